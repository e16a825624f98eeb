// Shared host/device helpers of the gfx950 kernels (wave64, DPP cross-lane ops).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "slimfit.h"

namespace slimfit {

constexpr int kWave = 64;

// ---- host-side helpers (api.cpp) --------------------------------------------
int32_t check_device_range(const void *p, size_t bytes);   // pointer checks, see slimfit.h
// Declared at the top of every entry point that takes a stream: while that stream is being captured into a
// graph the pointer look-ups (runtime queries a capture does not allow) are skipped for this thread's call.
struct StreamScope {
    explicit StreamScope(void *stream);
    ~StreamScope();
    StreamScope(const StreamScope &) = delete;
    StreamScope &operator=(const StreamScope &) = delete;
private:
    bool prev_;
};
int32_t launch_status();                                    // hipGetLastError -> status

// A grid's threads are counted in 32 bits: a launch of 2^32 or more starts what the low bits say and reports no error.
// More work goes out in launches of kMaxGridThreads, or is refused.
constexpr int64_t kMaxGridThreads = (int64_t)1 << 31;
inline bool grid_fits(int64_t blocks, int threads) { return blocks <= 0xFFFFFFFFLL / threads; }

// short rows that keep few entries have a kernel of their own (prune_short.hip)
constexpr int kShortPruneMaxCols = 256;
constexpr int kShortPruneMaxK = 16;                     // bf16 rows
constexpr int kShortPruneMaxKF32 = 12;                  // fp32 rows
bool prune_short_eligible(const void *p, int32_t dt, int64_t rows, int cols, int k, int mode, bool softmax);
void launch_prune_short(const void *p, int32_t dt, int64_t rows, int cols, int k, int mode, float tau, void *vals,
                        uint16_t *idx, int32_t *counts, hipStream_t st);
void launch_softmax_prune_short(const void *logits, int32_t dt, int64_t rows, int cols, int k, void *probs, void *vals,
                                uint16_t *idx, hipStream_t st);

#if defined(__HIPCC__)
// kernel<<<grid, block, lds, stream>>>(args...) in one call of the runtime instead of three (the launch's shape is not
// pushed and popped on the way): 2.77 us of host time a call for 2.85.  launch_status() has the error.
template <typename T> struct Same { using type = T; };
template <typename... P>
inline void launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, typename Same<P>::type... args)
{
    void *at[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    (void)hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, at, lds, stream);
}
#endif

inline bool aligned_to(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }
inline bool dtype_ok(int32_t dt) { return dt == SLIMFIT_F32 || dt == SLIMFIT_BF16; }
inline size_t dtype_size(int32_t dt) { return dt == SLIMFIT_F32 ? 4 : 2; }

#if defined(__HIPCC__)
// ---- 128/64-bit global access, optionally non-temporal (streamed once) ----------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <bool NT, typename V>
__device__ __forceinline__ V load_global(const V *p)
{
    return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT, typename V>
__device__ __forceinline__ void store_global(V *p, V v)
{
    if (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// ---- DPP lane exchange --------------------------------------------------------
// A DPP "row" is 16 consecutive lanes.  The controls used here only permute
// inside a row, so every source lane exists.
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7-i inside each 8
constexpr int kDppMirror = 0x140;     // lane i <-> 15-i inside each 16

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v)
{
    // every source lane exists, so `old` is never seen; bound_ctrl lets the move fold into the instruction that uses it
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __builtin_bit_cast(float, dpp_u32<CTRL>(__builtin_bit_cast(uint32_t, v)));
}

// max over groups of G consecutive lanes (G = 4 .. 64, a power of two; it need not be a constant, but is wave-uniform);
// every lane of a group receives the group's result.
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v, int G)
{
    v = max(v, dpp_u32<kDppXor1>(v));
    v = max(v, dpp_u32<kDppXor2>(v));
    if (G >= 8) v = max(v, dpp_u32<kDppHalfMirror>(v));
    if (G >= 16) v = max(v, dpp_u32<kDppMirror>(v));
    if (G >= 32) {                                          // exchanges rows of 16 lanes, then halves of the wave
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = max(r[0], r[1]);
    }
    if (G >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = max(r[0], r[1]);
    }
    return v;
}

// Alg. 2 with one scale per block: code = clamp(round_half_even(x * mult), qmin, qmax)
// -- one fp32 multiply -- where mult = qmax / a and the stored scale = a / qmax for a
// block whose largest magnitude is a (two IEEE fp32 divisions); a block of zeros, or one
// whose multiplier would overflow, gets scale 0 and codes 0.
//
// The code is left in the low BITS bits of the result (two's complement), whatever is above them: clamping to whole
// numbers commutes with rounding, and adding 1.5 * 2^23 rounds to a whole number (half to even) in the low mantissa bits.
constexpr uint32_t kRoundBits = 0x4B400000u;               // 1.5 * 2^23
template <int BITS>
__device__ __forceinline__ uint32_t quantise_one(float x, float mult)
{
    constexpr float qmax = (float)((1 << (BITS - 1)) - 1);
    constexpr float qmin = -(float)(1 << (BITS - 1));
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(x * mult, qmin, qmax) + __builtin_bit_cast(float, kRoundBits));
}
// the E codes of a vector, element i in bits [i*BITS, (i+1)*BITS) of the 64-bit result (two words)
template <int BITS, int E>
__device__ __forceinline__ void pack_codes(const float (&f)[E], float mult, uint32_t (&w)[2])
{
    static_assert(E == 4 || E == 8, "a 16-byte vector");
    uint32_t b[E];
#pragma unroll
    for (int i = 0; i < E; ++i) b[i] = quantise_one<BITS>(f[i], mult);
    w[0] = w[1] = 0u;
    if constexpr (BITS == 8) {
#pragma unroll
        for (int i = 0; i < E; i += 4)                      // the low bytes of four words
            w[i / 4] = __builtin_amdgcn_perm(b[i + 1], b[i], 0x0C0C0400u) | __builtin_amdgcn_perm(b[i + 3], b[i + 2], 0x04000C0Cu);
    } else {
        // sum of (kRoundBits + c_i) 16^i, the kRoundBits' share taken out; with 8 added to every c_i the fields borrow
        // nothing from one another, and flipping their top bits takes the 8 away again
        constexpr uint32_t ones = E == 4 ? 0x1111u : 0x11111111u;
        uint32_t v = b[E - 1];
#pragma unroll
        for (int i = E - 2; i >= 0; --i) v = (v << 4) + b[i];
        v = (v + (8u - kRoundBits) * ones) ^ (8u * ones);
        w[0] = E == 4 ? v & 0xFFFFu : v;
    }
}
template <int BITS>
__device__ __forceinline__ void block_scale(float a, float &mult, float &scale)       // a >= 0, not NaN
{
    constexpr float qmax = (float)((1 << (BITS - 1)) - 1);
    const float m = qmax / a, s = a / qmax;
    const bool ok = !__builtin_isinf(m);                   // a of 0 as well
    mult = ok ? m : 0.0f;
    scale = ok ? s : 0.0f;
}
// The same for N <= 4 blocks whose maxima all lanes of a quad hold: lane l of the quad does the divisions of block l and
// the quad exchanges the multipliers; `scale` is that of block (lane & 3), meant for lanes with (lane & 3) < N.  (Every
// lane's divisions for every block were a quarter of the quantiser's instructions.)
template <int BITS, int N>
__device__ __forceinline__ void quad_scales(const uint32_t (&a)[N], int lane, float (&mult)[N], float &scale)
{
    static_assert(N >= 1 && N <= 4, "a quad");
    const uint32_t a0 = a[0], a1 = a[N >= 2 ? 1 : 0], a2 = a[N >= 3 ? 2 : 0], a3 = a[N - 1];
    const uint32_t low = (lane & 1) ? a1 : a0, high = (lane & 1) ? a3 : a2;
    const uint32_t mine = N >= 3 && (lane & 2) ? high : low;
    float m;
    block_scale<BITS>(__builtin_bit_cast(float, mine), m, scale);
    mult[0] = dpp_f32<0x00>(m);                            // quad_perm: lane 0's to all four, and so on
    if constexpr (N >= 2) mult[1] = dpp_f32<0x55>(m);
    if constexpr (N >= 3) mult[2] = dpp_f32<0xAA>(m);
    if constexpr (N >= 4) mult[3] = dpp_f32<0xFF>(m);
}
// field i of BITS bits of a packed word, sign-extended
template <int BITS>
__device__ __forceinline__ int code_field(uint32_t word, int i)
{
    const int sh = i * BITS;
    return (int)(word << (32 - BITS - sh)) >> (32 - BITS);
}

// The whole wave's largest unsigned key, wave-uniform (SGPR).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = max(v, dpp_u32<kDppXor1>(v));
    v = max(v, dpp_u32<kDppXor2>(v));
    v = max(v, dpp_u32<kDppHalfMirror>(v));
    v = max(v, dpp_u32<kDppMirror>(v));
    uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return max(max(a, b), max(c, d));
}

// number of set bits of `mask` strictly below this lane
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// ---- bf16 -----------------------------------------------------------------------
__device__ __forceinline__ float bf16_widen(uint32_t h) { return __builtin_bit_cast(float, h << 16); }

// fp32 -> bf16, round to nearest even, denormals kept, NaN stays NaN.  gfx950 has the conversion in
// hardware (one instruction for a pair); the integer form is kept for comparison.
#ifndef SLIMFIT_HW_BF16_CVT
#define SLIMFIT_HW_BF16_CVT 1
#endif
__device__ __forceinline__ uint32_t bf16_narrow(float f)
{
#if SLIMFIT_HW_BF16_CVT
    return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)f);
#else
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
    return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? ((u >> 16) | 0x40u) : r;
#endif
}

// two at once, a in the low half
__device__ __forceinline__ uint32_t bf16_narrow2(float a, float b)
{
#if SLIMFIT_HW_BF16_CVT
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const bf16x2_t h = __builtin_convertvector(f32x2_t{a, b}, bf16x2_t);
    return __builtin_bit_cast(uint32_t, h);
#else
    return bf16_narrow(a) | (bf16_narrow(b) << 16);
#endif
}

// Order-preserving map float -> uint32 (larger float <=> larger key) and back.
__device__ __forceinline__ uint32_t float_to_key(float f)
{
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_to_float(uint32_t k)
{
    uint32_t u = (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
    return __builtin_bit_cast(float, u);
}
#endif  // __HIPCC__

}  // namespace slimfit
