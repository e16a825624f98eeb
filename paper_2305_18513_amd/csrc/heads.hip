// The reorderings around attention's products, for gfx950: the rows of the QKV projection (batch, token, [q | k | v],
// head, element) apart into the operands of Q K^T and P V -- q and v as (batch, head, token, element), k transposed, as
// (batch, head, element, token) -- and their gradients together again.  One pass over each byte; the factor of Q K^T goes
// onto q on the way (and onto its gradient on the way back).
//
// A workgroup owns 64 tokens x 64 elements of one head of one of the three parts.  q and v are rows of consecutive
// elements on both sides: 16-byte loads and stores.  k passes through LDS (rows 65 words apart, so that neither the
// writes along the elements nor the reads along the tokens queue at a bank); its token rows move 16 bytes at a time too,
// or by single elements where they are not aligned to that.
// Bound by HBM: 4096 x 2304 fp32 (75 MB) 12.6 us apart and 13.0 together, 6.0 and 5.8 TB/s.  torch's reshapes and
// transposes of the three parts, the division of the products and their gradient by sqrt(dim) and the concatenation of
// the gradients took 45 and 49 us there.
#include "common.hpp"

namespace slimfit {
namespace {

constexpr int kThreads = 256;
constexpr int kSide = 64;                  // tokens and elements of a workgroup's piece
constexpr int kPitch = kSide + 1;          // LDS row of the transposed part

template <typename T> struct Vec16;
template <> struct Vec16<float> {
    static constexpr int E = 4;
    __device__ static void load(const float *p, float (&f)[4])
    {
        const f32x4 r = *reinterpret_cast<const f32x4 *>(p);
        f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w;
    }
    __device__ static void store(float *p, const float (&f)[4]) { *reinterpret_cast<f32x4 *>(p) = f32x4{f[0], f[1], f[2], f[3]}; }
    __device__ static float load1(const float *p) { return *p; }
    __device__ static void store1(float *p, float f) { *p = f; }
};
template <> struct Vec16<uint16_t> {       // bf16, widened on the way in and rounded to nearest even on the way out
    static constexpr int E = 8;
    __device__ static void load(const uint16_t *p, float (&f)[8])
    {
        const u32x4 r = *reinterpret_cast<const u32x4 *>(p);
        const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __builtin_bit_cast(float, w[i] << 16);
            f[2 * i + 1] = __builtin_bit_cast(float, w[i] & 0xFFFF0000u);
        }
    }
    __device__ static void store(uint16_t *p, const float (&f)[8])
    {
        *reinterpret_cast<u32x4 *>(p) =
            u32x4{bf16_narrow2(f[0], f[1]), bf16_narrow2(f[2], f[3]), bf16_narrow2(f[4], f[5]), bf16_narrow2(f[6], f[7])};
    }
    __device__ static float load1(const uint16_t *p) { return bf16_widen(*p); }
    __device__ static void store1(uint16_t *p, float f) { *p = (uint16_t)bf16_narrow(f); }
};

struct Shape {
    int tokens, heads, dim;                // dim: a multiple of a 16-byte vector's elements
    int token_blocks, dim_blocks;
    float q_scale;
};

// SPLIT: fused -> (q, kt, v); otherwise the other way round
template <typename T, bool SPLIT>
__global__ void __launch_bounds__(kThreads)
heads_kernel(T *fused, T *q, T *kt, T *v, Shape s, unsigned first)
{
    using V = Vec16<T>;
    constexpr int E = V::E, kCols = kSide / E, kRows = kThreads / kCols;        // vectors across a piece, rows a step
    __shared__ float piece[kSide * kPitch];
    unsigned at = first + blockIdx.x;                       // of all launches' blocks (below 2^31)
    const int part = (int)(at % 3);
    at /= 3;
    const int d0 = (int)(at % (unsigned)s.dim_blocks) * kSide;
    at /= (unsigned)s.dim_blocks;
    const int t0 = (int)(at % (unsigned)s.token_blocks) * kSide;
    at /= (unsigned)s.token_blocks;                                   // batch * heads + head
    const int64_t head = at % (unsigned)s.heads, width = (int64_t)s.heads * s.dim;
    T *const rows = fused + ((int64_t)(at / (unsigned)s.heads) * s.tokens * 3 + part) * width + head * s.dim;       // token 0's; 3 * width apart
    const int n_t = min(kSide, s.tokens - t0), n_d = min(kSide, s.dim - d0);
    const int c = threadIdx.x % kCols * E, r0 = threadIdx.x / kCols;
    if (part != 1) {
        T *const apart = (part == 0 ? q : v) + (int64_t)at * s.tokens * s.dim;
        const float scale = part == 0 ? s.q_scale : 1.0f;
        float f[kSide / kRows][E];
#pragma unroll
        for (int i = 0; i < kSide / kRows; ++i) {
            const int r = i * kRows + r0;
            if (r < n_t && c < n_d)
                V::load(SPLIT ? rows + (int64_t)(t0 + r) * 3 * width + d0 + c : apart + (int64_t)(t0 + r) * s.dim + d0 + c, f[i]);
        }
#pragma unroll
        for (int i = 0; i < kSide / kRows; ++i) {
            const int r = i * kRows + r0;
            if (r < n_t && c < n_d) {
#pragma unroll
                for (int e = 0; e < E; ++e) f[i][e] *= scale;
                V::store(SPLIT ? apart + (int64_t)(t0 + r) * s.dim + d0 + c : rows + (int64_t)(t0 + r) * 3 * width + d0 + c, f[i]);
            }
        }
        return;
    }
    T *const turned = kt + (int64_t)at * s.tokens * s.dim + (int64_t)d0 * s.tokens + t0;       // element 0's; s.tokens apart
    const bool whole = s.tokens % E == 0;                   // every row of tokens begins on 16 bytes (t0 is a multiple of 64)
    auto token_rows = [&](auto vec, auto one) {             // the piece's rows along the tokens
        if (whole) {
#pragma unroll
            for (int i = 0; i < kSide / kRows; ++i) {
                const int r = i * kRows + r0;
                if (r < n_d && c < n_t) vec(turned + (int64_t)r * s.tokens + c, r, c);
            }
        } else {
            for (int i = threadIdx.x; i < kSide * kSide; i += kThreads) {
                const int r = i / kSide, t = i % kSide;
                if (r < n_d && t < n_t) one(turned + (int64_t)r * s.tokens + t, r, t);
            }
        }
    };
    auto element_rows = [&](auto f) {                       // its rows along the elements
#pragma unroll
        for (int i = 0; i < kSide / kRows; ++i) {
            const int r = i * kRows + r0;
            if (r < n_t && c < n_d) f(rows + (int64_t)(t0 + r) * 3 * width + d0 + c, r, c);
        }
    };
    if constexpr (SPLIT) {
        element_rows([&](T *p, int t, int d) {
            float f[E];
            V::load(p, f);
#pragma unroll
            for (int e = 0; e < E; ++e) piece[t * kPitch + d + e] = f[e];
        });
        __syncthreads();
        token_rows(
            [&](T *p, int d, int t) {
                float f[E];
#pragma unroll
                for (int e = 0; e < E; ++e) f[e] = piece[(t + e) * kPitch + d];
                V::store(p, f);
            },
            [&](T *p, int d, int t) { V::store1(p, piece[t * kPitch + d]); });
    } else {
        token_rows(
            [&](T *p, int d, int t) {
                float f[E];
                V::load(p, f);
#pragma unroll
                for (int e = 0; e < E; ++e) piece[(t + e) * kPitch + d] = f[e];
            },
            [&](T *p, int d, int t) { piece[t * kPitch + d] = V::load1(p); });
        __syncthreads();
        element_rows([&](T *p, int t, int d) {
            float f[E];
#pragma unroll
            for (int e = 0; e < E; ++e) f[e] = piece[t * kPitch + d + e];
            V::store(p, f);
        });
    }
}

template <bool SPLIT>
int32_t heads_entry(void *fused, int32_t dt, int64_t batch, int32_t tokens, int32_t heads, int32_t head_dim, float q_scale, void *q, void *kt,
                    void *v, void *stream)
{
    if (!dtype_ok(dt) || batch < 0 || tokens < 0 || heads < 1 || head_dim < 1) return SLIMFIT_ERR_INVALID_ARG;
    const int E = dt == SLIMFIT_F32 ? 4 : 8;
    if (head_dim % E != 0) return SLIMFIT_ERR_UNSUPPORTED;
    if (batch == 0 || tokens == 0) return SLIMFIT_OK;
    if (batch > (int64_t)1 << 31) return SLIMFIT_ERR_UNSUPPORTED;
    if (!fused || !q || !kt || !v) return SLIMFIT_ERR_INVALID_ARG;
    if (!aligned_to(fused, 16) || !aligned_to(q, 16) || !aligned_to(kt, 16) || !aligned_to(v, 16)) return SLIMFIT_ERR_ALIGNMENT;
    Shape s = {tokens, heads, head_dim, (tokens + kSide - 1) / kSide, (head_dim + kSide - 1) / kSide, q_scale};
    // (each factor is below 2^31 or 2^26: the products are looked at one by one)
    const double blocks = 3.0 * (double)batch * heads * s.token_blocks * s.dim_blocks;
    if (blocks > 2147483647.0 || (double)batch * tokens * heads * head_dim > 4.0e18) return SLIMFIT_ERR_UNSUPPORTED;
    const size_t bytes = (size_t)batch * (size_t)tokens * (size_t)heads * (size_t)head_dim * dtype_size(dt);
    int32_t rc;
    if ((rc = check_device_range(fused, 3 * bytes)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(q, bytes)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(kt, bytes)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(v, bytes)) != SLIMFIT_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    constexpr int64_t kMost = kMaxGridThreads / kThreads;    // blocks of a launch
    const int64_t all = (int64_t)blocks;
    for (int64_t first = 0; first < all; first += kMost) {
        const unsigned here = (unsigned)(all - first < kMost ? all - first : kMost);
        if (dt == SLIMFIT_F32)
            launch(heads_kernel<float, SPLIT>, here, kThreads, 0, st, static_cast<float *>(fused), static_cast<float *>(q),
                                                                  static_cast<float *>(kt), static_cast<float *>(v), s, (unsigned)first);
        else
            launch(heads_kernel<uint16_t, SPLIT>, here, kThreads, 0, st, static_cast<uint16_t *>(fused), static_cast<uint16_t *>(q),
                                                                     static_cast<uint16_t *>(kt), static_cast<uint16_t *>(v), s,
                                                                     (unsigned)first);
    }
    return launch_status();
}

}  // namespace
}  // namespace slimfit

using namespace slimfit;

extern "C" int32_t slimfit_split_heads(const void *qkv, int32_t dt, int64_t batch, int32_t tokens, int32_t heads, int32_t head_dim,
                                       float q_scale, void *q, void *kt, void *v, void *stream)
{
    StreamScope capture_aware(stream);
    return heads_entry<true>(const_cast<void *>(qkv), dt, batch, tokens, heads, head_dim, q_scale, q, kt, v, stream);
}

extern "C" int32_t slimfit_merge_heads(const void *q, const void *kt, const void *v, int32_t dt, int64_t batch, int32_t tokens, int32_t heads,
                                       int32_t head_dim, float q_scale, void *qkv, void *stream)
{
    StreamScope capture_aware(stream);
    return heads_entry<false>(qkv, dt, batch, tokens, heads, head_dim, q_scale, const_cast<void *>(q), const_cast<void *>(kt),
                              const_cast<void *>(v), stream);
}
