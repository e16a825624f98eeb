// Products of fp32 matrices on the bf16 matrix instructions (not in the paper: the dense products of the wrapped encoder
// block's linear layers).
//
// An fp32 number is the exact sum of three bf16 numbers, x = h + m + l (8 of its 24 bits, rounded to nearest, 8 of what is
// left, the rest), so a product of two is the sum of nine bf16 products, each exact in fp32.  The matrix cores add up the six
// from h h down to h l and m m; the other three are at most 2^-24 of the product.  A step's 32 elements are added up by
// themselves and then to what there was, so that a sum of K products is rounded K / 32 times at its own size: against 64 bits
// 1.5e-7 at K = 768 and 1.8e-7 at 3072, where torch's fp32 product has 5.0e-7 and 9.9e-7 (with every instruction adding to
// the whole sum 4.3e-7 and 6.2e-7, and 5 % less time).  Entries are split at 2^24 times their size, where
// the last bit of the smallest subnormal still has a normal bf16 number to go to (2 % of the time, in two multiplications more a
// pair).  Infinities, NaN, and entries and results too large for that (2^104, 2^80), are left to the fp32 matrix instructions
// at the end of the tile they fall into.
//
// Bound by power and by how far splitting (vector instructions) and multiplying overlap: 4096 x 768 x 3072 takes 103 us,
// 188 TFLOP/s of fp32 or 1.13 PFLOP/s of bf16 (an 8192^3 product in bf16 reaches 1.2 to 1.4 on the card); with operands of zeros a
// sixth less, with one of the six products a quarter.  torch's fp32 product: 140.
#include "common.hpp"

namespace slimfit {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kStep = 32;                  // depth of a step: one v_mfma_f32_16x16x32_bf16
constexpr int kRowBytes = kStep * 2;       // a row of one part in LDS
constexpr int kGroup = 256;                // threads that share a step
constexpr int kTileM = 128;

struct Parts {
    u32x4 h, m, l;                         // eight bf16 each
};
constexpr float kUp = 0x1p24f, kBack = 0x1p-48f;            // of an operand and of a product of two
__device__ __forceinline__ void split_pair(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    a *= kUp;
    b *= kUp;
    h = bf16_narrow2(a, b);
    a -= __builtin_bit_cast(float, h << 16);
    b -= __builtin_bit_cast(float, h & 0xFFFF0000u);
    m = bf16_narrow2(a, b);
    a -= __builtin_bit_cast(float, m << 16);
    b -= __builtin_bit_cast(float, m & 0xFFFF0000u);
    l = bf16_narrow2(a, b);
}
__device__ __forceinline__ Parts split(const float (&f)[8])
{
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pair(f[2 * i], f[2 * i + 1], h[i], m[i], l[i]);
    return Parts{{h[0], h[1], h[2], h[3]}, {m[0], m[1], m[2], m[3]}, {l[0], l[1], l[2], l[3]}};
}
// Where 16 bytes (eight elements deep) of a row lie: those of eight consecutive rows, and the four of two, are in different
// banks (SQ_LDS_BANK_CONFLICT counts none).
__device__ __forceinline__ int chunk_at(int row, int chunk) { return row * kRowBytes + ((chunk ^ ((row >> 1) & 3)) << 4); }

// A thread's share of ROWS rows of an operand, a step at a time.  Row r starts at base + r * ld (DEEP) or, its elements ld
// apart, at base + r.
template <int ROWS, bool DEEP, int GROUPS>
struct Loader {
    static constexpr int ITEMS = (ROWS * 4 + kGroup - 1) / kGroup;      // of eight elements
    using Held = float[ITEMS][8];
    const float *p[ITEMS];
    int64_t ld;
    __device__ __forceinline__ static bool has(int q, int t) { return (q + 1) * kGroup <= ROWS * 4 || t + q * kGroup < ROWS * 4; }   // wave-uniform
    __device__ __forceinline__ static int row(int q, int t) { return DEEP ? (t + q * kGroup) >> 2 : (t + q * kGroup) % ROWS; }
    __device__ __forceinline__ static int chunk(int q, int t) { return DEEP ? (t + q * kGroup) & 3 : (t + q * kGroup) / ROWS; }
    // rows past the last are read as the last, items past the share as its first
    __device__ __forceinline__ void init(const float *base, int64_t first, int64_t rows, int64_t ld_, int64_t k0, int t)
    {
        ld = ld_;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const int64_t r = min(first + (has(q, t) ? row(q, t) : 0), rows - 1);
            const int64_t k = k0 + 8 * (has(q, t) ? chunk(q, t) : 0);
            p[q] = base + (DEEP ? r * ld + k : k * ld + r);
        }
    }
    // No branch around any load, so that each is waited for by itself.  more: there is a step after this one; otherwise the
    // next call reads the same again.
    __device__ __forceinline__ void load(Held &f, bool more)
    {
        const int64_t on = more ? GROUPS * kStep * (DEEP ? 1 : ld) : 0;
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            if constexpr (DEEP) {
                const f32x4 a = reinterpret_cast<const f32x4 *>(p[q])[0], b = reinterpret_cast<const f32x4 *>(p[q])[1];
                f[q][0] = a.x; f[q][1] = a.y; f[q][2] = a.z; f[q][3] = a.w;
                f[q][4] = b.x; f[q][5] = b.y; f[q][6] = b.z; f[q][7] = b.w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) f[q][i] = p[q][i * ld];
            }
            p[q] += on;
        }
    }
    __device__ __forceinline__ static void store(const Held &f, char *lds, int t)
    {
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            if (!has(q, t)) continue;
            const Parts s = split(f[q]);
            char *at = lds + chunk_at(row(q, t), chunk(q, t));
            *reinterpret_cast<u32x4 *>(at) = s.h;
            *reinterpret_cast<u32x4 *>(at + ROWS * kRowBytes) = s.m;
            *reinterpret_cast<u32x4 *>(at + 2 * ROWS * kRowBytes) = s.l;
        }
    }
};

// out[i][j] = sum over k of a[i][k] b[j][k]; DEEP_B: b is N x K, otherwise K x N.  A group of four waves takes a step at a
// time, 64 x TN/2 of the tile a wave: its rows are split into LDS, and what was split is multiplied.
//   GROUPS 1  three workgroups a compute unit fill one another's waits: where there are tiles for that
//             (4096 x 2304 x 768 87 us, with two groups 97).  168 registers, which is why only one row of a's parts is held.
//   GROUPS 2  two groups of a workgroup take every other step of the same tile, one splitting while the other multiplies
//             (a barrier swaps them), and add their sums up at the end: where a compute unit has one tile
//             (4096 x 768 x 3072 103 us, with one group 153; 4096 x 768 x 768 29 and 42).
// AHEAD: steps of operands on their way in registers (one group has none to spare for two; two groups with one: 9 % slower).
template <int TN, bool DEEP_B, int GROUPS>
__global__ void __launch_bounds__(GROUPS * kGroup, GROUPS == 2 ? 2 : 3)
product_kernel(const float *__restrict__ a, const float *__restrict__ b, int64_t M, int64_t N, int64_t K, float *__restrict__ out, int tiles_m,
               int tiles_n)
{
    constexpr int WM = kTileM / 2, WN = TN / 2, FM = WM / 16, FN = WN / 16, AHEAD = GROUPS;
    constexpr int PART_A = kTileM * kRowBytes, PART_B = TN * kRowBytes, STAGE = 3 * (PART_A + PART_B);
    __shared__ __align__(16) char lds[GROUPS * STAGE];
    const int t = threadIdx.x & (kGroup - 1), lane = t & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6), group = GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    // Workgroups go to the eight XCDs in turn; an XCD's take bands of four tile rows, column by column, so that those at
    // work together share operands in its L2.
    const int per = tiles_m * tiles_n / 8, b0 = (int)blockIdx.x, id = b0 < per * 8 ? (b0 % 8) * per + b0 / 8 : b0;
    const int band = id / (4 * tiles_n), in_band = id % (4 * tiles_n), height = min(4, tiles_m - 4 * band);
    const int64_t m0 = (int64_t)(band * 4 + in_band % height) * kTileM, n0 = (int64_t)(in_band / height) * TN;

    char *stage = lds + group * STAGE;
    Loader<kTileM, true, GROUPS> la;
    Loader<TN, DEEP_B, GROUPS> lb;
    const int steps = (int)(K / kStep), mine = GROUPS == 1 ? steps : (steps + 1 - group) / 2, rounds = GROUPS == 1 ? steps : (steps + 1) / 2;
    const int64_t k0 = group < steps ? group * kStep : 0;
    la.init(a, m0, M, K, k0, t);
    lb.init(b, n0, N, DEEP_B ? K : N, k0, t);
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    typename Loader<kTileM, true, GROUPS>::Held ha[AHEAD];
    typename Loader<TN, DEEP_B, GROUPS>::Held hb[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
        la.load(ha[u], u + 1 < mine);
        lb.load(hb[u], u + 1 < mine);
    }
    const int wm = (wave >> 1) * WM, wn = (wave & 1) * WN;
    const char *read_a = stage + chunk_at(wm + (lane & 15), lane >> 4);
    const char *read_b = stage + 3 * PART_A + chunk_at(wn + (lane & 15), lane >> 4);
    auto step = [&](auto &held_a, auto &held_b, int s) {
        la.store(held_a, stage, t);
        lb.store(held_b, stage + 3 * PART_A, t);
        la.load(held_a, s + AHEAD + 1 < mine);
        lb.load(held_b, s + AHEAD + 1 < mine);
        __syncthreads();
        if (s < mine) {                                     // uniform for the group
            __builtin_amdgcn_s_setprio(1);                  // without: 10 % slower
            bf16x8 fb[3][FN];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int j = 0; j < FN; ++j) fb[p][j] = *reinterpret_cast<const bf16x8 *>(read_b + p * PART_B + j * 16 * kRowBytes);
            }
            constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                bf16x8 fa[3];
#pragma unroll
                for (int p = 0; p < 3; ++p) fa[p] = *reinterpret_cast<const bf16x8 *>(read_a + p * PART_A + i * 16 * kRowBytes);
                f32x4 part[FN];
#pragma unroll
                for (int j = 0; j < FN; ++j) part[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int u = 0; u < 6; ++u) {
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        part[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[PA[u]], fb[PB[u]][j], part[j], 0, 0, 0);
                }
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] += part[j];
            }
            __builtin_amdgcn_s_setprio(0);
        }
        __syncthreads();
    };
    // every thread passes the same number of barriers: the second group waits once before, the first once after; with two
    // groups the rounds are made even, and one past the end splits the last step again and multiplies nothing
    if (GROUPS == 2 && group == 1) __syncthreads();
    for (int s = 0; s < rounds; s += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) step(ha[u], hb[u], s + u);
    }
    constexpr int OWN = FM / GROUPS;                        // rows of sixteen that a group finishes
    f32x4 sum[OWN][FN];
    if constexpr (GROUPS == 2) {
        if (group == 0) __syncthreads();
        // each group hands the other half of its sums over and finishes the rest
        static_assert(FM % 2 == 0 && 2 * STAGE >= 2 * 4 * OWN * FN * kWave * 16, "the sums fit the stages");
        f32x4 *give = reinterpret_cast<f32x4 *>(lds) + ((1 - group) * 4 + wave) * (OWN * FN * kWave);
        const f32x4 *take = reinterpret_cast<const f32x4 *>(lds) + (group * 4 + wave) * (OWN * FN * kWave);
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4 low = acc[i][j], high = acc[OWN + i][j];
                give[(i * FN + j) * kWave + lane] = group == 0 ? high : low;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4 low = acc[i][j], high = acc[OWN + i][j];
                sum[i][j] = ((group == 0 ? low : high) + take[(i * FN + j) * kWave + lane]) * kBack;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) sum[i][j] = acc[i][j] * kBack;
        }
    }
    const int64_t first_row = m0 + wm + group * OWN * 16, first_col = n0 + wn;
    // An operand that is infinite, NaN or too large for a part, or a sum that overflows: what comes out there is what the fp32
    // matrix instructions make of the operands, for which the wave computes its share of the tile again (4096 x 3072 x 768 with
    // all entries of a NaN 290 us in all; by a loop over the depth for each output, one after the other, 17000).
    bool odd = false;
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) odd |= !(__builtin_fabsf(sum[i][j][q]) < __builtin_inff());
        }
    }
    if (__builtin_amdgcn_ballot_w64(odd) != 0u) {
        const int64_t deep = (lane >> 4) * 4;               // lane l holds depths k + 4 (l / 16) + q of both in the q-th of four instructions
        const float *pa[OWN], *pb[FN];
        f32x4 plain[OWN][FN];
#pragma unroll
        for (int i = 0; i < OWN; ++i) pa[i] = a + min(first_row + i * 16 + (lane & 15), M - 1) * K + deep;
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int64_t col = min(first_col + j * 16 + (lane & 15), N - 1);
            pb[j] = DEEP_B ? b + col * K + deep : b + deep * N + col;
#pragma unroll
            for (int i = 0; i < OWN; ++i) plain[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int64_t k = 0; k < K; k += 16) {
            f32x4 fa[OWN], fb[FN];
#pragma unroll
            for (int i = 0; i < OWN; ++i) fa[i] = *reinterpret_cast<const f32x4 *>(pa[i] + k);
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                if constexpr (DEEP_B) {
                    fb[j] = *reinterpret_cast<const f32x4 *>(pb[j] + k);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) fb[j][q] = pb[j][(k + q) * N];
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int i = 0; i < OWN; ++i) {
#pragma unroll
                    for (int j = 0; j < FN; ++j) plain[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][q], fb[j][q], plain[i][j], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
#pragma unroll
                for (int q = 0; q < 4; ++q) sum[i][j][q] = __builtin_fabsf(sum[i][j][q]) < __builtin_inff() ? sum[i][j][q] : plain[i][j][q];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < OWN; ++i) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const int64_t col = first_col + j * 16 + (lane & 15);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t row = first_row + i * 16 + (lane >> 4) * 4 + q;
                if (row < M && col < N) out[row * N + col] = sum[i][j][q];
            }
        }
    }
}

int64_t tiles_of(int64_t n, int tile) { return (n + tile - 1) / tile; }

template <int TN, int GROUPS>
void launch_tiles(const float *a, const float *b, bool b_deep, int64_t M, int64_t N, int64_t K, float *out, hipStream_t s)
{
    const int tm = (int)tiles_of(M, kTileM), tn = (int)tiles_of(N, TN);
    if (b_deep) launch(product_kernel<TN, true, GROUPS>, (unsigned)(tm * tn), GROUPS * kGroup, 0, s, a, b, M, N, K, out, tm, tn);
    else launch(product_kernel<TN, false, GROUPS>, (unsigned)(tm * tn), GROUPS * kGroup, 0, s, a, b, M, N, K, out, tm, tn);
}

}  // namespace
}  // namespace slimfit

using namespace slimfit;

static int32_t validate(int64_t M, int64_t N, int64_t K)
{
    if (M < 0 || N < 0 || K < 0) return SLIMFIT_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return SLIMFIT_OK;
    if (K == 0 || K % kStep != 0 || K > 0x7FFFFFFFLL) return SLIMFIT_ERR_UNSUPPORTED;
    // (each factor is below 2^63: the products are looked at in floating point first)
    if ((double)M * (double)K > 1.0e18 || (double)N * (double)K > 1.0e18 || (double)M * (double)N > 1.0e18) return SLIMFIT_ERR_UNSUPPORTED;
    if ((double)tiles_of(M, kTileM) * (double)tiles_of(N, 64) > (double)(kMaxGridThreads / (2 * kGroup))) return SLIMFIT_ERR_UNSUPPORTED;
    return SLIMFIT_OK;
}

// The operands are split on their way into LDS: no workspace is needed.
extern "C" int32_t slimfit_product_workspace(int64_t M, int64_t N, int64_t K, size_t *bytes)
{
    const int32_t rc = validate(M, N, K);
    if (rc != SLIMFIT_OK) return rc;
    if (!bytes) return SLIMFIT_ERR_INVALID_ARG;
    *bytes = 0;
    return SLIMFIT_OK;
}

extern "C" int32_t slimfit_product(const float *a, const float *b, int32_t b_deep, int64_t M, int64_t N, int64_t K, float *out, void *workspace,
                                   size_t workspace_bytes, void *stream)
{
    StreamScope capture_aware(stream);
    (void)workspace;
    (void)workspace_bytes;
    int32_t rc = validate(M, N, K);
    if (rc != SLIMFIT_OK || M == 0 || N == 0) return rc;
    if (!a || !b || !out) return SLIMFIT_ERR_INVALID_ARG;
    if (!aligned_to(a, 16) || !aligned_to(b, 16) || !aligned_to(out, 4)) return SLIMFIT_ERR_ALIGNMENT;
    if ((rc = check_device_range(a, (size_t)M * (size_t)K * 4)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(b, (size_t)N * (size_t)K * 4)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(out, (size_t)M * (size_t)N * 4)) != SLIMFIT_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // A tile for each of the 256 compute units at most: the narrowest tiles of which that holds, two groups on each (4096 x
    // 768 x 3072 in tiles of 96 columns 103 us, of 128, which leave 64 units idle, 112).  More: one group (tiles of 64 columns
    // 4096 x 2304 x 768 95 us, of 96 87; of 128 they need more registers than three workgroups have).
    constexpr int64_t kUnits = 256;
    const int64_t tm = tiles_of(M, kTileM);
    if (tm * tiles_of(N, 64) <= kUnits) launch_tiles<64, 2>(a, b, b_deep != 0, M, N, K, out, s);
    else if (tm * tiles_of(N, 96) <= kUnits) launch_tiles<96, 2>(a, b, b_deep != 0, M, N, K, out, s);
    else if (tm * tiles_of(N, 128) <= kUnits) launch_tiles<128, 2>(a, b, b_deep != 0, M, N, K, out, s);
    else launch_tiles<96, 1>(a, b, b_deep != 0, M, N, K, out, s);
    return launch_status();
}
