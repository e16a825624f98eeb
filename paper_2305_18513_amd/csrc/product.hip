// Products of fp32 matrices on the fp16 matrix instructions (not in the paper: the dense products of the wrapped encoder
// block's linear layers).
//
// A row of an operand, brought to below 2^15 by a power of two of its own, is the sum of two fp16 numbers, h and 2^-12 l, but
// for the last of its 24 bits where l would need a twelfth (at most 2^-23 of the entry; l is kept 2^12 times its size so that
// entries down to 2^-28 of the row's largest are as exact).  A product of two is then h h + 2^-12 (h l + l h), each exact in
// fp32, and l l, at most 2^-22 of it and 2^-26 in the mean, which is left out.  split_kernel writes both operands' parts in the
// order in which product_kernel's fragments take them; a step's h l + l h are added up by themselves and then to h h.  Against
// 64 bits 1.6e-7 to 2.1e-7 at K = 768 and 2.9e-7 to 4.0e-7 at 3072, where torch's fp32 product has 5.0e-7 and 9.9e-7.  A row
// with an infinity or a NaN, and results too large for fp32, are computed by plain arithmetic at the end of their tile.
//
// The products are bound by power: 4096 x 3072 x 768 takes 56 us in an encoder block, 1.04 PFLOP/s of fp16 (an 8192^3 product
// in bf16 reaches 1.21 on the card), 4096 x 768 x 3072 58 to 63; splitting by memory: 119 MB in 25 us for the latter, 44 MB in
// 11 for the former, two thirds of what a copy reaches, since a workgroup first reads its rows and then writes them.
// Together 67 and 80 us, where three bf16 parts of each operand, split on their way into LDS, and six products took 106 and 99
// and torch's fp32 product takes 141 and 138.
#include "common.hpp"

namespace slimfit {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kStep = 32;                  // depth of a step: one v_mfma_f32_16x16x32_f16
constexpr int kFragRows = 16;
constexpr int kPartBytes = kWave * 16;     // one part of a fragment: 16 rows, a step deep, lane l's eight elements at 16 l
constexpr int kFragBytes = 2 * kPartBytes; // h, then l

__host__ __device__ inline int64_t frags_of(int64_t rows) { return (rows + kFragRows - 1) / kFragRows; }

// ---------------------------------------------------------------------------------------------------- splitting

constexpr int kSplitWaves = 16;            // of a workgroup, at most: one for each HELD steps

// The power of two that brings magnitudes up to `top` (bits of the largest) below 2^15; 2^126 at most.
__device__ __forceinline__ uint32_t scale_bits(uint32_t top) { return min(268u - (top >> 23), 253u); }

__device__ __forceinline__ void split8(const float (&f)[8], float scale, bool odd, u32x4 &h, u32x4 &l)
{
    f16x8 hh, ll;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float x = f[i] * scale;
        hh[i] = (_Float16)x;
        ll[i] = (_Float16)((x - (float)hh[i]) * 4096.0f);
    }
    h = __builtin_bit_cast(u32x4, hh);
    l = __builtin_bit_cast(u32x4, ll);
    if (odd) {
        h = u32x4{0x7E007E00u, 0x7E007E00u, 0x7E007E00u, 0x7E007E00u};
        l = u32x4{0u, 0u, 0u, 0u};
    }
}

// Sixteen rows a workgroup, over their whole depth; element k of row r at x[r * ld + k] (DEEP) or x[k * ld + r].  Rows past the
// last repeat it.  A wave holds HELD steps in registers between the two passes; deeper rows are read twice.
template <bool DEEP, int HELD>
__device__ __forceinline__ void split_rows(const float *__restrict__ x, int64_t frag, int64_t rows, int64_t ld, int64_t steps, char *__restrict__ parts,
                                           float *__restrict__ unscale, uint32_t (&top)[kSplitWaves][kFragRows])
{
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x / kWave, row = lane & 15;
    const int64_t r = min(frag * kFragRows + row, rows - 1), k = (lane >> 4) * 8;
    const float *p = DEEP ? x + r * ld + k : x + k * ld + r;
    auto load = [&](int64_t s, float (&f)[8]) {
        const float *at = p + (DEEP ? s * kStep : s * kStep * ld);
        if constexpr (DEEP) {
            const f32x4 a = reinterpret_cast<const f32x4 *>(at)[0], b = reinterpret_cast<const f32x4 *>(at)[1];
            f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
            f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) f[i] = at[i * ld];
        }
    };
    uint32_t most = 0;
    auto look = [&](const float (&f)[8]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) most = max(most, __builtin_bit_cast(uint32_t, f[i]) & 0x7FFFFFFFu);
    };
    float held[HELD][8];
#pragma unroll
    for (int q = 0; q < HELD; ++q) {
        const int64_t s = wave + q * waves;
        load(s < steps ? s : 0, held[q]);
    }
#pragma unroll
    for (int q = 0; q < HELD; ++q) {
        if (wave + q * waves < steps) look(held[q]);
    }
    for (int64_t s = wave + HELD * waves; s < steps; s += waves) {
        float f[8];
        load(s, f);
        look(f);
    }
    most = max(most, (uint32_t)__shfl_xor((int)most, 16));
    most = max(most, (uint32_t)__shfl_xor((int)most, 32));
    if (lane < kFragRows) top[wave][lane] = most;
    __syncthreads();
    for (int w = 0; w < waves; ++w) most = max(most, top[w][row]);
    const bool odd = most >= 0x7F800000u;
    const uint32_t bits = odd ? 127u : scale_bits(most);
    const float scale = __builtin_bit_cast(float, bits << 23);
    if (threadIdx.x < kFragRows) unscale[frag * kFragRows + lane] = __builtin_bit_cast(float, (254u - bits) << 23);
    auto store = [&](int64_t s, const float (&f)[8]) {
        u32x4 h, l;
        split8(f, scale, odd, h, l);
        u32x4 *at = reinterpret_cast<u32x4 *>(parts + (frag * steps + s) * kFragBytes) + lane;
        at[0] = h;
        at[kWave] = l;
    };
#pragma unroll
    for (int q = 0; q < HELD; ++q) {
        const int64_t s = wave + q * waves;
        if (s < steps) store(s, held[q]);
    }
    for (int64_t s = wave + HELD * waves; s < steps; s += waves) {
        float f[8];
        load(s, f);
        store(s, f);
    }
}

struct Split {
    char *parts;                           // [fragments][steps][kFragBytes]
    float *unscale;                        // [fragments * 16]
};

template <bool DEEP_B, int HELD>
__global__ void __launch_bounds__(kSplitWaves * kWave, HELD > 4 ? 4 : 8)
split_kernel(const float *__restrict__ a, const float *__restrict__ b, int64_t M, int64_t N, int64_t K, Split sa, Split sb)
{
    __shared__ uint32_t top[kSplitWaves][kFragRows];
    const int64_t of_a = frags_of(M), id = blockIdx.x, steps = K / kStep;
    if (id < of_a) split_rows<true, HELD>(a, id, M, K, steps, sa.parts, sa.unscale, top);
    else split_rows<DEEP_B, HELD>(b, id - of_a, N, DEEP_B ? K : N, steps, sb.parts, sb.unscale, top);
}

// -------------------------------------------------------------------------------------------------- multiplying

// out[i][j] = sum over k of a[i][k] b[j][k]; b_deep: b is N x K, otherwise K x N (a and b are read only where plain arithmetic decides).
// A group of WY x WX waves takes a step at a time, TM/WY x TN/WX of the tile a wave; the step's fragments go from the split
// operands straight to LDS, one step ahead.  GROUPS groups of a workgroup take every GROUPS-th step of the same tile and add
// their sums up at the end.  Twelve waves, three a SIMD, fill one another's waits better than eight of larger parts: 4096 x 3072 x
// 768 in tiles of 256 x 192 68 us and 73.
template <int TM, int TN, int WY, int WX, int GROUPS>
__global__ void __launch_bounds__(GROUPS * WY * WX * kWave, 2)
product_kernel(Split sa, Split sb, int64_t M, int64_t N, int64_t K, float *__restrict__ out, int tiles_m, int tiles_n, const float *__restrict__ a,
               const float *__restrict__ b, bool b_deep)
{
    constexpr int FM = TM / WY / 16, FN = TN / WX / 16, WAVES = WY * WX;
    constexpr int PARTS_A = TM / 16 * 2, PARTS = PARTS_A + TN / 16 * 2, OWN_PARTS = (PARTS + WAVES - 1) / WAVES, STAGE = PARTS * kPartBytes;
    __shared__ __align__(16) char lds[GROUPS * 2 * STAGE];
    const int lane = threadIdx.x & (kWave - 1);
    const int in_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = in_all % WAVES, group = in_all / WAVES;
    // Workgroups go to the eight XCDs in turn; an XCD's take bands of four tile rows, column by column, so that those at
    // work together share operands in its L2.
    const int per = tiles_m * tiles_n / 8, b0 = (int)blockIdx.x, id = b0 < per * 8 ? (b0 % 8) * per + b0 / 8 : b0;
    const int band = id / (4 * tiles_n), in_band = id % (4 * tiles_n), height = min(4, tiles_m - 4 * band);
    const int64_t m0 = (int64_t)(band * 4 + in_band % height) * TM, n0 = (int64_t)(in_band / height) * TN;

    char *stage = lds + group * 2 * STAGE;
    const int steps = (int)(K / kStep), mine = (steps + GROUPS - 1 - group) / GROUPS, rounds = (steps + GROUPS - 1) / GROUPS;
    const int64_t most_a = frags_of(M) - 1, most_b = frags_of(N) - 1;
    const char *from[OWN_PARTS];
#pragma unroll
    for (int q = 0; q < OWN_PARTS; ++q) {
        const int part = min(wave * OWN_PARTS + q, PARTS - 1), f = part < PARTS_A ? part >> 1 : (part - PARTS_A) >> 1;
        const char *base = part < PARTS_A ? sa.parts + min(m0 / 16 + f, most_a) * steps * kFragBytes : sb.parts + min(n0 / 16 + f, most_b) * steps * kFragBytes;
        from[q] = base + (part & 1) * kPartBytes + group * kFragBytes;
    }
    // step s of this group into its stage s & 1
    auto fetch = [&](int s) {
#pragma unroll
        for (int q = 0; q < OWN_PARTS; ++q) {
            if (PARTS % WAVES != 0 && wave * OWN_PARTS + q >= PARTS) break;      // wave-uniform
            typedef __attribute__((address_space(3))) void lds_void;
            typedef const __attribute__((address_space(1))) void global_void;
            __builtin_amdgcn_global_load_lds((global_void *)(from[q] + (int64_t)s * (GROUPS * kFragBytes) + lane * 16),
                                             (lds_void *)(stage + (s & 1) * STAGE + (wave * OWN_PARTS + q) * kPartBytes), 16, 0, 0);
        }
    };
    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    const int frag_a = wave / WX * FM, frag_b = wave % WX * FN;
    const char *read_a = stage + frag_a * kFragBytes + lane * 16, *read_b = stage + PARTS_A * kPartBytes + frag_b * kFragBytes + lane * 16;
    if (mine > 0) fetch(0);
    for (int s = 0; s < rounds; ++s) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                 // what this wave fetched is in LDS: vmcnt(0)
        __syncthreads();                                    // and what the others did; the other stage has been read
        if (s < mine) {                                     // uniform for the group
            const int at = (s & 1) * STAGE;
            f16x8 fa[FM][2], fb[FN][2];
#pragma unroll
            for (int j = 0; j < FN; ++j) {
#pragma unroll
                for (int p = 0; p < 2; ++p) fb[j][p] = *reinterpret_cast<const f16x8 *>(read_b + at + j * kFragBytes + p * kPartBytes);
            }
#pragma unroll
            for (int i = 0; i < FM; ++i) {
#pragma unroll
                for (int p = 0; p < 2; ++p) fa[i][p] = *reinterpret_cast<const f16x8 *>(read_a + at + i * kFragBytes + p * kPartBytes);
            }
            if (s + 1 < mine) fetch(s + 1);
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                f32x4 low[FN];
#pragma unroll
                for (int j = 0; j < FN; ++j) low[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i][0], fb[j][1], f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
                for (int j = 0; j < FN; ++j) low[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i][1], fb[j][0], low[j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i][0], fb[j][0], acc[i][j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < FN; ++j) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[i][j][q] = __builtin_fmaf(low[j][q], 0x1p-12f, acc[i][j][q]);
                }
            }
        }
    }
    constexpr int OWN = FM / GROUPS;                        // rows of sixteen that a group finishes
    const int64_t col0 = n0 + frag_b * 16 + (lane & 15), row0 = m0 + (frag_a + group * OWN) * 16 + (lane >> 4) * 4;
    bool odd = false;
    auto put = [&](int i, int j, f32x4 v) {
        const int64_t col = col0 + j * 16;
        const float r[4] = {v.x, v.y, v.z, v.w};
        const float by = sb.unscale[min(col, N - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t row = row0 + i * 16 + q;
            const float value = r[q] * sa.unscale[min(row, M - 1)] * by;
            odd |= !(__builtin_fabsf(value) < 3.0e38f);
            if (row < M && col < N) out[row * N + col] = value;
        }
    };
    static_assert(GROUPS == 1 || GROUPS == 2, "");
    if constexpr (GROUPS == 2) {
        __syncthreads();                                    // the stages have been read
        // each group hands the other half of its sums over and finishes the rest
        static_assert(FM % 2 == 0 && 4 * STAGE >= 2 * WAVES * OWN * FN * kWave * 16, "the sums fit the stages");
        f32x4 *give = reinterpret_cast<f32x4 *>(lds) + ((1 - group) * WAVES + wave) * (OWN * FN * kWave);
        const f32x4 *take = reinterpret_cast<const f32x4 *>(lds) + (group * WAVES + wave) * (OWN * FN * kWave);
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4 first = acc[i][j], second = acc[OWN + i][j];
                give[(i * FN + j) * kWave + lane] = group == 0 ? second : first;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) {
                const f32x4 first = acc[i][j], second = acc[OWN + i][j];
                put(i, j, (group == 0 ? first : second) + take[(i * FN + j) * kWave + lane]);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < OWN; ++i) {
#pragma unroll
            for (int j = 0; j < FN; ++j) put(i, j, acc[i][j]);
        }
    }
    // A row that holds an infinity or a NaN, or a sum that overflows: plain arithmetic decides what comes out.
    if (__builtin_amdgcn_ballot_w64(odd) != 0u) {
        for (int i = 0; i < OWN * FN * 4; ++i) {
            const int64_t row = row0 + i / (FN * 4) * 16 + i % 4, col = col0 + i / 4 % FN * 16;
            if (row >= M || col >= N || __builtin_fabsf(out[row * N + col]) < 3.0e38f) continue;
            float sum = 0.0f;
            for (int64_t k = 0; k < K; ++k) sum += a[row * K + k] * (b_deep ? b[col * K + k] : b[k * N + col]);
            out[row * N + col] = sum;
        }
    }
}

int64_t tiles_of(int64_t n, int tile) { return (n + tile - 1) / tile; }
int64_t parts_bytes(int64_t rows, int64_t K) { return frags_of(rows) * (K / kStep) * kFragBytes; }

template <bool DEEP_B, int HELD>
void launch_split(const float *a, const float *b, int64_t M, int64_t N, int64_t K, const Split &sa, const Split &sb, hipStream_t s)
{
    const int64_t waves = (K / kStep + HELD - 1) / HELD;
    launch(split_kernel<DEEP_B, HELD>, (unsigned)(frags_of(M) + frags_of(N)), (unsigned)(waves < kSplitWaves ? waves : kSplitWaves) * kWave, 0, s, a, b, M, N,
           K, sa, sb);
}
template <int TM, int TN, int WY, int WX, int GROUPS>
void launch_tiles(const float *a, const float *b, bool b_deep, int64_t M, int64_t N, int64_t K, float *out, const Split &sa, const Split &sb,
                  hipStream_t s)
{
    const int tm = (int)tiles_of(M, TM), tn = (int)tiles_of(N, TN);
    launch(product_kernel<TM, TN, WY, WX, GROUPS>, (unsigned)(tm * tn), GROUPS * WY * WX * kWave, 0, s, sa, sb, M, N, K, out, tm, tn, a, b, b_deep);
}

int32_t validate(int64_t M, int64_t N, int64_t K)
{
    if (M < 0 || N < 0 || K < 0) return SLIMFIT_ERR_INVALID_ARG;
    if (M == 0 || N == 0) return SLIMFIT_OK;
    if (K == 0 || K % kStep != 0 || K > 0x7FFFFFFFLL) return SLIMFIT_ERR_UNSUPPORTED;
    // (each factor is below 2^63: the products are looked at in floating point first)
    if ((double)M * (double)K > 1.0e18 || (double)N * (double)K > 1.0e18 || (double)M * (double)N > 1.0e18) return SLIMFIT_ERR_UNSUPPORTED;
    if ((double)tiles_of(M, 128) * (double)tiles_of(N, 64) > (double)(kMaxGridThreads / 512)) return SLIMFIT_ERR_UNSUPPORTED;
    if ((double)(frags_of(M) + frags_of(N)) > (double)(kMaxGridThreads / (kSplitWaves * kWave))) return SLIMFIT_ERR_UNSUPPORTED;
    return SLIMFIT_OK;
}

}  // namespace
}  // namespace slimfit

using namespace slimfit;

extern "C" int32_t slimfit_product_workspace(int64_t M, int64_t N, int64_t K, size_t *bytes)
{
    const int32_t rc = validate(M, N, K);
    if (rc != SLIMFIT_OK) return rc;
    if (!bytes) return SLIMFIT_ERR_INVALID_ARG;
    *bytes = M == 0 || N == 0 ? 0 : (size_t)(parts_bytes(M, K) + parts_bytes(N, K) + (frags_of(M) + frags_of(N)) * kFragRows * 4);
    return SLIMFIT_OK;
}

extern "C" int32_t slimfit_product(const float *a, const float *b, int32_t b_deep, int64_t M, int64_t N, int64_t K, float *out, void *workspace,
                                   size_t workspace_bytes, void *stream)
{
    StreamScope capture_aware(stream);
    size_t need = 0;
    int32_t rc = slimfit_product_workspace(M, N, K, &need);
    if (rc != SLIMFIT_OK || M == 0 || N == 0) return rc;
    if (!a || !b || !out || !workspace) return SLIMFIT_ERR_INVALID_ARG;
    if (!aligned_to(a, 16) || !aligned_to(b, 16) || !aligned_to(out, 4) || !aligned_to(workspace, 16)) return SLIMFIT_ERR_ALIGNMENT;
    if (workspace_bytes < need) return SLIMFIT_ERR_WORKSPACE;
    if ((rc = check_device_range(a, (size_t)M * (size_t)K * 4)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(b, (size_t)N * (size_t)K * 4)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(out, (size_t)M * (size_t)N * 4)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(workspace, need)) != SLIMFIT_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *at = static_cast<char *>(workspace);
    float *scales = reinterpret_cast<float *>(at + parts_bytes(M, K) + parts_bytes(N, K));
    const Split sa{at, scales}, sb{at + parts_bytes(M, K), scales + frags_of(M) * kFragRows};
    if (K <= 3 * kSplitWaves * kStep) b_deep ? launch_split<true, 3>(a, b, M, N, K, sa, sb, s) : launch_split<false, 3>(a, b, M, N, K, sa, sb, s);
    else b_deep ? launch_split<true, 6>(a, b, M, N, K, sa, sb, s) : launch_split<false, 6>(a, b, M, N, K, sa, sb, s);
    // A compute unit holds one workgroup; the tiles that take the fewest rounds of 256, a round's time being its tile's elements
    // and 8192 more (its first fetch and its stores).  That picks the fastest of these seven for 18 of 19 sizes tried (4096 x
    // 2304 x 768 in tiles of 256 x 144 57 us, of 256 x 192 62, of 128 x 96 67; 4096 x 3072 x 768 89, 68 and 84; 4096 x 768 x 768
    // 50, 59 and 32).  Two groups where a tile is so small that one would leave a SIMD a single wave.
    struct Tile {
        int tm, tn;
        void (*go)(const float *, const float *, bool, int64_t, int64_t, int64_t, float *, const Split &, const Split &, hipStream_t);
    };
    static constexpr Tile kTiles[] = {
        {256, 192, launch_tiles<256, 192, 4, 3, 1>}, {256, 144, launch_tiles<256, 144, 4, 3, 1>}, {256, 96, launch_tiles<256, 96, 4, 3, 1>},
        {128, 144, launch_tiles<128, 144, 2, 3, 2>}, {128, 128, launch_tiles<128, 128, 2, 2, 2>}, {128, 96, launch_tiles<128, 96, 2, 3, 2>},
        {128, 64, launch_tiles<128, 64, 2, 2, 2>}};
    constexpr int64_t kUnits = 256;
    const Tile *best = kTiles;
    double least = 0.0;
    for (const Tile &tile : kTiles) {
        const double takes = (double)tiles_of(tiles_of(M, tile.tm) * tiles_of(N, tile.tn), kUnits) * (tile.tm * tile.tn + 8192);
        if (&tile == kTiles || takes < least) {
            best = &tile;
            least = takes;
        }
    }
    best->go(a, b, b_deep != 0, M, N, K, out, sa, sb, s);
    return launch_status();
}
