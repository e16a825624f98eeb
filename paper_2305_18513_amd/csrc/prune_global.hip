// Alg. 5 applied to a whole flattened tensor (the form the paper uses for the
// standardised input of LayerNorm: keep int(numel * 0.1) entries with their
// indices, restore by zeros + scatter).
//
// A full sort is not needed to know which k entries a descending sort would put
// first: the k-th largest key T and the number of keys equal to T that belong to
// the kept set decide it.  The survivors are emitted in ascending index order
// (ties at T go to the lowest indices).
//
//   keys      order-preserving unsigned images of the elements: |x| as the IEEE
//             bit pattern without its sign (by magnitude) or the usual signed
//             fold with -0 mapped onto +0 (by value); 32 bits for fp32, 16 for
//             bf16.  A key's top 12 bits name its bin (1/16 of a binade by
//             magnitude, 1/8 by value).
//   sample    16 workgroups histogram the bins of up to 1024 vectors each, drawn one
//             from each equal stretch of the tensor; of 16 neighbouring stretches each
//             workgroup takes one, in an order that is shuffled from sixteen to sixteen.
//             Each fixes a bracket of its own, the bin of its sample's entry of T's
//             rank; the sweep joins the 16.  Nothing depends on the sample being right: the sweep's counts
//             show whether T lies inside the joint bracket.
//   sweep     one pass over the tensor, a workgroup per tile of 4096 elements:
//             the candidates (keys not below the bracket) are collected in index
//             order in LDS and leave as a contiguous run of (value, position)
//             records, 6 bytes each; the keys inside the bracket (1.5 - 3 % of a
//             bell-shaped tensor) are also filed in the tile's key list.
//   digits    T from the key lists, first in 2^9 .. 2^12 steps of the bracket's
//             width, then to the last bit (at most 2^14 steps).
//   count     keys above T and equal to T, per tile and per group of tiles.
//   write     a wave per tile reads the tile's records, drops those that T
//             rejects, and stores (value, index) pairs at their final places,
//             with the optional tile and row pointers.  The first output slot of a
//             tile is the sum of the group counts and of the counts of its own
//             group's earlier tiles.  A tile that holds more candidates than it has
//             record slots is read from the tensor instead (so are all tiles when
//             more than one entry in nine is kept: no records are made then).
//
// Plain route: a bracket that holds too much of the sample (heavy ties), a list
// that overflows (bunched keys) or a sample that missed T leaves the lists
// unused; the same launches then read the tensor once per digit (12 | 8 | 12
// bits, bf16 12 | 4), once for the counts and once to write, and the last launch,
// which otherwise returns at once, is the write.  When k / n is too close to 0 or
// to 1 for a sample to bracket T, the tensor's own histogram takes its place.
//
// No kernel waits on another workgroup: every step that needs the whole of the
// one before is a launch of its own (a last-workgroup ticket needs an agent-scope
// release in every workgroup, which on this part writes back the XCD's whole L2
// and made the sweeps 2-25x slower when it was tried), but a step that one
// workgroup could do is done by every workgroup of the next launch for itself.
#include "common.hpp"
#include "key_order.hpp"

#include <cmath>
#include <type_traits>

namespace slimfit {
namespace {

constexpr int kTileThreads = 256;          // sweep and write: 4 waves
constexpr int kVecPerThread = 4;           // 16-byte vectors a thread holds in a tensor histogram
constexpr int kWideThreads = 1024;         // histogram, count and single-workgroup kernels
constexpr int kWideWaves = kWideThreads / kWave;
constexpr int kTop = 12;                   // leading key bits that name a bin
constexpr int kTopBins = 1 << kTop;
constexpr int64_t kPtrTile = SLIMFIT_GLOBAL_TILE;   // granularity of the tile pointers, and the tile of every kernel
constexpr int kTileElems = (int)kPtrTile;
constexpr int kWaveElems = kTileElems / 4; // a tile is four rounds of 1024 elements, one a wave of the sweep

constexpr int kSampleWgs = 16;             // at most; a thread of them takes one vector
constexpr int kListSlots = kTileElems * 3 / 32;     // a tile's key list (in a workspace without records: fewer)
constexpr int kMinListSlots = 192;         // fewer are not worth the sweep; the readers load 128 ahead
constexpr int kRecSlots = 640;             // a tile's records: 10 % kept and 3 % more in the bracket, plus 5 standard deviations
constexpr int kRecShare = 9;               // records are made when k * 9 <= n
constexpr int kMaxBracketBins = 64;
constexpr int kMaxDigit3 = 14;             // bits of the last digit over the lists
constexpr int kListGrid = 128;             // workgroups that add a first-digit histogram of the lists (each adds its non-empty bins with global atomics)
constexpr int kWideGrid = 256;
constexpr unsigned kPlainGrid = 2048;      // plain route: workgroups that count and write (those of the last launch usually return at once)
constexpr int kCounters = 64;              // the sweep's totals, spread over as many cache lines
constexpr int kMaxGroups = kWideGrid;      // groups of tiles whose counts are summed ahead of the write
constexpr int kMaxGroupTiles = 2048;       // 2^31 elements are 2^19 tiles
constexpr int64_t kApartTiles = 4096;      // 1024 workgroups of the write

struct State {                             // first 128 bytes of the workspace
    uint32_t plain;                        // the sweep made no lists
    uint32_t overflow;                     // set by the sweep: a tile's key list ran out of slots
    uint32_t lo, last;                     // the bracket's smallest and largest key
    uint32_t digit2, shift2;               // bits of the first digit over the lists, and where it starts
    uint32_t use_plain;                    // set after the sweep: what every later launch goes by
    uint32_t prefix;                       // plain route: the top digit
    uint32_t lo2;                          // list route: lower edge of the first digit's step that holds T
    uint32_t k_rem, k_rem2, k_rem3;        // entries still to take ahead of each digit
    uint32_t prefix3;                      // plain route: all key bits but the last digit's
    uint32_t T, take_eq;                   // k-th largest key; how many keys equal to T are kept
    uint32_t pad[17];
};
static_assert(sizeof(State) == 128, "state size");

// bf16 elements that enter the selection widened to fp32: the rows of a bf16 tensor that is standardised
// on the way in (the standardised values are fp32, and so are the kept values)
struct Bf16Row {
    uint16_t h;
};
template <typename T> struct Elem;
template <> struct Elem<float> {
    static constexpr int EPV = 4;          // elements per 16-byte vector
    static constexpr int KEYBITS = 32;
    using Out = float;                     // type of the kept values
    using Key = float;                     // type whose key / digit plan applies
};
template <> struct Elem<uint16_t> {
    static constexpr int EPV = 8;
    static constexpr int KEYBITS = 16;
    static constexpr bool WIDEN = false;
    using Out = uint16_t;
    using Key = uint16_t;
};
template <> struct Elem<Bf16Row> {
    static constexpr int EPV = 8;
    static constexpr int KEYBITS = 32;
    static constexpr bool WIDEN = true;    // raw bits are the fp32 pattern of the widened element
    using Out = float;
    using Key = float;
};

// raw element bits -> key (larger key <=> earlier in the descending order)
template <typename T, bool MAG> __device__ __forceinline__ uint32_t make_key(uint32_t bits) { return key_of<Elem<T>::KEYBITS, MAG>(bits); }

__device__ __forceinline__ uint32_t raw_bits(const float *p) { return __builtin_bit_cast(uint32_t, *p); }
__device__ __forceinline__ uint32_t raw_bits(const uint16_t *p) { return *p; }
__device__ __forceinline__ uint32_t raw_bits(const Bf16Row *p) { return (uint32_t)p->h << 16; }
// the eight halves of a 16-byte vector, as they are or widened to fp32 bit patterns
template <bool WIDEN>
__device__ __forceinline__ void split_halves(const u32x4 &w, uint32_t (&bits)[8])
{
    const uint32_t q[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        bits[2 * i] = WIDEN ? q[i] << 16 : q[i] & 0xFFFFu;
        bits[2 * i + 1] = WIDEN ? q[i] & 0xFFFF0000u : q[i] >> 16;
    }
}

// The EPV raw elements of vector `v` (element offset v*EPV); returns how many of
// them lie inside [0, n).  A vector that straddles n is read element by element.
template <typename T, bool NT = false>
__device__ __forceinline__ int load_vec(const T *x, int64_t n, int64_t v, uint32_t (&bits)[Elem<T>::EPV])
{
    constexpr int EPV = Elem<T>::EPV;
    const int64_t e0 = v * EPV;
    if (e0 + EPV <= n) {
        const u32x4 w = load_global<NT>(reinterpret_cast<const u32x4 *>(x + e0));
        if constexpr (EPV == 4) {
            bits[0] = w.x; bits[1] = w.y; bits[2] = w.z; bits[3] = w.w;
        } else {
            split_halves<Elem<T>::WIDEN>(w, bits);
        }
        return EPV;
    }
    int valid = 0;
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
        bits[e] = 0u;
        if (e0 + e < n) {
            bits[e] = raw_bits(x + e0 + e);
            ++valid;
        }
    }
    return valid;
}

// INSIDE: the caller has established (uniformly for the workgroup) that every vector it touches lies
// wholly below n, so the load is unconditional and the code after it is straight-line; otherwise the
// vector may straddle n or lie past it.
template <typename T, bool INSIDE, bool NT = false>
__device__ __forceinline__ int load_tile_vec(const T *x, int64_t n, int64_t nvec, int64_t v,
                                             uint32_t (&bits)[Elem<T>::EPV])
{
    constexpr int EPV = Elem<T>::EPV;
    if constexpr (INSIDE) {
        const u32x4 w = load_global<NT>(reinterpret_cast<const u32x4 *>(x + v * EPV));
        if constexpr (EPV == 4) {
            bits[0] = w.x; bits[1] = w.y; bits[2] = w.z; bits[3] = w.w;
        } else {
            split_halves<Elem<T>::WIDEN>(w, bits);
        }
        return EPV;
    } else {
#pragma unroll
        for (int e = 0; e < EPV; ++e) bits[e] = 0u;
        return v < nvec ? load_vec<T, NT>(x, n, v, bits) : 0;
    }
}

// Optional standardisation on the way in (fp32 tensors): element j of row r
// enters the selection as x~ = fl(fl(x - mean[r]) * rstd[r]), two fp32 operations
// that every sweep repeats bit for bit, so the LayerNorm's standardised input is
// pruned without ever being stored.  r = j / H by a multiply-high with a magic
// number (exact for j < 2^31: magic = ceil(2^(31+l) / H), l = ceil(log2 H),
// r = mulhi(j, magic) >> (l - 1)).
struct Std {
    const float *mean, *rstd;
    uint32_t magic, shift;
    uint32_t vec_uniform;        // H is a multiple of 64 vectors: the 64 vectors a wave loads together share a row
    uint32_t last_row;
    uint32_t H;
    int32_t *row_ptr;            // optional output: survivors ahead of every row (rows + 1 entries)
};
// Applied to a vector after all of the thread's loads have been issued, so that
// the loads still overlap.  SCATTERED: the wave's vectors are not 64 consecutive
// ones, so every lane has a row of its own whatever H is.
template <typename T, bool STD, bool SCATTERED = false>
__device__ __forceinline__ void standardise(uint32_t (&bits)[Elem<T>::EPV], int valid, int64_t v, const Std &sd)
{
    constexpr int EPV = Elem<T>::EPV;
    if constexpr (STD) {
        // H is a multiple of EPV: a vector lies in one row.  No branch on `valid`: a vector past the end
        // takes the last row's statistics and its result is never looked at, and the statistic loads of
        // all of a thread's vectors can be issued together.
        (void)valid;
        uint32_t row = min(__umulhi((uint32_t)(v * EPV), sd.magic) >> sd.shift, sd.last_row);
        if (!SCATTERED && sd.vec_uniform) row = (uint32_t)__builtin_amdgcn_readfirstlane((int)row);    // scalar loads
        const float mu = sd.mean[row], rs = sd.rstd[row];
#pragma unroll
        for (int e = 0; e < EPV; ++e)
            bits[e] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(float, bits[e]) - mu) * rs);
    }
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v)            // absent sources contribute 0
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
// inclusive prefix sum over the 64 lanes of a wave
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v)
{
    v += dpp_or_zero<0x111, 0xF>(v);       // row_shr:1
    v += dpp_or_zero<0x112, 0xF>(v);       // row_shr:2
    v += dpp_or_zero<0x114, 0xF>(v);       // row_shr:4
    v += dpp_or_zero<0x118, 0xF>(v);       // row_shr:8
    v += dpp_or_zero<0x142, 0xA>(v);       // row_bcast:15 into rows 1 and 3
    v += dpp_or_zero<0x143, 0xC>(v);       // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ uint32_t wave_total_u32(uint32_t inclusive)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)inclusive, 63);
}

__device__ __forceinline__ uint32_t row_of(uint32_t e, const Std &sd) { return __umulhi(e, sd.magic) >> sd.shift; }

// vector (tile, round, group j, lane): a round is kGroups * 64 consecutive vectors
template <typename T> constexpr int kGroups = kWaveElems / (kWave * Elem<T>::EPV);      // 4 (fp32) or 2 (bf16)
template <typename T>
__device__ __forceinline__ int64_t round_vec(int64_t tile, int round, int j, int lane)
{
    return tile * (int64_t)(kTileElems / Elem<T>::EPV) + (int64_t)((round * kGroups<T> + j) * kWave + lane);
}
// a wave's round of a tile, standardised; INSIDE: the whole tile lies below n
template <typename T, bool STD, bool INSIDE, bool NT = false>
__device__ __forceinline__ void load_round(const T *__restrict__ x, int64_t n, int64_t tile, int round, int lane,
                                           uint32_t (&bits)[kGroups<T>][Elem<T>::EPV], int (&valid)[kGroups<T>],
                                           const Std &sd)
{
    const int64_t nvec = (n + Elem<T>::EPV - 1) / Elem<T>::EPV;
#pragma unroll
    for (int j = 0; j < kGroups<T>; ++j)
        valid[j] = load_tile_vec<T, INSIDE, NT>(x, n, nvec, round_vec<T>(tile, round, j, lane), bits[j]);
#pragma unroll
    for (int j = 0; j < kGroups<T>; ++j) standardise<T, STD>(bits[j], valid[j], round_vec<T>(tile, round, j, lane), sd);
}

// exclusive prefix sum of one value per thread over a workgroup of NT threads; two barriers
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *wave_sums)
{
    constexpr int NW = NT / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const uint32_t incl = wave_scan_u32(v);
    __syncthreads();                                       // wave_sums may still be read from a previous call
    if (lane == kWave - 1) wave_sums[wave] = incl;
    __syncthreads();
    uint32_t before = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) before += (w < wave) ? wave_sums[w] : 0u;
    return before + incl - v;
}

// The bin, counted from the top of a histogram of 2^bits bins, at which the running count reaches k_rem, and how
// many of its entries are still to take.  Every thread of the workgroup (NT threads, bits <= 14, 2^bits <= 16 NT)
// gets the answer.
struct Choice {
    uint32_t bin, left;
};
template <int NT, int PER>
__device__ __forceinline__ Choice select_bin_per(const uint32_t *hist, int bits, uint32_t k_rem)
{
    __shared__ uint32_t wave_sums[NT / kWave];
    __shared__ Choice found;
    const int top = (1 << bits) - 1 - (int)threadIdx.x * PER;              // this thread's highest bin
    uint32_t h[PER];
    uint32_t mine = 0u;
    if constexpr (PER == 1) {
        h[0] = hist[max(top, 0)];
    } else {                                               // 16 bytes a load (2^bits is a multiple of PER): 2^14 bins in 7.6 us, 14.0 in 4-byte loads
        static_assert(PER % 4 == 0, "vectors");
        const u32x4 *v = reinterpret_cast<const u32x4 *>(hist + max(top + 1 - PER, 0));
#pragma unroll
        for (int q = 0; q < PER / 4; ++q) {
            const u32x4 w = v[q];
            h[PER - 1 - 4 * q] = w.x; h[PER - 2 - 4 * q] = w.y; h[PER - 3 - 4 * q] = w.z; h[PER - 4 - 4 * q] = w.w;
        }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        h[j] = top >= 0 ? h[j] : 0u;
        mine += h[j];
    }
    if (threadIdx.x == 0) found = Choice{0u, 1u};
    uint32_t above = block_exclusive_scan<NT>(mine, wave_sums);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (above < k_rem && k_rem <= above + h[j]) found = Choice{(uint32_t)(top - j), k_rem - above};   // one thread, one j
        above += h[j];
    }
    __syncthreads();
    return found;
}
template <int NT>
__device__ __forceinline__ Choice select_bin(const uint32_t *hist, int bits, uint32_t k_rem)
{
    if ((1 << bits) <= NT) return select_bin_per<NT, 1>(hist, bits, k_rem);
    if ((1 << bits) <= 4 * NT) return select_bin_per<NT, 4>(hist, bits, k_rem);
    return select_bin_per<NT, 16>(hist, bits, k_rem);
}

// the counters, group sums and histograms, one contiguous piece of the workspace
__device__ __forceinline__ void clear_block(u32x4 *zero, int n16)
{
    for (int i = blockIdx.x * kWideThreads + threadIdx.x; i < n16; i += gridDim.x * kWideThreads) zero[i] = u32x4{0u, 0u, 0u, 0u};
}
__global__ void __launch_bounds__(kWideThreads) clear_kernel(u32x4 *zero, int n16, State *plain)      // plain: no sample and no sweep follow
{
    clear_block(zero, n16);
    if (plain && blockIdx.x == 0 && threadIdx.x == 0) plain->plain = 1u;      // (the thread that cleared it)
}

// ---- the sample ------------------------------------------------------------------------
// A workgroup's own bracket: the bins of its sample's entries of the ranks rank_hi <= rank_lo, counted from the largest,
// and how many of its entries lie between.  The sweep's bracket runs from the lowest to the highest of the workgroups'.
struct alignas(8) Edges {
    uint16_t hi, lo;
    uint32_t within;
};
// hist: kTopBins counts; the threads of a workgroup of kWideThreads call it, thread 0 gets the answer
__device__ __forceinline__ Edges find_edges(const uint32_t *hist, uint32_t rank_hi, uint32_t rank_lo)
{
    __shared__ uint32_t wave_sums[kWideWaves];
    __shared__ uint32_t edge[4];                           // highest bin, entries above it, lowest bin, entries down to it
    constexpr int PER = kTopBins / kWideThreads;           // 4
    const int slot = kWideThreads - 1 - (int)threadIdx.x;  // bins 4 * slot .. 4 * slot + 3, highest first
    const u32x4 f = reinterpret_cast<const u32x4 *>(hist)[slot];
    const uint32_t h[PER] = {f.w, f.z, f.y, f.x};
    if (threadIdx.x < 4) edge[threadIdx.x] = 0u;           // ranks outside the sample leave a bracket at the bottom: T is missed
    uint32_t above = block_exclusive_scan<kWideThreads>(h[0] + h[1] + h[2] + h[3], wave_sums);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t bin = (uint32_t)(4 * slot + PER - 1 - j);
        if (above < rank_hi && rank_hi <= above + h[j]) { edge[0] = bin; edge[1] = above; }
        if (above < rank_lo && rank_lo <= above + h[j]) { edge[2] = bin; edge[3] = above + h[j]; }
        above += h[j];
    }
    __syncthreads();
    return Edges{(uint16_t)edge[0], (uint16_t)edge[2], edge[3] - edge[1]};
}

__device__ __forceinline__ uint32_t mix(uint32_t i)
{
    uint32_t h = i * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    return h ^ (h >> 13);
}

// One vector of each of `total` equal stretches of the tensor (all vectors when there are no more than that), for
// stretch i at a place in it that depends on i only.  step: length of a stretch times 2^16.  Of each 16 stretches a
// workgroup takes one, which one being as good as random, so that columns of unlike scale come to all workgroups alike.
// Taken in turn, a workgroup saw the same columns of every row where a row is a multiple of 16 stretches, and the brackets
// lay apart: 512 x 128 with scales over a factor of e either way had 18 % of the tensor in the joint one, now 3 (without such columns 3
// either way).  Bound by latency (16 workgroups; one vector, its row's statistics, the histogram, the scan): a launch of one
// workgroup that added up the histograms and chose one bracket took 5 us after it.
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kWideThreads)
sample_kernel(const T *__restrict__ x, uint32_t total, uint64_t step, uint32_t rank_hi, uint32_t rank_lo, Edges *__restrict__ edges,
              State *st, u32x4 *zero, int n16, Std sd)
{
    constexpr int EPV = Elem<T>::EPV;
    __shared__ alignas(16) uint32_t bins[kTopBins];
    static_assert((kSampleWgs & (kSampleWgs - 1)) == 0, "gridDim.x, kSampleWgs or 1, is a power of two");
    const uint32_t mine = threadIdx.x * gridDim.x + ((blockIdx.x + (mix(threadIdx.x) >> 28)) & (gridDim.x - 1u)), i = min(mine, total - 1u);
    const uint64_t v0 = (i * step) >> 16, v1 = ((i + 1) * step) >> 16;
    const int64_t at = (int64_t)v0 + __umulhi(mix(i), (uint32_t)(v1 - v0));
    uint32_t bits[EPV];
    load_tile_vec<T, true>(x, 0, 0, at, bits);
    for (int b = threadIdx.x; b < kTopBins; b += kWideThreads) bins[b] = 0u;
    clear_block(zero, n16);
    __syncthreads();
    if (mine < total) {
        standardise<T, STD, true>(bits, EPV, at, sd);
#pragma unroll
        for (int e = 0; e < EPV; ++e) atomicAdd(&bins[make_key<T, MAG>(bits[e]) >> (Elem<T>::KEYBITS - kTop)], 1u);
    }
    __syncthreads();
    const Edges e = find_edges(bins, rank_hi, rank_lo);
    if (threadIdx.x < kSampleWgs / gridDim.x) edges[blockIdx.x + threadIdx.x] = e;      // (gridDim.x is kSampleWgs or 1)
    if (blockIdx.x == 0 && threadIdx.x == 0) st->overflow = 0u;
}

// The same from the tensor's own top digit, where T's rank is too close to an end for a sample.
// (The histogram is cleared again.)
__global__ void __launch_bounds__(kWideThreads) edges_kernel(uint32_t *hist, uint32_t k, Edges *__restrict__ edges, State *st)
{
    Edges e = find_edges(hist, k, k);
    // sixteen times this has to fit 32 bits below; a fourteenth of the largest tensor, from which on it is too much, is less
    e.within = min(e.within, 0xFFFFFFFFu / kSampleWgs);
    static_assert(0xFFFFFFFFu / kSampleWgs > 0x7FFFFFFFu / 14, "still too much");
    reinterpret_cast<u32x4 *>(hist)[threadIdx.x] = u32x4{0u, 0u, 0u, 0u};
    if (threadIdx.x < kSampleWgs) edges[threadIdx.x] = e;
    if (threadIdx.x == 0) st->overflow = 0u;
}

// The sweep's bracket; every workgroup works it out for itself.  size: entries that the sixteen edges were found among.
struct Bracket {
    uint32_t lo, last;                     // its smallest and largest key
    int range_bits, digit2;
    bool plain;                            // too wide for the digits, too much for the lists or among the NaN
};
__device__ __forceinline__ bool too_much(uint32_t bins, uint32_t within, uint64_t size, int list_slots)
{
    // the lists: on average 1/14 of the tensor where they hold 1/10.7 of a tile
    return bins > (uint32_t)kMaxBracketBins || (uint64_t)within * (14 * kListSlots) > size * (uint32_t)list_slots;
}
template <int KEYBITS, bool MAG>
__device__ __forceinline__ Bracket join_edges(u32x2 mine, uint64_t size, int list_slots)
{
    // a lane of each sixteen per pair of edges; by scalar loads and instructions, which a compute unit starts one at a time,
    // the sweep of 49152 x 1024 took 4 us longer
    static_assert(kSampleWgs == 16, "a DPP row");
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)group_max_u32(mine.x & 0xFFFFu, 16));
    const uint32_t lo = ~(uint32_t)__builtin_amdgcn_readfirstlane((int)group_max_u32(~(mine.x >> 16), 16));
    uint32_t sum = mine.y;
    sum += dpp_u32<kDppXor1>(sum);
    sum += dpp_u32<kDppXor2>(sum);
    sum += dpp_u32<kDppHalfMirror>(sum);
    sum += dpp_u32<kDppMirror>(sum);
    const uint32_t within = (uint32_t)__builtin_amdgcn_readfirstlane((int)sum);
    constexpr int shift = KEYBITS - kTop;
    const uint32_t nb = hi - lo + 1u;
    const int log_nb = nb > 1u ? 32 - __builtin_clz(nb - 1u) : 0;
    Bracket b;
    b.lo = lo << shift;
    b.last = b.lo + ((nb << shift) - 1u);
    b.range_bits = min(log_nb, 12) + shift;
    // the rest is at most 14 bits, 12 for the usual brackets of up to 16 bins: every workgroup of the count reads that
    // histogram whole (2^14 bins: 4096 x 768 in all 44.3 us, 2^12 40.9); more in this digit is more global atomics
    b.digit2 = min(b.range_bits, min(kTop, max(9, log_nb + 8)));
    b.plain = too_much(nb, within, size, list_slots) || !reach_exists<KEYBITS, MAG>(b.lo);
    return b;
}

// ---- the sweep: records, key lists and totals --------------------------------------------
// Bound by the read of the tensor and the records (0.7 bytes an element), with instruction issue close behind (bf16):
// 50.3 M fp32 39 us, 6.1 TB/s; 51.6 M bf16 28 us, 5.2 TB/s.  A candidate's place comes from prefix sums over the
// lanes' counts; a lane per element and two v_mbcnt each instead (4-byte loads, no counts) took 50 and 52 us.  The
// records pass through LDS so that they leave in whole lines: 37 MB written here and read by the write below in
// place of a second read of the tensor with one scattered store per survivor (42 us, bf16 44).  A candidate is compared,
// counted and staged by its lane's bit of one mask; making and comparing its key for each, branching around each store and
// leaving in 4-byte stores took 41.5 and 30 us.  Two tiles a workgroup: fp32 1.4 us slower, bf16 the same.
// Leaves tile_cnt[tile] = (keys above the bracket | candidates << 16, keys filed).
// byte address of a __shared__ object in the workgroup's LDS
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void *)p);
}
// Those lanes store two words at LDS byte address `at` and move 8 bytes on.  As an instruction sequence under the lane
// mask: from `if` the compiler makes a branch around every store, which nearly always some lane of the 64 has to follow
// there and back.
__device__ __forceinline__ void stage_if(uint64_t lanes, uint32_t &at, uint32_t first, uint32_t second)
{
    uint64_t all;
    asm volatile("s_and_saveexec_b64 %1, %2\n\t"
                 "ds_write2_b32 %0, %3, %4 offset1:1\n\t"
                 "v_add_u32_e32 %0, 8, %0\n\t"
                 "s_mov_b64 exec, %1"
                 : "+v"(at), "=&s"(all)
                 : "s"(lanes), "v"(first), "v"(second)
                 : "memory", "scc");
}
constexpr uint32_t kTooMany = 0x8000u;                      // in place of a tile's candidate count: it has no records
// REC: make records; the tensor is not read again then, and its loads are non-temporal.
template <bool REC>
struct SweepLds {
    alignas(16) u32x2 stage[REC ? kRecSlots : 2];           // (element bits, place in the tile)
    uint32_t wave_cnt[kTileThreads / kWave];
    uint32_t filed;
};
template <typename T, bool MAG, bool STD, bool INSIDE, bool REC>
__device__ __forceinline__ void
sweep_tile(const T *__restrict__ x, int64_t n, u32x2 edges, uint64_t size, State *st, uint64_t *__restrict__ counters, u32x2 *__restrict__ tile_cnt,
           uint32_t *__restrict__ lists, int list_slots, uint32_t *__restrict__ rec_val, uint16_t *__restrict__ rec_pos, const Std &sd,
           SweepLds<REC> &lds)
{
    constexpr int EPV = Elem<T>::EPV, G = kGroups<T>;
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = blockIdx.x;
    if (threadIdx.x == 0) lds.filed = 0u;
    uint32_t bits[G][EPV];
    int valid[G];
    load_round<T, STD, INSIDE, REC>(x, n, tile, wave, lane, bits, valid, sd);
    const Bracket br = join_edges<Elem<T>::KEYBITS, MAG>(edges, size, list_slots);
    if (blockIdx.x == 0 && threadIdx.x == 0) {             // for the launches that follow
        st->plain = br.plain ? 1u : 0u;
        st->lo = br.lo;
        st->last = br.last;
        st->digit2 = (uint32_t)br.digit2;
        st->shift2 = (uint32_t)(br.range_bits - br.digit2);
    }
    if (br.plain) return;
    const uint32_t lo = br.lo, last = br.last;

    uint64_t cand[G][EPV];                                  // lane masks of the candidates
    auto mark = [&](auto reach) {
#pragma unroll
        for (int j = 0; j < G; ++j) {
#pragma unroll
            for (int e = 0; e < EPV; ++e) cand[j][e] = __builtin_amdgcn_ballot_w64((INSIDE || e < valid[j]) && reach(bits[j][e]));
        }
    };
    constexpr int BITS = Elem<T>::KEYBITS;
    if (!MAG && reach_is_positive<BITS>(lo)) {              // uniform
        mark([&](uint32_t b) { return reaches_positive<BITS>(b, lo); });
    } else {
        const Reach edge = reach_of<BITS, MAG>(lo);
        mark([&](uint32_t b) { return reaches<BITS, MAG>(b, edge); });
    }
    // candidates per group of 64 vectors: three 10-bit fields (at most 512 each) in one prefix sum
    uint32_t packed[2] = {0u, 0u};
#pragma unroll
    for (int j = 0; j < G; ++j) {
        uint32_t c = 0u;
#pragma unroll
        for (int e = 0; e < EPV; ++e) c += __builtin_amdgcn_inverse_ballot_w64(cand[j][e]) ? 1u : 0u;
        packed[j / 3] += c << (10 * (j % 3));
    }
    uint32_t incl[2], total[2];
#pragma unroll
    for (int w = 0; w < (G + 2) / 3; ++w) {
        incl[w] = wave_scan_u32(packed[w]);
        total[w] = wave_total_u32(incl[w]);
    }
    uint32_t wave_total = 0u;
#pragma unroll
    for (int j = 0; j < G; ++j) wave_total += (total[j / 3] >> (10 * (j % 3))) & 1023u;
    if (lane == 0) lds.wave_cnt[wave] = wave_total;
    __syncthreads();                                        // `filed` is zero as well
    uint32_t pos = 0u, n_cand = 0u;
#pragma unroll
    for (int w = 0; w < kTileThreads / kWave; ++w) {
        const uint32_t c = lds.wave_cnt[w];
        pos += (w < wave) ? c : 0u;
        n_cand += c;
    }
    n_cand = (uint32_t)__builtin_amdgcn_readfirstlane((int)n_cand);
    uint32_t *keys = lists + tile * list_slots;
    const bool whole = REC && n_cand <= (uint32_t)kRecSlots;       // workgroup-uniform
    if (whole) {
#pragma unroll
        for (int j = 0; j < G; ++j) {
            uint32_t at = lds_address(lds.stage) + 8u * (pos + (((incl[j / 3] - packed[j / 3]) >> (10 * (j % 3))) & 1023u));
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                stage_if(cand[j][e], at, bits[j][e], (uint32_t)(((wave * G + j) * kWave + lane) * EPV + e));
            pos += (total[j / 3] >> (10 * (j % 3))) & 1023u;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the compiler does not count stage_if's writes
        __syncthreads();
        // four records a lane
        uint32_t *rv = rec_val + tile * kRecSlots;
        uint16_t *rp = rec_pos + tile * kRecSlots;
        static_assert(kRecSlots % 4 == 0 && kRecSlots <= 4 * kTileThreads, "one round");
        const uint32_t t = 4u * threadIdx.x;
        if ((uint32_t)(4 * kWave * wave) < n_cand) {        // wave-uniform
            const u32x4 *r = reinterpret_cast<const u32x4 *>(lds.stage + min(t, (uint32_t)kRecSlots - 4u));
            const u32x4 r0 = r[0], r1 = r[1];
            const uint32_t v[4] = {r0.x, r0.z, r1.x, r1.z};
            if (t < n_cand) {                               // (the slots up to the next vector take what is staged there)
                *reinterpret_cast<u32x4 *>(rv + t) = u32x4{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<u32x2 *>(rp + t) = u32x2{r0.y | (r0.w << 16), r1.y | (r1.w << 16)};
            }
            uint64_t m[4];
            uint32_t n_keys = 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                m[q] = __builtin_amdgcn_ballot_w64(t + q < n_cand && make_key<T, MAG>(v[q]) <= last);
                n_keys += (uint32_t)__builtin_popcountll(m[q]);
            }
            if (n_keys != 0u) {                             // wave-uniform
                uint32_t slot = 0u;
                if (lane == 0) slot = atomicAdd(&lds.filed, n_keys);
                slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t at = slot + lanes_below(m[q]);
                    if (__builtin_amdgcn_inverse_ballot_w64(m[q]) && at < (uint32_t)list_slots) keys[at] = make_key<T, MAG>(v[q]);
                    slot += (uint32_t)__builtin_popcountll(m[q]);
                }
            }
        }
    } else {
        uint32_t in_bracket = 0u;
#pragma unroll
        for (int j = 0; j < G; ++j) {
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                const uint32_t key = make_key<T, MAG>(bits[j][e]);
                in_bracket += ((INSIDE || e < valid[j]) && key >= lo && key <= last) ? 1u : 0u;
            }
        }
        const uint32_t upto = wave_scan_u32(in_bracket), all = wave_total_u32(upto);
        if (all) {                                          // wave-uniform
            uint32_t slot = 0u;
            if (lane == 0) slot = atomicAdd(&lds.filed, all);
            slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot) + upto - in_bracket;
#pragma unroll
            for (int j = 0; j < G; ++j) {
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const uint32_t key = make_key<T, MAG>(bits[j][e]);
                    if ((INSIDE || e < valid[j]) && key >= lo && key <= last) {
                        if (slot < (uint32_t)list_slots) keys[slot] = key;
                        ++slot;
                    }
                }
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t f = lds.filed, gt = n_cand - f;
        tile_cnt[tile] = u32x2{gt | ((whole ? n_cand : kTooMany) << 16), min(f, (uint32_t)list_slots)};
        if (f > (uint32_t)list_slots) st->overflow = 1u;
        atomicAdd(reinterpret_cast<unsigned long long *>(counters + (tile & (kCounters - 1)) * 8),
                  (unsigned long long)gt | ((unsigned long long)f << 32));
    }
}

template <typename T, bool MAG, bool STD, bool REC>
__global__ void __launch_bounds__(kTileThreads)
sweep_kernel(const T *__restrict__ x, int64_t n, const Edges *__restrict__ edges, uint64_t size, State *st, uint64_t *__restrict__ counters, u32x2 *__restrict__ tile_cnt,
             uint32_t *__restrict__ lists, int list_slots, uint32_t *__restrict__ rec_val, uint16_t *__restrict__ rec_pos, Std sd)
{
    __shared__ SweepLds<REC> lds;
    const u32x2 mine = reinterpret_cast<const u32x2 *>(edges)[threadIdx.x & (kSampleWgs - 1)];
    // The tile is asked for before the edges have arrived, unless one pair of them says that it may not be needed.
    const u32x2 one = reinterpret_cast<const u32x2 *>(edges)[blockIdx.x & (kSampleWgs - 1)];
    if (too_much((one.x & 0xFFFFu) - (one.x >> 16) + 1u, one.y * kSampleWgs, size, list_slots) && blockIdx.x != 0 &&
        join_edges<Elem<T>::KEYBITS, MAG>(mine, size, list_slots).plain)
        return;
    if (((int64_t)blockIdx.x + 1) * kTileElems <= n)        // workgroup-uniform: the whole tile lies below n
        sweep_tile<T, MAG, STD, true, REC>(x, n, mine, size, st, counters, tile_cnt, lists, list_slots, rec_val, rec_pos, sd, lds);
    else
        sweep_tile<T, MAG, STD, false, REC>(x, n, mine, size, st, counters, tile_cnt, lists, list_slots, rec_val, rec_pos, sd, lds);
}

// ---- one digit: LDS histogram of the matching keys, non-empty bins added to the global one ----
// Of the tensor; FIRST: the top digit, every key matches and there is no branch around the ds_add.  The top digit
// keeps kCopies histograms, one per lane modulo kCopies: the plain route is the one of tensors with few distinct
// values, whose lanes would queue for a handful of LDS words (50.3 M fp32 multiples of a half: 89 us with one, 62 with
// four, 58 with eight).
constexpr int kCopies = 8;
constexpr int kCopyStride = kTopBins + 8;      // a bin's copies lie in banks of their own (at kTopBins all in one: bf16 ties 59.4 us, now 38.2)
constexpr int kCopyWords = kCopies * kCopyStride;
template <typename T, bool MAG, bool STD, bool FIRST>
__device__ __forceinline__ void tensor_hist(const T *__restrict__ x, int64_t n, uint32_t prefix, uint32_t mask, int shift,
                                            int nbins, uint32_t *bins, const Std &sd)
{
    constexpr int EPV = Elem<T>::EPV;
    const int64_t nvec = (n + EPV - 1) / EPV;
    const int64_t nfull = n / EPV;                            // vectors wholly below n
    const int64_t chunk = (int64_t)kWideThreads * kVecPerThread;
    const uint32_t copy = (threadIdx.x % kCopies) * kCopyStride;
    auto sweep = [&](auto inside_tag, int64_t base) {
        constexpr bool INSIDE = decltype(inside_tag)::value;
        uint32_t bits[kVecPerThread][EPV];
        int valid[kVecPerThread];
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j)
            valid[j] = load_tile_vec<T, INSIDE>(x, n, nvec, base + (int64_t)j * kWideThreads + threadIdx.x, bits[j]);
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j)
            standardise<T, STD>(bits[j], valid[j], base + (int64_t)j * kWideThreads + threadIdx.x, sd);
#pragma unroll
        for (int j = 0; j < kVecPerThread; ++j) {
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                if (INSIDE || e < valid[j]) {
                    const uint32_t key = make_key<T, MAG>(bits[j][e]);
                    if (FIRST) atomicAdd(&bins[copy + (key >> shift)], 1u);
                    else if ((key & mask) == prefix) atomicAdd(&bins[(key >> shift) & (uint32_t)(nbins - 1)], 1u);
                }
            }
        }
    };
    for (int64_t base = (int64_t)blockIdx.x * chunk; base < nvec; base += (int64_t)gridDim.x * chunk) {
        if (base + chunk <= nfull) sweep(std::true_type{}, base);      // workgroup-uniform
        else sweep(std::false_type{}, base);
    }
}
// The key lists of four tiles t, t + stride, ...: counts and first 128 slots (those past the count hold anything).
struct FourLists {
    u32x2 cnt[4];
    uint32_t a[4], b[4];
    __device__ __forceinline__ void load(const u32x2 *__restrict__ tile_cnt, const uint32_t *__restrict__ lists, int list_slots,
                                         int64_t t, int64_t stride, int64_t end)
    {
        const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t at = min(t + u * stride, end - 1);
            cnt[u] = tile_cnt[at];
            a[u] = lists[at * list_slots + lane];
            b[u] = lists[at * list_slots + lane + kWave];
        }
    }
    template <typename F>
    __device__ __forceinline__ void each(int u, const uint32_t *__restrict__ keys, F f) const
    {
        const uint32_t lane = threadIdx.x & (kWave - 1), n = cnt[u].y;
        if (lane < n) f(a[u]);
        if (lane + kWave < n) f(b[u]);
        for (uint32_t i = lane + 2 * kWave; i < n; i += kWave) f(keys[i]);
    }
};
// f(key) for every filed key, a wave per tile; first: the wave's first four, loaded ahead by the caller
template <typename F>
__device__ __forceinline__ void for_each_filed(FourLists &first, const u32x2 *__restrict__ tile_cnt,
                                               const uint32_t *__restrict__ lists, int list_slots, int64_t ntiles, int grid, F f)
{
    const int64_t waves = (int64_t)grid * kWideWaves;
    for (int64_t t = (int64_t)blockIdx.x * kWideWaves + (threadIdx.x >> 6); t < ntiles;) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (t + u * waves < ntiles) first.each(u, lists + (t + u * waves) * list_slots, f);
        t += 4 * waves;
        if (t < ntiles) first.load(tile_cnt, lists, list_slots, t, waves, ntiles);
    }
}
__device__ __forceinline__ void clear_bins(uint32_t *bins, int nbins)
{
    for (int i = threadIdx.x; i < nbins; i += kWideThreads) bins[i] = 0u;
}
template <int COPIES = 1>
__device__ __forceinline__ void add_bins(const uint32_t *bins, uint32_t *__restrict__ hist, int nbins)
{
    for (int i = threadIdx.x; i < nbins; i += kWideThreads) {
        uint32_t c = 0u;
#pragma unroll
        for (int u = 0; u < COPIES; ++u) c += bins[u * kCopyStride + i];
        if (c) atomicAdd(&hist[i], c);
    }
}

// the tensor's own top digit, in place of the sample
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kWideThreads)
top_digit_kernel(const T *__restrict__ x, int64_t n, uint32_t *__restrict__ hist, Std sd)
{
    __shared__ uint32_t bins[kCopyWords];
    clear_bins(bins, kCopyWords);
    __syncthreads();
    tensor_hist<T, MAG, STD, true>(x, n, 0u, 0u, Elem<T>::KEYBITS - kTop, kTopBins, bins, sd);
    __syncthreads();
    add_bins<kCopies>(bins, hist, kTopBins);
}

// The verdict on the bracket, and the first digit (list route: of the bracket; plain route: the top one).
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kWideThreads)
digit_kernel(const T *__restrict__ x, int64_t n, State *st, const uint64_t *__restrict__ counters,
             const u32x2 *__restrict__ tile_cnt, const uint32_t *__restrict__ lists, int list_slots, uint32_t *__restrict__ hist2,
             int64_t ntiles, uint32_t k, Std sd)
{
    __shared__ uint32_t bins[kCopyWords];
    const int lane = threadIdx.x & (kWave - 1);
    static_assert(kCounters == kWave, "a lane per counter");
    const int grid = min((int)gridDim.x, kListGrid);
    FourLists first;
    first.load(tile_cnt, lists, list_slots, (int64_t)blockIdx.x * kWideWaves + (threadIdx.x >> 6), (int64_t)grid * kWideWaves, ntiles);
    const uint64_t c = counters[lane * 8];
    const uint32_t gt = wave_total_u32(wave_scan_u32((uint32_t)c)), in = wave_total_u32(wave_scan_u32((uint32_t)(c >> 32)));
    const bool plain = st->plain || st->overflow || gt >= k || k - gt > in;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->use_plain = plain ? 1u : 0u;
        st->k_rem = plain ? k : k - gt;
    }
    if (!plain && (int)blockIdx.x >= grid) return;
    const int nbins = plain ? kTopBins : 1 << st->digit2;
    clear_bins(bins, plain ? kCopyWords : nbins);
    __syncthreads();
    if (plain) {
        tensor_hist<T, MAG, STD, true>(x, n, 0u, 0u, Elem<T>::KEYBITS - kTop, kTopBins, bins, sd);
    } else {
        const uint32_t lo = st->lo, shift = st->shift2, top = (uint32_t)nbins - 1u;
        for_each_filed(first, tile_cnt, lists, list_slots, ntiles, grid, [&](uint32_t key) { atomicAdd(&bins[min((key - lo) >> shift, top)], 1u); });
    }
    __syncthreads();
    if (plain) add_bins<kCopies>(bins, hist2, kTopBins);
    else add_bins(bins, hist2, nbins);
}

// 32-bit keys: the second digit (list route: the rest of the key).
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kWideThreads)
second_digit_kernel(const T *__restrict__ x, int64_t n, State *st, const u32x2 *__restrict__ tile_cnt,
                    const uint32_t *__restrict__ lists, int list_slots, const uint32_t *__restrict__ hist2,
                    uint32_t *__restrict__ hist3, int64_t ntiles, Std sd)
{
    __shared__ uint32_t bins[1 << kMaxDigit3];
    FourLists first;
    first.load(tile_cnt, lists, list_slots, (int64_t)blockIdx.x * kWideWaves + (threadIdx.x >> 6), (int64_t)gridDim.x * kWideWaves, ntiles);
    const bool plain = st->use_plain != 0u;
    const Choice c = select_bin<kWideThreads>(hist2, plain ? kTop : (int)st->digit2, st->k_rem);
    const uint32_t shift = st->shift2;
    const uint32_t lo2 = st->lo + (c.bin << shift);
    const uint32_t prefix = c.bin << (32 - kTop), mask = ~0u << (32 - kTop);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->k_rem2 = c.left;
        st->lo2 = lo2;
        st->prefix = prefix;
    }
    const int nbins = plain ? 256 : 1 << shift;
    clear_bins(bins, nbins);
    __syncthreads();
    if (plain)
        tensor_hist<T, MAG, STD, false>(x, n, prefix, mask, 12, nbins, bins, sd);
    else
        for_each_filed(first, tile_cnt, lists, list_slots, ntiles, (int)gridDim.x, [&](uint32_t key) {
            if (key - lo2 < (uint32_t)nbins) atomicAdd(&bins[key - lo2], 1u);
        });
    __syncthreads();
    add_bins(bins, hist3, nbins);
}

// List route: T, then the keys above T and equal to T per group of tiles and, inside a group, ahead of every tile.
// Plain route: the last digit.
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kWideThreads)
count_kernel(const T *__restrict__ x, int64_t numel, State *st, const u32x2 *__restrict__ tile_cnt, const uint32_t *__restrict__ lists,
             int list_slots,
             const uint32_t *__restrict__ hist2, const uint32_t *__restrict__ hist3, uint32_t *__restrict__ hist4,
             u32x2 *__restrict__ tile_sum, u32x2 *__restrict__ group_sum, int64_t ntiles, int group_tiles, Std sd)
{
    constexpr bool WIDE_KEY = Elem<T>::KEYBITS == 32;
    __shared__ uint32_t bins[kTopBins];                     // list route: the group's tiles' sums
    __shared__ uint32_t wave_sums[kWideWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * group_tiles, t1 = min(t0 + group_tiles, ntiles);
    FourLists four;
    four.load(tile_cnt, lists, list_slots, t0 + wave, kWideWaves, t1);
    const bool plain = st->use_plain != 0u;
    const Choice c = WIDE_KEY ? select_bin<kWideThreads>(hist3, plain ? 8 : (int)st->shift2, st->k_rem2)
                              : select_bin<kWideThreads>(hist2, plain ? kTop : (int)st->digit2, st->k_rem);
    if (plain) {
        const uint32_t prefix = WIDE_KEY ? st->prefix | (c.bin << 12) : c.bin << 4;
        constexpr uint32_t low = WIDE_KEY ? 0xFFFu : 0xFu;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            st->prefix3 = prefix;
            st->k_rem3 = c.left;
        }
        clear_bins(bins, (int)low + 1);
        __syncthreads();
        tensor_hist<T, MAG, STD, false>(x, numel, prefix, ~low, 0, (int)low + 1, bins, sd);
        __syncthreads();
        add_bins(bins, hist4, (int)low + 1);
        return;
    }
    const uint32_t Tk = (WIDE_KEY ? st->lo2 : st->lo) + c.bin;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->T = Tk;
        st->take_eq = c.left;
    }
    u32x2 *sum = reinterpret_cast<u32x2 *>(bins);
    for (int64_t t = t0 + wave; t < t1;) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t tile = t + u * kWideWaves;
            if (tile >= t1) break;                          // wave-uniform
            uint32_t gt = 0u, eq = 0u;
            four.each(u, lists + tile * list_slots, [&](uint32_t key) {
                gt += key > Tk ? 1u : 0u;
                eq += key == Tk ? 1u : 0u;
            });
            const uint32_t both = wave_total_u32(wave_scan_u32(gt | (eq << 16)));
            if (lane == 0) sum[tile - t0] = u32x2{(four.cnt[u].x & 0xFFFFu) + (both & 0xFFFFu), both >> 16};
        }
        t += 4 * kWideWaves;
        if (t < t1) four.load(tile_cnt, lists, list_slots, t, kWideWaves, t1);
    }
    __syncthreads();
    // the sums ahead of every tile of the group, and the group's own; two tiles a thread
    static_assert(kMaxGroupTiles <= 2 * kWideThreads && kMaxGroupTiles * 2 <= kTopBins, "group size");
    const int n = (int)(t1 - t0), i = 2 * (int)threadIdx.x;
    const u32x2 zero = {0u, 0u}, s0 = i < n ? sum[i] : zero, s1 = i + 1 < n ? sum[i + 1] : zero;
    const u32x2 a = {block_exclusive_scan<kWideThreads>(s0.x + s1.x, wave_sums), block_exclusive_scan<kWideThreads>(s0.y + s1.y, wave_sums)};
    if (i < n) tile_sum[t0 + i] = a;
    if (i + 1 < n) tile_sum[t0 + i + 1] = a + s0;
    if (i < n && i + 2 >= n) group_sum[blockIdx.x] = a + s0 + s1;
}

template <typename T> __device__ __forceinline__ void store_raw(T *p, uint32_t bits);
template <> __device__ __forceinline__ void store_raw<float>(float *p, uint32_t bits) { *p = __builtin_bit_cast(float, bits); }
template <> __device__ __forceinline__ void store_raw<uint16_t>(uint16_t *p, uint32_t bits) { *p = (uint16_t)bits; }

__device__ __forceinline__ void stream_raw(float *p, uint32_t bits) { __builtin_nontemporal_store(__builtin_bit_cast(float, bits), p); }
__device__ __forceinline__ void stream_raw(uint16_t *p, uint32_t bits) { __builtin_nontemporal_store((uint16_t)bits, p); }

// Where the outputs go.
template <typename T>
struct Out {
    typename Elem<T>::Out *vals;
    int32_t *idx, *tile_ptr;
    uint32_t k;
};

// keys above T / equal to T of a tile, from the tensor (a workgroup, a wave a round); the sums are thread 0's
template <typename T, bool MAG, bool STD, bool INSIDE>
__device__ __forceinline__ u32x2 count_tensor_tile(const T *__restrict__ x, int64_t n, int64_t tile, uint32_t Tk, const Std &sd)
{
    constexpr int EPV = Elem<T>::EPV, G = kGroups<T>;
    __shared__ uint32_t part[kTileThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    uint32_t bits[G][EPV];
    int valid[G];
    load_round<T, STD, INSIDE>(x, n, tile, wave, lane, bits, valid, sd);
    uint32_t packed = 0u;
#pragma unroll
    for (int j = 0; j < G; ++j) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const uint32_t key = make_key<T, MAG>(bits[j][e]);
            if (INSIDE || e < valid[j]) packed += (key > Tk ? 1u : 0u) + (key == Tk ? 1u << 16 : 0u);
        }
    }
    const uint32_t sum = wave_total_u32(wave_scan_u32(packed));    // at most 1024 in either half
    __syncthreads();                                        // the previous tile's sums have been read
    if (lane == 0) part[wave] = sum;
    __syncthreads();
    u32x2 r = {0u, 0u};
#pragma unroll
    for (int w = 0; w < kTileThreads / kWave; ++w) {
        r.x += part[w] & 0xFFFFu;
        r.y += part[w] >> 16;
    }
    return r;
}

// the survivors of a tile in ascending index order, from the tensor (a workgroup, a wave a round)
template <typename T, bool MAG, bool STD, bool INSIDE>
__device__ __forceinline__ void write_tensor_tile(const T *__restrict__ x, int64_t n, int64_t tile, uint32_t Tk, uint32_t out_base,
                                                  uint32_t budget, const Out<T> &out, const Std &sd)
{
    constexpr int EPV = Elem<T>::EPV, G = kGroups<T>;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    __shared__ uint32_t part[kTileThreads / kWave];
    uint32_t bits[G][EPV];
    int valid[G];
    load_round<T, STD, INSIDE>(x, n, tile, wave, lane, bits, valid, sd);
    uint32_t packed[G], incl[G];                            // keys above T | keys equal T << 16: at most 512 per group and field
    uint32_t mine = 0u;
#pragma unroll
    for (int j = 0; j < G; ++j) {
        packed[j] = 0u;
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const uint32_t key = make_key<T, MAG>(bits[j][e]);
            if (INSIDE || e < valid[j]) packed[j] += (key > Tk ? 1u : 0u) + (key == Tk ? 1u << 16 : 0u);
        }
        incl[j] = wave_scan_u32(packed[j]);
        mine += wave_total_u32(incl[j]);
    }
    __syncthreads();                                        // the previous tile's sums have been read
    if (lane == 0) part[wave] = mine;
    __syncthreads();
    uint32_t run_gt = 0u, run_eq = 0u;                      // survivors / ties of this tile ahead of the current group
#pragma unroll
    for (int w = 0; w < kTileThreads / kWave; ++w) {
        run_gt += w < wave ? part[w] & 0xFFFFu : 0u;
        run_eq += w < wave ? part[w] >> 16 : 0u;
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const uint32_t excl = incl[j] - packed[j], group = wave_total_u32(incl[j]);
        uint32_t my_gt = run_gt + (excl & 0xFFFFu);
        uint32_t my_eq = run_eq + (excl >> 16);
        const int64_t e0 = round_vec<T>(tile, wave, j, lane) * EPV;
        if constexpr (STD) {
            if (sd.row_ptr && valid[j]) {                   // rows start on vector boundaries
                const uint32_t row = row_of((uint32_t)e0, sd);
                if ((uint32_t)e0 == row * sd.H) sd.row_ptr[row] = (int32_t)(out_base + my_gt + min(my_eq, budget));
            }
        }
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            if (INSIDE || e < valid[j]) {
                const uint32_t key = make_key<T, MAG>(bits[j][e]);
                const bool above = key > Tk;
                const bool tie = key == Tk;
                if (above || (tie && my_eq < budget)) {
                    const uint32_t pos = out_base + my_gt + min(my_eq, budget);
                    if (pos < out.k) {                      // always true for consistent counts; guards the stores
                        store_raw<typename Elem<T>::Out>(out.vals + pos, bits[j][e]);
                        out.idx[pos] = (int32_t)(e0 + e);
                    }
                }
                my_gt += above ? 1u : 0u;
                my_eq += tie ? 1u : 0u;
            }
        }
        run_gt += group & 0xFFFFu;
        run_eq += group >> 16;
    }
}

// the survivors of a tile from its records (a wave; n_cand <= kRecSlots of them, four a lane and chunk): they pass through
// the wave's LDS and leave as aligned 16-byte vectors, and a row's pointer is found among them by bisection.  Bound by
// latency (a wave's one round of loads, 2.4 waves a slot): 50.3 M fp32 entries, 5.03 M kept, 19 us for 80 MB, 51.6 M bf16 16;
// 22 and 19 with a record a lane, 4-byte stores and the pointers from each survivor's left neighbour.
constexpr int kRecChunk = 4 * kWave;
constexpr int kRecChunks = (kRecSlots + kRecChunk - 1) / kRecChunk;
constexpr int kFirstChunks = 2;            // loaded before the count is known
constexpr int kWriteSlots = kRecSlots + 4; // a wave's survivors in LDS, behind up to three unused slots
template <typename T, bool MAG, bool STD>
__device__ __forceinline__ void write_record_tile(const u32x4 (&v)[kRecChunks], const u32x2 (&p)[kRecChunks], uint32_t n_cand,
                                                  int64_t n, int64_t tile, uint32_t Tk, uint32_t out_base, uint32_t budget,
                                                  const Out<T> &out, const Std &sd, u32x2 *lds)
{
    using Val = typename Elem<T>::Out;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t t0 = (uint32_t)(tile * kTileElems);
    // survivor s goes to lds[phase + s], so that where both outputs lie alike an aligned vector of theirs is one of lds
    const uint32_t phase = ((uint32_t)(reinterpret_cast<uintptr_t>(out.idx) / 4) + out_base) & 3u;
    uint32_t run_gt = 0u, run_eq = 0u;
#pragma unroll
    for (int u = 0; u < kRecChunks; ++u) {
        if ((uint32_t)(u * kRecChunk) >= n_cand) break;     // wave-uniform
        const uint32_t i = (uint32_t)(u * kRecChunk + 4 * lane);
        const uint32_t r[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
        const uint32_t at[4] = {p[u].x & 0xFFFFu, p[u].x >> 16, p[u].y & 0xFFFFu, p[u].y >> 16};
        uint64_t above[4], tie[4];                          // lane masks
        uint32_t c = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t key = make_key<T, MAG>(r[q]);
            above[q] = __builtin_amdgcn_ballot_w64(i + q < n_cand && key > Tk);
            tie[q] = __builtin_amdgcn_ballot_w64(i + q < n_cand && key == Tk);
            c += __builtin_amdgcn_inverse_ballot_w64(above[q]) ? 1u : 0u;
        }
        if ((tie[0] | tie[1] | tie[2] | tie[3]) != 0u) {    // wave-uniform
#pragma unroll
            for (int q = 0; q < 4; ++q) c += __builtin_amdgcn_inverse_ballot_w64(tie[q]) ? 1u << 16 : 0u;
        }
        const uint32_t incl = wave_scan_u32(c), all = wave_total_u32(incl);
        uint32_t my_eq = run_eq + ((incl - c) >> 16);
        uint32_t to = lds_address(lds) + 8u * (phase + run_gt + ((incl - c) & 0xFFFFu) + min(my_eq, budget));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint64_t keep = above[q];
            if (tie[q] != 0u) {                             // wave-uniform
                const bool t = __builtin_amdgcn_inverse_ballot_w64(tie[q]);
                keep |= __builtin_amdgcn_ballot_w64(t && my_eq < budget);
                my_eq += t ? 1u : 0u;
            }
            stage_if(keep, to, r[q], t0 + at[q]);
        }
        run_gt += all & 0xFFFFu;
        run_eq += all >> 16;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the compiler does not count stage_if's writes
    const uint32_t kept = run_gt + min(run_eq, budget);
    const uint32_t first = min(out_base, out.k), end = phase + min(kept, out.k - first);     // (consistent counts never pass k)
    const bool alike = sizeof(Val) == 4 && ((reinterpret_cast<uintptr_t>(out.vals) ^ reinterpret_cast<uintptr_t>(out.idx)) & 15u) == 0u;
    if (alike) {
        for (uint32_t b = 0u; b < end; b += kRecChunk) {
            const uint32_t i = b + 4u * (uint32_t)lane;
            const u32x4 *pair = reinterpret_cast<const u32x4 *>(lds + min(i, (uint32_t)kWriteSlots - 4u));
            const u32x4 a = pair[0], c = pair[1];
            const uint32_t val[4] = {a.x, a.z, c.x, c.z}, idx[4] = {a.y, a.w, c.y, c.w};
            const int64_t o = (int64_t)first + i - phase;   // output slot of lds[i]
            if (i >= phase && i + 4u <= end) {
                __builtin_nontemporal_store(u32x4{val[0], val[1], val[2], val[3]}, reinterpret_cast<u32x4 *>(out.vals + o));
                __builtin_nontemporal_store(u32x4{idx[0], idx[1], idx[2], idx[3]}, reinterpret_cast<u32x4 *>(out.idx + o));
            } else {                                        // the vectors shared with the tiles before and after
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (i + q >= phase && i + q < end) {
                        stream_raw(out.vals + o + q, val[q]);
                        __builtin_nontemporal_store((int32_t)idx[q], out.idx + o + q);
                    }
                }
            }
        }
    } else {
        for (uint32_t i = phase + (uint32_t)lane; i < end; i += kWave) {
            const u32x2 r = lds[i];
            stream_raw(out.vals + (first + i - phase), r.x);
            __builtin_nontemporal_store((int32_t)r.y, out.idx + (first + i - phase));
        }
    }
    if constexpr (STD) {
        if (sd.row_ptr) {
            // the rows that begin in the tile: how many survivors lie ahead of their first element
            const int r0 = t0 > 0u ? (int)row_of(t0 - 1u, sd) + 1 : 0, r1 = (int)row_of((uint32_t)(min((int64_t)t0 + kTileElems, n) - 1), sd);
            for (int r = r0 + lane; r <= r1; r += kWave) {
                const uint32_t e = (uint32_t)r * sd.H;
                uint32_t before = 0u;
#pragma unroll
                for (uint32_t step = 512u; step > 0u; step >>= 1) {
                    const uint32_t to = before + step;
                    if (to <= kept && lds[phase + min(to, (uint32_t)kRecSlots) - 1u].y < e) before = to;
                }
                sd.row_ptr[r] = (int32_t)(out_base + before);
            }
        }
    }
}

// List route: keys above T / equal to T ahead of a tile: those ahead of it in its group plus the sums of the groups
// ahead (a wave, no barrier).
__device__ __forceinline__ u32x2 sums_ahead(const u32x2 *__restrict__ tile_sum, const u32x2 *__restrict__ group_sum, int64_t tile,
                                            int group_tiles)
{
    const int lane = threadIdx.x & (kWave - 1), group = (int)(tile / group_tiles);
    u32x2 a = {0u, 0u};
#pragma unroll
    for (int u = 0; u < kMaxGroups / kWave; ++u) {
        const u32x2 s = group_sum[u * kWave + lane];        // (past the last group: zeros)
        a += u * kWave + lane < group ? s : u32x2{0u, 0u};
    }
    return tile_sum[tile] + u32x2{wave_total_u32(wave_scan_u32(a.x)), wave_total_u32(wave_scan_u32(a.y))};
}
// The same on the plain route, whose tile sums are the tiles' own (a workgroup).
__device__ __forceinline__ u32x2 plain_sums_ahead(const u32x2 *__restrict__ tile_sum, const u32x2 *__restrict__ group_sum, int64_t first,
                                            int group_tiles)
{
    __shared__ uint32_t part[2][kTileThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
    const int group = (int)(first / group_tiles);
    u32x2 a = {0u, 0u};
    static_assert(kMaxGroups <= kTileThreads, "a thread per group");
    if ((int)threadIdx.x < group) a = group_sum[threadIdx.x];
    for (int64_t t = (int64_t)group * group_tiles + threadIdx.x; t < first; t += kTileThreads) {
        const u32x2 s = tile_sum[t];
        a.x += s.x;
        a.y += s.y;
    }
    const uint32_t gx = wave_total_u32(wave_scan_u32(a.x)), gy = wave_total_u32(wave_scan_u32(a.y));
    __syncthreads();                                        // `part` may still be read from the previous tile
    if (lane == 0) {
        part[0][wave] = gx;
        part[1][wave] = gy;
    }
    __syncthreads();
    u32x2 sum = {0u, 0u};
#pragma unroll
    for (int w = 0; w < kTileThreads / kWave; ++w) {
        sum.x += part[0][w];
        sum.y += part[1][w];
    }
    return sum;
}
template <typename T>
__device__ __forceinline__ void write_pointers(const Out<T> &out, int64_t tile, int64_t ntiles, uint32_t out_base, const Std &sd, bool std)
{
    if ((threadIdx.x & (kWave - 1)) != 0) return;
    if (out.tile_ptr) {
        out.tile_ptr[tile] = (int32_t)out_base;
        if (tile == ntiles - 1) out.tile_ptr[ntiles] = (int32_t)out.k;
    }
    if (std && sd.row_ptr && tile == ntiles - 1) sd.row_ptr[sd.last_row + 1u] = (int32_t)out.k;
}

// Plain route: T, then the counts per tile and group (few enough workgroups that the search for T is amortised).
template <typename T, bool MAG, bool STD>
__device__ __forceinline__ void plain_count(const T *__restrict__ x, int64_t n, State *st, const uint32_t *__restrict__ hist4,
                                            u32x2 *tile_sum, u32x2 *group_sum, int64_t ntiles, int group_tiles, const Std &sd)
{
    const int64_t grid = min((int64_t)gridDim.x, (int64_t)kPlainGrid);
    if ((int64_t)blockIdx.x >= grid) return;
    const Choice c = select_bin<kTileThreads>(hist4, Elem<T>::KEYBITS == 32 ? 12 : 4, st->k_rem3);
    const uint32_t Tk = st->prefix3 | c.bin;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->T = Tk;
        st->take_eq = c.left;
    }
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += grid) {              // workgroup-uniform
        const u32x2 r = (tile + 1) * kTileElems <= n ? count_tensor_tile<T, MAG, STD, true>(x, n, tile, Tk, sd)
                                                     : count_tensor_tile<T, MAG, STD, false>(x, n, tile, Tk, sd);
        if (threadIdx.x == 0) {
            tile_sum[tile] = r;
            uint32_t *g = reinterpret_cast<uint32_t *>(group_sum + tile / group_tiles);
            atomicAdd(g, r.x);
            atomicAdd(g + 1, r.y);
        }
    }
}
// the survivors of one tile, from the tensor (a workgroup)
template <typename T, bool MAG, bool STD>
__device__ __forceinline__ void dense_tile(const T *__restrict__ x, int64_t n, const State *st,
                                           u32x2 ahead, int64_t tile, int64_t ntiles, const Out<T> &out, const Std &sd)
{
    const uint32_t Tk = st->T, take_eq = st->take_eq;
    const uint32_t out_base = ahead.x + min(ahead.y, take_eq), budget = take_eq > ahead.y ? take_eq - ahead.y : 0u;
    if (threadIdx.x < kWave) write_pointers<T>(out, tile, ntiles, out_base, sd, STD);
    if ((tile + 1) * kTileElems <= n)
        write_tensor_tile<T, MAG, STD, true>(x, n, tile, Tk, out_base, budget, out, sd);
    else
        write_tensor_tile<T, MAG, STD, false>(x, n, tile, Tk, out_base, budget, out, sd);
}

// The survivors from the records (list route; on the plain route the counts).
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kTileThreads)
write_kernel(const T *__restrict__ x, int64_t n, State *st, const u32x2 *__restrict__ tile_cnt, const uint32_t *__restrict__ rec_val,
             const uint16_t *__restrict__ rec_pos, const uint32_t *__restrict__ hist4, u32x2 *tile_sum, u32x2 *group_sum, int64_t ntiles,
             int group_tiles, Out<T> out, Std sd)
{
    if (st->use_plain != 0u) {
        plain_count<T, MAG, STD>(x, n, st, hist4, tile_sum, group_sum, ntiles, group_tiles, sd);
        return;
    }
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // a workgroup's tiles: four in a row or, where the workgroups all run at once, a quarter of the tensor apart, so that
    // tiles without records, which come in a row, don't meet in one workgroup (4096 x 768, an eighth of the rows ten times
    // the rest: the launch 6.2 us against 11.6; apart on large tensors costs 1 - 3 us: 50432 x 1024 bf16 81.0 -> 83.7)
    const bool apart = ntiles <= kApartTiles;
    const int64_t tile0 = apart ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4, step = apart ? (int64_t)gridDim.x : 1;
    const int64_t tile = tile0 + step * wave;
    const uint32_t Tk = st->T, take_eq = st->take_eq;
    // the records travel while the sums ahead are added up; no branch around any load
    const int64_t here = min(tile, ntiles - 1);
    const uint32_t n_cand = tile_cnt[here].x >> 16;
    const u32x4 *rv = reinterpret_cast<const u32x4 *>(rec_val + here * kRecSlots);
    const u32x2 *rp = reinterpret_cast<const u32x2 *>(rec_pos + here * kRecSlots);
    static_assert(kRecSlots % 4 == 0 && kFirstChunks * kRecChunk <= kRecSlots, "whole vectors");
    u32x4 v[kRecChunks];
    u32x2 p[kRecChunks];
#pragma unroll
    for (int u = 0; u < kFirstChunks; ++u) {                // (a list's unused slots hold anything)
        v[u] = rv[u * kWave + lane];
        p[u] = rp[u * kWave + lane];
    }
    const bool more = n_cand > (uint32_t)(kFirstChunks * kRecChunk) && n_cand != kTooMany;
#pragma unroll
    for (int u = kFirstChunks; u < kRecChunks; ++u) {
        v[u] = u32x4{0u, 0u, 0u, 0u};
        p[u] = u32x2{0u, 0u};
        if (more) {
            const int i = min(u * kWave + lane, kRecSlots / 4 - 1);
            v[u] = rv[i];
            p[u] = rp[i];
        }
    }
    const u32x2 ahead = sums_ahead(tile_sum, group_sum, here, group_tiles);
    const uint32_t out_base = ahead.x + min(ahead.y, take_eq), budget = take_eq > ahead.y ? take_eq - ahead.y : 0u;
    // A tile that holds more candidates than records (18 % of them where the rows' scale has a log-normal spread of 0.3) is
    // written from the tensor by the whole workgroup, whose waves read a quarter each.  By its own wave alone, a quarter
    // after another, the launch waited for it: such rows 50432 x 1024 bf16 100.8 us in all against 96.6, 49152 x 1024 fp32
    // 113.6 against 111.3.
    __shared__ alignas(16) u32x2 kept[4][kWriteSlots];
    __shared__ u32x2 left[4];                               // such tiles: first output slot, ties to keep
    if (lane == 0) left[wave] = tile < ntiles && n_cand == kTooMany ? u32x2{out_base, budget} : u32x2{~0u, 0u};
    if (tile < ntiles) {
        write_pointers<T>(out, tile, ntiles, out_base, sd, STD);
        if (n_cand != kTooMany) write_record_tile<T, MAG, STD>(v, p, n_cand, n, tile, Tk, out_base, budget, out, sd, kept[wave]);
    }
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        const u32x2 at = left[w];
        if (at.x == ~0u) continue;                          // workgroup-uniform
        const int64_t t = tile0 + step * w;
        if ((t + 1) * kTileElems <= n)
            write_tensor_tile<T, MAG, STD, true>(x, n, t, Tk, at.x, at.y, out, sd);
        else
            write_tensor_tile<T, MAG, STD, false>(x, n, t, Tk, at.x, at.y, out, sd);
    }
}

// The same when the sweep has made no records: a workgroup per tile, from the tensor.
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kTileThreads)
dense_write_kernel(const T *__restrict__ x, int64_t n, State *st, const uint32_t *__restrict__ hist4, u32x2 *tile_sum, u32x2 *group_sum,
                   int64_t ntiles, int group_tiles, Out<T> out, Std sd)
{
    if (st->use_plain != 0u) plain_count<T, MAG, STD>(x, n, st, hist4, tile_sum, group_sum, ntiles, group_tiles, sd);
    else dense_tile<T, MAG, STD>(x, n, st, sums_ahead(tile_sum, group_sum, blockIdx.x, group_tiles), blockIdx.x, ntiles, out, sd);
}

// Plain route: the survivors.
template <typename T, bool MAG, bool STD>
__global__ void __launch_bounds__(kTileThreads)
plain_write_kernel(const T *__restrict__ x, int64_t n, const State *st, const u32x2 *__restrict__ tile_sum,
                   const u32x2 *__restrict__ group_sum, int64_t ntiles, int group_tiles, Out<T> out, Std sd)
{
    if (st->use_plain == 0u) return;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x)           // workgroup-uniform
        dense_tile<T, MAG, STD>(x, n, st, plain_sums_ahead(tile_sum, group_sum, tile, group_tiles), tile, ntiles, out, sd);
}

// ---- restore without tile pointers: zeros, then scatter -----------------------------------
__global__ void __launch_bounds__(kTileThreads) zero_kernel(u32x4 *__restrict__ out, int64_t nvec16, uint8_t *tail, int tail_bytes)
{
    const int64_t v = (int64_t)blockIdx.x * (kTileThreads * kVecPerThread) + threadIdx.x;
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < kVecPerThread; ++j) {
        const int64_t i = v + (int64_t)j * kTileThreads;
        if (i < nvec16) out[i] = z;
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < tail_bytes) tail[threadIdx.x] = 0;
}

template <typename T>
__global__ void __launch_bounds__(kTileThreads)
scatter_kernel(const T *__restrict__ vals, const int32_t *__restrict__ idx, int64_t k, int64_t n, T *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * kTileThreads + threadIdx.x;
    if (i >= k) return;
    const int32_t at = idx[i];
    if (at >= 0 && (int64_t)at < n) out[at] = vals[i];
}

// ---- restore with tile pointers: each 4096-element tile of the output is built in LDS
// (zeros + its own records) and written once ------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(kTileThreads)
restore_tiles_kernel(const T *__restrict__ vals, const int32_t *__restrict__ idx, const int32_t *__restrict__ tile_ptr,
                     int64_t k, int64_t n, T *__restrict__ out)
{
    constexpr int PER16 = 16 / (int)sizeof(T);
    constexpr int kVecs = (int)kPtrTile / PER16;
    __shared__ alignas(16) T tile[kPtrTile];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * kPtrTile;
    const int m = (int)min(kPtrTile, n - t0);                  // >= 1 by the launch size

    int64_t p0 = tile_ptr[blockIdx.x], p1 = tile_ptr[blockIdx.x + 1];
    p0 = min(max(p0, (int64_t)0), k);                          // pointers that do not fit the record arrays are cut
    p1 = min(max(p1, p0), min(k, p0 + kPtrTile));
    const int n_rec = (int)(p1 - p0);

    // the first records of every thread are fetched before the tile is cleared,
    // so their latency overlaps the zero-fill and the barrier
    constexpr int PRE = 2;
    int pre_at[PRE];
    T pre_val[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
        const int j = tid + u * kTileThreads;
        pre_at[u] = -1;
        pre_val[u] = T(0);
        if (j < n_rec) {
            const int64_t at = (int64_t)idx[p0 + j] - t0;
            pre_at[u] = (at >= 0 && at < m) ? (int)at : -1;
            pre_val[u] = vals[p0 + j];
        }
    }
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (int v = tid; v < kVecs; v += kTileThreads) reinterpret_cast<u32x4 *>(tile)[v] = z;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PRE; ++u)
        if (pre_at[u] >= 0) tile[pre_at[u]] = pre_val[u];
    for (int j = tid + PRE * kTileThreads; j < n_rec; j += kTileThreads) {
        const int64_t at = (int64_t)idx[p0 + j] - t0;
        if (at >= 0 && at < m) tile[at] = vals[p0 + j];
    }
    __syncthreads();
    const int full = m / PER16;                                // whole 16-byte vectors inside the tensor
    u32x4 *dst = reinterpret_cast<u32x4 *>(out + t0);
    for (int v = tid; v < full; v += kTileThreads)
        __builtin_nontemporal_store(reinterpret_cast<const u32x4 *>(tile)[v], dst + v);
    for (int e = full * PER16 + tid; e < m; e += kTileThreads) out[t0 + e] = tile[e];
}

// Workspace: state | counters | group sums | three histograms | the sample's edges | tile counts | tile sums | key lists | records.
// From the counters to the histograms everything has to be zero at the start.
//
// That is 1.3 bytes an element.  Before the records there was a quarter of a byte, and a caller may hold a workspace of
// that size: it is still served, in one of two smaller layouts.
//   lists   no records (the survivors are written from the tensor), and as many list slots as there is room for;
//   plain   where not even 192 slots fit beside the histograms (below 4 - 6 M elements): no sample and no sweep, the
//           plain route's launches alone, with the state, two histograms and the sums.
struct Workspace {
    State *st;
    uint64_t *counters;
    u32x2 *group_sum;
    uint32_t *hist2, *hist3, *hist4;
    Edges *edges;
    u32x2 *tile_cnt, *tile_sum;
    uint32_t *lists, *rec_val;
    uint16_t *rec_pos;
    int list_slots;                        // 0: the plain layout
    bool records;
    u32x4 *zero;
    int zero16;
    size_t bytes;
};
struct Carver {
    char *base;
    size_t off;
    template <typename P> P *take(size_t bytes)
    {
        char *p = base + off;
        off += (bytes + 127) / 128 * 128;
        return reinterpret_cast<P *>(p);
    }
};
size_t tiles_of(int64_t n) { return (size_t)((n + kPtrTile - 1) / kPtrTile); }
int group_tiles_for(int64_t ntiles) { return (int)(((ntiles + kMaxGroups - 1) / kMaxGroups + 3) / 4 * 4); }
Workspace carve(void *base, int64_t n, int list_slots, bool records)
{
    Workspace w = {};
    Carver c = {static_cast<char *>(base), 0};
    const size_t tiles = tiles_of(n);
    w.list_slots = list_slots;
    w.records = records;
    w.st = c.take<State>(sizeof(State));
    w.counters = c.take<uint64_t>(kCounters * 64);
    w.group_sum = c.take<u32x2>(kMaxGroups * 8);
    w.hist2 = c.take<uint32_t>((size_t)kTopBins * 4);
    w.hist3 = c.take<uint32_t>((size_t)4 << kMaxDigit3);
    w.hist4 = c.take<uint32_t>((size_t)kTopBins * 4);
    w.zero = reinterpret_cast<u32x4 *>(w.counters);
    w.zero16 = (int)((c.off - sizeof(State)) / 16);
    w.edges = c.take<Edges>(kSampleWgs * sizeof(Edges));
    w.tile_cnt = c.take<u32x2>(tiles * 8);
    w.tile_sum = c.take<u32x2>(tiles * 8);
    w.lists = c.take<uint32_t>(tiles * (size_t)list_slots * 4);
    if (records) {
        w.rec_val = c.take<uint32_t>(tiles * kRecSlots * 4);
        w.rec_pos = c.take<uint16_t>(tiles * kRecSlots * 2);
    }
    w.bytes = c.off;
    return w;
}
Workspace carve_plain(void *base, int64_t n)
{
    Workspace w = {};
    Carver c = {static_cast<char *>(base), 0};
    const int64_t tiles = (int64_t)tiles_of(n);
    const int per = group_tiles_for(tiles);
    w.st = c.take<State>(sizeof(State));
    w.group_sum = c.take<u32x2>((size_t)((tiles + per - 1) / (per > 0 ? per : 1)) * 8);
    w.hist2 = c.take<uint32_t>((size_t)kTopBins * 4);
    w.hist3 = c.take<uint32_t>(256 * 4);
    w.zero = reinterpret_cast<u32x4 *>(w.st);
    w.zero16 = (int)(c.off / 16);
    w.tile_sum = c.take<u32x2>((size_t)tiles * 8);
    w.bytes = c.off;
    return w;
}
char origin[1];                            // where only offsets are wanted
size_t workspace_bytes_for(int64_t n) { return carve(origin, n, kListSlots, true).bytes; }
// The least that is accepted: state, one histogram, two words and 256 list slots a tile.  (The plain layout is smaller.)
size_t least_workspace_for(int64_t n)
{
    Carver c = {origin, 0};
    const size_t tiles = tiles_of(n);
    c.take<char>(sizeof(State) + (size_t)kTopBins * 4);
    c.take<char>(tiles * 8);
    c.take<char>(tiles * 8);
    c.take<char>((tiles + 1) * 1024);
    return c.off;
}
Workspace carve_room(void *base, int64_t n, size_t room)            // room >= least_workspace_for(n)
{
    if (room >= workspace_bytes_for(n)) return carve(base, n, kListSlots, true);
    const size_t bare = carve(origin, n, 0, false).bytes, tiles = tiles_of(n);
    if (room >= bare) {
        const size_t fit = (room - bare) / (tiles * 4);             // (whole lines: a multiple of 32)
        const int slots = (int)(fit < (size_t)kListSlots ? fit / 32 * 32 : (size_t)kListSlots);
        if (slots >= kMinListSlots) return carve(base, n, slots, false);
    }
    return carve_plain(base, n);
}

// Which ranks of a workgroup's sample bound its bracket: those next to T's own, f = k / n of the sample.  The 16 samples are
// as good as independent of one another, and T is as likely above a workgroup's bracket as below it: it is missed on one
// side of all 16 once in 2^15 tensors, as long as neighbouring stretches are as good as exchangeable (and hardly ever where the workgroups see every vector:
// 16 counts cannot all lie on one side of their mean).  The joint bracket spans 3.5 standard deviations sqrt(size f (1 - f)) of
// a workgroup's rank, 1.7 % of the tensor at f = 0.1, and the rest of its outer bins.  (One bracket of six deviations either
// way from the sum of the 16 histograms, 1.4 %, took a launch of one workgroup more: 4096 x 768 37.3 us in all and 33.7
// now, 8192 x 1024 bf16 41.8 and 38.3, 49152 x 1024 87.7 and 88.2.)
struct SamplePlan {
    bool use;                              // false: T's rank is too close to an end, the tensor's own histogram is taken
    int wgs;
    uint32_t total, hi, lo, size;
    uint64_t step;
};
SamplePlan plan_sample(int64_t n, int64_t k, int epv)
{
    SamplePlan p = {false, 0, 0u, 0u, 0u, 0u, 0u};
    const int64_t vectors = n / epv, most = (int64_t)kSampleWgs * kWideThreads;
    if (vectors == 0) return p;
    const int64_t total = vectors < most ? vectors : most, rest = n - vectors * epv;
    p.total = (uint32_t)total;
    p.size = (uint32_t)(total * epv);
    p.step = ((uint64_t)vectors << 16) / (uint64_t)total;
    int64_t hi, lo, size;
    if (vectors <= kWideThreads) {         // one workgroup sees every vector: only the last few entries were not seen
        p.wgs = 1;
        size = total * epv;
        hi = k - rest;
        lo = k;
    } else {
        const double f = (double)k / (double)n;
        if (vectors > most && (f * p.size < 256 || (1.0 - f) * p.size < 256)) return p;
        p.wgs = kSampleWgs;
        size = total / kSampleWgs * epv;   // (some have a vector more)
        const double r = f * (double)size;
        hi = (int64_t)r;
        lo = (int64_t)r + 1;
    }
    p.use = true;
    p.hi = (uint32_t)(hi < 1 ? 1 : hi);
    p.lo = (uint32_t)(lo > size ? size : lo);
    if (p.hi > p.lo) p.hi = p.lo;
    return p;
}

template <typename T, bool MAG, bool STD>
void launch_select(const T *x, int64_t n, uint32_t k, typename Elem<T>::Out *vals, int32_t *idx, int32_t *tile_ptr,
                   const Workspace &w, const Std &sd, hipStream_t s)
{
    const int64_t ntiles = (n + kTileElems - 1) / kTileElems;
    // at most kMaxGroups groups of tiles; also the workgroups of the digit and count launches
    const int group_tiles = group_tiles_for(ntiles);
    const unsigned groups = (unsigned)((ntiles + group_tiles - 1) / group_tiles);
    const Out<T> out = {vals, idx, tile_ptr, k};
    const unsigned plain_grid = (unsigned)(ntiles < kPlainGrid ? ntiles : kPlainGrid);
    if (w.list_slots == 0) {
        // The plain layout.  The digit launches look at a list's head before they know the route: they are told of one
        // tile and given the histogram to look at.  The first digit's histogram serves again as the last one's.
        const u32x2 *no_cnt = reinterpret_cast<const u32x2 *>(w.hist2);
        launch(clear_kernel, 1, kWideThreads, 0, s, w.zero, w.zero16, w.st);
        launch(digit_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.st, reinterpret_cast<const uint64_t *>(w.hist2), no_cnt, w.hist2,
                                                                  0, w.hist2, 1, k, sd);
        uint32_t *last = w.hist3;
        if constexpr (Elem<T>::KEYBITS == 32) {
            launch(second_digit_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.st, no_cnt, w.hist2, 0, w.hist2, w.hist3, 1, sd);
            last = w.hist2;
            launch(clear_kernel, 1, kWideThreads, 0, s, reinterpret_cast<u32x4 *>(last), kTopBins / 4, nullptr);
        }
        launch(count_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.st, no_cnt, w.hist2, 0, w.hist2, w.hist3, last, w.tile_sum,
                                                                  w.group_sum, 1, group_tiles, sd);
        launch(dense_write_kernel<T, MAG, STD>, plain_grid, kTileThreads, 0, s, x, n, w.st, last, w.tile_sum, w.group_sum, ntiles, group_tiles,
                                                                            out, sd);
        launch(plain_write_kernel<T, MAG, STD>, plain_grid, kTileThreads, 0, s, x, n, w.st, w.tile_sum, w.group_sum, ntiles, group_tiles, out,
                                                                            sd);
        return;
    }
    const bool records = w.records && (int64_t)k * kRecShare <= n;
    const SamplePlan plan = plan_sample(n, (int64_t)k, Elem<T>::EPV);

    if (plan.use) {
        launch(sample_kernel<T, MAG, STD>, plan.wgs, kWideThreads, 0, s, x, plan.total, plan.step, plan.hi, plan.lo, w.edges, w.st, w.zero,
                                                                     w.zero16, sd);
    } else {
        launch(clear_kernel, 1, kWideThreads, 0, s, w.zero, w.zero16, nullptr);
        launch(top_digit_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.hist4, sd);
        launch(edges_kernel, 1, kWideThreads, 0, s, w.hist4, k, w.edges, w.st);
    }
    const uint64_t size = plan.use && plan.wgs == kSampleWgs ? plan.size : (plan.use ? (uint64_t)plan.size : (uint64_t)n) * kSampleWgs;
    if (records)
        launch(sweep_kernel<T, MAG, STD, true>, (unsigned)ntiles, kTileThreads, 0, s, x, n, w.edges, size, w.st, w.counters, w.tile_cnt, w.lists, w.list_slots,
                                                                                 w.rec_val, w.rec_pos, sd);
    else
        launch(sweep_kernel<T, MAG, STD, false>, (unsigned)ntiles, kTileThreads, 0, s, x, n, w.edges, size, w.st, w.counters, w.tile_cnt, w.lists, w.list_slots,
                                                                                  nullptr, nullptr, sd);
    launch(digit_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.st, w.counters, w.tile_cnt, w.lists, w.list_slots, w.hist2,
                                                              ntiles, k, sd);
    if constexpr (Elem<T>::KEYBITS == 32)
        launch(second_digit_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.st, w.tile_cnt, w.lists, w.list_slots, w.hist2, w.hist3,
                                                                         ntiles, sd);
    launch(count_kernel<T, MAG, STD>, groups, kWideThreads, 0, s, x, n, w.st, w.tile_cnt, w.lists, w.list_slots, w.hist2, w.hist3, w.hist4, w.tile_sum,
                                                              w.group_sum, ntiles, group_tiles, sd);
    if (records)
        launch(write_kernel<T, MAG, STD>, (unsigned)((ntiles + 3) / 4), kTileThreads, 0, s, x, n, w.st, w.tile_cnt, w.rec_val, w.rec_pos, w.hist4,
                                                                                       w.tile_sum, w.group_sum, ntiles, group_tiles, out, sd);
    else
        launch(dense_write_kernel<T, MAG, STD>, (unsigned)ntiles, kTileThreads, 0, s, x, n, w.st, w.hist4, w.tile_sum, w.group_sum, ntiles,
                                                                                 group_tiles, out, sd);
    launch(plain_write_kernel<T, MAG, STD>, plain_grid, kTileThreads, 0, s, x, n, w.st, w.tile_sum, w.group_sum, ntiles, group_tiles, out, sd);
}

}  // namespace
}  // namespace slimfit

using namespace slimfit;

extern "C" int32_t slimfit_prune_global_workspace(int64_t n, size_t *bytes)
{
    if (!bytes || n < 0 || n > 0x7FFFFFFFLL) return SLIMFIT_ERR_INVALID_ARG;
    *bytes = workspace_bytes_for(n);
    return SLIMFIT_OK;
}

extern "C" int64_t slimfit_global_tile_ptr_len(int64_t n)
{
    if (n < 0 || n > 0x7FFFFFFFLL) return -1;
    return (n + kPtrTile - 1) / kPtrTile + 1;
}

namespace {

// Shared body of the two pruning entry points.  H == 0: plain; otherwise the
// tensor is rows of H elements standardised with mean / rstd on the way in.
int32_t prune_global_entry(const void *x, int32_t dt, int64_t n, int64_t H, const float *mean, const float *rstd,
                           int64_t k, int32_t by_magnitude, void *vals, int32_t *idx, int32_t *tile_ptr,
                           int32_t *row_ptr, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!dtype_ok(dt) || n < 0 || k < 0 || k > n) return SLIMFIT_ERR_INVALID_ARG;
    if (n > 0x7FFFFFFFLL) return SLIMFIT_ERR_UNSUPPORTED;                 // indices are int32
    const bool standardised = H != 0;
    const int64_t epv = dt == SLIMFIT_F32 ? 4 : 8;            // a row has to be whole 16-byte vectors
    if (standardised && (H < epv || H % epv != 0 || n % H != 0)) return SLIMFIT_ERR_INVALID_ARG;
    if (k == 0) return SLIMFIT_OK;
    if (!x || !vals || !idx || !workspace || (standardised && (!mean || !rstd))) return SLIMFIT_ERR_INVALID_ARG;
    const size_t esz = dtype_size(dt);
    const size_t vsz = standardised ? 4 : esz;                // standardised values are fp32 whatever the input
    if (!aligned_to(x, 16) || !aligned_to(vals, vsz) || !aligned_to(idx, 4) || !aligned_to(workspace, 16) ||
        (tile_ptr && !aligned_to(tile_ptr, 4)) || (row_ptr && !aligned_to(row_ptr, 4)) ||
        (standardised && (!aligned_to(mean, 4) || !aligned_to(rstd, 4))))
        return SLIMFIT_ERR_ALIGNMENT;
    if (workspace_bytes < least_workspace_for(n)) return SLIMFIT_ERR_WORKSPACE;
    const Workspace w = carve_room(workspace, n, workspace_bytes);
    int32_t rc;
    if ((rc = check_device_range(x, (size_t)n * esz)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(vals, (size_t)k * vsz)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(idx, (size_t)k * 4)) != SLIMFIT_OK) return rc;
    if ((rc = check_device_range(workspace, w.bytes)) != SLIMFIT_OK) return rc;
    if (tile_ptr && (rc = check_device_range(tile_ptr, (size_t)slimfit_global_tile_ptr_len(n) * 4)) != SLIMFIT_OK)
        return rc;
    Std sd = {nullptr, nullptr, 0u, 0u, 0u, 0u, 0u, nullptr};
    if (standardised) {
        const size_t rows = (size_t)(n / H);
        if ((rc = check_device_range(mean, rows * 4)) != SLIMFIT_OK) return rc;
        if ((rc = check_device_range(rstd, rows * 4)) != SLIMFIT_OK) return rc;
        if (row_ptr && (rc = check_device_range(row_ptr, (rows + 1) * 4)) != SLIMFIT_OK) return rc;
        int l = 0;
        while (((int64_t)1 << l) < H) ++l;                              // ceil(log2 H) >= 2
        const uint64_t pow = (uint64_t)1 << (31 + l);
        sd.mean = mean;
        sd.rstd = rstd;
        sd.magic = (uint32_t)((pow + (uint64_t)H - 1) / (uint64_t)H);   // < 2^32 because H > 2^(l-1)
        sd.shift = (uint32_t)(l - 1);
        sd.vec_uniform = (H % (kWave * epv) == 0) ? 1u : 0u;
        sd.last_row = (uint32_t)(rows - 1);
        sd.H = (uint32_t)H;
        sd.row_ptr = row_ptr;
    }

    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t kk = (uint32_t)k;
    if (dt == SLIMFIT_F32) {
        const float *xf = static_cast<const float *>(x);
        float *vf = static_cast<float *>(vals);
        if (standardised) {
            if (by_magnitude) launch_select<float, true, true>(xf, n, kk, vf, idx, tile_ptr, w, sd, s);
            else launch_select<float, false, true>(xf, n, kk, vf, idx, tile_ptr, w, sd, s);
        } else {
            if (by_magnitude) launch_select<float, true, false>(xf, n, kk, vf, idx, tile_ptr, w, sd, s);
            else launch_select<float, false, false>(xf, n, kk, vf, idx, tile_ptr, w, sd, s);
        }
    } else if (standardised) {
        const Bf16Row *xr = static_cast<const Bf16Row *>(x);
        float *vf = static_cast<float *>(vals);
        if (by_magnitude) launch_select<Bf16Row, true, true>(xr, n, kk, vf, idx, tile_ptr, w, sd, s);
        else launch_select<Bf16Row, false, true>(xr, n, kk, vf, idx, tile_ptr, w, sd, s);
    } else {
        const uint16_t *xh = static_cast<const uint16_t *>(x);
        uint16_t *vh = static_cast<uint16_t *>(vals);
        if (by_magnitude) launch_select<uint16_t, true, false>(xh, n, kk, vh, idx, tile_ptr, w, sd, s);
        else launch_select<uint16_t, false, false>(xh, n, kk, vh, idx, tile_ptr, w, sd, s);
    }
    return launch_status();
}

}  // namespace

extern "C" int32_t slimfit_prune_global(const void *x, int32_t dt, int64_t n, int64_t k, int32_t by_magnitude,
                                        void *vals, int32_t *idx, int32_t *tile_ptr, void *workspace,
                                        size_t workspace_bytes, void *stream)
{
    StreamScope capture_aware(stream);
    return prune_global_entry(x, dt, n, 0, nullptr, nullptr, k, by_magnitude, vals, idx, tile_ptr, nullptr, workspace,
                              workspace_bytes, stream);
}

extern "C" int32_t slimfit_prune_global_standardized(const void *x, int32_t dt, int64_t n, int64_t H,
                                                     const float *mean, const float *rstd, int64_t k,
                                                     int32_t by_magnitude, void *vals, int32_t *idx,
                                                     int32_t *tile_ptr, int32_t *row_ptr, void *workspace,
                                                     size_t workspace_bytes, void *stream)
{
    StreamScope capture_aware(stream);
    if (H == 0) return SLIMFIT_ERR_INVALID_ARG;
    return prune_global_entry(x, dt, n, H, mean, rstd, k, by_magnitude, vals, idx, tile_ptr, row_ptr, workspace,
                              workspace_bytes, stream);
}

extern "C" int32_t slimfit_restore_global(const void *vals, const int32_t *idx, const int32_t *tile_ptr, int64_t k,
                                          int32_t dt, int64_t n, void *out, void *stream)
{
    StreamScope capture_aware(stream);
    if (!dtype_ok(dt) || n < 0 || k < 0 || k > n) return SLIMFIT_ERR_INVALID_ARG;
    if (n > 0x7FFFFFFFLL) return SLIMFIT_ERR_UNSUPPORTED;
    if (n == 0) return SLIMFIT_OK;
    if (!out || (k > 0 && (!vals || !idx))) return SLIMFIT_ERR_INVALID_ARG;
    const size_t esz = dtype_size(dt);
    if (!aligned_to(out, 16) || (k > 0 && (!aligned_to(vals, esz) || !aligned_to(idx, 4))) ||
        (tile_ptr && !aligned_to(tile_ptr, 4)))
        return SLIMFIT_ERR_ALIGNMENT;
    int32_t rc;
    if ((rc = check_device_range(out, (size_t)n * esz)) != SLIMFIT_OK) return rc;
    if (k > 0) {
        if ((rc = check_device_range(vals, (size_t)k * esz)) != SLIMFIT_OK) return rc;
        if ((rc = check_device_range(idx, (size_t)k * 4)) != SLIMFIT_OK) return rc;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (tile_ptr && k > 0) {
        const int64_t tiles = (n + kPtrTile - 1) / kPtrTile;
        if ((rc = check_device_range(tile_ptr, (size_t)(tiles + 1) * 4)) != SLIMFIT_OK) return rc;
        if (dt == SLIMFIT_F32)
            launch(restore_tiles_kernel<float>, (unsigned)tiles, kTileThreads, 0, s, 
                static_cast<const float *>(vals), idx, tile_ptr, k, n, static_cast<float *>(out));
        else
            launch(restore_tiles_kernel<uint16_t>, (unsigned)tiles, kTileThreads, 0, s, 
                static_cast<const uint16_t *>(vals), idx, tile_ptr, k, n, static_cast<uint16_t *>(out));
        return launch_status();
    }
    const size_t bytes = (size_t)n * esz;
    const int64_t nvec16 = (int64_t)(bytes / 16);
    const int tail_bytes = (int)(bytes % 16);
    const int64_t per_block = (int64_t)kTileThreads * kVecPerThread;
    int64_t zblocks = (nvec16 + per_block - 1) / per_block;
    if (zblocks < 1) zblocks = 1;
    launch(zero_kernel, (unsigned)zblocks, kTileThreads, 0, s, static_cast<u32x4 *>(out), nvec16,
                                                          static_cast<uint8_t *>(out) + (size_t)nvec16 * 16, tail_bytes);
    if (k > 0) {
        const unsigned sblocks = (unsigned)((k + kTileThreads - 1) / kTileThreads);
        if (dt == SLIMFIT_F32)
            launch(scatter_kernel<float>, sblocks, kTileThreads, 0, s, static_cast<const float *>(vals), idx, k, n,
                                                                   static_cast<float *>(out));
        else
            launch(scatter_kernel<uint16_t>, sblocks, kTileThreads, 0, s, static_cast<const uint16_t *>(vals), idx, k, n,
                                                                      static_cast<uint16_t *>(out));
    }
    return launch_status();
}
