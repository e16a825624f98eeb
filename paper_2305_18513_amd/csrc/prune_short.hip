// Pruning of short score rows that keep few entries (Alg. 5 applied per row; the
// appendix on pruning), for gfx950: rows of at most 256 columns, k <= 16 (bf16)
// or k <= 12 (fp32).
//
// With 197-column rows a wave that owns one row at a time spends most of its
// instructions on per-row bookkeeping (wave reductions, a bin scan, scalar
// popcounts) that does not shrink with the row.  Here nothing is done per row by
// a whole wave.  G lanes (2 or 4; 4 or 8 of wide softmax rows) share a row, so a wave works on R = 64 / G
// consecutive rows at once, and every lane owns one contiguous segment of its
// row (E = ceil(cols / G) entries):
//
//   stage    the wave's R consecutive rows are one contiguous, 16-byte aligned
//            piece of the tensor: copied to LDS with 16-byte non-temporal loads
//            (the only pass over HBM);
//   select   each lane keeps the largest CH keys of its segment in a sorted
//            register list: inserting a key is one v_max plus CH-1 v_med3
//            (new s[i] = median(s[i-1], s[i], key)), no branch, no cross-lane step.
//            Where a lane has many (bf16), only the larger of two neighbours is
//            inserted, and the partners of those that stayed afterwards.
//            A key carries the entry's column below its value (bf16: the 16 value
//            bits and the column; fp32: the upper 24 bits of the value's image and
//            the column), so ties go to the lower column and the list itself names
//            the columns.
//   merge    the G sorted lists of a row are merged by DPP exchanges between its
//            lanes (the partner's j-th largest can only land at position >= j).
//   fp32     24 value bits decide the kept set exactly unless the k-th and the
//            (k+1)-th largest agree in all of them (or, with a threshold, an entry
//            agrees with the threshold in all of them): about 0.1 % of 197-column
//            softmax rows, 1.5 % of their waves.  A wave that has such a row repeats the selection on the full
//            32-bit images (no columns), then walks its segment once more to
//            place the kept columns: the exact route, same result.
//   output   the kept columns are sorted in registers, staged in LDS in output
//            order and leave as contiguous runs; fp32 values (and bf16 ones when
//            a sign bit was seen, so that -0 stays -0) are re-read from the staged
//            rows.
//
// Keys: the bit patterns themselves, read as signed integers, order positive
// entries correctly and put zeros and negative entries below them, which is all
// a row needs whose kept entries are positive (every softmax row).  A wave that
// meets a row whose k-th largest entry is not positive starts over with
// sign * magnitude keys (-0 and +0 coincide, as float comparison has it).
#include "common.hpp"
#include "short_rows.hpp"

#include <climits>
#include <utility>

namespace slimfit {
namespace {

#ifndef SLIMFIT_SHORT_NT
#define SLIMFIT_SHORT_NT 1             // the rows are streamed once
#endif
#ifndef SLIMFIT_SHORT_NT_STORE
#define SLIMFIT_SHORT_NT_STORE 0       // the pairs leave through the cache: plain stores are acknowledged sooner
#endif
#ifndef SLIMFIT_SHORT_FORCE_EXACT
#define SLIMFIT_SHORT_FORCE_EXACT 0    // tests of the exact route: take it for every wave
#endif

__device__ __forceinline__ int med3_i32(int a, int b, int c)
{
    // written as an instruction: max(min(a, b), min(max(a, b), c)) compiles to the same v_med3_i32, but chains
    // of it take the optimiser minutes to analyse
    int d;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// (a & mask) | b in one instruction; mask sits in a register because the three-operand encoding takes no literal
__device__ __forceinline__ int and_or_i32(int a, int mask, int b)
{
    int d;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(mask), "s"(b));
    return d;
}

// s is sorted in descending order; afterwards it holds the CH largest of s + {key}
template <int CH>
__device__ __forceinline__ void chain_insert(int (&s)[CH], int key)
{
#pragma unroll
    for (int i = CH - 1; i >= 1; --i) s[i] = med3_i32(s[i - 1], s[i], key);
    s[0] = max(s[0], key);
}

// the same for a key that is not above s[J]
template <int CH, int J>
__device__ __forceinline__ void chain_insert_below(int (&s)[CH], int key)
{
#pragma unroll
    for (int i = CH - 1; i >= J + 2; --i) s[i] = med3_i32(s[i - 1], s[i], key);
    s[J + 1] = max(s[J + 1], key);
}

// the same for b[0] >= b[1] >= ...: b[j] cannot land above position j
template <int CH>
__device__ __forceinline__ void chain_merge(int (&m)[CH], const int (&b)[CH])
{
#pragma unroll
    for (int j = 0; j < CH; ++j) {
#pragma unroll
        for (int i = CH - 1; i >= (j > 1 ? j : 1); --i) m[i] = med3_i32(m[i - 1], m[i], b[j]);
        if (j == 0) m[0] = max(m[0], b[0]);
    }
}

// every lane of a row ends with the merged list of the row's G lanes
template <int G, int CH>
__device__ __forceinline__ void merge_row(int (&m)[CH])
{
    int b[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) b[i] = (int)dpp_u32<kDppXor1>((uint32_t)m[i]);
    chain_merge<CH>(m, b);
    if constexpr (G >= 4) {
#pragma unroll
        for (int i = 0; i < CH; ++i) b[i] = (int)dpp_u32<kDppXor2>((uint32_t)m[i]);
        chain_merge<CH>(m, b);
    }
    if constexpr (G >= 8) {                                // (the lanes of a quad hold the same list by now)
#pragma unroll
        for (int i = 0; i < CH; ++i) b[i] = (int)dpp_u32<kDppHalfMirror>((uint32_t)m[i]);
        chain_merge<CH>(m, b);
    }
}

// ascending, in place (odd-even transposition)
template <int N>
__device__ __forceinline__ void sort_ascending(uint32_t (&c)[N])
{
#pragma unroll
    for (int round = 0; round < N; ++round) {
#pragma unroll
        for (int i = round & 1; i + 1 < N; i += 2) {
            const uint32_t lo = min(c[i], c[i + 1]), hi = max(c[i], c[i + 1]);
            c[i] = lo;
            c[i + 1] = hi;
        }
    }
}

// sign * magnitude of a float's bits (-0 -> 0)
__device__ __forceinline__ int signed_key_f32(uint32_t u)
{
    const int s = (int)u >> 31;
    return (int)(((u & 0x7FFFFFFFu) ^ (uint32_t)s) - (uint32_t)s);
}
// the same for 16 bits held sign-extended
__device__ __forceinline__ int signed_key_16(int v)
{
    const int s = v >> 31;
    return ((v & 0x7FFF) ^ s) - s;
}

struct ShortArgs {
    int64_t rows;
    int cols, k, mode;
    float tau;
    uint32_t div_magic;            // t / k == (t * div_magic) >> 16 for t < 64 * k
};

constexpr uint32_t kNoPair = 0xFFFF0000u;              // staging slot of an unused output position: column 0xFFFF

template <int... J, typename F>
__device__ __forceinline__ void static_for(std::integer_sequence<int, J...>, F f)
{
    (f(std::integral_constant<int, J>{}), ...);
}

// T: float or bf16 bits; G: lanes a row; K: largest k served; NV: 16-byte vectors a lane holds
template <typename T, int G, int K, int NV>
struct ShortRows {
    static constexpr bool BF = sizeof(T) == 2;
    static constexpr int R = kWave / G;
    static constexpr int CHP = BF ? K : K + 1;                 // list length: fp32 also wants the (k+1)-th largest
    static constexpr int LANE_BITS = G == 2 ? 1 : (G == 4 ? 2 : 3);
    static constexpr int TAG_BITS = 8 - LANE_BITS;             // entry's rank inside the lane's segment (at most 256 columns)
    static constexpr int N_OUT = (R * K + kWave - 1) / kWave;  // output pairs a lane stores
    // Whether the larger of two neighbours stands for both in the selection's walk: where a lane has 65 entries or more (bf16
    // rows of more than 128 columns; NV is 4, 8, 13 or 16).  806 912 x 197, k = 9: 86.5 -> 78.0 us, 49 152 x 160, k = 16 12.5 -> 11.8,
    // x 250, k = 12 14.1 -> 12.7; few rows of 130 columns lose (8192, k = 13 7.6 -> 8.0).  With fewer entries the partners cost
    // as much or more: 98 304 x 100 9.3 / 9.3, x 70 7.9 -> 8.1, and so do fp32 rows of 33 to 64 entries a lane: 98 304 x 160
    // 19.7 -> 20.5, nine tenths masked 18.9 -> 20.4, 49 152 x 224 17.7 -> 18.4, 302 592 x 197 55.6 -> 54.2.
    static constexpr bool kPaired = BF && NV >= 13;

    // Visits the lane's entries e = 0 .. E-1 in column order: f(e, bits, ok) with the entry's bits (fp32: its
    // 32; bf16: its 16, zero-extended, or sign-extended when SEXT) and ok = "this lane has an entry e".  seg:
    // the lane's segment among the staged rows (LDS).  Blocks of kBlk entries; two register buffers take
    // turns, so a block's LDS reads are in flight while the one before it is worked on (f may hold asm
    // statements, which a run-time trip count cannot be unrolled around: blocks by hand).
    static constexpr int kBlk = 8;
    template <bool SEXT, typename F>
    static __device__ __forceinline__ void for_each_entry(const T *seg, int E, int len, int e_all, F f)
    {
        auto bits_at = [&](int e) -> int {
            if constexpr (BF) return SEXT ? (int)(int16_t)seg[e] : (int)seg[e];
            else return (int)__builtin_bit_cast(uint32_t, seg[e]);
        };
        const int n_blk = e_all / kBlk;                    // blocks every lane has in full
        int A[kBlk], B[kBlk];
        if (n_blk > 0) {
#pragma unroll
            for (int u = 0; u < kBlk; ++u) A[u] = bits_at(u);
        }
        for (int bi = 0; bi < n_blk; bi += 2) {
            if (bi + 1 < n_blk) {
#pragma unroll
                for (int u = 0; u < kBlk; ++u) B[u] = bits_at((bi + 1) * kBlk + u);
            }
#pragma unroll
            for (int u = 0; u < kBlk; ++u) f(bi * kBlk + u, A[u], true);
            if (bi + 1 < n_blk) {
                if (bi + 2 < n_blk) {
#pragma unroll
                    for (int u = 0; u < kBlk; ++u) A[u] = bits_at((bi + 2) * kBlk + u);
                }
#pragma unroll
                for (int u = 0; u < kBlk; ++u) f((bi + 1) * kBlk + u, B[u], true);
            }
        }
        // the ragged end: entries some lanes do not have.  Such a lane reads a few entries past its segment
        // (the next row's, or at most G - 1 entries past the staged rows, which the launch's LDS has room for).
        for (int e0 = n_blk * kBlk; e0 < E; e0 += kBlk) {
#pragma unroll
            for (int u = 0; u < kBlk; ++u) {
                if (e0 + u < E) A[u] = bits_at(e0 + u);    // wave-uniform
            }
#pragma unroll
            for (int u = 0; u < kBlk; ++u) {
                if (e0 + u < E) f(e0 + u, A[u], e0 + u < len);
            }
        }
    }

    // NEG: keys are sign * magnitude.  Without it the bit patterns themselves serve as (signed) keys, which orders
    // the positive entries correctly and puts everything else (zeros of either sign, negative values in reversed
    // order) below them: enough whenever every kept entry is positive.  The plain pass notices when that fails for
    // one of the wave's rows and returns false before it has written anything; the caller then runs the signed pass.
    // Held: entries that are in registers already: each_held<NEG>(f) visits the lane's as f(e, bits, ok), and a row of one
    // value (constant_rows) keeps its first columns: it neither starts the selection over nor takes the exact route.  The kept columns are left in oc, kept is the row's count.
    struct NotHeld {
        static constexpr bool HELD = false;
    };
    template <bool NEG, typename Held>
    static __device__ __forceinline__ bool select(const ShortArgs &a, const T *rows_lds, uint32_t *oc, int lane, int &kept,
                                                  const Held &held)
    {
        const int cols = a.cols, k = a.k;
        const int r = lane / G, q = lane % G;
        const int E = (cols + G - 1) / G;                  // entries a lane
        const int len = min(max(cols - q * E, 0), E);      // this lane's
        const int e_all = max(cols - (G - 1) * E, 0);      // the last lane's: the shortest segment
        const T *seg = rows_lds + r * cols + q * E;
        constexpr int TAG_TOP = (1 << TAG_BITS) - 1;
        constexpr uint32_t COL_MASK = (1u << (TAG_BITS + LANE_BITS)) - 1u;      // rank in the segment, lane of the row

        // ---- selection on keys that carry the column ---------------------------------
        int m[CHP];
#pragma unroll
        for (int i = 0; i < CHP; ++i) m[i] = INT_MIN;
        int value_mask = (int)~COL_MASK;
        asm("" : "+v"(value_mask));                        // in a register, not a literal at every use
        // f(e, bits, ok) for the lane's entries, from registers if they are there
        auto walk = [&](auto f) {
            if constexpr (Held::HELD) held.template each_held<NEG>(f);
            else for_each_entry<NEG>(seg, E, len, e_all, f);
        };
        // the earlier entry of the segment ranks higher
        auto key_of = [&](int e, int bits) -> int {
            if constexpr (BF) return (int)(((uint32_t)(NEG ? signed_key_16(bits) : bits) << 16) | (uint32_t)(TAG_TOP - e));
            else return ((NEG ? signed_key_f32((uint32_t)bits) : bits) & value_mask) | (TAG_TOP - e);
        };
        // PAIRED: of entries 2i and 2i + 1 only the larger goes into the list.  A lane's largest entries are then those in
        // the list or their partners: one that is not the larger of its pair has that one above it, so the pair is in the
        // list or CHP larger entries are.  Half as many insertions, then CHP - 1 short ones.
        constexpr bool PAIRED = kPaired && !Held::HELD;
        int waiting = INT_MIN;
        walk([&](int e, int bits, bool ok) {
            int key;
            if constexpr (!BF && !Held::HELD) key = and_or_i32(NEG ? signed_key_f32((uint32_t)bits) : bits, value_mask, TAG_TOP - e);
            else key = key_of(e, bits);                     // (fp32: e is a constant here, wave-uniform above)
            key = ok ? key : INT_MIN;
            if (!PAIRED) chain_insert<CHP>(m, key);
            else if (e & 1) chain_insert<CHP>(m, max(waiting, key));
            else waiting = key;
        });
        if constexpr (PAIRED) {
            if (E & 1) chain_insert<CHP>(m, waiting);
            int partner[CHP - 1];
#pragma unroll
            for (int j = 0; j < CHP - 1; ++j) {
                const int other = (TAG_TOP - (m[j] & TAG_TOP)) ^ 1;
                const bool has = m[j] != INT_MIN && other < len;
                const int bits = NEG ? (int)(int16_t)seg[has ? other : 0] : (int)seg[has ? other : 0];
                partner[j] = has ? key_of(other, bits) : INT_MIN;
            }
            static_for(std::make_integer_sequence<int, CHP - 1>{}, [&](auto j) { chain_insert_below<CHP, j>(m, partner[j]); });
        }
#pragma unroll
        for (int i = 0; i < CHP; ++i) m[i] |= (G - 1 - q) << TAG_BITS;     // lanes of lower columns rank higher
        merge_row<G, CHP>(m);

        auto column_of = [&](int key) {
            const int low = key & (int)COL_MASK;
            return (G - 1 - (low >> TAG_BITS)) * E + (TAG_TOP - (low & TAG_TOP));
        };
        int kk = k;
        bool exact = false;                                 // this row has to take the exact route (fp32 only)
        uint32_t c[K];                                      // kept (column << 16 | bf16 value bits), kNoPair beyond kk
        bool plain_ok = true;
        if constexpr (!NEG) {
            // all kept entries positive?  With k entries kept: the k-th largest is; with fewer (a threshold run): tau is.
            int cut_value = 0;
#pragma unroll
            for (int i = 0; i < K; ++i) cut_value = (i == k - 1) ? m[i] >> (BF ? 16 : TAG_BITS + LANE_BITS) : cut_value;
            plain_ok = cut_value > 0 || (a.mode == SLIMFIT_PRUNE_THRESHOLD && a.tau > 0.0f);
            if (!Held::HELD && __builtin_amdgcn_ballot_w64(!plain_ok) != 0) return false;
        }
        if constexpr (BF) {
            auto bits_of = [&](int key) -> uint32_t {
                const int k16 = key >> 16;
                if constexpr (NEG) return k16 < 0 ? ((uint32_t)(-k16) | 0x8000u) : (uint32_t)k16;
                else return (uint32_t)k16 & 0xFFFFu;
            };
            if (a.mode == SLIMFIT_PRUNE_THRESHOLD) {
                int n = 0;
#pragma unroll
                for (int i = 0; i < K; ++i) n += (i < k && bf16_widen(bits_of(m[i])) >= a.tau) ? 1 : 0;
                kk = n;
            }
#pragma unroll
            for (int i = 0; i < K; ++i)
                c[i] = i < kk ? ((uint32_t)min(column_of(m[i]), cols - 1) << 16) | bits_of(m[i]) : kNoPair;
        } else {
            int cut_v = INT_MIN, next_v = INT_MIN;          // value bits of the k-th and the (k+1)-th largest
#pragma unroll
            for (int i = 0; i < CHP; ++i) {
                cut_v = (i == k - 1) ? m[i] >> (TAG_BITS + LANE_BITS) : cut_v;
                next_v = (i == k) ? m[i] >> (TAG_BITS + LANE_BITS) : next_v;
            }
            exact = cut_v == next_v;
            if (a.mode == SLIMFIT_PRUNE_THRESHOLD) {
                const int tau_v = signed_key_f32(__builtin_bit_cast(uint32_t, a.tau)) >> (TAG_BITS + LANE_BITS);
                int n = 0;
                bool unsure = false;
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    const int v = m[i] >> (TAG_BITS + LANE_BITS);
                    n += (i < k && v > tau_v) ? 1 : 0;
                    unsure = unsure || (i < k && v == tau_v);
                }
                if (n < k) exact = false;                   // fewer than k pass: the kept set is {entries >= tau}
                kk = n;
                exact = exact || unsure;
            }
#pragma unroll
            for (int i = 0; i < K; ++i) c[i] = i < kk ? (uint32_t)min(column_of(m[i]), cols - 1) << 16 : kNoPair;
        }

        if constexpr (Held::HELD) {
            if (__builtin_amdgcn_ballot_w64(exact || !plain_ok) != 0) {
                const bool constant = held.constant_rows();
                if (!NEG && __builtin_amdgcn_ballot_w64(!plain_ok && !constant) != 0) return false;
                exact = exact && !constant;
#pragma unroll
                for (int i = 0; i < K; ++i) c[i] = constant ? (i < k ? (uint32_t)i << 16 : kNoPair) : c[i];
            }
        }
        uint32_t *orow = oc + r * k;
        const bool any_exact = !BF && (SLIMFIT_SHORT_FORCE_EXACT || __builtin_amdgcn_ballot_w64(exact) != 0);
        if (!any_exact) {
            sort_ascending<K>(c);
#pragma unroll
            for (int i = 0; i < K; ++i)
                if (i % G == q && i < k) orow[i] = c[i];
        }
        if constexpr (!BF) {
            if (any_exact) {
                // ---- the exact route: full 32-bit images, then a second walk over the entries ----
                constexpr int CH = K + 1;
                int s[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) s[i] = INT_MIN;
                auto full_key = [&](int bits) { return NEG ? signed_key_f32((uint32_t)bits) : bits; };
                walk([&](int e, int bits, bool ok) { chain_insert<CH>(s, ok ? full_key(bits) : INT_MIN); });
                int mm[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) mm[i] = s[i];
                merge_row<G, CH>(mm);
                int cut = INT_MIN, cut_next = INT_MIN;
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    cut = (i == k - 1) ? mm[i] : cut;
                    cut_next = (i == k) ? mm[i] : cut_next;
                }
                bool take_all_equal = cut_next != cut;      // exactly k entries reach the cut
                kk = k;
                if (a.mode == SLIMFIT_PRUNE_THRESHOLD) {
                    const int tau_key = signed_key_f32(__builtin_bit_cast(uint32_t, a.tau));
                    int n = 0;
#pragma unroll
                    for (int i = 0; i < K; ++i) n += (i < k && mm[i] >= tau_key) ? 1 : 0;
                    if (n < k) {                            // fewer than k pass: all of them are kept
                        kk = n;
                        cut = tau_key;
                        take_all_equal = true;
                    }
                }
                // from its own list a lane knows how many of its entries are above the cut and how many equal it
                int gt = 0, eq = 0;
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    gt += s[i] > cut ? 1 : 0;
                    eq += s[i] == cut ? 1 : 0;
                }
                int gt_of[G], eq_of[G];                     // the same of every lane of the row
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    gt_of[g] = __shfl(gt, (lane & ~(G - 1)) + g, kWave);
                    eq_of[g] = __shfl(eq, (lane & ~(G - 1)) + g, kWave);
                }
                int gt_all = 0;
#pragma unroll
                for (int g = 0; g < G; ++g) gt_all += gt_of[g];
                int need = take_all_equal ? INT_MAX : kk - gt_all;      // equal entries still to hand out, lower columns first
                int base = 0, take_eq = 0;
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const int t = min(max(need, 0), eq_of[g]);
                    if (g < q) base += gt_of[g] + t;
                    if (g == q) take_eq = t;
                    need = need == INT_MAX ? need : need - t;
                }
                // the same keys as in the selection, so the columns placed here are exactly the entries counted above
                uint32_t *out = orow + base;
                const int col0 = q * E;
                int seen = 0;
                walk([&](int e, int bits, bool ok) {
                    const int key = full_key(bits);
                    const bool is_eq = ok && key == cut;
                    if ((ok && key > cut) || (is_eq && seen < take_eq)) *out++ = (uint32_t)(col0 + e) << 16;
                    seen += is_eq ? 1 : 0;
                });
            }
        }

        kept = kk;
        return true;
    }
    // LDS serves a wave's accesses in order
    static __device__ __forceinline__ void settle()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // ---- the wave's pairs in output order; reread: the values come from the staged rows, not from oc ----
    static __device__ __forceinline__ void write_pairs(const ShortArgs &a, const T *rows_lds, const uint32_t *oc, bool reread, int lane,
                                                       int n_here, int64_t row0, int kept, T *__restrict__ vals,
                                                       uint16_t *__restrict__ idx, int32_t *__restrict__ counts)
    {
        const int cols = a.cols, k = a.k;
        const int n_out = n_here * k;
        T *ov = vals + row0 * (int64_t)k;
        uint16_t *oi = idx + row0 * (int64_t)k;
        uint32_t w[N_OUT];
        T v[N_OUT];
#pragma unroll
        for (int it = 0; it < N_OUT; ++it) {
            const int t = it * kWave + lane;
            w[it] = t < n_out ? oc[t] : kNoPair;
        }
#pragma unroll
        for (int it = 0; it < N_OUT; ++it) {
            const uint32_t t = (uint32_t)(it * kWave + lane);
            const uint32_t rl = min((t * a.div_magic) >> 16, (uint32_t)(R - 1));
            v[it] = (T)(w[it] & 0xFFFFu);                   // (0 of an unused slot)
            if (!BF || reread) {                            // wave-uniform
                const T x = rows_lds[rl * (uint32_t)cols + min(w[it] >> 16, (uint32_t)cols - 1u)];
                v[it] = w[it] != kNoPair ? x : T(0);
            }
        }
#pragma unroll
        for (int it = 0; it < N_OUT; ++it) {
            const int t = it * kWave + lane;
            if (t < n_out) {
                store_global<SLIMFIT_SHORT_NT_STORE != 0>(ov + t, v[it]);
                store_global<SLIMFIT_SHORT_NT_STORE != 0>(oi + t, (uint16_t)(w[it] >> 16));
            }
        }
        if (counts && lane % G == 0 && lane / G < n_here) counts[row0 + lane / G] = kept;
    }
};

// NV: 16-byte vectors a lane holds while the rows are staged (the wave's rows are 64 * cols bytes: NV >= cols / 16)
template <typename T, int G, int K, int NV>
__global__ __launch_bounds__(kWave) void prune_rows_short_kernel(const T *__restrict__ p, ShortArgs a,
                                                                 T *__restrict__ vals, uint16_t *__restrict__ idx,
                                                                 int32_t *__restrict__ counts)
{
    using S = ShortRows<T, G, K, NV>;
    extern __shared__ uint4 short_lds[];
    constexpr int R = S::R;
    constexpr int PER16 = 16 / (int)sizeof(T);
    static_assert(R * sizeof(T) % 16 == 0, "the wave's rows are a whole number of 16-byte vectors");
    const int lane = threadIdx.x;
    const int cols = a.cols, k = a.k;
    char *slab = reinterpret_cast<char *>(short_lds);
    const int slab_bytes = (int)short_rows_bytes(cols, G, (int)sizeof(T));
    uint32_t *oc = reinterpret_cast<uint32_t *>(slab + slab_bytes);        // R * k output slots
    u32x4 *dst_v = reinterpret_cast<u32x4 *>(slab);

    // The wave's R consecutive rows are one contiguous, 16-byte aligned piece of 64 * cols bytes.  No branch
    // around a load: lanes past the end of a short last piece re-read its last vector (and store it again where
    // it belongs), which keeps all NV loads in flight together.
    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int n_here = (int)min((int64_t)R, a.rows - row0);        // >= 1 by the launch size
    const int n_elem = n_here * cols;
    const int n_vec = n_elem / PER16;
    const u32x4 *src_v = reinterpret_cast<const u32x4 *>(p + row0 * (int64_t)cols);
    if (n_vec > (NV - 1) * kWave) {
        // (wave-uniform) the piece fills all NV rounds but perhaps the last: no index arithmetic on the others
        u32x4 v[NV];
        const int last = min((NV - 1) * kWave + lane, n_vec - 1);
#pragma unroll
        for (int u = 0; u < NV - 1; ++u) v[u] = load_global<SLIMFIT_SHORT_NT != 0>(src_v + u * kWave + lane);
        v[NV - 1] = load_global<SLIMFIT_SHORT_NT != 0>(src_v + last);
#pragma unroll
        for (int u = 0; u < NV - 1; ++u) dst_v[u * kWave + lane] = v[u];
        dst_v[last] = v[NV - 1];
    } else if (n_vec > 0) {
        // fewer rounds (narrow rows for this NV, or a short last piece): lanes past the end re-read the last vector
        // (and store it again where it belongs), which keeps the loads free of branches
        u32x4 v[NV];
#pragma unroll
        for (int u = 0; u < NV; ++u) v[u] = load_global<SLIMFIT_SHORT_NT != 0>(src_v + min(u * kWave + lane, n_vec - 1));
#pragma unroll
        for (int u = 0; u < NV; ++u) dst_v[min(u * kWave + lane, n_vec - 1)] = v[u];
    }
    {
        const int ei = n_vec * PER16 + lane;           // fewer than PER16 entries are left over (short last piece only)
        if (ei < n_elem) reinterpret_cast<T *>(slab)[ei] = p[row0 * (int64_t)cols + ei];
    }
    // unused output slots read as "no pair"
    for (int t = lane; t < R * k; t += kWave) oc[t] = kNoPair;
    S::settle();

    const T *rows_lds = reinterpret_cast<const T *>(slab);
    int kept;
    const typename S::NotHeld none;
    const bool plain = S::template select<false>(a, rows_lds, oc, lane, kept, none);
    if (!plain) S::template select<true>(a, rows_lds, oc, lane, kept, none);
    S::settle();
    S::write_pairs(a, rows_lds, oc, !plain, lane, n_here, row0, kept, vals, idx, counts);
}

// ---------------------------------------------------------------------------------------------------------------
// Row softmax and Alg. 5 in one pass over short rows of logits: the kept set is decided on the logits (which order
// a row exactly as its probabilities do), the dense probabilities are written once, and the kept values are the
// numbers the dense row holds.  The rows are staged as above; then every lane takes its part of its row into
// registers (the LDS of the staged rows lets about 20 waves into a compute unit at 197 columns, so there are registers
// enough for all of it), where selection, maximum, exponentials (hardware exp2), their sum (four running sums a lane, so that no
// sum is longer than a quarter of the lane's part; exchanged between the row's G lanes) and the division by it (one IEEE
// division a row) find it; the probabilities go back over the staged rows and leave for `probs` as one contiguous piece.
// Bound by the waves' lifetime on few rows and by HBM on many: 87 468 x 197 fp32 37.2 us when selection, maximum,
// exponentials and scaling each walked the staged rows, 34.2 from registers, 30.4 with eight lanes a row as well (4.7 TB/s);
// 302 592 rows 100 -> 90 (5.3 TB/s); 806 912 x 197 bf16 202 -> 162 (4.1 TB/s, bound by the list insertion).
template <typename T, int G, int K, int NV>
struct HeldRows {
    using S = ShortRows<T, G, K, NV>;
    static constexpr bool BF = sizeof(T) == 2, HELD = true;
    static constexpr int PER16 = 16 / (int)sizeof(T);
    static constexpr int kMost = NV * 16 / (int)sizeof(T), kBlk = kShortHeldBlock;      // entries a lane may have
    T *rows;                           // the staged rows (LDS)
    T *seg;                            // the lane's part
    T *out;                            // the wave's piece of the dense rows
    int lane, n_elem, E, len, e_all;
    float x[kMost];

    __device__ __forceinline__ HeldRows(int cols, T *rows_, T *out_, int lane_, int n_elem_) : rows(rows_), out(out_), lane(lane_), n_elem(n_elem_)
    {
        const int r = lane / G, q = lane % G;
        E = (cols + G - 1) / G;
        len = min(max(cols - q * E, 0), E);
        e_all = max(cols - (G - 1) * E, 0);                // entries every lane has
        seg = rows + r * cols + q * E;
        each_block([&](auto e0) {
            // (a lane without some of a block's entries reads the next row's, or at most G + 2 entries past the rows, which
            // the launch's LDS has room for)
#pragma unroll
            for (int u = 0; u < kBlk; ++u) x[e0 + u] = BF ? __builtin_bit_cast(float, (uint32_t)seg[e0 + u] << 16) : (float)seg[e0 + u];
        });
        each_block([&](auto e0) {
            if (e0 + kBlk <= e_all) return;
#pragma unroll
            for (int u = 0; u < kBlk; ++u) x[e0 + u] = e0 + u < len ? x[e0 + u] : -__builtin_inff();
        });
    }
    // f(first entry) for the blocks of kBlk entries that the widest lane has (unrolled as a pack: a loop this long would
    // not be, and its registers would become memory)
    template <typename F>
    __device__ __forceinline__ void each_block(F f) const
    {
        static_for(std::make_integer_sequence<int, kMost / kBlk>{}, [&](auto i) {
            if (i * kBlk < E) f(std::integral_constant<int, i * kBlk>{});          // wave-uniform
        });
    }
    // f(entry, its bits, whether the lane has it): bf16 16 bits, sign-extended with NEG; entries that the lane lacks are
    // -inf, below every kept entry of a plain pass, which is not told of them
    template <bool NEG, typename F>
    __device__ __forceinline__ void each_held(F f) const
    {
        each_block([&](auto e0) {
            const bool whole = !NEG || e0 + kBlk <= e_all;
#pragma unroll
            for (int u = 0; u < kBlk; ++u) {
                const int bits = __builtin_bit_cast(int, x[e0 + u]);
                f(e0 + u, !BF ? bits : (NEG ? bits >> 16 : (int)((uint32_t)bits >> 16)), whole || e0 + u < len);
            }
        });
    }
    // Is the row's every entry its first one?  Asked where a row would need a second pass, and so by the wave's whole; only
    // where the first three entries of each lane of some row agree are the others looked at (a few rows' waves decide how long
    // a launch of few rows takes: 24 576 x 192 8.7 us without this test, 9.5 with all entries at once, 8.7 so).
    __device__ __forceinline__ bool constant_rows() const
    {
        auto held_bits = [&](int e) { return __builtin_bit_cast(uint32_t, x[e]); };
        uint64_t alike = __builtin_amdgcn_ballot_w64(len < 3 || (held_bits(0) == held_bits(1) && held_bits(0) == held_bits(2)));
        alike &= alike >> 1;                                // of all the lanes of a row
        if (G >= 4) alike &= alike >> 2;
        if (G >= 8) alike &= alike >> 4;
        constexpr uint64_t firsts = G == 2 ? 0x5555555555555555u : (G == 4 ? 0x1111111111111111u : 0x0101010101010101u);
        if ((alike & firsts) == 0) return false;
        const uint32_t first = (uint32_t)__shfl((int)held_bits(0), lane & ~(G - 1), kWave);
        uint32_t differs = 0u;
        each_block([&](auto e0) {
#pragma unroll
            for (int u = 0; u < kBlk; ++u) differs |= e0 + u < len ? held_bits(e0 + u) ^ first : 0u;
        });
        differs |= dpp_u32<kDppXor1>(differs);
        if constexpr (G >= 4) differs |= dpp_u32<kDppXor2>(differs);
        if constexpr (G >= 8) differs |= dpp_u32<kDppHalfMirror>(differs);
        return differs == 0u;
    }
    // Has some row of the wave fewer than k entries without a sign?  Its k-th largest is negative then, and the selection on
    // plain bit patterns would be for nothing.  One instruction an entry: the signs are shifted into a register.  us with
    // both selections / with this, while the signed one walked the staged rows: negative logits 302 592 x 197 fp32 118 / 97,
    // 806 912 x 197 bf16 213 / 195; nine tenths masked 108 / 88, 211 / 195; plain rows 89.5 / 92.0, 170 / 170.  With both
    // selections from registers 97 and 167, 87 and 164, plain 90 and 162.  (Zeros have no sign: a row that they cut takes both.)
    __device__ __forceinline__ bool cut_is_negative(int k) const
    {
        uint32_t signs[(kMost + 31) / 32] = {};
        int n = 0;
        each_block([&](auto e0) {
#pragma unroll
            for (int u = 0; u < kBlk; ++u)
                signs[e0 / 32] = __builtin_amdgcn_alignbit(signs[e0 / 32], __builtin_bit_cast(uint32_t, x[e0 + u]), 31);
            n += kBlk;
        });
#pragma unroll
        for (int i = 0; i < (kMost + 31) / 32; ++i) n -= __builtin_popcount(signs[i]);      // (entries that a lane lacks hold -inf)
        n += (int)dpp_u32<kDppXor1>((uint32_t)n);
        if constexpr (G >= 4) n += (int)dpp_u32<kDppXor2>((uint32_t)n);
        if constexpr (G >= 8) n += (int)dpp_u32<kDppHalfMirror>((uint32_t)n);
        return __builtin_amdgcn_ballot_w64(n < k) != 0;
    }
    __device__ __forceinline__ void to_probabilities()
    {
        constexpr float kLog2e = 1.44269504088896340736f;
        float mx = -__builtin_inff();
        each_block([&](auto e0) {
            // the larger of two numbers (NaN is passed over)
#pragma unroll
            for (int u = 0; u < kBlk; ++u) mx = __builtin_amdgcn_fmed3f(x[e0 + u], mx, __builtin_inff());
        });
        mx = fmaxf(mx, dpp_f32<kDppXor1>(mx));
        if constexpr (G >= 4) mx = fmaxf(mx, dpp_f32<kDppXor2>(mx));
        if constexpr (G >= 8) mx = fmaxf(mx, dpp_f32<kDppHalfMirror>(mx));
        // (a lane of a row past the tensor's end, or one without entries, holds -inf here: its results are not used)
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        each_block([&](auto e0) {
#pragma unroll
            for (int u = 0; u < kBlk; ++u) {
                x[e0 + u] = __builtin_amdgcn_exp2f((x[e0 + u] - mx) * kLog2e);
                s[u] += x[e0 + u];
            }
        });
        float sum = (s[0] + s[1]) + (s[2] + s[3]);
        sum += dpp_f32<kDppXor1>(sum);
        if constexpr (G >= 4) sum += dpp_f32<kDppXor2>(sum);
        if constexpr (G >= 8) sum += dpp_f32<kDppHalfMirror>(sum);
        const float inv = 1.0f / sum;                       // IEEE division
        each_block([&](auto e0) {
            auto put = [&](int e) {
                if constexpr (BF) seg[e] = (T)bf16_narrow(x[e] * inv);
                else seg[e] = x[e] * inv;
            };
            if (e0 + kBlk <= e_all) {
#pragma unroll
                for (int u = 0; u < kBlk; ++u) put(e0 + u);
            } else {
#pragma unroll
                for (int u = 0; u < kBlk; ++u)
                    if (e0 + u < len) put(e0 + u);
            }
        });
        S::settle();
        // the dense rows leave as they came: one contiguous piece, 16 bytes a lane
        const int n_vec = n_elem / PER16;
        const u32x4 *src_v = reinterpret_cast<const u32x4 *>(rows);
        u32x4 *dst_v = reinterpret_cast<u32x4 *>(out);
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const int v = u * kWave + lane;
            if (v < n_vec) store_global<true>(dst_v + v, src_v[v]);
        }
        const int ei = n_vec * PER16 + lane;
        if (ei < n_elem) out[ei] = rows[ei];
    }
};

// Most waves a SIMD is to hold.  fp32 rows of 129 to 224 columns that keep 7 to 9 have registers for five, and are faster with
// four, whose loads queue less, but at the ends: 197 columns, 60 000 rows 22.7 us with four, 22.1 with five, 80 000 27.5 / 28.0,
// 98 304 32.2 / 32.9, 130 000 40.5 / 42.0, 160 000 48.8 / 50.8, 302 592 87.8 / 85.7.  Others lose with four (98 304 x 100, k = 5
// 18.8 / 17.0) or have registers for no more.
template <typename T, int G, int K, int NV> constexpr int kSoftmaxWaves = sizeof(T) == 4 && G == 8 && K == 9 && NV == 7 ? 4 : 8;

template <typename T, int G, int K, int NV>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, kSoftmaxWaves<T, G, K, NV>))) void softmax_prune_short_kernel(const T *__restrict__ p, ShortArgs a,
                                                                    T *__restrict__ probs, T *__restrict__ vals,
                                                                    uint16_t *__restrict__ idx)
{
    using S = ShortRows<T, G, K, NV>;
    extern __shared__ uint4 short_lds[];
    constexpr int R = S::R;
    constexpr int PER16 = 16 / (int)sizeof(T);
    const int lane = threadIdx.x;
    const int cols = a.cols, k = a.k;
    char *slab = reinterpret_cast<char *>(short_lds);
    const int slab_bytes = (int)short_rows_bytes(cols, G, (int)sizeof(T));
    uint32_t *oc = reinterpret_cast<uint32_t *>(slab + slab_bytes);        // R * k output slots
    u32x4 *slab_v = reinterpret_cast<u32x4 *>(slab);

    const int64_t row0 = (int64_t)blockIdx.x * R;
    const int n_here = (int)min((int64_t)R, a.rows - row0);        // >= 1 by the launch size
    const int n_elem = n_here * cols;
    const int n_vec = n_elem / PER16;
    const u32x4 *src_v = reinterpret_cast<const u32x4 *>(p + row0 * (int64_t)cols);
    if (n_vec > 0) {
        // lanes past the end of a short last piece re-read its last vector (and store it again where it belongs)
        u32x4 v[NV];
#pragma unroll
        for (int u = 0; u < NV; ++u) v[u] = load_global<SLIMFIT_SHORT_NT != 0>(src_v + min(u * kWave + lane, n_vec - 1));
#pragma unroll
        for (int u = 0; u < NV; ++u) slab_v[min(u * kWave + lane, n_vec - 1)] = v[u];
    }
    {
        const int ei = n_vec * PER16 + lane;           // fewer than PER16 entries are left over (short last piece only)
        if (ei < n_elem) reinterpret_cast<T *>(slab)[ei] = p[row0 * (int64_t)cols + ei];
    }
    for (int t = lane; t < R * k; t += kWave) oc[t] = kNoPair;
    S::settle();

    HeldRows<T, G, K, NV> held(cols, reinterpret_cast<T *>(slab), probs + row0 * (int64_t)cols, lane, n_elem);
    const T *rows_lds = reinterpret_cast<const T *>(slab);
    int kept;
    bool selected = false;
    if (!held.cut_is_negative(k)) selected = S::template select<false>(a, rows_lds, oc, lane, kept, held);
    if (!selected) S::template select<true>(a, rows_lds, oc, lane, kept, held);
    S::settle();
    held.to_probabilities();
    S::write_pairs(a, rows_lds, oc, true, lane, n_here, row0, kept, vals, idx, nullptr);
}

// Lanes to a softmax row: a wave that holds half as many rows lives half as long (and twice as many fit the LDS), which
// wide rows gain more from than they lose to one more merge of the lists.  Eight lanes (fp32) against four, us:
// 87 468 x 197 30.4 / 34.2, 49 152 x 197 20.1 / 22.8, 16 384 x 130 9.3 / 11.0, 8192 x 112 6.5 / 7.4, 98 304 x 112 18.7 / 17.9,
// x 79 14.7 / 14.0, x 50 10.3 / 8.2.  bf16, four against two: 806 912 x 197 169 / 175, 32 768 x 250 16.2 / 21.1, 8192 x 96
// 6.9 / 7.6, 98 304 x 96 12.9 / 12.6, x 79 14.2 / 13.4.  (bf16 with eight lanes: 183 at 806 912 x 197.)
constexpr int kSoftmaxWideCols = 96;
// With many rows their number hides a wave's lifetime and the one merge more is what counts, and the more so the longer the
// lists.  fp32, four lanes against eight: k = 9, 49 152 x 100 11.9 / 13.1, 98 304 x 100 20.3 / 22.0, x 112 21.8 / 22.5, x 127
// 24.7 / 23.5, 196 608 x 100 33.8 / 41.5 (few distinct values 43 / 58), x 120 36 / 41, x 127 42.3 / 43.8, 24 576 x 100 10.9 / 10.0;
// k = 12, 49 152 x 96 13.7 / 15.6, 196 608 x 100 37 / 50; k = 5, 98 304 x 100 17.3 / 17.8, 196 608 x 100 30.5 / 31.6 but x 96, whose
// 16 rows lie in two banks, 30.7 / 28.9.
bool softmax_wide(int32_t dt, int64_t rows, int cols, int k)
{
    if (cols < kSoftmaxWideCols) return false;
    if (dt != SLIMFIT_F32 || cols >= 128 || k <= 4) return true;
    if (k <= 6) return cols > 112 || cols == 96 || rows < 98304;
    return rows < (k > 9 || cols <= 112 ? 40000 : 131072);
}

// f(the call's arguments, its first row, its blocks) for pieces of rows that a grid has threads for
template <int G, typename F>
void in_pieces(const ShortArgs &a, F f)
{
    constexpr int R = kWave / G;
    constexpr int64_t kMost = kMaxGridThreads / kWave * R;     // rows (a multiple of 64: pieces begin on 16 bytes)
    for (int64_t row0 = 0; row0 < a.rows; row0 += kMost) {
        ShortArgs piece = a;
        piece.rows = a.rows - row0 < kMost ? a.rows - row0 : kMost;
        f(piece, row0, (unsigned)((piece.rows + R - 1) / R));
    }
}

template <typename T, int G, int K, int NV>
void launch_softmax_short(const T *p, const ShortArgs &a, T *probs, T *vals, uint16_t *idx, hipStream_t st)
{
    const size_t lds = short_lds_bytes(a.cols, a.k, G, (int)sizeof(T), kShortHeldBlock);
    in_pieces<G>(a, [&](const ShortArgs &piece, int64_t row0, unsigned blocks) {
        launch(softmax_prune_short_kernel<T, G, K, NV>, blocks, kWave, lds, st, p + row0 * a.cols, piece, probs + row0 * a.cols, vals + row0 * a.k,
                                                                            idx + row0 * a.k);
    });
}

// WIDE: rows of at least kSoftmaxWideCols columns, and so many lanes to a row
template <typename T, bool WIDE> constexpr int kSoftmaxLanes = (WIDE ? 2 : 1) * (sizeof(T) == 2 ? 2 : 4);

template <typename T, bool WIDE, int K>
void launch_softmax_short_nv(const T *p, const ShortArgs &a, T *probs, T *vals, uint16_t *idx, hipStream_t st)
{
    // rounds of 64 vectors a piece takes when it is 64, 128, 224 (197 columns) or 256 columns wide
    constexpr int G = kSoftmaxLanes<T, WIDE>;
    constexpr int kFull = kWave / G * (int)sizeof(T) * 256 / 16 / kWave, kMost = (kFull * 13 + 15) / 16;
    const int nv = (kWave / G * a.cols * (int)sizeof(T) / 16 + kWave - 1) / kWave;
    if constexpr (WIDE) {
        if (nv <= kFull / 2) launch_softmax_short<T, G, K, kFull / 2>(p, a, probs, vals, idx, st);
        else if (nv <= kMost) launch_softmax_short<T, G, K, kMost>(p, a, probs, vals, idx, st);
        else launch_softmax_short<T, G, K, kFull>(p, a, probs, vals, idx, st);
    } else {
        static_assert(kSoftmaxWideCols <= 128, "half the columns");
        if (nv <= kFull / 4) launch_softmax_short<T, G, K, kFull / 4>(p, a, probs, vals, idx, st);
        else launch_softmax_short<T, G, K, kFull / 2>(p, a, probs, vals, idx, st);
    }
}

template <typename T, bool WIDE>
void launch_softmax_short_k(const T *p, const ShortArgs &a, T *probs, T *vals, uint16_t *idx, hipStream_t st)
{
    if (a.k <= 2) launch_softmax_short_nv<T, WIDE, 2>(p, a, probs, vals, idx, st);
    else if (a.k <= 4) launch_softmax_short_nv<T, WIDE, 4>(p, a, probs, vals, idx, st);
    else if (a.k <= 6) launch_softmax_short_nv<T, WIDE, 6>(p, a, probs, vals, idx, st);
    else if (a.k <= 9) launch_softmax_short_nv<T, WIDE, 9>(p, a, probs, vals, idx, st);
    else if (a.k <= 12) launch_softmax_short_nv<T, WIDE, 12>(p, a, probs, vals, idx, st);
    else if constexpr (sizeof(T) == 2) launch_softmax_short_nv<T, WIDE, 16>(p, a, probs, vals, idx, st);
}

constexpr int kShortLongListF32 = 9;       // fp32 rows that keep more have lines of their own (prune_short_eligible)

template <typename T, int G, int K, int NV>
void launch_short(const T *p, const ShortArgs &a, T *vals, uint16_t *idx, int32_t *counts, hipStream_t st)
{
#ifndef SLIMFIT_SHORT_LDS_PAD
#define SLIMFIT_SHORT_LDS_PAD 0        // timing experiments only: LDS a wave claims beyond what it uses
#endif
    const size_t lds = short_lds_bytes(a.cols, a.k, G, (int)sizeof(T), 1) + SLIMFIT_SHORT_LDS_PAD;
    in_pieces<G>(a, [&](const ShortArgs &piece, int64_t row0, unsigned blocks) {
        launch(prune_rows_short_kernel<T, G, K, NV>, blocks, kWave, lds, st, p + row0 * a.cols, piece, vals + row0 * a.k, idx + row0 * a.k,
                                                                        counts ? counts + row0 : nullptr);
    });
}

template <typename T, int G, int K>
void launch_short_nv(const T *p, const ShortArgs &a, T *vals, uint16_t *idx, int32_t *counts, hipStream_t st)
{
    constexpr int R = kWave / G;
    const int nv = (R * a.cols * (int)sizeof(T) / 16 + kWave - 1) / kWave;      // rounds of 64 vectors a piece takes
    if (nv <= 4) launch_short<T, G, K, 4>(p, a, vals, idx, counts, st);
    else if (nv <= 8) launch_short<T, G, K, 8>(p, a, vals, idx, counts, st);
    else if constexpr (sizeof(T) == 2 || K <= kShortLongListF32) {     // (fp32 rows of the longest lists have under 128 columns)
        if (nv <= 13) launch_short<T, G, K, 13>(p, a, vals, idx, counts, st);   // 197 columns
        else launch_short<T, G, K, 16>(p, a, vals, idx, counts, st);
    }
}

template <typename T, int G>
void launch_short_k(const T *p, const ShortArgs &a, T *vals, uint16_t *idx, int32_t *counts, hipStream_t st)
{
    if (a.k <= 2) launch_short_nv<T, G, 2>(p, a, vals, idx, counts, st);
    else if (a.k <= 4) launch_short_nv<T, G, 4>(p, a, vals, idx, counts, st);
    else if (a.k <= 6) launch_short_nv<T, G, 6>(p, a, vals, idx, counts, st);
    else if (a.k <= 9) launch_short_nv<T, G, 9>(p, a, vals, idx, counts, st);
    else if (a.k <= 12) launch_short_nv<T, G, 12>(p, a, vals, idx, counts, st);
    else if constexpr (sizeof(T) == 2) launch_short_nv<T, G, 16>(p, a, vals, idx, counts, st);
}

}  // namespace

// Which short rows come here rather than to the wave-per-row kernel (prune.hip).  Both were measured on 33 .. 256 columns
// and 2048 .. 196 608 rows; times are this kernel's against the other's, in us:
//  - few enough kept entries: the list insertion grows with k.  fp32 rows that keep 13 to 16 lose (196 608 x 140, k = 14:
//    softmax 74 against 63, pruning 46 against 44).  Those that keep 10 to 12 gain from 32 768 rows on up to 96 columns (98 304
//    rows: softmax of 64 columns 18.7 against 29.7, pruning 14.4 / 19.5; 24 576 rows: pruning of 80 columns 8.0 / 8.8, softmax of
//    90 10.6 / 11.2) and from 65 536 rows on with more: pruning of 97 to 127 columns (100 columns 13.4 / 16.3, 127 15.3 / 16.6)
//    and of no more (49 152 x 197 18.7 / 15.9), softmax of all but 128 and 192 (98 304 x 192 34.6 / 33.5; 196 608 rows: 100
//    columns 37 / 56, 197 69 / 81, 250 82 / 101; 65 536 rows: 160 with negative logits 25.7 / 24.6).  Not with a threshold: rows
//    of which fewer than k pass it are done at once in the other kernel (98 304 rows: peaked ones of 64 columns 14.7 / 12.4,
//    of 112 20.5 / 13.4, masked 20.1 / 13.4; plain ones 15.2 / 18.9 and 21.0 / 22.5);
//  - strides that spread over the LDS banks: the lanes of a wave read the same entry of 16 rows at once, and at a
//    stride of a multiple of 64 dwords those lie in one bank (196 608 rows, fp32 pruning, from 128 columns on: 105 against
//    47 at 256, 54 against 38 at 128, but 18 against 34 at 64).  Softmax, whose fp32 waves hold 8 rows and go to the LDS once
//    to take them up and once to lay the probabilities down, loses on 256 columns (131 072 rows: fp32 123 against 51, bf16
//    63 against 53) and on few rows of 128 and 192 that keep more than 6 (k = 9, 24 576 rows: 192 12.2 against 11.3, negative
//    logits 14.6 / 11.4, 128 10.9 / 10.8 and 12.2 / 10.8; 49 152 rows: 19.2 / 19.0 and 21.4 / 19.0, 17.2 / 17.6 and 18.4 / 17.6,
//    few distinct values 23 / 47 and 20 / 42; 196 608 rows: 57 / 62, 52 / 56; k = 6, 24 576 rows: 10.5 / 11.4, 9.3 / 10.6);
//  - enough rows: a wave takes 8 to 32 of them and needs 7 - 15 us whatever their number, while the other kernel gives
//    few rows a wave each.  From 128 columns on, at 197 columns: fp32 pruning of 16 384 rows 11.2 against 8.3, 24 576 12.7 /
//    10.0, 49 152 17.6 / 15.9 (peaked 16.2 against 19.1, nine tenths masked 14.9 against 17.7), 196 608 40 / 47.  bf16
//    softmax of 16 384 rows 10.6 against 10.8 (250 columns 12.1 / 10.7), 20 000 12.5 / 15.5.  fp32 softmax of 20 000 rows
//    12.6 against 11.8 (250 columns 13.9 / 12.3), 24 576 12.6 / 14.3, 32 768 14.9 / 17.4, 49 152 19.7 / 25.2.
//    Below 128 columns the two are within 1 us of one another for few rows (fp32 pruning of 16 384 x 112 7.1 against 7.2)
//    and this one is ahead from 24 576 on, so their number is not looked at but for fp32 softmax of 64 and 96 columns, which
//    the other kernel has in whole slots (2048 rows, k = 9: 5.3 against 4.8, negative logits 6.6 / 4.7; 8192 rows: 6.2 / 6.4,
//    7.5 / 6.2, few distinct values 6.9 / 9.9; 16 384 rows 7.2 / 8.5).  Nor is it for bf16 pruning: plain rows gain in
//    the other kernel at k = 16 (16 384 x 197 9.5 against 8.1), but rows with masked columns, whose zeros share one
//    histogram bin there, lose more (9.6 against 14.8; peaked 9.5 against 9.7).
// What stays slower here or there: pruned fp32 rows of few distinct values (logits in steps of a half) take the other kernel's
// bisection to the last bit, 98 304 x 192 62 us here, 85 there, 16 384 x 197 12 and 20; constant rows 61 and 70, 12 and 16.
// fp32 softmax rows that are negative throughout, 24 576 x 197 15.7 and 14.3 (plain ones 12.6 and 14.3).
constexpr int64_t kShortMinRows = 20000, kShortMinRowsSoftmaxF32 = 24000, kStrideMinRowsSoftmaxF32 = 40000,
                  kNarrowMinRowsSoftmaxF32 = 6000, kLongListMinRows = 65536,
                  kLongListMinRowsNarrow = 32768;

bool prune_short_eligible(const void *p, int32_t dt, int64_t rows, int cols, int k, int mode, bool softmax)
{
    const bool bf16 = dt == SLIMFIT_BF16;
    if (cols > kShortPruneMaxCols || k > (bf16 ? kShortPruneMaxK : kShortPruneMaxKF32)) return false;
    if (!aligned_to(p, 16)) return false;              // (the rows are staged with 16-byte loads)
    if (!bf16 && k > kShortLongListF32) {
        if (mode == SLIMFIT_PRUNE_THRESHOLD) return false;
        if (cols <= 96) return rows >= kLongListMinRowsNarrow;
        return rows >= kLongListMinRows && (softmax ? cols % 64 != 0 : cols < 128);
    }
    if (softmax && bf16) return cols != 256 && (cols < 128 || rows >= kShortMinRows);
    if (softmax) {
        if (cols >= 128) return cols != 256 && rows >= (cols % 64 == 0 && k > 6 ? kStrideMinRowsSoftmaxF32 : kShortMinRowsSoftmaxF32);
        return !(cols >= 64 && cols % 32 == 0) || rows >= kNarrowMinRowsSoftmaxF32;
    }
    if (bf16) return true;
    return !(cols >= 128 && cols % 64 == 0) && (cols < 128 || rows >= kShortMinRows);
}

void launch_softmax_prune_short(const void *logits, int32_t dt, int64_t rows, int cols, int k, void *probs, void *vals,
                                uint16_t *idx, hipStream_t st)
{
    ShortArgs a;
    a.rows = rows;
    a.cols = cols;
    a.k = k;
    a.mode = SLIMFIT_PRUNE_TOPK;
    a.tau = 0.0f;
    a.div_magic = 65536u / (uint32_t)k + 1u;
    const bool wide = softmax_wide(dt, rows, cols, k);
    auto launch = [&](auto *x) {
        using T = std::remove_pointer_t<decltype(x)>;
        const T *in = static_cast<const T *>(logits);
        T *pr = static_cast<T *>(probs), *v = static_cast<T *>(vals);
        if (wide) launch_softmax_short_k<T, true>(in, a, pr, v, idx, st);
        else launch_softmax_short_k<T, false>(in, a, pr, v, idx, st);
    };
    if (dt == SLIMFIT_F32) launch(static_cast<float *>(nullptr));
    else launch(static_cast<uint16_t *>(nullptr));
}

void launch_prune_short(const void *p, int32_t dt, int64_t rows, int cols, int k, int mode, float tau, void *vals,
                        uint16_t *idx, int32_t *counts, hipStream_t st)
{
    ShortArgs a;
    a.rows = rows;
    a.cols = cols;
    a.k = k;
    a.mode = mode;
    a.tau = tau;
    a.div_magic = 65536u / (uint32_t)k + 1u;
#ifndef SLIMFIT_SHORT_G_F32
#define SLIMFIT_SHORT_G_F32 4
#endif
    if (dt == SLIMFIT_F32)
        launch_short_k<float, SLIMFIT_SHORT_G_F32>(static_cast<const float *>(p), a, static_cast<float *>(vals), idx, counts, st);
    else
#ifndef SLIMFIT_SHORT_G_BF16
#define SLIMFIT_SHORT_G_BF16 2
#endif
        launch_short_k<uint16_t, SLIMFIT_SHORT_G_BF16>(static_cast<const uint16_t *>(p), a, static_cast<uint16_t *>(vals), idx, counts, st);
}

}  // namespace slimfit
