// The whole-tensor pruner's order of elements (prune_global.hip), in plain C++ so that it can be checked on the host.
//
// An element's key is its magnitude's bits or the usual signed fold of its bits, with -0 ordered as +0; a larger key comes
// earlier.  NaN have keys as well: above the infinities by magnitude, beyond the infinity of their sign by value.
#pragma once
#include <cstdint>

namespace slimfit {

template <int BITS, bool MAG> constexpr uint32_t key_of(uint32_t b)        // BITS: 32 (fp32) or 16 (bf16)
{
    constexpr uint32_t sign = 1u << (BITS - 1), all = sign | (sign - 1u);
    if (MAG) return (b << 1) & all;
    if (b == sign) b = 0u;
    return b ^ ((b & sign) ? all : sign);
}

// Whether an element's key is at least `lo`, without making it.  By magnitude one comparison of numbers (`lo` is no NaN's key:
// whoever gets such a lower edge cannot use this).  By value the fold is the same for all elements: one that is wrong for the
// elements of the other sign than the edge's leaves them on their side of it.
struct Reach {
    uint32_t flip, from;
};
template <int BITS, bool MAG> constexpr bool reach_exists(uint32_t lo) { return !MAG || lo <= 0xFF000000u >> (32 - BITS); }
template <int BITS, bool MAG> constexpr Reach reach_of(uint32_t lo)
{
    constexpr uint32_t sign = 1u << (BITS - 1), all = sign | (sign - 1u);
    if (MAG) return Reach{0u, (lo << (32 - BITS)) >> 1};
    return lo > sign ? Reach{sign, lo} : Reach{all, lo == sign ? sign - 1u : lo};      // an edge of zero is reached by -0 too
}
template <int BITS, bool MAG> constexpr bool reaches(uint32_t b, Reach r)
{
    if (MAG) return !(__builtin_fabsf(__builtin_bit_cast(float, b << (32 - BITS))) < __builtin_bit_cast(float, r.from));
    return (b ^ r.flip) >= r.from;
}
// by value with an edge above zero: one comparison of signed whole numbers
template <int BITS> constexpr bool reach_is_positive(uint32_t lo) { return lo > 1u << (BITS - 1); }
template <int BITS> constexpr bool reaches_positive(uint32_t b, uint32_t lo)
{
    const uint32_t number = lo ^ (1u << (BITS - 1));
    return BITS == 16 ? (int16_t)b >= (int16_t)number : (int32_t)b >= (int32_t)number;
}

}  // namespace slimfit
