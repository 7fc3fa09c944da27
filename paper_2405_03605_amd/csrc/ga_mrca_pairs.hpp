// MRCA interval of one pair of surfaces, in a bounded number of integer
// operations for every policy (paper Fig. 1: relatedness estimated from the
// markers two genomes carry). Plain C++ for host and device.
//
// A rank is retained from its deposit until the deposit that overwrites its
// site, so two surfaces with deposit counters lo <= hi share exactly the ranks
// below lo that the one with hi still holds, and a rank sits at one site
// whatever the counter. U is the oldest shared rank whose fields differ (or
// lo), L sits kc shared ranks below U, plus one (0 if there are fewer).
//
// Tilted policy, one slot per level. With w = hi - 1 the ranks held are
// w - age(x), one for every x from 0 to bitlen(w) (at most 31), age(x) =
// (w mod 2^x) | 2^(x-1): one per doubling of age, in order. The zero bits k
// of w hold their level's rank at x = k + 1 and the one bits at x = (next one
// bit below k) + 1; level 31 counts as a one bit. So the oldest differing rank is
// the top differing zero-bit level or the top differing one-bit level, and the
// kc-th rank below it is at x + kc. With two slots per level the second
// newest rank of level k has age 2^(k+1) plus the low k + 1 bits of w with bit
// k flipped, and the ages in order are w mod 2^q plus (2 or 3) 2^q, two per
// doubling.
#pragma once

#include <stdint.h>

#ifdef __HIP__
#define GA_PAIR __host__ __device__ __forceinline__
#else
#define GA_PAIR inline
#endif

namespace ga {

// bits of v: 0 for 0, else the place of its top bit plus one
GA_PAIR uint32_t bitlen(uint32_t v) { return v ? 32u - (uint32_t)__builtin_clz(v) : 0u; }
// the bits below v's top bit
GA_PAIR uint32_t below_top(uint32_t v) { return 0x7FFFFFFFu >> __builtin_clz(v | 1u); }
GA_PAIR uint32_t low_bits(uint32_t v, uint32_t n) { return v & ((1u << n) - 1u); }  // n < 32

struct Interval {
  uint32_t lower, upper;
};

// The even and odd bits of a 64-bit string, each packed.
GA_PAIR uint32_t even_bits(uint64_t v) {
  v &= 0x5555555555555555ull;
  v = (v | (v >> 1)) & 0x3333333333333333ull;
  v = (v | (v >> 2)) & 0x0F0F0F0F0F0F0F0Full;
  v = (v | (v >> 4)) & 0x00FF00FF00FF00FFull;
  v = (v | (v >> 8)) & 0x0000FFFF0000FFFFull;
  return (uint32_t)(v | (v >> 16));
}

// ---- one slot per level ---------------------------------------------------------

// Age of the rank at place x (x <= 31), and the first place whose age is at
// least `age` (up to 32: none).
GA_PAIR uint32_t ring_age(uint32_t w, uint32_t x) { return low_bits(w, x) | ((1u << x) >> 1); }
GA_PAIR uint32_t ring_from(uint32_t w, uint32_t age) {
  const uint32_t x = bitlen(age);
  return x > 31u ? 32u : x + (ring_age(w, x) < age ? 1u : 0u);
}
GA_PAIR uint32_t ring_top(uint32_t w) {
  const uint32_t x = bitlen(w);
  return x < 31u ? x : 31u;
}
// Place of the oldest differing newest rank (-1: none), `diff` one bit per
// level. Levels that hold no rank yet do not count; places below the shared
// ones may be returned.
GA_PAIR int32_t ring_oldest(uint32_t w, uint32_t diff) {
  const uint32_t zeros = diff & ~w & below_top(w);
  const uint32_t ones = diff & (w | 0x80000000u);
  const int32_t z = zeros ? (int32_t)bitlen(zeros) : -1;
  const int32_t o = ones ? (int32_t)bitlen(w & below_top(ones)) : -1;
  return z > o ? z : o;
}

GA_PAIR Interval tilted_interval(uint32_t ta, uint32_t tb, uint32_t diff, uint32_t kc) {
  const uint32_t hi = ta > tb ? ta : tb, lo = ta > tb ? tb : ta;
  if (lo == 0u) return {0u, 0u};
  const uint32_t w = hi - 1u;
  const int32_t first = (int32_t)ring_from(w, hi - lo);
  const int32_t y = ring_oldest(w, diff);
  const bool differs = y >= first;
  const uint32_t at = differs ? (uint32_t)y : 0u;
  const uint32_t upper = differs ? w - ring_age(w, at) : lo;
  const uint32_t next = (uint32_t)((differs ? y : first - 1) + (int32_t)(kc < 64u ? kc : 64u));
  const uint32_t lower = next <= ring_top(w) ? w - ring_age(w, next & 31u) + 1u : 0u;
  return {lower, upper};
}

// ---- two slots per level --------------------------------------------------------

// Place in the order of ages of the cell `age` falls in, the age there, and the
// first place whose age is at least `age`.
GA_PAIR uint32_t pair_place(uint32_t age) {
  const uint32_t x = bitlen(age);
  return x < 2u ? x : 2u * x - 2u + ((age >> (x - 2u)) & 1u);
}
GA_PAIR uint32_t pair_age(uint32_t w, uint32_t z) {
  const uint32_t q = (z >> 1) - 1u;  // places 0 and 1: ages 0 and 1
  return z < 2u ? z : low_bits(w, q) + ((2u + (z & 1u)) << q);
}
GA_PAIR uint32_t pair_from(uint32_t w, uint32_t age) {
  const uint32_t z = pair_place(age);
  return z + (pair_age(w, z) < age ? 1u : 0u);
}

// d0, d1: one bit per level for each of its slots
GA_PAIR Interval tilted2_interval(uint32_t ta, uint32_t tb, uint32_t d0, uint32_t d1,
                                  uint32_t kc) {
  const uint32_t hi = ta > tb ? ta : tb, lo = ta > tb ? tb : ta;
  if (lo == 0u) return {0u, 0u};
  const uint32_t w = hi - 1u, top = 0x80000000u;
  // slot of each level's newest rank: the parity of its index along the level
  const uint32_t slot = (~(w ^ (w >> 1)) & ~top) | (w & top);
  const int32_t y = ring_oldest(w, (d0 & ~slot) | (d1 & slot));
  const uint32_t below = below_top(w);
  const uint32_t held = (below >> 1) | (w & (below | top));  // levels with a second rank
  const uint32_t second = ((d1 & ~slot) | (d0 & slot)) & held;
  const uint32_t k = bitlen(second) - 1u;  // when second != 0
  const uint32_t bit = 1u << (k & 31u);
  const uint32_t age2 = (second & top) ? w : (((w ^ bit) & (2u * bit - 1u)) | (2u * bit));
  uint32_t age = y >= 0 ? ring_age(w, (uint32_t)y) : 0u;
  if (second && age2 > age) age = age2;
  const bool differs = (y >= 0 || second) && age >= hi - lo;
  const uint32_t first = pair_from(w, hi - lo);
  const uint32_t upper = differs ? w - age : lo;
  const uint32_t next = (differs ? pair_place(age) + 1u : first) + (kc < 128u ? kc : 128u) - 1u;
  const uint32_t lower = next <= pair_place(w) ? w - pair_age(w, next) + 1u : 0u;
  return {lower, upper};
}

// ---- hybrid: a steady half on the even ranks, a tilted half on the odd ones --------

// steady a, b: the halves' strings thinned to the shared epoch E, shared ranks
// 2 j 2^E for j < shared; diff: the tilted half's levels.
GA_PAIR Interval hybrid_interval(uint32_t ta, uint32_t tb, uint32_t sa, uint32_t sb, uint32_t E,
                                 uint32_t shared, uint32_t diff, uint32_t kc) {
  const uint32_t lo = ta < tb ? ta : tb;
  uint32_t upper = lo;
  const uint32_t hit = (sa ^ sb) & (shared >= 32u ? 0xFFFFFFFFu : (1u << shared) - 1u);
  if (hit) upper = 2u * ((uint32_t)__builtin_ctz(hit) << E);
  const uint32_t hi1 = (ta > tb ? ta : tb) >> 1, lo1 = lo >> 1;
  const bool ring = lo1 != 0u;
  const uint32_t w = ring ? hi1 - 1u : 0u;
  const int32_t first = ring ? (int32_t)ring_from(w, hi1 - lo1) : 32;
  const int32_t y = ring_oldest(w, diff);
  if (y >= first) {
    const uint32_t r = 2u * (w - ring_age(w, (uint32_t)y)) + 1u;
    if (r < upper) upper = r;
  }
  // The kc-th shared rank below upper: of two descending lists a (tilted, from
  // place x on) and b (steady, j ranks) the k-th largest is the greatest
  // min(a_i, b_(k-i)), with nothing smaller than an absent a_0 or b_0. Ranks are
  // held plus one, 0 for none.
  uint32_t x = 32u;
  if (ring && upper > 1u) {
    const uint32_t under = (upper - 2u) >> 1;  // the ranks 2 q + 1 with q <= under
    const uint32_t from = ring_from(w, under < w ? w - under : 0u);
    x = from > (uint32_t)first ? from : (uint32_t)first;
  }
  uint32_t j = 0u;
  if (upper != 0u) {
    j = ((upper - 1u) >> (E + 1u)) + 1u;
    j = j < shared ? j : shared;
  }
  const uint32_t k = kc < 65u ? kc : 65u;  // neither list has more than 32
  uint32_t lower = j >= k ? ((j - k) << (E + 1u)) + 1u : 0u;  // b_k
  const uint32_t held = ring ? w + 1u : 0u;
  uint64_t bit = 1ull << x;  // 2^place; places from 32 on hold nothing
  for (uint32_t i = 1; i <= k && bit <= 0x80000000ull; ++i, bit <<= 1) {
    const uint32_t age = (w & ((uint32_t)bit - 1u)) | ((uint32_t)bit >> 1);
    const uint32_t a = 2u * ((held > age ? held : age) - age);  // 0 past the last one
    uint32_t b = 0xFFFFFFFFu;
    if (i < k) b = j >= k - i ? ((j - (k - i)) << (E + 1u)) + 1u : 0u;
    const uint32_t least = a < b ? a : b;
    lower = least > lower ? least : lower;
  }
  return {lower, upper};
}

}  // namespace ga
