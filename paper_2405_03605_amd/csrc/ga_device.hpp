// Device building blocks of the generation step, shared by every kernel
// family (per-generation streaming, LDS-resident tiles, asynchronous, batched):
// the counter-based RNG, the surface policy, cross-lane permutes, the torus
// geometry, coherent word accesses, and `breed`, the per-child part of a
// generation (tournament, copy, mutation, stratum deposit; paper Sec. 2).
#pragma once

#include <type_traits>

#include "ga_internal.hpp"

namespace ga {

constexpr uint32_t kMulA = 0xD2511F53u;   // Philox4x32 round multipliers
constexpr uint32_t kMulB = 0xCD9E8D57u;
constexpr uint32_t kMulAInverse = 0x991A7CDBu;  // kMulA * kMulAInverse = 1 mod 2^32
static_assert(kMulA * kMulAInverse == 1u, "inverse of the first multiplier");
constexpr uint32_t kWeylA = 0x9E3779B9u;  // key schedule increments
constexpr uint32_t kWeylB = 0xBB67AE85u;

constexpr uint32_t kStreamSelect = 0u;
constexpr uint32_t kStreamMigrate = 1u;
constexpr uint32_t kStreamSample = 2u;
constexpr uint32_t kStreamMutate = 3u;

struct Block {
  uint32_t x, y, z, w;
};

// a ^ b ^ c in one gfx950 three-input bitwise op (truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint32_t hi32(uint64_t v) { return (uint32_t)(v >> 32); }

// A copy of a wavefront-uniform value in a vector register.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t x) {
  uint32_t r;
  asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(x));
  return r;
}

// The value as it is, but opaque to the optimizer: an XOR of invariants stays
// one invariant instead of being split back over a loop's own operands.
__device__ __forceinline__ uint32_t whole(uint32_t x) {
  asm("" : "+v"(x));
  return x;
}

// (a & b) | c in one three-input bitwise op. On gfx950 the bitwise, add and
// immediate-shift ops issue in about 3 cycles a wavefront while no operand is
// a scalar register, against 4.7 with one, and 4.9 for v_and_or, v_bfi and
// shifts by a register whatever their operands (eight wavefronts per SIMD,
// nominal 2.4 GHz): the hot loops keep their constants in vector registers.
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xEA);
}

// The key of Philox round r: the run's key plus r Weyl increments. HELD keeps
// the keys of rounds 3..9 in vector registers for a kernel's lifetime (14
// registers; a round's two XORs then issue in 3 cycles each instead of 4.7);
// otherwise they are scalar sums.
template <bool HELD>
struct RoundKeys;

template <>
struct RoundKeys<false> {
  uint32_t k0, k1;
  __device__ __forceinline__ RoundKeys(uint32_t key0, uint32_t key1) : k0(key0), k1(key1) {}
  __device__ __forceinline__ uint32_t a(int r) const { return k0 + (uint32_t)r * kWeylA; }
  __device__ __forceinline__ uint32_t b(int r) const { return k1 + (uint32_t)r * kWeylB; }
};

template <>
struct RoundKeys<true> {
  uint32_t ka[7], kb[7];
  __device__ __forceinline__ RoundKeys(uint32_t key0, uint32_t key1) {
#pragma unroll
    for (int r = 0; r < 7; ++r) {
      ka[r] = in_vgpr(key0 + (uint32_t)(r + 3) * kWeylA);
      kb[r] = in_vgpr(key1 + (uint32_t)(r + 3) * kWeylB);
    }
  }
  __device__ __forceinline__ uint32_t a(int r) const { return ka[r - 3]; }
  __device__ __forceinline__ uint32_t b(int r) const { return kb[r - 3]; }
};

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11), rounds FIRST..9 applied
// to counter state (c0..c3): each round takes both halves of two 32x32->64
// products and mixes the high halves with the other two words and the round's
// key.
template <int FIRST, bool HELD>
__device__ __forceinline__ Block philox_rounds(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                               const RoundKeys<HELD>& key) {
#pragma unroll
  for (int round = FIRST; round < 10; ++round) {
    const uint64_t pa = (uint64_t)kMulA * c0;
    const uint64_t pb = (uint64_t)kMulB * c2;
    const uint32_t n0 = xor3(hi32(pb), c1, key.a(round));
    const uint32_t n2 = xor3(hi32(pa), c3, key.b(round));
    c1 = (uint32_t)pb;
    c3 = (uint32_t)pa;
    c0 = n0;
    c2 = n2;
  }
  return {c0, c1, c2, c3};
}

__device__ __forceinline__ Block philox10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                          uint32_t k0, uint32_t k1) {
  return philox_rounds<0, false>(c0, c1, c2, c3, RoundKeys<false>(k0, k1));
}

// Stream blocks for one lane across many islands. The counter is (slot,
// island, t_lo, t_hi*4 + stream): only the island word changes between a
// lane's blocks, so everything of rounds 0-2 that does not depend on it is
// computed once. The remaining per-block cost is 2 + 7*2 products and 4 + 7*2
// XORs.
struct SelectStream {
  uint32_t x0;      // round 0: c0' = x0 ^ island
  uint32_t inv_a;   // round 1: c2'' = hi(M0*c0') ^ inv_a
  uint32_t inv_b;   // round 2: c0''' = hi(M1*c2'') ^ inv_b
  uint32_t inv_c;   // round 2: c2''' = inv_c ^ lo(M0*c0')
  uint32_t inv_d;   // round 2: c3''' = inv_d

  __device__ __forceinline__ void init(uint32_t slot, uint32_t t_lo, uint32_t t_hi4, uint32_t key0,
                                       uint32_t key1, uint32_t stream) {
    // round 0 on (slot, island, t_lo, t_hi4)
    const uint64_t pa0 = (uint64_t)kMulA * slot;
    const uint64_t pb0 = (uint64_t)kMulB * t_lo;
    x0 = hi32(pb0) ^ key0;                       // c0' = hi(pb0) ^ island ^ k0
    const uint32_t c1_1 = (uint32_t)pb0;
    const uint32_t c2_1 = hi32(pa0) ^ (t_hi4 | stream) ^ key1;
    const uint32_t c3_1 = (uint32_t)pa0;
    // round 1: pb1 from c2_1 is invariant; pa1 from c0' is not
    const uint64_t pb1 = (uint64_t)kMulB * c2_1;
    const uint32_t c0_2 = hi32(pb1) ^ c1_1 ^ (key0 + kWeylA);
    const uint32_t c1_2 = (uint32_t)pb1;
    inv_a = c3_1 ^ (key1 + kWeylB);              // c2_2 = hi(pa1) ^ inv_a, c3_2 = lo(pa1)
    // round 2: pa2 from c0_2 is invariant; pb2 from c2_2 is not
    const uint64_t pa2 = (uint64_t)kMulA * c0_2;
    inv_b = c1_2 ^ (key0 + 2u * kWeylA);         // c0_3 = hi(pb2) ^ inv_b
    inv_c = hi32(pa2) ^ (key1 + 2u * kWeylB);    // c2_3 = inv_c ^ c3_2
    inv_d = (uint32_t)pa2;                       // c3_3
  }

  // The invariants as single vector registers (see whole).
  __device__ __forceinline__ void hold() {
    x0 = whole(x0);
    inv_a = whole(inv_a);
    inv_b = whole(inv_b);
    inv_c = whole(inv_c);
    inv_d = whole(inv_d);
  }

  // Round 1's product of the island word: the same for every slot and stream
  // of an island in a generation (and the island back from it: the multiplier
  // is odd, so its low word determines the counter word).
  __device__ __forceinline__ uint64_t of_island(uint32_t island) const {
    return (uint64_t)kMulA * (x0 ^ island);
  }
  __device__ __forceinline__ uint32_t island_of(uint64_t pa1) const {
    return ((uint32_t)pa1 * kMulAInverse) ^ x0;
  }

  template <bool HELD>
  __device__ __forceinline__ Block block(uint32_t island, const RoundKeys<HELD>& key) const {
    return block_from(of_island(island), key);
  }
  template <bool HELD>
  __device__ __forceinline__ Block block_from(uint64_t pa1, const RoundKeys<HELD>& key) const {
    const uint32_t c2_2 = hi32(pa1) ^ inv_a;
    const uint32_t c3_2 = (uint32_t)pa1;
    const uint64_t pb2 = (uint64_t)kMulB * c2_2;
    const uint32_t c0_3 = hi32(pb2) ^ inv_b;
    const uint32_t c1_3 = (uint32_t)pb2;
    const uint32_t c2_3 = inv_c ^ c3_2;
    return philox_rounds<3, HELD>(c0_3, c1_3, c2_3, inv_d, key);
  }
};

// One agent's genome in registers: fitness, deposit counter, surface words
// and, for a genome model with a string, its two words.
struct Genome {
  float f = 0.f;
  uint32_t T = 0, D0 = 0, D1 = 0;
  uint32_t P0 = 0, P1 = 0;
};

// What a model's mutate may use beyond the child's selection-stream block:
// the mutation probability (and the treatment law's thresholds) and, for
// draws of its own, the lane's mutation stream at the child's island.
template <bool HELD>
struct MutateArgs {
  uint32_t p32, law, p_ben, p_any;
  const SelectStream* mut;
  const RoundKeys<HELD>* key;
  uint64_t island;  // the island's product (SelectStream::of_island)
  __device__ __forceinline__ Block draw() const { return mut->block_from(island, *key); }
};

}  // namespace ga

#include "models/models.hpp"

namespace ga {

// Site written by the deposit of stratum rank r on S = 2^s sites when r >= S
// and r is a multiple of 2^e, e = bitlen(r) - s ("doubling steady" surface):
// the j-th rank written in epoch e takes over the site of rank (2j+1) << (e-1),
// which left the retained set when epoch e began. Written ranks have the form
// odd << shift, so the walk only renormalises the odd part until the rank
// falls below S.
__device__ __forceinline__ uint32_t surface_site_walk(uint32_t r, uint32_t e, uint32_t s) {
  const uint32_t half = 1u << (s - 1u);
  uint32_t odd = (((r >> e) - half) << 1) | 1u;
  uint32_t shift = e - 1u;
  for (;;) {
    const uint32_t len = 32u - __clz(odd);
    if (len + shift <= s) return odd << shift;
    const uint32_t lead = odd << (s - len);  // rank >> its epoch, in [S/2, S)
    shift = len + shift - s - 1u;
    odd = ((lead - half) << 1) | 1u;
  }
}

__device__ __forceinline__ uint32_t permute(uint32_t value, uint32_t byte_addr) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute((int)byte_addr, (int)value);
}
__device__ __forceinline__ float permute(float value, uint32_t byte_addr) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute((int)byte_addr, __float_as_int(value)));
}

// Island next to (x, y) in direction q on the W x H torus:
// 0 north (y-1), 1 east (x+1), 2 south (y+1), 3 west (x-1).
__device__ __forceinline__ void torus_xy(uint32_t x, uint32_t y, uint32_t q, uint32_t W,
                                         uint32_t H, uint32_t* nx, uint32_t* ny) {
  const uint32_t xe = (x + 1u == W) ? 0u : x + 1u;
  const uint32_t xw = (x == 0u ? W : x) - 1u;
  const uint32_t yn = (y == 0u ? H : y) - 1u;
  const uint32_t ys = (y + 1u == H) ? 0u : y + 1u;
  *nx = q == 1u ? xe : (q == 3u ? xw : x);
  *ny = q == 0u ? yn : (q == 2u ? ys : y);
}
__device__ __forceinline__ uint32_t torus_step(uint32_t x, uint32_t y, uint32_t q, uint32_t W,
                                               uint32_t H) {
  uint32_t nx, ny;
  torus_xy(x, y, q, W, H, &nx, &ny);
  return ny * W + nx;
}

template <typename P>
__device__ __forceinline__ P* at_byte(P* base, uint32_t byte_off) {
  return reinterpret_cast<P*>(reinterpret_cast<char*>(base) + byte_off);
}
template <typename P>
__device__ __forceinline__ const P* at_byte(const P* base, uint32_t byte_off) {
  return reinterpret_cast<const P*>(reinterpret_cast<const char*>(base) + byte_off);
}

// Word accesses to memory that other workgroups (on any XCD) read and write
// while this one runs: relaxed atomics at device scope. Each such access is
// coherent across the XCDs by itself (its scope bits send it past the per-XCD
// L2's non-coherent state), so ordering two of them only needs the first to
// have completed before the second issues: drain_memory() waits for every
// memory access this wavefront has in flight. A device-scope fence would do
// the same but also write back and invalidate the whole L2 of the XCD, which
// under thousands of wavefronts streaming the population costs far more than
// the exchange itself.
__device__ __forceinline__ uint32_t load_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(uint32_t* p, uint32_t value) {
  __hip_atomic_store(p, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Two words at once (8-byte aligned), for entries whose stability the
// exchange protocol already guarantees while they are read.
__device__ __forceinline__ uint2 load_agent2(const uint32_t* p) {
  const uint64_t x = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  return make_uint2((uint32_t)x, (uint32_t)(x >> 32));
}
__device__ __forceinline__ void store_agent2(uint32_t* p, uint32_t lo, uint32_t hi) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), ((uint64_t)hi << 32) | lo, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void drain_memory() {
  // also a compiler barrier: no memory access moves across it
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// A kernel's dynamic LDS by byte offset (it starts at 0: no kernel that uses
// these has any other).
template <typename T>
__device__ __forceinline__ T lds_get(uint32_t byte) {
  return *(__attribute__((address_space(3))) T*)byte;
}
template <typename T>
__device__ __forceinline__ void lds_put(uint32_t byte, T x) {
  *(__attribute__((address_space(3))) T*)byte = x;
}
// Keeps the compiler from moving memory accesses across it (the LDS executes a
// wavefront's accesses in order by itself).
__device__ __forceinline__ void keep_order() { asm volatile("" ::: "memory"); }

// The dispatcher hands workgroups to the eight XCDs in turn (group g to XCD
// g mod 8), each XCD with its own L2. Renumbering the groups so that every XCD
// takes one contiguous band of the grid keeps an island's four neighbours, and
// the outbox entries it reads from them, mostly on its own XCD.
// The renumbering of groups g < n (a permutation of [0, n)), for grids whose
// first n groups are the ones with work.
__device__ __forceinline__ uint32_t xcd_band(uint32_t g, uint32_t n) {
  const uint32_t x = g & 7u, q = n >> 3, r = n & 7u;
  return (x < r ? x * (q + 1u) : r * (q + 1u) + (x - r) * q) + (g >> 3);
}
__device__ __forceinline__ uint32_t xcd_band_group() { return xcd_band(blockIdx.x, gridDim.x); }

// Per-lane constants of one generation's children: the lane's slot in its
// island, the address its island's members are found at (see the parent
// accessors below), and the selection (and, under the treatment law, mutation)
// stream with everything hoisted that depends only on the slot and the
// generation.
struct BreedLane {
  uint32_t slot;
  uint32_t base;       // address of the island's slot 0
  uint32_t slot_mask;  // (N - 1) * 4: a draw's bits that pick a slot, in place
  uint32_t t_lo, t_hi4;
  SelectStream sel, mut;
  // the mutation thresholds, compared lane by lane: held in vector registers
  // so that the loops do not keep (or reload) them in scalar ones
  uint32_t p32, p_ben, p_any;
};

template <int LC>
__device__ __forceinline__ BreedLane breed_lane(const RunView& v, uint64_t t) {
  const uint32_t L = LC >= 0 ? (uint32_t)LC : v.log2n;
  const uint32_t lane = __lane_id();
  BreedLane b;
  b.slot = lane & ((1u << L) - 1u);
  b.base = (lane & ~((1u << L) - 1u)) << 2;
  b.slot_mask = in_vgpr(((1u << L) - 1u) << 2);
  b.t_lo = (uint32_t)t;
  b.t_hi4 = (uint32_t)(t >> 32) << 2;
  b.sel.init(b.slot, b.t_lo, b.t_hi4, v.seed, v.run_id, kStreamSelect);
  if (v.law) b.mut.init(b.slot, b.t_lo, b.t_hi4, v.seed, v.run_id, kStreamMutate);
  b.p32 = in_vgpr(v.p32);
  b.p_ben = in_vgpr(v.p_ben);
  b.p_any = in_vgpr(v.p_any);
  return b;
}

// Where a tournament finds the members of the lane's island. The address of a
// member is its island's base | slot * 4, the slot taken from byte m of the
// draw without leaving its place: ((word >> s) & slot_mask) | base.

// Members in the registers of this wavefront's lanes (cross-lane permutes;
// every lane must take part).
template <int SW, bool STR>
struct LaneParents {
  const Genome& g;
  __device__ __forceinline__ float fitness(uint32_t at) const { return permute(g.f, at); }
  __device__ __forceinline__ void copy(Genome& c, uint32_t at) const {
    c.T = permute(g.T, at);
    c.D0 = permute(g.D0, at);
    c.D1 = SW > 1 ? permute(g.D1, at) : 0u;
    if (STR) {
      c.P0 = permute(g.P0, at);
      c.P1 = permute(g.P1, at);
    }
  }
};

// The steady policy's deposit of rank q on 2^s sites writes iff q has no set
// bit below its top s bits (every rank below 2^s; after that the multiples of
// 2^e, e = bitlen(q) - s). May: three ops, true for every rank that writes and
// (rounded to binary32) for a few from 2^24 on that do not; writes: exact.
__device__ __forceinline__ bool steady_may_write(uint32_t q, uint32_t s) {
  return (__float_as_uint((float)q) & ((1u << (24u - s)) - 1u)) == 0u;
}
__device__ __forceinline__ bool steady_writes(uint32_t q, uint32_t s) {
  const uint32_t len = 32u - __clz(q);
  return len <= s || (q & ((1u << (len - s)) - 1u)) == 0u;
}

// Steps 3-7 of generation t for the child in this lane's slot of `island`
// (paper Sec. 2): evaluation (the fitness word), a tournament of k entrants
// drawn with replacement from the lane's island (first strict maximum in draw
// order wins; neutral runs take entrant 0), the winner's genome copied from
// `parents`, the model's mutation, and one stratum deposit at rank T followed
// by T + 1. `island` is its product in the lane's streams (of_island), `r` the
// child's selection block.
// LC / SWC: log2 N and surface words fixed at compile time, or -1 to read
// them from the view.
// PLAIN: a tournament of two under the discrete mutation law, the common run,
// known at compile time.
template <int LC, int SWC, typename Model, bool WIDE, bool PLAIN, bool HELD, typename Parents>
__device__ __forceinline__ Genome breed(const RunView& v, const BreedLane& b,
                                        const Parents& parents, const Block& r, uint64_t island,
                                        const RoundKeys<HELD>& key) {
  const uint32_t L = LC >= 0 ? (uint32_t)LC : v.log2n;
  const uint32_t SW = SWC >= 0 ? (uint32_t)SWC : v.words;
  // surface: S = 2^s_log sites of 2^dlog-bit differentia under the steady
  // policy; one bit on 32 or 64 sites is fixed at compile time, WIDE reads
  // the width, the site count and the policy from the view
  const uint32_t dlog = WIDE ? v.dlog : 0u;
  const bool tilted = WIDE && v.policy == 1u;
  const bool hybrid = WIDE && v.policy == 2u;
  const uint32_t s_log = WIDE ? v.s_log : 4u + SW;

  // 3-5. evaluate (read fitness) and run the tournament: entrant m takes byte
  // m of (w0, w1), little-endian. Entrant 1 is taken apart (k = 2 is the
  // common size); beyond it entrants go in pairs, all of a pair's members
  // fetched before any is compared, an odd last one left out of the
  // comparison. The conditions are uniform.
  auto entrant = [&](uint32_t word, uint32_t byte) {
    return and_or(word >> (8u * byte + 6u - L), b.slot_mask, b.base);
  };
  uint32_t best = entrant(r.x, 0);
  float fbest = parents.fitness(best);
  const uint32_t k = PLAIN ? 2u : v.selection ? v.k : 1u;
  auto meet = [&](uint32_t at, float f, bool in) {
    const bool wins = in && f > fbest;
    best = wins ? at : best;
    fbest = wins ? f : fbest;
  };
  if (k > 1u) {
    const uint32_t a1 = entrant(r.x, 1);
    const float f1 = parents.fitness(a1);
    if (k > 2u) {
      const uint32_t a2 = entrant(r.x, 2), a3 = entrant(r.x, 3);
      const float f2 = parents.fitness(a2), f3 = parents.fitness(a3);
      if (k > 4u) {
        const uint32_t a4 = entrant(r.y, 0), a5 = entrant(r.y, 1);
        const float f4 = parents.fitness(a4), f5 = parents.fitness(a5);
        meet(a1, f1, true);
        meet(a2, f2, true);
        meet(a3, f3, true);
        meet(a4, f4, true);
        meet(a5, f5, k > 5u);
        if (k > 6u) {
          const uint32_t a6 = entrant(r.y, 2), a7 = entrant(r.y, 3);
          const float f6 = parents.fitness(a6), f7 = parents.fitness(a7);
          meet(a6, f6, true);
          meet(a7, f7, k > 7u);
        }
      } else {
        meet(a1, f1, true);
        meet(a2, f2, true);
        meet(a3, f3, k > 3u);
      }
    } else {
      meet(a1, f1, true);
    }
  }
  Genome c;
  parents.copy(c, best);
  c.f = fbest;

  // 6. mutation, by the genome model
  MutateArgs<HELD> ma{b.p32, PLAIN ? 0u : v.law, b.p_ben, b.p_any, &b.mut, &key, island};
  Model::mutate(c, r, ma);

  // 7. stratum deposit at rank T, then T + 1. The hybrid policy sends even
  //    ranks 2q to a 32-site steady half (sites 0..31) and odd ranks 2q + 1
  //    to a 32-site tilted half (sites 32..63), each as its rank q.
  uint32_t q = c.T, q_log = s_log, site_base = 0u;
  bool on_tilted = tilted;
  if (hybrid) {
    q = c.T >> 1;
    q_log = 5u;
    on_tilted = (c.T & 1u) != 0u;
    site_base = on_tilted ? 32u : 0u;
  }
  if (on_tilted || steady_may_write(q, q_log)) {
    uint32_t site = q;
    bool write = true;
    if (on_tilted) {
      // level k = trailing zeros of q (capped at 31; q = 0 counts as 31), slot
      // (q >> (k+1)) mod m ((q >> 31) mod m on level 31), m = sites / 32
      const uint32_t m_log = q_log - 5u;
      const uint32_t lev = q ? min((uint32_t)__ffs(q) - 1u, 31u) : 31u;
      const uint32_t ring = (lev < 31u ? q >> (lev + 1u) : q >> 31) & ((1u << m_log) - 1u);
      site = (lev << m_log) + ring;
    } else if (q >= (1u << q_log)) {
      write = steady_writes(q, q_log);
      if (write) site = surface_site_walk(q, (32u - __clz(q)) - q_log, q_log);
    }
    site += site_base;
    // the differentia: one bit, the top bit of the selection block's w3;
    // b = 2^dlog > 1 bits, the top b bits of word 0 of a block of their own
    // (mutation stream, counter word 0 = slot + 256), drawn only by the
    // lanes that write
    const uint32_t pos = site << dlog;
    uint32_t value = (uint32_t)((int32_t)r.w >> 31);  // the bit, in every place
    uint32_t field = 1u << (pos & 31u);
    if (WIDE && dlog != 0u) {
      value = philox10(b.slot + 256u, b.sel.island_of(island), b.t_lo, b.t_hi4 | kStreamMutate,
                       v.seed, v.run_id).x >>
              (32u - (1u << dlog)) << (pos & 31u);
      field = ((2u << ((1u << dlog) - 1u)) - 1u) << (pos & 31u);
    }
    field = write ? field : 0u;
    if (SW == 1 || pos < 32u) {
      c.D0 = (c.D0 & ~field) | (value & field);
    } else {
      c.D1 = (c.D1 & ~field) | (value & field);
    }
  }
  c.T += 1u;
  return c;
}

// ---------------------------------------------------------------------------
// Host-side dispatch to a kernel's compile-time shape.
// ---------------------------------------------------------------------------
template <int V>
using IntC = std::integral_constant<int, V>;
template <bool V>
using BoolC = std::integral_constant<bool, V>;

template <typename M, bool WD, typename F>
hipError_t dispatch_shapes(uint32_t L, uint32_t SW, F& f) {
  switch (L * 2u + (SW - 1u)) {
    case 0: return f(IntC<0>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 1: return f(IntC<0>{}, IntC<2>{}, M{}, BoolC<WD>{});
    case 2: return f(IntC<1>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 3: return f(IntC<1>{}, IntC<2>{}, M{}, BoolC<WD>{});
    case 4: return f(IntC<2>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 5: return f(IntC<2>{}, IntC<2>{}, M{}, BoolC<WD>{});
    case 6: return f(IntC<3>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 7: return f(IntC<3>{}, IntC<2>{}, M{}, BoolC<WD>{});
    case 8: return f(IntC<4>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 9: return f(IntC<4>{}, IntC<2>{}, M{}, BoolC<WD>{});
    case 10: return f(IntC<5>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 11: return f(IntC<5>{}, IntC<2>{}, M{}, BoolC<WD>{});
    case 12: return f(IntC<6>{}, IntC<1>{}, M{}, BoolC<WD>{});
    case 13: return f(IntC<6>{}, IntC<2>{}, M{}, BoolC<WD>{});
    default: return hipErrorInvalidValue;
  }
}

// Calls f(IntC<log2 N>, IntC<surface words>, Model, BoolC<wide differentia
// or another policy>) for the run's shape; f returns a hipError_t. Every
// kernel family is instantiated for every model of GA_FOR_EACH_MODEL.
template <typename F>
hipError_t dispatch(const RunView& v, F&& f) {
  const bool wide = v.dlog != 0u || v.policy != 0u;
#define GA_MODEL_CASE(ID, M)                                                   \
  case ID:                                                                     \
    return wide ? dispatch_shapes<M, true>(v.log2n, v.words, f)                \
                : dispatch_shapes<M, false>(v.log2n, v.words, f);
  switch (v.model) {
    GA_FOR_EACH_MODEL(GA_MODEL_CASE)
    default: return hipErrorInvalidValue;
  }
#undef GA_MODEL_CASE
}

// The template arguments of a kernel from dispatch's tag arguments
#define GA_SHAPE_ARGS(LC, SWC, M, WD) \
  decltype(LC)::value, decltype(SWC)::value, decltype(M), decltype(WD)::value

}  // namespace ga
