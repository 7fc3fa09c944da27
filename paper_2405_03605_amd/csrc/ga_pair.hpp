// Two generations of the streaming form in one launch, the population through
// HBM once for both.
//
// A wavefront takes a chunk of 16 islands (at most 512 agents, 256 of the larger
// genomes) into LDS, runs
// generations t and t + 1 there and writes the chunk back. Within a generation
// islands depend on each other only through the emissions of the one before,
// so what the second generation needs from outside the chunk is its neighbours'
// emissions of t, and an emission is fixed before anything of its generation
// is bred: it is the member in the drawn slot, unless an arrival of t took
// that slot. So beside the outbox entries (emissions of t - 1) every island
// leaves its candidate for t, the member its draw of t picks as it is before
// immigration, with that draw; a neighbour then has the island's emission
// without a draw of its own: the candidate or, where the drawn slots say that
// an arrival may have replaced it (one in eight of those sent, at 32 members),
// what the outbox entries of the island's own neighbours say. Results are those
// of the single-generation kernel.
//
// A launch reads the outbox plane and the candidate plane its predecessor
// wrote and writes the other ones (other wavefronts still read the first), so
// two launches, four generations, bring the outbox back to the plane a
// single-generation launch expects; the host runs them in fours.
//
// Bound: the matrix cores have nothing to do here; HBM (26 bytes per agent a
// launch, 5.9 of the 7.2 TB/s an in-place update reaches) and VALU (77
// instructions per 64 children, 59 of them in the loop; 0.89 of the issue slots)
// together. 1024 x 512 x 32, k = 2: 37 us per generation (74 a launch) against
// 62 for the single-generation kernel; 300 x 200 x 64 trap-4 on the hybrid
// surface, k = 3: 18.7 against 34.2; it is ahead at every
// grid and island size from four members up (16 x 16 x 32: 1.8 against 3.2,
// 4096 x 1024 x 32: 326 against 645). What made it so: arrivals and draws kept
// in registers, four lanes an island, so that LDS holds 24 wavefronts a CU
// instead of 18, and the neighbours' draws read, not drawn (43 -> 37 us);
// workgroups of one wavefront (43.8 at four). Full chunks: 8 islands 42 us,
// 4 islands 56. Unrolling the loop four times left it where it was; a register
// cap for more wavefronts per SIMD where both loops share a kernel spills (43).
#pragma once

#include "ga_device.hpp"

namespace ga {

// Members in the chunk's planes: `at` is the byte offset of the fitness word.
template <int SW, bool STR, uint32_t PLANE>
struct ChunkParents {
  __device__ __forceinline__ float fitness(uint32_t at) const { return lds_get<float>(at); }
  __device__ __forceinline__ void copy(Genome& c, uint32_t at) const {
    c.T = lds_get<uint32_t>(at + PLANE);
    c.D0 = lds_get<uint32_t>(at + 2u * PLANE);
    c.D1 = SW > 1 ? lds_get<uint32_t>(at + 3u * PLANE) : 0u;
    if (STR) {
      c.P0 = lds_get<uint32_t>(at + (2u + SW) * PLANE);
      c.P1 = lds_get<uint32_t>(at + (3u + SW) * PLANE);
    }
  }
  __device__ __forceinline__ void put(const Genome& c, uint32_t at) const {
    lds_put(at, c.f);
    lds_put(at + PLANE, c.T);
    lds_put(at + 2u * PLANE, c.D0);
    if (SW > 1) lds_put(at + 3u * PLANE, c.D1);
    if (STR) {
      lds_put(at + (2u + SW) * PLANE, c.P0);
      lds_put(at + (3u + SW) * PLANE, c.P1);
    }
  }
};

// The word of an outbox or candidate entry that genome word k sits in (with a
// string an entry always has two surface words).
template <int SW, bool STR>
__device__ __forceinline__ uint32_t entry_word(uint32_t k) {
  return STR && SW == 1 && k >= 3u ? k + 1u : k;
}

// A tournament of two under the discrete mutation law (what breed's PLAIN is).
__host__ __device__ __forceinline__ bool is_plain(const RunView& v) {
  return v.k == 2u && v.selection && !v.law;
}

// A lane's value handed to the other lanes of its group of four: lane FROM's.
template <int FROM>
__device__ __forceinline__ uint32_t from_quad(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, FROM * 0x55, 0xF, 0xF, true);
}

// An island's migration draw in the word after its candidate's genome: byte d
// holds the slot for the arrival from d in its top six bits, where the draw has
// it (islands have at most 64 members); the low two bits of byte k are bits 2k
// and 2k + 1 of direction (top two) and emigrant slot.
__device__ __forceinline__ uint32_t pack_draw(uint32_t x, uint32_t y, uint32_t z) {
  const uint32_t e = (y >> 30 << 6) | (x >> 26);
  uint32_t s = (e | (e << 12)) & 0x000F000Fu;
  s = (s | (s << 6)) & 0x03030303u;
  return (z & 0xFCFCFCFCu) | s;
}
// Direction in the top two bits, the emigrant slot in the six below.
__device__ __forceinline__ uint32_t unpack_sent(uint32_t w) {
  return (w & 0x03030303u) * ((1u << 24) + (1u << 18) + (1u << 12) + (1u << 6));
}

// Generations t and t + 1 of islands [base, base + v.ipw) by one wavefront
// whose LDS starts at 0. `plane`: the outbox plane that holds the emissions of
// t - 1 (those of t + 1 go to the other one); the candidates of t are in the
// plane of t's second bit.
template <int LC, int SWC, typename Model, bool WIDE, bool PLAIN>
__device__ __forceinline__ void chunk_pair(const RunView& v, uint32_t base, uint64_t t,
                                           uint32_t plane) {
  constexpr uint32_t L = (uint32_t)LC;
  constexpr uint32_t SW = (uint32_t)SWC;
  constexpr bool kStr = Model::kString;
  constexpr uint32_t kw = pair_words(SW, kStr);
  constexpr uint32_t kAgents = pair_agents(L, kw), kPlane = pair_plane(L, kw);
  constexpr uint32_t obs = (SW == 1 && !kStr) ? 4u : 8u;
  constexpr uint32_t ob_hdr = kStr ? 6u : 2u + SW;
  const uint32_t lane = __lane_id(), q = lane & 3u, li = lane >> 2;
  const uint32_t W = v.width, H = v.height;
  const uint32_t n_iter = v.ipw >> (6u - L);
  const uint32_t prod = kw * kPlane;
  const uint32_t* in_ob = plane ? v.ob[1] : v.ob[0];
  uint32_t* out_ob = plane ? v.ob[0] : v.ob[1];
  const size_t cand_plane = (size_t)v.island_stride * obs;
  const bool odd = (t & 2u) != 0u;
  // without migration there are no candidates and nobody sends
  const uint32_t* in_cand = v.migration ? v.cand + (odd ? cand_plane : 0u) : in_ob;
  uint32_t* out_cand = v.cand + (odd ? 0u : cand_plane);
  const ChunkParents<SWC, kStr, kPlane> pop;
  typedef uint32_t Quad __attribute__((ext_vector_type(4)));

  // ---- what comes from other islands on its way, lane (island, direction) ------
  const bool ok = li < v.ipw && base + li < v.islands;
  const uint32_t bx = base % W, by = base / W;
  uint32_t x = bx + (ok ? li : 0u), y = by;
  if (W >= kAgents >> L) {
    y += x >= W ? 1u : 0u;
    x -= x >= W ? W : 0u;
  } else {
    y += x / W;
    x = x % W;
  }
  uint32_t nx, ny;
  torus_xy(x, y, q, W, H, &nx, &ny);
  const uint32_t nb = ny * W + nx;
  uint32_t a0[8], a1[8];  // the neighbour's outbox entry and its candidate
  auto load = [](uint32_t (&to)[8], const uint32_t* from) __attribute__((always_inline)) {
#pragma unroll
    for (uint32_t k = 0; k < obs; k += 4) {
      const Quad w4 = *reinterpret_cast<const Quad*>(from + k);
      to[k] = w4.x;
      to[k + 1] = w4.y;
      to[k + 2] = w4.z;
      to[k + 3] = w4.w;
    }
  };
  load(a0, in_ob + (size_t)nb * obs);
  load(a1, in_cand + (size_t)nb * obs);

  // ---- and the chunk's population on its way into LDS, 16 bytes a lane ----------
  // (all of a full chunk: what a shorter one reads too much is not written back)
  const size_t first_agent = (size_t)base << L;
  auto plane_of = [&](uint32_t k) __attribute__((always_inline)) -> uint32_t* {
    return k == 0u ? reinterpret_cast<uint32_t*>(v.pop_f)
           : k == 1u ? v.pop_T
           : k < 2u + SW ? v.pop_D + (k - 2u) * (size_t)v.agent_stride
                         : v.pop_P + (k - 2u - SW) * (size_t)v.agent_stride;
  };
  if (kAgents >= 256u || 4u * lane < kAgents)
#pragma unroll
    for (uint32_t k = 0; k < kw; ++k)
#pragma unroll
      for (uint32_t h = 0; h < kAgents; h += 256u)
        __builtin_amdgcn_global_load_lds(
            (__attribute__((address_space(1))) void*)(plane_of(k) + first_agent + h + 4u * lane),
            (__attribute__((address_space(3))) void*)(k * kPlane + 4u * h), 16, 0, 0);

  // ---- the island's draws: lanes 0, 1, 2 of its four that of t, t + 1, t + 2 -----
  const RoundKeys<true> key(v.seed, v.run_id);
  const uint32_t slot_mask = in_vgpr(((1u << L) - 1u) << 2);
  const uint64_t tq = t + (q < 2u ? q : 2u);
  SelectStream later;
  later.init(0u, (uint32_t)tq, (uint32_t)(tq >> 32) << 2, v.seed, v.run_id, kStreamMigrate);
  const Block mine = later.block(y * W + x, key);
  const uint32_t home = 4u * (li << L);
  const uint32_t q_shift = 8u * q + 6u - L;  // byte q of a draw, as a slot in place
  uint32_t at = and_or(from_quad<0>(mine.z) >> q_shift, slot_mask, home);
  uint32_t at1 = and_or(from_quad<1>(mine.z) >> q_shift, slot_mask, home);
  // the member this island sends at t + 1 and its candidate for t + 2, as places
  // of this lane's word
  const uint32_t em1 =
      and_or(from_quad<1>(mine.x) >> (30u - L), slot_mask, home) + q * kPlane;
  const uint32_t hdr1 = v.migration ? kMetaValid | (from_quad<1>(mine.y) >> 30) : 0u;
  const uint32_t em2 =
      and_or(from_quad<2>(mine.x) >> (30u - L), slot_mask, home) + q * kPlane;
  const uint32_t draw2 = from_quad<2>(pack_draw(mine.x, mine.y, mine.z));

  // ---- the neighbour's emission of t: its candidate, or the last arrival drawn
  // into that slot --------------------------------------------------------------
  const uint32_t sent_to = unpack_sent(a1[ob_hdr]);
  const bool sent = ok && v.migration && (sent_to >> 30) == (q ^ 2u);
  const uint32_t emig = (sent_to >> (28u - L)) & slot_mask;
  uint32_t maybe = 0u;  // bit d: the neighbour's arrival from d draws that slot
#pragma unroll
  for (uint32_t d = 0; d < 4; ++d)
    maybe |= ((a1[ob_hdr] >> (8u * d + 6u - L)) & slot_mask) == emig ? 1u << d : 0u;
  maybe = sent ? maybe : 0u;
  while (__builtin_amdgcn_ballot_w64(maybe != 0u) != 0ull) {
    if (maybe) {
      const uint32_t d = 31u - __clz(maybe);
      uint32_t a2[8];
      load(a2, in_ob + (size_t)torus_step(nx, ny, d, W, H) * obs);
      const bool hit = a2[ob_hdr] == (kMetaValid | (d ^ 2u));
#pragma unroll
      for (uint32_t k = 0; k < kw; ++k) {
        const uint32_t w = entry_word<SWC, kStr>(k);
        a1[w] = hit ? a2[w] : a1[w];
      }
      maybe = hit ? 0u : maybe & ~(1u << d);
    }
  }
  at = ok && a0[ob_hdr] == (kMetaValid | (q ^ 2u)) ? at : kDiscard;
  at1 = sent ? at1 : kDiscard;
  auto genome = [](const uint32_t (&a)[8]) __attribute__((always_inline)) {
    Genome e;
    e.f = __uint_as_float(a[0]);
    e.T = a[1];
    e.D0 = a[2];
    e.D1 = SW > 1 ? a[3] : 0u;
    if (kStr) {
      e.P0 = a[4];
      e.P1 = a[5];
    }
    return e;
  };
  Genome arrival = genome(a0);
  const Genome arrival1 = genome(a1);

  drain_memory();  // the population is in LDS
  BreedLane bl = breed_lane<LC>(v, t);
  const uint32_t group = bl.base;
#pragma unroll 1
  for (uint32_t g = 0; g < 2u; ++g) {
    const uint64_t tg = t + g;
    bl.t_lo = (uint32_t)tg;
    bl.t_hi4 = (uint32_t)(tg >> 32) << 2;
    bl.sel.init(bl.slot, bl.t_lo, bl.t_hi4, v.seed, v.run_id, kStreamSelect);
    bl.sel.hold();
    if (v.law) bl.mut.init(bl.slot, bl.t_lo, bl.t_hi4, v.seed, v.run_id, kStreamMutate);
    // arrivals into their drawn slots, one direction after the other, so the
    // last to draw a slot keeps it; the islands' products
    keep_order();
#pragma unroll
    for (uint32_t d = 0; d < 4; ++d) {
      if (at != kDiscard && q == d) pop.put(arrival, at);
      keep_order();
    }
    if (q == 0u) lds_put(prod + 8u * li, bl.sel.of_island(base + li));
    if (g == 1u && ok) {
      // this island's emission of t + 1, a word or two a lane
      uint32_t* o = out_ob + (size_t)(base + li) * obs;
      if (q < kw) o[entry_word<SWC, kStr>(q)] = lds_get<uint32_t>(em1);
      if (kw > 4u && q + 4u < kw)
        o[entry_word<SWC, kStr>(q + 4u)] = lds_get<uint32_t>(em1 + 4u * kPlane);
      if (q == 3u) o[ob_hdr] = hdr1;
    }
    keep_order();
    uint32_t next = prod + 8u * (lane >> L);
    uint64_t island = lds_get<uint64_t>(next);
    bl.base = group;
#pragma unroll 1
    for (uint32_t it = 0; it < n_iter; ++it) {
      next += 512u >> L;  // read ahead; the table has one iteration's room more
      const uint64_t next_island = lds_get<uint64_t>(next);
      const Block r = bl.sel.block_from(island, key);
      const Genome cld = breed<LC, SWC, Model, WIDE, PLAIN>(v, bl, pop, r, island, key);
      pop.put(cld, bl.base + 4u * bl.slot);
      bl.base += 256u;
      island = next_island;
    }
    arrival = arrival1;
    at = at1;
  }

  // ---- the chunk back, 16 bytes a lane, and the candidates of t + 2 ---------------
  keep_order();
  const uint32_t chunk = n_iter << 6;  // agents
#pragma unroll
  for (uint32_t h = 0; h < kAgents; h += 256u)
    if (h + 4u * lane < chunk)
#pragma unroll
      for (uint32_t k = 0; k < kw; ++k)
        *reinterpret_cast<Quad*>(plane_of(k) + first_agent + h + 4u * lane) =
            lds_get<Quad>(k * kPlane + 4u * h + 16u * lane);
  if (v.migration && ok) {
    uint32_t* o = out_cand + (size_t)(base + li) * obs;
    if (q < kw) o[entry_word<SWC, kStr>(q)] = lds_get<uint32_t>(em2);
    if (kw > 4u && q + 4u < kw)
      o[entry_word<SWC, kStr>(q + 4u)] = lds_get<uint32_t>(em2 + 4u * kPlane);
    if (q == 3u) o[ob_hdr] = draw2;
  }
}

// The candidates of generation t of an island from its population as it is.
__device__ __forceinline__ void leave_candidate(const RunView& v, uint32_t i, uint64_t t) {
  const Block b = philox10(0u, i, (uint32_t)t, ((uint32_t)(t >> 32) << 2) | kStreamMigrate, v.seed,
                           v.run_id);
  const bool strings = model_has_string(v.model);
  const size_t a = ((size_t)i << v.log2n) + (v.log2n ? b.x >> (32u - v.log2n) : 0u);
  uint32_t* o = v.cand + ((t & 2u) ? (size_t)v.island_stride * v.ob_stride : 0u) +
                (size_t)i * v.ob_stride;
  o[0] = reinterpret_cast<const uint32_t*>(v.pop_f)[a];
  o[1] = v.pop_T[a];
  for (uint32_t w = 0; w < v.words; ++w) o[2u + w] = v.pop_D[w * (size_t)v.agent_stride + a];
  if (strings)
    for (uint32_t w = 0; w < 2u; ++w) o[4u + w] = v.pop_P[w * (size_t)v.agent_stride + a];
  o[strings ? 6u : 2u + v.words] = pack_draw(b.x, b.y, b.z);
}

}  // namespace ga
