// LDS-resident persistent form of the synchronous generation step.
//
// The torus is cut into tiles of tile_w x tile_h islands (ragged at the right
// and bottom edges); one workgroup owns one tile for the whole launch and keeps
// its population in LDS across generations, the way each processing element
// of the paper's wafer-scale design keeps its island in local memory (Sec. 2
// Methods). HBM then carries the population once at the start and once at the
// end of a launch, and in between only the emissions of the islands on a
// tile's edge (one entry each per generation).
//
// Each wavefront owns a fixed share of the tile's islands (a contiguous run of
// whole 64-agent iterations) and takes them from one generation to the next by
// itself. Generation t of a wavefront, with the same results as the
// per-generation streaming kernel (and the oracle):
//   island pass   four lanes per island, one per direction: the migration draw;
//                 the neighbour's emission of generation t-1 (from the LDS
//                 outbox, or from the exchange area in HBM for a neighbour in
//                 another tile); arrivals written into their drawn slots of
//                 the LDS population, later directions over earlier ones; the
//                 drawn emigrant (post-immigration) copied to the LDS outbox of
//                 parity t&1 and, for an island on the tile's edge, to the
//                 exchange area;
//   iterations    lanes are agent slots, 64/N islands per iteration:
//                 tournament, copy, mutation and deposit (`breed`), the
//                 entrants' fitness and the winner's genome gathered straight
//                 from the island's planes in LDS, children written in place.
// The only order between wavefronts is that a pass of generation t+1 follows
// every wavefront's pass of generation t: each arrives on an LDS counter after
// its pass and waits on the counter before its next one, a whole set of
// iterations later, so the wait is normally already met and no wavefront idles
// at a barrier. (DS operations of a wavefront execute in order, so its outbox
// writes are in LDS before its arrival, and another wavefront's reads after
// it has seen the arrival.)
//
// Exchange between tiles. An edge island's emission of generation t goes to its
// slot of parity t&1 in the exchange area, one 64-bit word per genome word: the
// word below, and above it the generation (31 bits) and one bit of the
// direction. 64-bit accesses are single, so a reader that finds generation t in
// each word has the whole entry: no flag, no drain, no order between the words,
// and one memory round trip between a store and the neighbour's use of it,
// which the iterations hide (the reader's first try goes out halfway through
// them). A slot is overwritten two generations later, after its owner has
// read the emission of t+1 of every neighbour outside its tile, which each of
// them sends only after reading the slot. The same order keeps a tile that is
// done from writing its last emissions over the pending ones of the HBM outbox
// that a neighbour has yet to read (the same plane after an even number of
// generations); without migration nothing is sent, and the host runs an odd
// number of generations a launch.
//
// Every tile's workgroup must be resident at once (the host sizes the tiling
// by the occupancy query); each wait on another tile is bounded, and a wait
// that gave up is counted, which the host reports as an error when the state
// is read.
//
// Bound: VALU issue (256 x 256 x 32 on 32 x 8 tiles: 2,390 vector instructions
// per SIMD and generation in 10,800 cycles), so what is not Philox is kept
// short: parents are gathered from planes by address (no permutes, no arrival
// test, no record read and write: 4.3 cycles a gather against 7.3 a permute),
// constants sit in vector registers (see and_or in ga_device.hpp), and a
// pass's Philox block, an island's direction and a genome's word share the
// same lanes. The rotating priority below keeps a SIMD's wavefronts together:
// served oldest first they finished one after the other, the last alone on its
// SIMD at one instruction in nine cycles. Measured, microseconds per
// generation, against the form before (16-byte records, one thread per island
// in a pass between two workgroup barriers, per-tile progress words):
// 256 x 256 x 32 6.0 to 4.4 (5.2 with the hardware's priority; 4.6 where waiting
// wavefronts retry without a pause), 100 x 100 x 32 treatments 5.4 to 2.8, 37 x 23 x
// 16 k = 5 3.9 to 1.6 (2.2 on tiles of 2,048 agents), 8 x 8 x 32 2.6 to 1.7.
#include <algorithm>

#include "ga_device.hpp"

namespace ga {
namespace {

// LDS words of a tile: the population in blocks of 64 agents (an iteration),
// each block one plane of 64 words per genome word (fitness, T, surface words,
// string words), so that a block's planes are reached from one address with
// constant offsets and 64 lanes' reads of a plane meet no bank twice; the
// islands' products (SelectStream::of_island) of the current generation; the
// outbox for both parities (TI entries of ob_stride words each); the halo, one
// such entry for each pair of an edge island and a direction out of the tile
// (at most 2 (tile_w + tile_h)), and the island each comes from; a counter of
// pairs given out and the arrival counter.
__host__ __device__ inline uint32_t tile_agents_padded(uint32_t ti_full, uint32_t log2n) {
  return ((ti_full << log2n) + 63u) & ~63u;
}
__host__ __device__ inline uint32_t tile_agent_words(uint32_t words, bool strings) {
  return 2u + words + (strings ? 2u : 0u);
}
// The product table, two words an island, padded so that what follows stays
// 16-byte aligned. The iterations read one block ahead: past the last block that
// ends in the outbox and halo behind the table (tile_lds_bytes has room for it
// where those are shorter: a few islands of one or two agents).
__host__ __device__ inline uint32_t tile_table_words(uint32_t ta, uint32_t log2n) {
  return (2u * (ta >> log2n) + 3u) & ~3u;
}

typedef uint32_t Quad __attribute__((ext_vector_type(4)));

// Members in LDS: `at` is the byte offset of the member's fitness.
template <int SW, bool STR>
struct TileParents {
  __device__ __forceinline__ float fitness(uint32_t at) const { return lds_get<float>(at); }
  __device__ __forceinline__ void copy(Genome& c, uint32_t at) const {
    c.T = lds_get<uint32_t>(at + 256u);
    c.D0 = lds_get<uint32_t>(at + 512u);
    c.D1 = SW > 1 ? lds_get<uint32_t>(at + 768u) : 0u;
    if (STR) {
      c.P0 = lds_get<uint32_t>(at + 256u * (2u + SW));
      c.P1 = lds_get<uint32_t>(at + 256u * (3u + SW));
    }
  }
  __device__ __forceinline__ Genome get(uint32_t at) const {
    Genome c;
    copy(c, at);
    c.f = fitness(at);
    return c;
  }
  __device__ __forceinline__ void put(const Genome& c, uint32_t at) const {
    lds_put(at, c.f);
    lds_put(at + 256u, c.T);
    lds_put(at + 512u, c.D0);
    if (SW > 1) lds_put(at + 768u, c.D1);
    if (STR) {
      lds_put(at + 256u * (2u + SW), c.P0);
      lds_put(at + 256u * (3u + SW), c.P1);
    }
  }
};

// A pass's lane: island li of the tile (id `island`), direction q = lane & 3,
// which is also the genome word the lane sends on. LDS byte offsets: `home`,
// the island's slot 0; `in`, the neighbour's entry of generation t - 1 (in the
// outbox, or in the halo for one outside the tile); `out`, this lane's word of
// the island's outbox entry of t. `to`: the byte offset of this lane's word of
// the island's exchange slot of t; `prod`, the island's product. out and to change parity with every
// generation, and in by `step` (0 in the halo).
struct PassLane {
  uint32_t island, home, in, step, out, to, prod;
  bool ok, edge;  // edge: one of the island's neighbours is outside
};

// DENSE: held to the registers of six wavefronts per SIMD (five with more than
// one surface word or a string, seven for islands of one agent), for tilings of
// many small tiles that are only all resident at that occupancy; it spills some.
// The plain form takes up to 128 registers, four wavefronts per SIMD.
template <int LC, int SWC, typename Model>
constexpr int kDenseWaves = SWC == 1 && !Model::kString ? (LC == 0 ? 7 : 6) : 5;

template <bool DENSE, int LC, int SWC, typename Model, bool WIDE>
__global__ __launch_bounds__(1024)
__attribute__((amdgpu_waves_per_eu(DENSE ? kDenseWaves<LC, SWC, Model> : 4)))
void tile_kernel(RunView v, uint32_t n_gens) {
  constexpr uint32_t L = (uint32_t)LC;
  constexpr uint32_t SW = (uint32_t)SWC;
  constexpr uint32_t N = 1u << L;
  constexpr bool kStr = Model::kString;
  // words per outbox entry (f, T, surface, header; with a string f, T, D0,
  // D1, P0, P1, header) and the header's word, as in the HBM outbox
  constexpr uint32_t obs = (SW == 1 && !kStr) ? 4u : 8u;
  constexpr uint32_t ob_hdr = kStr ? 6u : 2u + SW;
  constexpr uint32_t kWords = 2u + SW + (kStr ? 2u : 0u);  // genome words
  constexpr uint32_t kBlock = 256u * kWords;               // LDS bytes of 64 agents
  constexpr uint32_t kSlot = 8u * exchange_words(kStr);    // bytes of an exchange slot
  // passes of 16 islands whose lanes' places stay in registers for the launch
  // (most wavefronts have no more; further ones are worked out each time)
  constexpr uint32_t kHeld = DENSE ? 1u : (L >= 4 || kStr) ? 2u : SW == 1 ? 4u : 3u;
  const uint32_t tid = threadIdx.x, nthreads = blockDim.x;
  const uint32_t lane = __lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t nwaves = nthreads >> 6;
  const uint32_t W = v.width, H = v.height;

  // this workgroup's tile and its actual extent
  const uint32_t tile = xcd_band_group();
  const uint32_t tx = tile % v.tiles_x, ty = tile / v.tiles_x;
  const uint32_t x0 = tx * v.tile_w, y0 = ty * v.tile_h;
  const uint32_t w = min(v.tile_w, W - x0), h = min(v.tile_h, H - y0);
  const uint32_t ti = w * h;
  const uint32_t TI = v.tile_w * v.tile_h;
  const uint32_t TA = tile_agents_padded(ti, L);
  const uint32_t n_iter = TA >> 6;

  const TileParents<SWC, kStr> pop;
  const uint32_t lprod = n_iter * kBlock;                    // [li]: the island's product
  const uint32_t lob = lprod + 4u * tile_table_words(TA, L);  // [(p * TI + li) * obs + k]
  const uint32_t halo = lob + 8u * TI * obs;                       // [pair * obs + k]
  const uint32_t n_halo = 2u * (v.tile_w + v.tile_h);
  const uint32_t halo_isl = halo + 4u * n_halo * obs;              // [pair]: island it comes from
  const uint32_t given = halo_isl + 4u * n_halo, arrivals = given + 4u;
  auto agent_at = [&](uint32_t la) { return (la >> 6) * kBlock + ((la & 63u) << 2); };

  // this wavefront's iterations (the wavefronts of a ragged tile that get none
  // take no part in the generations) and islands
  const uint32_t active = min(nwaves, n_iter);
  const uint32_t it0 = wave < active ? wave * n_iter / active : 0u;
  const uint32_t it1 = wave < active ? (wave + 1u) * n_iter / active : 0u;
  const uint32_t li0 = (it0 << 6) >> L;
  const uint32_t li1 = min((it1 << 6) >> L, ti);

  // island li of the tile
  auto island_id = [&](uint32_t li) {
    const uint32_t ly = li / w;
    return (y0 + ly) * W + x0 + (li - ly * w);
  };

  // ---- load: population, pending outbox --------------------------------------
  if (tid == 0u) {
    lds_put(given, 0u);
    lds_put(arrivals, 0u);
  }
  __syncthreads();
  const uint64_t t0 = *v.gen;
  const uint32_t p_first = ((uint32_t)t0 & 1u) ^ 1u;
  for (uint32_t la = tid; la < TA; la += nthreads) {
    const uint32_t li = la >> L;
    const uint32_t a = (island_id(li) << L) + (la & (N - 1u));
    Genome g;
    if (li < ti) {
      g.f = v.pop_f[a];
      g.T = v.pop_T[a];
      g.D0 = v.pop_D[a];
      if (SW > 1) g.D1 = v.pop_D[v.agent_stride + a];
      if (kStr) {
        g.P0 = v.pop_P[a];
        g.P1 = v.pop_P[v.agent_stride + a];
      }
    }
    pop.put(g, agent_at(la));
  }
  for (uint32_t k = tid; k < ti * obs; k += nthreads) {
    const uint32_t li = k / obs, j = k - li * obs;
    lds_put(lob + 4u * ((p_first * TI + li) * obs + j),
            v.ob[p_first][(size_t)island_id(li) * obs + j]);
  }
  __syncthreads();

  // ---- this wavefront's pass lanes ---------------------------------------------
  const uint32_t q = lane & 3u;
  const uint32_t lob_parity = 4u * TI * obs;       // bytes from parity 0 to 1
  const uint32_t ex_parity = v.islands * kSlot;
  // the neighbour of island r of the tile in this lane's direction
  auto neighbour = [&](uint32_t r, uint32_t* nx, uint32_t* ny) {
    const uint32_t ly = r / w;
    torus_xy(x0 + (r - ly * w), y0 + ly, q, W, H, nx, ny);
    return *nx - x0 < w && *ny - y0 < h;  // inside the tile
  };
  // The lane's place in pass `round` for generation t; the pairs of the
  // passes before it take the halo entries from `pair` on, which moves past
  // this pass's.
  auto place = [&](uint32_t round, uint32_t t_lo, uint32_t* pair) __attribute__((always_inline)) {
    PassLane pl;
    const uint32_t li = li0 + round * 16u + (lane >> 2);
    pl.ok = li < li1;
    const uint32_t r = pl.ok ? li : 0u;
    uint32_t nx, ny;
    const bool inside = neighbour(r, &nx, &ny);
    const uint64_t out_of = __builtin_amdgcn_ballot_w64(pl.ok && !inside);
    const uint32_t mine = *pair + __builtin_amdgcn_mbcnt_hi(
                                      (uint32_t)(out_of >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)out_of, 0u));
    *pair += (uint32_t)__popcll(out_of);
    const uint32_t p_out = t_lo & 1u, p_in = p_out ^ 1u;
    pl.island = island_id(r);
    pl.home = agent_at(r << L);
    pl.prod = lprod + 8u * r;
    pl.step = inside ? lob_parity : 0u;
    pl.in = inside ? lob + 4u * ((ny - y0) * w + (nx - x0)) * obs + p_in * lob_parity
                   : halo + 4u * mine * obs;
    pl.out = lob + 4u * (r * obs + q) + p_out * lob_parity;
    pl.to = pl.island * kSlot + 8u * q + p_out * ex_parity;
    pl.edge = ((out_of >> (lane & ~3u)) & 15ull) != 0ull;
    return pl;
  };
  // this wavefront's pairs: how many, and the islands they come from
  const uint32_t n_rounds = (li1 - li0 + 15u) >> 4;
  uint32_t n_pairs = 0u;
  for (uint32_t r = 0; r < n_rounds; ++r) (void)place(r, 0u, &n_pairs);
  uint32_t first = 0u;
  if (lane == 0u && n_pairs)
    first = __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t*)given, n_pairs,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  first = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
  for (uint32_t r = 0, pair = first; r < n_rounds; ++r) {
    const PassLane pl = place(r, 0u, &pair);
    uint32_t nx, ny;
    if (pl.ok && !neighbour(li0 + r * 16u + (lane >> 2), &nx, &ny))
      lds_put(halo_isl + (pl.in - halo) / obs, ny * W + nx);
  }
  keep_order();
  // The pending emissions (generation t0 - 1) come from the HBM outbox.
  for (uint32_t k = lane; k < n_pairs * obs; k += 64u) {
    const uint32_t p = first + k / obs, j = k % obs;
    lds_put(halo + 4u * (p * obs + j),
            v.ob[p_first][(size_t)lds_get<uint32_t>(halo_isl + 4u * p) * obs + j]);
  }
  keep_order();
  // From then on lane j fetches pair j (lane j + 64, ... the further ones of
  // a wavefront with more than 64): the emission's words as they are in the
  // exchange area.
  struct Sent {
    uint64_t w[kWords];
  };
  const bool fetches = lane < n_pairs;
  const uint32_t far = fetches ? lds_get<uint32_t>(halo_isl + 4u * (first + lane)) * kSlot : 0u;
  auto fetch = [&](bool on, uint32_t from, Sent& s) {
    if (on) {
      const unsigned long long* e = at_byte(v.exchange, from);
#pragma unroll
      for (uint32_t k = 0; k < kWords; ++k)
        s.w[k] = __hip_atomic_load(e + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  // whether a lane's words are not all of the generation stamped `stamp`
  auto stale = [&](bool on, uint32_t stamp, const Sent& s) {
    uint32_t off = 0u;
#pragma unroll
    for (uint32_t k = 0; k < kWords; ++k) off |= (uint32_t)(s.w[k] >> 32) ^ stamp;
    return __builtin_amdgcn_ballot_w64(on && off > 1u) != 0ull;
  };
  // the words as an outbox entry in the halo
  auto settle = [&](bool on, uint32_t pair, const Sent& s) {
    if (on) {
      const uint32_t hdr = kMetaValid | ((uint32_t)(s.w[0] >> 32) & 1u) |
                           (((uint32_t)(s.w[1] >> 32) & 1u) << 1);
      const uint32_t to = halo + 4u * pair * obs;
      const uint32_t f = (uint32_t)s.w[0], T = (uint32_t)s.w[1], D0 = (uint32_t)s.w[2];
      const uint32_t D1 = SW > 1 ? (uint32_t)s.w[3] : 0u;
      lds_put(to, Quad{f, T, D0, (SW > 1 || kStr) ? D1 : hdr});
      if (kStr)
        lds_put(to + 16u, Quad{(uint32_t)s.w[kWords - 2], (uint32_t)s.w[kWords - 1], hdr, 0u});
      else if (SW > 1)
        lds_put(to + 16u, Quad{hdr, 0u, 0u, 0u});
    }
  };
  // fetch and settle, as often as it takes (one long wait at most). Between tries
  // a wavefront of the dense form sleeps (1.7 us) at the lowest priority, one of the
  // plain form after 16 of them: 20 wavefronts of a CU that retry at once keep its
  // one address unit busy, and a wavefront whose stores some of them wait for gets
  // no turn until their tries run out (islands of one agent in 20 one-wavefront
  // tiles a CU: single passes held up for 30 to 52 ms, the run invalid). 24 such
  // tiles a CU: 13.5 us per generation, 18.8 asleep half as long, 34 a quarter, 68
  // with the first 16 tries at once; 24 tiles a CU of two 32-agent islands 3.67
  // against 3.55.
  uint32_t gave_up = 0u;
  auto wait_for = [&](bool on, uint32_t from, uint32_t stamp, uint32_t pair) {
    for (uint32_t spin = gave_up ? kLockSpins : 0u;; ++spin) {
      Sent s = {};
      fetch(on, from, s);
      if (!stale(on, stamp, s) || spin == kLockSpins) {
        gave_up += spin == kLockSpins ? 1u : 0u;
        settle(on, pair, s);
        break;
      }
      if (DENSE || spin >= 16u) {
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_s_sleep(64);
      }
    }
  };

  PassLane held[kHeld];
  Sent sent = {};
  uint32_t held_pairs = first;
#pragma unroll
  for (uint32_t r = 0; r < kHeld; ++r)
    if (r < n_rounds) held[r] = place(r, (uint32_t)t0, &held_pairs);

  const RoundKeys<!DENSE> key(v.seed, v.run_id);
  BreedLane bl = breed_lane<LC>(v, t0);
  const uint32_t group = bl.base;                     // bytes to the lane's island in its block
  const uint32_t slot_mask = bl.slot_mask;            // (N - 1) * 4
  const uint32_t q_shift = 8u * q + 6u - L;           // byte q of the draw, as a slot in place
  const uint32_t arrival = kMetaValid | (q ^ 2u);     // header of an arrival from direction q
  const bool plain = v.k == 2u && v.selection && !v.law;
  const bool exchanging = v.migration && n_pairs != 0u;

  for (uint32_t g = 0; wave < active && g < n_gens; ++g) {
    const uint64_t t = t0 + g;
    const uint32_t t_lo = (uint32_t)t;
    const uint32_t t_hi4 = (uint32_t)(t >> 32) << 2;
    const uint32_t stamp = t_lo << 1, stamp_in = (t_lo - 1u) << 1;
    const bool arriving = v.migration || g == 0u;

    // the wavefronts of a SIMD (every fourth one) take turns at its priorities,
    // a generation each
    switch (((wave >> 2) + g) & 3u) {
      case 0: __builtin_amdgcn_s_setprio(0); break;
      case 1: __builtin_amdgcn_s_setprio(1); break;
      case 2: __builtin_amdgcn_s_setprio(2); break;
      default: __builtin_amdgcn_s_setprio(3); break;
    }

    // ---- island pass ----------------------------------------------------------
    SelectStream migrate;
    migrate.init(0u, t_lo, t_hi4, v.seed, v.run_id, kStreamMigrate);
    // every wavefront's pass of generation t - 1 is done
    while ((uint32_t)__builtin_amdgcn_readfirstlane((int)lds_get<volatile uint32_t>(arrivals)) <
           g * active) {
      __builtin_amdgcn_s_sleep(1);
    }
    keep_order();
    // the halo: the emissions of t - 1 from outside (a run without migration
    // keeps the launch's pending ones for its first generation only)
    if (g != 0u && n_pairs != 0u && v.migration) {
      const uint32_t ex_in = (t_lo & 1u) ? 0u : ex_parity;
      if (!stale(fetches, stamp_in, sent))
        settle(fetches, first + lane, sent);
      else
        wait_for(fetches, far + ex_in, stamp_in, first + lane);
      for (uint32_t p = 64u + lane; __builtin_amdgcn_ballot_w64(p < n_pairs) != 0ull; p += 64u) {
        const bool on = p < n_pairs;
        const uint32_t from =
            on ? lds_get<uint32_t>(halo_isl + 4u * (first + p)) * kSlot + ex_in : 0u;
        wait_for(on, from, stamp_in, first + p);
      }
    }
    keep_order();
    auto pass = [&](const PassLane& pl) __attribute__((always_inline)) {
      const uint64_t product = migrate.of_island(pl.island);
      const Block mig = migrate.block_from(product, key);
      // the neighbour's emission of t - 1
      const Quad a = lds_get<Quad>(pl.in);
      Genome e;
      e.f = __uint_as_float(a.x);
      e.T = a.y;
      e.D0 = a.z;
      uint32_t hdr = a.w;
      if (SW > 1 || kStr) {
        e.D1 = a.w;
        const Quad b = lds_get<Quad>(pl.in + 16u);
        e.P0 = b.x;
        e.P1 = b.y;
        hdr = kStr ? b.z : b.x;
      }
      // arrivals into their drawn slots: one direction after the other, so
      // the last to draw a slot keeps it
      const bool hit = pl.ok && arriving && hdr == arrival;
      const uint32_t at = and_or(mig.z >> q_shift, slot_mask, pl.home);
      if (pl.ok && q == 0u) lds_put(pl.prod, product);  // for the iterations
      keep_order();
#pragma unroll
      for (uint32_t d = 0; d < 4; ++d) {
        if (hit && q == d) pop.put(e, at);
        keep_order();
      }
      // the emission, the drawn member after immigration: each lane of the
      // island sends on the genome words q, q + 4
      if (pl.ok) {
        const uint32_t emig = and_or(mig.x >> (30u - L), slot_mask, pl.home + 256u * q);
        const uint32_t dir = mig.y >> 30;
        const uint32_t ohdr = v.migration ? (kMetaValid | dir) : 0u;
        uint32_t word = q < kWords ? lds_get<uint32_t>(emig) : ohdr;
        uint32_t more = 0u;  // outbox word q + 4
        if (kStr) {
          // outbox words: f, T, D0, D1, P0, P1, header, 0
          if (SW == 1) {  // planes f, T, D0, P0, P1
            more = q == 0u ? lds_get<uint32_t>(emig + 768u)
                           : q == 1u ? lds_get<uint32_t>(emig + 768u) : q == 2u ? ohdr : 0u;
            word = q < 3u ? word : 0u;
          } else {
            more = q < 2u ? lds_get<uint32_t>(emig + 1024u) : q == 2u ? ohdr : 0u;
          }
          lds_put(pl.out + 16u, more);
        } else if (SW > 1) {
          lds_put(pl.out + 16u, q == 0u ? ohdr : 0u);
        }
        lds_put(pl.out, word);
        if (pl.edge && exchanging && g + 1u < n_gens) {
          // the exchange's words are the genome's: f, T, surface, string
          const uint64_t hi = (uint64_t)(stamp | ((dir >> q) & 1u)) << 32;
          unsigned long long* x = at_byte(v.exchange, pl.to);
          if (kStr && SW == 1) {
            if (q < 3u)
              __hip_atomic_store(x, hi | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (q < 2u)  // words 3 and 4
              __hip_atomic_store(x + 3, ((uint64_t)stamp << 32) | more, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
          } else {
            if (q < kWords)
              __hip_atomic_store(x, hi | word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (kWords > 4u && q + 4u < kWords)
              __hip_atomic_store(x + 4, ((uint64_t)stamp << 32) | more, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
    };
#pragma unroll
    for (uint32_t r = 0; r < kHeld; ++r)
      if (r < n_rounds) pass(held[r]);
    for (uint32_t r = kHeld, pair = held_pairs; r < n_rounds; ++r) pass(place(r, t_lo, &pair));
    keep_order();
    if (lane == 0u)
      __hip_atomic_fetch_add((__attribute__((address_space(3))) uint32_t*)arrivals, 1u,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    // the held lanes' places change parity
#pragma unroll
    for (uint32_t r = 0; r < kHeld; ++r) {
      const bool odd = (t_lo & 1u) != 0u;
      held[r].out += odd ? 0u - lob_parity : lob_parity;
      held[r].to += odd ? 0u - ex_parity : ex_parity;
      held[r].in += odd ? held[r].step : 0u - held[r].step;
    }

    // ---- iterations: lanes are agent slots ----------------------------------
    bl.t_lo = t_lo;
    bl.t_hi4 = t_hi4;
    bl.sel.init(bl.slot, t_lo, t_hi4, v.seed, v.run_id, kStreamSelect);
    bl.sel.hold();
    if (v.law) bl.mut.init(bl.slot, t_lo, t_hi4, v.seed, v.run_id, kStreamMutate);
    auto iterations = [&](auto fixed, uint32_t from, uint32_t to) __attribute__((always_inline)) {
      constexpr bool kPlain = decltype(fixed)::value;
      if (from >= to) return;
      // the islands' products are read an iteration ahead
      uint32_t next = lprod + 8u * (((from << 6) + lane) >> L);
      uint64_t island = lds_get<uint64_t>(next);
      bl.base = group + from * kBlock;
#pragma unroll 1
      for (uint32_t it = from; it < to; ++it) {
        next += 512u >> L;
        const uint64_t next_island = lds_get<uint64_t>(next);
        const Block r = bl.sel.block_from(island, key);
        const Genome c = breed<LC, SWC, Model, WIDE, kPlain>(v, bl, pop, r, island, key);
        pop.put(c, bl.base + 4u * bl.slot);  // padding past the last island too
        bl.base += kBlock;
        island = next_island;
      }
    };
    // halfway through, the first try for the neighbours' emissions of t goes out
    const uint32_t half = it0 + ((it1 - it0 + 1u) >> 1);
    auto run = [&](uint32_t from, uint32_t to) __attribute__((always_inline)) {
      if (plain)
        iterations(BoolC<true>{}, from, to);
      else
        iterations(BoolC<false>{}, from, to);
    };
    run(it0, half);
    if (exchanging && g + 1u < n_gens) fetch(fetches, far + (t_lo & 1u) * ex_parity, sent);
    run(half, it1);
  }
  __syncthreads();

  // ---- store: population and the last generation's outbox -------------------
  for (uint32_t la = tid; la < (ti << L); la += nthreads) {
    const uint32_t a = (island_id(la >> L) << L) + (la & (N - 1u));
    const Genome c = pop.get(agent_at(la));
    v.pop_f[a] = c.f;
    v.pop_T[a] = c.T;
    v.pop_D[a] = c.D0;
    if (SW > 1) v.pop_D[v.agent_stride + a] = c.D1;
    if (kStr) {
      v.pop_P[a] = c.P0;
      v.pop_P[v.agent_stride + a] = c.P1;
    }
  }
  if (n_gens > 0) {
    const uint32_t p_last = (uint32_t)(t0 + n_gens - 1u) & 1u;
    uint32_t* gob = v.ob[p_last];
    for (uint32_t k = tid; k < ti * obs; k += nthreads) {
      const uint32_t li = k / obs, j = k - li * obs;
      gob[(size_t)island_id(li) * obs + j] =
          lds_get<uint32_t>(lob + 4u * ((p_last * TI + li) * obs + j));
    }
  }
  if (lane == 0u && gave_up)
    __hip_atomic_fetch_add(v.waits, (unsigned long long)gave_up, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

size_t tile_lds_bytes(uint32_t tile_w, uint32_t tile_h, uint32_t log2n, uint32_t words,
                      uint32_t model, uint32_t ob_stride) {
  const uint32_t TI = tile_w * tile_h;
  const uint32_t TA = tile_agents_padded(TI, log2n);
  const size_t pop = (size_t)tile_agent_words(words, model_has_string(model)) * TA;
  const size_t all = pop + tile_table_words(TA, log2n) + 2u * (size_t)TI * ob_stride +
                     2u * (size_t)(tile_w + tile_h) * (ob_stride + 1u) + 2u;
  return 4u * std::max(all, pop + 2u * (size_t)((TA + 64u) >> log2n));
}

uint32_t tile_threads(uint32_t tile_w, uint32_t tile_h, uint32_t log2n) {
  const uint32_t iters = tile_agents_padded(tile_w * tile_h, log2n) >> 6;
  return 64u * (iters < 16u ? iters : 16u);
}

// Wavefronts per CU of the plain form (its 128-register budget).
constexpr uint32_t kPlainWaves = 16;

hipError_t tile_occupancy(const RunView& v, uint32_t threads, size_t lds, int* groups_per_cu) {
  return dispatch(v, [&](auto LC, auto SWC, auto M, auto WD) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        groups_per_cu, tile_kernel<true, GA_SHAPE_ARGS(LC, SWC, M, WD)>, (int)threads, lds);
  });
}

hipError_t launch_tiles(const RunView& v, uint64_t n_gens, hipStream_t stream) {
  if (n_gens == 0) return hipSuccess;
  const uint32_t n_tiles = v.tiles_x * v.tiles_y;
  // without an exchange area (or a neighbour to exchange with) a launch of
  // several tiles runs one generation, which needs no exchange
  if (n_tiles > 1 && n_gens > 1 && v.migration && !v.exchange) return hipErrorInvalidValue;
  const uint32_t threads = tile_threads(v.tile_w, v.tile_h, v.log2n);
  const size_t lds = tile_lds_bytes(v.tile_w, v.tile_h, v.log2n, v.words, v.model, v.ob_stride);
  int device = 0, cus = 0;
  hipError_t e = hipGetDevice(&device);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
  if (e != hipSuccess) return e;
  // the plain form while all tiles are resident at its occupancy
  const uint32_t per_cu = (n_tiles + (uint32_t)cus - 1u) / (uint32_t)cus;
  const bool dense = per_cu * (threads / 64u) > kPlainWaves;
  return dispatch(v, [&](auto LC, auto SWC, auto M, auto WD) {
    if (dense)
      tile_kernel<true, GA_SHAPE_ARGS(LC, SWC, M, WD)><<<dim3(n_tiles), dim3(threads), lds, stream>>>(
          v, (uint32_t)n_gens);
    else
      tile_kernel<false, GA_SHAPE_ARGS(LC, SWC, M, WD)><<<dim3(n_tiles), dim3(threads), lds, stream>>>(
          v, (uint32_t)n_gens);
    return hipGetLastError();
  });
}

}  // namespace ga
