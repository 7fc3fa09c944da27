// Stand-ins for the HIP runtime and the kernel launch wrappers that carry out
// the plan of generations the C ABI's host logic (ga_api.hip) hands them: device
// memory is host memory, a launch moves an agent's deposit counter T by the
// generations it would run and aborts if the agent is not at the generation the
// launch says, launches on a capturing stream run when their graph is launched.
// So T at the end of a call says which generations were planned. Also checked:
// candidates are left for the generation a launch of two starts from, whole in
// memory of their own. plan_* below are for the tests.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdio>
#include <functional>
#include <map>
#include <string>
#include <vector>
#include "ga_internal.hpp"

struct ihipStream_t { int x; };
struct ihipEvent_t { int x; };
struct ihipGraph_t { std::vector<std::function<void()>> nodes; };
struct ihipGraphExec_t { std::vector<std::function<void()>> nodes; };

namespace {
std::map<uint8_t*, size_t> blocks;  // live device allocations
size_t malloc_limit = SIZE_MAX;     // larger ones fail
std::vector<size_t> mallocs;        // sizes asked for
std::vector<uint64_t> tile_gens;    // generations of each tile launch
unsigned frees = 0, captures = 0, persistent = 0;
unsigned batch_tiles = 0;            // tiles of the last batch launch
hipStream_t capturing = nullptr;
ihipGraph_t* graph = nullptr;

[[noreturn]] void stop(const char* what) {
  fprintf(stderr, "plan: %s\n", what);
  abort();
}
hipError_t run(hipStream_t s, std::function<void()> f) {
  if (capturing && s == capturing)
    graph->nodes.push_back(std::move(f));
  else
    f();
  return hipSuccess;
}
}  // namespace

extern "C" {
void plan_reset(size_t limit) {
  malloc_limit = limit;
  mallocs.clear();
  tile_gens.clear();
  frees = captures = persistent = 0;
}
unsigned plan_count(const char* what) {
  const std::string w(what);
  if (w == "mallocs") return (unsigned)mallocs.size();
  if (w == "frees") return frees;
  if (w == "captures") return captures;
  if (w == "persistent") return persistent;
  if (w == "batch tiles") return batch_tiles;
  if (w == "tile launches") return (unsigned)tile_gens.size();
  stop("no such count");
}
uint64_t plan_tile_gens(unsigned i) { return tile_gens[i]; }
int roctxRangePushA(const char*) { return 0; }
int roctxRangePop() { return 0; }
}

const char* hipGetErrorString(hipError_t) { return "plan"; }
hipError_t hipMalloc(void** p, size_t n) {
  mallocs.push_back(n);
  if (n > malloc_limit) return hipErrorInvalidValue;
  *p = calloc(1, n);
  blocks[static_cast<uint8_t*>(*p)] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  frees += 1;
  blocks.erase(static_cast<uint8_t*>(p));
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memmove(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = new ihipStream_t(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = new ihipEvent_t(); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, int) { capturing = s; graph = new ihipGraph_t(); captures += 1; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = graph; capturing = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, void*, void*, size_t) { *x = new ihipGraphExec_t{g->nodes}; return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { delete g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete x; return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) { for (auto& f : x->nodes) f(); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, int, int) { *v = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }

namespace ga {
namespace {

// Islands [first, first + ipw) of v from generation t on by n.
void breed(const RunView& v, uint32_t first, uint32_t ipw, uint64_t t, uint32_t n) {
  const uint32_t end = std::min(first + ipw, v.islands);
  for (size_t a = (size_t)first << v.log2n; a < (size_t)end << v.log2n; ++a) {
    if (v.pop_T[a] != (uint32_t)t) stop("an agent is not at the launch's generation");
    v.pop_T[a] += n;
  }
}

size_t cand_plane(const RunView& v) { return (size_t)v.island_stride * v.ob_stride; }

// Candidates of generation t: the generation and the run they belong to, in the
// whole of their plane, which must be part of one allocation.
void leave(const RunView& v, uint64_t t, uint32_t run) {
  uint32_t* p = v.cand + ((t & 2u) ? cand_plane(v) : 0u);
  bool inside = false;
  for (const auto& b : blocks)
    inside |= (uint8_t*)v.cand >= b.first &&
              (uint8_t*)(v.cand + 2 * cand_plane(v)) <= b.first + b.second;
  if (!inside) stop("candidates outside the library's memory");
  for (size_t k = 0; k < cand_plane(v); ++k) p[k] = (uint32_t)t * 4096u + run;
}
void take(const RunView& v, uint64_t t, uint32_t run) {
  if (!v.migration) return;
  const uint32_t* p = v.cand + ((t & 2u) ? cand_plane(v) : 0u);
  for (size_t k = 0; k < cand_plane(v); ++k)
    if (p[k] != (uint32_t)t * 4096u + run) stop("no candidates for the launch's generation");
}

RunView member(const RunView* views, uint32_t run) {
  RunView v = views[run];
  const uintptr_t at = reinterpret_cast<uintptr_t>(views);
  auto fix = [&](auto& p) { p = reinterpret_cast<std::decay_t<decltype(p)>>(reinterpret_cast<uintptr_t>(p) + at); };
  fix(v.pop_f), fix(v.pop_T), fix(v.pop_D), fix(v.ob[0]), fix(v.ob[1]), fix(v.gen), fix(v.left), fix(v.cand);
  return v;
}

}  // namespace

hipError_t launch_generation(const RunView& v, uint32_t off, uint32_t waves, uint32_t, hipStream_t s) {
  return run(s, [=] {
    const uint64_t t = *v.gen + off;
    switch (v.span) {
      case kSpanCandidates: leave(v, t, 0); return;
      case kSpanFromMail: case kSpanToMail: return;
      case kSpanTwo:
        take(v, t, 0);
        if ((v.ipw << v.log2n) > pair_agents(v.log2n, pair_words(v.words, v.model != 0))) stop("chunk larger than its LDS");
        [[fallthrough]];
      case kSpanOne:
        for (uint32_t w = 0; w < waves; ++w) breed(v, w * v.ipw, v.ipw, t, v.span);
        if (v.span == kSpanTwo && v.migration) leave(v, t + 2, 0);
        return;
    }
    stop("unknown span");
  });
}
hipError_t launch_tiles(const RunView& v, uint64_t n, hipStream_t s) {
  return run(s, [=] {
    tile_gens.push_back(n);
    breed(v, 0, v.islands, *v.gen, (uint32_t)n);
  });
}
size_t tile_lds_bytes(uint32_t w, uint32_t h, uint32_t l, uint32_t words, uint32_t, uint32_t o) {
  return 4 * ((size_t)w * h * ((2 + words) << l) + 2 * w * h * o);
}
uint32_t tile_threads(uint32_t w, uint32_t h, uint32_t l) {
  return 64u * std::min(16u, ((w * h << l) + 63u) / 64u);
}
hipError_t tile_occupancy(const RunView&, uint32_t threads, size_t, int* g) { *g = (int)(1024u / threads); return hipSuccess; }
// What a CU holds at once of groups of `wpg` wavefronts: 32 wavefronts, and LDS,
// given out in pieces of `piece` bytes.
uint32_t resident(const RunView& v, uint32_t wpg, size_t piece) {
  const size_t lds = (lds_bytes(v.ipw, wpg, v.model) + piece - 1) / piece * piece;
  return (uint32_t)std::min<size_t>(32u / wpg, (160u << 10) / lds) * 256u;
}
hipError_t launch_async(const RunView& v, uint64_t n, uint32_t waves, uint32_t, uint32_t wpg, uint32_t, uint32_t, hipStream_t s) {
  if ((waves + wpg - 1) / wpg > resident(v, wpg, 1280)) stop("more groups than are resident");
  return run(s, [=] { breed(v, 0, v.islands, *v.gen, (uint32_t)n); });
}
hipError_t launch_lockstep(const RunView& v, uint64_t gen, uint64_t n, uint32_t waves, uint32_t, uint32_t wpg, hipStream_t s) {
  if ((waves + wpg - 1) / wpg > resident(v, wpg, 1280)) stop("more groups than are resident");
  return run(s, [=] {
    if (gen != *v.gen) stop("lockstep launch at another generation");
    persistent += 1;
    breed(v, 0, v.islands, gen, (uint32_t)n);
  });
}
// as the occupancy query, which does not know the pieces
hipError_t async_capacity(const RunView& v, uint32_t wpg, bool, uint32_t* w) { *w = resident(v, wpg, 1) * wpg; return hipSuccess; }
hipError_t launch_advance(unsigned long long* g, uint64_t n, hipStream_t s) { return run(s, [=] { *g += n; }); }
hipError_t launch_init(const RunView&, hipStream_t) { return hipSuccess; }
bool model_has_string_host(uint32_t id) { return id != 0; }
uint32_t model_count() { return 3; }
size_t lds_bytes(uint32_t ipw, uint32_t waves, uint32_t model) { return (5u * ipw + 1u) * 16u * (model ? 2u : 1u) * waves; }
hipError_t launch_fill(uint32_t* p, uint32_t v, size_t n, hipStream_t) { for (size_t i = 0; i < n; ++i) p[i] = v; return hipSuccess; }
hipError_t launch_sample(const RunView& v, uint32_t* ids, hipStream_t) { for (uint32_t i = 0; i < v.islands; ++i) ids[i] = i << v.log2n; return hipSuccess; }
hipError_t launch_gather(const RunView& v, const uint32_t* ids, uint32_t n, uint32_t* T, uint32_t*, hipStream_t) {
  for (uint32_t j = 0; j < n; ++j) T[j] = v.pop_T[ids[j]];
  return hipSuccess;
}
hipError_t launch_batch_all(const RunView* views, const Tile* tiles, uint32_t grid, uint32_t off, uint32_t, uint32_t, hipStream_t s) {
  return run(s, [=] {
    std::map<uint32_t, bool> seen;
    batch_tiles = (unsigned)std::count_if(tiles, tiles + grid, [](const Tile& t) { return t.cls != kNoTile; });
    for (uint32_t w = 0; w < grid; ++w) {
      const Tile tile = tiles[w];
      if (tile.cls == kNoTile) continue;
      const RunView v = member(views, tile.run);
      const uint64_t t0 = *v.gen, left = *v.left;
      const bool first = !seen[tile.run];
      seen[tile.run] = true;
      if (off >= kBatchCandidates) {
        if (v.migration && first) leave(v, t0, 1u + tile.run);
      } else if (off >= kBatchSingle) {
        const uint64_t n = (off & ~kBatchSingle) >> 2, takes = std::min(left, n);
        const uint64_t ran = (takes & ~3ull) + (off & 3u);
        if (ran < takes) breed(v, tile.first, v.ipw, t0 + ran, 1);
      } else if (off >= kBatchPair) {
        const uint32_t ran = off & ~kBatchPair;
        if ((left & ~3ull) <= ran) continue;
        if (first) take(v, t0 + ran, 1u + tile.run);
        breed(v, tile.first, v.ipw, t0 + ran, 2);
      } else if (left > off) {
        breed(v, tile.first, v.ipw, t0 + off, 1);
      }
    }
    // after the launch: what the pair leaves, once no tile reads any more
    if (off >= kBatchPair && off < kBatchSingle)
      for (const auto& m : seen) {
        const RunView v = member(views, m.first);
        const uint32_t ran = off & ~kBatchPair;
        if ((*v.left & ~3ull) > ran && v.migration) leave(v, *v.gen + ran + 2, 1u + m.first);
      }
  });
}
hipError_t launch_store_u64(unsigned long long* p, unsigned long long v, hipStream_t) { *p = v; return hipSuccess; }
hipError_t launch_batch_advance(const RunView* views, const uint32_t* n, uint32_t, uint64_t block, hipStream_t s) {
  return run(s, [=] {
    for (uint32_t m = 0; m < *n; ++m) {
      const RunView v = member(views, m);
      const uint64_t adv = std::min<uint64_t>(*v.left, block);
      *v.gen += adv;
      *v.left -= adv;
    }
  });
}
hipError_t launch_roof_inplace(void*, size_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_roof_philox(uint32_t*, uint32_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_roof_valu(uint32_t*, uint32_t, uint32_t, uint32_t, hipStream_t) { return hipSuccess; }
size_t mrca_workspace_bytes(size_t n) { return n * 16; }
hipError_t launch_mrca_matrix_noalloc(const uint32_t*, const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t*, uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_mrca_matrix(const uint32_t*, const uint32_t*, uint32_t, uint32_t, uint32_t, uint32_t, uint32_t, void*, uint32_t*, uint32_t*, hipStream_t) { return hipSuccess; }
}  // namespace ga
