// All-pairs MRCA-interval estimation from hereditary-stratigraphy surfaces on
// gfx950: the primitive under post hoc phylogenetic reconstruction (paper
// Fig. 1: markers on genomes let relatedness be estimated after the run; Sec. 3
// reconstructs from 10k sampled end-state genomes).
//
// For two surfaces with deposit counters Ta, Tb on S sites, the ranks both
// retain are the multiples of 2^e, e = max(e(Ta), e(Tb)), below min(Ta, Tb)
// (e(n) = max(0, ceil(log2 n) - log2 S), "doubling steady" surface). Ranks
// older than the MRCA hold identical differentia, so the first common rank
// whose differentia differ bounds the MRCA's counter from above (U); kc
// matching common ranks in a row below U make an MRCA earlier than them a
// 2^-(b kc) event for b-bit differentia (L).
//
// Layout of the work: `normalize_kernel` turns each surface into its retained
// differentia in rank order (field j, b bits wide, = rank j * 2^e(T)), a
// 64-bit string (S * b <= 64); for one-bit differentia a pair keeps every
// 2^(e - e(T))-th bit of each string (stride compaction), XORs them and
// takes the lowest set bit, O(1) per pair; wider fields are compared field by
// field up to the first mismatch (at most S <= 32 of them). The tilted and
// hybrid policies need no pass of their own (ga_mrca_pairs.hpp). Integer only.
#include <mutex>

#include "ga_internal.hpp"
#include "ga_mrca_pairs.hpp"

namespace ga {
namespace {

struct Normalized {
  unsigned long long bits;  // retained differentia in rank order
  uint32_t T;
  uint32_t epoch;
};

__device__ __forceinline__ uint32_t epoch_of(uint32_t n, uint32_t s) {
  // max(0, ceil(log2 n) - s); ceil(log2 n) = bitlen(n - 1) for n >= 1
  const uint32_t c = n <= 1u ? 0u : 32u - __clz(n - 1u);
  return c > s ? c - s : 0u;
}

// Site of rank r (a retained rank, so never a discard): ranks below S keep
// site r; otherwise walk to the rank whose site the j-th rank of its epoch
// took over, as in the generation step's deposit.
__device__ uint32_t site_of_retained(uint32_t r, uint32_t s) {
  const uint32_t half = 1u << (s - 1u);
  if (r < (half << 1)) return r;
  const uint32_t e = (32u - __clz(r)) - s;
  uint32_t odd = (((r >> e) - half) << 1) | 1u;
  uint32_t shift = e - 1u;
  for (;;) {
    const uint32_t len = 32u - __clz(odd);
    if (len + shift <= s) return odd << shift;
    const uint32_t lead = odd << (s - len);
    shift = len + shift - s - 1u;
    odd = ((lead - half) << 1) | 1u;
  }
}

// One wavefront per surface, lane l deciding bit l of the string.
__global__ __launch_bounds__(256) void normalize_kernel(const uint32_t* __restrict__ T,
                                                        const uint32_t* __restrict__ D, uint32_t n,
                                                        uint32_t s, uint32_t dlog,
                                                        Normalized* out) {
  const uint32_t a = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (a >= n) return;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t words = (1u << (s + dlog)) >> 5;  // S * b / 32
  const uint32_t t = T[a];
  const uint32_t e = epoch_of(t, s);
  const uint32_t count = t == 0u ? 0u : ((t - 1u) >> e) + 1u;  // ceil(t / 2^e) <= S
  const uint32_t j = lane >> dlog;                             // the bit's field
  uint32_t bit = 0u;
  if (j < count) {
    const uint32_t at = (site_of_retained(j << e, s) << dlog) + (lane & ((1u << dlog) - 1u));
    bit = (D[(size_t)a * words + (at >> 5)] >> (at & 31u)) & 1u;
  }
  const unsigned long long bits = __builtin_amdgcn_ballot_w64(bit != 0u);
  if (lane == 0u) out[a] = Normalized{bits, t, e};
}

// keep bits 0, 2^d, 2*2^d, ... of x, packed to the bottom
__device__ __forceinline__ unsigned long long compact_stride(unsigned long long x, uint32_t d) {
  for (uint32_t i = 0; i < d; ++i) {
    x &= 0x5555555555555555ull;
    x = (x | (x >> 1)) & 0x3333333333333333ull;
    x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
    x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
    x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
    x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
  }
  return x;
}

// Interval for the pair (a, b) of normalised surfaces.
__device__ __forceinline__ uint2 pair_interval(const Normalized& a, const Normalized& b,
                                               uint32_t dlog, uint32_t kc) {
  const uint32_t e = a.epoch > b.epoch ? a.epoch : b.epoch;
  const uint32_t tmin = a.T < b.T ? a.T : b.T;
  const uint32_t common = tmin == 0u ? 0u : ((tmin - 1u) >> e) + 1u;  // ranks j*2^e < tmin
  uint32_t j = common;  // first mismatching common rank index, or common
  if (dlog == 0u) {
    const unsigned long long diff =
        compact_stride(a.bits, e - a.epoch) ^ compact_stride(b.bits, e - b.epoch);
    const unsigned long long mask = common >= 64u ? ~0ull : ((1ull << common) - 1ull);
    const unsigned long long hit = diff & mask;
    if (hit) j = (uint32_t)__ffsll((long long)hit) - 1u;
  } else if (a.epoch == b.epoch) {
    // common rank i is field i of both strings: the first differing field
    // holds the lowest set bit of the XOR
    const uint32_t used = common << dlog;  // bits of the common fields
    const unsigned long long mask = used >= 64u ? ~0ull : ((1ull << used) - 1ull);
    const unsigned long long hit = (a.bits ^ b.bits) & mask;
    if (hit) j = ((uint32_t)__ffsll((long long)hit) - 1u) >> dlog;
  } else {
    // common rank i is field i << (e - epoch) of each string
    const unsigned long long fmask = (1ull << (1u << dlog)) - 1ull;
    const uint32_t da = e - a.epoch, db = e - b.epoch;
    for (uint32_t i = 0; i < common; ++i) {
      const unsigned long long fa = (a.bits >> ((i << da) << dlog)) & fmask;
      const unsigned long long fb = (b.bits >> ((i << db) << dlog)) & fmask;
      if (fa != fb) {
        j = i;
        break;
      }
    }
  }
  const uint32_t upper = j < common ? j << e : tmin;
  const uint32_t lower = j < kc ? 0u : ((j - kc) << e) + 1u;
  return make_uint2(lower, upper);
}

// Keep bits 0, 2^d, 2 * 2^d, ... of a 32-bit string, packed to the bottom.
__device__ __forceinline__ uint32_t compact_stride32(uint32_t x, uint32_t d) {
  for (uint32_t i = 0; i < d && i < 5u; ++i) {
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    x = (x | (x >> 8)) & 0x0000FFFFu;
  }
  return x;
}

// Steady pairs: nothing but writes (8 bytes a pair). One thread per pair (x, y) in
// each of eight passes over 2,048 consecutive y (256 per pass, lane-consecutive,
// so loads and the two output rows are coalesced); rows of the grid are x.
// 10,000 x 10,000: 144 us with the normalisation. The order the stores come out in
// matters more than the instructions before them: with the differentia width
// fixed at compile time the same kernel takes 157.
__global__ __launch_bounds__(256) void steady_pairs_kernel(const Normalized* __restrict__ nz,
                                                           uint32_t n, uint32_t dlog, uint32_t kc,
                                                           uint32_t* __restrict__ L,
                                                           uint32_t* __restrict__ U) {
  const uint32_t x = blockIdx.y;
  const Normalized a = nz[x];
  const size_t row = (size_t)x * n;
#pragma unroll
  for (uint32_t pass = 0; pass < 8; ++pass) {
    const uint32_t y = blockIdx.x * 2048u + pass * 256u + threadIdx.x;
    if (y < n) {
      const uint2 r = pair_interval(a, nz[y], dlog, kc);
      U[row + y] = r.y;
      L[row + y] = r.x;
    }
  }
}

// What a pair needs of a surface, in the four words a row or column keeps.
typedef uint32_t Quad __attribute__((ext_vector_type(4)));
enum Kind { kTilted, kTilted2, kTiltedWide, kHybrid };

struct PairArgs {
  const uint32_t* __restrict__ T;
  const uint32_t* __restrict__ D;
  uint32_t kc;
};

// Sites of the hybrid's steady half in rank order, one row of 32 for each of
// its epochs: 0 to 26, for up to 2^31 deposits.
constexpr uint32_t kEpochs = 27;

template <int KIND>
__device__ __forceinline__ Quad surface(const PairArgs& a, uint32_t x, const uint8_t* sites) {
  const uint32_t t = a.T[x];
  if (KIND == kTilted) return Quad{a.D[x], 0u, t, 0u};
  const uint32_t lo = a.D[(size_t)x * 2], hi = a.D[(size_t)x * 2 + 1];
  if (KIND == kTilted2 || KIND == kTiltedWide) {
    // slots 0 and 1 of every level, or bits 0 and 1 of every field
    const uint64_t w = (uint64_t)hi << 32 | lo;
    return Quad{even_bits(w), even_bits(w >> 1), t, 0u};
  }
  // hybrid: the steady half (sites 0..31) in rank order, (t + 1) / 2 deposits
  // on the even ranks; the tilted half's levels
  const uint32_t nh = (t >> 1) + (t & 1u);
  const uint32_t e = epoch_of(nh, 5u);
  const uint32_t count = nh == 0u ? 0u : ((nh - 1u) >> e) + 1u;  // <= 32
  uint32_t bits = 0u;
  for (uint32_t j = 0; j < count; ++j) bits |= ((lo >> sites[e * 32u + j]) & 1u) << j;
  return Quad{bits, hi, t, e};
}

template <int KIND>
__device__ __forceinline__ Interval interval(const PairArgs& g, const Quad& a, const Quad& b) {
  if (KIND == kTilted) return tilted_interval(a.z, b.z, a.x ^ b.x, g.kc);
  if (KIND == kTiltedWide) return tilted_interval(a.z, b.z, (a.x ^ b.x) | (a.y ^ b.y), g.kc);
  if (KIND == kTilted2) return tilted2_interval(a.z, b.z, a.x ^ b.x, a.y ^ b.y, g.kc);
  const uint32_t E = a.w > b.w ? a.w : b.w;
  const uint32_t na = (a.z >> 1) + (a.z & 1u), nb = (b.z >> 1) + (b.z & 1u);
  const uint32_t nmin = na < nb ? na : nb;
  const uint32_t shared = nmin == 0u ? 0u : ((nmin - 1u) >> E) + 1u;  // <= 32
  return hybrid_interval(a.z, b.z, compact_stride32(a.x, E - a.w), compact_stride32(b.x, E - b.w),
                         E, shared, a.y ^ b.y, g.kc);
}

// All pairs under the tilted and hybrid policies. A workgroup takes `rows`
// consecutive rows x by 1,024 columns: a thread keeps four columns' surfaces in
// registers (256 apart, so a store is a wavefront's 256 consecutive bytes) and
// reads each row's from LDS (one address for the whole wavefront). The writes
// take 117 to 124 us of a 10,000 x 10,000 matrix (a plain fill of both outputs);
// with 60 to 230 vector instructions a pair it takes, against comparing all S
// sites of a pair in mirrored 64 x 64 blocks: tilted S = 32 147 us (601), S = 64
// 267 (1,164), S = 32 of 2 bits 160 (601), hybrid 505 (858). Bound: the writes,
// VALU for S = 64 and the hybrid. Four consecutive columns a thread (16-byte
// stores) or 32 rows measured 2% and 10% slower.
constexpr uint32_t kCols = 4;  // columns a thread keeps
constexpr uint32_t kMaxRows = 8;

template <int KIND>
__global__ __launch_bounds__(256) void pairs_kernel(PairArgs args, uint32_t n, uint32_t rows,
                                                    uint32_t* __restrict__ L,
                                                    uint32_t* __restrict__ U) {
  __shared__ Quad row[kMaxRows];
  __shared__ uint8_t sites[KIND == kHybrid ? kEpochs * 32u : 1u];
  const uint32_t x0 = blockIdx.y * rows, x1 = min(x0 + rows, n);
  if (KIND == kHybrid) {
    for (uint32_t k = threadIdx.x; k < kEpochs * 32u; k += 256u)
      sites[k] = (uint8_t)site_of_retained((k & 31u) << (k >> 5), 5u);
    __syncthreads();
  }
  for (uint32_t x = x0 + threadIdx.x; x < x1; x += 256u)
    row[x - x0] = surface<KIND>(args, x, sites);
  const uint32_t y = blockIdx.x * (256u * kCols) + threadIdx.x;
  Quad col[kCols];
#pragma unroll
  for (uint32_t c = 0; c < kCols; ++c)
    col[c] = surface<KIND>(args, min(y + 256u * c, n - 1u), sites);
  __syncthreads();
#pragma unroll 1
  for (uint32_t x = x0; x < x1; ++x) {
    const Quad a = row[x - x0];
    const size_t at = (size_t)x * n + y;
#pragma unroll
    for (uint32_t c = 0; c < kCols; ++c) {
      const Interval r = interval<KIND>(args, a, col[c]);
      if (y + 256u * c < n) {
        U[at + 256u * c] = r.upper;
        L[at + 256u * c] = r.lower;
      }
    }
  }
}

// Rows per workgroup: as many as leave about eight workgroups per CU (2,048), so
// that a small matrix still spreads over the chip.
template <int KIND>
hipError_t launch_pairs(const PairArgs& args, uint32_t n, uint32_t* L, uint32_t* U,
                        hipStream_t stream) {
  const uint32_t columns = (n + 256u * kCols - 1u) / (256u * kCols);
  const uint32_t rows = max(1u, min(kMaxRows, (uint32_t)((uint64_t)columns * n / 2048u)));
  pairs_kernel<KIND><<<dim3(columns, (n + rows - 1u) / rows), dim3(256), 0, stream>>>(
      args, n, rows, L, U);
  return hipGetLastError();
}

}  // namespace

size_t mrca_workspace_bytes(size_t n) { return n * sizeof(Normalized); }

// Workspace of the allocation-free relatedness call: one normalised surface
// per sample for up to kScratchSurfaces samples, in a file-scope device array.
// Each GPU the library runs on holds its own copy until the process ends.
// In host code `scratch` only names the symbol: its device address, per
// device, comes from hipGetSymbolAddress.
static __device__ __align__(256) Normalized scratch[kScratchSurfaces];

constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void* scratch_ptr[kMaxDevices] = {};

// Device address of the current device's copy of `scratch`, looked up once
// per device (with that device current) and kept.
hipError_t scratch_address(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> hold(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    scratch_ptr[dev] = p;
  }
  *out = scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_mrca_matrix(const uint32_t* T, const uint32_t* D, uint32_t n, uint32_t s_log,
                              uint32_t dlog, uint32_t policy, uint32_t kc, void* workspace,
                              uint32_t* L, uint32_t* U, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const PairArgs args{T, D, kc};
  if (policy == 2u) return launch_pairs<kHybrid>(args, n, L, U, stream);
  if (policy == 1u) {
    if (s_log == 6u && dlog == 0u) return launch_pairs<kTilted2>(args, n, L, U, stream);
    if (s_log == 5u && dlog == 0u) return launch_pairs<kTilted>(args, n, L, U, stream);
    if (s_log == 5u && dlog == 1u) return launch_pairs<kTiltedWide>(args, n, L, U, stream);
    return hipErrorInvalidValue;
  }
  Normalized* nz = static_cast<Normalized*>(workspace);
  normalize_kernel<<<dim3((n + 3) / 4), dim3(256), 0, stream>>>(T, D, n, s_log, dlog, nz);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((n + 2047) / 2048, n);
  steady_pairs_kernel<<<grid, dim3(256), 0, stream>>>(nz, n, dlog, kc, L, U);
  return hipGetLastError();
}

hipError_t launch_mrca_matrix_noalloc(const uint32_t* T, const uint32_t* D, uint32_t n,
                                      uint32_t s_log, uint32_t dlog, uint32_t policy, uint32_t kc,
                                      uint32_t* L, uint32_t* U, hipStream_t stream) {
  if (n > kScratchSurfaces) return hipErrorInvalidValue;
  void* ws = nullptr;
  if (n != 0 && policy == 0u) {
    // the normalise pass writes every one of the n entries it reads back,
    // so nothing left from an earlier call needs clearing
    const hipError_t e = scratch_address(&ws);
    if (e != hipSuccess) return e;
  }
  return launch_mrca_matrix(T, D, n, s_log, dlog, policy, kc, ws, L, U, stream);
}

}  // namespace ga
