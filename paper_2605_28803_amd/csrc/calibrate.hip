// Calibration of the static per-step, per-channel activation steps
// (Section 4.2, eq:perstep_scale): Delta_j = sigma_hat(|Y[:, j]|) / q_max with
// the robust peak sigma_hat taken as the nearest-rank p-th percentile of the
// magnitudes of column j (p = 99.9 in the paper's calibration settings).
//
// The percentile is an order statistic, computed exactly over the bit patterns
// of |y|: for non-negative floats the unsigned order of the pattern is the
// numeric order (NaN patterns sort above +inf).  Two routes.
//
// High percentiles (the m-th largest of n with m small: 9 of 8160 at 99.9):
// one pass over Y takes the maximum of each of up to 256 groups of consecutive
// rows per column.  The m-th largest group maximum L is a lower bound of the
// result (m groups hold a value >= L), and only groups whose maximum exceeds L
// (fewer than m) hold values above it.  One wave per column finds L, re-reads
// just those groups, keeps the values above L, and selects the m-th largest of
// them, or L itself if there are fewer than m.  Bound by the one read of Y:
// 8160 x 2048 takes 27 us (11 the read, 16 the selection: its scattered re-reads touch
// most cache lines of Y once more) against 229 us for the radix route's four reads.
//
// Otherwise radix selection: four passes of 8 bits each, most significant
// first.  A pass histograms, per column, the next 8-bit digit of every value
// whose higher bits equal the prefix fixed so far, then one wave per column
// scans the 256 bins, finds the bin holding the remaining rank, appends its
// digit to the prefix and subtracts the counts below it.
//
// Work split of a histogram pass: a workgroup owns 64 columns (one per lane,
// so a wave reads 256 contiguous bytes of a row) and a chunk of rows; the 4
// waves walk the chunk's rows and count in an LDS histogram [256][64]
// (lanes of one wave never share an address), which is flushed to the global
// histogram [K][256] with one atomic per non-zero bin.  The row chunks give
// the launch enough workgroups to fill the chip for any column count.
#include <cmath>
#include <mutex>

#include "common.h"

namespace oq {
namespace {

constexpr int kSlab = 64;           // columns per workgroup
constexpr int kMaxRowSplits = 2048;  // row chunks per column slab

constexpr int kGroups = 256;        // row groups per column (their maxima use the histogram's memory)
constexpr int kTopCap = 2048;       // values re-read per column: (m - 1) groups
constexpr int kTopWaves = 8;        // columns per workgroup of the second kernel

// gmax[g][col] = max |Y| bits of rows [g gs, (g + 1) gs) of a column; VEC
// columns per lane (4: 16-byte loads, rows 16-byte aligned and K % 4 == 0).
template <int VEC>
__global__ __launch_bounds__(64) void top_group_kernel(const float* __restrict__ Y, int64_t n, int64_t K, int64_t ldy,
                                                       int gs, uint32_t* __restrict__ gmax) {
  typedef float vec __attribute__((ext_vector_type(VEC)));
  const int64_t col = (static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x) * VEC;
  if (col >= K) return;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * gs;
  const int64_t r1 = r0 + gs < n ? r0 + gs : n;
  const float* y = Y + col;
  uint32_t best[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) best[e] = 0;
  auto take = [&](const vec& v) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) best[e] = max(best[e], __float_as_uint(v[e]) & 0x7FFFFFFFu);
  };
  int64_t r = r0;
  for (; r + 8 <= r1; r += 8) {  // eight rows in flight
    vec v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const vec*>(y + (r + u) * ldy);
#pragma unroll
    for (int u = 0; u < 8; ++u) take(v[u]);
  }
  for (; r < r1; ++r) take(*reinterpret_cast<const vec*>(y + r * ldy));
  uint32_t* o = gmax + static_cast<int64_t>(blockIdx.y) * K + col;
#pragma unroll
  for (int e = 0; e < VEC; ++e) o[e] = best[e];
}

// One wave per column: L, the values above L, the m-th largest.
__global__ __launch_bounds__(64 * kTopWaves) void top_select_kernel(const float* __restrict__ Y, int64_t n, int64_t K,
                                                                    int64_t ldy, int gs, int groups, int m,
                                                                    const uint32_t* __restrict__ gmax, double qmax,
                                                                    float* __restrict__ out) {
  __shared__ uint32_t cand[kTopWaves][kTopCap];
  __shared__ uint16_t glist[kTopWaves][kGroups];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t col = static_cast<int64_t>(blockIdx.x) * kTopWaves + wv;
  if (col >= K) return;  // (no barrier below: each wave keeps to its own LDS)
  const uint64_t below = (uint64_t(1) << lane) - 1;
  uint32_t g[kGroups / 64];
#pragma unroll
  for (int i = 0; i < kGroups / 64; ++i) {
    const int gi = i * 64 + lane;
    g[i] = gi < groups ? gmax[static_cast<int64_t>(gi) * K + col] : 0u;
  }
  // The largest L with at least m maxima >= L (m <= groups; absent groups are 0).
  uint32_t L = 0;
  for (int bit = 30; bit >= 0; --bit) {
    const uint32_t t = L | (1u << bit);
    int c = 0;
#pragma unroll
    for (int i = 0; i < kGroups / 64; ++i) c += __popcll(__ballot(g[i] >= t));
    if (c >= m) L = t;
  }
  int ng = 0;
#pragma unroll
  for (int i = 0; i < kGroups / 64; ++i) {
    const bool hit = g[i] > L;
    const uint64_t b = __ballot(hit);
    if (hit) glist[wv][ng + __popcll(b & below)] = static_cast<uint16_t>(i * 64 + lane);
    ng += __popcll(b);
  }
  // ng < m, so the re-read values number at most (m - 1) gs <= kTopCap.
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  int nc = 0;
  const int total = ng * gs;
  for (int i0 = 0; i0 < total; i0 += 256) {  // four loads in flight
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + 64 * u + lane, ic = i < total ? i : 0;
      const int64_t r = static_cast<int64_t>(glist[wv][ic / gs]) * gs + ic % gs;
      v[u] = __float_as_uint(Y[(r < n ? r : n - 1) * ldy + col]) & 0x7FFFFFFFu;
      if (i >= total || r >= n) v[u] = 0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool hit = v[u] > L;
      const uint64_t b = __ballot(hit);
      if (hit) cand[wv][nc + __popcll(b & below)] = v[u];
      nc += __popcll(b);
    }
  }
  uint32_t res = L;
  if (nc >= m) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t v0 = lane < nc ? cand[wv][lane] : 0u;
    res = 0;
    for (int bit = 30; bit >= 0; --bit) {
      const uint32_t t = res | (1u << bit);
      int c = __popcll(__ballot(v0 >= t));
      for (int i0 = 64; i0 < nc; i0 += 64) c += __popcll(__ballot(i0 + lane < nc && cand[wv][i0 + lane] >= t));
      if (c >= m) res = t;
    }
  }
  if (lane == 0) out[col] = static_cast<float>(static_cast<double>(__uint_as_float(res)) / qmax);
}

// hist = 0, prefix = 0, rank = k for every column.
__global__ __launch_bounds__(256) void quantile_init_kernel(uint32_t* __restrict__ hist, uint32_t* __restrict__ prefix,
                                                            uint32_t* __restrict__ rank, int64_t K, uint32_t k) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < K * 64) reinterpret_cast<uint4*>(hist)[i] = make_uint4(0, 0, 0, 0);
  if (i < K) {
    prefix[i] = 0;
    rank[i] = k;
  }
}

__global__ __launch_bounds__(256) void quantile_hist_kernel(const float* __restrict__ Y, int64_t n, int64_t K,
                                                            int64_t ldy, int64_t chunk, int shift,
                                                            const uint32_t* __restrict__ prefix,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256 * kSlab];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t col = static_cast<int64_t>(blockIdx.x) * kSlab + lane;
  const bool cok = col < K;
  for (int i = threadIdx.x; i < 256 * kSlab; i += 256) h[i] = 0;
  __syncthreads();
  const uint32_t pre = cok ? prefix[col] : 0u;
  const uint32_t hi_mask = shift >= 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * chunk;
  const int64_t r1 = r0 + chunk < n ? r0 + chunk : n;
  const float* yc = Y + (cok ? col : 0);
  // Four rows per wave in flight: loads first, then the counts.
  int64_t r = r0 + wv;
  for (; r + 12 < r1; r += 16) {
    uint32_t b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) b[u] = __float_as_uint(yc[(r + 4 * u) * ldy]) & 0x7FFFFFFFu;
    if (cok) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if ((b[u] & hi_mask) == pre) atomicAdd(&h[((b[u] >> shift) & 255u) * kSlab + lane], 1u);
    }
  }
  for (; r < r1; r += 4) {
    const uint32_t b = __float_as_uint(yc[r * ldy]) & 0x7FFFFFFFu;
    if (cok && (b & hi_mask) == pre) atomicAdd(&h[((b >> shift) & 255u) * kSlab + lane], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 256 * kSlab; i += 256) {
    const int d = i / kSlab, c = i % kSlab;
    const uint32_t v = h[i];
    const int64_t cc = static_cast<int64_t>(blockIdx.x) * kSlab + c;
    if (v != 0u && cc < K) atomicAdd(&hist[cc * 256 + d], v);
  }
}

// One wave per column: lane l holds bins 4l .. 4l + 3.  Finds the bin that
// holds the remaining rank, updates prefix and rank, clears the column's
// histogram for the next pass; the last pass writes prefix / q_max.
__global__ __launch_bounds__(256) void quantile_select_kernel(uint32_t* __restrict__ hist, int64_t K, int shift,
                                                              uint32_t* __restrict__ prefix,
                                                              uint32_t* __restrict__ rank, bool last, double qmax,
                                                              float* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t col = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (col >= K) return;
  uint4* hc = reinterpret_cast<uint4*>(hist + col * 256) + lane;
  const uint4 c = *hc;
  const uint32_t s = c.x + c.y + c.z + c.w;
  // Inclusive prefix sum of s over the wave.
  uint32_t incl = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  const uint32_t k = rank[col];
  const uint64_t hit = __ballot(incl >= k);
  // The candidates of this pass number at least k, so some lane reaches k;
  // a histogram that does not (it cannot happen) selects the top bin.
  const int L = hit ? __builtin_ctzll(hit) : 63;
  const uint32_t below_lane = __shfl(incl - s, L, 64);
  const uint4 cl = make_uint4(__shfl(c.x, L, 64), __shfl(c.y, L, 64), __shfl(c.z, L, 64), __shfl(c.w, L, 64));
  *hc = make_uint4(0, 0, 0, 0);
  if (lane != 0) return;
  uint32_t acc = below_lane;
  int d = 4 * L;
  const uint32_t cc[4] = {cl.x, cl.y, cl.z, cl.w};
  int i = 0;
  for (; i < 3; ++i) {
    if (acc + cc[i] >= k) break;
    acc += cc[i];
  }
  d += i;
  const uint32_t p = prefix[col] | (static_cast<uint32_t>(d) << shift);
  prefix[col] = p;
  rank[col] = k - acc;
  if (last) out[col] = static_cast<float>(static_cast<double>(__uint_as_float(p)) / qmax);
}

// Launches of one calibration: work = hist [K][256] | prefix [K] | rank [K].
int calibrate_launch(const float* Y, int64_t n, int64_t K, int64_t ldy, double p, float qmax, float* delta,
                     uint32_t* work, hipStream_t s) {
  // Nearest rank: the k-th smallest with k = ceil(p n / 100), in [1, n].  p is
  // taken to 1e-6 percent and the product formed in integers (pm n <= 1e8 *
  // INT32_MAX < 2^63): in floating point 99.9 / 100 * 1000 = 999.0000000000001
  // would round up to the maximum.
  const int64_t pm = std::llround(p * 1e6);
  int64_t k = (pm * n + 99999999) / 100000000;
  if (k < 1) k = 1;
  if (k > n) k = n;
  // The m-th largest by group maxima where m groups exist and the re-read
  // values fit the second kernel's LDS (99.9%: n <= 22 thousand rows).  Ahead of the
  // radix route wherever it applies, us: 22000 x 64 at 99.9% 19 / 62, a million x 64 at
  // 100% (one group maximum each; 256 waves in flight) 199 / 600.
  const int64_t m = n - k + 1, gs = (n + kGroups - 1) / kGroups, groups = (n + gs - 1) / gs;
  if (m <= groups && (m - 1) * gs <= kTopCap) {
    const bool vec = K % 4 == 0 && ldy % 4 == 0 && aligned(Y, 16);
    const int64_t cpw = vec ? 256 : 64;
    const dim3 grid(static_cast<unsigned>((K + cpw - 1) / cpw), static_cast<unsigned>(groups));
    if (vec) hipLaunchKernelGGL(top_group_kernel<4>, grid, dim3(64), 0, s, Y, n, K, ldy, static_cast<int>(gs), work);
    else hipLaunchKernelGGL(top_group_kernel<1>, grid, dim3(64), 0, s, Y, n, K, ldy, static_cast<int>(gs), work);
    hipLaunchKernelGGL(top_select_kernel, dim3(static_cast<unsigned>((K + kTopWaves - 1) / kTopWaves)),
                       dim3(64 * kTopWaves), 0, s, Y, n, K, ldy, static_cast<int>(gs), static_cast<int>(groups),
                       static_cast<int>(m), work, static_cast<double>(qmax), delta);
    return launch_status();
  }
  uint32_t* hist = work;
  uint32_t* prefix = hist + K * 256;
  uint32_t* rank = prefix + K;
  hipLaunchKernelGGL(quantile_init_kernel, dim3(static_cast<unsigned>((K * 64 + 255) / 256)), dim3(256), 0, s,
                     hist, prefix, rank, K, static_cast<uint32_t>(k));
  const int64_t slabs = (K + kSlab - 1) / kSlab;
  // Enough row chunks for ~8 workgroups per CU over the slabs, at least 64
  // rows per chunk.
  int64_t splits = (2048 + slabs - 1) / slabs;
  if (splits > kMaxRowSplits) splits = kMaxRowSplits;
  if (splits > (n + 63) / 64) splits = (n + 63) / 64;
  if (splits < 1) splits = 1;
  const int64_t chunk = (n + splits - 1) / splits;
  splits = (n + chunk - 1) / chunk;
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    hipLaunchKernelGGL(quantile_hist_kernel, dim3(static_cast<unsigned>(slabs), static_cast<unsigned>(splits)),
                       dim3(256), 0, s, Y, n, K, ldy, chunk, shift, prefix, hist);
    hipLaunchKernelGGL(quantile_select_kernel, dim3(static_cast<unsigned>((K + 3) / 4)), dim3(256), 0, s, hist,
                       K, shift, prefix, rank, pass == 3, static_cast<double>(qmax), delta);
  }
  return launch_status();
}

// Argument checks shared by both entry points (before any launch).
int calibrate_check(const float* Y, int64_t n, int64_t K, int64_t ldy, double p, float qmax, float* delta) {
  if (n < 0 || K < 0 || n > INT32_MAX || K > (int64_t(1) << 24) || ldy < K) return OQ_ERR_SHAPE;
  if (!(p > 0.0 && p <= 100.0) || !(qmax > 0.0f) || !std::isfinite(qmax)) return OQ_ERR_ARG;
  if (K == 0) return OQ_OK;
  if (n == 0) return OQ_ERR_SHAPE;  // no order statistic of an empty column
  if (!Y || !delta) return OQ_ERR_NULL;
  if (!aligned(Y, 4) || !aligned(delta, 4)) return OQ_ERR_ALIGN;
  return OQ_OK;
}

// ---- the allocation-free variant -----------------------------------------
// Its histogram, prefixes and ranks live in a file-scope device array, one
// copy per GPU for the life of the process, sized for kScratchMaxK columns.
constexpr int64_t kScratchMaxK = 16384;
constexpr size_t kScratchWords = static_cast<size_t>(kScratchMaxK) * (256 + 2);  // 16.9 MB
constexpr int kMaxDevices = 64;

// The array's address on each device, from hipGetSymbolAddress with that
// device current (the host-side name is not a device address).
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};

}  // namespace
}  // namespace oq

static __device__ __align__(256) uint32_t scratch[oq::kScratchWords];

namespace oq {
namespace {

int scratch_for_current_device(uint32_t** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return OQ_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return OQ_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return OQ_ERR_HIP;
    g_scratch_ptr[dev] = static_cast<uint32_t*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return OQ_OK;
}

}  // namespace
}  // namespace oq

extern "C" size_t oq_calibrate_workspace_bytes(int64_t K) {
  if (K <= 0) return 0;
  return static_cast<size_t>(K) * (256 + 2) * sizeof(uint32_t);
}

extern "C" int oq_calibrate_step_scales(const float* Y, int64_t n, int64_t K, int64_t ldy, double p, float qmax,
                                        float* delta, void* work, size_t work_bytes, void* stream) {
  int e = oq::calibrate_check(Y, n, K, ldy, p, qmax, delta);
  if (e != OQ_OK || K == 0) return e;
  if (!work) return OQ_ERR_NULL;
  if (work_bytes < oq_calibrate_workspace_bytes(K)) return OQ_ERR_SHAPE;
  if (!oq::aligned(work, 16)) return OQ_ERR_ALIGN;
  if ((e = oq::device_check()) != OQ_OK) return e;
  return oq::calibrate_launch(Y, n, K, ldy, p, qmax, delta, static_cast<uint32_t*>(work),
                              static_cast<hipStream_t>(stream));
}

extern "C" int oq_calibrate_step_scales_noalloc(const float* Y, int64_t n, int64_t K, int64_t ldy, double p,
                                                float qmax, float* delta, void* stream) {
  int e = oq::calibrate_check(Y, n, K, ldy, p, qmax, delta);
  if (e != OQ_OK || K == 0) return e;
  if (K > oq::kScratchMaxK) return OQ_ERR_WORKSPACE;
  if ((e = oq::device_check()) != OQ_OK) return e;
  uint32_t* work = nullptr;
  if ((e = oq::scratch_for_current_device(&work)) != OQ_OK) return e;
  return oq::calibrate_launch(Y, n, K, ldy, p, qmax, delta, work, static_cast<hipStream_t>(stream));
}
