// Offline preparation of a weight for the full composite rotation, on the
// GPU (Section 4.1: zigzag permutation P from weight channel energies, the
// per-block factor U_b of the SVD of each block's weight rows, R_b = U_b H_64 /
// 8, and the fold W' = W P R_hat with round-to-nearest per output channel).
//
// Orientation: the weight is stored [N][K] (output-major), so input channel j
// is column j and block b's weight rows (the paper's C_in x C_out orientation)
// are the 64 columns perm[64 b .. 64 b + 63] of W, a 64 x N matrix W_b.
//
//  * Channel energies e_j = sum_n W[n][j]^2 in fp64, one workgroup per 16 to
//    64 columns with a fixed reduction order (deterministic, so exactly equal
//    columns get exactly equal energies).
//  * Zigzag order: the descending rank of e_j (ties to the lower index) by
//    counting, then the snake deal over the blocks.
//  * U_b: the left singular vectors of W_b are the eigenvectors of the Gram
//    matrix G_b = W_b W_b^T, with sigma_i^2 its eigenvalues.  G_b is formed on
//    the fp64 matrix cores (exact products of fp16 values) and diagonalized by
//    the cyclic Jacobi method in fp64: the 2016 index pairs in 63 steps of 32
//    disjoint pairs (round-robin order), the 32 rotations of a step applied
//    together, until 63 steps in a row (every pair) apply none (at most 40
//    sweeps).  Eigenpairs are ordered by descending eigenvalue (ties to the
//    lower index) and each vector's sign is fixed so that its entry of largest
//    magnitude (the first on ties) is positive.  One workgroup per block.
//  * R_b = U_b H_64 / 8 in fp64, rounded once to fp16 (round half to even)
//    and stored column-major per block, the operand the online composite
//    kernel reads.
//  * The fold and RTN are the online composite rotate-quantize applied to
//    the weight rows (s_t = 1): codes per output channel and its scale.
#include <cmath>

#include "common.h"

extern "C" int oq_rotate_quantize_act_composite(const void* X, int64_t M, int64_t K, int64_t ldx,
                                                const int32_t* perm, const void* Rt, const float* s_table,
                                                int32_t t, uint8_t* Xq, float* x_scale, void* stream);

namespace oq {
namespace {

constexpr int kB = 64;        // block size (the paper's)
constexpr int kLd = kB + 1;   // padded LDS row of the 64 x 64 matrices
constexpr int kMaxSteps = 40 * 63;

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double h2d(uint16_t h) {
  return static_cast<double>(static_cast<float>(__builtin_bit_cast(_Float16, h)));
}

// fp64 -> fp16 bits, one rounding (half to even), from the fp64 bit pattern:
// the 53-bit significand is shifted to the fp16 precision of the value's
// binade (10 fraction bits for normal fp16, fewer for subnormal) with an
// exact remainder test.  |x| >= 65520 gives infinity (R_b entries are
// bounded by 1).
__device__ __forceinline__ uint16_t f64_to_f16_rne(double x) {
  const uint64_t bits = __double_as_longlong(x);
  const uint16_t sign = static_cast<uint16_t>((bits >> 48) & 0x8000u);
  const int e = static_cast<int>((bits >> 52) & 0x7FF);
  if (e == 0) return sign;                    // zero or fp64 subnormal: far below fp16 range
  if (e == 0x7FF) return sign | 0x7C00u;      // inf (NaN is not produced here)
  const int ue = e - 1023;                    // unbiased exponent
  if (ue >= 16) return sign | 0x7C00u;
  const uint64_t mant = (bits & ((uint64_t(1) << 52) - 1)) | (uint64_t(1) << 52);
  const int e16 = ue + 15;                    // biased fp16 exponent if normal
  const int shift = e16 >= 1 ? 42 : 42 + (1 - e16);
  if (shift >= 54) return sign;               // below half the smallest subnormal
  uint64_t q = mant >> shift;
  const uint64_t rem = mant & ((uint64_t(1) << shift) - 1);
  const uint64_t half = uint64_t(1) << (shift - 1);
  if (rem > half || (rem == half && (q & 1))) ++q;
  uint32_t r;
  if (e16 >= 1) r = (static_cast<uint32_t>(e16) << 10) + static_cast<uint32_t>(q) - 1024u;  // carry moves the exponent
  else r = static_cast<uint32_t>(q);                                                       // subnormal (q = 1024: smallest normal)
  if (r >= 0x7C00u) r = 0x7C00u;
  return sign | static_cast<uint16_t>(r);
}

// e[j] = sum_n W[n][j]^2: CW columns per workgroup, 1024 / CW threads per column
// (thread g takes rows g, g + 1024 / CW, ...), their sums added in order.  Bound
// by the one read of W, if the columns are spread over the chip and a row's
// piece is not so narrow that its cache lines are fetched several times: 2560 x
// 2048 at 64 / 32 / 16 columns 8.4 / 5.3 / 9.8 us, 2560 x 1024 8.3 / 5.1 / 3.7, 4096 x 4096 14.2 /
// 12.6 / 22.0, 2048 x 16384 11.0 / 21.4 / 43.0.
template <int CW>
__global__ __launch_bounds__(1024) void energy_kernel(const uint16_t* __restrict__ W, int64_t N, int64_t K,
                                                      int64_t ldw, double* __restrict__ e) {
  constexpr int G = 1024 / CW;
  __shared__ double part[G][CW];
  const int c = threadIdx.x % CW, g = threadIdx.x / CW;
  const int64_t col = static_cast<int64_t>(blockIdx.x) * CW + c;
  const bool ok = col < K;
  const uint16_t* wc = W + (ok ? col : 0);
  double acc = 0.0;
  int64_t n = g;
  for (; n + 7 * G < N; n += 8 * G) {
    uint16_t w[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) w[u] = wc[(n + G * u) * ldw];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc = fma(h2d(w[u]), h2d(w[u]), acc);
  }
  for (; n < N; n += G) {
    const double a = h2d(wc[n * ldw]);
    acc = fma(a, a, acc);
  }
  part[g][c] = acc;
  __syncthreads();
  if (threadIdx.x < CW && ok) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < G; ++w) s += part[w][c];
    e[col] = s;
  }
}

// perm from energies: 64 channels per workgroup; wave w counts the channels of
// its sixteenth of every 2048, or of as many as there are (sixteenths of 2048 left
// one wave to count all of a short row: K = 64 7.3 -> 2.3 us, 1024 9.0 -> 8.4), that rank
// before channel j (larger energy, or equal energy and lower index); rank i is
// dealt to round i / nb and block (round even ? i % nb : nb - 1 - i % nb), slot round.
__global__ __launch_bounds__(1024) void zigzag_kernel(const double* __restrict__ e, int K, int nb,
                                                      int32_t* __restrict__ perm) {
  __shared__ double chunk[2048];
  __shared__ int part[16][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = blockIdx.x * 64 + lane;
  const double ej = j < K ? e[j] : 0.0;
  int rank = 0;
  for (int base = 0; base < K; base += 2048) {
    const int len = K - base < 2048 ? K - base : 2048;
    __syncthreads();
    for (int i = threadIdx.x; i < len; i += 1024) chunk[i] = e[base + i];
    __syncthreads();
    // (Every channel before this workgroup's 64 wins a tie, every one after loses it.)
    const int per = (len + 15) / 16, i0 = min(wv * per, len), i1 = min(i0 + per, len);
    const int lo = min(max(static_cast<int>(blockIdx.x) * 64 - base, i0), i1);
    const int hi = min(max(static_cast<int>(blockIdx.x) * 64 + 64 - base, i0), i1);
#pragma unroll 8
    for (int i = i0; i < lo; ++i) rank += chunk[i] >= ej ? 1 : 0;
    for (int i = lo; i < hi; ++i) rank += (chunk[i] > ej || (chunk[i] == ej && base + i < j)) ? 1 : 0;
#pragma unroll 8
    for (int i = hi; i < i1; ++i) rank += chunk[i] > ej ? 1 : 0;
  }
  part[wv][lane] = rank;
  __syncthreads();
  if (wv != 0 || j >= K) return;
  rank = 0;
  for (int w = 0; w < 16; ++w) rank += part[w][lane];
  const int c = K / nb;
  const int r = rank / nb, p = rank % nb;
  const int b = (r & 1) ? nb - 1 - p : p;
  perm[b * c + r] = j;
}

// G_b = W_b W_b^T in fp64 on v_mfma_f64_16x16x4 (lane l holds row k = l / 16 of
// W_b^T, column l % 16, for either operand; element i of the result is row
// 4 i + l / 16, column l % 16): the ten 16 x 16 tiles on and above the diagonal.
// The waves take four rows in turn each; their sums are added in order.  Bound
// by the gather (2-byte loads of permuted columns: each touches a cache line of
// its own, which other blocks want at about the same time), so by the number of
// gathers while there are few blocks to spread over the chip, and by how much
// of the weight is in flight, and stays in L2, when there are many.
//
// gram_split_kernel: the tiles of a block on six workgroups, each with at most
// two groups of 16 columns to gather: (0,0)(0,1), (1,1)(1,2), (2,2)(2,3),
// (3,3)(3,0), (0,2), (1,3).  Three gathers of the weight in all.
// gram_kernel: one workgroup per block, one gather.
// us, six workgroups / one: 2560 x 1024 29 / 87, 2560 x 2048 49 / 93, 1024 x 3072 57 / 45,
// 4096 x 4096 325 / 171, 8192 x 8192 2314 / 421, 2048 x 16384 1166 / 134.
__device__ __forceinline__ int gram_column(const int32_t* perm, int b, int g, int lane, int64_t K) {
  const int32_t c = perm[b * kB + 16 * g + (lane & 15)];  // clamped: an out-of-range entry cannot address outside the row
  return c < 0 ? 0 : (c >= K ? static_cast<int>(K - 1) : c);
}

__global__ __launch_bounds__(512) void gram_split_kernel(const uint16_t* __restrict__ W, int64_t N, int64_t K,
                                                         int64_t ldw, const int32_t* __restrict__ perm,
                                                         double* __restrict__ G) {
  __shared__ double red[8][2][256];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x / 6, t = blockIdx.x % 6;
  const int g0 = t < 4 ? t : t - 4, g1 = t < 4 ? (t + 1) & 3 : t - 2;
  const bool two = t < 4;  // the diagonal tile (g0, g0) as well
  const int kr = lane >> 4;
  const uint16_t *w0 = W + gram_column(perm, b, g0, lane, K), *w1 = W + gram_column(perm, b, g1, lane, K);
  v4d d = {0, 0, 0, 0}, x = {0, 0, 0, 0};
  constexpr int UN = 8;
  for (int64_t n0 = 4 * wv; n0 < N; n0 += 32 * UN) {
    uint16_t a[UN], c[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t n = n0 + 32 * u + kr, nc = n < N ? n : N - 1;  // clamped row; its value is replaced by 0
      a[u] = w0[nc * ldw];
      c[u] = w1[nc * ldw];
      if (n >= N) a[u] = c[u] = 0;
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const double av = h2d(a[u]), cv = h2d(c[u]);
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(av, cv, x, 0, 0, 0);
      if (two) d = __builtin_amdgcn_mfma_f64_16x16x4f64(av, av, d, 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    red[wv][0][(4 * i + kr) * 16 + (lane & 15)] = x[i];
    red[wv][1][(4 * i + kr) * 16 + (lane & 15)] = d[i];
  }
  __syncthreads();
  const int which = threadIdx.x >> 8, el = threadIdx.x & 255;
  if (which && !two) return;
  double s = 0.0;
  for (int w = 0; w < 8; ++w) s += red[w][which][el];
  const int i = 16 * g0 + el / 16, j = 16 * (which ? g0 : g1) + el % 16;
  double* g = G + static_cast<int64_t>(b) * kB * kB;
  g[i * kB + j] = s;
  if (!which) g[j * kB + i] = s;
}

__global__ __launch_bounds__(256) void gram_kernel(const uint16_t* __restrict__ W, int64_t N, int64_t K, int64_t ldw,
                                                   const int32_t* __restrict__ perm, double* __restrict__ G) {
  constexpr int WV = 4, UN = 4;
  __shared__ double red[WV][256];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x, kr = lane >> 4;
  const uint16_t* w[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) w[g] = W + gram_column(perm, b, g, lane, K);
  v4d x[4][4];  // (on and above the diagonal)
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int f = g; f < 4; ++f) x[g][f] = v4d{0, 0, 0, 0};
  for (int64_t n0 = 4 * wv; n0 < N; n0 += 4 * WV * UN) {
    uint16_t a[UN][4];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int64_t n = n0 + 4 * WV * u + kr, nc = n < N ? n : N - 1;  // clamped row; its values are replaced by 0
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        a[u][g] = w[g][nc * ldw];
        if (n >= N) a[u][g] = 0;
      }
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      double v[4];
#pragma unroll
      for (int g = 0; g < 4; ++g) v[g] = h2d(a[u][g]);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int f = g; f < 4; ++f) x[g][f] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[g], v[f], x[g][f], 0, 0, 0);
    }
  }
  double* gb = G + static_cast<int64_t>(b) * kB * kB;
  const int el = threadIdx.x;
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int f = g; f < 4; ++f) {
      __syncthreads();  // (the last tile's sums are read)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wv][(4 * i + kr) * 16 + (lane & 15)] = x[g][f][i];
      __syncthreads();
      double s = 0.0;
#pragma unroll
      for (int v = 0; v < WV; ++v) s += red[v][el];
      const int i = 16 * g + el / 16, j = 16 * f + el % 16;
      gb[i * kB + j] = s;
      if (g != f) gb[j * kB + i] = s;
    }
}

// The round-robin order: at step k (mod 63) slot m of 32 holds the pair (p, q) =
// (k, 63) for m = 0 and ((k + m) mod 63, (k - m) mod 63) otherwise; every
// unordered pair meets in exactly one of 63 steps.
__device__ __forceinline__ int rr_top(int k, int m) { return k + m < 63 ? k + m : k + m - 63; }
__device__ __forceinline__ int rr_bot(int k, int m) { return m == 0 ? 63 : k - m >= 0 ? k - m : k - m + 63; }

// Lane i gets lane i + 1's (i - 1's) double.
template <int CTRL>
__device__ __forceinline__ double wave_move(double x) {
  const uint64_t u = __double_as_longlong(x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), CTRL, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(static_cast<uint64_t>(hi) << 32 | lo);
}
__device__ __forceinline__ double wave_next(double x) { return wave_move<0x130>(x); }
__device__ __forceinline__ double wave_prev(double x) { return wave_move<0x138>(x); }

// One Newton step for y ~ 1 / sqrt(x).
__device__ __forceinline__ double rsq_step(double x, double y) { return y * fma(-0.5 * x * y, y, 1.5); }

// Eigenvectors of G_b (GU holds G on entry, U on return), one workgroup of 14
// waves per 64-channel block.  What bounds it is the chain of steps: 500 or so,
// each depending on the last.  So a step is one barrier long and three parts of
// it run side by side:
//  * wave 0 forms the next step's rotations, from this step's matrix and
//    rotations (the three entries that each coming pair needs, ten old ones
//    per pair) rather than waiting for the updated matrix;
//  * waves 1-5 apply this step's rotations to the matrix, from one LDS buffer to
//    the other, in 2 x 2 blocks of slot pairs (rows and columns at once); by
//    symmetry only slot pairs at cyclic distance 0 .. 16 are computed, each
//    written twice;
//  * waves 6-13 rotate the accumulated vectors in registers: a lane is a slot
//    and holds eight rows' pairs (four per half wave), and since the slots'
//    contents move by one slot per step, the columns move by one lane.
// 2560 x 2048 (32 blocks, 410 steps): 324 us, 0.8 us a step, the length of wave
// 0's chain of fp64 operations.  (Before: parameters, column pass and row pass in turn through LDS with three
// barriers, the Gram matrix on the vector units of the same 32 workgroups:
// 1456 us with the Gram matrix, now 51 us in a kernel of its own.)
__global__ __launch_bounds__(896) void block_eig_kernel(double* __restrict__ GU, double* __restrict__ lam) {
  // The Jacobi iterate, double-buffered.  Rows unpadded: a lane's row and column both move by one
  // per slot, up or down, so the lanes' addresses are 65 or 63 doubles apart: no bank conflicts
  // (a row of 65 doubles would put them 64 apart, all on one bank).
  __shared__ double A[2][kB][kB];
  __shared__ double2 rot[2][32];     // (c, s) of the slots, double-buffered
  __shared__ int done[2];
  __shared__ double dg[kB];
  __shared__ int rk[kB];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 31;
  double* g = GU + static_cast<int64_t>(blockIdx.x) * kB * kB;
  for (int i = tid; i < kB * kB; i += 896) A[0][i >> 6][i & 63] = g[i];
  if (tid < 32) rot[0][tid] = make_double2(1.0, 0.0);
  __syncthreads();
  double trace = 0.0;
  for (int i = 0; i < kB; ++i) trace += A[0][i][i];
  const double floor2 = 0x1p-104 * trace * trace;

  // (wave 0) Rotations of step k + 1 (mod 63) from the matrix and rotations of
  // step k.  A pair is rotated unless |a_pq| is negligible against the diagonal,
  // |a_pq| <= 2^-53 sqrt(|a_pp a_qq|), or at the rounding level of the whole
  // matrix, |a_pq| <= 2^-52 trace(G) (entries of a numerically null eigenspace
  // would otherwise keep rotating among themselves).  The angle needs no last
  // bit, since what it leaves of the pair stays in the matrix (the hardware's
  // reciprocals and one Newton step give a few ulp); c^2 + s^2 = 1 does, so c
  // takes two Newton steps.  Returns whether any pair rotates.
  auto next_rotations = [&](int x, int k) -> bool {
    // Slots that hold the coming pair now: its top comes from the top of slot
    // m + 1 (slot 31: its own bottom), its bottom from the bottom of slot m - 1
    // (slot 1: the top of slot 0; slot 0 keeps 63).
    const int sa = m < 31 ? m + 1 : 31, sb = m < 2 ? 0 : m - 1;
    const double2 ra = rot[x][sa], rb = rot[x][sb];
    const int ap = rr_top(k, sa), aq = rr_bot(k, sa), bp = rr_top(k, sb), bq = rr_bot(k, sb);
    const double (*M)[kB] = A[x];
    const double app = M[ap][ap], apq = M[ap][aq], aqq = M[aq][aq];
    const double bpp = M[bp][bp], bpq = M[bp][bq], bqq = M[bq][bq];
    const double x00 = M[ap][bp], x01 = M[ap][bq], x10 = M[aq][bp], x11 = M[aq][bq];
    const double a0 = m < 31 ? ra.x : ra.y, a1 = m < 31 ? -ra.y : ra.x;    // top (c, -s) / bottom (s, c)
    const double b0 = m == 1 ? rb.x : rb.y, b1 = m == 1 ? -rb.y : rb.x;
    const double dp = a0 * a0 * app + 2.0 * a0 * a1 * apq + a1 * a1 * aqq;
    const double dq = b0 * b0 * bpp + 2.0 * b0 * b1 * bpq + b1 * b1 * bqq;
    const double o = a0 * (b0 * x00 + b1 * x01) + a1 * (b0 * x10 + b1 * x11);
    double c = 1.0, s = 0.0;
    // t = tan of the angle: the smaller root, sign(d) 2 o / (|d| + sqrt(d^2 + 4 o^2)).
    if (o * o > fmax(0x1p-106 * fabs(dp * dq), floor2)) {
      const double d = dq - dp, o2 = 2.0 * o, r = fma(d, d, o2 * o2);
      const double den = fma(r, rsq_step(r, __builtin_amdgcn_rsq(r)), fabs(d));
      double rc = __builtin_amdgcn_rcp(den);
      rc = rc * fma(-den, rc, 2.0);
      const double t = (d >= 0.0 ? o2 : -o2) * rc;
      const double u = fma(t, t, 1.0);
      c = rsq_step(u, rsq_step(u, __builtin_amdgcn_rsq(u)));
      s = t * c;
      if (s == 0.0) c = 1.0;
    }
    if (lane < 32) rot[x ^ 1][m] = make_double2(c, s);
    return __ballot(s != 0.0) != 0;
  };

  // Rows 8 (wv - 6) + 4 (lane / 32) + j of V in slot order: top and bottom of slot m.
  const int vr = 8 * (wv - 6) + 4 * (lane >> 5);
  double vt[4], vb[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    vt[j] = vr + j == rr_top(0, m) ? 1.0 : 0.0;
    vb[j] = vr + j == rr_bot(0, m) ? 1.0 : 0.0;
  }

  // Step 0's rotations: the identity applied to G as if at step 62.  (rot[0] is
  // the identity; the result lands in rot[1], so the matrix moves there too.)
  int idle = 0;  // (wave 0) steps in a row without a rotation
  if (wv == 0) {
    idle = next_rotations(0, 62) ? 0 : 1;
    if (lane == 0) done[1] = 0;
  }
  for (int i = tid; i < kB * kB; i += 896) A[1][i >> 6][i & 63] = A[0][i >> 6][i & 63];
  __syncthreads();
  int k = 0, x = 1;
  for (int step = 0; step < kMaxSteps && !done[x]; ++step) {
    if (wv == 0) {
      idle = next_rotations(x, k) ? 0 : idle + 1;
      if (lane == 0) done[x ^ 1] = idle >= 63;
    } else if (wv < 6) {
      // Distances dist = 2 i + lane / 32, i = wv - 1 and wv + 4; both loaded before either is stored.
      const double2 r1 = rot[x][m];
      const int p1 = rr_top(k, m), q1 = rr_bot(k, m);
      double2 r2[2];
      int p2[2], q2[2];
      double e00[2], e01[2], e10[2], e11[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int m2 = (m + 2 * (wv - 1 + 5 * i) + (lane >> 5)) & 31;
        r2[i] = rot[x][m2];
        p2[i] = rr_top(k, m2);
        q2[i] = rr_bot(k, m2);
        e00[i] = A[x][p1][p2[i]];
        e01[i] = A[x][p1][q2[i]];
        e10[i] = A[x][q1][p2[i]];
        e11[i] = A[x][q1][q2[i]];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int dist = 2 * (wv - 1 + 5 * i) + (lane >> 5);
        const double f00 = r2[i].x * e00[i] - r2[i].y * e01[i], f01 = r2[i].y * e00[i] + r2[i].x * e01[i];
        const double f10 = r2[i].x * e10[i] - r2[i].y * e11[i], f11 = r2[i].y * e10[i] + r2[i].x * e11[i];
        const double h00 = r1.x * f00 - r1.y * f10, h11 = r1.y * f01 + r1.x * f11;
        const double h01 = r1.x * f01 - r1.y * f11;
        double h10 = r1.y * f00 + r1.x * f10;
        // In a slot's own block both off-diagonal entries are one value, what the rotation left of the pair.
        if (dist == 0) h10 = h01;
        if (dist < 16 || (dist == 16 && m < 16)) {
          A[x ^ 1][p1][p2[i]] = h00;
          A[x ^ 1][p1][q2[i]] = h01;
          A[x ^ 1][q1][p2[i]] = h10;
          A[x ^ 1][q1][q2[i]] = h11;
          if (dist != 0) {
            A[x ^ 1][p2[i]][p1] = h00;
            A[x ^ 1][q2[i]][p1] = h01;
            A[x ^ 1][p2[i]][q1] = h10;
            A[x ^ 1][q2[i]][q1] = h11;
          }
        }
      }
    } else {
      const double2 r = rot[x][m];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double t = r.x * vt[j] - r.y * vb[j], bo = r.y * vt[j] + r.x * vb[j];
        const double down = m == 0 ? t : bo;  // moves to the next slot's bottom
        const double up = wave_next(t), pr = wave_prev(down);
        vt[j] = m == 31 ? bo : up;
        vb[j] = m == 0 ? bo : pr;
      }
    }
    __syncthreads();
    x ^= 1;
    k = k == 62 ? 0 : k + 1;
  }

  // Order and signs.
  if (tid < kB) dg[tid] = A[x][tid][tid];
  if (wv >= 6) {
    const int p = rr_top(k, m), q = rr_bot(k, m);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      A[x ^ 1][vr + j][p] = vt[j];
      A[x ^ 1][vr + j][q] = vb[j];
    }
  }
  __syncthreads();
  const double (*V)[kB] = A[x ^ 1];
  if (tid < kB) {
    const double li = dg[tid];
    int r = 0;
    for (int j = 0; j < kB; ++j) r += (dg[j] > li || (dg[j] == li && j < tid)) ? 1 : 0;
    rk[tid] = r;
    lam[static_cast<int64_t>(blockIdx.x) * kB + r] = li;
    int arg = 0;
    double best = -1.0;
    for (int rr = 0; rr < kB; ++rr) {
      const double a = fabs(V[rr][tid]);
      if (a > best) {
        best = a;
        arg = rr;
      }
    }
    A[x][0][tid] = V[arg][tid] < 0.0 ? -1.0 : 1.0;  // (the iterate is spent) the sign of column tid
  }
  __syncthreads();
  for (int it = tid; it < kB * kB; it += 896) {
    const int r = it >> 6, i = it & 63;
    g[r * kB + rk[i]] = A[x][0][i] * V[r][i];
  }
}

// Rt[b][j][r] = fp16(R_b[r][j]), R_b[r][j] = sum_i U_b[r][i] H[i][j] / 8: four
// workgroups per block, a wave per column j, a lane per row r.
__global__ __launch_bounds__(1024) void block_rot_kernel(const double* __restrict__ U, uint16_t* __restrict__ Rt) {
  __shared__ double u[kB][kLd];
  const int b = blockIdx.x >> 2, lane = threadIdx.x & 63;
  const int j = (blockIdx.x & 3) * 16 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double* ub = U + static_cast<int64_t>(b) * kB * kB;
  for (int i = threadIdx.x; i < kB * kB; i += 1024) u[i >> 6][i & 63] = ub[i];
  __syncthreads();
  double s = 0.0;
#pragma unroll 16
  for (int i = 0; i < kB; ++i) s += (__popc(i & j) & 1) ? -u[lane][i] : u[lane][i];
  Rt[(static_cast<int64_t>(b) * kB + j) * kB + lane] = f64_to_f16_rne(s * 0.125);
}

int check_weight(const void* W, int64_t N, int64_t K, int64_t ldw) {
  if (N < 1 || K < kB || K % kB != 0 || K > 16384 || ldw < K) return OQ_ERR_SHAPE;
  if (!W) return OQ_ERR_NULL;
  if (!aligned(W, 2)) return OQ_ERR_ALIGN;
  return OQ_OK;
}

}  // namespace
}  // namespace oq

extern "C" int oq_channel_energy(const void* W, int64_t N, int64_t K, int64_t ldw, double* energy, void* stream) {
  if (N < 1 || K < 1 || ldw < K) return OQ_ERR_SHAPE;
  if (!W || !energy) return OQ_ERR_NULL;
  if (!oq::aligned(W, 2) || !oq::aligned(energy, 8)) return OQ_ERR_ALIGN;
  int st = oq::device_check();
  if (st != OQ_OK) return st;
  hipStream_t h = static_cast<hipStream_t>(stream);
  const uint16_t* w = static_cast<const uint16_t*>(W);
#define OQ_ENERGY(CW) \
  hipLaunchKernelGGL(oq::energy_kernel<CW>, dim3(static_cast<unsigned>((K + CW - 1) / CW)), dim3(1024), 0, h, w, N, K, ldw, energy)
  // The widest piece that still gives about a hundred workgroups.
  if (K >= 6144) OQ_ENERGY(64);
  else if (K >= 2048) OQ_ENERGY(32);
  else OQ_ENERGY(16);
#undef OQ_ENERGY
  return oq::launch_status();
}

extern "C" int oq_zigzag_permutation(const double* energy, int64_t K, int32_t block, int32_t* perm, void* stream) {
  if (block < 1 || K < block || K % block != 0 || K > 65536) return OQ_ERR_SHAPE;
  if (!energy || !perm) return OQ_ERR_NULL;
  if (!oq::aligned(energy, 8) || !oq::aligned(perm, 4)) return OQ_ERR_ALIGN;
  int st = oq::device_check();
  if (st != OQ_OK) return st;
  hipLaunchKernelGGL(oq::zigzag_kernel, dim3(static_cast<unsigned>((K + 63) / 64)), dim3(1024), 0,
                     static_cast<hipStream_t>(stream), energy, static_cast<int>(K), static_cast<int>(K / block),
                     perm);
  return oq::launch_status();
}

extern "C" int oq_block_svd(const void* W, int64_t N, int64_t K, int64_t ldw, const int32_t* perm, int32_t block,
                            double* U, double* sigma2, void* stream) {
  int st = oq::check_weight(W, N, K, ldw);
  if (st != OQ_OK) return st;
  if (block != oq::kB) return OQ_ERR_SHAPE;
  if (!perm || !U || !sigma2) return OQ_ERR_NULL;
  if (!oq::aligned(perm, 4) || !oq::aligned(U, 8) || !oq::aligned(sigma2, 8)) return OQ_ERR_ALIGN;
  if ((st = oq::device_check()) != OQ_OK) return st;
  // (U holds the Gram matrices in between.)
  hipStream_t h = static_cast<hipStream_t>(stream);
  const uint16_t* w = static_cast<const uint16_t*>(W);
  const unsigned nb = static_cast<unsigned>(K / oq::kB);
  if (nb > 32) hipLaunchKernelGGL(oq::gram_kernel, dim3(nb), dim3(256), 0, h, w, N, K, ldw, perm, U);
  else hipLaunchKernelGGL(oq::gram_split_kernel, dim3(6 * nb), dim3(512), 0, h, w, N, K, ldw, perm, U);
  hipLaunchKernelGGL(oq::block_eig_kernel, dim3(nb), dim3(896), 0, h, U, sigma2);
  return oq::launch_status();
}

extern "C" int oq_block_rotations(const double* U, int64_t K, int32_t block, uint16_t* Rt, void* stream) {
  if (block != oq::kB || K < oq::kB || K % oq::kB != 0 || K > 16384) return OQ_ERR_SHAPE;
  if (!U || !Rt) return OQ_ERR_NULL;
  if (!oq::aligned(U, 8) || !oq::aligned(Rt, 2)) return OQ_ERR_ALIGN;
  int st = oq::device_check();
  if (st != OQ_OK) return st;
  hipLaunchKernelGGL(oq::block_rot_kernel, dim3(static_cast<unsigned>(4 * (K / oq::kB))), dim3(1024), 0,
                     static_cast<hipStream_t>(stream), U, Rt);
  return oq::launch_status();
}

extern "C" size_t oq_prepare_weights_workspace_bytes(int64_t K) {
  if (K <= 0) return 0;
  // energies K doubles, U K * 64 doubles, sigma^2 K doubles
  return static_cast<size_t>(K) * (1 + oq::kB + 1) * sizeof(double);
}

extern "C" int oq_prepare_weights_composite(const void* W, int64_t N, int64_t K, int64_t ldw, int32_t* perm,
                                            uint16_t* Rt, uint8_t* Wq, float* w_scale, void* work,
                                            size_t work_bytes, void* stream) {
  int st = oq::check_weight(W, N, K, ldw);
  if (st != OQ_OK) return st;
  if (!perm || !Rt || !Wq || !w_scale || !work) return OQ_ERR_NULL;
  if (work_bytes < oq_prepare_weights_workspace_bytes(K)) return OQ_ERR_SHAPE;
  if (ldw % 8 != 0) return OQ_ERR_ALIGN;
  if (!oq::aligned(W, 16) || !oq::aligned(perm, 4) || !oq::aligned(Rt, 16) || !oq::aligned(Wq, 16) ||
      !oq::aligned(w_scale, 4) || !oq::aligned(work, 16))
    return OQ_ERR_ALIGN;
  if ((st = oq::device_check()) != OQ_OK) return st;
  double* energy = static_cast<double*>(work);
  double* U = energy + K;
  double* sigma2 = U + K * oq::kB;
  if ((st = oq_channel_energy(W, N, K, ldw, energy, stream)) != OQ_OK) return st;
  if ((st = oq_zigzag_permutation(energy, K, oq::kB, perm, stream)) != OQ_OK) return st;
  if ((st = oq_block_svd(W, N, K, ldw, perm, oq::kB, U, sigma2, stream)) != OQ_OK) return st;
  if ((st = oq_block_rotations(U, K, oq::kB, Rt, stream)) != OQ_OK) return st;
  return oq_rotate_quantize_act_composite(W, N, K, ldw, perm, Rt, nullptr, 0, Wq, w_scale, stream);
}
