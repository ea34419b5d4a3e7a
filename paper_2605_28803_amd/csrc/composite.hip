// Online composite rotation of Section 4.1 with per-token int4 quantization.
//
// eq:transform: X' = X P R_hat with P a channel permutation and R_hat =
// BlockDiag(R_1 .. R_K), R_b = U_b H_c (eq:blockdiag), block size c = 64 (the
// paper's setting).  Then the step scale and the per-token quantizer of
// Section 4.2 (eq:scale, eq:quant; eq:perstep_scale in its per-(layer, step)
// scalar form): z = s_t y, Delta = max|z| / 7, q = round_half_even(z / Delta),
// x_scale = Delta / s_t.
//
// Three kernels.  rq_composite_x_kernel takes rows of one chunk (K = 512, 1024,
// 1536, 2048, 3072, 4096: every y in registers, one pass), and above K = 4096
// rows split into chunks of channels whose workgroups exchange their partial
// row maxima (one pass, each y computed once).  Other K up to 4096 take
// rq_composite1_kernel (whole rows in LDS, one pass), other K above it the
// two-pass rq_composite_kernel described next.
//
// Two-pass kernel: one workgroup of four waves owns RW rows.  The rows are
// staged in LDS as fp16.  Pass 1: wave w takes the 64-channel blocks b = w, w + 4, ...; for
// each, the A fragment (rows x 32 permuted channels) is gathered from LDS
// through perm (the v_mfma_f32_16x16x32_f16 operand layout: lane l holds row
// l % 16 and the 8 consecutive k values 8 (l / 16) .. + 7), the B fragment is
// one 16-byte load of the column-major block matrix (lane l holds output
// column l % 16 and the same 8 k values), and the 16 x 16 fp32 products give
// y for four 16-channel column groups; only the row maxima are kept.  The
// maxima are combined across lanes and waves, then pass 2 recomputes y and
// writes int8 codes to LDS, which are packed two per byte and stored
// coalesced.  fp16 x fp16 products are exact in fp32; the 64-term sums are
// the only rounding of the transform.  Rows past RW in a fragment are zero.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "rq_device.h"

namespace oq {
namespace {

typedef _Float16 c8h __attribute__((ext_vector_type(8)));
typedef float c4f __attribute__((ext_vector_type(4)));

constexpr int kCB = 64;  // block size c

// Address-space-qualified pointers for the direct global -> LDS load builtin.
typedef __attribute__((address_space(1))) void gmem_void;
typedef __attribute__((address_space(3))) void lds_void;

// Two nibbles per byte from 16 two's-complement int8 codes (even channel low).
__device__ __forceinline__ uint32_t pack4codes(uint32_t d) {
  const uint32_t e = d & 0x000F000Fu;          // codes 0, 2 -> bits 0-3, 16-19
  const uint32_t o = (d >> 4) & 0x00F000F0u;   // codes 1, 3 -> bits 4-7, 20-23
  const uint32_t t = e | o;
  return (t & 0xFFu) | ((t >> 8) & 0xFF00u);
}

template <int RW, int KMAX, int G, bool GATHER>
__global__ __launch_bounds__(256) void rq_composite_kernel(const uint16_t* __restrict__ X, int64_t M, int K,
                                                           int64_t ldx, const int32_t* __restrict__ perm,
                                                           const uint16_t* __restrict__ Rt, float s_t,
                                                           uint8_t* __restrict__ Xq, float* __restrict__ xs) {
  // fp16 rows, padded by 16 bytes: the 16 rows of a gather read the same
  // permuted column, and the pad puts them in different LDS banks.
  constexpr int XS = KMAX + 8;
  __shared__ __attribute__((aligned(16))) uint16_t sx[GATHER ? RW * XS : 8];
  __shared__ __attribute__((aligned(16))) int32_t sp[GATHER ? KMAX : 4];  // the permutation
  __shared__ __attribute__((aligned(16))) uint8_t sc[RW * KMAX / 2];  // packed codes
  __shared__ float red[4][16];
  __shared__ float gscale[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * RW;
  const int nb = K / kCB;
  const int vpr = K / 8;  // 16-byte pieces per row

  // Stage the rows (rows past M are zeros) and the permutation (clamped into
  // range: a non-permutation keeps every access inside the staged rows).
  if constexpr (GATHER) {
    for (int p0 = tid; p0 < RW * vpr; p0 += 256 * 8) {
      uint4 v[8];
      bool ok[8];
  #pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int p = p0 + u * 256;
        const int r = p / vpr, c8 = p - r * vpr;
        ok[u] = p < RW * vpr && row0 + r < M;
        const int64_t gr = ok[u] ? row0 + r : 0;
        v[u] = *reinterpret_cast<const uint4*>(X + gr * ldx + (ok[u] ? c8 * 8 : 0));
      }
  #pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int p = p0 + u * 256;
        const int r = p / vpr, c8 = p - r * vpr;
        if (p < RW * vpr) *reinterpret_cast<uint4*>(&sx[r * XS + c8 * 8]) = ok[u] ? v[u] : make_uint4(0, 0, 0, 0);
      }
    }
    for (int k4 = tid; k4 < K / 4; k4 += 256) {
      int4 pv = *reinterpret_cast<const int4*>(perm + 4 * k4);
      pv.x = min(max(pv.x, 0), K - 1);
      pv.y = min(max(pv.y, 0), K - 1);
      pv.z = min(max(pv.z, 0), K - 1);
      pv.w = min(max(pv.w, 0), K - 1);
      *reinterpret_cast<int4*>(&sp[4 * k4]) = pv;
    }
  }
  __syncthreads();

  const int r16 = lane & 15, q = lane >> 4;
  const bool rok = r16 < RW;
  const uint16_t* xrow = &sx[GATHER && rok ? r16 * XS : 0];

  // A fragment: rows x 32 permuted channels of block b, k step kk (without a
  // permutation: one 16-byte load per lane from global memory, rows past RW
  // or M zero).
  const bool gok = rok && row0 + r16 < M;
  auto gather = [&](int b, int kk) -> c8h {
    if constexpr (!GATHER) {
      const c8h v = *reinterpret_cast<const c8h*>(X + (gok ? row0 + r16 : 0) * ldx + b * kCB + kk * 32 + 8 * q);
      return gok ? v : c8h{};
    }
    const int k0 = b * kCB + kk * 32 + 8 * q;
    const int4 pa = *reinterpret_cast<const int4*>(&sp[k0]);
    const int4 pb = *reinterpret_cast<const int4*>(&sp[k0 + 4]);
    const int idx[8] = {pa.x, pa.y, pa.z, pa.w, pb.x, pb.y, pb.z, pb.w};
    c8h a;
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = __builtin_bit_cast(_Float16, rok ? xrow[idx[j]] : uint16_t(0));
    return a;
  };
  // B fragments of G consecutive blocks of this wave (blocks b0 + 4 g), all
  // loads issued together; blocks past the end read block 0 and are skipped.
  c8h bf[G][4][2];
  auto load_b = [&](int b0) {
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
      const int b = b0 + 4 * gi < nb ? b0 + 4 * gi : 0;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
          bf[gi][cb][kk] = *reinterpret_cast<const c8h*>(
              Rt + (static_cast<int64_t>(b) * kCB + cb * 16 + r16) * kCB + kk * 32 + 8 * q);
    }
  };

  // Pass 1: row maxima of |y|.  The B fragments of the next group are in
  // flight while the current group is multiplied (the scheduling barrier
  // keeps the loads ahead of the products).
  float amax[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  load_b(wave);
  for (int b0 = wave; b0 < nb; b0 += 4 * G) {
    c8h cur[G][4][2];
#pragma unroll
    for (int gi = 0; gi < G; ++gi)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        cur[gi][cb][0] = bf[gi][cb][0];
        cur[gi][cb][1] = bf[gi][cb][1];
      }
    if (b0 + 4 * G < nb) load_b(b0 + 4 * G);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
      const int b = b0 + 4 * gi;
      if (b < nb) {
        const c8h a0 = gather(b, 0), a1 = gather(b, 1);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          c4f acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, cur[gi][cb][0], c4f{0, 0, 0, 0}, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, cur[gi][cb][1], acc, 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) amax[e] = fmaxf(amax[e], fabsf(acc[e]));
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float m = amax[e];
    m = fmaxf(m, rqd::lane_xor<1>(m));
    m = fmaxf(m, rqd::lane_xor<2>(m));
    m = fmaxf(m, rqd::lane_xor<4>(m));
    m = fmaxf(m, rqd::lane_xor<8>(m));
    if (r16 == 0) red[wave][4 * q + e] = m;
  }
  __syncthreads();
  if (tid < 16) {
    const float m = fmaxf(fmaxf(red[0][tid], red[1][tid]), fmaxf(red[2][tid], red[3][tid]));
    // a_z = max|s_t y|, Delta = a_z / 7, code = round(y s_t / Delta).
    const float a_z = m * s_t;
    const float delta = a_z / 7.0f;
    gscale[tid] = delta > 0.0f ? s_t / delta : 0.0f;
    if (tid < RW && row0 + tid < M) xs[row0 + tid] = delta / s_t;
  }
  __syncthreads();

  // Pass 2: codes.  Lanes r16 and r16 ^ 1 hold channels 2i and 2i + 1 of
  // the same row; the even lane packs both into one byte.
  float g[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) g[e] = gscale[4 * q + e];
  load_b(wave);
  for (int b0 = wave; b0 < nb; b0 += 4 * G) {
    c8h cur[G][4][2];
#pragma unroll
    for (int gi = 0; gi < G; ++gi)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        cur[gi][cb][0] = bf[gi][cb][0];
        cur[gi][cb][1] = bf[gi][cb][1];
      }
    if (b0 + 4 * G < nb) load_b(b0 + 4 * G);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int gi = 0; gi < G; ++gi) {
      const int b = b0 + 4 * gi;
      if (b < nb) {
        const c8h a0 = gather(b, 0), a1 = gather(b, 1);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          c4f acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, cur[gi][cb][0], c4f{0, 0, 0, 0}, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, cur[gi][cb][1], acc, 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t code = __float_as_uint(fmaf(acc[e], g[e], rqd::kRoundMagic)) & 0xFu;
            const uint32_t other = __float_as_uint(rqd::lane_xor<1>(__uint_as_float(code)));
            const int row = 4 * q + e;
            if (row < RW && (r16 & 1) == 0)
              sc[row * (KMAX / 2) + (b * kCB + cb * 16 + r16) / 2] = static_cast<uint8_t>(code | (other << 4));
          }
        }
      }
    }
  }
  __syncthreads();

  // Store 16 packed bytes per thread.
  const int ppr = K / 32;
  for (int p = tid; p < RW * ppr; p += 256) {
    const int r = p / ppr, c32 = p - r * ppr;
    if (row0 + r >= M) continue;
    *reinterpret_cast<uint4*>(Xq + (row0 + r) * static_cast<int64_t>(K / 2) + c32 * 16) =
        *reinterpret_cast<const uint4*>(&sc[r * (KMAX / 2) + c32 * 16]);
  }
}

// Single pass for K <= 4096: eight waves, RG row groups of 16 rows (RW = 16 RG
// rows per workgroup), every y value kept in registers until the row maxima
// are known, so each block matrix is read once per workgroup and reused by
// the RG row groups.  Codes are packed across lanes (channel pairs, then 4
// and 8 channels) and stored as dwords by the lanes holding the first of 8
// channels.
template <int RG, int KMAX, bool GATHER>
__global__ __launch_bounds__(512) void rq_composite1_kernel(const uint16_t* __restrict__ X, int64_t M, int K,
                                                            int64_t ldx, const int32_t* __restrict__ perm,
                                                            const uint16_t* __restrict__ Rt, float s_t,
                                                            uint8_t* __restrict__ Xq, float* __restrict__ xs) {
  constexpr int WAVES = 8, RW = 16 * RG, XS = KMAX + 8;
  constexpr int NBW = KMAX / kCB / WAVES;  // blocks per wave at K = KMAX
  __shared__ __attribute__((aligned(16))) uint16_t sx[GATHER ? RW * XS : 8];
  __shared__ __attribute__((aligned(16))) int32_t sp[GATHER ? KMAX : 4];
  __shared__ float red[WAVES][RW];
  __shared__ float gscale[RW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * RW;
  const int nb = K / kCB;
  const int vpr = K / 8;

  if constexpr (GATHER) {
    for (int p0 = tid; p0 < RW * vpr; p0 += 512 * 8) {
      uint4 v[8];
      bool ok[8];
  #pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int p = p0 + u * 512;
        const int r = p / vpr, c8 = p - r * vpr;
        ok[u] = p < RW * vpr && row0 + r < M;
        const int64_t gr = ok[u] ? row0 + r : 0;
        v[u] = *reinterpret_cast<const uint4*>(X + gr * ldx + (ok[u] ? c8 * 8 : 0));
      }
  #pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int p = p0 + u * 512;
        const int r = p / vpr, c8 = p - r * vpr;
        if (p < RW * vpr) *reinterpret_cast<uint4*>(&sx[r * XS + c8 * 8]) = ok[u] ? v[u] : make_uint4(0, 0, 0, 0);
      }
    }
    for (int k4 = tid; k4 < K / 4; k4 += 512) {
      int4 pv = *reinterpret_cast<const int4*>(perm + 4 * k4);
      pv.x = min(max(pv.x, 0), K - 1);
      pv.y = min(max(pv.y, 0), K - 1);
      pv.z = min(max(pv.z, 0), K - 1);
      pv.w = min(max(pv.w, 0), K - 1);
      *reinterpret_cast<int4*>(&sp[4 * k4]) = pv;
    }
  }
  __syncthreads();

  const int r16 = lane & 15, q = lane >> 4;
  // Without a permutation (X already in the permuted channel order): the A
  // fragment of rows rg*16 .. + 15 and k step kk of block b is one 16-byte
  // load per lane straight from global memory; rows past M read row 0 and
  // are zeroed where used.
  bool rv[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) rv[rg] = row0 + rg * 16 + r16 < M;
  auto load_a = [&](int b, c8h (&f)[RG][2]) {
    const int bb = b < nb ? b : 0;
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      const int64_t gr = rv[rg] ? row0 + rg * 16 + r16 : 0;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        f[rg][kk] = *reinterpret_cast<const c8h*>(X + gr * ldx + bb * kCB + kk * 32 + 8 * q);
    }
  };
  auto gather = [&](int b, int kk, int rg) -> c8h {
    const int k0 = b * kCB + kk * 32 + 8 * q;
    const int4 pa = *reinterpret_cast<const int4*>(&sp[k0]);
    const int4 pb = *reinterpret_cast<const int4*>(&sp[k0 + 4]);
    const int idx[8] = {pa.x, pa.y, pa.z, pa.w, pb.x, pb.y, pb.z, pb.w};
    const uint16_t* xrow = &sx[(rg * 16 + r16) * XS];
    c8h a;
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = __builtin_bit_cast(_Float16, xrow[idx[j]]);
    return a;
  };

  c4f y[NBW][4][RG];
  float amax[RG][4];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg)
#pragma unroll
    for (int e = 0; e < 4; ++e) amax[rg][e] = 0.0f;
  // The block matrix fragments of block i + 1 are loaded while block i is
  // multiplied (blocks past the end read block 0 and are not used).
  auto load_b = [&](int b, c8h (&f)[4][2]) {
    const int bb = b < nb ? b : 0;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        f[cb][kk] = *reinterpret_cast<const c8h*>(Rt + (static_cast<int64_t>(bb) * kCB + cb * 16 + r16) * kCB +
                                                  kk * 32 + 8 * q);
  };
  c8h bnext[4][2];
  c8h anext[GATHER ? 1 : RG][2];
  load_b(wave, bnext);
  if constexpr (!GATHER) load_a(wave, anext);
#pragma unroll
  for (int i = 0; i < NBW; ++i) {
    const int b = wave + WAVES * i;
    c8h bf[4][2];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      bf[cb][0] = bnext[cb][0];
      bf[cb][1] = bnext[cb][1];
    }
    c8h af[GATHER ? 1 : RG][2];
    if constexpr (!GATHER) {
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        af[rg][0] = anext[rg][0];
        af[rg][1] = anext[rg][1];
      }
    }
    if (i + 1 < NBW) {
      load_b(b + WAVES, bnext);
      if constexpr (!GATHER) load_a(b + WAVES, anext);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (b < nb) {
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        c8h a0, a1;
        if constexpr (GATHER) {
          a0 = gather(b, 0, rg);
          a1 = gather(b, 1, rg);
        } else {
          a0 = rv[rg] ? af[rg][0] : c8h{};
          a1 = rv[rg] ? af[rg][1] : c8h{};
        }
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          c4f acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, bf[cb][0], c4f{0, 0, 0, 0}, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, bf[cb][1], acc, 0, 0, 0);
          y[i][cb][rg] = acc;
#pragma unroll
          for (int e = 0; e < 4; ++e) amax[rg][e] = fmaxf(amax[rg][e], fabsf(acc[e]));
        }
      }
    }
  }
#pragma unroll
  for (int rg = 0; rg < RG; ++rg)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float m = amax[rg][e];
      m = fmaxf(m, rqd::lane_xor<1>(m));
      m = fmaxf(m, rqd::lane_xor<2>(m));
      m = fmaxf(m, rqd::lane_xor<4>(m));
      m = fmaxf(m, rqd::lane_xor<8>(m));
      if (r16 == 0) red[wave][rg * 16 + 4 * q + e] = m;
    }
  __syncthreads();
  if (tid < RW) {
    float m = red[0][tid];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) m = fmaxf(m, red[w][tid]);
    const float a_z = m * s_t;
    const float delta = a_z / 7.0f;
    gscale[tid] = delta > 0.0f ? s_t / delta : 0.0f;
    if (row0 + tid < M) xs[row0 + tid] = delta / s_t;
  }
  __syncthreads();

#pragma unroll
  for (int i = 0; i < NBW; ++i) {
    const int b = wave + WAVES * i;
    if (b < nb) {
#pragma unroll
      for (int rg = 0; rg < RG; ++rg)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = rg * 16 + 4 * q + e;
          const float g = gscale[row];
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) {
            // code of channel b*64 + cb*16 + r16; pack 8 consecutive channels
            uint32_t c = __float_as_uint(fmaf(y[i][cb][rg][e], g, rqd::kRoundMagic)) & 0xFu;
            c |= __float_as_uint(rqd::lane_xor<1>(__uint_as_float(c))) << 4;
            c |= __float_as_uint(rqd::lane_xor<2>(__uint_as_float(c))) << 8;
            c |= __float_as_uint(rqd::lane_xor<4>(__uint_as_float(c))) << 16;
            if ((r16 & 7) == 0 && row0 + row < M)
              *reinterpret_cast<uint32_t*>(Xq + (row0 + row) * static_cast<int64_t>(K / 2) +
                                           (b * kCB + cb * 16 + r16) / 2) = c;
          }
        }
    }
  }
}

// ---------------------------------------------------------------------------
// Rows wider than a workgroup can stage (K > 4096, and K = 4096 with P
// folded): the permuted channels of a row are cut into nq = K / C chunks of C
// channels, and each (tile of R = 16 RG rows, chunk) pair is one workgroup, so
// that each block matrix R_b is read once per R rows instead of once per few
// rows.  The nq workgroups of a tile exchange their rows' partial maxima and
// each quantizes its own chunk, so every y value is computed once and stays in
// registers.
//
// Staging with the online permutation: a row at a time goes through registers
// (16-byte loads, four rows ahead) into a raw LDS row, from which each thread
// gathers the C / 512 channels of its consecutive positions (2-byte LDS reads)
// and stores them with one write into the chunk's row.  The whole row is read
// by each of the nq workgroups (from L2: the tile's workgroups are placed on
// one XCD, adjacent in dispatch order).  What the other forms are bound by:
// storing from registers the channels that fall into the chunk under a mask
// keeps 1 / nq of the store lanes at work (4080 x 16384: 166 us); loading them
// from global memory 2 bytes each in source order runs at one lane per clock
// (120 us); this, with the block matrices and the packing below, takes 84 us.
// At C = 4096 and K = 16384 the two buffers are all of the LDS, so the chunk's
// rows are not padded: 16-byte piece p of row r is stored at p ^ r, which
// spreads the operand reads of 16 rows over the banks.  Without a permutation
// the chunk's columns are copied directly to the same places.
//
// Exchange: through the call's own output, so that any number of calls may run
// at once.  Until chunk q stores its codes, its part of the tile's first row of
// Xq carries the maxima of the tile's R rows and, behind them, the nq chunks'
// acknowledgements (together in a few cache lines: a word in each row instead
// took up to 40% longer).  comp_words_kernel sets
// them all to kWait (sign bit set; a maximum is >= 0).  A workgroup publishes
// its maxima, waits for every chunk's, acknowledges to the others that it has
// read them, and stores its codes over the words once all the others have
// acknowledged.  The tile's workgroups are dispatched together (ids x + 8 (nq t' +
// q) for XCD x), so a workgroup only waits for partners dispatched at the same
// time.  The waits poll with agent-scope atomic loads and are bounded, and a
// workgroup that gives up goes on without storing codes, so the grid always
// drains.  The token scales are formed by atomic maximum over the bits, from 0:
// chunk 0 gives the scale, any chunk that gives up a NaN, which is above every
// number, so no order of the two hides it.  (Chunk 0 waiting for a word from
// every other took 0.7 us more.)  give_up: the chunk that gives up at once on the maxima (chunk p: p) or
// on the acknowledgements (nq + p); -1 but in a test.
// ---------------------------------------------------------------------------
constexpr int kPollLimit = 1 << 20;

// Workgroup barrier for LDS alone: loads from global memory stay in flight
// (__syncthreads waits for them).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

constexpr uint32_t kWait = 0xFFFFFFFFu, kNaN = 0x7FC00000u;

// Word w of chunk p's part of a row of codes (C / 8 words).
__device__ __forceinline__ uint32_t* exchange_word(uint8_t* Xq, int64_t row, int K, int C, int p, int w) {
  return reinterpret_cast<uint32_t*>(Xq + row * (K / 2) + p * (C / 2)) + w;
}
__device__ __forceinline__ void exchange_store(uint32_t* w, uint32_t v) {
  __hip_atomic_store(w, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits until a word is no longer kWait, for at most kPollLimit polls.
__device__ __forceinline__ uint32_t exchange_wait(const uint32_t* w, bool give_up) {
  if (give_up) return kWait;
  uint32_t v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int it = 0; (v >> 31) && it < kPollLimit; ++it) {
    __builtin_amdgcn_s_sleep(2);
    v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return v;
}

// n = nq (R + nq) > R words per tile, and the token scales.
__global__ __launch_bounds__(256) void comp_words_kernel(uint8_t* __restrict__ Xq, float* __restrict__ xs, int64_t M,
                                                         int ntiles, int K, int C, int nq, int R) {
  const int per = R + nq, n = nq * per;
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x, tile = i / n;
  if (i < M) xs[i] = 0.0f;
  const int in = static_cast<int>(i - tile * n);
  if (tile < ntiles) *exchange_word(Xq, tile * R, K, C, in / per, in % per) = kWait;
}

template <int RG, int C, bool GATHER, int WAVES, int PF, int KMAX>
__global__ __launch_bounds__(64 * WAVES) void rq_composite_x_kernel(
    const uint16_t* __restrict__ X, int64_t M, int K, int64_t ldx, const int32_t* __restrict__ perm,
    const uint16_t* __restrict__ Rt, float s_t, uint8_t* __restrict__ Xq, float* __restrict__ xs, int nq, int ntiles,
    int give_up) {
  constexpr int NT = 64 * WAVES;
  constexpr int R = 16 * RG, XS = C;
  constexpr int NBC = C / kCB, NBW = NBC / WAVES;  // blocks per chunk, per wave
  static_assert(NBW >= 1 && NBC % WAVES == 0, "chunk blocks per wave");
  static_assert(PF >= 2, "block matrix ring depth");
  // The chunk's rows (later the codes); then a region for, in turn, the raw rows
  // (with the permutation), 2 KB of block matrix per wave, the maxima and scales.
  // RPS raw rows (KMAX >= K channels each) are staged at a time.
  constexpr int RPS = KMAX >= 1024 ? 16384 / KMAX : 16;
  constexpr int AUXB = GATHER && RPS * KMAX * 2 > WAVES * 2048 ? RPS * KMAX * 2 : WAVES * 2048;
  __shared__ __attribute__((aligned(16))) uint8_t smem[R * XS * 2 + AUXB];
  constexpr int NQMAX = 16384 / C;
  static_assert((WAVES * R + R + NQMAX * R + 1) * 4 <= AUXB && WAVES * 2048 <= AUXB, "auxiliary region");
  static_assert(R + NQMAX <= C / 8, "exchange words");
  uint16_t* sx = reinterpret_cast<uint16_t*>(smem);
  uint16_t* raw = sx + R * XS;
  float (*red)[R] = reinterpret_cast<float (*)[R]>(raw);
  float* gscale = reinterpret_cast<float*>(raw) + WAVES * R;
  float* pmax = gscale + R;  // [nq][R] the chunks' maxima
  int& timed_out = *reinterpret_cast<int*>(pmax + NQMAX * R);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int xcd = blockIdx.x % 8, idx = blockIdx.x / 8;
  const int q = idx % nq;
  const int tile = (idx / nq) * 8 + xcd;
  if (tile >= ntiles) return;  // every workgroup of such a tile id returns
  const int64_t row0 = static_cast<int64_t>(tile) * R;
  const int cbase = q * C;

  // ---- y = x_chunk . BlockDiag(R_b) for this wave's NBW blocks, kept in
  // registers.  The block matrices run through a ring of PF register stages;
  // the first PF - 1 are requested before the rows are staged.
  const int r16 = lane & 15, qq = lane >> 4;
  const int wb0 = wave * NBW;  // first block of this wave within the chunk
  // (Block matrices are loaded as they lie in memory, 1 KB of consecutive bytes
  // per instruction, and turned into operands through LDS: loaded directly, the
  // lanes of an operand are 128 bytes apart and a load takes 64 cycles instead of 16.)
  auto load_b = [&](int i, c8h (&f)[4][2]) {
    const uint16_t* rb = Rt + (static_cast<int64_t>(q) * NBC + wb0 + (i < NBW ? i : 0)) * kCB * kCB + 8 * lane;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int h = 0; h < 2; ++h) f[cb][h] = *reinterpret_cast<const c8h*>(rb + cb * 1024 + h * 512);
  };
  c8h bring[PF][4][2];
#pragma unroll
  for (int i = 0; i < PF - 1; ++i)
    if (i < NBW) load_b(i, bring[i]);
  // ---- Stage the chunk of R rows in LDS (rows past M read row M - 1; their
  // results are not stored).
  if constexpr (GATHER) {
    constexpr int EPT = C / NT;                  // positions per thread
    static_assert(EPT >= 1 && C % NT == 0, "positions per thread");
    // Stored VW at a time, so that a store stays within a 16-byte piece.
    constexpr int VW = EPT % 8 == 0 ? 8 : EPT % 4 == 0 ? 4 : EPT % 2 == 0 ? 2 : 1;
    typedef uint16_t vec __attribute__((ext_vector_type(VW)));
    int idx[EPT];                                // their channels (clamped: never outside the row)
#pragma unroll
    for (int e = 0; e < EPT; ++e) idx[e] = min(max(perm[cbase + tid * EPT + e], 0), K - 1);
    static_assert(R % RPS == 0, "rows per step");
    constexpr int STEPS = R / RPS, AHEAD = STEPS < 4 ? STEPS : 4;
    constexpr int PPR = KMAX / 8;                // 16-byte pieces of a raw row
    constexpr int PMAX = RPS * PPR / NT;         // pieces of a step per thread
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    u4 v[AHEAD][PMAX];
#define OQ_LOAD_STEP(ST, S)                                                                    \
  {                                                                                            \
    _Pragma("unroll") for (int i_ = 0; i_ < PMAX; ++i_) {                                      \
      const int p_ = tid + NT * i_, rl_ = (ST) * RPS + p_ / PPR, c_ = p_ % PPR;                \
      const int64_t gr_ = row0 + rl_ < M ? row0 + rl_ : M - 1;                                 \
      v[S][i_] = *reinterpret_cast<const u4*>(X + gr_ * ldx + (8 * c_ < K ? 8 * c_ : 0));      \
    }                                                                                          \
  }
    static_for<AHEAD>([&](auto S_) { OQ_LOAD_STEP(decltype(S_)::value, decltype(S_)::value) });
    static_for<STEPS>([&](auto R_) {  // (constant ring slots: the loads stay in registers)
      constexpr int st = decltype(R_)::value, sl = st % AHEAD;
#pragma unroll
      for (int i = 0; i < PMAX; ++i)
        *reinterpret_cast<u4*>(raw + 8 * (tid + NT * i)) = v[sl][i];  // (past K: never gathered)
      if constexpr (st + AHEAD < STEPS) OQ_LOAD_STEP(st + AHEAD, sl)
      lds_barrier();
#pragma unroll
      for (int rl = 0; rl < RPS; ++rl) {
        const int r = st * RPS + rl;
#pragma unroll
        for (int e0 = 0; e0 < EPT; e0 += VW) {
          vec g;
          if constexpr (VW == 1) {
            g = raw[rl * KMAX + idx[e0]];
          } else {
#pragma unroll
            for (int e = 0; e < VW; ++e) g[e] = raw[rl * KMAX + idx[e0 + e]];
          }
          const int at = tid * EPT + e0;         // piece at / 8 moves to (at / 8) ^ (r mod 16)
          *reinterpret_cast<vec*>(sx + r * XS + (at ^ ((r & 15) * 8))) = g;
        }
      }
      lds_barrier();
    });
#undef OQ_LOAD_STEP
  } else {
    // The chunk's columns of each row go straight from global memory into
    // LDS (global_load_lds_dwordx4: lane l's 16 bytes land at the given LDS
    // address + 16 l), 1 KB (512 channels) per wave instruction, with no
    // registers in between, so every row of the tile is in flight at once.
    // Rows past M read row M - 1 (their results are not stored).
    constexpr int PARTS = C / 512;
    for (int j = wave; j < R * PARTS; j += WAVES) {
      const int r = j / PARTS, h = j % PARTS;
      const int64_t gr = row0 + r < M ? row0 + r : M - 1;
      const uint16_t* src = X + gr * ldx + cbase + 512 * h + 8 * (lane ^ (r & 15));
      __builtin_amdgcn_global_load_lds((gmem_void*)src, (lds_void*)(sx + r * XS + 512 * h), 16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0);
  }
  __syncthreads();

  c4f y[NBW][4][RG];
  float amax[RG][4];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg)
#pragma unroll
    for (int e = 0; e < 4; ++e) amax[rg][e] = 0.0f;
  // This wave's 2 KB of the auxiliary region hold 16 columns at a time: column c of
  // 128 bytes, its 16-byte piece p at slot p ^ (c / 2).  (A wave's LDS operations
  // execute in order, so the next columns may be stored behind the reads.)
  uint16_t* wbuf = raw + wave * 1024;
  const int wslot = (lane >> 3) * 64, wp = lane & 7;
  const int rslot = r16 * 64, rsw = (r16 >> 1) & 7;
#pragma unroll
  for (int i = 0; i < NBW; ++i) {
    if (i + PF - 1 < NBW) load_b(i + PF - 1, bring[(i + PF - 1) % PF]);
    __builtin_amdgcn_sched_barrier(0);
    const c8h (&bf)[4][2] = bring[i % PF];
    c8h a[RG][2];
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      const uint16_t* ap = &sx[(rg * 16 + r16) * XS];
      const int at = (wb0 + i) * kCB + 8 * qq;
      a[rg][0] = *reinterpret_cast<const c8h*>(ap + (at ^ (r16 * 8)));
      a[rg][1] = *reinterpret_cast<const c8h*>(ap + ((at + 32) ^ (r16 * 8)));
    }
    c8h b[4][2];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
      for (int h = 0; h < 2; ++h)  // columns 8 h + lane / 8
        *reinterpret_cast<c8h*>(wbuf + h * 512 + wslot + ((wp ^ (4 * h + (lane >> 4))) * 8)) = bf[cb][h];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
        b[cb][kk] = *reinterpret_cast<const c8h*>(wbuf + rslot + (((4 * kk + qq) ^ rsw) * 8));
      asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        c4f acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rg][0], b[cb][0], c4f{0, 0, 0, 0}, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rg][1], b[cb][1], acc, 0, 0, 0);
        y[i][cb][rg] = acc;
#pragma unroll
        for (int e = 0; e < 4; ++e) amax[rg][e] = fmaxf(amax[rg][e], fabsf(acc[e]));
      }
  }
  __syncthreads();  // the waves' block matrices are spent: the region holds the maxima and scales
  if (tid == 0) timed_out = 0;
  // Chunk maxima per row: across the 16 lanes of a row group, then the waves.
#pragma unroll
  for (int rg = 0; rg < RG; ++rg)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float m = amax[rg][e];
      m = fmaxf(m, rqd::lane_xor<1>(m));
      m = fmaxf(m, rqd::lane_xor<2>(m));
      m = fmaxf(m, rqd::lane_xor<4>(m));
      m = fmaxf(m, rqd::lane_xor<8>(m));
      if (r16 == 0) red[wave][rg * 16 + 4 * qq + e] = m;
    }
  __syncthreads();  // also: every wave's reads of sx are done (sx is reused for the codes)
  if (tid < R) {
    float m = red[0][tid];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) m = fmaxf(m, red[w][tid]);
    red[0][tid] = m;
    if (nq > 1) exchange_store(exchange_word(Xq, row0, K, C, q, tid), __float_as_uint(m));
  }
  if (nq > 1) {
    // Thread t < nq R waits for partner t / R's maximum of row t % R (its own
    // chunk's included).
    for (int t = tid; t < nq * R; t += NT) {
      uint32_t v = exchange_wait(exchange_word(Xq, row0, K, C, t / R, t % R), give_up == q);
      if (v >> 31) {
        timed_out = 1;
        v = 0;
      }
      pmax[t] = __uint_as_float(v);
    }
    __syncthreads();
    if (tid < nq && tid != q) exchange_store(exchange_word(Xq, row0, K, C, tid, R + q), 0);
    if (tid < R) {
      float m = 0.0f;
      for (int p = 0; p < nq; ++p) m = fmaxf(m, pmax[p * R + tid]);
      red[0][tid] = m;
    }
  }
  __syncthreads();
  if (tid < R) {
    const float m = red[0][tid];
    const float a_z = m * s_t;
    const float delta = a_z / 7.0f;
    gscale[tid] = delta > 0.0f ? s_t / delta : 0.0f;
    const float scale = delta / s_t;
    if (q == 0 && row0 + tid < M) {
      if (nq == 1) xs[row0 + tid] = scale;
      else atomicMax(reinterpret_cast<uint32_t*>(xs) + row0 + tid, __float_as_uint(scale));
    }
  }
  __syncthreads();

  // ---- Codes: 8 consecutive channels packed into a dword across lanes and
  // staged in LDS (the chunk's rows, C / 2 bytes each), then stored as 16-byte
  // pieces.  A lane's four rows travel together, one per byte: lane pairs form
  // a row's two nibbles, then two byte exchanges (lane ^ 2, ^ 4) leave lanes 0,
  // 4, 2, 6 of eight with the dword of rows 0, 1, 2, 3.
  uint32_t* scodes = reinterpret_cast<uint32_t*>(sx);  // [R][C / 8] dwords
  const uint32_t sel2 = (lane & 2) ? 0x03070206u : 0x05010400u;
  const uint32_t sel4 = (lane & 4) ? 0x03020706u : 0x05040100u;
  const int crow = 4 * qq + (lane & 2) + ((lane >> 2) & 1);
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    float g[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = gscale[rg * 16 + 4 * qq + e];
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        uint32_t c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = __float_as_uint(fmaf(y[i][cb][rg][e], g[e], rqd::kRoundMagic));
        const uint32_t v = (__builtin_amdgcn_perm(c[1], c[0], 0x0C0C0400u) |
                            __builtin_amdgcn_perm(c[3], c[2], 0x04000C0Cu)) & 0x0F0F0F0Fu;
        const uint32_t w = v | __float_as_uint(rqd::lane_xor<1>(__uint_as_float(v))) << 4;
        const uint32_t h = __builtin_amdgcn_perm(__float_as_uint(rqd::lane_xor<2>(__uint_as_float(w))), w, sel2);
        const uint32_t d = __builtin_amdgcn_perm(__float_as_uint(rqd::lane_xor_dpp<4>(__uint_as_float(h))), h, sel4);
        if ((lane & 1) == 0)
          scodes[(rg * 16 + crow) * (C / 8) + ((wb0 + i) * kCB + cb * 16 + (r16 & 8)) / 8] = d;
      }
  }
  if (nq > 1 && tid < nq && tid != q)  // (the other chunks have read this one's maxima)
    if (exchange_wait(exchange_word(Xq, row0, K, C, q, R + tid), give_up == nq + q) >> 31) timed_out = 1;
  __syncthreads();
  if (nq > 1 && timed_out) {
    if (tid < R && row0 + tid < M) atomicMax(reinterpret_cast<uint32_t*>(xs) + row0 + tid, kNaN);
    return;
  }
  constexpr int CPR = C / 32;  // 16-byte code pieces per row of the chunk
  for (int p = tid; p < R * CPR; p += NT) {
    const int r = p / CPR, c16 = p % CPR;
    if (row0 + r >= M) continue;
    *reinterpret_cast<uint4*>(Xq + (row0 + r) * static_cast<int64_t>(K / 2) + cbase / 2 + 16 * c16) =
        *reinterpret_cast<const uint4*>(&scodes[r * (C / 8) + 4 * c16]);
  }
}

template <int RG, int C, bool GATHER, int KMAX = C, int WAVES = 8, int PF = 2>
int launch_composite_x(const void* X, int64_t M, int64_t K, int64_t ldx, const int32_t* perm, const void* Rt,
                       float s, uint8_t* Xq, float* x_scale, hipStream_t stream, int give_up = -1) {
  constexpr int R = 16 * RG;
  const int64_t ntiles = (M + R - 1) / R;
  const int nq = static_cast<int>(K / C);
  if (ntiles > (int64_t{1} << 26)) return OQ_ERR_SHAPE;
  if (nq > 1) {
    const int64_t words = ntiles * nq * (R + nq);
    hipLaunchKernelGGL(comp_words_kernel, dim3(static_cast<unsigned>((words + 255) / 256)), dim3(256), 0, stream, Xq,
                       x_scale, M, static_cast<int>(ntiles), static_cast<int>(K), C, nq, R);
    const int st = launch_status();
    if (st != OQ_OK) return st;
  }
  const int64_t grid = (ntiles + 7) / 8 * 8 * nq;
  hipLaunchKernelGGL((rq_composite_x_kernel<RG, C, GATHER, WAVES, PF, KMAX>), dim3(static_cast<unsigned>(grid)),
                     dim3(64 * WAVES), 0, stream, static_cast<const uint16_t*>(X), M, static_cast<int>(K), ldx,
                     perm, static_cast<const uint16_t*>(Rt), s, Xq, x_scale, nq, static_cast<int>(ntiles), give_up);
  return launch_status();
}

// Chunk width: the widest of 4096 / 2048 / 1024 / 512 that divides K, at
// most `cap` (0: none; the two-pass kernel is used).  With the online
// permutation every chunk's workgroup reads whole rows, so 16-row tiles of the
// widest chunk (fewest re-reads) are best.  With P folded into the input a
// workgroup reads only its chunk's columns and the block matrices dominate
// the traffic from L2 (128 K / R bytes per row for R-row tiles), so 32-row
// tiles of at most 1024 channels (64 KB of LDS, two workgroups per CU) are
// best (measured at K = 4096 - 16384).
int comp_chunk(int64_t K, int cap) {
  for (int c : {4096, 2048, 1024, 512})
    if (c <= cap && K % c == 0) return c;
  return 0;
}

int launch_composite_chunked(bool gather, int C, const void* X, int64_t M, int64_t K, int64_t ldx,
                             const int32_t* perm, const void* Rt, float s, uint8_t* Xq, float* x_scale,
                             hipStream_t h, int give_up = -1) {
  if (gather) {
#define OQ_CX(CC, KM) return launch_composite_x<1, CC, true, KM>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h, give_up)
    switch (C) {
      case 4096:
        if (K <= 8192) OQ_CX(4096, 8192);
        OQ_CX(4096, 16384);
      case 2048: OQ_CX(2048, 16384);
      case 1024: OQ_CX(1024, 16384);
      case 512: OQ_CX(512, 16384);
      default: return OQ_ERR_SHAPE;
    }
#undef OQ_CX
  }
  switch (C) {
    case 1024: return launch_composite_x<2, 1024, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h, give_up);
    case 512: return launch_composite_x<2, 512, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h, give_up);
    default: return OQ_ERR_SHAPE;
  }
}

// Rows that one chunk holds: the chunked kernel with nq = 1, without exchange.
// *st is set and true returned if K is one of the widths built (512, 1024, 1536,
// 2048, 3072, 4096).  2560 and 3584 would fit the kernel too; no instance is built
// for them, so they take rq_composite1_kernel (4080 rows: 26 and 30 us with the
// permutation).  (Against rq_composite1_kernel, which stays for the other K
// up to 4096: 4080 x 2048 22 -> 11 us, 16384 x 1024 23 -> 18 us, 700 x 4096 28 ->
// 16 us; with P folded 22 -> 9, 25 -> 12, 28 -> 11 us.)
bool launch_composite_one(bool gather, const void* X, int64_t M, int64_t K, int64_t ldx, const int32_t* perm,
                          const void* Rt, float s, uint8_t* Xq, float* x_scale, hipStream_t h, int* st) {
#define OQ_C1(RG, CC, G, KM) *st = launch_composite_x<RG, CC, G, KM>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h)
  // Folded rows of up to 1024 channels: 32-row tiles read the block matrices half as often, 16-row
  // tiles spread few rows over more CUs.
#define OQ_C1_CASE(CC, KM)               \
  case CC:                               \
    if (gather) OQ_C1(1, CC, true, KM);  \
    else if (CC <= 1024 && M > 1024) OQ_C1((CC <= 1024 ? 2 : 1), CC, false, CC); \
    else OQ_C1(1, CC, false, CC);        \
    return true;
  switch (K) {
    OQ_C1_CASE(512, 512)
    OQ_C1_CASE(1024, 1024)
    OQ_C1_CASE(1536, 2048)
    OQ_C1_CASE(2048, 2048)
    OQ_C1_CASE(3072, 4096)
    OQ_C1_CASE(4096, 4096)
    default: return false;
  }
#undef OQ_C1_CASE
#undef OQ_C1
}

template <int RG, int KMAX, bool GATHER = true>
int launch_composite1(const void* X, int64_t M, int64_t K, int64_t ldx, const int32_t* perm, const void* Rt,
                      float s, uint8_t* Xq, float* x_scale, hipStream_t stream) {
  const unsigned grid = static_cast<unsigned>((M + 16 * RG - 1) / (16 * RG));
  hipLaunchKernelGGL((rq_composite1_kernel<RG, KMAX, GATHER>), dim3(grid), dim3(512), 0, stream,
                     static_cast<const uint16_t*>(X), M, static_cast<int>(K), ldx, perm,
                     static_cast<const uint16_t*>(Rt), s, Xq, x_scale);
  return launch_status();
}

template <int RW, int KMAX, bool GATHER = true>
int launch_composite(const void* X, int64_t M, int64_t K, int64_t ldx, const int32_t* perm, const void* Rt,
                     float s, uint8_t* Xq, float* x_scale, hipStream_t stream) {
  const unsigned grid = static_cast<unsigned>((M + RW - 1) / RW);
  hipLaunchKernelGGL((rq_composite_kernel<RW, KMAX, 2, GATHER>), dim3(grid), dim3(256), 0, stream,
                     static_cast<const uint16_t*>(X), M, static_cast<int>(K), ldx, perm,
                     static_cast<const uint16_t*>(Rt), s, Xq, x_scale);
  return launch_status();
}

}  // namespace
}  // namespace oq

extern "C" int oq_rotate_quantize_act_composite(const void* X, int64_t M, int64_t K, int64_t ldx,
                                                const int32_t* perm, const void* Rt, const float* s_table,
                                                int32_t t, uint8_t* Xq, float* x_scale, void* stream) {
  if (M < 0 || K < 64 || K % 64 != 0 || K > 16384 || ldx < K) return OQ_ERR_SHAPE;
  if (ldx % 8 != 0) return OQ_ERR_ALIGN;
  if (t < 0) return OQ_ERR_ARG;
  if (M == 0) return OQ_OK;
  if (!X || !Rt || !Xq || !x_scale) return OQ_ERR_NULL;
  if (!oq::aligned(X, 16) || (perm && !oq::aligned(perm, 16)) || !oq::aligned(Rt, 16) || !oq::aligned(Xq, 16) ||
      !oq::aligned(x_scale, 4))
    return OQ_ERR_ALIGN;
  const float s = s_table ? s_table[t] : 1.0f;
  if (!(s > 0.0f) || !std::isfinite(s)) return OQ_ERR_ARG;
  int st = oq::device_check();
  if (st != OQ_OK) return st;
  hipStream_t h = static_cast<hipStream_t>(stream);
  // K = 4096 folded with many rows: 1024-channel chunks of 32-row tiles read the
  // block matrices half as often as one workgroup per 16 whole rows (M = 2000 / 4080 / 16384: 10.5 / 15.4 / 48 against
  // 12.6 / 16.2 / 60 us).
  if (!perm && K == 4096 && M > 1024)
    return oq::launch_composite_chunked(false, 1024, X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  if (oq::launch_composite_one(perm != nullptr, X, M, K, ldx, perm, Rt, s, Xq, x_scale, h, &st)) return st;
  // Other K.  Without a permutation the rows are read straight into the MFMA
  // operands (no LDS staging): row groups sized to the register budget.
  if (!perm) {
    // Few rows: one row group per workgroup, so the rows spread over more CUs.
    if (M <= 1024 && K <= 1024) return oq::launch_composite1<1, 1024, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    if (M <= 1024 && K <= 2048) return oq::launch_composite1<1, 2048, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    if (K <= 1024) return oq::launch_composite1<2, 1024, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    if (K <= 2048) return oq::launch_composite1<2, 2048, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    if (K <= 4096) return oq::launch_composite1<1, 4096, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    if (const int c = oq::comp_chunk(K, 1024))
      return oq::launch_composite_chunked(false, c, X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    if (K <= 8192) return oq::launch_composite<16, 8192, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
    return oq::launch_composite<16, 16384, false>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  }
  // Single pass (y in registers) up to K = 4096, row groups sized to the
  // LDS budget; deeper rows take the two-pass kernel.
  // Few rows: one row group per workgroup, so the rows spread over more CUs.
  if (M <= 1024 && K <= 2048) return oq::launch_composite1<1, 2048>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  if (K <= 1024) return oq::launch_composite1<4, 1024>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  if (K <= 2048) return oq::launch_composite1<2, 2048>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  if (K <= 4096) return oq::launch_composite1<1, 4096>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  if (const int c = oq::comp_chunk(K, 4096))
    return oq::launch_composite_chunked(true, c, X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  if (K <= 8192) return oq::launch_composite<4, 8192>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
  return oq::launch_composite<2, 16384>(X, M, K, ldx, perm, Rt, s, Xq, x_scale, h);
}

// A call that exchanges in which one chunk gives up (see the exchange above):
// for the tests of how a failure is reported; not part of the interface.
extern "C" int oq_test_composite_give_up(const void* X, int64_t M, int64_t K, int64_t ldx, const int32_t* perm,
                                         const void* Rt, uint8_t* Xq, float* x_scale, int32_t give_up, void* stream) {
  const int c = !perm && K == 4096 ? 1024 : K > 4096 && K <= 16384 ? oq::comp_chunk(K, perm ? 4096 : 1024) : 0;
  if (M < 1 || c == 0 || ldx < K || ldx % 8 != 0) return OQ_ERR_SHAPE;
  if (!X || !Rt || !Xq || !x_scale) return OQ_ERR_NULL;
  const int st = oq::device_check();
  if (st != OQ_OK) return st;
  return oq::launch_composite_chunked(perm != nullptr, c, X, M, K, ldx, perm, Rt, 1.0f, Xq, x_scale,
                                      static_cast<hipStream_t>(stream), give_up);
}
