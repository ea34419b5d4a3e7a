// W4A4 product with int32 accumulation and the fused dequantization epilogue.
//
// eq:lowbit_linear: X'W' ~= Delta_X' Delta_W' Q_X' Q_W'.  acc[i][n] =
// sum_k q[i][k] wq[n][k] is formed exactly on the int8 matrix cores
// (v_mfma_i32_32x32x32_i8); the per-token and per-output-channel steps (and the
// bias) are applied to the accumulator in the epilogue, as the Implementation
// Details fold every scale into dequantization.
//
// CDNA4 has no int4 integer MFMA, so codes are widened to int8 in registers.
// A packed byte holds two codes (low nibble = even channel).  Masking instead
// of sign-extending keeps each code in the HIGH nibble of an int8 lane:
// (w << 4) & 0xF0F0F0F0 gives 16*q_even per byte and w & 0xF0F0F0F0 gives
// 16*q_odd, both correctly signed.  Every product is then 256*q*wq;
// |256 * 49 * K| < 2^31 for K <= 16384, and the exact accumulator is recovered
// with an arithmetic shift by 8.  A and B take the channels in the same order,
// so the dot products are unchanged.
//
// Two kernels.  M > 64 (and fewer rows of wide products): LDS-staged tiles on
// v_mfma_i32_32x32x32_i8 (gemm_ring.h; kernel and tile by the rules of gemm_rules.h).
// Other M <= 64 (and token codes in the 16-row tiled layout): a weight-streaming kernel on
// v_mfma_i32_16x16x64_i8 with the operands loaded straight into registers
// (details at gemm_small_kernel).  8-bit token codes (W4A8) use both with
// the A operand loaded as bytes.
#include "common.h"
#include "gemm_ring.h"
#include "gemm_rules.h"

namespace oq {
namespace {

constexpr int BK = 64;  // K granularity in codes (one MFMA k step of 64 codes = 32 packed bytes)

__device__ __forceinline__ v4i widen16_u2(uint2 p) {
  const uint32_t m = 0xF0F0F0F0u;
  v4i r;
  r[0] = static_cast<int>((p.x << 4) & m);
  r[1] = static_cast<int>(p.x & m);
  r[2] = static_cast<int>((p.y << 4) & m);
  r[3] = static_cast<int>(p.y & m);
  return r;
}

// 16 bytes of 8-bit codes (natural channel order) in the order that
// widen16_u2 gives packed codes: within each group of 8 channels the even
// channels first, [0 2 4 6 1 3 5 7], so that a W4A8 A operand meets the
// widened weight fragment channel for channel.
__device__ __forceinline__ v4i order16_i8(uint4 p) {
  v4i r;
  r[0] = static_cast<int>(__builtin_amdgcn_perm(p.y, p.x, 0x06040200u));
  r[1] = static_cast<int>(__builtin_amdgcn_perm(p.y, p.x, 0x07050301u));
  r[2] = static_cast<int>(__builtin_amdgcn_perm(p.w, p.z, 0x06040200u));
  r[3] = static_cast<int>(__builtin_amdgcn_perm(p.w, p.z, 0x07050301u));
  return r;
}

// ---------------------------------------------------------------------------
// Small-M product (the DiT's 50 action tokens, decode): weight-bandwidth and
// latency bound, so the weight is spread over many small workgroups.  A
// workgroup owns 16 MB rows x 16 NB columns of the output and all of K; its
// WAVES waves take contiguous ranges of 128-code units (64 packed bytes per
// row).  Every operand fragment is one 16-byte load per lane that feeds two
// v_mfma_i32_16x16x64_i8 steps (the two 8-byte halves, widened to int8 in
// registers); all of a wave's loads of UB units are issued before the first
// MFMA.  A comes either from the 16-row tiled layout -- one load is 1024
// contiguous bytes, 8 whole cache lines -- or from [M][K/2] rows (16 rows x
// 64 bytes per load).  The token codes are re-read by every workgroup, so the
// tiled form is what the DiT's fused producers write.  K % 128 == 64 (row
// layout only) ends with one 64-code step in 8-byte pieces on the last wave.
// The waves' partial accumulators are summed through LDS before the shared
// epilogue.
// ---------------------------------------------------------------------------

// Epilogue of one output from the exact accumulator; the per-row / per-column
// operands are passed in (loaded early by the caller).
template <int EPI>
__device__ __forceinline__ void store_out(const GemmArgs& a, int64_t off, int v, float xs, float ws, float bias,
                                          float gate, float resid) {
  if (EPI == EPI_I32) {
    static_cast<int32_t*>(a.C)[off] = v;
    return;
  }
  const float y = static_cast<float>(v) * xs * ws + bias;
  if (EPI == EPI_F16) {
    static_cast<_Float16*>(a.C)[off] = static_cast<_Float16>(y);
  } else if (EPI == EPI_GELU_F16) {
    static_cast<_Float16*>(a.C)[off] =
        static_cast<_Float16>(gelu_tanh(static_cast<float>(static_cast<_Float16>(y))));
  } else if (EPI == EPI_BF16) {
    static_cast<uint16_t*>(a.C)[off] = f32_to_bf16_rne(y);
  } else {
    static_cast<float*>(a.C)[off] = fmaf(gate, y, resid);
  }
}

// A8 (row layout only): 8-bit token codes, 32 bytes per lane and unit,
// reordered in registers; the accumulator is shifted by 4.
template <int EPI, int NB, int WAVES, int MB, int UB, bool TILED, bool A8 = false>
__global__ __launch_bounds__(64 * WAVES) void gemm_small_kernel(GemmArgs a) {
  static_assert(!(A8 && TILED), "8-bit token codes use the row layout");
  constexpr int BNs = 16 * NB, ROWS = 16 * MB, NOUT = ROWS * BNs, NT = 64 * WAVES;
  constexpr int OPT = (NOUT + NT - 1) / NT;  // outputs per thread
  static_assert(NT % BNs == 0, "a thread keeps one output column");
  __shared__ int red[WAVES][NOUT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // scalar: the unit range bounds MFMA loops
  const int64_t n0 = static_cast<int64_t>(blockIdx.x) * BNs;
  const int64_t m0 = static_cast<int64_t>(blockIdx.y) * ROWS;
  const int64_t Kb = a.K / 2;
  const int nu = static_cast<int>(a.K / 128);
  const int ubeg = (nu * wave) / WAVES, uend = (nu * (wave + 1)) / WAVES;

  // Row-block bases: tiled -> block (m0 / 16 + rb) at unit 0 plus this lane's
  // 16 bytes; rows -> row m0 + 16 rb + lane % 16 at byte 0.  Out-of-range
  // blocks / rows read a clamped valid address; their fragments are replaced
  // by zeros where they are used.  Every load is unconditional, so the
  // compiler counts them exactly and each MFMA waits only for its own
  // operands.
  const uint8_t* abase[MB];
  bool aok[MB];
#pragma unroll
  for (int rb = 0; rb < MB; ++rb) {
    if (TILED) {
      const int64_t blk = m0 / 16 + rb;
      aok[rb] = blk * 16 < a.M;
      abase[rb] = a.A + (aok[rb] ? blk : 0) * nu * 1024 + lane * 16;
    } else {
      const int64_t r = m0 + rb * 16 + (lane & 15);
      aok[rb] = r < a.M;
      abase[rb] = a.A + (aok[rb] ? r : 0) * Kb * (A8 ? 2 : 1);
    }
  }
  const uint8_t* bbase[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) bbase[nb] = a.B + min<int64_t>(n0 + nb * 16 + (lane & 15), a.N - 1) * Kb;
  const int piece = 16 * (lane >> 4);  // this lane's 16 bytes of a 64-byte unit (row layout)

  // Fragments of UB units starting at u0 (a unit past uend reads unit uend - 1
  // or 0 again; its MFMAs are skipped).
  constexpr int AH = A8 ? 2 : 1;  // 16-byte A loads per unit and row block
  uint4 fa[UB ? UB : 1][MB][AH], fb[UB ? UB : 1][NB];
  auto load_units = [&](int u0) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int uu = u0 + u < uend ? u0 + u : max(uend - 1, 0);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) fb[u][nb] = *reinterpret_cast<const uint4*>(bbase[nb] + uu * 64 + piece);
#pragma unroll
      for (int rb = 0; rb < MB; ++rb)
#pragma unroll
        for (int c = 0; c < AH; ++c)
          fa[u][rb][c] = *reinterpret_cast<const uint4*>(
              TILED ? abase[rb] + static_cast<int64_t>(uu) * 1024
                    : abase[rb] + uu * 64 * AH + piece * AH + 16 * c);
    }
  };
  // The first units' loads go out before anything else.
  load_units(ubeg);

  // Epilogue operands of this thread's outputs (row (tid + u NT) / BNs,
  // column tid % BNs), loaded while the fragments are in flight, from clamped
  // addresses (the values of outputs that are not stored do not matter).
  const int ecol = tid % BNs;
  const int64_t egc = n0 + ecol;
  const bool ecol_ok = egc < a.N;
  const int64_t egc_c = ecol_ok ? egc : 0;
  float e_ws = 0.0f, e_bias = 0.0f, e_gate = 1.0f;
  float e_xs[OPT], e_res[OPT];
  if (EPI != EPI_I32) {
    e_ws = a.ws[egc_c];
    if (a.bias) e_bias = static_cast<float>(__builtin_bit_cast(_Float16, a.bias[egc_c]));
    if (EPI == EPI_RESID_F32 && a.gate) e_gate = static_cast<float>(__builtin_bit_cast(_Float16, a.gate[egc_c]));
  }
#pragma unroll
  for (int u = 0; u < OPT; ++u) {
    const int64_t gr = m0 + (tid + u * NT) / BNs;
    const int64_t gr_c = gr < a.M ? gr : 0;
    e_xs[u] = 0.0f;
    e_res[u] = 0.0f;
    if (EPI != EPI_I32) {
      e_xs[u] = a.xs[gr_c];
      if (EPI == EPI_RESID_F32) e_res[u] = static_cast<const float*>(a.C)[gr_c * a.ldc + egc_c];
    }
  }

  v4i acc[MB][NB];
#pragma unroll
  for (int rb = 0; rb < MB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[rb][nb] = v4i{0, 0, 0, 0};
  auto mfma_units = [&](int u0) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      if (u0 + u < uend) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          v4i wb[NB];
#pragma unroll
          for (int nb = 0; nb < NB; ++nb)
            wb[nb] = widen16_u2(h ? make_uint2(fb[u][nb].z, fb[u][nb].w) : make_uint2(fb[u][nb].x, fb[u][nb].y));
#pragma unroll
          for (int rb = 0; rb < MB; ++rb) {
            v4i xa;
            if constexpr (A8) {
              xa = order16_i8(aok[rb] ? fa[u][rb][h] : make_uint4(0, 0, 0, 0));
            } else {
              const uint2 pa = h ? make_uint2(fa[u][rb][0].z, fa[u][rb][0].w) : make_uint2(fa[u][rb][0].x, fa[u][rb][0].y);
              xa = widen16_u2(aok[rb] ? pa : make_uint2(0, 0));
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              acc[rb][nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, wb[nb], acc[rb][nb], 0, 0, 0);
          }
        }
      }
    }
  };
  // First round straight-line (the MFMAs of a unit wait only for that unit's
  // loads); deeper K continues in rounds of UB units.
  if constexpr (UB > 0) {
    mfma_units(ubeg);
    for (int u0 = ubeg + UB; u0 < uend; u0 += UB) {
      load_units(u0);
      mfma_units(u0);
    }
  }
  if (!TILED && (a.K & 127) && wave == WAVES - 1) {
    // Final 64 codes: 32 packed bytes per row, 8 per lane.
    const int64_t off = static_cast<int64_t>(nu) * 64 + 8 * (lane >> 4);
    v4i wb[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) wb[nb] = widen16_u2(*reinterpret_cast<const uint2*>(bbase[nb] + off));
#pragma unroll
    for (int rb = 0; rb < MB; ++rb) {
      v4i xa;
      if constexpr (A8)
        xa = order16_i8(aok[rb] ? *reinterpret_cast<const uint4*>(abase[rb] + 2 * off) : make_uint4(0, 0, 0, 0));
      else
        xa = widen16_u2(aok[rb] ? *reinterpret_cast<const uint2*>(abase[rb] + off) : make_uint2(0, 0));
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[rb][nb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, wb[nb], acc[rb][nb], 0, 0, 0);
    }
  }

  // 16x16 accumulator layout: element e of lane l is row 4*(l/16) + e, column l%16.
#pragma unroll
  for (int rb = 0; rb < MB; ++rb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[wave][(rb * 16 + 4 * (lane >> 4) + e) * BNs + nb * 16 + (lane & 15)] = acc[rb][nb][e];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < OPT; ++u) {
    const int i = tid + u * NT;
    const int64_t gr = m0 + i / BNs;
    if (i >= NOUT || gr >= a.M || !ecol_ok) continue;
    int sum = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) sum += red[w][i];
    store_out<EPI>(a, gr * a.ldc + egc, sum >> (A8 ? 4 : 8), e_xs[u], e_ws, e_bias, e_gate, e_res[u]);
  }
}

template <int EPI, bool TILED, int MB, bool A8 = false>
int launch_small_mb(const GemmArgs& a, hipStream_t stream) {
  const SmallShape sh = small_shape(a.N, a.K, A8);
  const int bn = 16 * sh.nb;
  const dim3 grid(static_cast<unsigned>((a.N + bn - 1) / bn), static_cast<unsigned>((a.M + 16 * MB - 1) / (16 * MB)));
  const dim3 block(64 * sh.waves);
#define OQ_SMALL(NB, WV, UB)                                                                             \
  if (sh.nb == NB && sh.waves == WV && sh.ub == UB) {                                                    \
    hipLaunchKernelGGL((gemm_small_kernel<EPI, NB, WV, MB, UB, TILED, A8>), grid, block, 0, stream, a);  \
    return launch_status();                                                                              \
  }
  if constexpr (!TILED) {  // (the tiled layout has K % 128 == 0)
    OQ_SMALL(1, 4, 0)
    OQ_SMALL(2, 8, 0)
  }
  OQ_SMALL(1, 4, 2)
  OQ_SMALL(2, 8, 1)
  OQ_SMALL(1, 16, 1)
  OQ_SMALL(2, 8, 2)
  if constexpr (!A8) {
    OQ_SMALL(1, 16, 2)
    OQ_SMALL(2, 8, 4)
  }
#undef OQ_SMALL
  return OQ_ERR_SHAPE;
}

// Row blocks of 16 (one per workgroup) spread a small-M product over four
// times the workgroups of 64-row blocks; that pays while the grid stays
// within 16 waves per CU (the 50-row DiT linears: q|k|v, o and down, 1.5 to
// 5 thousand waves; not the 8192-column gate|up, whose 32-column workgroups of
// 8 waves would make 8 thousand).
bool small_row_blocks_of_16(const GemmArgs& a) {
  const SmallShape sh = small_shape(a.N, a.K, false);
  const int64_t bn = 16 * sh.nb;
  const int64_t total = (a.N + bn - 1) / bn * ((a.M + 15) / 16) * sh.waves;
  return a.M <= 16 || total <= 4096;
}

template <int EPI, bool TILED>
int launch_small(const GemmArgs& a, hipStream_t stream) {
  return small_row_blocks_of_16(a) ? launch_small_mb<EPI, TILED, 1>(a, stream) : launch_small_mb<EPI, TILED, 4>(a, stream);
}

template <int EPI>
int launch_small_any(const GemmArgs& a, hipStream_t stream) {
  if (a.a_i8)
    return a.M <= 16 ? launch_small_mb<EPI, false, 1, true>(a, stream) : launch_small_mb<EPI, false, 4, true>(a, stream);
  return a.a_tiled ? launch_small<EPI, true>(a, stream) : launch_small<EPI, false>(a, stream);
}

}  // namespace

int gemm_validate(const uint8_t* Xq, int64_t M, const uint8_t* Wq, int64_t N, int64_t K, const void* C,
                  int64_t ldc, int64_t ldc_align) {
  if (M < 0 || N < 1 || K < BK || K % BK != 0 || K > 16384 || ldc < N) return OQ_ERR_SHAPE;
  if (ldc % ldc_align != 0) return OQ_ERR_ALIGN;
  if (M == 0) return OQ_OK;  // nothing is read or written; pointers may be NULL
  if (!Xq || !Wq || !C) return OQ_ERR_NULL;
  if (!aligned(Xq, 16) || !aligned(Wq, 16) || !aligned(C, 16) || ldc % ldc_align != 0) return OQ_ERR_ALIGN;
  return OQ_OK;
}

template <int WM, int WN, int TM, int TN, bool A8, int P, int NS, int KG, int SPREAD>
int launch_ring(const GemmArgs& a, Epilogue epi, hipStream_t stream) {
  constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 g(static_cast<unsigned>(tiles)), b(64 * WM * WN * KG);
#define OQ_RING(E) hipLaunchKernelGGL((gemm_ring_kernel<E, WM, WN, TM, TN, A8, P, NS, KG, SPREAD>), g, b, 0, stream, a)
  switch (epi) {
    case EPI_I32: OQ_RING(EPI_I32); break;
    case EPI_F16: OQ_RING(EPI_F16); break;
    case EPI_BF16: OQ_RING(EPI_BF16); break;
    case EPI_GELU_F16:
      if constexpr (A8) return OQ_ERR_ARG;  // a DiT path only
      else OQ_RING(EPI_GELU_F16);
      break;
    case EPI_RESID_F32:
      if constexpr (A8) return OQ_ERR_ARG;  // the residual epilogue is a W4A4 DiT path only
      else OQ_RING(EPI_RESID_F32);
      break;
    default: return OQ_ERR_ARG;
  }
#undef OQ_RING
  return launch_status();
}

int gemm_launch(const GemmArgs& a, Epilogue epi, hipStream_t stream) {
  if (a.M == 0) return OQ_OK;
  if (a.a_i8 && (epi == EPI_RESID_F32 || epi == EPI_GELU_F16)) return OQ_ERR_ARG;
  if (few_rows(a.M, a.N, a.K, a.a_i8, a.a_tiled)) {
    switch (epi) {
      case EPI_I32: return launch_small_any<EPI_I32>(a, stream);
      case EPI_F16: return launch_small_any<EPI_F16>(a, stream);
      case EPI_BF16: return launch_small_any<EPI_BF16>(a, stream);
      case EPI_RESID_F32: return launch_small_any<EPI_RESID_F32>(a, stream);
      case EPI_GELU_F16: return launch_small_any<EPI_GELU_F16>(a, stream);
      default: return OQ_ERR_ARG;
    }
  }
  if (a.a_i8) {
    switch (ring_tiling(a.M, a.N, a.K, true)) {
      case 0: return launch_ring<2, 4, 4, 2, true, 4, 3, 1, 2>(a, epi, stream);
      case 1: return launch_ring<2, 2, 2, 2, true, 4, 3, 1, 1>(a, epi, stream);
      default: return launch_ring<1, 2, 2, 1, true, 8, 2, 2, 1>(a, epi, stream);
    }
  }
  switch (ring_tiling(a.M, a.N, a.K, false)) {
    case 0: return launch_ring<2, 4, 4, 2, false, 8, 2, 1, 4>(a, epi, stream);
    case 1: return launch_ring<2, 2, 2, 2, false, 8, 2, 1, 1>(a, epi, stream);
    case 2: return launch_ring<2, 2, 2, 1, false, 8, 2, 1, 1>(a, epi, stream);
    case 3: return launch_ring<1, 2, 2, 1, false, 16, 2, 4, 1>(a, epi, stream);
    case 4: return launch_ring<2, 2, 1, 1, false, 16, 2, 1, 1>(a, epi, stream);
    case 5: return launch_ring<2, 2, 1, 1, false, 4, 2, 1, 1>(a, epi, stream);
    default: return launch_ring<2, 2, 2, 1, false, 4, 2, 1, 1>(a, epi, stream);
  }
}

}  // namespace oq

extern "C" int oq_w4a4_linear(const uint8_t* Xq, const float* x_scale, int64_t M, const uint8_t* Wq,
                              const float* w_scale, const void* bias, int64_t N, int64_t K, void* Y,
                              int64_t ldy, int32_t out_dtype, void* stream) {
  int st = oq::gemm_validate(Xq, M, Wq, N, K, Y, ldy, 8);
  if (st != OQ_OK || M == 0) return st;
  if (!x_scale || !w_scale) return OQ_ERR_NULL;
  if (out_dtype != OQ_OUT_F16 && out_dtype != OQ_OUT_BF16) return OQ_ERR_ARG;
  if (!oq::aligned(x_scale, 4) || !oq::aligned(w_scale, 4) || (bias && !oq::aligned(bias, 2))) return OQ_ERR_ALIGN;
  if ((st = oq::device_check()) != OQ_OK) return st;
  oq::GemmArgs a{Xq, Wq, x_scale, w_scale, static_cast<const uint16_t*>(bias), Y, nullptr, M, N, K, ldy};
  return oq::gemm_launch(a, out_dtype == OQ_OUT_F16 ? oq::EPI_F16 : oq::EPI_BF16, static_cast<hipStream_t>(stream));
}

extern "C" int oq_w4a4_gemm_i32(const uint8_t* Xq, int64_t M, const uint8_t* Wq, int64_t N, int64_t K,
                                int32_t* acc, int64_t ldc, void* stream) {
  int st = oq::gemm_validate(Xq, M, Wq, N, K, acc, ldc, 4);
  if (st != OQ_OK || M == 0) return st;
  if ((st = oq::device_check()) != OQ_OK) return st;
  oq::GemmArgs a{Xq, Wq, nullptr, nullptr, nullptr, acc, nullptr, M, N, K, ldc};
  return oq::gemm_launch(a, oq::EPI_I32, static_cast<hipStream_t>(stream));
}

extern "C" int oq_w4a4_linear_tiled(const uint8_t* Xt, const float* x_scale, int64_t M, const uint8_t* Wq,
                                    const float* w_scale, const void* bias, int64_t N, int64_t K, void* Y,
                                    int64_t ldy, int32_t out_dtype, void* stream) {
  int st = oq::gemm_validate(Xt, M, Wq, N, K, Y, ldy, 8);
  if (st != OQ_OK) return st;
  if (K % 128 != 0) return OQ_ERR_SHAPE;
  if (M == 0) return OQ_OK;
  if (!x_scale || !w_scale) return OQ_ERR_NULL;
  if (out_dtype != OQ_OUT_F16 && out_dtype != OQ_OUT_BF16) return OQ_ERR_ARG;
  if (!oq::aligned(x_scale, 4) || !oq::aligned(w_scale, 4) || (bias && !oq::aligned(bias, 2))) return OQ_ERR_ALIGN;
  if ((st = oq::device_check()) != OQ_OK) return st;
  oq::GemmArgs a{Xt, Wq, x_scale, w_scale, static_cast<const uint16_t*>(bias), Y, nullptr, M, N, K, ldy, true};
  return oq::gemm_launch(a, out_dtype == OQ_OUT_F16 ? oq::EPI_F16 : oq::EPI_BF16, static_cast<hipStream_t>(stream));
}

extern "C" int oq_w4a4_gemm_i32_tiled(const uint8_t* Xt, int64_t M, const uint8_t* Wq, int64_t N, int64_t K,
                                      int32_t* acc, int64_t ldc, void* stream) {
  int st = oq::gemm_validate(Xt, M, Wq, N, K, acc, ldc, 4);
  if (st != OQ_OK) return st;
  if (K % 128 != 0) return OQ_ERR_SHAPE;
  if (M == 0) return OQ_OK;
  if ((st = oq::device_check()) != OQ_OK) return st;
  oq::GemmArgs a{Xt, Wq, nullptr, nullptr, nullptr, acc, nullptr, M, N, K, ldc, true};
  return oq::gemm_launch(a, oq::EPI_I32, static_cast<hipStream_t>(stream));
}

extern "C" int oq_w4a8_linear(const int8_t* Xq8, const float* x_scale, int64_t M, const uint8_t* Wq,
                              const float* w_scale, const void* bias, int64_t N, int64_t K, void* Y,
                              int64_t ldy, int32_t out_dtype, void* stream) {
  const uint8_t* A = reinterpret_cast<const uint8_t*>(Xq8);
  int st = oq::gemm_validate(A, M, Wq, N, K, Y, ldy, 8);
  if (st != OQ_OK || M == 0) return st;
  if (!x_scale || !w_scale) return OQ_ERR_NULL;
  if (out_dtype != OQ_OUT_F16 && out_dtype != OQ_OUT_BF16) return OQ_ERR_ARG;
  if (!oq::aligned(x_scale, 4) || !oq::aligned(w_scale, 4) || (bias && !oq::aligned(bias, 2))) return OQ_ERR_ALIGN;
  if ((st = oq::device_check()) != OQ_OK) return st;
  oq::GemmArgs a{A, Wq, x_scale, w_scale, static_cast<const uint16_t*>(bias), Y, nullptr, M, N, K, ldy, false, true};
  return oq::gemm_launch(a, out_dtype == OQ_OUT_F16 ? oq::EPI_F16 : oq::EPI_BF16, static_cast<hipStream_t>(stream));
}

extern "C" int oq_w4a8_gemm_i32(const int8_t* Xq8, int64_t M, const uint8_t* Wq, int64_t N, int64_t K,
                                int32_t* acc, int64_t ldc, void* stream) {
  const uint8_t* A = reinterpret_cast<const uint8_t*>(Xq8);
  int st = oq::gemm_validate(A, M, Wq, N, K, acc, ldc, 4);
  if (st != OQ_OK || M == 0) return st;
  if ((st = oq::device_check()) != OQ_OK) return st;
  oq::GemmArgs a{A, Wq, nullptr, nullptr, nullptr, acc, nullptr, M, N, K, ldc, false, true};
  return oq::gemm_launch(a, oq::EPI_I32, static_cast<hipStream_t>(stream));
}
