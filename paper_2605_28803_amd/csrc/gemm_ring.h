// Products with M > 64 (prefill and batched shapes): packed codes streamed
// straight into an LDS ring, widened between the matrix instructions.
//
// A workgroup of WM x WN x KG waves owns a (32 TM WM) x (32 TN WN) output
// tile; a wave owns (32 TM) x (32 TN) of v_mfma_i32_32x32x32_i8 blocks.  K is
// walked in stages of 32 P codes.  A stage's packed rows (16 P bytes each) go
// from global memory into one of NS ring buffers with 16-byte direct-to-LDS
// loads: no load ring in registers, no store phase, half the LDS bytes of
// widened codes, and NS - 1 stages in flight at no register cost.  A lane
// reads 16 packed bytes of a row (32 codes) at once; their even channels
// ((w << 4) & 0xF0F0F0F0: 16 * code per byte, signed) feed one matrix
// instruction and their odd ones (w & 0xF0F0F0F0) the next, the same order in
// A and B.  Every product is then 256 q wq, exact in int32 for K <= 16384, and
// the accumulator is shifted right by 8.
//
// What bounds it and why it is built so.  Widening costs 12 vector operations
// per 16 bytes; with two waves per SIMD up to six vector operations hide
// behind each 32-cycle matrix instruction, with one wave none do (measured: a
// lone wave issues one vector operation every 8 cycles), so every
// configuration keeps at least two waves per SIMD on a full chip.  The wide
// wave tiles (128 x 64: 4.5 operations per matrix instruction) are for large
// problems.  Each pair of 32-code halves is two phases: while the even
// channels are multiplied the odd ones are widened and the next pair is read
// from LDS; while the odd ones are multiplied the next pair's even channels
// are widened.  The only wait per stage is one barrier, placed before the last
// pair, when every wave holds all of the stage's fragments: it both publishes
// the next stage and frees this one's buffer for refilling.  The refill is
// spread over the next SPREAD phases: a whole stage's loads issued at once
// hold the waves at the CU's 64-byte-per-clock load path (16384 x 8192 x 8192:
// 835 us in one burst, 782 over four phases).
// Against the kernel it replaced (packed codes through a register ring,
// widened into padded LDS rows): 16384 x 8192 x 8192 907 -> 779 us,
// 816 x 32768 x 2048 75 -> 56 us, 4080 x 2048 x 16384 154 -> 108 us,
// 1024 x 6144 x 1536 22.8 -> 13.9 us, 1024 x 1536 x 6144 24.0 -> 16.6 us,
// 1024 x 1536 x 1536 11.4 -> 7.1 us.
//
// LDS rows are not padded (a direct load writes 1 KB of consecutive bytes);
// instead the 16-byte pieces of a row are stored at slot piece ^ swz(row),
// which spreads any 16 consecutive rows of one piece over all banks.
//
// KG > 1: KG groups of WM x WN waves share the ring and take the pairs of a
// stage in turn; their accumulators are summed through LDS (exact integers)
// before the epilogue.
//
// The direct loads are written in assembly because the compiler waits for
// every outstanding direct load before any LDS read; the loads have no
// register outputs, and each is waited for by count (vmcnt, in order) before
// the barrier that publishes it.  The compiler's own counts only become
// stricter by loads it does not see.
#pragma once
#include "common.h"

namespace oq {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t b = __float_as_uint(f);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return static_cast<uint16_t>(b >> 16);
}

// Map a linear workgroup id to an output tile (tm, tn): consecutive ids go to
// different XCDs (id % 8), so XCD x takes the x-th contiguous chunk of the
// tiles, and each chunk is walked in groups of GM tile rows (shared A rows and
// B columns stay in that XCD's L2).
__device__ __forceinline__ void ring_tile(int id, int tiles_m, int tiles_n, int* tm, int* tn) {
  const int total = tiles_m * tiles_n;
  const int x = id & 7, per = total >> 3, rem = total & 7;
  const int lin = x * per + min(x, rem) + (id >> 3);
  constexpr int GM = 4;
  const int group = lin / (GM * tiles_n);
  const int first_m = group * GM;
  const int gsize = min(GM, tiles_m - first_m);
  const int in = lin - group * GM * tiles_n;
  *tm = __builtin_amdgcn_readfirstlane(first_m + in % gsize);
  *tn = __builtin_amdgcn_readfirstlane(in / gsize);
}

// Direct-to-LDS loads: lane l's 16 (4) bytes at base + voff land at LDS byte
// lds + 16 l (4 l).
__device__ __forceinline__ void dma16(uint32_t lds, uint32_t voff, const uint8_t* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory", "m0");
}
__device__ __forceinline__ void dma4(uint32_t lds, uint32_t voff, const void* base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory", "m0");
}
// At most N loads still outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N < 64, "vmcnt has six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Slot of piece p of a row of P pieces: p ^ swz<P>(row).
template <int P>
__device__ __forceinline__ int swz(int row) {
  static_assert(P == 4 || P == 8 || P == 16, "pieces per row");
  return P == 4 ? (row >> 2) & 3 : P == 8 ? (row >> 1) & 7 : row & 15;
}

// A8: the token operand holds 8-bit codes (W4A8), one byte each, 32 P bytes
// per row and stage: a lane reads the 32 bytes that belong to its 16 packed
// weight bytes and picks their even, then their odd bytes; the products are
// 16 q wq and the accumulator is shifted by 4.
template <int EPI, int WM, int WN, int TM, int TN, bool A8, int P, int NS, int KG, int SPREAD>
__global__ __launch_bounds__(64 * WM * WN * KG, 2)
void gemm_ring_kernel(GemmArgs a) {
  constexpr int NW = WM * WN * KG;
  constexpr int NT = 64 * NW;
  constexpr int BM = 32 * TM * WM, BN = 32 * TN * WN;
  constexpr int PA = A8 ? 2 * P : P;                 // A pieces of a row per stage
  constexpr int ABYTES = BM * PA * 16, BBYTES = BN * P * 16;
  constexpr int STAGE = ABYTES + BBYTES;
  constexpr int LA = ABYTES / 1024, LB = BBYTES / 1024;  // 1 KB loads of a stage
  static_assert((LA + LB) % NW == 0, "loads per wave");
  constexpr int LPW = (LA + LB) / NW;
  constexpr int NP = P / 2 / KG;                      // 64-code pairs per stage and group
  static_assert(P % (2 * KG) == 0 && NP >= 1, "pairs");
  // Output by one of three routes.  ROWS: int32 partial tiles (one per K group)
  // go through LDS in row order and every thread of the workgroup finishes
  // pieces of V consecutive columns; used where those tiles fit the ring and
  // either the K groups have to be summed or the residual is to be read (16-byte
  // accesses by all waves: the residual epilogue of the 64 x 64 tile with 4 K
  // groups took 13 us longer from the accumulators of group 0).  STAGED: 16-bit
  // results of the accumulators go through LDS and leave as 16-byte row pieces.
  // Else the accumulators are stored directly.
  constexpr bool HALF = EPI == EPI_F16 || EPI == EPI_BF16 || EPI == EPI_GELU_F16;
  constexpr int TILEB = BM * BN * 4;
  constexpr bool ROWS = KG > 1 || (EPI == EPI_RESID_F32 && TILEB <= NS * STAGE);
  constexpr bool STAGED = HALF && !ROWS;
  constexpr int V = HALF ? 8 : 4;
  constexpr int TP = BN + 8;                           // halves per staged output row
  constexpr int OUTB = ROWS ? KG * TILEB : STAGED ? BM * TP * 2 : 0;
  constexpr int LDSB = NS * STAGE > OUTB ? NS * STAGE : OUTB;
  // The ring (after the K loop: the output tile), then the scales of the tile's rows and columns.
  __shared__ __attribute__((aligned(16))) uint8_t smem[LDSB + (BM + BN) * 4];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = wv / (WM * WN), wave = wv % (WM * WN);
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_m = static_cast<int>((a.M + BM - 1) / BM);
  const int tiles_n = static_cast<int>((a.N + BN - 1) / BN);
  int tm, tn;
  ring_tile(static_cast<int>(blockIdx.x), tiles_m, tiles_n, &tm, &tn);
  const int64_t m0 = static_cast<int64_t>(tm) * BM;
  const int64_t n0 = static_cast<int64_t>(tn) * BN;
  const int64_t Kb = a.K / 2;
  const int64_t Ka = A8 ? a.K : Kb;
  const int n64 = static_cast<int>(a.K / 64);          // 64-code pairs
  const int nk = (n64 + P / 2 - 1) / (P / 2);          // stages

  // 32 x 32 accumulator layout: element e of lane l is row 8 (e / 4) + 4 (l / 32) + e % 4, column l % 32.
  const int col_in = lane & 31;
  const int row_grp = 4 * (lane >> 5);
  // Bias and gate of this thread's output columns, and with few pieces per
  // thread the old residual values: loaded first, used last.
  constexpr int NC = ROWS ? V : TN;                    // columns per thread
  static_assert(NT % (BN / V) == 0, "a thread keeps its columns in the row route");
  const int rcol = (tid % (BN / V)) * V;               // (row route) first column within the tile
  uint16_t biasb[NC], gateb[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int64_t gc = n0 + (ROWS ? rcol + j : wn * 32 * TN + j * 32 + col_in);
    const int64_t gcc = gc < a.N ? gc : a.N - 1;
    biasb[j] = 0;
    gateb[j] = 0x3C00;
    if (EPI != EPI_I32 && a.bias) biasb[j] = a.bias[gcc];
    if (EPI == EPI_RESID_F32 && a.gate) gateb[j] = a.gate[gcc];
  }
  constexpr int RSTEP = NT / (BN / V);                 // (row route) rows between a thread's pieces
  constexpr int NPC = ROWS ? (BM + RSTEP - 1) / RSTEP : 1;
  static_assert(!ROWS || BM % RSTEP == 0, "pieces per thread");
  constexpr bool EARLY = ROWS && EPI == EPI_RESID_F32 && NPC <= 8;
  float4 rearly[EARLY ? NPC : 1];
  // (A resid row is 16-byte aligned in every column multiple of 4; the last
  // columns of a ragged N are read one by one at the end.)
  if constexpr (EARLY) {
#pragma unroll
    for (int c = 0; c < NPC; ++c) {
      const int64_t r = m0 + tid / (BN / V) + c * RSTEP, gr = r < a.M ? r : a.M - 1;
      const int64_t gc = n0 + rcol + 4 <= a.N ? n0 + rcol : 0;
      rearly[c] = *reinterpret_cast<const float4*>(static_cast<const float*>(a.C) + gr * a.ldc + gc);
    }
  }
  // Wave wv issues loads wv LPW .. wv LPW + LPW - 1 of a stage (A's first), each
  // 1 KB: lane l's 16 bytes are slot l of 64 / pieces rows.  Rows past M (N)
  // read the last one; their outputs are not stored.
  uint32_t voff[LPW];
  const uint8_t* base[LPW];
  uint32_t lofs[LPW];
  int pc[LPW];
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
      (__attribute__((address_space(3))) uint8_t*)smem));
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int l = wv * LPW + i;
    const bool isA = l < LA;
    const int ll = isA ? l : l - LA;
    const int pr = isA ? PA : P;
    const int row = ll * (64 / pr) + lane / pr;
    const int slot = lane % pr;
    const int piece = slot ^ (isA ? swz<PA>(row) : swz<P>(row));
    const int64_t lim = (isA ? a.M - m0 : a.N - n0) - 1;
    const int64_t rr = row < lim ? row : lim;
    voff[i] = static_cast<uint32_t>(rr * (isA ? Ka : Kb)) + piece * 16;
    pc[i] = (isA && A8) ? piece >> 1 : piece;
    base[i] = isA ? a.A + m0 * Ka : a.B + n0 * Kb;
    lofs[i] = lds0 + l * 1024;
  }
  // Loads [I0, I1) of stage s into ring buffer b.  The last stage may be short
  // (K is a multiple of 64 codes, two pieces): pieces past K read piece 0 of the
  // stage, and their pairs multiply zero A fragments.
  auto issue = [&](int s, int b, auto I0, auto I1) {
    const int left = n64 * 2 - s * P;  // valid pieces
#pragma unroll
    for (int i = decltype(I0)::value; i < decltype(I1)::value; ++i) {
      const bool isA = wv * LPW + i < LA;
      const uint8_t* p = base[i] + static_cast<int64_t>(s) * ((isA && A8) ? 32 * P : 16 * P);
      uint32_t v = voff[i];
      if (left < P) {
        const int over = pc[i] >= left ? pc[i] : 0;
        v -= over * ((isA && A8) ? 32 : 16);
      }
      dma16(lofs[i] + b * STAGE, v, p);
    }
  };
  // The refill of a buffer, spread over SLOTS phases.
  constexpr int SLOTS = SPREAD < 2 * NP ? SPREAD : 2 * NP;
  auto issue_slot = [&](int s, int b, auto SL) {
    constexpr int sl = decltype(SL)::value;
    if constexpr (sl < SLOTS) {
      if (s < nk) issue(s, b, std::integral_constant<int, LPW * sl / SLOTS>{}, std::integral_constant<int, LPW * (sl + 1) / SLOTS>{});
    }
  };

  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

  const int frow = lane & 31, half = lane >> 5;
  const int arow = wm * 32 * TM + frow, brow = wn * 32 * TN + frow;
  const int sa = swz<PA>(frow), sb = swz<P>(frow);  // (the same in every 32-row block)
  const uint8_t* fA = smem + arow * PA * 16;
  const uint8_t* fB = smem + ABYTES + brow * P * 16;

  constexpr int AH = A8 ? 2 : 1;
  static_assert(NP % 2 == 0, "pairs alternate between two register sets");
  uint4 pa[2][TM][AH], pb[2][TN];
  auto read = [&](int b, int pair, int set) {
    const int q = 2 * pair + half;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int h = 0; h < AH; ++h)
        pa[set][i][h] = *reinterpret_cast<const uint4*>(fA + b * STAGE + i * 32 * PA * 16 + (((AH * q + h) ^ sa) * 16));
#pragma unroll
    for (int j = 0; j < TN; ++j)
      pb[set][j] = *reinterpret_cast<const uint4*>(fB + b * STAGE + j * 32 * P * 16 + ((q ^ sb) * 16));
  };
  v4i wa[2][TM], wb[2][TN];
  // Widen the even (odd = 0) or odd channels of packed set `set` into w*[odd].
  auto widen = [&](int set, int odd, uint32_t mm) {
    constexpr uint32_t m = 0xF0F0F0F0u;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (A8) {
        // (Selector 0x0C: a zero byte.)
        const uint32_t sel = !mm ? 0x0C0C0C0Cu : odd ? 0x07050301u : 0x06040200u;
        const uint4 x = pa[set][i][0], y = pa[set][i][AH - 1];
        wa[odd][i][0] = static_cast<int>(__builtin_amdgcn_perm(x.y, x.x, sel));
        wa[odd][i][1] = static_cast<int>(__builtin_amdgcn_perm(x.w, x.z, sel));
        wa[odd][i][2] = static_cast<int>(__builtin_amdgcn_perm(y.y, y.x, sel));
        wa[odd][i][3] = static_cast<int>(__builtin_amdgcn_perm(y.w, y.z, sel));
      } else {
        const uint4 x = pa[set][i][0];
        wa[odd][i][0] = (odd ? x.x : x.x << 4) & mm;
        wa[odd][i][1] = (odd ? x.y : x.y << 4) & mm;
        wa[odd][i][2] = (odd ? x.z : x.z << 4) & mm;
        wa[odd][i][3] = (odd ? x.w : x.w << 4) & mm;
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const uint4 x = pb[set][j];
      wb[odd][j][0] = (odd ? x.x : x.x << 4) & m;
      wb[odd][j][1] = (odd ? x.y : x.y << 4) & m;
      wb[odd][j][2] = (odd ? x.z : x.z << 4) & m;
      wb[odd][j][3] = (odd ? x.w : x.w << 4) & m;
    }
  };
  auto mfma = [&](int odd) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa[odd][i], wb[odd][j], acc[i][j], 0, 0, 0);
  };
  // The scales of the tile's rows and columns.
  if constexpr (EPI != EPI_I32) {
#pragma unroll
    for (int i = 0; i < ((BM + BN) / 64 + NW - 1) / NW; ++i) {
      const int l = wv + i * NW;
      if (l < (BM + BN) / 64) {
        const bool isx = l < BM / 64;
        const int64_t idx = (isx ? l : l - BM / 64) * 64 + lane, lim = isx ? a.M - 1 - m0 : a.N - 1 - n0;
        dma4(lds0 + LDSB + l * 256, static_cast<uint32_t>(idx < lim ? idx : lim) * 4, isx ? a.xs + m0 : a.ws + n0);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nk) issue(s, s, std::integral_constant<int, 0>{}, std::integral_constant<int, LPW>{});
  // Wait for a stage, with `ahead` whole stages issued after it.
  auto wait_stage = [&](int ahead) {
    if (ahead >= NS - 1) wait_vm<(NS - 1) * LPW>();
    else if (NS > 2 && ahead == NS - 2) wait_vm<(NS > 2 ? NS - 2 : 0) * LPW>();
    else if (NS > 3 && ahead == NS - 3) wait_vm<(NS > 3 ? NS - 3 : 0) * LPW>();
    else wait_vm<0>();
  };
  wait_stage(nk - 1);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read(0, grp, 0);
  widen(0, 0, grp < n64 ? 0xF0F0F0F0u : 0u);
  // (Opaque, so that the loop's widening stays where it is written.)
#pragma unroll
  for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(wa[0][i]));
#pragma unroll
  for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(wb[0][j]));
  int b = 0, bp = NS - 1;
  for (int s = 0; s < nk; ++s) {
    const int bn = b + 1 == NS ? 0 : b + 1;
    const int pair0 = s * (P / 2) + grp;
    const int sprev = s > 0 ? s - 1 + NS : nk;
    static_for<NP>([&](auto P_) {
      constexpr int p = decltype(P_)::value;
      constexpr int sl = p + 1 == NP ? 0 : 2 + 2 * p;
      const bool on = pair0 + p * KG < n64;
      const bool onn = pair0 + (p + 1 < NP ? (p + 1) * KG : P / 2) < n64;
      if (p + 1 == NP && s + 1 < nk) {
        // Fragments of this stage are in registers; stage s + 1 has landed.
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wait_stage(min(nk - 1 - (s + 1), NS - 2));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      // Phase A: even channels multiplied, odd ones widened, next pair read.
      issue_slot(p + 1 == NP ? s + NS : sprev, p + 1 == NP ? b : bp, std::integral_constant<int, sl>{});
      __builtin_amdgcn_sched_barrier(0);
      if (p + 1 < NP) read(b, grp + (p + 1) * KG, (p + 1) & 1);
      else read(bn, grp, 0);
      mfma(0);
      widen(p & 1, 1, on ? 0xF0F0F0F0u : 0u);
      // Phase B: odd channels multiplied, the next pair's even ones widened.
      issue_slot(p + 1 == NP ? s + NS : sprev, p + 1 == NP ? b : bp, std::integral_constant<int, sl + 1>{});
      __builtin_amdgcn_sched_barrier(0);
      mfma(1);
      widen((p + 1) & 1, 0, onn ? 0xF0F0F0F0u : 0u);
    });
    bp = b;
    b = bn;
  }
  // Epilogue.
  constexpr int SH = A8 ? 4 : 8;
  const float* sxs = reinterpret_cast<const float*>(smem + LDSB);
  const float* sws = sxs + BM;
  float bias[NC], gate[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    bias[j] = static_cast<float>(__builtin_bit_cast(_Float16, biasb[j]));
    gate[j] = static_cast<float>(__builtin_bit_cast(_Float16, gateb[j]));
  }
  auto half_of = [](float y) -> uint16_t {
    if constexpr (EPI == EPI_F16) return __builtin_bit_cast(uint16_t, static_cast<_Float16>(y));
    else if constexpr (EPI == EPI_GELU_F16)
      return __builtin_bit_cast(uint16_t, static_cast<_Float16>(gelu_tanh(static_cast<float>(static_cast<_Float16>(y)))));
    else return f32_to_bf16_rne(y);
  };
  auto store8 = [&](int64_t gr, int64_t gc, uint4 v) {  // 8 16-bit outputs (ldc % 8 == 0: 16-byte aligned)
    uint16_t* C = static_cast<uint16_t*>(a.C);
    if (gc + 8 <= a.N) {
      *reinterpret_cast<uint4*>(C + gr * a.ldc + gc) = v;
    } else {
      const uint16_t h[8] = {static_cast<uint16_t>(v.x), static_cast<uint16_t>(v.x >> 16),
                             static_cast<uint16_t>(v.y), static_cast<uint16_t>(v.y >> 16),
                             static_cast<uint16_t>(v.z), static_cast<uint16_t>(v.z >> 16),
                             static_cast<uint16_t>(v.w), static_cast<uint16_t>(v.w >> 16)};
      for (int e = 0; e < 8 && gc + e < a.N; ++e) C[gr * a.ldc + gc + e] = h[e];
    }
  };
  if constexpr (ROWS || STAGED) __syncthreads();  // every fragment read of the last stage is done
  if constexpr (ROWS) {
    int32_t* part = reinterpret_cast<int32_t*>(smem) + grp * (BM * BN);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          part[(wm * 32 * TM + i * 32 + 8 * (e / 4) + row_grp + e % 4) * BN + wn * 32 * TN + j * 32 + col_in] = acc[i][j][e];
    __syncthreads();
    const int64_t gc = n0 + rcol;
    if (gc >= a.N) return;
    float w[V];
#pragma unroll
    for (int e = 0; e < V; ++e) w[e] = EPI != EPI_I32 ? sws[rcol + e] : 0.0f;
#pragma unroll
    for (int c = 0; c < NPC; ++c) {
      const int lr = tid / (BN / V) + c * RSTEP;
      const int64_t gr = m0 + lr;
      if (gr >= a.M) break;
      int v[V];
#pragma unroll
      for (int e = 0; e < V; ++e) v[e] = 0;
#pragma unroll
      for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int e = 0; e < V; e += 4) {
          const v4i p = *reinterpret_cast<const v4i*>(smem + (static_cast<size_t>(g) * BM * BN + lr * BN + rcol + e) * 4);
#pragma unroll
          for (int u = 0; u < 4; ++u) v[e + u] += p[u];
        }
      if constexpr (EPI == EPI_I32) {
        int32_t* o = static_cast<int32_t*>(a.C) + gr * a.ldc + gc;  // (ldc % 4 == 0: 16-byte aligned)
        if (gc + 4 <= a.N) *reinterpret_cast<v4i*>(o) = v4i{v[0] >> SH, v[1] >> SH, v[2] >> SH, v[3] >> SH};
        else
          for (int e = 0; e < 4 && gc + e < a.N; ++e) o[e] = v[e] >> SH;
      } else {
        float y[V];
#pragma unroll
        for (int e = 0; e < V; ++e) y[e] = static_cast<float>(v[e] >> SH) * sxs[lr] * w[e] + bias[e];
        if constexpr (EPI == EPI_RESID_F32) {
          float* o = static_cast<float*>(a.C) + gr * a.ldc + gc;
          if (gc + 4 <= a.N) {
            float4 r;
            if constexpr (EARLY) r = rearly[c];
            else r = *reinterpret_cast<const float4*>(o);
            *reinterpret_cast<float4*>(o) = make_float4(fmaf(gate[0], y[0], r.x), fmaf(gate[1], y[1], r.y),
                                                        fmaf(gate[2], y[2], r.z), fmaf(gate[3], y[3], r.w));
          } else {
            for (int e = 0; e < 4 && gc + e < a.N; ++e) o[e] = fmaf(gate[e], y[e], o[e]);
          }
        } else {
          uint32_t h[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            h[e] = half_of(y[(2 * e) % V]) | static_cast<uint32_t>(half_of(y[(2 * e + 1) % V])) << 16;
          store8(gr, gc, make_uint4(h[0], h[1], h[2], h[3]));
        }
      }
    }
    return;
  }
  // From the accumulators: each lane's rows come in runs of four.
  uint16_t* tile = reinterpret_cast<uint16_t*>(smem);
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    // (Every old residual value of the block is read before its first store.)
    float rold[4][TN][4];
    if constexpr (EPI == EPI_RESID_F32) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int64_t r = m0 + wm * 32 * TM + i * 32 + 8 * q + row_grp + u, gr = r < a.M ? r : a.M - 1;
            const int64_t gc = n0 + wn * 32 * TN + j * 32 + col_in, gcc = gc < a.N ? gc : a.N - 1;
            rold[q][j][u] = static_cast<const float*>(a.C)[gr * a.ldc + gcc];
          }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int lr0 = wm * 32 * TM + i * 32 + 8 * q + row_grp;  // row within the tile
      const float4 x4 = EPI != EPI_I32 ? *reinterpret_cast<const float4*>(sxs + lr0) : make_float4(0, 0, 0, 0);
      const float xr[4] = {x4.x, x4.y, x4.z, x4.w};
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int lc = wn * 32 * TN + j * 32 + col_in;
        const int64_t gc = n0 + lc;
        const float wsc = EPI != EPI_I32 ? sws[lc] : 0.0f;
        if constexpr (STAGED) {
          // Rows / columns past the edge are staged but not written back.
#pragma unroll
          for (int u = 0; u < 4; ++u)
            tile[(lr0 + u) * TP + lc] = half_of(static_cast<float>(acc[i][j][4 * q + u] >> SH) * xr[u] * wsc + bias[j]);
          continue;
        }
        if (gc >= a.N) continue;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int64_t gr = m0 + lr0 + u;
          if (gr >= a.M) continue;
          const int v = acc[i][j][4 * q + u] >> SH;
          const int64_t off = gr * a.ldc + gc;
          if constexpr (EPI == EPI_I32) {
            static_cast<int32_t*>(a.C)[off] = v;
          } else if constexpr (EPI == EPI_RESID_F32) {
            const float y = static_cast<float>(v) * xr[u] * wsc + bias[j];
            static_cast<float*>(a.C)[off] = fmaf(gate[j], y, rold[q][j][u]);
          }
        }
      }
    }
  }
  if constexpr (STAGED) {
    static_assert((BM * BN / 8) % NT == 0, "output pieces per thread");
    __syncthreads();
#pragma unroll
    for (int c = 0; c < (BM * BN / 8) / NT; ++c) {
      const int id = tid + NT * c;
      const int lr = id / (BN / 8), pcx = (id % (BN / 8)) * 8;
      const int64_t gr = m0 + lr, gc = n0 + pcx;
      if (gr >= a.M || gc >= a.N) continue;
      store8(gr, gc, *reinterpret_cast<const uint4*>(&tile[lr * TP + pcx]));
    }
  }
}

}  // namespace
}  // namespace oq
