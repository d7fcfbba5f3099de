// Streaming projection GEMM for K = 256 / 512 (gfx950): C[M,N] = A[M,K] * Wt[N,K]^T with A given
// as a head/tail pair of fp16 planes.
//
// Same division of labour as the streaming output projection: a workgroup keeps its tile of A
// (32 or 64 rows, both planes) in the LDS for its whole life, filled once straight from global
// memory, and the weights - stored at load time in MFMA fragment order - stream through
// registers, one fully coalesced 1 KiB load per fragment, running a few k-steps ahead of their
// use.  The main loop has no LDS writes, no barriers and no address arithmetic; against the tiled
// kernel (both operand tiles written to and read from the LDS for every 64 MFMAs) the LDS
// traffic per MFMA drops to a quarter.  Both planes are multiplied with the same weight
// fragment into one fp32 accumulator.
//
// A wave owns strips of 64 output columns (wave, wave + 8, ... of the workgroup's range) and all
// rows of the tile; the epilogue does what the tiled kernel's does (bias, scale, ReLU, residual, two
// destinations, optional tail plane).  Here the A fragment is the row operand of the MFMA, so a
// lane owns an output column and a store instruction covers 128 contiguous bytes per row.  Tiles
// inside the matrix take an epilogue without branches, so that the stores of a strip are issued
// back to back; encoder-sized launches mark their whole-line streams non-temporal.
//
// Fragment order of Wp: [strip = n / 64][ks = k / 16][nb = (n % 64) / 32][lane][8 halfs] with
// lane = n % 32 + 32 * ((k % 16) / 8).
#include "nt_kernels.h"

#include <mutex>
#include <type_traits>

namespace nt {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int GS_WAVES = 8;

bool gemm_stream_supported(int N, int K) { return (K == 256 || K == 512) && N % 64 == 0; }

// Rows wave, wave + 8, ... of a tile, element lane * NE + j of the i-th in xv[i][j]: LayerNorm (fp32 statistics: mean first, then the
// biased variance or mean absolute deviation of the centred values), split into head (and tail) planes in the LDS.
template <int NE, int RPW, int TM, bool TAIL>
__device__ __forceinline__ void gs_normalise(const float (&xv)[RPW][NE], const GemmLayerNorm &ln, _Float16 *sh, int wave, int lane) {
  constexpr int K = NE * 64, LD = K + 8;
  float gam[NE], bet[NE];
#pragma unroll
  for (int j = 0; j < NE; j += 4) {
    *(float4 *)&gam[j] = *(const float4 *)(ln.gamma + lane * NE + j);
    *(float4 *)&bet[j] = *(const float4 *)(ln.beta + lane * NE + j);
  }
  float mean[RPW], rstd[RPW];
#pragma unroll
  for (int i = 0; i < RPW; i++) {
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < NE; j++) sum += xv[i][j];
    mean[i] = sum;
  }
#pragma unroll
  for (int i = 0; i < RPW; i++) mean[i] = wave_sum(mean[i]);
#pragma unroll
  for (int i = 0; i < RPW; i++) {
    mean[i] = mean[i] / (float)K;
    float q = 0.f;
#pragma unroll
    for (int j = 0; j < NE; j++) {
      const float c = xv[i][j] - mean[i];
      q += ln_term(c, ln.eps.l1);
    }
    rstd[i] = q;
  }
#pragma unroll
  for (int i = 0; i < RPW; i++) rstd[i] = wave_sum(rstd[i]);
#pragma unroll
  for (int i = 0; i < RPW; i++) {
    rstd[i] = ln_rscale(rstd[i] / (float)K, ln.eps);
    typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
    halfNE hi, lo;
#pragma unroll
    for (int j = 0; j < NE; j++) {
      const float y = as_f32(gam[j] * ((xv[i][j] - mean[i]) * rstd[i]) + bet[j]);
      hi[j] = (_Float16)y;
      lo[j] = (_Float16)(y - (float)hi[j]);
    }
    const int R = wave + GS_WAVES * i;
    *(halfNE *)(sh + R * LD + lane * NE) = hi;
    if (TAIL) *(halfNE *)(sh + (R + TM) * LD + lane * NE) = lo;
  }
}

// RB = 32-row blocks per tile (1: decoder-sized M; 2: encoder-sized M).
// LN = true: A_hi points to fp32 rows X[M][lda] instead; the tile is LayerNorm-ed (fp32 statistics: mean first, then
// the biased variance of the centred values) and split into head/tail planes while it is written to the LDS, which
// saves the separate LayerNorm kernel and the round trip of its output through memory.
// TAIL = false: only the head plane of A is multiplied (11 significant bits: half the MFMA work and half the tile).
// NB = 32-column blocks per wave.  2: strips of 64 columns through a ring of eight k-steps.  1: strips of 32 columns whose
// fragments (all of them for K = 256 / 512, sixteen k-steps ahead for several passes) are requested before the tile is
// filled - for launches of few workgroups, whose time is the latency of a wave's stream: half the columns and one turn of the
// memory system instead of five.  The sums are the same, term by term.
// NC > 1: the contraction runs over NC * K columns of A in NC passes over the K-wide tile (K = 512, planes from memory):
// between passes the tile is refilled behind a barrier while the weight ring keeps streaming, and every wave keeps the
// accumulators of its one strip (N is 512 per column group) - the second matrix of an FFN, whose K is the FFN width.
// CHAIN: the rows that are normalised are made here, x += A * Wo^T + bias (A: planes, Wo: K x K), see GemmChain.
template <int RB, int K, bool C_F32, bool LN, bool TAIL, int NC, int NB, bool CHAIN>
__device__ __forceinline__ void gs_tile(const _Float16 *__restrict__ A_hi, const _Float16 *__restrict__ A_lo, long lda, int M,
                                        const _Float16 *__restrict__ Wp, int N, int col_groups, const GemmEpilogue &e, const GemmLayerNorm &ln,
                                        const GemmChain &ch) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  _Float16 *sh = (_Float16 *)smem;
  constexpr int TM = 32 * RB, ROWS = (TAIL ? 2 : 1) * TM;  // LDS fragment rows: head rows, then tail rows
  constexpr int LD = K + 8;                   // halfs per LDS row: the 16 B pad keeps the fragment reads conflict-free
  constexpr int KS = K / 16;
  // register slots of W fragments per wave; the lookahead is SL - 1 k-steps.  (A deeper ring did not shorten the
  // decoder-sized launches, and fewer registers leave room for other kernels' waves on the same CU.)
  constexpr int SL = NB == 2 ? 8 : NC > 1 ? 16 : KS;
  constexpr int LA = SL == KS && NC == 1 ? SL : SL - 1;  // k-steps requested ahead
  constexpr int SW = 32 * NB;                            // columns of a strip
  constexpr int NOPS = (TAIL ? 2 : 1) * RB;
  static_assert(KS % SL == 0, "the ring of W slots must divide the k-steps of a strip");
  static_assert(NC == 1 || (K == 512 && !LN), "several passes: 512-wide tiles of planes only");
  static_assert(!CHAIN || (K == 512 && LN && TAIL && NC == 1 && NB == 2), "the chain's tile has both planes of 512 columns");
  constexpr int KST = NC * KS;  // k-steps of a whole strip
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mt = blockIdx.x / col_groups, cg = blockIdx.x % col_groups;
  const int m0 = mt * TM;
  const int NS = N / SW;
  const int sb0 = (int)((long)cg * NS / col_groups), sb1 = (int)((long)(cg + 1) * NS / col_groups);
  // first fragment of a strip
  auto strip_at = [&](int s) { return NB == 2 ? s * (KST * 2048) : (s >> 1) * (KST * 2048) + (s & 1) * 1024; };

  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, N * (NC * K) * 2, 0x00020000);
  const int wlane = lane * 16;
  auto wload = [&](int soff, int nb) -> half8 {
    u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + nb * 1024, soff, 0);
    return __builtin_bit_cast(half8, t);
  };

  half8 wb[SL][NB];
  int strip = sb0 + wave;
  const bool have = strip < sb1;
  auto preload = [&]() {
    if (!have) return;
    const int sp = strip_at(strip);
#pragma unroll
    for (int q = 0; q < LA; q++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) wb[q][nb] = wload(sp + q * 2048, nb);
  };

  // ---- the A tile: global memory -> LDS.  Rows past M repeat row M - 1 (their results are never stored) ----
  // planes, K = 512: one wave instruction moves one row of one plane (1 KiB) without passing through registers;
  // pass c of NC takes columns c * K .. c * K + K - 1 of A
  auto fill_planes = [&](int c) {
#pragma unroll
    for (int i = 0; i < ROWS / GS_WAVES; i++) {
      const int R = wave + GS_WAVES * i;
      const _Float16 *src = R >= TM ? A_lo : A_hi;
      int m = m0 + (R % TM);
      m = m < M ? m : M - 1;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(src + (long)m * lda + c * K + lane * 8),
          (__attribute__((address_space(3))) void *)(sh + R * LD), 16, 0, RB == 2 ? 2 : 0);
    }
  };
  floatx16 acc[RB][NB];
  // fragment row of operand op: head rows of block op % RB, then the tail rows; two base registers, because the
  // byte offsets of the upper half do not fit the 16-bit offset field
  const _Float16 *hrow = sh + li * LD + g * 8;
  constexpr int HALF = ROWS > 32 ? ROWS / 2 : ROWS;  // LDS rows reached from the first base register
  int off2 = HALF * LD;
  asm volatile("" : "+v"(off2));
  const _Float16 *hrow2 = hrow + off2;
  auto frag = [&](int op, int ks) -> half8 {
    const int R0 = op * 32;  // ops 0 .. RB-1: head planes, RB .. 2RB-1: tail planes
    return *(const half8 *)((R0 < HALF ? hrow : hrow2) + (R0 % HALF) * LD + ks * 16);
  };
  half8 hf[NOPS];
  if constexpr (CHAIN) {
    // The projection before: one strip of 64 columns per wave, both planes; its ring runs on into this product's first strip.  The
    // product goes through the LDS, where the planes were, to be normalised as rows that come from memory are: the same sums in
    // the same order as two launches.
    constexpr int NE = K / 64, RPW = TM / GS_WAVES, LDX = K + 8;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc((void *)ch.Wo, 0, K * K * 2, 0x00020000);
    auto oload = [&](int soff, int nb) -> half8 {
      return __builtin_bit_cast(half8, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(ors, wlane + nb * 1024, soff, 0));
    };
    const int ocur = wave * (KS * 2048), onext = strip_at(strip);
    float obias[NB], xv[RPW][NE];
    fill_planes(0);
#pragma unroll
    for (int nb = 0; nb < NB; nb++) obias[nb] = ch.bias[wave * 64 + nb * 32 + li];
#pragma unroll
    for (int q = 0; q < LA; q++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) wb[q][nb] = oload(ocur + q * 2048, nb);
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    auto request_rows = [&]() {
#pragma unroll
      for (int i = 0; i < RPW; i++) {
        const float *xr = ch.x + (long)min(m0 + wave + GS_WAVES * i, M - 1) * K + lane * NE;
#pragma unroll
        for (int j = 0; j < NE; j += 4) {
          const f32x4 t = *(const f32x4 *)(xr + j);
          xv[i][j] = t[0], xv[i][j + 1] = t[1], xv[i][j + 2] = t[2], xv[i][j + 3] = t[3];
        }
      }
    };
#pragma unroll
    for (int op = 0; op < NOPS; op++) hf[op] = frag(op, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const int tgt = ks + LA;
      // the residual rows, behind the last fragments of this product: nothing of it waits for them (from the start 1 to 2 % slower).
      // Cached, unlike the rows of the other form: 16,375 tokens 841 -> 797 us a whole encoder
      if (tgt == KS) {
        request_rows();
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int op = 0; op < NOPS; op++) {
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
          if (ks == 0 && op < RB) {
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            acc[op % RB][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[op], wb[ks % SL][nb], zero, 0, 0, 0);
          } else {
            acc[op % RB][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[op], wb[ks % SL][nb], acc[op % RB][nb], 0, 0, 0);
          }
        }
        if (ks + 1 < KS) hf[op] = frag(op, ks + 1);
        if (op == 0) {
#pragma unroll
          for (int nb = 0; nb < NB; nb++) wb[tgt % SL][nb] = tgt < KS ? oload(ocur + tgt * 2048, nb) : wload(onext + (tgt - KS) * 2048, nb);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();  // every wave is done with the planes: the product takes their place, whole rows of it are read back
    float *sx = (float *)smem;
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++)
          sx[(rb * 32 + (v >> 2) * 8 + g * 4 + (v & 3)) * LDX + wave * 64 + nb * 32 + li] = acc[rb][nb][v] + obias[nb];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPW; i++)
#pragma unroll
      for (int j = 0; j < NE; j += 4) {
        const f32x4 t = *(const f32x4 *)(sx + (wave + GS_WAVES * i) * LDX + lane * NE + j);
        xv[i][j] += t[0], xv[i][j + 1] += t[1], xv[i][j + 2] += t[2], xv[i][j + 3] += t[3];
      }
    __syncthreads();
    gs_normalise<NE, RPW, TM, TAIL>(xv, ln, sh, wave, lane);
    auto put_row = [&](int i) {
      float *xr = ch.x + (long)(m0 + wave + GS_WAVES * i) * K + lane * NE;
#pragma unroll
      for (int j = 0; j < NE; j += 4) {
        const f32x4 t = {xv[i][j], xv[i][j + 1], xv[i][j + 2], xv[i][j + 3]};
        if (RB == 2) __builtin_nontemporal_store(t, (f32x4 *)(xr + j));
        else *(f32x4 *)(xr + j) = t;
      }
    };
    if (__builtin_expect(m0 + TM <= M, 1)) {
#pragma unroll
      for (int i = 0; i < RPW; i++) put_row(i);
    } else {
#pragma unroll
      for (int i = 0; i < RPW; i++)
        if (m0 + wave + GS_WAVES * i < M) put_row(i);
    }
  } else if constexpr (LN) {
    // a wave takes rows wave, wave + 8, ...; a lane holds NE consecutive elements of the row
    constexpr int NE = K / 64, RPW = TM / GS_WAVES;
    const float *X = (const float *)A_hi;
    float xv[RPW][NE];
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      int m = m0 + wave + GS_WAVES * i;
      m = m < M ? m : M - 1;
      const float *xr = X + (long)m * lda + lane * NE;
#pragma unroll
      for (int j = 0; j < NE; j += 4) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        // encoder-sized launches stream their rows, residuals and fp32 outputs past the L2 (non-temporal), so that
        // the weight fragments, which every workgroup reads, stay in it.  Only whole-line accesses are marked:
        // where a line is consumed or produced in pieces (the q/k/v reads and half-line context stores of the encoder
        // attention), the pieces rely on the cache and the hint cost 7 % of the whole job
        const f32x4 t = RB == 2 ? __builtin_nontemporal_load((const f32x4 *)(xr + j)) : *(const f32x4 *)(xr + j);
        xv[i][j] = t[0], xv[i][j + 1] = t[1], xv[i][j + 2] = t[2], xv[i][j + 3] = t[3];
      }
    }
    if (NB == 1) {  // behind the rows: their wait does not include the fragments
      __builtin_amdgcn_sched_barrier(0);
      preload();
    }
    gs_normalise<NE, RPW, TM, TAIL>(xv, ln, sh, wave, lane);
  } else if (K == 512) {
    fill_planes(0);
    if (NB == 1) preload();
  } else {
    constexpr int CPR = K / 8, PER_T = ROWS * CPR / (GS_WAVES * 64);
    if (NB == 1) preload();
    u32x4 fr[PER_T];
#pragma unroll
    for (int i = 0; i < PER_T; i++) {
      const int c = tid + GS_WAVES * 64 * i, R = c / CPR, kc = c % CPR;
      const _Float16 *src = R >= TM ? A_lo : A_hi;
      int m = m0 + (R % TM);
      m = m < M ? m : M - 1;
      fr[i] = *(const u32x4 *)(src + (long)m * lda + kc * 8);
    }
#pragma unroll
    for (int i = 0; i < PER_T; i++) {
      const int c = tid + GS_WAVES * 64 * i, R = c / CPR, kc = c % CPR;
      *(u32x4 *)(sh + R * LD + kc * 8) = fr[i];
    }
  }
  if (!CHAIN) {
    if (NB == 2) preload();
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's rows have landed in the LDS before the barrier
  }
  __syncthreads();
  if (!have) {
    if (NC > 1) {  // a wave without a strip still fills its rows of every pass
#pragma unroll 1
      for (int c = 1; c < NC; c++) {
        __syncthreads();
        fill_planes(c);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
      }
    }
    return;
  }
  // Two waves share a SIMD.  With equal priority they take turns at the matrix pipe, finish their strips together
  // and then both sit in the store phase of the epilogue (the long one when the output is fp32) while the pipe
  // idles.  Giving one of them priority makes the phases alternate instead.
  if (wave < GS_WAVES / 2) __builtin_amdgcn_s_setprio(2);

#pragma unroll
  for (int op = 0; op < NOPS; op++) hf[op] = frag(op, 0);

  if (NC > 1) {
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[rb][nb][v] = 0.f;
  }
  for (; strip < sb1; strip += GS_WAVES) {
    const bool more = strip + GS_WAVES < sb1;
    int pcur = strip_at(strip);
    const int pend = pcur + (KST - 1) * 2048;
    const int pnext = strip_at(more ? strip + GS_WAVES : strip);
    // bias and scale of the strip's columns, requested here so that the epilogue does not wait for them behind the
    // weight fragments in flight
    float bias[NB], scl[NB];
#pragma unroll
    for (int nb = 0; nb < NB; nb++) {
      const int n = strip * SW + nb * 32 + li;
      bias[nb] = e.bias ? e.bias[n] : 0.f;
      scl[nb] = (n < e.scale_cols) ? e.scale : 1.f;
    }
    // The k-loop of a strip, over the head plane's row blocks alone (NO = RB) or over both planes' (NO = NOPS): the
    // epilogue's tail_col0 .. tail_col1 name the output columns whose strips take the tail plane as well.
    auto k_loop = [&](auto nops_tag, const float (&bias_)[NB], const float (&scl_)[NB]) {
      constexpr int NO = decltype(nops_tag)::value;
#pragma unroll
      for (int ks = 0; ks < KS; ks++) {
        const int tgt = ks + LA;
        // several passes: the ring simply runs on into the next pass's fragments of the same strip (at the end of the
        // last pass it re-reads the strip's last fragment)
        const int pf = NC > 1 ? min(pcur + tgt * 2048, pend) : tgt < KS ? pcur + tgt * 2048 : pnext + (tgt - KS) * 2048;
        const int ksn = (ks + 1) % KS;
#pragma unroll
        for (int op = 0; op < NO; op++) {
#pragma unroll
          for (int nb = 0; nb < NB; nb++) {
            if (NC == 1 && ks == 0 && op < RB) {
              const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
              acc[op % RB][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[op], wb[ks % SL][nb], zero, 0, 0, 0);
            } else {
              acc[op % RB][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[op], wb[ks % SL][nb], acc[op % RB][nb], 0, 0, 0);
            }
          }
          // refill what was just consumed; the scheduling barrier keeps the loads this far ahead of their use
          hf[op] = frag(op, ksn);
          if (LA < SL && op == 0) {
#pragma unroll
            for (int nb = 0; nb < NB; nb++) wb[tgt % SL][nb] = wload(pf, nb);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        // the wait for bias and scale is taken here, where it counts only the fragments requested since; left to the
        // epilogue it becomes a wait for everything in flight
        if (NB == 2 && ks == SL) asm volatile("" ::"v"(bias_[0]), "v"(bias_[NB - 1]), "v"(scl_[0]), "v"(scl_[NB - 1]));
      }
    };
    const bool with_tail = TAIL && strip * SW >= e.tail_col0 && strip * SW < e.tail_col1;
#pragma unroll 1
    for (int c = 0; c < NC; c++) {
      if (NC > 1 && c > 0) {
        // next pass: every wave is done with the tile, it is refilled, and the first fragments are read again
        __syncthreads();
        fill_planes(c);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
#pragma unroll
        for (int op = 0; op < NOPS; op++) hf[op] = frag(op, 0);
        pcur += KS * 2048;
      }
      // (the choice by output columns is for the single-pass form; a second instance of the loop here costs registers)
      if (NC > 1 || with_tail) k_loop(std::integral_constant<int, NOPS>{}, bias, scl);
      else k_loop(std::integral_constant<int, RB>{}, bias, scl);
    }
    // ---- epilogue of the strip: acc[rb][nb][v] is C[m0 + rb*32 + (v/4)*8 + g*4 + v%4][strip*64 + nb*32 + li] ----
    // Addresses are a uniform 64-bit base per 32 x 32 block plus a 32-bit lane offset (n_split is a multiple of 32,
    // so a block never straddles the two destinations).
    //
    // The stores of a strip must go out back to back.  Loads and stores of a wave complete in order on one counter;
    // with a per-row guard around every store the compiler can no longer count what is outstanding and waits for
    // the counter to reach zero before each store, i.e. for the acknowledgement of the previous one (150 ns each,
    // 10 us per strip).  So the guards are hoisted: a tile that lies within M (all but the last) and the
    // presence of a residual are decided once, uniformly, and the path taken is straight-line code.  The residual
    // may be the destination itself (in-place update); a block's residual values are requested before the
    // stores of the block before it, so that waiting for them does not wait for those stores.
    constexpr int CE = C_F32 ? 4 : 2;
    constexpr int NBLK = NB * RB;  // 32 x 32 blocks of the strip: block = nb * RB + rb
    // ce: bytes per element of the block's destination (fp32 kernels may write their first destination as plain
    // fp16: GemmEpilogue::first_f16; the choice is uniform over a block)
    auto block_at = [&](int blk, char *&dblock, const char *&rblock, unsigned &dlane, unsigned &rlane, long &ld,
                        int &mb, int &ce) {
      const int nb = blk / RB, rb = blk % RB;
      const int nbase = strip * SW + nb * 32;  // uniform
      const bool first = nbase < e.n_split;
      char *dst = (char *)(first ? e.dst0 : e.dst1);
      ld = first ? e.ld0 : e.ld1;
      const int ncb = first ? nbase : nbase - e.n_split;
      mb = m0 + rb * 32;  // uniform
      ce = (C_F32 && e.first_f16 && first) ? 2 : CE;
      dblock = dst + ((long)mb * ld + ncb) * ce;
      rblock = (const char *)e.resid + ((long)mb * e.ldr + nbase) * 4;
      dlane = (unsigned)((g * 4 * ld + li) * ce);
      rlane = (unsigned)((g * 4 * e.ldr + li) * 4);
      // the per-row offsets derived from these do not depend on the strip; computed once and kept, they would hold
      // dozens of registers through the main loop
      asm volatile("" : "+v"(dlane), "+v"(rlane));
    };
    auto finish = [&](int blk, int v, float r) -> float {
      float val = (acc[blk % RB][blk / RB][v] + bias[blk / RB]) * scl[blk / RB];
      if (e.relu) val = fmaxf(val, 0.f);
      return val + r;
    };
    auto put = [&](char *at_, float val, int ce) {
      if (C_F32 && ce == 2) {
        *(_Float16 *)at_ = (_Float16)val;
      } else if (C_F32) {
        if (RB == 2) __builtin_nontemporal_store(val, (float *)at_);
        else *(float *)at_ = val;
      } else {
        val = as_f32(val);
        const _Float16 hi = (_Float16)val;
        *(_Float16 *)at_ = hi;  // 64 bytes per row and instruction: the other half of the line follows, keep it cached
        if (e.dst_lo_offset) *((_Float16 *)at_ + e.dst_lo_offset) = (_Float16)(val - (float)hi);
      }
    };
    // The projections that follow a LayerNorm add no residual, and the others all do: the straight-line path is
    // compiled for that case only; anything else takes the guarded path below.
    constexpr bool RESID = !LN;
    if (__builtin_expect(m0 + TM <= M && RESID == (e.resid != nullptr), 1)) {
      float res[RESID ? 2 : 1][16];
      auto request = [&](int blk) {
        char *dblock; const char *rblock; unsigned dlane, rlane; long ld; int mb, ce;
        block_at(blk, dblock, rblock, dlane, rlane, ld, mb, ce);
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int r = (v >> 2) * 8 + (v & 3);
          const float *rp = (const float *)(rblock + (rlane + (unsigned)(r * e.ldr * 4)));
          res[blk & 1][v] = RB == 2 ? __builtin_nontemporal_load(rp) : *rp;
        }
      };
      if (RESID) request(0);
#pragma unroll
      for (int blk = 0; blk < NBLK; blk++) {
        __builtin_amdgcn_sched_barrier(0);  // one block at a time: bounds the loads and addresses in flight
        if (RESID && blk + 1 < NBLK) request(blk + 1);
        __builtin_amdgcn_sched_barrier(0);
        char *dblock; const char *rblock; unsigned dlane, rlane; long ld; int mb, ce;
        block_at(blk, dblock, rblock, dlane, rlane, ld, mb, ce);
        if (C_F32 && ce == 2) {  // uniform: the stores of a block stay straight-line code of one kind
#pragma unroll
          for (int v = 0; v < 16; v++) {
            const int r = (v >> 2) * 8 + (v & 3);
            put(dblock + (dlane + (unsigned)(r * ld * 2)), finish(blk, v, RESID ? res[blk & 1][v] : 0.f), 2);
          }
        } else {
#pragma unroll
          for (int v = 0; v < 16; v++) {
            const int r = (v >> 2) * 8 + (v & 3);
            put(dblock + (dlane + (unsigned)(r * ld * CE)), finish(blk, v, RESID ? res[blk & 1][v] : 0.f), CE);
          }
        }
      }
    } else {
      // the last row tile (or the unusual residual case): every row is checked against M
#pragma unroll
      for (int blk = 0; blk < NBLK; blk++) {
        __builtin_amdgcn_sched_barrier(0);
        char *dblock; const char *rblock; unsigned dlane, rlane; long ld; int mb, ce;
        block_at(blk, dblock, rblock, dlane, rlane, ld, mb, ce);
        // read the 16 residual values of the block first, then compute and store
        float res[16];
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int r = (v >> 2) * 8 + (v & 3);
          res[v] = (e.resid && mb + r + g * 4 < M) ? *(const float *)(rblock + (rlane + (unsigned)(r * e.ldr * 4))) : 0.f;
        }
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int r = (v >> 2) * 8 + (v & 3);
          if (mb + r + g * 4 >= M) continue;
          put(dblock + (dlane + (unsigned)(r * ld * ce)), finish(blk, v, res[v]), ce);
        }
      }
      // Nothing of this path may be left in flight at the end of the iteration: what is pending here (loads into
      // registers that the other path reuses) is also assumed pending there, and costs it a full wait per strip.
      __builtin_amdgcn_s_waitcnt(0x0F70);
    }
  }
}

template <int RB, int K, bool C_F32, bool LN, bool TAIL, int NC, int NB>
__global__ __launch_bounds__(GS_WAVES * 64) void gemm_stream_kernel(const _Float16 *__restrict__ A_hi,
                                                                   const _Float16 *__restrict__ A_lo, long lda, int M,
                                                                   const _Float16 *__restrict__ Wp, int N, int col_groups,
                                                                   GemmEpilogue e, GemmLayerNorm ln) {
  gs_tile<RB, K, C_F32, LN, TAIL, NC, NB, false>(A_hi, A_lo, lda, M, Wp, N, col_groups, e, ln, GemmChain{});
}
template <int RB>
__global__ __launch_bounds__(GS_WAVES * 64) void gemm_chain_kernel(const _Float16 *__restrict__ A_hi, const _Float16 *__restrict__ A_lo, long lda,
                                                                  int M, const _Float16 *__restrict__ Wp, int N, GemmEpilogue e, GemmLayerNorm ln,
                                                                  GemmChain ch) {
  gs_tile<RB, 512, true, true, true, 1, 2, true>(A_hi, A_lo, lda, M, Wp, N, 1, e, ln, ch);
}

// ---------------------------------------------------------------------------------------------------------------------
// An FFN in one launch: x += relu(LayerNorm(x) W1^T + b1) W2^T + b2, d = 512, hidden width 512 NC.  A workgroup has 32 rows; 512 hidden
// columns at a time go from the first product's accumulators through ReLU and the split into a second pair of planes in the LDS
// and straight into the second product, whose accumulators a wave keeps for its 64 output columns.  As two launches the hidden state
// travelled through memory as planes, 8 KB a row each way: 108 + 76 us at 16,384 tokens and 313 + 262 at 65,536 (F = 2,048), 131 and about
// 490 as one; 30 + 6 layer teacher 107.0 -> 102.2 ms, 8 heads and FFN 95.5 -> 91.4, submitted student 101.7 -> 97.4.  The matrix cores
// are busy 54 % of the time; the stream of both matrices (4 MB a tile at the CU's 64 bytes a clock) takes as long as their products.  The weight ring runs through both products without a break; a
// workgroup takes the tiles blockIdx.x, + gridDim.x, ... and requests the next tile's rows before the last product of this one.  The
// sums are those of the two launches, term by term.
// ---------------------------------------------------------------------------------------------------------------------
template <int NC>
__global__ __launch_bounds__(GS_WAVES * 64) void gemm_ffn_kernel(float *__restrict__ x, int M, GemmLayerNorm ln, const _Float16 *__restrict__ W1p,
                                                                const float *__restrict__ b1, const _Float16 *__restrict__ W2p,
                                                                const float *__restrict__ b2) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int K = 512, TM = 32, LD = K + 8, KS = K / 16, SL = 8, NE = K / 64, RPW = TM / GS_WAVES;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  _Float16 *sx = (_Float16 *)smem, *su = sx + 2 * TM * LD;  // planes of the rows and of the hidden state: head rows, then tail rows
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tiles = (M + TM - 1) / TM;
  const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc((void *)W1p, 0, NC * K * K * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc((void *)W2p, 0, NC * K * K * 2, 0x00020000);
  auto wload = [&](const __amdgpu_buffer_rsrc_t &r, int soff, int nb) -> half8 {
    return __builtin_bit_cast(half8, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(r, lane * 16 + nb * 1024, soff, 0));
  };
  auto at1 = [&](int c) { return (c * GS_WAVES + wave) * (KS * 2048); };       // this wave's strip of chunk c of the first matrix
  auto at2 = [&](int c) { return wave * (NC * KS * 2048) + c * (KS * 2048); };  // and the k-range of chunk c of its strip of the second

  half8 wb[SL][2];
  floatx16 acc2[2];
  float xv[RPW][NE];
  auto request_rows = [&](int m0) {  // rows past M repeat row M - 1
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      const float *xr = x + (long)min(m0 + wave + GS_WAVES * i, M - 1) * K + lane * NE;
#pragma unroll
      for (int j = 0; j < NE; j += 4) {
        const f32x4 t = *(const f32x4 *)(xr + j);
        xv[i][j] = t[0], xv[i][j + 1] = t[1], xv[i][j + 2] = t[2], xv[i][j + 3] = t[3];
      }
    }
  };
  // 32 k-steps over both planes; the ring holds k-steps 0 .. SL - 2 of `cur` on entry and of `next` on exit
  auto k_loop = [&](const _Float16 *planes, const __amdgpu_buffer_rsrc_t &rc, int cur, const __amdgpu_buffer_rsrc_t &rn, int next, floatx16 (&acc)[2],
                    auto fresh_tag) __attribute__((always_inline)) {
    constexpr bool FRESH = decltype(fresh_tag)::value;
    const _Float16 *hrow = planes + li * LD + g * 8;
    half8 hf[2];
    hf[0] = *(const half8 *)hrow;
    hf[1] = *(const half8 *)(hrow + TM * LD);
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int op = 0; op < 2; op++) {
#pragma unroll
        for (int nb = 0; nb < 2; nb++) {
          if (FRESH && ks == 0 && op == 0) {
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[op], wb[ks % SL][nb], zero, 0, 0, 0);
          } else {
            acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hf[op], wb[ks % SL][nb], acc[nb], 0, 0, 0);
          }
        }
        // refill what was just consumed; the scheduling barrier keeps the loads this far ahead of their use
        hf[op] = *(const half8 *)(hrow + op * TM * LD + (ks + 1) % KS * 16);
        if (op == 0) {
          const int tgt = ks + SL - 1;
#pragma unroll
          for (int nb = 0; nb < 2; nb++) wb[tgt % SL][nb] = tgt < KS ? wload(rc, cur + tgt * 2048, nb) : wload(rn, next + (tgt - KS) * 2048, nb);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  };

  int tile = blockIdx.x;
  if (tile >= tiles) return;
  request_rows(tile * TM);
#pragma unroll
  for (int q = 0; q < SL - 1; q++)
#pragma unroll
    for (int nb = 0; nb < 2; nb++) wb[q][nb] = wload(r1, at1(0) + q * 2048, nb);
  float bias2[2];
#pragma unroll
  for (int nb = 0; nb < 2; nb++) bias2[nb] = b2[wave * 64 + nb * 32 + li];
  if (wave < GS_WAVES / 2) __builtin_amdgcn_s_setprio(2);  // as in gemm_stream_kernel

  for (; tile < tiles; tile += gridDim.x) {
    const int m0 = tile * TM;
    gs_normalise<NE, RPW, TM, true>(xv, ln, sx, wave, lane);
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < 2; nb++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc2[nb][v] = 0.f;
    float res[2][16];
    float *xo = x + (long)(m0 + g * 4) * K + wave * 64 + li;
    auto chunk = [&](int c, auto last_tag) __attribute__((always_inline)) {
      constexpr bool LAST = decltype(last_tag)::value;
      float bias1[2];
#pragma unroll
      for (int nb = 0; nb < 2; nb++) bias1[nb] = b1[(c * GS_WAVES + wave) * 64 + nb * 32 + li];
      floatx16 acc1[2];
      k_loop(sx, r1, at1(c), r2, at2(c), acc1, std::true_type{});
      __syncthreads();  // every wave is done with the hidden planes of the chunk before
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const float u = as_f32(fmaxf(acc1[nb][v] + bias1[nb], 0.f));
          const _Float16 hi = (_Float16)u;
          _Float16 *p = su + ((v >> 2) * 8 + g * 4 + (v & 3)) * LD + wave * 64 + nb * 32 + li;
          p[0] = hi;
          p[TM * LD] = (_Float16)(u - (float)hi);
        }
      __syncthreads();
      if (LAST) {  // residual, and the next tile's rows (the last tile reads its own again)
#pragma unroll
        for (int nb = 0; nb < 2; nb++)
#pragma unroll
          for (int v = 0; v < 16; v++) {
            const int r = (v >> 2) * 8 + (v & 3);
            res[nb][v] = xo[(long)(min(m0 + g * 4 + r, M - 1) - m0 - g * 4) * K + nb * 32];
          }
        request_rows((tile + (int)gridDim.x < tiles ? tile + (int)gridDim.x : tile) * TM);
      }
      k_loop(su, r2, at2(c), r1, at1(LAST ? 0 : c + 1), acc2, std::false_type{});
    };
#pragma unroll 1
    for (int c = 0; c < NC - 1; c++) chunk(c, std::false_type{});
    chunk(NC - 1, std::true_type{});
    if (__builtin_expect(m0 + TM <= M, 1)) {  // straight-line stores, as in gemm_stream_kernel
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++) xo[((v >> 2) * 8 + (v & 3)) * K + nb * 32] = acc2[nb][v] + bias2[nb] + res[nb][v];
    } else {
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++)
          if (m0 + g * 4 + (v >> 2) * 8 + (v & 3) < M) xo[((v >> 2) * 8 + (v & 3)) * K + nb * 32] = acc2[nb][v] + bias2[nb] + res[nb][v];
      __builtin_amdgcn_s_waitcnt(0x0F70);
    }
  }
}

// workgroups per row tile with 32-column strips: four strips each, or two where N is an odd multiple of 64
static int gs_narrow_groups(int N) { return N % 128 == 0 ? N / 128 : N / 64; }

template <int RB, int K, bool C_F32, bool LN, bool TAIL, int NC = 1, int NB = 2>
static hipError_t gs_launch(const _Float16 *A, const _Float16 *A_lo, long lda, int M, const _Float16 *Wp, int N,
                            const GemmEpilogue &e, const GemmLayerNorm &ln, hipStream_t s) {
  auto kern = gemm_stream_kernel<RB, K, C_F32, LN, TAIL, NC, NB>;
  const size_t lds = (size_t)(TAIL ? 64 : 32) * RB * (K + 8) * 2;
  // raising the dynamic LDS limit is per kernel, once per process (several host threads may get here at once)
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  });
  if (attr_err != hipSuccess) return attr_err;
  const int row_tiles = (M + 32 * RB - 1) / (32 * RB), NS = N / (32 * NB);
  // The strips of a row tile are split over several workgroups where that shortens the launch: rounds of workgroups (one to a CU)
  // times the fill of the tile, which takes as long as a strip, and a wave's strips.  With as many workgroups as fit a few rounds
  // instead, every round began with a fill of its own: an encoder of six layers 516 against 439 us at 8,192 tokens, 888 against 754
  // at 16,384, 1,341 against 1,206 at 32,768; 8 heads and FFN 2,048 1,113 / 941, 2,039 / 1,767, 3,580 / 3,386 (20,480 tokens, just past
  // a round: the same both ways).
  int col_groups = 1;
  long best = 0;
  for (int cg = 1; cg * GS_WAVES <= NS; cg++) {
    if (NS % cg != 0) continue;
    const long cost = ((long)row_tiles * cg + 255) / 256 * (1 + (NS / cg + GS_WAVES - 1) / GS_WAVES);
    if (best == 0 || cost < best) best = cost, col_groups = cg;
  }
  if (NC > 1) col_groups = NS / GS_WAVES;  // several passes: exactly one strip per wave
  if (NB == 1) col_groups = gs_narrow_groups(N);
  hipLaunchKernelGGL(kern, dim3(row_tiles * col_groups), dim3(GS_WAVES * 64), lds, s, A, A_lo, lda, M, Wp, N, col_groups, e,
                     ln);
  return hipGetLastError();
}

// 32-column strips, two or four to a workgroup, while that is one round of workgroups: there the launch is one wave's latency (22 rows,
// N = 1536 / 512: 10.1 / 7.4 us against 15.7 / 13.4; a 30 + 6 layer model at an 8,192-token budget 138 against 158 ms).
// Beyond, filling the same rows for more workgroups costs the other lanes more than the launch gains (up to two rounds:
// 127.7 against 125.3 ms on the 8-head model at 16,384 tokens).
// N = 192 (three groups) at 3,200 / 8,000 rows, a whole encoder: 0.45 / 0.70 ms narrow, 0.40 / 0.62 wide.  A matrix of 64 columns is narrow at any
// number of rows: its one wide strip leaves one of eight waves working, two narrow ones two (19,200 / 64,000 rows, a whole
// encoder: 1.36 / 3.52 ms narrow, 1.45 / 3.64 wide).
static bool gs_narrow(int M, int N) { return N == 64 || (long)((M + 31) / 32) * gs_narrow_groups(N) <= 256; }

template <bool LN>
static hipError_t gs_dispatch(bool c_f32, const _Float16 *A, const _Float16 *A_lo, long lda, const _Float16 *Wp, int M,
                              int N, int K, const GemmEpilogue &e, const GemmLayerNorm &ln, bool tail, hipStream_t s) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (!gemm_stream_supported(N, K) || e.n_split % 32 != 0) return hipErrorInvalidValue;
  const bool small = M <= 8192;  // 32-row tiles: twice the workgroups
  if (gs_narrow(M, N)) {
#define NT_GS_CASE(K_, CF_)                                                                              \
  if (K == K_ && c_f32 == CF_)                                                                           \
    return tail ? gs_launch<1, K_, CF_, LN, true, 1, 1>(A, A_lo, lda, M, Wp, N, e, ln, s)                \
                : gs_launch<1, K_, CF_, LN, false, 1, 1>(A, A_lo, lda, M, Wp, N, e, ln, s);
    NT_GS_CASE(512, true) NT_GS_CASE(512, false) NT_GS_CASE(256, true) NT_GS_CASE(256, false)
#undef NT_GS_CASE
  }
#define NT_GS_CASE(RB_, K_, CF_)                                                                                       \
  if (small == (RB_ == 1) && K == K_ && c_f32 == CF_)                                                                  \
    return tail ? gs_launch<RB_, K_, CF_, LN, true>(A, A_lo, lda, M, Wp, N, e, ln, s)                                  \
                : gs_launch<RB_, K_, CF_, LN, false>(A, A_lo, lda, M, Wp, N, e, ln, s);
  NT_GS_CASE(1, 512, true) NT_GS_CASE(1, 512, false) NT_GS_CASE(2, 512, true) NT_GS_CASE(2, 512, false)
  NT_GS_CASE(1, 256, true) NT_GS_CASE(1, 256, false) NT_GS_CASE(2, 256, true) NT_GS_CASE(2, 256, false)
#undef NT_GS_CASE
  return hipErrorInvalidValue;
}

// The same product for few rows: a workgroup takes 32 rows and one strip of 32 columns, its waves an eighth of the k-range each,
// whose fragments of both operands are requested at once, straight into registers (a row's 16-byte pieces share their lines over
// four k-steps); the eight partial blocks meet in the LDS.  In passes over a tile the launch is a chain of fill, barrier and
// k-loop per 512 columns.  fp32 output, one destination.
// Up to kSplitKRows rows (N = 512, K = 2,048, a 30 + 6 layer model): 45 / 240 rows 16.9 -> 16.1 / 22.5 -> 21.4 ms a batch, 2,048
// sentences 112.8 -> 108.5 ms.  Up to 512 rows the rows are read by 16 workgroups per tile where two would do: 109.8 ms, and
// 115.4 -> 117.5 on the 8-head model with its 300 to 700 rows.
template <int K, bool TAIL>
__global__ __launch_bounds__(512) void gemm_split_k_kernel(const _Float16 *__restrict__ A_hi, const _Float16 *__restrict__ A_lo,
                                                           long lda, int M, const _Float16 *__restrict__ Wp, int N,
                                                           GemmEpilogue e) {
  constexpr int KS = K / 16, KSW = KS / GS_WAVES;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  __shared__ f32x4 red[GS_WAVES][4][64];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NS = N / 32, m0 = blockIdx.x / NS * 32, strip = blockIdx.x % NS;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, N * K * 2, 0x00020000);
  const int w0 = (strip >> 1) * (KS * 2048) + (strip & 1) * 1024 + wave * (KSW * 2048);
  const long arow = (long)min(m0 + li, M - 1) * lda + wave * (KSW * 16) + g * 8;
  half8 w[KSW], a[TAIL ? 2 : 1][KSW];
#pragma unroll
  for (int q = 0; q < KSW; q++) {
    w[q] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16, w0 + q * 2048, 0));
    a[0][q] = *(const half8 *)(A_hi + arow + q * 16);
    if (TAIL) a[TAIL][q] = *(const half8 *)(A_lo + arow + q * 16);
  }
  // this thread's two results: rows row0, row0 + 1 of the block, column li
  const int part = wave >> 1, row0 = m0 + part * 8 + g * 4 + (wave & 1) * 2, n = strip * 32 + li;
  const float bias = e.bias ? e.bias[n] : 0.f, scl = n < e.scale_cols ? e.scale : 1.f;
  float res[2];
#pragma unroll
  for (int v = 0; v < 2; v++) res[v] = e.resid && row0 + v < M ? e.resid[(long)(row0 + v) * e.ldr + n] : 0.f;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.f;
#pragma unroll
  for (int q = 0; q < KSW; q++)
#pragma unroll
    for (int op = 0; op < (TAIL ? 2 : 1); op++) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[op][q], w[q], acc, 0, 0, 0);
#pragma unroll
  for (int q = 0; q < 4; q++) red[wave][q][lane] = f32x4{acc[q * 4], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
  __syncthreads();
  f32x2 t = ((const f32x2 *)&red[0][part][lane])[wave & 1];
#pragma unroll
  for (int p = 1; p < GS_WAVES; p++) t += ((const f32x2 *)&red[p][part][lane])[wave & 1];
#pragma unroll
  for (int v = 0; v < 2; v++) {
    float val = (t[v] + bias) * scl;
    if (e.relu) val = fmaxf(val, 0.f);
    if (row0 + v < M) ((float *)e.dst0)[(long)(row0 + v) * e.ld0 + n] = val + res[v];
  }
}

// K = 1024 / 2048 in passes over a 512-wide tile; N a multiple of 512 (one strip per wave and column group)
static constexpr int kSplitKRows = 256;
bool gemm_stream_k_supported(int N, int K) { return (K == 1024 || K == 2048) && N >= 512 && N % 512 == 0; }

hipError_t launch_gemm_stream_k(bool c_f32, const _Float16 *A, const _Float16 *A_lo, long lda, const _Float16 *Wp, int M,
                                int N, int K, const GemmEpilogue &e, hipStream_t s, bool tail, int shape_rows) {
  if (M <= 0 || N <= 0) return hipSuccess;
  if (!gemm_stream_k_supported(N, K) || e.n_split % 32 != 0) return hipErrorInvalidValue;
  tail = tail && A_lo != nullptr;
  if (c_f32 && e.n_split == N && !e.first_f16 && (shape_rows > 0 ? shape_rows : M) <= kSplitKRows) {
    const dim3 grid((unsigned)((M + 31) / 32 * (N / 32)));
#define NT_SPLIT_K(K_, TL_) \
  if (K == K_ && tail == TL_) hipLaunchKernelGGL((gemm_split_k_kernel<K_, TL_>), grid, dim3(512), 0, s, A, A_lo, lda, M, Wp, N, e);
    NT_SPLIT_K(1024, true) NT_SPLIT_K(1024, false) NT_SPLIT_K(2048, true) NT_SPLIT_K(2048, false)
#undef NT_SPLIT_K
    return hipGetLastError();
  }
  const GemmLayerNorm ln{};
#define NT_GSK_CASE(NC_, CF_, TL_)                        \
  if (K == 512 * NC_ && c_f32 == CF_ && tail == TL_)      \
    return gs_narrow(M, N) ? gs_launch<1, 512, CF_, false, TL_, NC_, 1>(A, A_lo, lda, M, Wp, N, e, ln, s) : M <= 8192 ? gs_launch<1, 512, CF_, false, TL_, NC_>(A, A_lo, lda, M, Wp, N, e, ln, s) \
                     : gs_launch<2, 512, CF_, false, TL_, NC_>(A, A_lo, lda, M, Wp, N, e, ln, s);
  NT_GSK_CASE(2, true, true) NT_GSK_CASE(2, true, false) NT_GSK_CASE(4, true, true) NT_GSK_CASE(4, true, false)
#undef NT_GSK_CASE
  return hipErrorInvalidValue;
}

bool gemm_ffn_supported(int M, int d, int F) { return d == 512 && (F == 1024 || F == 2048) && M >= kFfnMinRows; }

template <int NC>
static hipError_t gf_launch(float *x, int M, const GemmLayerNorm &ln, const _Float16 *W1p, const float *b1, const _Float16 *W2p, const float *b2, hipStream_t s) {
  auto kern = gemm_ffn_kernel<NC>;
  constexpr int lds = 4 * 32 * (512 + 8) * 2;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds); });
  if (attr_err != hipSuccess) return attr_err;
  const int tiles = (M + 31) / 32;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles < 256 ? tiles : 256)), dim3(GS_WAVES * 64), lds, s, x, M, ln, W1p, b1, W2p, b2);
  return hipGetLastError();
}

hipError_t launch_gemm_ffn(float *x, int M, int F, const GemmLayerNorm &ln, const _Float16 *W1p, const float *b1, const _Float16 *W2p, const float *b2,
                           hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (F == 1024) return gf_launch<2>(x, M, ln, W1p, b1, W2p, b2, s);
  if (F == 2048) return gf_launch<4>(x, M, ln, W1p, b1, W2p, b2, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_stream(bool c_f32, const _Float16 *A, const _Float16 *A_lo, long lda, const _Float16 *Wp, int M,
                              int N, int K, const GemmEpilogue &e, hipStream_t s, bool tail) {
  return gs_dispatch<false>(c_f32, A, A_lo, lda, Wp, M, N, K, e, GemmLayerNorm{}, tail && A_lo != nullptr, s);
}

bool gemm_chain_supported(int M, int N, int K) { return K == 512 && N % 512 == 0 && M > kChainRows; }

template <int RB>
static hipError_t gc_launch(const _Float16 *A, const _Float16 *A_lo, long lda, const GemmChain &ch, const GemmLayerNorm &ln, const _Float16 *Wp, int M,
                            int N, const GemmEpilogue &e, hipStream_t s) {
  auto kern = gemm_chain_kernel<RB>;
  constexpr int lds = 2 * 32 * RB * (512 + 8) * 2;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds); });
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL(kern, dim3((unsigned)((M + 32 * RB - 1) / (32 * RB))), dim3(GS_WAVES * 64), lds, s, A, A_lo, lda, M, Wp, N, e, ln, ch);
  return hipGetLastError();
}

hipError_t launch_gemm_chain(const _Float16 *A, const _Float16 *A_lo, long lda, const GemmChain &ch, const GemmLayerNorm &ln, const _Float16 *Wp, int M,
                             int N, const GemmEpilogue &e, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (N <= 0 || N % 512 != 0 || e.n_split % 32 != 0) return hipErrorInvalidValue;
  return M <= 8192 ? gc_launch<1>(A, A_lo, lda, ch, ln, Wp, M, N, e, s) : gc_launch<2>(A, A_lo, lda, ch, ln, Wp, M, N, e, s);
}

hipError_t launch_gemm_stream_ln(bool c_f32, const float *X, long ldx, const GemmLayerNorm &ln, const _Float16 *Wp, int M,
                                 int N, int K, const GemmEpilogue &e, hipStream_t s, bool tail) {
  return gs_dispatch<true>(c_f32, (const _Float16 *)X, nullptr, ldx, Wp, M, N, K, e, ln, tail, s);
}

}  // namespace nt
