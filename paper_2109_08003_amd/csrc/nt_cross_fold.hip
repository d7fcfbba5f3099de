// Folded cross caches of one-layer one-head decoders as 16-bit integers (gfx950): the matrix at load, and per batch one launch from the
// encoder's residual stream to the cache.
//
// A decoder step multiplies its row with Wq before the cross-attention and the context with Wo after it; both can be done once per source
// token instead: q . k = y . (k Wq^T) + b_q . k, and (sum p v) Wo = sum p (v Wo).  With x^ the encoder's row, normalised without gain g and
// offset h (k = (g x^ + h) Wk + b_k, v likewise), what the step attends over is
//     keys   x^ [g (Wk Wq^T)] and a constant x^ . [g (Wk b_q)],     values   x^ [g (Wv Wo)];
// h and the biases only add the same to every key's score, which a softmax does not see, and a constant to the context.  Every column of
// the two products is divided by its size, the key columns' sizes go into the gain and offset of the normalisation the query comes from,
// the value columns' are multiplied back with the context: a vector's integers have one scale, which its largest element sets.
// So a vector is rounded once, as it is without folding, and its columns are of one magnitude.  The products are formed in double and
// kept as head and tail planes, 22 bits, as the factors of 11 bits they are made of are exact.
//
// 54,069 tokens, d = 512: 171 us without the tail plane and 262 with it, where projection and quantisation as two launches, the keys and
// values in fp32 between them, took 195 and 229; what a step gains is in nt_dec1.hip.  0.66 PFLOP/s are issued (both planes of the matrix,
// 1.5 times the products with the tail) and the matrix pipes are busy for 38 % of the time: the fill of a tile, the products and the two
// exchanges per vector follow one another.
//
// The kernel has the shape of nt_gemm_stream.hip's: a tile of 32 or 64 normalised rows in the LDS, the matrix through a ring of
// registers.  The matrix is the row operand, so that a lane owns a row of the tile and half of a wave's 64 columns: the largest element of
// a vector is a maximum over the lane's registers, one exchange with the other half and one through the LDS with the other waves, and
// the codes leave through the LDS as whole vectors.
#include <algorithm>
#include <mutex>

#include "nt_kernels.h"

namespace nt {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int CF_WAVES = 8;

// W: [strip = n / 64][k / 16][plane][(n % 64) / 32][lane][8 halfs], lane = n % 32 + 32 * ((k % 16) / 8); then five vectors of d
static size_t cf_matrix_bytes(int d) { return (size_t)d * 2 * d * 2 * 2; }
size_t cross_fold_bytes(int d) { return cf_matrix_bytes(d) + (size_t)5 * d * 4; }
CrossFold cross_fold_at(void *dst, int d) {
  const float *v = (const float *)((char *)dst + cf_matrix_bytes(d));
  return CrossFold{(const _Float16 *)dst, v, v + d, v + 2 * d, v + 3 * d, v + 4 * d};
}

// ---- at load --------------------------------------------------------------------------------------------------------
// C [d][2 d] = gain times the two products, 64 x 64 per workgroup, 4 x 4 per lane
constexpr int CP_T = 64, CP_K = 32;
__global__ __launch_bounds__(256) void cross_fold_product_kernel(CrossFoldWeights w, int d, double *C) {
  __shared__ double sa[CP_K][CP_T + 2], sb[CP_K][CP_T + 2];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int x0 = blockIdx.y * CP_T, n0 = blockIdx.x * CP_T, half = n0 >= d, j0 = half ? n0 - d : n0;
  double acc[4][4] = {};
  for (int m0 = 0; m0 < d; m0 += CP_K) {
    for (int i = tid; i < CP_T * CP_K; i += 256) {
      const int c = i % CP_T, m = i / CP_T;
      sa[m][c] = (double)(float)w.Wkv[(long)(half * d + m0 + m) * d + x0 + c];
      if (!half) sb[m][c] = (double)(float)w.Wq[(long)(m0 + m) * d + j0 + c];
    }
    if (half)
      for (int i = tid; i < CP_T * CP_K; i += 256) sb[i % CP_K][i / CP_K] = (double)(float)w.Wo[(long)(j0 + i / CP_K) * d + m0 + i % CP_K];
    __syncthreads();
    for (int m = 0; m < CP_K; m++) {
      double a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; i++) a[i] = sa[m][ty * 4 + i], b[i] = sb[m][tx + i * 16];
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] += a[i] * b[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int x = x0 + ty * 4 + i;
    const double g = (double)w.enc_gamma[x] * (half ? 1.0 : (double)w.q_scale);
#pragma unroll
    for (int j = 0; j < 4; j++) C[(long)x * 2 * d + n0 + tx + j * 16] = g * acc[i][j];
  }
}
__device__ __forceinline__ double cf_sum(double v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}
// one wave: block m < d: t[m] = b_v[m] + h . Wv[:, m]; block d + x: u[x] = q_scale g[x] Wk[x, :] . b_q
__global__ __launch_bounds__(64) void cross_fold_vector_kernel(CrossFoldWeights w, int d, double *t, float *u) {
  const int lane = threadIdx.x, i = blockIdx.x % d;
  double s = 0.0;
  if ((int)blockIdx.x < d) {
    for (int x = lane; x < d; x += 64) s += (double)w.enc_beta[x] * (double)(float)w.Wkv[(long)(d + i) * d + x];
    s = cf_sum(s);
    if (lane == 0) t[i] = s + (double)w.bkv[d + i];
  } else {
    for (int m = lane; m < d; m += 64) s += (double)w.bq[m] * (double)(float)w.Wkv[(long)m * d + i];
    s = cf_sum(s);
    if (lane == 0) u[i] = (float)(s * (double)w.enc_gamma[i] * (double)w.q_scale);
  }
}
// one wave per column: its size (root mean square: elements of order one, whose tails are no subnormals), planes, scale
__global__ __launch_bounds__(64) void cross_fold_pack_kernel(CrossFoldWeights w, int d, const double *C, const double *t, _Float16 *W,
                                                             float *gamma2, float *beta2, float *value_scale, float *value_const) {
  const int lane = threadIdx.x, n = blockIdx.x, half = n >= d, j = half ? n - d : n, KS = d / 16;
  double s = 0.0;
  for (int x = lane; x < d; x += 64) s += C[(long)x * 2 * d + n] * C[(long)x * 2 * d + n];
  s = cf_sum(s);
  float size = (float)sqrt(s / (double)d);
  if (!(size > 0.f && size < INFINITY)) size = 1.f;
  for (int x = lane; x < d; x += 64) {
    const float c = (float)(C[(long)x * 2 * d + n] / (double)size);
    const _Float16 hi = (_Float16)c, lo = (_Float16)(c - (float)hi);
    _Float16 *p = W + ((((long)(n >> 6) * KS + (x >> 4)) * 4 + ((n >> 5) & 1)) * 64 + (n & 31) + 32 * ((x >> 3) & 1)) * 8 + (x & 7);
    p[0] = hi;
    p[2 * 64 * 8] = lo;
  }
  if (!half) {
    if (lane == 0) gamma2[j] = w.gamma2[j] * size, beta2[j] = w.beta2[j] * size;
    return;
  }
  double o = 0.0;
  for (int m = lane; m < d; m += 64) o += t[m] * (double)(float)w.Wo[(long)j * d + m];
  o = cf_sum(o);
  if (lane == 0) value_scale[j] = size, value_const[j] = (float)(o + (double)w.bo[j]);
}

hipError_t cross_fold_build(const CrossFoldWeights &w, int d, void *dst, hipStream_t s) {
  if (d != 256 && d != 512) return hipErrorInvalidValue;
  double *tmp = nullptr;
  hipError_t e = hipMalloc((void **)&tmp, ((size_t)d * 2 * d + d) * sizeof(double));
  if (e != hipSuccess) return e;
  double *C = tmp, *t = tmp + (size_t)d * 2 * d;
  const CrossFold f = cross_fold_at(dst, d);
  hipLaunchKernelGGL(cross_fold_product_kernel, dim3(2 * d / CP_T, d / CP_T), dim3(256), 0, s, w, d, C);
  hipLaunchKernelGGL(cross_fold_vector_kernel, dim3(2 * d), dim3(64), 0, s, w, d, t, (float *)f.u);
  hipLaunchKernelGGL(cross_fold_pack_kernel, dim3(2 * d), dim3(64), 0, s, w, d, C, t, (_Float16 *)f.W, (float *)f.gamma2, (float *)f.beta2,
                     (float *)f.value_scale, (float *)f.value_const);
  e = hipGetLastError();
  const hipError_t done = hipStreamSynchronize(s);
  (void)hipFree(tmp);
  return e != hipSuccess ? e : done;
}

// ---- per batch ------------------------------------------------------------------------------------------------------
// A workgroup: a tile of 32 RB rows, and the strips of 64 columns p * 8 + wave, p = part's share of the matrix (split == 2: the keys or
// the values; a vector of 256 columns is four waves' strips, so that one turn makes both).
template <int K, int RB, bool TAIL>
__global__ __launch_bounds__(CF_WAVES * 64) void cross_fold_kernel(const float *__restrict__ x, int M, LnEps eps, const _Float16 *__restrict__ Wp,
                                                                   const float *__restrict__ u, int split, short *__restrict__ cache,
                                                                   float *__restrict__ sc) {
  constexpr int TM = 32 * RB, LD = K + 8, KS = K / 16, NE = K / 64, RPW = TM / CF_WAVES, NOPS = (TAIL ? 2 : 1) * RB;
  constexpr int SL = 4;                    // ring of k-steps, four fragments each (lookahead SL - 1)
  constexpr int CLD = 512 + 8;             // codes of one turn: [row][8 strips of 64]
  constexpr int TURNS = 2 * K / 512, WPV = K / 64;  // turns; waves per vector
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  _Float16 *sh = (_Float16 *)smem;
  short *sCode = (short *)(smem + (TAIL ? 2 : 1) * TM * LD * 2);
  float *sMax = (float *)(sCode + TM * CLD);  // [8][TM]
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = (int)blockIdx.x / split * TM, part = (int)blockIdx.x % split;
  const int turn0 = part * (TURNS / split), turn1 = turn0 + TURNS / split;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, 2 * K * K * 4, 0x00020000);
  auto wload = [&](int soff, int f) -> half8 {
    return __builtin_bit_cast(half8, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16 + f * 1024, soff, 0));
  };
  auto strip_at = [&](int turn) { return (turn * CF_WAVES + wave) * (KS * 4096); };

  // ---- the tile: normalised rows (fp32 statistics: mean first, then the terms of the centred values); rows past M repeat row M - 1 ----
  half8 wb[SL][4];  // plane * 2 + column block
  {
    float xv[RPW][NE], uv[NE];
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      const int m = min(m0 + wave + CF_WAVES * i, M - 1);
#pragma unroll
      for (int j = 0; j < NE; j += 4) {
        const f32x4 t = *(const f32x4 *)(x + (long)m * K + lane * NE + j);
        xv[i][j] = t[0], xv[i][j + 1] = t[1], xv[i][j + 2] = t[2], xv[i][j + 3] = t[3];
      }
    }
#pragma unroll
    for (int j = 0; j < NE; j += 4) *(float4 *)&uv[j] = *(const float4 *)(u + lane * NE + j);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < SL - 1; q++)
#pragma unroll
      for (int f = 0; f < 4; f++) wb[q][f] = wload(strip_at(turn0) + q * 4096, f);
    float mean[RPW], rs[RPW], c[RPW];
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NE; j++) s += xv[i][j];
      mean[i] = s;
    }
#pragma unroll
    for (int i = 0; i < RPW; i++) mean[i] = wave_sum(mean[i]) / (float)K;
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NE; j++) s += ln_term(xv[i][j] - mean[i], eps.l1);
      rs[i] = s;
    }
#pragma unroll
    for (int i = 0; i < RPW; i++) rs[i] = ln_rscale(wave_sum(rs[i]) / (float)K, eps);
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
      halfNE hi, lo;
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < NE; j++) {
        const float y = as_f32((xv[i][j] - mean[i]) * rs[i]);
        hi[j] = (_Float16)y;
        lo[j] = (_Float16)(y - (float)hi[j]);
        s += y * uv[j];
      }
      const int R = wave + CF_WAVES * i;
      *(halfNE *)(sh + R * LD + lane * NE) = hi;
      if (TAIL) *(halfNE *)(sh + (R + TM) * LD + lane * NE) = lo;
      c[i] = s;
    }
#pragma unroll
    for (int i = 0; i < RPW; i++) c[i] = wave_sum(c[i]);
    if (part == 0 && lane == 0) {
#pragma unroll
      for (int i = 0; i < RPW; i++)
        if (m0 + wave + CF_WAVES * i < M) sc[(long)(m0 + wave + CF_WAVES * i) * 4 + 2] = c[i];
    }
  }
  __syncthreads();

  const _Float16 *hrow = sh + li * LD + g * 8;
  constexpr int ROWS = (TAIL ? 2 : 1) * TM, HALF = ROWS > 32 ? ROWS / 2 : ROWS;
  int off2 = HALF * LD;  // second base register: the offsets of the upper half do not fit the offset field
  asm volatile("" : "+v"(off2));
  const _Float16 *hrow2 = hrow + off2;
  auto frag = [&](int op, int ks) -> half8 { return *(const half8 *)((op * 32 < HALF ? hrow : hrow2) + (op * 32 % HALF) * LD + ks * 16); };
  half8 hf[NOPS];
#pragma unroll
  for (int op = 0; op < NOPS; op++) hf[op] = frag(op, 0);
  floatx16 acc[2][RB];
#pragma unroll 1
  for (int turn = turn0; turn < turn1; turn++) {
    const int cur = strip_at(turn), next = strip_at(turn + 1 < turn1 ? turn + 1 : turn);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const int tgt = ks + SL - 1, pf = tgt < KS ? cur + tgt * 4096 : next + (tgt - KS) * 4096;
#pragma unroll
      for (int op = 0; op < NOPS; op++) {  // head rows: both planes of the matrix; tail rows: its head
#pragma unroll
        for (int f = 0; f < (op < RB ? 4 : 2); f++) {
          if (ks == 0 && op < RB && f < 2) {
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            acc[f & 1][op % RB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wb[ks % SL][f], hf[op], zero, 0, 0, 0);
          } else {
            acc[f & 1][op % RB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wb[ks % SL][f], hf[op], acc[f & 1][op % RB], 0, 0, 0);
          }
        }
        hf[op] = frag(op, (ks + 1) % KS);
        if (op == 0) {
#pragma unroll
          for (int f = 0; f < 4; f++) wb[tgt % SL][f] = wload(pf, f);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // ---- acc[nb][rb][v] is column nb * 32 + (v / 4) * 8 + g * 4 + v % 4 of the strip, row rb * 32 + li of the tile ----
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      float top = 0.f;
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++) top = fmaxf(top, fabsf(acc[nb][rb][v]));
      top = wave_pair32(top, top, WaveMax{});
      if (g == 0) sMax[wave * TM + rb * 32 + li] = top;
    }
    __syncthreads();
    const int first = wave / WPV * WPV;  // first wave of this wave's vector
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      float top = 0.f;
#pragma unroll
      for (int w = 0; w < WPV; w++) top = fmaxf(top, sMax[(first + w) * TM + rb * 32 + li]);
      const float scale = top > 0.f ? top / 32767.f : 1.f, inv = 1.f / scale;
      const int m = m0 + rb * 32 + li;
      if (wave == first && g == 0 && m < M) sc[(long)m * 4 + (turn * CF_WAVES + wave) / WPV] = scale;
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
          short4v q;
#pragma unroll
          for (int t = 0; t < 4; t++) q[t] = (short)(int)fminf(fmaxf(rintf(acc[nb][rb][v + t] * inv), -32767.f), 32767.f);
          *(short4v *)(sCode + (rb * 32 + li) * CLD + wave * 64 + nb * 32 + v * 2 + g * 4) = q;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      const int R = wave + CF_WAVES * i;
      if (m0 + R < M) *(short8v *)(cache + (long)(m0 + R) * 2 * K + turn * 512 + lane * 8) = *(const short8v *)(sCode + R * CLD + lane * 8);
    }
  }
}

template <int K, int RB, bool TAIL>
static hipError_t cf_launch(const float *x, int M, LnEps eps, const CrossFold &f, short *cache, float *sc, hipStream_t s) {
  auto kern = cross_fold_kernel<K, RB, TAIL>;
  constexpr int lds = (TAIL ? 2 : 1) * 32 * RB * (K + 8) * 2 + 32 * RB * (512 + 8) * 2 + CF_WAVES * 32 * RB * 4;
  // raising the dynamic LDS limit is per kernel, once per process (several host threads may get here at once)
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds); });
  if (attr_err != hipSuccess) return attr_err;
  const int tiles = (M + 32 * RB - 1) / (32 * RB), split = K == 512 && tiles <= 128 ? 2 : 1;
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * split)), dim3(CF_WAVES * 64), lds, s, x, M, eps, f.W, f.u, split, cache, sc);
  return hipGetLastError();
}

hipError_t launch_cross_fold(const float *x, int M, int d, LnEps eps, const CrossFold &f, bool tail, short *cache, float *sc, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (d != 256 && d != 512) return hipErrorInvalidValue;
  const bool wide = M > 8192 && !tail;  // 64-row tiles (with the tail plane the tile and its codes do not fit)
#define NT_CF(K_, RB_, TL_) \
  if (d == K_ && wide == (RB_ == 2) && tail == TL_) return cf_launch<K_, RB_, TL_>(x, M, eps, f, cache, sc, s);
  NT_CF(512, 1, false) NT_CF(512, 2, false) NT_CF(512, 1, true) NT_CF(256, 1, false) NT_CF(256, 2, false) NT_CF(256, 1, true)
#undef NT_CF
  return hipErrorInvalidValue;
}

}  // namespace nt
