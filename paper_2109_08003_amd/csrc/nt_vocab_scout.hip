// Output projection with row arg-max for many rows (gfx950): an 8-bit scout pass over the whole vocabulary, exact logits for the
// entries it cannot rule out.
//
// Greedy search wants one id per row, and all but a few of the 32,000 logits lose by far.  The scout multiplies 8-bit codes of the
// states with 8-bit codes of the matrix on the int8 matrix cores - twice the rate and half the bytes of fp16 - and what it leaves
// out is bounded: with x = a + e (a the rounded state, e the rest) and w = b + f likewise,
//     x . w - a . b = e . w + a . f,     |x . w - a . b| <= ||e|| ||w|| + ||a|| ||f||        (Cauchy-Schwarz)
// where ||e||, ||a|| come per row from the kernel that writes the state and ||w||, ||f|| per strip from load time.  An entry whose
// scout logit plus its bound stays below the best scout logit minus that one's bound is not the arg-max.  What is left (16 of
// 32,000 entries per row on flat random logits, d = 512; 5 of 4,000 at d = 256) gets its logit from the state's head + tail planes
// and the fp16 matrix in fp32, and the largest of these wins, lowest id on ties: the same tokens as a pass over everything with
// both planes, but for ties within fp32 rounding.  A row with more than kPickCap candidates has every logit computed.
//
// The matrix is centred before it is rounded: its mean row adds the same to every logit of a row, so it changes no arg-max, and
// a common offset of the entries would only widen the range of the codes.  Entries are sorted by their largest element, so that the
// 64 entries of a strip, which share one scale, are alike.
//
// The columns are levelled and mixed before either side is rounded, because a row has one scale: a column that is larger than the
// others (an offset or a gain of the final normalisation, a column of the matrix) would leave the others few of its steps.
//   levelled: x . w = sum (x_k 2^l_k) (w_k 2^-l_k), where l_k takes half of the column's size, x_k against the spread of w_k, to either
//   side (all of it on one side only moves the trouble to the other);
//   mixed: eight columns at a time (four at d = 256), the elements of a lane, by an orthogonal matrix of signs on both sides, which
//   spreads what is left of such a column over eight.
// Candidates of a row, d = 512, 32,000 flat random entries, median / largest of 400 states (with the groups of which all are taken,
// see below; neither: without them), both, levelled only, neither: an offset of 25 on one column 45 / 336, 483 / 1,700, 802 / 2,600; two gains of 16 15 / 253,
// 194 / 1,678, 277 / 3,104; a column of the matrix 16 times the others 15 / 302, 85 / 1,719, 842 / 2,626; none of these 12 / 85 each way.
// Eight steps of 400 rows with any of these 0.24 to 0.29 ms, 0.24 with none; before, when one row or another of every launch had each
// logit computed, 4.8 to 5.1 ms.  The 4,096-, 16,384- and 65,536-token budgets take the same time as without, to 0.3 %.
//
// The scout has the shape of the 8-bit output layer's kernel (nt_vocab_q8.hip): 128 rows of codes in the LDS, fragments of the
// matrix through a ring of registers, a wave owns a strip of 64 entries for all rows of the tile, a lane owns a row of each 32-row
// block.  A lane's 32 products of a strip are one group (|sum| <= 127^2 512 < 2^23): the largest and the runner-up leave with their
// places and a bound on the third, in two integers, so that only a group that may hold three candidates (one row in a thousand)
// has all its entries computed; four instructions per product.
//
// Measured, d = 512, 32,000 entries: scout 30.5 us (2.0 POP/s) and pick 10.5 us at 1,460 rows on average (40,000 sentences, 65,536-token budget),
// 11.5 and 7.7 at 400, 8.0 and 5.6 at 260, where a pass over the head plane that certified its winners, the certification and the recompute
// of the rest took 61, 5.5 and 11 us at 1,900 rows, and a pass with both planes 14 to 28 us for 65 to 512.  The scout is bound by the matrix
// cores (operand loads, folds and the ends of strips take a good half, as in nt_vocab_q8.hip; a wave's
// priority, waves started apart and a ring of eight slots changed nothing), the pick by its chain of dependent loads.
// One scale per strip instead of per entry costs 16 candidates a row instead of 13 and saves two instructions per product.
#include "nt_kernels.h"
#include "nt_pick.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <numeric>
#include <type_traits>
#include <vector>

namespace nt {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int SC_ROWS = 128, SC_WAVES = 8;
constexpr int SC_LEVEL = 32;         // largest power of two of a column

static size_t scout_code_bytes(int N, int K) { return (size_t)((N + 63) / 64) * 64 * K; }
// codes, then per strip {scale, largest ||w||, largest ||f||, unused}, then the id of every place (-1: none), then the matrix's rows in
// the order of the places (the exact logits then need no look-up before their row), then the states' levels l_k
static size_t scout_level_at(int N, int K) { return scout_code_bytes(N, K) + (size_t)((N + 63) / 64) * (16 + 64 * 4 + 64 * (size_t)K * 2); }
size_t vocab_scout_bytes(int N, int K) { return scout_level_at(N, K) + (size_t)K; }
const int8_t *vocab_scout_levels(const void *matrix, int N, int K) { return (const int8_t *)matrix + scout_level_at(N, K); }

// ---- at load, on the device (50 MB for 32,000 x 512; the same loops on the host took 350 ms of a load of 200) ----------------------
constexpr int SP_ROWS = 256;  // rows per partial sum of the mean

// Elements that are no finite numbers stay out of the mean and of the codes; the strip of such an entry has norms without end, which
// makes its entries candidates of every row, and the exact logits decide.
__device__ __forceinline__ bool scout_finite(_Float16 w) { return fabsf((float)w) <= 65504.f; }

__global__ __launch_bounds__(512) void scout_sum_kernel(const _Float16 *W, int N, int K, double *sums) {
  const int k = threadIdx.x, v0 = blockIdx.x * SP_ROWS, v1 = v0 + SP_ROWS < N ? v0 + SP_ROWS : N;
  double s = 0.0, s2 = 0.0;
  for (int v = v0; v < v1; v++) {
    const _Float16 w = W[(long)v * K + k];
    const double x = scout_finite(w) ? (double)(float)w : 0.0;
    s += x;
    s2 += x * x;
  }
  sums[((long)blockIdx.x * 2) * K + k] = s;
  sums[((long)blockIdx.x * 2 + 1) * K + k] = s2;
}
// Mean of every column, and its level: half the ratio of what the final normalisation makes of the state there (gain and offset; 3.3: the
// largest of 512 normal deviates) to the column's spread, against the mean of all columns' halves.  A column that is always 0 on
// one side gives all of its size to the other.
__global__ __launch_bounds__(512) void scout_mean_kernel(const double *sums, int n, int N, int K, const float *gamma, const float *beta, float *mean,
                                                         int8_t *level) {
  __shared__ float ratio[512];
  const int k = threadIdx.x;
  double s = 0.0, s2 = 0.0;
  for (int i = 0; i < n; i++) s += sums[((long)i * 2) * K + k], s2 += sums[((long)i * 2 + 1) * K + k];
  s /= (double)N;
  mean[k] = (float)s;
  const double spread2 = s2 / (double)N - s * s;
  const float state = fabsf(beta[k]) + 3.3f * fabsf(gamma[k]), matrix = spread2 > 0.0 ? (float)sqrt(spread2) : 0.f;
  const bool both = state > 0.f && state < INFINITY && matrix > 0.f;
  const float half = both ? 0.5f * log2f(state / matrix) : 0.f;
  ratio[k] = both ? half : INFINITY;
  __syncthreads();
  float all = 0.f;
  int of = 0;
  for (int i = 0; i < K; i++)
    if (ratio[i] < INFINITY) all += ratio[i], of++;
  int l = 0;
  if (both) l = (int)rintf(half - all / (float)of);
  else if (state == 0.f && matrix > 0.f) l = -SC_LEVEL;
  else if (matrix == 0.f && state > 0.f && state < INFINITY) l = SC_LEVEL;
  level[k] = (int8_t)-(l < -SC_LEVEL ? -SC_LEVEL : l > SC_LEVEL ? SC_LEVEL : l);
}
// This lane's elements of row v as they are coded: centred, levelled, mixed (which on both sides multiplies a product by NE).
// false: one of them is no finite number; it counts as 0.
template <int NE>
__device__ __forceinline__ bool scout_entry(const _Float16 *W, long v, const float *mean, const int8_t *level, int lane, _Float16 (&w)[NE], double (&x)[NE]) {
  bool finite = true;
#pragma unroll
  for (int e = 0; e < NE; e++) {
    const int k = lane * NE + e;
    w[e] = W[v * (NE * 64) + k];
    const bool f = scout_finite(w[e]);
    x[e] = f ? ldexp((double)(float)w[e] - (double)mean[k], -level[k]) * (1.0 / NE) : 0.0;
    finite &= f;
  }
  scout_mix<NE>(x);
  return finite;
}
// largest of them in every row, a wave each; infinite (last in the order) where an element is not finite
template <int NE>
__global__ __launch_bounds__(256) void scout_top_kernel(const _Float16 *W, int N, const float *mean, const int8_t *level, float *top) {
  const int lane = threadIdx.x & 63, v = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (v >= N) return;
  _Float16 w[NE];
  double x[NE];
  float m = scout_entry<NE>(W, v, mean, level, lane, w, x) ? 0.f : INFINITY;
#pragma unroll
  for (int e = 0; e < NE; e++) m = fmaxf(m, fabsf((float)x[e]));
  m = wave_max(m);
  if (lane == 0) top[v] = m;
}
// one strip per workgroup, sixteen rows per wave
template <int NE>
__global__ __launch_bounds__(256) void scout_pack_kernel(const _Float16 *W, int N, const float *mean, const int8_t *level, const float *top,
                                                         const int32_t *order, int8_t *codes, float4 *consts, int32_t *ids, _Float16 *sorted) {
  constexpr int K = NE * 64, KS = K / 32;
  __shared__ float norms[2][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, s = blockIdx.x;
  const int n = N - s * 64 < 64 ? N - s * 64 : 64;
  const float own = lane < n ? top[order[s * 64 + lane]] : 0.f, largest = wave_max(own < INFINITY ? own : 0.f);
  const float scale = largest > 0.f ? largest / 127.f : 1.f, inv = 1.f / scale;
  float wn = 0.f, fn = 0.f;
  for (int i = wave * 16; i < wave * 16 + 16; i++) {
    const int v = i < n ? order[s * 64 + i] : -1;
    if (lane == 0) ids[s * 64 + i] = v;
    _Float16 w[NE] = {};
    double x[NE] = {}, w2 = 0.0, f2 = 0.0;
    if (v >= 0 && !scout_entry<NE>(W, v, mean, level, lane, w, x)) w2 = f2 = INFINITY;
#pragma unroll
    for (int e = 0; e < NE; e++) {
      const int k = lane * NE + e;
      const float c = fminf(fmaxf(rintf((float)x[e] * inv), -127.f), 127.f);
      const double f = x[e] - (double)c * (double)scale;
      w2 += x[e] * x[e];
      f2 += f * f;
      sorted[((long)s * 64 + i) * K + k] = w[e];
      // the fragment order of nt_vocab_q8.hip
      codes[((((long)s * KS + k / 32) * 2 + i / 32) * 64 + i % 32 + 32 * ((k % 32) / 16)) * 16 + k % 16] = (int8_t)(int)c;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      w2 += __shfl_xor(w2, m, 64);
      f2 += __shfl_xor(f2, m, 64);
    }
    wn = fmaxf(wn, (float)(sqrt(w2) * 1.0001));
    fn = fmaxf(fn, (float)(sqrt(f2) * 1.0001));
  }
  if (lane == 0) norms[0][wave] = wn, norms[1][wave] = fn;
  __syncthreads();
  if (threadIdx.x == 0)
    consts[s] = make_float4(scale, fmaxf(fmaxf(norms[0][0], norms[0][1]), fmaxf(norms[0][2], norms[0][3])),
                            fmaxf(fmaxf(norms[1][0], norms[1][1]), fmaxf(norms[1][2], norms[1][3])), 0.f);
}

hipError_t vocab_scout_build(const _Float16 *W, int N, int K, const float *gamma, const float *beta, void *dst, hipStream_t s) {
  if (K != 256 && K != 512) return hipErrorInvalidValue;
  const int NS = (N + 63) / 64, parts = (N + SP_ROWS - 1) / SP_ROWS;
  int8_t *codes = (int8_t *)dst;
  float4 *consts = (float4 *)(codes + scout_code_bytes(N, K));
  int32_t *ids = (int32_t *)(consts + NS);
  _Float16 *sorted = (_Float16 *)(ids + 64 * (size_t)NS);
  int8_t *level = (int8_t *)dst + scout_level_at(N, K);
  std::vector<float> h_top((size_t)N);  // (before the device memory: they may throw)
  std::vector<int32_t> h_order((size_t)N);
  char *tmp = nullptr;
  hipError_t e = hipMalloc((void **)&tmp, (size_t)parts * K * 16 + (size_t)K * 4 + (size_t)N * 8);
  if (e != hipSuccess) return e;
  double *sums = (double *)tmp;
  float *mean = (float *)(sums + (size_t)parts * 2 * K), *top = mean + K;
  int32_t *order = (int32_t *)(top + N);
  hipLaunchKernelGGL(scout_sum_kernel, dim3(parts), dim3(K), 0, s, W, N, K, sums);
  hipLaunchKernelGGL(scout_mean_kernel, dim3(1), dim3(K), 0, s, sums, parts, N, K, gamma, beta, mean, level);
  hipLaunchKernelGGL(K == 512 ? scout_top_kernel<8> : scout_top_kernel<4>, dim3((N + 3) / 4), dim3(256), 0, s, W, N, mean, level, top);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(h_top.data(), top, (size_t)N * 4, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  std::iota(h_order.begin(), h_order.end(), 0);
  std::stable_sort(h_order.begin(), h_order.end(), [&](int32_t a, int32_t b) { return h_top[(size_t)a] < h_top[(size_t)b]; });
  if (e == hipSuccess) e = hipMemcpyAsync(order, h_order.data(), (size_t)N * 4, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(K == 512 ? scout_pack_kernel<8> : scout_pack_kernel<4>, dim3(NS), dim3(256), 0, s, W, N, mean, level, top, order, codes,
                       consts, ids, sorted);
    e = hipGetLastError();
  }
  const hipError_t done = hipStreamSynchronize(s);
  (void)hipFree(tmp);
  return e != hipSuccess ? e : done;
}

// ---------------------------------------------------------------------------------------------------------------------
struct ScSplit {
  int m_tiles, G, per_xcd;
};
static ScSplit sc_split(int M, int NS) {
  ScSplit p;
  p.m_tiles = (M + SC_ROWS - 1) / SC_ROWS;
  p.G = std::max(1, std::min(256 / p.m_tiles, NS));
  p.per_xcd = (p.m_tiles * p.G + 7) / 8;
  return p;
}

// What a group leaves, of its three largest products << 5 | place
__device__ __forceinline__ i32x2 scout_pair(const int (&top)[3]) {
  const int apart = ((top[1] >> 5) - (top[2] >> 5)) >> SC_APART;
  const int second = top[1] > SC_NONE / 2 ? top[1] : SC_LOW * 32;
  return i32x2{top[0], (second >> 5) << 8 | (apart > 7 ? 7 : apart) << 5 | (second & 31)};
}

// part[m][2 strip + g]: {largest product << 5 | place, runner-up << 8 | min(7, distance to the third >> SC_APART) << 5 | place}
template <int K>
__global__ __launch_bounds__(SC_WAVES * 64) void vocab_scout_kernel(const int8_t *__restrict__ codes, int M, const int8_t *__restrict__ Wq,
                                                                   int N, int m_tiles, int G, int per_xcd, int ns_div_g, int ns_mod_g,
                                                                   unsigned int m_tiles_magic, i32x2 *__restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int LD = K + 16;  // bytes per LDS row: the pad keeps the 16-byte fragment reads conflict-free
  constexpr int KS = K / 32;
  constexpr int SL = 4;       // ring of fragment slots per wave (lookahead SL - 1 k-steps)
  static_assert(KS % SL == 0, "the ring of slots must divide the k-steps of a strip");
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int total = m_tiles * G;
  const int idx = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  {
    const int end = ((blockIdx.x & 7) + 1) * per_xcd;
    if (idx >= (end < total ? end : total)) return;  // uniform over the workgroup
  }
  // idx / m_tiles by multiply-high, which stays in scalar registers (exact for idx * m_tiles < 2^32)
  const int gi = m_tiles_magic ? (int)__umulhi((unsigned int)idx, m_tiles_magic) : idx;
  const int m0 = (idx - gi * m_tiles) * SC_ROWS;
  const int NS = (N + 63) >> 6;
  const int sb0 = gi * ns_div_g + (gi < ns_mod_g ? gi : ns_mod_g);
  const int sb1 = sb0 + ns_div_g + (gi < ns_mod_g ? 1 : 0);

  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wq, 0, NS * 64 * K, 0x00020000);
  const int wlane = lane * 16;
  auto wload = [&](int soff, int nb) -> i32x4 {
    u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(wrs, wlane + nb * 1024, soff, 0);
    return __builtin_bit_cast(i32x4, t);
  };
  i32x4 wb[SL][2];
  int strip = sb0 + wave;
  const bool have = strip < sb1;
  {  // the tile of codes: global memory -> registers -> LDS.  Rows past M repeat row M - 1 (never stored)
    constexpr int CPR = K / 16, PER_T = SC_ROWS * CPR / (SC_WAVES * 64);
    u32x4 fr[PER_T];
#pragma unroll
    for (int i = 0; i < PER_T; i++) {
      const int c = tid + SC_WAVES * 64 * i, R = c / CPR, kc = c % CPR;
      const int m = m0 + R < M ? m0 + R : M - 1;
      fr[i] = *(const u32x4 *)(codes + (long)m * K + kc * 16);
    }
    if (have) {
#pragma unroll
      for (int q = 0; q < SL - 1; q++) {
        wb[q][0] = wload(strip * (KS * 2048) + q * 2048, 0);
        wb[q][1] = wload(strip * (KS * 2048) + q * 2048, 1);
      }
    }
#pragma unroll
    for (int i = 0; i < PER_T; i++) {
      const int c = tid + SC_WAVES * 64 * i, R = c / CPR, kc = c % CPR;
      *(u32x4 *)(smem + R * LD + kc * 16) = fr[i];
    }
  }
  __syncthreads();
  if (!have) return;

  i32x16 acc[4][2];
  const unsigned char *hrow = smem + li * LD + g * 16;
  int off2 = 64 * LD;  // second base register: the offsets of rows 64.. do not fit the 16-bit immediate
  asm volatile("" : "+v"(off2));
  const unsigned char *hrow2 = hrow + off2;
  i32x4 hf[4];
#pragma unroll
  for (int op = 0; op < 4; op++) hf[op] = *(const i32x4 *)((op < 2 ? hrow : hrow2) + (op & 1) * 32 * LD);
  i32x2 *out = part + (long)(m0 + li) * (2 * NS) + g;
  const bool full = m0 + SC_ROWS <= M;
  for (; strip < sb1; strip += SC_WAVES) {
    const bool more = strip + SC_WAVES < sb1;
    const int pcur = strip * (KS * 2048);
    const int pnext = (more ? strip + SC_WAVES : strip) * (KS * 2048);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const int tgt = ks + SL - 1;
      const int pf = tgt < KS ? pcur + tgt * 2048 : pnext + (tgt - KS) * 2048;
      const int ksn = (ks + 1) % KS;
#pragma unroll
      for (int op = 0; op < 4; op++) {
#pragma unroll
        for (int nb = 0; nb < 2; nb++) {
          if (ks == 0) {
            const i32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            acc[op][nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wb[ks % SL][nb], hf[op], zero, 0, 0, 0);
          } else {
            acc[op][nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wb[ks % SL][nb], hf[op], acc[op][nb], 0, 0, 0);
          }
        }
        // refill what was just consumed; the scheduling barrier keeps the loads this far ahead of their use
        hf[op] = *(const i32x4 *)((op < 2 ? hrow : hrow2) + (op & 1) * 32 * LD + ksn * 32);
        if (op == 0) {
          wb[tgt % SL][0] = wload(pf, 0);
          wb[tgt % SL][1] = wload(pf, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // ---- strip done: the three largest of this lane's 32 products per row, with their places ----
    int top[4][3];
    auto fold = [&](auto masked_tag) {
      constexpr bool MASKED = decltype(masked_tag)::value;
#pragma unroll
      for (int a = 0; a < 4; a++) top[a][0] = top[a][1] = top[a][2] = SC_NONE;
#pragma unroll
      for (int nb = 0; nb < 2; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++)
#pragma unroll
          for (int a = 0; a < 4; a++) {
            int x = (acc[a][nb][v] << 5) | (nb * 16 + v), second, third;
            if (MASKED) x = strip * 64 + nb * 32 + (v >> 2) * 8 + g * 4 + (v & 3) < N ? x : SC_NONE;
            asm("v_med3_i32 %0, %1, %2, %3" : "=v"(third) : "v"(top[a][1]), "v"(top[a][2]), "v"(x));
            asm("v_med3_i32 %0, %1, %2, %3" : "=v"(second) : "v"(top[a][0]), "v"(top[a][1]), "v"(x));
            top[a][2] = third;
            top[a][1] = second;
            top[a][0] = top[a][0] > x ? top[a][0] : x;
          }
    };
    auto pair = [&](int a) { return scout_pair(top[a]); };
    if (strip * 64 + 64 <= N) fold(std::false_type{}); else fold(std::true_type{});
    // straight-line stores for whole tiles (a guard around each makes it wait for the one before)
    if (full) {
#pragma unroll
      for (int a = 0; a < 4; a++) out[(long)a * 32 * (2 * NS) + 2 * strip] = pair(a);
    } else {
#pragma unroll
      for (int a = 0; a < 4; a++)
        if (m0 + a * 32 + li < M) out[(long)a * 32 * (2 * NS) + 2 * strip] = pair(a);
    }
  }
}

// The same for up to 64 rows (32 RBS): a wave per strip and block of 32 rows, four to a workgroup.  The launch is one wave's latency there: all
// fragments of the strip are requested at once, behind the tile's codes, and a wave has a quarter of the products that a strip of the kernel
// above has, where 45 rows waited for 128.  A step of 33 / 45 / 64 rows alone 17.6 / 17.8 / 18.1 us -> 16.9 / 17.1 / 17.5; 65 / 90 / 128 rows, four
// blocks of 32, would take 19.9 / 20.6 / 21.4 where the kernel above takes 19.4 / 20.2 / 20.7.
template <int K, int RBS>
__global__ __launch_bounds__(256) void vocab_scout_few_kernel(const int8_t *__restrict__ codes, int M, const int8_t *__restrict__ Wq, int N,
                                                              i32x2 *__restrict__ part) {
  constexpr int LD = K + 16, KS = K / 32, CPR = K / 16, PER_T = 32 * RBS * CPR / 256;
  __shared__ __attribute__((aligned(16))) unsigned char smem[32 * RBS * LD];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rb = wave % RBS;
  const int NS = (N + 63) >> 6, strip = blockIdx.x * (4 / RBS) + wave / RBS;
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wq, 0, NS * 64 * K, 0x00020000);
  u32x4 fr[PER_T];
#pragma unroll
  for (int i = 0; i < PER_T; i++) {  // rows past M repeat row M - 1 (never stored)
    const int c = tid + 256 * i, R = c / CPR, kc = c % CPR;
    fr[i] = *(const u32x4 *)(codes + (long)min(R, M - 1) * K + kc * 16);
  }
  __builtin_amdgcn_sched_barrier(0);
  i32x4 w[KS][2];  // (past the end of the matrix: zeros)
#pragma unroll
  for (int ks = 0; ks < KS; ks++)
#pragma unroll
    for (int nb = 0; nb < 2; nb++)
      w[ks][nb] = __builtin_bit_cast(i32x4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16 + nb * 1024, (strip * KS + ks) * 2048, 0));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < PER_T; i++) {
    const int c = tid + 256 * i, R = c / CPR, kc = c % CPR;
    *(u32x4 *)(smem + R * LD + kc * 16) = fr[i];
  }
  __syncthreads();
  i32x16 acc[2];
#pragma unroll
  for (int nb = 0; nb < 2; nb++)
#pragma unroll
    for (int v = 0; v < 16; v++) acc[nb][v] = 0;
  const unsigned char *hrow = smem + (rb * 32 + li) * LD + g * 16;
#pragma unroll
  for (int ks = 0; ks < KS; ks++) {
    const i32x4 x = *(const i32x4 *)(hrow + ks * 32);
#pragma unroll
    for (int nb = 0; nb < 2; nb++) acc[nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[ks][nb], x, acc[nb], 0, 0, 0);
  }
  int top[3] = {SC_NONE, SC_NONE, SC_NONE};
#pragma unroll
  for (int nb = 0; nb < 2; nb++)
#pragma unroll
    for (int v = 0; v < 16; v++) {
      int x = (acc[nb][v] << 5) | (nb * 16 + v), second, third;
      x = strip * 64 + nb * 32 + (v >> 2) * 8 + g * 4 + (v & 3) < N ? x : SC_NONE;
      asm("v_med3_i32 %0, %1, %2, %3" : "=v"(third) : "v"(top[1]), "v"(top[2]), "v"(x));
      asm("v_med3_i32 %0, %1, %2, %3" : "=v"(second) : "v"(top[0]), "v"(top[1]), "v"(x));
      top[2] = third;
      top[1] = second;
      top[0] = top[0] > x ? top[0] : x;
    }
  const int m = rb * 32 + li;
  if (strip < NS && m < M) part[(long)m * (2 * NS) + 2 * strip + g] = scout_pair(top);
}

constexpr int PK_WAVES = 8;
// Up to so many rows, a workgroup each: 5.3 us against 5.8 with two (45 rows), 5.6 against 5.8 (260), 7.7 against 7.8 (400), but 11.8
// against 9.9 at 1,000, where the workgroups no longer fit the chip at once.
constexpr int kPickOneRow = 512;

template <int K, int PK_ROWS>
__global__ __launch_bounds__(PK_WAVES * 64) void vocab_pick_kernel(PickArgs a, int M, int32_t *tok, int32_t *slot_of_row) {
  __shared__ PickShared<K, PK_ROWS, PK_WAVES> sh;
  pick_rows<K, PK_ROWS, PK_WAVES>(a, sh, blockIdx.x * PK_ROWS, M);
  const int i = blockIdx.x * PK_ROWS + threadIdx.x;
  if (threadIdx.x < PK_ROWS && i < M) {
    tok[a.row0 + i] = (int32_t)(0xFFFFFFFFu - (unsigned int)sh.best[threadIdx.x]);
    slot_of_row[a.row0 + i] = -1;
  }
}

// Rows per launch: their pairs stay within 64 MiB
static int scout_chunk(int N) {
  const size_t per_row = (size_t)((N + 63) / 64) * 16;
  return (int)std::max<size_t>(SC_ROWS, std::min<size_t>(8192, ((size_t)64 << 20) / per_row / SC_ROWS * SC_ROWS));
}
size_t vocab_scout_scratch_bytes(int N, int rows) {
  return (size_t)std::min(scout_chunk(N), (rows + SC_ROWS - 1) / SC_ROWS * SC_ROWS) * (size_t)((N + 63) / 64) * 16;
}

bool vocab_scout_one_launch(int N, int rows) { return rows <= scout_chunk(N); }
static PickArgs pick_args(const VocabScout &v, const _Float16 *h, const _Float16 *h_lo, long ldh, const VocabWeights &w, int row0, bool distrust) {
  const int NS = (w.N + 63) / 64;
  const float4 *consts = (const float4 *)((const int8_t *)v.matrix + scout_code_bytes(w.N, w.K));
  const int32_t *ids = (const int32_t *)(consts + NS);
  return PickArgs{v.scratch, v.row_consts, consts, ids, NS, row0, distrust ? INFINITY : 0.f, h, h_lo, ldh, (const _Float16 *)(ids + 64 * (size_t)NS)};
}

constexpr int kScoutFewRows = 64;
template <int K, int RBS>
static hipError_t scout_few_launch(const VocabScout &v, int M, int N, hipStream_t s) {
  const int NS = (N + 63) / 64, per = 4 / RBS;
  hipLaunchKernelGGL((vocab_scout_few_kernel<K, RBS>), dim3((NS + per - 1) / per), dim3(256), 0, s, v.codes, M, (const int8_t *)v.matrix, N, (i32x2 *)v.scratch);
  return hipGetLastError();
}

template <int K>
static hipError_t scout_launch(const VocabScout &v, const _Float16 *h, const _Float16 *h_lo, long ldh, const VocabWeights &w, int M, bool distrust,
                               int32_t *tok, int32_t *slot_of_row, PickArgs *later, hipStream_t s) {
  const int NS = (w.N + 63) / 64, chunk = scout_chunk(w.N);
  const int8_t *Wq = (const int8_t *)v.matrix;
  constexpr int lds = SC_ROWS * (K + 16);  // 66 KiB at K = 512
  // raising the dynamic LDS limit is per kernel, once per process (several host threads may get here at once)
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [] { attr_err = hipFuncSetAttribute((const void *)vocab_scout_kernel<K>, hipFuncAttributeMaxDynamicSharedMemorySize, lds); });
  if (attr_err != hipSuccess) return attr_err;
  for (int r0 = 0; r0 < M; r0 += chunk) {
    const int rows = std::min(chunk, M - r0);
    hipError_t e;
    if (M <= kScoutFewRows) {
      e = M <= 32 ? scout_few_launch<K, 1>(v, M, w.N, s) : scout_few_launch<K, 2>(v, M, w.N, s);
    } else {
      const ScSplit p = sc_split(rows, NS);
      const unsigned int magic = p.m_tiles > 1 ? (unsigned int)((0x100000000ull + (unsigned)p.m_tiles - 1) / (unsigned)p.m_tiles) : 0u;
      hipLaunchKernelGGL((vocab_scout_kernel<K>), dim3(8 * p.per_xcd), dim3(SC_WAVES * 64), lds, s, v.codes + (long)r0 * K, rows, Wq, w.N,
                         p.m_tiles, p.G, p.per_xcd, NS / p.G, NS % p.G, magic, (i32x2 *)v.scratch);
      e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    if (later) {  // (vocab_scout_one_launch)
      *later = pick_args(v, h, h_lo, ldh, w, 0, distrust);
      return hipSuccess;
    }
    const PickArgs args = pick_args(v, h, h_lo, ldh, w, r0, distrust);
    auto pick = [&](auto rows_tag) {
      constexpr int PR = decltype(rows_tag)::value;
      hipLaunchKernelGGL((vocab_pick_kernel<K, PR>), dim3((rows + PR - 1) / PR), dim3(PK_WAVES * 64), 0, s, args, rows, tok, slot_of_row);
    };
    if (rows <= kPickOneRow) pick(std::integral_constant<int, 1>{}); else pick(std::integral_constant<int, 2>{});
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_vocab_scout(const VocabScout &v, const _Float16 *h, const _Float16 *h_lo, long ldh, const VocabWeights &w, int M, bool distrust,
                              int32_t *tok, int32_t *slot_of_row, PickArgs *later, hipStream_t s) {
  if (later && !vocab_scout_one_launch(w.N, M)) return hipErrorInvalidValue;
  if (w.K == 512) return scout_launch<512>(v, h, h_lo, ldh, w, M, distrust, tok, slot_of_row, later, s);
  if (w.K == 256) return scout_launch<256>(v, h, h_lo, ldh, w, M, distrust, tok, slot_of_row, later, s);
  return hipErrorInvalidValue;
}

}  // namespace nt
