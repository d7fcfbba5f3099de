// The attention half of a decoder layer in one launch (gfx950): one-head models of width 256 / 512, and eight heads of 64.
//
// Between the Q | K | V projection and the output layer a decoder row passes through
//   self-attention -> output projection + residual -> LayerNorm -> query projection -> cross-attention ->
//   output projection + residual -> [LayerNorm -> FFN + residual ->] final LayerNorm,
// and no step of it reads another row.  A workgroup carries its rows through the whole chain - 2 with eight waves, 4 to 16 with
// sixteen, and where nothing is left but attention also 1 with four or eight and 2 with four (the paper's cure for many small dependent
// nodes is fewer, larger ones, Sec. 3.3 "Graph Optimization"); what passes from one phase to the next stays in the LDS.  As four launches (two attention kernels with a wave per row, two kernels that
// streamed the 512 KB matrices for 32-row tiles) the chain took 24 + 24 + 28 + 16 us at 1,900 rows and 38 us at one row,
// most of it the start and end of launches and, in the projections, 60 workgroups or fewer on 256 CUs.
//
// Attention phases: streams of 16-bit integer keys and values with one fp32 scale per vector (value = code * scale,
// absmax / 32767: an rms error of about 3e-5 of a vector's spread where fp16 leaves 2.8e-4 of every element); the query,
// scores, softmax and context are fp32 (Sec. 3.1 "FP16 Inference").  Lane l holds elements l * NE .. l * NE + NE - 1 of
// every vector, so a wave instruction reads one whole vector.  Keys are taken four at a time: their sums are reduced together in the
// vector unit (wave_fold), wave-uniform scores, one rescale of the online softmax per block.  A row's blocks are dealt to 1 (1,024 rows or more)
// or 4 partial softmaxes (folded: also 2 or 8) that are merged in order, however many waves compute them.
//
// First layer: token -> z, query, key and value by table (Dec1Table in nt_kernels.h), so the step starts here: one sentence reads
// one row of 6 KB where a launch of its own streamed the 1.5 MB matrix (9 to 11 us up to 512 rows, 15 to 21 us from there on, of
// which 1 to 3 us remain here, most of them hidden behind the caches' first blocks).  The table of a 32,000-entry vocabulary at
// d = 512 has 198 MB (264 where batches of both kinds occur, folded and not) and takes 2 ms of a load of 200 ms.  With the launch against by table: one sentence
// 1,008 -> 811 us, 45 sentences 3,225 -> 2,505, 8 sentences of the 256-wide model 1,188 -> 920 us, a 4,096-token budget
// 28.4 -> 25.2 ms, 16,384 tokens 76.0 -> 68.2, 65,536 tokens 559 -> 521, 320 rows of 180 tokens 22.7 -> 20.5, the model with
// 8 heads and FFN 2,048 116.8 -> 109.0 ms, the 30 + 6 layer teacher 110.4 -> 109.1.  It is the faster form at every row count, so
// every layer of this file's kinds takes it; only the shapes without a layer in one launch keep dec_qkv_kernel.
//
// Projection phases: every workgroup pulls the whole matrix through its CU (64 B per clock: 3.9 us for 512 KB at
// 2.1 GHz), which is what bounds them.  A wave owns D / 8 or D / 16 output columns.  With at most eight rows the head and
// the tail plane of the activations share one 16-row operand (rows 0-7 head, 8-15 tail) and the two halves of the result
// meet in one lane exchange; sixteen rows take one 16x16x32 MFMA per plane.  (A 32x32x16 operand would be mostly empty: four
// times the matrix time.)  The weight fragments of the next projection are requested before the attention or LayerNorm
// phase that precedes it.
//
// Folded attention (one-layer decoders).  q . k = (W y + b) . k = y . (W^T k) + b . k,
// and Wo (sum p v) + bo = sum p (Wo v + bo).  With the cross keys and values of a sentence multiplied by the two matrices once,
// when the batch is encoded, and the self values projected by the product of value and output matrix (formed at load, the last
// group of columns of the table), a step's attention half has no projection left.  The self values are cached without their constant, which a
// softmax passes through unchanged, and with every column divided by its norm: either would set the one scale of a vector's
// integers for all its elements (eight output biases of 16, or eight output columns 16 times as large, leave 1.3e-5 / 1.1e-4 of
// the context's norm instead of 2.5e-6 / 2.7e-5).  Batches of up to kDec1FoldRows rows: the cross products are formed from the rounded
// (integer) vectors, so nothing is rounded that was not before, and kept in fp32: twice the bytes (a 4,096-token budget, batches of 36 to 341 rows: 27.5 ms folded up to 256 rows, 26.7 up to
// 512; batches alone on the chip, 300 / 450 rows of 35 padded tokens: 3.14 -> 2.74 / 3.89 -> 3.52 ms folded; 320 rows of 180:
// 24.0 ms with, 23.9 without, which puts the line for kDec1FoldTokens below that).  What is left is latency: a row per workgroup of four or eight waves.  One row 20.6 us without folding, 12.8 with the cross cache folded,
// 45 rows 26 and 17.8; with the self values too, one sentence 1119 -> 1012 us, 45 sentences 3742 -> 3207 us, 8 sentences of
// the 256-wide model 1253 -> 1175 us, a 4,096-token budget 28.0 -> 27.5 ms (each with the projection as a launch of its own).
//
// A folded row's time is its chain of dependent steps, by the clock of one wave (a sentence of 22 tokens, about 2.4 clocks per ns): 4,500 until
// the arguments and the last step's partial keys are there, 1,300 for the token, 2,300 for the table's rows, 1,000 for their
// combination, 1,200 per four keys of a wave, 900 for a merge of partial softmaxes, 800 per normalisation, 1,400 to the end.  So what
// depends on no row is staged in the LDS meanwhile (fold_const, fold_pos; requested where it was used it came to three more turns of
// the memory system), the caches' first keys travel with the table's rows, the row's waves all hold it and merge a share of the
// columns each, and the pair that is appended is rounded by the wave with the fewest keys.  One row of 22 tokens 10.3 -> 9.2 us, 45 rows
// 13.4 -> 11.6, 300 of 13 14.0 -> 12.8, integer caches 320 rows of 150 31.8 -> 30.1, 2,000 of 27 40.4 -> 37.6; with an FFN 45 rows
// 24.0 -> 21.6.  One sentence 690 -> 655 us, 45 sentences 2,120 -> 1,970, a 4,096-token budget 19.2 -> 18.8 ms.
//
// Larger batches keep the products as 16-bit integers, the same bytes as without folding (nt_cross_fold.hip).  A step's layer alone, us,
// against three matrices per workgroup: 2,000 rows of 27 tokens 55 -> 40, 700 of 40 44 -> 25, 1,000 of 55 55 -> 34, 320 of 150 49 -> 32;
// with an FFN of the model's width 70 -> 57, 55 -> 37 (700 of 40), 58 -> 44.  200,000 sentences at 65,536 tokens 457 -> 430 ms, 320 rows of 150
// tokens 18.7 -> 14.9 ms, 32,768 through the submitted student 96 -> 89.5 ms.  Not before an 8-bit output layer (fold_all in
// nt_host.hip); several layers have no folded form.
//
// Registers: three forms spill some of theirs - eight heads with two rows (28 bytes of scratch per lane) and with eight rows
// (56 bytes), folded in fp32 with two rows and the FFN at d = 512 (56 bytes, 44 with a row map).  The others use no scratch.
//
// Measured per step of 1,900 / 45 / 1 rows, alone: 92 / 42 / 38 us as four launches, 71 / 30 / 25 us as one, without
// the launch that projected Q | K | V (21 / 11 / 9 us).  With the table in its place and folded caches one row now takes 7.1 to 7.4 us.
//
// Eight heads of 64 (HEADS): the caches stay fp32 (self) and fp16 (cross); a vector still lies across one wave instruction, a
// head on eight of its lanes, so that every lane keeps its own head's softmax and a score costs three DPP adds.  Relative keys
// enter as one number per (head, clipped distance), computed once per row.  Against two attention launches, two chains and a
// projection per layer: 2,048 sentences through the 30 + 6 layer teacher 139 -> 123 ms, 16,384 through the model with 8 heads
// and FFN 2,048 119 -> 115 ms.
//
// Caches: row c (a sentence), position p: keys at kv[((c * row_positions + p) * 2) * d], values d elements later; scales
// at sc[(c * row_positions + p) * 2 + {0: key, 1: value}].  The newest pair arrives as fp32 from the projection, is used
// at full precision and appended in integer form.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "nt_kernels.h"
#include "nt_pick.h"

namespace nt {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D1_NK = 4;     // keys per block
constexpr int D1_SL = 4;     // ring of weight fragments: k-steps of 32 in flight per wave

bool attn_i16_supported(int d, int heads, int clip) { return heads == 1 && clip == 0 && (d == 256 || d == 512); }
bool dec1_heads_supported(int d, int heads) { return d == 512 && heads == 8; }

template <int NE>
__device__ __forceinline__ void d1_load(const float *p, float (&x)[NE]) {
#pragma unroll
  for (int e = 0; e < NE; e += 4) {
    const float4 t = *(const float4 *)(p + e);
    x[e] = t.x, x[e + 1] = t.y, x[e + 2] = t.z, x[e + 3] = t.w;
  }
}

// x (NE elements per lane, one vector per wave) -> integer codes at dst, scale at *sc; x becomes code * scale
template <int NE>
__device__ __forceinline__ void d1_quantize_store(float (&x)[NE], short *dst, float *sc, int lane) {
  typedef short shortNE __attribute__((ext_vector_type(NE)));
  float amax = 0.f;
#pragma unroll
  for (int e = 0; e < NE; e++) amax = fmaxf(amax, fabsf(x[e]));
  amax = wave_max(amax);
  const float scale = amax > 0.f ? amax / 32767.f : 1.f;
  const float inv = 1.f / scale;
  shortNE qv;
#pragma unroll
  for (int e = 0; e < NE; e++) {
    float c = rintf(x[e] * inv);
    c = fminf(fmaxf(c, -32767.f), 32767.f);
    qv[e] = (short)(int)c;
    x[e] = c * scale;
  }
  *(shortNE *)(dst + lane * NE) = qv;
  if (lane == 0) *sc = scale;
}

// fp32 rows [M][2 d] (key | value of one position each) -> integer cache + scales.
// PLANES (the folded cross cache below): the rounded vectors also as head / tail planes, and key_const[m] = u . key.
template <int NE, bool PLANES>
__global__ __launch_bounds__(256) void quantize_kv_i16_kernel(const float *x, long M, short *cache, float *sc, KvPlanes pl) {
  constexpr int D = NE * 64;
  const int lane = threadIdx.x & 63;
  const long m = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (m >= M) return;
#pragma unroll
  for (int which = 0; which < 2; which++) {
    float v[NE];
    const float *src = x + (m * 2 + which) * D + lane * NE;
#pragma unroll
    for (int e = 0; e < NE; e += 4) {
      const f32x4 t = __builtin_nontemporal_load((const f32x4 *)(src + e));  // read once
      v[e] = t[0], v[e + 1] = t[1], v[e + 2] = t[2], v[e + 3] = t[3];
    }
    d1_quantize_store<NE>(v, cache + (m * 2 + which) * D, sc + m * 2 + which, lane);
    if constexpr (PLANES) {  // v holds code * scale now
      typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
      halfNE hi, lo;
#pragma unroll
      for (int e = 0; e < NE; e++) {
        v[e] = as_f32(v[e]);
        hi[e] = (_Float16)v[e];
        lo[e] = (_Float16)(v[e] - (float)hi[e]);
      }
      _Float16 *dst = (which ? pl.v : pl.k) + m * D + lane * NE;
      *(halfNE *)dst = hi;
      *(halfNE *)(dst + pl.lo_offset) = lo;
      if (which == 0) {
        float u[NE], s = 0.f;
        d1_load<NE>(pl.u + lane * NE, u);
#pragma unroll
        for (int e = 0; e < NE; e++) s += u[e] * v[e];
        s = wave_sum(s);
        if (lane == 0) pl.key_const[m] = s * pl.scale;
      }
    }
  }
}

hipError_t launch_quantize_kv_i16(const float *x, long M, int d, short *cache, float *sc, const KvPlanes *planes, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  const dim3 grid((unsigned)((M + 3) / 4)), block(256);
  if (d != 512 && d != 256) return hipErrorInvalidValue;
#define NT_QKV(NE_, P_) hipLaunchKernelGGL((quantize_kv_i16_kernel<NE_, P_>), grid, block, 0, s, x, M, cache, sc, planes ? *planes : KvPlanes{})
  if (d == 512) { if (planes) NT_QKV(8, true); else NT_QKV(8, false); }
  else { if (planes) NT_QKV(4, true); else NT_QKV(4, false); }
#undef NT_QKV
  return hipGetLastError();
}

// The first layer's projection table (Dec1Table): centred rows x B in double, once per load.  64 rows x 64 columns per
// workgroup, 4 x 4 per lane.
constexpr int DT_T = 64, DT_K = 32;
__global__ __launch_bounds__(256) void dec1_table_kernel(const _Float16 *E, const float *pe, const float *gamma, const float *beta,
                                                         const double *B, const double *bias, int vocab, int max_len, int d, int N, float *rows) {
  __shared__ double sa[DT_K][DT_T + 2], sb[DT_K][DT_T], sm[DT_T];
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4, n0 = blockIdx.x % (N / DT_T) * DT_T;
  const long r0 = (long)(blockIdx.x / (N / DT_T)) * DT_T, R = (long)vocab + max_len + 1;
  const double root = sqrt((double)d);
  auto element = [&](long r, int k) { return r < vocab ? root * (double)(float)E[r * d + k] : r < R - 1 ? (double)pe[(r - vocab) * d + k] : 0.0; };
  {  // means of the rows, four lanes each
    double s = 0.0;
    for (int k = tid & 3; k < d; k += 4) s += element(r0 + (tid >> 2), k);
    s += __shfl_xor(s, 1, 64);
    s += __shfl_xor(s, 2, 64);
    if ((tid & 3) == 0) sm[tid >> 2] = s / (double)d;
  }
  __syncthreads();
  double acc[4][4] = {};
  for (int k0 = 0; k0 < d; k0 += DT_K) {
    for (int i = tid; i < DT_T * DT_K; i += 256) {
      const int k = k0 + i % DT_K;
      const long r = r0 + i / DT_K;
      sa[i % DT_K][i / DT_K] = r < R - 1 ? (element(r, k) - sm[i / DT_K]) * (double)gamma[k] : r == R - 1 ? (double)beta[k] : 0.0;
      sb[i / DT_T][i % DT_T] = B[(long)(k0 + i / DT_T) * N + n0 + i % DT_T];
    }
    __syncthreads();
    for (int k = 0; k < DT_K; k++) {
      double x[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; i++) x[i] = sa[k][ty * 4 + i], w[i] = sb[k][tx + i * 16];
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] += x[i] * w[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const long r = r0 + ty * 4 + i;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int n = n0 + tx + j * 16;
      if (r < R) rows[r * N + n] = (float)(acc[i][j] + (r == R - 1 ? bias[n] : 0.0));
    }
  }
}

size_t dec1_table_bytes(int vocab, int max_len, int d, int parts) { return ((size_t)vocab + max_len + 1) * parts * d * sizeof(float); }

hipError_t launch_dec1_table(const _Float16 *E, const float *pe, const float *gamma, const float *beta, const double *B, const double *bias,
                             int vocab, int max_len, int d, int parts, float *rows, hipStream_t s) {
  const long R = (long)vocab + max_len + 1;
  const int N = parts * d;
  if (d % DT_K != 0 || N % DT_T != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(dec1_table_kernel, dim3((unsigned)((R + DT_T - 1) / DT_T * (N / DT_T))), dim3(256), 0, s, E, pe, gamma, beta, B, bias,
                     vocab, max_len, d, N, rows);
  return hipGetLastError();
}

// Dec1Args::fold_const (for either form of the caches, 13 vectors each) and fold_pos, one vector per workgroup
constexpr int DF_CONST = 13;
__global__ __launch_bounds__(256) void dec1_fold_vectors_kernel(Dec1FoldVectors v, int d, float *dst) {
  const int i = blockIdx.x, form = i / DF_CONST, u = i % DF_CONST, ffn = v.ln3.gamma != nullptr;
  const long ld = (long)v.table.parts * d;
  const float *src = nullptr;
  if (form < 2) {
    const float *offset = v.table.rows + (v.vocab + v.table.max_len) * ld;
    const bool two = form == 1 && v.gamma2;
    const float *all[DF_CONST] = {two ? v.gamma2 : v.ln2.gamma, two ? v.beta2 : v.ln2.beta, v.ln3.gamma, v.ln3.beta, v.lnf.gamma, v.lnf.beta,
                                  v.fold_scale, v.fold_bias, v.cross_scale, v.cross_const, offset, offset + d, offset + ld - d};
    src = u < 2 || ffn ? all[u] : u + 2 < DF_CONST ? all[u + 2] : nullptr;
  } else {
    const int t = (i - 2 * DF_CONST) / 4, w = (i - 2 * DF_CONST) % 4;
    const float *pos = v.table.rows + (v.vocab + t) * ld;
    src = w == 3 ? v.pe + (long)t * d : w == 2 ? pos + ld - d : pos + w * d;
  }
  for (int k = threadIdx.x; k < d; k += 256) dst[(long)i * d + k] = src ? src[k] : 0.f;
}
size_t dec1_fold_vectors_bytes(int d, int max_len) { return (size_t)(2 * DF_CONST + 4 * max_len) * d * sizeof(float); }
hipError_t launch_dec1_fold_vectors(const Dec1FoldVectors &v, int d, float *dst, hipStream_t s) {
  hipLaunchKernelGGL(dec1_fold_vectors_kernel, dim3((unsigned)(2 * DF_CONST + 4 * v.table.max_len)), dim3(256), 0, s, v, d, dst);
  return hipGetLastError();
}
const float *dec1_fold_const(const float *vectors, int d, int folded) { return vectors + (long)(folded - 1) * DF_CONST * d; }
const float *dec1_fold_pos(const float *vectors, int d) { return vectors + 2L * DF_CONST * d; }

// One partial softmax over some of a row's keys.
template <int NE>
struct D1Part {
  float m, l, acc[NE];
  __device__ __forceinline__ void clear() {
    m = -INFINITY, l = 0.f;
#pragma unroll
    for (int e = 0; e < NE; e++) acc[e] = 0.f;
  }
  __device__ __forceinline__ void merge(const D1Part &o) {
    const float mn = fmaxf(m, o.m);
    const float ca = (m == -INFINITY) ? 0.f : __expf(m - mn);
    const float cb = (o.m == -INFINITY) ? 0.f : __expf(o.m - mn);
    l = l * ca + o.l * cb;
#pragma unroll
    for (int e = 0; e < NE; e++) acc[e] = acc[e] * ca + o.acc[e] * cb;
    m = mn;
  }
};

// Relative keys of one row (several heads only): what a key adds to the score of this lane's head, by its distance to the
// query, clipped; p == nullptr: none.
constexpr int D1_MAX_CLIP = 16;
struct D1Rel {
  const float *p = nullptr;
  int clip = 0, t = 0;  // the query's position
  __device__ __forceinline__ float at(int j) const { return p[max(j - t + clip, 0) * 8]; }
};

// The keys of one block and their fold into a partial softmax; positions past the end repeat the last key and get
// weight 0.  KIND: integers with scales (sc[2 p], sc[2 p + 1]); fp32 keys and values, each key with an additive constant (sc[p]); or
// integers with scales and such a constant (sc[4 p .. 4 p + 2]).
// These numbers, which every lane needs, come through scalar loads (earlier launches wrote them): 16 to 24 vector registers less, which
// are what two blocks in flight take in a wave of 128, and a third of the load instructions (a 4,096-token budget 19.7 -> 19.4 ms).
enum D1Kind { D1_CODES, D1_FLOATS, D1_CODES_CONST };
template <int NE, D1Kind KIND>
struct D1Block {
  static constexpr bool F32 = KIND == D1_FLOATS;
  typedef short shortNE __attribute__((ext_vector_type(NE)));
  typedef float floatNE __attribute__((ext_vector_type(NE)));
  typedef typename std::conditional<F32, floatNE, shortNE>::type Vec;
  typedef typename std::conditional<F32, float, short>::type Elt;
  Vec k[D1_NK], v[D1_NK];
  float ks[D1_NK], vs[D1_NK], kc[D1_NK];

  __device__ __forceinline__ void load(const void *kv, const float *sc, long pos0, int j0, int n, int lane) {
    constexpr int D = NE * 64;
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      const int j = j0 + i < n ? j0 + i : n - 1;
      const long p = pos0 + j;
      const char *kp = (const char *)kv + p * (2 * D * (long)sizeof(Elt));  // (uniform)
      k[i] = *(const Vec *)(kp + (unsigned)lane * sizeof(Vec));
      v[i] = *(const Vec *)(kp + (unsigned)lane * sizeof(Vec) + D * sizeof(Elt));
      typedef const __attribute__((address_space(4))) float *Uniform;
      const Uniform u = (Uniform)(unsigned long long)(sc + p * (F32 ? 1 : KIND == D1_CODES ? 2 : 4));
      ks[i] = F32 ? 1.f : u[0];
      vs[i] = F32 ? 1.f : u[1];
      kc[i] = F32 ? u[0] : KIND == D1_CODES_CONST ? u[2] : 0.f;
    }
  }
  __device__ __forceinline__ void fold(const float (&q)[NE], int j0, int n, int lane, D1Part<NE> &a, const D1Rel &) const {
    float p[D1_NK];
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < NE; e++) s += q[e] * (float)k[i][e];
      p[i] = s;
    }
    // reduce-scatter: after the exchanges over the two top lane bits a lane holds the sum over those bits of the key
    // numbered by them; the remaining exchanges complete it.  Lanes 16 i .. 16 i + 15 then hold the product of key i
    static_assert(D1_NK == 4, "blocks of four keys");
    float r1 = wave_pair16(wave_pair32(p[0], p[2], WaveAdd{}), wave_pair32(p[1], p[3], WaveAdd{}), WaveAdd{});
    r1 = wave_fold16(r1, WaveAdd{});
    float s[D1_NK], bm = -INFINITY;
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      const float dot = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(r1), 16 * i));
      s[i] = F32 ? dot + kc[i] : KIND == D1_CODES_CONST ? dot * ks[i] + kc[i] : dot * ks[i];
      if (j0 + i >= n) s[i] = -INFINITY;
      bm = fmaxf(bm, s[i]);
    }
    const float mn = fmaxf(a.m, bm);  // j0 < n: at least one finite score
    const float corr = (a.m == -INFINITY) ? 0.f : __expf(a.m - mn);
    float w[D1_NK], wsum = 0.f;
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      w[i] = __expf(s[i] - mn);  // exp(-inf) = 0 for the positions past the end
      wsum += w[i];
      if (!F32) w[i] *= vs[i];
    }
    a.l = a.l * corr + wsum;
#pragma unroll
    for (int e = 0; e < NE; e++) {
      float t = a.acc[e] * corr;
#pragma unroll
      for (int i = 0; i < D1_NK; i++) t += w[i] * (float)v[i][e];
      a.acc[e] = t;
    }
    a.m = mn;
  }
};

// The same for heads of eight lanes (64 of 512 columns each): every lane keeps its head's maximum and sum, a score is the sum
// over eight lanes (three DPP adds), and nothing is uniform over the wave but the positions.
__device__ __forceinline__ float d1_head_sum(float v) {
  auto add = [](float x, auto ctrl) {
    return x + __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v = add(v, std::integral_constant<int, 0xB1>{});   // quad_perm: lane ^ 1
  v = add(v, std::integral_constant<int, 0x4E>{});   // quad_perm: lane ^ 2
  return add(v, std::integral_constant<int, 0x141>{});  // mirrored within eight lanes: the other four
}

template <int NE, typename Elt>
struct D1HeadBlock {
  typedef Elt Vec __attribute__((ext_vector_type(NE)));
  Vec k[D1_NK], v[D1_NK];

  __device__ __forceinline__ void load(const void *kv, const float *, long pos0, int j0, int n, int lane) {
    constexpr int D = NE * 64;
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      const int j = j0 + i < n ? j0 + i : n - 1;
      const char *kp = (const char *)kv + (pos0 + j) * (2 * D * (long)sizeof(Elt));  // (uniform)
      k[i] = *(const Vec *)(kp + (unsigned)lane * sizeof(Vec));
      v[i] = *(const Vec *)(kp + (unsigned)lane * sizeof(Vec) + D * sizeof(Elt));
    }
  }
  __device__ __forceinline__ void fold(const float (&q)[NE], int j0, int n, int, D1Part<NE> &a, const D1Rel &rel) const {
    float s[D1_NK], mn = a.m;
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      float p = 0.f;
#pragma unroll
      for (int e = 0; e < NE; e++) p += q[e] * (float)k[i][e];
      s[i] = d1_head_sum(p);
      if (rel.p) s[i] += rel.at(j0 + i < n ? j0 + i : n - 1);
      if (j0 + i >= n) s[i] = -INFINITY;
      mn = fmaxf(mn, s[i]);
    }
    const float corr = (a.m == -INFINITY) ? 0.f : __expf(a.m - mn);
    float w[D1_NK], wsum = 0.f;
#pragma unroll
    for (int i = 0; i < D1_NK; i++) {
      w[i] = __expf(s[i] - mn);
      wsum += w[i];
    }
    a.l = a.l * corr + wsum;
#pragma unroll
    for (int e = 0; e < NE; e++) {
      float t = a.acc[e] * corr;
#pragma unroll
      for (int i = 0; i < D1_NK; i++) t += w[i] * (float)v[i][e];
      a.acc[e] = t;
    }
    a.m = mn;
  }
};
// The input token of a wave's row, in two halves so that the loads between them travel with it: BOS, the given token, or the
// arg-max of the previous step, which the row's first wave also stores.
struct D1Token {
  unsigned long long key[4];  // a lane's first partial keys
  int tok, slot;
  __device__ __forceinline__ void request(const Dec1Args &a, int row, int lane) {
    const StepBeginArgs &b = a.sb;
    tok = b.pad_id, slot = -1;
#pragma unroll
    for (int u = 0; u < 4; u++) key[u] = 0ull;
    if (a.tok_in) {
      if (row < a.rows) tok = a.tok_in[row];
    } else if (b.t > 0 && row < b.rows_prev) {
      if (b.prev_cert == kPrevPick) {
      } else if (b.prev_cert) {
        tok = b.tok[row];
        slot = b.slot_of_row[row];
      } else if (b.pk) {
#pragma unroll
        for (int u = 0; u < 4; u++)
          if (lane + 64 * u < b.n_partials) key[u] = b.pk[(long)row * b.n_partials + lane + 64 * u];
      }
    }
  }
  // picked: the row's key, where the launch has picked it
  __device__ __forceinline__ int resolve(const Dec1Args &a, int row, bool first_wave, int lane, unsigned long long picked) {
    const StepBeginArgs &b = a.sb;
    int y = tok;
    if (!a.tok_in) {
      if (b.t == 0) {
        y = b.bos_id;
      } else if (row < b.rows_prev && (b.prev_cert || b.pk)) {
        if (b.prev_cert == kPrevPick) {
          y = (int)(0xFFFFFFFFu - (unsigned int)picked);
        } else if (b.prev_cert) {
          if (slot >= 0) y = (int)(0xFFFFFFFFu - (unsigned int)b.final_key[slot]);
        } else {
          unsigned long long top = 0ull;
#pragma unroll
          for (int u = 0; u < 4; u++) top = key[u] > top ? key[u] : top;
          for (int q = lane + 256; q < b.n_partials; q += 64) {
            const unsigned long long c = b.pk[(long)row * b.n_partials + q];
            top = c > top ? c : top;
          }
          y = (int)(0xFFFFFFFFu - (unsigned int)wave_max_u64(top));
        }
        if (y < 0 || y >= b.vocab) y = b.pad_id;  // a row none of whose logits is a number
        if (first_wave && lane == 0) b.out[(long)row * b.out_ld + b.t - 1] = y;
      }
      if (b.forced && row < a.rows) {
        y = b.forced[(long)row * b.forced_ld + b.t];
        if (y < 0 || y >= b.vocab) {
          if (lane == 0) b.flags[0] = 1;
          y = b.pad_id;
        }
      }
      if (b.cert_count && blockIdx.x == 0 && threadIdx.x == 0) *b.cert_count = 0;
    }
    if (row >= a.rows) y = b.pad_id;  // computes on the padding token and stores nothing
    return __builtin_amdgcn_readfirstlane(y);
  }
};

// First layer without folding: z = sqrt(d) E[y] + PE[t], and from its mean and scale the query, and (first wave of a row) the key and
// value, by the table (see Dec1Table).  Every wave of a row computes the statistics for itself.
template <int NE>
__device__ __forceinline__ void first_layer_start(const Dec1Args &a, int y, int lane, bool first_wave, float (&q)[NE], float (&z)[NE],
                                                  float (&kx)[NE], float (&vx)[NE]) {
  constexpr int D = NE * 64;
  typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
  const long ld = (long)a.table.parts * D;
  const float *by_token = a.table.rows + y * ld + lane * NE, *by_pos = a.table.rows + (a.sb.vocab + a.sb.t) * ld + lane * NE,
              *offset = a.table.rows + (a.sb.vocab + a.table.max_len) * ld + lane * NE;
  const halfNE ev = *(const halfNE *)(a.sb.E + (long)y * D + lane * NE);
  float pv[NE], tq[NE], tk[NE], tv[NE];
  d1_load<NE>(a.sb.pe + (long)a.sb.t * D + lane * NE, pv);
  d1_load<NE>(by_token, tq);
  if (first_wave) {
    d1_load<NE>(by_token + D, tk);
    d1_load<NE>(by_token + 2 * D, tv);
  }
  const float sc = sqrtf((float)D);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < NE; e++) {
    z[e] = sc * (float)ev[e] + pv[e];
    s += z[e];
  }
  const float mean = wave_sum(s) / (float)D;
  float v = 0.f;
#pragma unroll
  for (int e = 0; e < NE; e++) v += ln_term(z[e] - mean, a.eps.l1);
  const float rs = ln_rscale(wave_sum(v) / (float)D, a.eps);
  auto combine = [&](const float (&t)[NE], int col, float (&x)[NE]) {
    float p[NE], c[NE];
    d1_load<NE>(by_pos + col, p);
    d1_load<NE>(offset + col, c);
#pragma unroll
    for (int e = 0; e < NE; e++) x[e] = rs * (t[e] + p[e]) + c[e];
  };
  combine(tq, 0, q);
  if (first_wave) {
    combine(tk, D, kx);
    combine(tv, 2 * D, vx);
  }
}

// D: model width.  RW: rows per workgroup, NWAVES / RW waves each.  PARTS: partial softmaxes per row.  IND: row r uses cache
// row origin[r] (< 0: no row, zero context).  FFN: the layer's FFN (of width D) is part of the chain.  FOLD32, FOLD16 (0 / 1): the
// caches hold folded vectors, in fp32 or as integers.  HEADS: eight heads of 64 columns, self cache fp32, cross cache fp16, optional
// relative keys.
template <int D, int RW, int NWAVES, int PARTS, int FOLD16, bool IND, bool FFN, bool FOLD32, bool HEADS>
__global__ __launch_bounds__(NWAVES * 64) void dec1_kernel(Dec1Args args) {
  constexpr int NE = D / 64, WR = NWAVES / RW, PW = PARTS / WR;  // elements per lane; waves per row; partials per wave
  constexpr int NC = D / NWAVES, NT = NC / 16;                   // output columns of a wave, in tiles of 16
  constexpr int LD = D + 8, ZLD = D + 4, KS = D / 32, KS16 = D / 16;
  static_assert(PARTS % WR == 0 && KS % D1_SL == 0, "");
  // whether the next matrix's first fragments are requested before an attention phase: 32 of 128 registers, which a wave
  // with several partial softmaxes does not have
  constexpr bool EARLY = !(NWAVES == 16 && (PW > 1 || HEADS));
  constexpr bool FOLD = FOLD32 || FOLD16;
  // folded: what is requested before it is needed: 2 both caches' first blocks before the row's start, 1 a cache's at a time, 0 nothing
  constexpr int AHEAD = !FOLD ? 0 : NWAVES < 16 ? 2 : FFN ? 0 : 1;
  static_assert(!FOLD || PW == 1, "");
  static_assert(!HEADS || (D == 512 && !FOLD && !FFN), "heads are eight lanes of eight elements");
  typedef typename std::conditional<HEADS, D1HeadBlock<NE, float>, D1Block<NE, D1_CODES>>::type SelfBlock;
  typedef typename std::conditional<HEADS, D1HeadBlock<NE, _Float16>,
                                    D1Block<NE, FOLD32 ? D1_FLOATS : FOLD16 ? D1_CODES_CONST : D1_CODES>>::type CrossBlock;
  typedef D1Part<NE> Part;
  __shared__ __attribute__((aligned(16))) _Float16 sA[FOLD && !FFN ? 8 : 2 * RW * LD];  // head rows, then tail rows
  __shared__ __attribute__((aligned(16))) float sZ[RW * ZLD];                     // residual stream
  __shared__ __attribute__((aligned(16))) float sQ[FOLD && !FFN ? 4 : RW * (D + 8)];    // cross-attention query, later:
  _Float16 *sU = (_Float16 *)sQ;                                                  // FFN hidden state, head rows, then tail rows
  // partial softmaxes: of the waves pg > 0, or (folded) of all waves
  __shared__ __attribute__((aligned(16))) float sPart[WR > 1 ? RW * (FOLD ? PARTS * (D + 2) : (PARTS - PW) * (NE + 2) * 64) : 4];
  constexpr int NV = FFN ? 6 : 4, LN2 = 0, LN3 = 2, LNF = NV - 2;  // vectors of the normalisations
  // folded: and, as in Dec1Args::fold_const, scale and constant of either context (VC) and the first layer's constants (VS), and as in
  // fold_pos what goes by the position (VP)
  constexpr int VC = NV, VS = VC + 4, VP = VS + 3, NVT = FOLD ? VP + 4 : NV, NVW = (NVT + NWAVES - 1) / NWAVES;
  __shared__ __attribute__((aligned(16))) float sNorm[NVT * D];
  constexpr bool PICKS = WR > 1 && !IND && !HEADS;  // dec1_picks; the EOS mode's steps start with launches that want the tokens
  __shared__ typename std::conditional<PICKS, PickShared<D, PICKS ? RW : 1, NWAVES>, int>::type sPick;
  __shared__ float sRel[HEADS ? RW * (D1_MAX_CLIP + 1) * 8 : 1];                  // per row: [distance][head]
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 4, c16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = wave / WR, pg = wave % WR;
  const int row0 = blockIdx.x * RW;
  const bool valid = row0 + rw < args.rows;
  D1Token token;
  if (FOLD || args.table.rows) token.request(args, row0 + rw, lane);
  // the normalisations' gains and offsets go to the LDS while the start of the row travels, a vector per wave: read where they are used,
  // each would be another turn of the memory system in the row's chain
  float norm[NVW][NE];
  const float *norm_src[NVW];
#pragma unroll
  for (int u = 0; u < NVW; u++) {
    const int i = wave + u * NWAVES;
    if constexpr (FOLD) {
      norm_src[u] = i < VP ? args.fold_const + i * D : i < NVT ? args.fold_pos + (args.sb.t * 4L + (i - VP)) * D : nullptr;
    } else {
      const GemmLayerNorm &of = i < 2 ? args.ln2 : FFN && i < 4 ? args.ln3 : args.lnf;
      norm_src[u] = i < NV ? (i & 1 ? of.beta : of.gamma) : nullptr;  // (no final one: nullptr)
    }
    if (norm_src[u]) d1_load<NE>(norm_src[u] + lane * NE, norm[u]);
  }
  unsigned long long picked = 0ull;
  if constexpr (PICKS) {
    if (args.sb.prev_cert == kPrevPick) {
      pick_rows<D, RW, NWAVES>(args.sb.pick, sPick, row0, args.sb.rows_prev);
      picked = sPick.best[rw];
    }
  }
  // Without folding the arguments are read again from here on: kept across the pick they took 59 to 85 scalar registers more than there
  // are, moved to vector registers and back in launches that do not pick as well (two such layers, 1 / 16 / 300 rows, us a step: d = 512 56.9 / 66.8 /
  // 71.4 -> 55.9 / 65.5 / 70.0, d = 256 30.2 / 35.6 / 43.4 -> 28.7 / 33.8 / 41.5).
  const Dec1Args *later = &args;
  if constexpr (PICKS && !FOLD) {
    typedef const __attribute__((address_space(4))) Dec1Args *Segment;
    Segment segment = (Segment)__builtin_amdgcn_kernarg_segment_ptr();  // (starts with the only argument)
    asm volatile("" : "+s"(segment));
    later = (const Dec1Args *)segment;
  }
  const Dec1Args &a = *later;
  const int r = valid ? row0 + rw : 0;
  int rc = r;
  if (IND) rc = valid ? a.origin[r] : -1;
  const bool live = valid && rc >= 0;
  rc = __builtin_amdgcn_readfirstlane(live ? rc : 0);

  // ---- weight fragments: [n / 64][k / 16][(n % 64) / 32][n % 32 + 32 * ((k % 16) / 8)][8]; a 16 x 32 operand is four
  // runs of 256 bytes ----
  half8 wb[D1_SL][NT];
  const int n0 = wave * NC;
  const int w_wave = (n0 >> 6) * (KS16 * 2048) + ((n0 >> 5) & 1) * 1024 + ((n0 >> 4) & 1) * 256;  // this wave's first columns
  const int w_lane = (h >> 1) * 2048 + (h & 1) * 512 + c16 * 16;
  auto w_load = [&](const __amdgpu_buffer_rsrc_t &rs, int ks, int t) {
    return __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(rs, w_lane + ((t >> 1) & 1) * 1024 + (t & 1) * 256, w_wave + ks * 4096, 0));
  };
  auto matrix = [&](const _Float16 *W) { return __builtin_amdgcn_make_buffer_rsrc((void *)W, 0, D * D * 2, 0x00020000); };
  auto preload = [&](const _Float16 *W) {
    const __amdgpu_buffer_rsrc_t rs = matrix(W);
#pragma unroll
    for (int q = 0; q < D1_SL; q++)
#pragma unroll
      for (int t = 0; t < NT; t++) wb[q][t] = w_load(rs, q, t);
  };
  // acc[t][v], summed over both planes: row (h & 1) * 4 + v, column n0 + t * 16 + c16 (in lane groups h and h + 2 alike).
  // The ring holds k-steps 0 .. D1_SL - 1 of W on entry.
  f32x4 acc[NT];
  auto project = [&](const _Float16 *W, const _Float16 *planes) {
    const __amdgpu_buffer_rsrc_t rs = matrix(W);
    const _Float16 *ap = planes + (RW == 16 ? c16 : (c16 < 8 ? 0 : RW) + (c16 & (RW - 1))) * LD + h * 8;
#pragma unroll
    for (int t = 0; t < NT; t++) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // D1_SL k-steps per turn; the slot just used is refilled for the next turn, the last turn refills nothing
    auto turn = [&](int kb, auto refill_tag) {
      constexpr bool REFILL = decltype(refill_tag)::value;
      const _Float16 *xp = ap + kb * (D1_SL * 32);
      half8 x[D1_SL], xl[D1_SL];
#pragma unroll
      for (int q = 0; q < D1_SL; q++) {
        x[q] = *(const half8 *)(xp + q * 32);
        if (RW == 16) xl[q] = *(const half8 *)(xp + RW * LD + q * 32);
      }
#pragma unroll
      for (int q = 0; q < D1_SL; q++) {
#pragma unroll
        for (int t = 0; t < NT; t++) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(x[q], wb[q][t], acc[t], 0, 0, 0);
        if (RW == 16) {
#pragma unroll
          for (int t = 0; t < NT; t++) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xl[q], wb[q][t], acc[t], 0, 0, 0);
        }
        if (REFILL) {
#pragma unroll
          for (int t = 0; t < NT; t++) wb[q][t] = w_load(rs, (kb + 1) * D1_SL + q, t);
        }
        __builtin_amdgcn_sched_barrier(0);  // keeps the loads this far ahead of their use
      }
    };
#pragma nounroll
    for (int kb = 0; kb + 1 < KS / D1_SL; kb++) turn(kb, std::true_type{});
    turn(KS / D1_SL - 1, std::false_type{});
    if (RW == 16) return;
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int v = 0; v < 4; v++) acc[t][v] = wave_pair32(acc[t][v], acc[t][v], WaveAdd{});
  };
  // f(row, column, value) for every result of the wave; the lane groups that only duplicate rows stay out
  auto results = [&](auto f) {
    if (RW < 16 && (h >= 2 || (RW < 8 && h != 0))) return;
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int v = 0; v < (RW < 4 ? RW : 4); v++) f((RW == 16 ? h : h & 1) * 4 + v, n0 + t * 16 + c16, acc[t][v]);
  };
  float bias[NT];  // of the wave's columns, requested ahead of the product
  auto request_bias = [&](const float *b) {
#pragma unroll
    for (int t = 0; t < NT; t++) bias[t] = b[n0 + t * 16 + c16];
  };
  auto add_residual = [&]() {
    results([&](int i, int n, float x) { float *z = sZ + i * ZLD + n; *z = x + bias[(n - n0) >> 4] + *z; });
  };
  auto store_planes = [&](const float (&y)[NE]) {
    typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
    halfNE hi, lo;
#pragma unroll
    for (int e = 0; e < NE; e++) {
      const float x = as_f32(y[e]);
      hi[e] = (_Float16)x;
      lo[e] = (_Float16)(x - (float)hi[e]);
    }
    *(halfNE *)(sA + rw * LD + lane * NE) = hi;
    *(halfNE *)(sA + (RW + rw) * LD + lane * NE) = lo;
  };
  auto store_norms = [&]() {
#pragma unroll
    for (int u = 0; u < NVW; u++)
      if (norm_src[u]) {
#pragma unroll
        for (int e = 0; e < NE; e += 4)
          *(float4 *)(sNorm + (wave + u * NWAVES) * D + lane * NE + e) = make_float4(norm[u][e], norm[u][e + 1], norm[u][e + 2], norm[u][e + 3]);
      }
  };
  // LayerNorm of a row of the residual stream: fp32, mean first, then the variance of the centred values
  auto normalise_row = [&](int which, float (&y)[NE]) {
    float ga[NE], be[NE];
    d1_load<NE>(sNorm + which * D + lane * NE, ga);
    d1_load<NE>(sNorm + (which + 1) * D + lane * NE, be);
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < NE; e++) s += y[e];
    const float mean = wave_sum(s) / (float)D;
    float q = 0.f;
#pragma unroll
    for (int e = 0; e < NE; e++) q += ln_term(y[e] - mean, a.eps.l1);
    const float rs = ln_rscale(wave_sum(q) / (float)D, a.eps);
#pragma unroll
    for (int e = 0; e < NE; e++) y[e] = ga[e] * ((y[e] - mean) * rs) + be[e];
  };
  auto normalise = [&](int which, float (&y)[NE]) {  // of this wave's row in the LDS
    d1_load<NE>(sZ + rw * ZLD + lane * NE, y);
    normalise_row(which, y);
  };
  // attention of this wave's row over n cached keys; the partials may hold the newest key already.  The merged context
  // goes to done(ctx) in the row's first wave
  // Two blocks in flight: the next one of the wave's only partial, or one of each of its two.
  constexpr int STEP = PARTS * D1_NK;
  const int j_first = pg * PW * D1_NK;
  auto first_block = [&](auto &b, int which, const void *kv, const float *sc, long pos0, int n) {
    if (j_first + which * STEP < n) b.load(kv, sc, pos0, j_first + which * STEP, n, lane);
  };
  // the wave's share of the keys; b holds the first two blocks already if `preloaded`
  auto fold_keys = [&](auto (&b)[2], auto preloaded, const float (&q)[NE], const void *kv, const float *sc, long pos0, int n, const D1Rel &rel, Part (&st)[PW]) {
    if constexpr (NWAVES == 16 && !decltype(preloaded)::value) {  // 128 registers: one block at a time
      for (int j = j_first; j < n; j += STEP)
#pragma unroll
        for (int u = 0; u < PW; u++)
          if (j + u * D1_NK < n) {
            b[0].load(kv, sc, pos0, j + u * D1_NK, n, lane);
            b[0].fold(q, j + u * D1_NK, n, lane, st[u], rel);
          }
    } else if constexpr (PW == 1) {
      if constexpr (!decltype(preloaded)::value) {
        first_block(b[0], 0, kv, sc, pos0, n);
        first_block(b[1], 1, kv, sc, pos0, n);
      }
      for (int j = j_first; j < n; j += 2 * STEP) {
        b[0].fold(q, j, n, lane, st[0], rel);
        if (j + 2 * STEP < n) b[0].load(kv, sc, pos0, j + 2 * STEP, n, lane);
        if (j + STEP < n) b[1].fold(q, j + STEP, n, lane, st[0], rel);
        if (j + 3 * STEP < n) b[1].load(kv, sc, pos0, j + 3 * STEP, n, lane);
      }
    } else {
      static_assert(PW == 2, "one or two partials per wave");
      for (int j = j_first; j < n; j += STEP) {
        b[0].load(kv, sc, pos0, j, n, lane);
        if (j + D1_NK < n) b[1].load(kv, sc, pos0, j + D1_NK, n, lane);
        b[0].fold(q, j, n, lane, st[0], rel);
        if (j + D1_NK < n) b[1].fold(q, j + D1_NK, n, lane, st[1], rel);
      }
    }
  };
  auto attend = [&](auto (&b)[2], const float (&q)[NE], const void *kv, const float *sc, long pos0, int n, const D1Rel &rel, Part (&st)[PW], auto done) {
    fold_keys(b, std::false_type{}, q, kv, sc, pos0, n, rel, st);
    if constexpr (WR > 1) {
      if (pg > 0) {
#pragma unroll
        for (int u = 0; u < PW; u++) {
          float *p = sPart + ((rw * (PARTS - PW) + (pg - 1) * PW + u) * (NE + 2)) * 64 + lane;
          p[0] = st[u].m;
          p[64] = st[u].l;
#pragma unroll
          for (int e = 0; e < NE; e++) p[(2 + e) * 64] = st[u].acc[e];
        }
      }
      __syncthreads();
    }
    if (pg == 0) {
      Part &t = st[0];
#pragma unroll
      for (int k = 1; k < PARTS; k++) {
        if (k < PW) {
          t.merge(st[k]);
        } else {
          const float *p = sPart + ((rw * (PARTS - PW) + k - PW) * (NE + 2)) * 64 + lane;
          Part o;
          o.m = p[0];
          o.l = p[64];
#pragma unroll
          for (int e = 0; e < NE; e++) o.acc[e] = p[(2 + e) * 64];
          t.merge(o);
        }
      }
      const float inv = (t.l > 0.f) ? 1.f / t.l : 0.f;
      float ctx[NE];
#pragma unroll
      for (int e = 0; e < NE; e++) ctx[e] = t.acc[e] * inv;
      done(ctx);
    }
    __syncthreads();
  };

  const int n_self = __builtin_amdgcn_readfirstlane(live ? a.n_keys : 0);
  const int n_cross = __builtin_amdgcn_readfirstlane(live ? a.len[rc] : 0);
  SelfBlock sb[2];
  CrossBlock cb[2];
  const long cross0 = (long)rc * a.cross_positions, self0 = (long)rc * a.self_positions;
  const int n_cached = n_self > 0 ? n_self - 1 : 0;
  float q[NE], z[NE], kx[NE], vx[NE];
  if constexpr (FOLD) {
    // ---- folded: start of the row, two attentions; the row stays in the registers of all its waves, each of which merges their partial
    // softmaxes for itself, so that an attention costs one exchange ----
    typedef std::integral_constant<bool, (AHEAD > 0)> Ahead;
    const int y = token.resolve(a, row0 + rw, pg == 0, lane, picked);
    if (row0 >= a.rows) return;  // rows that were kept to collect their last tokens
    typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
    const float *by_token = a.table.rows + (long)y * a.table.parts * D + lane * NE;
    const halfNE ev = *(const halfNE *)(a.sb.E + (long)y * D + lane * NE);
    d1_load<NE>(by_token, q);
    d1_load<NE>(by_token + D, kx);
    d1_load<NE>(by_token + (a.table.parts - 1) * D, vx);
    store_norms();
    __syncthreads();
    if constexpr (AHEAD == 2) {  // the first blocks of both caches travel with the table's rows
      first_block(sb[0], 0, a.self_kv, a.self_sc, self0, n_cached);
      first_block(cb[0], 0, a.cross_kv, a.cross_sc, cross0, n_cross);
    }
    {  // z = sqrt(d) E[y] + PE[t]; query, key and value by table (Dec1Table)
      float pv[NE];
      d1_load<NE>(sNorm + (VP + 3) * D + lane * NE, pv);
      const float sc = sqrtf((float)D);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < NE; e++) {
        z[e] = sc * (float)ev[e] + pv[e];
        s += z[e];
      }
      const float mean = wave_sum(s) / (float)D;
      float v = 0.f;
#pragma unroll
      for (int e = 0; e < NE; e++) v += ln_term(z[e] - mean, a.eps.l1);
      const float rs = ln_rscale(wave_sum(v) / (float)D, a.eps);
      auto combine = [&](float (&x)[NE], int which) {
        float p[NE], c[NE];
        d1_load<NE>(sNorm + (VP + which) * D + lane * NE, p);
        d1_load<NE>(sNorm + (VS + which) * D + lane * NE, c);
#pragma unroll
        for (int e = 0; e < NE; e++) x[e] = rs * (x[e] + p[e]) + c[e];
      };
      combine(q, 0);
      combine(kx, 1);
      combine(vx, 2);
    }
    if constexpr (AHEAD == 1) {
      __builtin_amdgcn_sched_barrier(0);
      first_block(sb[0], 0, a.self_kv, a.self_sc, self0, n_cached);
    }
    auto put_z = [&]() {
#pragma unroll
      for (int e = 0; e < NE; e += 4) *(float4 *)(sZ + rw * ZLD + lane * NE + e) = make_float4(z[e], z[e + 1], z[e + 2], z[e + 3]);
    };
    if (pg == 0) put_z();
    // A context into the residual stream.  The partial softmaxes of a row's waves meet in the LDS; each wave merges its share of the columns,
    // all with one set of weights (in the chain of pairwise merges in one wave, which the others waited for, a context took 1,000 clocks).
    auto add_context = [&](const Part &st, int which) {
      // (FOLD32: of the folded values of the cross cache nothing is left to do)
      auto added = [&](float z_, float ctx, float c, float b) {
        if (FOLD32) return which == 0 ? z_ + b + ctx * c : z_ + ctx;
        return z_ + (ctx * c + b);
      };
      const float *scale = sNorm + (VC + 2 * which) * D, *constant = scale + D;
      if constexpr (WR == 1) {
        float c[NE], b[NE];
        d1_load<NE>(sZ + rw * ZLD + lane * NE, z);
        d1_load<NE>(scale + lane * NE, c);
        d1_load<NE>(constant + lane * NE, b);
        const float inv = (st.l > 0.f) ? 1.f / st.l : 0.f;
#pragma unroll
        for (int e = 0; e < NE; e++) z[e] = added(z[e], st.acc[e] * inv, c[e], b[e]);
        put_z();
      } else {
        constexpr int CW = D / WR, CL = CW < 64 ? 1 : CW / 64;  // columns of a wave, of a lane
        float *base = sPart + rw * PARTS * (D + 2);
        float2 *ml = (float2 *)(base + PARTS * D);
#pragma unroll
        for (int e = 0; e < NE; e += 4)
          *(float4 *)(base + pg * D + lane * NE + e) = make_float4(st.acc[e], st.acc[e + 1], st.acc[e + 2], st.acc[e + 3]);
        if (lane == 0) ml[pg] = make_float2(st.m, st.l);
        __syncthreads();
        if (CW >= 64 || lane < CW) {
          const int col = pg * CW + lane * CL;
          float m[PARTS], l = 0.f, top = -INFINITY, ctx[CL] = {}, x[PARTS][CL];
#pragma unroll
          for (int k = 0; k < PARTS; k++) {
#pragma unroll
            for (int c = 0; c < CL; c++) x[k][c] = base[k * D + col + c];
          }
#pragma unroll
          for (int k = 0; k < PARTS; k++) m[k] = ml[k].x, top = fmaxf(top, m[k]);
#pragma unroll
          for (int k = 0; k < PARTS; k++) {
            const float w = m[k] == -INFINITY ? 0.f : __expf(m[k] - top);
            l += w * ml[k].y;
#pragma unroll
            for (int c = 0; c < CL; c++) ctx[c] += w * x[k][c];
          }
          const float inv = (l > 0.f) ? 1.f / l : 0.f;
          float *zc = sZ + rw * ZLD + col;
#pragma unroll
          for (int c = 0; c < CL; c++) zc[c] = added(zc[c], ctx[c] * inv, scale[col + c], constant[col + c]);
        }
        __syncthreads();
      }
    };
    // (z is in the LDS while keys are read: the registers are theirs)
    {
      Part st[1];
      st[0].clear();
      if (pg == 0 && n_self > 0) {  // the pair computed in this step: used as it is
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < NE; e++) s += q[e] * kx[e];
        st[0].m = wave_sum(s);
        st[0].l = 1.f;
#pragma unroll
        for (int e = 0; e < NE; e++) st[0].acc[e] = vx[e];
      }
      if (pg == WR - 1 && n_self > 0) {  // and appended in integer form, by the wave with the fewest other keys
        const long p = self0 + (n_self - 1);
        short *dst = (short *)a.self_kv + p * 2 * D;
        d1_quantize_store<NE>(kx, dst, a.self_sc + p * 2, lane);
        d1_quantize_store<NE>(vx, dst + D, a.self_sc + p * 2 + 1, lane);
      }
      if constexpr (AHEAD > 0) {  // the second blocks when the start no longer needs its registers
        __builtin_amdgcn_sched_barrier(0);
        first_block(sb[1], 1, a.self_kv, a.self_sc, self0, n_cached);
        if constexpr (AHEAD == 2) first_block(cb[1], 1, a.cross_kv, a.cross_sc, cross0, n_cross);
      }
      fold_keys(sb, Ahead{}, q, a.self_kv, a.self_sc, self0, n_cached, D1Rel{}, st);
      add_context(st[0], 0);
    }
    if constexpr (AHEAD == 1) {
      __builtin_amdgcn_sched_barrier(0);
      first_block(cb[0], 0, a.cross_kv, a.cross_sc, cross0, n_cross);
      first_block(cb[1], 1, a.cross_kv, a.cross_sc, cross0, n_cross);
    }
    // ---- cross-attention: the normalised row is the query ----
    normalise(LN2, q);
    if (FFN && EARLY) preload(a.W1);
    Part st[1];
    st[0].clear();
    fold_keys(cb, Ahead{}, q, a.cross_kv, a.cross_sc, cross0, n_cross, D1Rel{}, st);
    if (FFN && !EARLY) preload(a.W1);
    add_context(st[0], 1);
    if constexpr (FFN) {
      if (pg == 0) {
        normalise(LN3, q);
        store_planes(q);
      }
    }
  } else {
  // ---- self-attention ----
  if (EARLY) preload(a.Wo_self);
  if (a.table.rows) {
    const int y = token.resolve(a, row0 + rw, pg == 0, lane, picked);
    if (row0 >= a.rows) return;  // rows that were kept to collect their last tokens
    first_layer_start<NE>(a, y, lane, pg == 0, q, z, kx, vx);
  } else {
    d1_load<NE>(a.q + (long)r * D + lane * NE, q);
    if (pg == 0) {
      d1_load<NE>(a.z + (long)r * D + lane * NE, z);
      d1_load<NE>(a.kv_new + (long)r * 2 * D + lane * NE, kx);
      d1_load<NE>(a.kv_new + (long)r * 2 * D + D + lane * NE, vx);
    }
  }
  store_norms();
  if (pg == 0) {  // (z, kx, vx: the row's first wave)
#pragma unroll
    for (int e = 0; e < NE; e += 4) *(float4 *)(sZ + rw * ZLD + lane * NE + e) = make_float4(z[e], z[e + 1], z[e + 2], z[e + 3]);
  }
  D1Rel rel;
  if constexpr (HEADS) {
    if (a.rk) {  // this row's query against the relative keys it can meet (distances -clip .. 0), shared by the row's waves
      rel.p = sRel + rw * (D1_MAX_CLIP + 1) * 8 + (lane >> 3), rel.clip = a.clip, rel.t = n_self - 1;
      for (int o = pg; o <= a.clip; o += WR) {
        float k[NE], s = 0.f;
        d1_load<NE>(a.rk + o * 64 + (lane & 7) * 8, k);
#pragma unroll
        for (int e = 0; e < NE; e++) s += q[e] * k[e];
        s = d1_head_sum(s);
        if ((lane & 7) == 0) sRel[rw * (D1_MAX_CLIP + 1) * 8 + o * 8 + (lane >> 3)] = s;
      }
      __syncthreads();
    }
  }
  {
    Part st[PW];
#pragma unroll
    for (int u = 0; u < PW; u++) st[u].clear();
    if (pg == 0 && n_self > 0) {  // the pair computed in this step: used as it is, and appended in integer form
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < NE; e++) s += q[e] * kx[e];
      st[0].m = HEADS ? d1_head_sum(s) + (rel.p ? rel.at(rel.t) : 0.f) : wave_sum(s);
      st[0].l = 1.f;
#pragma unroll
      for (int e = 0; e < NE; e++) st[0].acc[e] = vx[e];
      const long p = self0 + (n_self - 1);
      if constexpr (HEADS) {
        float *dst = (float *)a.self_kv + p * 2 * D + lane * NE;
#pragma unroll
        for (int e = 0; e < NE; e += 4) {
          *(float4 *)(dst + e) = make_float4(kx[e], kx[e + 1], kx[e + 2], kx[e + 3]);
          *(float4 *)(dst + D + e) = make_float4(vx[e], vx[e + 1], vx[e + 2], vx[e + 3]);
        }
      } else {
        short *dst = (short *)a.self_kv + p * 2 * D;
        d1_quantize_store<NE>(kx, dst, a.self_sc + p * 2, lane);
        d1_quantize_store<NE>(vx, dst + D, a.self_sc + p * 2 + 1, lane);
      }
    }
    attend(sb, q, a.self_kv, a.self_sc, self0, n_cached, rel, st, store_planes);
  }
  // ---- output projection + residual, LayerNorm, cross-attention query ----
  if (!EARLY) preload(a.Wo_self);
  request_bias(a.bo_self);
  project(a.Wo_self, sA);
  preload(a.Wq);
  add_residual();
  __syncthreads();
  {
    float y[NE];
    normalise(LN2, y);
    if (pg == 0) store_planes(y);
  }
  __syncthreads();
  request_bias(a.bq);
  project(a.Wq, sA);
  if (EARLY) preload(a.Wo_cross);
  {
    results([&](int i, int n, float x) { sQ[i * ZLD + n] = (x + bias[(n - n0) >> 4]) * a.q_scale; });
  }
  __syncthreads();
  // ---- cross-attention, output projection + residual ----
  {
    Part st[PW];
#pragma unroll
    for (int u = 0; u < PW; u++) st[u].clear();
    d1_load<NE>(sQ + rw * ZLD + lane * NE, q);
    attend(cb, q, a.cross_kv, a.cross_sc, cross0, n_cross, D1Rel{}, st, store_planes);
  }
  if (!EARLY) preload(a.Wo_cross);
  request_bias(a.bo_cross);
  project(a.Wo_cross, sA);
  if (FFN) preload(a.W1);
  add_residual();
  __syncthreads();
  if constexpr (FFN) {
    float y[NE];
    normalise(LN3, y);
    if (pg == 0) store_planes(y);
  }
  }
  if constexpr (FFN) {
    __syncthreads();
    request_bias(a.b1);
    project(a.W1, sA);
    preload(a.W2);
    results([&](int i, int n, float x) {
      const float u = as_f32(fmaxf(x + bias[(n - n0) >> 4], 0.f));
      const _Float16 hi = (_Float16)u;
      sU[i * LD + n] = hi;
      sU[(RW + i) * LD + n] = (_Float16)(u - (float)hi);
    });
    __syncthreads();
    request_bias(a.b2);
    project(a.W2, sU);
    add_residual();
    __syncthreads();
  }
  // ---- the residual stream back, and / or the final hidden state as planes with the norm of the tail ----
  if (pg != 0 || !valid) return;
  d1_load<NE>(sZ + rw * ZLD + lane * NE, z);
  if (a.write_z) {
#pragma unroll
    for (int e = 0; e < NE; e += 4) *(float4 *)(a.z + (long)r * D + lane * NE + e) = make_float4(z[e], z[e + 1], z[e + 2], z[e + 3]);
  }
  if (a.h_hi) {
    typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
    unsigned int level[NE / 4];
    if (a.scout.codes) scout_levels<NE>(a.scout, lane, level);
    float (&y)[NE] = z;
    normalise_row(LNF, y);
    halfNE hi, lo;
    float tail2 = 0.f;
#pragma unroll
    for (int e = 0; e < NE; e++) {
      const float x = as_f32(y[e]);
      hi[e] = (_Float16)x;
      lo[e] = (_Float16)(x - (float)hi[e]);
      tail2 += (float)lo[e] * (float)lo[e];
    }
    tail2 = wave_sum(tail2);
    *(halfNE *)(a.h_hi + (long)r * D + lane * NE) = hi;
    *(halfNE *)(a.h_hi + a.h_lo_offset + (long)r * D + lane * NE) = lo;
    if (lane == 0) a.lo_norm[r] = sqrtf(tail2) * 1.0001f;  // rounded up: it is used as a bound
    if (a.scout.codes) scout_emit<NE>(y, level, a.scout, r, lane);
  }
}

template <int D, bool FFN, bool HEADS>
static hipError_t d1_launch(const Dec1Args &a, hipStream_t s) {
  // The form goes by shape_rows, never by what else is running or by a count the host happened to read: the forms differ in
  // the last bit (number of partial softmaxes, contraction of products and sums).
  // 1,024 rows and more: sixteen rows per workgroup.  With eight the launch alone is as fast (71 us at 1,900 rows), but
  // its 238 workgroups pull the matrices through twice as many CUs for the same rows; with 119 the other lanes' matrix
  // kernels get the rest of the chip and the job is 4 % faster (200,000 sentences: 560 against 582 ms).
  // Up to 512 rows two per workgroup (320 rows of 180 tokens alone: 24.4 against 26.7 ms with four), in between eight
  // (65,536 tokens: 550 against 554 ms with four).  Eight heads, whose keys are fp32: a CU pulls some 55 KB of them a us whatever is in
  // flight, so few rows are spread over more CUs: two per workgroup up to 192 rows (a step of the 30 + 6 layer teacher, 100 / 160 rows
  // alone: 320 / 326 us, with four 344 / 350; with 8 heads and FFN 2,048, 160 rows of 100 70 and 80), four up to 512 (teacher, 260 /
  // 320 rows 402 / 414 us, with eight 473 / 486; 300 / 500 rows with FFN 2,048 73.5 / 79.2 and 83.4 / 87.5).  Beside other lanes the CUs are not
  // idle: 2,048 sentences through the teacher 97.9 ms with these lines, 100.2 with 64 and 256, 98.9 with 256 and 512, 100.5 with 512 for
  // two; the model with FFN 2,048 takes the same time but for 1,023 in place of 512 (92 against 91 ms).
  const int shape = a.shape_rows > 0 ? a.shape_rows : a.rows;
  const int rows = a.table.rows && !a.tok_in ? std::max(a.rows, a.sb.rows_prev) : a.rows;  // those that only collect a token, too
#define NT_D1F(RW_, NW_, P_, F16_, F32_)                                                                                  \
  do {                                                                                                                   \
    const dim3 grid((unsigned)((rows + RW_ - 1) / RW_));                                                                 \
    if (a.origin) hipLaunchKernelGGL((dec1_kernel<D, RW_, NW_, P_, F16_, true, FFN, F32_, HEADS>), grid, dim3(64 * NW_), 0, s, a); \
    else hipLaunchKernelGGL((dec1_kernel<D, RW_, NW_, P_, F16_, false, FFN, F32_, HEADS>), grid, dim3(64 * NW_), 0, s, a);         \
  } while (0)
#define NT_D1(RW_, NW_, P_, F32_) NT_D1F(RW_, NW_, P_, 0, F32_)
  if constexpr (!HEADS) {
    if (a.folded == 2) {
      // Integer folded caches.  1,024 rows and more: a wave per row, sixteen rows per workgroup, which fills half of the chip's CUs and
      // leaves the other lanes' kernels the rest (2,000 rows of 27 tokens / 1,100 of 40 alone 40 / 39 us; four or eight rows of a wave each 34 /
      // 30 to 32, two rows of four waves 56 / 40; 200,000 sentences at 65,536 tokens 430 ms, 432 to 446 and 495).  Fewer rows: two waves each
      // (900 rows of 40, 620 of 55: 25 / 28 us, with four 31 / 31), and four as long as their workgroups, two to a CU at d = 512, are one round, that is up
      // to 512 rows (a step, four waves / two: 301 rows of 110 tokens 35.4 / 36.3, 400 36.7 / 38.4, 512 42.4 / 43.3, 513 49.6 / 45.1, of 22 tokens 35.7 /
      // 32.3; d = 256, more to a CU, 520 rows of 110 32.4 / 34.7, of 22 23.7 / 24.7).  With an FFN, whose matrices every workgroup pulls: sixteen rows,
      // four (900 rows of 40 / 560 of 60: 39 / 40 us, with eight 44 / 48, with two 52 / 56), two up to the same line (a step, two rows / four: 301 rows of 110
      // tokens 43.2 / 48.3, 400 46.6 / 50.3, 512 52.5 / 54.2, 513 71.3 / 56.0, of 22 tokens 56.3 / 44.2).
      constexpr int kOneRound = D == 512 ? 512 : 520;
      if constexpr (FFN) {
        if (shape >= 1024) NT_D1F(16, 16, 1, 1, false);
        else if (shape > kOneRound) NT_D1F(4, 16, 4, 1, false);
        else NT_D1F(2, 8, 4, 1, false);
      } else {
        if (shape >= 1024) NT_D1F(16, 16, 1, 1, false);
        else if (shape > kOneRound) NT_D1F(2, 4, 2, 1, false);
        else NT_D1F(1, 4, 4, 1, false);
      }
      return hipGetLastError();
    }
    if (a.folded) {
      // A row per workgroup, up to 256 rows, which is one round; more, two of them with four waves each (a step of 250 / 300 / 400 / 511 rows
      // alone: 31.8 / 40.3 / 41.9 / 45.3 us and 32.4 / 36.1 / 37.9 / 41.6).  Eight waves for a row up to 64 rows: 45 rows of 22 tokens 11.6
      // us with eight and 12.2 with four, 60 of 100 17.4 and 18.7; 100 rows of 30 11.2 both ways, 200 of 20 11.9 and 11.4, and beside other
      // lanes they cost more (a 4,096-token budget 19.5 against 18.8 ms).  Four for a row alone, which is mostly a short sentence: 22
      // tokens 9.5 us with eight and 9.3 with four (150: 15.3 and 16.5).
      if (FFN || shape > 256) NT_D1(2, 8, 4, true);
      else if constexpr (!FFN) {
        if (shape > 1 && shape <= 64) NT_D1(1, 8, 8, true);
        else NT_D1(1, 4, 4, true);
      }
      return hipGetLastError();
    }
  }
  if (shape >= 1024) {
    NT_D1(16, 16, 1, false);
  } else if (shape <= (HEADS ? 192 : 512)) {
    NT_D1(2, 8, 4, false);
  } else {
    if constexpr (HEADS) {
      if (shape <= 512) {
        NT_D1(4, 16, 4, false);
        return hipGetLastError();
      }
    }
    NT_D1(8, 16, 4, false);
  }
#undef NT_D1
#undef NT_D1F
  return hipGetLastError();
}

// The pick of the last step's arg-max inside the layer saves its launch: 400 rows of 30 tokens 2.76 -> 2.67 ms, 320 of 150 13.6 -> 13.2, 700 of 40
// 3.91 -> 3.82, 45 of 22 1.94 -> 1.89, with an FFN 300 / 700 rows of 30 2.65 -> 2.57 / 3.90 -> 3.74 (batches alone); 4,096- and
// 16,384-token budgets 18.4 -> 18.2 and 49.5 -> 46.2 ms.  Not where a row has one wave for it, nor with eight heads (the 30 + 6 layer teacher's
// batch of 250 rows 20.4 -> 20.6 ms: sixteen waves wait for four rows' picks in one layer of six; with a single eight-head layer it has not been tried).
bool dec1_picks(int shape_rows, int heads) { return heads <= 1 && shape_rows < 1024; }

hipError_t launch_dec1(const Dec1Args &a, int d, hipStream_t s) {
  if (a.rows <= 0) return hipSuccess;
  const bool ffn = a.W1 != nullptr;
  if (a.folded && !a.table.rows) return hipErrorInvalidValue;
  if (a.table.rows && a.sb.prev_cert == kPrevPick && (a.origin || a.tok_in || !dec1_picks(a.shape_rows > 0 ? a.shape_rows : a.rows, a.heads)))
    return hipErrorInvalidValue;
  if (a.heads > 1) {
    if (!dec1_heads_supported(d, a.heads) || ffn || a.folded || a.clip > D1_MAX_CLIP) return hipErrorInvalidValue;
    return d1_launch<512, false, true>(a, s);
  }
  if (d == 512) return ffn ? d1_launch<512, true, false>(a, s) : d1_launch<512, false, false>(a, s);
  if (d == 256) return ffn ? d1_launch<256, true, false>(a, s) : d1_launch<256, false, false>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace nt
