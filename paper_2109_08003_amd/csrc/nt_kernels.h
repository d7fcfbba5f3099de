// Internal launch interface between the host side of libnt and its gfx950 kernels.
// Every launcher validates nothing: the host code checks shapes before calling.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace nt {

// ---- GEMM: C[M,N] = A[M,K] * Wt[N,K]^T, fp16 MFMA with fp32 accumulation -------------
// Epilogue, applied to acc (fp32):  v = acc + bias[n];  if (n < scale_cols) v *= scale;
// if (relu) v = max(v,0);  if (resid) v += resid[m*ldr+n];  then columns [0,n_split) go to
// dst0[m*ld0+n] and columns [n_split,N) to dst1[m*ld1+(n-n_split)].
// Flavour of a layer normalisation y = gamma * (x - mean) * r + beta.  Vanilla: r = 1 / sqrt(var + eps) with the
// biased variance.  L1-norm (Sec. 3.1 "FP16 Inference"): r = 1 / (sqrt(pi/2) * mean|x - mean| + eps), the scaled
// mean absolute deviation, which equals the standard deviation for normally distributed activations.
struct LnEps {
  float eps = 0.f;
  int l1 = 0;
};
#ifdef __HIPCC__
// A computed value, as the fp32 number it is, before it is split into an fp16 head and the tail against it.  Left alone, the
// compiler folds the product that formed x into the conversion to fp16 where it can (v_fma_mixlo_f16: one rounding) and
// converts the rounded x where it packs two heads (v_cvt_pk_f16_f32).  Near the middle between two fp16 numbers (one value in
// 8,192) the two differ: the head that is stored or multiplied and the head that the tail was formed against are then one fp16
// step apart, and the pair is good to 2^-11 instead of 2^-22.
__device__ __forceinline__ float as_f32(float x) {
  asm("" : "+v"(x));
  return x;
}
// what a row sums over its centred elements, and how the mean of those terms becomes the scale r
__device__ __forceinline__ float ln_term(float c, int l1) { return l1 ? fabsf(c) : c * c; }
__device__ __forceinline__ float ln_rscale(float mean_term, LnEps e) {
  return e.l1 ? 1.0f / (1.2533141373f * mean_term + e.eps) : 1.0f / sqrtf(mean_term + e.eps);
}
#endif

struct GemmEpilogue {
  const float *bias = nullptr;
  float scale = 1.f;
  int scale_cols = 0;
  int relu = 0;
  const float *resid = nullptr;
  long ldr = 0;
  void *dst0 = nullptr;
  long ld0 = 0;
  int n_split = 0;  // set to N when there is a single destination
  void *dst1 = nullptr;
  long ld1 = 0;
  // streaming kernels with a head/tail A operand: only the strips of 64 output columns that start in
  // [tail_col0, tail_col1) multiply the tail plane too (the others see fp16 activations: half the MFMA work)
  int tail_col0 = 0, tail_col1 = 1 << 30;
  int first_f16 = 0;       // streaming kernels with fp32 destinations: the first destination is plain fp16 instead
  long dst_lo_offset = 0;  // fp16 destinations only: if != 0 the tail fp16(v - fp16(v)) is also stored, this many
                           // elements after the head (the result becomes a head/tail plane pair)
};

// How the A operand is given (see nt_gemm.hip): one fp16 plane, a head/tail pair of fp16 planes
// (~22 significant bits, two MFMA passes), or fp32 that the kernel splits while staging.
enum AMode { A_F16 = 0, A_PLANES = 1, A_F32 = 2 };

// a_mode: AMode; A_lo is the tail plane for A_PLANES (ignored otherwise).  c_f32: destinations are
// fp32, else fp16.  K must be a multiple of 64; lda in elements.
// Wp (optional): the same weights in MFMA fragment order (vocab_pack layout); with A_PLANES and a supported
// shape the streaming kernel is used, and tail = false then leaves the tail plane out of the product.
// shape_rows selects the kernel form (0: M), as in Dec1Args.
hipError_t launch_gemm(int a_mode, bool c_f32, const void *A, const void *A_lo, long lda, const _Float16 *Wt, int M,
                       int N, int K, const GemmEpilogue &e, hipStream_t s, const _Float16 *Wp = nullptr, bool tail = true,
                       int shape_rows = 0);

// Streaming form for K = 256 / 512 and N % 64 == 0 (nt_gemm_stream.hip): the A tile (head/tail planes) stays in
// the LDS, the weights stream through registers in fragment order.
struct GemmLayerNorm {
  const float *gamma = nullptr, *beta = nullptr;
  LnEps eps;
};
bool gemm_stream_supported(int N, int K);
// C = LayerNorm(X) * Wt^T: X [M][ldx] fp32 is normalised and split into planes while the tile is loaded
// The same with K = 1024 / 2048 (an FFN's second matrix), fp32 results: NC passes over a 512-wide tile of the planes,
// Wp = vocab_pack of Wt [N][K]; N a multiple of 512.
bool gemm_stream_k_supported(int N, int K);
hipError_t launch_gemm_stream_k(bool c_f32, const _Float16 *A, const _Float16 *A_lo, long lda, const _Float16 *Wp, int M,
                                int N, int K, const GemmEpilogue &e, hipStream_t s, bool tail = true, int shape_rows = 0);
// tail = false: only the head plane of A enters the product (fp16 activations: half the matrix-core work)
hipError_t launch_gemm_stream_ln(bool c_f32, const float *X, long ldx, const GemmLayerNorm &ln, const _Float16 *Wp, int M,
                                 int N, int K, const GemmEpilogue &e, hipStream_t s, bool tail = true);
hipError_t launch_gemm_stream(bool c_f32, const _Float16 *A, const _Float16 *A_lo, long lda, const _Float16 *Wp, int M,
                              int N, int K, const GemmEpilogue &e, hipStream_t s, bool tail = true);

// x [M][512] += relu(LayerNorm(x) W1^T + b1) W2^T + b2 in one launch; both matrices in fragment order, hidden width F.  A tile of 32 rows takes
// its workgroup 65 us at F = 2,048, so the line lies where two launches, which spread a tile over several, take as long: six layers with 8
// heads at 2,048 / 3,072 / 4,096 tokens 469 / 509 / 541 us with it and 418 / 562 / 625 without; 8,192, 16,384, 65,536: 832 / 1,535 / 6,079
// against 976 / 1,828 / 6,581.  Past a full round of 8,192 tokens, where a few workgroups take one tile more, the two launches have begun a
// round of theirs: 8,224 / 9,216 / 10,240 / 12,288 tokens 1,247 / 1,171 / 1,183 / 1,241 against 1,332 / 1,189 / 1,235 / 1,370; 16,416, 24,608,
// 32,800: 2,109 / 2,704 / 3,680 against 2,716 / 3,151 / 4,333.  F = 1,024 crosses at the same place: 2,048 / 2,560 / 3,072 tokens 361 / 383 / 403
// against 349 / 408 / 425; 8,224, 9,216, 10,240: 963 / 905 / 933 against 1,056 / 935 / 971; 16,416, 65,536: 1,659 / 4,552 against 2,040 / 4,891.
constexpr int kFfnMinRows = 2560;
bool gemm_ffn_supported(int M, int d, int F);  // and worth it
hipError_t launch_gemm_ffn(float *x, int M, int F, const GemmLayerNorm &ln, const _Float16 *W1p, const float *b1, const _Float16 *W2p, const float *b2,
                           hipStream_t s);

// The output projection of an attention and the LayerNorm + projection that follow it, one launch: x += A Wo^T + bias (rows of 512, in
// place), then as launch_gemm_stream_ln with both planes (e.tail_col0 .. tail_col1) over those rows.  Wp, Wo: vocab_pack order.
// The launch keeps the rows on the chip where two wrote and read them, 2 KB a row, and fill a tile twice; it stays bound by the phases
// of its workgroups that follow one another (context in, product, residual in, product with stores between its strips: at 65,536 tokens
// 275 us where the matrix cores need 110 at the clock they hold and the memory 137).  A tile is a workgroup's from end to end: up to
// kChainRows rows two launches, which spread one over several, are as fast.  Six layers, one head, no FFN, tokens as sentences
// of 25, 100 and 200: 2,500 / 3,075 / 4,000 (100) / 4,000 (200) tokens 323 / 324 / 432 / 625 us with it and 293 / 313 / 424 / 613
// without; 4,100, 5,000, 8,200, 16,375, 32,750, 65,525: 350, 367, 567, 825, 1,345, 2,402 against 371, 392, 612, 883, 1,424, 2,534.
struct GemmChain {
  const _Float16 *Wo = nullptr;
  const float *bias = nullptr;
  float *x = nullptr;
};
constexpr int kChainRows = 4096;
bool gemm_chain_supported(int M, int N, int K);  // and worth it
hipError_t launch_gemm_chain(const _Float16 *A, const _Float16 *A_lo, long lda, const GemmChain &ch, const GemmLayerNorm &ln, const _Float16 *Wp, int M,
                             int N, const GemmEpilogue &e, hipStream_t s);

// Decoder-step variant for small M (fp32 A and C): 32 x 32 tiles, whole-K operand panels loaded
// in one round trip.  If ln_g != nullptr the rows of A are LayerNorm-ed first (requires K to be
// the row width, 256 or 512).  K must be a multiple of 256.
bool skinny_gemm_supported(int K, bool with_ln);
hipError_t launch_skinny_gemm(const float *A, long lda, const _Float16 *Wt, int M, int N, int K, const float *ln_g,
                              const float *ln_b, LnEps ln_eps, const GemmEpilogue &e, hipStream_t s);

// ---- output projection fused with row arg-max ------------------------------------------
// For every row m < M: the largest of h[m,:] . W_out[v,:] over v < N, lowest v on ties, as packed
// keys.  Each workgroup reduces a range of the vocabulary; partial keys go to pk[m * n_partials + p].
//
// Key = (order-preserving bits of the fp32 logit) << 32 | (0xFFFFFFFF - v): the maximum key is the
// largest logit and, among equal logits, the lowest id.  Max over keys is associative and
// commutative, so the result does not depend on the tiling: deterministic without float atomics.
__device__ __forceinline__ unsigned long long argmax_key(float val, int v) {
  unsigned int b = __float_as_uint(val);
  b = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
  return ((unsigned long long)b << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned int)v);
}
__device__ __forceinline__ float key_value(unsigned long long key) {
  unsigned int b = (unsigned int)(key >> 32);
  b = (b & 0x80000000u) ? (b & 0x7FFFFFFFu) : ~b;
  return __uint_as_float(b);
}

// Reductions over a wave in the vector unit.  An exchange through the LDS unit (ds_bpermute, what __shfl_xor becomes) takes about 60
// clocks, six of them in a row make a sum, and a decoder row passes a dozen such chains one after the other; a v_permlane swap or a
// DPP operand takes a few.  The steps pair lanes as xor 32, 16, 8, 4, 2, 1 do (a rotation by 8 or 4 within 16 lanes is such a
// pairing once the larger steps are done), so the results are those of the exchanges, bit for bit.  One sentence 808 -> 726 us (of which
// about a third is the arg-max's 250 partial keys requested together), 45 sentences 2,508 -> 2,241, the 256-wide model 930 -> 832, a
// 4,096-token budget 21.7 -> 20.4 ms, 65,536 tokens 465 -> 461.
// wave_fold: all 64 lanes; wave_fold16: groups of 16.  op is commutative.
template <int CTRL>
__device__ __forceinline__ unsigned int wave_dpp(unsigned int x) {
  return (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
template <typename T, class Op>
__device__ __forceinline__ T wave_fold16(T x, Op op) {
  static_assert(sizeof(T) == 4, "");
  auto step = [&](T v, auto ctrl) { return op(v, __builtin_bit_cast(T, wave_dpp<decltype(ctrl)::value>(__builtin_bit_cast(unsigned int, v)))); };
  x = step(x, std::integral_constant<int, 0x128>{});  // row_ror 8, 4
  x = step(x, std::integral_constant<int, 0x124>{});
  x = step(x, std::integral_constant<int, 0x4E>{});   // quad_perm: lane ^ 2, lane ^ 1
  return step(x, std::integral_constant<int, 0xB1>{});
}
// x of this lane's half paired with y of the other half (halves: lanes 0-31, 32-63): the lower half gets op(x, x'), the upper
// op(y, y')
template <typename T, class Op>
__device__ __forceinline__ T wave_pair32(T x, T y, Op op) {
  const auto p = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned int, x), __builtin_bit_cast(unsigned int, y), false, false);
  return op(__builtin_bit_cast(T, (unsigned int)p[0]), __builtin_bit_cast(T, (unsigned int)p[1]));
}
template <typename T, class Op>
__device__ __forceinline__ T wave_pair16(T x, T y, Op op) {  // likewise with lanes 0-15 / 16-31 of each half
  const auto p = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned int, x), __builtin_bit_cast(unsigned int, y), false, false);
  return op(__builtin_bit_cast(T, (unsigned int)p[0]), __builtin_bit_cast(T, (unsigned int)p[1]));
}
template <typename T, class Op>
__device__ __forceinline__ T wave_fold(T x, Op op) {
  x = wave_pair32(x, x, op);
  x = wave_pair16(x, x, op);
  return wave_fold16(x, op);
}
struct WaveAdd { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; } };
struct WaveMax { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a > b ? a : b; }
                 __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct WaveMin { __device__ __forceinline__ float operator()(float a, float b) const { return fminf(a, b); } };
__device__ __forceinline__ float wave_sum(float v) { return wave_fold(v, WaveAdd{}); }
__device__ __forceinline__ float wave_max(float v) { return wave_fold(v, WaveMax{}); }
// the largest 64-bit key: the high words first, then the low words of those that have it
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long x) {
  const unsigned int hi = wave_fold((unsigned int)(x >> 32), WaveMax{});
  const unsigned int lo = wave_fold((unsigned int)(x >> 32) == hi ? (unsigned int)x : 0u, WaveMax{});
  return (unsigned long long)hi << 32 | lo;
}
__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long x, int mask) {
  unsigned int lo = (unsigned int)x, hi = (unsigned int)(x >> 32);
  lo = __shfl_xor(lo, mask, 64);
  hi = __shfl_xor(hi, mask, 64);
  return ((unsigned long long)hi << 32) | lo;
}

// The output matrix in two layouts: Wt [N][K] row-major, and Wp in MFMA fragment order (see
// vocab_pack_bytes / vocab_pack; built once at load time).  The streaming kernels need K = 256 or
// 512 (vocab_stream_supported); other widths, or force_tiled, take the tiled kernels on Wt.
struct VocabWeights {
  const _Float16 *Wt = nullptr;
  const _Float16 *Wp = nullptr;
  int N = 0, K = 0;
  bool force_tiled = false;
};
bool vocab_stream_supported(int K);
size_t vocab_pack_bytes(int N, int K);
// host: dst[vocab_pack_bytes] <- fragment order of Wt [N][K]
void vocab_pack(const _Float16 *Wt, int N, int K, _Float16 *dst);

// n_partials of the launch configuration used with M rows (exact: head + tail planes; certified: tiled kernels' head plane
// first, none in the scout's).
// wide: vocab_wide of a row count at least M.  Up to a tile of 32 rows, and, of up to 256 strips of 64 entries (one to a workgroup), more where strips
// times tiles are at most kVocabWideStrips, take a kernel of its own, more the scout, which is two launches (and whose sums run in another order, so a
// caller whose M depends on timing decides by a row count that does not, and nobody by what happens to be running).  A decoder step alone, us, d = 512,
// wide / scout, with strips x tiles: 1,000 entries, 33 rows (32) 12.3 / 20.2, 512 rows (256) 16.6 / 27.5; 4,000 entries, 128 rows (252) 13.2 / 21.5,
// 300 rows (630) 21.1 / 24.4, 512 rows (1,008) 26.1 / 26.4; 8,000 entries, 64 rows (250) 12.9 / 19.2, 160 rows (625) 19.5 / 20.2, 200 rows (875)
// 21.5 / 20.5.  d = 256: 4,000 entries, 300 rows (630) 14.6 / 19.0.  More than 256 strips, rows of 22 tokens, 17 / 24 / 32 rows and the scout from 33 rows on: eight
// heads 29.3 / 30.1 / 31.1 and 34.5 / 34.5 / 34.5, the EOS mode of one head 21.9 / 22.8 / 23.6 and 24.5, d = 256 18.5 / 18.9 / 19.3 and 20.2, with an FFN of the
// model's width 25.8 / 26.9 / 27.9 and 28.7.
// line: the largest row count that takes the wide kernel with more than 256 strips.
//  - kVocabWideRows for a batch that is alone (figures above).
//  - Alone, and the pick is no launch but part of the next step's only layer (DecodeCursor::prev_pick), without an FFN: kVocabFewRows, d = 256 kVocabFewRows256.
//    17 / 20 / 24 / 28 / 32 rows, 32,000 entries 15.7 / 16.0 / 16.3 / 16.7 / 17.1 and 15.7 / 15.9 / 16.0 / 16.4 / 16.5, 20,000 15.1 / 15.3 / 15.8 / 16.2 / 16.6 and 15.2 /
//    15.5 / 15.7 / 15.9 / 16.0, 16,500 14.8 / 15.2 / 15.6 / 16.0 / 16.4 and 14.8 / 15.1 / 15.2 / 15.3 / 15.3; d = 256, 32,000 entries, 20 / 24 / 28 / 32 rows 12.3 / 12.3 /
//    12.5 / 12.8 and 12.5 / 12.6 / 12.5 / 12.8, 16,500 12.0 / 12.1 / 12.4 / 12.6 and 12.3 / 12.2 / 12.2 / 12.2.  (Two decoder layers of 512, 18 / 24 / 28 / 32 rows 67.8 /
//    68.7 / 69.7 / 67.6 and 68.9 / 69.0 / 69.2 / 66.6; of 256, 28 rows 35.6 and 36.3: no line of their own.)
//  - A call with several batches, whose lanes share the memory system that one wide kernel fills: kVocabFewRows.  1,500 sentences in batches of at most 24 and 32
//    rows, wide against scout: the submitted student 30.7 against 24.0 and 25.0 against 18.8 ms, eight heads and FFN 2,048 47.3 against 42.2 and 37.7 against 33.1,
//    the 256-wide model (24 rows) 13.1 against 10.8; a 4,096-token budget of one head 17.9 with the line at 32 rows, 17.4 at 4 to 16.  In the EOS mode, which the
//    host paces, one launch less is worth more: 24 rows of one head 29.3 against 30.8 (37 against 43 in processes whose host is the slower), of the submitted
//    student 33.4 against 31.1 (39 against 42): the same line all the same, so that its tokens are those of the fixed-length call by construction.
constexpr int kVocabWideStrips = 640, kVocabWideRows = 32, kVocabFewRows = 16, kVocabFewRows256 = 24;
bool vocab_wide(const VocabWeights &w, int rows, int line);
int vocab_argmax_partials(const VocabWeights &w, int M, bool certified, bool wide);
// h is a head/tail pair of fp16 planes.
hipError_t launch_vocab_argmax(const _Float16 *h, const _Float16 *h_lo, long ldh, const VocabWeights &w, int M,
                               unsigned long long *pk, bool wide, hipStream_t s);

// Arg-max of many rows (nt_vocab_scout.hip): an 8-bit pass with a rigorous bound leaves a few candidates per row, which get
// exact logits.  K = 256 / 512.
struct VocabScout {
  const void *matrix;   // vocab_scout_build of the output matrix
  int8_t *codes;        // [rows][K] and
  float4 *row_consts;   // [rows]: written by the kernel that writes the hidden state (scout_emit)
  void *scratch;        // vocab_scout_scratch_bytes
};
size_t vocab_scout_bytes(int N, int K);
// dst [vocab_scout_bytes] <- W [N][K], gamma / beta [K]: the final normalisation, all on the device; returns when it is done (load time)
hipError_t vocab_scout_build(const _Float16 *W, int N, int K, const float *gamma, const float *beta, void *dst, hipStream_t s);
const int8_t *vocab_scout_levels(const void *matrix, int N, int K);  // within the packed matrix
size_t vocab_scout_scratch_bytes(int N, int rows);
// Where a hidden state goes besides its planes (codes == nullptr: nowhere), and the powers of two that level its columns
struct ScoutOut {
  int8_t *codes = nullptr;
  float4 *row_consts = nullptr;
  const int8_t *levels = nullptr;
};
#ifdef __HIPCC__
// An orthogonal matrix of signs, times the root of NE, on a lane's elements.  (The two signs in front: equal elements stay spread.)
template <int NE, typename T>
__device__ __forceinline__ void scout_mix(T (&x)[NE]) {
  static_assert(NE == 4 || NE == 8, "");
  x[3] = -x[3];
  if (NE == 8) x[6] = -x[6];
#pragma unroll
  for (int m = 1; m < NE; m *= 2)
#pragma unroll
    for (int e = 0; e < NE; e++)
      if (!(e & m)) {
        const T a = x[e], b = x[e | m];
        x[e] = a + b;
        x[e | m] = a - b;
      }
}
// the same where element lane & (NE - 1) of a group is this lane's
template <int NE>
__device__ __forceinline__ float scout_mix_lanes(float x, int lane) {
  auto step = [&](float v, float o, int m) { return lane & m ? o - v : v + o; };
  auto from = [](float v, auto ctrl) { return __uint_as_float(wave_dpp<decltype(ctrl)::value>(__float_as_uint(v))); };
  const int e = lane & (NE - 1);
  if (e == 3 || (NE == 8 && e == 6)) x = -x;
  x = step(x, from(x, std::integral_constant<int, 0xB1>{}), 1);  // quad_perm: lane ^ 1, lane ^ 2
  x = step(x, from(x, std::integral_constant<int, 0x4E>{}), 2);
  if (NE == 8)  // row_half_mirror, quad_perm: (lane ^ 7) ^ 3
    x = step(x, from(from(x, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{}), 4);
  return x;
}
// One levelled and mixed row, NE elements per lane of a wave: codes in [-127, 127] and {scale, ||y - scale code||, ||scale code||, 0}, the norms
// rounded up (they are bounds).
template <int NE>
__device__ __forceinline__ float4 scout_round(const float (&y)[NE], int (&code)[NE]) {
  float top = 0.f;
#pragma unroll
  for (int e = 0; e < NE; e++) top = fmaxf(top, fabsf(y[e]));
  top = wave_max(top);
  const float scale = top > 0.f ? top / 127.f : 1.f, inv = 1.f / scale;
  float e2 = 0.f, a2 = 0.f;
#pragma unroll
  for (int e = 0; e < NE; e++) {
    const float c = fminf(fmaxf(rintf(y[e] * inv), -127.f), 127.f), a = c * scale;
    code[e] = (int)c;
    e2 += (y[e] - a) * (y[e] - a);
    a2 += a * a;
  }
  e2 = wave_sum(e2);
  a2 = wave_sum(a2);
  return make_float4(scale, sqrtf(e2) * 1.001f, sqrtf(a2) * 1.0001f, 0.f);
}
// the same for a row whose lanes hold consecutive elements; level: theirs, four to a word
template <int NE>
__device__ __forceinline__ void scout_emit(const float (&y)[NE], const unsigned int (&level)[NE / 4], const ScoutOut &o, long row, int lane) {
  int code[NE];
  float x[NE];
#pragma unroll
  for (int e = 0; e < NE; e++) x[e] = ldexpf(y[e], (int)(int8_t)(level[e / 4] >> (e % 4 * 8)));
  scout_mix<NE>(x);
  const float4 rc = scout_round<NE>(x, code);
#pragma unroll
  for (int e = 0; e < NE; e += 4)
    *(unsigned int *)(o.codes + row * (NE * 64) + lane * NE + e) =
        (code[e] & 0xFF) | (code[e + 1] & 0xFF) << 8 | (code[e + 2] & 0xFF) << 16 | (unsigned int)code[e + 3] << 24;
  if (lane == 0) o.row_consts[row] = rc;
}
template <int NE>
__device__ __forceinline__ void scout_levels(const ScoutOut &o, int lane, unsigned int (&level)[NE / 4]) {
#pragma unroll
  for (int w = 0; w < NE / 4; w++) level[w] = ((const unsigned int *)(o.levels + lane * NE))[w];
}
#endif
// What the second half, the pick, reads (nt_pick.h)
struct PickArgs {
  const void *part;            // the scout's groups
  const float4 *row_consts, *strip_consts;
  const int32_t *ids;
  int NS, row0;
  float distrust;
  const _Float16 *h_hi, *h_lo; // the states
  long ldh;
  const _Float16 *Ws;          // the matrix in the scout's order
};
// Results: tok[m], and slot_of_row[m] = -1.  distrust: every row has every logit computed.  later: only the scout runs; the first decoder
// layer of the next step picks (StepBeginArgs::pick), which takes rows that are one launch.
bool vocab_scout_one_launch(int N, int rows);
hipError_t launch_vocab_scout(const VocabScout &v, const _Float16 *h, const _Float16 *h_lo, long ldh, const VocabWeights &w, int M,
                              bool distrust, int32_t *tok, int32_t *slot_of_row, PickArgs *later, hipStream_t s);

// Same result as launch_vocab_argmax for many rows, usually at less work: the scout above, or (tiled kernels) a head-only
// pass whose winner is certified against a rigorous bound on the contribution of the tail (lo_norm[m] = ||tail of row m||,
// w_norm_max = max_v ||W_out[v,:]||); rows that cannot be certified are recomputed with both planes.
// Results: tok[m] when slot_of_row[m] < 0, else the key in final_key[slot_of_row[m]].
// *count must be 0 when the call starts (the start of the step clears it).  list [M]: scratch of the recompute.
bool vocab_tiled(const VocabWeights &w);               // only the tiled kernels fit (or are forced)
bool vocab_scouted(const VocabWeights &w, bool wide);  // the scout is the kernel for this choice
hipError_t launch_vocab_argmax_certified(const VocabScout &v, const _Float16 *h, const _Float16 *h_lo, long ldh,
                                         const VocabWeights &w, int M, const float *lo_norm, float w_norm_max,
                                         unsigned long long *pk, float *ps, int32_t *tok, int32_t *slot_of_row, int32_t *list,
                                         int32_t *count, unsigned long long *final_key, PickArgs *later, hipStream_t s);

// the tiled implementations (nt_gemm.hip) and their certification kernel
int vocab_argmax_partials_tiled(int M, int N);
hipError_t launch_vocab_argmax_tiled(const _Float16 *h, const _Float16 *h_lo, long ldh, const _Float16 *Wt, int M, int N,
                                     int K, unsigned long long *pk, hipStream_t s);
hipError_t launch_vocab_argmax_certified_tiled(const _Float16 *h, const _Float16 *h_lo, long ldh, const _Float16 *Wt, int M,
                                               int N, int K, const float *lo_norm, float w_norm_max,
                                               unsigned long long *pk, float *ps, int32_t *tok, int32_t *slot_of_row,
                                               int32_t *list, int32_t *count, unsigned long long *final_key, hipStream_t s);
hipError_t launch_argmax_select(const unsigned long long *pk, const float *ps, int n_partials, int M, const float *lo_norm,
                                float w_norm_max, int32_t *tok, int32_t *slot_of_row, int32_t *list, int32_t *count,
                                unsigned long long *final_key, hipStream_t s);

// ---- 8-bit output layer fused with the row arg-max (nt_vocab_q8.hip; Sec. 3.2, Eq. 3-6) ----------------------------
bool vocab_q8_supported(int K);
size_t vocab_q8_pack_bytes(int N, int K);
size_t vocab_q8_const_bytes(int N);
// Host: quantise Wt [N][K] per vocabulary entry and lay the codes out in MFMA fragment order, the per-entry
// constants (scale, zero point, sum of codes - K * zero point) in accumulator order.
void vocab_q8_pack(const _Float16 *Wt, int N, int K, int8_t *codes, void *consts);
// Host: Eq. 3, 4 for one vocabulary entry (what vocab_q8_pack applies to every row)
void vocab_q8_quantize_row(const _Float16 *w, int K, int8_t *q, float *scale, int32_t *zero);
// x [M][d] fp32 -> [LayerNorm if gamma != nullptr ->] unsigned 8-bit codes per row, stored as signed bytes
// (code - 128) in codes [M][d]; a_scale [M]; c [M] = 128 - zero point; sa [M] = sum of the signed bytes.  d = 256 / 512.
hipError_t launch_q8_rows(const float *x, int M, int d, const float *gamma, const float *beta, LnEps eps, int8_t *codes,
                          float *a_scale, int32_t *c_out, int32_t *sa_out, hipStream_t s);
// partial keys per row that launch_vocab_q8_argmax writes for M rows
int vocab_q8_partials(int M);
// pk[m * vocab_q8_partials(M) + p]: largest b_scale[v] * float(I[m][v]) of a range of the vocabulary, as packed keys
hipError_t launch_vocab_q8_argmax(const int8_t *codes, const int32_t *c_row, const int32_t *sa_row, int M,
                                  const int8_t *Wq, const void *consts, int N, int K, unsigned long long *pk,
                                  hipStream_t s);
// logits[m * ld + v] = a_scale[m] * (b_scale[v] * float(I[m][v])) by the definition (debug / teacher-forced path)
hipError_t launch_q8_logits(const int8_t *codes, const float *a_scale, const int32_t *c_row, int M, const int8_t *Wq,
                            const void *consts, int N, int K, float *logits, long ld, hipStream_t s);

// ---- row kernels --------------------------------------------------------------------
// x[r,:] = sqrt(d) * E[id] + PE[pos]; rows r = b*S + s, pos = s.  Out-of-range ids are
// replaced by pad_id and flags[0] is set.  Also clamps len into [1,S] -> len_out.
hipError_t launch_embed_src(const int32_t *src, const int32_t *len, int32_t *len_out, int B, int S, int d, int vocab,
                            int pad_id, const _Float16 *E, const float *pe, float *x, int32_t *flags, hipStream_t s);

// out = gamma * (x - mean) * r + beta per row of d, r as LnEps says.
enum OutMode { OUT_F16 = 0, OUT_F32 = 1, OUT_PLANES = 2 };  // OUT_PLANES: fp16 head at out, tail at out + lo_offset
// lo_norm (OUT_PLANES only, optional): receives the Euclidean norm of every row's tail plane.  scout (OUT_PLANES, d = 256 / 512).
hipError_t launch_layer_norm(const float *x, int M, int d, const float *gamma, const float *beta, LnEps eps,
                             void *out, int out_mode, long lo_offset, hipStream_t s, float *lo_norm = nullptr, ScoutOut scout = ScoutOut());

// out[i] = hi[i] + lo[i] (debug readback of a head/tail plane pair)
hipError_t launch_planes_to_float(const _Float16 *hi, const _Float16 *lo, float *out, long n, hipStream_t s);

// fp16 -> fp32 copy (debug readback)
hipError_t launch_half_to_float(const _Float16 *in, float *out, long n, hipStream_t s);
hipError_t launch_fill_i32(int32_t *p, long n, int32_t v, hipStream_t s);
// one wave that busy-waits for `ticks` periods of the 100 MHz wall clock (bounded); sink is never written
hipError_t launch_spin(long ticks, int *sink, hipStream_t s);

// Probes: `blocks` workgroups of four waves, each wave `iters` x 4 independent 32x32x16 fp16 MFMAs (2 * 32 * 32 * 16
// flops each); a grid-stride read of `bytes` bytes (a multiple of 16).  sink is never written.
// workgroups of eight waves, iters (a multiple of 8) rounds of eight independent 32x32x16 fp16 MFMAs per wave
hipError_t launch_probe_mfma(int iters, int blocks, bool random_operands, float *sink, hipStream_t s);
hipError_t launch_probe_read(const void *src, long bytes, float *sink, hipStream_t s);
// reads bytes of buf and writes them back in place (the contents do not change)
hipError_t launch_probe_copy(void *buf, long bytes, hipStream_t s);

// Start of decoder step t for rows [0, rows_prev): (1) if t > 0, reduce the arg-max partials of
// step t-1 and store the token in out[r*out_ld + t-1]; (2) for rows < rows_now: take the input
// token (BOS at t = 0, forced[r*forced_ld + t] if forced, else the token just reduced),
// z = sqrt(d) * E[y] + PE[t], and a = LayerNorm(z) unless a == nullptr.
struct StepBeginArgs {
  int t, rows_prev, rows_now, d, vocab, bos_id, pad_id;
  const unsigned long long *pk;
  int n_partials;
  int32_t *out;
  long out_ld;
  const int32_t *forced;
  long forced_ld;
  const _Float16 *E;
  const float *pe;
  const float *gamma, *beta;
  LnEps eps;
  float *z, *a;
  int32_t *flags;
  // certified arg-max of the previous step (prev_cert != 0): token = tok[r], or the key in
  // final_key[slot_of_row[r]] when the row had to be recomputed; cert_count is cleared for this step
  // prev_cert == kPrevPick: the token is picked here (first decoder layer in one launch, dec1_picks)
  int prev_cert;
  const int32_t *tok, *slot_of_row;
  const unsigned long long *final_key;
  int32_t *cert_count;
  PickArgs pick;
};
constexpr int kPrevPick = 2;
hipError_t launch_step_begin(const StepBeginArgs &a, hipStream_t s);

// ---- fused decoder-step kernels (nt_decoder.hip), model widths 256 / 512 ----------------------------------------
bool dec_fused_supported(int K);
// Step start fused into the first layer's self-attention projection: tokens as launch_step_begin takes them (or
// tok_in[r] directly when tok_in != nullptr: the EOS mode's dense rows), z = sqrt(d) * E[y] + PE[t] written to sb.z,
// LayerNorm (sb.gamma, sb.beta), then [q|k|v] = a * Wp^T with epilogue e (N columns; Wp in MFMA fragment order).
// sb.a is ignored.  Rows in [rows_now, rows_prev) only have their token collected.
struct DecQkvArgs {
  StepBeginArgs sb;
  const int32_t *tok_in;
  const _Float16 *Wp;
  int N;
  GemmEpilogue e;
  int shape_rows;  // row count that selects the kernel form (0: rows_now), as in Dec1Args
};
hipError_t launch_dec_qkv(const DecQkvArgs &a, hipStream_t s);
// One launch for: z' = A * W1^T + b1 + z (A: head/tail planes [M][lda], W1 [K][K] in fragment order; z' is written
// back to z if write_z), y = LayerNorm(z'), then either (W2p == nullptr) y as head/tail planes at h_hi /
// h_hi + h_lo_offset with row stride K, plus lo_norm[m] = ||tail|| (optional), or C = y * W2^T with epilogue e2
// (N2 columns, fp32 or fp16 destinations).
struct DecChainArgs {
  const _Float16 *A_hi, *A_lo;
  long lda;
  const _Float16 *W1p;
  const float *b1;
  float *z;
  long ldz;
  int write_z;
  int M;
  const float *gamma, *beta;
  LnEps eps;
  _Float16 *h_hi;
  long h_lo_offset;
  float *lo_norm;
  ScoutOut scout;
  const _Float16 *W2p;
  int N2;
  GemmEpilogue e2;
};
hipError_t launch_dec_chain(const DecChainArgs &a, int K, bool c2_f32, hipStream_t s);

// Start of decoder step t when sentences end at EOS (Sec. 3.3 "Greedy Search"): the rows still decoding are kept
// as a dense prefix.  Dense row r of a step belongs to batch row origin[r] (-1: no row; such rows compute on the
// padding token and store nothing).  Three launches:
//   collect  (t > 0) token of step t-1 for every previous dense row -> out[b][t-1]; a row ends when the token is
//            eos_id or when it has cap[b] tokens, and then gets out_len[b] = t
//   compact  stable compaction of the rows that go on -> origin / tok_in of step t, their count -> *live and, if
//            progress != nullptr, progress_tag | t << 32 | count into that host-visible word.  At t == 0 the rows
//            with cap > 0 start with bos_id.
//   embed    z[r] = sqrt(d) * E[tok_in[r]] + PE[t] for r < rows_now (tok_in is pad_id where origin[r] < 0)
// rows_prev: dense rows of step t-1 (B at t == 0); rows_now <= rows_prev: dense rows step t will run on, an upper
// bound of the count the compaction finds.
struct EosStepArgs {
  int t, rows_prev, rows_now, d, vocab, bos_id, pad_id, eos_id;
  // arg-max result of step t-1, as in StepBeginArgs
  const unsigned long long *pk;
  int n_partials, prev_cert;
  const int32_t *tok, *slot_of_row;
  const unsigned long long *final_key;
  int32_t *cert_count;
  int32_t *out;
  long out_ld;
  int32_t *out_len;
  const int32_t *cap;          // [B] most tokens of each batch row
  const int32_t *origin_prev;  // [rows_prev] of step t-1 (unused at t == 0)
  int32_t *origin;             // [rows_prev] of step t
  int32_t *y;                  // [rows_prev] scratch: token of a previous dense row that goes on, else -1
  int32_t *tok_in;             // [rows_prev] input token of each dense row of step t
  int32_t *live;
  unsigned long long *progress;
  unsigned long long progress_tag;
  const _Float16 *E;
  const float *pe;
  float *z;
  int skip_embed;              // != 0: no embedding launch (the first projection of the step embeds tok_in itself)
};
hipError_t launch_eos_step_begin(const EosStepArgs &a, hipStream_t s);

// ---- attention ------------------------------------------------------------------------
// Encoder self-attention on a padded batch.  qkv [B*S, 3d] (q already scaled | k | v), len [B];
// ctx [B*S, d].  f32: qkv is fp32 (split-precision MFMA inside) and ctx is written as a head/tail
// pair of fp16 planes (tail ctx_lo_offset elements after the head); else both are fp16.  Keys >=
// len get weight exactly 0; query rows >= len get 0.  rk: optional relative keys [2*clip+1, dh].
hipError_t launch_enc_attention(const void *qkv, bool f32, const int32_t *len, void *ctx, long ctx_lo_offset, int B,
                                int S, int d, int heads, const float *rk, int clip, hipStream_t s);
// The register-resident form with the scaled query and the key as plain fp16 (qk [B*S, 2d]: q | k) and the value as
// fp32 (v [B*S, d]); sentences of at most 128 tokens, no relative keys (enc_attention_qk16_supported).  Scores then
// take one MFMA per product instead of three; probabilities, values and the context keep head + tail.
bool enc_attention_qk16_supported(int S, int d, int heads, const float *rk);
hipError_t launch_enc_attention_qk16(const _Float16 *qk, const float *v, const int32_t *len, void *ctx, long ctx_lo_offset,
                                     int B, int S, int d, int heads, hipStream_t s);

// Single-query attention against a cache, one query per (row, head).
//   q [rows, d] fp32 (scaled); ctx [rows, d] fp32.
//   cache row r: kv + r*row_stride elements, position j at + j*2d: k[d] then v[d].
//   n_keys: fixed count (self-attention: t+1) when len == nullptr, else len[r] (cross).
//   kv_f32 selects fp32 or fp16 cache elements.
//   rk (self only): relative keys; the query sits at position qpos, key j at position j.
//   ctx_lo_offset != 0: ctx is written as a head/tail pair of fp16 planes instead (head at ctx, tail that many
//   elements later).
//   origin (optional): query row r uses cache row (and len entry) origin[r]; origin[r] < 0 gives a zero context.
//   kv_new (optional, fp32 caches with a fixed key count only): [rows, 2d], the key and value of position
//   n_keys-1 of every query row; they are used from there and stored into the cache by this kernel.
hipError_t launch_attn_decode(const float *q, const void *kv, bool kv_f32, long row_stride, const int32_t *len,
                              int n_keys, int rows, int d, int heads, const float *rk, int clip, int qpos,
                              float *ctx, hipStream_t s, long ctx_lo_offset = 0, const int32_t *origin = nullptr,
                              const float *kv_new = nullptr);

// ---- attention half of a decoder layer, d = 256 / 512 (nt_dec1.hip) ---------------------------------------------------
// Several heads (dec1_heads_supported): fp32 self cache, fp16 cross cache, laid out as for launch_attn_decode; optional
// relative keys.  One head, no relative keys (attn_i16_supported): both caches hold 16-bit integers with one fp32 scale per vector.  Cache row c, position p: key codes at
// kv + ((c * positions + p) * 2) * d, value codes d elements later; their scales at sc[(c * positions + p) * 2] and
// [... + 1] (value = code * scale).
bool attn_i16_supported(int d, int heads, int clip);
bool dec1_heads_supported(int d, int heads);
// The first layer's Q | K | V projection depends on the input token y and the position t alone, and LayerNorm is affine in
// the row once its scale r is known: with c(v) = v - mean(v),
//   q|k|v = r (sqrt(d) (gamma c(E[y])) W + (gamma c(PE[t])) W) + (beta W + b).
// The three products are formed at load, in double, and kept in fp32: rows 0 .. vocab - 1 by token, then max_len rows by
// position, then beta W + b.  A row has `parts` groups of d columns: scaled query, key, value, and, last, for folded batches the
// value multiplied by the output matrix with its columns scaled (three where all batches are folded, or none; else four).
struct Dec1Table {
  const float *rows;  // nullptr: no table
  int parts, max_len;
};
size_t dec1_table_bytes(int vocab, int max_len, int d, int parts);
// B [d][parts * d] and bias [parts * d] in double on the device
hipError_t launch_dec1_table(const _Float16 *E, const float *pe, const float *gamma, const float *beta, const double *B,
                             const double *bias, int vocab, int max_len, int d, int parts, float *rows, hipStream_t s);
struct Dec1Args {
  // first layer (table.rows != nullptr): the launch is the start of the step as launch_dec_qkv has it - the previous step's
  // tokens are collected, rows beyond `rows` only for that, z is computed here - and q, kv_new are not read
  Dec1Table table;
  StepBeginArgs sb;        // gamma / beta / a / rows_now unused
  const int32_t *tok_in;   // EOS mode: tokens of the dense rows
  int heads;             // 0 / 1: one head
  const float *rk;       // several heads: relative keys [2 clip + 1][64], or nullptr
  int clip;
  int rows;
  int shape_rows;        // row count that selects the kernel form (0: rows).  The forms differ in the last bit, so a
                         // caller whose row count depends on timing passes one that does not
  const int32_t *origin; // optional: row r uses cache row origin[r] (< 0: zero context)
  LnEps eps;
  float *z;              // [rows, d] residual stream; written back if write_z
  int write_z;
  // self-attention: scaled query and this step's key | value pair (fp32), appended to the cache at position n_keys - 1
  const float *q, *kv_new;
  void *self_kv;
  float *self_sc;
  long self_positions;
  int n_keys;
  // output projection, LayerNorm, cross-attention query (matrices in fragment order)
  const _Float16 *Wo_self, *Wq, *Wo_cross;
  const float *bo_self, *bq, *bo_cross;
  float q_scale;
  GemmLayerNorm ln2;
  const void *cross_kv;  // integers with scales in cross_sc, or (folded == 1) fp32 [position][2 d] with one constant per key in
  const float *cross_sc; // cross_sc: keys multiplied by the query matrix and scale, values by the output matrix (+ bias)
  // folded: the self values then are already multiplied by the output matrix, too, column j divided by a scale; the whole constant of the
  // self context is b_v W_o + b_o.  Neither a bias nor the columns' different sizes may enter the cache: its integers have one scale per
  // vector, which the largest element sets for all.
  // folded == 2: the cross cache as integers of the products (CrossFold; {key scale, value scale, key's constant, unused} per
  // position in cross_sc).
  // What a row's start and its contexts need besides the row, one behind the other as a workgroup stages it (dec1_fold_vectors):
  // fold_const: gain and offset before the cross-attention, [before the FFN,] of the final normalisation; scale and constant of the self
  // context, of the cross context (folded == 2); the table's constants of query, key and value.
  // fold_pos [position][4]: the table's query, key and value of a position, and the embedding's offset
  int folded;
  const float *fold_const, *fold_pos;
  long cross_positions;
  const int32_t *len;    // keys of each cache row
  // FFN of width d (W1 == nullptr: none, or not part of this launch)
  GemmLayerNorm ln3;
  const _Float16 *W1, *W2;
  const float *b1, *b2;
  // final hidden state: LayerNorm as head / tail planes and the norm of the tail (h_hi == nullptr: not wanted)
  GemmLayerNorm lnf;
  _Float16 *h_hi;
  long h_lo_offset;
  float *lo_norm;
  ScoutOut scout;
};
hipError_t launch_dec1(const Dec1Args &a, int d, hipStream_t s);
// dst [dec1_fold_vectors_bytes] <- the above, at load: constants (of folded == 1, then of folded == 2 where gamma2 is given), then positions
struct Dec1FoldVectors {
  GemmLayerNorm ln2, ln3, lnf;         // ln3.gamma == nullptr: no FFN inside the layer
  const float *fold_scale, *fold_bias; // of the self context
  const float *gamma2, *beta2, *cross_scale, *cross_const;  // folded == 2 (gamma2 == nullptr: not used)
  const float *pe;
  Dec1Table table;
  int vocab;
};
size_t dec1_fold_vectors_bytes(int d, int max_len);
hipError_t launch_dec1_fold_vectors(const Dec1FoldVectors &v, int d, float *dst, hipStream_t s);
const float *dec1_fold_const(const float *vectors, int d, int folded);
const float *dec1_fold_pos(const float *vectors, int d);
// whether the layer's form for so many rows takes the pick of the previous step's arg-max into its start
bool dec1_picks(int shape_rows, int heads);
constexpr int kDec1FoldRows = 512, kDec1FoldTokens = 32768;
// What larger batches of one-layer one-head decoders fold (nt_cross_fold.hip): the encoder's final normalisation without gain and offset
// times [gain (Wk Wq^T) | gain (Wv Wo)], each column divided by its size, and what that leaves for the decoder.
struct CrossFold {
  const _Float16 *W;                      // the matrix as head and tail planes in fragment order
  const float *u;                         // [d]: a key's constant is its row . u
  const float *gamma2, *beta2;            // [d]: normalisation before the cross-attention, times the key columns' sizes
  const float *value_scale, *value_const; // [d]: sizes of the value columns; b_v Wo + b_o with the encoder's offset in it
};
size_t cross_fold_bytes(int d);
CrossFold cross_fold_at(void *dst, int d);
// dst [cross_fold_bytes] <- the matrices ([out][in], as the projections have them), all on the device; returns when it is done (load time)
struct CrossFoldWeights {
  const _Float16 *Wkv, *Wq, *Wo;
  const float *bkv, *bq, *bo, *enc_gamma, *enc_beta, *gamma2, *beta2;
  float q_scale;
};
hipError_t cross_fold_build(const CrossFoldWeights &w, int d, void *dst, hipStream_t s);
// x [M][d]: the encoder's residual stream -> codes [M][2][d], sc [M][4] (see Dec1Args).  tail: the normalised rows keep head + tail.
hipError_t launch_cross_fold(const float *x, int M, int d, LnEps eps, const CrossFold &f, bool tail, short *cache, float *sc, hipStream_t s);
// x [M][2 d] fp32 (key | value of M positions) -> codes [M][2][d] and scales [M][2]; planes (optional): the rounded
// vectors as head / tail planes [M][d] (tail lo_offset elements after the head) and key_const[m] = scale * (u . key)
struct KvPlanes {
  _Float16 *k, *v;
  long lo_offset;
  const float *u;
  float scale;
  float *key_const;
};
hipError_t launch_quantize_kv_i16(const float *x, long M, int d, short *cache, float *sc, const KvPlanes *planes, hipStream_t s);

// max dynamic LDS the encoder attention needs for (S, dh); used to validate shapes at load.
size_t enc_attention_lds_bytes(int S, int dh, bool f32);

}  // namespace nt
