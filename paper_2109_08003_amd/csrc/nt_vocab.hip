// Output projection fused with the row arg-max (gfx950): the fragment order of the output matrix, the kernel for a few rows, and the
// choice among the kernels.
//
// The log-softmax of the output layer is not needed for greedy search (Sec. 3.3 "Graph Optimization"), and the logits never reach
// memory: a lane owns a row and folds the logits in its accumulators into the row's best.  A few rows, or a
// few hundred with a small vocabulary, take vocab_wide_kernel below (vocab_wide), more the scout of nt_vocab_scout.hip, model widths other than 256 and 512 the tiled kernels of nt_gemm.hip.
//
// Fragment order of Wp: [strip = v / 64][ks = k / 16][nb = (v % 64) / 32][lane][8 halfs] with
// lane = v % 32 + 32 * ((k % 16) / 8): lane l of the MFMA row operand holds W[v = l % 32][k = 8 * (l / 32) .. + 7].  A wave fetches a
// fragment with one fully coalesced 1 KiB load directly into the registers the MFMA reads.
#include "nt_kernels.h"

namespace nt {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

bool vocab_stream_supported(int K) { return K == 256 || K == 512; }

size_t vocab_pack_bytes(int N, int K) { return (size_t)((N + 63) / 64) * 64 * K * 2; }

void vocab_pack(const _Float16 *Wt, int N, int K, _Float16 *dst) {
  const int NS = (N + 63) / 64, KS = K / 16;
  for (int strip = 0; strip < NS; strip++)
    for (int ks = 0; ks < KS; ks++)
      for (int nb = 0; nb < 2; nb++)
        for (int lane = 0; lane < 64; lane++) {
          const int v = strip * 64 + nb * 32 + (lane & 31), k = ks * 16 + (lane >> 5) * 8;
          _Float16 *o = dst + ((((size_t)strip * KS + ks) * 2 + nb) * 64 + lane) * 8;
          for (int e = 0; e < 8; e++) o[e] = v < N ? Wt[(size_t)v * K + k + e] : (_Float16)0.f;
        }
}

// ---------------------------------------------------------------------------------------------------------------------
// A few rows with the chip to themselves (one request at a time).  The launch is then the time the output matrix (32 MB) takes to
// arrive, and with a strip per wave, streamed through a ring of registers, it arrived at 2.6 TB/s.  Here KP waves share a strip,
// each a range of its k-steps, all of whose fragments are requested at once (16 KB per wave, 128 KB per CU, the whole
// matrix in one round of workgroups); the rows' operands come straight from memory in the same way, so nothing waits for
// a tile to be filled.  They are requested first (loads return in order, and theirs are short) and a scheduling barrier keeps every
// load ahead of the first product: a step of 1 / 8 rows 14.8 / 15.6 us, with the rows last 15.0 / 16.0, left to the compiler, which
// requests the matrix in portions, 16.1 / 16.9.  Partial logits meet in the LDS.  The matrix is read past the L2 (non-temporal): it
// does not fit there and would evict the decoder's other weights at every step.  (Several tiles of 32 rows, which share a small one,
// read it through the L2.)
// One row: 7.0 us against 12.7, and 20 instead of 25 us for the decoder layer that follows.
// ---------------------------------------------------------------------------------------------------------------------
constexpr int VW_ROWS = 32;
static_assert(kVocabWideRows == VW_ROWS, "two strips per workgroup: one tile");
template <int K, int SPW, bool TILES>
__global__ __launch_bounds__(512) void vocab_wide_kernel(const _Float16 *__restrict__ h_hi, const _Float16 *__restrict__ h_lo,
                                                         long ldh, int M, const _Float16 *__restrict__ Wp, int N, int G,
                                                         unsigned long long *__restrict__ pk) {
  constexpr int KP = 8 / SPW, KS = K / 16, KSW = KS / KP, GPW = 8 / KP;  // k-parts; k-steps and register groups of a wave
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  __shared__ f32x4 red[8 * 8 * 64];  // [wave][register group][lane]
  __shared__ unsigned long long skey[8][32];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int NS = (N + 63) >> 6, kp = wave % KP, slot = wave / KP;
  const int strip_want = blockIdx.x * SPW + slot;
  const int strip = strip_want < NS ? strip_want : NS - 1;  // past the end: the last strip again (same keys)
  const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)Wp, 0, NS * 64 * K * 2, 0x00020000);
  const int w0 = (strip * KS + kp * KSW) * 2048;
  const int m0 = TILES ? blockIdx.y * VW_ROWS : 0, m = m0 + li < M ? m0 + li : M - 1;
  const long at_ = (long)m * ldh + kp * (KSW * 16) + g * 8;
  half8 xh[KSW], xl[KSW];
#pragma unroll
  for (int ks = 0; ks < KSW; ks++) {
    xh[ks] = *(const half8 *)(h_hi + at_ + ks * 16);
    xl[ks] = *(const half8 *)(h_lo + at_ + ks * 16);
  }
  __builtin_amdgcn_sched_barrier(0);
  half8 w[KSW][2];
#pragma unroll
  for (int ks = 0; ks < KSW; ks++)
#pragma unroll
    for (int nb = 0; nb < 2; nb++)
      w[ks][nb] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(wrs, lane * 16 + nb * 1024, w0 + ks * 2048, TILES ? 0 : 2));
  __builtin_amdgcn_sched_barrier(0);
  floatx16 acc[2];
#pragma unroll
  for (int nb = 0; nb < 2; nb++)
#pragma unroll
    for (int v = 0; v < 16; v++) acc[nb][v] = 0.f;
#pragma unroll
  for (int ks = 0; ks < KSW; ks++)
#pragma unroll
    for (int nb = 0; nb < 2; nb++) {
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[ks][nb], xh[ks], acc[nb], 0, 0, 0);
      acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(w[ks][nb], xl[ks], acc[nb], 0, 0, 0);
    }
#pragma unroll
  for (int q = 0; q < 8; q++)
    red[(wave * 8 + q) * 64 + lane] = f32x4{acc[q >> 2][(q & 3) * 4], acc[q >> 2][(q & 3) * 4 + 1], acc[q >> 2][(q & 3) * 4 + 2], acc[q >> 2][(q & 3) * 4 + 3]};
  __syncthreads();
  // this wave sums and folds register groups kp * GPW .. + GPW - 1 of its strip; columns ascend
  float best = -INFINITY;
  int at_best = 0;
#pragma unroll
  for (int u = 0; u < GPW; u++) {
    const int q = kp * GPW + u;
    f32x4 t = red[(slot * KP * 8 + q) * 64 + lane];
#pragma unroll
    for (int p = 1; p < KP; p++) t += red[((slot * KP + p) * 8 + q) * 64 + lane];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int n = strip * 64 + (q >> 2) * 32 + (q & 3) * 8 + g * 4 + e;
      const bool gt = n < N && t[e] > best;
      best = gt ? t[e] : best;
      at_best = gt ? n : at_best;
    }
  }
  unsigned long long key = best == -INFINITY ? 0ull : argmax_key(best, at_best);
  const unsigned long long other = shfl_xor_u64(key, 32);
  key = other > key ? other : key;
  if (g == 0) skey[wave][li] = key;
  __syncthreads();
  if (tid < VW_ROWS && m0 + tid < M) {
    unsigned long long k = skey[0][tid];
#pragma unroll
    for (int i = 1; i < 8; i++) k = skey[i][tid] > k ? skey[i][tid] : k;
    pk[(long)(m0 + tid) * G + blockIdx.x] = k;
  }
}

// Strips per workgroup of the wide kernel: one (eight k-parts) as long as that is one round of workgroups, else two
static int vw_strips(int N) { return (N + 63) / 64 <= 256 ? 1 : 2; }
static int vw_groups(int N) { return ((N + 63) / 64 + vw_strips(N) - 1) / vw_strips(N); }
static bool use_stream(const VocabWeights &w) { return !w.force_tiled && w.Wp && vocab_stream_supported(w.K); }

bool vocab_tiled(const VocabWeights &w) { return !use_stream(w); }
bool vocab_wide(const VocabWeights &w, int rows, int line) {
  if (!use_stream(w)) return false;
  const int tiles = (rows + VW_ROWS - 1) / VW_ROWS, NS = (w.N + 63) / 64;
  if (vw_strips(w.N) == 1) return tiles == 1 || (long)tiles * NS <= kVocabWideStrips;
  return rows <= line && vw_groups(w.N) <= 512;
}
bool vocab_scouted(const VocabWeights &w, bool wide) { return use_stream(w) && !wide; }

int vocab_argmax_partials(const VocabWeights &w, int M, bool certified, bool wide) {
  if (!use_stream(w)) return vocab_argmax_partials_tiled(M, w.N);
  return !certified && wide ? vw_groups(w.N) : 0;
}

hipError_t launch_vocab_argmax(const _Float16 *h, const _Float16 *h_lo, long ldh, const VocabWeights &w, int M,
                               unsigned long long *pk, bool wide, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (!use_stream(w)) return launch_vocab_argmax_tiled(h, h_lo, ldh, w.Wt, M, w.N, w.K, pk, s);
  if (!wide) return hipErrorInvalidValue;
  const int G = vw_groups(w.N), spw = vw_strips(w.N);
#define NT_VW(K_, S_, T_) \
  if (w.K == K_ && spw == S_ && (M > VW_ROWS) == T_) {                                                                                            \
    hipLaunchKernelGGL((vocab_wide_kernel<K_, S_, T_>), dim3(G, (M + VW_ROWS - 1) / VW_ROWS), dim3(512), 0, s, h, h_lo, ldh, M, w.Wp, w.N, G, pk); \
    return hipGetLastError();                                                                                                                     \
  }
  NT_VW(512, 1, false) NT_VW(512, 1, true) NT_VW(512, 2, false) NT_VW(256, 1, false) NT_VW(256, 1, true) NT_VW(256, 2, false)
#undef NT_VW
  return hipErrorInvalidValue;  // (two strips per workgroup: one tile, see vocab_wide)
}

hipError_t launch_vocab_argmax_certified(const VocabScout &v, const _Float16 *h, const _Float16 *h_lo, long ldh,
                                         const VocabWeights &w, int M, const float *lo_norm, float w_norm_max,
                                         unsigned long long *pk, float *ps, int32_t *tok, int32_t *slot_of_row, int32_t *list,
                                         int32_t *count, unsigned long long *final_key, PickArgs *later, hipStream_t s) {
  if (M <= 0) return hipSuccess;
  if (!use_stream(w) && later) return hipErrorInvalidValue;
  if (!use_stream(w))
    return launch_vocab_argmax_certified_tiled(h, h_lo, ldh, w.Wt, M, w.N, w.K, lo_norm, w_norm_max, pk, ps, tok,
                                               slot_of_row, list, count, final_key, s);
  return launch_vocab_scout(v, h, h_lo, ldh, w, M, w_norm_max > 1e29f, tok, slot_of_row, later, s);
}

}  // namespace nt
