// The candidates the scout has left, their exact logits and the arg-max of the rows of a workgroup (gfx950): a launch of its own
// (nt_vocab_scout.hip), or the start of the next step's first decoder layer (nt_dec1.hip).
#pragma once
#include "nt_kernels.h"

namespace nt {

constexpr int SC_NONE = -(1 << 30);  // below every packed product (places past the end of the vocabulary)
constexpr int SC_LOW = -(1 << 23);   // below every product
constexpr int SC_APART = 13;         // the distance to the third leaves in units of 2^13
constexpr int kPickCap = 1024;       // candidates of a row

#ifdef __HIPCC__
// All waves of a row find its candidates; the logits are then dealt to groups of 16 lanes, because the rows differ (16 on average, 70 at most in a
// thousand on flat random logits) and one wave with its own row's took as long as the worst row.
// Bound by its chain of dependent loads (the scout's groups, then the candidates' rows of the matrix), so a row is spread over as many
// waves as find work in it.  With four rows per workgroup and four entries in flight per group - most of them loads of an entry that
// was not there, 16 to 64 candidates for 128 places - it took 7.6, 8.2, 9.9 and 12.6 us at 45, 260, 400 and 1,000 rows on average,
// now 5.3, 5.6, 7.7 and 9.9.
// Rows with more than kPickCap candidates have every entry computed, by the same function, once all others are done.
// ---------------------------------------------------------------------------------------------------------------------

// Reductions over a wave in the vector unit (data-parallel primitives: rows of 16 lanes, then their broadcasts): a tenth of the
// latency of an exchange through the LDS unit.
template <int CTRL, int ROWS>
__device__ __forceinline__ int pk_dpp(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int pk_scan(int x) {  // inclusive sum over the lanes
  x += pk_dpp<0x111, 0xf>(0, x);  // row_shr 1, 2, 4, 8
  x += pk_dpp<0x112, 0xf>(0, x);
  x += pk_dpp<0x114, 0xf>(0, x);
  x += pk_dpp<0x118, 0xf>(0, x);
  x += pk_dpp<0x142, 0xa>(0, x);  // the last lane of rows 0 and 2 to rows 1 and 3, then of row 1 to rows 2 and 3
  return x + pk_dpp<0x143, 0xc>(0, x);
}
__device__ __forceinline__ float pk_max(float x) {  // over all lanes
  auto step = [](float v, auto ctrl, auto rows) {
    return fmaxf(v, __int_as_float(pk_dpp<decltype(ctrl)::value, decltype(rows)::value>(__float_as_int(-INFINITY), __float_as_int(v))));
  };
  typedef std::integral_constant<int, 0xf> all;
  x = step(x, std::integral_constant<int, 0x111>{}, all{});
  x = step(x, std::integral_constant<int, 0x112>{}, all{});
  x = step(x, std::integral_constant<int, 0x114>{}, all{});
  x = step(x, std::integral_constant<int, 0x118>{}, all{});
  x = step(x, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
  x = step(x, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ float pk_sum16(float x) {  // over 16 lanes (rotations: every lane gets it)
  x += __int_as_float(pk_dpp<0x128, 0xf>(0, __float_as_int(x)));
  x += __int_as_float(pk_dpp<0x124, 0xf>(0, __float_as_int(x)));
  x += __int_as_float(pk_dpp<0x122, 0xf>(0, __float_as_int(x)));
  return x + __int_as_float(pk_dpp<0x121, 0xf>(0, __float_as_int(x)));
}


template <int K, int ROWS, int NWAVES>
struct PickShared {
  __attribute__((aligned(16))) float x[ROWS][K];
  int32_t cand[ROWS][kPickCap];
  int count[ROWS];
  float floors[NWAVES];
  unsigned long long best[ROWS];
};
// Rows first_row .. first_row + ROWS - 1 (of M; row r of the launch's is row row0 + r of the states): their keys in sh.best, there for all
// waves on return.  The whole workgroup calls it.
template <int K, int ROWS, int NWAVES>
__device__ __forceinline__ void pick_rows(const PickArgs &a, PickShared<K, ROWS, NWAVES> &sh, int first_row, int M) {
  constexpr int WPR = NWAVES / ROWS;  // waves that find a row's candidates
  constexpr int CH = 8 / WPR;              // strips per lane at a time
  constexpr int STEP = WPR * 64 * CH;
  constexpr int KC = K / 128;         // runs of 128 elements: 16 lanes x 8
  constexpr int NG = NWAVES * 4;    // groups of 16 lanes
  constexpr int NE = K / 64;
  typedef _Float16 half8 __attribute__((ext_vector_type(8)));
  typedef int i32x4 __attribute__((ext_vector_type(4)));
  auto &sx = sh.x;
  auto &cand = sh.cand;
  auto &count = sh.count;
  auto &floors = sh.floors;
  auto &best = sh.best;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), e16 = lane & 15, group = threadIdx.x >> 4;
  const int own_row = wave / WPR, half = wave % WPR;
  const int i = first_row + own_row;
  const bool valid = i < M;
  const int r = a.row0 + (valid ? i : 0);
  {
    typedef _Float16 halfNE __attribute__((ext_vector_type(NE)));
    const i32x4 *mine = (const i32x4 *)a.part + (long)(valid ? i : 0) * a.NS;
    i32x4 p[CH];
    float4 sc[CH];
    auto load = [&](int s0) {
#pragma unroll
      for (int c = 0; c < CH; c++) {
        const int s = s0 + (WPR * c + half) * 64 + lane;
        const int at = s < a.NS ? s : a.NS - 1;  // past the end: the last strip again, left out below
        p[c] = mine[at];
        sc[c] = a.strip_consts[at];
      }
    };
    load(0);
    const float4 rc = a.row_consts[r];  // {scale, ||e||, ||a||}
    const halfNE xh = *(const halfNE *)(a.h_hi + (long)r * a.ldh + lane * NE), xl = *(const halfNE *)(a.h_lo + (long)r * a.ldh + lane * NE);
    // what a strip's scout logits may be off by, with what fp32 loses on either side
    auto bound = [&](const float4 &c) { return 1.0001f * (rc.y * c.y + rc.z * c.z) + 3e-6f * (rc.y + rc.z) * c.y + a.distrust; };
    float floor_ = -INFINITY;
    for (int s0 = 0;;) {
#pragma unroll
      for (int c = 0; c < CH; c++) {
        const int top = (p[c][0] > p[c][2] ? p[c][0] : p[c][2]) >> 5;
        floor_ = fmaxf(floor_, rc.x * sc[c].x * (float)top - bound(sc[c]));
      }
      if ((s0 += STEP) >= a.NS) break;
      load(s0);
    }
    floor_ = pk_max(floor_);
    if (lane == 0) {
      floors[wave] = floor_;
      if (half == 0) count[own_row] = 0, best[own_row] = 0ull;
    }
    if (half == 0) {
#pragma unroll
      for (int e = 0; e < NE; e += 4)
        *(float4 *)&sx[own_row][lane * NE + e] = make_float4((float)xh[e] + (float)xl[e], (float)xh[e + 1] + (float)xl[e + 1],
                                                             (float)xh[e + 2] + (float)xl[e + 2], (float)xh[e + 3] + (float)xl[e + 3]);
    }
    __syncthreads();
    floor_ = floors[WPR * own_row];
#pragma unroll
    for (int w = 1; w < WPR; w++) floor_ = fmaxf(floor_, floors[WPR * own_row + w]);
    // every lane counts its own groups' candidates, then all write theirs
    for (int s0 = 0; s0 < a.NS && valid; s0 += STEP) {
      if (a.NS > STEP) load(s0);
      unsigned firsts = 0u, seconds = 0u, thirds = 0u;
#pragma unroll
      for (int c = 0; c < CH; c++) {
        const float unit = rc.x * sc[c].x, least = floor_ - bound(sc[c]);
        const bool there = s0 + (WPR * c + half) * 64 + lane < a.NS;
#pragma unroll
        for (int g = 0; g < 2; g++) {
          const int second = p[c][2 * g + 1] >> 8, apart = p[c][2 * g + 1] >> 5 & 7;
          auto in = [&](int product) { return !(unit * (float)product < least); };  // (a NaN is a candidate)
          const bool one = there && p[c][2 * g] > SC_NONE / 2 && in(p[c][2 * g] >> 5), two = one && second > SC_LOW && in(second);
          firsts |= one ? 1u << (2 * c + g) : 0u;
          seconds |= two ? 1u << (2 * c + g) : 0u;
          thirds |= two && in(second - (apart << SC_APART)) ? 1u << (2 * c + g) : 0u;  // as large as a third can be
        }
      }
      const int own = __popc(firsts) + __popc(seconds) + 32 * __popc(thirds), upto = pk_scan(own);
      const int all = __builtin_amdgcn_readlane(upto, 63);
      if (all == 0) continue;
      int base = 0;
      if (lane == 0) base = atomicAdd(&count[own_row], all);
      int at = __builtin_amdgcn_readfirstlane(base) + upto - own;
      auto add = [&](int c, int g, int code) {
        if (at < kPickCap)
          cand[own_row][at] = (s0 + (WPR * c + half) * 64 + lane) * 64 + (code >> 4) * 32 + ((code & 15) >> 2) * 8 + g * 4 + (code & 3);
        at++;
      };
#pragma unroll
      for (int c = 0; c < CH; c++)
#pragma unroll
        for (int g = 0; g < 2; g++) {
          if (firsts >> (2 * c + g) & 1u) add(c, g, p[c][2 * g] & 31);
          if (seconds >> (2 * c + g) & 1u) add(c, g, p[c][2 * g + 1] & 31);
          if (thirds >> (2 * c + g) & 1u)  // rare: all 32 of the group
            for (int code = 0; code < 32; code++) add(c, g, code);
        }
    }
  }
  __syncthreads();
  // logit of row `row` and the entry whose elements lane e16 of a group holds in w; every lane of the group gets it
  auto dot = [&](const half8 (&w)[KC], int row) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < KC; j++) {
      const float4 x0 = *(const float4 *)&sx[row][j * 128 + e16 * 8], x1 = *(const float4 *)&sx[row][j * 128 + e16 * 8 + 4];
      const float x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
      for (int t = 0; t < 8; t++) s += x[t] * (float)w[j][t];
    }
    return pk_sum16(s);
  };
  auto key = [](float s, int id) { return s > -INFINITY ? argmax_key(s, id) : 0ull; };  // (not for a NaN, which argmax_key ranks first)
  auto fetch = [&](half8 (&w)[KC], int place) {
#pragma unroll
    for (int j = 0; j < KC; j++) w[j] = *(const half8 *)(a.Ws + (long)place * K + j * 128 + e16 * 8);
  };
  int first[ROWS + 1];  // of the rows' candidates, laid end to end
  unsigned many = 0u;
  first[0] = 0;
#pragma unroll
  for (int w = 0; w < ROWS; w++) {
    const int n = count[w];
    many |= n > kPickCap ? 1u << w : 0u;
    first[w + 1] = first[w] + (n > kPickCap ? 0 : n);
  }
  // (a wave without a candidate left drops out; within a wave all groups load, which is faster than a branch around the loads)
  for (int c0 = wave * 4; c0 < first[ROWS]; c0 += NG) {
    const int c = c0 + (lane >> 4);
    int row = 0, from = 0;
#pragma unroll
    for (int q = 1; q < ROWS; q++)
      if (c >= first[q]) row = q, from = first[q];
    const bool there = c < first[ROWS];
    const int place = there ? cand[row][c - from] : 0;
    half8 w[KC];
    fetch(w, place);
    const int id = there ? a.ids[place] : -1;
    const unsigned long long k = key(dot(w, row), id);
    if (e16 == 0 && id >= 0) atomicMax(&best[row], k);
  }
  if (many) {
    unsigned long long mine[ROWS] = {};
    for (int v0 = 0; v0 < a.NS * 64; v0 += NG) {
      const int id = a.ids[v0 + group];
      half8 w[KC];
      fetch(w, v0 + group);
#pragma unroll
      for (int q = 0; q < ROWS; q++)
        if (many >> q & 1u) {
          const unsigned long long k = key(dot(w, q), id);
          mine[q] = id >= 0 && k > mine[q] ? k : mine[q];
        }
    }
#pragma unroll
    for (int q = 0; q < ROWS; q++)
      if (e16 == 0 && (many >> q & 1u)) atomicMax(&best[q], mine[q]);
  }
  __syncthreads();
}
#endif

}  // namespace nt
