// Tri-state tailor (Sec. IV-F eq. 10, Alg. 1 "KV Cache Tailor") and the prompt commit.
//
//   choose  : heavy-hitter score S = mu + gamma*var (eq. 9) -> 64-bit selection key
//             (fp32 bits of S) << 32 | (0xFFFFFFFF - position); larger key = better rank, so ties in
//             S go to the older token and the order is total.  0 marks "not eligible".
//             exact k-th largest key by radix select, for k = n_o and k = b together;
//             classification of every slot and the lists that compact both pools in place
//   move    : quantise the demoted rows into free Q slots, fill holes with tail rows
//
// Everything that decides a state or a code is integer or single-rounded fp32 arithmetic in a fixed
// order (this file must be compiled with -ffp-contract=off).
#include <hip/hip_fp16.h>

#include <algorithm>
#include <type_traits>

#include "arkv_dev.h"

namespace arkv {

typedef uint32_t u32x4t __attribute__((ext_vector_type(4)));   // 16 bytes; arrays of it stay in registers (arrays of uint4 do not)

// ------------------------------------------------------------------------------------------
// score -> key
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float hh_moments_score(float mu, float ex2, float gamma) {
  const float var = fmaxf(ex2 - mu * mu, 0.0f);
  return mu + gamma * var;
}
__device__ __forceinline__ float hh_score(float s1, float s2, int n, float gamma) {
  const float nf = (float)n;
  return hh_moments_score(s1 / nf, s2 / nf, gamma);
}

// The radix select looks at digits of (score - smallest score), and a row that is not ranked must not match one that is: kNoScore
// lies at least 2^21 above every score, so after the first digit (which leaves at most 21 bits) its leading bits differ from
// every candidate's.  Scores are >= 0 or NaN; negative NaNs above that line count as the largest value below it.
__device__ __forceinline__ uint64_t make_key(float S, int pos) {
  return ((uint64_t)min(__float_as_uint(S), 0xFFDFFFFFu) << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)pos);
}

// ------------------------------------------------------------------------------------------
// exact k-th largest key for two ranks at once, by one workgroup of 1024 threads.
//
// Radix select, most significant digit first, on digits of up to 11 bits of (score - smallest score): the scores of a unit
// share most of their leading bits, so digits of the difference spread them over the bins from the first pass on, and two
// passes usually leave one candidate per rank (digits of the score itself: three passes, the first one held up by lanes that
// met on the few exponents' bins).  The position is only looked at where scores tie at a rank.  Bound by the one CU's
// instruction issue and the passes' barriers, not by bytes, hence: the unit's scores as 32-bit words in LDS, four to a read,
// and rolled loops over them (in registers they took unrolled code with the ballots of every round live at once: hundreds of
// spilled scalar registers), and both ranks in the same passes.  Once the chosen bin holds a single candidate the remaining
// passes are skipped.
// ------------------------------------------------------------------------------------------
constexpr uint32_t kNoScore = 0xFFFFFFFFu;   // not ranked (above every score, see make_key)
constexpr int kLdsRows = 32768;              // units of up to this many rows keep their scores in LDS (128 KB)
constexpr int kFusedRows = 8192;             // prompts of up to this many positions are scored by the workgroup that selects
constexpr int kRounds = 32;                  // rounds of 1024 rows per list chunk
constexpr int kBins = 2048, kDigit = 11;
constexpr int kFew = 64;                     // candidates of a rank that one wave ranks among themselves, a lane each
constexpr int kQuad = 4096;                  // rows of a round of the selection: four adjacent ones per thread
__host__ __device__ constexpr int quads(int rows) { return (rows + kQuad - 1) / kQuad; }
template <typename Row>                      // Row: integer that holds a row index
struct SelectLds {
  union {
    int hist[2 * kBins];                     // one histogram per rank
    struct { uint32_t score[2][kFew]; int row[2][kFew]; } list;      // a rank's last candidates
    struct {                                 // behind the selection, per 64 rows of a list chunk (see k_tailor_choose)
      uint64_t stay[kRounds * 16], dem[kRounds * 16];
      uint32_t off[3][kRounds * 16];         // places of the rows' first entries in the lists, two of 16 bits each
    };
  };
  Row who[2 * kBins];                        // a row that fell into the bin (the row, where only one did)
  uint32_t wsum[2][16], lo[16], hi[16];
  uint64_t thr[2];
  int sel[2], k[2], cnt[2];
  int crowded[6];                            // per pass over the scores
  int listed[2];
};

// The k-th best (1: the best) of n <= kFew listed rows, by one wave; its threshold as select_two gives it.  Equal scores go by
// the keys' low words.
template <typename Key>
__device__ __forceinline__ void rank_few(const uint32_t* scores, const int* rows, int n, int k, Key&& key, uint64_t* thr) {
  const int lane = threadIdx.x & 63;
  const bool mine = lane < n;
  const uint32_t s = mine ? scores[lane] : 0u;
  int better = 0, equal = 0;
  for (int j = 0; j < n; ++j) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)s, j);
    better += o > s ? 1 : 0;
    equal += o == s ? 1 : 0;
  }
  const bool hit = mine && better < k && k <= better + equal;
  const unsigned long long hits = __ballot(hit);
  if (__popcll(hits) == 1) {
    if (hit) *thr = (uint64_t)s << 32;
    return;
  }
  const uint64_t full = hit ? key(rows[lane]) : 0ull;
  int older = 0;
  for (unsigned long long todo = hits; todo; todo &= todo - 1)
    older += (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)full, __ffsll(todo) - 1) > (uint32_t)full ? 1 : 0;
  if (hit && better + older == k - 1) *thr = full;
}

// inclusive sum over the wave's lanes up to this one (DPP: row shifts by 1, 2, 4, 8, then the rows' last lanes)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_prefix_sum(uint32_t v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);
  return dpp_add<0x143, 0xc>(v);
}

// Sums of 16 waves' values in LDS: of the waves before this one (w, uniform), and of all.
struct WaveSums { uint32_t before, total; };
__device__ __forceinline__ WaveSums wave_sums(const uint32_t* sums /*[16]*/, int lane, int w) {
  uint32_t v = sums[lane & 15];
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  const uint32_t up_to = (uint32_t)__builtin_amdgcn_readlane((int)v, w), own = sums[w];
  return {up_to - own, (uint32_t)__builtin_amdgcn_readlane((int)v, 15)};
}

// Smallest and largest score seen so far; over the wave's lanes.
struct ScoreRange {
  uint32_t lo = kNoScore, hi = 0;
  __device__ __forceinline__ void add(uint32_t sb) {
    lo = min(lo, sb);
    hi = max(hi, sb == kNoScore ? 0u : sb);
  }
  // over the wave's lanes, in the last one (the steps of wave_prefix_sum)
  template <int CTRL, int ROWS>
  __device__ __forceinline__ void step() {
    lo = min(lo, (uint32_t)__builtin_amdgcn_update_dpp((int)kNoScore, (int)lo, CTRL, ROWS, 0xf, false));
    hi = max(hi, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, ROWS, 0xf, false));
  }
  __device__ __forceinline__ void wave() {
    step<0x111, 0xf>(); step<0x112, 0xf>(); step<0x114, 0xf>(); step<0x118, 0xf>(); step<0x142, 0xa>(); step<0x143, 0xc>();
  }
};

// The lanes of a wave that share the first adding lane's bin (all lanes of the wave must be here).
struct Shared { int first, bin, lanes; };
__device__ __forceinline__ Shared shared_bin(int bin, bool add, unsigned long long adding) {
  const int first = __ffsll(adding) - 1, b = __builtin_amdgcn_readlane(bin, first);
  return {first, b, (int)__popcll(__ballot(add && bin == b))};
}

// load(q, s) must give the scores s[0 .. 3] of rows 4096 q + 4 * thread .. + 3, q < nq (kNoScore: not a candidate);
// score(row), key(row) = a candidate's, for any thread; range: of the scores this thread has seen, all threads' together of
// all candidates.  sm.thr[x]: the candidates whose key is at least that are the best k_x.  It is the key of rank k_x, its low
// word left out (0) where no other candidate has that score, or ~0 when k_x = 0 or there is no candidate (nothing
// qualifies); k_x is clamped to the number of candidates, so "fewer candidates than b" keeps everything.  Ends with a barrier.
template <typename Row, typename Load, typename Score, typename Key>
__device__ __forceinline__ void select_two(int nq, Load&& load, Score&& score_at, Key&& key, ScoreRange range, int k0, int k1,
                                           SelectLds<Row>& sm) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t prefix[2] = {0, 0};               // digits found so far: of the score, then (tie) of the low word
  uint32_t base = 0, score[2] = {0, 0};      // the smallest score; tie passes: the rank's whole score
  int k[2] = {k0, k1};
  bool done[2] = {k0 <= 0, k1 <= 0};
  int left[2] = {0, 0}, total = 0;           // candidates of a rank after the last pass, and at the start
  range.wave();
  if (lane == 63) { sm.lo[w] = range.lo; sm.hi[w] = range.hi; }
  if (tid < 2) sm.thr[tid] = ~0ull;
  if (tid < 6) sm.crowded[tid] = 0;
  if (tid < 2) sm.listed[tid] = 0;
  bool tie = false;                          // scores are used up: digits of the low word among equal scores
  int rest = 0;                              // bits of the score (low word) not looked at yet
  for (int pass = 0;; ++pass) {
    if (done[0] && done[1]) break;
    const int top = kBins - 1 - 2 * tid;     // this thread's bins: top and top - 1
    *reinterpret_cast<int2*>(&sm.hist[top - 1]) = make_int2(0, 0);
    *reinterpret_cast<int2*>(&sm.hist[kBins + top - 1]) = make_int2(0, 0);
    if (pass == 0) {
      __syncthreads();                       // (also for keys that lie in memory: load reads other threads')
      uint32_t lo = kNoScore, hi = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) { lo = min(lo, sm.lo[i]); hi = max(hi, sm.hi[i]); }
      base = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
      hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
      if (base == kNoScore) break;           // no candidate: rows that are not ranked must not count as equal scores
      rest = hi > base ? 32 - __builtin_clz(hi - base) : 0;
    }
    if (rest == 0) {
      if (tie) break;                        // (positions are distinct: a bin of the last pass holds one candidate)
      tie = true;
      rest = 32;
      for (int x = 0; x < 2; ++x) { score[x] = base + prefix[x]; prefix[x] = 0; }
    }
    const bool low_first = tie && rest == 32;
    const int width = min(rest, kDigit);
    rest -= width;
    const bool shared = prefix[0] == prefix[1] && score[0] == score[1];    // both ranks still look at the same candidates
    const bool use0 = !done[0] || shared, use1 = !done[1] && !shared;
    const bool few = 3 * ((use0 ? left[0] : 0) + (use1 ? left[1] : 0)) <= total;
    // bin_of(score, row, bin): whether the row is counted in this pass, and in which bin, which remembers a row.
    // Accesses to one LDS word are served lane by lane, and equal scores (or the leading digits of neighbouring positions)
    // put whole waves on one bin.  So every wave looks at a row per lane, spread over the unit; if any finds more than 24
    // lanes on one bin, the pass counts the lanes that share the first one's at once.  Otherwise it does not: that costs ten
    // instructions per round.  Nor does it look where less than a third of the rows are candidates (a wave then has 21 of
    // them).
    auto count_shared = [&](auto&& bin_of) {
      for (int q = 0; q < nq; ++q) {
        uint32_t s4[4];
        load(q, s4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int row = kQuad * q + 4 * tid + e;
          int bin = 0;
          const bool add = bin_of(s4[e], row, bin);
          const unsigned long long adding = __ballot(add);
          if (adding == 0) continue;
          const Shared s = shared_bin(bin, add, adding);
          if (lane == s.first || (add && bin != s.bin)) {
            atomicAdd(&sm.hist[bin], lane == s.first ? s.lanes : 1);
            sm.who[bin] = (Row)row;
          }
        }
      }
    };
    auto count = [&](auto&& bin_of) {
      if (!few) {
        const int q = (w * nq) >> 4;
        uint32_t s4[4];
        load(q, s4);
        int bin = 0;
        const bool add = bin_of(s4[0], kQuad * q + 4 * tid, bin);
        const unsigned long long adding = __ballot(add);
        if (adding != 0 && shared_bin(bin, add, adding).lanes > 24 && lane == 0) sm.crowded[pass] = 1;
      }
      __syncthreads();
      if (!few && sm.crowded[pass]) {
        count_shared(bin_of);
      } else {
        for (int q = 0; q < nq; ++q) {
          uint32_t s4[4];
          load(q, s4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int row = kQuad * q + 4 * tid + e;
            int bin = 0;
            if (bin_of(s4[e], row, bin)) {
              atomicAdd(&sm.hist[bin], 1);
              sm.who[bin] = (Row)row;
            }
          }
        }
      }
    };
    if (pass == 0 && !tie) {
      if (rest + width <= 6) {               // (nearly) equal scores: whole waves meet on a bin
        count_shared([&](uint32_t sb, int, int& bin) { bin = (int)((sb - base) >> rest); return sb != kNoScore; });
      } else {
        // the second histogram is free in this pass, so odd lanes count there and half as many lanes meet on a bin
        const int odd = (lane & 1) * kBins;
        for (int q = 0; q < nq; ++q) {
          uint32_t s4[4];
          load(q, s4);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (s4[e] != kNoScore) atomicAdd(&sm.hist[odd + (int)((s4[e] - base) >> rest)], 1);
        }
      }
    } else if (!tie) {
      const int up = rest + width;
      count([&](uint32_t sb, int, int& bin) {
        const uint32_t v = sb - base, hi = v >> up;    // (kNoScore never matches: it lies at least 2^21 above every score)
        const bool c0 = use0 && hi == prefix[0], c1 = use1 && hi == prefix[1];
        bin = (int)__builtin_amdgcn_ubfe(v, rest, width) + (c0 ? 0 : kBins);
        return c0 || c1;
      });
    } else {
      __syncthreads();                       // (the keys may lie in memory)
      count_shared([&](uint32_t sb, int row, int& bin) {
        bool c0 = use0 && sb == score[0], c1 = use1 && sb == score[1];
        if (c0 || c1) {
          const uint32_t lw = (uint32_t)key(row), hi = low_first ? 0u : lw >> (rest + width);
          c0 = c0 && hi == prefix[0];
          c1 = c1 && hi == prefix[1];        // (not both: two ranks with the same digits share the first histogram)
          bin = (int)__builtin_amdgcn_ubfe(lw, rest, width) + (c0 ? 0 : kBins);
        }
        return c0 || c1;
      });
    }
    __syncthreads();
    // ge = candidates in bins top - 1 and above
    int2 a = *reinterpret_cast<const int2*>(&sm.hist[top - 1]);
    const int2 b = *reinterpret_cast<const int2*>(&sm.hist[kBins + top - 1]);
    if (pass == 0 && !tie) { a.x += b.x; a.y += b.y; }
    uint32_t ge0 = wave_prefix_sum((uint32_t)(a.x + a.y)), ge1 = wave_prefix_sum((uint32_t)(b.x + b.y));
    if (lane == 63) { sm.wsum[0][w] = ge0; sm.wsum[1][w] = ge1; }
    __syncthreads();
    const WaveSums w0 = wave_sums(sm.wsum[0], lane, w), w1 = wave_sums(sm.wsum[1], lane, w);
    const uint32_t tot0 = w0.total;
    ge0 += w0.before;
    ge1 += w1.before;
    if (pass == 0) {
      total = (int)tot0;
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        if (k[x] > (int)tot0) k[x] = (int)tot0;         // fewer candidates than k: keep them all
        if (k[x] <= 0) done[x] = true;
      }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      if (done[x]) continue;
      const bool first = x == 0 || shared;
      const int hi_cnt = first ? a.y : b.y, lo_cnt = first ? a.x : b.x;
      const int g = (int)(first ? ge0 : ge1);                         // >= bin top - 1
      const int above = g - hi_cnt - lo_cnt;                          // > bin top
      if (above < k[x] && k[x] <= above + hi_cnt) { sm.sel[x] = top; sm.k[x] = k[x] - above; sm.cnt[x] = hi_cnt; }
      else if (above + hi_cnt < k[x] && k[x] <= g) { sm.sel[x] = top - 1; sm.k[x] = k[x] - above - hi_cnt; sm.cnt[x] = lo_cnt; }
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      if (done[x]) continue;
      prefix[x] = (prefix[x] << width) | (uint32_t)sm.sel[x];
      k[x] = sm.k[x];
      left[x] = sm.cnt[x];
      if (sm.cnt[x] == 1 && (pass > 0 || tie)) {         // one candidate left
        const int row = (int)sm.who[(x == 0 || shared ? 0 : kBins) + sm.sel[x]];
        if (tid == 0) sm.thr[x] = tie ? key(row) : (uint64_t)score_at(row) << 32;
        done[x] = true;
      }
    }
    // Few candidates left: they are listed and a wave per rank ranks them among themselves, instead of another pass with its
    // histogram, sums and three barriers (a commit's selection, 32 units x 32768 positions: 23 -> 21.4 us; 64 at most, a lane each)
    if (!tie && !(done[0] && done[1]) && (done[0] || left[0] <= kFew) && (done[1] || left[1] <= kFew)) {
      const bool same = !done[0] && !done[1] && prefix[0] == prefix[1];
      const bool use0 = !done[0], use1 = !done[1] && !same;
      for (int q = 0; q < nq; ++q) {
        uint32_t s4[4];
        load(q, s4);
        bool in0[4], in1[4], any = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t hi = (s4[e] - base) >> rest;
          in0[e] = use0 && hi == prefix[0];
          in1[e] = use1 && hi == prefix[1];
          any = any || in0[e] || in1[e];
        }
        if (any) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (in0[e] || in1[e]) {
              const int x = in0[e] ? 0 : 1, i = atomicAdd(&sm.listed[x], 1);
              sm.list.score[x][i] = s4[e];
              sm.list.row[x][i] = kQuad * q + 4 * tid + e;
            }
          }
        }
      }
      __syncthreads();
      if (w == 0 && !done[0]) rank_few(sm.list.score[0], sm.list.row[0], left[0], k[0], key, &sm.thr[0]);
      if (w == 1 && !done[1]) rank_few(sm.list.score[same ? 0 : 1], sm.list.row[same ? 0 : 1], left[1], k[1], key, &sm.thr[1]);
      break;
    }
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------------------
// block-wide exclusive scan of NF words of packed counters, 1024 threads; ends with a barrier
// ------------------------------------------------------------------------------------------
template <int NF>
__device__ __forceinline__ void block_excl_scan(uint32_t (&v)[NF], uint32_t (*sm)[16] /*[NF][16]*/, uint32_t (&total)[NF]) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t inc[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    inc[f] = wave_prefix_sum(v[f]);
    if (lane == 63) sm[f][w] = inc[f];
  }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const WaveSums ws = wave_sums(sm[f], lane, w);
    total[f] = ws.total;
    v[f] = ws.before + inc[f] - v[f];
  }
  __syncthreads();
}

// a row's place behind the rows before it in the wave that set the same flag
__device__ __forceinline__ int place(unsigned long long flags, int lane) {
  return __popcll(flags & ((1ull << lane) - 1ull));
}

// ------------------------------------------------------------------------------------------
// quantiser: one K or V row held by LPR lanes, 8 channels each (fp32 from bf16)
// ------------------------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dppf(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               0xf, 0xf, true));
}

__device__ __forceinline__ uint16_t f2h(float x) { return __half_as_ushort(__float2half_rn(x)); }
__device__ __forceinline__ float h2f(uint16_t h) { return __half2float(__ushort_as_half(h)); }
__device__ __forceinline__ uint16_t h_next_down(uint16_t h) {
  if ((h & 0x7fffu) == 0) return 0x8001u;
  return (h & 0x8000u) ? (uint16_t)(h + 1) : (uint16_t)(h - 1);
}
__device__ __forceinline__ uint16_t h_next_up(uint16_t h) {
  if ((h & 0x7fffu) == 0) return 0x0001u;
  return (h & 0x8000u) ? (uint16_t)(h - 1) : (uint16_t)(h + 1);
}

// x: the 8 channels of this lane; the 4 lanes of an aligned quad form one group of 32 channels.
// Returns the lane's packed codes (8*BITS bits) and the group's meta word (scale | zero << 16).
template <int BITS>
__device__ __forceinline__ void quantize8(const float (&x)[8], uint32_t& codes, uint32_t& meta) {
  const float qmax = (float)((1 << BITS) - 1);
  float mn = x[0], mx = x[0];
#pragma unroll
  for (int c = 1; c < 8; ++c) { mn = fminf(mn, x[c]); mx = fmaxf(mx, x[c]); }
  mn = fminf(mn, dppf<0xB1>(mn)); mx = fmaxf(mx, dppf<0xB1>(mx));
  mn = fminf(mn, dppf<0x4E>(mn)); mx = fmaxf(mx, dppf<0x4E>(mx));
  uint16_t zh = f2h(mn);
  float z = h2f(zh);
  if (z > mn) { zh = h_next_down(zh); z = h2f(zh); }
  const float r = mx - z;
  uint16_t sh = 0;
  codes = 0;
  if (r != 0.0f) {
    const float s = r / qmax;
    sh = f2h(s);
    float sc = h2f(sh);
    if (sc * qmax < r) { sh = h_next_up(sh); sc = h2f(sh); }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      float t = rintf((x[c] - z) / sc);
      t = fminf(fmaxf(t, 0.0f), qmax);
      codes |= (uint32_t)t << (BITS * c);
    }
  }
  meta = (uint32_t)sh | ((uint32_t)zh << 16);
}

__device__ __forceinline__ void unpack8(const uint4& r, float (&f)[8]) {
  f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
  f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
  f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
  f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
}

// fp8 rows with one scale per token (Alg. 1 "Reconstruction Before Attention": x~ = q^ * s).
// |t| <= 448 -> nearest E4M3 code (sign, 4 exponent bits with bias 7, 3 mantissa bits, subnormals below
// 2^-6, no infinities), ties to the even code, in integer arithmetic on the fp32 bits.
__device__ __forceinline__ uint32_t e4m3_code(float t) {
  const float a = fminf(fabsf(t), 448.0f);
  uint32_t code;
  if (a < 0.015625f) {
    code = (uint32_t)rintf(a * 512.0f);             // subnormals are multiples of 2^-9; 8 = the smallest normal
  } else {
    uint32_t b = __float_as_uint(a);
    b += 0x7FFFFu + ((b >> 20) & 1u);               // round to 3 mantissa bits, ties to even
    code = (((b >> 23) - 120u) << 3) | ((b >> 20) & 7u);
  }
  return code;
}

// x: the 8 channels of this lane; the LPR lanes of a row share one scale.
// Returns the lane's 8 codes (byte c = channel c) and the row's scale (fp16 bits).
template <int LPR>
__device__ __forceinline__ void quantize8_fp8(const float (&x)[8], uint2& codes, uint32_t& meta) {
  float amax = fabsf(x[0]);
#pragma unroll
  for (int c = 1; c < 8; ++c) amax = fmaxf(amax, fabsf(x[c]));
  amax = fmaxf(amax, dppf<0xB1>(amax));
  amax = fmaxf(amax, dppf<0x4E>(amax));
  amax = fmaxf(amax, dppf<0x141>(amax));             // 8 lanes
  if (LPR == 16) amax = fmaxf(amax, dppf<0x140>(amax));
  uint16_t sh = 0;
  codes = make_uint2(0, 0);
  if (amax != 0.0f) {
    const float s = amax / 448.0f;
    sh = f2h(s);
    float sc = h2f(sh);
    if (sc * 448.0f < amax) { sh = h_next_up(sh); sc = h2f(sh); }
    uint32_t w[2] = {0, 0};
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const uint32_t code = e4m3_code(x[c] / sc) | (x[c] < 0.0f ? 0x80u : 0u);
      w[c >> 2] |= code << (8 * (c & 3));
    }
    codes = make_uint2(w[0], w[1]);
  }
  meta = sh;
}

// 2 LPR adjacent lanes (lane = 0 .. 2 LPR - 1 among them) quantise a token into Q slot dst of unit gu: lanes [0, LPR) the
// K row, the others the V row.  A wave takes 64 / (2 LPR) tokens at once; every lane runs the arithmetic (the lane
// exchanges need them active), lanes without store write nothing.
template <int D, int BITS>
__device__ __forceinline__ void quantize_into(const Pools& P, int gu, int dst, const uint16_t* krow,
                                              const uint16_t* vrow, int lane, bool store) {
  constexpr int LPR = D / 8, CB = D * BITS / 8, NG = metas_per_row(D, BITS);
  const bool isv = lane >= LPR;
  const int sub = lane % LPR;
  const uint16_t* src = (isv ? vrow : krow) + sub * 8;
  const uint4 raw = *reinterpret_cast<const uint4*>(src);
  float x[8];
  unpack8(raw, x);
  // K: canonical row-major packing.  V: the same bytes, token-minor in blocks of kVBlock tokens (see Pools).
  uint8_t* cdst = P.qkc + ((size_t)gu * P.capQ + dst) * CB;
  uint32_t* mdst = P.qkm + ((size_t)gu * P.capQ + dst) * NG;
  uint8_t* vcu = P.qvc + (size_t)gu * P.capQv * CB;
  constexpr int MH = vmeta_per_row(D, BITS);
  uint16_t* vmu = P.qvm + (size_t)gu * P.capQv * MH;
  if constexpr (BITS == 8) {
    uint2 codes;
    uint32_t meta;
    quantize8_fp8<LPR>(x, codes, meta);
    if (!store) return;
    if (lane < LPR) {
      *reinterpret_cast<uint2*>(cdst + ((sub & 3) * (D / 32) + (sub >> 2)) * 8) = codes;     // see kcode_index
      if (sub == 0) mdst[0] = meta;
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        vcu[vcode_index(dst, 8 * sub + i, CB, BITS)] = (uint8_t)((i < 4 ? codes.x >> (8 * i) : codes.y >> (8 * (i - 4))) & 0xffu);
      if (sub == 0) vmu[vmeta_index(dst, 0, MH)] = (uint16_t)meta;
    }
  } else {
    uint32_t codes, meta;
    quantize8<BITS>(x, codes, meta);
    if (!store) return;
    if (lane < LPR) {
      const int chunk = (sub & 3) * (D / 32) + (sub >> 2);                                   // see kcode_index
      if (BITS == 4) *reinterpret_cast<uint32_t*>(cdst + chunk * 4) = codes;
      else *reinterpret_cast<uint16_t*>(cdst + chunk * 2) = (uint16_t)codes;
      if ((sub & 3) == 0) mdst[sub >> 2] = meta;
    } else {
#pragma unroll
      for (int i = 0; i < BITS; ++i) vcu[vcode_index(dst, BITS * sub + i, CB, BITS)] = (uint8_t)((codes >> (8 * i)) & 0xffu);
      if ((sub & 3) == 0) {
        vmu[vmeta_index(dst, sub >> 2, MH)] = (uint16_t)(meta & 0xffffu);              // scale
        vmu[vmeta_index(dst, D / kGroup + (sub >> 2), MH)] = (uint16_t)(meta >> 16);   // zero point
      }
    }
  }
}

// What one workgroup of a launch writes and another reads inside the same launch goes through device-scope relaxed atomics
// (write-through stores, loads that do not hit a stale L2 line of another XCD); no cache-wide flush.
__device__ __forceinline__ void st_dev8(void* p, uint64_t v) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_dev8(const void* p) {
  return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a row's running sums, `dev`: which another workgroup of this launch may have written
__device__ __forceinline__ float2 row_sums(const float2* p, bool dev) {
  return dev ? __builtin_bit_cast(float2, ld_dev8(p)) : *p;
}

// The unit's counts behind its tailor, by one thread.  The host's copy spares a copy of its own behind every tailor.
__device__ __forceinline__ void publish_counts(const Pools& P, const TailorLaunch& L, int gu, int o, int q) {
  P.cnt[gu] = make_int2(o, q);
  if (L.tell_host)
    __hip_atomic_store(P.cnt_host + gu, count_word(o, q, L.seq[(gu - L.unit_begin) / P.U]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The moves of a unit's tailor.  first: index of this wave among the `waves` that share them.
// nD demoted rows into free Q slots (TPW tokens per wave at once), nM tail rows of the Q pool into holes.  list(l, i): entry i
// of a list.
enum MoveList { kOHole = 0, kOMov, kDem, kQFree, kQMov, kMoveLists };
// where a list begins in a unit's plan
__device__ __forceinline__ size_t list_begin(const Pools& P, int l) {
  return (size_t)kPlanHdr + (size_t)(l < kQMov ? l : kQFree) * P.capO + (size_t)(l < kQMov ? 0 : P.capQ);
}
template <int D, int BITS, typename List>
__device__ __forceinline__ void tailor_move_q(const Pools& P, int gu, int nD, int nM, int first, int waves, int lane, bool dev,
                                              List&& list) {
  constexpr int CB = D * BITS / 8, NG = metas_per_row(D, BITS);
  constexpr int LPT = 2 * (D / 8), TPW = 64 / LPT;
  const int t = lane / LPT, sl = lane % LPT;
  for (int i0 = first * TPW; i0 < nD; i0 += waves * TPW) {
    const int item = min(i0 + t, nD - 1), dst = list(kQFree, item);
    const size_t o = (size_t)gu * P.capO + list(kDem, item);
    quantize_into<D, BITS>(P, gu, dst, P.ok + o * D, P.ov + o * D, sl, i0 + t < nD);
    if (sl == 0 && i0 + t < nD) {
      P.qpos[(size_t)gu * P.capQ + dst] = P.opos[o];
      P.qacc[(size_t)gu * P.capQ + dst] = row_sums(P.oacc + o, dev);
    }
  }
  for (int item = first; item < nM; item += waves) {
    const int dst = list(kQFree, nD + item), src = list(kQMov, item);
    const size_t so = (size_t)gu * P.capQ + src, d_ = (size_t)gu * P.capQ + dst;
    // K: code bytes, 4 per lane; V: one byte column per lane (token-minor blocks)
    for (int b = lane * 4; b < CB; b += 256)
      *reinterpret_cast<uint32_t*>(P.qkc + d_ * CB + b) = *reinterpret_cast<const uint32_t*>(P.qkc + so * CB + b);
    uint8_t* vcu = P.qvc + (size_t)gu * P.capQv * CB;
    for (int b = lane; b < CB; b += 64) vcu[vcode_index(dst, b, CB, BITS)] = vcu[vcode_index(src, b, CB, BITS)];
    constexpr int MH = vmeta_per_row(D, BITS);
    uint16_t* vmu = P.qvm + (size_t)gu * P.capQv * MH;
    if (lane < MH) vmu[vmeta_index(dst, lane, MH)] = vmu[vmeta_index(src, lane, MH)];
    if (lane < NG) P.qkm[d_ * NG + lane] = P.qkm[so * NG + lane];
    if (lane == 0) { P.qpos[d_] = P.qpos[so]; P.qacc[d_] = row_sums(P.qacc + so, dev); }
  }
}

// nM tail rows of the O pool into holes: after every demoted row of the unit has been read.
template <int D, typename List>
__device__ __forceinline__ void tailor_move_o(const Pools& P, int gu, int nM, int first, int waves, int lane, bool dev, List&& list) {
  constexpr int LPR = D / 8, LPT = 2 * LPR, TPW = 64 / LPT;
  const int t = lane / LPT, sl = lane % LPT, sub = sl % LPR;
  uint16_t* base = sl < LPR ? P.ok : P.ov;
  for (int item = first * TPW + t; item < nM; item += waves * TPW) {
    const size_t so = (size_t)gu * P.capO + list(kOMov, item), d_ = (size_t)gu * P.capO + list(kOHole, item);
    *reinterpret_cast<uint4*>(base + d_ * D + sub * 8) = *reinterpret_cast<const uint4*>(base + so * D + sub * 8);
    if (sl == 0) { P.opos[d_] = P.opos[so]; P.oacc[d_] = row_sums(P.oacc + so, dev); }
  }
}

// ------------------------------------------------------------------------------------------
// in-place tailor: keys (eq. 9's score per row), the two thresholds, and the lists that compact both pools.
// One launch; one workgroup per unit chooses, bound by its CU's instruction issue and round trips.  Where the step's logits have
// to be turned into probabilities as well, the scores of many rows are the unit's workgroups' work (tailor_parts): they leave
// keys and sums at the device's coherence point, and the one that draws the last ticket reads the keys back and goes on.
// 32 units x 8192 rows with kept logits, one row moved per step: 20.2 us with the launch's start and end; 25.6 with one
// workgroup for everything (scores 9.3, selection 4.4, fates 3.3, lists 1.7, moves 3.1), a ballot per 64 rows for the fates and
// the lists of the moved rows fetched back from memory (the last two 1.2 us together).
// Fates are kept as a bit per row (two words per 64 rows), so that the lists' counts are one thread's work per 64 rows and words
// with nothing to list are skipped.
//   plan: header | ohole[capO] | omov[capO] | dem[capO] | qfree[capQ] | qmov[capQ]
// ------------------------------------------------------------------------------------------
// bits 0 .. n - 1 of a word whose first bit is row `row0`: the rows below `end`
__device__ __forceinline__ uint64_t rows_below(int row0, int end) {
  const int n = end - row0;
  return n <= 0 ? 0ull : n >= 64 ? ~0ull : (1ull << n) - 1ull;
}
// What a list gets of 64 rows: Original rows to fill (hole), Original rows behind the new end that stay (mov), demoted rows
// (dem), free Quantized slots below the new end (fr), Quantized rows behind it that stay (qm).
struct ListFlags { uint64_t hole, mov, dem, fr, qm; };
__device__ __forceinline__ ListFlags list_flags(uint64_t stay, uint64_t dem, int row0, int cO, int n, int cOn, int cQn) {
  const uint64_t o = rows_below(row0, cO), on = rows_below(row0, cOn), all = rows_below(row0, n), q = rows_below(row0, cO + cQn);
  return {~stay & on, stay & o & ~on, dem, ~stay & all & q & ~o, stay & all & ~o & ~q};
}

// Sum and sum of squares of a step's probabilities of one row over the unit's heads, added up as k_flush_scores does.
// fin: the step's final (max, 1/sum) per head.
template <int G>
__device__ __forceinline__ float2 step_moments(const float (&x)[G], const float2 (&fin)[G]) {
  constexpr int HB = (G + 3) / 4, HPL = G < 4 ? G : 4;
  float2 m[HB];
#pragma unroll
  for (int b = 0; b < HB; ++b) {
    m[b] = make_float2(0.f, 0.f);
#pragma unroll
    for (int i = 0; i < HPL; ++i) {
      const float p = __builtin_amdgcn_exp2f(x[4 * b + i] - fin[4 * b + i].x) * fin[4 * b + i].y;
      m[b].x += p;
      m[b].y = fmaf(p, p, m[b].y);
    }
  }
  if constexpr (HB == 2) { m[0].x += m[1].x; m[0].y += m[1].y; }
  return m[0];
}

// KEPT: the pending step's logits are in Pools::logit (see k_decode_attend); its probabilities are added to the sums here.
// L.few_moves (with and without them): the moves are made here as well.
constexpr int kNearList = 64;
template <int G, bool IN_LDS, bool KEPT>
__global__ __launch_bounds__(1024) void k_tailor_choose(Pools P, TailorLaunch L) {
  extern __shared__ __align__(16) uint32_t row_word[];      // IN_LDS: score of row i
  __shared__ __align__(16) SelectLds<typename std::conditional<IN_LDS, uint16_t, uint32_t>::type> sel;
  __shared__ uint32_t scan_sm[3][16];
  __shared__ int tot[3];
  __shared__ int32_t near_list[kMoveLists][kNearList];
  const int gu = L.unit_begin + blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int parts = IN_LDS && KEPT ? (int)gridDim.y : 1, part = blockIdx.y;
  const int2 cnt = P.cnt[gu];
  const int cO = cnt.x, cQ = cnt.y, n = cO + cQ;           // rows: the O pool's, then the Q pool's
  uint64_t* keys = P.keys + (size_t)gu * (P.capO + P.capQ);
  const int32_t* opos = P.opos + (size_t)gu * P.capO;
  const int32_t* qpos = P.qpos + (size_t)gu * P.capQ;
  float2* oacc = P.oacc + (size_t)gu * P.capO;
  float2* qacc = P.qacc + (size_t)gu * P.capQ;
  const float* logit = KEPT ? P.logit + (size_t)(gu - P.logit_unit0) * P.logit_stride : nullptr;   // (may be this unit's plan)
  float2 fin[G];
  if constexpr (KEPT) {
    const float2* f = P.fin + (size_t)((L.slot + kRing - 1) % kRing) * P.fin_stride + (size_t)gu * G;
#pragma unroll
    for (int h = 0; h < G; ++h) fin[h] = f[h];
  }
  const int slot_q = P.capO - cO;                           // row i >= cO: key slot i + slot_q
  const int nq = quads(n), rounds = (n + 1023) / 1024;
  ScoreRange range;
  // (a __syncthreads of the selection stands between these stores and another thread's read of a key: its fence orders the
  // workgroup's accesses to memory, which on this target needs no wait for the stores, they pass the CU's L1 in order)
  constexpr int BATCH = 4;                                  // rows requested together, one batch ahead of their use
  struct Rows { int pos[BATCH]; float2 acc[BATCH]; float x[KEPT ? BATCH : 1][G]; };
  auto fetch_rounds = [&](int round, int step, Rows& r) {      // BATCH rounds of 1024 rows, `step` apart
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int i = min(1024 * (round + step * j) + tid, n - 1);
      r.pos[j] = i < cO ? opos[i] : qpos[i - cO];
      r.acc[j] = i < cO ? oacc[i] : qacc[i - cO];
      if constexpr (KEPT) {
        typedef float Vec __attribute__((ext_vector_type(G < 4 ? G : 4)));
        const Vec* p = reinterpret_cast<const Vec*>(logit + (size_t)i * G);
        if constexpr (G == 1) r.x[j][0] = *reinterpret_cast<const float*>(p);
        else
#pragma unroll
          for (int v = 0; v < (G + 3) / 4; ++v) {
            const Vec t = p[v];
#pragma unroll
            for (int h = 0; h < (G < 4 ? G : 4); ++h) r.x[j][4 * v + h] = t[h];
          }
      }
    }
  };
  auto fetch = [&](int q, Rows& r) { fetch_rounds(4 * q, 1, r); };
  // key of row i (0: not ranked), its sums brought up to date
  auto score_row = [&](int i, int pos, float2& acc, const float (&x)[G]) -> uint64_t {
    if constexpr (KEPT) {
      const float2 m = step_moments<G>(x, fin);
      acc.x += m.x; acc.y += m.y;
    }
    if (i >= n || pos >= L.position + 1 - L.window) return 0;
    const int first = pos > L.t_prefill - L.window ? pos : L.t_prefill - L.window;
    return make_key(hh_score(acc.x, acc.y, G * (L.position - first + 1), L.gamma), pos);
  };
  auto score_rows = [&](int q, Rows& r) {
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int i = kQuad * q + 1024 * j + tid;
      if (kQuad * q + 1024 * j >= n) {                      // a round without rows
        if constexpr (IN_LDS) row_word[i] = kNoScore;
        continue;
      }
      const uint64_t key = score_row(i, r.pos[j], r.acc[j], r.x[KEPT ? j : 0]);
      if (KEPT && i < n) *(i < cO ? oacc + i : qacc + (i - cO)) = r.acc[j];
      const uint32_t sb = key ? (uint32_t)(key >> 32) : kNoScore;
      range.add(sb);
      if (i < n) keys[i < cO ? i : i + slot_q] = key;
      if constexpr (IN_LDS) row_word[i] = sb;               // (whole quads)
    }
  };
  if (parts > 1) {
    // This workgroup's rounds of 1024 rows, every parts-th; the unit's last workgroup reads all keys back and goes on alone.
    Rows r;
    for (int j0 = part; j0 < rounds; j0 += parts * BATCH) {
      fetch_rounds(j0, parts, r);
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const int i = 1024 * (j0 + j * parts) + tid;
        if (i >= n) continue;
        const uint64_t key = score_row(i, r.pos[j], r.acc[j], r.x[KEPT ? j : 0]);
        st_dev8(i < cO ? oacc + i : qacc + (i - cO), __builtin_bit_cast(uint64_t, r.acc[j]));
        st_dev8(keys + (i < cO ? i : i + slot_q), key);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // this wave's stores are at the device's coherence point
    __syncthreads();
    if (tid == 0) {
      int* const ticket = P.ticket + (size_t)gu * (kTicketWaves * kTicketPitch);      // (zero between launches)
      const int done = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
      if (done == parts) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      tot[0] = done;
    }
    __syncthreads();
    if (tot[0] != parts) return;
    constexpr int AHEAD = 8;
    for (int j0 = 0; j0 < 4 * nq; j0 += AHEAD) {
      uint64_t k[AHEAD];
#pragma unroll
      for (int j = 0; j < AHEAD; ++j) {
        const int i = min(1024 * (j0 + j) + tid, n - 1);
        k[j] = ld_dev8(keys + (i < cO ? i : i + slot_q));
      }
#pragma unroll
      for (int j = 0; j < AHEAD; ++j) {
        const int i = 1024 * (j0 + j) + tid;
        if (j0 + j >= 4 * nq) break;
        const uint32_t sb = i < n && k[j] ? (uint32_t)(k[j] >> 32) : kNoScore;
        range.add(sb);
        if constexpr (IN_LDS) row_word[i] = sb;
      }
    }
    __syncthreads();                                        // (tot is read above and cleared below)
  } else {
    Rows ra, rb;
    fetch(0, ra);
    for (int q = 0; q < nq; q += 2) {
      fetch(min(q + 1, nq - 1), rb);
      score_rows(q, ra);
      if (q + 1 < nq) {
        fetch(min(q + 2, nq - 1), ra);
        score_rows(q + 1, rb);
      }
    }
  }
  auto key_of = [&](int i) -> uint64_t {
    const uint64_t* k = keys + (i < cO ? i : i + slot_q);
    return parts > 1 ? ld_dev8(k) : *k;
  };
  auto score_of = [&](int i) -> uint32_t {
    if constexpr (IN_LDS) return row_word[i];
    const uint64_t k = key_of(i);
    return k ? (uint32_t)(k >> 32) : kNoScore;
  };
  auto load = [&](int q, uint32_t (&s)[4]) {
    const int i = kQuad * q + 4 * tid;
    if constexpr (IN_LDS) {
      const uint4 v = *reinterpret_cast<const uint4*>(row_word + i);
      s[0] = v.x; s[1] = v.y; s[2] = v.z; s[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] = i + e < n ? score_of(i + e) : kNoScore;
    }
  };
  if (tid < 3) tot[tid] = 0;
  select_two(nq, load, score_of, key_of, range, P.n_o[gu], P.nb[gu], sel);
  const uint64_t thr_o = sel.thr[0], thr_b = sel.thr[1];

  // What becomes of the rows: each stays in its pool (window rows do), is demoted, or (neither) is evicted.  Most stay: a
  // chunk's words start out so, and only the rows that leave touch them, four adjacent ones at once (with a ballot for every
  // 64 rows this took 3.3 us of 22 for 8192 rows).
  const uint32_t so = (uint32_t)(thr_o >> 32), sq = (uint32_t)(thr_b >> 32);
  const bool ties = __builtin_amdgcn_readfirstlane((uint32_t)thr_o | (uint32_t)thr_b) != 0;
  // the rows of rounds j0 .. j0 + nj - 1 of 1024: marks them in the words, and counts those that leave their pool
  auto fates = [&](int j0, int nj, bool mark, bool count) {
    if (mark) {
      if (tid < 16 * nj) { sel.stay[tid] = rows_below(1024 * j0 + 64 * tid, n); sel.dem[tid] = 0; }
      __syncthreads();
    }
    uint32_t leaveO = 0, demoted = 0, leaveQ = 0;
    for (int q = 0; q < quads(1024 * nj); ++q) {
      uint32_t s4[4];
      load(j0 / 4 + q, s4);
      const int i0 = 1024 * j0 + kQuad * q + 4 * tid;
      uint32_t gone = 0, dem = 0;                            // of the four rows
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = i0 + e;
        const uint32_t sb = s4[e];
        const bool o = i < cO, none = sb == kNoScore;
        bool geo = sb >= so, geb = sb >= sq;                 // (a row that is not ranked: both, and it stays Original)
        if (ties && !none && (sb == so || sb == sq)) {       // scores that tie with a threshold: the whole key decides
          const uint64_t key = key_of(i);
          geo = key >= thr_o; geb = key >= thr_b;
        }
        if (i < n && !(o ? geo : geb && !none)) {
          const bool d = o && geb;
          leaveO += o ? 1 : 0; demoted += d ? 1 : 0; leaveQ += o ? 0 : 1;
          gone |= 1u << e;
          dem |= d ? 1u << e : 0u;
        }
      }
      if (mark && gone) {
        const int word = (i0 - 1024 * j0) >> 5;
        atomicAnd(reinterpret_cast<uint32_t*>(sel.stay) + word, ~(gone << (i0 & 31)));
        if (dem) atomicOr(reinterpret_cast<uint32_t*>(sel.dem) + word, dem << (i0 & 31));
      }
    }
    if (count && __any((leaveO | leaveQ) != 0)) {
      const uint32_t a = wave_prefix_sum(leaveO), b = wave_prefix_sum(demoted), c = wave_prefix_sum(leaveQ);
      if (lane == 63) { atomicAdd(&tot[0], (int)a); atomicAdd(&tot[1], (int)b); atomicAdd(&tot[2], (int)c); }
    }
    __syncthreads();
  };
  const bool one_chunk = rounds <= kRounds;
  fates(0, rounds, one_chunk, true);
  const int cOn = cO - tot[0], nD = tot[1], cQn = cQ - tot[2] + nD;

  int32_t* plan = P.plan + (size_t)gu * P.plan_stride;
  // a list's first entries stay in LDS where this workgroup makes the moves
  const bool here = L.few_moves;
  auto put = [&](int l, int i, int32_t v) {
    if (here && i < kNearList) near_list[l][i] = v;
    else plan[list_begin(P, l) + i] = v;
  };
  int base_hole = 0, base_mov = 0, base_dem = 0, base_free = 0, base_qmov = 0;
  for (int j0 = 0; j0 < rounds; j0 += kRounds) {
    const int nj = rounds - j0 < kRounds ? rounds - j0 : kRounds, entries = 16 * nj;
    if (!one_chunk) fates(j0, nj, true, false);
    uint32_t v[3] = {0, 0, 0}, total[3];
    if (tid < entries) {                                    // thread = 64 rows
      const ListFlags f = list_flags(sel.stay[tid], sel.dem[tid], 1024 * j0 + 64 * tid, cO, n, cOn, cQn);
      v[0] = (uint32_t)__popcll(f.hole) | ((uint32_t)__popcll(f.mov) << 16);
      v[1] = (uint32_t)__popcll(f.dem) | ((uint32_t)__popcll(f.fr) << 16);
      v[2] = (uint32_t)__popcll(f.qm);
    }
    block_excl_scan<3>(v, scan_sm, total);
    if (tid < entries) { sel.off[0][tid] = v[0]; sel.off[1][tid] = v[1]; sel.off[2][tid] = v[2]; }
    __syncthreads();
    // wave: its share of the entries, a lane each, of which most have nothing to list in the long run
    const int mine = 16 * lane + w;
    uint64_t m_stay = 0, m_dem = 0;
    bool some = false;
    if (mine < entries) {
      m_stay = sel.stay[mine]; m_dem = sel.dem[mine];
      const ListFlags f = list_flags(m_stay, m_dem, 1024 * j0 + 64 * mine, cO, n, cOn, cQn);
      some = (f.hole | f.mov | f.dem | f.fr | f.qm) != 0;
    }
    for (unsigned long long todo = __ballot(some); todo; todo &= todo - 1) {
      const int l = __ffsll(todo) - 1, e = 16 * l + w, row0 = 1024 * j0 + 64 * e, i = row0 + lane;
      auto of = [&](uint64_t m) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)m, l) | ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(m >> 32), l) << 32);
      };
      const ListFlags f = list_flags(of(m_stay), of(m_dem), row0, cO, n, cOn, cQn);
      const uint32_t hm = sel.off[0][e], df = sel.off[1][e], qm = sel.off[2][e];
      auto has = [&](uint64_t m) { return ((m >> lane) & 1) != 0; };
      if (has(f.hole)) put(kOHole, base_hole + (int)(hm & 0xFFFF) + place(f.hole, lane), i);
      if (has(f.mov)) put(kOMov, base_mov + (int)(hm >> 16) + place(f.mov, lane), i);
      if (has(f.dem)) put(kDem, base_dem + (int)(df & 0xFFFF) + place(f.dem, lane), i);
      if (has(f.fr)) put(kQFree, base_free + (int)(df >> 16) + place(f.fr, lane), i - cO);
      if (has(f.qm)) put(kQMov, base_qmov + (int)qm + place(f.qm, lane), i - cO);
    }
    base_hole += (int)(total[0] & 0xFFFF); base_mov += (int)(total[0] >> 16);
    base_dem += (int)(total[1] & 0xFFFF); base_free += (int)(total[1] >> 16);
    base_qmov += (int)total[2];
    if (j0 + kRounds < rounds) __syncthreads();            // the next chunk's flags go into the same table
  }
  // slots behind the Q pool's old end
  for (int i = tid; i < cQn - cQ; i += 1024) put(kQFree, base_free + i, cQ + i);
  if (tid == 0) {
    plan[PL_CO_NEW] = cOn; plan[PL_CQ_NEW] = cQn; plan[PL_N_DEM] = nD;
    plan[PL_N_QMOV] = base_qmov; plan[PL_N_OMOV] = base_mov;
    plan[PL_CO_OLD] = cO; plan[PL_CQ_OLD] = cQ;
  }
  if (!here) return;
  __syncthreads();                                        // the lists
  auto list = [&](int l, int i) { return i < kNearList ? near_list[l][i] : plan[list_begin(P, l) + i]; };
  auto moves = [&](auto d, auto bits) {
    tailor_move_q<decltype(d)::value, decltype(bits)::value>(P, gu, nD, base_qmov, w, 16, lane, parts > 1, list);
    __syncthreads();                                      // every demoted row has been read
    tailor_move_o<decltype(d)::value>(P, gu, base_mov, w, 16, lane, parts > 1, list);
  };
  using std::integral_constant;
  if (P.D == 128) {
    const integral_constant<int, 128> d;
    if (P.bits == 4) moves(d, integral_constant<int, 4>()); else if (P.bits == 2) moves(d, integral_constant<int, 2>()); else moves(d, integral_constant<int, 8>());
  } else {
    const integral_constant<int, 64> d;
    if (P.bits == 4) moves(d, integral_constant<int, 4>()); else if (P.bits == 2) moves(d, integral_constant<int, 2>()); else moves(d, integral_constant<int, 8>());
  }
  if (tid == 0) publish_counts(P, L, gu, cOn, cQn);
}

template <int D, int BITS>
__global__ __launch_bounds__(256) void k_tailor_move_q(Pools P, TailorLaunch L) {
  const int gu = L.unit_begin + blockIdx.y;
  const int32_t* plan = P.plan + (size_t)gu * P.plan_stride;
  tailor_move_q<D, BITS>(P, gu, plan[PL_N_DEM], plan[PL_N_QMOV], blockIdx.x * 4 + (threadIdx.x >> 6), gridDim.x * 4, threadIdx.x & 63, false,
                         [&](int l, int i) { return plan[list_begin(P, l) + i]; });
}

template <int D>
__global__ __launch_bounds__(256) void k_tailor_move_o(Pools P, TailorLaunch L) {
  const int gu = L.unit_begin + blockIdx.y;
  const int32_t* plan = P.plan + (size_t)gu * P.plan_stride;
  tailor_move_o<D>(P, gu, plan[PL_N_OMOV], blockIdx.x * 4 + (threadIdx.x >> 6), gridDim.x * 4, threadIdx.x & 63, false,
                   [&](int l, int i) { return plan[list_begin(P, l) + i]; });
  if (blockIdx.x == 0 && threadIdx.x == 0) publish_counts(P, L, gu, plan[PL_CO_NEW], plan[PL_CQ_NEW]);
}

// ------------------------------------------------------------------------------------------
// prompt commit: scores of the prompt's positions, the two thresholds, and the survivors' way into the empty pools
// ------------------------------------------------------------------------------------------
struct BudgetArgs { int n_o[64], nb[64]; };       // per sequence
// Scratch of a commit: scores [units][pitch] (rows of a whole number of 16-byte vectors), each 64 positions' range of them
// [units][commit_ranges], and what k_commit_select says of the blocks of 1024 positions.
struct CommitScratch { uint32_t* scores; int pitch; uint2* ranges; int4* blocks; };
__host__ __device__ constexpr int commit_ranges(int T) { return (T + 63) / 64; }
__host__ __device__ constexpr int commit_blocks(int T) { return (T + 1023) / 1024; }

// Scores of a long prompt's positions (kNoScore: window, and what fills the pitch), over the whole chip (two IEEE divisions per
// position: in the one workgroup that selects they took longer than the selection; see launch_commit for the line), each 64 positions' range of scores, and
// the layer's budgets (a launch of their own took 5 us).
__global__ __launch_bounds__(256) void k_commit_keys(Pools P, CommitLaunch L, CommitScratch C, int hkv, BudgetArgs budgets) {
  const int lu = blockIdx.y;
  if (hkv > 0 && blockIdx.x == 0 && threadIdx.x == 0) {
    P.n_o[L.unit_begin + lu] = budgets.n_o[lu / hkv];
    P.nb[L.unit_begin + lu] = budgets.nb[lu / hkv];
  }
  const int j = blockIdx.x * 256 + threadIdx.x;
  uint32_t sb = kNoScore;
  if (j < L.T - L.window) {
    const float2 a = L.pre[(size_t)lu * L.T + j];
    sb = (uint32_t)(make_key(hh_score(a.x, a.y, P.G * L.window, L.gamma), j) >> 32);
  }
  if (j < C.pitch) C.scores[(size_t)lu * C.pitch + j] = sb;
  ScoreRange r;
  r.add(sb);
  r.wave();
  if ((threadIdx.x & 63) == 63 && j - 63 < C.pitch) C.ranges[(size_t)lu * commit_ranges(L.T) + j / 64] = make_uint2(r.lo, r.hi);
}

// Parts into which a block with that many survivors is cut.
__device__ __forceinline__ uint32_t commit_parts(uint32_t survivors, int share_rows) {
  return (survivors + (uint32_t)share_rows - 1) / (uint32_t)share_rows;
}

// One workgroup per unit: 23 us for 32 units x 32768 positions, of which 15.7 between a workgroup's first instruction and its
// last (scores into LDS 1.9, selection 9.4, blocks 4.4) and the rest is the launch's start and end; 21.4 since one wave ranks
// the last candidates.  35 us with digits of the
// plain score, one score per LDS read and 64-bit keys in memory (whole commits of 32 x 32768 88 -> 74 us, 8 x 131072 159 -> 96,
// 8 x 1000 20.2 -> 19.4).  The two thresholds of a unit, and per block of 1024 positions (blocks [units][rounds + 1], the
// last one the totals) the rows in front of it that become Original and Quantized and the parts in front of it into which
// k_commit_scatter cuts blocks: as many as hold share_rows survivors each, wherever in the prompt the survivors sit.
//
// SCORES: the scores are formed here as well (and stored for k_commit_scatter), and the budgets come with this launch: short
// prompts, see launch_commit.
template <bool IN_LDS, bool SCORES>
__global__ __launch_bounds__(1024) void k_commit_select(Pools P, CommitLaunch L, CommitScratch C, int share_rows, int hkv, BudgetArgs budgets) {
  extern __shared__ __align__(16) uint32_t row_word[];     // IN_LDS: the positions' scores
  __shared__ __align__(16) SelectLds<typename std::conditional<IN_LDS, uint16_t, uint32_t>::type> sel;
  __shared__ uint32_t cnt[kRounds / 4][16];  // per (round of 4096 positions, wave): Original | Quantized << 16
  const int lu = blockIdx.x, gu = L.unit_begin + lu, tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T = L.T, rounds = commit_blocks(T), nq = quads(T);
  const int n_cand = T - L.window;           // positions behind them are the window
  const uint32_t* scores = C.scores + (size_t)lu * C.pitch;
  auto fetch = [&](int q) -> u32x4t {
    const int i = kQuad * q + 4 * tid;
    const u32x4t none = {kNoScore, kNoScore, kNoScore, kNoScore};
    return i < C.pitch ? *reinterpret_cast<const u32x4t*>(scores + i) : none;
  };
  ScoreRange range;
  int k_o, k_b;
  if constexpr (SCORES) {
    k_o = budgets.n_o[lu / hkv];
    k_b = budgets.nb[lu / hkv];
    if (tid == 0) { P.n_o[gu] = k_o; P.nb[gu] = k_b; }
    const float2* pre = L.pre + (size_t)lu * T;
    const int samples = P.G * L.window;
    const bool pow2 = (samples & (samples - 1)) == 0;        // the usual window: a product gives the quotient's very bits
    const float inv = 1.0f / (float)samples;
    float2 a[kFusedRows / kQuad][4];         // (all requested together)
#pragma unroll
    for (int q = 0; q < kFusedRows / kQuad; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[q][e] = pre[min(kQuad * q + 4 * tid + e, T - 1)];
#pragma unroll
    for (int q = 0; q < kFusedRows / kQuad; ++q) {
      const int i = kQuad * q + 4 * tid;
      u32x4t v = {kNoScore, kNoScore, kNoScore, kNoScore};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 t = a[q][e];
        const float S = pow2 ? hh_moments_score(t.x * inv, t.y * inv, L.gamma) : hh_score(t.x, t.y, samples, L.gamma);
        if (i + e < n_cand) v[e] = (uint32_t)(make_key(S, i + e) >> 32);
        range.add(v[e]);
      }
      if (i < C.pitch) *reinterpret_cast<u32x4t*>(C.scores + (size_t)lu * C.pitch + i) = v;
      if (q < nq) *reinterpret_cast<u32x4t*>(row_word + i) = v;
    }
  } else {
    k_o = P.n_o[gu];
    k_b = P.nb[gu];
    for (int i = tid; i < commit_ranges(T); i += 1024) {
      const uint2 r = C.ranges[(size_t)lu * commit_ranges(T) + i];
      range.lo = min(range.lo, r.x);
      range.hi = max(range.hi, r.y);
    }
  }
  if constexpr (IN_LDS && !SCORES) {
    u32x4t v[kLdsRows / kQuad];              // (all requested together; a thread only reads what it stores here)
#pragma unroll
    for (int q = 0; q < kLdsRows / kQuad; ++q)
      if (q < nq) v[q] = fetch(q);
#pragma unroll
    for (int q = 0; q < kLdsRows / kQuad; ++q)
      if (q < nq) *reinterpret_cast<u32x4t*>(row_word + kQuad * q + 4 * tid) = v[q];
  }
  auto load = [&](int q, uint32_t (&s)[4]) {
    u32x4t v;
    if constexpr (IN_LDS) v = *reinterpret_cast<const u32x4t*>(row_word + kQuad * q + 4 * tid);
    else v = fetch(q);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = v[e];
  };
  auto score_of = [&](int i) -> uint32_t {
    if constexpr (IN_LDS) return row_word[i];
    else return scores[i];
  };
  auto key_of = [&](int i) -> uint64_t { return ((uint64_t)score_of(i) << 32) | (0xFFFFFFFFu - (uint32_t)i); };
  select_two(nq, load, score_of, key_of, range, k_o, k_b, sel);
  const uint64_t thr_o = sel.thr[0], thr_b = sel.thr[1];
  int4* blocks = C.blocks + (size_t)lu * (rounds + 1);
  int bo = 0, bq = 0, bp = 0;
  for (int j0 = 0; j0 < rounds; j0 += kRounds) {
    const int nj = rounds - j0 < kRounds ? rounds - j0 : kRounds;
    for (int q = 0; q < quads(1024 * nj); ++q) {
      uint32_t s[4], no = 0, nb = 0;         // a wave's positions of the round are a quarter of a block
      load(j0 / 4 + q, s);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = 1024 * j0 + kQuad * q + 4 * tid + e;
        const uint64_t k = ((uint64_t)s[e] << 32) | (0xFFFFFFFFu - (uint32_t)i);
        no += (uint32_t)__popcll(__ballot(i < n_cand ? k >= thr_o : i < T));
        nb += (uint32_t)__popcll(__ballot(i < n_cand ? k >= thr_b : i < T));     // (n_o <= b)
      }
      if (lane == 0) cnt[q][w] = no | ((nb - no) << 16);
    }
    __syncthreads();
    // lane j of wave 0: round j (kRounds <= 64)
    if (w == 0) {
      uint32_t o = 0, q = 0;
      if (lane < nj)
#pragma unroll
        for (int i = 0; i < 4; ++i) { const uint32_t c = cnt[lane / 4][4 * (lane % 4) + i]; o += c & 0xFFFFu; q += c >> 16; }
      const uint32_t p = commit_parts(o + q, share_rows);
      const uint32_t io = wave_prefix_sum(o), iq = wave_prefix_sum(q), ip = wave_prefix_sum(p);
      if (lane < nj) blocks[j0 + lane] = make_int4(bo + (int)(io - o), bq + (int)(iq - q), bp + (int)(ip - p), 0);
      bo += __builtin_amdgcn_readlane((int)io, 63);
      bq += __builtin_amdgcn_readlane((int)iq, 63);
      bp += __builtin_amdgcn_readlane((int)ip, 63);
    }
    __syncthreads();
  }
  if (tid == 0) {
    P.thr[(size_t)gu * 2] = thr_o; P.thr[(size_t)gu * 2 + 1] = thr_b;
    P.cnt[gu] = make_int2(bo, bq);
    blocks[rounds] = make_int4(bo, bq, bp, 0);
  }
}

// A prompt that fits its cache: every row becomes Original.  The workgroups of a unit go through its rows side by side, a
// wave two (d = 64: four) tokens at a time.  Bound by the bytes (32 units x 16384 rows, 537 MB in and out, with the budgets'
// launch: 104 us; 8 units x 1000 rows 10.0).  Several rows in flight per lane, 512 to 8192 workgroups: slower or the same.
template <int D>
__global__ __launch_bounds__(256) void k_commit_copy(Pools P, CommitLaunch L) {
  constexpr int LPR = D / 8, LPT = 2 * LPR, TPW = 64 / LPT;      // as in k_commit_scatter
  const int lu = blockIdx.y, gu = L.unit_begin + lu, lane = threadIdx.x & 63, w = threadIdx.x >> 6, T = L.T;
  const int t = lane / LPT, sl = lane % LPT;
  const uint16_t* src = (sl < LPR ? L.k : L.v) + (size_t)lu * T * D + (sl % LPR) * 8;
  uint16_t* dst = (sl < LPR ? P.ok : P.ov) + (size_t)gu * P.capO * D + (sl % LPR) * 8;
  for (int i = (4 * blockIdx.x + w) * TPW + t; i < T; i += 4 * TPW * gridDim.x) {
    *reinterpret_cast<uint4*>(dst + (size_t)i * D) = *reinterpret_cast<const uint4*>(src + (size_t)i * D);
    if (sl == 0) {
      P.opos[(size_t)gu * P.capO + i] = i;
      P.oacc[(size_t)gu * P.capO + i] = L.pre[(size_t)lu * T + i];
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) P.cnt[gu] = make_int2(T, 0);
}

// The survivors of a selection into the pools: a workgroup takes one part of a block of 1024 positions (see k_commit_select).
// It lists the block's survivors in LDS (positions stay in ascending order), copies its share of the Original rows, several
// in flight per wave, and quantises its share of the others straight from the caller's rows.  Bound by the gathered rows'
// bytes where the grid fills the chip (32 units x 6152 of 32768 rows, 200 MB: 43 us), by a workgroup's chain of rounds where it
// does not, hence the parts: with one workgroup per block a whole commit of 16 units x 2200 positions (1100 kept, all packed)
// took 62 us instead of 26 (24 with the present selection), and one of 32 x 32768 whose survivors sit in few blocks (equal
// scores) 335 instead of 132 (89).
template <int D, int BITS>
__global__ __launch_bounds__(256) void k_commit_scatter(Pools P, CommitLaunch L, CommitScratch C, int share_rows) {
  constexpr int LPR = D / 8, LPT = 2 * LPR;         // lanes per K (V) row, per token
  constexpr int TPW = 64 / LPT;                     // tokens per wave and round
  __shared__ uint16_t so[1024], sq[1024];
  __shared__ uint32_t cnt[16];
  // the units run fastest: workgroups behind a unit's last part end at once, and with the slots fastest they left the CUs
  // with unequal shares of the others (32 units x 32768 positions, total of the commit: 105 to 128 us by their number, where
  // this order took 89)
  const int lu = (int)(blockIdx.x % (unsigned)L.n_units), slot = (int)(blockIdx.x / (unsigned)L.n_units);
  const int gu = L.unit_begin + lu, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, T = L.T;
  // the block whose parts this workgroup falls among: the last one with no more parts in front of it (lane = block)
  const int n_blocks = commit_blocks(T);
  const int4* blocks = C.blocks + (size_t)lu * (n_blocks + 1);
  int block = 0, part = 0;
  int2 base = make_int2(0, 0);
  for (int b0 = 0; b0 <= n_blocks; b0 += 64) {
    const int4 e = blocks[min(b0 + lane, n_blocks)];
    const int in_front = __popcll(__ballot(b0 + lane <= n_blocks && e.z <= slot));
    if (in_front > 0) {
      block = b0 + in_front - 1;
      base = make_int2(__builtin_amdgcn_readlane(e.x, in_front - 1), __builtin_amdgcn_readlane(e.y, in_front - 1));
      part = slot - __builtin_amdgcn_readlane(e.z, in_front - 1);
    }
    if (in_front < 64) break;
  }
  if (block == n_blocks) return;                    // behind the last part
  const int j0 = 1024 * block;
  const uint16_t* K = L.k + (size_t)lu * T * D;
  const uint16_t* V = L.v + (size_t)lu * T * D;
  const float2* pre = L.pre + (size_t)lu * T;
  int no, nq, parts;
  {
    const uint64_t thr_o = P.thr[(size_t)gu * 2], thr_b = P.thr[(size_t)gu * 2 + 1];
    uint32_t sb[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) sb[r] = C.scores[(size_t)lu * C.pitch + min(j0 + 256 * r + tid, T - 1)];
    bool o[4], q[4];
    int po[4], pq[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = j0 + 256 * r + tid;
      const uint64_t key = ((uint64_t)sb[r] << 32) | (0xFFFFFFFFu - (uint32_t)i);
      o[r] = i < T && (sb[r] == kNoScore || key >= thr_o);           // kNoScore: window position
      q[r] = i < T && !o[r] && key >= thr_b;
      const unsigned long long bo = __ballot(o[r]), bq = __ballot(q[r]);
      po[r] = place(bo, lane); pq[r] = place(bq, lane);
      if (lane == 0) cnt[4 * r + w] = (uint32_t)__popcll(bo) | ((uint32_t)__popcll(bq) << 16);
    }
    __syncthreads();
    uint32_t run = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      if (e % 4 == w) {
        const int r = e / 4;
        if (o[r]) so[(run & 0xFFFFu) + po[r]] = (uint16_t)(256 * r + tid);
        if (q[r]) sq[(run >> 16) + pq[r]] = (uint16_t)(256 * r + tid);
      }
      run += cnt[e];
    }
    no = (int)(run & 0xFFFFu); nq = (int)(run >> 16);
    parts = (int)commit_parts((uint32_t)(no + nq), share_rows);
  }
  __syncthreads();
  const int o0 = no * part / parts, o1 = no * (part + 1) / parts, q0 = nq * part / parts, q1 = nq * (part + 1) / parts;
  const size_t ob = (size_t)gu * P.capO + base.x, qb = (size_t)gu * P.capQ + base.y;
  const int t = lane / LPT, sl = lane % LPT;        // token of the wave's round, lane inside it: K row, then V row
  constexpr int ROUND = 4 * TPW;                    // tokens of the workgroup's round
  {
    const uint16_t* src = (sl < LPR ? K : V) + (size_t)j0 * D + (sl % LPR) * 8;
    uint16_t* dst = (sl < LPR ? P.ok : P.ov) + ob * D + (sl % LPR) * 8;
    constexpr int U = 4;                            // rounds in flight
    for (int i0 = o0 + w * TPW + t; i0 < o1; i0 += ROUND * U) {
      u32x4t v[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + ROUND * u < o1) v[u] = *reinterpret_cast<const u32x4t*>(src + (size_t)so[i0 + ROUND * u] * D);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (i0 + ROUND * u < o1) *reinterpret_cast<u32x4t*>(dst + (size_t)(i0 + ROUND * u) * D) = v[u];
    }
  }
  for (int i = o0 + tid; i < o1; i += 256) { const int j = j0 + so[i]; P.opos[ob + i] = j; P.oacc[ob + i] = pre[j]; }
  // (all lanes of a wave stay together: the quantiser exchanges values between them)
  for (int i0 = q0 + w * TPW; i0 < q1; i0 += ROUND) {
    const int i = i0 + t, j = j0 + sq[min(i, q1 - 1)];
    quantize_into<D, BITS>(P, gu, base.y + i, K + (size_t)j * D, V + (size_t)j * D, sl, i < q1);
  }
  for (int i = q0 + tid; i < q1; i += 256) { const int j = j0 + sq[i]; P.qpos[qb + i] = j; P.qacc[qb + i] = pre[j]; }
}

// The selection by itself (parity hook): thresholds of a list of scores whose keys are a commit's.
template <bool IN_LDS>
__global__ __launch_bounds__(1024) void k_select_probe(const uint32_t* scores, int n, int k0, int k1, uint64_t* thr) {
  extern __shared__ __align__(16) uint32_t row_word[];
  __shared__ __align__(16) SelectLds<typename std::conditional<IN_LDS, uint16_t, uint32_t>::type> sel;
  const int tid = threadIdx.x, nq = quads(n);
  ScoreRange range;
  for (int i = tid; i < kQuad * nq; i += 1024) {
    const uint32_t sb = i < n ? scores[i] : kNoScore;
    range.add(sb);
    if constexpr (IN_LDS) row_word[i] = sb;
  }
  __syncthreads();
  auto score_of = [&](int i) -> uint32_t {
    if constexpr (IN_LDS) return row_word[i];
    else return i < n ? scores[i] : kNoScore;
  };
  auto load = [&](int q, uint32_t (&s)[4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = score_of(kQuad * q + 4 * tid + e);
  };
  auto key_of = [&](int i) -> uint64_t { return ((uint64_t)score_of(i) << 32) | (0xFFFFFFFFu - (uint32_t)i); };
  select_two(nq, load, score_of, key_of, range, k0, k1, sel);
  if (tid < 2) thr[tid] = sel.thr[tid];
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
// One workgroup of 1024 threads per unit with a 32-bit word of LDS per row (whole rounds of the selection).
template <typename... Params, typename... Args>
static hipError_t launch_rows(void (*kernel)(Params...), dim3 grid, int lds_rows, hipStream_t s, Args... args) {
  const size_t shm = (size_t)quads(lds_rows) * kQuad * sizeof(uint32_t);
  if (shm > 32 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, grid, dim3(1024), shm, s, args...);
  return hipGetLastError();
}

static int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

template <int D, int BITS>
static void launch_tailor_moves(const Pools& P, const TailorLaunch& a, hipStream_t s) {
  dim3 gq(clampi((P.capQ + 3) / 4, 1, 256), a.n_units), go(clampi((P.capO + 3) / 4, 1, 256), a.n_units);
  hipLaunchKernelGGL((k_tailor_move_q<D, BITS>), gq, dim3(256), 0, s, P, a);
  hipLaunchKernelGGL((k_tailor_move_o<D>), go, dim3(256), 0, s, P, a);
}

// Workgroups of a unit that score its rows where they have the step's logits to turn into probabilities: a CU reads 28 bytes a
// row (G = 4) and writes 16, which takes one 9 us for 8192 rows.  Spread over several, the scores' way through memory and the
// ticket cost about 4 us (a step with a tailor, one workgroup / several: 32 units x 8192 rows 42.2 / 39.6 us, 8 x 6000 30.9 /
// 29.3, 8 x 30000 69.0 / 54.8, 32 x 4000 32.0 / 31.8, 8 x 3000 25.2 / 25.9, 8 x 1200 23.0 / 24.2).
static int tailor_parts(int n_units, int max_rows) {
  return max_rows <= kQuad ? 1 : std::max(1, std::min((max_rows + 1023) / 1024, 256 / n_units));
}

hipError_t launch_tailor(const Pools& P, const TailorLaunch& a, hipStream_t s) {
  if (a.n_pending > 0 && !a.kept) {
    hipError_t e = launch_flush_scores(P, a.unit_begin, a.n_units, a.n_pending, a.slot, s);
    if (e != hipSuccess) return e;
  }
  // the scores of a unit stay in LDS between the passes where they fit
  const bool lds = a.max_rows <= kLdsRows;
  const int rows = lds ? a.max_rows : 0;
  const dim3 grid(a.n_units, lds && a.kept ? tailor_parts(a.n_units, a.max_rows) : 1);
#define ARKV_CH(G_)                                                                                                     \
  case G_:                                                                                                              \
    e = a.kept ? (lds ? launch_rows(k_tailor_choose<G_, true, true>, grid, rows, s, P, a)                               \
                      : launch_rows(k_tailor_choose<G_, false, true>, grid, rows, s, P, a))                             \
               : (lds ? launch_rows(k_tailor_choose<G_, true, false>, grid, rows, s, P, a)                              \
                      : launch_rows(k_tailor_choose<G_, false, false>, grid, rows, s, P, a));                           \
    break;
  hipError_t e = hipErrorInvalidValue;
  switch (P.G) { ARKV_CH(1) ARKV_CH(2) ARKV_CH(4) ARKV_CH(8) }
  if (e != hipSuccess) return e;
#undef ARKV_CH
  if (a.few_moves) return hipSuccess;                       // done by the choosing workgroups
  if (P.D == 128 && P.bits == 4) launch_tailor_moves<128, 4>(P, a, s);
  else if (P.D == 128 && P.bits == 2) launch_tailor_moves<128, 2>(P, a, s);
  else if (P.D == 64 && P.bits == 4) launch_tailor_moves<64, 4>(P, a, s);
  else if (P.D == 64 && P.bits == 2) launch_tailor_moves<64, 2>(P, a, s);
  else if (P.D == 128 && P.bits == 8) launch_tailor_moves<128, 8>(P, a, s);
  else if (P.D == 64 && P.bits == 8) launch_tailor_moves<64, 8>(P, a, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// The layer's budgets (per sequence: Original target and survivor count) reach the device as launch
// arguments, so that the commit stays ordered on the caller's stream without a staging buffer.
__global__ void k_set_budgets(int32_t* n_o, int32_t* nb, int unit_begin, int hkv, int seq0, int n_seq, BudgetArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_seq * hkv) return;
  const int u = unit_begin + seq0 * hkv + i;
  n_o[u] = a.n_o[i / hkv];
  nb[u] = a.nb[i / hkv];
}

static BudgetArgs budget_args(const int32_t* n_o_seq, const int32_t* nb_seq, int n) {
  BudgetArgs a;
  for (int i = 0; i < 64; ++i) { a.n_o[i] = i < n ? n_o_seq[i] : 0; a.nb[i] = i < n ? nb_seq[i] : 0; }
  return a;
}

static void launch_set_budgets(const Pools& P, int unit_begin, int hkv, int batch, const int32_t* n_o_seq,
                               const int32_t* nb_seq, hipStream_t s) {
  for (int s0 = 0; s0 < batch; s0 += 64) {
    const int n = batch - s0 < 64 ? batch - s0 : 64;
    hipLaunchKernelGGL(k_set_budgets, dim3((n * hkv + 255) / 256), dim3(256), 0, s, P.n_o, P.nb, unit_begin, hkv, s0, n,
                       budget_args(n_o_seq + s0, nb_seq + s0, n));
  }
}

static int commit_pitch(int T) { return (T + 3) / 4 * 4; }
size_t commit_scratch_words(int n_units, int T) {       // 8-byte words; the blocks' entries are 16-byte aligned
  return (size_t)n_units * ((size_t)commit_pitch(T) / 2 + (size_t)commit_ranges(T) + 2 * ((size_t)commit_blocks(T) + 1)) + 1;
}
static CommitScratch commit_scratch(uint64_t* p, int n_units, int T) {
  CommitScratch c;
  c.pitch = commit_pitch(T);
  c.scores = reinterpret_cast<uint32_t*>(p);
  uint64_t* ranges = p + (size_t)n_units * c.pitch / 2;
  c.ranges = reinterpret_cast<uint2*>(ranges);
  c.blocks = reinterpret_cast<int4*>(p + (((size_t)(ranges - p) + (size_t)n_units * commit_ranges(T) + 1) / 2 * 2));
  return c;
}
// the key of the unit's i-th position in a commit's scratch (0: not ranked)
uint64_t commit_key(const uint32_t* scores, int i) {
  return scores[i] == kNoScore ? 0 : ((uint64_t)scores[i] << 32) | (0xFFFFFFFFu - (uint32_t)i);
}
int commit_score_pitch(int T) { return commit_pitch(T); }

hipError_t launch_commit(const Pools& P, const CommitLaunch& a, int hkv, const int32_t* n_o_seq, const int32_t* nb_seq,
                         uint64_t* scratch, hipStream_t s) {
  const int batch = a.n_units / hkv;
  const bool with_keys = a.select && batch <= 64;           // the budgets ride with the keys' launch
  if (!with_keys) launch_set_budgets(P, a.unit_begin, hkv, batch, n_o_seq, nb_seq, s);
  if (!a.select) {
    // a workgroup per round of its four waves while they are few, then 64 per CU that go through the rows side by side (32
    // units x 16384 rows: 99 us at 16384 workgroups, 103 at 8192, 111 at 2048; 8 x 16384: 28.6, 27.9, 29.4)
    const int rounds = (a.T + 4 * (256 / P.D) - 1) / (4 * (256 / P.D));
    const dim3 grid(clampi(rounds, 1, std::max(1, 16384 / a.n_units)), a.n_units);
    if (P.D == 128) hipLaunchKernelGGL(k_commit_copy<128>, grid, dim3(256), 0, s, P, a);
    else hipLaunchKernelGGL(k_commit_copy<64>, grid, dim3(256), 0, s, P, a);
    return hipGetLastError();
  }
  const CommitScratch c = commit_scratch(scratch, a.n_units, a.T);
  const BudgetArgs budgets = budget_args(n_o_seq, nb_seq, with_keys ? batch : 0);
  // Short prompts: the selecting workgroup forms its unit's scores itself and a launch falls away (a whole ingest, with / without
  // the scores' own launch: 8 units x 1000 positions 43.5 / 40.8 us, 32 x 2000 52.3 / 49.3, 8 x 4000 44.3 / 41.8, 8 x 8192 58.0 /
  // 57.0, 32 x 8192 88.5 / 87.5; beyond that one CU takes longer over 8 bytes a position than the launch).
  const bool fused = with_keys && a.T <= kFusedRows;
  if (!fused)
    hipLaunchKernelGGL(k_commit_keys, dim3((a.T + 255) / 256, a.n_units), dim3(256), 0, s, P, a, c, with_keys ? hkv : 0, budgets);
  int kept = 0;                                             // the most rows that a unit keeps
  for (int i = 0; i < batch; ++i) kept = std::max(kept, std::min(nb_seq[i], a.T - a.window) + a.window);
  // about four workgroups per CU; below 8 rows a workgroup's lists cost more than its rows (8 units x 1000 positions, 500
  // kept: 21 us for the whole commit, 52 in one part per block), above 96 nothing is gained (32 units x 32768 positions,
  // 6152 kept: 89 to 95 us at 64 to 1024 rows; all with an earlier selection that took 2 and 12 us more)
  const int share_rows = clampi((int)((long long)a.n_units * kept / 1024 + 7) / 8 * 8, 8, 96);
  const hipError_t e = fused ? launch_rows(k_commit_select<true, true>, dim3(a.n_units), a.T, s, P, a, c, share_rows, hkv, budgets)
                       : a.T <= kLdsRows ? launch_rows(k_commit_select<true, false>, dim3(a.n_units), a.T, s, P, a, c, share_rows, hkv, budgets)
                                         : launch_rows(k_commit_select<false, false>, dim3(a.n_units), 0, s, P, a, c, share_rows, hkv, budgets);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)a.n_units * (unsigned)(kept / share_rows + commit_blocks(a.T)));   // (a block's last part may be short)
#define ARKV_SC(D_, B_)                                                                                                      \
  if (P.D == D_ && P.bits == B_) {                                                                                           \
    hipLaunchKernelGGL((k_commit_scatter<D_, B_>), grid, dim3(256), 0, s, P, a, c, share_rows);                              \
    return hipGetLastError();                                                                                                \
  }
  ARKV_SC(128, 4) ARKV_SC(128, 2) ARKV_SC(128, 8) ARKV_SC(64, 4) ARKV_SC(64, 2) ARKV_SC(64, 8)
#undef ARKV_SC
  return hipErrorInvalidValue;
}

bool select_in_lds(int n) { return n <= kLdsRows; }
hipError_t launch_select_probe(const uint32_t* scores, int n, int k0, int k1, bool in_lds, uint64_t* thr, hipStream_t s) {
  return in_lds ? launch_rows(k_select_probe<true>, dim3(1), n, s, scores, n, k0, k1, thr)
                : launch_rows(k_select_probe<false>, dim3(1), 0, s, scores, n, k0, k1, thr);
}

}  // namespace arkv
