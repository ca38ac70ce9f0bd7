// Prefill scorer (Sec. IV-C eqs. 2-5, and the first samples of the eq. 9 moments).
//
// Per unit (sequence, kv-head) the last W queries of the G heads of the group form M = G*W query
// rows; their logits against all T keys are a dense [T x d] x [d x M] contraction -> MFMA
// (v_mfma_f32_32x32x16_bf16, keys on the M side so that a lane owns ONE query row and the softmax
// statistics of a row are in-register reductions).  The causal softmax needs each row's max and
// sum before any probability exists, so the keys are streamed twice:
//   k_prefill_rows     per (key chunk, unit): row max / row sum partials
//   k_prefill_rowfinal per unit: c_r = max_r + log2(sum_r)
//   k_prefill_cols     per (key chunk, unit): p = 2^(x - c_r); per key sum_r p and sum_r p^2 -> pre
//   k_prefill_stats    per sequence: p_k over keys < T-W aggregated over all heads, entropy,
//                      variance, kurtosis (fp64 reductions; the normaliser's partial sums come from
//                      k_prefill_cols, the last workgroup of a sequence finishes)
#include <type_traits>

#include "arkv_dev.h"

namespace arkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr float kNegBigP = -1.0e30f;

// 2^x as one v_exp_f32 (arguments are <= 0 up to rounding, or hugely negative -> 0)
__device__ __forceinline__ float pexp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <int CTRL>
__device__ __forceinline__ float dpp_p(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL,
                                                               0xf, 0xf, true));
}
// sum over the 32 lanes that share lane/32
__device__ __forceinline__ float sum32(float x) {
  x += dpp_p<0xB1>(x);
  x += dpp_p<0x4E>(x);
  x += dpp_p<0x141>(x);
  x += dpp_p<0x140>(x);
  x += __shfl_xor(x, 16);
  return x;
}

// Stage the unit's query rows in LDS: row r = (head r / W, window query r % W) at byte r*(2D+16), rows >= M
// zero.  q points at the unit's first head; heads are head_stride elements apart.
template <int D, int NT>
__device__ __forceinline__ void stage_q(unsigned char* sm, const uint16_t* q, size_t head_stride, int W, int M, int MP) {
  constexpr int RB = 2 * D + 16;
  constexpr int VPR = D / 8;  // uint4 per row
  constexpr int BATCH = 8;    // loads in flight per thread (one at a time, every load costs a memory round trip)
  for (int i0 = threadIdx.x; i0 < MP * VPR; i0 += NT * BATCH) {
    uint4 v[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int i = i0 + b * NT, r = i / VPR, c = i % VPR;
      v[b] = make_uint4(0, 0, 0, 0);
      if (r < M) v[b] = *reinterpret_cast<const uint4*>(q + (size_t)(r / W) * head_stride + (size_t)(r % W) * D + c * 8);
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int i = i0 + b * NT, r = i / VPR, c = i % VPR;
      if (i < MP * VPR) *reinterpret_cast<uint4*>(sm + (size_t)r * RB + c * 16) = v[b];
    }
  }
}

template <int D>
__device__ __forceinline__ void load_keys(u32x4 (&kf)[D / 16], const uint16_t* k, int j0, int T, int lane) {
  int key = j0 + (lane & 31);
  if (key > T - 1) key = T - 1;
  const uint16_t* p = k + (size_t)key * D + (lane >> 5) * 8;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) kf[kk] = *reinterpret_cast<const u32x4*>(p + kk * 16);
}

// One step of the two passes' software pipeline: the D/16 MFMAs that form the NEXT step's 32x32 logits tile
// (key operands kx, query operands of row tile rt_next read from LDS two MFMAs ahead), with the vector work on
// THIS step's tile dealt out between them by `work(kk)`.  A wave's MFMAs only run in the background of its own
// vector instructions if the two alternate in the instruction stream, and left to itself the compiler groups
// them apart (scheduling barriers do not help: the instruction selector has already grouped them).  The order is
// therefore pinned by data: after slot kk an empty volatile asm takes the two running sums of the vector work
// (p0, p1: every slot's work must read and write them) together with the key operand of MFMA kk + 1, so that
// work(kk) lies before it and MFMA kk + 1 after it.
// KEYS_ON_M: the keys are the MFMA's M side (a lane owns one query row), else its N side (a lane owns one key).
// qoff: the lane's byte offset inside a row tile, (lane % 32) * row pitch + (lane / 32) * 16; it goes through an
// empty asm so that the optimiser cannot hoist the LDS reads (the same for every key tile) out of the key loop,
// where they would take 32 RT registers.
// LDS operands are requested this many MFMAs ahead, across steps (a whole step ahead measured the same and costs
// 16 registers more)
template <int D> constexpr int kQAheadOf = 3;

// The first kQAhead operands of row tile rt: what a step expects to be in flight when it starts.
template <int D>
__device__ __forceinline__ void prime_operands(uint4 (&qb)[kQAheadOf<D> + 1], const unsigned char* sm, int rt, int qoff) {
  constexpr int RB = 2 * D + 16;
  constexpr int kQAhead = kQAheadOf<D>;
  asm volatile("" : "+v"(qoff));
#pragma unroll
  for (int i = 0; i < kQAhead; ++i) qb[i] = *reinterpret_cast<const uint4*>(sm + rt * 32 * RB + qoff + i * 32);
}

// rt_next: the row tile whose logits this step's MFMAs form; rt_after: the row tile of the step after it, whose
// first kQAhead operands are requested in this step's last slots (ring qb, slot = operand index % (kQAhead + 1);
// D/16 is a multiple of the ring size, so the slots line up from step to step).
template <int D, bool KEYS_ON_M, typename Work>
__device__ __forceinline__ f32x16 pipeline_step(u32x4 (&kx)[D / 16], uint4 (&qb)[kQAheadOf<D> + 1], const unsigned char* sm,
                                                int rt_next, int rt_after, int qoff, float& p0, float& p1, Work work) {
  constexpr int RB = 2 * D + 16;
  constexpr int KK = D / 16;
  constexpr int kQAhead = kQAheadOf<D>;
  static_assert(KK % (kQAhead + 1) == 0 && KK > kQAhead, "ring slots must line up across steps");
  asm volatile("" : "+v"(qoff));
  const unsigned char* qrow = sm + rt_next * 32 * RB + qoff;
  const unsigned char* qrow2 = sm + rt_after * 32 * RB + qoff;
  f32x16 C = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int ahead = kk + kQAhead;
    qb[ahead % (kQAhead + 1)] = *reinterpret_cast<const uint4*>(ahead < KK ? qrow + ahead * 32 : qrow2 + (ahead - KK) * 32);
    const uint4 qc = qb[kk % (kQAhead + 1)];
    if constexpr (KEYS_ON_M)
      C = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kx[kk]), __builtin_bit_cast(bf16x8, qc), C, 0, 0, 0);
    else
      C = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, qc), __builtin_bit_cast(bf16x8, kx[kk]), C, 0, 0, 0);
    work(kk);
    if (kk + 1 < KK) {
      // (resident since the previous key tile: pinning it waits for nothing)
      asm volatile("" : "+v"(p0), "+v"(p1), "+v"(kx[kk + 1]));
    }
  }
  return C;
}

// NW waves per workgroup: 4, or 8 where the staged queries leave room for only one workgroup per CU (more than
// 256 query rows), so that a SIMD still has two waves.
// Logits tile of the first pass: C[i] at key j0 + 8(i/4) + 4(lane/32) + i%4, row rt*32 + lane%32.
template <int D, int RT, int NW>
__global__ __launch_bounds__(64 * NW, (NW == 4 && RT < 8) ? 3 : 2) void k_prefill_rows(PrefillLaunch L) {
  extern __shared__ __align__(16) unsigned char sm[];
  constexpr int NT = 64 * NW;
  constexpr int KK = D / 16;
  const int chunk = blockIdx.x, u = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int M = L.G * L.W, MP = RT * 32, T = L.T;
  stage_q<D, NT>(sm, L.q_win + (size_t)u * L.G * L.q_head_stride, L.q_head_stride, L.W, M, MP);
  __syncthreads();
  const uint16_t* k = L.k + (size_t)u * T * D;
  float m[RT], l[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) { m[rt] = kNegBigP; l[rt] = 0.f; }
  const int jbeg = chunk * L.chunk, jend = min(jbeg + L.chunk, T);
  const int qoff = (lane & 31) * (2 * D + 16) + (lane >> 5) * 16;
  const float scale2 = L.scale2;
  u32x4 kf[KK], kn[KK];
  if (jbeg + w * 32 < jend) load_keys<D>(kf, k, jbeg + w * 32, T, lane);
  float pin0 = 0.f, pin1 = 0.f;
  uint4 qb[kQAheadOf<D> + 1];
  prime_operands<D>(qb, sm, 0, qoff);
  f32x16 C = pipeline_step<D, true>(kf, qb, sm, 0, RT > 1 ? 1 : 0, qoff, pin0, pin1, [](int) {});
  // One key tile against all row tiles; every step also issues the next step's MFMAs.  FULL: no key of the tile
  // is masked for any row (padded rows are rows of zeros whose statistics nobody reads), and then nothing in the
  // body branches.
  auto key_tile = [&](int j0, auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
    load_keys<D>(kn, k, j0 + 32 * NW, T, lane);        // next tile of this wave (clamped past the end)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float x[16];
      float mn = 0.f, s = 0.f;
      auto work = [&](int kk) {
        if (kk == 0) {
          if constexpr (FULL) {
            // the scale is positive, so the maximum is taken on the raw dot products
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = C[i];
            float mt = fmaxf(x[0], x[1]);
#pragma unroll
            for (int i = 2; i < 16; i += 2) mt = fmaxf(fmaxf(mt, x[i]), x[i + 1]);
            mn = fmaxf(m[rt], mt * scale2);
          } else {
            const int r = rt * 32 + (lane & 31);
            const int lastv = r < M ? T - L.W + (r % L.W) : -1;   // last visible key of this row
            float mt = kNegBigP;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int j = j0 + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3);
              x[i] = j <= lastv ? C[i] * scale2 : kNegBigP;       // scaled here: the sentinel stays the sentinel
              mt = fmaxf(mt, x[i]);
            }
            mn = fmaxf(m[rt], mt);
          }
          s = l[rt] * pexp2(m[rt] - mn);
        } else {
          // the 16 logits are dealt over the remaining KK - 1 slots; FULL: 2^(scale x - max) is one fma and one exp
          const int i0 = (kk - 1) * 16 / (KK - 1), i1 = kk * 16 / (KK - 1);
#pragma unroll
          for (int i = i0; i < i1; ++i) {
            if constexpr (FULL) s += pexp2(fmaf(x[i], scale2, -mn));
            else s += pexp2(x[i] - mn);                           // masked entries: 2^(-1e30 - mn) = 0
          }
        }
      };
      constexpr int RT2 = RT > 1 ? 1 : 0;          // the row tile after row tile 0
      const f32x16 Cn = rt + 1 < RT ? pipeline_step<D, true>(kf, qb, sm, rt + 1, rt + 2 < RT ? rt + 2 : 0, qoff, mn, s, work)
                                    : pipeline_step<D, true>(kn, qb, sm, 0, RT2, qoff, mn, s, work);
      if constexpr (!FULL) { if (!(mn > 0.5f * kNegBigP)) s = 0.f; }      // nothing visible yet: 16 * 2^0 dropped
      m[rt] = mn; l[rt] = s;
      C = Cn;
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = kn[kk];
  };
  int j0 = jbeg + w * 32;
  for (; j0 < jend && j0 + 32 <= T - L.W; j0 += 32 * NW) key_tile(j0, std::true_type{});
  for (; j0 < jend; j0 += 32 * NW) key_tile(j0, std::false_type{});
  // merge the two lane halves, then the waves
  float* red = reinterpret_cast<float*>(sm);   // reuse after everyone is done with the queries
  __syncthreads();
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const float mo = __shfl_xor(m[rt], 32), lo = __shfl_xor(l[rt], 32);
    const float mn = fmaxf(m[rt], mo);
    l[rt] = l[rt] * exp2f(m[rt] - mn) + lo * exp2f(mo - mn);
    m[rt] = mn;
    if (lane < 32) { red[(w * MP + rt * 32 + lane) * 2] = m[rt]; red[(w * MP + rt * 32 + lane) * 2 + 1] = l[rt]; }
  }
  __syncthreads();
  for (int r = tid; r < MP; r += NT) {
    float mn = kNegBigP;
    for (int i = 0; i < NW; ++i) mn = fmaxf(mn, red[(i * MP + r) * 2]);
    float s = 0.f;
    for (int i = 0; i < NW; ++i) s += red[(i * MP + r) * 2 + 1] * exp2f(red[(i * MP + r) * 2] - mn);
    L.rowstat[((size_t)u * L.n_chunks + chunk) * MP + r] = make_float2(mn, s);
  }
}

__global__ __launch_bounds__(256) void k_prefill_rowfinal(PrefillLaunch L, int MP, float* rowc) {
  // grid (MP/32, U): 32 rows per workgroup, 8 threads per row share the chunks
  __shared__ float sm_m[32][8], sm_s[32][8];
  const int u = blockIdx.y, r = blockIdx.x * 32 + (threadIdx.x >> 3), part = threadIdx.x & 7;
  float mn = kNegBigP;
  for (int c = part; c < L.n_chunks; c += 8) mn = fmaxf(mn, L.rowstat[((size_t)u * L.n_chunks + c) * MP + r].x);
  sm_m[threadIdx.x >> 3][part] = mn;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) mn = fmaxf(mn, sm_m[threadIdx.x >> 3][i]);
  float s = 0.f;
  for (int c = part; c < L.n_chunks; c += 8) {
    const float2 t = L.rowstat[((size_t)u * L.n_chunks + c) * MP + r];
    s += t.y * pexp2(t.x - mn);
  }
  sm_s[threadIdx.x >> 3][part] = s;
  __syncthreads();
  if (part == 0) {
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) tot += sm_s[threadIdx.x >> 3][i];
    rowc[(size_t)u * MP + r] = tot > 0.f ? mn + log2f(tot) : 0.f;
  }
}

__device__ __forceinline__ double block_sum_d(double v, double* sm) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sm[w] = v;
  __syncthreads();
  double t = 0;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sm[i];
  return t;
}

// the same for N values at once: one pair of barriers
template <int N>
__device__ __forceinline__ void block_sums_d(double (&v)[N], double* sm /*[N][4]*/) {
#pragma unroll
  for (int k = 0; k < N; ++k)
    for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) sm[4 * k + w] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    v[k] = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[k] += sm[4 * k + i];
  }
}

// c_r = max + log2(sum) of a row from the first pass's partials per key chunk (rowstat: the row's first, MP apart), by one
// thread.  Partials are requested 16 at a time and added in CHAINS chains: one for up to 16 chunks, eight for more, as in
// k_prefill_rowfinal, from whose bits this can differ where a later batch moves the maximum.
template <int CHAINS>
__device__ __forceinline__ float row_constant(const float2* rowstat, int n_chunks, int MP) {
  float mn = kNegBigP, s[CHAINS];
#pragma unroll
  for (int i = 0; i < CHAINS; ++i) s[i] = 0.f;
  for (int c0 = 0; c0 < n_chunks; c0 += 16) {
    float2 t[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) t[i] = rowstat[(size_t)min(c0 + i, n_chunks - 1) * MP];
    float m = mn;
#pragma unroll
    for (int i = 0; i < 16; ++i) m = fmaxf(m, t[i].x);
    const float f = pexp2(mn - m);
#pragma unroll
    for (int i = 0; i < CHAINS; ++i) s[i] *= f;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (c0 + i < n_chunks) s[i % CHAINS] += t[i].y * pexp2(t[i].x - m);
    mn = m;
  }
  float tot = s[0];
#pragma unroll
  for (int i = 1; i < CHAINS; ++i) tot += s[i];
  return tot > 0.f ? mn + log2f(tot) : 0.f;
}

// The same of 8 GROUPS rows (r, r + 8 waves, ...) from up to 8 J chunks, by a wave: eight lanes a row, each every eighth chunk,
// added up in k_prefill_rowfinal's order, so that a constant's bits do not depend on which of the two forms it.  All partials
// are requested together and stay in registers between the maximum and the sum.
template <int MP, int NW, int J, int GROUPS>
__device__ __forceinline__ void row_constants_of(const float2* rowstat, int n_chunks, int r, int M, float* crow) {
  const int lane = threadIdx.x & 63, part = lane >> 3;
  float2 t[GROUPS][J];
#pragma unroll
  for (int g = 0; g < GROUPS; ++g)
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int c = part + 8 * j;
      const unsigned at = (unsigned)(min(c, n_chunks - 1) * MP + r + 8 * NW * g) * 8u;
      t[g][j] = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(rowstat) + at);
      if (c >= n_chunks) t[g][j].y = 0.f;                 // (adds nothing; its maximum is another's)
    }
#pragma unroll
  for (int g = 0; g < GROUPS; ++g) {
    float m = kNegBigP, s = 0.f, tot = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j) m = fmaxf(m, t[g][j].x);
#pragma unroll
    for (int o = 8; o < 64; o *= 2) m = fmaxf(m, __shfl_xor(m, o));
#pragma unroll
    for (int j = 0; j < J; ++j) s += t[g][j].y * pexp2(t[g][j].x - m);
#pragma unroll
    for (int p = 0; p < 8; ++p) tot += __shfl(s, 8 * p + (lane & 7));
    const int row = r + 8 * NW * g;
    if (part == 0) crow[row] = row < M ? -(tot > 0.f ? m + log2f(tot) : 0.f) : kNegBigP;
  }
}

// crow[r] = -c_r of all rows, by the whole workgroup, from 17 to 64 chunks.  Up to 128 rows (the whole scorer with eight lanes / a
// thread per row: 256 rows 5 % slower, 128 rows the same, 64 and 32 rows 2 to 9 % faster, d = 128, 8 units x 6000 keys 20.1 / 21.4 us;
// beyond 64 chunks 16 partials a lane at a time leave too few rows in flight, 128 rows 7 to 27 % slower).
constexpr int kWaveChunks = 64, kWaveRows = 128;
template <int MP, int NW>
__device__ __forceinline__ void row_constants(const float2* rowstat, int n_chunks, int M, float* crow) {
  constexpr int ALL = MP / (8 * NW);                      // groups of eight rows per wave
  const int r0 = 8 * (threadIdx.x >> 6) + (threadIdx.x & 7);
  auto all = [&](auto j) {
    constexpr int J = decltype(j)::value, GROUPS = ALL < 16 / J ? ALL : 16 / J;
#pragma unroll 1
    for (int i = 0; i < ALL; i += GROUPS) row_constants_of<MP, NW, J, GROUPS>(rowstat, n_chunks, r0 + 8 * NW * i, M, crow);
  };
  using std::integral_constant;
  if (n_chunks <= 32) all(integral_constant<int, 4>()); else all(integral_constant<int, 8>());
}

// Second pass.  Here the MFMA is turned round (query rows on the M side, keys on the N side) so that a
// lane owns ONE key and the sums over the M = G*W query rows are in-register additions: C[i] is row
// rt*32 + 8(i/4) + 4(lane/32) + i%4 against key j0 + lane%32.  The row constants c_r come from LDS.
// (The launch bounds keep the prologue from taking more registers than the loop: 96 at d = 64.)
template <int D, int RT, int NW>
__global__ __launch_bounds__(64 * NW, NW > 4 ? 2 : D == 64 && RT <= 4 ? 5 : 3) void k_prefill_cols(PrefillLaunch L, const float* rowc, double* zpart) {
  extern __shared__ __align__(16) unsigned char sm[];
  constexpr int RB = 2 * D + 16;
  constexpr int NT = 64 * NW;
  constexpr int KK = D / 16;
  const int chunk = blockIdx.x, u = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int M = L.G * L.W, MP = RT * 32, T = L.T;
  stage_q<D, NT>(sm, L.q_win + (size_t)u * L.G * L.q_head_stride, L.q_head_stride, L.W, M, MP);
  float* crow = reinterpret_cast<float*>(sm + (size_t)MP * RB);   // [MP] -c_r (padded rows: -1e30 -> p = 0)
  int* lastk = reinterpret_cast<int*>(crow + MP);                 // [MP] last visible key of the row
  const bool by_wave = MP <= kWaveRows && L.merge_rows && L.n_chunks > 16 && L.n_chunks <= kWaveChunks;
  const float2* rowstat = L.rowstat + (size_t)u * L.n_chunks * MP;
  if constexpr (RT * 32 <= kWaveRows) {
    if (by_wave) row_constants<RT * 32, NW>(rowstat, L.n_chunks, M, crow);
  }
  for (int r = tid; r < MP; r += NT) {
    // the row constant in base-2 units: from the first pass / the attention pass, or from the caller's
    // log-sum-exp (natural log of the sum over visible keys of exp(scale q.k), what attention kernels commonly
    // return per query row; row r = (head inside the group) * W + (window query))
    float cr = 0.f;
    if (L.merge_rows) {
      if (!by_wave) cr = L.n_chunks <= 16 ? row_constant<1>(rowstat + r, L.n_chunks, MP) : row_constant<8>(rowstat + r, L.n_chunks, MP);
    } else if (r < M) cr = L.lse ? L.lse[((size_t)u * L.G + r / L.W) * L.W + r % L.W] * 1.4426950408889634f : rowc[(size_t)u * MP + r];
    if (!by_wave) crow[r] = r < M ? -cr : kNegBigP;
    lastk[r] = r < M ? T - L.W + (r % L.W) : -1;
  }
  __syncthreads();
  const uint16_t* k = L.k + (size_t)u * T * D;
  const int jbeg = chunk * L.chunk, jend = min(jbeg + L.chunk, T);
  float2* pre = L.pre + (size_t)u * T;
  const int hl = lane >> 5, kl = lane & 31;
  const int qoff = kl * RB + hl * 16;
  const float scale2 = L.scale2;
  double zacc = 0.0;                                              // this workgroup's share of eq. 3's normaliser
  u32x4 kf[KK], kn[KK];
  if (jbeg + w * 32 < jend) load_keys<D>(kf, k, jbeg + w * 32, T, lane);
  float pin0 = 0.f, pin1 = 0.f;
  uint4 qb[kQAheadOf<D> + 1];
  prime_operands<D>(qb, sm, 0, qoff);
  f32x16 C = pipeline_step<D, false>(kf, qb, sm, 0, RT > 1 ? 1 : 0, qoff, pin0, pin1, [](int) {});
  float4 nc_nxt = *reinterpret_cast<const float4*>(crow + 4 * hl);      // row tile 0, first group
  // FULL: no key of the tile is masked for any row (padded rows have c_r = -1e30, so p = 0 without a test)
  auto key_tile = [&](int j0, auto full_c) {
    constexpr bool FULL = decltype(full_c)::value;
    load_keys<D>(kn, k, j0 + 32 * NW, T, lane);
    const int j = j0 + kl;
    float a1 = 0.f, a2 = 0.f;
    // the row constants are the same for every key tile too: opaque offset, see pipeline_step
    int c0 = 4 * hl;
    asm volatile("" : "+v"(c0));
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      // a slot handles PER logits: rows 8 g4 + 4 hl .. + 3 of the tile for g4 = first logit / 4.  The four row
      // constants of a group are requested from LDS one group ahead (nc_nxt; across steps and key tiles as well:
      // used right after the request, every group would wait for an LDS round trip)
      const int rt_n = rt + 1 < RT ? rt + 1 : 0;        // the tile the next step works on
      float4 nc;
      int4 lk;
      auto work = [&](int kk) {
        static_assert(KK == 8 || KK == 4, "two or four logits per slot");
        constexpr int PER = 16 / KK;                      // logits per slot
        const int i0 = kk * PER;
        if (i0 % 4 == 0) {
          const int g4 = i0 / 4;
          nc = nc_nxt;
          nc_nxt = *reinterpret_cast<const float4*>(crow + (g4 + 1 < 4 ? rt * 32 + 8 * (g4 + 1) : rt_n * 32) + c0);
          if constexpr (!FULL) lk = *reinterpret_cast<const int4*>(lastk + rt * 32 + 8 * g4 + c0);
        }
        const float ncv[4] = {nc.x, nc.y, nc.z, nc.w};
        const int lkv[4] = {lk.x, lk.y, lk.z, lk.w};
#pragma unroll
        for (int i = i0; i < i0 + PER; ++i) {
          float p = pexp2(fmaf(C[i], scale2, ncv[i % 4]));
          if constexpr (!FULL) p = j <= lkv[i % 4] ? p : 0.f;
          a1 += p;
          a2 = fmaf(p, p, a2);
        }
      };
      constexpr int RT2 = RT > 1 ? 1 : 0;          // the row tile after row tile 0
      const f32x16 Cn = rt + 1 < RT ? pipeline_step<D, false>(kf, qb, sm, rt + 1, rt + 2 < RT ? rt + 2 : 0, qoff, a1, a2, work)
                                    : pipeline_step<D, false>(kn, qb, sm, 0, RT2, qoff, a1, a2, work);
      C = Cn;
    }
    a1 += __shfl_xor(a1, 32);
    a2 += __shfl_xor(a2, 32);
    if (hl == 0 && j < T) pre[j] = make_float2(a1, a2);
    if (hl == 0 && j < T - L.W) zacc += (double)a1;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) kf[kk] = kn[kk];
  };
  int j0 = jbeg + w * 32;
  for (; j0 < jend && j0 + 32 <= T - L.W; j0 += 32 * NW) key_tile(j0, std::true_type{});
  for (; j0 < jend; j0 += 32 * NW) key_tile(j0, std::false_type{});
  // sum over the chunk's keys before the window of the attention they received, in a fixed order
  zacc = block_sum_d(zacc, reinterpret_cast<double*>(sm));       // (its first barrier ends the use of the queries)
  if (tid == 0) zpart[(size_t)u * L.n_chunks + chunk] = zacc;
}

// Results that one workgroup writes and another reads inside the same launch go through device-scope relaxed
// atomics (write-through stores, loads that do not hit a stale L2 line of another XCD); no cache-wide flush.
__device__ __forceinline__ void st_dev_d(double* p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double ld_dev_d(const double* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Aggregated key distribution over ALL heads of a sequence and its three statistics (eqs. 3-5), fp64, every
// sum in a fixed order: the normaliser Z from the column pass's per-workgroup sums; per chunk of keys the sums
// of -p ln p, (p - 1/n)^2, (p - 1/n)^4; the workgroup of a sequence that finishes last (a ticket) adds the
// chunks up and writes the statistics.
constexpr int kStatChunk = 512;    // keys per workgroup
// Bound by its chain of round trips and barriers (keys' loads, normaliser, sums, ticket, sums): the keys' loads go out
// before the normaliser is reduced and the three sums share their barriers (2000 keys x 8 heads: 13 -> 8 us).
// Up to 1024 keys one workgroup does it all and the chain ends with the first sums: no ticket, no second reading (the whole
// scorer, 8 heads x 400 keys 19.1 -> 17.5 us, x 600 19.1 -> 17.8, x 1000 19.0 -> 18.5; with 1024 threads for up to 2048 keys the
// logarithms took longer than that saves, 2000 keys 18.7 -> 20.4).

template <int KPT>                  // keys per thread
__global__ __launch_bounds__(256) void k_prefill_stats(PrefillLaunch L, const double* zpart, double* mpart) {
  __shared__ double sm[16];
  __shared__ int last;
  const int b = blockIdx.y, ch = blockIdx.x, n = L.T - L.W, nch = gridDim.x;
  const float2* pre = L.pre + (size_t)b * L.Hkv * L.T;
  // the keys' sums over the heads do not wait for the normaliser: their loads are on the way while it is reduced
  constexpr int kChunk = 256 * KPT;
  double c[KPT];
#pragma unroll
  for (int i = 0; i < KPT; ++i) c[i] = 0;
#pragma unroll 8
  for (int g = 0; g < L.Hkv; ++g)
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      c[i] += (double)pre[(size_t)g * L.T + min(ch * kChunk + (int)threadIdx.x + 256 * i, n - 1)].x;
  double Z = 0;
  for (int i = threadIdx.x; i < L.Hkv * L.n_chunks; i += 256) Z += zpart[(size_t)b * L.Hkv * L.n_chunks + i];
  Z = block_sum_d(Z, sm);
  const double pbar = 1.0 / (double)n;
  double m[3] = {0, 0, 0};            // sums of -p ln p, (p - pbar)^2, (p - pbar)^4
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    if (ch * kChunk + (int)threadIdx.x + 256 * i < n) {
      const double p = c[i] / Z;
      if (p > 0) m[0] -= p * log(p);
      const double d = p - pbar, d2 = d * d;
      m[1] += d2; m[2] += d2 * d2;
    }
  }
  block_sums_d(m, sm);
  if (nch > 1) {                                      // (uniform)
    if (threadIdx.x == 0) {
      double* o = mpart + ((size_t)b * nch + ch) * 3;
      st_dev_d(o, m[0]); st_dev_d(o + 1, m[1]); st_dev_d(o + 2, m[2]);
      __builtin_amdgcn_s_waitcnt(0);                    // the partials are at the device's coherence point
      last = __hip_atomic_fetch_add(L.stat_ticket + b, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nch - 1;
    }
    __syncthreads();
    if (!last) return;
    m[0] = m[1] = m[2] = 0;
    for (int i = threadIdx.x; i < nch; i += 256) {
      const double* o = mpart + ((size_t)b * nch + i) * 3;
      m[0] += ld_dev_d(o); m[1] += ld_dev_d(o + 1); m[2] += ld_dev_d(o + 2);
    }
    block_sums_d(m, sm);
    if (threadIdx.x == 0) __hip_atomic_store(L.stat_ticket + b, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
  }
  if (threadIdx.x != 0) return;
  const double m2 = m[1] / (double)n, m4 = m[2] / (double)n;
  L.stats[b * 3 + 0] = (float)m[0];
  L.stats[b * 3 + 1] = (float)m2;
  L.stats[b * 3 + 2] = m2 > 0 ? (float)(m4 / (m2 * m2)) : 0.f;
}

// Up to kMergeChunks key chunks, or more of them in a launch of up to kMergeGrid workgroups of up to 128 query rows (half as many
// of 256, a quarter of 512), the column pass puts the row constants together itself, in its prologue, and k_prefill_rowfinal, a
// launch of 5 us, is left out.  Otherwise every workgroup of the column pass reads more than the launch costs: 8 bytes per row
// and chunk.  In the column pass / with the launch, us, d = 128, 128 rows: 8 units x 4000 keys (32 chunks) 19.8 / 21.7, 2 x 3000 19.2 /
// 20.8, 32 x 32768 (32) 109.5 / 111.5, 8 x 10000 (79 chunks, 632 workgroups) 33.7 / 34.3, 2 x 32768 (256, 512) 34.6 / 37.3; 16 x 8192
// (64, 1024) 43.3 / 43.6, 8 x 16384 (128, 1024) 49.9 / 47.3, 24 x 10000 (79, 1896) 66.3 / 61.3.  256 rows: 2 x 9000 (141 workgroups)
// 26.5 / 28.3, 4 x 18763 (588, d = 64) 43.6 / 39.7.  512 rows: 1 x 36919 (289) 84.9 / 68.8, 4 x 9324 (292, d = 64) 47.8 / 45.2.
constexpr int kMergeChunks = 32, kMergeGrid = 640;

template <int D, int RT>
static hipError_t launch_prefill_t(const PrefillLaunch& a, float* rowc, hipStream_t s) {
  const int U = a.B * a.Hkv, MP = RT * 32;
  constexpr int NW = RT > 8 ? 8 : 4;
  const size_t shm = (size_t)MP * (2 * D + 16);
  if (shm + (size_t)MP * 8 > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_prefill_rows<D, RT, NW>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_prefill_cols<D, RT, NW>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)(shm + (size_t)MP * 8));
    if (e != hipSuccess) return e;
  }
  dim3 grid(a.n_chunks, U);
  if (!a.have_rowc) {
    hipLaunchKernelGGL((k_prefill_rows<D, RT, NW>), grid, dim3(64 * NW), shm, s, a);
    if (!a.merge_rows) hipLaunchKernelGGL(k_prefill_rowfinal, dim3(MP / 32, U), dim3(256), 0, s, a, MP, rowc);
  }
  const int n = a.T - a.W;
  const bool one = n > kStatChunk && n <= 2 * kStatChunk;      // one workgroup of twice the keys: no ticket
  const int nch = one ? 1 : (n + kStatChunk - 1) / kStatChunk;
  double* zpart = reinterpret_cast<double*>(rowc + (size_t)U * MP);      // [U][n_chunks], then [B][nch][3]
  double* mpart = zpart + (size_t)U * a.n_chunks;
  hipLaunchKernelGGL((k_prefill_cols<D, RT, NW>), grid, dim3(64 * NW), shm + (size_t)MP * 8, s, a, (const float*)rowc, zpart);
  if (one) hipLaunchKernelGGL(k_prefill_stats<2 * kStatChunk / 256>, dim3(nch, a.B), dim3(256), 0, s, a, (const double*)zpart, mpart);
  else hipLaunchKernelGGL(k_prefill_stats<kStatChunk / 256>, dim3(nch, a.B), dim3(256), 0, s, a, (const double*)zpart, mpart);
  return hipGetLastError();
}

// rowc: scratch [U][MP] floats followed by U*n_chunks + 3*B*ceil((T-W)/512) doubles for the statistics partials
hipError_t launch_prefill_stats(const PrefillLaunch& launch, float* rowc, hipStream_t s) {
  PrefillLaunch a = launch;
  const int M = a.G * a.W;
  int RT = 1;
  while (RT * 32 < M) RT *= 2;
  if (RT > 16) return hipErrorInvalidValue;
  const long long wgs = (long long)a.n_chunks * a.B * a.Hkv;
  a.merge_rows = !a.have_rowc && (a.n_chunks <= kMergeChunks || (wgs <= kMergeGrid && 32 * RT * wgs <= 128 * kMergeGrid)) ? 1 : 0;
#define ARKV_PF(D_, RT_) if (a.D == D_ && RT == RT_) return launch_prefill_t<D_, RT_>(a, rowc, s);
  ARKV_PF(128, 1) ARKV_PF(128, 2) ARKV_PF(128, 4) ARKV_PF(128, 8) ARKV_PF(128, 16)
  ARKV_PF(64, 1) ARKV_PF(64, 2) ARKV_PF(64, 4) ARKV_PF(64, 8) ARKV_PF(64, 16)
#undef ARKV_PF
  return hipErrorInvalidValue;
}

}  // namespace arkv
