// Causal prefill attention with the scorer's first pass fused (Sec. IV-C: eq. 2 is a slice of the prompt's
// causal attention, so the pass that computes the prompt's outputs already holds the window rows' softmax
// maxima and sums).
//
// One workgroup = 32 QB query positions of one (sequence, kv-head) x H of the G heads of its group (all of them up to
// G = 4, four or eight at G = 8, see launch_prefill_attn); a wave takes 32
// positions of one head.  QB = 4 / H for H < 4 (else 1), so that at least four waves share every key and value tile,
// which is fetched from HBM once per workgroup and staged
// in LDS (keys in three buffers, values in two, one barrier per 32-key tile); the loads of a tile have two steps to
// arrive (a step takes 0.4-1.1 us, a load that misses the L2 0.5-1 us), and their conversion and way into LDS is
// dealt out between the PV MFMAs of the second.  With one step to arrive and the staging behind the MFMAs: 32768 tokens x
// 8 units 8736 -> 8206 us, 512 x 16411 x 8 units 164 -> 152 us (147 since, see kPrio), 2003 x 32 units (d = 64, G = 1) 43.1 -> 33.0 us;
// the earlier loads alone gave 1 / 4 / 15 %.  Keys are on the M side of the
// logits MFMA (v_mfma_f32_32x32x16_bf16, S^T = K Q^T), which leaves ONE query row per lane: the online softmax
// is per-lane arithmetic (the two lane halves of a row talk only when the row's reference maximum moves, which
// is rare: see the step below).  The probabilities a lane then holds
// (keys 8(i/4) + 4(lane/32) + i%4 of the tile) are, eight at a time, exactly a B operand of the PV MFMA
// (O^T = V^T P^T) if the contraction index is read in that key order; the value tile is staged transposed
// ([channel][key], fp16) with its key columns permuted so that the matching A operand is one 16-byte read.
// Probabilities are rounded to fp16 (values to fp16 exactly: bf16 has fewer mantissa bits; magnitudes
// beyond fp16's range are not supported), accumulation fp32.
#include <hip/hip_fp16.h>

#include "arkv.h"
#include "arkv_dev.h"

namespace arkv {

typedef __bf16 bf16x8a __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8a __attribute__((ext_vector_type(8)));
typedef float f32x16a __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4a __attribute__((ext_vector_type(4)));   // a 16-byte chunk the compiler keeps in registers
// N dwords that one load or store moves
template <int N> struct WordsOf { typedef uint32_t type __attribute__((ext_vector_type(N))); };
template <> struct WordsOf<1> { typedef uint32_t type; };
template <int N> using Words = typename WordsOf<N>::type;
template <int N> __device__ __forceinline__ Words<N> buffer_words(__amdgpu_buffer_rsrc_t r, uint32_t byte) {
  if constexpr (N == 4) return __builtin_amdgcn_raw_buffer_load_b128(r, byte, 0, 0);
  else if constexpr (N == 2) return __builtin_amdgcn_raw_buffer_load_b64(r, byte, 0, 0);
  else return __builtin_amdgcn_raw_buffer_load_b32(r, byte, 0, 0);
}
template <typename V> __device__ __forceinline__ uint32_t word(const V& v, int i) {
  if constexpr (sizeof(V) == 4) return v;
  else return v[i];
}

constexpr float kNegBigA = -1.0e30f;
constexpr int kVtPitch = 40;   // halves per channel row of the transposed value tile: 32 keys + 8 (16-byte reads, 20-dword stride)

__device__ __forceinline__ float aexp2(float x) { return __builtin_amdgcn_exp2f(x); }

// two bf16 values (each in the LOW half of its dword) -> packed fp16 pair (a low, b high)
__device__ __forceinline__ uint32_t bf16_pair_to_f16x2(uint32_t a, uint32_t b) {
  const __half2 h = __floats2half2_rn(__uint_as_float(a << 16), __uint_as_float(b << 16));
  return *reinterpret_cast<const uint32_t*>(&h);
}

// column of key j (0..31) in the transposed value tile: the eight keys 16 jj + 8 a + 4 hh + r (a = 0, 1;
// r = 0..3) that lane half hh contracts in PV step jj sit side by side at 16 jj + 8 hh + 4 a + r
__device__ __forceinline__ int vt_col(int j) { return (j & 16) | ((j & 4) << 1) | ((j & 8) >> 1) | (j & 3); }

template <int D>
struct AttnLds {
  static constexpr int KP = D + 8;              // halves per key row: 16-byte reads of 16 keys hit 64 banks
  uint16_t k[3][32][KP];                        // key tiles t + 1 (logits now), t + 2 (operands prefetched), t + 3 (being staged)
  _Float16 vt[2][D][kVtPitch];
};

// sched_group_barrier classes
constexpr int kSgValu = 0x2, kSgMfma = 0x8, kSgDsRead = 0x100;
typedef _Float16 f16x2a __attribute__((ext_vector_type(2)));
constexpr float kSumLimit = 16384.0f;   // a lane's 16 probabilities may sum to this before the reference maximum moves

// Profiling builds (-DARKV_PHASE_TRACE): shader-clock and 100 MHz timestamps around the longest workgroup,
// from which the shader clock the kernel ran at follows.  Product builds compile none of it.
#ifdef ARKV_PHASE_TRACE
__device__ unsigned long long g_attn_clock[4];
#endif

// At least four waves per workgroup: fetching and staging a tile is work of the workgroup, and with one or two waves to
// share it (LDS also admits few such workgroups per CU) the matrix pipe idled behind it.  One block of 32 positions at
// G = 1, 2 against QB = 4 / G, 4096-token prompt, 8 kv-heads: d = 128 211 -> 97 us and 233 -> 119 us; d = 64, 2003 tokens,
// 32 units, G = 1: 80.6 -> 51.7 us.
template <int H> constexpr int kQBlocks = H < 4 ? 4 / H : 1;     // H: heads of a workgroup

// four adjacent channels of an output row: bf16, and fp32 for the parity hook
template <int D>
__device__ __forceinline__ void store_out4(const AttnLaunch& L, size_t orow, int c, const float (&val)[4]) {
  uint16_t o[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t bits = __float_as_uint(val[e]);
    bits += 0x7fffu + ((bits >> 16) & 1u);      // round to nearest even (finite values)
    o[e] = (uint16_t)(bits >> 16);
  }
  if (L.outf) *reinterpret_cast<float4*>(L.outf + orow * D + c) = make_float4(val[0], val[1], val[2], val[3]);
  *reinterpret_cast<uint2*>(L.out + orow * D + c) =
      make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
}

// Split over the keys, for launches whose workgroups do not fill the chip or whose longest workgroup outlasts the
// average (attn_split decides).  A workgroup's key tiles whose first key every one of its rows sees are cut into
// pieces of at most piece_tiles; the last piece also takes the tiles of the causal diagonal.  So every row sees the
// first key of every piece, and no piece leaves a row's softmax reference unset.
struct AttnPieces { int n, visible; };    // pieces; tiles that start at or before the first row's position
__host__ __device__ inline AttnPieces attn_pieces(int first_pos, int piece_tiles) {
  const int visible = first_pos / 32 + 1;
  return {piece_tiles > 0 ? (visible + piece_tiles - 1) / piece_tiles : 1, visible};
}
// A piece's partial result per wave, in the order in which its lanes hold it: 4 * (D / 32) float4 per lane
// [channel block][row group][lane] (unnormalised sums), then (reference maximum, sum) per row [32], then the sum of the
// unrounded probabilities per row [32] (EXACT).
template <int D> constexpr int kPieceFloats = 32 * D + 96;

// A launch whose workgroups take H of a unit's G heads has G / H shares per unit; the shares of a unit lie eight apart (as
// many as there are units left in the last eight), on the same XCD, whose L2 then serves both.  share: 0 .. units G / H - 1.
template <int G, int H>
__host__ __device__ __forceinline__ void unit_share(int share, int units, int& u, int& head0) {
  constexpr int N = G / H;
  const int first = share / (8 * N) * 8, r = share % (8 * N), n = units - first < 8 ? units - first : 8;
  u = first + r % n;
  head0 = H * (r / n);
}

// Which unit and block of query positions a workgroup takes.  grid (units, blocks, pieces; or units, up to kMaxGridY
// blocks, rest): the unit runs fastest, so the longest blocks of ALL units start first and the short ones fill the gaps at
// the end, and with a multiple of 8 units a unit's workgroups share the L2 of one XCD (workgroups go to the XCDs in turn).
// With the block fastest, the last unit's long blocks started late: 4096 tokens x 8 units, d = 128, G = 4 205 -> 156 us,
// x 24 units 551 -> 450 us, 2003 x 32, d = 64, G = 1 51.6 -> 43.5 us.
// Units whose keys and values together exceed the last-level cache go in groups that fit (L.group units, see
// attn_group), one group after the other: 32 units x 32768 tokens (537 MB) 36.7 ms all at once, 35.0 one unit at a time,
// 34.3 in groups of eight; 64 x 8192 4.73 -> 4.49 ms against one at a time.
// A launch of at most two workgroups per CU starts all at once: there the second half runs from the shortest up, so that
// a CU that got a long one first gets a short one next (4096 x 8 units, G = 1: 65 -> 60 us; 1000 x 8, G = 4: 26.3 -> 25.7).
constexpr int kMaxGridY = 65535;
// x of units workgroups side by side, rank of the blocks (0: the longest)
__host__ __device__ __forceinline__ bool query_block(unsigned units, unsigned x, unsigned rank, int nqb, int group, int& u, int& qb) {
  if (rank >= (unsigned)nqb) return false;
  u = (int)x;
  if ((unsigned)group < units) {
    const unsigned id = x + units * rank, per = (unsigned)group * (unsigned)nqb;
    const unsigned g = id / per, rem = id % per, first = g * (unsigned)group;
    const unsigned n = first + (unsigned)group < units ? (unsigned)group : units - first;  // units of this group
    u = (int)(first + rem % n);
    rank = rem / n;
  } else if (units * (unsigned)nqb <= 512u && (int)rank >= (nqb + 1) / 2) {
    qb = (int)rank - (nqb + 1) / 2;
    return true;
  }
  qb = nqb - 1 - (int)rank;
  return true;
}
// Units that run side by side: as many as 128 MB of keys and values, in eights (one per XCD), at least eight; in a split
// launch all of them.
static int attn_group(int D, int T, int units, bool split) {
  const long long per_unit = 4ll * D * T;
  const long long n = (128ll << 20) / per_unit / 8 * 8;
  return split ? units : (int)(n < 8 ? (units < 8 ? units : 8) : (n < units ? n : units));
}

// EXACT (a split launch that also hands the scorer its row constants): the window rows' normalisers are summed from the
// probabilities before their rounding to fp16 as well.  The rounded sum is the right one for the outputs (numerator and
// denominator then see the same numbers); as a normaliser it carries the roundings of few large probabilities, which
// depend on the reference maximum and so on the cut.
template <int D, int G, int H, bool EXACT>
__global__ __launch_bounds__(64 * H * kQBlocks<H>, 2) void k_prefill_attn(AttnLaunch L) {
#ifdef ARKV_PHASE_TRACE
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) { g_attn_clock[0] = clock64(); g_attn_clock[1] = wall_clock64(); }
#endif
  constexpr int KK = D / 16;          // k-steps of the logits MFMA
  constexpr int KH = KK / 2;          // operands carried from the previous phase
  constexpr int CBN = D / 32;         // 32-channel blocks of the output
  constexpr int NPV = 2 * CBN;        // PV MFMAs per tile
  constexpr int QB = kQBlocks<H>;     // blocks of 32 query positions per workgroup
  constexpr int NT = 64 * H * QB;
  // Staging items of a tile, the same number for every thread (a branch would end the region in which they are
  // dealt out between MFMAs): KW channels of a key; VW channels of a pair of adjacent keys' values.
  constexpr int KW = 32 * D / NT < 8 ? 32 * D / NT : 8, KPR = D / KW, KPT = 32 * KPR / NT;
  constexpr int VW = 16 * D / NT;
  static_assert(KW * KPR == D && KPT * NT == 32 * KPR && VW >= 2 && VW <= 8, "equal shares");
  // Of the two waves on a SIMD the one in phase A issues first, then the one in phase B: they share the issue port, and the
  // phase with vector work beside its MFMAs is the longer one.  512 queries x 16411 keys x 8 units 160-164 -> 147-156 us, 8192
  // tokens x 8 units 533 -> 527, the same at G = 8; nothing at G = 1 (164.4, 165.3) or d = 64 (321, 323).
  constexpr bool kPrio = D == 128 && H >= 4;
  static_assert(NPV >= KH && NPV >= KPT + VW / 2, "operand prefetch pattern; one staging item per PV MFMA at most");
  using KItem = Words<KW / 2>;
  using VItem = Words<VW / 2>;
  __shared__ __align__(16) AttnLds<D> sm;
  const int nqb = (L.Tq + 32 * QB - 1) / (32 * QB);
  int u, qb;
  const bool split = L.piece_tiles > 0;
  if (!query_block(gridDim.x, blockIdx.x, blockIdx.y + (split ? 0u : blockIdx.z * (unsigned)kMaxGridY), nqb, L.group, u, qb)) return;
  const int share = u;                              // of a unit's heads; also where its partials lie
  int head0 = 0;
  if constexpr (H < G) unit_share<G, H>(share, L.B * L.Hkv, u, head0);
  const int b = u / L.Hkv, g = u % L.Hkv;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = head0 + wave % H, wq = QB * qb + wave / H; // head of the unit, block of 32 query positions
  const int n = lane & 31, hh = lane >> 5;
  const int T = L.T, Tq = L.Tq, q0 = T - Tq;
  const int row = 32 * wq + n;                     // query row inside the block of T_q queries
  const int rowc_ = row < Tq ? row : Tq - 1;
  const int pos = q0 + rowc_;                      // its position: sees keys j <= pos
  const int jmax = min(T, q0 + 32 * QB * (qb + 1));  // keys any row of this workgroup can see
  const int ntiles = (jmax + 31) / 32;
  const AttnPieces pc = attn_pieces(q0 + 32 * QB * qb, L.piece_tiles);
  const int piece = split ? (int)blockIdx.z : 0;
  if (piece >= pc.n) return;
  const int t0 = pc.visible * piece / pc.n, t1 = piece + 1 < pc.n ? pc.visible * (piece + 1) / pc.n : ntiles;
  const int jfull = q0 + 32 * wq - 31;             // tiles starting at or before this need no mask
  const uint16_t* kbase = L.k + (size_t)u * T * D;
  const uint16_t* vbase = L.v + (size_t)u * T * D;
  const float scale2 = L.scale2;

  // query operand (B of S^T = K Q^T): row n, channels 16 kk + 8 hh .. +7
  u32x4a qreg[KK];
  {
    const uint16_t* qp = L.q + ((size_t)(b * L.Hq + g * G + w) * Tq + rowc_) * D + 8 * hh;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qreg[kk] = *reinterpret_cast<const u32x4a*>(qp + 16 * kk);
  }
  // global -> registers -> LDS staging of one tile.  A tile is a buffer of its own: a uniform base, a per-thread constant
  // offset, and as many rows as the prompt still has (none for the prefetch past it), so that the last, partial tile needs
  // no branch and no clamped address (1-3 %); the rows it lacks read as zero and are masked.
  KItem ks[2][KPT];
  VItem vs[2][2];
  const uint32_t koff = 2 * KW * tid, voff = 2 * (2 * (tid % 16) * D + VW * (tid / 16));
  auto rows_from = [&](const uint16_t* base, int j0) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base) + (size_t)j0 * D, 0,
                                             2 * D * __builtin_amdgcn_readfirstlane(min(max(T - j0, 0), 32)), 0x00027000);
  };
  auto fetch_k = [&](int j0, KItem (&to)[KPT]) {
    const __amdgpu_buffer_rsrc_t r = rows_from(kbase, j0);
#pragma unroll
    for (int c = 0; c < KPT; ++c) to[c] = buffer_words<KW / 2>(r, koff + 2 * KW * NT * c);
  };
  auto fetch_v = [&](int j0, VItem (&to)[2]) {
    const __amdgpu_buffer_rsrc_t r = rows_from(vbase, j0);
    to[0] = buffer_words<VW / 2>(r, voff);
    to[1] = buffer_words<VW / 2>(r, voff + 2 * D);
  };
  auto stage_k1 = [&](int buf, int c, const KItem (&from)[KPT]) {
    const int ch = tid + NT * c;
    *reinterpret_cast<KItem*>(&sm.k[buf][ch / KPR][KW * (ch % KPR)]) = from[c];
  };
  auto stage_v1 = [&](int buf, int e, const VItem (&from)[2]) {      // channels 2 e, 2 e + 1 of the thread's share
    const int col = vt_col(2 * (tid % 16)), c0 = VW * (tid / 16);
    const uint32_t a = word(from[0], e), b = word(from[1], e);
    *reinterpret_cast<uint32_t*>(&sm.vt[buf][c0 + 2 * e][col]) = bf16_pair_to_f16x2(a, b);
    *reinterpret_cast<uint32_t*>(&sm.vt[buf][c0 + 2 * e + 1][col]) = bf16_pair_to_f16x2(a >> 16, b >> 16);
  };
  auto k_operand = [&](int buf, int kk) { return *reinterpret_cast<const u32x4a*>(&sm.k[buf][n][16 * kk + 8 * hh]); };
  // A of O^T = V^T P^T, PV MFMA r = jj * CBN + cb: channel 32 cb + n, keys 16 jj + 4 hh + (0..3) and
  // 16 jj + 8 + 4 hh + (0..3), adjacent in LDS
  auto v_operand = [&](int buf, int r) {
    return *reinterpret_cast<const u32x4a*>(&sm.vt[buf][32 * (r % CBN) + n][16 * (r / CBN) + 8 * hh]);
  };

  f32x16a acc[CBN];
#pragma unroll
  for (int cb = 0; cb < CBN; ++cb)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[cb][i] = 0.f;
  float m_run = kNegBigA, l_run = 0.f, le_run = 0.f;
  u32x4a kop[KK], vop[NPV];
  int kA = 1, kB = 2, kW = 0;       // LDS buffers of key tiles t + 1, t + 2 and t + 3 (= the one tile t leaves)

  // fresh logits of the tile starting at j0 (C[i]: row n against key j0 + 8(i/4) + 4hh + i%4, unscaled):
  // what lies beyond the row gets a logit whose probability is zero
  auto mask = [&](f32x16a& C, int j0) {
    if (j0 > jfull) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (j0 + 8 * (i >> 2) + 4 * hh + (i & 3) > pos) C[i] = kNegBigA;
    }
  };
  // probabilities of logits C against the running reference m_run, as fp16 pairs (ph[e]: elements 2e, 2e + 1),
  // and their sum as rounded (the same numbers the PV MFMA multiplies)
  auto probs = [&](const f32x16a& C, int i, uint32_t (&ph)[8], float& lt, float& le) {
    const float p0 = aexp2(fmaf(C[i], scale2, -m_run)), p1 = aexp2(fmaf(C[i + 1], scale2, -m_run));
    const __half2 h2 = __floats2half2_rn(p0, p1);
    ph[i / 2] = *reinterpret_cast<const uint32_t*>(&h2);
    lt = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2a, ph[i / 2]), f16x2a{(_Float16)1.0f, (_Float16)1.0f}, lt, false);
    if constexpr (EXACT) { le += p0; le += p1; }
  };

  // One step of the two-stage pipeline over tiles.  Phase A: the logits MFMAs of tile t + 1 (into Cn), each
  // followed in issue order by one LDS operand read for a later MFMA and by its share of tile t's softmax
  // arithmetic (from C): the matrix pipe works in the background of the same wave's vector instructions only
  // if the two alternate.  Phase B: the PV MFMAs of tile t between operand reads for the next step and the
  // conversion and staging of the tiles fetched at the top of the step before: one item behind each MFMA, pinned there by
  // an empty asm that takes an operand of the next MFMA (group barriers alone let the MFMAs run together at the end).
  // The reference maximum is lazy: probabilities are taken against the row's current m_run, and only when a
  // lane's sum shows that they grew large (or the reference is still unset) does the row move its reference
  // to the tile's maximum and redo the tile.  A row decides from its own numbers only.
  auto step = [&](f32x16a& C, f32x16a& Cn, int t, const int vb) {     // vb: the buffer that holds the value tile
    const int j0 = 32 * t;
    fetch_k(j0 + 128, ks[vb]);
    fetch_v(j0 + 64, vs[vb]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kPrio) __builtin_amdgcn_s_setprio(2);
    uint32_t ph[8];
    float lt0 = 0.f, lt1 = 0.f, le0 = 0.f, le1 = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) Cn[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + KH < KK) kop[kk + KH] = k_operand(kA, kk + KH);
      else vop[kk + KH - KK] = v_operand(vb, kk + KH - KK);
      Cn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8a, kop[kk]), __builtin_bit_cast(bf16x8a, qreg[kk]), Cn, 0, 0, 0);
      constexpr int EPK = 16 / KK;                    // softmax elements per MFMA (2 at D = 128, 4 at D = 64)
#pragma unroll
      for (int e = 0; e < EPK; e += 2) probs(C, EPK * kk + e, ph, ((kk + e / 2) & 1) ? lt1 : lt0, ((kk + e / 2) & 1) ? le1 : le0);
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      __builtin_amdgcn_sched_group_barrier(kSgMfma, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSgDsRead, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSgValu, (EXACT ? 8 : 6) * 16 / (2 * KK), 0);
    }
    float lt = lt0 + lt1;
    if (__any(!(lt <= kSumLimit))) {                  // rare after the first tile
      const float lo = __shfl_xor(lt, 32);
      const bool move = !(fmaxf(lt, lo) <= kSumLimit);   // both lane halves of a row agree
      float mt = C[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mt = fmaxf(mt, C[i]);
      mt *= scale2;                                   // scale2 > 0: the maximum commutes with the scaling
      mt = fmaxf(mt, __shfl_xor(mt, 32));
      const float mn = move ? fmaxf(m_run, mt) : m_run;
      const float f = aexp2(m_run - mn);
      m_run = mn;
      l_run *= f;
      le_run *= f;
#pragma unroll
      for (int cb = 0; cb < CBN; ++cb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb][i] *= f;
      lt0 = 0.f; lt1 = 0.f; le0 = 0.f; le1 = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) probs(C, i, ph, lt0, le0);
      lt = lt0;
    }
    l_run += lt;
    if constexpr (EXACT) le_run += le0 + le1;
    if constexpr (kPrio) __builtin_amdgcn_s_setprio(1);
    // PV: probabilities eight per k-step: jj = 0 -> elements 0..7, jj = 1 -> 8..15
#pragma unroll
    for (int r = 0; r < NPV; ++r) {
      if (r + KH < NPV) vop[r + KH] = v_operand(vb, r + KH);
      else kop[r + KH - NPV] = k_operand(kB, r + KH - NPV);
      const int jj = r / CBN, cb = r % CBN;
      const u32x4a pb = {ph[4 * jj], ph[4 * jj + 1], ph[4 * jj + 2], ph[4 * jj + 3]};
      acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8a, vop[r]), __builtin_bit_cast(f16x8a, pb), acc[cb], 0, 0, 0);
      if (r < VW / 2) stage_v1(vb ^ 1, r, vs[vb ^ 1]);                  // tile t + 1; that buffer was last read one step ago
      else if (r < VW / 2 + KPT) stage_k1(kW, r - VW / 2, ks[vb ^ 1]);  // tile t + 3 into the buffer tile t's logits came from
      if (r + 1 < NPV) asm volatile("" : "+v"(ph[4 * ((r + 1) / CBN)]) : : "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (kPrio) __builtin_amdgcn_s_setprio(0);
    mask(Cn, j0 + 32);
    const int k0 = kA; kA = kB; kB = kW; kW = k0;
    __syncthreads();
  };

  {
    // Everything the first steps need is requested before any of it is waited for: one round trip to memory in front of the
    // first step, where the third tile's request behind the first one's arrival made it two (144 calls on 150 to 600 keys 2 %
    // at the median, up to 10; 2003 x 32 units 33.1 -> 32.8 us; nothing on long prompts).
    KItem first[3][KPT];
#pragma unroll
    for (int i = 0; i < 3; ++i) fetch_k(32 * (t0 + i), first[i]);
    fetch_v(32 * t0, vs[0]);
    fetch_v(32 * t0 + 32, vs[1]);
    fetch_k(32 * t0 + 96, ks[1]);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int c = 0; c < KPT; ++c) stage_k1(i, c, first[i]);
#pragma unroll
    for (int e = 0; e < VW / 2; ++e) stage_v1(0, e, vs[0]);
  }
  __syncthreads();
  f32x16a C0, C1;
  {
#pragma unroll
    for (int i = 0; i < 16; ++i) C0[i] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      C0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8a, k_operand(0, kk)), __builtin_bit_cast(bf16x8a, qreg[kk]), C0, 0, 0, 0);
    mask(C0, 32 * t0);
#pragma unroll
    for (int kk = 0; kk < KH; ++kk) kop[kk] = k_operand(1, kk);
  }
  __syncthreads();       // the first step stages into buffer 0: every wave, also one whose query rows came late, has read it
  for (int t = t0; t < t1; t += 2) {
    step(C0, C1, t, 0);
    if (t + 1 < t1) step(C1, C0, t + 1, 1);
  }

#ifdef ARKV_PHASE_TRACE
  if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) { g_attn_clock[2] = clock64(); g_attn_clock[3] = wall_clock64(); }
#endif
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if (pc.n > 1) {
    float* part = L.part + ((((size_t)share * nqb + qb) * gridDim.z + piece) * (H * QB) + wave) * kPieceFloats<D>;
#pragma unroll
    for (int cb = 0; cb < CBN; ++cb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        *reinterpret_cast<float4*>(part + ((cb * 4 + i4) * 64 + lane) * 4) =
            make_float4(acc[cb][4 * i4], acc[cb][4 * i4 + 1], acc[cb][4 * i4 + 2], acc[cb][4 * i4 + 3]);
    if (hh == 0) *reinterpret_cast<float2*>(part + 32 * D + 2 * n) = make_float2(m_run, l_tot);
    if constexpr (EXACT) {
      const float le = le_run + __shfl_xor(le_run, 32);
      if (hh == 0) part[32 * D + 64 + n] = le;
    }
    return;
  }
  const float inv = 1.0f / l_tot;
  if (row < Tq) {
    const size_t orow = (size_t)(b * L.Hq + g * G + w) * Tq + row;
#pragma unroll
    for (int cb = 0; cb < CBN; ++cb)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4) {
        const float val[4] = {acc[cb][4 * i4] * inv, acc[cb][4 * i4 + 1] * inv, acc[cb][4 * i4 + 2] * inv, acc[cb][4 * i4 + 3] * inv};
        store_out4<D>(L, orow, 32 * cb + 8 * i4 + 4 * hh, val);
      }
    // the scorer's row constant c = max + log2(sum) of the window rows (row index: head-major, W per head)
    float l_row = l_tot;
    if constexpr (EXACT) l_row = le_run + __shfl_xor(le_run, 32);
    if (L.rowc && hh == 0 && pos >= T - L.W)
      L.rowc[(size_t)u * L.MP + w * L.W + (pos - (T - L.W))] = m_run + log2f(l_row);
  }
}

// Adds up the pieces of the workgroups that have more than one.  grid (query blocks, units, D / 32), the same waves and
// lanes as above; a wave takes one block of 32 channels.  Bound by the partials' bytes (34 MB written and read at 512
// queries x 16411 keys x 32 heads: 9 us of 147).
template <int D, int G, int H>
__global__ __launch_bounds__(64 * H * kQBlocks<H>) void k_prefill_attn_merge(AttnLaunch L, int max_pieces) {
  constexpr int QB = kQBlocks<H>;
  const int qb = blockIdx.x, cb = blockIdx.z;
  int u = blockIdx.y, head0 = 0;
  if constexpr (H < G) unit_share<G, H>(blockIdx.y, L.B * L.Hkv, u, head0);
  const int b = u / L.Hkv, g = u % L.Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = head0 + wave % H, n = lane & 31, hh = lane >> 5;
  const int T = L.T, Tq = L.Tq, q0 = T - Tq, row = 32 * (QB * qb + wave / H) + n;
  const AttnPieces pc = attn_pieces(q0 + 32 * QB * qb, L.piece_tiles);
  if (pc.n < 2 || row >= Tq) return;
  const float* part = L.part + (((size_t)blockIdx.y * gridDim.x + qb) * max_pieces * (H * QB) + wave) * kPieceFloats<D>;
  const size_t stride = (size_t)(H * QB) * kPieceFloats<D>;
  float M = kNegBigA;
  for (int p = 0; p < pc.n; ++p) M = fmaxf(M, part[p * stride + 32 * D + 2 * n]);
  float l = 0.f, le = 0.f, acc[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  for (int p = 0; p < pc.n; ++p) {
    const float* pp = part + p * stride;
    const float2 ml = *reinterpret_cast<const float2*>(pp + 32 * D + 2 * n);
    const float f = aexp2(ml.x - M);
    l = fmaf(ml.y, f, l);
    if (L.rowc && cb == 0) le = fmaf(pp[32 * D + 64 + n], f, le);
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
      const float4 v = *reinterpret_cast<const float4*>(pp + ((cb * 4 + i4) * 64 + lane) * 4);
      acc[4 * i4] = fmaf(v.x, f, acc[4 * i4]);
      acc[4 * i4 + 1] = fmaf(v.y, f, acc[4 * i4 + 1]);
      acc[4 * i4 + 2] = fmaf(v.z, f, acc[4 * i4 + 2]);
      acc[4 * i4 + 3] = fmaf(v.w, f, acc[4 * i4 + 3]);
    }
  }
  const float inv = 1.0f / l;
  const size_t orow = (size_t)(b * L.Hq + g * G + w) * Tq + row;
#pragma unroll
  for (int i4 = 0; i4 < 4; ++i4) {
    const float val[4] = {acc[4 * i4] * inv, acc[4 * i4 + 1] * inv, acc[4 * i4 + 2] * inv, acc[4 * i4 + 3] * inv};
    store_out4<D>(L, orow, 32 * cb + 8 * i4 + 4 * hh, val);
  }
  if (L.rowc && cb == 0 && hh == 0 && q0 + row >= T - L.W)
    L.rowc[(size_t)u * L.MP + w * L.W + (q0 + row - (T - L.W))] = M + log2f(le);
}

// Floats of scratch the pieces of such a launch take.
size_t attn_part_floats(int D, int G, int units, int Tq, int max_pieces) {
  const int qb_rows = 32 * (G < 4 ? 4 / G : 1);
  return max_pieces < 2 ? 0 : (size_t)units * ((Tq + qb_rows - 1) / qb_rows) * max_pieces * (G < 4 ? 4 : G) *
                              (size_t)(D == 64 ? kPieceFloats<64> : kPieceFloats<128>);
}

// How far to split over the keys: tiles per piece (0: no split) and the largest number of pieces of a workgroup.
// The model: a tile step takes `alone` us in a workgroup that has its CU to itself and `shared` us where two share it, so a
// launch takes `alone` x the longest workgroup's tiles or half of `shared` x the tiles per CU, whichever is more; the merge costs
// 3 us, 0.1 per piece and its partials' way out and back.  (A step timed by itself takes 0.54 and 1.04 us, d = 64: 0.43 and
// 0.66; the constants are those with which the model chooses best.)  Split pays where few workgroups walk many tiles: 512
// queries x 16411 keys x 8 kv-heads 290 -> 146 us (4 pieces), 32 x 1100 x 8 units (d = 64) 19.9 -> 12.1.  It does not pay for a
// whole short prompt, whose imbalance is only the causal triangle (1100 tokens x 8 kv-heads: 29.6 us unsplit, 32.9 us in 2
// pieces; 972 x 4, 23.1 and 24.7 in 3; d = 64, 1379 x 4 22.5 and 25.0 in 4), hence `triangle`; with most CUs idle it pays earlier (d = 64, 1249 x
// 1 20.6 and 15.3 in 5, 1272 x 1 20.7 and 15.0).  Calls on up to 992 keys (kUnsplitKeys, whatever a workgroup's rows make
// of their tiles) are never split, so that a prompt of that length gives the same bits however it is cut into chunks (32 x 600
// keys: 12-17 us where the best split takes 10-13).
// Every number of pieces timed for 1700 drawn calls (1-32 units, 993-13000 keys, 16 queries to the whole prompt, every G): the
// chosen one takes 3.8 % longer than the best on average, 12 % at the ninth decile, 42 at most (with constants fitted to an older
// loop 6.2, 17 and 65).  394 of them are cut otherwise than with those, these take 9 % less at the mean (-39 to +12 %, 34
// above +3).
constexpr int kUnsplitKeys = 992;
void attn_split(int D, int G, int units, int T, int Tq, int* piece_tiles, int* max_pieces) {
  *piece_tiles = 0; *max_pieces = 1;
  const double alone = D == 64 ? 0.36 : 0.6, shared = D == 64 ? 0.6 : 0.95;
  const int H = G < 4 ? G : 4, QB = 4 / H, nqb = (Tq + 32 * QB - 1) / (32 * QB), q0 = T - Tq;
  const long long wgs = (long long)nqb * units * (G / H);
  const int v0 = attn_pieces(q0, 0).visible, vmax = v0 + QB * (nqb - 1);         // visible tiles: v0 + QB i, i < nqb
  const double mean = 0.5 * ((double)v0 + vmax);
  const double triangle = D == 128 ? 9.5 : wgs > 128 ? 7.5 : 6.6;                // us of the average workgroup
  if (T <= kUnsplitKeys || wgs > 4 * 256 || alone * mean < triangle) return;
  const double busy = 0.5 * shared * mean * (double)wgs / 256;
  double best = 1.05 * (alone * vmax > busy ? alone * vmax : busy);
  for (int ns = 2; ns <= 16; ++ns) {
    const int pt = (vmax + ns - 1) / ns;
    const size_t floats = attn_part_floats(D, G, units, Tq, ns);
    if (pt < 8 || floats > kAttnPartFloats) break;
    long long items = 0;
    for (int p = 0; p < ns; ++p) {                                               // workgroups with more than p pieces
      const int i0 = (p * pt + 1 - v0 + QB - 1) / QB;                            // the first one (v0 + QB i > p pt)
      items += nqb - (p * pt + 1 <= v0 ? 0 : (i0 < nqb ? i0 : nqb));
    }
    items *= units * (G / H);
    double t = items <= 256 ? alone * pt : items <= 512 ? shared * pt : busy + 0.5 * shared * pt;
    if (t < busy) t = busy;
    t += 3.0 + 0.1 * ns + 1.0e-6 * (double)floats;
    if (t < best) { best = t; *piece_tiles = pt; *max_pieces = ns; }
  }
}

template <int D, int G, int H>
static hipError_t launch_attn_t(const AttnLaunch& launch, int max_pieces, hipStream_t s) {
  AttnLaunch a = launch;
  constexpr int rows = 32 * kQBlocks<H>, nt = 64 * H * kQBlocks<H>;
  const int units = a.B * a.Hkv * (G / H), nqb = (a.Tq + rows - 1) / rows;
  a.group = attn_group(a.D, a.T, a.B * a.Hkv, max_pieces > 1) * (G / H);
  const dim3 grid(units, nqb < kMaxGridY ? nqb : kMaxGridY, max_pieces > 1 ? max_pieces : (nqb + kMaxGridY - 1) / kMaxGridY);
  if (max_pieces > 1 && a.rowc) hipLaunchKernelGGL((k_prefill_attn<D, G, H, true>), grid, dim3(nt), 0, s, a);
  else hipLaunchKernelGGL((k_prefill_attn<D, G, H, false>), grid, dim3(nt), 0, s, a);
  if (max_pieces > 1)
    hipLaunchKernelGGL((k_prefill_attn_merge<D, G, H>), dim3(nqb, units, D / 32), dim3(nt), 0, s, a, max_pieces);
  return hipGetLastError();
}

// Heads of a unit that a workgroup takes.
static int attn_heads(int D, int G, int units, int T, int Tq, bool split) {
  // Four heads per workgroup at G = 8: four waves leave twice as many workgroups to spread over the CUs as eight, and a
  // wave that has its SIMD to itself takes a step in 0.54 us (d = 64: 0.43) instead of 0.76 (0.55).  4 / 8 heads, us: 300 x 8 units
  // 11.9 / 16.5, 32 x 1100 x 8 (split) 14.4 / 18.4, 2003 x 8 78.7 / 91.6 (d = 64: 51.3 / 62.0), 2003 x 32 309 / 314; the best of
  // every split taken on both sides, 138 calls on 150 to 10007 keys, 2 to 32 units: 13 % less at the median, up to 33.  Long
  // prompts that fill the chip many times over read each key tile once for all eight heads (10007 x 8 1562 / 1589, 1024 x
  // 10007 x 32 1179 / 1211, d = 128; 5000 x 32 the same; d = 64 956 / 994 the other way).  At d = 64 a CU holds three
  // workgroups of four waves or two of eight: where blocks that are much alike fill at most two of eight per CU, but more than
  // three of four, the smaller ones take a second round (474 x 2688 x 32 units, 480 blocks, 121 / 105; 499 x 6055 x 32, 512
  // blocks, 267 / 233; 102 calls of 385 to 512 blocks with at most 0.4 of the keys as queries 9 % on average, -7 to 24; of 330 to 384
  // and 513 to 590 blocks 9 to 27 % the other way, and where the blocks' lengths differ more).
  const long long blocks = (long long)units * ((Tq + 31) / 32);
  const bool eight = !split && (D == 128 ? T >= 8192 && blocks >= 512 : blocks > 3 * 128 && blocks <= 4 * 128 && 5ll * Tq <= 2ll * T);
  return G < 8 ? G : eight ? 8 : 4;
}

hipError_t launch_prefill_attn(const AttnLaunch& a, int max_pieces, hipStream_t s) {
  const int G = a.Hq / a.Hkv, H = attn_heads(a.D, G, a.B * a.Hkv, a.T, a.Tq, max_pieces > 1);
#define ARKV_AT(D_, G_, H_) if (a.D == D_ && G == G_ && H == H_) return launch_attn_t<D_, G_, H_>(a, max_pieces, s);
  ARKV_AT(128, 8, 8) ARKV_AT(64, 8, 8)
  ARKV_AT(128, 1, 1) ARKV_AT(128, 2, 2) ARKV_AT(128, 4, 4) ARKV_AT(128, 8, 4)
  ARKV_AT(64, 1, 1) ARKV_AT(64, 2, 2) ARKV_AT(64, 4, 4) ARKV_AT(64, 8, 4)
#undef ARKV_AT
  return hipErrorInvalidValue;
}

}  // namespace arkv

extern "C" int arkv_debug_attention_split(int32_t head_dim, int32_t group, int32_t units, int32_t T, int32_t T_q, int32_t* out) {
  if (!out || (head_dim != 64 && head_dim != 128) || (group != 1 && group != 2 && group != 4 && group != 8) || units < 1 ||
      T_q < 1 || T_q > T)
    return ARKV_EINVAL;
  int tiles, pieces;
  arkv::attn_split(head_dim, group, units, T, T_q, &tiles, &pieces);
  const int rows = 32 * (group < 4 ? 4 / group : 1), last = (T_q - 1) / rows;
  out[0] = tiles; out[1] = pieces;
  out[2] = arkv::attn_pieces(T - T_q, tiles).n;
  out[3] = arkv::attn_pieces(T - T_q + rows * last, tiles).n;
  return ARKV_OK;
}

extern "C" int arkv_debug_attention_block(int32_t head_dim, int32_t units, int32_t T, int32_t n_blocks, int32_t split, int32_t index,
                                          int32_t* out) {
  if (!out || (head_dim != 64 && head_dim != 128) || units < 1 || T < 1 || n_blocks < 1 || index < 0 ||
      (long long)index >= (long long)units * n_blocks)
    return ARKV_EINVAL;
  const unsigned x = (unsigned)index % (unsigned)units, rank = (unsigned)index / (unsigned)units;
  int u = -1, qb = -1;
  if (!arkv::query_block((unsigned)units, x, rank, n_blocks, arkv::attn_group(head_dim, T, units, split != 0), u, qb))
    return ARKV_EINVAL;
  out[0] = u; out[1] = qb;
  return ARKV_OK;
}

extern "C" int arkv_debug_attention_heads(int32_t head_dim, int32_t group, int32_t units, int32_t T, int32_t T_q, int32_t index, int32_t* out) {
  if (!out || (head_dim != 64 && head_dim != 128) || (group != 1 && group != 2 && group != 4 && group != 8) || units < 1 ||
      T_q < 1 || T_q > T || index < 0)
    return ARKV_EINVAL;
  int tiles, pieces;
  arkv::attn_split(head_dim, group, units, T, T_q, &tiles, &pieces);
  const int H = arkv::attn_heads(head_dim, group, units, T, T_q, pieces > 1), shares = group / H;
  const int rows = 32 * (H < 4 ? 4 / H : 1), nqb = (T_q + rows - 1) / rows;
  if ((long long)index >= (long long)units * shares * nqb) return ARKV_EINVAL;
  const unsigned n = (unsigned)(units * shares), x = (unsigned)index % n, rank = (unsigned)index / n;
  int u = -1, qb = -1, head0 = 0;
  if (!arkv::query_block(n, x, rank, nqb, arkv::attn_group(head_dim, T, units, pieces > 1) * shares, u, qb)) return ARKV_EINVAL;
  if (shares == 2) { const int share = u; arkv::unit_share<8, 4>(share, units, u, head0); }
  out[0] = u; out[1] = head0; out[2] = H; out[3] = qb;
  return ARKV_OK;
}

namespace arkv {
// the prefill attention's four clock words (shader clock and 100 MHz counter at the start and the end of workgroup 0)
hipError_t phase_trace_attn(unsigned long long* host, bool* built) {
#ifdef ARKV_PHASE_TRACE
  *built = true;
  return hipMemcpyFromSymbol(host, HIP_SYMBOL(g_attn_clock), 4 * sizeof(unsigned long long));
#else
  (void)host;
  *built = false;
  return hipSuccess;
#endif
}
}  // namespace arkv
