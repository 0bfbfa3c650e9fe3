// Per-sample adaptive steps after a block (Algorithm 1, Sec. III-B..E):
//   merge router and count (Eq. 4-5), bipartite soft matching with
//   size-weighted merging (Sec. III-C), exit check on the CLS head
//   (Eq. 6-7), CLS-attention top-k pruning of continuing samples (Eq. 8),
// followed by a separate compaction kernel that re-packs the surviving
// samples and tokens (exclusive scans over new lengths and keep flags).
// The fp32 rows of x never move: a token keeps its physical row (a merge
// updates the destination row in place) and the compaction re-packs the row
// map, the sizes and the origin ids.
//
// One 512-thread workgroup per live sample (the compaction uses 256).  No
// float atomics: every reduction has a fixed order, so results do not depend
// on scheduling or on the rest of the batch.
//
// The per-sample kernel is a chain of short dependent phases, bound by their
// latency (one workgroup per CU, few waves): it loads what a phase needs
// together with the phase before, reduces with lane moves instead of LDS
// shuffles, ranks four keys per LDS read or searches thresholds within a wave,
// and keeps two barriers between the choice of the pairs and the merge.
// Per launch, averaged over the blocks of a run: one 224 x 224 image 21.3 ->
// 17.7 us (blocks of 130 to 197 tokens) and 14.1 -> 12.7 us (up to 128), 64
// images with few merges 17.9 -> 12.9 us, 64 images at 384 x 384 21.8 -> 13.9
// us and 26.0 -> 23.2 us for similarity_kernel.  Of 37,000 cycles at 189
// tokens the similarity takes 26,500.
#include "kernels.h"

#include <algorithm>

namespace fusion {

constexpr int AD_TMAX = 640;  // tokens per sample (CLS included), largest size class
constexpr int AD_NT = 512;    // threads per workgroup (8 waves)

// Size classes of the per-sample kernel: TMAX tokens (CLS included), so
// |A| = ceil(N/2) and |B| = floor(N/2) are at most TMAX/2.  The smallest
// class (T <= 128, picked from the host's token bound of the block) stages
// 64 features per chunk: its chunk loop is latency-bound, and half the
// chunks halve the barriers.
template <int TMAX_, int WC_ = (TMAX_ <= 128 ? 4 : TMAX_ <= 256 ? 2 : 4)> struct AdSize {
  static constexpr int TMAX = TMAX_;
  static constexpr int AMAX = TMAX_ / 2;
  static constexpr int BMAX = TMAX_ / 2;
  static constexpr int SKC = TMAX_ <= 128 ? 64 : 32;  // features per chunk (MFMA K steps of 32)
  // LDS row of a staged chunk (bf16): 32-feature chunks are unpadded 64-byte
  // rows with their four 16-byte pieces XOR-permuted by (row / 4) % 4 (the
  // 16-byte operand reads of 16 consecutive rows then hit disjoint banks);
  // 64-feature chunks are padded to 144-byte rows
  static constexpr bool SWZ = SKC == 32;
  static constexpr int SKP = SWZ ? SKC : SKC + 8;
  // similarity wave layout: WC column groups of B tiles, AD_NT / 64 / WC
  // groups of 32 A rows; SAG A rows per pass
  static constexpr int WC = WC_;
  static constexpr int SAG = 32 * (AD_NT / 64 / WC);
  static constexpr int NBT = BMAX / 16;        // B tiles of 16 rows
  static constexpr int NBW = NBT / WC;         // B tiles per wave
  static constexpr int BG = TMAX_ <= 128 ? 1 : TMAX_ <= 256 ? 4 : 5;  // B tiles per MFMA group
  static constexpr int SPT = ((SAG + BMAX) * (SKC / 4) + AD_NT - 1) / AD_NT;  // slots / thread
};

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int merge_count(float m, double rho, int r_b, int N, int rule) {
  // budget:   r = clamp(floor(((2 rho) m) r_b + 1/2), 0, floor(N/2));
  // fraction: r = min(floor(((rho m) N) / 2), floor(N/2)) (Sec. III-C with
  //           the rescaled ratio of Eq. 5);
  // every step an individually rounded IEEE double operation.
  const double t =
      rule == 1 ? __dmul_rn(__dmul_rn(__dmul_rn(rho, (double)m), (double)N), 0.5)
                : __dadd_rn(__dmul_rn(__dmul_rn(__dmul_rn(2.0, rho), (double)m), (double)r_b), 0.5);
  int r = (int)floor(t);
  if (r < 0) r = 0;
  if (r > N / 2) r = N / 2;
  return r;
}

// Block-wide reductions for AD_NT threads (8 waves).  red: 8 entries that no
// thread still reads; every write of the workgroup before the call is visible
// after it.
__device__ __forceinline__ float bsum(float v, float* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < AD_NT / 64; w++) s += red[w];
  return s;
}
__device__ __forceinline__ float bmax(float v, float* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = red[0];
#pragma unroll
  for (int w = 1; w < AD_NT / 64; w++) s = fmaxf(s, red[w]);
  return s;
}

// Lanes that share one element's rank count when n elements are ranked by
// the workgroup: the largest power of two (at most 16) with n * P <= AD_NT.
__device__ __forceinline__ int rank_lanes(int n) {
  int P = 1;
  while (P < 16 && n * (2 * P) <= AD_NT) P *= 2;
  return P;
}
// Sum over the P adjacent lanes (P = 1, 2, 4, 8 or 16) of each group.
__device__ __forceinline__ int lanes_sum(int v, int P) {
  if (P > 1) v += lane_xor_i<1>(v);
  if (P > 2) v += lane_xor_i<2>(v);
  if (P > 4) v += lane_xor_i<4>(v);
  if (P > 8) v += lane_xor_i<8>(v);
  return v;
}

// Order-preserving key of a float, never 0: for a, b not NaN, a < b iff
// order_key(a) < order_key(b), and a == b iff the keys are equal (-0 and +0
// share the key of +0).  NaNs take keys of their own at the two ends.
__device__ __forceinline__ unsigned order_key(float f) {
  const unsigned u = f == 0.f ? 0u : __float_as_uint(f);
  const unsigned k = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return k ? k : 1u;
}

// Selections rank keys[0 .. n), padded with 0 up to a multiple of 4 (rank_of)
// or 64 (wave_top); key 0 marks an element that does not take part.  An
// element is chosen iff fewer than c elements precede it, a larger key or an
// equal key at a lower index coming first.
//
// rank_of: elements that precede e (key k >= 1), counted over this lane's
// share (lane p of P) of the keys, four to a 16-byte LDS read: at indices
// below e a key of at least k counts, above it one larger than k, which is
// one compare and one add with carry per key outside e's own group of four.
__device__ __forceinline__ int rank_of(const unsigned* keys, int n, int e, unsigned k, int p,
                                       int P) {
  int rank = 0;
  const int n4 = (n + 3) >> 2, qe = e >> 2;
#pragma unroll 4
  for (int q = p; q < n4; q += P) {
    const uint4 v = ((const uint4*)keys)[q];
    const unsigned t = q < qe ? k - 1u : k;
    rank += v.x > t;
    rank += v.y > t;
    rank += v.z > t;
    rank += v.w > t;
  }
  if (qe % P == p) {  // equal keys below e in its own group
    const uint4 v = ((const uint4*)keys)[qe];
    rank += ((e & 3) > 0) & (v.x == k);
    rank += ((e & 3) > 1) & (v.y == k);
    rank += ((e & 3) > 2) & (v.z == k);
  }
  return rank;
}

// wave_top: the c elements chosen of n <= 64 NJ, as this wave's ballots; bit
// l of sel[j] is element 64 j + l.  The c-th largest key is found bit by bit
// from the top: the wave holds all keys in registers and counts those at or
// above the next threshold with ballots, so there is no LDS round trip and no
// barrier in the search (a workgroup-wide digit search with one barrier per
// round took 7,000 to 13,000 cycles for 288 keys), which ends early once
// exactly c keys remain.
template <int NJ>
__device__ __forceinline__ void wave_top(const unsigned* keys, int n, int c,
                                         unsigned long long (&sel)[NJ]) {
  const int lane = threadIdx.x & 63;
  const int nj = (n + 63) >> 6;
  c = __builtin_amdgcn_readfirstlane(c);
  unsigned k[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    k[j] = j < nj ? keys[64 * j + lane] : 0u;
    sel[j] = 0ull;
  }
  if (c <= 0) return;
  unsigned prefix = 0;
  for (int bit = 31; bit >= 0; bit--) {
    const unsigned t = prefix | (1u << bit);
    int m = 0;
#pragma unroll
    for (int j = 0; j < NJ; j++) m += (int)__popcll(__ballot(k[j] >= t));
    if (m >= c) prefix = t;
    if (m == c) break;  // the keys from the threshold on are the c largest
  }
  // prefix is at most the c-th key and above the next one: all larger keys,
  // then equal ones in index order
  int need = c;
#pragma unroll
  for (int j = 0; j < NJ; j++) need -= (int)__popcll(__ballot(k[j] > prefix));
  const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int j = 0; j < NJ; j++) {
    const unsigned long long eq = __ballot(k[j] == prefix);
    sel[j] = __ballot(k[j] > prefix || (k[j] == prefix && (int)__popcll(eq & lt) < need));
    need = max(need - (int)__popcll(eq), 0);
  }
}

// Candidates above which wave_top replaces the all-pairs rank count (whole
// prune step at 188 candidates: 4,800 against 8,300 cycles).
constexpr int SEL_WAVE_MIN = 128;

// Cosine similarities of the A tokens (even patch slots) with the B tokens
// (odd slots) of one sample, and the best B for every A.
//
// One pass over the features in chunks of SKC, double-buffered in LDS.
// The token rows are read from x through prow (the sample's physical row of
// each token slot).  Every thread owns a fixed set of (row, 4-feature)
// slots: the A rows of the pass first, then the B rows (clamped to the last
// real row, so
// the loads need no branch; padding rows only feed outputs that are never
// read).  The loads run two chunks ahead in two register sets.  A chunk's
// values are split into bf16 hi + lo (hi = RNE(v), lo = RNE(v - hi)), with
// the row's sum of squares accumulated on the way, and written to the LDS
// buffer that the MFMAs of the current chunk do not read: one barrier per
// chunk.  The dot products take hi.hi' + hi.lo' + lo.hi' on
// v_mfma_f32_16x16x32_bf16 with fp32 accumulation (absolute error of a
// cosine <= ~1.2e-5, the dropped lo.lo' term included), per output in
// feature order, the three terms in that order within each 32 features.
// The B fragment is the MFMA's row operand, so lane l of a 16 x 16 output
// tile holds S[b = 4 (l / 16) + j][a = l % 16] (j = 0..3): the candidates
// of one A token sit in 4 lanes x 4 registers per B tile.  Wave w owns A
// rows 32 (w / WC) .. +31 of the pass against B tiles NBW (w % WC) .. +NBW-1.
// Cosines are dot * (1 / n_a) * (1 / n_b) with the clamped norms
// max(||x||, 1e-12).  The argmax over B (ties to the lowest B index, NaN
// never wins) runs in-lane, then across the 4 lanes of a token with the
// lane-swap instructions, then over the WC wave groups in B order through
// LDS (pbv, pbi: WC SAG entries each).  rn holds the reciprocal norms:
// A rows of the pass at [0, SAG), B rows at [SAG, SAG + BMAX).  Passes of SAG
// A rows run from A row ag_first, at most n_pass of them; bestsim / best may
// point to LDS or to global memory (indexed by A row).
template <class Z>
__device__ void similarity_argmax(const float* __restrict__ x, const int* prow, int d,
                                  int nA, int nB, float* rn, float* bestsim,
                                  int* best, bf16_t* Ahi, bf16_t* Alo,
                                  bf16_t* Bhi, bf16_t* Blo, float* pbv, int* pbi,
                                  int ag_first = 0, int n_pass = 1 << 30) {
  constexpr int SKC = Z::SKC, SKP = Z::SKP, SPT = Z::SPT, NBW = Z::NBW, BG = Z::BG;
  constexpr int SAG = Z::SAG, WC = Z::WC, BMAX = Z::BMAX;
  constexpr int Q = SKC / 4;  // 16-byte slots per row and chunk
  static_assert(SKC % 32 == 0, "whole MFMA K steps per chunk");
  static_assert(SPT * AD_NT == (SAG + BMAX) * Q, "slots must tile the staged rows exactly");
  static_assert(Q == 8 || Q == 16, "lanes of a staged row");
  static_assert(NBW % BG == 0 && NBW * WC == Z::NBT, "wave layout: B tiles split evenly");
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 4, c = lane & 15;
  const int wr = wave / WC, wc = wave % WC;
  const int nbt = (nB + 15) >> 4, nck = d / SKC;
  for (int ag = ag_first, pass = 0; ag < nA && pass < n_pass; ag += SAG, pass++) {
    const float* xs = x;
    uint32_t soff[SPT];  // slot offsets into x, in floats (physical row * d + feature)
    bool sval[SPT];
    float ss[SPT];
#pragma unroll
    for (int w = 0; w < SPT; w++) {
      const int u = tid + w * AD_NT;
      const int r = u / Q, q = (u % Q) * 4;
      if (r < SAG) {
        sval[w] = ag + r < nA;
        soff[w] = (uint32_t)prow[1 + 2 * min(ag + r, nA - 1)] * d + q;
      } else {
        sval[w] = r - SAG < nB;
        soff[w] = (uint32_t)prow[2 + 2 * min(r - SAG, nB - 1)] * d + q;
      }
      ss[w] = 0.f;
    }
    auto load = [&](float4(&cx)[SPT], int kc) {
#pragma unroll
      for (int w = 0; w < SPT; w++) cx[w] = *(const float4*)(xs + soff[w] + kc * SKC);
    };
    // split chunk values into hi / lo and write them to LDS buffer `buf`
    auto stage = [&](const float4(&cx)[SPT], int buf) {
#pragma unroll
      for (int w = 0; w < SPT; w++) {
        const float4 e = cx[w];
        ss[w] = fmaf(e.x, e.x, ss[w]);
        ss[w] = fmaf(e.y, e.y, ss[w]);
        ss[w] = fmaf(e.z, e.z, ss[w]);
        ss[w] = fmaf(e.w, e.w, ss[w]);
        const uint32_t h01 = pack_bf16x2(e.x, e.y), h23 = pack_bf16x2(e.z, e.w);
        const uint2 hv = make_uint2(h01, h23);
        const uint2 lv = make_uint2(pack_bf16x2(e.x - __uint_as_float(h01 << 16),
                                                e.y - __uint_as_float(h01 & 0xFFFF0000u)),
                                    pack_bf16x2(e.z - __uint_as_float(h23 << 16),
                                                e.w - __uint_as_float(h23 & 0xFFFF0000u)));
        const int u = tid + w * AD_NT;
        const int r = u / Q, q = (u % Q) * 4;
        bf16_t* H = r < SAG ? Ahi + (buf * SAG + r) * SKP : Bhi + (buf * BMAX + r - SAG) * SKP;
        bf16_t* Lo = r < SAG ? Alo + (buf * SAG + r) * SKP : Blo + (buf * BMAX + r - SAG) * SKP;
        // (SAG and BMAX are multiples of 16, so r % 16 is the LDS row's)
        const int qs = Z::SWZ ? ((((q >> 3) ^ (r >> 2)) & 3) << 3) | (q & 4) : q;
        *(uint2*)(H + qs) = hv;
        *(uint2*)(Lo + qs) = lv;
      }
    };
    f32x4_t acc[2][NBW];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int t = 0; t < NBW; t++) acc[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // wave-uniform: does this wave's block hold any real (A, B) pair
    const bool act = ag + 32 * wr < nA && wc * NBW < nbt;
    auto mfma = [&](int buf) {
      if (!act) return;
      // column of this lane's 16-byte piece (rows r with r % 16 == c)
      const int gs = Z::SWZ ? ((g ^ (c >> 2)) << 3) : 8 * g;
#pragma unroll
      for (int kk = 0; kk < SKC / 32; kk++) {
        bf16x8_t ah[2], al[2];
#pragma unroll
        for (int i = 0; i < 2; i++) {
          const int row = buf * SAG + 32 * wr + 16 * i + c;
          ah[i] = *(const bf16x8_t*)(Ahi + row * SKP + 32 * kk + gs);
          al[i] = *(const bf16x8_t*)(Alo + row * SKP + 32 * kk + gs);
        }
#pragma unroll
        for (int t0 = 0; t0 < NBW; t0 += BG) {
          bf16x8_t bh[BG], bl[BG];
#pragma unroll
          for (int j = 0; j < BG; j++) {
            const int row = buf * BMAX + (wc * NBW + t0 + j) * 16 + c;
            bh[j] = *(const bf16x8_t*)(Bhi + row * SKP + 32 * kk + gs);
            bl[j] = *(const bf16x8_t*)(Blo + row * SKP + 32 * kk + gs);
          }
#pragma unroll
          for (int j = 0; j < BG; j++)
#pragma unroll
            for (int i = 0; i < 2; i++)
              acc[i][t0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[j], ah[i], acc[i][t0 + j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < BG; j++)
#pragma unroll
            for (int i = 0; i < 2; i++)
              acc[i][t0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl[j], ah[i], acc[i][t0 + j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < BG; j++)
#pragma unroll
            for (int i = 0; i < 2; i++)
              acc[i][t0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bh[j], al[i], acc[i][t0 + j], 0, 0, 0);
        }
      }
    };
    // chunk kc: MFMAs on buffer kc & 1; chunk kc + 1 (in registers `nx`)
    // staged into the other buffer; chunk kc + 3 loaded into `nx`.  The two
    // do not depend on each other: of the two waves on each SIMD one stages
    // first, so that vector and matrix work overlap.
    float4 r0[SPT], r1[SPT];
    auto step = [&](int kc, float4(&nx)[SPT]) {
      if (wave & 4) {
        if (kc + 1 < nck) stage(nx, (kc + 1) & 1);
        if (kc + 3 < nck) load(nx, kc + 3);
        mfma(kc & 1);
      } else {
        mfma(kc & 1);
        if (kc + 1 < nck) stage(nx, (kc + 1) & 1);
        if (kc + 3 < nck) load(nx, kc + 3);
      }
      __syncthreads();
    };
    load(r0, 0);
    if (nck > 1) load(r1, 1);
    stage(r0, 0);
    if (nck > 2) load(r0, 2);
    __syncthreads();
    for (int kc = 0; kc < nck; kc += 2) {
      step(kc, r1);
      if (kc + 1 < nck) step(kc + 1, r0);
    }
    // reciprocal row norms: the Q threads of a row are adjacent lanes
#pragma unroll
    for (int w = 0; w < SPT; w++) {
      float v = ss[w];
      v += lane_xor<1>(v);
      v += lane_xor<2>(v);
      v += lane_xor<4>(v);
      if (Q > 8) v += lane_xor<8>(v);
      const int u = tid + w * AD_NT;
      // (the B rows of the padding get a NaN, whose products never win)
      if ((u % Q) == 0 && (sval[w] || u / Q >= SAG))
        rn[u / Q] = sval[w] ? 1.0f / fmaxf(sqrtf(v), 1e-12f) : NAN;
    }
    __syncthreads();
    // best B per A over this wave's tiles (A rows past nA are never read; a
    // wave without a real pair has zero products, kept out by `act`)
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int ar = 32 * wr + 16 * i + c;  // A row within the pass
      const float ra = rn[min(ar, max(nA - ag, 1) - 1)];
      float bv = -INFINITY;
      int bi = 0x7fffffff;
#pragma unroll
      for (int t = 0; t < NBW; t++) {
        const int b0 = (wc * NBW + t) * 16 + 4 * g;
        const float4 rb = *(const float4*)(rn + SAG + b0);
        const float rbj[4] = {rb.x, rb.y, rb.z, rb.w};
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const float v = (acc[i][t][j] * ra) * rbj[j];
          const bool take = v > bv;
          bv = take ? v : bv;
          bi = take ? b0 + j : bi;
        }
      }
      // combine the 4 lanes of the token (lanes c, c + 16, c + 32, c + 48):
      // each swap yields the lane's own pair and its partner's
      {
        const auto v16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(bv), __float_as_uint(bv), false, false);
        const auto i16 = __builtin_amdgcn_permlane16_swap((unsigned)bi, (unsigned)bi, false, false);
        const float v0 = __uint_as_float(v16[0]), v1 = __uint_as_float(v16[1]);
        const int i0 = (int)i16[0], i1 = (int)i16[1];
        const bool t1 = v1 > v0 || (v1 == v0 && i1 < i0);
        bv = t1 ? v1 : v0;
        bi = t1 ? i1 : i0;
      }
      {
        const auto v32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(bv), __float_as_uint(bv), false, false);
        const auto i32 = __builtin_amdgcn_permlane32_swap((unsigned)bi, (unsigned)bi, false, false);
        const float v0 = __uint_as_float(v32[0]), v1 = __uint_as_float(v32[1]);
        const int i0 = (int)i32[0], i1 = (int)i32[1];
        const bool t1 = v1 > v0 || (v1 == v0 && i1 < i0);
        bv = t1 ? v1 : v0;
        bi = t1 ? i1 : i0;
      }
      if (g == 0) {
        pbv[wc * SAG + ar] = act ? bv : -INFINITY;
        pbi[wc * SAG + ar] = act ? bi : 0x7fffffff;
      }
    }
    __syncthreads();
    // partial results in B order: a later group wins only on a larger value
    for (int e = tid; e < SAG && ag + e < nA; e += AD_NT) {
      float v0 = pbv[e];
      int i0 = pbi[e];
#pragma unroll
      for (int w = 1; w < WC; w++) {
        const float v1 = pbv[w * SAG + e];
        const int i1 = pbi[w * SAG + e];
        if (v1 > v0 || (v1 == v0 && i1 < i0)) {
          v0 = v1;
          i0 = i1;
        }
      }
      bestsim[ag + e] = v0;
      best[ag + e] = i0 < nB ? i0 : 0;  // i0 >= nB only with non-finite x
    }
    __syncthreads();
  }
}

// Samples whose merge step has its best matches from similarity_kernel keep no
// similarity operands in LDS (SIM = false).
template <class Z, bool SIM>
__global__ __launch_bounds__(AD_NT) void adapt_kernel(AdaptArgs a) {
  const int i = blockIdx.x;
  // (the offsets and the live map hold an entry per workgroup of the grid:
  // nothing here waits for the counter)
  const int base = a.cu[i], T = a.cu[i + 1] - base, N = T - 1;
  const int orig = a.live[i];
  if (i >= a.cnt->nlive) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int d = a.d;
  const size_t tr_row = (size_t)(a.b - 1) * a.B + orig;

  constexpr int TMAX = Z::TMAX, AMAX = Z::AMAX, BMAX = Z::BMAX, SKP = Z::SKP, SAG = Z::SAG;
  static_assert(AMAX <= AD_NT && TMAX % 64 == 0 && AMAX % 64 == 0, "selection ranges");
  // the host's token bound selects the size class and is exact; a sample
  // beyond it (never produced by the library itself) is dropped rather than
  // overrunning the per-token LDS arrays
  if (T > TMAX || T < 1) {
    if (tid == 0) a.newlen[i] = 0;
    return;
  }
  __shared__ float sc[TMAX];
  __shared__ float szs[TMAX];
  __shared__ int prow[TMAX];  // physical row of x for each of the sample's tokens
  __shared__ int keepf[TMAX];
  // reciprocal norms of the similarity, then the keys of the selections
  __shared__ __attribute__((aligned(16))) float rn[TMAX];
  unsigned* keys = (unsigned*)rn;
  __shared__ float bestsim[AMAX];
  __shared__ int best[AMAX];
  __shared__ int pairs[AMAX];  // chosen pairs, destination << 10 | A slot
  __shared__ int srt[AMAX];    // the same in ascending order
  // similarity operands, two buffers each
  __shared__ __attribute__((aligned(16))) bf16_t Ahi[SIM ? 2 * SAG * SKP : 8];
  __shared__ __attribute__((aligned(16))) bf16_t Alo[SIM ? 2 * SAG * SKP : 8];
  __shared__ __attribute__((aligned(16))) bf16_t Bhi[SIM ? 2 * BMAX * SKP : 8];
  __shared__ __attribute__((aligned(16))) bf16_t Blo[SIM ? 2 * BMAX * SKP : 8];
  __shared__ float pbv[SIM ? Z::WC * SAG : 1];
  __shared__ int pbi[SIM ? Z::WC * SAG : 1];
  __shared__ float red[3][8];

  // CLS-attention scores are gathered here and follow the merge; learned
  // scores are computed after the merge from the merged hidden states
  const bool attnP = a.isP && a.prune_rule == 0;
  const bool router = a.isM && !a.r_fixed;
  float z = 0.f;
  if (router) {
    const float* xc = a.x + (size_t)a.rmap[base] * d;
    for (int k = tid; k < d; k += AD_NT) z = fmaf(a.router_w[k], xc[k], z);
  }
  for (int t = tid; t < T; t += AD_NT) {
    keepf[t] = 1;
    szs[t] = a.size[base + t];
    prow[t] = a.rmap[base + t];
  }
  if (attnP) {
    for (int t = tid; t < T; t += AD_NT) {
      // (three heads' scores in flight; a head past H adds nothing)
      const float* cs = a.cls_scores + (size_t)i * a.H * a.tmax + t;
      float s = cs[0];
      for (int h = 1; h < a.H; h += 3) {
        float v[3];
#pragma unroll
        for (int u = 0; u < 3; u++) v[u] = cs[(size_t)min(h + u, a.H - 1) * a.tmax];
#pragma unroll
        for (int u = 0; u < 3; u++) s = h + u < a.H ? s + v[u] : s;
      }
      sc[t] = s / (float)a.H;
    }
  }
  const int nA = (N + 1) / 2, nB = N / 2;
  if (!SIM && a.isM) {
    // best matches computed by similarity_kernel, one workgroup per pass
    for (int e = tid; e < nA; e += AD_NT) {
      bestsim[e] = a.sim_v[(base >> 1) + e];
      best[e] = a.sim_i[(base >> 1) + e];
    }
  }

  // ---------------------------------------------------------- merge --
  int r = 0;
  if (router) {
    z = bsum(z, red[0]) + a.router_b[0];
    const float m = 1.0f / (1.0f + expf(-z));
    r = merge_count(m, a.rho, a.r_b, N, a.merge_rule);
    if (tid == 0) {
      if (a.tr_r) a.tr_r[tr_row] = r;
      if (a.tr_m) a.tr_m[tr_row] = m;
    }
  } else {
    if (a.isM) {
      r = min(max(a.r_fixed[i], 0), N / 2);
      if (tid == 0 && a.tr_r) a.tr_r[tr_row] = r;
    }
    __syncthreads();
  }
  if (r > 0) {
    if (SIM)
      similarity_argmax<Z>(a.x, prow, d, nA, nB, rn, bestsim, best, Ahi, Alo, Bhi, Blo, pbv,
                           pbi);
    // top-r of A by best similarity, ties to the lower A slot
    {
      const int wide = nA > SEL_WAVE_MIN;
      const int npad = wide ? (nA + 63) & ~63 : (nA + 3) & ~3;  // <= AMAX <= AD_NT
      if (tid < npad) keys[tid] = tid < nA ? order_key(bestsim[tid]) : 0u;
    }
    __syncthreads();
    // the chosen pairs, in any order
    if (AMAX > SEL_WAVE_MIN && nA > SEL_WAVE_MIN) {
      unsigned long long sel[AMAX / 64];
      wave_top<AMAX / 64>(keys, nA, r, sel);
      int at = 0;
#pragma unroll
      for (int j = 0; j < AMAX / 64; j++) {
        if (wave == j && (sel[j] >> lane & 1)) {
          pairs[at + (int)__popcll(sel[j] & ((1ull << lane) - 1ull))] = best[tid] << 10 | tid;
          keepf[1 + 2 * tid] = 0;
        }
        at += (int)__popcll(sel[j]);
      }
    } else {
      // P adjacent lanes split the comparisons of one token (nA P <= AD_NT:
      // one round)
      const int P = rank_lanes(nA), p = tid & (P - 1), aa = tid / P;
      int rank = 0;
      if (aa < nA) rank = rank_of(keys, nA, aa, keys[aa], p, P);
      rank = lanes_sum(rank, P);
      if (aa < nA && p == 0 && rank < r) {
        pairs[rank] = best[aa] << 10 | aa;
        keepf[1 + 2 * aa] = 0;
      }
    }
    __syncthreads();
    // sorted: the sources of one destination form a group, contiguous in srt
    // and in ascending A slot.  Groups are merged independently.
    {
      const int P = rank_lanes(r), p = tid & (P - 1), q = tid / P;
      int rank = 0, key = 0;
      if (q < r) {
        key = pairs[q];
#pragma unroll 4
        for (int q2 = p; q2 < r; q2 += P) rank += pairs[q2] < key;
      }
      rank = lanes_sum(rank, P);
      if (q < r && p == 0) srt[rank] = key;
    }
    __syncthreads();
    // size-weighted merge into each receiving destination: a half wave per
    // group, its lanes at 16-byte pieces f, f + 32, f + 64 of the rows, the
    // sources SU at a time, so that their loads are in flight together (many
    // sources can share a destination: one load after the other took up to
    // 20,000 cycles at 577 tokens).  A group reads A rows and its own B row.
    constexpr int FU = 3, SU = 4, HW = AD_NT / 32;
    const int hw = tid >> 5, hl = tid & 31, d4 = d / 4;
    float4* x4 = (float4*)a.x;
    for (int q = hw; q < r; q += HW) {
      const int bb = srt[q] >> 10, a0 = srt[q] & 1023;
      if (q > 0 && srt[q - 1] >> 10 == bb) continue;
      const int tb = 2 + 2 * bb, ta0 = 1 + 2 * a0;
      float4* xb4 = x4 + (size_t)prow[tb] * d4;
      const float4* xa4 = x4 + (size_t)prow[ta0] * d4;
      const float sb = szs[tb], sa0 = szs[ta0];
      for (int f0 = hl; f0 - hl < d4; f0 += 32 * FU) {
        float4 num[FU], xa0[FU];
#pragma unroll
        for (int u = 0; u < FU; u++) {
          const int f = min(f0 + 32 * u, d4 - 1);
          num[u] = xb4[f];
          xa0[u] = xa4[f];
        }
#pragma unroll
        for (int u = 0; u < FU; u++) {
          num[u] = make_float4(sb * num[u].x, sb * num[u].y, sb * num[u].z, sb * num[u].w);
          num[u].x = num[u].x + sa0 * xa0[u].x;
          num[u].y = num[u].y + sa0 * xa0[u].y;
          num[u].z = num[u].z + sa0 * xa0[u].z;
          num[u].w = num[u].w + sa0 * xa0[u].w;
        }
        float den = sb + sa0;
        float s2 = attnP ? sc[tb] + sc[ta0] : 0.f;
        for (int pp = q + 1; pp < r && srt[pp] >> 10 == bb; pp += SU) {
          float4 xa[SU][FU];
          float sa[SU], se[SU];
          bool in[SU];
#pragma unroll
          for (int v = 0; v < SU; v++) {
            const int pr = srt[min(pp + v, r - 1)], ta = 1 + 2 * (pr & 1023);
            in[v] = pp + v < r && pr >> 10 == bb;
            sa[v] = szs[ta];
            se[v] = attnP ? sc[ta] : 0.f;
            const float4* xs4 = x4 + (size_t)prow[ta] * d4;
#pragma unroll
            for (int u = 0; u < FU; u++) xa[v][u] = xs4[min(f0 + 32 * u, d4 - 1)];
          }
#pragma unroll
          for (int v = 0; v < SU; v++) {
            if (!in[v]) break;
#pragma unroll
            for (int u = 0; u < FU; u++) {
              num[u].x = num[u].x + sa[v] * xa[v][u].x;
              num[u].y = num[u].y + sa[v] * xa[v][u].y;
              num[u].z = num[u].z + sa[v] * xa[v][u].z;
              num[u].w = num[u].w + sa[v] * xa[v][u].w;
            }
            den = den + sa[v];
            s2 = s2 + se[v];
          }
        }
#pragma unroll
        for (int u = 0; u < FU; u++)
          if (f0 + 32 * u < d4)
            xb4[f0 + 32 * u] =
                make_float4(num[u].x / den, num[u].y / den, num[u].z / den, num[u].w / den);
        if (f0 + 32 * FU >= d4 + hl && hl == 0) {  // the group's last pieces
          a.size[base + tb] = den;
          if (attnP) sc[tb] = s2;
        }
      }
    }
    if (a.tr_merge) {
      for (int q = tid; q < r; q += AD_NT) {
        const int so = a.origin[base + 1 + 2 * (srt[q] & 1023)];
        if (so >= 0 && so <= a.n0)
          a.tr_merge[tr_row * (a.n0 + 1) + so] = a.origin[base + 2 + 2 * (srt[q] >> 10)];
      }
    }
    __syncthreads();
  }

  // ------------------------------------------------------------ exit --
  bool fire = false;
  if (a.isE) {
    const float* lg = a.head_buf + (size_t)i * a.C;
    float lm = -INFINITY;
    for (int k = tid; k < a.C; k += AD_NT) lm = fmaxf(lm, lg[k]);
    lm = bmax(lm, red[1]);
    float s = 0.f;
    for (int k = tid; k < a.C; k += AD_NT) s += expf(lg[k] - lm);
    s = bsum(s, red[2]);
    const float c = 1.0f / s;
    fire = (a.delta < 1.0f) && (c >= a.delta);
    if (tid == 0 && a.tr_c) a.tr_c[tr_row] = c;
    if (fire) {
      for (int k = tid; k < a.C; k += AD_NT) a.logits[(size_t)orig * a.C + k] = lg[k];
      if (tid == 0) a.exit_block[orig] = a.b;
    }
  }

  // ----------------------------------------------------------- prune --
  if (a.isP && !fire && a.prune_rule == 1) {
    // s_t = w . z_t + beta on the merged rows (Eq. 8): one half wave per
    // token, 16-byte pieces, fixed-order half-wave sum, the rows of RU tokens
    // loaded together.  The merge's row writes above are visible here: same
    // workgroup, past a barrier.
    constexpr int RU = 4, HW = AD_NT / 32;
    const int hw = tid >> 5, hl = tid & 31, d4 = d >> 2;
    const float4* w4 = (const float4*)a.prune_w;
    const float pb = a.prune_b[0];
    for (int t0 = 1 + hw; t0 < T; t0 += RU * HW) {
      const float4* xr[RU];
      float s[RU];
#pragma unroll
      for (int u = 0; u < RU; u++) {
        xr[u] = (const float4*)(a.x + (size_t)prow[min(t0 + u * HW, T - 1)] * d);
        s[u] = 0.f;
      }
#pragma unroll 3
      for (int q = hl; q < d4; q += 32) {
        const float4 w = w4[q];
#pragma unroll
        for (int u = 0; u < RU; u++) {
          const float4 v = xr[u][q];
          s[u] = fmaf(v.x, w.x, s[u]);
          s[u] = fmaf(v.y, w.y, s[u]);
          s[u] = fmaf(v.z, w.z, s[u]);
          s[u] = fmaf(v.w, w.w, s[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < RU; u++) {
        const float v = half_sum(s[u]);
        if (hl == 0 && t0 + u * HW < T) sc[t0 + u * HW] = v + pb;
      }
    }
    __syncthreads();
  }
  int kept = T - r;  // rows kept: all but the merged sources, or the pruned ones
  if (a.isP && !fire) {
    const int k = (int)floor(__dmul_rn(a.tau_eff, (double)(N - r)));
    kept = 1 + k;
    // top-k of the kept patch tokens t = 1 + e by score, ties to the lower
    // slot (N <= 2 AD_NT)
    const bool wide = TMAX > SEL_WAVE_MIN && N > SEL_WAVE_MIN;
    const int npad = wide ? (N + 63) & ~63 : (N + 3) & ~3;  // <= TMAX
    for (int e = tid; e < npad; e += AD_NT)
      keys[e] = e < N && keepf[1 + e] ? order_key(sc[1 + e]) : 0u;
    __syncthreads();
    if (wide) {
      unsigned long long sel[TMAX / 64];
      wave_top<TMAX / 64>(keys, N, k, sel);
#pragma unroll
      for (int j = 0; j < TMAX / 64; j++)
        if ((j & 7) == wave && 64 * j + lane < N) keepf[1 + 64 * j + lane] = (sel[j] >> lane) & 1;
    } else {
      const int P = rank_lanes(N), p = tid & (P - 1);
      const int e = tid / P;
      const unsigned key = e < N ? keys[e] : 0u;
      int rank = 0;
      if (key) rank = rank_of(keys, N, e, key, p, P);
      rank = lanes_sum(rank, P);
      if (e < N && p == 0) keepf[1 + e] = key && rank < k;
    }
    __syncthreads();
  }

  for (int t = tid; t < T; t += AD_NT) a.keep[base + t] = fire ? 0 : keepf[t];
  if (tid == 0) a.newlen[i] = fire ? 0 : kept;
}

// Best matches of the merge step for long samples, one workgroup per (live
// sample, pass of SAG A rows): the same passes similarity_argmax makes one
// after the other inside adapt_kernel, spread over workgroups so that a
// small batch of long samples fills the GPU.  Results go to a.sim_v /
// a.sim_i (a sample's floor(T / 2) A tokens from half its first packed row on);
// adapt_kernel reads them instead.
template <class Z>
__global__ __launch_bounds__(AD_NT) void similarity_kernel(AdaptArgs a) {
  const int i = blockIdx.x, pass = blockIdx.y;
  if (i >= a.cnt->nlive) return;
  const int base = a.cu[i], T = a.cu[i + 1] - base, N = T - 1;
  if (T > Z::TMAX || T < 1) return;
  const int nA = (N + 1) / 2, nB = N / 2;
  if (nB < 1 || pass * Z::SAG >= nA) return;
  constexpr int TMAX = Z::TMAX, BMAX = Z::BMAX, SKP = Z::SKP, SAG = Z::SAG;
  __shared__ int prow[TMAX];
  __shared__ __attribute__((aligned(16))) float rn[TMAX];
  __shared__ __attribute__((aligned(16))) bf16_t Ahi[2 * SAG * SKP];
  __shared__ __attribute__((aligned(16))) bf16_t Alo[2 * SAG * SKP];
  __shared__ __attribute__((aligned(16))) bf16_t Bhi[2 * BMAX * SKP];
  __shared__ __attribute__((aligned(16))) bf16_t Blo[2 * BMAX * SKP];
  __shared__ float pbv[Z::WC * SAG];
  __shared__ int pbi[Z::WC * SAG];
  for (int t = threadIdx.x; t < T; t += AD_NT) prow[t] = a.rmap[base + t];
  __syncthreads();
  similarity_argmax<Z>(a.x, prow, a.d, nA, nB, rn, a.sim_v + (base >> 1), a.sim_i + (base >> 1),
                       Ahi, Alo, Bhi, Blo, pbv, pbi, pass * SAG, 1);
}

hipError_t launch_adapt(const AdaptArgs& a, hipStream_t s) {
  if (a.nlive_ub <= 0) return hipSuccess;
  if (a.T_ub <= 128 && a.d % AdSize<128>::SKC == 0) {
    adapt_kernel<AdSize<128>, true><<<a.nlive_ub, AD_NT, 0, s>>>(a);
  } else if (a.T_ub <= 256) {
    if (a.d % AdSize<256>::SKC != 0) return hipErrorInvalidValue;
    adapt_kernel<AdSize<256>, true><<<a.nlive_ub, AD_NT, 0, s>>>(a);
  } else {
    typedef AdSize<AD_TMAX> Z;
    // the split similarity: passes of 128 A rows (8 waves as 4 groups of 32
    // A rows x 2 column groups), so that each sample's B rows are read
    // ceil(nA / 128) times
    typedef AdSize<AD_TMAX, 2> ZS;
    static_assert(ZS::AMAX == Z::AMAX, "one match stride for both kernels");
    if (a.T_ub > AD_TMAX || a.d % Z::SKC != 0) return hipErrorInvalidValue;
    if (a.isM && !(a.sim_v && a.sim_i)) {
      adapt_kernel<Z, true><<<a.nlive_ub, AD_NT, 0, s>>>(a);
      return hipGetLastError();
    }
    if (a.isM) {
      // several passes of A rows: one workgroup each
      const int passes = (a.T_ub / 2 + ZS::SAG - 1) / ZS::SAG;
      similarity_kernel<ZS><<<dim3(a.nlive_ub, passes), AD_NT, 0, s>>>(a);
    }
    adapt_kernel<Z, false><<<a.nlive_ub, AD_NT, 0, s>>>(a);
  }
  return hipGetLastError();
}

// --------------------------------------------------------- compaction --
// Grid: (live sample, part); every workgroup of a sample recomputes the
// sample's offsets (cheap scans) and moves one contiguous range of its rows.
// Bound by a chain of dependent loads (counters, lengths, keep flags, row id,
// row) when the batch is small, else by the rows read and their LayerNorm
// written.  Each wave takes all keep flags of the sample in one batch of
// loads and counts a token's packed slot in their ballots, and a small batch
// is split into more parts: 13.9 -> 12.9 us per launch for DeiT-S at batch
// 256, 7.7 -> 5.3 us at batch 1, 14.8 -> 11.0 us for 64 samples at 384 x 384.
// CP_CHUNKS: wave masks that cover the longest sample; FILL: the entries past
// the survivors are written as well.
template <typename T, int CP_CHUNKS, bool FILL>
__global__ __launch_bounds__(256) void compact_kernel(CompactArgs a) {
  const int i = blockIdx.x, part = blockIdx.y;
  const int nl = a.cnt->nlive;
  // Workgroup (0, 0) always publishes the next counters, also when no sample
  // is live any more (the next block must see nlive = 0, not a stale value).
  if (i >= nl && (i != 0 || part != 0)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  __shared__ int ired[16];
  __shared__ int dsts[AD_TMAX / 8], prow[AD_TMAX / 8];  // packed slot (-1: dropped), physical row

  // offset of this sample's rows and its place among the kept samples; for
  // workgroup (0, 0) the totals instead
  const bool first = i == 0 && part == 0;
  const int lim = first || FILL ? nl : i;
  int off = 0, j = 0, tot = 0, nn = 0;
  for (int t = tid; t < lim; t += 256) {
    const int n = a.newlen[t];
    if (FILL) {
      tot += n;
      nn += n > 0;
    }
    if (!FILL || t < i) {
      off += n;
      j += n > 0;
    }
  }
  off = wave_sum_i(off);
  j = wave_sum_i(j);
  if (FILL) {
    tot = wave_sum_i(tot);
    nn = wave_sum_i(nn);
  }
  if (lane == 0) {
    ired[tid >> 6] = off;
    ired[4 + (tid >> 6)] = j;
    if (FILL) {
      ired[8 + (tid >> 6)] = tot;
      ired[12 + (tid >> 6)] = nn;
    }
  }
  __syncthreads();
  off = ired[0] + ired[1] + ired[2] + ired[3];
  j = ired[4] + ired[5] + ired[6] + ired[7];
  if (FILL) {
    tot = ired[8] + ired[9] + ired[10] + ired[11];
    nn = ired[12] + ired[13] + ired[14] + ired[15];
  } else if (first) {
    tot = off;
    nn = j;
    off = j = 0;
  }
  if (first) {
    if (tid == 0) {
      a.cnt2->nlive = nn;
      a.cnt2->M = tot;
      a.cu2[nn] = tot;
    }
    if (FILL) {
      for (int t = nn + 1 + tid; t <= a.B; t += 256) a.cu2[t] = -1;
      for (int t = nn + tid; t < a.B; t += 256) a.live2[t] = -1;
    }
  }
  if (FILL) {
    const int wg = i * (int)gridDim.y + part, nwg = (int)(gridDim.x * gridDim.y);
    for (int t = tot + wg * 256 + tid; t < a.fill_rows; t += nwg * 256) {
      a.rmap2[t] = -1;
      a.size2[t] = -1.f;
      a.origin2[t] = -1;
    }
    if (a.ln_out) {
      const size_t end = (size_t)a.fill_rows * a.d, step = (size_t)nwg * 256 * 4;
      for (size_t t = (size_t)tot * a.d + (size_t)(wg * 256 + tid) * 4; t < end; t += step)
        Store4<T>::put((T*)a.ln_out + t, make_float4(0.f, 0.f, 0.f, 0.f));
    }
  }
  if (i >= nl || a.newlen[i] == 0) return;
  const int base = a.cu[i], Tn = a.cu[i + 1] - base;
  if (Tn > 64 * CP_CHUNKS || Tn > a.n0 + 1 || Tn < 1) return;  // never kept by the adapt kernel (newlen 0)
  const int orig = a.live[i];
  if (tid == 0 && part == 0) {
    a.cu2[j] = off;
    a.live2[j] = orig;
  }
  // this part's rows (the sample's rows split into gridDim.y ranges)
  const int per = (Tn + (int)gridDim.y - 1) / (int)gridDim.y;
  const int t0 = part * per, t1 = min(Tn, t0 + per);
  if (t0 >= t1) return;
  // one thread per row of the part (AD_TMAX rows in at least 8 parts): its row id, size and origin move to the packed slot
  const bool mine = tid < t1 - t0;
  const int t = t0 + tid, tb = base + (mine ? t : t0);
  const int pr = a.rmap[tb], og = a.origin[tb];
  const float sz = a.size[tb];
  int kf[CP_CHUNKS];
#pragma unroll
  for (int c = 0; c < CP_CHUNKS; c++)
    if (c * 64 < t1) kf[c] = a.keep[base + min(c * 64 + lane, Tn - 1)];
  int n = 0;
  unsigned long long m = 0;
#pragma unroll
  for (int c = 0; c < CP_CHUNKS; c++)
    if (c * 64 < t1) {
      const unsigned long long msk = __ballot(c * 64 + lane < Tn && kf[c] != 0);
      n += c < (t >> 6) ? __popcll(msk) : 0;
      m = c == (t >> 6) ? msk : m;
    }
  const unsigned long long bit = 1ull << (t & 63);
  if (mine) {
    const int dj = (m & bit) ? n + __popcll(m & (bit - 1ull)) : -1;
    dsts[tid] = dj;
    prow[tid] = pr;
    if (dj >= 0) {
      a.rmap2[off + dj] = pr;
      a.size2[off + dj] = sz;
      a.origin2[off + dj] = og;
      if (a.tr_ids) a.tr_ids[((size_t)(a.b - 1) * a.B + orig) * (a.n0 + 1) + dj] = og;
    }
  }
  if (!a.ln_out) return;
  __syncthreads();
  // one half wave per kept row writes its LayerNorm for the next block
  // (16-byte pieces); the row itself stays where it is
  for (int q = tid >> 5; q < t1 - t0; q += 8) {
    const int dj = dsts[q];
    if (dj < 0) continue;
    ln_row_half<T>(a.x + (size_t)prow[q] * a.d, a.d, lane & 31, a.ln_g, a.ln_b,
                   (T*)a.ln_out + (size_t)(off + dj) * a.d, nullptr);
  }
}

template <typename T>
hipError_t launch_compact(const CompactArgs& a, hipStream_t s) {
  if (a.nlive_ub <= 0) return hipSuccess;
  if (a.n0 + 1 > AD_TMAX || a.d % 4 != 0 || a.d > 4 * 32 * LN_MAXV) return hipErrorInvalidValue;
  // 8 parts per sample, more while the launch stays under 1024 workgroups, up
  // to one row per half wave (per launch, averaged over the blocks of a run,
  // with 8 / more parts: 1 sample of 197 tokens 6.5 / 5.3 us, 64 samples of
  // 577 12.8 / 11.0; 4096 workgroups were slower at 256 samples, 17.0 / 12.9)
  const int parts = std::min((a.n0 + 1 + 7) / 8, std::max(8, 1024 / a.nlive_ub));
  const dim3 grid(a.nlive_ub, parts);
  if (a.fill_rows > 0) {
    if (a.n0 + 1 <= 256)
      compact_kernel<T, 4, true><<<grid, 256, 0, s>>>(a);
    else
      compact_kernel<T, AD_TMAX / 64, true><<<grid, 256, 0, s>>>(a);
  } else if (a.n0 + 1 <= 256) {
    compact_kernel<T, 4, false><<<grid, 256, 0, s>>>(a);
  } else {
    compact_kernel<T, AD_TMAX / 64, false><<<grid, 256, 0, s>>>(a);
  }
  return hipGetLastError();
}
template hipError_t launch_compact<float>(const CompactArgs&, hipStream_t);
template hipError_t launch_compact<bf16_t>(const CompactArgs&, hipStream_t);

}  // namespace fusion
