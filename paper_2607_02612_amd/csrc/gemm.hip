// Token GEMMs C[M,N] = A[M,K] . W[N,K]^T with fused epilogues (bias, GELU,
// residual add into the fp32 stream, patch-embedding scatter, fp32 logits).
//
// bf16 path: MFMA v_mfma_f32_32x32x16_bf16 on 128x128 tiles staged through
// LDS, fp32 accumulation.  fp32 path (no rounding): MFMA
// v_mfma_f32_16x16x4_f32, or LDS-tiled VALU FMA where the operands do not
// have its form.
// Rows are the packed live tokens of all samples, so ragged lengths are
// invisible here: M is read from the device counters and the grid is sized
// for an upper bound (tiles past M return at once).
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace fusion {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ void epilogue(const Epi& e, int r, int n, float acc) {
  switch (e.mode) {
    case EPI_STORE:
      ((T*)e.out)[(size_t)r * e.ldo + n] = St<T>::put(acc + e.bias[n]);
      break;
    case EPI_GELU:
      ((T*)e.out)[(size_t)r * e.ldo + n] = St<T>::put(gelu_erf(acc + e.bias[n]));
      break;
    case EPI_RESID: {
      float* p = (float*)e.out + (size_t)(e.rows ? e.rows[r] : r) * e.ldo + n;
      *p = *p + (acc + e.bias[n]);
      break;
    }
    case EPI_F32: {
      const int orow = e.rows ? e.rows[r] : r;
      ((float*)e.out)[(size_t)orow * e.ldo + n] = acc + e.bias[n];
      break;
    }
    case EPI_PATCH: {
      const int s = r / e.n0, j = r - s * e.n0;
      const size_t xr = (size_t)s * (e.n0 + 1) + 1 + j;
      ((float*)e.out)[xr * e.ldo + n] =
          (acc + e.bias[n]) + e.pos[(size_t)(1 + j) * e.ldo + n];
      break;
    }
  }
}

// ------------------------------------------------------------ fp32 VALU --
template <typename T>
__global__ __launch_bounds__(256) void gemm_valu(const T* __restrict__ A,
                                                 int lda,
                                                 const T* __restrict__ W,
                                                 int N, int K,
                                                 const int* M_dev, int M_host,
                                                 Epi e) {
  const int M = M_dev ? *M_dev : M_host;
  const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
  if (m0 >= M) return;
  __shared__ float As[16][68];
  __shared__ float Ws[16][68];
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < K; k0 += 16) {
    for (int idx = threadIdx.x; idx < 64 * 16; idx += 256) {
      const int r = idx >> 4, kk = idx & 15;
      const int gk = k0 + kk;
      const int gr = m0 + r, gn = n0 + r;
      As[kk][r] = (gr < M && gk < K) ? St<T>::get(A[(size_t)gr * lda + gk]) : 0.f;
      Ws[kk][r] = (gn < N && gk < K) ? St<T>::get(W[(size_t)gn * K + gk]) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; kk++) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; i++) {
        a[i] = As[kk][ty * 4 + i];
        w[i] = Ws[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = m0 + ty * 4 + i;
    if (r >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int n = n0 + tx * 4 + j;
      if (n < N) epilogue<T>(e, r, n, acc[i][j]);
    }
  }
}

// ------------------------------------------------------------ bf16 MFMA --
// MBx128 output tile per workgroup (MB = 256: 8 waves in a 4x2 grid; 128: 4
// waves, 2x2; 64: 2 waves side by side), each wave a 64x64 sub-tile of 2x2
// v_mfma_f32_32x32x16_bf16 blocks; launches with few 64-row tiles split
// each into 4 waves of 32x64 (1x2 blocks) instead, which changes no result.
//
// K is consumed in steps of KSV = 32 through a ring of three LDS stages
// (64-wide steps with two stages measured slower in these workgroups of 4
// waves on every shape, long K included).  A and W tiles reach LDS through the gfx950 asynchronous
// global->LDS path (global_load_lds_dwordx4): each wave-wide instruction
// writes 64 lanes x 16 bytes contiguously, i.e. 16 rows of 64 bytes,
// without passing through VGPRs, so later K steps are in
// flight while the matrix cores work on the current one (two or three
// workgroups share a CU and cover each other's load latency).  The loads
// are issued from inline assembly and their completion is awaited with
// explicit vmcnt counts (a compiler-visible LDS DMA would make every LDS
// read wait for all outstanding loads).  Each load names a wave-uniform
// operand base in SGPRs and a per-lane 32-bit byte offset, and the K loop is
// unrolled by the three ring stages, so that the loop's address arithmetic
// is scalar and the LDS reads take immediate offsets: no vector ALU work is
// left in the K loop (fc1 + GELU, which is bound by vector instruction
// issue, ran 11 % faster than with per-lane 64-bit pointers).  The 16-byte chunks of a staged row
// are XOR-permuted by (row / 4) % 4, which makes the per-lane 16-byte
// operand reads of 16 consecutive rows hit 16 disjoint bank groups.  Rows
// past M or N are clamped to the last valid row for the loads (every
// address stays in bounds) and masked in the epilogue.
//
// Epilogue: the accumulators start at the bias, and every load the epilogue
// needs (residual or position rows) is issued as one batch; for the staged
// fp32 epilogues the first round's row-map entries and addend rows are
// fetched during the last two K steps.  bf16 outputs are staged through LDS
// (the drained K ring) so that global stores are whole 256-byte row
// segments instead of 16-byte pieces of 32 different rows; the fp32
// residual update and the patch embedding are staged the same way as fp32
// rows (512-byte segments), on tiles of up to 128 rows; fp32 logits and
// 256-row tiles write directly.
//
// Tile order: blocks are dispatched round-robin over the 8 XCDs (block id %
// 8); the linear id is remapped so that each XCD walks whole row panels (all
// N tiles of one M tile back to back) and reuses the A panel in its own L2.
//
// Operand layout of v_mfma_f32_32x32x16_bf16 (64 lanes): lane l supplies
// A[row l%32][k 8*(l/32) .. +7] and B[k 8*(l/32) .. +7][col l%32]; result
// element q of lane l is C[8*(q/4) + 4*(l/32) + q%4][l%32].
constexpr int NB = 128;
constexpr int NXCD = 8;
// 64-row tiles below which a bf16 launch splits them over 32-row waves
constexpr long THIN_TILES = 768;
// 32 x 32 blocks up to which a bf16 launch takes the small-launch kernel: it
// saves the waits of a long K, while the medium kernel, which writes rows
// through LDS in whole lines, wins the sooner the less there is to wait for
// (us at the blocks, medium / small kernel: K = 64, 576 columns 432 3.1 / 2.8,
// 594 3.1 / 3.1, 1530 3.5 / 4.7; K = 192, 576 columns 594 4.2 / 4.5, 384 with
// residual 600 5.2 / 5.5, but 768 with GELU 576 5.2 / 4.8, 1512 5.4 / 5.6; K =
// 256, 384 columns 900 5.0 / 4.9, 1524 5.2 / 6.1; K = 768, 2304 columns 2016
// 11.2 / 9.0).  GELU runs slower on two medium workgroups of a CU than on the
// small ones (x64, see mid_blocks, above 32: 2713 x 768 x 192 6.6 / 6.1).
constexpr long SMALL_TILES = 2048;
inline long small_tiles(int mode, int K, long x64) {
  if (K > 320 || (mode == EPI_GELU && x64 > 32)) return SMALL_TILES;
  return K <= (mode == EPI_GELU || mode == EPI_F32 ? 128 : 192) ? 512 : 1024;
}

// 16-byte chunk c of staged row r (64-byte rows: four chunks)
__device__ __forceinline__ int kslot(int r, int c) { return c ^ ((r >> 2) & 3); }

// 16-byte store per lane: a wave-uniform 64-bit base in SGPRs plus the
// lane's 32-bit byte offset
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st16s(const void* sbase, unsigned voff, u32x4_t v) {
  asm volatile("global_store_dwordx4 %0, %1, %2" :: "v"(voff), "v"(v), "s"(sbase) : "memory");
}
// global -> LDS copy of 16 bytes per lane: a wave-uniform 64-bit base in
// SGPRs plus the lane's 32-bit byte offset (advancing to the next K step is
// scalar arithmetic); the LDS destination is the wave-uniform m0
__device__ __forceinline__ void dma16s(const void* sbase, unsigned voff, unsigned lds_byte_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds_byte_addr))
               : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// MB = 256, 128 or 64 rows per tile; each wave owns WR * 32 rows x 64
// columns (WR = 2: 2 x 2 MFMA blocks, WR = 1: 1 x 2), the waves in a grid of
// MB / (32 WR) rows x 2 columns.  Every layout accumulates each output
// element over the same 16-wide K pieces in the same order from the same
// bias start, so the results do not depend on MB or WR.  KSV = K step (32).
template <int EPI, int MB, int KSV, int WR>
__global__ __launch_bounds__(MB / (32 * WR) * 128, MB == 128 ? 3 : 1) void gemm_mfma_bf16(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W,
    int N, int K, const int* M_dev, int M_host, int n_mt, Epi e) {
  static_assert(KSV == 32, "K step of 32");
  constexpr int KS = KSV, NSTG = 3;
  constexpr int ROWB = KS * 2;                        // bytes per staged row
  constexpr int CPR = KS / 8;                         // 16-byte chunks per staged row
  constexpr int RPI = 64 / CPR;                       // rows per DMA instruction
  static_assert(WR == 1 || WR == 2, "32 or 64 rows per wave");
  constexpr int WMR = 32 * WR;                        // rows per wave
  constexpr int NWV = MB / WMR * 2;                   // waves
  constexpr int NT = NWV * 64;                        // threads
  constexpr int STGB = (MB + NB) * ROWB;              // bytes per stage
  constexpr int DMA_PER_WAVE = (MB + NB) / RPI / NWV; // DMA instructions per wave and stage
  static_assert((MB + NB) / RPI % NWV == 0, "stage split");
  const int M = M_dev ? *M_dev : M_host;
  const int n_nt = (N + NB - 1) / NB;
  const int id = blockIdx.x;
  const int xcd = id % NXCD, local = id / NXCD;
  const int mt = (local / n_nt) * NXCD + xcd, nt = local % n_nt;
  const int m0 = mt * MB, n0 = nt * NB;
  if (mt >= n_mt || m0 >= M) return;
  __shared__ __attribute__((aligned(16))) char smem[NSTG * STGB];
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  // the accumulators start at the bias of their columns (lane l owns columns
  // n0 + wn 64 + 32 j + 8 (q / 4) + 4 (l / 32) + q % 4; columns past N, never
  // stored, take a clamped bias), so no epilogue adds it
  // (with N % 8 == 0 the column base is clamped as a whole, since the lane
  // halves' columns c and c + 4 are on the same side of N: the addresses are
  // scalar; else each lane clamps its own.  Each accumulator set loads its
  // own copy, which costs no vector ALU moves)
  f32x16_t acc[WR][2];
  auto load_bias = [&](auto col) {
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const float* bp = col(n0 + wn * 64 + j * 32 + 8 * q4);
#pragma unroll
        for (int i = 0; i < WR; i++) {
          const float4 bv = *(const float4*)bp;
          acc[i][j][4 * q4 + 0] = bv.x;
          acc[i][j][4 * q4 + 1] = bv.y;
          acc[i][j][4 * q4 + 2] = bv.z;
          acc[i][j][4 * q4 + 3] = bv.w;
        }
      }
  };
  const float* bias_l = e.bias + 4 * (lane >> 5);
  if (EPI == EPI_STORE || EPI == EPI_GELU || N % 8 == 0)
    load_bias([&](int c) { return bias_l + min(c, N - 8); });
  else
    load_bias([&](int c) { return e.bias + min(c + 4 * (lane >> 5), N - 4); });

  // this lane's source row and LDS slot for each of the wave's DMA
  // instructions (8-row blocks: A rows first, then W rows)
  // per DMA instruction: a wave-uniform base (A or W) and LDS slot, and the
  // lane's byte offset from that base (rows past M or N clamped)
  const bf16_t* sbase[DMA_PER_WAVE];
  unsigned voff[DMA_PER_WAVE];
  unsigned dst[DMA_PER_WAVE];
#pragma unroll
  for (int u = 0; u < DMA_PER_WAVE; u++) {
    const int q = wave * DMA_PER_WAVE + u;
    const bool isA = q < MB / RPI;
    const int r = (isA ? q : q - MB / RPI) * RPI + lane / CPR;
    const int chunk = kslot(r, lane % CPR);
    if (isA) {
      const int gr = min(m0 + r, M - 1);
      sbase[u] = A;
      voff[u] = (unsigned)(((size_t)gr * lda + chunk * 8) * 2);
      dst[u] = q * RPI * ROWB;
    } else {
      const int gr = min(n0 + r, N - 1);
      sbase[u] = W;
      voff[u] = (unsigned)(((size_t)gr * K + chunk * 8) * 2);
      dst[u] = MB * ROWB + (q - MB / RPI) * RPI * ROWB;
    }
  }
  const int nk = K / KS;
#pragma unroll
  for (int st = 0; st < NSTG - 1; st++)
    if (st < nk) {
#pragma unroll
      for (int u = 0; u < DMA_PER_WAVE; u++)
        dma16s(sbase[u] + st * KS, voff[u], lds0 + st * STGB + dst[u]);
    }
  // staged residual / patch epilogue: the first round's row-map entries and
  // addend rows are fetched during the last two K steps, so that their
  // latency overlaps the final MFMAs
  constexpr bool STAGED = (EPI == EPI_RESID || EPI == EPI_PATCH) && MB <= 128;
  constexpr int RR = NSTG * STGB >= MB * NB * 4 ? MB : 64;  // rows per epilogue round
  constexpr int PER = RR * (NB / 4) / NT;                   // 16-byte pieces per thread
  float4 xpre[STAGED ? PER : 1];
  int ppre[STAGED ? PER : 1];
  auto row_map = [&](int rb, int* prow) {
    // one uniform branch for the whole batch: a select per entry would make
    // each load wait for every earlier memory access of the wave
    if (EPI == EPI_RESID && e.rows) {
#pragma unroll
      for (int k = 0; k < PER; k++)
        prow[k] = e.rows[min(m0 + rb + (tid + k * NT) / (NB / 4), M - 1)];
    } else {
#pragma unroll
      for (int k = 0; k < PER; k++) prow[k] = min(m0 + rb + (tid + k * NT) / (NB / 4), M - 1);
    }
  };
  auto addend = [&](int rb, const int* prow, float4* xv) {
    // the residual row (x += ...) or, for the patch embedding, the position
    // embedding of patch token 1 + j, whose output row is s (n0 + 1) + 1 + j
    // for packed row r = s n0 + j
#pragma unroll
    for (int k = 0; k < PER; k++) {
      const int idx = tid + k * NT;
      const int r = idx / (NB / 4), ch = idx % (NB / 4);
      const int m = min(m0 + rb + r, M - 1), n = min(n0 + ch * 4, N - 4);
      if (EPI == EPI_RESID) {
        xv[k] = *(const float4*)((const float*)e.out + (size_t)prow[k] * e.ldo + n);
      } else {
        const int pj = m - (m / e.n0) * e.n0;
        xv[k] = *(const float4*)(e.pos + (size_t)(1 + pj) * e.ldo + n);
      }
    }
  };
  // one K step; ST = kt % NSTG is a template argument so that the LDS
  // offsets of the stage are immediates
  auto kstep = [&](int kt, auto st_c) {
    constexpr int ST = decltype(st_c)::value;
    // stage kt has landed once at most the later stages are outstanding
    if (NSTG > 2 && kt + NSTG - 2 < nk)
      wait_vm<DMA_PER_WAVE * (NSTG - 2)>();
    else
      wait_vm<0>();
    __syncthreads();
    const int kn = kt + NSTG - 1;
    if (kn < nk) {
      constexpr int SN = (ST + NSTG - 1) % NSTG;
#pragma unroll
      for (int u = 0; u < DMA_PER_WAVE; u++)
        dma16s(sbase[u] + kn * KS, voff[u], lds0 + SN * STGB + dst[u]);
    }
    if constexpr (STAGED) {
      if (kt == max(nk - 2, 0)) row_map(0, ppre);
      if (kt == nk - 1) addend(0, ppre, xpre);
    }
    const char* Ab = smem + ST * STGB;
    const char* Bb = Ab + MB * ROWB;
#pragma unroll
    for (int ks = 0; ks < KS; ks += 16) {
      bf16x8_t a[2], b[2];
      const int c = (ks >> 3) + (lane >> 5);
#pragma unroll
      for (int i = 0; i < WR; i++) {
        const int r = wm * WMR + i * 32 + (lane & 31);
        a[i] = *(const bf16x8_t*)(Ab + r * ROWB + (kslot(r, c) << 4));
      }
#pragma unroll
      for (int j = 0; j < 2; j++) {
        const int r = wn * 64 + j * 32 + (lane & 31);
        b[j] = *(const bf16x8_t*)(Bb + r * ROWB + (kslot(r, c) << 4));
      }
      // transposed product: acc[i][j] holds C^T, so lane l owns output row
      // m = .. + (l % 32) and columns n = .. + 8 (q / 4) + 4 (l / 32) + q % 4
#pragma unroll
      for (int i = 0; i < WR; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
    }
  };
  static_assert(NSTG == 3, "the K loop is unrolled by three stages");
  for (int kt = 0; kt < nk; kt += NSTG) {
    kstep(kt, std::integral_constant<int, 0>{});
    if (kt + 1 < nk) kstep(kt + 1, std::integral_constant<int, 1>{});
    if (kt + 2 < nk) kstep(kt + 2, std::integral_constant<int, 2>{});
  }

  if (EPI == EPI_STORE || EPI == EPI_GELU) {
    // bf16 tile -> LDS -> global, 16 lanes per 256-byte row segment.  After
    // GELU (bound by vector instruction issue) the staged rows are 256
    // bytes padded to 272, so that every staging address is one per-lane
    // base plus an immediate; the plain store keeps unpadded rows with the
    // 16-byte chunk c of row r at c ^ (r % 16) (conflict-free, and faster
    // for the 256-row QKV tiles)
    constexpr bool PAD = EPI == EPI_GELU;
    constexpr int SROW = PAD ? NB * 2 + 16 : NB * 2;
    static_assert(MB * SROW <= NSTG * STGB, "epilogue staging fits");
    __syncthreads();
    char* sl = smem + (wm * WMR + (lane & 31)) * SROW + (PAD ? wn * 128 + (lane >> 5) * 8 : 0);
#pragma unroll
    for (int j = 0; j < 2; j++) {
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        // (N % 8 == 0: the lane halves' columns c and c + 4 are on the
        // same side of N, so the check is uniform)
        if (n0 + wn * 64 + j * 32 + 8 * q4 >= N) continue;
#pragma unroll
        for (int i = 0; i < WR; i++) {
          float v0 = acc[i][j][4 * q4 + 0], v1 = acc[i][j][4 * q4 + 1];
          float v2 = acc[i][j][4 * q4 + 2], v3 = acc[i][j][4 * q4 + 3];
          if (EPI == EPI_GELU) {
            v0 = gelu_erf(v0); v1 = gelu_erf(v1); v2 = gelu_erf(v2); v3 = gelu_erf(v3);
          }
          const uint2 pk = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
          if (PAD) {
            *(uint2*)(sl + i * 32 * SROW + j * 64 + q4 * 16) = pk;
          } else {
            const int r = wm * WMR + i * 32 + (lane & 31);
            const int c = wn * 64 + j * 32 + 8 * q4 + 4 * (lane >> 5);
            *(uint2*)(smem + r * SROW + (((c >> 3) ^ (r & 15)) << 4) + ((c >> 2) & 1) * 8) = pk;
          }
        }
      }
    }
    __syncthreads();
    // lane: row tid / 16 + 16 it, 16-byte piece tid % 16; the stores take a
    // uniform row-block base in SGPRs plus the lane's 32-bit byte offset
    const unsigned lo = (unsigned)(((tid >> 4) * e.ldo + (tid & 15) * 8) * 2);
    const int mr = M - m0 - (tid >> 4);   // rows from the lane's first row to M
    const bool col_ok = n0 + (tid & 15) * 8 < N;
#pragma unroll
    for (int it = 0; it < MB * (NB / 8) / NT; it++) {
      const int r = (tid >> 4) + it * (NT / 16), cc = tid & 15;
      const u32x4_t v = PAD ? *(const u32x4_t*)(smem + r * SROW + cc * 16)
                            : *(const u32x4_t*)(smem + r * SROW + ((cc ^ (r & 15)) << 4));
      if (it * (NT / 16) < mr && col_ok)
        st16s((const bf16_t*)e.out + (size_t)(m0 + it * (NT / 16)) * e.ldo + n0, lo, v);
    }
    return;
  }
  if ((EPI == EPI_RESID || EPI == EPI_PATCH) && MB <= 128) {
    // residual update (and patch embedding) through LDS: the accumulator
    // rows (bias included) are staged in fp32
    // (512-byte rows, 16-byte chunk c of row r at c ^ (r % 32)), then the
    // workgroup adds them to x with whole-row accesses (32 lanes per
    // 512-byte row segment) instead of 16-byte pieces of 32 rows per
    // instruction.  RR rows per round: the whole tile when the drained ring
    // holds it (64-row tiles), else rounds of 64 rows.
    float* x = (float*)e.out;
#pragma unroll
    for (int rb = 0; rb < MB; rb += RR) {
      __syncthreads();
      if (wm * WMR >= rb && wm * WMR < rb + RR) {
#pragma unroll
        for (int j = 0; j < 2; j++) {
#pragma unroll
          for (int i = 0; i < WR; i++) {
            const int r = wm * WMR + i * 32 + (lane & 31) - rb;
#pragma unroll
            for (int q4 = 0; q4 < 4; q4++) {
              const int c = wn * 64 + j * 32 + 8 * q4 + 4 * (lane >> 5);
              *(float4*)(smem + r * (NB * 4) + (((c >> 2) ^ (r & 31)) << 4)) =
                  make_float4(acc[i][j][4 * q4 + 0], acc[i][j][4 * q4 + 1],
                              acc[i][j][4 * q4 + 2], acc[i][j][4 * q4 + 3]);
            }
          }
        }
      }
      __syncthreads();
      float4 xv[PER];
      int prow[PER];
      if (rb == 0) {
#pragma unroll
        for (int k = 0; k < PER; k++) {
          xv[k] = xpre[k];
          prow[k] = ppre[k];
        }
      } else {
        row_map(rb, prow);
        addend(rb, prow, xv);
      }
#pragma unroll
      for (int k = 0; k < PER; k++) {
        const int idx = tid + k * NT;
        const int r = idx / (NB / 4), ch = idx % (NB / 4);
        const int m = m0 + rb + r, n = n0 + ch * 4;
        const float4 sv = *(const float4*)(smem + r * (NB * 4) + ((ch ^ (r & 31)) << 4));
        if (m < M && n < N) {
          size_t orow = (size_t)prow[k];
          if (EPI == EPI_PATCH) {
            const int sidx = m / e.n0;
            orow = (size_t)sidx * (e.n0 + 1) + 1 + (m - sidx * e.n0);
          }
          *(float4*)(x + orow * e.ldo + n) =
              make_float4(sv.x + xv[k].x, sv.y + xv[k].y, sv.z + xv[k].z, sv.w + xv[k].w);
        }
      }
    }
    return;
  }
  // residual update (other tile heights), fp32 logits (row scatter) and the
  // patch embedding: direct vector accesses
#pragma unroll
  for (int i = 0; i < WR; i++) {
    const int m = m0 + wm * WMR + i * 32 + (lane & 31);
    if (m >= M) continue;
    size_t orow = (size_t)m;
    int pj = 0;
    if (EPI == EPI_F32 || EPI == EPI_RESID) orow = e.rows ? (size_t)e.rows[m] : (size_t)m;
    if (EPI == EPI_PATCH) {
      const int sidx = m / e.n0;
      pj = m - sidx * e.n0;
      orow = (size_t)sidx * (e.n0 + 1) + 1 + pj;
    }
#pragma unroll
    for (int j = 0; j < 2; j++) {
      // all loads of the column block first (the residual or position
      // rows), then the arithmetic and the stores
      float4 xv[4];
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const int nb = min(n0 + wn * 64 + j * 32 + 8 * q4 + 4 * (lane >> 5), N - 4);
        if (EPI == EPI_RESID) xv[q4] = *(const float4*)((const float*)e.out + orow * e.ldo + nb);
        if (EPI == EPI_PATCH) xv[q4] = *(const float4*)(e.pos + (size_t)(1 + pj) * e.ldo + nb);
      }
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        const int nb = n0 + wn * 64 + j * 32 + 8 * q4 + 4 * (lane >> 5);
        if (nb >= N) continue;
        const float v0 = acc[i][j][4 * q4 + 0], v1 = acc[i][j][4 * q4 + 1];
        const float v2 = acc[i][j][4 * q4 + 2], v3 = acc[i][j][4 * q4 + 3];
        float4* po = (float4*)((float*)e.out + orow * e.ldo + nb);
        if (EPI == EPI_RESID) {
          *po = make_float4(xv[q4].x + v0, xv[q4].y + v1, xv[q4].z + v2, xv[q4].w + v3);
        } else if (EPI == EPI_F32) {
          *po = make_float4(v0, v1, v2, v3);
        } else {  // EPI_PATCH: + position embedding of token 1 + pj
          *po = make_float4(v0 + xv[q4].x, v1 + xv[q4].y, v2 + xv[q4].z, v3 + xv[q4].w);
        }
      }
    }
  }
}


// ----------------------------------------------- bf16 MFMA, small launches --
// Launches whose tiles leave most CUs idle are bound by the latency of one
// wave's chain: copies issued, stage waited for, operands read, MFMAs.  Here
// each of WM x WN waves of a workgroup computes one 32 x 32 block, NWV >= WM
// WN waves share the copies (one wave alone spends more cycles issuing them
// than in its MFMAs: 197 x 384 x 1536 took 8.7 us with one wave and 6.9 with
// three loading ones beside it), the ring holds NSTG K steps of 64, and the
// next step's operands are read before the current step's MFMAs.  The blocks
// accumulate the same 16-wide K pieces in the same order from the bias as the
// large tiles, and the epilogue does the same arithmetic, so results are
// bit-identical to theirs.  Staged rows are 128 bytes with their eight
// 16-byte chunks XOR-permuted by row % 8.  Row-map entries and residual rows
// are fetched right after the ring's first loads.  The blocks follow the
// dispatch order (a panel walk per XCD would leave XCDs idle here).
template <int EPI, int WM, int WN, int NSTG, int NWV>
__global__ __launch_bounds__(64 * NWV) void gemm_mfma_bf16_small(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int N, int K,
    const int* M_dev, int M_host, Epi e) {
  constexpr int KS = 64, ROWB = 128, RPI = 8;  // K step, bytes per staged row, rows per DMA
  constexpr int MB = 32 * WM, NBS = 32 * WN;
  constexpr bool HELP = NWV > WM * WN;
  constexpr int STGB = (MB + NBS) * ROWB;
  constexpr int DPW = (MB + NBS) / RPI / NWV;  // DMA instructions per wave and stage
  static_assert((MB + NBS) / RPI % NWV == 0, "stage split");
  const int M = M_dev ? *M_dev : M_host;
  const int n_nt = (N + NBS - 1) / NBS;
  const int mt = blockIdx.x / n_nt, nt = blockIdx.x - mt * n_nt;
  const int m0 = mt * MB, n0 = nt * NBS;
  if (m0 >= M) return;
  __shared__ __attribute__((aligned(16))) char smem[NSTG * STGB];
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const bool mm = !HELP || wave < WM * WN;
  const int wm = mm ? wave / WN : 0, wn = wave % WN, hh = lane >> 5, l32 = lane & 31;
  // this lane's output row and its physical row
  const int m = m0 + wm * 32 + l32, mc = min(m, M - 1);
  int orow = mc;
  if ((EPI == EPI_RESID || EPI == EPI_F32) && e.rows) orow = e.rows[mc];
  f32x4_t bias[4];
  const int nb = n0 + wn * 32;
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++)
    bias[q4] = *(const f32x4_t*)(e.bias + min(nb + 8 * q4 + 4 * hh, N - 4));
  const bf16_t* sbase[DPW];
  unsigned voff[DPW], dst[DPW];
#pragma unroll
  for (int u = 0; u < DPW; u++) {
    const int q = wave * DPW + u;
    const bool isA = q < MB / RPI;
    const int r = (isA ? q : q - MB / RPI) * RPI + (lane >> 3);
    const int gr = isA ? min(m0 + r, M - 1) : min(n0 + r, N - 1);
    sbase[u] = isA ? A : W;
    voff[u] = (unsigned)(((size_t)gr * (isA ? lda : K) + (((lane & 7) ^ (r & 7)) << 3)) * 2);
    dst[u] = q * RPI * ROWB;
  }
  const int nk = K / KS;
#pragma unroll
  for (int st = 0; st < NSTG - 1; st++)
    if (st < nk) {
#pragma unroll
      for (int u = 0; u < DPW; u++) dma16s(sbase[u] + st * KS, voff[u], lds0 + st * STGB + dst[u]);
    }
  f32x4_t xv[4];
  float* xr = nullptr;
  if (EPI == EPI_PATCH) {
    const int s = mc / e.n0, j = mc - s * e.n0;
    orow = s * (e.n0 + 1) + 1 + j;
    xr = (float*)e.pos + (size_t)(1 + j) * e.ldo;
  } else if (EPI == EPI_RESID) {
    xr = (float*)e.out + (size_t)orow * e.ldo;
  }
  if (EPI == EPI_RESID || EPI == EPI_PATCH) {
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++)
      xv[q4] = *(const f32x4_t*)(xr + min(nb + 8 * q4 + 4 * hh, N - 4));
  }
  f32x16_t acc;
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++)
#pragma unroll
    for (int q = 0; q < 4; q++) acc[4 * q4 + q] = bias[q4][q];
  bf16x8_t fa[2][4], fb[2][4];
  auto fetch = [&](int st, int p) {
    const char* Ab = smem + st * STGB + (wm * 32 + l32) * ROWB;
    const char* Bb = smem + st * STGB + (MB + wn * 32 + l32) * ROWB;
#pragma unroll
    for (int ks = 0; ks < 4; ks++) {
      const int ch = ((2 * ks + hh) ^ (l32 & 7)) << 4;
      fa[p][ks] = *(const bf16x8_t*)(Ab + ch);
      fb[p][ks] = *(const bf16x8_t*)(Bb + ch);
    }
  };
  // step kt: MFMAs on the operands in registers; operands of step kt + 1 read
  // once its stage has landed; the stage of step kt + NSTG loaded into the
  // slot that step kt was read from
  auto landed = [&](int kt) {  // stage kt and every earlier one
    if (kt + NSTG - 2 < nk)
      wait_vm<DPW * (NSTG - 2)>();
    else
      wait_vm<0>();
    __syncthreads();
  };
  int sr = 0, sw = NSTG - 1;
  auto step = [&](int kt, int p) {
    if (kt + 1 < nk) {
      if (kt + NSTG - 1 < nk) {
        // (slot sw held step kt - 1, whose operands every wave has read)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int u = 0; u < DPW; u++)
          dma16s(sbase[u] + (kt + NSTG - 1) * KS, voff[u], lds0 + sw * STGB + dst[u]);
        sw = sw + 1 == NSTG ? 0 : sw + 1;
      }
      sr = sr + 1 == NSTG ? 0 : sr + 1;
      landed(kt + 1);
      if (mm) fetch(sr, p ^ 1);
    }
    if (mm)
#pragma unroll
    for (int ks = 0; ks < 4; ks++)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[p][ks], fa[p][ks], acc, 0, 0, 0);
  };
  landed(0);
  if (mm) fetch(0, 0);
  for (int kt = 0; kt < nk; kt += 2) {
    step(kt, 0);
    if (kt + 1 < nk) step(kt + 1, 1);
  }
  if (m >= M || !mm) return;
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++) {
    const int n = nb + 8 * q4 + 4 * hh;
    if (n >= N) continue;
    f32x4_t v = {acc[4 * q4], acc[4 * q4 + 1], acc[4 * q4 + 2], acc[4 * q4 + 3]};
    if (EPI == EPI_STORE || EPI == EPI_GELU) {
      if (EPI == EPI_GELU) {
#pragma unroll
        for (int q = 0; q < 4; q++) v[q] = gelu_erf(v[q]);
      }
      *(uint2*)((bf16_t*)e.out + (size_t)m * e.ldo + n) =
          make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
    } else {
      if (EPI == EPI_RESID) v = xv[q4] + v;
      if (EPI == EPI_PATCH) v = v + xv[q4];
      *(f32x4_t*)((float*)e.out + (size_t)orow * e.ldo + n) = v;
    }
  }
}

// Workgroups by the number of 32 x 32 blocks (us per launch at the rows, N x
// K given; large-tile kernel / 1 block / 2 blocks / 4 blocks a workgroup):
//   up to 256, one per CU: one block and four loading waves
//     (197, 384 x 1536: 15.2 / 6.9 / 8.2 / 9.5; 197, 1152 x 384: 5.3 / 3.5 / 3.8 / 4.6)
//   up to 1024, two workgroups per CU: two blocks (788, 1152 x 384: 5.6 / 5.0 /
//     4.7 / 5.1; 1337, 768 x 3072, 1008 blocks: two 18.7, four 20.2; but 2907,
//     384 x 1536, 1092 blocks: two 17.4, four 15.5)
//   up to small_tiles(): four blocks, which load each operand row for two
//     (1576, 1152 x 384: 6.9 / 8.2 / 7.7 / 6.2; 2400, 768 x 3072: 35.6 / 41 / 37 / 26)
//   beyond, the medium kernel (2201, 1152 x 384: 7.7 against 8.6)
template <int EPI>
void launch_small(const bf16_t* A, int lda, const bf16_t* W, int N, int K, const int* M_dev,
                  int M_host, int M_ub, long t32, const Epi& e, hipStream_t s) {
  const int m32 = (M_ub + 31) / 32, m64 = (M_ub + 63) / 64, n32 = (N + 31) / 32, n64 = (N + 63) / 64;
  if (t32 <= 256)
    gemm_mfma_bf16_small<EPI, 1, 1, 4, 4><<<m32 * n32, 256, 0, s>>>(A, lda, W, N, K, M_dev, M_host, e);
  else if (t32 <= 1024)
    gemm_mfma_bf16_small<EPI, 1, 2, 4, 4><<<m32 * n64, 256, 0, s>>>(A, lda, W, N, K, M_dev, M_host, e);
  else
    gemm_mfma_bf16_small<EPI, 2, 2, 3, 4><<<m64 * n64, 256, 0, s>>>(A, lda, W, N, K, M_dev, M_host, e);
}

// ---------------------------------------------- bf16 MFMA, medium launches --
// Launches whose 64- or 128-row tiles fit the chip once are bound by how fast
// a CU gets its operands: the three workgroups that share an A panel fetch the
// same lines, so few distinct bytes are in flight, and 64-byte rows use half
// of each cache line (197 images, fc2: the K loop without its copies took half
// the time; without its MFMAs or LDS reads it took all of it).  Here K steps
// of 64 stage whole 128-byte lines, and 8 waves of BI 32 x 32 blocks (two
// workgroups a CU, so 16 waves) hide more of each other's latency: the
// operands of each half step are read while the other half multiplies.  128 x
// 128 tiles (BI = 2) in two stages, 64 x 128 (BI = 1) in three.  The blocks
// accumulate the same 16-wide K pieces in the same order from the bias as the
// other kernels, and the epilogue does the same arithmetic, so results are
// bit-identical to theirs.  Staged rows are 128 bytes with their eight 16-byte
// chunks XOR-permuted by row % 8.  Every wave stages its own 32-row blocks
// through the drained ring, so its output rows are written in 128-byte (fp32)
// or 64-byte (bf16) pieces without another barrier.
template <int EPI, int BI, int NSTG>
__global__ __launch_bounds__(512, 2) void gemm_mfma_bf16_mid(
    const bf16_t* __restrict__ A, int lda, const bf16_t* __restrict__ W, int N, int K,
    const int* M_dev, int M_host, int n_mt, Epi e) {
  constexpr int KS = 64, ROWB = 128, RPI = 8;     // K step, bytes per staged row, rows per DMA
  constexpr int WM = 2, WN = 4, NWV = WM * WN;    // wave grid
  constexpr int WR = 32 * BI, MB = WR * WM;       // rows per wave and tile; NB = 32 WN columns
  constexpr int STGB = (MB + NB) * ROWB;
  constexpr int DPW = (MB + NB) / RPI / NWV;      // DMA instructions per wave and stage
  static_assert((MB + NB) / RPI % NWV == 0 && NB == 32 * WN, "stage split");
  const int M = M_dev ? *M_dev : M_host;
  const int n_nt = (N + NB - 1) / NB;
  const int id = blockIdx.x;
  const int xcd = id % NXCD, local = id / NXCD;
  const int mt = (local / n_nt) * NXCD + xcd, nt = local % n_nt;
  const int m0 = mt * MB, n0 = nt * NB;
  if (mt >= n_mt || m0 >= M) return;
  __shared__ __attribute__((aligned(16))) char smem[NSTG * STGB];
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave / WN, wn = wave % WN, hh = lane >> 5, l32 = lane & 31;
  const int nw = n0 + wn * 32;                    // the wave's first column
  const bf16_t* sbase[DPW];
  unsigned voff[DPW], dst[DPW];
#pragma unroll
  for (int u = 0; u < DPW; u++) {
    const int q = wave * DPW + u;
    const bool isA = q < MB / RPI;
    const int r = (isA ? q : q - MB / RPI) * RPI + (lane >> 3);
    const int gr = isA ? min(m0 + r, M - 1) : min(n0 + r, N - 1);
    sbase[u] = isA ? A : W;
    voff[u] = (unsigned)(((size_t)gr * (isA ? lda : K) + (((lane & 7) ^ (r & 7)) << 3)) * 2);
    dst[u] = q * RPI * ROWB;
  }
  const int nk = K / KS;
#pragma unroll
  for (int st = 0; st < NSTG - 1; st++)
    if (st < nk) {
#pragma unroll
      for (int u = 0; u < DPW; u++) dma16s(sbase[u] + st * KS, voff[u], lds0 + st * STGB + dst[u]);
    }
  f32x16_t acc[BI];
#pragma unroll
  for (int q4 = 0; q4 < 4; q4++) {
    const f32x4_t bv = *(const f32x4_t*)(e.bias + min(nw + 8 * q4 + 4 * hh, N - 4));
#pragma unroll
    for (int i = 0; i < BI; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) acc[i][4 * q4 + q] = bv[q];
  }
  bf16x8_t fa[2][2][BI], fb[2][2];
  auto fetch = [&](auto st_c, auto p_c) {  // half p of the stage in slot ST
    constexpr int ST = decltype(st_c)::value, p = decltype(p_c)::value;
    const char* Ab = smem + ST * STGB + (wm * WR + l32) * ROWB;
    const char* Bb = smem + ST * STGB + (MB + wn * 32 + l32) * ROWB;
#pragma unroll
    for (int ks = 0; ks < 2; ks++) {
      const int c = ((4 * p + 2 * ks + hh) ^ (l32 & 7)) << 4;
#pragma unroll
      for (int i = 0; i < BI; i++) fa[p][ks][i] = *(const bf16x8_t*)(Ab + i * 32 * ROWB + c);
      fb[p][ks] = *(const bf16x8_t*)(Bb + c);
    }
  };
  auto mma = [&](auto p_c) {
    constexpr int p = decltype(p_c)::value;
#pragma unroll
    for (int ks = 0; ks < 2; ks++)
#pragma unroll
      for (int i = 0; i < BI; i++)
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[p][ks], fa[p][ks][i], acc[i], 0, 0, 0);
  };
  auto landed = [&](int kt) {  // stage kt and every earlier one
    if (kt + NSTG - 2 < nk)
      wait_vm<DPW * (NSTG - 2)>();
    else
      wait_vm<0>();
    __syncthreads();
  };
  // step kt, its first half's operands in registers: stage kt + NSTG - 1 goes
  // into the slot of step kt - 1, whose operands every wave had read before
  // the barrier that step kt - 1 ended with
  typedef std::integral_constant<int, 0> H0;
  typedef std::integral_constant<int, 1> H1;
  auto step = [&](int kt, auto st_c) {
    constexpr int ST = decltype(st_c)::value;
    if (kt + NSTG - 1 < nk) {
      constexpr int SN = (ST + NSTG - 1) % NSTG;
#pragma unroll
      for (int u = 0; u < DPW; u++)
        dma16s(sbase[u] + (kt + NSTG - 1) * KS, voff[u], lds0 + SN * STGB + dst[u]);
    }
    fetch(st_c, H1{});
    mma(H0{});
    if (kt + 1 < nk) {
      landed(kt + 1);
      fetch(std::integral_constant<int, (ST + 1) % NSTG>{}, H0{});
    }
    mma(H1{});
  };
  landed(0);
  fetch(H0{}, H0{});
  for (int kt = 0; kt < nk; kt += NSTG) {
    step(kt, std::integral_constant<int, 0>{});
    if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>{});
    if constexpr (NSTG > 2)
      if (kt + 2 < nk) step(kt + 2, std::integral_constant<int, 2>{});
  }
  static_assert(NSTG == 2 || NSTG == 3, "the K loop is unrolled by the stages");
  __syncthreads();  // the ring is drained
  if constexpr (EPI == EPI_STORE || EPI == EPI_GELU) {
    constexpr int SROW = 64 + 16;  // staged bf16 row of 32 columns
    static_assert(NWV * WR * SROW <= NSTG * STGB, "epilogue staging fits");
    char* sw = smem + wave * WR * SROW;
#pragma unroll
    for (int i = 0; i < BI; i++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        float v0 = acc[i][4 * q4 + 0], v1 = acc[i][4 * q4 + 1];
        float v2 = acc[i][4 * q4 + 2], v3 = acc[i][4 * q4 + 3];
        if (EPI == EPI_GELU) {
          v0 = gelu_erf(v0); v1 = gelu_erf(v1); v2 = gelu_erf(v2); v3 = gelu_erf(v3);
        }
        *(uint2*)(sw + (i * 32 + l32) * SROW + q4 * 16 + hh * 8) =
            make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
      }
    // 4 lanes per row
#pragma unroll
    for (int k = 0; k < WR / 16; k++) {
      const int r = (lane >> 2) + 16 * k, n = nw + (lane & 3) * 8, m = m0 + wm * WR + r;
      const uint4 v = *(const uint4*)(sw + r * SROW + (lane & 3) * 16);
      if (m < M && n < N) *(uint4*)((bf16_t*)e.out + (size_t)m * e.ldo + n) = v;
    }
  } else {
    constexpr int SROW = 128 + 16;  // staged fp32 row
    static_assert(NWV * 32 * SROW <= NSTG * STGB, "epilogue staging fits");
    char* sw = smem + wave * 32 * SROW;
    const int nc = nw + (lane & 7) * 4, ncc = min(nc, N - 4);  // this lane's columns
#pragma unroll
    for (int i = 0; i < BI; i++) {
      // 8 lanes per row: output rows and addend rows of the lane's 4 pieces
      float4 xv[4];
      size_t orow[4];
      int m[4];
#pragma unroll
      for (int k = 0; k < 4; k++) {
        m[k] = m0 + wm * WR + i * 32 + (lane >> 3) + 8 * k;
        orow[k] = (size_t)min(m[k], M - 1);
      }
      if ((EPI == EPI_RESID || EPI == EPI_F32) && e.rows) {
#pragma unroll
        for (int k = 0; k < 4; k++) orow[k] = (size_t)e.rows[orow[k]];
      }
#pragma unroll
      for (int k = 0; k < 4; k++) {
        if (EPI == EPI_RESID) xv[k] = *(const float4*)((const float*)e.out + orow[k] * e.ldo + ncc);
        if (EPI == EPI_PATCH) {
          const int sm = (int)orow[k] / e.n0, pj = (int)orow[k] - sm * e.n0;
          orow[k] = (size_t)sm * (e.n0 + 1) + 1 + pj;
          xv[k] = *(const float4*)(e.pos + (size_t)(1 + pj) * e.ldo + ncc);
        }
      }
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++)
        *(float4*)(sw + l32 * SROW + q4 * 32 + hh * 16) = make_float4(
            acc[i][4 * q4], acc[i][4 * q4 + 1], acc[i][4 * q4 + 2], acc[i][4 * q4 + 3]);
#pragma unroll
      for (int k = 0; k < 4; k++) {
        float4 v = *(const float4*)(sw + ((lane >> 3) + 8 * k) * SROW + (lane & 7) * 16);
        if (EPI != EPI_F32)
          v = make_float4(v.x + xv[k].x, v.y + xv[k].y, v.z + xv[k].z, v.w + xv[k].w);
        if (m[k] < M && nc < N) *(float4*)((float*)e.out + orow[k] * e.ldo + nc) = v;
      }
    }
  }
}

// Medium launches by the tiles of the XCD that gets the most row panels (all
// column tiles of a panel run on one XCD, whose 32 CUs hold 64 of these
// workgroups at a time; of the 3-stage kernel's 128-row ones 96).  82 panels of
// 6 tiles are 492 in all, but 66 on two XCDs: 10431 x 768 x 768 took 39.0 us as
// "fits once" and takes 35 in the 3-stage kernel; 5200 x 768 x 192 + GELU, 66
// 64-row tiles there, 9.4 and 8.4 in 128-row ones.  us per launch on cold
// operands, 3-stage kernel / this one:
//   64-row tiles fit once: BI = 1 (384 x 1536 with residual: 2400 rows 18.5 /
//     13.4, 9000 rows 24.8 / 20.4; 1536 x 384 with GELU: 2400 rows 10.1 / 8.5)
//   128-row tiles fit once: BI = 2 (384 x 1536: 12608 rows 35.9 / 26.2, 20000
//     rows 46.9 / 33.1; 768 x 3072: 9456 rows 85.9 / 52.2; 1152 x 384: 6304
//     rows 14.8 / 10.8; 1536 x 384: 4700 rows 17.7 / 12.5)
//   up to 96: the 3-stage kernel, which holds them all (384 x 1536: 28000
//     rows 58.9 / 60.8; 1152 x 384: 9000 rows 15.7 / 16.8)
//   up to 128: BI = 2 in two even rounds (384 x 1536: 36928 rows 87.5 / 77.4;
//     384 x 384: 40000 rows 41.6 / 37.8), not with GELU, whose vector work
//     prefers three independent workgroups (1536 x 384 inside a pass: 9500
//     rows 25.4 / 28.0)
//   plain store further: K of 384 and more up to 240 (2304 x 768: 12608 rows
//     66.2 / 57.2; 1152 x 384 inside a pass, operands just written: 19200 rows
//     29.2 / 27.4, 23500 rows 34.4 / 33.6), below to 112 (576 x 192: 20922 rows
//     15.2 / 14.7, 24898 17.1 / 17.6, inside a pass 39400 rows 20.8 / 21.7)
//   beyond, the 3-stage kernel (384 x 1536: 50432 rows 109.9 / 108.8)
int mid_blocks(int mode, int K, long x64, long x128) {
  if (x64 <= 64) return 1;
  const long most = mode == EPI_GELU ? 64
                    : mode != EPI_STORE ? 128 : K >= 384 ? 240 : 112;
  if (x128 <= 64 || (x128 > 96 && x128 <= most)) return 2;
  return 0;
}
template <int EPI>
void launch_mid(int bi, const bf16_t* A, int lda, const bf16_t* W, int N, int K, const int* M_dev,
                int M_host, int M_ub, const Epi& e, hipStream_t s) {
  const int n_mt = (M_ub + 64 * bi - 1) / (64 * bi);
  const int grid = (n_mt + NXCD - 1) / NXCD * NXCD * ((N + NB - 1) / NB);
  if (bi == 1)
    gemm_mfma_bf16_mid<EPI, 1, 3><<<grid, 512, 0, s>>>(A, lda, W, N, K, M_dev, M_host, n_mt, e);
  else
    gemm_mfma_bf16_mid<EPI, 2, 2><<<grid, 512, 0, s>>>(A, lda, W, N, K, M_dev, M_host, n_mt, e);
}

// ------------------------------------------------------------ fp32 MFMA --
// MB x MB output tile per workgroup, 4 waves in a 2 x 2 grid, each wave
// (MB / 32)^2 blocks of v_mfma_f32_16x16x4_f32.  K is consumed KS floats at a
// time through a ring of NSTG stages filled by the asynchronous global -> LDS
// path: 32 (128-byte rows, their eight chunks XOR-permuted by row % 8) or,
// where K is not a multiple of it, 16 (64-byte rows, the bf16 kernel's staged
// layout).  A lane's 16-byte piece of a staged row feeds four MFMA steps: slot
// g = l / 16 of step i is k = 16 kt + 4 g + i, in this order for every tile
// size and KS, so a row's result does not depend on the tile.  Large products
// are bound by the fp32 matrix rate (nominal 157 TFLOP/s), small ones by the
// latency of the first stages and the barriers of the K steps (1573 x 1152 x
// 384: 62 us for the general kernel, 20 for this one).  The product is
// transposed (W as the row operand): lane (g, c) holds row m = .. + c, columns
// n = .. + 4 g + q.
template <int MB, int NSTG, int KS>
__global__ __launch_bounds__(256) void gemm_mfma_f32(const float* __restrict__ A, int lda,
                                                     const float* __restrict__ W, int N, int K,
                                                     const int* M_dev, int M_host, int n_mt,
                                                     int vec, Epi e) {
  constexpr int ROWB = KS * 4, CPR = KS / 4, RPI = 64 / CPR;  // bytes, chunks per row; rows per DMA
  constexpr int WB = MB / 2, NW = WB / 16;       // wave tile rows, 16-row blocks
  constexpr int STGB = 2 * MB * ROWB;            // bytes per stage: A rows, W rows
  constexpr int DPW = 2 * MB / RPI / 4;          // DMA instructions per wave and stage
  static_assert(KS == 16 || KS == 32, "64- or 128-byte rows");
  const int M = M_dev ? *M_dev : M_host;
  const int n_nt = (N + MB - 1) / MB;
  const int id = blockIdx.x;
  const int xcd = id % NXCD, local = id / NXCD;
  const int mt = (local / n_nt) * NXCD + xcd, nt = local % n_nt;
  const int m0 = mt * MB, n0 = nt * MB;
  if (mt >= n_mt || m0 >= M) return;
  __shared__ __attribute__((aligned(16))) char smem[NSTG * STGB];
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 4, c = lane & 15;

  // 16-byte chunk c of staged row r
  auto slot = [](int r, int c) { return KS == 16 ? kslot(r, c) : c ^ (r & 7); };
  const float* sbase[DPW];
  unsigned voff[DPW], dst[DPW];
#pragma unroll
  for (int u = 0; u < DPW; u++) {
    const int q = wave * DPW + u;  // block of RPI rows: A rows first, then W rows
    const bool isA = q < MB / RPI;
    const int r = (isA ? q : q - MB / RPI) * RPI + lane / CPR;
    // (from the tile's first row: operands of any size within 32-bit offsets)
    const int dr = isA ? min(r, M - 1 - m0) : min(r, N - 1 - n0);
    sbase[u] = isA ? A + (size_t)m0 * lda : W + (size_t)n0 * K;
    voff[u] = (unsigned)((dr * (isA ? lda : K) + slot(r, lane % CPR) * 4) * 4);
    dst[u] = q * RPI * ROWB;
  }
  const int nk = K / KS;
#pragma unroll
  for (int st = 0; st < NSTG - 1; st++)
    if (st < nk) {
#pragma unroll
      for (int u = 0; u < DPW; u++) dma16s(sbase[u] + st * KS, voff[u], lds0 + st * STGB + dst[u]);
    }
  f32x4_t acc[NW][NW];
#pragma unroll
  for (int i = 0; i < NW; i++)
#pragma unroll
    for (int j = 0; j < NW; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int st = 0, sn = NSTG - 1;  // ring slots of step kt and of step kt + NSTG - 1
  for (int kt = 0; kt < nk; kt++) {
    if (kt + NSTG - 2 < nk)
      wait_vm<DPW * (NSTG - 2)>();
    else
      wait_vm<0>();
    __syncthreads();
    if (kt + NSTG - 1 < nk) {
#pragma unroll
      for (int u = 0; u < DPW; u++)
        dma16s(sbase[u] + (kt + NSTG - 1) * KS, voff[u], lds0 + sn * STGB + dst[u]);
    }
    const char* Ab = smem + st * STGB;
    const char* Bb = Ab + MB * ROWB;
    f32x4_t av[KS / 16][NW], bv[KS / 16][NW];
#pragma unroll
    for (int h = 0; h < KS / 16; h++)
#pragma unroll
      for (int i = 0; i < NW; i++) {
        const int ra = wm * WB + i * 16 + c, rb = wn * WB + i * 16 + c;
        av[h][i] = *(const f32x4_t*)(Ab + ra * ROWB + (slot(ra, 4 * h + g) << 4));
        bv[h][i] = *(const f32x4_t*)(Bb + rb * ROWB + (slot(rb, 4 * h + g) << 4));
      }
#pragma unroll
    for (int h = 0; h < KS / 16; h++)
#pragma unroll
      for (int q = 0; q < 4; q++)
#pragma unroll
        for (int i = 0; i < NW; i++)
#pragma unroll
          for (int j = 0; j < NW; j++)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv[h][j][q], av[h][i][q], acc[i][j], 0, 0, 0);
    st = st + 1 == NSTG ? 0 : st + 1;
    sn = sn + 1 == NSTG ? 0 : sn + 1;
  }
#pragma unroll
  for (int i = 0; i < NW; i++) {
    const int m = m0 + wm * WB + i * 16 + c;
    if (m >= M) continue;
    if (!vec) {  // rows or columns that 16-byte accesses do not fit
#pragma unroll
      for (int j = 0; j < NW; j++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int n = n0 + wn * WB + j * 16 + 4 * g + q;
          if (n < N) epilogue<float>(e, m, n, acc[i][j][q]);
        }
      continue;
    }
    size_t orow = (size_t)m, prow = 0;
    if (e.mode == EPI_PATCH) {
      const int s = m / e.n0;
      prow = 1 + (m - s * e.n0);
      orow = (size_t)s * (e.n0 + 1) + prow;
    } else if (e.rows) {
      orow = (size_t)e.rows[m];
    }
#pragma unroll
    for (int j = 0; j < NW; j++) {
      const int n = n0 + wn * WB + j * 16 + 4 * g;
      if (n >= N) continue;
      f32x4_t v = acc[i][j] + *(const f32x4_t*)(e.bias + n);
      f32x4_t* po = (f32x4_t*)((float*)e.out + orow * e.ldo + n);
      if (e.mode == EPI_GELU) {
#pragma unroll
        for (int q = 0; q < 4; q++) v[q] = gelu_erf(v[q]);
      }
      if (e.mode == EPI_RESID) v = *po + v;
      if (e.mode == EPI_PATCH) v = v + *(const f32x4_t*)(e.pos + prow * e.ldo + n);
      *po = v;
    }
  }
}

template <>
hipError_t launch_gemm<float>(const float* A, int lda, const float* W, int N,
                              int K, const int* M_dev, int M_host, int M_ub, int M_est,
                              const Epi& e, hipStream_t s) {
  if (M_ub <= 0) return hipSuccess;
  const int Mx = M_est > 0 ? std::min(M_est, M_ub) : M_ub;
  // matrix cores: whole 16-float K steps, 16-byte aligned operand rows, a
  // tile's 64 rows within 32-bit byte offsets (so whether a row takes this
  // order of sums does not depend on the number of rows); anything else takes
  // the general kernel
  if (K >= 16 && K % 16 == 0 && lda % 4 == 0 && ((uintptr_t)A | (uintptr_t)W) % 16 == 0 &&
      std::max(lda, K) <= 1 << 22) {
    const int vec = N % 4 == 0 && e.ldo % 4 == 0 &&
                    ((uintptr_t)e.out | (uintptr_t)e.bias | (uintptr_t)e.pos) % 16 == 0;
    auto tiles = [&](int mb) { return (long)((Mx + mb - 1) / mb) * ((N + mb - 1) / mb); };
    auto grid = [&](int mb) {
      return ((M_ub + mb - 1) / mb + NXCD - 1) / NXCD * NXCD * ((N + mb - 1) / mb);
    };
    // K steps of 32 (whole 128-byte lines) where K has them: 32-row tiles in
    // three stages, of which more run at once and wait for less, or 64-row
    // tiles in two, which read each operand half as often.  The 64-row ones
    // win with more than three of them a CU, the sooner the longer K (us,
    // 32-row / 64-row tiles at the number of 64-row tiles: K = 192, 384
    // columns 1800 37.3 / 38.5, 1152 columns 2394 43.3 / 42.2; K = 384, 1536
    // columns 1200 39.8 / 41.7, 2400 74.8 / 69.2; K = 768, 384 columns 1056
    // 65.4 / 67.1, 1536 columns 1128 68.3 / 63.8; K = 1536, 888 110 / 98;
    // over 231 shapes the rule loses 0.5 % to the better of the two)
    auto go = [&](auto mb_c, auto st_c, auto ks_c) {
      constexpr int MB = decltype(mb_c)::value;
      gemm_mfma_f32<MB, decltype(st_c)::value, decltype(ks_c)::value><<<grid(MB), 256, 0, s>>>(
          A, lda, W, N, K, M_dev, M_host, (M_ub + MB - 1) / MB, vec, e);
    };
    typedef std::integral_constant<int, 16> I16;
    typedef std::integral_constant<int, 32> I32;
    typedef std::integral_constant<int, 64> I64;
    if (K % 32 == 0) {
      if (tiles(64) >= 768 + (3 << 16) / std::max(K, 192))
        go(I64{}, std::integral_constant<int, 2>{}, I32{});
      else
        go(I32{}, std::integral_constant<int, 3>{}, I32{});
    } else if (tiles(64) >= 512) {
      go(I64{}, std::integral_constant<int, 6>{}, I16{});
    } else {
      go(I32{}, std::integral_constant<int, 8>{}, I16{});
    }
    return hipGetLastError();
  }
  dim3 grid((M_ub + 63) / 64, (N + 63) / 64);
  gemm_valu<float><<<grid, 256, 0, s>>>(A, lda, W, N, K, M_dev, M_host, e);
  return hipGetLastError();
}

template <>
hipError_t launch_gemm<bf16_t>(const bf16_t* A, int lda, const bf16_t* W,
                               int N, int K, const int* M_dev, int M_host,
                               int M_ub, int M_est, const Epi& e, hipStream_t s) {
  if (M_ub <= 0) return hipSuccess;
  // the kernel is chosen for the rows expected, the grid covers the bound
  // (every kernel gives the same bits)
  const int Mx = M_est > 0 ? std::min(M_est, M_ub) : M_ub;
  // The K steps need K % 32 == 0 and 16-byte aligned rows; the vector
  // epilogues need N and the output stride to be multiples of 8 (bf16
  // outputs) or 4 (fp32 outputs).  The model creation rejects bf16 shapes
  // that do not satisfy this.
  if (K % 32 != 0 || lda % 8 != 0 || K <= 0) return hipErrorInvalidValue;
  if (N % 4 != 0 || e.ldo % 4 != 0) return hipErrorInvalidValue;
  // the loads take 32-bit byte offsets from the operand bases
  if ((size_t)M_ub * lda * 2 > 0xFFFFFFFFull || (size_t)N * K * 2 > 0xFFFFFFFFull)
    return hipErrorInvalidValue;
  if ((e.mode == EPI_STORE || e.mode == EPI_GELU) && (N % 8 != 0 || e.ldo % 8 != 0))
    return hipErrorInvalidValue;
  const int n_nt = (N + NB - 1) / NB;
  // tiles of mb rows of the XCD that gets the most row panels
  auto per_xcd = [&](int mb) { return (long)((Mx + mb * NXCD - 1) / (mb * NXCD)) * n_nt; };
  const long t32 = (long)((Mx + 31) / 32) * ((N + 31) / 32);
  if (K % 64 == 0 && t32 <= small_tiles(e.mode, K, per_xcd(64))) {
    switch (e.mode) {
      case EPI_STORE: launch_small<EPI_STORE>(A, lda, W, N, K, M_dev, M_host, M_ub, t32, e, s); break;
      case EPI_GELU: launch_small<EPI_GELU>(A, lda, W, N, K, M_dev, M_host, M_ub, t32, e, s); break;
      case EPI_RESID: launch_small<EPI_RESID>(A, lda, W, N, K, M_dev, M_host, M_ub, t32, e, s); break;
      case EPI_F32: launch_small<EPI_F32>(A, lda, W, N, K, M_dev, M_host, M_ub, t32, e, s); break;
      case EPI_PATCH: launch_small<EPI_PATCH>(A, lda, W, N, K, M_dev, M_host, M_ub, t32, e, s); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  const int bi = K % 64 == 0 ? mid_blocks(e.mode, K, per_xcd(64), per_xcd(128)) : 0;
  if (bi) {
    switch (e.mode) {
      case EPI_STORE: launch_mid<EPI_STORE>(bi, A, lda, W, N, K, M_dev, M_host, M_ub, e, s); break;
      case EPI_GELU: launch_mid<EPI_GELU>(bi, A, lda, W, N, K, M_dev, M_host, M_ub, e, s); break;
      case EPI_RESID: launch_mid<EPI_RESID>(bi, A, lda, W, N, K, M_dev, M_host, M_ub, e, s); break;
      case EPI_F32: launch_mid<EPI_F32>(bi, A, lda, W, N, K, M_dev, M_host, M_ub, e, s); break;
      case EPI_PATCH: launch_mid<EPI_PATCH>(bi, A, lda, W, N, K, M_dev, M_host, M_ub, e, s); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  // tile rows: 256 (8 waves) when there are enough tiles to fill the CUs
  // several times over, 64 when 128-row tiles would leave CUs idle (only K
  // that the medium kernel does not take)
  const bool small = K % 64 != 0 && (long)((Mx + 127) / 128) * n_nt < 512;
  // (256 rows not for the GELU epilogue, whose vector work overlaps better with
  // three 4-wave workgroups per CU than with two 8-wave ones.  The direct
  // residual epilogue of 256-row tiles needs four of them a CU: 39500 x 768 x
  // 768, 930 tiles, takes 103 us in 128-row tiles and 124 in 256-row ones, 87000
  // x 384 x 384, 1020 tiles, 80 and 106.  The plain store, which both stage
  // alike, takes them where the medium kernel ends: 26700 x 1152 x 384 inside a
  // pass, 945 tiles, 36.4 and 34.0, 13800 x 2304 x 768 72.9 and 68.3)
  const bool big = e.mode != EPI_GELU &&
                   (long)((Mx + 255) / 256) * n_nt >= (e.mode == EPI_STORE ? 925 : 1024);
  const int mb = small ? 64 : big ? 256 : 128;
  const int n_mt = (M_ub + mb - 1) / mb;
  const int grid = (n_mt + NXCD - 1) / NXCD * NXCD * n_nt;
  // 32-row waves (twice the waves per tile) for 64-row tiles when the launch
  // has fewer tiles than the CUs hold at once (us, 64- / 32-row waves: 197 x
  // 1152 x 96 4.2 / 3.5, with residual 6.0 / 4.9; 3000 x 768 x 352 8.1 / 7.4;
  // from K about 1000 on they are even)
  const bool thin = small && (long)((Mx + 63) / 64) * n_nt < THIN_TILES;
#define FUSION_GEMM_LAUNCH(E)                                                                    \
  if (thin)                                                                                     \
    gemm_mfma_bf16<E, 64, 32, 1><<<grid, 256, 0, s>>>(A, lda, W, N, K, M_dev, M_host, n_mt, e); \
  else if (small)                                                                               \
    gemm_mfma_bf16<E, 64, 32, 2><<<grid, 128, 0, s>>>(A, lda, W, N, K, M_dev, M_host, n_mt, e); \
  else if (big)                                                                                 \
    gemm_mfma_bf16<E, 256, 32, 2><<<grid, 512, 0, s>>>(A, lda, W, N, K, M_dev, M_host, n_mt, e); \
  else                                                                                          \
    gemm_mfma_bf16<E, 128, 32, 2><<<grid, 256, 0, s>>>(A, lda, W, N, K, M_dev, M_host, n_mt, e)
  switch (e.mode) {
    case EPI_STORE: FUSION_GEMM_LAUNCH(EPI_STORE); break;
    case EPI_GELU: FUSION_GEMM_LAUNCH(EPI_GELU); break;
    case EPI_RESID: FUSION_GEMM_LAUNCH(EPI_RESID); break;
    case EPI_F32: FUSION_GEMM_LAUNCH(EPI_F32); break;
    case EPI_PATCH: FUSION_GEMM_LAUNCH(EPI_PATCH); break;
    default: return hipErrorInvalidValue;
  }
#undef FUSION_GEMM_LAUNCH
  return hipGetLastError();
}

}  // namespace fusion
