// C = A B^T for fp32 A (M x K) and B (N x K) on the fp16 matrix cores with fp32 accuracy to
// about 2^-22: each row of an operand is scaled by a power of two (its largest magnitude near
// 2^14) and split into two fp16 pieces, x = hi + lo with |lo| <= 2^-11 |hi| (22 significant
// bits), and
//     A B^T = Ahi Bhi^T + Ahi Blo^T + Alo Bhi^T        (+ Alo Blo^T, below 2^-22, dropped)
// is accumulated in fp32 by v_mfma_f32_32x32x16_f16.  Used for G = W H (T-update, Eq. (7): H is
// symmetric, so its rows serve as the rows of B), for F = E H of the objective (Eq. (9)) - both
// have a relative tolerance of 1e-4 downstream - and for the columns far to the right in the
// S-update.  The trailing updates of large Cholesky factorizations have a kernel of their own here
// (pair_syrk256_kernel).
//
// Both pieces of 32 columns share one 128-byte line, [hi x 32 | lo x 32], so one LDS stage (32 k,
// 256 + 256 lines) feeds all three piece products: 48 MFMAs per wavefront and stage, where reading
// the pieces as three separate products moves 1.5 times the bytes per MFMA.  The product kernel is
// the H = X X^T kernel's skeleton otherwise: 8 wavefronts of 128 x 64, tiles loaded straight into
// LDS (buffer_load ... lds) with XOR-permuted 16-byte chunks, two stages, one barrier per step;
// small tiles are 4 wavefronts of 64 x 64, two workgroups per compute unit.
// The reads of a step are spread over its MFMAs, each row of 16 lanes in banks of its own: the S-update's
// products of an 8192 x 28672 sweep 19.0 -> 18.5 ms, large tiles 35.4 -> 35.2 (power takes the rest).
// Bound by MFMA issue and power at large sizes: 8192 x 28672 x 28672 38.3 -> 32.0 ms (1.26 PFLOP/s
// issued, what a large bf16 library product reaches on the same card), 4096^3 365 -> 320 us,
// 2048^3 141 -> 66 us; making the pieces 26 + 10 -> 7 us per 2048 x 2048 operand (a row's exponent
// comes from the pass that splits it; a maximum over the whole matrix was a pass of its own).
#include "ganq_internal.h"

namespace ganq {
namespace {

constexpr int PLINE = 128;       // bytes of one row's line: 32 hi, 32 lo
constexpr int FLUSH = 8;         // steps of 32 columns that one accumulator of the small tiles sums

// One workgroup per row: the exponent that brings the row's largest finite magnitude near 2^14, and
// the row's pieces, zero for cols <= k < kp.  The second pass over the row finds it in the cache.
__global__ __launch_bounds__(256) void pair_split_kernel(const float* __restrict__ X, int64_t cols, int64_t ld,
                                                         int64_t kp, _Float16* __restrict__ dst,
                                                         int* __restrict__ ex) {
  __shared__ float red[4];
  const int64_t r = blockIdx.x;
  const int tid = threadIdx.x;
  const float* __restrict__ xr = X + r * ld;
  const bool vec = ((uintptr_t)xr & 15) == 0;
  auto load8 = [&](int64_t k, float (&v)[8]) {
    if (vec && k + 8 <= cols) {
      const float4 a = *reinterpret_cast<const float4*>(xr + k), b = *reinterpret_cast<const float4*>(xr + k + 4);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
      v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = (k + u < cols) ? xr[k + u] : 0.f;
    }
  };
  float mx = 0.f;
  for (int64_t k = 8 * tid; k < cols; k += 8 * 256) {
    float v[8];
    load8(k, v);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float a = fabsf(v[u]);
      if (a < __builtin_huge_valf() && a > mx) mx = a;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if ((tid & 63) == 0) red[tid >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  const int e = (mx > 0.f) ? 14 - ilogbf(mx) : 0;
  if (tid == 0) ex[r] = e;
  for (int64_t k = 8 * tid; k < kp; k += 8 * 256) {
    float v[8];
    load8(k, v);
    half8 hi, lo;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float s = ldexpf(v[u], e);
      hi[u] = (_Float16)s;
      lo[u] = (_Float16)(s - (float)hi[u]);
    }
    _Float16* d = dst + r * 2 * kp + (k >> 5) * 64 + (k & 31);
    *reinterpret_cast<half8*>(d) = hi;
    *reinterpret_cast<half8*>(d + 32) = lo;
  }
}

// Asks the scheduler for the reads of a step (RD of them, the first AHEAD in front) spread over its MF MFMAs.
template <int RD, int AHEAD, int MF>
__device__ inline void spread_reads() {
  __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
  for (int u = 0; u < RD - AHEAD; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, MF - (RD - AHEAD), 0);
}

// C[sp] = (sum over the three piece pairs, k steps of split sp of A_p B_p^T) scaled back
template <int TILE>
__global__ __launch_bounds__(TILE * 2, 2) void pair_gemm_kernel(const _Float16* __restrict__ A,
                                                             const _Float16* __restrict__ B, int64_t M, int64_t N,
                                                             int64_t ldp, int step0, int nsteps, int splits,
                                                             const int* __restrict__ ea,
                                                             const int* __restrict__ eb, float* __restrict__ C,
                                                             int64_t ldc, int64_t cstride) {
  constexpr int NWV = TILE / 32;             // wavefronts: 2 x 4 of 128 x 64, or 2 x 2 of 64 x 64
  constexpr int WC = TILE / 64;
  constexpr int TI = TILE / 64, TJ = 2;      // 32 x 32 MFMA tiles per wavefront
  constexpr int TILEB = TILE * PLINE, STAGEB = 2 * TILEB;
  constexpr int DPW = TILE / 8 / NWV;        // wavefront loads per operand and stage
  // Workgroups are dealt to the 8 XCDs round-robin by flat index; each XCD takes a contiguous run
  // of the item list, which walks the tiles in groups of 8 tile rows, column by column: 32
  // workgroups side by side on one XCD share 8 + 4 blocks of operand rows through its L2.
  const int tm = (int)ceil_div(M, TILE), tn = (int)ceil_div(N, TILE);
  const int64_t tiles = (int64_t)tm * tn, total = tiles * splits;
  const int64_t per = (total + 7) / 8;
  const int64_t q = blockIdx.x >> 3;
  const int64_t item = (int64_t)(blockIdx.x & 7) * per + q;
  if (q >= per || item >= total) return;
  const int sp = (int)(item / tiles);
  const int t = (int)(item % tiles);
  const int grp = t / (8 * tn), rem = t % (8 * tn);
  const int gsz = (tm - 8 * grp < 8) ? tm - 8 * grp : 8;
  // divisions are done on the vector unit; what they yield is the same in every lane
  const int bm = __builtin_amdgcn_readfirstlane(8 * grp + rem % gsz), bn = __builtin_amdgcn_readfirstlane(rem / gsz);

  extern __shared__ __attribute__((aligned(16))) unsigned char gsm[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)gsm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave / WC, wc = wave % WC;
  const int kh = lane >> 5, l32 = lane & 31;
  const int64_t m0 = (int64_t)bm * TILE, n0 = (int64_t)bn * TILE;
  const int64_t rowsA = (M - m0 < TILE) ? M - m0 : TILE;
  const int64_t rowsB = (N - n0 < TILE) ? N - n0 : TILE;

  // lane -> (row of 8, 16-byte chunk): chunk c of row r sits at position c ^ ((r >> 1) & 7), so that the 16
  // rows an LDS read serves at a time fall into different banks
  const int dr = lane >> 3, dc = (lane & 7) ^ (((wave & 1) << 2) | (dr >> 1));
  uint32_t voff[DPW];
#pragma unroll
  for (int j = 0; j < DPW; ++j) voff[j] = (uint32_t)(((int64_t)((wave + NWV * j) * 8 + dr) * ldp + dc * 8) * 2);
  const int4v rsA = make_rsrc(A + m0 * ldp, rowsA * ldp * 2);
  const int4v rsB = make_rsrc(B + n0 * ldp, rowsB * ldp * 2);
  const int sb = step0 + __builtin_amdgcn_readfirstlane((int)((int64_t)nsteps * sp / splits));
  const int se = step0 + __builtin_amdgcn_readfirstlane((int)((int64_t)nsteps * (sp + 1) / splits));
  auto issue = [&](int s, int st) {
    const uint32_t soff = (uint32_t)(s * PLINE);
    const uint32_t sbase = lds0 + st * STAGEB;
#pragma unroll
    for (int j = 0; j < DPW; ++j) {
      load16_to_lds(rsA, sbase + (wave + NWV * j) * 1024, voff[j], soff);
      load16_to_lds(rsB, sbase + TILEB + (wave + NWV * j) * 1024, voff[j], soff);
    }
  };

  // The small tiles have registers for two more sets of accumulators.  The cross products, 2^-11 of the
  // others, round among themselves, and every FLUSH steps the main sum moves to a total of its own: the
  // rounding of an fp32 accumulator grows with the length and the size of what it has summed.
  constexpr bool TWO = TILE == 128;
  floatx16 acc[TI][TJ], crs[TWO ? TI : 1][TWO ? TJ : 1], tot[TWO ? TI : 1][TWO ? TJ : 1];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        acc[i][j][v] = 0.f;
        if constexpr (TWO) crs[i][j][v] = tot[i][j][v] = 0.f;
      }

  const int rswz = (l32 >> 1) & 7;
  if (sb < se) issue(sb, 0);
  int st = 0;
#pragma unroll 1
  for (int s = sb; s < se; ++s) {
    wait_all_loads();
    __syncthreads();
    if (s + 1 < se) issue(s + 1, st ^ 1);
    if constexpr (TWO) {
      if (s > sb && (s - sb) % FLUSH == 0) {
#pragma unroll
        for (int i = 0; i < TI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              tot[i][j][v] += acc[i][j][v];
              acc[i][j][v] = 0.f;
            }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char* Asm = gsm + st * STAGEB + (wr * (TILE / 2) + l32) * PLINE;
    const unsigned char* Bsm = gsm + st * STAGEB + TILEB + (wc * 64 + l32) * PLINE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      half8 ah[TI], al[TI], bh[TJ], bl[TJ];
      const int ph = ((2 * ks + kh) ^ rswz) * 16, pl = ((4 + 2 * ks + kh) ^ rswz) * 16;
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        ah[i] = *reinterpret_cast<const half8*>(Asm + i * 32 * PLINE + ph);
        al[i] = *reinterpret_cast<const half8*>(Asm + i * 32 * PLINE + pl);
      }
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        bh[j] = *reinterpret_cast<const half8*>(Bsm + j * 32 * PLINE + ph);
        bl[j] = *reinterpret_cast<const half8*>(Bsm + j * 32 * PLINE + pl);
      }
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[i], bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          floatx16& a = TWO ? crs[TWO ? i : 0][TWO ? j : 0] : acc[i][j];
          a = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[i], bh[j], a, 0, 0, 0);
        }
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          floatx16& a = TWO ? crs[TWO ? i : 0][TWO ? j : 0] : acc[i][j];
          a = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[i], bl[j], a, 0, 0, 0);
        }
    }
    spread_reads<4 * (TI + TJ), TI + TJ, 6 * TI * TJ>();
    __builtin_amdgcn_sched_barrier(0);
    st ^= 1;
  }

  float* __restrict__ Cs = C + sp * cstride;
  int ebj[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int64_t col = n0 + wc * 64 + j * 32 + l32;
    ebj[j] = (col < N) ? eb[col] : 0;
  }
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int64_t row = m0 + wr * (TILE / 2) + i * 32 + (v >> 2) * 8 + kh * 4 + (v & 3);
      if (row >= M) continue;
      const int e = ea[row];
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const int64_t col = n0 + wc * 64 + j * 32 + l32;
        float r = acc[i][j][v];
        if constexpr (TWO) r = tot[i][j][v] + (r + crs[i][j][v]);
        if (col < N) Cs[row * ldc + col] = ldexpf(r, -(e + ebj[j]));
      }
    }
}

// ---- C(lower) -= A A^T for A of exactly 256 columns: the trailing update of the blocked Cholesky ----

// One wavefront per row of 256 columns: its exponent and its pieces (rows of 512 halves).
__global__ __launch_bounds__(256) void pair_split256_kernel(const float* __restrict__ X, int64_t rows, int64_t ld,
                                                            _Float16* __restrict__ dst, int* __restrict__ ex) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const float4 q = *reinterpret_cast<const float4*>(X + r * ld + 4 * lane);
  const float v[4] = {q.x, q.y, q.z, q.w};
  float mx = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float a = fabsf(v[u]);
    if (a < __builtin_huge_valf() && a > mx) mx = a;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  const int e = (mx > 0.f) ? 14 - ilogbf(mx) : 0;
  if (lane == 0) ex[r] = e;
  half4 hi, lo;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const float s = ldexpf(v[u], e);
    hi[u] = (_Float16)s;
    lo[u] = (_Float16)(s - (float)hi[u]);
  }
  _Float16* d = dst + r * 512 + (lane >> 3) * 64 + (lane & 7) * 4;
  *reinterpret_cast<half4*>(d) = hi;
  *reinterpret_cast<half4*>(d + 32) = lo;
}

// 128 x 128 tiles on or below the diagonal, 4 wavefronts of 64 x 64, all 256 columns in eight steps
// through two LDS stages, two workgroups per compute unit.  The cross products have accumulators of
// their own.  The product of the low pieces is dropped except in the diagonal tiles: there it is a sum of
// squares, 1.5e-8 of H_jj that every pivot would keep (where the pivots shrink to 1 / 17 of H_jj their
// relative error was 1.6 times that of the fp32 update; with it, and in |L L^T - H| anyway, the errors are
// level or lower).  Bound by C: 128 KB of it move per tile against 2.6 us of MFMA.  Factorization on
// its own, fp32 matrix units before:
// n = 28672 94.6 -> 57.0 ms, 11008 10.0 -> 7.9 ms, 8192 5.85 -> 5.1 ms.
__global__ __launch_bounds__(256, 2) void pair_syrk256_kernel(const _Float16* __restrict__ A, int64_t M,
                                                              const int* __restrict__ ea, float* __restrict__ C,
                                                              int64_t ldc) {
  constexpr int TILE = 128, TILEB = TILE * PLINE, STAGEB = 2 * TILEB, STEPS = 8, LDP = 512;
  // flat index -> tile (bm, bn) of the lower triangle, row by row
  const int64_t t = blockIdx.x;
  int bm = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while ((int64_t)bm * (bm + 1) / 2 > t) --bm;
  while ((int64_t)(bm + 1) * (bm + 2) / 2 <= t) ++bm;
  bm = __builtin_amdgcn_readfirstlane(bm);       // found on the vector unit, the same in every lane
  const int bn = __builtin_amdgcn_readfirstlane((int)(t - (int64_t)bm * (bm + 1) / 2));

  extern __shared__ __attribute__((aligned(16))) unsigned char gsm[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)gsm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave >> 1, wc = wave & 1;
  const int kh = lane >> 5, l32 = lane & 31;
  const int64_t m0 = (int64_t)bm * TILE, n0 = (int64_t)bn * TILE;
  const int64_t rowsA = (M - m0 < TILE) ? M - m0 : TILE, rowsB = (M - n0 < TILE) ? M - n0 : TILE;
  const int dr = lane >> 3, dc = (lane & 7) ^ (((wave & 1) << 2) | (dr >> 1));
  uint32_t voff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) voff[j] = (uint32_t)((((wave + 4 * j) * 8 + dr) * LDP + dc * 8) * 2);
  const int4v rsA = make_rsrc(A + m0 * LDP, rowsA * LDP * 2);
  const int4v rsB = make_rsrc(A + n0 * LDP, rowsB * LDP * 2);
  auto issue = [&](int s, int st) {
    const uint32_t soff = (uint32_t)(s * PLINE), sbase = lds0 + st * STAGEB;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      load16_to_lds(rsA, sbase + (wave + 4 * j) * 1024, voff[j], soff);
      load16_to_lds(rsB, sbase + TILEB + (wave + 4 * j) * 1024, voff[j], soff);
    }
  };
  issue(0, 0);
  floatx16 acc[2][2], crs[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = crs[i][j][v] = 0.f;
  const int rswz = (l32 >> 1) & 7;
#pragma unroll 1
  for (int s = 0; s < STEPS; ++s) {
    wait_all_loads();
    __syncthreads();
    if (s + 1 < STEPS) issue(s + 1, (s + 1) & 1);
    const unsigned char* Asm = gsm + (s & 1) * STAGEB + (wr * 64 + l32) * PLINE;
    const unsigned char* Bsm = gsm + (s & 1) * STAGEB + TILEB + (wc * 64 + l32) * PLINE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int ph = ((2 * ks + kh) ^ rswz) * 16, pl = ((4 + 2 * ks + kh) ^ rswz) * 16;
      half8 ah[2], al[2], bh[2], bl[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        ah[i] = *reinterpret_cast<const half8*>(Asm + i * 32 * PLINE + ph);
        al[i] = *reinterpret_cast<const half8*>(Asm + i * 32 * PLINE + pl);
        bh[i] = *reinterpret_cast<const half8*>(Bsm + i * 32 * PLINE + ph);
        bl[i] = *reinterpret_cast<const half8*>(Bsm + i * 32 * PLINE + pl);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[i], bh[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) crs[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[i], bh[j], crs[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) crs[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[i], bl[j], crs[i][j], 0, 0, 0);
      if (bm == bn) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) crs[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[i], bl[j], crs[i][j], 0, 0, 0);
      }
    }
  }
  const bool full = (m0 + TILE <= M) && (bn < bm);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t row = m0 + wr * 64 + i * 32 + kh * 4, col = n0 + wc * 64 + j * 32 + l32;
      float* __restrict__ cp = C + row * ldc + col;
      if (full) {
        const int ec = ea[col];
        float cin[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) cin[v] = cp[((v >> 2) * 8 + (v & 3)) * ldc];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int dv = (v >> 2) * 8 + (v & 3);
          cp[dv * ldc] = cin[v] - ldexpf(acc[i][j][v] + crs[i][j][v], -(ea[row + dv] + ec));
        }
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int dv = (v >> 2) * 8 + (v & 3);
          if (row + dv < M && col <= row + dv)
            cp[dv * ldc] -= ldexpf(acc[i][j][v] + crs[i][j][v], -(ea[row + dv] + ea[col]));
        }
      }
    }
}

}  // namespace

// kp = pair_columns(K): columns rounded up to whole lines.  A piece matrix holds rows x 2 kp halves:
// the pieces of X[r][k] sit at [r][(k / 32) * 64 + k % 32] (hi) and 32 further on (lo), scaled by 2^ex[r].
hipError_t launch_pair_split(hipStream_t s, const float* X, int64_t rows, int64_t cols, int64_t ld,
                             _Float16* dst, int* ex) {
  hipLaunchKernelGGL(pair_split_kernel, dim3((unsigned)rows), dim3(256), 0, s, X, cols, ld, pair_columns(cols), dst, ex);
  return hipGetLastError();
}

// C + sp * cstride (sp < splits) = the share of split sp of the sum over the 32-column steps
// [step0, step1) of A B^T, both given as piece matrices with rows of 2 kp halves.
// small_tiles: 128 x 128 tiles, whose sums are the more accurate ones (FLUSH); the S-update asks for them.
// Mean error of its targets in units of 2^-24 of their size, with sums of everything to the right in
// the fp32 matrix units / with large tiles (m = 8192) / now: 5000 columns 5.5 / 6.3 / 1.7, with the
// dominant features on the left 2.7 / 8.1 / 2.0; 27648 columns 11.6 / 10.7 / 2.1.  It costs 2.4 of the
// 22.4 ms of an 8192 x 28672 sweep.  Otherwise 256 x 256 tiles where there are at least 192 of them, 128 x
// 128 tiles below (G = W H with its pieces, large / small tiles: 64 large tiles, 2048 x 2048, 141 / 66 us;
// 128, 2048 x 4096, 310 / 246; 144, 3072 x 3072, 226 / 246; 169, 252 / 282; 192, 4096 x 3072, 247 / 268; 256,
// 4096 x 4096, 396 / 451).  Time alone would put the line near 140; between there and 192 the small
// tiles' accuracy costs up to a tenth.
hipError_t launch_pair_gemm(hipStream_t s, const _Float16* A, const _Float16* B, int64_t M, int64_t N, int64_t kp,
                            int step0, int step1, int splits, const int* ea, const int* eb, float* C, int64_t ldc,
                            int64_t cstride, bool small_tiles) {
  hipError_t e;
  if (!small_tiles && ceil_div(M, 256) * ceil_div(N, 256) * splits >= 192) {
    constexpr int lds = 4 * 256 * PLINE;
    static std::atomic<uint64_t> lds_set{0};
    if ((e = ensure_dynamic_lds((const void*)pair_gemm_kernel<256>, lds, lds_set)) != hipSuccess) return e;
    const int64_t total = ceil_div(M, 256) * ceil_div(N, 256) * splits;
    hipLaunchKernelGGL(pair_gemm_kernel<256>, dim3((unsigned)(8 * ceil_div(total, 8))), dim3(512), lds, s, A, B, M,
                       N, 2 * kp, step0, step1 - step0, splits, ea, eb, C, ldc, cstride);
  } else {
    constexpr int lds = 4 * 128 * PLINE;
    static std::atomic<uint64_t> lds_set{0};
    if ((e = ensure_dynamic_lds((const void*)pair_gemm_kernel<128>, lds, lds_set)) != hipSuccess) return e;
    const int64_t total = ceil_div(M, 128) * ceil_div(N, 128) * splits;
    hipLaunchKernelGGL(pair_gemm_kernel<128>, dim3((unsigned)(8 * ceil_div(total, 8))), dim3(256), lds, s, A, B, M,
                       N, 2 * kp, step0, step1 - step0, splits, ea, eb, C, ldc, cstride);
  }
  return hipGetLastError();
}

size_t pair_bytes(int64_t rows, int64_t cols) { return align_up((size_t)rows * 2 * pair_columns(cols) * sizeof(_Float16)); }

size_t gemm_split_scratch_bytes(int64_t M, int64_t N, int64_t K) {
  return align_up((size_t)M * sizeof(int)) + align_up((size_t)N * sizeof(int)) + pair_bytes(M, K) + pair_bytes(N, K);
}

// C (M x N) = A (M x K) * B (N x K)^T.  scratch: [exponents of A's rows][of B's][A pieces][B pieces].
hipError_t launch_gemm_split(hipStream_t s, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                             const float* B, int64_t ldb, float* C, int64_t ldc, void* scratch) {
  char* p = (char*)scratch;
  int* ea = (int*)p;
  int* eb = (int*)(p += align_up((size_t)M * sizeof(int)));
  _Float16* As = (_Float16*)(p += align_up((size_t)N * sizeof(int)));
  _Float16* Bs = (_Float16*)(p + pair_bytes(M, K));
  hipError_t e;
  if ((e = launch_pair_split(s, A, M, K, lda, As, ea)) != hipSuccess) return e;
  if ((e = launch_pair_split(s, B, N, K, ldb, Bs, eb)) != hipSuccess) return e;
  const int64_t kp = pair_columns(K);
  return launch_pair_gemm(s, As, Bs, M, N, kp, 0, (int)(kp / 32), 1, ea, eb, C, ldc, 0, false);
}

size_t pair_syrk256_scratch_bytes(int64_t M) {
  return align_up((size_t)M * 512 * sizeof(_Float16)) + align_up((size_t)M * sizeof(int));
}

// C (M x M, lower triangle) -= A A^T with A of M x 256; needs lda % 4 == 0 and a 16-byte aligned A.
hipError_t launch_pair_syrk256(hipStream_t s, int64_t M, const float* A, int64_t lda, float* C, int64_t ldc,
                               void* scratch) {
  if (M <= 0) return hipSuccess;
  if ((lda % 4) != 0 || (((uintptr_t)A) % 16) != 0) return hipErrorInvalidValue;
  _Float16* Ap = (_Float16*)scratch;
  int* ex = (int*)((char*)scratch + align_up((size_t)M * 512 * sizeof(_Float16)));
  constexpr int lds = 4 * 128 * PLINE;
  static std::atomic<uint64_t> lds_set{0};
  hipError_t e = ensure_dynamic_lds((const void*)pair_syrk256_kernel, lds, lds_set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pair_split256_kernel, dim3((unsigned)ceil_div(M, 4)), dim3(256), 0, s, A, M, lda, Ap, ex);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t nt = ceil_div(M, 128);
  hipLaunchKernelGGL(pair_syrk256_kernel, dim3((unsigned)(nt * (nt + 1) / 2)), dim3(256), lds, s, Ap, M, ex, C, ldc);
  return hipGetLastError();
}

}  // namespace ganq
