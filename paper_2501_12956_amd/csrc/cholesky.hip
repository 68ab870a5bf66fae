// L = Cholesky(H) or of its preconditioned form (Eq. (10), Remark 3.1,
// Appendix A Eq. (23)-(24)), blocked, fp32 storage.
//
// The lower triangle of H (plus the preconditioner) is copied to a working matrix W; L is
// written once and never read back as input of the same kernel that writes it.  Columns go
// in outer panels of 256, each of four inner blocks of 64:
//   inner block (one launch): every workgroup owns 64 rows below the diagonal block and
//     repeats the small shared part itself - it brings the 64 x 64 diagonal block up to date
//     with the earlier inner blocks of the panel (left-looking, from L), factors it and
//     inverts the factor in LDS - then updates its own rows the same way and multiplies
//     them by that inverse.  No second launch and no grid-wide dependency for the solve.  The
//     serial chain of the four 16 x 16 leaves bounds it; the other wavefronts work beside it.
//   outer panel: W22 -= L21 L21^T with K = 256, on the fp32 matrix cores or, for large remainders,
//     as split products on the fp16 ones.
#include "ganq_internal.h"

namespace ganq {
namespace {

constexpr int NB = 64;

__global__ void fill_i32_kernel(int* p, int v) { *p = v; }

// W <- lower triangle of H (+ preconditioner on the diagonal), L <- 0.
// delta (if used) must already hold the diagonal offsets.
// thr[i] = pivot threshold of column i: tau times the diagonal entry that is factorised.
// One thread takes four consecutive columns (16-byte loads and stores where VEC says that rows of
// H, W and L allow them).  Entries of W right of the diagonal inside the group that holds the
// diagonal are written as 0; the rest of the upper triangle of W is never read.
template <bool VEC>
__global__ __launch_bounds__(256) void copy_lower_kernel(const float* __restrict__ H, int64_t n,
                                                         int64_t ldh, float* __restrict__ W,
                                                         float* __restrict__ L, int64_t ldl,
                                                         int precond, float lambda,
                                                         const float* __restrict__ delta, float tau,
                                                         float* __restrict__ thr) {
  const int64_t j0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  const int64_t i = blockIdx.y;
  if (j0 >= n) return;
  const int cnt = (int)((n - j0 < 4) ? n - j0 : 4);
  if (VEC) {
    *reinterpret_cast<float4*>(L + i * ldl + j0) = float4{0.f, 0.f, 0.f, 0.f};
  } else {
    for (int t = 0; t < cnt; ++t) L[i * ldl + j0 + t] = 0.f;
  }
  if (j0 > i) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    const float4 h = *reinterpret_cast<const float4*>(H + i * ldh + j0);
    v[0] = h.x; v[1] = h.y; v[2] = h.z; v[3] = h.w;
  } else {
    for (int t = 0; t < cnt; ++t) v[t] = H[i * ldh + j0 + t];
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int64_t j = j0 + t;
    if (j > i) v[t] = 0.f;
    if (j == i) {
      if (precond == GANQ_PRECOND_LAMBDA) v[t] += lambda;
      if (precond == GANQ_PRECOND_DIAGDOM) v[t] += delta[i];
      // a diagonal that is not positive and finite fails at once (threshold +inf: no pivot passes)
      thr[i] = (v[t] > 0.f && v[t] < 3.0e38f) ? tau * v[t] : __builtin_huge_valf();
    }
  }
  if (VEC) {
    *reinterpret_cast<float4*>(W + i * n + j0) = float4{v[0], v[1], v[2], v[3]};
  } else {
    for (int t = 0; t < cnt; ++t)
      if (j0 + t <= i) W[i * n + j0 + t] = v[t];
  }
}

// delta_i = max(sum_j |H_ij| - 2 H_ii, 1e-8), Appendix A Eq. (23); one workgroup per row.
__global__ __launch_bounds__(256) void diagdom_delta_kernel(const float* __restrict__ H, int64_t n,
                                                            int64_t ldh, float* __restrict__ delta) {
  const int64_t i = blockIdx.x;
  double s = 0.0;
  for (int64_t j = threadIdx.x; j < n; j += 256) s += fabs((double)H[i * ldh + j]);
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double d = red[0] - 2.0 * (double)H[i * ldh + i];
    delta[i] = (float)(d > 1e-8 ? d : 1e-8);
  }
}

// ---- 64 x 64 diagonal block: factor and inverse of the factor, one workgroup ----
//
// The block lives in LDS and is processed as 4 x 4 leaves of 16 x 16.  What takes time is the chain of 64
// dependent columns, so everything else runs beside it.  Per leaf column kb:
// P (wavefront 0) the 16 x 16 diagonal leaf is factored and the leaves under it are solved at the same time:
//     every row of 16 lanes holds the leaf's rows, and each of the first three the rows of one leaf below,
//     columns in registers; pivots and multipliers travel by DPP row broadcasts, no LDS round trip and no
//     barrier inside the 16 steps.  The other wavefronts finish the trailing update of the column before
//     and the inverse as far as it is known.
// Q the leaves of the next column are brought up to date, one per wavefront; the leaf just factored is
//     inverted by forward substitution (one column per lane) as soon as a wavefront is free.
// Only the last leaf's inverse and the last row of the block inverse remain at the end.  Two barriers per leaf
// column instead of one per matrix column.  On a bad pivot the 1-based global index of
// the first one is recorded in *info (if still 0) and the pivot is replaced by 1 so that
// the kernel terminates normally.
constexpr int BLD = NB + 1;    // LDS row stride (floats)

// value of lane LANE of the same row of 16 lanes (DPP row broadcast, folds into the consumer)
template <int LANE>
__device__ inline float row_bcast(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + LANE,
                                                                0xf, 0xf, true));
}

// acc += bcast * y, where bcast is x of lane LANE of the same row of 16 lanes: one VOP2 DPP
// instruction.  The caller separates the write of x from the first such read by two wait
// states (dpp_wait), which the compiler does not do for inline assembly.
template <int LANE>
__device__ inline void fmac_row_bcast(float& acc, float x, float y) {
  asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
               : "+v"(acc) : "v"(x), "v"(y), "n"(LANE));
}
// two wait states between the (earlier) write of v and its (later) DPP reads
__device__ inline void dpp_wait(float& v) { asm volatile("s_nop 1" : "+v"(v)); }

// Columns C .. 15 of step K: a[C] -= L[C][K] L[r][K] in the leaf, b[C] -= L[C][K] P[r][K] below it.
template <int K, int C, bool PANEL>
struct LeafCols {
  static __device__ inline void update(float (&a)[16], float (&b)[16], float lk, float nlk, float nlb) {
    fmac_row_bcast<C>(a[C], lk, nlk);
    if constexpr (PANEL) fmac_row_bcast<C>(b[C], lk, nlb);
    LeafCols<K, C + 1, PANEL>::update(a, b, lk, nlk, nlb);
  }
};
template <int K, bool PANEL>
struct LeafCols<K, 16, PANEL> {
  static __device__ inline void update(float (&)[16], float (&)[16], float, float, float) {}
};

// Step K takes its pivot from the step before, which broadcasts it as soon as that one column is done and
// has its other columns still to do: the next reciprocal root is computed under them.
template <int K, bool PANEL>
struct LeafSteps {
  // branch-free: a bad pivot (not positive, or not finite) is replaced by 1 and the first
  // such column of the leaf is remembered in badk
  static __device__ inline void run(float (&a)[16], float (&b)[16], float (&rsv)[16], int r, int& badk, float thr,
                                    float piv) {
    const bool bad = !(piv > row_bcast<K>(thr)) || !(piv < 3.0e38f);
    badk = (bad && badk == 16) ? K : badk;
    piv = bad ? 1.f : piv;
    const float rs = __builtin_amdgcn_rsqf(piv);      // 1 ulp
    rsv[K] = rs;
    const float akk = (bad && r == K) ? 1.f : a[K];
    float lk = (r >= K) ? akk * rs : 0.f;             // L[r][K]; row K gets piv * rs = sqrt(piv)
    a[K] = lk;
    const float nlk = -lk;
    float nlb = 0.f;
    if constexpr (PANEL) {
      b[K] *= rs;
      nlb = -b[K];
    }
    dpp_wait(lk);
    if constexpr (K < 15) {
      fmac_row_bcast<K + 1>(a[K + 1], lk, nlk);
      dpp_wait(a[K + 1]);
      const float next = row_bcast<K + 1>(a[K + 1]);
      if constexpr (PANEL) fmac_row_bcast<K + 1>(b[K + 1], lk, nlb);
      LeafCols<K, K + 2, PANEL>::update(a, b, lk, nlk, nlb);
      LeafSteps<K + 1, PANEL>::run(a, b, rsv, r, badk, thr, next);
    }
  }
};

// Forward substitution L x = e_j with one column j per lane: once x[K] is known every later
// row's running sum takes its term, s[RR] -= L[RR][K] x[K] (independent instructions).
template <int K, int RR>
struct LeafInvRows {
  static __device__ inline void update(const float (&a)[16], float (&sv)[16], float nx) {
    fmac_row_bcast<RR>(sv[RR], a[K], nx);            // a[K] of lane RR is L[RR][K]
    LeafInvRows<K, RR + 1>::update(a, sv, nx);
  }
};
template <int K>
struct LeafInvRows<K, 16> {
  static __device__ inline void update(const float (&)[16], float (&)[16], float) {}
};
template <int K>
struct LeafInv {
  static __device__ inline void run(const float (&a)[16], const float (&rsv)[16], float (&sv)[16]) {
    sv[K] *= rsv[K];                                 // x[K]
    const float nx = -sv[K];
    LeafInvRows<K, K + 1>::update(a, sv, nx);
    LeafInv<K + 1>::run(a, rsv, sv);
  }
};
template <>
struct LeafInv<16> {
  static __device__ inline void run(const float (&)[16], const float (&)[16], float (&)[16]) {}
};

// One wavefront: factors the leaf at rows o .. o+15 of M and solves the `below` leaves under it.  Lane l holds
// matrix row l % 16 of the leaf and of leaf l / 16 below, 16 columns in registers.
__device__ inline void factor_leaf(float (*M)[BLD], float (*Inv)[BLD], int o, int below, int nb, int64_t k0,
                                   int* __restrict__ info, const float* __restrict__ thr) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  float a[16], b[16], rsv[16];
  const bool has = g < below;
  const int pr = has ? o + 16 + 16 * g + r : o + r;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    a[c] = M[o + r][o + c];
    b[c] = M[pr][o + c];
  }
  // lane r holds the threshold of the leaf's column r (0 for the identity padding beyond nb)
  float th = (o + r < nb) ? thr[k0 + o + r] : 0.f;
  dpp_wait(th);
  int badk = 16;
  dpp_wait(a[0]);
  const float piv = row_bcast<0>(a[0]);
  if (below > 0)
    LeafSteps<0, true>::run(a, b, rsv, r, badk, th, piv);
  else
    LeafSteps<0, false>::run(a, b, rsv, r, badk, th, piv);
  if (badk < 16 && lane == 0 && o + badk < nb) atomicCAS(info, 0, (int)(k0 + o + badk + 1));
  if (lane < 16) {
#pragma unroll
    for (int c = 0; c < 16; ++c) M[o + r][o + c] = a[c];
  }
  if (has) {
#pragma unroll
    for (int c = 0; c < 16; ++c) M[pr][o + c] = b[c];
  }
  if (below == 0) {
    // the last leaf's inverse follows at once: lane j solves L x = e_j
    float x[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) x[c] = (c == r) ? 1.f : 0.f;
    LeafInv<0>::run(a, rsv, x);
    if (lane < 16) {
#pragma unroll
      for (int c = 0; c < 16; ++c) Inv[o + c][o + r] = x[c];
    }
  }
}

// One wavefront: the inverse of the factored leaf at rows o .. o+15 of M.
__device__ inline void invert_leaf(const float (*M)[BLD], float (*Inv)[BLD], int o) {
  const int lane = threadIdx.x & 63, r = lane & 15;
  float a[16], x[16], rsv[16];
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    a[c] = M[o + r][o + c];
    rsv[c] = __builtin_amdgcn_rcpf(M[o + c][o + c]);      // 1 ulp
    x[c] = (c == r) ? 1.f : 0.f;
  }
#pragma unroll
  for (int c = 0; c < 16; ++c) dpp_wait(a[c]);
  LeafInv<0>::run(a, rsv, x);
  if (lane < 16) {
#pragma unroll
    for (int c = 0; c < 16; ++c) Inv[o + c][o + r] = x[c];
  }
}

// Leaf products on the matrix cores, one wavefront each (v_mfma_f32_16x16x4_f32: lane l supplies
// A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[4 (l / 16) + r][l % 16], r = 0..3).
// d += sign * A B^T: rows ra of A, rows rb of B, columns k of both
__device__ inline void leaf_abt(floatx4& d, const float (*A)[BLD], int ra, const float (*B)[BLD], int rb, int k, float sign) {
  const int lm = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int kk = 0; kk < 16; kk += 4)
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(sign * A[ra + lm][k + kk + lk], B[rb + lm][k + kk + lk], d, 0, 0, 0);
}
// d += sign * A B: rows ra and columns ka of A, rows kb and columns cb of B
__device__ inline void leaf_ab(floatx4& d, const float (*A)[BLD], int ra, int ka, const float (*B)[BLD], int kb, int cb, float sign) {
  const int lm = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int kk = 0; kk < 16; kk += 4)
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(sign * A[ra + lm][ka + kk + lk], B[kb + kk + lk][cb + lm], d, 0, 0, 0);
}
__device__ inline floatx4 leaf_load(const float (*X)[BLD], int r0, int c0) {
  const int lm = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
  return floatx4{X[r0 + 4 * lk][c0 + lm], X[r0 + 4 * lk + 1][c0 + lm], X[r0 + 4 * lk + 2][c0 + lm], X[r0 + 4 * lk + 3][c0 + lm]};
}
__device__ inline void leaf_store(float (*X)[BLD], int r0, int c0, const floatx4& d) {
  const int lm = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) X[r0 + 4 * lk + r][c0 + lm] = d[r];
}
// M(i, j) -= M(i, k) M(j, k)^T in leaves
__device__ inline void leaf_update(float (*M)[BLD], int i, int j, int k) {
  floatx4 d = leaf_load(M, 16 * i, 16 * j);
  leaf_abt(d, M, 16 * i, M, 16 * j, 16 * k, -1.f);
  leaf_store(M, 16 * i, 16 * j, d);
}
// Inv(i, j) = -Inv(i, i) sum_{j <= k < i} L(i, k) Inv(k, j); the sum goes through Tmp(i, j), where the same
// wavefront reads it back, as it may read Inv(i, j) for a leaf further down
__device__ inline void leaf_inverse(const float (*M)[BLD], float (*Inv)[BLD], float (*Tmp)[BLD], int i, int j) {
  floatx4 t = {0.f, 0.f, 0.f, 0.f};
  for (int k = j; k < i; ++k) leaf_ab(t, M, 16 * i, 16 * k, Inv, 16 * k, 16 * j, 1.f);
  leaf_store(Tmp, 16 * i, 16 * j, t);
  lds_handover();
  floatx4 x = {0.f, 0.f, 0.f, 0.f};
  leaf_ab(x, Inv, 16 * i, 16 * i, Tmp, 16 * i, 16 * j, -1.f);
  leaf_store(Inv, 16 * i, 16 * j, x);
  lds_handover();
}

// M: the block (lower triangle meaningful on entry, identity beyond nb); on exit its lower
// triangle is the factor (strict upper part of the leaves zero) and Inv its inverse (leaves on and below the diagonal).
// Tmp is scratch.  Called by all wavefronts of the workgroup: 0 to 3 do this work, the others call
// other(0) .. other(3) between the barriers, beside the four leaves.  Ends with a barrier.
template <typename F>
__device__ inline void factor_block(float (*M)[BLD], float (*Inv)[BLD], float (*Tmp)[BLD], int nb,
                                    int64_t k0, int* __restrict__ info, const float* __restrict__ thr, const F& other) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // P0
  if (wave == 0) factor_leaf(M, Inv, 0, 3, nb, k0, info, thr);
  if (wave >= 4) other(0);
  __syncthreads();
  // Q0
  if (wave < 3) leaf_update(M, wave + 1, 1, 0);
  __syncthreads();
  // P1
  if (wave == 0) factor_leaf(M, Inv, 16, 2, nb, k0, info, thr);
  if (wave == 1) leaf_update(M, 2, 2, 0);
  if (wave == 2) leaf_update(M, 3, 2, 0);
  if (wave == 3) {
    leaf_update(M, 3, 3, 0);
    invert_leaf(M, Inv, 0);
  }
  if (wave >= 4) other(1);
  __syncthreads();
  // Q1
  if (wave < 2) leaf_update(M, wave + 2, 2, 1);
  if (wave == 2) leaf_update(M, 3, 3, 1);
  __syncthreads();
  // P2
  if (wave == 0) factor_leaf(M, Inv, 32, 1, nb, k0, info, thr);
  if (wave == 3) invert_leaf(M, Inv, 16);
  if (wave >= 4) other(2);
  __syncthreads();
  // Q2
  if (wave == 0) leaf_update(M, 3, 3, 2);
  if (wave == 3) invert_leaf(M, Inv, 32);
  __syncthreads();
  // P3; the sums of the last row of the inverse wait in Tmp for the last leaf
  if (wave == 0) factor_leaf(M, Inv, 48, 0, nb, k0, info, thr);
  if (wave == 1) leaf_inverse(M, Inv, Tmp, 1, 0);
  if (wave == 1 || wave == 2) leaf_inverse(M, Inv, Tmp, 2, wave - 1);
  if (wave >= 1 && wave < 4) {
    const int j = wave - 1;
    floatx4 t = {0.f, 0.f, 0.f, 0.f};
    for (int k = j; k < 3; ++k) leaf_ab(t, M, 48, 16 * k, Inv, 16 * k, 16 * j, 1.f);
    leaf_store(Tmp, 48, 16 * j, t);
  }
  if (wave >= 4) other(3);
  __syncthreads();
  if (wave >= 1 && wave < 4) {
    const int j = wave - 1;
    floatx4 x = {0.f, 0.f, 0.f, 0.f};
    leaf_ab(x, Inv, 48, 48, Tmp, 48, 16 * j, -1.f);
    leaf_store(Inv, 48, 16 * j, x);
  }
  __syncthreads();
}

constexpr int PLD = 3 * NB + 1;   // LDS stride of the diagonal rows' earlier columns

// Inner block at columns c0 .. c0 + nb of the outer panel that starts at column J.
// Workgroup w owns rows c0 + 64 + 64 w .. (if any); workgroup 0 also stores the diagonal block.
// Eight wavefronts.  While 0 to 3 factor the diagonal block, 5 to 7 bring the workgroup's own rows up to date;
// 4 shares its SIMD with wavefront 0, whose dependent steps fp32 MFMAs would hold up, and only waits.  With
// four wavefronts doing all of it in turn a launch took 24.5 us on average (n = 2048), now 18.9.
// vec: rows of L start on 16 bytes.
constexpr int PTH = 512;
__global__ __launch_bounds__(PTH) void chol_panel_kernel(const float* __restrict__ W, float* __restrict__ L,
                                                         int64_t ldl, int64_t n, int64_t J, int64_t c0,
                                                         int nb, int vec, int* __restrict__ info,
                                                         const float* __restrict__ thr) {
  extern __shared__ __attribute__((aligned(16))) float psm[];
  float (*M)[BLD] = reinterpret_cast<float (*)[BLD]>(psm);
  float (*Inv)[BLD] = reinterpret_cast<float (*)[BLD]>(psm + NB * BLD);
  float (*Tmp)[BLD] = reinterpret_cast<float (*)[BLD]>(psm + 2 * NB * BLD);
  float (*X)[BLD] = reinterpret_cast<float (*)[BLD]>(psm + 3 * NB * BLD);
  float (*Pd)[PLD] = reinterpret_cast<float (*)[PLD]>(psm + 4 * NB * BLD);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lm = lane & 15, lk = lane >> 4;
  const int Kp = (int)(c0 - J);               // columns of this panel already factored: 0, 64, 128, 192
  const int64_t r0 = c0 + NB + (int64_t)blockIdx.x * NB;
  const bool own = r0 < n;

  // raw diagonal block (identity beyond nb, strict upper part zero) and the diagonal rows'
  // earlier columns of L; all loads are issued before the first use
  {
    float ld[8], pd[3][8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = tid + PTH * u, rr = e >> 6, cc = e & 63;
      const bool in = rr < nb && cc <= rr;
      const float v = W[(c0 + (in ? rr : 0)) * n + c0 + (in ? cc : 0)];
      ld[u] = in ? v : ((rr == cc) ? 1.f : 0.f);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q * NB < Kp) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int e = tid + PTH * u, rr = e >> 6, cc = e & 63;
          const float v = L[(c0 + (rr < nb ? rr : 0)) * ldl + J + q * NB + cc];
          pd[q][u] = rr < nb ? v : 0.f;
        }
      }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = tid + PTH * u;
      M[e >> 6][e & 63] = ld[u];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (q * NB < Kp) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int e = tid + PTH * u;
          Pd[e >> 6][q * NB + (e & 63)] = pd[q][u];
        }
      }
  }
  // own rows: X = W[rows, block] - L[rows, earlier columns] (diagonal rows' earlier columns)^T in tiles of 16 x
  // 16, tile (strip s, columns t): wavefront 5 strip 0, 6 strip 1, 7 strip 2, and strip 3 column by column (5
  // two of its four tiles)
  const int w5 = wave - 5;
  auto strip = [&](int x) { return x < 4 ? w5 : 3; };
  auto tilec = [&](int x) { return x < 4 ? x : x == 4 ? w5 : 3; };
  const int ntile = w5 == 0 ? 6 : 5;
  floatx4 acc[6];
  floatx4 av[2][12];            // this lane's columns 16 b + 4 lk .. + 3 of row lm of the two strips
  if (own && w5 >= 0) {
#pragma unroll
    for (int x = 0; x < 6; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = r0 + 16 * strip(x) + 4 * lk + r;
        const int col = 16 * tilec(x) + lm;
        const bool in = row < n && col < nb;
        const float v = W[(in ? row : r0) * n + c0 + (in ? col : 0)];
        acc[x][r] = in ? v : 0.f;
      }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t row = r0 + 16 * (h == 0 ? w5 : 3) + lm;
      const float* __restrict__ lp = L + (row < n ? row : r0) * ldl + J + 4 * lk;
#pragma unroll
      for (int b = 0; b < 12; ++b)
        if (16 * b < Kp) {
          if (vec) {
            av[h][b] = *reinterpret_cast<const floatx4*>(lp + 16 * b);
          } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) av[h][b][u] = lp[16 * b + u];
          }
        }
    }
  }
  __syncthreads();
  // diagonal block -= (earlier columns) (earlier columns)^T: leaves on or below the diagonal, dealt to the
  // wavefronts
  if (Kp > 0) {
    for (int t = wave; t < 10; t += 8) {
      const int ti = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3, tj = t - ti * (ti + 1) / 2;
      floatx4 d = leaf_load(M, 16 * ti, 16 * tj);
      for (int k = 0; k < Kp; k += 4)
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(-Pd[16 * ti + lm][k + lk], Pd[16 * tj + lm][k + lk], d, 0, 0, 0);
      leaf_store(M, 16 * ti, 16 * tj, d);
    }
    __syncthreads();
  }
  // a quarter of the own rows' columns beside each leaf
  auto rows = [&](int quarter) {
    if (!own || w5 < 0) return;
#pragma unroll
    for (int b = 0; b < 12; ++b) {
      // 4, 8 or 12 blocks of 16 columns
      if (16 * b >= Kp || b / (Kp >> 6) != quarter) continue;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int x = 0; x < 6; ++x)
          if (x < ntile)
            acc[x] = __builtin_amdgcn_mfma_f32_16x16x4f32(-av[x < 4 ? 0 : 1][b][u], Pd[16 * tilec(x) + lm][16 * b + 4 * lk + u],
                                                         acc[x], 0, 0, 0);
    }
    if (quarter == 3) {
#pragma unroll
      for (int x = 0; x < 6; ++x)
        if (x < ntile) leaf_store(X, 16 * strip(x), 16 * tilec(x), acc[x]);
    }
  };
  factor_block(M, Inv, Tmp, nb, c0, info, thr, rows);
  if (blockIdx.x == 0) {
    for (int e = tid; e < NB * NB; e += PTH) {
      const int rr = e >> 6, cc = e & 63;
      if (rr < nb && cc <= rr) L[(c0 + rr) * ldl + c0 + cc] = M[rr][cc];
    }
  }
  if (!own) return;
  // rows = X inv(factor)^T; column tile t takes columns up to its own of the lower triangle: tiles 0 and 3 or 1
  // and 2 to a wavefront
  const int s = wave & 3;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int t = (wave >> 2) == 0 ? 3 * h : 1 + h;
    floatx4 d = {0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k <= t; ++k) leaf_abt(d, X, 16 * s, Inv, 16 * t, 16 * k, 1.f);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = r0 + 16 * s + 4 * lk + r;
      const int col = 16 * t + lm;
      if (row < n && col < nb) L[row * ldl + c0 + col] = d[r];
    }
  }
}

}  // namespace

constexpr int kOuter = 4 * NB;
// Trailing updates of more rows than this run on the fp16 units (split pieces, two launches).  The split
// saves 3 % of a factorization of 5120, 7 % at 6656, 11 % at 8192 and 40 % at 28672; a line at 3072 or 2048
// rows would save another 1 to 3 % from n = 4096 on and nothing below, not enough to leave fp32 products
// for.
constexpr int64_t kSplitRows = 4096;
constexpr int kPanelLds = (4 * NB * BLD + NB * PLD) * (int)sizeof(float);

size_t cholesky_scratch_bytes(int64_t n) {
  return kAlign + 2 * align_up((size_t)n * sizeof(float)) + align_up((size_t)n * n * sizeof(float)) +
         (n > kSplitRows ? pair_syrk256_scratch_bytes(n) : 0);
}

hipError_t launch_cholesky(hipStream_t s, const float* H, int64_t n, int64_t ldh, int precond,
                           float lambda, float* L, int64_t ldl, int* info_dev) {
  // info_dev points at scratch: [int info][pad to 256][float delta[n]][float thr[n]][float W[n x n]][pieces of a panel, large n]
  float* delta = reinterpret_cast<float*>(reinterpret_cast<char*>(info_dev) + kAlign);
  float* thr = reinterpret_cast<float*>(reinterpret_cast<char*>(delta) + align_up((size_t)n * sizeof(float)));
  float* W = reinterpret_cast<float*>(reinterpret_cast<char*>(thr) + align_up((size_t)n * sizeof(float)));
  void* pieces = reinterpret_cast<char*>(W) + align_up((size_t)n * n * sizeof(float));
  // A pivot at or below tau times its column's diagonal entry is rounding noise of the fp32
  // Schur complement (about sqrt(n) 2^-24 of that entry), not information: the matrix is then
  // numerically singular and the factor would be useless to the S-update.
  const float tau = 8.f * sqrtf((float)n) * 5.9604645e-8f;
  hipError_t e;
  static std::atomic<uint64_t> lds_set{0};
  if ((e = ensure_dynamic_lds((const void*)chol_panel_kernel, kPanelLds, lds_set)) != hipSuccess) return e;
  hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(1), 0, s, info_dev, 0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (precond == GANQ_PRECOND_DIAGDOM) {
    hipLaunchKernelGGL(diagdom_delta_kernel, dim3((unsigned)n), dim3(256), 0, s, H, n, ldh, delta);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const bool vec = (n % 4) == 0 && (ldh % 4) == 0 && (ldl % 4) == 0 && (((uintptr_t)H | (uintptr_t)L) & 15) == 0;
  const dim3 cgrid((unsigned)ceil_div(n, 1024), (unsigned)n);
  if (vec)
    hipLaunchKernelGGL(copy_lower_kernel<true>, cgrid, dim3(256), 0, s, H, n, ldh, W, L, ldl, precond, lambda,
                       delta, tau, thr);
  else
    hipLaunchKernelGGL(copy_lower_kernel<false>, cgrid, dim3(256), 0, s, H, n, ldh, W, L, ldl, precond, lambda,
                       delta, tau, thr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int64_t J = 0; J < n; J += kOuter) {
    for (int64_t c0 = J; c0 < n && c0 < J + kOuter; c0 += NB) {
      const int nb = (int)((n - c0 < NB) ? n - c0 : NB);
      const int64_t rem = n - c0 - NB;
      const unsigned wgs = rem > 0 ? (unsigned)ceil_div(rem, NB) : 1u;
      hipLaunchKernelGGL(chol_panel_kernel, dim3(wgs), dim3(PTH), kPanelLds, s, W, L, ldl, n, J, c0, nb,
                         (ldl % 4) == 0 && (((uintptr_t)L) & 15) == 0 ? 1 : 0, info_dev, thr);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int64_t rem = n - J - kOuter;
    if (rem <= 0) break;
    // W22 -= L21 L21^T, lower tiles only
    const float* L21 = L + (J + kOuter) * ldl + J;
    float* W22 = W + (J + kOuter) * n + (J + kOuter);
    const bool al16 = (ldl % 4) == 0 && (((uintptr_t)L21) % 16) == 0;
    if (al16 && rem > kSplitRows)
      e = launch_pair_syrk256(s, rem, L21, ldl, W22, n, pieces);
    else if (al16 && 128 * ldl * 4 < ((int64_t)1 << 31))
      e = launch_syrk256_f32(s, rem, L21, ldl, W22, n);
    else
      e = launch_gemm_f32(s, /*transb=*/1, /*lower_only=*/1, rem, rem, kOuter, -1.f, L21, ldl, L21, ldl, 1.f, W22, n);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ganq
