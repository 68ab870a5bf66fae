// S-update of GANQ: back-substitution on the Cholesky factor L, Eq. (13)-(22)
// and the inner loop of Algorithm 1.
//
// For j = n-1 .. 0 and every row i:
//     tgt  = W_ij + (sum_{u>j} E_iu L_uj) / L_jj,     E_iu = W_iu - T_i[Q_iu]
//     Q_ij = argmin_s |tgt - T_is|   (lowest s on ties)
//
// Rows are independent and columns are sequential.  The columns go in super-blocks of
// 1024 from the right, two launches each:
//   products   F[m x 1024] = E[:, right of the super-block] L[.., super-block] on the fp16
//              matrix cores with both operands split into two fp16 pieces (gemm_split.hip: 22
//              significant bits, fp32 accumulation): the whole chip works on one product, L is read
//              once per row tile and the rate is that of the fp16 units / 3.  L's pieces are made
//              once per layer (transposed, an exponent per column), those of E leave the sweep as
//              the columns are decided (an exponent per row, from max |W_i| + max |T_i|).
//   sweep      one workgroup owns 16 rows and walks the super-block's columns in blocks of 64.
//              Four wavefronts decide the columns of a block one by one in fp32 (16 lanes per row);
//              each decided residual updates the rest of the block and the whole next block
//              (right-looking).  The other four meanwhile multiply, for the next block, the columns
//              right of the current one (the same split products, residual pieces in LDS, pieces of L
//              streamed from L2 up to 12 k steps ahead), stage the next 64 x 128 piece of L in LDS and
//              write out what the block before decided.  So a block costs its 64 dependent steps and one
//              LDS-only barrier.  The product is not done on the fp32 matrix units because those hold
//              up the vector unit of the deciding wavefront on the same SIMD: its steps got slower by
//              exactly the MFMA time (8.0k cycles a block without them, 12.7k with 512 columns' worth).
//
// A step: each row's codebook is sorted once (stable); lane c holds the midpoint between sorted
// codes c and c+1, so the nearest code of a target is the number of midpoints below it: one
// compare, one ballot, one popcount.  The residual of the chosen code is picked out of the 16
// lanes with an exact one-hot lane-row sum (DPP).  A target exactly on a midpoint takes the lower
// code; two equal codes resolve to the lower index.
//
// Infinite weights and NaN act as in an fp32 evaluation: the residual is that of the code written to
// Q (the lowest for a target of -inf or NaN), and as pieces they travel in the low one alone.
//
// Bounds: the dependent steps (n x about 125 cycles and 1.2k cycles of hand-over per 64 of them,
// whatever m up to 16 rows per compute unit) and the products (3 m n^2 flops on the fp16 units).
// Measured per sweep, before (one workgroup walking all n columns, its sums over everything to the
// right on the fp32 matrix units) and now: 4096 x 4096 0.94 -> 0.54 ms (88 us of sweep and 60 us of
// products per super-block), 4096 x 11008 5.4 -> 2.5 ms, 8192 x 28672 71.4 -> 24.8 ms, 256 x 512
// 62 -> 38 us.
#include "ganq_internal.h"

namespace ganq {
namespace {

constexpr int SB = 64;          // columns per block
constexpr int SR = kSlabRows;   // rows per workgroup
constexpr int PU = 12;          // k steps of 32 in flight per multiplying wavefront
constexpr int NW = 8;           // wavefronts per workgroup: 4 decide, 4 multiply
constexpr int NP = 4;
constexpr int WSB = 1024;       // columns per super-block
constexpr int WSPLIT = 2;       // most k-splits of a product
constexpr int LF_COLS16 = WSB / 32 * 2 * 512;   // halves of LF per 16 columns: [k step][piece][lane][8 k]

// One super-block: the sums over the columns right of it are in F (nsplit partial sums, rows of
// WSB); the residuals of its own columns also leave as fp16 pieces (gemm_split.hip) where a
// super-block further left needs them.
struct BlockArgs {
  int64_t jlo, jhi;          // its columns
  const float* F;
  int64_t fstride;
  int nsplit;                // 0: nothing to the right
  _Float16* Ep;              // residual pieces of the whole layer
  const _Float16* LF;        // pieces of L inside the super-blocks, in the order of the sweep's loads
  int64_t kp;                // rows of Ep hold 2 kp halves
  const float* wmax;         // max |W_i|; null where no residual is ever multiplied as pieces
  int* ea;                   // exponents of the rows of Ep, written by the first super-block
  const int* eb;             // exponents of the columns of L
};

template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ inline int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
// value of lane K of this lane's 16-lane row
template <int K>
__device__ inline float row_bcast(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + K, 0xf, 0xf, true));
}
template <int K>
__device__ inline int row_bcast_i(int v) { return dpp_i<0x150 + K>(v); }


// Stable rank of this lane's code within its row, and "is lane k's code equal to mine".
template <int K>
struct RankLoop {
  __device__ static inline void run(float tc, int c, int& rank) {
    const float tk = row_bcast<K>(tc);
    rank += (tk < tc || (tk == tc && K < c)) ? 1 : 0;
    if constexpr (K > 0) RankLoop<K - 1>::run(tc, c, rank);
  }
};
template <int K>
struct RepLoop {
  // lowest original index among the sorted positions that hold the same value as mine
  __device__ static inline void run(float ts, int orig, int& rep) {
    const float tk = row_bcast<K>(ts);
    const int ok = row_bcast_i<K>(orig);
    if (tk == ts && ok < rep) rep = ok;
    if constexpr (K > 0) RepLoop<K - 1>::run(ts, orig, rep);
  }
};

// One column of the sequential phase (local column JL of the block).  The row of L that a step
// multiplies by (d: the block's own columns, x: the next block's) is read from LDS two steps ahead.
// Only the update of the register that the next step reads is on the dependency chain; the others
// are left to the next step (ep, prev), where they fill the slots between its dependent operations.
struct LRow {
  float4 d, x;
};
constexpr int LPITCH = 2 * SB;        // floats per staged row: column 16 q + c sits at 4 c + q, next block first
__device__ inline LRow load_lrow(const float* Ld, int jl, int c) {
  LRow r;
  r.x = *reinterpret_cast<const float4*>(Ld + jl * LPITCH + 4 * c);
  r.d = *reinterpret_cast<const float4*>(Ld + jl * LPITCH + SB + 4 * c);
  return r;
}
__device__ inline float part(const float4& v, int q) { return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w; }

// `hook` runs in front of column 47: the requests for the next block, which at the block's start would
// queue behind those of the multiplying wavefronts.
template <int JL, bool FULL, typename HOOK>
struct Step {
  // lo, hi: midpoints on either side of this lane's code; votes: lane JL collects the lanes that
  // step JL chose (a bit per lane of the wavefront).  The scheduling barriers keep two independent
  // operations behind each result that a lane-row operation reads (it waits two slots for it).
  __device__ static inline void run(int bw, int c, float ts, float lo, float hi, const float (&Wr)[4],
                                    const float (&rd)[4], float (&acc)[4], float (&accn)[4], float (&Er)[4],
                                    uint32_t (&votes)[2], const float* Ld, float ep, const LRow& prev,
                                    const LRow& cur, const LRow& nx1,
                                    const HOOK& hook) {
    if constexpr (JL == 47) hook();
    LRow nx2;
    if constexpr (JL >= 2) nx2 = load_lrow(Ld, JL - 2, c);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int co = JL & 15, qo = JL >> 4;
    float e = 0.f;
    if (FULL || JL < bw) {
      const float tl = fmaf(acc[qo], rd[qo], Wr[qo]);
      __builtin_amdgcn_sched_barrier(0);
      accn[0] = fmaf(ep, prev.x.x, accn[0]);
      const float cand = row_bcast<co>(Wr[qo]) - ts;
      float cand0 = (c == 0) ? cand : 0.f;
      asm("" : "+v"(cand0));
      __builtin_amdgcn_sched_barrier(0);
      const float tg = row_bcast<co>(tl);
      // lane 0 holds for every target that is not above its midpoint; for -inf and NaN there is no vote
      const unsigned long long upto = __builtin_amdgcn_ballot_w64(!(tg > hi)), from = __builtin_amdgcn_ballot_w64(tg > lo);
      float x = (tg > lo) ? cand : cand0;
      asm("" : "+v"(x));      // selects one after the other: combining masks would take a detour over the scalar unit
      x = (tg > hi) ? 0.f : x;
      __builtin_amdgcn_sched_barrier(0);
      accn[1] = fmaf(ep, prev.x.y, accn[1]);
      accn[2] = fmaf(ep, prev.x.z, accn[2]);
      __builtin_amdgcn_sched_barrier(0);
      x += dpp_f<0xB1>(x);    // quad_perm [1,0,3,2]
      __builtin_amdgcn_sched_barrier(0);
      accn[3] = fmaf(ep, prev.x.w, accn[3]);
      if constexpr (qo > 0) acc[0] = fmaf(ep, prev.d.x, acc[0]);
      __builtin_amdgcn_sched_barrier(0);
      x += dpp_f<0x4E>(x);    // quad_perm [2,3,0,1]
      __builtin_amdgcn_sched_barrier(0);
      const unsigned long long chosen = from & upto;
      asm("v_writelane_b32 %0, %1, %2" : "+v"(votes[0]) : "s"((uint32_t)chosen), "n"(JL));
      asm("v_writelane_b32 %0, %1, %2" : "+v"(votes[1]) : "s"((uint32_t)(chosen >> 32)), "n"(JL));
      __builtin_amdgcn_sched_barrier(0);
      x += dpp_f<0x141>(x);   // row_half_mirror
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (qo > 1) acc[1] = fmaf(ep, prev.d.y, acc[1]);
      if constexpr (qo > 2) acc[2] = fmaf(ep, prev.d.z, acc[2]);
      __builtin_amdgcn_sched_barrier(0);
      e = x + dpp_f<0x140>(x);   // row_mirror
      // the register the next step reads
      constexpr int qn = (JL > 0) ? (JL - 1) >> 4 : 0;
      if constexpr (JL > 0) {
        acc[qn] = fmaf(e, part(cur.d, qn), acc[qn]);
      }
      if (c == co) Er[qo] = e;
    }
    if constexpr (JL > 0) {
      Step<JL - 1, FULL, HOOK>::run(bw, c, ts, lo, hi, Wr, rd, acc, accn, Er, votes, Ld, e, cur, nx1, nx2, hook);
    } else {
      accn[0] = fmaf(e, cur.x.x, accn[0]);
      accn[1] = fmaf(e, cur.x.y, accn[1]);
      accn[2] = fmaf(e, cur.x.z, accn[2]);
      accn[3] = fmaf(e, cur.x.w, accn[3]);
    }
  }
};

constexpr int EP_HALVES = WSB * SR;               // one piece of the super-block's residuals: [k / 8][row][k % 8]
constexpr int LD_FLOATS = SB * LPITCH;            // one staged piece of L
constexpr int RPITCH = SB + 4;
constexpr int RED_FLOATS = SR * RPITCH;           // a block's sums: [row][column]
constexpr int S_LDS_BYTES = 2 * EP_HALVES * 2 + 2 * LD_FLOATS * 4 + 2 * RED_FLOATS * 4 + 2 * NP * SB * 8 + SR * 16 * 4 + SR * 4;

// LDS is handed over; loads and stores in flight to memory stay in flight.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <bool VECL>
__global__ __launch_bounds__(64 * NW) void update_S_kernel(const float* __restrict__ W, int64_t m, int64_t n,
                                                       int64_t ldw, const float* __restrict__ L, int64_t ldl,
                                                       const float* __restrict__ rdiag,
                                                       const float* __restrict__ T, int C,
                                                       uint8_t* __restrict__ Q, int64_t ldq, BlockArgs sb) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  _Float16* Eh = reinterpret_cast<_Float16*>(smem);             // residual pieces, high
  _Float16* Elo = Eh + EP_HALVES;                               // and low
  float* Ldb = reinterpret_cast<float*>(Elo + EP_HALVES);       // two staged pieces: 64 rows x (next block | this block)
  float* red = Ldb + 2 * LD_FLOATS;                             // two blocks' sums over the columns further right
  unsigned long long* votes = reinterpret_cast<unsigned long long*>(red + 2 * RED_FLOATS);   // [2][wavefront][column]
  int* repl = reinterpret_cast<int*>(votes + 2 * NP * SB);      // [row][sorted position] -> original index
  int* eal = repl + SR * 16;                                    // [row] exponent of the pieces

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, g = lane >> 4;
  const bool p2 = wv < NP;                        // wavefronts that decide columns (4 rows each)
  const int64_t row0 = (int64_t)blockIdx.x * SR;

  const int64_t jlo = sb.jlo, jhi = sb.jhi;
  const int nblk = (int)ceil_div(jhi - jlo, SB);  // blocks of this super-block
  const int64_t kend = jlo + (int64_t)nblk * SB;  // its padded end: columns >= n have E = 0

  if (p2) {
    const int r = 4 * wv + g;                         // row within the slab
    const int64_t row = row0 + r;
    const bool row_ok = row < m;
    // ---- sort this row's codebook (stable), build midpoints and tie representatives ----
    float tc = __builtin_huge_valf();
    if (c < C) tc = row_ok ? T[row * C + c] : 0.f;
    int rank = 0;
    RankLoop<15>::run(tc, c, rank);
    const int paddr = ((lane & 48) | rank) << 2;
    const float ts = __builtin_bit_cast(float, __builtin_amdgcn_ds_permute(paddr, __builtin_bit_cast(int, tc)));
    const int orig = __builtin_amdgcn_ds_permute(paddr, c);
    int rep = orig;
    RepLoop<15>::run(ts, orig, rep);
    const float tnext = dpp_f<0x101>(ts);             // row_shl:1 -> value of lane c + 1
    const float mid = (c < 15) ? 0.5f * (ts + tnext) : __builtin_huge_valf();
    const float below = dpp_f<0x111>(mid);            // row_shr:1 -> midpoint of lane c - 1
    const float lo = (c > 0) ? below : -__builtin_huge_valf();
    repl[r * 16 + c] = rep;
    // |E_ij| <= max |W_i| + max |T_i| is brought below 2^15
    float tm = fabsf(tc);
    tm = (tm < __builtin_huge_valf()) ? tm : 0.f;
    tm = fmaxf(tm, dpp_f<0xB1>(tm));
    tm = fmaxf(tm, dpp_f<0x4E>(tm));
    tm = fmaxf(tm, dpp_f<0x141>(tm));
    tm = fmaxf(tm, dpp_f<0x140>(tm));
    tm += (row_ok && sb.wmax != nullptr) ? sb.wmax[row] : 0.f;
    // (the sum of two finite maxima may itself be out of range: it is below 2^129 then)
    const int ea = (tm > 0.f) ? 14 - (tm < __builtin_huge_valf() ? ilogbf(tm) : 128) : 0;
    if (c == 0) {
      eal[r] = ea;
      if (sb.jhi == n && row_ok) sb.ea[row] = ea;     // for the products of the super-blocks to come
    }
    lds_barrier();

    // a block's weights, reciprocals and sums from the right are requested one block ahead
    const int64_t rowc = row_ok ? row : m - 1;
    const float* Wp = W + rowc * ldw + c;
    const float* Rp = rdiag + c;
    const float* Fp = sb.F + rowc * WSB + c;
    float Wr[4], rd[4], fr[WSPLIT][4];
#pragma unroll
    for (int sp = 0; sp < WSPLIT; ++sp)
#pragma unroll
      for (int q = 0; q < 4; ++q) fr[sp][q] = 0.f;
    auto fetch = [&](int b) {
      const int64_t j0 = jlo + (int64_t)b * SB;
      if (j0 + SB <= n) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          Wr[q] = Wp[j0 + 16 * q];
          rd[q] = Rp[j0 + 16 * q];
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool ok = j0 + 16 * q + c < n;
          Wr[q] = ok ? Wp[j0 + 16 * q] : 0.f;
          rd[q] = ok ? Rp[j0 + 16 * q] : 0.f;
        }
      }
      // sums from the right exist where the super-block is whole
#pragma unroll
      for (int sp = 0; sp < WSPLIT; ++sp)
        if (sp < sb.nsplit) {
#pragma unroll
          for (int q = 0; q < 4; ++q) fr[sp][q] = Fp[sp * sb.fstride + b * SB + 16 * q];
        }
    };
    fetch(nblk - 1);
    float accn[4] = {0.f, 0.f, 0.f, 0.f};
    for (int b = nblk - 1; b >= 0; --b) {
      const int64_t j0 = jlo + (int64_t)b * SB;
      const int bw = (int)((n - j0 < SB) ? n - j0 : SB);
      float acc[4], Wc[4], rc[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float sum = accn[q];
        if (b + 2 < nblk) sum += red[(b & 1) * RED_FLOATS + r * RPITCH + 16 * q + c];
#pragma unroll
        for (int sp = 0; sp < WSPLIT; ++sp) sum += fr[sp][q];
        acc[q] = sum;
        accn[q] = 0.f;
        Wc[q] = Wr[q];
        rc[q] = rd[q];
      }
      auto next = [&]() {
        if (b > 0) fetch(b - 1);
      };

      float Er[4] = {0.f, 0.f, 0.f, 0.f};
      uint32_t vt[2] = {0u, 0u};
      const float* Ld = Ldb + ((nblk - 1 - b) & 1) * LD_FLOATS;
      LRow zero;
      zero.d = zero.x = make_float4(0.f, 0.f, 0.f, 0.f);
      const LRow l0 = load_lrow(Ld, SB - 1, c), l1 = load_lrow(Ld, SB - 2, c);
      if (bw == SB)
        Step<SB - 1, true, decltype(next)>::run(bw, c, ts, lo, mid, Wc, rc, acc, accn, Er, vt, Ld, 0.f, zero, l0, l1, next);
      else
        Step<SB - 1, false, decltype(next)>::run(bw, c, ts, lo, mid, Wc, rc, acc, accn, Er, vt, Ld, 0.f, zero, l0, l1, next);

#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // an infinite residual or NaN goes into the low piece alone: every product of it is then one with
        // L's high piece, infinite or NaN as in fp32 (inf in the high piece would meet a low piece of L
        // that is zero or of the other sign)
        const float v = ldexpf(Er[q], ea);
        const _Float16 hi = (_Float16)((fabsf(v) < __builtin_huge_valf()) ? v : 0.f);
        const int at = ((b * 8 + 2 * q + (c >> 3)) * SR + r) * 8 + (c & 7);
        Eh[at] = hi;
        Elo[at] = (_Float16)(v - (float)hi);
      }
      votes[((b & 1) * NP + wv) * SB + lane] = (unsigned long long)vt[1] << 32 | vt[0];
      lds_barrier();     // residuals and choices of this block; sums and L of the next one
    }
  } else {
    // ---- the other wavefronts, per block b: write out block b + 1; the sums of block b - 1 over the
    // columns right of b; the piece of L for block b - 1 ----
    const int wq = wv - NP, ft = tid - 64 * NP;
    // rows [j0, j0 + 64) of L, columns of the block before (x) and of the block itself (d), permuted for
    // load_lrow; a thread takes 4 columns of every eighth row.  Rows from n on and columns left of the
    // super-block lie outside the descriptor and read as zero.  What stands on and above the diagonal
    // only reaches the sums of columns that are already decided.
    const int srow = ft >> 5, scol = (ft & 31) * 4;      // column j0 - 64 + scol
    auto stage_load = [&](int b, int hf, float4 (&v)[4]) {
      const int64_t j0 = jlo + (int64_t)b * SB;
      const int64_t rows = (n - j0 < SB) ? n - j0 : SB;
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(L + j0 * ldl), 0, (int)(((rows - 1) * ldl + n) * (int64_t)sizeof(float)), 0x00020000);
      const int64_t gc = j0 - SB + scol;
      const uint32_t vo = (gc >= jlo) ? (uint32_t)((srow * ldl + gc) * sizeof(float)) : 0x7ffffff0u;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t so = (uint32_t)(8 * (4 * hf + u) * ldl * sizeof(float));
        if (VECL) {
          v[u] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo, so, 0));
        } else {
          v[u].x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, 0));
          v[u].y = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo + 4, so, 0));
          v[u].z = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo + 8, so, 0));
          v[u].w = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo + 12, so, 0));
        }
      }
    };
    auto stage_store = [&](float* dst, int hf, const float4 (&v)[4]) {
      const int half = scol >> 6, cl = scol & 63;        // column cl of its block: 16 q + c
      float* d = dst + (srow + 32 * hf) * LPITCH + half * SB + (cl >> 4) + 4 * (cl & 15);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        d[8 * u * LPITCH] = v[u].x;
        d[8 * u * LPITCH + 4] = v[u].y;
        d[8 * u * LPITCH + 8] = v[u].z;
        d[8 * u * LPITCH + 12] = v[u].w;
      }
    };
    {
      float4 v[4];
      for (int hf = 0; hf < 2; ++hf) {
        stage_load(nblk - 1, hf, v);
        stage_store(Ldb, hf, v);
      }
    }
    lds_barrier();
    const int orow = ft >> 4, oc = 4 * (ft & 15);     // four decided columns of one row
    const int64_t grow = row0 + orow;
    auto write_out = [&](int b) {
      const int64_t col = jlo + (int64_t)b * SB + oc;
      if (grow < m) {
        uint32_t q4 = 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          // the lane of this row that the column's step chose; no vote means the lowest code
          const unsigned long long v = votes[((b & 1) * NP + (orow >> 2)) * SB + oc + u];
          const uint32_t v16 = (uint32_t)(v >> (16 * (orow & 3))) & 0xffffu;
          const int q = repl[orow * 16 + (v16 != 0u ? __builtin_ctz(v16) : 0)];
          q4 |= (uint32_t)q << (8 * u);
        }
        uint8_t* dst = Q + grow * ldq + col;
        if (col + 4 <= n && ((uintptr_t)dst & 3) == 0) {
          *reinterpret_cast<uint32_t*>(dst) = q4;
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (col + u < n) dst[u] = (uint8_t)(q4 >> (8 * u));
        }
      }
      // pieces for the products of the super-blocks further left: 8 columns of one row a thread
      if (jlo > 0) {
        const int prow = ft & 15, k8 = (ft >> 4) & 7, piece = ft >> 7;
        const int64_t pc = jlo + (int64_t)b * SB + 8 * k8;
        if (row0 + prow < m && pc < sb.kp)
          *reinterpret_cast<half8*>(sb.Ep + (row0 + prow) * 2 * sb.kp + (pc >> 5) * 64 + 32 * piece + (pc & 31)) =
              *reinterpret_cast<const half8*>((piece ? Elo : Eh) + ((b * 8 + k8) * SR + prow) * 8);
      }
    };
    int ear[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) ear[v] = eal[4 * g + v];
    // lane l supplies column 16 wq + l % 16 of the block and 8 k from 8 (l / 16) of a step; the pieces
    // lie in that order, a kilobyte of each per 16 columns and step (read out of LT's rows, which are a
    // power of two apart as often as not, the 16 lines of a load fell on one cache channel: 3.3k cycles
    // per 12 steps).  Steps run from the right end (the oldest residuals) to the left.
    const int64_t kmax = (kend < sb.kp) ? kend : sb.kp;
    const uint32_t loff = (uint32_t)(lane * 16);
    struct Frag {
      half8 h, l;
    };
    for (int b = nblk - 1; b >= 0; --b) {
      const int64_t k0 = jlo + (int64_t)(b + 1) * SB;
      if (b > 0) {
        const int nst = (int)((kmax - k0) / 32);
        const int64_t jb = k0 - 2 * SB;                        // first column of block b - 1
        const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(sb.LF + (jb / 16 + wq) * LF_COLS16), 0, LF_COLS16 * 2, 0x00020000);
        const uint32_t s0 = (uint32_t)(((kmax - jlo) / 32 - 1) * 2048);
        auto fetch = [&](int st) {
          Frag f;
          const uint32_t so = s0 - 2048u * (uint32_t)(st < nst ? st : nst - 1);
          f.h = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(rl, loff, so, 0));
          f.l = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(rl, loff + 1024, so, 0));
          return f;
        };
        floatx4 mhh = {0.f, 0.f, 0.f, 0.f}, mlh = mhh, mhl = mhh;
        const int ebase = (int)((kmax - jlo) / 8 - 4);
        auto mma = [&](const Frag& f, int st) {
          const int at = ((ebase - 4 * st + g) * SR + c) * 8;
          const half8 ah = *reinterpret_cast<const half8*>(Eh + at), al = *reinterpret_cast<const half8*>(Elo + at);
          mhh = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, f.h, mhh, 0, 0, 0);
          mlh = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, f.h, mlh, 0, 0, 0);
          mhl = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, f.l, mhl, 0, 0, 0);
        };
        Frag f[PU];
        if (nst > 0) {
#pragma unroll
          for (int u = 0; u < PU; ++u) f[u] = fetch(u);
        }
        const int ebj = sb.eb[jb + 16 * wq + c];
        float* Ldn = Ldb + ((nblk - b) & 1) * LD_FLOATS;
        float4 v[4];
        stage_load(b - 1, 0, v);
        if (b + 1 < nblk) write_out(b + 1);
        stage_store(Ldn, 0, v);
        stage_load(b - 1, 1, v);
        int s = 0;
        for (; s + PU <= nst; s += PU) {
#pragma unroll
          for (int u = 0; u < PU; ++u) {
            mma(f[u], s + u);
            f[u] = fetch(s + u + PU);          // past the last step: the last one again, never used
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int u = 0; u < PU; ++u)
          if (s + u < nst) mma(f[u], s + u);
        if (nst > 0) {
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4)
            red[((b - 1) & 1) * RED_FLOATS + (4 * g + v4) * RPITCH + 16 * wq + c] =
                ldexpf(mhh[v4] + (mlh[v4] + mhl[v4]), -(ear[v4] + ebj));
        }
        stage_store(Ldn, 1, v);
      } else if (nblk > 1) {
        write_out(1);
      }
      lds_barrier();
    }
    write_out(0);
  }
}

// ---- operands of the products ----

// rdiag[j] = 1 / L_jj and eb[j]: the exponent that brings max |L_kj| over k > j near 2^14.  One
// workgroup per 64 columns, 16 rows side by side.
__global__ __launch_bounds__(1024) void l_column_kernel(const float* __restrict__ L, int64_t n, int64_t ldl,
                                                        float* __restrict__ rdiag, int* __restrict__ eb) {
  __shared__ float red[16][64];
  const int jj = threadIdx.x & 63, kk = threadIdx.x >> 6;
  const int64_t j0 = (int64_t)blockIdx.x * 64, j = j0 + jj;
  float mx = 0.f;
  if (j < n) {
#pragma unroll 8
    for (int64_t k = j0 + 1 + kk; k < n; k += 16) {
      const float v = fabsf(L[k * ldl + j]);
      if (k > j && v < __builtin_huge_valf() && v > mx) mx = v;
    }
  }
  red[kk][jj] = mx;
  __syncthreads();
  if (kk == 0 && j < n) {
#pragma unroll
    for (int u = 1; u < 16; ++u) mx = fmaxf(mx, red[u][jj]);
    eb[j] = (mx > 0.f) ? 14 - ilogbf(mx) : 0;
    rdiag[j] = 1.f / L[j * ldl + j];
  }
}

// Pieces of L, 64 x 64 tiles through LDS.  Right of column j's super-block they go to row j of LT (the
// products' operand; each line of 32 k leaves whole), inside it and right of j's block of 64 to LF.
__global__ __launch_bounds__(256) void l_pieces_kernel(const float* __restrict__ L, int64_t n, int64_t ldl,
                                                       const int* __restrict__ eb, int64_t kp,
                                                       _Float16* __restrict__ LT, _Float16* __restrict__ LF) {
  __shared__ float tile[64][65];
  const int64_t j0 = (int64_t)blockIdx.x * 64, k0 = (int64_t)blockIdx.y * 64;
  if (k0 <= j0) return;
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int kk = u * 4 + (tid >> 6), jj = tid & 63;
    tile[kk][jj] = (k0 + kk < n) ? L[(k0 + kk) * ldl + j0 + jj] : 0.f;     // j0 + 63 < k0 <= n - 1
  }
  __syncthreads();
  const int jj = tid >> 2, kq = (tid & 3) * 16;
  const int e = eb[j0 + jj];
  if (k0 + kq >= kp) return;
  half8 hi[2], lo[2];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const float v = ldexpf(tile[kq + u][jj], e);
    const _Float16 h = (_Float16)((fabsf(v) < __builtin_huge_valf()) ? v : 0.f);      // as for the residuals
    hi[u >> 3][u & 7] = h;
    lo[u >> 3][u & 7] = (_Float16)(v - (float)h);
  }
  if (k0 / WSB == j0 / WSB) {
    _Float16* d = LF + ((j0 + jj) / 16 * (WSB / 32) + (k0 % WSB + kq) / 32) * 1024 + ((kq & 31) / 8 * 16 + (jj & 15)) * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      *reinterpret_cast<half8*>(d + 128 * h) = hi[h];
      *reinterpret_cast<half8*>(d + 512 + 128 * h) = lo[h];
    }
  } else {
    _Float16* d = LT + (j0 + jj) * 2 * kp + ((k0 + kq) >> 5) * 64 + (kq & 31);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      *reinterpret_cast<half8*>(d + 8 * h) = hi[h];
      *reinterpret_cast<half8*>(d + 32 + 8 * h) = lo[h];
    }
  }
}

// wmax[i] = max |W_ij|
__global__ __launch_bounds__(256) void s_rowmax_kernel(const float* __restrict__ W, int64_t n, int64_t ldw,
                                                       float* __restrict__ wmax) {
  __shared__ float red[4];
  const int64_t row = blockIdx.x;
  float mx = 0.f;
  for (int64_t k = threadIdx.x; k < n; k += 256) {
    const float v = fabsf(W[row * ldw + k]);
    if (v < __builtin_huge_valf() && v > mx) mx = v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) wmax[row] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// E = W - T[Q], one workgroup per row (rows on x: this call takes more of them than the y axis holds)
__global__ __launch_bounds__(256) void s_residual_kernel(const float* W, int64_t n, int64_t ldw,
                                                         const float* __restrict__ T, int C,
                                                         const uint8_t* __restrict__ Q, int64_t ldq, float* E,
                                                         int64_t lde) {
  __shared__ float tr[16];
  const int64_t i = blockIdx.x;
  if ((int)threadIdx.x < C) tr[threadIdx.x] = T[i * C + threadIdx.x];
  __syncthreads();
  for (int64_t j = threadIdx.x; j < n; j += 256) E[i * lde + j] = W[i * ldw + j] - tr[Q[i * ldq + j]];
}

// Scratch of the S-update, carved in one place.
struct SScratch {
  float *rdiag, *wmax;
  int *ea, *eb;
  _Float16 *LF, *LT, *Ep;
  float* F;
  size_t bytes;
  SScratch(void* base, int64_t m, int64_t n) {
    size_t off = 0;
    auto take = [&](size_t b) {
      const size_t at = off;
      off += align_up(b);
      return base != nullptr ? (char*)base + at : nullptr;
    };
    rdiag = (float*)take((size_t)n * sizeof(float));
    wmax = (float*)take((size_t)m * sizeof(float));
    ea = (int*)take((size_t)m * sizeof(int));
    eb = (int*)take((size_t)n * sizeof(int));
    LF = (_Float16*)take((size_t)ceil_div(n, 64) * 4 * LF_COLS16 * sizeof(_Float16));
    // only where there is more than one super-block
    LT = (_Float16*)take(n > WSB ? pair_bytes(n, n) : 0);
    Ep = (_Float16*)take(n > WSB ? pair_bytes(m, n) : 0);
    F = (float*)take(n > WSB ? (size_t)WSPLIT * m * WSB * sizeof(float) : 0);
    bytes = off;
  }
};

}  // namespace

size_t update_s_scratch_bytes(int64_t m, int64_t n) { return SScratch(nullptr, m, n).bytes; }

hipError_t launch_update_S_prepare(hipStream_t s, const float* W, int64_t m, int64_t n, int64_t ldw, const float* L,
                                   int64_t ldl, void* scratch) {
  const SScratch sc(scratch, m, n);
  hipError_t e;
  if (n > 2 * SB) {
    hipLaunchKernelGGL(s_rowmax_kernel, dim3((unsigned)m), dim3(256), 0, s, W, n, ldw, sc.wmax);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const unsigned c64 = (unsigned)ceil_div(n, 64);
  hipLaunchKernelGGL(l_column_kernel, dim3(c64), dim3(1024), 0, s, L, n, ldl, sc.rdiag, sc.eb);
  if ((e = hipGetLastError()) != hipSuccess || c64 < 2) return e;
  hipLaunchKernelGGL(l_pieces_kernel, dim3(c64, c64), dim3(256), 0, s, L, n, ldl, sc.eb, pair_columns(n), sc.LT, sc.LF);
  return hipGetLastError();
}

hipError_t launch_update_S(hipStream_t s, const float* W, int64_t m, int64_t n, int64_t ldw,
                           const float* L, int64_t ldl, const float* T, int nbits, uint8_t* Q,
                           int64_t ldq, float* E, int64_t lde, void* scratch) {
  const SScratch sc(scratch, m, n);
  const int C = 1 << nbits;
  const int64_t kp = pair_columns(n);
  hipError_t e;
  const bool vec = (ldl % 4 == 0) && (((uintptr_t)L) % 16 == 0);
  static std::atomic<uint64_t> lds_a{0}, lds_b{0};
  e = vec ? ensure_dynamic_lds((const void*)update_S_kernel<true>, S_LDS_BYTES, lds_a)
          : ensure_dynamic_lds((const void*)update_S_kernel<false>, S_LDS_BYTES, lds_b);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)ceil_div(m, SR)), block(64 * NW);
  for (int64_t jlo = (n - 1) / WSB * WSB; jlo >= 0; jlo -= WSB) {
    BlockArgs sb{};
    sb.jlo = jlo;
    sb.jhi = (jlo + WSB < n) ? jlo + WSB : n;
    sb.F = sc.F;
    sb.fstride = m * WSB;
    sb.Ep = sc.Ep;
    sb.LF = sc.LF;
    sb.kp = kp;
    sb.wmax = (n > 2 * SB) ? sc.wmax : nullptr;     // a block and the one after it update each other in fp32
    sb.ea = sc.ea;
    sb.eb = sc.eb;
    if (sb.jhi < n) {
      const int s0 = (int)(sb.jhi / 32), s1 = (int)(kp / 32);
      // Two k-splits where one gives no more than a tile per compute unit, which holds two, and they still
      // have 16 steps each.  8192 x 8192 with one split 2.85 ms, with two 2.94; 4096 rows with one leave
      // half the slots empty.
      sb.nsplit = (s1 - s0 >= 32 && ceil_div(m, 128) * (WSB / 128) <= 256) ? 2 : 1;
      if ((e = launch_pair_gemm(s, sc.Ep, sc.LT + jlo * 2 * kp, m, WSB, kp, s0, s1, sb.nsplit, sc.ea, sc.eb + jlo,
                                sc.F, WSB, sb.fstride, true)) != hipSuccess) return e;
    }
    if (vec)
      hipLaunchKernelGGL(update_S_kernel<true>, grid, block, S_LDS_BYTES, s, W, m, n, ldw, L, ldl, sc.rdiag, T, C, Q,
                         ldq, sb);
    else
      hipLaunchKernelGGL(update_S_kernel<false>, grid, block, S_LDS_BYTES, s, W, m, n, ldw, L, ldl, sc.rdiag, T, C, Q,
                         ldq, sb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // the residuals themselves, for a caller who asked for them: W - T[Q] as the sweep formed them
  if (E != nullptr)
    hipLaunchKernelGGL(s_residual_kernel, dim3((unsigned)m), dim3(256), 0, s, W, n, ldw, T, C, Q, ldq, E, lde);
  return hipGetLastError();
}

}  // namespace ganq
