// Factorisation of the real-shifted coarsest operator A3 (eq. 3.6) on the GPU (set-up, FP64).
//
// Fronts are processed by height in the nested-dissection tree (nd_plan.cpp).  A front
// matrix F (nF x nF, row major, S nodes first) is assembled from the original coefficients
// and the children's Schur complements (extend-add).  With A = F_SS, B = F_SB, C = F_BS,
// D = F_BB the front then gives
//     L = [A^-1; C A^-1],   W = -A^-1 B   (stored in the substitution's precision)
//     D + C W                             (its Schur complement, for the parent).
// A is inverted by Gauss-Jordan exchange steps with partial pivoting among the S rows; the
// rest are dense products with the whole inverse, on the FP64 matrix cores:
//     W = -A^-1 B  (depth nS),  C A^-1  (depth nS),  D += C W  (depth nS).
// Taking them once per front, after the inversion, keeps B, C and D (most of the front) out
// of the pivoting: a panel covers the nS rows of A instead of all nF, the products run at
// full depth instead of in slices of 8 to 128, and no row swap touches B.  FP32 factors are
// those of a 5/7-point operator, which is complex symmetric: there C A^-1 = -W^T needs no product
// and D + C W is formed for its lower tiles only, nS^3 + nS^2 nB + nS nB^2 / 2 complex
// multiply-adds instead of nS (nS + nB)^2.  FP64 factors take every product: W and C A^-1 round
// apart where A is ill-conditioned, and the transpose of one for the other costs digits that FP32
// factors don't hold (undamped 428x484, 44x48x80 and 28x64x28 grids: 9e-8, 6e-9 and 6e-10 against
// 7e-11, 5e-12 and 2e-12; 1.2 to 1.4 times the error on damped ones; 1 % of a 600x640 step).
// Set-up times against exchanging the S pivots over all nF rows
// and columns: 228 -> 121 ms (256^3), 6.8 -> 4.8 ms (1024^2), 62.7 -> 41.7 ms (192x192x72
// compact), 17.5 -> 11.3 ms (1024^2 compact), 1.19 -> 0.74 ms (128^2).
//
// Exchange steps without row swaps.  Exchanging pivot (p, k) in y = Q x makes row p stand
// for x_k and column k for y_p:
//     Q[i][j] -= Q[i][k] Q[p][j] / Q[p][k],   Q[i][k] = Q[i][k] / Q[p][k],
//     Q[p][j] = -Q[p][j] / Q[p][k],           Q[p][k] = 1 / Q[p][k].
// Rows stay where they are; pm[k] is the pivot row of column k, ip its inverse.  Once every
// column is exchanged, A^-1[k][pm[l]] = Q[pm[k]][l] (k_inv_final).
//
// A run of pivots K is taken in three nested sizes: panels of KB columns in registers
// (k_inv_panel), blocks of several panels, and windows of at most HELM_ND_WIN rows.  After
// a run, every column J outside it takes one product
//     Q[:, J] = Q0[:, J] (pivot rows: 0) - Q'[:, K] Q0[pm[K], J]           (k_inv_gemm),
// read from one copy of A and written to the other (the front itself and a scratch copy,
// parity 0 and 1), so that a launch reads no entry that it writes.  The pivots of a window's
// columns come from the window's rows; the rows of A outside the window take their part of the
// run's columns from the finished window, Q'[i, K] = Q0[i, K] Q'[pm[K], K] (k_inv_outer).
//
// Windows bound the rows that a panel searches and keeps in registers, but the rows of one may
// hold no good pivots where the whole separator does: a window's block is the operator with
// zero values beyond it, and near a resonance of that part of the grid it is singular (without
// damping; 1536 rows, 2 windows, at such a frequency: the coarsest solve was wrong in every digit,
// 1e-14 with pivots from all rows).  The loss shows as large entries Q'[i, K] in the rows still to
// be pivoted, the multipliers of the window's elimination: the error grows about as their square
// (largest multiplier 1.3, 4.6, 46, 460: 1.3, 26, 75, 25000 times that with pivots from all rows).
// k_inv_outer reports any beyond 1, which pivoting over all rows keeps every step to, and the
// factorisation is then taken again with one window per separator, whose panels search all its
// rows.  Multipliers of at most 1 cost nothing (ratios of 0.94 to 1.24, geometric mean 1.00, over 88
// grids).  With an absorbing layer or a complex shift they are 0.25 to 1 at 144^3 to 256^3 (G = 5 to
// 12), without either 4 to 16; of the 2D roots merged to 1025 to 1100 rows some exceed 1, for
// homogeneous media above all (up to 6).
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace helm {

__global__ void __launch_bounds__(256) k_nd_assemble(const NDFrontDev* __restrict__ hf,
                                                     const NDAsm* __restrict__ asmv, const cd* __restrict__ coef,
                                                     cd* __restrict__ Fp) {
  const NDFrontDev f = hf[blockIdx.y];
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < f.asm_cnt;
       e += (long long)gridDim.x * blockDim.x) {
    NDAsm a = asmv[f.asm_off + e];
    cd* F = Fp + f.F_off;
    F[(long long)a.row * f.nF + a.col] += coef[a.cidx];
  }
}

// A front from its children's Schur complements: F[i][j] = sum over the children that hold both
// i and j.  A work-group owns EXT_R rows of 256 columns, a thread one column; for each child it
// inverts the child's position map over those rows and columns in LDS (positions outside: -1)
// and adds the child's entries, so every entry of F is written once and nothing is cleared
// before.  Bound by the memory it moves; the maps are a few loads per thread from the L2.  As
// one read-add-write launch per child over a cleared F, extending took 11.0 ms at 256^3 and
// clearing 3.8; together they now take 7.3.
#define EXT_R 8
__global__ void __launch_bounds__(256) k_nd_extend(const NDFrontDev* __restrict__ hf,
                                                   const NDFrontDev* __restrict__ fr,
                                                   const int* __restrict__ children,
                                                   const long long* __restrict__ child_map_off,
                                                   const int* __restrict__ maps, cd* __restrict__ Fp) {
  __shared__ int s_r[EXT_R], s_c[256];
  const NDFrontDev f = hf[blockIdx.y];
  const int nc = (f.nF + 255) / 256, t = threadIdx.x;
  const int i0 = (int)blockIdx.x / nc * EXT_R, j0 = (int)blockIdx.x % nc * 256;
  if (i0 >= f.nF) return;
  cd acc[EXT_R];
#pragma unroll
  for (int r = 0; r < EXT_R; ++r) acc[r] = mk(0.0, 0.0);
  for (int q = 0; q < f.nchild; ++q) {
    const NDFrontDev fc = fr[children[f.child_off + q]];
    const int* __restrict__ mp = maps + child_map_off[f.child_off + q];
    s_c[t] = -1;
    if (t < EXT_R) s_r[t] = -1;
    __syncthreads();
    for (int k = t; k < fc.nB; k += 256) {
      const int m = mp[k];
      if (m >= i0 && m < i0 + EXT_R) s_r[m - i0] = k;
      if (m >= j0 && m < j0 + 256) s_c[m - j0] = k;
    }
    __syncthreads();
    const int kc = s_c[t];
    const cd* __restrict__ Fc = Fp + fc.F_off + (long long)fc.nS * fc.nF + fc.nS + max(kc, 0);
    // 8 rows' loads in flight before any is added
#pragma unroll
    for (int r = 0; r < EXT_R; r += 8) {
      cd v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int kr = __builtin_amdgcn_readfirstlane(s_r[r + u]);
        v[u] = mk(0.0, 0.0);
        if (kr >= 0)
          if (kc >= 0) v[u] = Fc[(long long)kr * fc.nF];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[r + u] += v[u];
    }
    __syncthreads();
  }
  cd* __restrict__ F = Fp + f.F_off + (long long)i0 * f.nF + j0 + t;
  if (j0 + t < f.nF)
#pragma unroll
    for (int r = 0; r < EXT_R; ++r)
      if (i0 + r < f.nF) F[(long long)r * f.nF] = acc[r];
}

// ----------------------------------------------------------------- inversion of A ----
// one front's inversion: the two copies of A, its pivot maps and the window in work
struct InvFront {
  int nS, nwin, w0, wn;      // window rows and columns [w0, w0 + wn); wn <= 0: nothing to do
  cd *q0, *q1;
  int ld0, ld1;
  int *pm, *ip;
  __device__ __forceinline__ cd* q(int par) const { return par ? q1 : q0; }
  __device__ __forceinline__ long long ld(int par) const { return par ? ld1 : ld0; }
};
__device__ __forceinline__ InvFront inv_front(const NDInv& v, int y, int w) {
  const NDFrontDev f = v.hf[y];
  InvFront a;
  a.nS = f.nS;
  a.nwin = win_count(f.nS, v.win);
  const int wsz = win_size(f.nS, v.win);
  a.w0 = w * wsz;
  a.wn = w < a.nwin ? min(wsz, f.nS - a.w0) : 0;
  a.q0 = v.F + f.F_off;
  a.q1 = v.G + v.goff[y];
  a.ld0 = f.nF;
  a.ld1 = f.nS;
  a.pm = v.pm + f.perm_off;
  a.ip = v.ip + f.perm_off;
  return a;
}
__device__ __forceinline__ int steps_of(int n, int step) { return (n + step - 1) / step; }

template <int CTRL, int RMASK>
__device__ __forceinline__ unsigned dpp_umax(unsigned v) {
  return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, RMASK, 0xf, false));
}
// largest of the 64 lanes' values (pair and quad swaps, row mirrors, row broadcasts)
__device__ __forceinline__ unsigned wave_umax(unsigned v) {
  v = dpp_umax<0xB1, 0xf>(v);
  v = dpp_umax<0x4E, 0xf>(v);
  v = dpp_umax<0x141, 0xf>(v);
  v = dpp_umax<0x140, 0xf>(v);
  v = dpp_umax<0x142, 0xa>(v);
  v = dpp_umax<0x143, 0xc>(v);
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// a - b c in four fused multiply-adds
__device__ __forceinline__ cd csubmul(cd a, cd b, cd c) {
  return mk(fma(b.y, c.y, fma(-b.x, c.x, a.x)), fma(-b.y, c.x, fma(-b.x, c.y, a.y)));
}

// lane L (of each row of 16 lanes)'s v
template <int L>
__device__ __forceinline__ cd row_cd(cd v) {
  const double x = __builtin_amdgcn_update_dpp(0.0, v.x, 0x150 + L, 0xf, 0xf, true);
  const double y = __builtin_amdgcn_update_dpp(0.0, v.y, 0x150 + L, 0xf, 0xf, true);
  return mk(x, y);
}
// slots [J, J1) of a panel's rows less ck times the pivot row's entries (lane l of rl: slot l);
// ROT: slot j takes what is left of slot j + 1
template <int ROT, int J, int J1, int KS, int R>
__device__ __forceinline__ void panel_update(cd (&a)[R][KS], const cd (&ck)[R], cd rl) {
  if constexpr (J < J1) {
    const cd rj = row_cd<J + ROT>(rl);
#pragma unroll
    for (int r = 0; r < R; ++r) a[r][J] = csubmul(a[r][J + ROT], ck[r], rj);
    panel_update<ROT, J + 1, J1, KS, R>(a, ck, rl);
  }
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (N > 0) {
    static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>());
  }
}

// A row's key for the pivot search: the leading bits of |Q[i][k]|^2 (a positive double's bits
// order as its value) with the row in the last B (10 up to 1024 rows), lower rows first among
// equals.  The chosen pivot is within 2^(B - 20) of the largest in |.|^2.  Zero and NaN
// come last, but before exchanged rows (key 0): the one row that is left is found even if it is the
// last one and holds no pivot.
template <int B>
__device__ __forceinline__ unsigned pivot_key(cd a, bool open, int row) {
  constexpr unsigned ROWS = 1u << B;
  const double v = abs2(a);
  const unsigned hb = v >= 0.0 ? (unsigned)__double2hiint(v) & ~(ROWS - 1) : 0u;
  return open ? max(hb, ROWS) | (ROWS - 1 - (unsigned)row) : 0u;
}

// Panel [w0 + k0, + KB) of the window's rows, one work-group of NT threads per front.  The
// threads are Q groups of NR: group q owns the columns q, q + Q, ... (KS = KB / Q of them) and
// its thread t the rows t + r NR, r < R, with those entries in registers.  Bound by the chain
// of its pivots, each of them
//   the new column's keys and, by DPP, the wave's best (the group that owns the column, while
//   the others still update theirs), its entries into LDS;  barrier;
//   the pivot row, KS entries by each of its Q threads, into LDS;  barrier;
//   the rank-1 update, the next pivot's column first.
// Q groups: the rows of a small front fill one wave per 64, so that the update and the row's way
// through LDS (24 cycles per entry of a single lane) would run on one SIMD of four; over more
// rows the waves suffice and Q is 1.  The division of a thread's own candidate and the search
// stand before the first barrier, which the other columns' update shares; the pivot row
// reaches the update by DPP.  Without row swaps no other row is exchanged.  The column loop
// stays rolled but for one pivot of each group (unrolled it overflows the instruction cache),
// so the entries are kept rotated: after m such rounds slot j holds the group's column
// (m + j) mod KS.
// Rows pass through LDS 8 columns (a cache line) at a time on their way in and out: taken
// directly, every 16-byte access of a wave would touch 64 lines.
template <int KB, int Q, int R, int NT>
__global__ void __launch_bounds__(NT) k_inv_panel(NDInv v, int w, int k0, int par) {
  constexpr int NR = NT / Q, KS = KB / Q, GW = NR / 64, CB = 8, CQ = CB / Q, LS = CB + 1;
  constexpr int KEY = NR * R > 1024 ? 11 : 10;
  static_assert(NR % 64 == 0 && CB % Q == 0 && KS >= 2 && KS <= 16 && (KS & (KS - 1)) == 0, "panel split");
  __shared__ cd s_row[KB];                 // the pivot row, by group and slot
  __shared__ unsigned s_key[GW];
  __shared__ int s_piv[KB];
  __shared__ cd s_t[NR * LS];
  static_assert(R <= LS, "the column fits the staging buffer");
  cd* s_col = s_t;                         // the pivot column, by row
  const InvFront f = inv_front(v, blockIdx.x, w);
  if (k0 >= f.wn) return;
  const int kbb = min(KB, f.wn - k0), t = threadIdx.x, lane = t & 63;
  const int q = __builtin_amdgcn_readfirstlane(t / NR), tr = t - q * NR;
  const cd* __restrict__ src = f.q(par) + (long long)f.w0 * f.ld(par) + f.w0 + k0;
  cd* __restrict__ dst = f.q(par ^ 1) + (long long)f.w0 * f.ld(par ^ 1) + f.w0 + k0;
  const unsigned ls = (unsigned)f.ld(par), ldd = (unsigned)f.ld(par ^ 1);
  int bad = 0;
  cd a[R][KS];
  bool open[R];
  // entry (row e / 8, column e % 8) of a pass of NR rows and 8 columns, e = t + NT u
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < KS; c += CQ)
#pragma unroll
      for (int u = 0; u < CQ; ++u) {
        const int e = t + NT * u;
        // byte offsets of a window stay far below 4 GB (at most 1152 rows)
        const unsigned off = 16u * ((unsigned)min(r * NR + e / CB, f.wn - 1) * ls + min(c * Q + e % CB, kbb - 1));
        a[r][c + u] = *(const cd*)((const char*)src + off);
      }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = r * NR + tr;
    open[r] = i < f.wn && f.ip[f.w0 + min(i, f.wn - 1)] < 0;
#pragma unroll
    for (int c = 0; c < KS; c += CQ) {
      __syncthreads();
#pragma unroll
      for (int u = 0; u < CQ; ++u) {
        const int e = t + NT * u;
        s_t[e / CB * LS + e % CB] = a[r][c + u];
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < CQ; ++u) a[r][c + u] = s_t[tr * LS + q + Q * u];
    }
  }
  // slot 0 into LDS; the wave's best key; the reciprocal of this thread's best row in it (zero
  // or NaN: ok is 0 and the pivot taken as 1)
  cd ri = mk(1.0, 0.0);
  bool ok = true;
  auto search = [&]() {
    cd c0 = a[0][0];
    unsigned key = pivot_key<KEY>(a[0][0], open[0], tr);
    if (Q > 1) s_col[tr] = a[0][0];
#pragma unroll
    for (int r = 1; r < R; ++r) {
      const unsigned kr = pivot_key<KEY>(a[r][0], open[r], r * NR + tr);
      const bool up = kr > key;
      c0.x = up ? a[r][0].x : c0.x;
      c0.y = up ? a[r][0].y : c0.y;
      key = up ? kr : key;
      if (Q > 1) s_col[r * NR + tr] = a[r][0];
    }
    const unsigned wk = wave_umax(key);
    if (lane == 0) s_key[tr >> 6] = wk;
    const double d = abs2(c0), di = 1.0 / d;
    ok = d > 0.0;
    ri = ok ? mk(c0.x * di, -c0.y * di) : mk(1.0, 0.0);
    asm("" : "+v"(ri.x), "+v"(ri.y));      // divided here, not by the winner after the barrier
  };
  __syncthreads();
  if (q == 0) search();
  __syncthreads();
  // one pivot of each group in turn, each group's in its slot 0; the last one's update also
  // rotates the slots
  for (int k1 = 0; k1 < kbb; k1 += Q)
    static_for<Q>([&](auto qc) {
      constexpr int QO = decltype(qc)::value, LAST = QO == Q - 1;
      const int kk = k1 + QO;
      if (kk >= kbb) return;               // uniform: a last panel of fewer columns
      unsigned bk = s_key[0];
#pragma unroll
      for (int g = 1; g < GW; ++g) bk = max(bk, s_key[g]);
      cd ck[R];
#pragma unroll
      for (int r = 0; r < R; ++r) ck[r] = Q > 1 ? s_col[r * NR + tr] : mk(a[r][0].x, a[r][0].y);
      constexpr int RM = (1 << KEY) - 1;
      const int p = RM - (__builtin_amdgcn_readfirstlane((int)bk) & RM);   // the pivot row, from w0
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r * NR + tr == p) {
#pragma unroll
          for (int j = 1; j < KS; ++j) s_row[q * KS + j] = a[r][j];
          if (q == QO) {
            s_row[q * KS] = ri;                        // the reciprocal of the pivot
            if (!ok) bad = 1;                          // a zero or NaN pivot is recorded
            s_piv[kk] = p;
          } else {
            s_row[q * KS] = a[r][0];
          }
          // the pivot row becomes -row / pivot, 1 / pivot: ck below is 1 / pivot for it
          open[r] = false;
#pragma unroll
          for (int j = 0; j < KS; ++j) a[r][j] = mk(0.0, 0.0);
        }
      __syncthreads();
      const cd rl = s_row[q * KS + (t & (KS - 1))];
      const cd inv = s_row[QO * KS];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        ck[r] = ck[r] * inv;
        if (r * NR + tr == p) ck[r] = inv;
      }
      // the pivot's column becomes ck; the next pivot's column first, so that its search and
      // division overlap the other columns
      cd s0[R];
      const cd r0 = row_cd<0>(rl);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        s0[r] = csubmul(a[r][0], ck[r], r0);
        if (q == QO) s0[r] = ck[r];
      }
      if constexpr (LAST) {
        panel_update<1, 0, 1, KS, R>(a, ck, rl);
        if (q == 0) search();
        panel_update<1, 1, KS - 1, KS, R>(a, ck, rl);
#pragma unroll
        for (int r = 0; r < R; ++r) a[r][KS - 1] = s0[r];
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) a[r][0] = s0[r];
        if (q == QO + 1) search();
        panel_update<0, 1, KS, KS, R>(a, ck, rl);
      }
      __syncthreads();
    });
  if (bad) atomicOr(v.err, f.nwin > 1 ? ND_GROWTH : ND_SINGULAR);
  if (t < kbb) {
    f.pm[f.w0 + k0 + t] = f.w0 + s_piv[t];
    f.ip[f.w0 + s_piv[t]] = f.w0 + k0 + t;
  }
  // slot j of group g now holds its column (m + j) mod KS, after m rotations
  const int m = kbb / Q;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < KS; c += CQ) {
      __syncthreads();
#pragma unroll
      for (int u = 0; u < CQ; ++u) s_t[tr * LS + q + Q * u] = a[r][c + u];
      __syncthreads();
#pragma unroll
      for (int u = 0; u < CQ; ++u) {
        const int e = t + NT * u, i = r * NR + e / CB;
        const int col = e % Q + Q * ((m + c + e % CB / Q) % KS);
        if (i < f.wn && col < kbb) *(cd*)((char*)dst + 16u * ((unsigned)i * ldd + col)) = s_t[e / CB * LS + e % CB];
      }
    }
}

// A panel of any number of rows, one work-group per front, 8 threads per row: the panel is
// copied and then exchanged in place, every pivot from all open rows; the threads of the next
// pivot's column search it as they write it.  Taken where a window's own rows hold no good
// pivots, so it is kept simple: bound by one CU's reads and writes of the panel per pivot, hence 8
// columns (set-up of 256^3, 4225 rows: 96 ms, 240 with this pass, 287 with 16 columns; 160^3:
// 15.9, 34.9, 42.1).
#define WIDE_KB 8
__global__ void __launch_bounds__(1024) k_inv_panel_wide(NDInv v, int w, int k0, int par) {
  constexpr int KB = WIDE_KB, NT = 1024, NW = NT / 64;
  __shared__ cd s_row[KB];
  __shared__ double s_v[NW];
  __shared__ int s_i[NW];
  const InvFront f = inv_front(v, blockIdx.x, w);
  if (k0 >= f.wn) return;
  const int kbb = min(KB, f.wn - k0), t = threadIdx.x, lane = t & 63, c = t % KB;
  const bool on = c < kbb;
  const long long ls = f.ld(par), ld = f.ld(par ^ 1);
  const cd* __restrict__ src = f.q(par) + f.w0 * ls + f.w0 + k0 + (on ? c : 0);
  cd* dst = f.q(par ^ 1) + f.w0 * ld + f.w0 + k0 + (on ? c : 0);
  int* ip = f.ip + f.w0;
  // this thread's candidate of the column in search: the largest |entry|^2 among the open rows
  // (zero and NaN: 0), the lower row among equals
  double bv = -1.0;
  int bi = f.wn - 1;
  auto offer = [&](cd a, int i, int done) {
    const double q = abs2(a), x = q > 0.0 ? q : 0.0;
    if (x > bv && done < 0) {
      bv = x;
      bi = i;
    }
  };
  // RU rows' loads in flight (past the last row: repeated, not used)
  constexpr int RU = 8, RS = NT / KB;
  for (int i0 = t / KB; i0 < f.wn; i0 += RU * RS) {
    cd x[RU];
    int done[RU];
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int i = min(i0 + u * RS, f.wn - 1);
      x[u] = src[i * ls];
      done[u] = ip[i];
    }
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      const int i = i0 + u * RS;
      if (i >= f.wn) break;
      if (on) dst[i * ld] = x[u];
      if (c == 0) offer(x[u], i, done[u]);
    }
  }
  int bad = 0;
  for (int kk = 0; kk < kbb; ++kk) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ov = __shfl_xor(bv, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (ov > bv || (ov == bv && oi < bi)) {
        bv = ov;
        bi = oi;
      }
    }
    if (lane == 0) {
      s_v[t >> 6] = bv;
      s_i[t >> 6] = bi;
    }
    __syncthreads();
    bv = s_v[0];
    bi = s_i[0];
    for (int g = 1; g < NW; ++g)
      if (s_v[g] > bv || (s_v[g] == bv && s_i[g] < bi)) {
        bv = s_v[g];
        bi = s_i[g];
      }
    const int p = bi;
    const bool ok = bv > 0.0;
    if (!ok) bad = 1;
    if (t < kbb) s_row[t] = dst[p * ld];
    if (t == 0) {
      f.pm[f.w0 + k0 + kk] = f.w0 + p;
      ip[p] = f.w0 + k0 + kk;
    }
    __syncthreads();
    const cd inv = ok ? cdiv(mk(1.0, 0.0), s_row[kk]) : mk(1.0, 0.0);
    const cd rc = on ? s_row[c] : mk(0.0, 0.0);
    bv = -1.0;
    bi = f.wn - 1;
    for (int i0 = t / KB; i0 < f.wn; i0 += RU * RS) {
      cd x[RU];
      int done[RU];
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const int i = min(i0 + u * RS, f.wn - 1);
        x[u] = dst[i * ld];
        done[u] = ip[i];
      }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const int i = i0 + u * RS;
        const cd xk = mk(__shfl(x[u].x, (lane & ~(KB - 1)) + kk, 64), __shfl(x[u].y, (lane & ~(KB - 1)) + kk, 64));
        const cd ck = i == p ? inv : xk * inv;
        const cd y = c == kk ? ck : csubmul(i == p ? mk(0.0, 0.0) : x[u], ck, rc);
        if (i >= f.wn || !on) continue;
        dst[i * ld] = y;
        if (c == kk + 1) offer(y, i, done[u]);
      }
    }
    __syncthreads();
  }
  if (bad && t == 0) atomicOr(v.err, f.nwin > 1 ? ND_GROWTH : ND_SINGULAR);
}

// ------------------------------------------------------ complex FP64 products (MFMA) ----
// C tile of GT x GT (64 or 32), K deep: a work-group of 4 wavefronts, each a quarter of 2 x 2
// or 1 x 1 blocks of the 16 x 16 x 4 FP64 MFMA, real and imaginary parts accumulated separately:
//   Cr += Ar Br - Ai Bi,  Ci += Ar Bi + Ai Br  (four real MFMAs per k group).
// MFMA lane layout: A[m][k] from lane m + 16 k, B[k][n] from lane n + 16 k, and lane l
// holds D[l / 16 + 4 i][l % 16], i < 4.  Panels of A and B pass through LDS, 16 k at a time;
// the next 16 are loaded into registers while the matrix cores work on these.
#define GK 16
typedef double mfma_d4 __attribute__((ext_vector_type(4)));
template <int GT>
struct GemmLds {
  cd a[GK][GT + 1], b[GK][GT + 1];
};
template <int GT>
struct GemmAcc {
  mfma_d4 r[GT / 32][GT / 32], i[GT / 32][GT / 32];
};
// la(row, k) and lb(k, col): entries of the tile's operands; both are called for every
// row and column of the tile and every k < K rounded up to 16, and return 0 outside
template <int GT, class LA, class LB>
__device__ __forceinline__ void gemm_tile(GemmLds<GT>& s, int K, GemmAcc<GT>& acc, LA la, LB lb) {
  constexpr int NQ = GT / 32;            // 16 x 16 blocks of a wavefront per axis
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wr = (wv >> 1) * (GT / 2), wc = (wv & 1) * (GT / 2), lm = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int a = 0; a < NQ; ++a)
#pragma unroll
    for (int b = 0; b < NQ; ++b) {
      acc.r[a][b] = mfma_d4{0.0, 0.0, 0.0, 0.0};
      acc.i[a][b] = mfma_d4{0.0, 0.0, 0.0, 0.0};
    }
  constexpr int NLD = GK * GT / 256;
  cd ra[NLD], rb[NLD];
  auto load = [&](int kk0) {
#pragma unroll
    for (int it = 0; it < NLD; ++it) {
      const int p = (int)threadIdx.x + 256 * it;
      ra[it] = la(p / GK, kk0 + p % GK);             // consecutive threads along a row of A
      rb[it] = lb(kk0 + p / GT, p % GT);             // consecutive threads along a row of B
    }
  };
  load(0);
  for (int kk0 = 0; kk0 < K; kk0 += GK) {
#pragma unroll
    for (int it = 0; it < NLD; ++it) {
      const int p = (int)threadIdx.x + 256 * it;
      s.a[p % GK][p / GK] = ra[it];
      s.b[p / GT][p % GT] = rb[it];
    }
    __syncthreads();
    if (kk0 + GK < K) load(kk0 + GK);
#pragma unroll
    for (int k4 = 0; k4 < GK; k4 += 4) {
      cd av[NQ], bv[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        av[q] = s.a[k4 + lk][wr + 16 * q + lm];
        bv[q] = s.b[k4 + lk][wc + 16 * q + lm];
      }
      // the four products of a block go to two accumulators: issue them in rounds over the
      // accumulators, so that no MFMA waits for the one just before it
#pragma unroll
      for (int qa = 0; qa < NQ; ++qa)
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
          acc.r[qa][qb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[qa].x, bv[qb].x, acc.r[qa][qb], 0, 0, 0);
          acc.i[qa][qb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[qa].x, bv[qb].y, acc.i[qa][qb], 0, 0, 0);
        }
#pragma unroll
      for (int qa = 0; qa < NQ; ++qa)
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
          acc.r[qa][qb] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[qa].y, bv[qb].y, acc.r[qa][qb], 0, 0, 0);
          acc.i[qa][qb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[qa].y, bv[qb].x, acc.i[qa][qb], 0, 0, 0);
        }
    }
    __syncthreads();
  }
}
// st(row, col, value, old) for the tile's entries, old = ld(row, col); the loads of a 16-column
// strip are issued together (ld clamps its indices, so they stand under no branch)
template <int GT, class LD, class ST>
__device__ __forceinline__ void gemm_store(const GemmAcc<GT>& acc, LD ld, ST st) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int wr = (wv >> 1) * (GT / 2), wc = (wv & 1) * (GT / 2), lm = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int qb = 0; qb < GT / 32; ++qb) {
    cd o[GT / 32][4];
#pragma unroll
    for (int qa = 0; qa < GT / 32; ++qa)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[qa][i] = ld(wr + 16 * qa + lk + 4 * i, wc + 16 * qb + lm);
#pragma unroll
    for (int qa = 0; qa < GT / 32; ++qa)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        st(wr + 16 * qa + lk + 4 * i, wc + 16 * qb + lm, mk(acc.r[qa][qb][i], acc.i[qa][qb][i]), o[qa][i]);
  }
}
__device__ __forceinline__ cd no_old(int, int) { return mk(0.0, 0.0); }
#define GEMM_KERNEL __global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3)))

// Columns outside a run K = [w0 + k0, + kw) of pivots (clipped to the window).  cmode 0: the
// other columns of the block [w0 + b0, + bw) (after a panel), 1: of the window (after a
// block), over the window's rows; 2: of A (after a window), over all rows.  The run's own
// entries Q'[:, K] are in copy pa, Q0 in copy par, and the result goes to copy par ^ 1.
// pa < 0: a block's entries, whose copy depends on its number of panels of kb columns; where
// that is copy par, they are copied over.
template <int GT>
GEMM_KERNEL k_inv_gemm(NDInv v, int w, int k0, int kw, int cmode, int b0, int bw, int par, int pa, int kb) {
  const InvFront f = inv_front(v, blockIdx.y, w);
  if (k0 >= f.wn || (cmode == 2 && f.nwin == 1)) return;
  const int kn = min(kw, f.wn - k0);
  const int r0 = cmode == 2 ? 0 : f.w0, M = cmode == 2 ? f.nS : f.wn;
  const int c0 = cmode == 0 ? f.w0 + b0 : cmode == 1 ? f.w0 : 0;
  const int nc = cmode == 0 ? min(bw, f.wn - b0) : cmode == 1 ? f.wn : f.nS;
  if (nc == kn && pa >= 0) return;
  const int tilesN = steps_of(nc, GT), tilesM = steps_of(M, GT);
  if ((int)blockIdx.x >= tilesM * tilesN) return;
  const int tm = blockIdx.x / tilesN * GT, tn = blockIdx.x % tilesN * GT;
  if (pa < 0) pa = par ^ (steps_of(kn, kb) & 1);
  const int K0 = f.w0 + k0, po = par ^ 1;
  const cd* __restrict__ A = f.q(pa) + (long long)r0 * f.ld(pa) + K0;
  const cd* __restrict__ Q0 = f.q(par);
  cd* __restrict__ O = f.q(po);
  const long long la = f.ld(pa), l0 = f.ld(par), lo = f.ld(po);
  const int* __restrict__ pm = f.pm + K0;
  const bool inside = c0 + tn >= K0 && c0 + min(tn + GT, nc) <= K0 + kn;   // only columns of K
  if (inside && pa == po) return;
  __shared__ GemmLds<GT> s;
  GemmAcc<GT> acc;
  if (!inside)
    gemm_tile<GT>(
        s, kn, acc,
        [&](int r, int k) { return tm + r < M && k < kn ? A[(tm + r) * la + k] : mk(0.0, 0.0); },
        [&](int k, int c) {
          return tn + c < nc && k < kn ? Q0[pm[k] * l0 + c0 + tn + c] : mk(0.0, 0.0);
        });
  gemm_store<GT>(
      acc,
      [&](int r, int c) {
        // old entry; 0 in the run's pivot rows.  Columns of K: the entry to copy
        const int i = r0 + min(tm + r, M - 1), j = c0 + min(tn + c, nc - 1);
        const bool own = j >= K0 && j < K0 + kn;
        const cd* __restrict__ src = own ? A + (i - r0) * la + (j - K0) : Q0 + i * l0 + j;
        const int q = f.ip[i];
        const cd o = *src;
        return !own && q >= K0 && q < K0 + kn ? mk(0.0, 0.0) : o;
      },
      [&](int r, int c, cd x, cd o) {
        const int i = r0 + tm + r, j = c0 + tn + c;
        if (tm + r >= M || tn + c >= nc) return;
        if (j >= K0 && j < K0 + kn) {
          if (pa != po) O[i * lo + j] = o;
        } else {
          O[i * lo + j] = o - x;
        }
      });
}

// a finished window's columns in the rows outside it: Q'[i, K] = Q0[i, K] Q'[pm[K], K]; the
// window's own rows are copied where its result is not in copy par ^ 1 already
template <int GT>
GEMM_KERNEL k_inv_outer(NDInv v, int w, int par, int kout) {
  const InvFront f = inv_front(v, blockIdx.y, w);
  if (f.nwin == 1 || f.wn <= 0) return;
  const int M = f.nS, N = f.wn;
  const int tilesN = steps_of(N, GT), tilesM = steps_of(M, GT);
  if ((int)blockIdx.x >= tilesM * tilesN) return;
  const int tm = blockIdx.x / tilesN * GT, tn = blockIdx.x % tilesN * GT;
  const int po = par ^ 1, pr = par ^ (steps_of(f.wn, kout) & 1);
  const cd* __restrict__ A = f.q(par) + f.w0;
  const cd* __restrict__ B = f.q(pr) + f.w0;
  cd* __restrict__ O = f.q(po) + f.w0;
  const long long la = f.ld(par), lb = f.ld(pr), lo = f.ld(po);
  const int* __restrict__ pm = f.pm + f.w0;
  const bool inside = tm >= f.w0 && min(tm + GT, M) <= f.w0 + f.wn;
  if (inside && pr == po) return;
  __shared__ GemmLds<GT> s;
  GemmAcc<GT> acc;
  if (!inside)
    gemm_tile<GT>(
        s, N, acc, [&](int r, int k) { return tm + r < M && k < N ? A[(tm + r) * la + k] : mk(0.0, 0.0); },
        [&](int k, int c) { return tn + c < N && k < N ? B[pm[k] * lb + tn + c] : mk(0.0, 0.0); });
  int big = 0;
  gemm_store<GT>(acc, no_old, [&](int r, int c, cd x, cd) {
    const int i = tm + r, j = tn + c;
    if (i >= M || j >= N) return;
    if (i >= f.w0 && i < f.w0 + f.wn) {
      if (pr != po) O[i * lo + j] = B[i * lb + j];
    } else {
      O[i * lo + j] = x;
      if (f.ip[i] < 0 && !(abs2(x) <= v.growth2)) big = 1;      // (NaN counts as large)
    }
  });
  if (big) atomicOr(v.err, ND_GROWTH);
}

// the copy that holds a front's exchanged A once every window is done
__device__ __forceinline__ int final_par(const InvFront& f, int kout) {
  return (f.nwin > 1 ? f.nwin : steps_of(f.nS, kout)) & 1;
}

// A^-1 in natural order, N[k][m] = Q[pm[k]][ip[m]], into the copy that Q does not occupy, and
// into the upper block of L (column major, in the substitution's precision; a 32 x 32 tile
// passes through LDS so that both are written in runs)
template <typename C>
__global__ void __launch_bounds__(256) k_inv_final(NDInv v, int kout, C* __restrict__ Lp) {
  const NDFrontDev fr = v.hf[blockIdx.y];
  const InvFront f = inv_front(v, blockIdx.y, 0);
  const int nt = steps_of(f.nS, 32);
  if ((int)blockIdx.x >= nt * nt) return;
  const int k0 = blockIdx.x / nt * 32, m0 = blockIdx.x % nt * 32;
  const int pf = final_par(f, kout), tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const cd* __restrict__ Q = f.q(pf);
  cd* __restrict__ N = f.q(pf ^ 1);
  const long long lq = f.ld(pf), ln = f.ld(pf ^ 1);
  __shared__ C t[32][33];
  const int q = f.ip[min(m0 + tx, f.nS - 1)];
  cd x[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) x[u] = Q[f.pm[min(k0 + ty + 8 * u, f.nS - 1)] * lq + q];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int k = k0 + ty + 8 * u;
    if (k < f.nS && m0 + tx < f.nS) N[k * ln + m0 + tx] = x[u];
    t[ty + 8 * u][tx] = conv<C>::from(x[u]);
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int m = m0 + ty + 8 * u, k = k0 + tx;
    if (k < f.nS && m < f.nS) Lp[fr.L_off + (long long)m * fr.ldL + k] = t[tx][ty + 8 * u];
  }
}

// W = -A^-1 B: in FP64 for the Schur product (T, nS x nB row major), in the substitution's
// precision into W and (SYM) as C A^-1 = (A^-1 B)^T into the
// lower block of L
template <int GT, typename C, int SYM>
GEMM_KERNEL k_nd_w(NDInv v, const long long* __restrict__ toff, int kout, cd* __restrict__ T, C* __restrict__ Lp,
                   C* __restrict__ Wp) {
  const NDFrontDev fr = v.hf[blockIdx.y];
  const int nS = fr.nS, nB = fr.nB;
  const int tilesN = steps_of(nB, GT), tilesM = steps_of(nS, GT);
  if ((int)blockIdx.x >= tilesM * tilesN) return;
  const int tm = blockIdx.x / tilesN * GT, tn = blockIdx.x % tilesN * GT;
  const InvFront f = inv_front(v, blockIdx.y, 0);
  const int pn = final_par(f, kout) ^ 1;
  const cd* __restrict__ N = f.q(pn);
  const cd* __restrict__ B = v.F + fr.F_off + nS;
  const long long ln = f.ld(pn), lf = fr.nF;
  cd* __restrict__ Tt = T + toff[blockIdx.y];
  __shared__ GemmLds<GT> s;
  GemmAcc<GT> acc;
  gemm_tile<GT>(
      s, nS, acc, [&](int r, int k) { return tm + r < nS && k < nS ? N[(tm + r) * ln + k] : mk(0.0, 0.0); },
      [&](int k, int c) { return tn + c < nB && k < nS ? B[k * lf + tn + c] : mk(0.0, 0.0); });
  gemm_store<GT>(acc, no_old, [&](int r, int c, cd x, cd) {
    const int k = tm + r, j = tn + c;
    if (k >= nS || j >= nB) return;
    Tt[(long long)k * nB + j] = -x;
    Wp[fr.W_off + (long long)j * fr.ldW + k] = conv<C>::from(-x);
    if (SYM) Lp[fr.L_off + (long long)k * fr.ldL + nS + j] = conv<C>::from(x);
  });
}

// C A^-1 into the lower block of L (FP64 factors)
template <int GT, typename C>
GEMM_KERNEL k_nd_x(NDInv v, int kout, C* __restrict__ Lp) {
  const NDFrontDev fr = v.hf[blockIdx.y];
  const int nS = fr.nS, nB = fr.nB;
  const int tilesN = steps_of(nS, GT), tilesM = steps_of(nB, GT);
  if ((int)blockIdx.x >= tilesM * tilesN) return;
  const int tm = blockIdx.x / tilesN * GT, tn = blockIdx.x % tilesN * GT;
  const InvFront f = inv_front(v, blockIdx.y, 0);
  const int pn = final_par(f, kout) ^ 1;
  const cd* __restrict__ N = f.q(pn);
  const cd* __restrict__ Cb = v.F + fr.F_off + (long long)nS * fr.nF;
  const long long ln = f.ld(pn), lf = fr.nF;
  __shared__ GemmLds<GT> s;
  GemmAcc<GT> acc;
  gemm_tile<GT>(
      s, nS, acc, [&](int r, int k) { return tm + r < nB && k < nS ? Cb[(tm + r) * lf + k] : mk(0.0, 0.0); },
      [&](int k, int c) { return tn + c < nS && k < nS ? N[k * ln + tn + c] : mk(0.0, 0.0); });
  gemm_store<GT>(acc, no_old, [&](int r, int c, cd x, cd) {
    if (tm + r < nB && tn + c < nS)
      Lp[fr.L_off + (long long)(tn + c) * fr.ldL + nS + tm + r] = conv<C>::from(x);
  });
}

// D += C W, the front's Schur complement; SYM: the tiles on and
// below the diagonal, the others being their mirror images
template <int GT, int SYM>
GEMM_KERNEL k_nd_schur(NDInv v, const long long* __restrict__ toff, const cd* __restrict__ T) {
  const NDFrontDev fr = v.hf[blockIdx.y];
  const int nS = fr.nS, nB = fr.nB, nt = steps_of(nB, GT);
  int bm, bn;
  if (SYM) {
    // tile x of the lower triangle, row by row
    bm = (int)((sqrt(8.0 * blockIdx.x + 1.0) - 1.0) * 0.5);
    while ((bm + 1) * (bm + 2) / 2 <= (int)blockIdx.x) ++bm;
    while (bm * (bm + 1) / 2 > (int)blockIdx.x) --bm;
    bn = (int)blockIdx.x - bm * (bm + 1) / 2;
  } else {
    bm = blockIdx.x / max(nt, 1);
    bn = blockIdx.x % max(nt, 1);
  }
  if (bm >= nt) return;
  const int tm = bm * GT, tn = bn * GT;
  cd* __restrict__ F = v.F + fr.F_off + (long long)nS * fr.nF;
  const cd* __restrict__ Tt = T + toff[blockIdx.y];
  const long long lf = fr.nF;
  __shared__ GemmLds<GT> s;
  GemmAcc<GT> acc;
  gemm_tile<GT>(
      s, nS, acc, [&](int r, int k) { return tm + r < nB && k < nS ? F[(tm + r) * lf + k] : mk(0.0, 0.0); },
      [&](int k, int c) { return tn + c < nB && k < nS ? Tt[(long long)k * nB + tn + c] : mk(0.0, 0.0); });
  gemm_store<GT>(acc, [&](int r, int c) { return F[min(tm + r, nB - 1) * lf + nS + min(tn + c, nB - 1)]; },
                 [&](int r, int c, cd x, cd o) {
    const int i = tm + r, j = tn + c;
    if (i >= nB || j >= nB) return;
    const cd d = o + x;
    F[i * lf + nS + j] = d;
    if (SYM && bm != bn) F[j * lf + nS + i] = d;
  });
}

__global__ void k_fill_int(int* __restrict__ p, long long n, int x) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    p[i] = x;
}

// ------------------------------------------------------------- launchers ----
static unsigned blocks256(long long n, unsigned cap) {
  return (unsigned)std::min<long long>(cap, std::max<long long>(1, (n + 255) / 256));
}
void nd_fill_int(int* p, long long n, int x, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_int, dim3(blocks256(n, 1024)), dim3(256), 0, s, p, n, x);
}
void nd_assemble(const NDInv& v, int nids, int max_asm, const NDAsm* asmv, const cd* coef, hipStream_t s) {
  hipLaunchKernelGGL(k_nd_assemble, dim3(blocks256(max_asm, 1024), nids), dim3(256), 0, s, v.hf, asmv, coef, v.F);
}
void nd_extend(const NDInv& v, const NDFrontDev* fr, int nids, int max_nF, const int* children,
               const long long* child_map_off, const int* maps, hipStream_t s) {
  const unsigned tiles = (unsigned)((max_nF + EXT_R - 1) / EXT_R) * ((max_nF + 255) / 256);
  hipLaunchKernelGGL(k_nd_extend, dim3(tiles, nids), dim3(256), 0, s, v.hf, fr, children, child_map_off, maps, v.F);
}

// the most rows of a register panel.  Windows end at 1024, where two threads' rows fit 512 threads;
// three rows per thread take the roots of up to 1100 rows that the default schedule merges in 2D,
// where their windows held no good pivots (about 1080 rows: set-up 3.1 ms, 6.8 with this second
// pass, 13.1 with k_inv_panel_wide; as the only pass 3.8, so the windows come first)
#define REG_ROWS 1152
// columns of a panel over a window of up to rows rows, and its split (k_inv_panel): 32 columns
// while their entries leave a thread at most 16, then 16.  A panel in us, split into 4 / 2
// groups or whole rows per thread: 64 rows 26.6 / 28.8 / 33, 128 rows 31.3 / 35.4 / 36,
// 256 rows 41.4 / 40.2 / 50; of 16 columns over 512 rows, 2 groups / whole rows 22.2 / 21.6,
// over 1024 34.6 / 31.7.  Panels in memory take WIDE_KB.
static int panel_cols(int rows) { return rows <= 256 ? 32 : rows <= REG_ROWS ? 16 : WIDE_KB; }
static void inv_panel(const NDInv& v, int nids, int rows, int w, int k0, int par, hipStream_t s) {
#define PANEL(KB, Q, R, NT) \
  hipLaunchKernelGGL((k_inv_panel<KB, Q, R, NT>), dim3(nids), dim3(NT), 0, s, v, w, k0, par)
  if (rows <= 64)
    PANEL(32, 4, 1, 256);
  else if (rows <= 128)
    PANEL(32, 4, 2, 256);
  else if (rows <= 256)
    PANEL(32, 2, 1, 512);
  else if (rows <= 512)
    PANEL(16, 1, 1, 512);
  else if (rows <= 1024)
    PANEL(16, 1, 2, 512);
  else if (rows <= REG_ROWS)
    PANEL(16, 1, 3, 384);
  else
    hipLaunchKernelGGL(k_inv_panel_wide, dim3(nids), dim3(1024), 0, s, v, w, k0, par);
}
// A product's tiles are 64 x 64, or 32 x 32 where 64 x 64 ones would not give every CU one:
// there the launch lasts as long as one tile (a 16-deep update of 577 columns: 16.3 us with
// 64 x 64 tiles and their old entries loaded one by one, 7.2 us).
static unsigned tiles(int m, int n, int gt) { return (unsigned)(((m + gt - 1) / gt) * ((n + gt - 1) / gt)); }
static bool small_tiles(int m, int n, int nids) { return (long long)tiles(m, n, 64) * nids < 256; }
#define LAUNCH_GEMM(m, n, nids, s, k64, k32, ...)                                                     \
  do {                                                                                                \
    if (small_tiles(m, n, nids))                                                                      \
      hipLaunchKernelGGL((k32), dim3(tiles(m, n, 32), nids), dim3(256), 0, s, __VA_ARGS__);           \
    else                                                                                              \
      hipLaunchKernelGGL((k64), dim3(tiles(m, n, 64), nids), dim3(256), 0, s, __VA_ARGS__);           \
  } while (0)

int nd_invert(const NDInv& v, int nids, int max_nS, int max_wn, int block_cols, hipStream_t s) {
  const int kb = panel_cols(max_wn);
  const int kout = std::max(1, block_cols / kb) * kb;
  const int nwin = win_count(max_nS, v.win);
  for (int w = 0; w < nwin; ++w) {
    for (int b0 = 0, blk = 0; b0 < max_wn; b0 += kout, ++blk) {
      const int cur = (w ^ blk) & 1;            // the copy that holds A before this block
      const int nb = std::min(kout, max_wn - b0);
      for (int k0 = b0, q = 0; k0 < b0 + nb; k0 += kb, ++q) {
        const int par = cur ^ (q & 1);
        inv_panel(v, nids, max_wn, w, k0, par, s);
        if (nb > kb)                             // the block's other panels, earlier ones included
          LAUNCH_GEMM(max_wn, nb, nids, s, k_inv_gemm<64>, k_inv_gemm<32>, v, w, k0, kb, 0, b0, kout, par, par ^ 1,
                      kb);
      }
      if (max_wn > kb)
        LAUNCH_GEMM(max_wn, max_wn, nids, s, k_inv_gemm<64>, k_inv_gemm<32>, v, w, b0, kout, 1, 0, 0, cur, -1, kb);
    }
    if (nwin > 1) {
      const int par = w & 1;
      LAUNCH_GEMM(max_nS, max_wn, nids, s, k_inv_outer<64>, k_inv_outer<32>, v, w, par, kout);
      LAUNCH_GEMM(max_nS, max_nS, nids, s, k_inv_gemm<64>, k_inv_gemm<32>, v, w, 0, max_wn, 2, 0, 0, par, par ^ 1, kb);
    }
  }
  return kout;
}

// FP32 factors (those of a complex symmetric 5/7-point operator) take the products that symmetry
// leaves; FP64 ones take all of them
template <typename C>
void nd_products(const NDInv& v, int nids, int max_nS, int max_nB, int kout, const long long* toff, cd* T, C* Lp,
                 C* Wp, hipStream_t s) {
  constexpr int SYM = sizeof(C) == sizeof(cf);
  const int nt = (max_nS + 31) / 32;
  const cd* Tc = T;
  hipLaunchKernelGGL((k_inv_final<C>), dim3(nt * nt, nids), dim3(256), 0, s, v, kout, Lp);
  if (max_nB == 0) return;
  LAUNCH_GEMM(max_nS, max_nB, nids, s, (k_nd_w<64, C, SYM>), (k_nd_w<32, C, SYM>), v, toff, kout, T, Lp, Wp);
  if constexpr (SYM) {
    const bool small = small_tiles(max_nB, max_nB / 2, nids);
    const int nb = (max_nB + (small ? 31 : 63)) / (small ? 32 : 64);
    if (small)
      hipLaunchKernelGGL((k_nd_schur<32, 1>), dim3(nb * (nb + 1) / 2, nids), dim3(256), 0, s, v, toff, Tc);
    else
      hipLaunchKernelGGL((k_nd_schur<64, 1>), dim3(nb * (nb + 1) / 2, nids), dim3(256), 0, s, v, toff, Tc);
  } else {
    LAUNCH_GEMM(max_nB, max_nS, nids, s, (k_nd_x<64, C>), (k_nd_x<32, C>), v, kout, Lp);
    LAUNCH_GEMM(max_nB, max_nB, nids, s, (k_nd_schur<64, 0>), (k_nd_schur<32, 0>), v, toff, Tc);
  }
}
template void nd_products<cf>(const NDInv&, int, int, int, int, const long long*, cd*, cf*, cf*, hipStream_t);
template void nd_products<cd>(const NDInv&, int, int, int, int, const long long*, cd*, cd*, cd*, hipStream_t);

}  // namespace helm
