// Kernels of the paper's compact fourth-order stack (eqs. 3.1-3.4): its Galerkin
// operators (FP64 set-up) and the steps of its cycle (cycle precision).  The layouts and
// operators are described in wide.h.
//
// The cycle steps are plain one-node-per-thread kernels: every neighbour and coefficient
// load is issued unconditionally (clamped index, zero weight), so a thread waits on one
// batch of loads.  Right-hand sides solved in lock-step are grid y, N entries apart.
#include <stdexcept>

#include "wide.h"

namespace helm {

namespace {

// node coordinates of flat index f
__device__ __forceinline__ void coords(const Geom& g, long long f, int& i0, int& i1, int& i2) {
  node_coords(g, f, i0, i1, i2);
}

// ---------------------------------------------------------------- set-up ----
// Galerkin product Ac = R A P for one coarse node I per wavefront (four per work-group):
//   q(j)      = sum_i R(I, i) A(i, j)            over the fine nodes j that R's row I reaches
//                                                 through A (a box of side 2(a + rin) + 1)
//   Ac(I, J)  = sum_j q(j) P(j, J)                for every coarse J = I + D, |D_a| <= rc
// R(I, i) = prod_a Rt.w[i_a - 2 I_a + Rt.a]; P(j, J) = prod_a 2 Pt.w[j_a - 2 J_a + Pt.a]
// (P = 2^d Pt^T); both truncated at the grid's ends.
//
// Bound by the instructions a wavefront spends per term, most of them index arithmetic: the
// radii are compile-time constants and every node takes the whole box (terms off the grid are
// zero), so that indices divide by constants.  The fine operator is linear in its coefficient
// scalar, A = L - s M diag(m (1 - i sigma)): one launch forms the two products and writes both
// of the set-up's operators, and the FP32 copy of the first.  With run-time radii and a launch per
// operator the 192 x 192 x 72 set-up spent 2 x 1.65 + 0.86 ms here and 0.2 on the copy, the
// 1024^2 one 2 x 0.23 + 0.20; now 1.07 + 0.69 and 0.15 + 0.13.
// The four nodes' results leave through LDS, four nodes (64 bytes of a plane) to a run.
template <int DIM_, int AR_, int RIN_, int BP_, int RC_>
struct GalBox {
  static constexpr int DIM = DIM_, AR = AR_, RIN = RIN_, BP = BP_, RC = RC_;
  static constexpr int S = 2 * (AR + RIN) + 1, S2 = DIM == 3 ? S : 1, W = 2 * RC + 1;
  static constexpr int NQ = S * S * S2, NT = W * S * S2, NU = W * W * S2, NO = W * W * (DIM == 3 ? W : 1);
  static_assert(NU <= NQ && NO <= NT, "passes in place");
};
struct GalArgs {
  Geom gf, gc;
  FineOp op;            // the fine operator's
  const double* m;
  cd sa, sb;
  const cd* A;          // planes of radius RIN
  Transfer1D Rt, Pt;
  cd *out, *outb;
  cf* out32;            // FP32 copy of out, or null
};

// this wavefront's coarse node; blocks in slabs, one per XCD (block b runs on XCD b % 8), so
// that neighbouring runs of a plane meet in one L2
__device__ __forceinline__ long long gal_node(const Geom& gc, int wv) {
  const long long per = ((long long)gridDim.x + 7) / 8;
  const long long b = (long long)(blockIdx.x % 8) * per + blockIdx.x / 8;
  return b * 4 + wv;
}

// q, of the box, into sum_j q(j) P(j, I + D): three one-axis passes (axis 0, then 1, then 2),
// each term 2 Pt.w[j_a - 2 J_a + BP] for the j_a in the box; the result in t, D0 fastest
template <class B>
__device__ __forceinline__ void gal_passes(cd* q, cd* t, const Transfer1D& Pt, int lane) {
  // term o of output D: box position 2 (D - RC) + AR + RIN - BP + o
  auto pass = [&](const cd* in, cd* out, int n, int stride, auto index) {
    for (int e = lane; e < n; e += 64) {
      int D, base;
      index(e, D, base);
      const int j0 = 2 * (D - B::RC) + B::AR + B::RIN - B::BP;
      cd acc = mk(0.0, 0.0);
#pragma unroll
      for (int o = 0; o <= 2 * B::BP; ++o)
        if (j0 + o >= 0 && j0 + o < B::S) acc += (2.0 * Pt.w[o]) * in[base + stride * (j0 + o)];
      out[e] = acc;
    }
    __syncthreads();
  };
  __syncthreads();
  pass(q, t, B::NT, 1, [](int e, int& D, int& base) { D = e % B::W; base = B::S * (e / B::W); });
  if constexpr (B::DIM == 3) {
    pass(t, q, B::NU, B::W, [](int e, int& D, int& base) {
      D = e / B::W % B::W;
      base = e % B::W + B::W * B::S * (e / (B::W * B::W));
    });
    pass(q, t, B::NO, B::W * B::W, [](int e, int& D, int& base) { D = e / (B::W * B::W); base = e % (B::W * B::W); });
  } else {
    pass(t, q, B::NO, B::W, [](int e, int& D, int& base) { D = e / B::W; base = e % B::W; });
    for (int e = lane; e < B::NO; e += 64) t[e] = q[e];
    __syncthreads();
  }
}
// the block's four results (nodes at sI), four consecutive threads an entry of each: in is false
// for J off the grid
template <class B, class ST>
__device__ __forceinline__ void gal_store(const GalArgs& a, const cd (*t)[B::NT], const int (*sI)[3], ST st) {
  const int nd = threadIdx.x % 4;
  const long long I = gal_node(a.gc, nd);
  if (I >= a.gc.tot) return;
  const int Ia[3] = {sI[nd][0], sI[nd][1], sI[nd][2]};
  for (int o = threadIdx.x / 4; o < B::NO; o += 64) {
    const int D[3] = {o % B::W, o / B::W % B::W, B::DIM == 3 ? o / (B::W * B::W) : B::RC};
    bool in = true;
    for (int d = 0; d < B::DIM; ++d) in = in && Ia[d] + D[d] >= B::RC && Ia[d] + D[d] - B::RC < a.gc.N[d];
    st((long long)o * a.gc.tot + I, in, t[nd][o], nd, D);
  }
}

// A weighs an offset by the number of axes it moves along, so with c_a = r_a(j_a) and s_a =
// r_a(j_a - 1) + r_a(j_a + 1), r_a the row of R along axis a (zero off its support and off the
// grid), the sums over i are those over the subsets of moved axes:
//   centre prod c, faces sum_a s_a prod_{b != a} c_b, edges (3D) sum_a c_a prod_{b != a} s_b
template <int DIM>
__device__ __forceinline__ double gal_lap(const double* c, const double* s) {
  if constexpr (DIM == 3) {
    const double cc = c[0] * c[1] * c[2];
    const double ff = s[0] * c[1] * c[2] + c[0] * s[1] * c[2] + c[0] * c[1] * s[2];
    const double ee = c[0] * s[1] * s[2] + s[0] * c[1] * s[2] + s[0] * s[1] * c[2];
    return 24.0 * cc - 2.0 * ff - ee;
  } else {
    return 20.0 * (c[0] * c[1]) - 4.0 * (s[0] * c[1] + c[0] * s[1]) - s[0] * s[1];
  }
}
template <int DIM>
__device__ __forceinline__ double gal_mass(const double* c, const double* s) {
  if constexpr (DIM == 3)
    return (6.0 / 12.0) * (c[0] * c[1] * c[2]) +
           (1.0 / 12.0) * (s[0] * c[1] * c[2] + c[0] * s[1] * c[2] + c[0] * c[1] * s[2]);
  else
    return (8.0 / 12.0) * (c[0] * c[1]) + (1.0 / 12.0) * (s[0] * c[1] + c[0] * s[1]);
}

// R L P is a sum of products over the axes: each axis's sums of c and s against P take a lane
// per offset, and only the product with M runs through the box
template <class B>
__global__ void __launch_bounds__(256) k_wgal_fine(GalArgs a) {
  __shared__ cd q[4][B::NQ], t[4][B::NT];
  __shared__ int sI[4][3];
  __shared__ double s1[4][2][B::DIM][B::W], sr[4][B::DIM][B::S + 2];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const long long I = gal_node(a.gc, wv), Ic = I < a.gc.tot ? I : 0;
  int Ia[3];
  coords(a.gc, Ic, Ia[0], Ia[1], Ia[2]);
  if (lane < 3) sI[wv][lane] = lane == 0 ? Ia[0] : lane == 1 ? Ia[1] : Ia[2];
  const long long sf1 = a.gf.N[0], sf2 = (long long)a.gf.N[0] * a.gf.N[1];
  // r_a at box positions -1 .. S (a table: lane-dependent reads of the arguments are loads)
  if (lane < B::DIM * (B::S + 2)) {
    const int d = lane / (B::S + 2), x = lane % (B::S + 2) - 1;
    const int J = d == 0 ? Ia[0] : d == 1 ? Ia[1] : Ia[2], n = d == 0 ? a.gf.N[0] : d == 1 ? a.gf.N[1] : a.gf.N[2];
    const int i = 2 * J - B::AR - B::RIN + x;
    sr[wv][d][x + 1] =
        x >= B::RIN && x <= B::RIN + 2 * B::AR && i >= 0 && i < n ? a.Rt.w[x - B::RIN] : 0.0;
  }
  __syncthreads();
  if (lane < 2 * B::DIM * B::W) {
    const int moved = lane % 2, D = lane / 2 % B::W, d = lane / 2 / B::W;
    const int J = d == 0 ? Ia[0] : d == 1 ? Ia[1] : Ia[2], n = d == 0 ? a.gf.N[0] : d == 1 ? a.gf.N[1] : a.gf.N[2];
    double acc = 0.0;
#pragma unroll
    for (int o = 0; o <= 2 * B::BP; ++o) {
      const int x = 2 * (D - B::RC) + B::AR + B::RIN - B::BP + o, j = 2 * J - B::AR - B::RIN + x;
      if (x < 0 || x >= B::S || j < 0 || j >= n) continue;
      acc += (2.0 * a.Pt.w[o]) * (moved ? sr[wv][d][x] + sr[wv][d][x + 2] : sr[wv][d][x + 1]);
    }
    s1[wv][moved][d][D] = acc;
  }
  for (int e = lane; e < B::NQ; e += 64) {
    const int r[3] = {e % B::S, e / B::S % B::S, B::DIM == 3 ? e / (B::S * B::S) : B::AR + B::RIN};
    int j[3] = {0, 0, 0};
    bool in = true;
    for (int d = 0; d < B::DIM; ++d) {
      j[d] = 2 * Ia[d] - B::AR - B::RIN + r[d];
      in = in && j[d] >= 0 && j[d] < a.gf.N[d];
    }
    cd acc = mk(0.0, 0.0);
    if (in) {
      double cv[3], sv[3];
      for (int d = 0; d < B::DIM; ++d) {
        cv[d] = sr[wv][d][r[d] + 1];
        sv[d] = sr[wv][d][r[d]] + sr[wv][d][r[d] + 2];
      }
      const double mj = a.m[j[0] + j[1] * sf1 + j[2] * sf2];
      acc = gal_mass<B::DIM>(cv, sv) * mk(mj, -mj * layer_sigma(a.op, j[0], j[1], j[2]));
    }
    q[wv][e] = acc;
  }
  gal_passes<B>(q[wv], t[wv], a.Pt, lane);
  const double ih = a.op.inv_h2 / 6.0;
  gal_store<B>(a, t, sI, [&](long long at, bool in, cd v, int nd, const int* D) {
    cd xa = mk(0.0, 0.0), xb = mk(0.0, 0.0);
    if (in) {
      double cv[3], sv[3];
      for (int d = 0; d < B::DIM; ++d) {
        cv[d] = s1[nd][0][d][D[d]];
        sv[d] = s1[nd][1][d][D[d]];
      }
      const cd l = mk(ih * gal_lap<B::DIM>(cv, sv), 0.0);
      xa = l - a.sa * v;
      xb = l - a.sb * v;
    }
    a.out[at] = xa;
    a.outb[at] = xb;
    if (a.out32) a.out32[at] = conv<cf>::from(xa);
  });
}

template <class B>
__global__ void __launch_bounds__(256) k_wgal_coarse(GalArgs a) {
  __shared__ cd q[4][B::NQ], t[4][B::NT];
  __shared__ int sI[4][3];
  constexpr int SW = 2 * B::RIN + 1;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const long long I = gal_node(a.gc, wv), Ic = I < a.gc.tot ? I : 0;
  int Ia[3];
  coords(a.gc, Ic, Ia[0], Ia[1], Ia[2]);
  if (lane < 3) sI[wv][lane] = lane == 0 ? Ia[0] : lane == 1 ? Ia[1] : Ia[2];
  const long long sf1 = a.gf.N[0], sf2 = (long long)a.gf.N[0] * a.gf.N[1];
  for (int e = lane; e < B::NQ; e += 64) {
    const int r[3] = {e % B::S, e / B::S % B::S, B::DIM == 3 ? e / (B::S * B::S) : B::AR + B::RIN};
    bool in = true;
    for (int d = 0; d < B::DIM; ++d) {
      const int j = 2 * Ia[d] - B::AR - B::RIN + r[d];
      in = in && j >= 0 && j < a.gf.N[d];
    }
    cd acc = mk(0.0, 0.0);
    if (in)
      // fine rows i = 2 I + o - AR on the grid within RIN of j (box position RIN + o): a row of
      // terms is loaded at clamped indices before any is added
      for (int o2 = 0; o2 <= (B::DIM == 3 ? 2 * B::AR : 0); ++o2) {
        const int i2 = B::DIM == 3 ? 2 * Ia[2] - B::AR + o2 : 0, k2 = B::DIM == 3 ? r[2] - o2 : 0;
        if (B::DIM == 3 && (i2 < 0 || i2 >= a.gf.N[2] || k2 < 0 || k2 >= SW)) continue;
#pragma unroll
        for (int o1 = 0; o1 <= 2 * B::AR; ++o1) {
          const int i1 = 2 * Ia[1] - B::AR + o1, k1 = r[1] - o1;
          const bool ok1 = i1 >= 0 && i1 < a.gf.N[1] && k1 >= 0 && k1 < SW;
          cd v[2 * B::AR + 1];
#pragma unroll
          for (int o0 = 0; o0 <= 2 * B::AR; ++o0) {
            const int i0 = 2 * Ia[0] - B::AR + o0, k0 = r[0] - o0;
            const bool ok = ok1 && i0 >= 0 && i0 < a.gf.N[0] && k0 >= 0 && k0 < SW;
            const long long at = (long long)(k0 + SW * (k1 + SW * k2)) * a.gf.tot + (i0 + i1 * sf1 + i2 * sf2);
            v[o0] = a.A[ok ? at : 0];
            v[o0].x = ok ? v[o0].x : 0.0;
            v[o0].y = ok ? v[o0].y : 0.0;
          }
#pragma unroll
          for (int o0 = 0; o0 <= 2 * B::AR; ++o0) {
            double w = a.Rt.w[o0] * a.Rt.w[o1];
            if (B::DIM == 3) w *= a.Rt.w[o2];
            acc += w * v[o0];
          }
        }
      }
    q[wv][e] = acc;
  }
  gal_passes<B>(q[wv], t[wv], a.Pt, lane);
  gal_store<B>(a, t, sI, [&](long long at, bool in, cd v, int, const int*) { a.out[at] = in ? mk(v.x, v.y) : mk(0.0, 0.0); });
}

// ----------------------------------------------------------- cycle steps ----
template <int DIM, typename R, typename CB, typename CO>
__global__ void __launch_bounds__(256) k_w1(WFine<R> A, int mode, int xz, const typename cplx<R>::type* __restrict__ x,
                                            const CB* __restrict__ b, R w, CO* __restrict__ out) {
  typedef typename cplx<R>::type C;
  const Geom& g = A.op.g;
  const long long f = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= g.tot) return;
  const long long off = (long long)blockIdx.y * g.tot;
  int i0, i1, i2;
  coords(g, f, i0, i1, i2);
  C dg;
  const C ax = wide_row<DIM, R, C>(A.op, A.s, A.m, x + off, f, i0, i1, i2, xz != 0, dg);
  C v;
  if (mode == WM_APPLY) {
    v = ax;
  } else {
    const C r = conv<C>::from(b[off + f]) - ax;
    if (mode == WM_RES) {
      v = r;
    } else {
      const C xo = xz ? mk((R)0, (R)0) : x[off + f];
      v = xo + w * cdiv(r, dg);
    }
  }
  out[off + f] = conv<CO>::from(v);
}

// planes of radius RAD: (A x)_i = sum_k coef[k N + i] x[i + d_k]
template <int DIM, int RAD, typename R>
__global__ void __launch_bounds__(256) k_w2(Geom g, const typename cplx<R>::type* __restrict__ coef, int mode, int xz,
                                            const typename cplx<R>::type* __restrict__ x,
                                            const typename cplx<R>::type* __restrict__ b, R w,
                                            typename cplx<R>::type* __restrict__ out) {
  typedef typename cplx<R>::type C;
  constexpr int SW = 2 * RAD + 1;
  const long long f = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= g.tot) return;
  const long long off = (long long)blockIdx.y * g.tot;
  int i0, i1, i2;
  coords(g, f, i0, i1, i2);
  const long long s1 = g.N[0], s2 = (long long)g.N[0] * g.N[1];
  constexpr int KC = DIM == 3 ? (SW * SW * SW) / 2 : (SW * SW) / 2;    // centre plane
  const C dg = coef[(long long)KC * g.tot + f];
  C ax = mk((R)0, (R)0);
  if (!xz) {
    // one plane of (2 RAD + 1)^2 taps in flight at a time: the fully unrolled 125-tap 3D
    // loop needed 512 registers and spilled
#pragma unroll 1
    for (int d2 = (DIM == 3 ? -RAD : 0); d2 <= (DIM == 3 ? RAD : 0); ++d2)
#pragma unroll
      for (int d1 = -RAD; d1 <= RAD; ++d1) {
        const bool in1 = i1 + d1 >= 0 && i1 + d1 <= g.n[1] && (DIM == 2 || (i2 + d2 >= 0 && i2 + d2 <= g.n[2]));
#pragma unroll
        for (int d0 = -RAD; d0 <= RAD; ++d0) {
          const int k = (d0 + RAD) + SW * (d1 + RAD) + (DIM == 3 ? SW * SW * (d2 + RAD) : 0);
          const bool in = in1 && i0 + d0 >= 0 && i0 + d0 <= g.n[0];
          const long long j = in ? f + d0 + d1 * s1 + d2 * s2 : f;
          const C a = coef[(long long)k * g.tot + f];
          const C xv = x[off + j];
          ax += (in ? (R)1 : (R)0) * (a * xv);
        }
      }
  }
  C v;
  if (mode == WM_APPLY) {
    v = ax;
  } else {
    const C r = b[off + f] - ax;
    if (mode == WM_RES) {
      v = r;
    } else {
      const C xo = xz ? mk((R)0, (R)0) : x[off + f];
      v = xo + w * cdiv(r, dg);
    }
  }
  out[off + f] = v;
}

// b_c(I) = sum_i R(I, i) v(i), one coarse node per thread.  The half-width A is a constant, so the
// weights are scalars and a row of terms is loaded (at clamped indices, 0 off the grid) before
// any is added: with bounds per thread every weight was a load and every term waited for the one
// before (192 x 192 x 72: 53 us, now 25)
template <int DIM, int A, typename C, typename CO>
__global__ void __launch_bounds__(256) k_wrestrict(Geom gf, const C* __restrict__ v, Geom gc, Transfer1D Rt,
                                                   CO* __restrict__ out) {
  typedef decltype(v[0].x) R;
  const long long I = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= gc.tot) return;
  v += (long long)blockIdx.y * gf.tot;
  out += (long long)blockIdx.y * gc.tot;
  int Ia[3];
  coords(gc, I, Ia[0], Ia[1], Ia[2]);
  const long long s1 = gf.N[0], s2 = (long long)gf.N[0] * gf.N[1];
  C acc = mk((R)0, (R)0);
#pragma unroll 1                    // a plane's terms in flight: all planes' take 256 registers
  for (int o2 = 0; o2 <= (DIM == 3 ? 2 * A : 0); ++o2) {
    const int i2 = DIM == 3 ? 2 * Ia[2] - A + o2 : 0;
    const bool ok2 = DIM < 3 || (i2 >= 0 && i2 < gf.N[2]);
    const R w2 = DIM == 3 ? (R)Rt.w[o2] : (R)1;
#pragma unroll
    for (int o1 = 0; o1 <= 2 * A; ++o1) {
      const int i1 = 2 * Ia[1] - A + o1;
      const bool ok1 = ok2 && i1 >= 0 && i1 < gf.N[1];
      const R w1 = w2 * (R)Rt.w[o1];
      C t[2 * A + 1];
#pragma unroll
      for (int o0 = 0; o0 <= 2 * A; ++o0) {
        const int i0 = 2 * Ia[0] - A + o0;
        const bool ok = ok1 && i0 >= 0 && i0 < gf.N[0];
        t[o0] = v[ok ? i0 + i1 * s1 + i2 * s2 : 0];
        t[o0].x = ok ? t[o0].x : (R)0;
        t[o0].y = ok ? t[o0].y : (R)0;
      }
#pragma unroll
      for (int o0 = 0; o0 <= 2 * A; ++o0) acc += (w1 * (R)Rt.w[o0]) * t[o0];
    }
  }
  out[I] = conv<CO>::from(acc);
}

// x (+)= P e, one fine node per thread: along an axis the coarse J = lo + k, k <= A, with weight
// 2 Pt.w[i - 2 J + A] (the last of an odd i - A is none); loads as in k_wrestrict (192 x 192 x 72:
// 77 us, now 42)
template <int DIM, int A, typename CE, typename C>
__global__ void __launch_bounds__(256) k_wprolong(Geom gc, const CE* __restrict__ e, Geom gf, Transfer1D Pt, int add,
                                                  C* __restrict__ x) {
  typedef decltype(x[0].x) R;
  const long long f = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= gf.tot) return;
  e += (long long)blockIdx.y * gc.tot;
  x += (long long)blockIdx.y * gf.tot;
  int ia[3];
  coords(gf, f, ia[0], ia[1], ia[2]);
  int lo[3];
  R w[3][A + 1];
  for (int d = 0; d < DIM; ++d) {
    lo[d] = (ia[d] - A + 1) >> 1;                  // ceil((i - A) / 2)
    const bool odd = (ia[d] - A) & 1;
#pragma unroll
    for (int k = 0; k <= A; ++k)
      w[d][k] = odd ? (k < A ? (R)(2.0 * Pt.w[2 * A - 1 - 2 * (k < A ? k : 0)]) : (R)0) : (R)(2.0 * Pt.w[2 * A - 2 * k]);
  }
  const long long s1 = gc.N[0], s2 = (long long)gc.N[0] * gc.N[1];
  const C xo = add ? x[f] : mk((R)0, (R)0);
  C acc = mk((R)0, (R)0);
#pragma unroll
  for (int k2 = 0; k2 <= (DIM == 3 ? A : 0); ++k2) {
    const int J2 = DIM == 3 ? lo[2] + k2 : 0;
    const bool ok2 = DIM < 3 || (J2 >= 0 && J2 < gc.N[2]);
    const R w2 = DIM == 3 ? w[2][k2] : (R)1;
#pragma unroll
    for (int k1 = 0; k1 <= A; ++k1) {
      const int J1 = lo[1] + k1;
      const bool ok1 = ok2 && J1 >= 0 && J1 < gc.N[1];
      const R w1 = w2 * w[1][k1];
      C t[A + 1];
#pragma unroll
      for (int k0 = 0; k0 <= A; ++k0) {
        const int J0 = lo[0] + k0;
        // (a term of weight 0 takes 0, whatever its entry)
        const bool ok = ok1 && J0 >= 0 && J0 < gc.N[0] && w1 * w[0][k0] != (R)0;
        t[k0] = conv<C>::from(e[ok ? J0 + J1 * s1 + J2 * s2 : 0]);
        t[k0].x = ok ? t[k0].x : (R)0;
        t[k0].y = ok ? t[k0].y : (R)0;
      }
#pragma unroll
      for (int k0 = 0; k0 <= A; ++k0) acc += (w1 * w[0][k0]) * t[k0];
    }
  }
  x[f] = add ? xo + acc : acc;
}

template <typename CI, typename CO>
__global__ void __launch_bounds__(256) k_wcopy(const CI* __restrict__ in, CO* __restrict__ out, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = conv<CO>::from(in[i]);
}

inline dim3 grid1(long long n, int nr) { return dim3((unsigned)((n + 255) / 256), (unsigned)nr); }

}  // namespace

// ------------------------------------------------------------- launchers ----
static dim3 gal_grid(const Geom& gc) { return dim3((unsigned)((gc.tot + 31) / 32 * 8)); }
// whether a transfer pair and radii are those of B
template <class B>
static bool gal_is(const Geom& g, const Transfer1D& Rt, int rin, const Transfer1D& Pt, int rc) {
  return g.dim == B::DIM && Rt.a == B::AR && rin == B::RIN && Pt.a == B::BP && rc == B::RC;
}

void wgal_fine(const FineOp& op, cd sa, cd sb, const double* m, const Geom& gc, const Transfer1D& Rt,
               const Transfer1D& Pt, int rc, cd* outa, cf* outa32, cd* outb, hipStream_t st) {
  typedef GalBox<3, 2, 1, 2, 2> B3;
  typedef GalBox<2, 2, 1, 2, 2> B2;
  GalArgs a{};
  a.gf = op.g;
  a.gc = gc;
  a.op = op;
  a.m = m;
  a.sa = sa;
  a.sb = sb;
  a.Rt = Rt;
  a.Pt = Pt;
  a.out = outa;
  a.outb = outb;
  a.out32 = outa32;
  if (gal_is<B3>(op.g, Rt, 1, Pt, rc))
    hipLaunchKernelGGL((k_wgal_fine<B3>), gal_grid(gc), dim3(256), 0, st, a);
  else if (gal_is<B2>(op.g, Rt, 1, Pt, rc))
    hipLaunchKernelGGL((k_wgal_fine<B2>), gal_grid(gc), dim3(256), 0, st, a);
  else
    throw std::runtime_error("wgal_fine: transfers");
}

void wgal_coarse(const Geom& g, const cd* A, int rin, const Geom& gc, const Transfer1D& Rt, const Transfer1D& Pt,
                 int rc, cd* out, hipStream_t st) {
  typedef GalBox<3, 1, 2, 2, 2> L3;       // level-dependent transfers
  typedef GalBox<2, 1, 2, 2, 2> L2;
  typedef GalBox<2, 2, 2, 2, 3> C2;       // cubic
  GalArgs a{};
  a.gf = g;
  a.gc = gc;
  a.A = A;
  a.Rt = Rt;
  a.Pt = Pt;
  a.out = out;
  if (gal_is<L3>(g, Rt, rin, Pt, rc))
    hipLaunchKernelGGL((k_wgal_coarse<L3>), gal_grid(gc), dim3(256), 0, st, a);
  else if (gal_is<L2>(g, Rt, rin, Pt, rc))
    hipLaunchKernelGGL((k_wgal_coarse<L2>), gal_grid(gc), dim3(256), 0, st, a);
  else if (gal_is<C2>(g, Rt, rin, Pt, rc))
    hipLaunchKernelGGL((k_wgal_coarse<C2>), gal_grid(gc), dim3(256), 0, st, a);
  else
    throw std::runtime_error("wgal_coarse: transfers");
}

template <typename R, typename CB, typename CO>
void w1_step(const WFine<R>& A, int mode, int xz, const typename cplx<R>::type* x, const CB* b, R w, CO* out, int nr,
             hipStream_t st) {
  const dim3 grid = grid1(A.op.g.tot, nr);
  if (xz) x = (const typename cplx<R>::type*)(const void*)out;   // not read; a valid address all the same
  if (A.op.g.dim == 3)
    hipLaunchKernelGGL((k_w1<3, R, CB, CO>), grid, dim3(256), 0, st, A, mode, xz, x, b, w, out);
  else
    hipLaunchKernelGGL((k_w1<2, R, CB, CO>), grid, dim3(256), 0, st, A, mode, xz, x, b, w, out);
}

template <typename R>
void w2_step(const Geom& g, const typename cplx<R>::type* coef, int r, int mode, int xz,
             const typename cplx<R>::type* x, const typename cplx<R>::type* b, R w, typename cplx<R>::type* out,
             int nr, hipStream_t st) {
  const dim3 grid = grid1(g.tot, nr);
  if (xz) x = out;                                    // not read; a valid address all the same
  if (g.dim == 3 && r == 2)
    hipLaunchKernelGGL((k_w2<3, 2, R>), grid, dim3(256), 0, st, g, coef, mode, xz, x, b, w, out);
  else if (g.dim == 2 && r == 2)
    hipLaunchKernelGGL((k_w2<2, 2, R>), grid, dim3(256), 0, st, g, coef, mode, xz, x, b, w, out);
  else
    throw std::runtime_error("w2_step: no kernel for this dimension and stencil radius");
}

template <typename CI, typename CO>
void w_restrict(const Geom& gf, const CI* v, const Geom& gc, const Transfer1D& Rt, CO* out, int nr, hipStream_t st) {
  const dim3 grid = grid1(gc.tot, nr);
  if (gf.dim == 3 && Rt.a == 1)
    hipLaunchKernelGGL((k_wrestrict<3, 1, CI, CO>), grid, dim3(256), 0, st, gf, v, gc, Rt, out);
  else if (gf.dim == 3)
    hipLaunchKernelGGL((k_wrestrict<3, 2, CI, CO>), grid, dim3(256), 0, st, gf, v, gc, Rt, out);
  else if (Rt.a == 1)
    hipLaunchKernelGGL((k_wrestrict<2, 1, CI, CO>), grid, dim3(256), 0, st, gf, v, gc, Rt, out);
  else
    hipLaunchKernelGGL((k_wrestrict<2, 2, CI, CO>), grid, dim3(256), 0, st, gf, v, gc, Rt, out);
}

template <typename CE, typename C>
void w_prolong(const Geom& gc, const CE* e, const Geom& gf, const Transfer1D& Pt, int add, C* x, int nr,
               hipStream_t st) {
  const dim3 grid = grid1(gf.tot, nr);
  if (gf.dim == 3 && Pt.a == 1)
    hipLaunchKernelGGL((k_wprolong<3, 1, CE, C>), grid, dim3(256), 0, st, gc, e, gf, Pt, add, x);
  else if (gf.dim == 3)
    hipLaunchKernelGGL((k_wprolong<3, 2, CE, C>), grid, dim3(256), 0, st, gc, e, gf, Pt, add, x);
  else if (Pt.a == 1)
    hipLaunchKernelGGL((k_wprolong<2, 1, CE, C>), grid, dim3(256), 0, st, gc, e, gf, Pt, add, x);
  else
    hipLaunchKernelGGL((k_wprolong<2, 2, CE, C>), grid, dim3(256), 0, st, gc, e, gf, Pt, add, x);
}

template <typename CI, typename CO>
void w_copy(const CI* in, CO* out, long long n, hipStream_t st) {
  hipLaunchKernelGGL((k_wcopy<CI, CO>), dim3(1024), dim3(256), 0, st, in, out, n);
}

template void w1_step<float, cd, cf>(const WFine<float>&, int, int, const cf*, const cd*, float, cf*, int, hipStream_t);
template void w1_step<float, cd, cd>(const WFine<float>&, int, int, const cf*, const cd*, float, cd*, int, hipStream_t);
template void w1_step<float, cf, cf>(const WFine<float>&, int, int, const cf*, const cf*, float, cf*, int, hipStream_t);
template void w1_step<double, cd, cd>(const WFine<double>&, int, int, const cd*, const cd*, double, cd*, int,
                                      hipStream_t);
template void w2_step<float>(const Geom&, const cf*, int, int, int, const cf*, const cf*, float, cf*, int, hipStream_t);
template void w2_step<double>(const Geom&, const cd*, int, int, int, const cd*, const cd*, double, cd*, int,
                              hipStream_t);
template void w_restrict<cf, cf>(const Geom&, const cf*, const Geom&, const Transfer1D&, cf*, int, hipStream_t);
template void w_restrict<cf, cd>(const Geom&, const cf*, const Geom&, const Transfer1D&, cd*, int, hipStream_t);
template void w_restrict<cd, cd>(const Geom&, const cd*, const Geom&, const Transfer1D&, cd*, int, hipStream_t);
template void w_restrict<cd, cf>(const Geom&, const cd*, const Geom&, const Transfer1D&, cf*, int, hipStream_t);
template void w_prolong<cf, cf>(const Geom&, const cf*, const Geom&, const Transfer1D&, int, cf*, int, hipStream_t);
template void w_prolong<cd, cf>(const Geom&, const cd*, const Geom&, const Transfer1D&, int, cf*, int, hipStream_t);
template void w_prolong<cd, cd>(const Geom&, const cd*, const Geom&, const Transfer1D&, int, cd*, int, hipStream_t);
template void w_prolong<cf, cd>(const Geom&, const cf*, const Geom&, const Transfer1D&, int, cd*, int, hipStream_t);
template void w_copy<cf, cf>(const cf*, cf*, long long, hipStream_t);
template void w_copy<cf, cd>(const cf*, cd*, long long, hipStream_t);
template void w_copy<cd, cd>(const cd*, cd*, long long, hipStream_t);
template void w_copy<cd, cf>(const cd*, cf*, long long, hipStream_t);

}  // namespace helm
