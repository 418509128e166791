// Internal declarations of libhelm (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <string>
#include <vector>

#include "../../include/helm.h"

namespace helm {

// ---------------------------------------------------------------------------
// complex numbers: interleaved (re, im) in FP32 (cf) and FP64 (cd).  Dedicated
// types rather than HIP's float2/double2, whose operators are element-wise.
// ---------------------------------------------------------------------------
struct __align__(8) cf { float x, y; };
struct __align__(16) cd { double x, y; };
template <typename R> struct cplx;
template <> struct cplx<float> { typedef cf type; };
template <> struct cplx<double> { typedef cd type; };

__host__ __device__ inline cf mk(float a, float b) { cf r; r.x = a; r.y = b; return r; }
__host__ __device__ inline cd mk(double a, double b) { cd r; r.x = a; r.y = b; return r; }
__host__ __device__ inline cf operator+(cf a, cf b) { return mk(a.x + b.x, a.y + b.y); }
__host__ __device__ inline cd operator+(cd a, cd b) { return mk(a.x + b.x, a.y + b.y); }
__host__ __device__ inline cf operator-(cf a, cf b) { return mk(a.x - b.x, a.y - b.y); }
__host__ __device__ inline cd operator-(cd a, cd b) { return mk(a.x - b.x, a.y - b.y); }
__host__ __device__ inline cf operator-(cf a) { return mk(-a.x, -a.y); }
__host__ __device__ inline cd operator-(cd a) { return mk(-a.x, -a.y); }
__host__ __device__ inline cf operator*(cf a, cf b) {
  return mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__host__ __device__ inline cd operator*(cd a, cd b) {
  return mk(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__host__ __device__ inline cf operator*(float s, cf a) { return mk(s * a.x, s * a.y); }
__host__ __device__ inline cd operator*(double s, cd a) { return mk(s * a.x, s * a.y); }
__host__ __device__ inline cf& operator+=(cf& a, cf b) { a.x += b.x; a.y += b.y; return a; }
__host__ __device__ inline cd& operator+=(cd& a, cd b) { a.x += b.x; a.y += b.y; return a; }
__host__ __device__ inline cf& operator-=(cf& a, cf b) { a.x -= b.x; a.y -= b.y; return a; }
__host__ __device__ inline cd& operator-=(cd& a, cd b) { a.x -= b.x; a.y -= b.y; return a; }
__host__ __device__ inline cf conjc(cf a) { return mk(a.x, -a.y); }
__host__ __device__ inline cd conjc(cd a) { return mk(a.x, -a.y); }
__host__ __device__ inline float abs2(cf a) { return a.x * a.x + a.y * a.y; }
__host__ __device__ inline double abs2(cd a) { return a.x * a.x + a.y * a.y; }
// a * conj(b) and conj(a) * b
__host__ __device__ inline cd cmulc(cd a, cd b) {  // conj(a) * b
  return mk(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__host__ __device__ inline cf cmulc(cf a, cf b) {
  return mk(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
__host__ __device__ inline cd cdiv(cd a, cd b) {
  double d = b.x * b.x + b.y * b.y;
  return mk((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}
__host__ __device__ inline cf cdiv(cf a, cf b) {
  float d = b.x * b.x + b.y * b.y;
  return mk((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}
// conversions between precisions
__host__ __device__ inline cf to_f(cd a) { return mk((float)a.x, (float)a.y); }
__host__ __device__ inline cf to_f(cf a) { return a; }
__host__ __device__ inline cd to_d(cf a) { return mk((double)a.x, (double)a.y); }
__host__ __device__ inline cd to_d(cd a) { return a; }
// streaming accesses of vectors that a pass reads or writes once (the Krylov basis):
// marked non-temporal so that they do not displace the data reused from pass to pass
// (the coarsest factors, the level-2 coefficients) in the caches
typedef double dvec2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ cd ld_nt(const cd* p) {
  const dvec2 v = __builtin_nontemporal_load((const dvec2*)p);
  return mk(v.x, v.y);
}
__device__ __forceinline__ void st_nt(cd* p, cd v) {
  dvec2 w;
  w.x = v.x;
  w.y = v.y;
  __builtin_nontemporal_store(w, (dvec2*)p);
}

template <typename C> struct conv;
template <> struct conv<cf> {
  __host__ __device__ static cf from(cd a) { return to_f(a); }
  __host__ __device__ static cf from(cf a) { return a; }
};
template <> struct conv<cd> {
  __host__ __device__ static cd from(cd a) { return a; }
  __host__ __device__ static cd from(cf a) { return to_d(a); }
};

// ---------------------------------------------------------------------------
// grid geometry of one level
// ---------------------------------------------------------------------------
struct Geom {
  int dim;
  int n[3];       // cells (1 node on unused axes: n = 0)
  int N[3];       // nodes per axis = n + 1 (1 on unused axes)
  long long tot;  // total nodes
};

// coordinates of flat node index f = i0 + N0 (i1 + N1 i2); a grid has fewer than 2^31 nodes,
// so 32-bit division serves (64-bit division has no instruction and costs some 40)
__device__ __forceinline__ void node_coords(const Geom& g, long long f, int& i0, int& i1, int& i2) {
  const unsigned u = (unsigned)f, N0 = (unsigned)g.N[0], N1 = (unsigned)g.N[1];
  const unsigned r = u / N0;
  i0 = (int)(u - r * N0);
  const unsigned q = r / N1;
  i1 = (int)(r - q * N1);
  i2 = (int)q;
}

inline Geom make_geom(int dim, const int* n) {
  Geom g;
  g.dim = dim;
  g.tot = 1;
  for (int a = 0; a < 3; ++a) {
    g.n[a] = a < dim ? n[a] : 0;
    g.N[a] = g.n[a] + 1;
    g.tot *= g.N[a];
  }
  return g;
}
inline Geom coarsen(const Geom& f) {
  int n[3] = {f.n[0] / 2, f.n[1] / 2, f.n[2] / 2};
  return make_geom(f.dim, n);
}

// fine level operator: -Lap_h - s * m (1 - i sigma) with a complex scalar s
struct FineOp {
  Geom g;
  int compact = 0;      // 1: the compact fourth-order operator (eqs. 3.1, 3.2) with its mass term
  double inv_h2;
  int layer[3][2];
  double sigma_max;
  // the layer profile's per-axis constants (set by set_layer_profile): reciprocal widths
  // (0 where a face has no layer) in FP64 and FP32, and the first node past the high face's
  // inner edge
  double inv_w[3][2];
  float inv_wf[3][2];
  int inner_hi[3];
};

// the profile's constants of op.layer and op.g
inline void set_layer_profile(FineOp& op) {
  for (int a = 0; a < 3; ++a) {
    for (int s = 0; s < 2; ++s) {
      const int w = a < op.g.dim ? op.layer[a][s] : 0;
      op.inv_w[a][s] = w > 0 ? 1.0 / w : 0.0;
      op.inv_wf[a][s] = (float)op.inv_w[a][s];
    }
    op.inner_hi[a] = op.g.n[a] - (a < op.g.dim ? op.layer[a][1] : 0);
  }
}

// sigma = sigma_max * sum over axes of (depth into the layer / width)^2, without branches:
// the depth below the low face's inner edge is max(lo - i, 0), past the high face's
// max(i - (n - hi), 0), and a face without a layer has reciprocal width 0
__host__ __device__ inline double layer_sigma(const FineOp& op, int i0, int i1, int i2) {
  const int ii[3] = {i0, i1, i2};
  double s = 0.0;
  for (int a = 0; a < op.g.dim; ++a) {
    const double tl = (double)max(op.layer[a][0] - ii[a], 0) * op.inv_w[a][0];
    const double th = (double)max(ii[a] - op.inner_hi[a], 0) * op.inv_w[a][1];
    s += tl * tl + th * th;
  }
  return op.sigma_max * s;
}

// number of stencil points of the stored coarse operators
__host__ __device__ inline int stencil_points(int dim) { return dim == 2 ? 9 : 27; }

// ---------------------------------------------------------------------------
// nested-dissection structure of the coarsest level (host side)
// ---------------------------------------------------------------------------
struct NDFrontDev {
  int nS, nB, nF;
  int nchild;           // children: plan.children[child_off .. child_off + nchild)
  int child_off;
  int height;
  long long idx_off;    // nF ints: S nodes then B nodes (level-3 flat indices)
  long long inv_off;    // nF+1 ints at cptr[inv_off]: contributions to position i are
                        // cidx[cptr[i] .. cptr[i+1]) (absolute indices into the update pool)
  long long F_off;      // nF*nF cd (row major), setup scratch; holds Schur block for parent
  long long L_off;      // nF x nS column major (ld ldL): left block column [A^-1; C A^-1] (cycle precision)
  long long W_off;      // nS x nB column major (ld ldW): top-right block -A^-1 B          (cycle precision)
  long long upd_off;    // nB update vector (cycle precision)
  long long perm_off;   // nS ints
  long long asm_off;    // assembly entries
  int asm_cnt;
  // leading dimensions of L and W: nF and nS rounded up to 128 bytes, with L_off and W_off
  // multiples of 128 bytes, so that a run of a column starts on a cache line
  int ldL, ldW;
  int pad;
};

// the factorisation's device arrays for the fronts of one height (slot order): the front
// matrices, the second copy of their separator blocks (offset goff per slot, nS x nS), the
// pivot rows pm (perm_off + column) and their inverse ip (-1: not yet a pivot row), the rows of
// an inversion window (a multiple of 16), and the square of the largest entry that a window may
// leave in a row that is still to be pivoted (k_inv_outer)
struct NDInv {
  const NDFrontDev* hf;
  const long long* goff;
  cd *F, *G;
  int *pm, *ip, *err;
  int win;
  double growth2;
};
// bits of the error word: a zero or NaN pivot among all rows of a separator; a window whose own
// rows hold no good pivots
#define ND_SINGULAR 1
#define ND_GROWTH 2

// windows of a separator of nS rows: nwin of wsz rows (a multiple of 16; the last shorter)
__host__ __device__ inline int win_count(int nS, int win) { return (nS + win - 1) / win; }
__host__ __device__ inline int win_size(int nS, int win) {
  const int n = win_count(nS, win);
  return ((nS + n - 1) / n + 15) / 16 * 16;
}

struct NDAsm {          // F[row][col] += coef[cidx]
  int row, col;
  long long cidx;
};

// Substitution launches: one per height and direction, of one of two kinds.
//   row blocks   items of at most rb rows of a front, each by `waves` wavefronts that split the
//                columns; the front's vector is gathered into LDS and the rows are finished
//                in the same launch
//   split-K      tiles of 256 rows x at most 128 columns write partial products, a second
//                launch sums them; for heights with large blocks, which one work-group per
//                row block would not spread over the chip
struct NDGather {       // an entry of a front's vector: r[rid] (rid >= 0) + its children's updates
  int rid, u0, u1, u2, u3;   // the first four updates inline (-1: none)
  int ca, cb;           // the others: cidx[ca .. cb)
  int pad;
};
struct NDRow {
  long long m_off;      // first entry of the front's block (L forward, W backward)
  long long idx_off;    // the front's node list
  long long upd_off;    // its updates
  int ld, r0, nr, K;    // leading dimension, rows [r0, r0 + nr), columns
  int nS, g0;           // forward: the front's first entry in the launch's gather list
};
struct NDTile {
  int front, r0, k0, k1;
  int pslot;            // partial sums P[pslot + t], t < 256
  int voff;             // the front's first entry in the flat gather list
};
struct NDRowTile {
  int front, r0, nkt, pslot, voff, pad;
};

struct NDLaunch {
  int kind = 1;                     // 1: row blocks, 2: split-K
  std::vector<NDGather> gath;       // per front one entry per row (forward) or column (backward)
  std::vector<NDRow> rows;
  int rb = 16, waves = 1, max_k = 0;   // rows of an item, its waves, most columns
  std::vector<NDTile> tiles;
  std::vector<NDRowTile> rtiles;
  long long p_elems = 0;            // partial products of the tiles
};

// several right-hand sides substituted by one launch (grid y): strides, in entries,
// between the vectors of consecutive right-hand sides
struct NDRhs {
  int n = 1;             // right-hand sides
  int pad = 0;
  long long vec = 0;     // r and x (N3)
  long long upd = 0;     // update pool
  long long part = 0;    // split-K partial products
};

struct NDLaunchDev {    // device copy of an NDLaunch, as the kernels see it
  int kind = 1, nrows = 0, ntiles = 0, nrt = 0;
  int rb = 16, waves = 1, max_k = 0;
  const NDGather* gath = nullptr;
  const NDRow* rows = nullptr;
  const NDTile* tiles = nullptr;
  const NDRowTile* rtiles = nullptr;
};

struct NDPlan {
  Geom g;                               // level-3 geometry
  std::vector<NDFrontDev> fronts;
  std::vector<int> idx, maps, cptr, cidx, children;
  std::vector<long long> child_map_off;   // per entry of `children`: offset of its map
  std::vector<NDAsm> asmv;
  std::vector<std::vector<int>> by_height;   // front ids per height
  int max_height = 0;
  long long F_total = 0, L_total = 0, W_total = 0, upd_total = 0, perm_total = 0;
  long long L_alloc = 0, W_alloc = 0;   // entries of the padded L and W storage
  int max_nS = 0, max_nB = 0, max_nF = 0;
  std::vector<NDLaunch> fwd, bwd;
};

// elem_bytes: bytes of a factor entry
// splitk_bytes: heights whose factor blocks hold at least this many bytes (per direction) and
// more than ND_SPLITK_COLS columns use split-K launches; 0: every height does
// merge_heights: heights of the dissection tree (leaves 0, before any merge) whose fronts are
// merged into their parents (fewer levels, larger fronts)
// radius: stencil radius of the coarsest operator (its (2 radius + 1)^dim coefficient planes,
// plane k of offset d = sum_a (d_a + radius) (2 radius + 1)^a)
void nd_plan(const Geom& g3, int leaf_max, int root_merge, int elem_bytes, long long splitk_bytes, NDPlan& plan,
             const std::vector<int>& merge_heights = std::vector<int>(), int radius = 1);
// LDS bytes of a row-block work-group for nr right-hand sides
size_t nd_rows_lds(int rb, int waves, int max_k, int nr, size_t elem_bytes);
#define ND_SPLITK_COLS 256
#define ND_ROWS_LDS (128 * 1024)   // the most a row-block work-group may take for one right-hand side

}  // namespace helm
