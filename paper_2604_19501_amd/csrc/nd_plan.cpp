// Symbolic analysis of the exact coarsest-grid solve.
//
// The coarsest operator (eq. 3.6) is a stencil of radius r on a regular node grid:
// 9-point (2D) / 27-point (3D) for the 5/7-point fine operator with full weighting
// (r = 1), 25- or 49-point (2D) and 125-point (3D) for the compact fourth-order stack
// with high-order or level-dependent transfers (r = 2 or 3).  It is solved exactly by
// block Gaussian elimination in a geometric nested-dissection order: a box of nodes is
// cut by a slab of r node planes normal to its longest axis (r planes separate the two
// halves for a stencil of radius r), recursively, until boxes hold at most leaf_max
// nodes.  Every tree node ("front") eliminates its separator S; its boundary B is the
// r-node halo of its box, which lies in ancestor separators.  After its subtree is
// eliminated, a front couples S and B densely.
//
// The separators of the top levels may be merged into one root front (a
// supernode): elimination stays exact, the tree gets shallower, and the solve
// needs fewer dependent steps at the price of a larger dense root block.
//
// This file builds, on the host: the tree, the S/B index lists, the child->parent
// position maps used by the extend-add of Schur complements and their inverses,
// the list of original matrix entries each front assembles, storage offsets, and
// the work schedules of the forward and backward substitutions.
#include <algorithm>
#include <cassert>
#include <cstdio>
#include <map>
#include <set>
#include <numeric>
#include <stdexcept>

#include "internal.h"

namespace helm {

namespace {

struct Box {
  int lo[3], hi[3];
};

struct Builder {
  Geom g;
  int leaf_max;
  int r = 1;            // stencil radius: separator slab thickness and halo width
  std::vector<Box> box;
  std::vector<std::vector<int>> S, B, kids;
  std::vector<int> parent;

  long long count(const Box& b) const {
    long long c = 1;
    for (int a = 0; a < g.dim; ++a) c *= (b.hi[a] - b.lo[a] + 1);
    return c;
  }
  int flat(int i0, int i1, int i2) const { return i0 + g.N[0] * (i1 + g.N[1] * i2); }

  int build(const Box& b, int par) {
    int id = (int)box.size();
    box.push_back(b);
    S.emplace_back();
    B.emplace_back();
    kids.emplace_back();
    parent.push_back(par);
    int ax = -1, ext = 0;
    for (int a = g.dim - 1; a >= 0; --a) {     // ties: prefer the slowest axis
      int e = b.hi[a] - b.lo[a] + 1;
      if (e > ext) { ext = e; ax = a; }
    }
    bool leaf = count(b) <= leaf_max || ext < r + 2;
    Box sep = b;
    if (!leaf) {
      int mid = (b.lo[ax] + b.hi[ax] - (r - 1)) / 2;     // the slab [mid, mid + r)
      sep.lo[ax] = mid;
      sep.hi[ax] = mid + r - 1;
      Box c0 = b, c1 = b;
      c0.hi[ax] = mid - 1;
      c1.lo[ax] = mid + r;
      int a0 = build(c0, id);
      int a1 = build(c1, id);
      kids[id] = {a0, a1};
    }
    for (int i2 = sep.lo[2]; i2 <= sep.hi[2]; ++i2)
      for (int i1 = sep.lo[1]; i1 <= sep.hi[1]; ++i1)
        for (int i0 = sep.lo[0]; i0 <= sep.hi[0]; ++i0) S[id].push_back(flat(i0, i1, i2));
    // r-node halo of the box inside the domain, increasing flat index
    int lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
      lo[a] = std::max(b.lo[a] - r, 0);
      hi[a] = std::min(b.hi[a] + r, g.N[a] - 1);
    }
    for (int i2 = lo[2]; i2 <= hi[2]; ++i2)
      for (int i1 = lo[1]; i1 <= hi[1]; ++i1)
        for (int i0 = lo[0]; i0 <= hi[0]; ++i0) {
          bool inside = i0 >= b.lo[0] && i0 <= b.hi[0] && i1 >= b.lo[1] && i1 <= b.hi[1] &&
                        i2 >= b.lo[2] && i2 <= b.hi[2];
          if (!inside) B[id].push_back(flat(i0, i1, i2));
        }
    return id;
  }
};

}  // namespace

size_t nd_rows_lds(int rb, int waves, int max_k, int nr, size_t elem_bytes) {
  const size_t ipw = (size_t)std::max(1, 4 / waves);     // items of a work-group (at least 4 waves)
  return elem_bytes * nr * ipw * ((size_t)max_k + (size_t)waves * rb);
}

void nd_plan(const Geom& g3, int leaf_max, int root_merge, int elem_bytes, long long splitk_bytes, NDPlan& plan,
             const std::vector<int>& merge_heights, int radius) {
  Builder bd;
  bd.g = g3;
  bd.leaf_max = std::max(leaf_max, 1);
  bd.r = std::max(1, radius);
  Box rootbox;
  for (int a = 0; a < 3; ++a) {
    rootbox.lo[a] = 0;
    rootbox.hi[a] = g3.N[a] - 1;
  }
  bd.build(rootbox, -1);
  const int nraw = (int)bd.box.size();
  std::vector<char> alive(nraw, 1);
  // ---- amalgamation: every front whose height in the dissection tree (leaves 0) is listed
  // in merge_heights joins its separator to its parent's, and its children become the
  // parent's.  The parent's box contains the child's, so its boundary is unchanged and the
  // elimination stays exact; the tree loses those levels, at the price of larger fronts.
  if (!merge_heights.empty()) {
    std::vector<int> hraw(nraw, 0), host(nraw);
    for (int t = nraw - 1; t >= 0; --t)        // children have larger ids than their parent
      for (int c : bd.kids[t]) hraw[t] = std::max(hraw[t], hraw[c] + 1);
    std::set<int> mh(merge_heights.begin(), merge_heights.end());
    for (int t = 0; t < nraw; ++t) {
      host[t] = t;
      if (t == 0 || !mh.count(hraw[t])) continue;
      const int q = host[bd.parent[t]];        // resolved first: parents precede children
      bd.S[q].insert(bd.S[q].end(), bd.S[t].begin(), bd.S[t].end());
      alive[t] = 0;
      host[t] = q;
    }
    for (int t = 0; t < nraw; ++t) bd.kids[t].clear();
    for (int t = 1; t < nraw; ++t)
      if (alive[t]) {
        bd.parent[t] = host[bd.parent[t]];
        bd.kids[bd.parent[t]].push_back(t);
      }
    for (int t = 0; t < nraw; ++t)
      if (alive[t]) std::sort(bd.S[t].begin(), bd.S[t].end());
  }
  // ---- merge whole levels of separators into the root while its separator stays <= root_merge
  {
    std::vector<int> frontier = bd.kids[0];
    while (!frontier.empty()) {
      size_t add = 0;
      for (int c : frontier) add += bd.S[c].size();
      if (bd.S[0].size() + add > (size_t)root_merge) break;
      std::vector<int> next;
      for (int c : frontier) {
        bd.S[0].insert(bd.S[0].end(), bd.S[c].begin(), bd.S[c].end());
        alive[c] = 0;
        next.insert(next.end(), bd.kids[c].begin(), bd.kids[c].end());
      }
      frontier = next;
    }
    std::sort(bd.S[0].begin(), bd.S[0].end());
    bd.kids[0] = frontier;
    for (int c : frontier) bd.parent[c] = 0;
  }
  // ---- renumber the surviving fronts (children keep larger ids than their parent)
  std::vector<int> nid(nraw, -1), oid;
  for (int t = 0; t < nraw; ++t)
    if (alive[t]) {
      nid[t] = (int)oid.size();
      oid.push_back(t);
    }
  const int nf = (int)oid.size();
  const long long N3 = g3.tot;
  std::vector<int> owner(N3, -1), pos_in_S(N3, -1);
  for (int t = 0; t < nf; ++t) {
    const std::vector<int>& s = bd.S[oid[t]];
    for (size_t i = 0; i < s.size(); ++i) {
      if (owner[s[i]] != -1) throw std::runtime_error("nd_plan: node in two separators");
      owner[s[i]] = t;
      pos_in_S[s[i]] = (int)i;
    }
  }
  for (long long v = 0; v < N3; ++v)
    if (owner[v] < 0) throw std::runtime_error("nd_plan: node in no separator");
  std::vector<std::vector<int>> kids(nf);
  std::vector<int> par(nf, -1), height(nf, 0);
  for (int t = 0; t < nf; ++t)
    for (int c : bd.kids[oid[t]]) {
      kids[t].push_back(nid[c]);
      par[nid[c]] = t;
    }
  for (int t = nf - 1; t >= 0; --t)
    for (int c : kids[t]) height[t] = std::max(height[t], height[c] + 1);

  plan.g = g3;
  plan.fronts.assign(nf, NDFrontDev());
  plan.idx.clear();
  plan.maps.clear();
  plan.asmv.clear();
  plan.children.clear();
  plan.child_map_off.clear();
  plan.max_height = 0;
  plan.max_nS = plan.max_nB = plan.max_nF = 0;
  long long F = 0, L = 0, W = 0, U = 0, P = 0, La = 0, Wa = 0;
  const long long line = std::max(1, 128 / std::max(1, elem_bytes));   // entries per 128 bytes
  auto pad_ld = [&](long long n) { return 4 * n <= 3 * line ? n : (n + line - 1) / line * line; };
  auto Bof = [&](int t) -> const std::vector<int>& { return bd.B[oid[t]]; };
  auto posF = [&](int t, int v) -> int {   // position of node v in front t's (S, B) list, -1 if absent
    if (owner[v] == t) return pos_in_S[v];
    const std::vector<int>& b = Bof(t);
    auto it = std::lower_bound(b.begin(), b.end(), v);
    if (it == b.end() || *it != v) return -1;
    return (int)bd.S[oid[t]].size() + (int)(it - b.begin());
  };
  for (int t = 0; t < nf; ++t) {
    NDFrontDev& f = plan.fronts[t];
    f.nS = (int)bd.S[oid[t]].size();
    f.nB = (int)Bof(t).size();
    f.nF = f.nS + f.nB;
    f.nchild = (int)kids[t].size();
    f.height = height[t];
    plan.max_height = std::max(plan.max_height, f.height);
    f.idx_off = (long long)plan.idx.size();
    plan.idx.insert(plan.idx.end(), bd.S[oid[t]].begin(), bd.S[oid[t]].end());
    plan.idx.insert(plan.idx.end(), Bof(t).begin(), Bof(t).end());
    f.F_off = F;  F += (long long)f.nF * f.nF;
    f.ldL = (int)pad_ld(f.nF);
    f.ldW = (int)pad_ld(f.nS);
    f.L_off = La; La += (long long)f.ldL * f.nS;
    f.W_off = Wa; Wa += (long long)f.ldW * f.nB;
    L += (long long)f.nF * f.nS;
    W += (long long)f.nS * f.nB;
    f.upd_off = U; U += f.nB;
    f.perm_off = P; P += f.nS;
    plan.max_nS = std::max(plan.max_nS, f.nS);
    plan.max_nB = std::max(plan.max_nB, f.nB);
    plan.max_nF = std::max(plan.max_nF, f.nF);
  }
  // child -> parent maps (setup extend-add) and, per parent position, the list of
  // child-update entries that add into it (solve gather), as CSR over positions
  plan.cptr.clear();
  plan.cidx.clear();
  for (int t = 0; t < nf; ++t) {
    NDFrontDev& f = plan.fronts[t];
    f.child_off = (int)plan.children.size();
    std::vector<std::vector<int>> contrib(f.nF);
    for (int c = 0; c < f.nchild; ++c) {
      int ch = kids[t][c];
      plan.children.push_back(ch);
      plan.child_map_off.push_back((long long)plan.maps.size());
      std::vector<char> seen(f.nF, 0);
      int k = 0;
      for (int v : Bof(ch)) {
        int p = posF(t, v);
        if (p < 0) throw std::runtime_error("nd_plan: child boundary outside parent front");
        if (seen[p]) throw std::runtime_error("nd_plan: map not injective");
        seen[p] = 1;
        plan.maps.push_back(p);
        long long a = plan.fronts[ch].upd_off + k++;
        if (a > 0x7fffffffLL) throw std::runtime_error("nd_plan: update pool too large");
        contrib[p].push_back((int)a);
      }
    }
    f.inv_off = (long long)plan.cptr.size();
    int acc = (int)plan.cidx.size();
    for (int p = 0; p < f.nF; ++p) {
      plan.cptr.push_back(acc);
      plan.cidx.insert(plan.cidx.end(), contrib[p].begin(), contrib[p].end());
      acc += (int)contrib[p].size();
    }
    plan.cptr.push_back(acc);
  }
  // assembly lists: entry (i, j) of the operator goes to the front where the first
  // eliminated of i, j is a separator node; the other one is then in that front too.
  const int dim = g3.dim;
  const int rr = bd.r, sw = 2 * bd.r + 1;   // stencil radius and width: plane k of offset d
  for (int t = 0; t < nf; ++t) {
    NDFrontDev& f = plan.fronts[t];
    f.asm_off = (long long)plan.asmv.size();
    const Box& bx = bd.box[oid[t]];
    const std::vector<int>& St = bd.S[oid[t]];
    for (int ps = 0; ps < f.nS; ++ps) {
      int s = St[ps];
      int s0 = s % g3.N[0], s1 = (s / g3.N[0]) % g3.N[1], s2 = s / (g3.N[0] * g3.N[1]);
      for (int d2 = (dim == 3 ? -rr : 0); d2 <= (dim == 3 ? rr : 0); ++d2)
        for (int d1 = -rr; d1 <= rr; ++d1)
          for (int d0 = -rr; d0 <= rr; ++d0) {
            int q0 = s0 + d0, q1 = s1 + d1, q2 = s2 + d2;
            if (q0 < 0 || q0 >= g3.N[0] || q1 < 0 || q1 >= g3.N[1] || q2 < 0 || q2 >= g3.N[2]) continue;
            int q = bd.flat(q0, q1, q2);
            int k = (d0 + rr) + sw * (d1 + rr) + (dim == 3 ? sw * sw * (d2 + rr) : 0);
            int kq = (-d0 + rr) + sw * (-d1 + rr) + (dim == 3 ? sw * sw * (-d2 + rr) : 0);
            if (owner[q] == t) {
              plan.asmv.push_back({ps, pos_in_S[q], (long long)k * N3 + s});
            } else {
              bool inbox = q0 >= bx.lo[0] && q0 <= bx.hi[0] && q1 >= bx.lo[1] && q1 <= bx.hi[1] &&
                           q2 >= bx.lo[2] && q2 <= bx.hi[2];
              if (inbox) continue;   // eliminated in a descendant, arrives via extend-add
              int pq = posF(t, q);
              if (pq < 0) throw std::runtime_error("nd_plan: neighbour outside front");
              plan.asmv.push_back({ps, pq, (long long)k * N3 + s});
              plan.asmv.push_back({pq, ps, (long long)kq * N3 + q});
            }
          }
    }
    f.asm_cnt = (int)((long long)plan.asmv.size() - f.asm_off);
  }
  plan.F_total = F;
  plan.L_total = L;
  plan.W_total = W;
  plan.L_alloc = La;
  plan.W_alloc = Wa;
  plan.upd_total = U;
  plan.perm_total = P;
  plan.by_height.assign(plan.max_height + 1, std::vector<int>());
  for (int t = 0; t < nf; ++t) plan.by_height[plan.fronts[t].height].push_back(t);

  // ---------------- solve schedules ----------------
  // one launch per height and direction (split-K: two): forward ascending, backward descending
  plan.fwd.clear();
  plan.bwd.clear();
  // a front's gather list.  Forward: row i reads r at its node (i < nS) and the children's
  // updates; backward: column j reads x at the boundary node
  auto add_gather = [&](NDLaunch& L, const NDFrontDev& f, int dir) -> int {
    const int g0 = (int)L.gath.size();
    const int* ids = plan.idx.data() + f.idx_off;
    if (dir == 1) {
      for (int j = 0; j < f.nB; ++j) L.gath.push_back({ids[f.nS + j], -1, -1, -1, -1, 0, 0, 0});
      return g0;
    }
    for (int i = 0; i < f.nF; ++i) {
      int ca = plan.cptr[f.inv_off + i];
      const int cb = plan.cptr[f.inv_off + i + 1];
      NDGather g{i < f.nS ? ids[i] : -1, -1, -1, -1, -1, 0, 0, 0};
      for (int* u : {&g.u0, &g.u1, &g.u2, &g.u3})
        if (ca < cb) *u = plan.cidx[ca++];
      g.ca = ca;
      g.cb = cb;
      L.gath.push_back(g);
    }
    return g0;
  };
  // row blocks: a wave takes 64 rows x 16 columns, 32 x 32 or 16 x 64 at a time.  Wide items
  // gather a front's vector less often, narrow ones spread long columns over more lanes; an
  // item has enough waves (up to 16) for one pass.
  auto build_rows = [&](NDLaunch& L, int h, int dir) {
    L.kind = 1;
    int K = 0, Rm = 0;
    for (int t : plan.by_height[h]) {
      const NDFrontDev& f = plan.fronts[t];
      K = std::max(K, dir == 0 ? f.nS : f.nB);
      Rm = std::max(Rm, dir == 0 ? f.nF : f.nS);
    }
    L.rb = K <= 64 ? 64 : K <= 256 ? 32 : 16;
    while (L.rb > 16 && L.rb >= 2 * Rm) L.rb /= 2;
    L.waves = 1;
    while (L.waves < 16 && L.waves * 16 * (64 / L.rb) < K) L.waves *= 2;
    L.max_k = K;
    for (int t : plan.by_height[h]) {
      const NDFrontDev& f = plan.fronts[t];
      const int R = dir == 0 ? f.nF : f.nS, k = dir == 0 ? f.nS : f.nB;
      if (R == 0 || k == 0) continue;      // (a front without a boundary: nothing backward)
      const int g0 = dir == 0 ? add_gather(L, f, 0) : 0;
      for (int r = 0; r < R; r += L.rb)
        L.rows.push_back({dir == 0 ? f.L_off : f.W_off, f.idx_off, f.upd_off, dir == 0 ? f.ldL : f.ldW, r,
                          std::min(L.rb, R - r), k, f.nS, g0});
    }
  };
  const int KT = 128;                                  // columns of a split-K tile
  auto build_splitk = [&](NDLaunch& L, int h, int dir) {
    L.kind = 2;
    for (int t : plan.by_height[h]) {
      const NDFrontDev& f = plan.fronts[t];
      const int R = dir == 0 ? f.nF : f.nS, K = dir == 0 ? f.nS : f.nB;
      if (R == 0 || K == 0) continue;
      const int voff = add_gather(L, f, dir);
      const int nkt = (K + KT - 1) / KT;
      for (int r0 = 0; r0 < R; r0 += 256) {
        const int ps0 = (int)L.p_elems;
        for (int kt = 0; kt < nkt; ++kt) {
          L.tiles.push_back({t, r0, kt * KT, std::min(K, (kt + 1) * KT), (int)L.p_elems, voff});
          L.p_elems += 256;
        }
        L.rtiles.push_back({t, r0, nkt, ps0, voff, 0});
      }
    }
  };
  std::vector<NDLaunch> bwd;
  for (int h = 0; h <= plan.max_height; ++h) {
    for (int dir = 0; dir < 2; ++dir) {
      long long bytes = 0;
      int K = 0;
      for (int t : plan.by_height[h]) {
        const NDFrontDev& f = plan.fronts[t];
        bytes += (long long)(dir == 0 ? f.nF : f.nB) * f.nS * elem_bytes;
        K = std::max(K, dir == 0 ? f.nS : f.nB);
      }
      if (bytes == 0) continue;
      NDLaunch L;
      // Split-K is for heights of large blocks.  Many small fronts reach the bytes too, but fill
      // a fraction of a 256 x 128 tile and spread over the chip by themselves: up to
      // ND_SPLITK_COLS columns they take row blocks, which read such a block in one pass of 32 or
      // 64 rows (a coarsest solve in ms, from any column count / from 257 on: 8192^2 3.29 / 1.81,
      // 4096^2 0.79 / 0.51, 2048^2 compact 0.88 / 0.79, 256^3 FP64 1.52 / 1.43; from 65 to 2049 on
      // the others are level within 3 %).  A vector too long for a row block's LDS takes tiles
      // whatever the size.
      const bool large = bytes >= splitk_bytes && (K > ND_SPLITK_COLS || splitk_bytes == 0);
      const bool fits = nd_rows_lds(64, 16, K, 1, elem_bytes) <= ND_ROWS_LDS;
      if (large || !fits)
        build_splitk(L, h, dir);
      else
        build_rows(L, h, dir);
      (dir == 0 ? plan.fwd : bwd).push_back(L);
    }
  }
  plan.bwd.assign(bwd.rbegin(), bwd.rend());
}


}  // namespace helm
