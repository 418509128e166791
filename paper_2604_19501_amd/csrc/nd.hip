// Exact solve of the real-shifted coarsest operator A3 (eq. 3.6) on the GPU: the substitution
// with the factors of nd_factor.hip, in the cycle's precision (FP64 for the compact stack).
// Per right-hand side, forward over the nested-dissection tree bottom-up,
//     [g_S; t_B] = [A^-1; C A^-1] f_S,   u_B = v_B - t_B  (passed to the parent),
// then backward top-down,  x_S = g_S + (-A^-1 B) x_B.
#include <stdexcept>

#include "internal.h"

namespace helm {

// ----------------------------------------------------------------- solve ----
template <typename C>
__device__ __forceinline__ C cmul_conj(C a, C x, int conj) {   // (conj? conj(a) : a) * x
  if (conj) a.y = -a.y;
  return a * x;
}


// one entry of a gather list: r at the row's node (rid >= 0), the first two updates inline
// and the rest through cidx; every load of the first level is issued unconditionally
template <typename C>
__device__ __forceinline__ C gather_list(const NDGather& g, const int* __restrict__ cidx, const C* __restrict__ upd,
                                         const C* __restrict__ r) {
  typedef decltype(r[0].x) R;
  const C a = r[max(g.rid, 0)], u0 = upd[max(g.u0, 0)], u1 = upd[max(g.u1, 0)];
  C v = g.rid >= 0 ? a : mk((R)0, (R)0);
  if (g.u0 >= 0) v += u0;
  if (g.u1 >= 0) v += u1;
  for (int q = g.ca; q < g.cb; ++q) v += upd[cidx[q]];
  return v;
}

// f_S (and v_B) entry i of front f: right-hand side on S plus the children's updates
// (contribution list cptr[i] .. cptr[i+1] of absolute indices into the update pool); F is
// the front record or a work item carrying its fields
template <typename C, typename F>
__device__ __forceinline__ C gather_entry(const F& f, const int* __restrict__ cptr,
                                          const int* __restrict__ cidx, const int* __restrict__ id,
                                          const C* __restrict__ upd, const C* __restrict__ r, int i) {
  typedef decltype(r[0].x) R;
  C v = i < f.nS ? r[id[i]] : mk((R)0, (R)0);
  const int* cp = cptr + f.inv_off;
  const int a = cp[i], b = cp[i + 1];
  for (int q = a; q < b; ++q) v += upd[cidx[q]];
  return v;
}

__device__ __forceinline__ size_t al16(size_t v) { return (v + 15) & ~(size_t)15; }

// the five parts of a task's schedule copied to LDS in one pass: eight independent loads
// per thread and round before the stores (word w of the concatenation belongs to part r
// when end[r - 1] <= w < end[r])
struct LdsCopy5 {
  const int *s0, *s1, *s2, *s3, *s4;
  int *d0, *d1, *d2, *d3, *d4;
  int end[5];
};
__device__ __forceinline__ void copy_lds5(const LdsCopy5& c) {
  const int tot = c.end[4], bd = blockDim.x;
  for (int w0 = threadIdx.x; w0 < tot; w0 += 8 * bd) {
    int v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int w = min(w0 + q * bd, tot - 1);
      const int* sp = w < c.end[0] ? c.s0 + w
                    : w < c.end[1] ? c.s1 + (w - c.end[0])
                    : w < c.end[2] ? c.s2 + (w - c.end[1])
                    : w < c.end[3] ? c.s3 + (w - c.end[2])
                                   : c.s4 + (w - c.end[3]);
      v[q] = *sp;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int w = w0 + q * bd;
      if (w >= tot) continue;
      int* dp = w < c.end[0] ? c.d0 + w
              : w < c.end[1] ? c.d1 + (w - c.end[0])
              : w < c.end[2] ? c.d2 + (w - c.end[1])
              : w < c.end[3] ? c.d3 + (w - c.end[2])
                             : c.d4 + (w - c.end[3]);
      *dp = v[q];
    }
  }
}

// a segment is processed by a whole wavefront: keep its fields in scalar registers
__device__ __forceinline__ int ufl(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ NDSeg uniform_seg(NDSeg a) {
  NDSeg b;
  b.m_off = ((long long)ufl((int)(a.m_off >> 32)) << 32) | (unsigned)ufl((int)(a.m_off & 0xffffffffLL));
  b.ld = ufl(a.ld);
  b.r0 = ufl(a.r0);
  b.nr = ufl(a.nr);
  b.k0 = ufl(a.k0);
  b.k1 = ufl(a.k1);
  b.vslot = ufl(a.vslot);
  b.pslot = ufl(a.pslot);
  b.pad = 0;
  return b;
}

// A segment of at most 16 (32) rows spreads 4 (2) groups of 16 columns over the wavefront:
// lane l takes row l mod g and columns k0 + 16 (l / g) .. + 16, g = lanes per group.
__device__ __forceinline__ int seg_group(const NDSeg& sg) { return sg.nr <= 16 ? 16 : sg.nr <= 32 ? 32 : 64; }

// the 16 matrix entries of a segment for one lane (row and column indices clamped)
template <typename C>
__device__ __forceinline__ void load_seg(const C* __restrict__ M, const NDSeg& sg, int lane, C* m) {
  const int gs = seg_group(sg), kq = sg.k0 + (lane / gs) * 16;
  const C* col = M + sg.m_off + sg.r0 + min(lane & (gs - 1), sg.nr - 1);
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) m[kk] = col[(long long)min(kq + kk, sg.k1 - 1) * sg.ld];
}

// Tree-block substitution: one work-group per subtree task, one stage per level.
//   gathers:  vec[slot] = src[rid] (+ children's updates)           all threads
//   segments: partial products of <= 64 rows over <= 16 columns       one wavefront, two at a time
//             (<= 32 rows over <= 32 columns, <= 16 rows over <= 64 columns)
//   outputs:  sum of a row block's partials, write x or the update    one wavefront each
// forward (FWD = 1): M = L = [A^-1; C A^-1] (ld ldL), src = r;  rows < nS give x_S = g_S,
//                    rows >= nS the update v_B - C A^-1 f_S of the parent
// backward:          M = W = -A^-1 B (ld ldW), src = x (the boundary solution);  x_S += W x_B
// The task's schedule is copied to LDS first, so a stage costs two dependent global
// accesses (gathered values, matrix entries) besides its barriers.
template <typename C, int FWD>
__global__ void __launch_bounds__(1024) k_nd_tree(const NDTask* __restrict__ tasks,
                                                  const NDStage* __restrict__ stages,
                                                  const NDGather* __restrict__ gath, const NDSeg* __restrict__ segs,
                                                  const NDOut* __restrict__ outs, const int* __restrict__ dst,
                                                  const int* __restrict__ cidx, const C* __restrict__ M,
                                                  C* __restrict__ upd, const C* __restrict__ src,
                                                  C* __restrict__ x, int conj, NDRhs rh) {
  typedef decltype(src[0].x) R;
  extern __shared__ __align__(16) char smem[];
  upd += blockIdx.y * rh.upd;          // right-hand side blockIdx.y
  src += blockIdx.y * rh.vec;
  x += blockIdx.y * rh.vec;
  const NDTask T = tasks[blockIdx.x];
  const int nst = T.st1 - T.st0, ng = T.g1 - T.g0, nsg = T.s1 - T.s0, no = T.o1 - T.o0, nd = T.d1 - T.d0;
  char* p = smem;
  NDStage* lst = (NDStage*)p;
  p += al16(sizeof(NDStage) * nst);
  NDGather* lg = (NDGather*)p;
  p += al16(sizeof(NDGather) * ng);
  NDSeg* lsg = (NDSeg*)p;
  p += al16(sizeof(NDSeg) * nsg);
  NDOut* lo = (NDOut*)p;
  p += al16(sizeof(NDOut) * no);
  int* ldst = (int*)p;
  p += al16(sizeof(int) * nd);
  // values forwarded between the task's levels: forward, the update vectors of fronts whose
  // parent is in the task; backward, the solution x_S of fronts with a descendant in it
  C* lupd = (C*)p;
  p += al16(sizeof(C) * T.nlu);
  C* lsrc = (C*)p;                     // per gather: r (forward) or x from outside the task
  p += al16(sizeof(C) * ng);
  C* lxg = (C*)p;                      // backward: x_S before the update, per output row
  p += al16(sizeof(C) * (FWD ? 0 : nd));
  C* work = (C*)p;
  // the launch-invariant inputs of the first 2 x blockDim gathers (and backward outputs)
  // take their indices from the schedule in global memory, so their loads overlap the copy
  const int bd = blockDim.x, tid = threadIdx.x;
  C pre[2], prx[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    pre[j] = prx[j] = mk((R)0, (R)0);
    if (ng > 0) {
      const NDGather g = gath[T.g0 + min(tid + j * bd, ng - 1)];
      const C v = src[max(g.rid, 0)];
      pre[j] = g.rid >= 0 && (FWD || g.u0 == -1) ? v : mk((R)0, (R)0);
    }
    if (!FWD && nd > 0) prx[j] = x[max(dst[T.d0 + min(tid + j * bd, nd - 1)], 0)];
  }
  {
    LdsCopy5 c;
    c.s0 = (const int*)(stages + T.st0);
    c.s1 = (const int*)(gath + T.g0);
    c.s2 = (const int*)(segs + T.s0);
    c.s3 = (const int*)(outs + T.o0);
    c.s4 = dst + T.d0;
    c.d0 = (int*)lst;
    c.d1 = (int*)lg;
    c.d2 = (int*)lsg;
    c.d3 = (int*)lo;
    c.d4 = ldst;
    c.end[0] = (int)(sizeof(NDStage) / 4) * nst;
    c.end[1] = c.end[0] + (int)(sizeof(NDGather) / 4) * ng;
    c.end[2] = c.end[1] + (int)(sizeof(NDSeg) / 4) * nsg;
    c.end[3] = c.end[2] + (int)(sizeof(NDOut) / 4) * no;
    c.end[4] = c.end[3] + nd;
    copy_lds5(c);
  }
  __syncthreads();
  const int nw = blockDim.x >> 6, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // prefetching holds a second segment in registers: FP32 only (FP64 would spill).  The
  // first stage's segments are requested together with the launch-invariant inputs below.
  constexpr bool PF = sizeof(C) == 8;
  NDSeg psg;
  C pm[PF ? 16 : 1];
  bool have_pf = false;
  if (PF && nst > 0 && lst[0].s0 + wv < lst[0].s1) {
    psg = uniform_seg(lsg[lst[0].s0 + wv]);
    load_seg(M, psg, lane, pm);
    have_pf = true;
  }
  // every stage's inputs that do not change during the launch: r (forward); x of fronts
  // above the task and x_S before the update (backward)
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (tid + j * bd < ng) lsrc[tid + j * bd] = pre[j];
    if (!FWD && tid + j * bd < nd) lxg[tid + j * bd] = prx[j];
  }
  for (int e = tid + 2 * bd; e < ng; e += bd) {
    const NDGather g = lg[e];
    const C v = src[max(g.rid, 0)];
    lsrc[e] = g.rid >= 0 && (FWD || g.u0 == -1) ? v : mk((R)0, (R)0);
  }
  if (!FWD)
    for (int e = tid + 2 * bd; e < nd; e += bd) lxg[e] = x[max(ldst[e], 0)];
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const NDStage S = lst[st];
    // loads are unconditional (clamped indices, zero weights) so that a wavefront keeps
    // all of them in flight instead of waiting on each one
    for (int e = S.g0 + (int)threadIdx.x; e < S.g1; e += blockDim.x) {
      const NDGather g = lg[e];
      C v = mk((R)0, (R)0);
      if (FWD) {
        // rhs from LDS; contributions of the task's own fronts from LDS, of fronts below
        // the task (the previous launch) from global memory
        v = lsrc[e];
        if (g.u0 >= 0 || g.u1 >= 0) {
          const C u0 = upd[max(g.u0, 0)], u1 = upd[max(g.u1, 0)];
          if (g.u0 >= 0) v += u0;
          if (g.u1 >= 0) v += u1;
        }
        if (g.u0 <= -2) v += lupd[-g.u0 - 2];
        if (g.u1 <= -2) v += lupd[-g.u1 - 2];
        for (int q = g.ca; q < g.cb; ++q) v += upd[cidx[q]];
      } else {
        v = g.u0 <= -2 ? lupd[-g.u0 - 2] : lsrc[e];    // x_B: from a task level above, or prefetched
      }
      work[g.slot] = v;
    }
    __syncthreads();
    // one segment per wavefront at a time, 16 matrix loads in flight; the first segment of
    // a wavefront in a stage was prefetched during the previous stage (the matrix does not
    // depend on the previous stage's results)
    for (int s0 = S.s0 + wv; s0 < S.s1; s0 += nw) {
      NDSeg sg;
      C mv[16];
      if (PF && s0 == S.s0 + wv && have_pf) {
        sg = psg;
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) mv[kk] = pm[PF ? kk : 0];
      } else {
        sg = uniform_seg(lsg[s0]);
        load_seg(M, sg, lane, mv);
      }
      const int gs = seg_group(sg), kq = sg.k0 + (lane / gs) * 16;
      C acc = mk((R)0, (R)0);
#pragma unroll
      for (int kk = 0; kk < 16; ++kk)
        if (kq + kk < sg.k1) acc += cmul_conj(mv[kk], work[sg.vslot + kq + kk], conj);
      for (int o = gs; o < 64; o <<= 1) {      // sum the column groups (every lane gets its row's sum)
        acc.x += __shfl_xor(acc.x, o, 64);
        acc.y += __shfl_xor(acc.y, o, 64);
      }
      work[sg.pslot + lane] = acc;
    }
    // prefetch this wavefront's first segment of the next stage
    have_pf = false;
    if (PF && st + 1 < nst) {
      const NDStage S2 = lst[st + 1];
      if (S2.s0 + wv < S2.s1) {
        psg = uniform_seg(lsg[S2.s0 + wv]);
        load_seg(M, psg, lane, pm);
        have_pf = true;
      }
    }
    __syncthreads();
    for (int o = S.o0 + wv; o < S.o1; o += nw) {
      const NDOut ob = lo[o];
      if (lane < ob.nr) {
        C acc = mk((R)0, (R)0);
        for (int q = 0; q < ob.nparts; ++q) acc += work[ob.pslot + 64 * q + lane];
        const int d = ldst[ob.d + lane];
        if (FWD) {
          if (d >= 0) {
            x[d] = acc;
          } else {
            const C u = work[ob.vslot + ob.r0 + lane] - acc;
            upd[-d - 1] = u;
            if (ob.lu_on) lupd[ob.lu + lane] = u;   // row >= nS: read by the parent's gather
          }
        } else {
          const C nx = lxg[ob.d + lane] + acc;
          x[d] = nx;
          if (ob.lu_on) lupd[ob.lu + lane] = nx;     // read by the gathers of lower levels
        }
      }
    }
    __syncthreads();
  }
}

// rows [r0, r1) (at most 16) of a big front: 16 row lanes x KS (16 or 64) k-splits per
// work-group, partial sums reduced through LDS; consecutive threads read consecutive rows
// of one column.  gemv16_load issues the thread's first 16 matrix entries, which do not
// depend on v, so callers start it before gathering v; gemv16_finish does the rest.
template <typename C, int KS = 16>
__device__ __forceinline__ void gemv16_load(const C* __restrict__ M, long long ld, int r0, int r1, int K, C* m) {
  const int row = threadIdx.x & 15, ks = threadIdx.x >> 4;
  const int kq = (K + KS - 1) / KS, kb = ks * kq, ke = min(K, kb + kq);
  const C* col = M + min(r0 + row, r1 - 1);
#pragma unroll
  for (int q = 0; q < 16; ++q) m[q] = col[(long long)max(0, min(kb + q, ke - 1)) * ld];
}
template <typename C, int KS = 16>
__device__ __forceinline__ C gemv16_finish(const C* __restrict__ M, long long ld, int r0, int r1, int K,
                                           const C* __restrict__ v, int conj, C* red, const C* m0) {
  typedef decltype(v[0].x) R;
  const int row = threadIdx.x & 15, ks = threadIdx.x >> 4;
  const int i = r0 + row;
  const int kq = (K + KS - 1) / KS, kb = ks * kq, ke = min(K, kb + kq);
  C acc = mk((R)0, (R)0);
  if (i < r1 && kb < ke) {
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (kb + q < ke) acc += cmul_conj(m0[q], v[kb + q], conj);
    // 16 matrix entries in flight per thread: load all (clamped), then accumulate
    const C* col = M + i;
    for (int k = kb + 16; k < ke; k += 16) {
      C m[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) m[q] = col[(long long)min(k + q, ke - 1) * ld];
#pragma unroll
      for (int q = 0; q < 16; ++q)
        if (k + q < ke) acc += cmul_conj(m[q], v[k + q], conj);
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (KS > 16) {                       // fold the k-splits 16 apart onto the first 256 threads
    C t = mk((R)0, (R)0);
    if (threadIdx.x < 256) {
      t = red[threadIdx.x];
#pragma unroll
      for (int g = 1; g < KS / 16; ++g) t += red[threadIdx.x + 256 * g];
    }
    __syncthreads();
    if (threadIdx.x < 256) red[threadIdx.x] = t;
    __syncthreads();
  }
  C tot = mk((R)0, (R)0);
  if (threadIdx.x < 16)
    for (int q = 0; q < 16; ++q) tot += red[q * 16 + threadIdx.x];
  return tot;
}

// forward substitution, big fronts: one work-group per chunk of at most 16 rows; KS = 64
// (1024 threads) as for the backward substitution
template <typename C, int KS>
__global__ void __launch_bounds__(16 * KS) k_nd_fwd_big(const NDGather* __restrict__ gath, const int* __restrict__ idx,
                                                         const int* __restrict__ cidx, const C* __restrict__ Lp,
                                                         C* __restrict__ upd, const NDItem* __restrict__ items,
                                                         const C* __restrict__ r, C* __restrict__ x,
                                                         C* __restrict__ gvec, int cap, int conj, NDRhs rh) {
  extern __shared__ char smem[];
  __shared__ C red[16 * KS];
  upd += blockIdx.y * rh.upd;
  r += blockIdx.y * rh.vec;
  x += blockIdx.y * rh.vec;
  C* vec = gvec ? gvec + blockIdx.y * rh.gvec + (long long)blockIdx.x * cap : (C*)smem;
  const NDItem f = items[blockIdx.x];
  const int* id = idx + f.idx_off;
  C m0[16];
  gemv16_load<C, KS>(Lp + f.m_off, f.ld, f.r0, f.r1, f.nS, m0);
  const NDGather* gl = gath + f.g0;
  for (int i = threadIdx.x; i < f.nS; i += 16 * KS) vec[i] = gather_list(gl[i], cidx, upd, r);
  for (int i = max(f.r0, f.nS) + threadIdx.x; i < f.r1; i += 16 * KS) vec[i] = gather_list(gl[i], cidx, upd, r);
  __syncthreads();
  C acc = gemv16_finish<C, KS>(Lp + f.m_off, f.ld, f.r0, f.r1, f.nS, vec, conj, red, m0);
  const int i = f.r0 + threadIdx.x;
  if (threadIdx.x < 16 && i < f.r1) {
    if (i < f.nS)
      x[id[i]] = acc;
    else
      upd[f.upd_off + i - f.nS] = vec[i] - acc;
  }
}

// backward substitution, big fronts: one work-group per chunk of at most 16 rows; KS = 64
// (1024 threads) for launches whose vectors exceed 256 entries and whose work-groups fit
// the chip at once (see big_threads), so that the gather of x_B takes one pass and a
// thread's k-slice one batch of loads
template <typename C, int KS>
__global__ void __launch_bounds__(16 * KS) k_nd_bwd_big(const NDFrontDev* __restrict__ fr, const int* __restrict__ idx,
                                                         const C* __restrict__ Wp, const NDItem* __restrict__ items,
                                                         C* __restrict__ x, C* __restrict__ gvec, int cap, int conj,
                                                         NDRhs rh) {
  extern __shared__ char smem[];
  __shared__ C red[16 * KS];
  x += blockIdx.y * rh.vec;
  C* vec = gvec ? gvec + blockIdx.y * rh.gvec + (long long)blockIdx.x * cap : (C*)smem;
  const NDItem f = items[blockIdx.x];
  const int* id = idx + f.idx_off;
  C m0[16];
  gemv16_load<C, KS>(Wp + f.m_off, f.ld, f.r0, f.r1, f.nB, m0);
  const int i = f.r0 + threadIdx.x;
  const int di = threadIdx.x < 16 && i < f.r1 ? id[i] : 0;
  for (int j = threadIdx.x; j < f.nB; j += 16 * KS) vec[j] = x[id[f.nS + j]];
  __syncthreads();
  C acc = gemv16_finish<C, KS>(Wp + f.m_off, f.ld, f.r0, f.r1, f.nB, vec, conj, red, m0);
  if (threadIdx.x < 16 && i < f.r1) x[di] = x[di] + acc;
}

// ---- split-K launches (kind 3) -------------------------------------------
// P[pslot + t] = sum_{k0 <= k < k1} M[k ld + r0 + t] vec[k]: one row per thread, 16 loads in
// flight.  The tile gathers its own k-slice of the front's input vector from the gather list
// (entry voff + k is the front's entry k), so no separate gather launch and buffer pass is
// needed; tiles of the same k-slice repeat its 128 gathers, which are small beside the
// 256 x 128 matrix block each of them streams.
template <typename C, int FWD>
__global__ void __launch_bounds__(256) k_nd_tile(const NDFrontDev* __restrict__ fr, const C* __restrict__ Mp,
                                                 const NDTile* __restrict__ tiles, const NDGather* __restrict__ gath,
                                                 const int* __restrict__ cidx, const C* __restrict__ upd,
                                                 const C* __restrict__ src, C* __restrict__ P, int conj, NDRhs rh) {
  typedef decltype(src[0].x) R;
  __shared__ C vec[128];
  upd += blockIdx.y * rh.upd;
  src += blockIdx.y * rh.vec;
  P += blockIdx.y * rh.part;
  const NDTile t = tiles[blockIdx.x];
  const NDFrontDev f = fr[t.front];
  const int ld = FWD ? f.ldL : f.ldW, rows = FWD ? f.nF : f.nS;
  const int nk = t.k1 - t.k0;
  const int i = min(t.r0 + (int)threadIdx.x, rows - 1);
  const C* col = Mp + (FWD ? f.L_off : f.W_off) + (long long)t.k0 * ld + i;
  // the first 16 matrix entries do not depend on the gathered slice: request them first
  C m0[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) m0[q] = col[(long long)min(q, nk - 1) * ld];
  if ((int)threadIdx.x < nk) vec[threadIdx.x] = gather_list(gath[t.voff + t.k0 + threadIdx.x], cidx, upd, src);
  __syncthreads();
  C acc = mk((R)0, (R)0);
#pragma unroll
  for (int q = 0; q < 16; ++q)
    if (q < nk) acc += cmul_conj(m0[q], vec[q], conj);
  for (int k = 16; k < nk; k += 16) {
    C m[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) m[q] = col[(long long)min(k + q, nk - 1) * ld];
#pragma unroll
    for (int q = 0; q < 16; ++q)
      if (k + q < nk) acc += cmul_conj(m[q], vec[k + q], conj);
  }
  P[t.pslot + threadIdx.x] = acc;
}

// rows of a row tile: the partials summed in k order, then x (or the update) written; the
// forward update rows gather their own input entry
template <typename C, int FWD>
__global__ void __launch_bounds__(256) k_nd_rowsum(const NDFrontDev* __restrict__ fr, const int* __restrict__ idx,
                                                   const NDRowTile* __restrict__ rt, const C* __restrict__ P,
                                                   const NDGather* __restrict__ gath, const int* __restrict__ cidx,
                                                   const C* __restrict__ src, C* __restrict__ upd,
                                                   C* __restrict__ x, NDRhs rh) {
  typedef decltype(src[0].x) R;
  P += blockIdx.y * rh.part;
  upd += blockIdx.y * rh.upd;
  src += blockIdx.y * rh.vec;
  x += blockIdx.y * rh.vec;
  const NDRowTile t = rt[blockIdx.x];
  const NDFrontDev f = fr[t.front];
  const int i = t.r0 + threadIdx.x;
  if (i >= (FWD ? f.nF : f.nS)) return;
  C acc = mk((R)0, (R)0);
  // in k order; groups of 8 loads are issued before their sums, so they are in flight together
  const C* pp = P + t.pslot + threadIdx.x;
  int q = 0;
  for (; q + 8 <= t.nkt; q += 8) {
    C v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = pp[256 * (q + u)];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += v[u];
  }
  for (; q < t.nkt; ++q) acc += pp[256 * q];
  if (FWD) {
    if (i < f.nS)
      x[idx[f.idx_off + i]] = acc;
    else
      upd[f.upd_off + i - f.nS] = gather_list(gath[t.voff + i], cidx, (const C*)upd, src) - acc;
  } else {
    const int id = idx[f.idx_off + i];
    x[id] = x[id] + acc;
  }
}

template <typename C, int FWD>
static void splitk(const NDLaunchDev& L, const NDFrontDev* fr, const int* idx, const int* cidx, const C* M, C* upd,
                   const C* src, C* x, C* P, int conj, const NDRhs& rh, hipStream_t s) {
  hipLaunchKernelGGL((k_nd_tile<C, FWD>), dim3(L.ntiles, rh.n), dim3(256), 0, s, fr, M, L.tiles, L.gath, cidx,
                     (const C*)upd, src, P, conj, rh);
  hipLaunchKernelGGL((k_nd_rowsum<C, FWD>), dim3(L.nrt, rh.n), dim3(256), 0, s, fr, idx, L.rtiles, (const C*)P,
                     L.gath, cidx, src, upd, x, rh);
}

// ------------------------------------------------------------- launchers ----
// LDS bytes above the default limit need the attribute on the kernel
template <typename C, int FWD>
static void tree_attr(size_t lds) {
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_nd_tree<C, FWD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// threads of a row-chunk launch: 1024 (64 k-splits) where the plan marks its vectors as
// longer than 256 entries and at most 512 work-groups run (two 16-wavefront work-groups
// per CU: one generation); otherwise 256.  A second generation doubles the launch's
// latency, which cost more than the shorter gather and k-slices save.
static int big_threads(const NDLaunchDev& L, const NDRhs& rh) {
  return L.threads == 1024 && (long long)L.ntasks * rh.n <= 512 ? 1024 : 256;
}

template <typename C>
void nd_fwd(const NDLaunchDev& L, const NDFrontDev* fr, const int* idx, const int* cptr, const int* cidx,
            const C* Lp, C* upd, const C* r, C* x, C* gvec, int cap, int conj, C* P, const NDRhs& rh,
            hipStream_t s) {
  if (L.kind == 3) {
    splitk<C, 1>(L, fr, idx, cidx, Lp, upd, r, x, P, conj, rh, s);
  } else if (L.kind == 2) {
    size_t lds = (size_t)L.lds_bytes;
    tree_attr<C, 1>(lds);
    hipLaunchKernelGGL((k_nd_tree<C, 1>), dim3(L.ntasks, rh.n), dim3(L.threads), lds, s, L.tasks, L.stages, L.gath,
                       L.segs, L.outs, L.dst, cidx, Lp, upd, r, x, conj, rh);
  } else {
    if (big_threads(L, rh) == 1024)
      hipLaunchKernelGGL((k_nd_fwd_big<C, 64>), dim3(L.ntasks, rh.n), dim3(1024), L.shm, s, L.gath, idx, cidx, Lp,
                         upd, L.items, r, x, gvec, cap, conj, rh);
    else
      hipLaunchKernelGGL((k_nd_fwd_big<C, 16>), dim3(L.ntasks, rh.n), dim3(256), L.shm, s, L.gath, idx, cidx, Lp,
                         upd, L.items, r, x, gvec, cap, conj, rh);
  }
}
template <typename C>
void nd_bwd(const NDLaunchDev& L, const NDFrontDev* fr, const int* idx, const int* cidx, const C* Wp, C* upd, C* x,
            C* gvec, int cap, int conj, C* P, const NDRhs& rh, hipStream_t s) {
  if (L.kind == 3) {
    splitk<C, 0>(L, fr, idx, cidx, Wp, upd, (const C*)x, x, P, conj, rh, s);
  } else if (L.kind == 2) {
    size_t lds = (size_t)L.lds_bytes;
    tree_attr<C, 0>(lds);
    hipLaunchKernelGGL((k_nd_tree<C, 0>), dim3(L.ntasks, rh.n), dim3(L.threads), lds, s, L.tasks, L.stages, L.gath,
                       L.segs, L.outs, L.dst, cidx, Wp, upd, (const C*)x, x, conj, rh);
  } else {
    if (big_threads(L, rh) == 1024)
      hipLaunchKernelGGL((k_nd_bwd_big<C, 64>), dim3(L.ntasks, rh.n), dim3(1024), L.shm, s, fr, idx, Wp, L.items, x,
                         gvec, cap, conj, rh);
    else
      hipLaunchKernelGGL((k_nd_bwd_big<C, 16>), dim3(L.ntasks, rh.n), dim3(256), L.shm, s, fr, idx, Wp, L.items, x,
                         gvec, cap, conj, rh);
  }
}

template void nd_fwd<cf>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const int*, const cf*, cf*,
                         const cf*, cf*, cf*, int, int, cf*, const NDRhs&, hipStream_t);
template void nd_fwd<cd>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const int*, const cd*, cd*,
                         const cd*, cd*, cd*, int, int, cd*, const NDRhs&, hipStream_t);
template void nd_bwd<cf>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const cf*, cf*, cf*, cf*, int,
                         int, cf*, const NDRhs&, hipStream_t);
template void nd_bwd<cd>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const cd*, cd*, cd*, cd*, int,
                         int, cd*, const NDRhs&, hipStream_t);


}  // namespace helm
