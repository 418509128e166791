// Exact solve of the real-shifted coarsest operator A3 (eq. 3.6) on the GPU: the substitution
// with the factors of nd_factor.hip, in the cycle's precision (FP64 for the compact stack).
// Per right-hand side, forward over the nested-dissection tree bottom-up,
//     [g_S; t_B] = [A^-1; C A^-1] f_S,   u_B = v_B - t_B  (passed to the parent),
// then backward top-down,  x_S = g_S + (-A^-1 B) x_B.
#include <stdexcept>

#include "internal.h"

namespace helm {

// ----------------------------------------------------------------- solve ----
__device__ __forceinline__ int ufl(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <typename C>
__device__ __forceinline__ C cmul_conj(C a, C x, int conj) {   // (conj? conj(a) : a) * x
  if (conj) a.y = -a.y;
  return a * x;
}


// ---- row blocks ------------------------------------------
// an entry of a gather list for NR right-hand sides (vectors sv and updates su entries apart;
// past the nq-th they repeat it): r at the entry's node, the first four updates inline and the
// rest through cidx.  Every load of the first level is in flight together; with several
// right-hand sides, where traffic counts more than one entry's latency, the third and fourth
// update (few entries have them) are loaded where they exist.
template <typename C, int NR>
__device__ __forceinline__ void gather_n(const NDGather& g, const int* __restrict__ cidx, const C* __restrict__ upd,
                                         const C* __restrict__ src, long long su, long long sv, int nq, C* v) {
  typedef decltype(src[0].x) R;
  constexpr int NI = NR == 1 ? 4 : 2;
  const int gu[4] = {g.u0, g.u1, g.u2, g.u3};
  C a[NR], u[NR][NI];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int qq = min(q, nq - 1);
    a[q] = src[qq * sv + max(g.rid, 0)];
#pragma unroll
    for (int i = 0; i < NI; ++i) u[q][i] = upd[qq * su + max(gu[i], 0)];
  }
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    v[q] = g.rid >= 0 ? a[q] : mk((R)0, (R)0);
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (gu[i] >= 0) v[q] += u[q][i];
  }
#pragma unroll
  for (int i = NI; i < 4; ++i)
    if (gu[i] >= 0) {
#pragma unroll
      for (int q = 0; q < NR; ++q) v[q] += upd[min(q, nq - 1) * su + gu[i]];
    }
  for (int c = g.ca; c < g.cb; ++c) {
    const int id = cidx[c];
#pragma unroll
    for (int q = 0; q < NR; ++q) v[q] += upd[min(q, nq - 1) * su + id];
  }
}

// One item (RB rows of a front) per W wavefronts; a wave covers RB rows x 64 / RB groups of 16
// columns at a time.  Bound by its chain of dependent accesses (item, gather record, gathered
// values, products, the waves' sums through LDS), 5 to 9 us a launch at 1024^2: everything
// that does not depend on the vector (a lane's first 16 entries, the rows' own inputs) is
// requested before the gather.  NR right-hand sides share the matrix entries: separately they
// read them from L2 or the last-level cache once each.  Against work-groups that walked whole
// subtrees with their schedule in LDS, and 16-row chunks above them, both one right-hand side
// per work-group: 600x640 FP64 255 -> 181 us per FGMRES iteration (with the levels merged that this
// kernel's one launch per level makes worth merging), 256^3 3.83 -> 3.66 ms, 192x192x72 compact
// 2.09 -> 1.81 ms, a batch of 6 media x 8 sources 205 -> 168 ms; 1024^2 level (260 us).
template <typename C, int RB, int NR, int FWD>
__global__ void __launch_bounds__(1024) k_nd_rows(const NDRow* __restrict__ rows, int nrows, int W, int vcap,
                                                  const NDGather* __restrict__ gath, const int* __restrict__ idx,
                                                  const int* __restrict__ cidx, const C* __restrict__ M,
                                                  C* __restrict__ upd, const C* __restrict__ src, C* __restrict__ x,
                                                  int conj, NDRhs rh) {
  typedef decltype(src[0].x) R;
  constexpr int U = 16, CG = 64 / RB, NO = NR > CG ? NR / CG : 1;   // NO: outputs of a thread, at most
  extern __shared__ __align__(16) char smem[];
  const int lane = threadIdx.x & 63, wv = ufl(threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
  const int ipw = nw / W, li = wv / W, w = wv % W;
  const int item = blockIdx.x * ipw + li;
  C* vec = (C*)smem + (long long)li * vcap * NR;
  C* part = (C*)smem + (long long)ipw * vcap * NR + (long long)li * W * RB * NR;
  const int q0 = blockIdx.y * NR, nq = min(NR, rh.n - q0);
  upd += q0 * rh.upd;
  src += q0 * rh.vec;
  x += q0 * rh.vec;
  const NDRow it = rows[min(item, nrows - 1)];
  const bool live = item < nrows;
  const int row = lane & (RB - 1), g = lane / RB;
  const C* __restrict__ col = M + it.m_off + it.r0 + min(row, it.nr - 1);
  // a lane's first 16 matrix entries do not depend on the vector
  C m[U];
  int kq = (w * CG + g) * U;
#pragma unroll
  for (int u = 0; u < U; ++u) m[u] = col[(long long)min(kq + u, it.K - 1) * it.ld];
  // this thread's outputs: its row of right-hand sides (w CG + g) + j W CG, j < NO
  const int orow = it.r0 + min(row, it.nr - 1);
  NDGather og;
  int oid = 0;
  if (FWD) og = gath[it.g0 + orow];
  else oid = idx[it.idx_off + orow];
  for (int k = w * 64 + lane; k < it.K; k += 64 * W) {
    if (FWD) {
      C v[NR];
      gather_n<C, NR>(gath[it.g0 + k], cidx, (const C*)upd, src, rh.upd, rh.vec, nq, v);
#pragma unroll
      for (int q = 0; q < NR; ++q) vec[k * NR + q] = v[q];
    } else {
      const int id = idx[it.idx_off + it.nS + k];
      C v[NR];
#pragma unroll
      for (int q = 0; q < NR; ++q) v[q] = src[min(q, nq - 1) * rh.vec + id];
#pragma unroll
      for (int q = 0; q < NR; ++q) vec[k * NR + q] = v[q];
    }
  }
  C ov[NO];
  const int oq = w * CG + g;
  if (FWD) {
    oid = og.rid;
    if (og.rid < 0) {
      // update rows: v_B of this thread's right-hand sides
#pragma unroll
      for (int j = 0; j < NO; ++j) {
        const int q = min(oq + j * W * CG, nq - 1);
        gather_n<C, 1>(og, cidx, (const C*)upd + q * rh.upd, src + q * rh.vec, 0, 0, 1, &ov[j]);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < NO; ++j) ov[j] = x[min(oq + j * W * CG, nq - 1) * rh.vec + oid];
  }
  __syncthreads();
  C acc[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) acc[q] = mk((R)0, (R)0);
  while (true) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (kq + u < it.K) {
#pragma unroll
        for (int q = 0; q < NR; ++q) acc[q] += cmul_conj(m[u], vec[(kq + u) * NR + q], conj);
      }
    }
    kq += W * CG * U;
    if (kq - g * U >= it.K) break;              // uniform over the wave
#pragma unroll
    for (int u = 0; u < U; ++u) m[u] = col[(long long)min(kq + u, it.K - 1) * it.ld];
  }
#pragma unroll
  for (int q = 0; q < NR; ++q) {
#pragma unroll
    for (int o = RB; o < 64; o <<= 1) {
      acc[q].x += __shfl_xor(acc[q].x, o, 64);
      acc[q].y += __shfl_xor(acc[q].y, o, 64);
    }
    if (g == 0) part[(w * NR + q) * RB + row] = acc[q];
  }
  __syncthreads();
  if (!live || row >= it.nr) return;
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    const int q = oq + j * W * CG;
    if (q >= nq) continue;
    C s = part[q * RB + row];
#pragma unroll 4
    for (int v = 1; v < W; ++v) s += part[(v * NR + q) * RB + row];
    if (!FWD)
      x[q * rh.vec + oid] = ov[j] + s;
    else if (oid >= 0)
      x[q * rh.vec + oid] = s;
    else
      upd[q * rh.upd + it.upd_off + it.r0 + row - it.nS] = ov[j] - s;
  }
}

template <typename C, int RB, int NR, int FWD>
static void launch_rows(const NDLaunchDev& L, const int* idx, const int* cidx, const C* M, C* upd, const C* src, C* x,
                        int conj, const NDRhs& rh, hipStream_t s) {
  const int ipw = std::max(1, 4 / L.waves), threads = 64 * ipw * L.waves;
  const size_t lds = nd_rows_lds(RB, L.waves, L.max_k, NR, sizeof(C));
  if (lds > 65536)
    (void)hipFuncSetAttribute((const void*)k_nd_rows<C, RB, NR, FWD>, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
  hipLaunchKernelGGL((k_nd_rows<C, RB, NR, FWD>), dim3((L.nrows + ipw - 1) / ipw, (rh.n + NR - 1) / NR), dim3(threads),
                     lds, s, L.rows, L.nrows, L.waves, L.max_k, L.gath, idx, cidx, M, upd, src, x, conj, rh);
}
template <typename C, int RB, int FWD>
static void rows_nr(const NDLaunchDev& L, const int* idx, const int* cidx, const C* M, C* upd, const C* src, C* x,
                    int conj, const NDRhs& rh, hipStream_t s) {
  // In FP64 at most 2: with 16 waves of 128 registers, 8 spill 100 of them and 4 spill 13 (us per
  // iteration of 9 right-hand sides, at most 8 / 4 / 2 / 1: 300^2 273 / 230 / 218 / 220, 800^2 1196 /
  // 991 / 974 / 1061, 72^3 846 / 737 / 707 / 743, 112^3 3240 / 2963 / 2926 / 3071; of 2: 800^2 - / - /
  // 327 / 348).  FP32 has no spills: 8 and 4 differ by 4 % at most, either way.
  constexpr int MAX_NR = sizeof(C) == sizeof(cf) ? 8 : 2;
  int nr = std::min(MAX_NR, rh.n >= 5 ? 8 : rh.n >= 3 ? 4 : rh.n);
  // Right-hand sides that share a work-group read each entry once, but make its chain longer: they
  // share only while the launch has 128 work-groups (us per FGMRES iteration of 8 right-hand sides,
  // shared always / with this line / with 256: 64^2 68 / 63 / 62, 96^2 77 / 69 / 76, 200^2 132 / 114 /
  // 123, 300^2 202 / 181 / 177, 32^3 179 / 148 / 149, 48^3 295 / 259 / 256; batches of 2 media x 7
  // on 580^2 13.1 / 12.0 / 12.0 ms, on 160^2 1.88 / 1.82 / 2.08)
  const int ipw = std::max(1, 4 / L.waves), blocks = (L.nrows + ipw - 1) / ipw;
  while (nr > 1 && blocks * ((rh.n + nr - 1) / nr) < 128) nr /= 2;
  while (nr > 1 && nd_rows_lds(RB, L.waves, L.max_k, nr, sizeof(C)) > 65536) nr /= 2;
  if constexpr (MAX_NR == 8) {
    if (nr == 8) return launch_rows<C, RB, 8, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
    if (nr == 4) return launch_rows<C, RB, 4, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
  }
  if (nr == 2) launch_rows<C, RB, 2, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
  else launch_rows<C, RB, 1, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
}
template <typename C, int FWD>
static void rows_launch(const NDLaunchDev& L, const int* idx, const int* cidx, const C* M, C* upd, const C* src, C* x,
                        int conj, const NDRhs& rh, hipStream_t s) {
  if (L.rb == 64) rows_nr<C, 64, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
  else if (L.rb == 32) rows_nr<C, 32, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
  else rows_nr<C, 16, FWD>(L, idx, cidx, M, upd, src, x, conj, rh, s);
}

// ---- split-K ------------------------------------------------------------
// P[pslot + t] = sum_{k0 <= k < k1} M[k ld + r0 + t] vec[k]: one row per thread, 16 loads in
// flight.  The tile gathers its own k-slice of the front's input vector from the gather list
// (entry voff + k is the front's entry k), so no separate gather launch and buffer pass is
// needed; tiles of the same k-slice repeat its 128 gathers, which are small beside the
// 256 x 128 matrix block each of them streams.  NR right-hand sides share the matrix entries.
template <typename C, int NR, int FWD>
__global__ void __launch_bounds__(256) k_nd_tile(const NDFrontDev* __restrict__ fr, const C* __restrict__ Mp,
                                                 const NDTile* __restrict__ tiles, const NDGather* __restrict__ gath,
                                                 const int* __restrict__ cidx, const C* __restrict__ upd,
                                                 const C* __restrict__ src, C* __restrict__ P, int conj, NDRhs rh) {
  typedef decltype(src[0].x) R;
  __shared__ C vec[128 * NR];
  const int q0 = blockIdx.y * NR, nq = min(NR, rh.n - q0);
  upd += q0 * rh.upd;
  src += q0 * rh.vec;
  P += q0 * rh.part;
  const NDTile t = tiles[blockIdx.x];
  const NDFrontDev f = fr[t.front];
  const int ld = FWD ? f.ldL : f.ldW, rows = FWD ? f.nF : f.nS;
  const int nk = t.k1 - t.k0;
  const int i = min(t.r0 + (int)threadIdx.x, rows - 1);
  const C* col = Mp + (FWD ? f.L_off : f.W_off) + (long long)t.k0 * ld + i;
  // the first 16 matrix entries do not depend on the gathered slice: request them first
  C m[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) m[u] = col[(long long)min(u, nk - 1) * ld];
  if ((int)threadIdx.x < nk) {
    C v[NR];
    gather_n<C, NR>(gath[t.voff + t.k0 + threadIdx.x], cidx, upd, src, rh.upd, rh.vec, nq, v);
#pragma unroll
    for (int q = 0; q < NR; ++q) vec[threadIdx.x * NR + q] = v[q];
  }
  __syncthreads();
  C acc[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) acc[q] = mk((R)0, (R)0);
  for (int k = 0;;) {
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (k + u < nk) {
#pragma unroll
        for (int q = 0; q < NR; ++q) acc[q] += cmul_conj(m[u], vec[(k + u) * NR + q], conj);
      }
    k += 16;
    if (k >= nk) break;
#pragma unroll
    for (int u = 0; u < 16; ++u) m[u] = col[(long long)min(k + u, nk - 1) * ld];
  }
#pragma unroll
  for (int q = 0; q < NR; ++q)
    if (q < nq) P[q * rh.part + t.pslot + threadIdx.x] = acc[q];
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
    if (i < f.nS) {
      x[idx[f.idx_off + i]] = acc;
    } else {
      C v;
      gather_n<C, 1>(gath[t.voff + i], cidx, (const C*)upd, src, 0, 0, 1, &v);
      upd[f.upd_off + i - f.nS] = v - acc;
    }
  } else {
    const int id = idx[f.idx_off + i];
    x[id] = x[id] + acc;
  }
}

template <typename C, int FWD>
static void splitk(const NDLaunchDev& L, const NDFrontDev* fr, const int* idx, const int* cidx, const C* M, C* upd,
                   const C* src, C* x, C* P, int conj, const NDRhs& rh, hipStream_t s) {
  const C* u = upd;
#define TILE(NR)                                                                                              \
  hipLaunchKernelGGL((k_nd_tile<C, NR, FWD>), dim3(L.ntiles, (rh.n + NR - 1) / NR), dim3(256), 0, s, fr, M, L.tiles, \
                     L.gath, cidx, u, src, P, conj, rh)
  if (rh.n >= 5) TILE(8);
  else if (rh.n >= 3) TILE(4);
  else if (rh.n == 2) TILE(2);
  else TILE(1);
#undef TILE
  hipLaunchKernelGGL((k_nd_rowsum<C, FWD>), dim3(L.nrt, rh.n), dim3(256), 0, s, fr, idx, L.rtiles, (const C*)P,
                     L.gath, cidx, src, upd, x, rh);
}

template <typename C>
void nd_fwd(const NDLaunchDev& L, const NDFrontDev* fr, const int* idx, const int* cidx, const C* Lp, C* upd,
            const C* r, C* x, int conj, C* P, const NDRhs& rh, hipStream_t s) {
  if (L.kind == 2)
    splitk<C, 1>(L, fr, idx, cidx, Lp, upd, r, x, P, conj, rh, s);
  else
    rows_launch<C, 1>(L, idx, cidx, Lp, upd, r, x, conj, rh, s);
}
template <typename C>
void nd_bwd(const NDLaunchDev& L, const NDFrontDev* fr, const int* idx, const int* cidx, const C* Wp, C* upd, C* x,
            int conj, C* P, const NDRhs& rh, hipStream_t s) {
  if (L.kind == 2)
    splitk<C, 0>(L, fr, idx, cidx, Wp, upd, (const C*)x, x, P, conj, rh, s);
  else
    rows_launch<C, 0>(L, idx, cidx, Wp, upd, (const C*)x, x, conj, rh, s);
}

template void nd_fwd<cf>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const cf*, cf*, const cf*, cf*,
                         int, cf*, const NDRhs&, hipStream_t);
template void nd_fwd<cd>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const cd*, cd*, const cd*, cd*,
                         int, cd*, const NDRhs&, hipStream_t);
template void nd_bwd<cf>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const cf*, cf*, cf*, int, cf*,
                         const NDRhs&, hipStream_t);
template void nd_bwd<cd>(const NDLaunchDev&, const NDFrontDev*, const int*, const int*, const cd*, cd*, cd*, int, cd*,
                         const NDRhs&, hipStream_t);

}  // namespace helm
