// Galerkin coarse operators (setup, FP64).
//
//   A2 = R1 H_s P1          eq. (2.2), s = alpha2^2 (1 - i beta) omega^2
//   A3 = R2 (R1 H_s' P1) P2 eq. (3.6), s' = alpha^2 (1 - i beta) omega^2 (real shift, eq. (3.5))
//
// R is full weighting ([1 2 1]/4 per axis, truncated at the ends) and P = 2^d R^T
// (d-linear interpolation).  For every coarse node I the kernels form the row
//   A_c(I, J) = sum_f R(I, f) sum_g A(f, g) P(g, J),  J - I in {-1, 0, 1}^d,
// over the restriction footprint f, the fine stencil g = f + t and the (at most 2^d)
// interpolation parents J of g.  Output: 3^d complex coefficients per coarse node, structure
// of arrays, offset k = (d0+1) + 3 (d1+1) + 9 (d2+1).
#include "internal.h"

namespace helm {

// a * P(g, J) into acc[J - I] for the parents J of the fine node g = 2 I + (d0, d1, d2),
// -2 <= d <= 2: along an axis an even d has the one parent I + d/2 (weight 1), an odd d
// the two parents I + (d -+ 1)/2 (weight 1/2 each).  Called from fully unrolled loops, so
// every index of acc is a constant and acc stays in registers.
template <int DIM>
__device__ __forceinline__ void add_parents(int d0, int d1, int d2, cd a, cd* acc) {
  const bool od0 = d0 & 1, od1 = d1 & 1, od2 = DIM == 3 && (d2 & 1);
  const double w = (od0 ? 0.5 : 1.0) * (od1 ? 0.5 : 1.0) * (od2 ? 0.5 : 1.0);
#pragma unroll
  for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
    for (int b1 = 0; b1 < 2; ++b1)
#pragma unroll
      for (int b0 = 0; b0 < 2; ++b0) {
        if ((od0 || !b0) && (od1 || !b1) && (od2 || !b2)) {
          const int J0 = od0 ? (b0 ? d0 + 1 : d0 - 1) / 2 : d0 / 2;
          const int J1 = od1 ? (b1 ? d1 + 1 : d1 - 1) / 2 : d1 / 2;
          const int J2 = DIM == 3 ? (od2 ? (b2 ? d2 + 1 : d2 - 1) / 2 : d2 / 2) : 0;
          acc[(J0 + 1) + 3 * (J1 + 1) + (DIM == 3 ? 9 * (J2 + 1) : 0)] += w * a;
        }
      }
}

// fine operator -Lap_h - s m (1 - i sigma) -> level 2.  Fine nodes outside the grid add
// zero terms, so the loops have constant trip counts.
template <int DIM>
__global__ void __launch_bounds__(128) k_gal_fine(FineOp op, cd s, const double* __restrict__ m,
                                                  Geom gc, cd* __restrict__ out) {
  constexpr int R2 = DIM == 3 ? 1 : 0, K = DIM == 3 ? 27 : 9;
  long long I = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= gc.tot) return;
  const Geom& g = op.g;
  const int Ic[3] = {(int)(I % gc.N[0]), (int)((I / gc.N[0]) % gc.N[1]),
                     DIM == 3 ? (int)(I / ((long long)gc.N[0] * gc.N[1])) : 0};
  cd acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = mk(0.0, 0.0);
  const double ih = op.inv_h2;
#pragma unroll
  for (int o2 = -R2; o2 <= R2; ++o2)
#pragma unroll
    for (int o1 = -1; o1 <= 1; ++o1)
#pragma unroll
      for (int o0 = -1; o0 <= 1; ++o0) {
        const int f[3] = {2 * Ic[0] + o0, 2 * Ic[1] + o1, 2 * Ic[2] + o2};
        const bool in = f[0] >= 0 && f[0] <= g.n[0] && f[1] >= 0 && f[1] <= g.n[1] &&
                        (DIM == 2 || (f[2] >= 0 && f[2] <= g.n[2]));
        const double wR = (o0 == 0 ? 0.5 : 0.25) * (o1 == 0 ? 0.5 : 0.25) * (DIM == 3 ? (o2 == 0 ? 0.5 : 0.25) : 1.0);
        cd diag = mk(0.0, 0.0);
        if (in) {
          const long long fl = f[0] + (long long)g.N[0] * (f[1] + (long long)g.N[1] * f[2]);
          const double sig = layer_sigma(op, f[0], f[1], f[2]);
          const double mm = m[fl];
          const cd c = s * mk(mm, -mm * sig);
          diag = mk(2.0 * DIM * ih - c.x, -c.y);
        }
        add_parents<DIM>(o0, o1, o2, wR * diag, acc);
#pragma unroll
        for (int a = 0; a < DIM; ++a)
#pragma unroll
          for (int sgn = -1; sgn <= 1; sgn += 2) {
            const int ga = f[a] + sgn;
            const bool ing = in && ga >= 0 && ga <= g.n[a];
            add_parents<DIM>(o0 + (a == 0 ? sgn : 0), o1 + (a == 1 ? sgn : 0), o2 + (a == 2 ? sgn : 0),
                             ing ? mk(-wR * ih, 0.0) : mk(0.0, 0.0), acc);
          }
      }
#pragma unroll
  for (int k = 0; k < K; ++k) out[(long long)k * gc.tot + I] = acc[k];
}

// out[J] = sum_t w(o + t, J) a[t], J = -1, 0, 1, along one axis: the interpolation weight of
// parent I + J in fine node 2 I + d is 1 at d = 2 J, 1/2 at d = 2 J -+ 1 and 0 beyond
__device__ __forceinline__ void gather_axis(int o, cd& a0, cd& a1, cd& a2) {
  const cd e = a0, c = a1, f = a2;      // t = -1, 0, 1
  if (o == 0) {
    a0 = 0.5 * e;
    a1 = c + 0.5 * (e + f);
    a2 = 0.5 * f;
  } else if (o < 0) {
    a0 = e + 0.5 * c;
    a1 = f + 0.5 * c;
    a2 = mk(0.0, 0.0);
  } else {
    a0 = mk(0.0, 0.0);
    a1 = e + 0.5 * c;
    a2 = f + 0.5 * c;
  }
}

// stored 3^d operator on level 2 -> level 3.  One thread per coarse node and fine row of its
// restriction footprint (3^d rows): its 3^d coefficients are loaded together and, P being a
// tensor product, taken to the coarse offsets one axis at a time; the rows' contributions
// are then summed through LDS in a fixed order.  Coefficients whose neighbour lies outside the grid
// are stored as 0.  With one thread per coarse node, walking rows, coefficients and parents
// one after the other, the launch was a chain of 729 loads: 0.49 ms at 17^3 coarse nodes and
// 3.5 ms at 65^3.
template <int DIM>
__global__ void __launch_bounds__(256) k_gal_coarse(Geom g, const cd* __restrict__ A, Geom gc,
                                                    cd* __restrict__ out) {
  constexpr int K = DIM == 3 ? 27 : 9, NN = DIM == 3 ? 9 : 28, KC = 9;
  __shared__ cd red[NN][K][KC];
  const int t = threadIdx.x, ln = t / K, o = t % K;
  const long long I = (long long)blockIdx.x * NN + ln;
  const bool on = ln < NN && I < gc.tot;
  const long long Iq = on ? I : 0;
  int i0, i1, i2;
  node_coords(gc, Iq, i0, i1, i2);
  const int o0 = o % 3 - 1, o1 = o / 3 % 3 - 1, o2 = DIM == 3 ? o / 9 - 1 : 0;
  const int f0 = 2 * i0 + o0, f1 = 2 * i1 + o1, f2 = DIM == 3 ? 2 * i2 + o2 : 0;
  const bool in = on && f0 >= 0 && f0 <= g.n[0] && f1 >= 0 && f1 <= g.n[1] &&
                  (DIM == 2 || (f2 >= 0 && f2 <= g.n[2]));
  const long long fl = in ? f0 + (long long)g.N[0] * (f1 + (long long)g.N[1] * f2) : 0;
  const double wR = in ? (o0 == 0 ? 0.5 : 0.25) * (o1 == 0 ? 0.5 : 0.25) * (DIM == 3 ? (o2 == 0 ? 0.5 : 0.25) : 1.0)
                       : 0.0;
  cd a[K];
#pragma unroll
  for (int k = 0; k < K; ++k) a[k] = A[(long long)k * g.tot + fl];
#pragma unroll
  for (int k = 0; k < K; k += 3) gather_axis(o0, a[k], a[k + 1], a[k + 2]);
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (k / 3 % 3 == 0) gather_axis(o1, a[k], a[k + 3], a[k + 6]);
  if (DIM == 3) {
#pragma unroll
    for (int k = 0; k < 9; ++k) gather_axis(o2, a[k], a[(k + 9) % K], a[(k + 18) % K]);
  }
#pragma unroll
  for (int c = 0; c < K; c += KC) {
    __syncthreads();
    if (ln < NN) {
#pragma unroll
      for (int k = 0; k < KC; ++k) red[ln][o][k] = in ? wR * a[c + k] : mk(0.0, 0.0);
    }
    __syncthreads();
    for (int e = t; e < NN * KC; e += 256) {
      const int n = e % NN, k = e / NN;
      const long long J = (long long)blockIdx.x * NN + n;
      if (J >= gc.tot) continue;
      cd v = mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < K; ++q) v += red[n][q][k];
      out[(long long)(c + k) * gc.tot + J] = v;
    }
  }
}

__global__ void k_cast_d2f(const cd* __restrict__ a, cf* __restrict__ b, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    b[i] = to_f(a[i]);
}

// m = kappa^2 from the slowness (is_m = 0), or m taken as given (is_m = 1)
__global__ void k_square(const double* __restrict__ kap, double* __restrict__ m64, float* __restrict__ m32,
                         long long n, int is_m) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    double v = is_m ? kap[i] : kap[i] * kap[i];
    m64[i] = v;
    m32[i] = (float)v;
  }
}

void gal_fine(const FineOp& op, cd s, const double* m, const Geom& gc, cd* out, hipStream_t st) {
  const dim3 grid((unsigned)((gc.tot + 127) / 128));
  if (op.g.dim == 3)
    hipLaunchKernelGGL(k_gal_fine<3>, grid, dim3(128), 0, st, op, s, m, gc, out);
  else
    hipLaunchKernelGGL(k_gal_fine<2>, grid, dim3(128), 0, st, op, s, m, gc, out);
}
void gal_coarse(const Geom& g, const cd* A, const Geom& gc, cd* out, hipStream_t st) {
  if (g.dim == 3)
    hipLaunchKernelGGL(k_gal_coarse<3>, dim3((unsigned)((gc.tot + 8) / 9)), dim3(256), 0, st, g, A, gc, out);
  else
    hipLaunchKernelGGL(k_gal_coarse<2>, dim3((unsigned)((gc.tot + 27) / 28)), dim3(256), 0, st, g, A, gc, out);
}
void cast_d2f(const cd* a, cf* b, long long n, hipStream_t st) {
  hipLaunchKernelGGL(k_cast_d2f, dim3(1024), dim3(256), 0, st, a, b, n);
}
void square_slowness(const double* kap, double* m64, float* m32, long long n, int is_m, hipStream_t st) {
  hipLaunchKernelGGL(k_square, dim3(1024), dim3(256), 0, st, kap, m64, m32, n, is_m);
}

}  // namespace helm
