// FP64 objective of libuot: the terms of Thm. duality at the plan R =
// e^{(u+v-C)/eps}, for data of either type.
#include <algorithm>

#include "uot_device.h"
#include "uot_launch.h"

// ---------------------------------------------------------------------------
// The products here are evaluated in FP64, whatever the type of the
// potentials: in FP32 a product of exponents near 10^3 is off by 1e-6 and
// more, as much as a converged solve's potentials are worth.
// Grids: FP64 line passes (uot_grid_line.hip) on weights built from the
// potentials (k_obj_weight).  The transport cost of FP64 data is a product per
// axis with that axis' kernel times its cost, a sum of positive terms; of FP32
// data
//   sum_ij R_ij |x_i - y_j|^2 = sum_i R_i. |x_i|^2 + sum_j R_.j |y_j|^2
//                               - 2 sum_i x_i . sum_j R_ij y_j,
// one line pass product per axis with the (positive) cell coordinates as
// weights: its cancellation, |x|^2 / cost, stays below what FP32 potentials
// leave, but took FP64's (4e-9 at 256 cells, eps 6e-6).
// Grids of the WF cost or of kernels of a few cells keep products in the data's
// type (uot_api.hip).
// Point clouds: one pass over the pairs (k_obj_points) gives a row's product
// and, for rows X, its cost moment and its row of K dy: the distance is shared,
// two exp2 per pair.  It is bound by FP64 issue (about 60 operations per pair;
// 100 with the WF cost); the one thread per row with library exp2 and log2
// calls that it replaces took 1.74 ms at 6000 x 5000 points (WF).
// ---------------------------------------------------------------------------
namespace uot {

namespace {

constexpr int kB = 256;

// terms of one element of a side, density pp, weight dd, potential u, plan
// marginal pi: d pi, d u pi, d f(pi | p), d f*(-u | p)
__device__ __forceinline__ void obj_terms(double u, double pi, double pp, double dd, double eps, const DivDev& F,
                                          double& a0, double& a1, double& a2, double& a3) {
  a0 = dd * pi;
  a1 = (pi > 0) ? dd * u * pi : 0.0;
  const double w = -u;   // conjugate argument
  const double lam = F.lam;
  switch (F.kind) {
    case 1:  // lam KL
      a2 = dd * lam * ((pi > 0 ? pi * ::log(pi / pp) : 0.0) - pi + pp);
      if (pp == 0.0 && pi > 0) a2 = __builtin_inf();
      a3 = (pp > 0) ? dd * lam * pp * ::expm1(w / lam) : 0.0;
      break;
    case 2:  // lam TV
      a2 = dd * lam * ::fabs(pi - pp);
      a3 = (w > lam * (1 + 1e-6)) ? __builtin_inf() : dd * pp * ::fmax(w, -lam);
      break;
    case 4: {  // growth, cap pp: F = s log kappa below kappa pp, s log(s/pp) - s + kappa pp above
      const double kap = 1.0 - lam;
      if (pp == 0.0) a2 = pi > 0 ? __builtin_inf() : 0.0;
      else a2 = dd * (pi <= kap * pp ? pi * ::log(kap) : pi * ::log(pi / pp) - pi + kap * pp);
      a3 = dd * pp * ::fmax(::exp(w) - kap, 0.0);
      break;
    }
    default:  // = / RG: indicator terms are not finite-valued; gap reported as NaN by the host
      a2 = 0.0;
      a3 = 0.0;
      if (F.kind == 0) a3 = (pp > 0) ? dd * pp * w : 0.0;
      else {
        const double al = F.has_lo ? ::exp(F.log_alpha) : 0.0;
        const double be = F.has_hi ? ::exp(F.log_beta) : __builtin_inf();
        a3 = (pp > 0) ? dd * pp * ((w > 0) ? be * w : al * w) : 0.0;
      }
      break;
  }
}

// block sums of Q doubles; thread q < Q writes out[q]
template <int Q> __device__ __forceinline__ void block_sums(const double (&v)[Q], double* out) {
  __shared__ double sm[Q][kB / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    double s = v[q];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) sm[q][wv] = s;
  }
  __syncthreads();
  if (threadIdx.x < Q) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kB / 64; ++k) s += sm[threadIdx.x][k];
    out[threadIdx.x] = s;
  }
}

// log2 of a reference weight, rounded as a solve on T data rounds it (see
// as_data)
template <typename T> __device__ __forceinline__ double obj_logd(T d) {
  return double(Num<T>::log(d) * T(kLog2e));
}
// log2 weight of a potential, pot / eps + log d, with le + lo = log2(e) / eps; a
// potential of +inf (left by a vanishing product) carries no mass
template <typename T>
__device__ __forceinline__ double obj_weight(const T* pot, const T* d, int64_t i, double le, double lo) {
  const double p = pot ? double(pot[i]) : 0.0, a = obj_logd<T>(d[i]);
  if (p == __builtin_inf()) return -__builtin_inf();
  return p == -__builtin_inf() ? p : __builtin_fma(p, le, __builtin_fma(p, lo, a));
}

}  // namespace

// out_i = weight of (pot, d; pot null: a zero potential), plus with axis >= 0
// log2 of that coordinate of the cell centre, with axis -2 log2 of its squared
// norm
template <typename T>
__global__ __launch_bounds__(kB) void k_obj_weight(const T* __restrict__ pot, const T* __restrict__ d, int64_t n,
                                                   double le, double lo, GridCells g, int axis,
                                                   double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (i >= n) return;
  double w = obj_weight<T>(pot, d, i, le, lo);
  if (axis != -1) {
    double x[3] = {0, 0, 0}, r = 0.0;
    int64_t j = i;
    for (int k = g.dim - 1; k >= 0; --k) {
      x[k] = (double(j % g.n[k]) + 0.5) * g.h[k];
      r = __builtin_fma(x[k], x[k], r);
      j /= g.n[k];
    }
    w += ::log2(axis >= 0 ? x[axis] : r);
  }
  out[i] = w;
}

// one side's terms from its product S (log2): 4 sums per block, the plan's
// marginal in pi_out
template <typename T>
__global__ __launch_bounds__(kB) void k_obj_side64(const T* __restrict__ pot, const double* __restrict__ S,
                                                   const T* __restrict__ p, const T* __restrict__ d, int64_t n,
                                                   double eps, DivDev F, T* __restrict__ pi_out,
                                                   double* __restrict__ part) {
  const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
  double a[4] = {0, 0, 0, 0};
  if (i < n) {
    const double u = double(pot[i]), s = S[i] * kLn2;
    // no mass where the potential or the product vanishes (0 times any potential)
    const double pi = (u == -__builtin_inf() || s == -__builtin_inf()) ? 0.0 : ::exp(u / eps + s);
    if (pi_out) pi_out[i] = T(pi);
    obj_terms(u, pi, double(p[i]), double(d[i]), eps, F, a[0], a[1], a[2], a[3]);
  }
  block_sums<4>(a, part + 4 * (int64_t)blockIdx.x);
}

// per-block sums of scale 2^{a_i + b_i}
__global__ __launch_bounds__(kB) void k_obj_sum(const double* __restrict__ a, const double* __restrict__ b, int64_t n,
                                                double* __restrict__ part) {
  const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
  const double v[1] = {i < n ? exp2_f64(a[i] + b[i]) : 0.0};
  block_sums<1>(v, part + blockIdx.x);
}

// Rows xr against one split of the columns: partial (m, s) of log2 sum_j 2^{w_j
// + log2 K_ij}, and with FULL the cost moment sum_j C_ij 2^{..} relative to 2^m
// and sum_j K_ij dy_j.  part[(split Q + q) Nr + i], Q = 4 or 2.
// grid = (ceil(Nr / 256), splits)
template <typename T, int DIM, int COST, bool FULL>
__global__ __launch_bounds__(kB) void k_obj_points(const T* __restrict__ xr, int64_t Nr, const T* __restrict__ yc,
                                                   const T* __restrict__ pot, const T* __restrict__ d, int64_t Mc,
                                                   int64_t cps, double le, double lo, double kc, double a2, double cut2,
                                                   double* __restrict__ part) {
  constexpr int C = 8, Q = FULL ? 4 : 2;
  __shared__ double ty[DIM][kB], tw[kB], tk[FULL ? kB : 1];
  const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
  double xi[DIM];
#pragma unroll
  for (int k = 0; k < DIM; ++k) xi[k] = double(xr[k * Nr + (i < Nr ? i : 0)]);
  const int64_t cb = (int64_t)blockIdx.y * cps, ce = cb + cps < Mc ? cb + cps : Mc;
  double m = -__builtin_inf(), s = 0.0, sc = 0.0, sk = 0.0;
  for (int64_t c0 = cb; c0 < ce; c0 += kB) {
    const int64_t j = c0 + threadIdx.x;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < DIM; ++k) ty[k][threadIdx.x] = j < ce ? double(yc[k * Mc + j]) : 0.0;
    tw[threadIdx.x] = j < ce ? obj_weight<T>(pot, d, j, le, lo) : -__builtin_inf();
    if (FULL) tk[threadIdx.x] = j < ce ? obj_logd<T>(d[j]) : -__builtin_inf();
    __syncthreads();
    const int cnt = ce - c0 < kB ? (int)(ce - c0) : kB;
    for (int jj = 0; jj < cnt; jj += C) {   // (columns past the end carry no weight)
      double t[C], cst[C], cm = -__builtin_inf();
#pragma unroll
      for (int k = 0; k < C; ++k) {
        double d2 = 0.0;
#pragma unroll
        for (int e = 0; e < DIM; ++e) {
          const double g = xi[e] - ty[e][jj + k];
          d2 = __builtin_fma(g, g, d2);
        }
        double g;
        if (COST == 1) {
          // log2 cos theta: C = -2 ln cos theta, log2 K = (2 / eps) log2 cos theta
          const double cv = CosSqrt<double>::eval(d2 * a2);
          const bool in = d2 < cut2 && cv > 0.0;
          const double lc = in ? ::log2(cv) : 0.0;
          cst[k] = -2.0 * kLn2 * lc;
          g = in ? kc * lc : -__builtin_inf();
        } else {
          cst[k] = d2;
          g = -kc * d2;
        }
        t[k] = tw[jj + k] + g;
        cm = __builtin_fmax(cm, t[k]);
        if (FULL) sk += exp2_f64(tk[jj + k] + g);
      }
      const double mn = __builtin_fmax(m, cm);
      if (mn == -__builtin_inf()) continue;
      const double r = exp2_f64(m - mn);
      s *= r;
      sc *= r;
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const double e = exp2_f64(t[k] - mn);
        s += e;
        if (FULL) sc = __builtin_fma(cst[k], e, sc);
      }
      m = mn;
    }
  }
  if (i >= Nr) return;
  double* o = part + (int64_t)blockIdx.y * Q * Nr + i;
  o[0] = m;
  o[Nr] = s;
  if (FULL) {
    o[2 * Nr] = sc;
    o[3 * Nr] = sk;
  }
}

// the splits of a row joined, and its terms: 6 sums per block (the side's
// four, the transport cost and the mass of K)
template <typename T, bool FULL>
__global__ __launch_bounds__(kB) void k_obj_points_finish(const double* __restrict__ part, int nsplit, int64_t Nr,
                                                          const T* __restrict__ pot, const T* __restrict__ p,
                                                          const T* __restrict__ d, double eps, DivDev F,
                                                          T* __restrict__ pi_out, double* __restrict__ out) {
  constexpr int Q = FULL ? 4 : 2;
  const int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x;
  double a[6] = {0, 0, 0, 0, 0, 0};
  if (i < Nr) {
    double m = -__builtin_inf(), s = 0.0, sc = 0.0, sk = 0.0;
    for (int k = 0; k < nsplit; ++k) m = __builtin_fmax(m, part[(int64_t)k * Q * Nr + i]);
    for (int k = 0; k < nsplit; ++k) {
      const double* o = part + (int64_t)k * Q * Nr + i;
      const double f = m == -__builtin_inf() ? 0.0 : exp2_f64(o[0] - m);
      s += f * o[Nr];
      if (FULL) {
        sc += f * o[2 * Nr];
        sk += o[3 * Nr];
      }
    }
    const double u = double(pot[i]), dd = double(d[i]);
    const bool none = u == -__builtin_inf() || u == __builtin_inf() || m == -__builtin_inf();
    const double pi = none ? 0.0 : ::exp(u / eps + (m + ::log2(s)) * kLn2);
    if (pi_out) pi_out[i] = T(pi);
    obj_terms(u, pi, double(p[i]), dd, eps, F, a[0], a[1], a[2], a[3]);
    if (FULL) {
      a[4] = none ? 0.0 : dd * pi * (sc / s);
      a[5] = dd * sk;
    }
  }
  block_sums<6>(a, out + 6 * (int64_t)blockIdx.x);
}

// A constant of the kernel, rounded as the products of a solve on T data round
// it (log reference weights likewise): the potentials belong to the kernel they
// were computed with, and at another one, 2^-24 away in its exponents, the
// plan's mass is off by about 1e-6, more than by anything else.
template <typename T> static double as_data(double k) { return double(T(k)); }

static unsigned obj_blocks(int64_t n) { return (unsigned)((n + kB - 1) / kB); }

template <typename T>
void launch_obj_weight(const T* pot, const T* d, int64_t n, double eps, const GridCells& g, int axis, double* out,
                       hipStream_t s) {
  const double le = kLog2e / eps;
  hipLaunchKernelGGL(k_obj_weight<T>, dim3(obj_blocks(n)), dim3(kB), 0, s, pot, d, n, le, le_rest(eps, le), g, axis, out);
}
template <typename T>
void launch_obj_side64(const T* pot, const double* S, const T* p, const T* d, int64_t n, double eps, const DivDev& F,
                       T* pi_out, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_obj_side64<T>, dim3(obj_blocks(n)), dim3(kB), 0, s, pot, S, p, d, n, eps, F, pi_out, part);
}
void launch_obj_sum(const double* a, const double* b, int64_t n, double* part, hipStream_t s) {
  hipLaunchKernelGGL(k_obj_sum, dim3(obj_blocks(n)), dim3(kB), 0, s, a, b, n, part);
}

template <typename T, bool FULL>
static void obj_points_t(int dim, const T* xr, int64_t Nr, const T* yc, const T* pot, const T* d, int64_t Mc, int nsplit,
                         double eps, const CostArgs& cost, double* part, hipStream_t s) {
  const double le = kLog2e / eps, lo = le_rest(eps, le);
  const int64_t cps = ((Mc + nsplit - 1) / nsplit + 7) / 8 * 8;
  const dim3 grid(obj_blocks(Nr), (unsigned)nsplit);
  const double a2 = as_data<T>(cost.kind == 1 ? 0.25 * M_PI * M_PI / (cost.cut * cost.cut) : 0.0);
  const double cut2 = as_data<T>(cost.cut * cost.cut);
  const double kc = as_data<T>(cost.kind == 1 ? 2.0 * kLn2 * le : le);
#define UOT_OP(D, C) \
  hipLaunchKernelGGL((k_obj_points<T, D, C, FULL>), grid, dim3(kB), 0, s, xr, Nr, yc, pot, d, Mc, cps, le, lo, kc, a2, cut2, part)
  if (cost.kind == 1) {
    if (dim == 1) UOT_OP(1, 1);
    else if (dim == 2) UOT_OP(2, 1);
    else UOT_OP(3, 1);
  } else {
    if (dim == 1) UOT_OP(1, 0);
    else if (dim == 2) UOT_OP(2, 0);
    else UOT_OP(3, 0);
  }
#undef UOT_OP
}

template <typename T>
void launch_obj_points(bool full, int dim, const T* xr, int64_t Nr, const T* yc, const T* pot_c, const T* dc, int64_t Mc,
                       int nsplit, double eps, const CostArgs& cost, const T* pot_r, const T* p, const T* dr,
                       const DivDev& F, T* pi_out, double* part, double* out, hipStream_t s) {
  if (full) {
    obj_points_t<T, true>(dim, xr, Nr, yc, pot_c, dc, Mc, nsplit, eps, cost, part, s);
    hipLaunchKernelGGL((k_obj_points_finish<T, true>), dim3(obj_blocks(Nr)), dim3(kB), 0, s, part, nsplit, Nr, pot_r, p,
                       dr, eps, F, pi_out, out);
  } else {
    obj_points_t<T, false>(dim, xr, Nr, yc, pot_c, dc, Mc, nsplit, eps, cost, part, s);
    hipLaunchKernelGGL((k_obj_points_finish<T, false>), dim3(obj_blocks(Nr)), dim3(kB), 0, s, part, nsplit, Nr, pot_r, p,
                       dr, eps, F, pi_out, out);
  }
}

#define UOT_OBJ_INST(T)                                                                                               \
  template void launch_obj_weight<T>(const T*, const T*, int64_t, double, const GridCells&, int, double*,             \
                                     hipStream_t);                                                                    \
  template void launch_obj_side64<T>(const T*, const double*, const T*, const T*, int64_t, double, const DivDev&, T*, \
                                     double*, hipStream_t);                                                           \
  template void launch_obj_points<T>(bool, int, const T*, int64_t, const T*, const T*, const T*, int64_t, int, double, \
                                     const CostArgs&, const T*, const T*, const T*, const DivDev&, T*, double*,       \
                                     double*, hipStream_t);
UOT_OBJ_INST(float)
UOT_OBJ_INST(double)

}  // namespace uot
