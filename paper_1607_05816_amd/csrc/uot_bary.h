// Barycentre combine of one cell (Table estimatebary, log form), shared by
// the combine kernels and the line passes of libuot.
#pragma once

#include "uot_device.h"
#include "uot_epilogue.h"
#include "uot_launch.h"

namespace uot {

// Table estimatebary (iii) lam TV / (iv) RG[b1, b2]: log h is a root of
//   TV: A0 + sum_{k: s_k>0} alpha_k clamp((x - log s_k) eps/lam, -1, 1)   (A0: weight of s_k = 0)
//   RG: sum_k alpha_k [b2 min(x + log b2 - log s_k, 0) + b1 max(x + log b1 - log s_k, 0)]
// in x = log h; both are non-decreasing and linear between their breakpoints
// (log s_k -+ lam/eps, log s_k - log b_i).  The smallest root is taken: the
// first breakpoint where the function is >= 0, linear interpolation from the
// breakpoint before it.  h = 0 (TV: A0 >= weight of the others; RG: some
// s_k = 0).  t2: log2 s_k at stride `stride`.

// breakpoint w (0, 1) of input k, natural log t: TV t -+ d, RG t - log b2 / t - log b1
template <typename T>
__device__ __forceinline__ T bary_break(bool tv, T t, int w, T d, T lb1, T lb2) {
  return tv ? (w == 0 ? t - d : t + d) : (w == 0 ? t - lb2 : t - lb1);
}

// TV / RG barycentre combine with L lanes per cell (L a power of two, 2..64):
// each lane evaluates f at its share of the cell's breakpoints, segmented
// shuffle reductions over the L lanes find the smallest breakpoint with
// f >= 0 and the largest one below it, and f is linear in between.  Spreading
// the breakpoints over lanes replaces one long dependent loop per cell, which
// left a launch of a few blocks waiting on memory.
template <typename T>
__device__ __forceinline__ T bary_fa(const T* t2, int64_t stride, int n, const BaryW& la, bool tv, T a0,
                                     T d, T lb1, T lb2, T b1, T b2, bool has_lo, T x) {
  T acc = tv ? a0 : T(0);
  for (int k = 0; k < n; ++k) {
    const T t = t2[k * stride] * T(kLn2);
    if (t == Num<T>::ninf()) continue;
    const T al = T(la.a[k]);
    if (tv) {
      const T y = (x - t) / d;
      acc += al * (y < T(-1) ? T(-1) : (y > T(1) ? T(1) : y));
    } else {
      const T up = x + lb2 - t, dn = x + lb1 - t;
      T term = b2 * (up < T(0) ? up : T(0));
      if (has_lo) term += b1 * (dn > T(0) ? dn : T(0));
      acc += al * term;
    }
  }
  return acc;
}

// lanes per cell: one to a breakpoint, up to a wave (two_breaks: TV, RG with a
// lower bound)
__host__ __device__ inline int bary_lanes(int nm, bool two_breaks) {
  const int nbp = two_breaks ? 2 * nm : nm;
  int L = 2;
  while (L < nbp && L < 64) L *= 2;
  return L;
}

// log h of TV / RG at one cell, by L lanes (a power of two; sub: this lane's
// index among them; every lane of the wave calls it): t2[k stride] = log2 s_k
template <typename T>
__device__ __forceinline__ T bary_root(const T* t2, int64_t stride, int nm, const BaryW& la, const DivDev& F2, T eps,
                                       int sub, int L) {
  const bool tv = F2.kind == 2;
  const bool lo = F2.has_lo != 0;
  T a0 = T(0), a1 = T(0), tmax = Num<T>::ninf(), tmin = Num<T>::pinf();
  for (int k = 0; k < nm; ++k) {
    const T t = t2[k * stride] * T(kLn2);
    const T al = T(la.a[k]);
    if (t == Num<T>::ninf()) {
      a0 += al;
    } else {
      a1 += al;
      tmax = t > tmax ? t : tmax;
      tmin = t < tmin ? t : tmin;
    }
  }
  // the cases with a closed answer: no mass (-inf), or RG with every input in
  // one band (the left end of the zero interval, exactly)
  bool closed = false;
  T logh = T(0);
  if (tv ? (a0 >= a1) : (a0 > T(0))) {
    closed = true;
    logh = Num<T>::ninf();
  } else if (!tv) {
    const T left = tmax - T(F2.log_beta);
    if (!lo || left <= tmin - T(F2.log_alpha)) {
      closed = true;
      logh = left;
    }
  }
  const T d = tv ? T(F2.lam) / eps : T(0);
  const T lb1 = lo ? T(F2.log_alpha) : T(0), lb2 = T(F2.log_beta);
  const T b1 = lo ? T(::exp(F2.log_alpha)) : T(0), b2 = T(::exp(F2.log_beta));
  const int per = tv ? 2 : (lo ? 2 : 1);
  const int nbp = nm * per;
  // smallest breakpoint with f >= 0 (and f there)
  T bhi = Num<T>::pinf(), fhi = T(0);
  for (int q = sub; q < nbp; q += L) {
    const int k = q / per, wq = q % per;
    const T t = t2[k * stride] * T(kLn2);
    if (t == Num<T>::ninf()) continue;
    const T b = bary_break<T>(tv, t, wq, d, lb1, lb2);
    const T fb = bary_fa<T>(t2, stride, nm, la, tv, a0, d, lb1, lb2, b1, b2, lo, b);
    if (fb >= T(0) && b < bhi) {
      bhi = b;
      fhi = fb;
    }
  }
  for (int o = L / 2; o >= 1; o >>= 1) {
    const T ob = __shfl_xor(bhi, o), of = __shfl_xor(fhi, o);
    if (ob < bhi || (ob == bhi && of < fhi)) {
      bhi = ob;
      fhi = of;
    }
  }
  // largest breakpoint below it
  T blo = Num<T>::ninf();
  for (int q = sub; q < nbp; q += L) {
    const int k = q / per, wq = q % per;
    const T t = t2[k * stride] * T(kLn2);
    if (t == Num<T>::ninf()) continue;
    const T b = bary_break<T>(tv, t, wq, d, lb1, lb2);
    if (b < bhi && b > blo) blo = b;
  }
  for (int o = L / 2; o >= 1; o >>= 1) {
    const T ob = __shfl_xor(blo, o);
    blo = ob > blo ? ob : blo;
  }
  if (!closed) {
    if (blo == Num<T>::ninf()) {
      logh = bhi;
    } else {
      const T flo = bary_fa<T>(t2, stride, nm, la, tv, a0, d, lb1, lb2, b1, b2, lo, blo);
      logh = blo + (T(0) - flo) * (bhi - blo) / (fhi - flo);
    }
  }
  return logh;
}

// log h of = (row (i)) or KL (row (ii)) at one cell
template <typename T>
__device__ __forceinline__ T bary_mean(const T* t2, int64_t stride, int nm, const BaryW& w, const DivDev& F2, T eps) {
  T logh;
  if (F2.kind == 0) {
    double acc = 0.0, asum = 0.0;
    for (int k = 0; k < nm; ++k) {
      const double al = w.a[k];
      acc += al * double(t2[k * stride]) * kLn2;
      asum += al;
    }
    logh = T(acc / asum);
  } else {
    // the power mean about the largest input, r + log(sum alpha_k e^{gam (t_k
    // - r)} / sum alpha) / gam with gam = eps / (eps + lam): 1 / gam magnifies
    // what the sum rounds (gam is small where transport matters), so a sum near 1
    // is carried as its difference from 1; a small one (the largest input has
    // little weight, the others lie far below it) would cancel there and is
    // taken as it is, its terms being positive
    const T gam = eps / (eps + T(F2.lam));
    T r = Num<T>::ninf();
    for (int k = 0; k < nm; ++k) r = Num<T>::fmax(r, t2[k * stride]);
    if (r == Num<T>::ninf()) return r;
    T acc = T(0), asum = T(0), sum = T(0);
    for (int k = 0; k < nm; ++k) {
      const T al = T(w.a[k]);
      T e;
      acc = Num<T>::fma(al, expm1_exp2(gam * (t2[k * stride] - r), e), acc);
      sum = Num<T>::fma(al, e, sum);
      asum += al;
    }
    // log y: of the small sum, or of 1 + x with what the addition rounds put back
    // (x in [-1/2, 0])
    const bool small = acc < T(-0.5) * asum;
    const T x = (small ? sum : acc) / asum;
    const T y = small ? x : T(1) + x;
    const T lost = small ? T(0) : x - (y - T(1));
    const T lg = Num<T>::log(y) + lost / y;
    logh = r * T(kLn2) + lg / gam;
  }
  return logh;
}

}  // namespace uot
