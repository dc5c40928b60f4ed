// Epilogue and control-step device helpers shared by the Gibbs-product
// kernels of libuot (uot_kernels.hip, uot_grid_tf.hip): the pointwise proxdiv
// epilogue with the residual partials, and the control step of an iteration.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "uot_device.h"
#include "uot_launch.h"

namespace uot {

constexpr int kBlock = 256;

// ---------------------------------------------------------------------------
// epilogue shared by every Gibbs product.  epi_elem handles one element with
// S2 = log2 of the product; epi_finish reduces the residual partials of the
// block (every thread of the block must call it).
// ---------------------------------------------------------------------------
template <typename T> struct ResAcc {
  T m, den, num, du;   // du: largest |u_new - u_old| seen
  __device__ __forceinline__ void init() {
    m = Num<T>::ninf();
    den = T(0);
    num = T(0);
    du = T(0);
  }
  __device__ __forceinline__ void add(T m2, T d2, T n2) { res_merge<T>(m, den, num, m2, d2, n2); }
};

// operands of one element's epilogue, loadable ahead of the product
template <typename T> struct EpiIn {
  T ld, uo, lp;
};

template <typename T>
__device__ __forceinline__ EpiIn<T> epi_load(int64_t e, const EpiArgs<T>& ep) {
  EpiIn<T> x;
  if (ep.mode == EPI_RAW) {
    x.ld = x.uo = x.lp = T(0);
    return x;
  }
  x.ld = ep.logd[e < ep.size ? e : e % ep.size];
  x.uo = ep.pot[e];
  x.lp = ep.logp[e];
  return x;
}

// The factors an epilogue multiplies by, once per thread: quotients by eps are
// products with a reciprocal carried in two parts (k + kl, so that pot k is
// rounded once), in place of an IEEE division per element and use.
template <typename T> struct EpiK {
  T zeta;
  T ke, kel;   // log2(e) / eps
  T kw, kwl;   // log2(e) / eps_w
  ProxK<T> k;  // eps, and the factor of KL or growth
};
// k + kl = log2(e) / eps (le: rounded to a double)
template <typename T> __device__ __forceinline__ void epi_parts(double eps, double le, T& k, T& kl) {
  k = T(le);
  kl = sizeof(T) == 4 ? T(le - double(k)) : T(le_rest(eps, le));
}
// from the control block's values (le: log2(e) / eps, eps_w and le_w those of w)
template <typename T>
__device__ __forceinline__ EpiK<T> epi_consts(double eps, double le, double eps_w, double le_w, double coef,
                                              double zeta) {
  EpiK<T> k;
  k.zeta = T(zeta);
  epi_parts<T>(eps, le, k.ke, k.kel);
  epi_parts<T>(eps_w, le_w, k.kw, k.kwl);
  k.k.set(eps, coef);
  return k;
}
// pot (k + kl) + a
template <typename T> __device__ __forceinline__ T epi_scale(T pot, T k, T kl, T a) {
  return Num<T>::fma(pot, k, Num<T>::fma(pot, kl, a));
}
// the weight of a potential in the next product, (pot / eps + log d) log2(e)
// with a = log d log2(e); infinite potentials stay what they are
template <typename T> __device__ __forceinline__ T epi_weight(T pot, T k, T kl, T a) {
  return Num<T>::fmax(pot, -pot) < Num<T>::pinf() ? epi_scale<T>(pot, k, kl, a) : pot;
}
// e^x - 1 at x = t ln 2: the Taylor polynomial to degree 7 for |x| < 1/4
// (remainder below 4e-10 of x), else 2^t - 1
__device__ __forceinline__ float expm1_poly(float x) {
  float p = 1.f / 5040.f;
  p = __builtin_fmaf(p, x, 1.f / 720.f);
  p = __builtin_fmaf(p, x, 1.f / 120.f);
  p = __builtin_fmaf(p, x, 1.f / 24.f);
  p = __builtin_fmaf(p, x, 1.f / 6.f);
  p = __builtin_fmaf(p, x, 0.5f);
  return __builtin_fmaf(p * x, x, x);
}
__device__ __forceinline__ float expm1_log2(float t) {
  const float x = t * float(kLn2);
  const float p = expm1_poly(x);
  return __builtin_fabsf(x) < 0.25f ? p : __builtin_amdgcn_exp2f(t) - 1.f;
}
// (and e = 2^t)
__device__ __forceinline__ float expm1_exp2(float t, float& e) {
  const float x = t * float(kLn2);
  e = __builtin_amdgcn_exp2f(t);
  return __builtin_fabsf(x) < 0.25f ? expm1_poly(x) : e - 1.f;
}
// ... t = n + f: 2^n (2^f - 1) + (2^n - 1), which is 2^f - 1 as it is for n = 0 and
// cancels less than two bits otherwise (|2^f - 1| <= 0.42)
__device__ __forceinline__ double expm1_exp2(double t, double& e) {
  const double tc = t < -1100.0 ? -1100.0 : t;
  const double n = __builtin_rint(tc);
  const double f = tc - n;
  double a, b;
  exp2_poly(f, a, b);
  const double m = __builtin_fma(b, f, a * (f * f)), s = __builtin_amdgcn_ldexp(1.0, (int)n);
  e = __builtin_fma(s, m, s);
  return __builtin_fma(s, m, s - 1.0);
}
__device__ __forceinline__ double expm1_log2(double t) { return ::expm1(t * kLn2); }

// The proxdiv epilogue of one element: writes the new potential (and lse_out),
// adds the residual or mass partial and returns the weight w of the next
// product; x.uo becomes the new potential.
template <typename T>
__device__ __forceinline__ T epi_core(int64_t e, T S2, EpiIn<T>& x, const EpiK<T>& K, const EpiArgs<T>& ep,
                                      ResAcc<T>& ra) {
  const T Sraw = S2 * T(kLn2);
  const T S = Sraw + K.zeta;                  // z K(.): log z of a total-mass penalty, else 0
  const T ld2 = x.ld * T(kLog2e);
  const T sd2 = S2 + K.zeta * T(kLog2e) + ld2;
  const T uo = x.uo;
  const T un = proxdiv_pot<T>(ep.F, x.lp, S, K.k);
  // a vanishing product (K b = 0 here, possible with exact zeros of K): the
  // row of the plan is zero whatever the potential, so the point carries no
  // marginal mass and enters the next product as -inf
  const bool vanish = Sraw == Num<T>::ninf();
  ep.pot[e] = un;
  x.uo = un;
  const T w = vanish ? Num<T>::ninf() : epi_weight<T>(un, K.kw, K.kwl, ld2);
  if (ep.lse_out) ep.lse_out[e] = S;
  if (vanish) return w;
  if (ep.part) {
    if (un == Num<T>::ninf()) {
      if (uo != Num<T>::ninf()) {
        ra.add(epi_scale<T>(uo, K.ke, K.kel, sd2), T(0), T(1));
        ra.du = Num<T>::pinf();           // a potential that jumped to -inf
      }
    } else {
      const T a = uo - un;
      const T d = expm1_log2(Num<T>::fmax(a, -a) < Num<T>::pinf() ? epi_scale<T>(a, K.ke, K.kel, T(0)) : a);
      ra.add(epi_scale<T>(un, K.ke, K.kel, sd2), T(1), Num<T>::fmax(d, -d));
      ra.du = Num<T>::fmax(ra.du, uo == Num<T>::ninf() ? Num<T>::pinf() : Num<T>::fmax(a, -a));
    }
  } else if (ep.mass_m) {
    // mass of the plan without z: the (m, den) pair of ra carries it
    ra.add(epi_scale<T>(un, K.ke, K.kel, S2 + ld2), T(1), T(0));
  }
  return w;
}

// the same value in every lane, kept in scalar registers
__device__ __forceinline__ float uniform(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}
__device__ __forceinline__ double uniform(double x) {
  const int2 v = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, int2{__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y)});
}

template <typename T> __device__ __forceinline__ EpiK<T> uniform(EpiK<T> k) {
  k.zeta = uniform(k.zeta);
  k.ke = uniform(k.ke), k.kel = uniform(k.kel);
  k.kw = uniform(k.kw), k.kwl = uniform(k.kwl);
  k.k.eps.c = uniform(k.k.eps.c), k.k.eps.cl = uniform(k.k.eps.cl);
  k.k.coef.c = uniform(k.k.coef.c), k.k.coef.cl = uniform(k.k.coef.cl);
  return k;
}

template <typename T>
__device__ __forceinline__ EpiK<T> epi_consts_of(const Ctrl* __restrict__ c, int side, const EpiArgs<T>& ep) {
  EpiK<T> k{};
  if (ep.mode == EPI_RAW) return k;
  // (w feeds the next half-step, at its eps)
  const int p = par_of(side), h = half_of(side);
  return epi_consts<T>(c->eps[p], c->le[p], c->eps[p ^ h], c->le[p ^ h], c->coef[p][h], c->zeta);
}

template <typename T>
__device__ __forceinline__ void epi_apply(int64_t e, T S2, const EpiIn<T>& x, const EpiK<T>& K, const EpiArgs<T>& ep,
                                          ResAcc<T>& ra) {
  if (ep.mode == EPI_RAW) {
    ep.out[e] = S2;
    return;
  }
  EpiIn<T> xi = x;
  const T w = epi_core<T>(e, S2, xi, K, ep, ra);
  if (ep.wnext) ep.wnext[e] = w;
}

template <typename T>
__device__ __forceinline__ void epi_elem(int64_t e, T S2, const EpiK<T>& K, const EpiArgs<T>& ep, ResAcc<T>& ra) {
  epi_apply<T>(e, S2, epi_load<T>(e, ep), K, ep, ra);
}

// Ragged batches, the in-solve mass balance: in the half-steps that run
// while the iteration counter equals ep.bal_iter, the plan's marginal mass
// over an item's rows (log2 units: S2 + (pot/eps + log d) log2(e), the row's
// a K b d, once its epilogue wrote the new potential) goes to one more
// block partial.  Rows with no mass (p = 0, or a vanishing product) add
// nothing.
template <typename T>
__device__ __forceinline__ bool bal_on(const EpiArgs<T>& ep, const Ctrl* __restrict__ c) {
  return ep.bal_m != nullptr && c->iter == ep.bal_iter;
}
// (m, s): a running log2-sum-exp in T precision, m + log2 s
template <typename T> struct MassAcc {
  T m, s;
  __device__ __forceinline__ void init() { m = Num<T>::ninf(); s = T(0); }
  __device__ __forceinline__ void add(T t) {
    if (t == Num<T>::ninf()) return;
    const T mn = Num<T>::fmax(m, t);
    s = s * Num<T>::exp2(m - mn) + Num<T>::exp2(t - mn);
    m = mn;
  }
};
template <typename T>
__device__ __forceinline__ void bal_elem(int64_t e, T S2, const Ctrl* __restrict__ c, int side, const EpiArgs<T>& ep,
                                         MassAcc<T>& mb) {
  if (S2 == Num<T>::ninf()) return;
  const T un = ep.pot[e];
  if (un == Num<T>::ninf() || un == Num<T>::pinf()) return;
  const T ld = ep.logd[e < ep.size ? e : e % ep.size];
  mb.add(S2 + (un / T(eps_of(c, side)) + ld) * T(kLog2e));
}

// log2-sum-exp (m, s) over a block in T precision (every thread calls it);
// thread 0 writes the result
template <typename T, int NT = kBlock>
__device__ __forceinline__ void block_lse_reduce(T m, T s, T* out_m, T* out_s) {
  __shared__ T sm[NT], ss[NT];
  sm[threadIdx.x] = m;
  ss[threadIdx.x] = s;
  __syncthreads();
  for (int off = NT / 2; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) {
      Lse2<T> a;
      a.m = sm[threadIdx.x];
      a.s = ss[threadIdx.x];
      a.merge(sm[threadIdx.x + off], ss[threadIdx.x + off]);
      sm[threadIdx.x] = a.m;
      ss[threadIdx.x] = a.s;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *out_m = sm[0];
    *out_s = ss[0];
  }
}

template <typename T, int NT = kBlock>
__device__ __forceinline__ void epi_finish(const EpiArgs<T>& ep, const ResAcc<T>& ra, int part_index) {
  if (ep.mode == EPI_RAW) return;
  if (ep.part) block_res_reduce<T, NT>(ra.m, ra.den, ra.num, ra.du, ep.part + part_index);
  else if (ep.mass_m) block_lse_reduce<T, NT>(ra.m, ra.den, ep.mass_m + part_index, ep.mass_s + part_index);
}

// ---------------------------------------------------------------------------
// control step of an iteration: reduce the residual partials of the X
// half-step, count the iteration, pick the next eps, stop when done.  It runs
// as its own launch (k_control) or in block 0 of the first pass of the Y
// half-step (grid solves of one problem: that pass only reads the slot of
// the current iteration, the step writes the slot of the next).
// ---------------------------------------------------------------------------
// what the control step of an iteration of parity par reads of the control
// block, loaded before the residual reduction so those loads overlap the
// loads of the partials
struct CtrlSnap {
  int64_t l, max_iter;
  int stage, n_stages, sn, sa;   // stages of this iteration, and of the two after it
  double tol;
};

__device__ __forceinline__ CtrlSnap ctrl_snap(const Ctrl* c, int par) {
  CtrlSnap s;
  s.l = c->iter;
  s.max_iter = c->max_iter;
  s.stage = c->stage[par];
  s.n_stages = c->n_stages;
  s.tol = c->tol;
  s.sn = stage_at(c, s.l + 1);
  s.sa = stage_at(c, s.l + 2);
  return s;
}
// the slot of the iteration after the one of `s`; not part of the snapshot, as
// a block that carries it through its own tile pays 12 registers for it
__device__ __forceinline__ CtrlSlot ctrl_next(const Ctrl* c, const CtrlSnap& s, int par) {
  return slot_values(c, s.sn, s.sa, par);
}

// one thread: record r, count the iteration, fill the slot of the next
// iteration (parity par ^ 1) with its eps stage, stop when done.  A stopped
// solve skips the next iteration; the control step of a skipped iteration
// passes the skip on (control_skip), so every later iteration skips too.
static __device__ void control_finish(Ctrl* c, const CtrlSnap& s, const CtrlSlot& next, double r, double du,
                                      double* __restrict__ hist, int par) {
  if (hist) hist[s.l] = r;
  c->res = r;
  c->du = du;
  c->iter = s.l + 1;
  set_slot(c, par ^ 1, next);
  const bool final_stage = s.stage >= s.n_stages;
  int status = 0;
  bool stop = false;
  if (r != r) {
    stop = true;
    status = -3;
  } else if (final_stage && r <= s.tol && s.l >= 1) {
    // (the first residual compares with the initial u and is not used to stop)
    stop = true;
    status = 0;
  } else if (s.l + 1 >= s.max_iter) {
    stop = true;
    status = 1;
  }
  if (stop) {
    c->status = status;
    c->stop = 1;
    c->skip[par ^ 1] = 1;
  }
}

__device__ __forceinline__ void control_skip(Ctrl* c, int par) { c->skip[par ^ 1] = 1; }

// this thread's share of the residual partials of one problem
template <int NT = kBlock>
__device__ __forceinline__ void ctl_load(const ResPart* __restrict__ part, int nparts, float& m, float& den,
                                         float& num, float& du) {
  m = -__builtin_inff();
  den = num = du = 0.f;
  for (int k = threadIdx.x; k < nparts; k += NT) {
    res_merge<float>(m, den, num, part[k].m, part[k].den, part[k].num);
    du = fmaxf(du, part[k].du);
  }
}

// block reduction of the shares and the control step (every thread of the
// block calls it)
template <int NT = kBlock>
__device__ __forceinline__ void ctl_reduce_finish(Ctrl* c, const CtrlSnap& snap, const CtrlSlot& next, float m,
                                                  float den, float num, float du, double* __restrict__ hist, int par) {
  __shared__ ResPart tot;
  __syncthreads();   // the block's own reductions before this one are complete
  block_res_reduce<float, NT>(m, den, num, du, &tot);
  __syncthreads();
  if (threadIdx.x == 0)
    control_finish(c, snap, next, res_ratio(double(tot.num), double(tot.den)), double(tot.du), hist, par);
}

// Control step of iteration parity par by one block of NT threads.  One
// problem (nfields 0): the partials and the control fields are loaded before
// the skip flag is tested.  Several: the partials form nfields equal ranges,
// and r is the largest per-field residual; the threads of a wave share the
// fields, L lanes (a power of two) to a field.
template <int NT = kBlock>
__device__ __forceinline__ void control_block(Ctrl* c, const ResPart* __restrict__ part, int nparts,
                                              double* __restrict__ hist, int nfields, int par) {
  const CtrlSnap snap = ctrl_snap(c, par);
  const CtrlSlot next = ctrl_next(c, snap, par);
  if (nfields == 0) {
    float m, den, num, du;
    ctl_load<NT>(part, nparts, m, den, num, du);
    asm volatile("" ::"v"(m), "v"(den), "v"(num), "v"(du));
    if (c->skip[par]) {
      if (threadIdx.x == 0) control_skip(c, par);
      return;
    }
    ctl_reduce_finish<NT>(c, snap, next, m, den, num, du, hist, par);
    return;
  }
  if (c->skip[par]) {
    if (threadIdx.x == 0) control_skip(c, par);
    return;
  }
  __shared__ float smax[NT], sdu[NT];
  float rmax = -1.0f, du = 0.f;
  const int per = nparts / nfields;
  int L = 1;
  while (L < 64 && L < per && L * nfields < NT) L *= 2;
  const int sub = threadIdx.x & (L - 1);
  // (every lane runs every round, for the shuffles; lanes past the last field repeat it)
  for (int f0 = 0; f0 < nfields; f0 += NT / L) {
    const int f = f0 + (int)threadIdx.x / L < nfields ? f0 + (int)threadIdx.x / L : nfields - 1;
    float m = -__builtin_inff(), den = 0.f, num = 0.f;
    for (int k = f * per + sub; k < (f + 1) * per; k += L) {
      res_merge<float>(m, den, num, part[k].m, part[k].den, part[k].num);
      du = fmaxf(du, part[k].du);
    }
    for (int o = 1; o < L; o <<= 1) {
      const float m2 = __shfl_xor(m, o), d2 = __shfl_xor(den, o), n2 = __shfl_xor(num, o);
      res_merge<float>(m, den, num, m2, d2, n2);
    }
    const float rf = float(res_ratio(double(num), double(den)));
    rmax = (rf != rf || rmax != rmax) ? rf : (rf > rmax ? rf : rmax);
  }
  smax[threadIdx.x] = rmax;
  sdu[threadIdx.x] = du;
  __syncthreads();
  for (int off = NT / 2; off >= 1; off >>= 1) {
    if ((int)threadIdx.x < off) {
      const float a = smax[threadIdx.x], b = smax[threadIdx.x + off];
      smax[threadIdx.x] = (a != a || b != b) ? (a != a ? a : b) : (a > b ? a : b);
      sdu[threadIdx.x] = fmaxf(sdu[threadIdx.x], sdu[threadIdx.x + off]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) control_finish(c, snap, next, double(smax[0]), double(sdu[0]), hist, par);
}

// The block that hosts the control step (the last in x, added by the launch; the
// others of its column have no work), true for the blocks the caller returns
// from.  A launch of its own for a step of one block cost 4.5 us of the 58.6 us of an
// iteration on 6000 x 5000 points under the WF cost.
__device__ __forceinline__ bool control_hosted(const CtlHost& host, int side) {
  if ((int)blockIdx.x != host.block) return false;
  if (blockIdx.y == 0 && blockIdx.z == 0)
    control_block<kBlock>(host.c, host.parts, host.nparts, host.hist, 0, par_of(side));
  return true;
}

}  // namespace uot
