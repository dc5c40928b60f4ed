// Separable grid passes of libuot on whole lines held in LDS, with the passes
// of consecutive half-steps fused where they run along the same axis.
#include <algorithm>

#include "uot_bary.h"
#include "uot_device.h"
#include "uot_epilogue.h"
#include "uot_launch.h"

// ---------------------------------------------------------------------------
// One 1-D pass is out_i = log2 sum_t 2^{w_t - c (i - t)^2} (c = h^2 log2(e) /
// eps) along every line of one axis.  Outputs are taken in tiles of 16 cells
// (centre cI, offsets e = i - cI in -7.5 .. 7.5), taps in segments of TS cells
// (centre r, offsets t' = t - r).  With d = r - cI the exponent splits exactly:
//   w_t - c (i - t)^2 = [w_t - c t'^2] - 2c t' d + 2c e t' - c (e - d)^2,
// so the segment's share of the 16 outputs of a tile is
//   2^{m - c (e - d)^2} sum_t A[e][t'] 2^{z_t - m},  A[e][t'] = 2^{2c e t'},
//   z_t = [w_t - c t'^2] - 2c d t',  m = max_t z_t.
// A depends on nothing but c: it is one 16 x TS matrix of a launch, and the
// (line, output tile) pairs are the columns of one matrix product A B,
// B[t][(line, tile)] = 2^{z_t - m}: v_mfma_f32_16x16x4f32, or
// v_mfma_f64_16x16x4f64 in FP64.  A column's segments are joined by a
// log-sum-exp per output.  Executed exp2 per output: taps / 16 for B and 2 per
// segment for the joins.
// The segment length TS keeps c TS <= 6 in FP32 (63 in FP64): |log2 A| is at
// most 7.5 c TS <= 45 (473), the largest term of row e is at least 2^-45, and
// a term that underflows in B (2^-126; 2^-1022) is below 2^-81, so what is
// lost stays under 2^-27 of the row's sum.
//
// Pair launches (k_line_pair) hold L lines of an axis per block: the last pass
// of a half-step, its proxdiv epilogue, and at once the first pass of the next
// half-step, which runs along the same axis (the X half-step takes the axes
// last to first, the Y half-step first to last; 1-D kernels commute).  On
// planes (k_plane_pair: the last two axes of a 3-D grid in one block) it is
// two passes, epilogue, two passes.  So an iteration of a 2-D or 3-D grid is
// two launches, and the weights between the half-steps never leave the block.
//
// What bounds it (counters, 100 iterations each): one field of 256 x 256 cells, 256
// blocks, by latency (a launch of 16.5 k cycles, 7 us: a block's waves wait 63 % of
// them, its launch, the round trip for the taps, two passes of a few dependent
// exp2 / MFMA chains); 256 fields of 64 x 64 by VALU issue (65 % of the 36 k cycles of
// a launch; the MFMA, which runs beside none of it, another 11 %; 42 VALU to an MFMA,
// most of them in the joins and the epilogue).
// ---------------------------------------------------------------------------
namespace uot {

namespace {

template <typename T> struct LineNum;

template <> struct LineNum<float> {
  typedef float V4 __attribute__((ext_vector_type(4)));
  typedef float V2 __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ V4 mma(float a, float b, V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // output row of result register r in lane quarter q
  static __device__ __forceinline__ int row(int q, int r) { return 4 * q + r; }
  static __device__ __forceinline__ float exp2(float x) { return __builtin_amdgcn_exp2f(x); }
  // maximum over the four lanes l % 16 + {0, 16, 32, 48}
  static __device__ __forceinline__ float max_rows(float x) { return max_over_rows(x); }
  // 2^x for x = a b: the rounding of the product (up to 2^-24 of an exponent of
  // 45, 2^-53 of one of 473 in FP64) put back as a factor
  static __device__ __forceinline__ float exp2_prod(float a, float b) {
    const float p = a * b;
    const float lo = __builtin_fmaf(a, b, -p);
    const float v = __builtin_amdgcn_exp2f(p);
    return __builtin_fmaf(v, lo * float(kLn2), v);
  }
};

template <> struct LineNum<double> {
  typedef double V4 __attribute__((ext_vector_type(4)));
  typedef double V2 __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ V4 mma(double a, double b, V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int q, int r) { return q + 4 * r; }
  static __device__ __forceinline__ double exp2(double x) { return exp2_f64(x); }
  static __device__ __forceinline__ double max_rows(double x) {
    x = __builtin_fmax(x, __shfl_xor(x, 16));
    return __builtin_fmax(x, __shfl_xor(x, 32));
  }
  static __device__ __forceinline__ double exp2_prod(double a, double b) {
    const double p = a * b;
    const double lo = __builtin_fma(a, b, -p);
    const double v = exp2(p);
    return __builtin_fma(v, lo * kLn2, v);
  }
};

// c = h2 log2(e) / eps of a pass, rounded once in FP64 too
template <typename T> __device__ __forceinline__ T line_c(double h2, double eps, double le) {
  const double p = h2 * le;
  if constexpr (sizeof(T) == 4) return T(p);
  return p + __builtin_fma(h2, le_rest(eps, le), __builtin_fma(h2, le, -p));
}

// The launch-wide operands of a pass at one c: lane (q, l) holds, for its taps
// b VB 4 + VB q + s of a segment (VB consecutive ones per block of 4 VB), the
// entries A[l][t'] and the factors -2c t'.
template <typename T, int TS> struct LineOp {
  static constexpr int TPL = TS / 4;                 // taps per lane
  static constexpr int VB = TPL < 4 ? TPL : 4;       // consecutive ones
  T c;
  T A[TPL], k2[TPL];
  __device__ __forceinline__ void init(T c_) {
    const int lane = threadIdx.x & 63, q = lane >> 4, li = lane & 15;
    c = c_;
    const T e = T(li) - T(7.5);
#pragma unroll
    for (int k = 0; k < TPL; ++k) {
      const T tp = T((k / VB) * (4 * VB) + VB * q + k % VB) - T(0.5 * (TS - 1));
      k2[k] = T(-2) * c * tp;
      A[k] = LineNum<T>::exp2_prod(T(2) * c, e * tp);
    }
  }
  // [w_t - c t'^2] as it is stored for the pass; -inf stays -inf
  static __device__ __forceinline__ T shifted(T w, int t, T c) {
    const T tp = T(t & (TS - 1)) - T(0.5 * (TS - 1));
    return Num<T>::fma(-c * tp, tp, w);
  }
};

// LDS shape of nl lines of n cells: taps padded to whole segments (-inf),
// outputs to whole tiles; the line strides keep the 16 columns of a wave on
// distinct banks
struct LineShape {
  int nl, n, nt, nseg, ldl, ldp, ksn, ksh;   // ksn = 2^ksh
  unsigned rn, rt;   // ceil(2^32 / n), ceil(2^32 / nt): quotients of indexes below 2^16 by one multiply
};
__device__ __forceinline__ int quot(int a, unsigned r, int d) { return d == 1 ? a : (int)__umulhi((unsigned)a, r); }

// The pass over nl lines in buf (line l, tap t at buf[l ldl + t], shifted):
// the block's waves take the groups of 16 columns and, ksn at a time, the
// segments; each leaves its partial (m, s) of every output i of a line at
// pm / ps[(ks nl + l) ldp + i].  PART: over tiles output tiles from tile0 of one
// line, outputs counted from there.
template <typename T, int TS, int NT, bool PART = false>
__device__ __forceinline__ void line_pass(const LineOp<T, TS>& op, const LineShape& S, const T* buf, T* pm, T* ps,
                                          int tile0 = 0, int tiles = 0) {
  using N = LineNum<T>;
  using V4 = typename N::V4;
  constexpr int TPL = TS / 4, VB = LineOp<T, TS>::VB;
  constexpr int W = NT / 64;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int q = lane >> 4, li = lane & 15;
  const int ks = wv & (S.ksn - 1), gstep = W >> S.ksh;
  const int ncol = PART ? tiles : S.nl * S.nt;
  const int G = (ncol + 15) >> 4;
  T er[4];   // offsets e of the result rows
#pragma unroll
  for (int r = 0; r < 4; ++r) er[r] = T(N::row(q, r)) - T(7.5);
  for (int g = wv >> S.ksh; g < G; g += gstep) {
    const int col = g * 16 + li;
    const int cc = col < ncol ? col : ncol - 1;
    const int line = PART || S.nl == 1 ? 0 : quot(cc, S.rt, S.nt);
    const int I = cc - line * S.nt;
    const T* wl = buf + line * S.ldl + VB * q;
    T M[4], R[4];
    // segment seg: al[r] (its shift for row r) and a[r] (its sum)
    auto segment = [&](int seg, T (&al)[4], T (&a)[4]) {
      const T d = T(seg * TS - (PART ? tile0 + I : I) * 16) + T(0.5 * (TS - 1) - 7.5);
      T z[TPL];
      T m = Num<T>::ninf();
#pragma unroll
      for (int b = 0; b < TPL / VB; ++b) {
        const T* src = wl + seg * TS + b * (4 * VB);
        T x[VB];
        if constexpr (VB == 4) {
          const V4 v = *reinterpret_cast<const V4*>(src);
          x[0] = v[0]; x[1] = v[1]; x[2] = v[2]; x[3] = v[3];
        } else {
#pragma unroll
          for (int s = 0; s < VB; ++s) x[s] = src[s];
        }
#pragma unroll
        for (int s = 0; s < VB; ++s) {
          z[b * VB + s] = Num<T>::fma(op.k2[b * VB + s], d, x[s]);
          m = Num<T>::fmax(m, z[b * VB + s]);
        }
      }
      m = N::max_rows(m);
      const T msh = m == Num<T>::ninf() ? T(0) : m;
      V4 acc = {T(0), T(0), T(0), T(0)}, acc2 = {T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int k = 0; k < TPL; k += 2) {
        acc = N::mma(op.A[k], N::exp2(z[k] - msh), acc);
        acc2 = N::mma(op.A[k + 1], N::exp2(z[k + 1] - msh), acc2);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const T ed = er[r] - d;
        al[r] = Num<T>::fma(-op.c * ed, ed, m);
        a[r] = acc[r] + acc2[r];
      }
    };
    if (ks < S.nseg) {
      segment(ks, M, R);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        M[r] = Num<T>::ninf();
        R[r] = T(0);
      }
    }
    for (int seg = ks + S.ksn; seg < S.nseg; seg += S.ksn) {
      T al[4], a[4];
      segment(seg, al, a);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const T mn = Num<T>::fmax(M[r], al[r]);
        const T sh = mn == Num<T>::ninf() ? T(0) : mn;
        R[r] = R[r] * N::exp2(M[r] - sh) + a[r] * N::exp2(al[r] - sh);
        M[r] = mn;
      }
    }
    if (col < ncol) {
      const int o = (ks * S.nl + line) * S.ldp + I * 16;
      if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<V4*>(pm + o + 4 * q) = V4{M[0], M[1], M[2], M[3]};
        *reinterpret_cast<V4*>(ps + o + 4 * q) = V4{R[0], R[1], R[2], R[3]};
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pm[o + N::row(q, r)] = M[r];
          ps[o + N::row(q, r)] = R[r];
        }
      }
    }
  }
}

// log2 of output i of line l from the ksn partials (a power of two up to 8)
// line_pass left: their maximum, then the scaled sums side by side
template <typename T, int K>
__device__ __forceinline__ T line_merge(const T* pm, const T* ps, int o, int st) {
  using N = LineNum<T>;
  T m[K], s[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    m[k] = pm[o + k * st];
    s[k] = ps[o + k * st];
  }
  T mx = m[0];
#pragma unroll
  for (int k = 1; k < K; ++k) mx = Num<T>::fmax(mx, m[k]);
  if constexpr (K == 1) return mx + Num<T>::log2(s[0]);
  const T sh = mx == Num<T>::ninf() ? T(0) : mx;
#pragma unroll
  for (int k = 0; k < K; ++k) s[k] *= N::exp2(m[k] - sh);
#pragma unroll
  for (int w = K / 2; w >= 1; w /= 2)
#pragma unroll
    for (int k = 0; k < w; ++k) s[k] += s[k + w];
  return mx + Num<T>::log2(s[0]);
}
template <typename T>
__device__ __forceinline__ T line_result(const LineShape& S, const T* pm, const T* ps, int l, int i) {
  const int st = S.nl * S.ldp, o = l * S.ldp + i;
  switch (S.ksn) {
    case 1: return line_merge<T, 1>(pm, ps, o, st);
    case 2: return line_merge<T, 2>(pm, ps, o, st);
    case 4: return line_merge<T, 4>(pm, ps, o, st);
    default: return line_merge<T, 8>(pm, ps, o, st);
  }
}

// taps past the end of the lines
template <typename T, int TS, int NT>
__device__ __forceinline__ void line_pad(const LineShape& S, T* buf) {
  const int pad = S.nseg * TS - S.n;
  for (int t = threadIdx.x; t < S.nl * pad; t += NT) {
    const int l = t / pad;
    buf[l * S.ldl + S.n + (t - l * pad)] = Num<T>::ninf();
  }
}

// line group of a block of a launch of nb: consecutive groups on one XCD
// (workgroups go round the 8 XCDs), as neighbouring groups share cache lines
// of what they read or write transposed
__device__ __forceinline__ unsigned xcd_group(unsigned nb) {
  return (nb & 7) == 0 ? (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
}

template <typename T> __device__ __forceinline__ T* line_lds() {
  extern __shared__ __align__(32) unsigned char line_raw[];
  return reinterpret_cast<T*>(line_raw);
}

}  // namespace

// ---------------------------------------------------------------------------
// One pass along the axis of cells (a, i, b), element a n B + i B + b, with the
// epilogue ep (raw output or proxdiv); a block takes L = 2^lsh lines: L
// consecutive b of one a (B > 1), or L consecutive a (B == 1).  c32: c rounded to
// FP32, as the passes on FP32 data round it.
// ---------------------------------------------------------------------------
template <typename T, int TS, int NT, int EPT>
__global__ __launch_bounds__(NT) void k_line(const T* __restrict__ in, int64_t A, int64_t B, int lsh, LineShape S,
                                             double h2, int side, const Ctrl* __restrict__ c, EpiArgs<T> ep,
                                             int c32) {
  using Op = LineOp<T, TS>;
  T* const buf = line_lds<T>();
  T* const pm = buf + S.nl * S.ldl;
  T* const ps = pm + S.ksn * S.nl * S.ldp;
  const int n = S.n;
  const unsigned grp = xcd_group(gridDim.x);
  int64_t base, lstep;
  int valid;   // lines of this block
  if (B > 1) {
    const unsigned gpa = (unsigned)((B + S.nl - 1) >> lsh);
    const unsigned a = grp / gpa;
    const int64_t b0 = (int64_t)(grp - a * gpa) << lsh;
    base = (int64_t)a * n * B + b0;
    lstep = 1;
    valid = B - b0 < S.nl ? (int)(B - b0) : S.nl;
  } else {
    const int64_t a0 = (int64_t)grp << lsh;
    base = a0 * n;
    lstep = n;
    valid = A - a0 < S.nl ? (int)(A - a0) : S.nl;
  }
  const bool skip = skip_side(c, side);
  const double eps = c->eps[par_of(side)], le = c->le[par_of(side)];
  const int tot = S.nl * n;
  int l[EPT], i[EPT];
  int64_t el[EPT];
  bool ok[EPT];
  T x[EPT];
  EpiIn<T> xe[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int id = threadIdx.x + k * NT;
    if (B > 1) {
      l[k] = id & (S.nl - 1);
      i[k] = id >> lsh;
    } else {
      l[k] = quot(id, S.rn, n);
      i[k] = id - l[k] * n;
    }
    ok[k] = id < tot && l[k] < valid;
    el[k] = ok[k] ? base + l[k] * lstep + i[k] * B : 0;
    x[k] = in[el[k]];
  }
#pragma unroll
  for (int k = 0; k < EPT; ++k) xe[k] = epi_load<T>(el[k], ep);
  __builtin_amdgcn_sched_barrier(0);
  Op op;
  op.init(c32 ? T(line_c<float>(h2, eps, le)) : line_c<T>(h2, eps, le));
  const EpiK<T> K = epi_consts_of<T>(c, side, ep);
  __builtin_amdgcn_sched_barrier(0);
  // (keeps the loads ahead of the branch)
#pragma unroll
  for (int k = 0; k < EPT; ++k) asm volatile("" : "+v"(x[k]), "+v"(xe[k].ld), "+v"(xe[k].uo), "+v"(xe[k].lp));
  if (skip) return;
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    if (threadIdx.x + k * NT < tot)
      buf[l[k] * S.ldl + i[k]] = ok[k] ? Op::shifted(x[k], i[k], op.c) : Num<T>::ninf();
  line_pad<T, TS, NT>(S, buf);
  __syncthreads();
  line_pass<T, TS, NT>(op, S, buf, pm, ps);
  __syncthreads();
  ResAcc<T> ra;
  ra.init();
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    if (ok[k]) epi_apply<T>(el[k], line_result<T>(S, pm, ps, l[k], i[k]), xe[k], K, ep, ra);
  epi_finish<T, NT>(ep, ra, (int)grp);
}

// ---------------------------------------------------------------------------
// One raw pass of lines as in k_line, few long ones: a block holds one line and
// takes `tiles` output tiles of it (parts blocks to a line).  One block a line
// left most of the chip idle: an objective of 3000 cells took 1.31 ms.
// ---------------------------------------------------------------------------
template <typename T, int TS, int NT, int EPT>
__global__ __launch_bounds__(NT) void k_line_part(const T* __restrict__ in, int64_t B, int tiles, unsigned parts,
                                                  LineShape S, double h2, int side, const Ctrl* __restrict__ c,
                                                  T* __restrict__ out, int c32) {
  using Op = LineOp<T, TS>;
  if (skip_side(c, side)) return;
  T* const buf = line_lds<T>();
  T* const pm = buf + S.ldl;
  T* const ps = pm + S.ksn * S.ldp;
  const int n = S.n;
  const unsigned line = blockIdx.x / parts, a = line / (unsigned)B;
  const int tile0 = (int)(blockIdx.x - line * parts) * tiles;
  const int64_t base = (int64_t)a * n * B + (line - a * (unsigned)B);
  const double eps = c->eps[par_of(side)], le = c->le[par_of(side)];
  Op op;
  op.init(c32 ? T(line_c<float>(h2, eps, le)) : line_c<T>(h2, eps, le));
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int i = threadIdx.x + k * NT;
    if (i < n) buf[i] = Op::shifted(in[base + i * B], i, op.c);
  }
  line_pad<T, TS, NT>(S, buf);
  __syncthreads();
  line_pass<T, TS, NT, true>(op, S, buf, pm, ps, tile0, tiles);
  __syncthreads();
  const int i0 = tile0 * 16, cnt = n - i0 < tiles * 16 ? n - i0 : tiles * 16;
  for (int i = threadIdx.x; i < cnt; i += NT) out[base + (i0 + i) * B] = line_result<T>(S, pm, ps, 0, i);
}

// ---------------------------------------------------------------------------
// Contiguous lines in, transposed lines out: F fields of R lines of n cells
// (element f R n + r n + i), output element f R n + i R + r, so the next
// launch, along the other axes, reads contiguous lines again (a strided read
// costs a cache line per element and sits on the critical path; a scattered
// store does not).  A block takes L = 2^lsh lines of one field (MODE 0, 1), or
// line r of every field (MODE 2).
//   MODE 0: one pass, raw
//   MODE 1: the pass, the proxdiv epilogue ep, and the next half-step's first
//           pass, raw; the second pass runs at the eps of the same iteration
//           after an X epilogue, of the next one after a Y epilogue
//   MODE 2: as MODE 1 with the barycentre combine over the fields between the
//           passes (bw: weights and their logs; ep carries F2, v, log dy and
//           log h in lse_out)
// A launch that hosts the control step has one more block for it: it only
// reads the slot of this iteration and writes the next one's.
// ---------------------------------------------------------------------------
template <typename T, int TS, int NT, int EPT, int MODE>
__global__ __launch_bounds__(NT, NT == 1024 || (sizeof(T) == 4 && NT == 256 && TS <= 32) ? 4 : 2) void k_line_pair(
    const T* __restrict__ in, int64_t R, int lsh, LineShape S, double h2, int side, const Ctrl* __restrict__ c,
    EpiArgs<T> ep, T* __restrict__ out, BaryW bw) {
  using Op = LineOp<T, TS>;
  const int par = par_of(side);
  unsigned nb = gridDim.x;
  if (ep.host_ctl) {
    --nb;
    if (blockIdx.x == nb) {
      control_block<NT>(ep.host_ctl, ep.host_parts, ep.host_nparts, ep.host_hist, ep.host_fields, par);
      return;
    }
  }
  T* const buf = line_lds<T>();
  T* const pm = buf + S.nl * S.ldl;
  T* const ps = pm + S.ksn * S.nl * S.ldp;
  const int n = S.n;
  const unsigned grp = xcd_group(nb);
  int64_t base, obase, lstep;   // element of (line 0, cell 0), of its output, and the line step
  int64_t ostep;
  int valid = S.nl;             // lines of this block
  if constexpr (MODE == 2) {
    base = (int64_t)grp * n;
    obase = grp;
    lstep = ostep = R * n;
  } else {
    const unsigned gpf = (unsigned)((R + S.nl - 1) >> lsh);
    const unsigned f = grp / gpf;
    const int64_t r0 = (int64_t)(grp - f * gpf) << lsh;
    base = ((int64_t)f * R + r0) * n;
    obase = (int64_t)f * R * n + r0;
    lstep = n;
    ostep = 1;
    valid = R - r0 < S.nl ? (int)(R - r0) : S.nl;
  }
  // the control fields (scalar loads), then this thread's elements (line l,
  // cell i): taps and epilogue operands, all in flight together; the operands
  // of the passes are built meanwhile
  const bool skip = skip_side(c, side);
  const bool same = half_of(side) == 0 || MODE == 0;
  const double eps = c->eps[par], eps_w = same ? eps : c->eps_after[par];
  const double le = c->le[par], le_w = same ? le : c->le_after[par];
  const int tot = S.nl * n;
  int l[EPT], i[EPT];
  int64_t el[EPT];
  bool ok[EPT];
  T x[EPT];
  EpiIn<T> xe[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int id = threadIdx.x + k * NT;
    l[k] = quot(id, S.rn, n);
    i[k] = id - l[k] * n;
    ok[k] = id < tot && l[k] < valid;
    el[k] = ok[k] ? base + l[k] * lstep + i[k] : 0;
    x[k] = in[el[k]];
  }
  if constexpr (MODE == 1) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) xe[k] = epi_load<T>(el[k], ep);
  } else if constexpr (MODE == 2) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      xe[k].ld = ep.logd[base + i[k]];
      xe[k].uo = xe[k].lp = T(0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  Op op;
  op.init(line_c<T>(h2, eps, le));
  EpiK<T> K{};
  if constexpr (MODE != 0) K = epi_consts<T>(eps, le, eps_w, le_w, c->coef[par][half_of(side)], c->zeta);
  __builtin_amdgcn_sched_barrier(0);
  // (keeps the loads ahead of the branch)
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    asm volatile("" : "+v"(x[k]));
    if constexpr (MODE != 0) asm volatile("" : "+v"(xe[k].ld), "+v"(xe[k].uo), "+v"(xe[k].lp));
  }
  if (skip) return;
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    if (threadIdx.x + k * NT < tot)
      buf[l[k] * S.ldl + i[k]] = ok[k] ? Op::shifted(x[k], i[k], op.c) : Num<T>::ninf();
  line_pad<T, TS, NT>(S, buf);
  __syncthreads();
  line_pass<T, TS, NT>(op, S, buf, pm, ps);
  __syncthreads();
  ResAcc<T> ra;
  ra.init();
  if constexpr (MODE == 1) {
    if (le_w != le) op.init(line_c<T>(h2, eps_w, le_w));
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      T w = Num<T>::ninf();
      if (ok[k]) w = epi_core<T>(el[k], line_result<T>(S, pm, ps, l[k], i[k]), xe[k], K, ep, ra);
      if (threadIdx.x + k * NT < tot) buf[l[k] * S.ldl + i[k]] = Op::shifted(w, i[k], op.c);
    }
  } else if constexpr (MODE == 2) {
    // the products of the line's cells, all fields side by side: field l,
    // cell i at t2[l n + i]
    T* const t2 = ps + S.ksn * S.nl * S.ldp;
    T* const lh = t2 + tot;
    if (le_w != le) op.init(line_c<T>(h2, eps_w, le_w));
    T r[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      r[k] = T(0);
      if (ok[k]) {
        r[k] = line_result<T>(S, pm, ps, l[k], i[k]);
        t2[l[k] * n + i[k]] = r[k];
      }
    }
    __syncthreads();
    const bool root = ep.F.kind == 2 || ep.F.kind == 3;
    if (root) {
      // L lanes to a cell; lanes past the last cell repeat it
      const int L = bary_lanes(S.nl, ep.F.kind == 2 || ep.F.has_lo);
      const int sub = threadIdx.x & (L - 1);
      for (int j0 = 0; j0 < n; j0 += NT / L) {
        const int j = j0 + (int)threadIdx.x / L;
        const T logh = bary_root<T>(t2 + (j < n ? j : n - 1), n, S.nl, bw, ep.F, K.k.eps.c, sub, L);
        if (sub == 0 && j < n) lh[j] = logh;
      }
      __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      if (!ok[k]) continue;
      const T logh = root ? lh[i[k]] : bary_mean<T>(t2 + i[k], n, S.nl, bw, ep.F, K.k.eps.c);
      if (l[k] == 0 && ep.lse_out) ep.lse_out[el[k]] = logh;
      const T vn = proxdiv_pot<T>(ep.F, logh, r[k] * T(kLn2), K.k);
      ep.pot[el[k]] = vn;
      const T w = r[k] == Num<T>::ninf() ? r[k] : epi_weight<T>(vn, K.kw, K.kwl, xe[k].ld * T(kLog2e));
      buf[l[k] * S.ldl + i[k]] = Op::shifted(w, i[k], op.c);
    }
  }
  if constexpr (MODE != 0) {
    __syncthreads();
    line_pass<T, TS, NT>(op, S, buf, pm, ps);
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int id = threadIdx.x + k * NT;
    if constexpr (MODE == 2) {
      if (ok[k]) out[obase + l[k] * ostep + i[k] * R] = line_result<T>(S, pm, ps, l[k], i[k]);
    } else {
      // (lines fastest: neighbouring lines are neighbours in the output)
      const int ol = id & (S.nl - 1), oi = id >> lsh;
      if (id < tot && ol < valid) out[obase + ol + (int64_t)oi * R] = line_result<T>(S, pm, ps, ol, oi);
    }
  }
  if constexpr (MODE == 1) epi_finish<T, NT>(ep, ra, (int)grp);
}

// ---------------------------------------------------------------------------
// Planes of the last two axes of a 3-D grid, one per block: F fields of n0
// planes of n1 x n2 cells.  FULL: the Y product's passes along axes 1 and 2,
// the proxdiv epilogue ep, and the next X product's passes along axes 2 and 1;
// else only the latter two.  The output is transposed (element f n0 n1 n2 + b n0
// + i0, b = i1 n2 + i2): contiguous lines of axis 0.
// S1: lines of axis 1 (n2 of them), S2: lines of axis 2 (n1).
// ---------------------------------------------------------------------------
template <typename T, int TS, int NT, int EPT, bool FULL>
__global__ __launch_bounds__(NT) void k_plane_pair(const T* __restrict__ in, int n0, LineShape S1, LineShape S2,
                                                   double h1, double h2, int side, const Ctrl* __restrict__ c,
                                                   EpiArgs<T> ep, T* __restrict__ out) {
  using Op = LineOp<T, TS>;
  const int par = par_of(side);
  unsigned nb = gridDim.x;
  if (ep.host_ctl) {
    --nb;
    if (blockIdx.x == nb) {
      control_block<NT>(ep.host_ctl, ep.host_parts, ep.host_nparts, ep.host_hist, ep.host_fields, par);
      return;
    }
  }
  T* const buf = line_lds<T>();
  const int lb1 = S1.nl * S1.ldl, lb2 = S2.nl * S2.ldl;
  const int pp1 = S1.ksn * S1.nl * S1.ldp, pp2 = S2.ksn * S2.nl * S2.ldp;
  T* const pm = buf + (lb1 > lb2 ? lb1 : lb2);
  T* const ps = pm + (pp1 > pp2 ? pp1 : pp2);
  const unsigned grp = xcd_group(nb);
  const int n2 = S2.n, tot = S1.n * n2;
  const int64_t base = (int64_t)grp * tot;
  const unsigned f = grp / (unsigned)n0;
  const int64_t obase = (int64_t)f * n0 * tot + (grp - f * (unsigned)n0);
  const bool skip = skip_side(c, side);
  const double eps = c->eps[par], eps_w = FULL ? c->eps_after[par] : eps;
  const double le = c->le[par], le_w = FULL ? c->le_after[par] : le;
  int i1[EPT], i2[EPT];
  int64_t el[EPT];
  bool ok[EPT];
  T x[EPT];
  EpiIn<T> xe[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int id = threadIdx.x + k * NT;
    i1[k] = quot(id, S2.rn, n2);
    i2[k] = id - i1[k] * n2;
    ok[k] = id < tot;
    el[k] = ok[k] ? base + id : 0;
    x[k] = in[el[k]];
  }
  if constexpr (FULL) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) xe[k] = epi_load<T>(el[k], ep);
  }
  __builtin_amdgcn_sched_barrier(0);
  const T c1 = line_c<T>(h1, eps, le), c2 = line_c<T>(h2, eps, le);
  Op op;
  op.init(FULL ? c1 : c2);
  EpiK<T> K{};
  if constexpr (FULL) K = epi_consts<T>(eps, le, eps_w, le_w, c->coef[par][1], c->zeta);
  __builtin_amdgcn_sched_barrier(0);
  // (keeps the loads ahead of the branch)
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    asm volatile("" : "+v"(x[k]));
    if constexpr (FULL) asm volatile("" : "+v"(xe[k].ld), "+v"(xe[k].uo), "+v"(xe[k].lp));
  }
  if (skip) return;
  ResAcc<T> ra;
  ra.init();
  if constexpr (FULL) {
    // axis 1: line i2, tap i1
#pragma unroll
    for (int k = 0; k < EPT; ++k)
      if (ok[k]) buf[i2[k] * S1.ldl + i1[k]] = Op::shifted(x[k], i1[k], c1);
    line_pad<T, TS, NT>(S1, buf);
    __syncthreads();
    line_pass<T, TS, NT>(op, S1, buf, pm, ps);
    __syncthreads();
    // axis 2: line i1, tap i2
    op.init(c2);
#pragma unroll
    for (int k = 0; k < EPT; ++k)
      if (ok[k]) buf[i1[k] * S2.ldl + i2[k]] = Op::shifted(line_result<T>(S1, pm, ps, i2[k], i1[k]), i2[k], c2);
    line_pad<T, TS, NT>(S2, buf);
    __syncthreads();
    line_pass<T, TS, NT>(op, S2, buf, pm, ps);
    __syncthreads();
    if (le_w != le) op.init(line_c<T>(h2, eps_w, le_w));
#pragma unroll
    for (int k = 0; k < EPT; ++k)
      if (ok[k]) {
        const T w = epi_core<T>(el[k], line_result<T>(S2, pm, ps, i1[k], i2[k]), xe[k], K, ep, ra);
        buf[i1[k] * S2.ldl + i2[k]] = Op::shifted(w, i2[k], op.c);
      }
  } else {
#pragma unroll
    for (int k = 0; k < EPT; ++k)
      if (ok[k]) buf[i1[k] * S2.ldl + i2[k]] = Op::shifted(x[k], i2[k], c2);
    line_pad<T, TS, NT>(S2, buf);
  }
  __syncthreads();
  line_pass<T, TS, NT>(op, S2, buf, pm, ps);
  __syncthreads();
  const T c1w = line_c<T>(h1, eps_w, le_w);
  op.init(c1w);
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    if (ok[k]) buf[i2[k] * S1.ldl + i1[k]] = Op::shifted(line_result<T>(S2, pm, ps, i1[k], i2[k]), i1[k], c1w);
  line_pad<T, TS, NT>(S1, buf);
  __syncthreads();
  line_pass<T, TS, NT>(op, S1, buf, pm, ps);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < EPT; ++k)
    if (ok[k])
      out[obase + (int64_t)(threadIdx.x + k * NT) * n0] = line_result<T>(S1, pm, ps, i2[k], i1[k]);
  if constexpr (FULL) epi_finish<T, NT>(ep, ra, (int)grp);
}

// ---------------------------------------------------------------------------
// Whole iterations of one problem on a 1-D grid, in one block: both half-steps
// run along the only axis, so the weights stay in LDS and the potentials in
// registers, and `chunk` iterations are one launch.  The block's first wave
// also takes the control step's decision.  exy[0], exy[1]: the X and Y
// epilogues (potentials, log densities, log weights, penalties).
// It is bound by the latency of a half-step (two per iteration): at 256 cells 5 k
// cycles in FP32 and 11 k in FP64 (one 16-column group whose segments go over 8
// waves; of these waves' time 40 % waits for memory or a barrier, 26 % for issue).
// ---------------------------------------------------------------------------
template <typename T, int TS, int NT, int EPT>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : 2) void k_line_loop(LineShape S, double h2, Ctrl* c, EpiArgs<T> ex,
                                                                      EpiArgs<T> ey, double* __restrict__ hist,
                                                                      int chunk) {
  using Op = LineOp<T, TS>;
  if (c->stop) return;
  __shared__ ResPart tot;
  __shared__ int stopped;   // 0 running, else 1 + the index of the status below
  T* const buf = line_lds<T>();
  T* const pm = buf + S.ldl;
  T* const ps = pm + S.ksn * S.ldp;
  const int n = S.n;
  EpiIn<T> xe[EPT], ye[EPT];
  T w[EPT];
  bool ok[EPT];
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int i = threadIdx.x + k * NT;
    ok[k] = i < n;
    xe[k] = epi_load<T>(ok[k] ? i : 0, ex);
    ye[k] = epi_load<T>(ok[k] ? i : 0, ey);
  }
  int64_t l = c->iter;
  const int64_t max_iter = c->max_iter;
  const int n_stages = c->n_stages;
  const double tol = c->tol;
  int sn = stage_at(c, l);
  double eps = c->eps_tab[sn], le = kLog2e / eps;
  EpiK<T> KX = uniform(epi_consts<T>(eps, le, eps, le, ctrl_coef(c, 0, eps), 0.0)), KY;
  Op op;
  op.init(line_c<T>(h2, eps, le));
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    const int i = threadIdx.x + k * NT;
    w[k] = ye[k].uo == Num<T>::pinf() ? Num<T>::ninf()
                                      : epi_weight<T>(ye[k].uo, KX.ke, KX.kel, ye[k].ld * T(kLog2e));
    if (ok[k]) buf[i] = Op::shifted(w[k], i, op.c);
  }
  line_pad<T, TS, NT>(S, buf);
  if (threadIdx.x == 0) stopped = 0;
  double r = 0.0, du = 0.0;
  for (int it = 0; it < chunk; ++it) {
    __syncthreads();
    line_pass<T, TS, NT>(op, S, buf, pm, ps);
    const int sn1 = stage_at(c, l + 1);
    const double eps1 = sn1 == sn ? eps : c->eps_tab[sn1], le1 = sn1 == sn ? le : kLog2e / eps1;
    if (it == 0 || sn1 != sn || KY.ke != KX.ke)
      KY = uniform(epi_consts<T>(eps, le, eps1, le1, ctrl_coef(c, 1, eps), 0.0));
    __syncthreads();
    ResAcc<T> ra;
    ra.init();
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int i = threadIdx.x + k * NT;
      if (ok[k]) {
        const T wu = epi_core<T>(i, line_result<T>(S, pm, ps, 0, i), xe[k], KX, ex, ra);
        buf[i] = Op::shifted(wu, i, op.c);
      }
    }
    block_res_reduce<T, NT>(ra.m, ra.den, ra.num, ra.du, &tot);   // (holds a barrier: the weights are in place)
    if (threadIdx.x == 0) {
      r = res_ratio(double(tot.num), double(tot.den));
      du = double(tot.du);
      if (hist) hist[l] = r;
      // (the first residual compares with the initial u and is not used to stop)
      if (r != r) stopped = 1;
      else if (sn >= n_stages && r <= tol && l >= 1) stopped = 2;
      else if (l + 1 >= max_iter) stopped = 3;
    }
    line_pass<T, TS, NT>(op, S, buf, pm, ps);
    __syncthreads();
    ++l;
    if (sn1 != sn) op.init(line_c<T>(h2, eps1, le1));
    ResAcc<T> none;
    none.init();
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int i = threadIdx.x + k * NT;
      if (ok[k]) {
        const T wv = epi_core<T>(i, line_result<T>(S, pm, ps, 0, i), ye[k], KY, ey, none);
        buf[i] = Op::shifted(wv, i, op.c);
      }
    }
    if (sn1 != sn) {
      sn = sn1;
      eps = eps1;
      le = le1;
      KX = uniform(epi_consts<T>(eps, le, eps, le, ctrl_coef(c, 0, eps), 0.0));
    }
    if (stopped) break;
  }
  if (threadIdx.x == 0) {
    c->iter = l;
    c->res = r;
    c->du = du;
    const int p = (int)(l & 1);
    set_slot(c, p, slot_values(c, stage_at(c, l), stage_at(c, l + 1), -1));
    if (stopped) {
      c->status = stopped == 1 ? -3 : stopped - 2;
      c->stop = 1;
      c->skip[p] = 1;
    }
  }
}

// dst[f][b][a] = src[f][a][b], or its log (log 1: densities, -inf where there is
// none; 2: weights), a block per 16 x 16 tile; grid = (ceil(Nb / 16), ceil(Na / 16), fields)
template <typename T>
__global__ __launch_bounds__(256) void k_transpose(const T* __restrict__ src, T* __restrict__ dst, int64_t Na,
                                                   int64_t Nb, int log) {
  __shared__ T t[16][17];
  const int x = threadIdx.x & 15, y = threadIdx.x >> 4;
  const int64_t fo = (int64_t)blockIdx.z * Na * Nb;
  const int64_t a = (int64_t)blockIdx.y * 16 + y, b = (int64_t)blockIdx.x * 16 + x;
  if (a < Na && b < Nb) {
    const T v = src[fo + a * Nb + b];
    t[y][x] = log == 0 ? v : (v > T(0) || log == 2) ? Num<T>::log(v) : Num<T>::ninf();
  }
  __syncthreads();
  const int64_t a2 = (int64_t)blockIdx.y * 16 + x, b2 = (int64_t)blockIdx.x * 16 + y;
  if (a2 < Na && b2 < Nb) dst[fo + b2 * Na + a2] = t[x][y];
}

// ---------------------------------------------------------------------------
// launch shapes
// ---------------------------------------------------------------------------
// longest segment for c (0: the pass does not apply).  FP32: c TS <= 6 and at
// least 8 taps, i.e. c <= 0.75; beyond that a kernel is a few cells wide and
// the direct passes take it.
// FP64: at most 32 taps, which take all 256 registers of a thread in blocks of 512 and
// spill 12 to 88 in those of 1024.
template <typename T> static int line_ts(double c) {
  const double top = sizeof(T) == 4 ? 6.0 : 63.0;
  for (int ts = sizeof(T) == 4 ? 64 : 32; ts >= (sizeof(T) == 4 ? 8 : 16); ts /= 2)
    if (c * ts <= top) return ts;
  return 0;
}

// Lines along a long axis that a line pass needs to keep up with the passes
// over parts of lines (0: any number will do), as a block holds a whole line.
// Measured (us an iteration, these passes / the others; tf: the tile-factored
// pass takes the axis; last: contiguous):
//   FP64, last: 24 x 560 51 / 47, 32 x 560 57 / 61, 16 x 850 77 / 60, 32 x 1000 94 / 91,
//     40 x 2048 303 / 328, 16 x 4096 1070 / 524; first: 4096 x 8 1071 / 2555
//   FP32 tf, last: 8 x 896 31 / 30, 64 x 1024 34 / 35, 64 x 2048 100 / 79, 72 x 2048 103 /
//     107, 72 x 4096 364 / 304, 100 x 4096 365 / 415; first: 512 x 8 16 / 23, 896 x 40
//     36 / 30, 1024 x 64 35 / 29, 1024 x 72 36 / 41, 2048 x 128 105 / 94, 2048 x 150 110 / 131
//   FP32 else, last: 8 x 1000 33 / 35, 30 x 1500 63 / 55, 64 x 1500 64 / 77, 64 x 2050 148 /
//     134, 100 x 2050 154 / 185; first: 1500 x 8 63 / 116
int64_t line_min_lines(bool f64, bool tf, bool last, int64_t n) {
  if (f64) return last && n > 512 ? (n < 768 ? 32 : 40) : 0;
  if (tf && last) return n < 1024 ? 0 : n < 3072 ? 72 : 96;
  if (tf) return n < 704 ? 0 : n < 1536 ? 72 : 144;
  return last && n > 1024 ? (n <= 2048 ? 56 : 72) : 0;
}

bool line_applies(bool f64, double c) { return (f64 ? line_ts<double>(c) : line_ts<float>(c)) > 0; }

// Lines per block: one while that gives fewer than 512 blocks (two per
// compute unit: a block's waves wait on its own barriers), else up to 1024
// elements (4 per thread), so that a wave's 16 columns and its operand set-up
// are shared; and never more than max_blocks blocks (the room of the residual
// partials).  `groups` groups of `per` lines each, no block across two groups.
static int line_lsh(int n, int64_t groups, int64_t per, int max_blocks) {
  auto blocks = [&](int lsh) { return groups * ((per + ((int64_t)1 << lsh) - 1) >> lsh); };
  int lsh = 0;
  while (((int64_t)n << (lsh + 1)) <= 1024 && lsh < 6 &&
         (blocks(lsh) > max_blocks || (lsh < 4 && blocks(lsh + 1) >= 512)))
    ++lsh;
  return lsh;
}

int64_t line_blocks(int n, int64_t groups, int64_t per, int max_blocks) {
  const int lsh = line_lsh(n, groups, per, max_blocks);
  return groups * ((per + ((int64_t)1 << lsh) - 1) >> lsh);
}

constexpr int kLineMaxCells = 4096;   // elements of a block: 1024 threads of 4
constexpr size_t kLineLds = 160 * 1024;   // LDS of a compute unit
// what a paired kernel of NT threads declares beside its dynamic LDS: the
// partials of block_lse_reduce and control_block, and the few of the others
template <typename T> constexpr size_t line_static_lds(int threads) {
  return (size_t)threads * (2 * sizeof(T) + 2 * sizeof(float)) + 1024;
}

// segment length and LDS shape of a pass over nl lines of n cells:
// the segments go over the waves when there are fewer groups of 16 columns
// than waves, in shorter segments if need be
// (tiles: a block's output tiles where it takes a part of one line)
static void line_shape(int nl, int n, int threads, int ts_max, int ts_min, LineShape& S, int& ts, int tiles = 0) {
  const int W = threads / 64;
  if (threads == 1024) ts_max = std::min(ts_max, 32);
  S.nl = nl;
  S.n = n;
  S.nt = (n + 15) / 16;
  const int G = ((tiles ? tiles : nl * S.nt) + 15) / 16;
  int ks = 1;
  while (ks < 8 && G * ks * 2 <= W) ks *= 2;
  ts = ts_max;
  while (ts > ts_min && ts > 16 && (n + ts - 1) / ts < ks) ts /= 2;
  S.nseg = (n + ts - 1) / ts;
  while (ks > S.nseg) ks /= 2;
  S.ksn = ks;
  S.ksh = 0;
  while ((1 << S.ksh) < ks) ++S.ksh;
  S.ldl = S.nseg * ts + 4;
  S.ldp = (tiles ? tiles : S.nt) * 16 + 4;
  S.rn = (unsigned)(((1ull << 32) + n - 1) / n);
  S.rt = (unsigned)(((1ull << 32) + S.nt - 1) / S.nt);
}

template <typename T> static size_t line_lds_bytes(const LineShape& S) {
  return sizeof(T) * ((size_t)S.nl * S.ldl + 2 * (size_t)S.ksn * S.nl * S.ldp);
}

template <typename K> static void line_big_lds(K kernel, size_t bytes) {
  if (bytes > 64 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)bytes);
}

// Threads of a block of `tot` elements in a launch of `blocks`: up to 512
// elements have a thread each of 512 (segments then go over 8 waves); up to
// 1024 a thread each of 1024 where the launch has about a block per compute
// unit or fewer (latency), else 256 threads with 4 each (throughput: the
// operand set-up of a wave is shared by more columns); beyond, 1024 with 4.
// Blocks of 1024 threads take segments of at most 32 taps (registers).
static int line_threads(int tot, int64_t blocks) {
  return tot <= 512 ? 512 : (tot <= 1024 && blocks > 320) ? 256 : 1024;
}

#define UOT_LINE_EPT(CALL, TS)                                             \
  if (tot <= 512) CALL(TS, 512, 1);                                        \
  else if (nthr == 256) CALL(TS, 256, 4);                                  \
  else if constexpr (TS <= 32) {                                           \
    if (tot <= 1024) CALL(TS, 1024, 1);                                    \
    else CALL(TS, 1024, 4);                                                \
  }
#define UOT_LINE_TS(CALL)                  \
  if (ts == 32) {                          \
    UOT_LINE_EPT(CALL, 32)                 \
  } else if (ts == 16) {                   \
    UOT_LINE_EPT(CALL, 16)                 \
  } else if constexpr (sizeof(T) == 4) {   \
    if (ts == 64) {                        \
      UOT_LINE_EPT(CALL, 64)               \
    } else {                               \
      UOT_LINE_EPT(CALL, 8)                \
    }                                      \
  }

// A raw pass over fewer than 256 lines of more than 16 tiles: parts of a line of
// at least 16 tiles (a wave's columns), up to 256 blocks
template <typename T>
static bool launch_line_part(const T* in, int64_t A, int n, int64_t B, double h, double c_max, int side, const Ctrl* c,
                             T* out, hipStream_t s, bool c32) {
  const int64_t lines = A * B;
  const int nt = (n + 15) / 16;
  if (nt <= 16 || lines > 128) return false;
  const int want = (int)std::min<int64_t>((nt + 15) / 16, 256 / lines);
  const int tiles = ((nt + want - 1) / want + 15) / 16 * 16;
  if (tiles >= nt) return false;
  const unsigned parts = (unsigned)((nt + tiles - 1) / tiles), blocks = (unsigned)lines * parts;
  const int tot = n;
  const int nthr = line_threads(tot, 1);
  LineShape S;
  int ts;
  line_shape(1, n, nthr, line_ts<T>(c_max), sizeof(T) == 4 ? 8 : 16, S, ts, tiles);
  const size_t lds = line_lds_bytes<T>(S);
#define UOT_LN(TS, NT, EPT)                                                                                        \
  do {                                                                                                             \
    if constexpr (NT != 256) {                                                                                     \
      line_big_lds(k_line_part<T, TS, NT, EPT>, lds);                                                              \
      hipLaunchKernelGGL((k_line_part<T, TS, NT, EPT>), dim3(blocks), dim3(NT), lds, s, in, B, tiles, parts, S,    \
                         h * h, side, c, out, c32 ? 1 : 0);                                                        \
    }                                                                                                              \
  } while (0)
  UOT_LINE_TS(UOT_LN)
#undef UOT_LN
  return true;
}

template <typename T>
void launch_line(const T* in, int64_t A, int n, int64_t B, double h, double c_max, int max_blocks, int side,
                 const Ctrl* c, const EpiArgs<T>& ep, hipStream_t s, bool c32) {
  if (ep.mode == EPI_RAW && launch_line_part<T>(in, A, n, B, h, c_max, side, c, ep.out, s, c32)) return;
  const int lsh = B > 1 ? line_lsh(n, A, B, max_blocks) : line_lsh(n, 1, A, max_blocks);
  const unsigned blocks = (unsigned)(B > 1 ? line_blocks(n, A, B, max_blocks) : line_blocks(n, 1, A, max_blocks));
  const int tot = n << lsh;
  const int nthr = line_threads(tot, blocks);
  LineShape S;
  int ts;
  line_shape(1 << lsh, n, nthr, line_ts<T>(c_max), sizeof(T) == 4 ? 8 : 16, S, ts);
  const size_t lds = line_lds_bytes<T>(S);
#define UOT_LN(TS, NT, EPT)                                                                                       \
  do {                                                                                                            \
    line_big_lds(k_line<T, TS, NT, EPT>, lds);                                                                    \
    hipLaunchKernelGGL((k_line<T, TS, NT, EPT>), dim3(blocks), dim3(NT), lds, s, in, A, B, lsh, S, h * h, side, c, \
                       ep, c32 ? 1 : 0);                                                                          \
  } while (0)
  UOT_LINE_TS(UOT_LN)
#undef UOT_LN
}

template <typename T>
void launch_line_pair(const T* in, int64_t F, int64_t R, int n, double h, double c_max, int max_blocks, int side,
                      const Ctrl* c, const EpiArgs<T>* ep, T* out, hipStream_t s) {
  const int lsh = line_lsh(n, F, R, max_blocks);
  const unsigned blocks = (unsigned)line_blocks(n, F, R, max_blocks) + (ep && ep->host_ctl ? 1 : 0);
  const int tot = n << lsh;
  const int nthr = line_threads(tot, blocks);
  LineShape S;
  int ts;
  line_shape(1 << lsh, n, nthr, line_ts<T>(c_max), sizeof(T) == 4 ? 8 : 16, S, ts);
  const size_t lds = line_lds_bytes<T>(S);
  const EpiArgs<T> none{};
#define UOT_LN(TS, NT, EPT)                                                                                       \
  do {                                                                                                            \
    if (ep) {                                                                                                     \
      line_big_lds(k_line_pair<T, TS, NT, EPT, 1>, lds);                                                          \
      hipLaunchKernelGGL((k_line_pair<T, TS, NT, EPT, 1>), dim3(blocks), dim3(NT), lds, s, in, R, lsh, S, h * h,  \
                         side, c, *ep, out, BaryW{});                                                        \
    } else {                                                                                                      \
      line_big_lds(k_line_pair<T, TS, NT, EPT, 0>, lds);                                                          \
      hipLaunchKernelGGL((k_line_pair<T, TS, NT, EPT, 0>), dim3(blocks), dim3(NT), lds, s, in, R, lsh, S, h * h,  \
                         side, c, none, out, BaryW{});                                                       \
    }                                                                                                             \
  } while (0)
  UOT_LINE_TS(UOT_LN)
#undef UOT_LN
}

// F fields of a line in one block, with room for their products side by side
// and a row of log h: launch shape and dynamic LDS
template <typename T> struct BaryShape {
  LineShape S;
  int ts, nthr;
  size_t lds;
  BaryShape(int F, int n, double c_max, int64_t blocks) {
    nthr = line_threads(F * n, blocks);
    line_shape(F, n, nthr, line_ts<T>(c_max), sizeof(T) == 4 ? 8 : 16, S, ts);
    lds = line_lds_bytes<T>(S) + sizeof(T) * (size_t)(F * n + n);
  }
  bool fits() const { return lds + line_static_lds<T>(nthr) <= kLineLds; }
};
// (launched over R rows, with and without the block of the control step)
template <typename T> static bool bary_fits(int64_t F, int64_t R, int n, double c_max) {
  return F * n <= kLineMaxCells && BaryShape<T>((int)F, n, c_max, R).fits() &&
         BaryShape<T>((int)F, n, c_max, R + 1).fits();
}
bool line_bary_fits(bool f64, int64_t F, int64_t R, int n, double c_max) {
  return f64 ? bary_fits<double>(F, R, n, c_max) : bary_fits<float>(F, R, n, c_max);
}

// Passes of a barycentre whose combine finds a root (TV, RG) over F inputs of
// R x n cells.  A block of the paired pass holds a row's n cells and searches
// them in rounds of NT / L, every round 2 F evaluations of F terms (bary_root),
// while the combine of its own launch spreads all cells over the chip: pairing
// wins while the rounds are few, or while a few inputs of many cells make the
// transposed store of the products the dearer part.  Where it does not, a pass
// per launch, except on the smallest grids, whose time is that of their
// launches and whose older passes (FP32: tile-factored axes, tf) take fewer
// cells a block.  Measured (us an iteration, TV, paired / a pass per launch /
// older passes): FP32 16 x 64 x 64 33.1 / 37.0 / 35.2, 10 x 112 x 112 46.0 / 40.5 /
// 40.2, 48 x 64 x 64 147 / 80 / 83, 10 x 80 x 80 40.0 / 41.5 / 33.1, 30 x 64 x 64
// - / 57.1 / 53.4, 20 x 50 x 50 - / 48.4 / 47.3, 10 x 150 x 150 65.5 / 70.3 / 95.6;
// FP64 8 x 64 x 64 35.4 / 37.3 / 41.0, 24 x 96 x 96 176 / 112 / 214, 12 x 48 x 48
// 57.4 / 55.5 / 51.7, 12 x 160 x 160 153 / 167 / 373.
int line_bary_root_passes(bool f64, int64_t F, int64_t R, int n, bool two_breaks, bool tf) {
  const int64_t cells = F * R * n;
  const int L = bary_lanes((int)F, two_breaks), NT = line_threads((int)F * n, R);
  const int64_t rounds = (n + NT / L - 1) / (NT / L), evals = rounds * F;
  const bool many = evals >= (f64 ? 24 : rounds > 2 ? 30 : 48);
  if (!many || (F <= 12 && cells >= 200000)) return 2;
  return cells < (!f64 && tf ? 130000 : 56000) ? 0 : 1;
}

template <typename T>
void launch_line_bary(const T* in, int64_t F, int64_t R, int n, double h, double c_max, int side, const Ctrl* c,
                      const EpiArgs<T>& ep, T* out, const BaryW& bw, hipStream_t s) {
  const unsigned blocks = (unsigned)R + (ep.host_ctl ? 1 : 0);
  const int tot = (int)F * n;
  const BaryShape<T> sh((int)F, n, c_max, blocks);
  const LineShape& S = sh.S;
  const int ts = sh.ts, nthr = sh.nthr;
  const size_t lds = sh.lds;
#define UOT_LN(TS, NT, EPT)                                                                                          \
  do {                                                                                                               \
    line_big_lds(k_line_pair<T, TS, NT, EPT, 2>, lds);                                                               \
    hipLaunchKernelGGL((k_line_pair<T, TS, NT, EPT, 2>), dim3(blocks), dim3(NT), lds, s, in, R, 0, S, h * h, side, c, \
                       ep, out, bw);                                                                         \
  } while (0)
  UOT_LINE_TS(UOT_LN)
#undef UOT_LN
}

// planes of n1 x n2 cells, one per block: launch shape and dynamic LDS
template <typename T> struct PlaneShape {
  LineShape S1, S2;
  int ts, nthr;
  size_t lds;
  PlaneShape(int n1, int n2, double c_max, int64_t blocks) {
    const int ts_min = sizeof(T) == 4 ? 8 : 16;
    int t2;
    nthr = line_threads(n1 * n2, blocks);
    // one segment length for both axes: the shorter of the two
    line_shape(n2, n1, nthr, line_ts<T>(c_max), ts_min, S1, ts);
    line_shape(n1, n2, nthr, ts, ts_min, S2, t2);
    if (t2 != ts) {
      ts = t2;
      line_shape(n2, n1, nthr, ts, ts, S1, t2);
    }
    const size_t lb = std::max((size_t)S1.nl * S1.ldl, (size_t)S2.nl * S2.ldl);
    const size_t pp = std::max((size_t)S1.ksn * S1.nl * S1.ldp, (size_t)S2.ksn * S2.nl * S2.ldp);
    lds = sizeof(T) * (lb + 2 * pp);
  }
  bool fits() const { return lds + line_static_lds<T>(nthr) <= kLineLds; }
  // taps that a wave of the block takes one after another in a pass along each axis
  int chain() const {
    auto of = [&](const LineShape& S) {
      const int G = (S.nl * S.nt + 15) / 16, gw = nthr / 64 / S.ksn;
      return (G + gw - 1) / gw * ((S.nseg + S.ksn - 1) / S.ksn) * ts;
    };
    return of(S1) + of(S2);
  }
};

// Whether a plane per block pays.  Thin planes pad their short lines to a
// segment and to a tile, up to 76 elements for a line of a few cells, so the
// LDS is counted in bytes, for the two block counts that one plan is launched
// with (the control step adds a block).  A plane's four passes are a chain in
// one block, which a pass per launch spreads over the chip.  Measured (us an
// iteration, paired / a pass per launch): FP32 chains of up to 128 taps 23.6 /
// 29.0 (8 x 48 x 48) and 26.1 / 26.9 (4 x 64 x 64), of 136 38.7 / 27.4 (4 x 8 x 256),
// of 272 66.7 / 31.2 (16 x 16 x 256).  FP64 (four elements a thread spill, 221
// registers): 1024 cells and chains of up to 64 taps 55.8 / 61.6 (64 x 20 x 48) and
// 41.3 / 48.5 (64 x 32 x 32), beyond either 45.3 / 35.0 (4 x 30 x 40), 79.4 / 58.3
// (64 x 4 x 200), 91.6 / 32.7 (4 x 64 x 64).
template <typename T> static bool plane_pays(int64_t blocks, int64_t n1, int64_t n2, double c_max) {
  constexpr bool f32 = sizeof(T) == 4;
  if (n1 * n2 > (f32 ? kLineMaxCells : 1024)) return false;
  for (int host = 0; host < 2; ++host) {
    const PlaneShape<T> sh((int)n1, (int)n2, c_max, blocks + host);
    if (!sh.fits() || sh.chain() > (f32 ? 128 : 64)) return false;
  }
  return true;
}
bool line_plane_pays(bool f64, int64_t planes, int64_t n1, int64_t n2, double c1_max, double c2_max) {
  const double c = std::max(c1_max, c2_max);
  return f64 ? plane_pays<double>(planes, n1, n2, c) : plane_pays<float>(planes, n1, n2, c);
}

template <typename T>
void launch_plane_pair(const T* in, int64_t F, int n0, int n1, int n2, double h1, double h2, double c1_max,
                       double c2_max, int side, const Ctrl* c, const EpiArgs<T>* ep, T* out, hipStream_t s) {
  const unsigned blocks = (unsigned)(F * n0) + (ep && ep->host_ctl ? 1 : 0);
  const int tot = n1 * n2;
  const PlaneShape<T> sh(n1, n2, std::max(c1_max, c2_max), blocks);
  const LineShape &S1 = sh.S1, &S2 = sh.S2;
  const int ts = sh.ts, nthr = sh.nthr;
  // (FP64: planes of up to 1024 cells, whose chains rule out 32 taps over 1024 threads)
  const size_t lds = sh.lds;
  const EpiArgs<T> none{};
#define UOT_LN(TS, NT, EPT)                                                                                         \
  do {                                                                                                              \
    if constexpr (sizeof(T) == 8 && (NT * EPT > 1024 || (TS > 16 && NT == 1024))) {                                 \
    } else if (ep) {                                                                                                \
      line_big_lds(k_plane_pair<T, TS, NT, EPT, true>, lds);                                                        \
      hipLaunchKernelGGL((k_plane_pair<T, TS, NT, EPT, true>), dim3(blocks), dim3(NT), lds, s, in, n0, S1, S2,      \
                         h1 * h1, h2 * h2, side, c, *ep, out);                                                      \
    } else {                                                                                                        \
      line_big_lds(k_plane_pair<T, TS, NT, EPT, false>, lds);                                                       \
      hipLaunchKernelGGL((k_plane_pair<T, TS, NT, EPT, false>), dim3(blocks), dim3(NT), lds, s, in, n0, S1, S2,     \
                         h1 * h1, h2 * h2, side, c, none, out);                                                     \
    }                                                                                                               \
  } while (0)
  UOT_LINE_TS(UOT_LN)
#undef UOT_LN
}

// Longest line the loop kernel is used for: one compute unit does what the
// chip shares in the launches it replaces, whose latency hardly depends on n.
// Measured (us per iteration, this kernel / the launches): FP32 64 cells 3.4 /
// 11.9, 256 4.3 / 15.5, 512 7.2 / 21.2, 768 17.3 / 22.4, 1024 26.3 / 22.7; FP64
// 64 5.3 / 15.5, 256 9.2 / 23.9, 512 22.2 / 31.2, 768 50.2 / 31.9.
int line_loop_max(bool f64) { return f64 ? 512 : 768; }   // (512 threads, in FP32 up to 1024)

template <typename T>
void launch_line_loop(int n, double h, double c_max, Ctrl* c, const EpiArgs<T>& ex, const EpiArgs<T>& ey, double* hist,
                      int chunk, hipStream_t s) {
  const int tot = n, nthr = line_threads(tot, 1);
  LineShape S;
  int ts;
  line_shape(1, n, nthr, line_ts<T>(c_max), sizeof(T) == 4 ? 8 : 16, S, ts);
  const size_t lds = line_lds_bytes<T>(S);
#define UOT_LN(TS, NT, EPT)                                                                                         \
  do {                                                                                                              \
    if constexpr (NT == 512 || (sizeof(T) == 4 && NT * EPT == 1024 && NT != 256))                                   \
      hipLaunchKernelGGL((k_line_loop<T, TS, NT, EPT>), dim3(1), dim3(NT), lds, s, S, h * h, c, ex, ey, hist, chunk); \
  } while (0)
  UOT_LINE_TS(UOT_LN)
#undef UOT_LN
}

template <typename T>
void launch_transpose(const T* src, T* dst, int64_t F, int64_t Na, int64_t Nb, int log, hipStream_t s) {
  for (int64_t f = 0; f < F; f += 65535) {
    const int64_t nf = std::min<int64_t>(65535, F - f);
    hipLaunchKernelGGL(k_transpose<T>, dim3((unsigned)((Nb + 15) / 16), (unsigned)((Na + 15) / 16), (unsigned)nf),
                       dim3(256), 0, s, src + f * Na * Nb, dst + f * Na * Nb, Na, Nb, log);
  }
}

#define UOT_LINE_INST(T)                                                                                              \
  template void launch_line<T>(const T*, int64_t, int, int64_t, double, double, int, int, const Ctrl*,                \
                               const EpiArgs<T>&, hipStream_t, bool);                                                 \
  template void launch_line_pair<T>(const T*, int64_t, int64_t, int, double, double, int, int, const Ctrl*,           \
                                    const EpiArgs<T>*, T*, hipStream_t);                                              \
  template void launch_line_bary<T>(const T*, int64_t, int64_t, int, double, double, int, const Ctrl*,                \
                                    const EpiArgs<T>&, T*, const BaryW&, hipStream_t);                        \
  template void launch_plane_pair<T>(const T*, int64_t, int, int, int, double, double, double, double, int,           \
                                     const Ctrl*, const EpiArgs<T>*, T*, hipStream_t);                                \
  template void launch_line_loop<T>(int, double, double, Ctrl*, const EpiArgs<T>&, const EpiArgs<T>&, double*, int,    \
                                    hipStream_t);                                                                     \
  template void launch_transpose<T>(const T*, T*, int64_t, int64_t, int64_t, int, hipStream_t);
UOT_LINE_INST(float)
UOT_LINE_INST(double)

}  // namespace uot
