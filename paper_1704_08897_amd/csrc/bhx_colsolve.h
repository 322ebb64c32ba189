// Kernels of the column solve.
#pragma once
#include "bhx_device.h"

namespace bhx {

// ---------------------------------------------------------------------------
// Column solve: t <- (lambda I + T)^-2 t along the last axis of every column
// of t (y in two dimensions, z in three), lambda the column's eigenvalue sum
// of the transformed axes and T the second difference of the axis.  This is
// the whole column part of the preconditioner, exactly: after the transforms
// of the other axes the operator is block diagonal with these tridiagonal
// (periodic: cyclic) blocks, so no transform along the last axis is needed.
//
// T + lambda I has constant coefficients and factors into two first-order
// recursions, (1/rho) (1 - rho S)(1 - rho S^-1) with S the shift and rho < 1
// the root of rho + 1/rho = 2 + lambda; the boundary rule only sets the state
// a recursion enters with.  Periodic and Neumann axes run (1 - rho S)^-2
// downwards, then (1 - rho S^-1)^-2 upwards; the entry states follow from the
// periodic (even) extension in closed form.  Dirichlet axes run the pivots of
// the tridiagonal's LDL^T factorisation, which are ratios of
// W_i = 1 - rho^(2(i+1)), so that each recursion starts from 0.  The one
// column with lambda = 0 (no Dirichlet rule on the transformed axes) is solved
// by running sums, the constant mode removed (Neumann, periodic).
//
// A block stages W neighbouring columns in LDS (t is read and written once, in
// runs of W elements).  A column is then one wave's (COLS = 1) or a sixteenth
// lane row's (COLS = 4): each lane keeps LC consecutive rows in registers, and
// the lanes' segments meet through their recursion states, scanned with the
// vector unit's own lane moves (DPP).  No barrier but around the staging.
//
// Bound: memory and launch latency up to about 1024^2 nodes, HBM beyond (16
// bytes and about 20 operations per node in FP64).  The transforms it replaces
// cost two FFTs per column, four of twice the length where Bluestein runs.  Per
// launch, transforms -> recursions: 1024^2 12.1 -> 10.7 us, 2048^2 32.2 -> 17.9
// (64 MB to load and store), 450^2 19.5 -> 7.3, 1231x877 69.2 -> 12.6 (17 MB), 40
// mixed instances 82.4 -> 13.2, 128^3 along z 21.0 -> 12.9.
// Relative to the spectral form its rounding is smaller in the energy norm
// that conjugate gradients work in (about 1e-11 against 1e-10 at 2048 nodes
// and the smallest lambda).
// ---------------------------------------------------------------------------

// DPP lane moves of a double; lanes without a source read 0.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  union { double d; int i[2]; } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, 0xf, 0xf, true);
  return b.d;
}
constexpr int kRowShl = 0x100, kRowShr = 0x110;      // + lanes, within rows of 16
__device__ __forceinline__ double lane_value(double v, int lane) {
  union { double d; int i[2]; } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_readlane(a.i[0], lane);
  b.i[1] = __builtin_amdgcn_readlane(a.i[1], lane);
  return b.d;
}

// sqrt(x), x > 0, from the hardware estimate of 1 / sqrt(x) by two Newton-
// Raphson steps and a correction of the root.
__device__ __forceinline__ double root(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  const double s = x * r;
  return fma(0.5 * r, fma(-s, s, x), s);
}
// 1 - (1 - d)^n by binary powering of m = 1 - (1 - d)^k: every step adds
// positive terms, so small results keep their relative accuracy.
__device__ __forceinline__ double one_minus_pow(double d, int n) {
  double m = 0.0;
#pragma unroll 1
  for (int b = 12; b >= 0; --b) {
    m = m * (2.0 - m);
    m = fma(((n >> b) & 1) ? d : 0.0, 1.0 - m, m);
  }
  return m;
}
// x^n by binary powering.
__device__ __forceinline__ double int_pow(double x, int n) {
  double r = 1.0;
#pragma unroll 1
  for (; n; n >>= 1) {
    r *= (n & 1) ? x : 1.0;
    x *= x;
  }
  return r;
}

// How a column of n rows lies in its lanes: LC rows per lane, nseg lanes in
// use; the last one misses `m` rows, which count as zeros.  A wave's rows of 16
// lanes are the stages of the scan: `row` (0 if COLS = 4) and place in it.
template <int LC, int COLS>
struct ColCut {
  int nseg, m, last, nl;     // last: row of the last segment; nl: segments in that row
  int li, l16, row;          // this lane: segment, place in its row, row of the column
  int below;                 // existing segments of its row after it
  __device__ __forceinline__ ColCut(int n) {
    const int lane = threadIdx.x & 63;
    nseg = (n + LC - 1) / LC;
    m = nseg * LC - n;
    last = (nseg - 1) >> 4;
    nl = nseg - 16 * last;
    l16 = lane & 15;
    row = COLS == 1 ? lane >> 4 : 0;
    li = 16 * row + l16;
    below = max(min(15, nseg - 1 - 16 * row) - l16, 0);
  }
  // value of lane `s` of the lane's own row
  __device__ __forceinline__ double in_row(double v, int s) const {
    return __shfl(v, ((int)threadIdx.x & 48) + s, 64);
  }
};

// rho^LC and its powers over 1, 2, 4, 8, 16 segments.
struct ColPow {
  double p[5];
  __device__ __forceinline__ ColPow(double pl) {
    p[0] = pl;
#pragma unroll
    for (int k = 1; k < 5; ++k) p[k] = p[k - 1] * p[k - 1];
  }
  // over s segments, s <= 15
  __device__ __forceinline__ double over(int s) const {
    double r = 1.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) r *= ((s >> k) & 1) ? p[k] : 1.0;
    return r;
  }
};

// Inclusive scan of the states within rows of 16 lanes, from the states of
// each segment alone.  TWO: second-order states (else s1 alone).
template <int LC, bool UP, bool TWO>
__device__ __forceinline__ void row_scan(const ColPow& P, double& s1, double& s2) {
  double len = LC;
  auto step = [&](double x1, double x2, double p) {
    if (TWO) s2 = fma(p, fma(len, x1, x2), s2);
    s1 = fma(p, x1, s1);
    len += len;
  };
  step(UP ? dpp<kRowShl + 1>(s1) : dpp<kRowShr + 1>(s1),
       !TWO ? 0.0 : UP ? dpp<kRowShl + 1>(s2) : dpp<kRowShr + 1>(s2), P.p[0]);
  step(UP ? dpp<kRowShl + 2>(s1) : dpp<kRowShr + 2>(s1),
       !TWO ? 0.0 : UP ? dpp<kRowShl + 2>(s2) : dpp<kRowShr + 2>(s2), P.p[1]);
  step(UP ? dpp<kRowShl + 4>(s1) : dpp<kRowShr + 4>(s1),
       !TWO ? 0.0 : UP ? dpp<kRowShl + 4>(s2) : dpp<kRowShr + 4>(s2), P.p[2]);
  step(UP ? dpp<kRowShl + 8>(s1) : dpp<kRowShr + 8>(s1),
       !TWO ? 0.0 : UP ? dpp<kRowShl + 8>(s2) : dpp<kRowShr + 8>(s2), P.p[3]);
}

// The recursions over a lane's segment: downwards (l up) or upwards from the
// states (s1, s2); x <- s2 if STORE.
template <int LC, bool UP, bool STORE>
__device__ __forceinline__ void col_sweep(double (&v)[LC], double rho, double& s1, double& s2) {
#pragma unroll
  for (int k = 0; k < LC; ++k) {
    const int l = UP ? LC - 1 - k : k;
    s1 = fma(rho, s1, v[l]);
    s2 = fma(rho, s2, s1);
    if (STORE) v[l] = s2;
  }
}
template <int LC>
__device__ __forceinline__ void col_clear_tail(double (&v)[LC], int len) {
  if (len >= LC) return;
#pragma unroll
  for (int l = 0; l < LC; ++l) v[l] = l < len ? v[l] : 0.0;
}

// Aggregates of the column's rows of 16 lanes, per lane of the column (rows
// past the last are unused).
template <int LC, int COLS, bool UP, bool TWO>
struct RowAgg {
  static constexpr int N = COLS == 1 ? 4 : 1;
  double a1[N], a2[N];
  __device__ __forceinline__ RowAgg(const ColCut<LC, COLS>& K, double s1, double s2) {
    if constexpr (COLS == 1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int at = 16 * r + (UP ? 0 : r == K.last ? K.nl - 1 : 15);
        a1[r] = lane_value(s1, at);
        a2[r] = TWO ? lane_value(s2, at) : 0.0;
      }
    } else {
      a1[0] = K.in_row(s1, UP ? 0 : K.nl - 1);
      a2[0] = TWO ? K.in_row(s2, UP ? 0 : K.nl - 1) : 0.0;
    }
  }
  // Takes the states (x1, x2) through the column; `pick` receives the states
  // that enter this lane's row.
  __device__ __forceinline__ void through(const ColCut<LC, COLS>& K, const ColPow& P, double plast,
                                          double& x1, double& x2, double& e1, double& e2) const {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const int r = UP ? N - 1 - k : k;
      if (r <= K.last) {
        if (r == K.row) {
          e1 = x1;
          e2 = x2;
        }
        const double p = r == K.last ? plast : P.p[4];
        const double len = r == K.last ? LC * K.nl : LC * 16;
        if (TWO) x2 = fma(p, fma(len, x1, x2), a2[r]);
        x1 = fma(p, x1, a1[r]);
      }
    }
  }
};

// Neumann and periodic axes.
template <int LC, int COLS>
__device__ __forceinline__ void col_even(double (&v)[LC], int n, bool neumann,
                                         const ColCut<LC, COLS>& K, int len, double pa) {
  const double rho = recip(1.0 + pa);
  double pl = rho;
#pragma unroll
  for (int l = 1; l < LC; l <<= 1) pl *= pl;
  const ColPow P(pl);
  const double plast = K.nl == 16 ? P.p[4] : P.over(K.nl);
  // rho^-m, rho^n and, with q = rho^period, 1 / (1 - q), 1 / (1 - rho) and
  // 1 / (1 - rho^2) from one reciprocal
  const double m = K.m, im = int_pow(1.0 + pa, K.m);
  const double pn = int_pow(P.p[4], K.last) * plast * im;
  const double q = neumann ? pn * pn : pn, per = neumann ? 2.0 * n : (double)n;
  const double iall = recip((1.0 - q) * pa * (1.0 + rho));
  const double iq = iall * pa * (1.0 + rho);
  const double id = (1.0 + pa) * iall * (1.0 - q) * (1.0 + rho);
  const double id2 = id * iall * (1.0 - q) * pa;
  const double pe = P.over(K.l16), pb = P.over(K.below);
  const double le = LC * K.l16, lb = LC * K.below;
#pragma unroll
  for (int l = 0; l < LC; ++l) v[l] *= rho * rho;
  // 1. aggregates from zero states: downwards and, for the even extension,
  //    upwards; the states entering the column from its extension
  double c1 = 0.0, c2 = 0.0;
  col_sweep<LC, false, false>(v, rho, c1, c2);
  row_scan<LC, false, true>(P, c1, c2);
  const RowAgg<LC, COLS, false, true> C(K, c1, c2);
  double x1 = 0.0, x2 = 0.0, e1 = 0.0, e2 = 0.0;
  C.through(K, P, plast, x1, x2, e1, e2);
  x1 *= im;                                  // before the missing rows
  x2 = fma(x2, im, -m * x1);
  if (neumann) {
    double b1 = 0.0, b2 = 0.0, y1 = 0.0, y2 = 0.0;
    col_sweep<LC, true, false>(v, rho, b1, b2);
    row_scan<LC, true, true>(P, b1, b2);
    const RowAgg<LC, COLS, true, true> U(K, b1, b2);
    U.through(K, P, plast, y1, y2, e1, e2);
    x2 = fma(pn, fma((double)n, x1, x2), y2);
    x1 = fma(pn, x1, y1);
  }
  double a1 = x1 * iq;
  double a2 = fma(per * q * iq, a1, x2 * iq);
  C.through(K, P, plast, a1, a2, e1, e2);
  // 2. downwards with the true states
  c1 = fma(pe, e1, dpp<kRowShr + 1>(c1));
  c2 = fma(pe, fma(le, e1, e2), dpp<kRowShr + 1>(c2));
  col_sweep<LC, false, true>(v, rho, c1, c2);
  col_clear_tail<LC>(v, len);
  // 3. aggregates upwards; the states entering from beyond the last row
  double b1 = 0.0, b2 = 0.0;
  col_sweep<LC, true, false>(v, rho, b1, b2);
  row_scan<LC, true, true>(P, b1, b2);
  const RowAgg<LC, COLS, true, true> U(K, b1, b2);
  double d1, d2;
  if (neumann) {
    // the solution and its half-way state are even about the boundary
    a1 *= im;
    a2 = fma(a2, im, -m * a1);
    d1 = fma(rho, a2, a1 * id) * id2;
    d2 = fma(rho, d1, a2) * id;
  } else {
    x1 = x2 = 0.0;
    U.through(K, P, plast, x1, x2, e1, e2);
    d1 = x1 * iq;
    d2 = fma(per * q * iq, d1, x2 * iq);
  }
  d1 *= im;                                  // past the missing rows
  d2 = fma(d2, im, -m * d1);
  U.through(K, P, plast, d1, d2, e1, e2);
  // 4. upwards
  b1 = fma(pb, e1, dpp<kRowShl + 1>(b1));
  b2 = fma(pb, fma(lb, e1, e2), dpp<kRowShl + 1>(b2));
  col_sweep<LC, true, true>(v, rho, b1, b2);
}

// Dirichlet axes: with W_i = 1 - rho^(2(i+1)) the LDL^T sweeps of T + lambda
// are C_i = W_i f_i + rho C_(i-1) downwards and y_i = rho (G_i + y_(i+1)),
// G_i = C_i / (W_i W_(i+1)), upwards, from zero states; the solution is
// W_i y_i.  Two applications.
template <int LC, int COLS>
__device__ __forceinline__ void col_odd(double (&v)[LC], const ColCut<LC, COLS>& K, int len,
                                        double pa) {
  const double rho = recip(1.0 + pa);
  const double r2 = rho * rho, d2 = pa * rho * (1.0 + rho);   // W_(i+1) = r2 W_i + d2
  const double w0 = one_minus_pow(d2, K.li * LC + 1);         // W of the segment's first row
  double pl = rho;
#pragma unroll
  for (int l = 1; l < LC; l <<= 1) pl *= pl;
  const ColPow P(pl);
  const double plast = K.nl == 16 ? P.p[4] : P.over(K.nl);
  const double pe = P.over(K.l16), pb = P.over(K.below);
#pragma unroll 1
  for (int rep = 0; rep < 2; ++rep) {
    // (the W_i are formed anew in each sweep: kept, they would take as many
    // registers as the rows)
    double wi = w0, cs = 0.0, ys = 0.0, none = 0.0, x1 = 0.0, e1 = 0.0;
    asm volatile("" : "+v"(wi));
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      v[l] *= wi;
      cs = fma(rho, cs, v[l]);
      wi = fma(r2, wi, d2);
    }
    row_scan<LC, false, false>(P, cs, none);
    const RowAgg<LC, COLS, false, false> C(K, cs, none);
    C.through(K, P, plast, x1, none, e1, none);
    cs = fma(pe, e1, dpp<kRowShr + 1>(cs));
    wi = w0;
    asm volatile("" : "+v"(wi));
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      cs = fma(rho, cs, v[l]);
      const double wn = fma(r2, wi, d2);
      v[l] = cs * recip(wi * wn);
      wi = wn;
    }
    col_clear_tail<LC>(v, len);
#pragma unroll
    for (int l = LC - 1; l >= 0; --l) ys = rho * (v[l] + ys);
    row_scan<LC, true, false>(P, ys, none);
    const RowAgg<LC, COLS, true, false> U(K, ys, none);
    x1 = 0.0;                                // nothing enters the last segment
    U.through(K, P, plast, x1, none, e1, none);
    ys = fma(pb, e1, dpp<kRowShl + 1>(ys));
#pragma unroll
    for (int l = LC - 1; l >= 0; --l) {
      ys = rho * (v[l] + ys);
      v[l] = ys;
    }
    wi = w0;
    asm volatile("" : "+v"(wi));
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      v[l] *= wi;
      wi = fma(r2, wi, d2);
    }
    col_clear_tail<LC>(v, len);
  }
}

// Running sum of v over the lanes of a column, without the lane's own value,
// and the column's total.
template <int COLS>
__device__ __forceinline__ double col_running_sum(double v, double& total) {
  const int lane = threadIdx.x & 63;
  double x = v;
  x += dpp<kRowShr + 1>(x);
  x += dpp<kRowShr + 2>(x);
  x += dpp<kRowShr + 4>(x);
  x += dpp<kRowShr + 8>(x);
  double s = dpp<kRowShr + 1>(x);
  if constexpr (COLS == 1) {
    const double r0 = lane_value(x, 15), r1 = lane_value(x, 31), r2 = lane_value(x, 47),
                 r3 = lane_value(x, 63);
    s += lane < 16 ? 0.0 : lane < 32 ? r0 : lane < 48 ? r0 + r1 : r0 + r1 + r2;
    total = r0 + r1 + (r2 + r3);
  } else {
    total = __shfl(x, (lane & 48) + 15, 64);
  }
  return s;
}

// The column with lambda = 0: T^+ T^+ (Neumann, periodic: the constant mode
// removed) or T^-2 (Dirichlet).  T u = f has fluxes g_i = u_i - u_(i+1): g is
// the running sum of f (less its mean) plus a constant, u minus the running
// sum of g plus a constant.
template <int LC, int COLS>
__device__ __forceinline__ void col_zero(double (&v)[LC], int n, int bc, int j0, int len) {
  const double inv = recip(bc == kDirichlet ? n + 1.0 : (double)n);
  double total;
#pragma unroll 1
  for (int rep = 0; rep < 2; ++rep) {
    double a = 0.0, j = j0;
    asm volatile("" : "+v"(j));          // (row numbers counted, not kept)
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      a += v[l];
      v[l] = a;
    }
    const double x = col_running_sum<COLS>(a, total);
    const double mean = bc == kDirichlet ? 0.0 : total * inv;
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      j += 1.0;
      v[l] = fma(-mean, j, x + v[l]);
    }
    col_clear_tail<LC>(v, len);
    a = 0.0;
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      const double g = v[l];
      v[l] = a;
      a += g;
    }
    const double y = col_running_sum<COLS>(a, total);
    const double c = bc == kNeumann ? 0.0 : total * inv;
    j = j0;
    asm volatile("" : "+v"(j));
#pragma unroll
    for (int l = 0; l < LC; ++l) {
      j += 1.0;
      v[l] = fma(c, j, -(y + v[l]));
    }
    col_clear_tail<LC>(v, len);
  }
  if (bc != kDirichlet) {
    double a = 0.0;
#pragma unroll
    for (int l = 0; l < LC; ++l) a += v[l];
    col_running_sum<COLS>(a, total);
    const double mean = total * inv;
#pragma unroll
    for (int l = 0; l < LC; ++l) v[l] -= mean;
  }
}

// One item: COLS columns a wave, 8 COLS columns from column c * 8 COLS.
// Staged as tile[column * cs + row + row / LC], cs = col_stride.
template <typename R, int LC, int COLS, bool ODD, bool d3>
__device__ __forceinline__ void col_item(R* tile, const Batch& B, const Inst& I, int c, bool zero) {
  constexpr int W = kColWaves * COLS;                // columns of the item
  constexpr int NR = kColThreads / W;                // rows staged at a time
  constexpr int NL = LC * (COLS == 1 ? 64 : 16) / NR;   // of them, at most
  // slots between rows NR apart (k of them); a row's own pad slots
  constexpr auto slots = [](int k) { return k * NR + (LC == 1 ? 0 : k * NR / LC); };
  const int n = d3 ? I.nz : I.ny, bc = d3 ? I.bcz : I.bcy;
  const int ncol = d3 ? I.nx * I.ny : I.nx;
  const int cs = col_stride(n, LC, W);
  const int e0 = c * W;
  // (opaque, so that nothing derived from it is kept from item to item)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  // 1. stage the columns; a thread's rows are NR apart
  const int gc = tid % W, gr = tid / W;
  BHX_GLOBAL R* tg =
      (BHX_GLOBAL R*)I.t + (size_t)min(gr, n - 1) * ncol + min(e0 + gc, ncol - 1);
  const size_t step = (size_t)NR * ncol;
  R raw[NL];
  {
    BHX_GLOBAL const R* a = tg;
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      if (k * NR < n) raw[k] = *a;
      a += gr + (k + 1) * NR < n ? step : 0;         // rows past the end: the last one again
    }
  }
  // the eigenvalue of the lane's column
  const int lane = tid & 63, wv = tid >> 6;
  const int cl = wv * COLS + (COLS == 1 ? 0 : lane >> 4);
  const int e = e0 + cl, ec = min(e, ncol - 1);
  BHX_GLOBAL const double* rt = (BHX_GLOBAL const double*)B.rtab[0];
  double lam = rt[I.lamx + (d3 ? ec % I.nx : ec)];
  if (d3) lam += rt[I.lamy + ec / I.nx];
  if (I.ctl->done) return;                           // (nothing changes it during this pass)
  const bool special = zero && e == 0;
  if (special) lam = 1.0;
  // rho = 1 / (1 + pa); 1 - rho = pa rho keeps its relative accuracy for small
  // lambda
  const double pa = 0.5 * (lam + root(lam * (lam + 4.0)));
  R* tl = tile + gc * cs + gr + (LC == 1 ? 0 : gr / LC);
  __syncthreads();                                   // the previous item's stores have read it
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    if ((k + 1) * NR <= n) tl[slots(k)] = raw[k];
    else if (gr + k * NR < n) tl[slots(k)] = raw[k];
  }
  __syncthreads();
  // 2. the lane's segment
  const ColCut<LC, COLS> K(n);
  const int j0 = K.li * LC, len = min(max(n - j0, 0), LC);
  R* ts = tile + cl * cs + (LC == 1 ? j0 : j0 + K.li);
  auto fetch = [&](double (&v)[LC]) {
#pragma unroll
    for (int l = 0; l < LC; ++l) v[l] = 0.0;
    if (len > 0) {
#pragma unroll
      for (int l = 0; l < LC; ++l) v[l] = (double)ts[l];
    }
    col_clear_tail<LC>(v, len);
  };
  auto put = [&](const double (&v)[LC], bool on) {
    if (on && len > 0) {
#pragma unroll
      for (int l = 0; l < LC; ++l) ts[l] = (R)v[l];
    }
  };
  const bool wave0 = zero && c == 0 && wv == 0;      // holds the column lambda = 0
  if (!(COLS == 1 && wave0)) {
    double v[LC];
    fetch(v);
    if constexpr (ODD) col_odd<LC, COLS>(v, K, len, pa);
    else col_even<LC, COLS>(v, n, bc == kNeumann, K, len, pa);
    put(v, !special);
  }
  if (wave0) {
    double v[LC];
    fetch(v);
    col_zero<LC, COLS>(v, n, bc, j0, len);
    put(v, special);
  }
  __syncthreads();
  // 3. back to t (addresses formed anew: kept, the loads' would take as many
  // registers as the rows)
  if (e0 + gc >= ncol) return;
  asm volatile("" : "+v"(tg));
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    if ((k + 1) * NR <= n) *tg = tl[slots(k)];
    else if (gr + k * NR < n) *tg = tl[slots(k)];
    tg += step;
  }
}

// PASS: the work list, kPassC (two dimensions) or kPassZ (three).  LONG: the
// class of the longest column (col_class); the longer ones take twice the
// registers, which would spill at the short ones' occupancy (and a kernel with
// spills pays for its scratch memory at every launch).  Class 3 has a launch of
// its own after the others' (launch_colsolve_odd64), which leave its columns
// alone and count the iteration for them.
template <typename R, int PASS, int LONG>
__global__ void __launch_bounds__(kColThreads, LONG ? 2 : 4)
    k_colsolve(const Batch* __restrict__ Bp, int count_iter) {
  constexpr bool d3 = PASS == kPassZ;
  const Batch B = *(BHX_CONST const Batch*)Bp;   // scalar loads, kept in registers
  extern __shared__ __align__(16) unsigned char smem[];
  debug_fill_lds(smem);
  R* tile = (R*)smem;
  for (int itm = logical_block(); itm < B.n_items[PASS]; itm += gridDim.x) {
    const int code = item_code(B, PASS, itm);
    const Inst I = B.inst[code >> kItemShift];
    const int c = code & kItemMask;
    BHX_GLOBAL Ctl* ctl = I.ctl;
    const bool zero = I.bcx != kDirichlet && (!d3 || I.bcy != kDirichlet);
    const int lc = col_rows(d3 ? I.nz : I.ny, d3 ? I.Gz : I.Gc);
    const bool wide = (d3 ? I.Gz : I.Gc) == 4 * kColWaves;
    const bool odd = (d3 ? I.bcz : I.bcy) == kDirichlet;
#define BHX_COL(LC)                                                        \
  case LC:                                                                 \
    if (wide) {                                                            \
      if (odd) col_item<R, LC, 4, true, d3>(tile, B, I, c, zero);          \
      else col_item<R, LC, 4, false, d3>(tile, B, I, c, zero);             \
    } else {                                                               \
      if (odd) col_item<R, LC, 1, true, d3>(tile, B, I, c, zero);          \
      else col_item<R, LC, 1, false, d3>(tile, B, I, c, zero);             \
    }                                                                      \
    break;
    if constexpr (LONG == 3) {
      if (odd && lc > 32) col_item<R, 64, 1, true, d3>(tile, B, I, c, zero);
    } else {
      switch (lc) {
        BHX_COL(1)
        BHX_COL(2)
        BHX_COL(4)
        BHX_COL(8)
        default:
          if constexpr (LONG > 0) {
            switch (lc) { BHX_COL(16) BHX_COL(32) }
          }
          if constexpr (LONG > 1)
            if (lc > 32 && !odd) col_item<R, 64, 1, false, d3>(tile, B, I, c, zero);
          break;
      }
      if (count_iter && c == 0 && threadIdx.x == 0 && !ctl->done) ctl->iter = ctl->iter + 1;
    }
#undef BHX_COL
  }
}

}  // namespace bhx
