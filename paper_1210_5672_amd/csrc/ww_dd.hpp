// Double-double (about 32 significant digits) DtN evaluation on gfx950: the GPU part
// of the quadruple-precision workflow of Wilkening & Yu (Sec. 2.2 on quadruple
// precision, Sec. 3.3): the matrices of eq. (fred) and (G) assembled in double-double,
// residuals of the solve formed in double-double by matrix products, corrections from
// the FP64 factors of the leading part (iterative refinement), and the spectral steps
// (gamma = mu', H gamma) by double-double FFTs.
//
// A double-double value is the unevaluated sum hi + lo of two doubles with
// |lo| <= ulp(hi)/2.  Arithmetic: Knuth's two-sum, the exact product by fma, and the
// accurate addition and multiplication of Hida, Li & Bailey ("Algorithms for
// quad-double precision floating point arithmetic", 2001), relative error about 2^-104;
// division by three quotient digits.  Arrays are stored as separate hi and lo planes.
#pragma once
#include "ww_kernels.hpp"

// No contraction of a product into a later sum inside the primitives: the error-free
// transformations need every product and sum rounded on its own (a product fused into
// the sum of a two-sum loses the low part).
#define CONTRACT_OFF _Pragma("clang fp contract(off)")

struct alignas(16) dd {   // (one 16-byte LDS access)
  double hi, lo;
};
struct cdd {
  dd re, im;
};

__host__ __device__ inline dd dd_of(double a) { return dd{a, 0.0}; }
__host__ __device__ inline dd dd_two_sum(double a, double b) {
  CONTRACT_OFF
  const double s = a + b;
  const double bb = s - a;
  return dd{s, (a - (s - bb)) + (b - bb)};
}
__host__ __device__ inline dd dd_quick(double a, double b) {   // |a| >= |b|
  CONTRACT_OFF
  const double s = a + b;
  return dd{s, b - (s - a)};
}
__host__ __device__ inline dd dd_two_prod(double a, double b) {
  CONTRACT_OFF
  const double p = a * b;
  return dd{p, fma(a, b, -p)};
}
__host__ __device__ inline dd dd_neg(dd a) { return dd{-a.hi, -a.lo}; }
__host__ __device__ inline dd dd_add(dd a, dd b) {
  CONTRACT_OFF
  dd s = dd_two_sum(a.hi, b.hi);
  const dd t = dd_two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = dd_quick(s.hi, s.lo);
  s.lo += t.lo;
  return dd_quick(s.hi, s.lo);
}
__host__ __device__ inline dd dd_sub(dd a, dd b) { return dd_add(a, dd_neg(b)); }
__host__ __device__ inline dd dd_add_d(dd a, double b) {
  CONTRACT_OFF
  dd s = dd_two_sum(a.hi, b);
  s.lo += a.lo;
  return dd_quick(s.hi, s.lo);
}
__host__ __device__ inline dd dd_mul(dd a, dd b) {
  CONTRACT_OFF
  dd p = dd_two_prod(a.hi, b.hi);
  p.lo += a.hi * b.lo + a.lo * b.hi;
  return dd_quick(p.hi, p.lo);
}
__host__ __device__ inline dd dd_mul_d(dd a, double b) {
  CONTRACT_OFF
  dd p = dd_two_prod(a.hi, b);
  p.lo += a.lo * b;
  return dd_quick(p.hi, p.lo);
}
__host__ __device__ inline dd dd_div(dd a, dd b) {
  CONTRACT_OFF
  const double q1 = a.hi / b.hi;
  dd r = dd_sub(a, dd_mul_d(b, q1));
  const double q2 = r.hi / b.hi;
  r = dd_sub(r, dd_mul_d(b, q2));
  const double q3 = r.hi / b.hi;
  return dd_add_d(dd_quick(q1, q2), q3);
}
__host__ __device__ inline dd dd_div_d(dd a, double b) { return dd_div(a, dd_of(b)); }
__host__ __device__ inline dd dd_sqrt(dd a) {   // one Newton step from the double root
  CONTRACT_OFF
  if (!(a.hi > 0.0)) return dd_of(0.0);
  const double x = sqrt(a.hi);
  const dd r = dd_sub(a, dd_two_prod(x, x));
  return dd_add_d(dd_of(x), r.hi / (2.0 * x));
}
__host__ __device__ inline cdd cdd_add(cdd a, cdd b) { return cdd{dd_add(a.re, b.re), dd_add(a.im, b.im)}; }
__host__ __device__ inline cdd cdd_sub(cdd a, cdd b) { return cdd{dd_sub(a.re, b.re), dd_sub(a.im, b.im)}; }
__host__ __device__ inline cdd cdd_mul(cdd a, cdd b) {
  return cdd{dd_sub(dd_mul(a.re, b.re), dd_mul(a.im, b.im)), dd_add(dd_mul(a.re, b.im), dd_mul(a.im, b.re))};
}

// pi and ln 2 as double-doubles (the standard hi/lo splits)
#define DD_PI_HI 3.141592653589793116e+00
#define DD_PI_LO 1.224646799147353207e-16
#define DD_LN2_HI 6.931471805599452862e-01
#define DD_LN2_LO 2.319046813846299558e-17

// 1/n for n < 28 as double-doubles: hi the quotient, lo its remainder (1 - hi n) / n, formed
// exactly from the upper 26 and the lower 27 bits of hi
struct DdInv {
  double hi[28], lo[28];
  constexpr DdInv() : hi{}, lo{} {
    for (int n = 1; n < 28; ++n) {
      const double q = 1.0 / n, c = q * 134217729.0, h = c - (c - q), l = q - h;
      hi[n] = q;
      lo[n] = ((1.0 - h * n) - l * n) / n;
    }
  }
};
__device__ constexpr DdInv dd_inv{};

// exp(a) and exp(-a) in double-double: a = k ln2 + r, |r| <= ln2/2, the even and the odd part
// of exp(r)'s Taylor series to the term r^27/27! (below 1e-37 for |r| <= 0.35), their sum and
// difference times 2^k and 2^-k.  No squarings: they would multiply the rounding of the
// series; no divisions: 27 of them took half of k_dd_prep.
__device__ inline void dd_exp_pm(dd a, dd* p, dd* m) {
  const double k = rint(a.hi / DD_LN2_HI);
  const dd ln2 = dd{DD_LN2_HI, DD_LN2_LO};
  const dd r = dd_sub(a, dd_mul_d(ln2, k));
  dd term = r, odd = r, even = dd_of(0.0);   // even: without the leading 1, which is added last
#pragma unroll 1
  for (int n = 2; n < 28; n += 2) {
    term = dd_mul(dd_mul(term, r), dd{dd_inv.hi[n], dd_inv.lo[n]});
    even = dd_add(even, term);
    term = dd_mul(dd_mul(term, r), dd{dd_inv.hi[n + 1], dd_inv.lo[n + 1]});
    odd = dd_add(odd, term);
  }
  const int ki = (int)k;
  const dd u = dd_add(dd_of(1.0), dd_add(even, odd)), v = dd_add(dd_of(1.0), dd_sub(even, odd));
  *p = dd{ldexp(u.hi, ki), ldexp(u.lo, ki)};
  *m = dd{ldexp(v.hi, -ki), ldexp(v.lo, -ki)};
}
__device__ inline dd dd_exp(dd a) {
  dd p, m;
  dd_exp_pm(a, &p, &m);
  return p;
}

// cot((x + i y)/2) from cos x, sin x, cosh y, sinh y by the two-branch formula of
// Sec. 2.2 (as the FP64 assembly), in double-double
__device__ inline void dd_cot_half(dd cx, dd sx, dd chy, dd shy, dd& re, dd& im) {
  if (cx.hi >= 0.0) {
    const dd num = dd_add(cx, chy);
    const dd den = dd_add(dd_mul(sx, sx), dd_mul(shy, shy));
    re = dd_div(dd_mul(num, sx), den);
    im = dd_neg(dd_div(dd_mul(num, shy), den));
  } else {
    const dd den = dd_sub(chy, cx);
    re = dd_div(sx, den);
    im = dd_neg(dd_div(shy, den));
  }
}

// -------------------------------------------------------------------------------------
// Radix-2 Stockham FFTs of N = 2^lg complex double-doubles in LDS, NB of them side by side by
// one workgroup; a = data, b = scratch, tw[j] = exp(-2 pi i j / N) for j < N/2.  dir -1
// forward, +1 inverse (with the 1/N).  a and b are exchanged as needed: the results are in a.
// Starts and ends with a barrier.
//
// Bound by the FP64 units of the one CU (156 operations a butterfly: 2.4 us of a transform at
// N = 512) and each stage's chain of dependent operations: transforms that do not depend on each
// other run together, indexing is shifts and masks, real and imaginary parts lie in planes
// of their own (16-byte steps from lane to lane, no bank conflicts).  Two threads per butterfly
// (one part each) took 1640 cycles a stage for their selects against 1500.  Measured at N = 512: 5.7 us a
// transform, 8.7 us two (one at a time, divisions for the indices, a scaling pass: 11 us each).
// -------------------------------------------------------------------------------------
#define DDF_NT 1024
struct CddBuf {
  dd *re, *im;
  __device__ cdd get(int t) const { return cdd{re[t], im[t]}; }
  __device__ void put(int t, cdd v) const {
    re[t] = v.re;
    im[t] = v.im;
  }
};
// buffer q of N values in the dynamic LDS (dd_lds_bytes: four and the twiddles' half)
__device__ inline CddBuf dd_buf(dd* lds, int q, int N) { return CddBuf{lds + (size_t)2 * q * N, lds + (size_t)(2 * q + 1) * N}; }
__device__ inline CddBuf dd_twiddles(dd* lds, const cdd* __restrict__ twg, int N) {
  const CddBuf tw{lds + (size_t)8 * N, lds + (size_t)8 * N + N / 2};
  for (int t = threadIdx.x; t < N / 2; t += blockDim.x) tw.put(t, twg[t]);
  return tw;
}
template <int NB>
__device__ inline void dd_fft(CddBuf (&a)[NB], CddBuf (&b)[NB], CddBuf tw, int N, int dir) {
  __syncthreads();
  const int lg = __builtin_ctz(N), half = N >> 1;
  const double sc = dir > 0 ? 1.0 / (double)N : 1.0;   // exact: N is a power of two
#pragma unroll 1
  for (int s = 0; s < lg; ++s) {
    const int Ns = 1 << s;
    for (int it = threadIdx.x; it < NB * half; it += blockDim.x) {
      const bool q = NB > 1 && it >= half;
      const int j = it & (half - 1), jm = j & (Ns - 1), o = 2 * j - jm;
      const CddBuf A = a[q ? NB - 1 : 0], B = b[q ? NB - 1 : 0];
      const cdd u = A.get(j);
      cdd v = A.get(j + half);
      if (s > 0) {
        cdd w = tw.get(jm << (lg - 1 - s));
        if (dir > 0) w.im = dd_neg(w.im);
        v = cdd_mul(v, w);
      }
      cdd x = cdd_add(u, v), y = cdd_sub(u, v);
      if (s + 1 == lg && dir > 0) {
        x = cdd{dd{x.re.hi * sc, x.re.lo * sc}, dd{x.im.hi * sc, x.im.lo * sc}};
        y = cdd{dd{y.re.hi * sc, y.re.lo * sc}, dd{y.im.hi * sc, y.im.lo * sc}};
      }
      B.put(o, x);
      B.put(o + Ns, y);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const CddBuf t = a[q];
      a[q] = b[q];
      b[q] = t;
    }
  }
}
__device__ inline void dd_fft1(CddBuf& a, CddBuf& b, CddBuf tw, int N, int dir) {
  CddBuf x[1] = {a}, y[1] = {b};
  dd_fft<1>(x, y, tw, N, dir);
  a = x[0];
  b = y[0];
}

// i k (with the Nyquist mode set to zero) times X
__device__ inline cdd dd_ik(cdd X, int k, int N) {
  if (2 * k == N || 2 * k == -N) return cdd{dd_of(0.0), dd_of(0.0)};
  const double kk = (double)k;
  return cdd{dd_neg(dd_mul_d(X.im, kk)), dd_mul_d(X.re, kk)};
}

// -------------------------------------------------------------------------------------
// Per-point quantities of a surface (one workgroup): eta' and eta'' (spectral, d/dx
// with the Nyquist mode set to zero, eta'' = d(eta')), exp(s) and exp(-s) of the
// surface height s (h + eta at finite depth, eta otherwise); domain (optional, finite
// depth): status bit 16 where s <= 0.  pt_hi / pt_lo: 4 planes
// of nmax values each: eta', eta'', exp(s), exp(-s).  Measured at N = 512: 21.7 us (62).
// -------------------------------------------------------------------------------------
__global__ __launch_bounds__(DDF_NT) void k_dd_prep(const double* __restrict__ eh, const double* __restrict__ el,
                                                    double hsurf, const cdd* __restrict__ twg, int N, int nmax,
                                                    double* __restrict__ pt_hi, double* __restrict__ pt_lo,
                                                    int* __restrict__ domain) {
  extern __shared__ dd ldsd[];
  CddBuf Z = dd_buf(ldsd, 0, N), W = dd_buf(ldsd, 1, N);
  const CddBuf tw = dd_twiddles(ldsd, twg, N);
  for (int t = threadIdx.x; t < N; t += blockDim.x) Z.put(t, cdd{dd{eh[t], el ? el[t] : 0.0}, dd_of(0.0)});
  dd_fft1(Z, W, tw, N, -1);
  CddBuf D[2] = {W, dd_buf(ldsd, 2, N)}, X[2] = {Z, dd_buf(ldsd, 3, N)};   // eta', eta''
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    const int k = t <= N / 2 ? t : t - N;
    const cdd d1 = dd_ik(Z.get(t), k, N);
    D[0].put(t, d1);
    D[1].put(t, dd_ik(d1, k, N));
  }
  dd_fft<2>(D, X, tw, N, +1);
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    const dd d1 = D[0].re[t], d2 = D[1].re[t];
    pt_hi[t] = d1.hi;
    pt_lo[t] = d1.lo;
    pt_hi[nmax + t] = d2.hi;
    pt_lo[nmax + t] = d2.lo;
    const dd sh = dd_add_d(dd{eh[t], el ? el[t] : 0.0}, hsurf);
    if (domain && !(sh.hi > 0.0)) atomicOr(domain, 16);   // finite depth: h + eta > 0
    dd ep, em;
    dd_exp_pm(sh, &ep, &em);
    pt_hi[2 * nmax + t] = ep.hi;
    pt_lo[2 * nmax + t] = ep.lo;
    pt_hi[3 * nmax + t] = em.hi;
    pt_lo[3 * nmax + t] = em.lo;
  }
}

// -------------------------------------------------------------------------------------
// Assembly in double-double (eq. (K1K2), the same formulas as k_assemble): A = I/2 +
// K/N and Gm = G/N, column-major Np x Np, hi and lo planes; Af receives the leading
// part of A, row-major, for the FP64 elimination.  cos, sin (of 2 pi d/N) and cot(pi d/N)/2 come
// from double-double circulant tables (d = (i - j) mod N).  N is a power of two, so the
// scaling by 1/N is exact.  One strip of 64 rows x 16 columns per workgroup.
// -------------------------------------------------------------------------------------
__global__ __launch_bounds__(WW_NT) void k_dd_assemble(const double* __restrict__ pt_hi,
                                                       const double* __restrict__ pt_lo, int nmax,
                                                       const double* __restrict__ tab_hi,
                                                       const double* __restrict__ tab_lo, int N, int Np, int finite,
                                                       double* __restrict__ A_hi, double* __restrict__ A_lo,
                                                       double* __restrict__ G_hi, double* __restrict__ G_lo,
                                                       double* __restrict__ Af) {
  constexpr int CW = 16;
  __shared__ double rt[WW_TB][CW + 1];   // the strip of A for the row-major copy
  const int i0 = blockIdx.x * WW_TB, j0 = blockIdx.y * CW;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int i = i0 + tx;
  const double sc = 1.0 / (double)N;
  const bool rin = i < N;
  const int ic = rin ? i : 0;
  const dd exi = dd{pt_hi[ic], pt_lo[ic]}, exxi = dd{pt_hi[nmax + ic], pt_lo[nmax + ic]};
  const dd epi = dd{pt_hi[2 * nmax + ic], pt_lo[2 * nmax + ic]};
  const dd emi = dd{pt_hi[3 * nmax + ic], pt_lo[3 * nmax + ic]};
  for (int jj = ty; jj < CW; jj += 4) {
    const int j = j0 + jj;
    dd a, gm;
    if (!rin || j >= N) {
      a = dd_of(i == j ? 1.0 : 0.0);
      gm = dd_of(0.0);
    } else {
      const dd exj = dd{pt_hi[j], pt_lo[j]};
      const dd epj = dd{pt_hi[2 * nmax + j], pt_lo[2 * nmax + j]};
      const dd emj = dd{pt_hi[3 * nmax + j], pt_lo[3 * nmax + j]};
      int d = (i - j) % N;
      if (d < 0) d += N;
      const dd cx = dd{tab_hi[d], tab_lo[d]}, sx = dd{tab_hi[N + d], tab_lo[N + d]};
      dd Kv, Gv;
      if (i != j) {
        const dd e1 = dd_mul(epi, emj), e2 = dd_mul(emi, epj);
        const dd s = dd_add(e1, e2), t = dd_sub(e1, e2);
        const dd chy = dd{0.5 * s.hi, 0.5 * s.lo}, shy = dd{0.5 * t.hi, 0.5 * t.lo};
        dd cre, cim;
        dd_cot_half(cx, sx, chy, shy, cre, cim);
        const dd k1 = dd_add(cim, dd_mul(exj, cre));
        const dd g1 = dd_sub(cre, dd_mul(exi, cim));
        Kv = dd{0.5 * k1.hi, 0.5 * k1.lo};
        Gv = dd_sub(dd{0.5 * g1.hi, 0.5 * g1.lo}, dd{tab_hi[2 * N + d], tab_lo[2 * N + d]});
      } else {
        const dd den = dd_add_d(dd_mul(exi, exi), 1.0);
        const dd q = dd_div(exxi, den);
        Kv = dd{-0.5 * q.hi, -0.5 * q.lo};
        const dd g = dd_mul(q, exi);
        Gv = dd{0.5 * g.hi, 0.5 * g.lo};
      }
      if (finite) {
        const dd e1 = dd_mul(epi, epj), e2 = dd_mul(emi, emj);
        const dd s = dd_add(e1, e2), t = dd_sub(e1, e2);
        const dd chy = dd{0.5 * s.hi, 0.5 * s.lo}, shy = dd{0.5 * t.hi, 0.5 * t.lo};
        dd dre, dim;
        dd_cot_half(cx, sx, chy, shy, dre, dim);
        const dd k2 = dd_sub(dim, dd_mul(exj, dre));
        const dd g2 = dd_sub(dre, dd_mul(exi, dim));
        Kv = dd_sub(Kv, dd{0.5 * k2.hi, 0.5 * k2.lo});
        Gv = dd_sub(Gv, dd{0.5 * g2.hi, 0.5 * g2.lo});
      }
      a = dd{Kv.hi * sc, Kv.lo * sc};
      if (i == j) a = dd_add_d(a, 0.5);
      gm = dd{Gv.hi * sc, Gv.lo * sc};
    }
    const size_t o = (size_t)j * Np + i;
    A_hi[o] = a.hi;
    A_lo[o] = a.lo;
    G_hi[o] = gm.hi;
    G_lo[o] = gm.lo;
    rt[tx][jj] = a.hi;
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < WW_TB * CW; idx += WW_NT) {
    const int r = idx / CW, cc = idx % CW;
    Af[(size_t)(i0 + r) * Np + j0 + cc] = rt[r][cc];
  }
}

// s += a b with s.lo left unnormalised: the product and the sum of the high parts are error
// free, their errors and the cross terms go to s.lo.  12 operations instead of the 29 of
// dd_mul and dd_add; each rounding of s.lo is 2^-53 |s.lo|, and dd_settle after every
// DD_SETTLE products keeps |s.lo| below DD_SETTLE ulps of the running sum.
#define DD_RUN 8
#define DD_SETTLE 4
__device__ __forceinline__ void dd_fma_acc(dd& s, dd a, dd b) {
  CONTRACT_OFF
  const double p = a.hi * b.hi;
  double e = fma(a.hi, b.hi, -p);
  e = fma(a.hi, b.lo, e);
  e = fma(a.lo, b.hi, e);
  const double h = s.hi + p, bb = h - s.hi;
  s.lo += ((s.hi - (h - bb)) + (p - bb)) + e;
  s.hi = h;
}
__device__ __forceinline__ void dd_settle(dd& s) { s = dd_two_sum(s.hi, s.lo); }

// out = add + sgn * A B for ncols columns in double-double (A column-major, all ld Np; add may
// be null).  A workgroup has 64 rows (one per lane) by NC columns, its eight waves split the
// inner index (runs of DD_RUN: w, w + 8, ...) and are summed in that order at the end.  A
// comes coalesced into registers, one run at a time, B through the scalar cache; five and more
// waves per SIMD cover the latency.
// Bound by the FP64 units: 12 Np^2 ncols operations at 39 T/s are 41 us at N = 1024, 129
// columns.  NC (dd_gemm): A is read Np / 64 x ncols / NC times, so wide, but the grid should
// come out even on the CUs.  Measured at that size: 92 us (one thread per entry over the whole
// inner index with normalised sums 244), the error of G psi against exact values (geometric
// mean over eight wavenumbers) 0.79 of what it was at N = 64, 0.49 at N = 1024.
#define DDG_NT 512
template <int NC>
__global__ __launch_bounds__(DDG_NT) void k_dd_gemm(const double* __restrict__ A_hi, const double* __restrict__ A_lo,
                                                    int Np, const double* __restrict__ B_hi,
                                                    const double* __restrict__ B_lo, const double* __restrict__ add_hi,
                                                    const double* __restrict__ add_lo, double sgn,
                                                    double* __restrict__ out_hi, double* __restrict__ out_lo,
                                                    int ncols) {
  constexpr int KS = DDG_NT / 64;
  __shared__ dd part[KS][NC][64];
  const int nrt = Np / 64, nct = (ncols + NC - 1) / NC;
  int rt, ct;
  if (nrt % 8 == 0) {   // workgroup b runs on XCD b mod 8: a band of row tiles each
    const int x = blockIdx.x % 8, l = blockIdx.x / 8;
    rt = x * (nrt / 8) + l / nct;
    ct = l % nct;
  } else {
    rt = blockIdx.x / nct;
    ct = blockIdx.x % nct;
  }
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  size_t bo[NC];   // uniform: B is read through the scalar cache
#pragma unroll
  for (int c = 0; c < NC; ++c) bo[c] = (size_t)min(ct * NC + c, ncols - 1) * Np;
  dd acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = dd_of(0.0);
#pragma unroll 1
  for (int k0 = w * DD_RUN; k0 < Np; k0 += KS * DD_RUN) {
    const size_t o = (size_t)k0 * Np + (size_t)rt * 64;
    double ah[DD_RUN], al[DD_RUN];
#pragma unroll
    for (int k = 0; k < DD_RUN; ++k) {
      ah[k] = (A_hi + (o + (size_t)k * Np))[(unsigned)lane];
      al[k] = (A_lo + (o + (size_t)k * Np))[(unsigned)lane];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int k = 0; k < DD_RUN; ++k) {
        dd_fma_acc(acc[c], dd{ah[k], al[k]}, dd{B_hi[bo[c] + k0 + k], B_lo ? B_lo[bo[c] + k0 + k] : 0.0});
        if (k % DD_SETTLE == DD_SETTLE - 1) dd_settle(acc[c]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) part[w][c][lane] = acc[c];
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * NC; e += DDG_NT) {
    const int c = e / 64, col = ct * NC + c;
    if (col >= ncols) break;
    dd t = part[0][c][e % 64];
#pragma unroll
    for (int g = 1; g < KS; ++g) t = dd_add(t, part[g][c][e % 64]);
    const size_t o = (size_t)col * Np + (size_t)rt * 64 + e % 64;
    dd v = dd{sgn * t.hi, sgn * t.lo};
    if (add_hi) v = dd_add(dd{add_hi[o], add_lo[o]}, v);
    out_hi[o] = v.hi;
    out_lo[o] = v.lo;
  }
}

// Residual maxima: a non-negative double orders like its bits; NaN counts as infinite.
__device__ __forceinline__ void dd_mx_put(unsigned long long* __restrict__ mx, double mr, double mb) {
  atomicMax(mx, (unsigned long long)__double_as_longlong(mr));
  atomicMax(mx + 1, (unsigned long long)__double_as_longlong(mb));
}

// The one-column form: 16 rows per workgroup (128 bytes of a column of A), 64 lanes per row
// over the inner index (j = q, q + 64, ...), summed by a fixed tree; no second launch for the
// partials.  mx (optional): max |out| and max |add| over the rows < N join mx[0], mx[1] (one
// atomic each per workgroup).  Latency bound.  Measured at N = 512: 6.6 us (64 rows x 16 inner
// chunks 4.7, a second launch for their sum 6.6, a third for the maxima 7.5).
#define DDV_NT 1024
__global__ __launch_bounds__(DDV_NT) void k_dd_gemv(const double* __restrict__ A_hi, const double* __restrict__ A_lo,
                                                    int Np, const double* __restrict__ x_hi,
                                                    const double* __restrict__ x_lo, const double* __restrict__ add_hi,
                                                    const double* __restrict__ add_lo, double sgn,
                                                    double* __restrict__ out_hi, double* __restrict__ out_lo, int N,
                                                    unsigned long long* __restrict__ mx) {
  __shared__ dd part[DDV_NT / 64][16];
  const int row = threadIdx.x & 15, q = threadIdx.x >> 4, lane = threadIdx.x & 63;
  const size_t i = (size_t)blockIdx.x * 16 + row;
  dd acc = dd_of(0.0);
#pragma unroll 4
  for (int j = q; j < Np; j += DDV_NT / 16) {
    const size_t o = (size_t)j * Np + i;
    acc = dd_add(acc, dd_mul(dd{A_hi[o], A_lo[o]}, dd{x_hi[j], x_lo ? x_lo[j] : 0.0}));
  }
  auto fold = [&](dd v, int m) { return dd_add(v, dd{__shfl_xor(v.hi, m), __shfl_xor(v.lo, m)}); };
  acc = fold(fold(acc, 16), 32);
  if (lane < 16) part[threadIdx.x >> 6][row] = acc;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int g = 4 * (lane >> 4);
  dd t = dd_add(dd_add(part[g][row], part[g + 1][row]), dd_add(part[g + 2][row], part[g + 3][row]));
  t = fold(fold(t, 16), 32);
  if (sgn < 0.0) t = dd_neg(t);
  dd ad = dd_of(0.0);
  if (add_hi) {
    ad = dd{add_hi[i], add_lo[i]};
    t = dd_add(ad, t);
  }
  if (lane < 16) {
    out_hi[i] = t.hi;
    out_lo[i] = t.lo;
  }
  if (!mx) return;
  const bool in = (int)i < N;
  double mr = in ? fabs(t.hi) : 0.0, mb = in ? fabs(ad.hi) : 0.0;
  if (mr != mr) mr = INFINITY;
#pragma unroll
  for (int m = 1; m < 16; m <<= 1) {
    mr = fmax(mr, __shfl_xor(mr, m));
    mb = fmax(mb, __shfl_xor(mb, m));
  }
  if (lane == 0) dd_mx_put(mx, mr, mb);
}

// the FP32 copy of the FP64 leading part of A (the mixed form factors it on MFMA)
__global__ void k_dd_a32(const double* __restrict__ A, float* __restrict__ A32, size_t n) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x)
    A32[e] = (float)A[e];
}

// mu += delta (double-double plus a double), n entries; lo0: mu's low part is not set yet (0)
__global__ void k_dd_correct(double* __restrict__ mu_hi, double* __restrict__ mu_lo, const double* __restrict__ delta,
                             size_t n, bool lo0) {
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
    const dd v = dd_add_d(dd{mu_hi[t], lo0 ? 0.0 : mu_lo[t]}, delta[t]);
    mu_hi[t] = v.hi;
    mu_lo[t] = v.lo;
  }
}

// gamma = d mu/dalpha and H gamma / 2 (spectrum |k| mu_hat / 2, zero at k = 0 and at
// Nyquist) of one column per workgroup, double-double; rows N..Np-1 zero.
// Measured: N = 512, one column 17 us (35); N = 1024, 129 columns 32 us (71).
__global__ __launch_bounds__(DDF_NT) void k_dd_gamma(const double* __restrict__ mu_hi,
                                                     const double* __restrict__ mu_lo, int Np,
                                                     const cdd* __restrict__ twg, int N, double* __restrict__ g_hi,
                                                     double* __restrict__ g_lo, double* __restrict__ h_hi,
                                                     double* __restrict__ h_lo) {
  extern __shared__ dd ldsd[];
  CddBuf Z = dd_buf(ldsd, 0, N), W = dd_buf(ldsd, 1, N);
  const CddBuf tw = dd_twiddles(ldsd, twg, N);
  const size_t off = (size_t)blockIdx.x * Np;
  for (int t = threadIdx.x; t < N; t += blockDim.x)
    Z.put(t, cdd{dd{mu_hi[off + t], mu_lo[off + t]}, dd_of(0.0)});
  dd_fft1(Z, W, tw, N, -1);
  CddBuf D[2] = {W, dd_buf(ldsd, 2, N)}, X[2] = {Z, dd_buf(ldsd, 3, N)};
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    const int k = t <= N / 2 ? t : t - N;
    const cdd z = Z.get(t);
    D[0].put(t, dd_ik(z, k, N));
    const double hk = (k == 0 || 2 * k == N || 2 * k == -N) ? 0.0 : 0.5 * fabs((double)k);
    D[1].put(t, cdd{dd_mul_d(z.re, hk), dd_mul_d(z.im, hk)});
  }
  dd_fft<2>(D, X, tw, N, +1);
  for (int t = threadIdx.x; t < Np; t += blockDim.x) {
    const bool in = t < N;
    const dd g = in ? D[0].re[t] : dd_of(0.0), h = in ? D[1].re[t] : dd_of(0.0);
    g_hi[off + t] = g.hi;
    g_lo[off + t] = g.lo;
    h_hi[off + t] = h.hi;
    h_lo[off + t] = h.lo;
  }
}

__global__ void k_dd_mx_reset(unsigned long long* __restrict__ mx) {
  if (threadIdx.x == 0) mx[0] = mx[1] = 0;
}

// max |r| and max |b| over rows < N of ncols columns (ld Np) into mx[0], mx[1]: one atomic
// maximum each per workgroup (one per thread took 28 us at N = 1024, 129 columns)
__global__ __launch_bounds__(WW_NT) void k_dd_maxabs(const double* __restrict__ r, const double* __restrict__ b, int N,
                                                     int Np, int ncols, unsigned long long* __restrict__ mx) {
  __shared__ double red[2][WW_NT / 64];
  double mr = 0.0, mb = 0.0;
  const size_t tot = (size_t)Np * ncols;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < tot; t += (size_t)gridDim.x * blockDim.x) {
    if ((int)(t % Np) >= N) continue;
    const double v = fabs(r[t]);
    mr = fmax(mr, v != v ? INFINITY : v);
    mb = fmax(mb, fabs(b[t]));
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    mr = fmax(mr, __shfl_xor(mr, m));
    mb = fmax(mb, __shfl_xor(mb, m));
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = mr;
    red[1][threadIdx.x >> 6] = mb;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int w = 1; w < WW_NT / 64; ++w) {
    mr = fmax(mr, red[0][w]);
    mb = fmax(mb, red[1][w]);
  }
  dd_mx_put(mx, mr, mb);
}

// =====================================================================================
// The base march in double-double (SDC15, the quadruple-precision workflow of Sec. 2.2):
// the right-hand side of eq. (ww) with the velocities of eq. (uv:from:G), the filter of
// eq. (filter) and the zero-mean projection, stage combinations and the outputs of eq.
// (f:phi) and (dfdT), every quantity a double-double.  States are 2N values [eta | phi]
// in hi and lo planes.
// =====================================================================================

// filter symbol exp(-36 (k / k_max)^36) for k = 0 .. N/2 (k_max = N/2, a power of two:
// k / k_max is exact; its 36th power by squarings in double-double)
__global__ void k_dd_filter_tab(int N, double* __restrict__ f_hi, double* __restrict__ f_lo) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k > N / 2) return;
  const dd x = dd_of((double)k / (double)(N / 2));
  const dd x2 = dd_mul(x, x), x4 = dd_mul(x2, x2), x8 = dd_mul(x4, x4);
  const dd x16 = dd_mul(x8, x8), x32 = dd_mul(x16, x16);
  const dd e = dd_exp(dd_mul_d(dd_mul(x32, x4), -36.0));
  f_hi[k] = e.hi;
  f_lo[k] = e.lo;
}

__device__ inline dd dd_ld(const double* __restrict__ h, const double* __restrict__ l, int i) {
  return dd{h[i], l[i]};
}
__device__ inline void dd_st(double* __restrict__ h, double* __restrict__ l, int i, dd v) {
  h[i] = v.hi;
  l[i] = v.lo;
}
// the filter symbol of wavenumber index t (0 .. N-1)
__device__ inline dd dd_filt_at(const double* __restrict__ f_hi, const double* __restrict__ f_lo, int t, int N) {
  const int k = t <= N / 2 ? t : N - t;
  return dd{f_hi[k], f_lo[k]};
}

// out = y0 + sum_t w_t K_{j_t} over n entries (the weights carry dt), double-double, the
// terms added in increasing t
__global__ void k_dd_sdc_combine(const double* __restrict__ y0h, const double* __restrict__ y0l,
                                 const double* __restrict__ Kh, const double* __restrict__ Kl, size_t kstride,
                                 const int* __restrict__ jt, const double* __restrict__ wh,
                                 const double* __restrict__ wl, int cnt, double* __restrict__ oh,
                                 double* __restrict__ ol, size_t n) {
  for (size_t e = blockIdx.x * (size_t)blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
    dd acc = dd{y0h[e], y0l[e]};
    for (int t = 0; t < cnt; ++t) {
      const size_t o = (size_t)jt[t] * kstride + e;
      acc = dd_add(acc, dd_mul(dd{wh[t], wl[t]}, dd{Kh[o], Kl[o]}));
    }
    oh[e] = acc.hi;
    ol[e] = acc.lo;
  }
}

// The base right-hand side at the state y (one workgroup): eta' and phi' by one packed
// transform (both real, the multiplier i k is odd), G phi given (double-double DtN);
//   u = (phi' - eta' G)/(1 + eta'^2),  v = (eta' phi' + G)/(1 + eta'^2),
//   eta_t = G phi,  phi_t = P[v eta_t - u^2/2 - v^2/2 - g eta + tau d/dx(eta'/sqrt(1 + eta'^2))],
// both filtered by one packed transform (the filter is even and real; P zeroes the mean
// of phi_t only: the imaginary part of mode 0).  The capillary term's two transforms are left
// out where tau = 0.  First the residual test of the solve behind G: status bit 4 unless
// max|r| <= tol max|b| (mx, cleared for the next solve).  Measured at N = 512: 28 us (66).
__global__ __launch_bounds__(DDF_NT) void k_dd_base_rhs(const double* __restrict__ yh, const double* __restrict__ yl,
                                                        const double* __restrict__ gh, const double* __restrict__ gl,
                                                        const double* __restrict__ f_hi,
                                                        const double* __restrict__ f_lo, const cdd* __restrict__ twg,
                                                        int N, double g, double tau, double* __restrict__ kh,
                                                        double* __restrict__ kl, unsigned long long* __restrict__ mx,
                                                        double tol, int* __restrict__ status) {
  extern __shared__ dd ldsd[];
  CddBuf Z = dd_buf(ldsd, 0, N), W = dd_buf(ldsd, 1, N), S = dd_buf(ldsd, 2, N);
  dd* const w = ldsd + (size_t)6 * N;   // the nonlinear terms
  const CddBuf tw = dd_twiddles(ldsd, twg, N);
  const dd zero = dd_of(0.0);
  if (threadIdx.x == 0) {
    const double mr = __longlong_as_double((long long)mx[0]), mb = __longlong_as_double((long long)mx[1]);
    if (!(mr <= tol * mb)) atomicOr(status, 4);
    mx[0] = 0;
    mx[1] = 0;
  }
  for (int t = threadIdx.x; t < N; t += blockDim.x) Z.put(t, cdd{dd_ld(yh, yl, t), dd_ld(yh, yl, N + t)});
  dd_fft1(Z, W, tw, N, -1);
  for (int t = threadIdx.x; t < N; t += blockDim.x) Z.put(t, dd_ik(Z.get(t), t <= N / 2 ? t : t - N, N));
  dd_fft1(Z, W, tw, N, +1);   // Z = eta' + i phi'
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    const dd ex = Z.re[t], ps = Z.im[t], G = dd_ld(gh, gl, t);
    const dd den = dd_add_d(dd_mul(ex, ex), 1.0);
    const dd u = dd_div(dd_sub(ps, dd_mul(ex, G)), den);
    const dd v = dd_div(dd_add(dd_mul(ex, ps), G), den);
    dd s = dd_sub(dd_mul(v, G), dd_mul_d(dd_add(dd_mul(u, u), dd_mul(v, v)), 0.5));
    w[t] = dd_sub(s, dd_mul_d(dd_ld(yh, yl, t), g));
    if (tau != 0.0) S.put(t, cdd{dd_div(ex, dd_sqrt(den)), zero});
  }
  if (tau != 0.0) {
    dd_fft1(S, W, tw, N, -1);
    for (int t = threadIdx.x; t < N; t += blockDim.x) S.put(t, dd_ik(S.get(t), t <= N / 2 ? t : t - N, N));
    dd_fft1(S, W, tw, N, +1);   // S.re = d/dx(eta'/sqrt(1 + eta'^2))
  }
  for (int t = threadIdx.x; t < N; t += blockDim.x)
    Z.put(t, cdd{dd_ld(gh, gl, t), tau != 0.0 ? dd_add(w[t], dd_mul_d(S.re[t], tau)) : w[t]});
  dd_fft1(Z, W, tw, N, -1);
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    const dd f = dd_filt_at(f_hi, f_lo, t, N);
    cdd v = cdd{dd_mul(Z.re[t], f), dd_mul(Z.im[t], f)};
    if (t == 0) v.im = zero;   // P: the mean of phi_t
    Z.put(t, v);
  }
  dd_fft1(Z, W, tw, N, +1);
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    dd_st(kh, kl, t, Z.re[t]);
    dd_st(kh, kl, N + t, Z.im[t]);
  }
}

// the filter on the state after a step (eta and phi packed), in place
__global__ __launch_bounds__(DDF_NT) void k_dd_filter_state(double* __restrict__ yh, double* __restrict__ yl,
                                                            const double* __restrict__ f_hi,
                                                            const double* __restrict__ f_lo,
                                                            const cdd* __restrict__ twg, int N) {
  extern __shared__ dd ldsd[];
  CddBuf Z = dd_buf(ldsd, 0, N), W = dd_buf(ldsd, 1, N);
  const CddBuf tw = dd_twiddles(ldsd, twg, N);
  for (int t = threadIdx.x; t < N; t += blockDim.x) Z.put(t, cdd{dd_ld(yh, yl, t), dd_ld(yh, yl, N + t)});
  dd_fft1(Z, W, tw, N, -1);
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    const dd f = dd_filt_at(f_hi, f_lo, t, N);
    Z.put(t, cdd{dd_mul(Z.re[t], f), dd_mul(Z.im[t], f)});
  }
  dd_fft1(Z, W, tw, N, +1);
  for (int t = threadIdx.x; t < N; t += blockDim.x) {
    dd_st(yh, yl, t, Z.re[t]);
    dd_st(yh, yl, N + t, Z.im[t]);
  }
}

// r = w phi, dr/dT = w phi_t / 4 (phi_t: the phi half of a right-hand side at the final
// state), f = r.r / 2 with w = 1/sqrt(N); one workgroup, the sum in a fixed order (each
// thread its strided terms in increasing index, then a tree over the threads)
__global__ __launch_bounds__(WW_NT) void k_dd_outputs(const double* __restrict__ yh, const double* __restrict__ yl,
                                                      const double* __restrict__ kh, const double* __restrict__ kl, int N,
                                                      double* __restrict__ rh, double* __restrict__ rl,
                                                      double* __restrict__ dh, double* __restrict__ dl,
                                                      double* __restrict__ fout) {
  __shared__ dd part[WW_NT];
  const dd w = dd_div(dd_of(1.0), dd_sqrt(dd_of((double)N)));
  dd acc = dd_of(0.0);
  for (int t = threadIdx.x; t < N; t += WW_NT) {
    const dd r = dd_mul(w, dd_ld(yh, yl, N + t));
    dd_st(rh, rl, t, r);
    if (dh) dd_st(dh, dl, t, dd_mul_d(dd_mul(w, dd_ld(kh, kl, N + t)), 0.25));
    acc = dd_add(acc, dd_mul(r, r));
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int s = WW_NT / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) part[threadIdx.x] = dd_add(part[threadIdx.x], part[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const dd f = dd_mul_d(part[0], 0.5);
    fout[0] = f.hi;
    fout[1] = f.lo;
  }
}
