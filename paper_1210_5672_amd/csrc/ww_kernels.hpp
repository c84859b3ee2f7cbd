// gfx950 kernels of the DtN / Jacobian hot path (Wilkening & Yu, overdetermined
// shooting for standing water waves).  FP64 throughout.
//
// Data layout (all device memory, column-major):
//   state column c (c = 0 base, c = 1..M Jacobian columns): 2N doubles,
//     [eta (N) | phi (N)], column stride 2N.
//   dense matrices A = I/2 + K/N and Gm = G/N: Np x Np, leading dimension Np, where
//     Np = N rounded up to the 64-row tile; the padding is the identity in A and zero
//     in Gm, so every blocked kernel works on whole 64x64 tiles.
//   solve arrays (right-hand sides, densities, gamma, DtN output): Np x R, ld Np.
//   per-point base arrays ("aux"): see AUX_* offsets.
#pragma once
#include <hip/hip_runtime.h>

#include "ww_fft.hpp"

#define WW_TB 64          // tile edge of the elimination
#define WW_NT 256         // threads per workgroup

// offsets of the mesh tables that the shared kernels read (see ww_mesh.hpp)
__device__ __forceinline__ size_t mesh_e(int nmax) { return (size_t)nmax; }
__device__ __forceinline__ size_t mesh_einv(int nmax) { return (size_t)2 * nmax; }

// per-point base quantities, each nmax doubles, at aux + AUX_x * nmax
enum {
  AUX_EX = 0,   // eta_x
  AUX_EXX,      // eta_xx
  AUX_PHS,      // varphi' (derivative of the surface potential along x)
  AUX_EP,       // exp(surface height)
  AUX_EM,       // exp(-surface height)
  AUX_U,        // phi_x on the surface
  AUX_V,        // phi_y on the surface
  AUX_W3,       // (1 + eta_x^2)^{3/2}
  AUX_COUNT
};

// Step coefficients in device memory (captured graphs stay valid when T changes):
//   coef[s * 16 + j] = a_sj dt,  coef[COEF_B + s] = b_s dt,  coef[COEF_DT] = dt
#define COEF_B 256
#define COEF_DT 300
#define COEF_SIZE 320

// Per-thread element sets: thread tid of a team of 256 owns t = tid + 256 m, m < PT.
// Global loads go through clamped, unconditional register loads (all in flight at once);
// only the stores are guarded by t < N.
#define NPT (WW_NMAX / WW_NT)

__device__ __forceinline__ int tidx(int m) { return threadIdx.x + WW_NT * m; }
__device__ __forceinline__ int tclamp(int m, int N) {
  const int t = tidx(m);
  return t < N ? t : N - 1;
}
// Pin register values at this point (stops the compiler from sinking their loads into
// later guarded blocks, which would serialise them).
template <int PT>
__device__ __forceinline__ void pin(const double (&v)[PT]) {
#pragma unroll
  for (int m = 0; m < PT; ++m) asm volatile("" ::"v"(v[m]));
}
template <int PT>
__device__ __forceinline__ void gload(double (&v)[PT], const double* __restrict__ p, int N, int tid = threadIdx.x) {
#pragma unroll
  for (int m = 0; m < PT; ++m) {
    const int t = tid + WW_NT * m;
    v[m] = p[t < N ? t : N - 1];
  }
}

// acc[m] = y[off + t_m] + sum_{j < stage} (a_sj dt) K[j][off + t_m]: stage values of the
// thread's elements; the loads of two stages for all elements are issued together.
// crow: the count weights (a_sj dt for a stage, b_s dt for the end of a step).
template <int PT>
__device__ __forceinline__ void stage_combine_vec(double (&acc)[PT], const double* __restrict__ y,
                                                  const double* __restrict__ K, size_t kstride, size_t off,
                                                  const double* __restrict__ crow, int count, int N,
                                                  int tid = threadIdx.x) {
  gload(acc, y + off, N, tid);
  for (int j0 = 0; j0 < count; j0 += 2) {
    const int j1 = (j0 + 1 < count) ? j0 + 1 : j0;
    const double a0 = crow[j0];
    const double a1 = (j0 + 1 < count) ? crow[j0 + 1] : 0.0;
    double k0[PT], k1[PT];
    gload(k0, K + (size_t)j0 * kstride + off, N, tid);
    gload(k1, K + (size_t)j1 * kstride + off, N, tid);
    pin(k0);
    pin(k1);
#pragma unroll
    for (int m = 0; m < PT; ++m) acc[m] = fma(a1, k1[m], fma(a0, k0[m], acc[m]));
  }
}

// Stage value at one element (column kernels: many threads, one element each).
__device__ __forceinline__ double stage_combine(double y0, const double* __restrict__ K, size_t kstride,
                                                size_t off, const double* __restrict__ coef, int stage) {
  double acc = y0;
  for (int j0 = 0; j0 < stage; j0 += 4) {
    double kv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = (j0 + q < stage) ? j0 + q : j0;
      kv[q] = K[(size_t)j * kstride + off];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (j0 + q < stage) acc = fma(coef[stage * 16 + j0 + q], kv[q], acc);
  }
  return acc;
}


// -------------------------------------------------------------------------------------
// state initialisation: q0 = q_fixed + basis @ params (column 0), Qdot(0) = basis
// -------------------------------------------------------------------------------------
__global__ void k_init_state(double* __restrict__ y, const double* __restrict__ basis,
                             const double* __restrict__ qfix, const double* __restrict__ params,
                             int N, int M) {
  const int R = M + 1;
  const int n2 = 2 * N;
  for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n2 * R; idx += gridDim.x * blockDim.x) {
    const int c = idx / n2, i = idx - c * n2;
    if (c == 0) {
      double s = qfix ? qfix[i] : 0.0;
      for (int k = 0; k < M; ++k) s += basis[(size_t)k * n2 + i] * params[k];
      y[i] = s;
    } else {
      y[(size_t)c * n2 + i] = basis[(size_t)(c - 1) * n2 + i];
    }
  }
}

// -------------------------------------------------------------------------------------
// base stage prep (one workgroup of two teams).  Stage value of the base column
//   Y_s = y + sum_{j<s} a_sj dt k_j,
// then eta_x, eta_xx (spectral), varphi', exp(+-surface height) and the Dirichlet
// data varphi into column 0 of the solve array (rows N..Np-1 zero).  Team 0 carries eta,
// team 1 varphi; the two inverse transforms run side by side.
// yhat (optional): the spectrum of eta + i varphi.  Dynamic LDS: 5 N complex (three work
// buffers, scratch, twiddles).
// -------------------------------------------------------------------------------------
#define PREP_NT 512

// failure detection: non-finite stage state (bit 2) or, at finite depth, a surface
// through the bottom (bit 16); status[2] keeps the first 16 step + stage
__device__ __forceinline__ void flag_state(int* __restrict__ status, bool bad, bool bed, int where) {
  if (status && (bad || bed)) {
    atomicOr(status, (bad ? 2 : 0) | (bed ? 16 : 0));
    atomicMin(status + 2, where);
  }
}

template <int NF>
__global__ __launch_bounds__(PREP_NT) void k_base_prep(
    const double* __restrict__ y, const double* __restrict__ K, double* __restrict__ Ys,
    const double* __restrict__ coef, int stage, size_t kstride, double* __restrict__ aux, int nmax,
    double* __restrict__ rhs0, int Np, const cplx* __restrict__ tw, int N, double hsurf, int* __restrict__ status,
    cplx* __restrict__ yhat) {
  constexpr int PT = FftSz<NF>::PT;
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* S = lds + 2 * N;
  cplx* X = lds + 3 * N;
  cplx* tws = lds + 4 * N;
  const FftPlan P = make_plan(N);
  const int tid = threadIdx.x & 255, team = threadIdx.x >> 8;
  load_twiddles<(PT + 1) / 2>(tws, tw, N);
  double v[PT];   // team 0: eta, team 1: varphi
  stage_combine_vec(v, y, K, kstride, team ? N : 0, coef + stage * 16, stage, N, tid);
  pin(v);
#pragma unroll
  for (int m = 0; m < PT; ++m) {
    const int t = tid + WW_NT * m;
    if (t < N) {
      Ys[team * N + t] = v[m];
      if (team) Z[t].y = v[m];
      else Z[t].x = v[m];
    }
  }
  FftSz<NF>::run(Z, W, tws, P, -1, tid, team == 0);   // spectrum of eta + i varphi
  for (int t = tid; t < N; t += WW_NT) {
    cplx E, F;
    split_pair(Z, t, N, E, F);
    const int k = wavenum(t, N);
    if (team) {
      S[t] = sym_deriv(F, k, N);
      if (yhat) yhat[t] = Z[t];
    } else {
      cplx ex = sym_deriv(E, k, N);
      W[t] = pack_pair(ex, sym_deriv(ex, k, N));
    }
  }
  // team 0: eta_x + i eta_xx; team 1: varphi' (imaginary part zero)
  FftSz<NF>::run(team ? S : W, team ? X : Z, tws, P, +1, tid, true);
  bool bad = false, bed = false;
#pragma unroll
  for (int m = 0; m < PT; ++m) {
    const int i = tid + WW_NT * m;
    if (i < N) {
      bad |= !isfinite(v[m]);
      if (team) {
        aux[AUX_PHS * nmax + i] = S[i].x;
        rhs0[i] = v[m];
      } else {
        aux[AUX_EX * nmax + i] = W[i].x;
        aux[AUX_EXX * nmax + i] = W[i].y;
        const double sh = v[m] + hsurf;
        aux[AUX_EP * nmax + i] = exp(sh);
        aux[AUX_EM * nmax + i] = exp(-sh);
        bed |= hsurf > 0.0 && sh <= 0.0;   // (a NaN height is reported as non-finite)
      }
    }
  }
  for (int i = N + (int)threadIdx.x; i < Np; i += PREP_NT) rhs0[i] = 0.0;
  // (status[1] counts the completed steps)
  if (status && (bad || bed)) flag_state(status, bad, bed, status[1] * 16 + stage);
}

typedef double dbl2v __attribute__((ext_vector_type(2)));
typedef float flt2v __attribute__((ext_vector_type(2)));

// -------------------------------------------------------------------------------------
// One row of y = add + sgn * M x from the row-major M (element type T, accumulation in
// double), by one wave: contiguous row reads, two entries a lane (x and M 2-entry aligned),
// eight pairs in flight, a fixed-order shuffle reduction.  Bound by memory latency.  With one
// entry a lane and load, sixteen in flight: f only N 1024 21.1 ms against 20.7, adjoint N 512
// 30.4 / 29.8.
// -------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void gemv_row_wave(const T* __restrict__ Mr, int Np, const double* __restrict__ x,
                                              const double* __restrict__ add, double sgn, double* __restrict__ y,
                                              int row, int lane) {
  typedef T T2 __attribute__((ext_vector_type(2)));
  const T2* mr = reinterpret_cast<const T2*>(Mr + (size_t)row * Np);
  const dbl2v* xr = reinterpret_cast<const dbl2v*>(x);
  const int n = Np / 2;
  double s0 = 0.0, s1 = 0.0;
  int j = lane;
  for (; j + 7 * 64 < n; j += 8 * 64) {
    T2 m[8];
    dbl2v xv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      m[q] = mr[j + 64 * q];
      xv[q] = xr[j + 64 * q];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      s0 = fma((double)m[q][0], xv[q][0], s0);
      s1 = fma((double)m[q][1], xv[q][1], s1);
    }
  }
#pragma unroll 4
  for (; j < n; j += 64) {
    const T2 m = mr[j];
    const dbl2v v = xr[j];
    s0 = fma((double)m[0], v[0], s0);
    s1 = fma((double)m[1], v[1], s1);
  }
  double s = s0 + s1;
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) y[row] = (add ? add[row] : 0.0) + sgn * s;
}

// -------------------------------------------------------------------------------------
// Kernel matrix assembly (Sec. 2.2 eq. (K1K2), App. A): A = I/2 + K/N, Gm = G/N.
//
// Entry (i, j), alpha_i - alpha_j = 2 pi d / N, d = (i - j) mod N:
//   C = cot((zeta_i - zeta_j)/2) by the branch formula of Sec. 2.2 with
//       cos x, sin x from a circulant table, cosh y, sinh y from exp(+-s_i) exp(-+s_j)
//   K1 = Im{zeta'_j C}/2,  G1 = Re{zeta'_i C}/2 - cot((alpha_i - alpha_j)/2)/2
//   diagonal: K1 = -Im{zeta''/(2 zeta')}, G1 = Re{zeta''/(2 zeta')}
//   finite depth (image surface conj zeta_j, all i, j):
//   D = cot((zeta_i - conj zeta_j)/2), K -= Im{conj(zeta'_j) D}/2, G -= Re{zeta'_i D}/2
// with zeta' = 1 + i eta_x, zeta'' = i eta_xx.  The image terms enter with a minus
// sign (the bracket of eq. (Phi) / (plemelj:1)-(plemelj:2)).
// The matrices are written row-major: thread (tx, ty) owns column tx of the strip and the
// rows ty + 4 m, so that every store is 64 consecutive doubles of a row.
// -------------------------------------------------------------------------------------
__device__ __forceinline__ void cot_half_branch(double cx, double sx, double chy, double shy,
                                                double& re, double& im) {
  if (cx >= 0.0) {
    const double num = cx + chy;
    const double inv = 1.0 / (sx * sx + shy * shy);
    re = num * sx * inv;
    im = -num * shy * inv;
  } else {
    const double inv = 1.0 / (chy - cx);
    re = sx * inv;
    im = -shy * inv;
  }
}

// Launch: grid (Np / 64, Np / ASM_CW): one workgroup per strip of ASM_CW rows x 64
// columns, several workgroups per 64-tile, so that enough waves are resident to hide
// the latency of the dependent FP64 chains (divisions of the cot branch formula).
// With a lagged inverse (Mx64 or Mx32, row-major), 16 more rows of workgroups follow
// the assembly grid: they form x0 = Mx psi (the first solve of the lagged-factor base
// chain, which does not need this stage's matrix), one wave per row.
// Writes A (row-major FP64: what the FP64 elimination starts from and what residuals
// multiply by), A32 (its FP32 copy, or null) and Gmr (row-major Gm).
template <int ASM_CW>
__global__ __launch_bounds__(WW_NT) void k_assemble(
    const double* __restrict__ aux, int nmax, const double* __restrict__ cosT,
    const double* __restrict__ sinT, const double* __restrict__ c0T, double* __restrict__ A,
    float* __restrict__ A32, double* __restrict__ Gmr, int N, int Np, int finite, const double* __restrict__ Mx64,
    const float* __restrict__ Mx32, const double* __restrict__ psi, double* __restrict__ x0) {
  if (blockIdx.y >= (unsigned)(Np / ASM_CW)) {
    // (uniform per workgroup: no barrier below is reached by these blocks)
    const int g = (blockIdx.y - Np / ASM_CW) * gridDim.x + blockIdx.x;
    const int row = g * (WW_NT / 64) + (threadIdx.x >> 6);
    if (row >= Np) return;
    if (Mx32)
      gemv_row_wave<float>(Mx32, Np, psi, nullptr, 1.0, x0, row, threadIdx.x & 63);
    else if (Mx64)
      gemv_row_wave<double>(Mx64, Np, psi, nullptr, 1.0, x0, row, threadIdx.x & 63);
    return;
  }
  // stage the per-point quantities of the strip's rows and 64 columns and the circulant
  // table entries d = i - j it touches in LDS
  __shared__ double rq[4][ASM_CW];           // eta_x, eta_xx, exp(s), exp(-s) of rows
  __shared__ double cq[3][WW_TB];            // eta_x, exp(s), exp(-s) of columns
  __shared__ double tb[3][WW_TB + ASM_CW];   // cos, sin, cot/2 of 2 pi d / N, d = i - j
  const int j0 = blockIdx.x * WW_TB, i0 = blockIdx.y * ASM_CW;
  const int t = threadIdx.x;
  {
    const int q = t >> 6, r = t & 63;
    const int jc = j0 + r;
    if (q < 3) cq[q][r] = (jc < N) ? aux[(q == 0 ? AUX_EX : q == 1 ? AUX_EP : AUX_EM) * nmax + jc] : 0.0;
    if (r < ASM_CW) {
      const int ir = i0 + r;
      rq[q][r] = (ir < N) ? aux[(q == 0 ? AUX_EX : q == 1 ? AUX_EXX : q == 2 ? AUX_EP : AUX_EM) * nmax + ir] : 0.0;
    }
    // table entries e <-> d = (i0 - j0 - 63 + e) mod N
    constexpr int NE = WW_TB + ASM_CW - 1;
    for (int e = t; e < 3 * NE; e += WW_NT) {
      const int which = e / NE, ee = e - which * NE;
      int d = (i0 - j0 - (WW_TB - 1) + ee) % N;
      if (d < 0) d += N;
      tb[which][ee] = which == 0 ? cosT[d] : which == 1 ? sinT[d] : c0T[d];
    }
  }
  __syncthreads();
  const int tx = t & 63;
  const int ty = t >> 6;
  const int j = j0 + tx;
  const double invN = 1.0 / (double)N;
  const double exj = cq[0][tx], epj = cq[1][tx], emj = cq[2][tx];
#pragma unroll
  for (int ii = ty; ii < ASM_CW; ii += 4) {
    const int i = i0 + ii;
    double a, gm;
    if (i >= N || j >= N) {
      a = (i == j) ? 1.0 : 0.0;
      gm = 0.0;
    } else {
      const double exi = rq[0][ii], exxi = rq[1][ii], epi = rq[2][ii], emi = rq[3][ii];
      const int e = ii - tx + (WW_TB - 1);
      const double cx = tb[0][e], sx = tb[1][e];
      double Kv, Gv;
      if (i != j) {
        const double e1 = epi * emj, e2 = emi * epj;   // exp(y), exp(-y), y = s_i - s_j
        const double chy = 0.5 * (e1 + e2), shy = 0.5 * (e1 - e2);
        double cre, cim;
        cot_half_branch(cx, sx, chy, shy, cre, cim);
        Kv = 0.5 * (cim + exj * cre);
        Gv = 0.5 * (cre - exi * cim) - tb[2][e];
      } else {
        const double den = 1.0 / (1.0 + exi * exi);
        Kv = -0.5 * exxi * den;
        Gv = 0.5 * exxi * exi * den;
      }
      if (finite) {
        const double e1 = epi * epj, e2 = emi * emj;   // exp(+-(s_i + s_j))
        const double chy = 0.5 * (e1 + e2), shy = 0.5 * (e1 - e2);
        double dre, dim;
        cot_half_branch(cx, sx, chy, shy, dre, dim);
        Kv -= 0.5 * (dim - exj * dre);
        Gv -= 0.5 * (dre - exi * dim);
      }
      a = Kv * invN + (i == j ? 0.5 : 0.0);
      gm = Gv * invN;
    }
    const size_t o = (size_t)i * Np + j;
    A[o] = a;
    if (A32) A32[o] = (float)a;
    Gmr[o] = gm;
  }
}

// -------------------------------------------------------------------------------------
// Matrix instructions v_mfma_f64_16x16x4f64 / v_mfma_f32_16x16x4f32.  Operand layout (lane
// l): A[row l%16][k l/16], B[k l/16][col l%16].  Result lane l holds column l%16 and rows
// row(i, l/16), i = 0..3: 4 i + l/16 (f64) or 4 (l/16) + i (f32).
// -------------------------------------------------------------------------------------
typedef double dbl4 __attribute__((ext_vector_type(4)));
typedef float flt4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mfma;
template <> struct Mfma<double> {
  typedef dbl4 V;
  static __device__ __forceinline__ V step(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row(i, rq) = rowc(i) + rowl(rq): the part common to the wave and the lane's
  static __device__ __forceinline__ int rowc(int i) { return 4 * i; }
  static __device__ __forceinline__ int rowl(int rq) { return rq; }
  static __device__ __forceinline__ int row(int i, int rq) { return rowc(i) + rowl(rq); }
  // element index and lane group (lane >> 4) of the result entries in row p
  static constexpr int row_elem(int p) { return p >> 2; }
  static constexpr int row_grp(int p) { return p & 3; }
};
template <> struct Mfma<float> {
  typedef flt4 V;
  static __device__ __forceinline__ V step(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int rowc(int i) { return i; }
  static __device__ __forceinline__ int rowl(int rq) { return 4 * rq; }
  static __device__ __forceinline__ int row(int i, int rq) { return rowc(i) + rowl(rq); }
  static constexpr int row_elem(int p) { return p & 3; }
  static constexpr int row_grp(int p) { return p >> 2; }
};

// Broadcast of lane n of each 16-lane row to the whole row (DPP row_newbcast).  n must
// fold to a constant (unrolled loops): the switch then reduces to one move.
template <int CTRL>
__device__ __forceinline__ double dpp_bcast(double v) {
  return __longlong_as_double((long long)__builtin_amdgcn_update_dpp(0LL, __double_as_longlong(v), CTRL, 0xf, 0xf,
                                                                     true));
}
template <int CTRL>
__device__ __forceinline__ float dpp_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <typename T>
__device__ __forceinline__ T row_bcast(T v, int n) {
  switch (n & 15) {
    case 0: return dpp_bcast<0x150>(v);
    case 1: return dpp_bcast<0x151>(v);
    case 2: return dpp_bcast<0x152>(v);
    case 3: return dpp_bcast<0x153>(v);
    case 4: return dpp_bcast<0x154>(v);
    case 5: return dpp_bcast<0x155>(v);
    case 6: return dpp_bcast<0x156>(v);
    case 7: return dpp_bcast<0x157>(v);
    case 8: return dpp_bcast<0x158>(v);
    case 9: return dpp_bcast<0x159>(v);
    case 10: return dpp_bcast<0x15a>(v);
    case 11: return dpp_bcast<0x15b>(v);
    case 12: return dpp_bcast<0x15c>(v);
    case 13: return dpp_bcast<0x15d>(v);
    case 14: return dpp_bcast<0x15e>(v);
    default: return dpp_bcast<0x15f>(v);
  }
}

// -------------------------------------------------------------------------------------
// Pivoting fallback.  The paper factors A without discussing pivoting (Sec. 3.3); A is
// diagonally dominant for the surfaces it treats, and the elimination runs without
// interchanges behind a pivot guard.  When a pivot falls below the guard, Gaussian
// elimination with partial pivoting (largest magnitude in the column, first row on
// ties) fixes a row order P; the elimination then runs on P A, whose pivots are the
// partial-pivoting ones, and every solve gathers its right-hand side by P.
// Two launches per column of the leading N x N block of W (column-major, ld Np):
// k_plu_pivot (one workgroup) picks the pivot, interchanges the two rows over all
// columns, records the interchange in perm ((P A) row i = A row perm[i]) and forms the
// multipliers; k_plu_update subtracts the rank-one update from the trailing block.
// Status bit 8: the largest candidate of a column is below the guard.
// -------------------------------------------------------------------------------------
#define PLU_NT 1024
__global__ __launch_bounds__(PLU_NT) void k_plu_pivot(double* __restrict__ W, int Np, int N, int k,
                                                       int* __restrict__ perm, double guard, int* __restrict__ status) {
  __shared__ double sv[PLU_NT / 64];
  __shared__ int si[PLU_NT / 64];
  __shared__ int sp;
  double* col = W + (size_t)k * Np;
  double bv = -1.0;
  int bi = N;
  for (int i = k + (int)threadIdx.x; i < N; i += PLU_NT) {   // rising rows: ties keep the first
    const double v = fabs(col[i]);
    if (v > bv) {
      bv = v;
      bi = i;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(bv, off);
    const int oi = __shfl_xor(bi, off);
    if (ov > bv || (ov == bv && oi < bi)) {
      bv = ov;
      bi = oi;
    }
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    sv[w] = bv;
    si[w] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = sv[0];
    int p = si[0];
    for (int q = 1; q < PLU_NT / 64; ++q)
      if (sv[q] > v || (sv[q] == v && si[q] < p)) {
        v = sv[q];
        p = si[q];
      }
    if (!(v >= guard)) atomicOr(status, 8);
    if (p < k || p >= N) p = k;   // no finite candidate (NaN column): keep the order
    sp = p;
    if (p != k) {
      const int t = perm[k];
      perm[k] = perm[p];
      perm[p] = t;
    }
  }
  __syncthreads();
  const int p = sp;
  if (p != k)
    for (int j = threadIdx.x; j < Np; j += PLU_NT) {
      double* cj = W + (size_t)j * Np;
      const double t = cj[k];
      cj[k] = cj[p];
      cj[p] = t;
    }
  __syncthreads();
  const double piv = col[k];
  for (int i = k + 1 + (int)threadIdx.x; i < N; i += PLU_NT) col[i] = col[i] / piv;
}

// W[i][j] -= W[i][k] W[k][j] for k < i, j < N: 64 rows x 16 columns per workgroup
__global__ __launch_bounds__(256) void k_plu_update(double* __restrict__ W, int Np, int N, int k) {
  const int i = k + 1 + blockIdx.x * 64 + (threadIdx.x & 63);
  if (i >= N) return;
  const double l = W[(size_t)k * Np + i];
  const int j0 = k + 1 + blockIdx.y * 16 + (threadIdx.x >> 6) * 4;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = j0 + q;
    if (j < N) W[(size_t)j * Np + i] -= l * W[(size_t)j * Np + k];
  }
}

__global__ void k_iota(int* __restrict__ p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = i;
}

// column-major copy of the row-major Np x Np matrix (the elimination's workspace)
__global__ void k_plu_copy(const double* __restrict__ A, double* __restrict__ W, int Np) {
  __shared__ double t[32][33];
  const int i0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) t[r][tx] = A[(size_t)(i0 + r) * Np + j0 + tx];
  __syncthreads();
  for (int c = ty; c < 32; c += 8) W[(size_t)(j0 + c) * Np + i0 + tx] = t[tx][c];
}
// the rows of the row-major Np x Np matrix by perm: dst row i = src row perm[i] (P A)
__global__ void k_gather_rows(const double* __restrict__ src, double* __restrict__ dst, const int* __restrict__ perm,
                              int Np) {
  const size_t i = blockIdx.x, q = perm[i];
  for (int j = threadIdx.x; j < Np; j += blockDim.x) dst[i * Np + j] = src[q * Np + j];
}

// rows of an Np x ncols column-major array (ld Np) by perm: gather dst[i] = src[perm[i]]
// (P x), or scatter dst[perm[i]] = src[i] (P^T x)
__global__ void k_permute_rows(const double* __restrict__ src, double* __restrict__ dst, const int* __restrict__ perm,
                               int Np, int ncols, int scatter) {
  const size_t tot = (size_t)Np * ncols;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < tot; idx += (size_t)gridDim.x * blockDim.x) {
    const size_t c = idx / Np;
    const int i = (int)(idx - c * Np);
    const int q = perm[i];
    if (scatter) dst[c * Np + q] = src[c * Np + i];
    else dst[c * Np + i] = src[c * Np + q];
  }
}

// -------------------------------------------------------------------------------------
// One right-hand side: y = add + sgn * M x, one wave per row (no cross-workgroup reduction).
// -------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(WW_NT) void k_gemv_row(const T* __restrict__ Mr, int Np,
                                                    const double* __restrict__ x, const double* __restrict__ add,
                                                    double sgn, double* __restrict__ y) {
  const int row = (blockIdx.x * WW_NT + threadIdx.x) >> 6;
  if (row >= Np) return;
  gemv_row_wave<T>(Mr, Np, x, add, sgn, y, row, threadIdx.x & 63);
}


// -------------------------------------------------------------------------------------
// Product with a row-major matrix for R right-hand sides:  out = add + sgn * M B
// (M: Np x Np row-major, element type T; B, add, out: Np x R column-major doubles,
// ld Np; B is rounded to T at the matrix instruction).  A workgroup's tile is 16 rows by 16 BC
// columns, its eight waves split the inner index (chunks of 16: w, w + 8, ...); the partial
// tiles are summed in LDS in a fixed order and stored once.
//
// Both operands have the inner index contiguous while a matrix instruction wants 16 rows (or
// columns) in consecutive lanes: loaded in that order, each lane's 16 bytes are an address of
// their own for the cache (60 cycles per load instruction; 23 us for N = 1024, R = 128).  So
// eight consecutive lanes load the 128 bytes of one row's chunk, and the wave turns the chunk
// round in its own piece of LDS (16-byte slots, slot s of row r at s ^ ((r >> 1) & 7): the 16
// rows that a lane group reads fall into the 16 slots of LDS's 256-byte bank row).  No barrier
// until the end, and D chunks per wave in flight in registers.
// The inner indices of instruction (h, e) are 8 h + 2 rq + e, the same in both operands.
//
// Bound by the matrix units (2 Np^2 R operations, 73 TFLOP/s) and, where a CU has one tile,
// by the latency of the first chunks and of the final sum.  Small tiles: larger ones read
// less from L2 but fill the CUs unevenly (R = 257 in 32 x 32 tiles, N 1024: 22 us against
// 18).  Workgroup b runs on XCD b mod 8: each XCD takes a band of row tiles with all their
// column tiles, so that its L2 holds that band of M and all of B.
// Measured, FP64, against 32 x 32 tiles whose operands the whole workgroup staged in LDS in
// 128-deep chunks: N x R = 256 x 64 2.7 us (7.8), 768 x 137 6.0 (15.2), 1024 x 128 7.8 (19.2;
// its operations 3.7), 2048 x 257 52 (94; 30).
// -------------------------------------------------------------------------------------
#define GEMM_NT 512
// The wave's own LDS accesses on either side stay in program order.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// One 16 x 16 operand block (rows r0 .. r0 + 15, 16 inner entries) of type T between global
// memory, registers and LDS.  Double: 2 loads of 8 rows; float: 1 load of 16 rows.
template <typename T> struct GemmOp;
template <> struct GemmOp<double> {
  static constexpr int L = 2, BYTES = 2048;   // loads, LDS bytes
  typedef dbl2v V;
  static __device__ int lrow(int lane) { return lane >> 3; }
  static __device__ int lcol(int lane) { return 2 * (lane & 7); }
  static __device__ int put_off(int lane, int l) {
    const int r = 8 * l + (lane >> 3);
    return r * 128 + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
  }
  static __device__ void get(const char* S, int cl, int rq, double (&v)[4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const dbl2v x = *reinterpret_cast<const dbl2v*>(S + cl * 128 + (((4 * h + rq) ^ (cl >> 1)) << 4));
      v[2 * h] = x[0];
      v[2 * h + 1] = x[1];
    }
  }
};
template <> struct GemmOp<float> {
  static constexpr int L = 1, BYTES = 1024;
  typedef flt4 V;
  static __device__ int lrow(int lane) { return lane >> 2; }
  static __device__ int lcol(int lane) { return 4 * (lane & 3); }
  static __device__ int put_off(int lane, int) {
    const int r = lane >> 2;
    return r * 64 + (((lane & 3) ^ (r >> 2)) << 4);
  }
  static __device__ void get(const char* S, int cl, int rq, float (&v)[4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const flt2v x =
          *reinterpret_cast<const flt2v*>(S + cl * 64 + (((2 * h + (rq >> 1)) ^ (cl >> 2)) << 4) + ((rq & 1) << 3));
      v[2 * h] = x[0];
      v[2 * h + 1] = x[1];
    }
  }
};

template <typename T, int BC, int D>
__global__ __launch_bounds__(GEMM_NT) void k_gemm_rm(const T* __restrict__ M, int Np, const double* __restrict__ B, int R,
                                                     const double* __restrict__ add, double sgn,
                                                     double* __restrict__ out) {
  constexpr int KS = GEMM_NT / 64, TR = 16, TC = 16 * BC, LD = TR + 1;
  constexpr int WB = GemmOp<T>::BYTES + BC * GemmOp<double>::BYTES;   // LDS bytes of a wave
  constexpr int SB = WB > TC * LD * 8 ? KS * WB : KS * TC * LD * 8;
  constexpr int LA = GemmOp<T>::L, LB = BC * GemmOp<double>::L;
  typedef typename Mfma<T>::V V;
  typedef typename GemmOp<T>::V VA;
  __shared__ __attribute__((aligned(256))) char sm[SB];
  const int nrt = Np / TR, nct = (R + TC - 1) / TC;
  int rt, ct;
  if (nrt % 8 == 0) {
    const int x = blockIdx.x % 8, l = blockIdx.x / 8;
    rt = x * (nrt / 8) + l / nct;
    ct = l % nct;
  } else {
    rt = blockIdx.x / nct;
    ct = blockIdx.x % nct;
  }
  const int lane = threadIdx.x & 63, cl = lane & 15, rq = lane >> 4;
  const int ks = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  char* const sa = sm + ks * WB;
  char* const sb = sa + GemmOp<T>::BYTES;
  const T* const ab = M + (size_t)(rt * TR) * Np + 16 * ks;
  const unsigned ao = (unsigned)(GemmOp<T>::lrow(lane) * Np + GemmOp<T>::lcol(lane));
  const double* bp[LB];
#pragma unroll
  for (int l = 0; l < LB; ++l)
    bp[l] = B + (size_t)min(ct * TC + 8 * l + GemmOp<double>::lrow(lane), R - 1) * Np + 16 * ks +
            GemmOp<double>::lcol(lane);
  const int n = (Np / 16 - ks + KS - 1) / KS;   // chunks of this wave
  VA a[D][LA];
  dbl2v b[D][LB];
  V acc[BC];
#pragma unroll
  for (int q = 0; q < BC; ++q) acc[q] = V{T(0), T(0), T(0), T(0)};
  auto fetch = [&](int d, int i) {
#pragma unroll
    for (int l = 0; l < LA; ++l)
      a[d][l] = *reinterpret_cast<const VA*>(ab + (size_t)(8 * l) * Np + (size_t)i * 16 * KS + ao);
#pragma unroll
    for (int l = 0; l < LB; ++l) b[d][l] = *reinterpret_cast<const dbl2v*>(bp[l] + (size_t)i * 16 * KS);
  };
  auto turn = [&](int d) {   // chunk of register set d into LDS
    wave_lds_order();
#pragma unroll
    for (int l = 0; l < LA; ++l)
      *reinterpret_cast<VA*>(sa + GemmOp<T>::put_off(lane, l)) = a[d][l];
#pragma unroll
    for (int l = 0; l < LB; ++l)
      *reinterpret_cast<dbl2v*>(sb + l / 2 * 2048 + GemmOp<double>::put_off(lane, l % 2)) = b[d][l];
    wave_lds_order();
  };
  auto product = [&](int dn) {   // chunk in LDS; the chunk of register set dn (>= 0) follows it
    T av[4];
    double bv[BC][4];
    GemmOp<T>::get(sa, cl, rq, av);
#pragma unroll
    for (int q = 0; q < BC; ++q) GemmOp<double>::get(sb + q * 2048, cl, rq, bv[q]);
    if (dn >= 0) turn(dn);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int q = 0; q < BC; ++q) acc[q] = Mfma<T>::step(av[j], (T)bv[q][j], acc[q]);
  };
  if (n > 0) {
    // prefetches past the last chunk repeat it (in bounds, unused)
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d, min(d, n - 1));
    turn(0);
    int i = 0;
    for (; i + D < n; i += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        fetch(d, min(i + d + D, n - 1));
        product((d + 1) % D);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (i + d < n) product(d + 1 < D ? d + 1 : -1);
  }
  __syncthreads();
  double* const Cs = reinterpret_cast<double*>(sm);
#pragma unroll
  for (int q = 0; q < BC; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) Cs[(ks * TC + 16 * q + cl) * LD + Mfma<T>::row(i, rq)] = (double)acc[q][i];
  __syncthreads();
  for (int e = threadIdx.x; e < TR * TC; e += GEMM_NT) {
    const int c = e / TR, r = e % TR, cc = ct * TC + c;
    if (cc >= R) break;
    double s = Cs[c * LD + r];
#pragma unroll
    for (int g = 1; g < KS; ++g) s += Cs[(g * TC + c) * LD + r];
    const size_t o = (size_t)cc * Np + rt * TR + r;
    out[o] = (add ? add[o] : 0.0) + sgn * s;
  }
}

// -------------------------------------------------------------------------------------
// gamma = d mu / d alpha and (1/2) H gamma for a pair of columns (eq. (G)):
// spectrum of mu_a + i mu_b, gamma_hat = i k mu_hat, (H gamma)_hat = |k| mu_hat
// (both zero at k = 0 and at Nyquist).  Rows N..Np-1 of the outputs are zero.  Two teams:
// the inverse transforms of the two columns run side by side.
// Dynamic LDS: 5 N complex (three work buffers, scratch and the twiddles).
// -------------------------------------------------------------------------------------
template <int NT>
__device__ inline void refine_check_col(const double* __restrict__ rc, const double* __restrict__ bc, int N,
                                        double tol, int* __restrict__ status, int flag, double* red);

template <int NF>
__global__ __launch_bounds__(PREP_NT) void k_gamma(const double* __restrict__ Mu, int Np, int ncols,
                                                   double* __restrict__ Gam, double* __restrict__ HG,
                                                   const cplx* __restrict__ tw, int N,
                                                   const double* __restrict__ chk_r, const double* __restrict__ chk_b,
                                                   double chk_tol, int* __restrict__ status, int chk_flag) {
  constexpr int PT = FftSz<NF>::PT;
  // the refinement test of the solve that produced Mu's first column, when chk_r is
  // given (the check kernel's work, folded into this launch)
  extern __shared__ cplx lds[];
  // (in the transform buffers: at N = 2048 they take all of a compute unit's LDS)
  if (chk_r && blockIdx.x == 0) {
    refine_check_col<PREP_NT>(chk_r, chk_b, N, chk_tol, status, chk_flag, reinterpret_cast<double*>(lds));
    __syncthreads();
  }
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* S = lds + 2 * N;
  cplx* X = lds + 3 * N;
  cplx* tws = lds + 4 * N;
  const FftPlan P = make_plan(N);
  const int tid = threadIdx.x & 255, team = threadIdx.x >> 8;
  load_twiddles<(PT + 1) / 2>(tws, tw, N);
  const int ca = 2 * blockIdx.x, cb = ca + 1;
  const bool hasb = cb < ncols;
  {
    double v[PT];
    gload(v, Mu + (size_t)(team && hasb ? cb : ca) * Np, N, tid);
    pin(v);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) {
        if (team) Z[t].y = hasb ? v[m] : 0.0;
        else Z[t].x = v[m];
      }
    }
  }
  FftSz<NF>::run(Z, W, tws, P, -1, tid, team == 0);
  for (int t = tid; t < N; t += WW_NT) {
    cplx A, B;
    split_pair(Z, t, N, A, B);
    const int k = wavenum(t, N);
    const double hk = (k == 0 || 2 * k == N || 2 * k == -N) ? 0.0 : 0.5 * fabs((double)k);
    if (team) S[t] = pack_pair(sym_deriv(B, k, N), cscale(B, hk));
    else W[t] = pack_pair(sym_deriv(A, k, N), cscale(A, hk));
  }
  FftSz<NF>::run(team ? S : W, team ? X : Z, tws, P, +1, tid, !team || hasb);
  if (team && !hasb) return;
  const cplx* V = team ? S : W;
  const size_t o = (size_t)(team ? cb : ca) * Np;
  for (int t = tid; t < Np; t += WW_NT) {
    const bool in = t < N;
    Gam[o + t] = in ? V[t].x : 0.0;
    HG[o + t] = in ? V[t].y : 0.0;
  }
}

// -------------------------------------------------------------------------------------
// Base DtN output of a lagged-factor stage in one launch (eq. (G)): every workgroup
// forms gamma = d mu/d alpha and (1/2) H gamma of the base density mu in LDS (one
// forward and one inverse FFT of its own), then, for its rows i (one wave per row),
//   G phi_i = (1/2) H gamma_i + sum_j Gm_ij gamma_j          (row-major Gm)
//   r_i     = psi_i - sum_j A_ij mu_j                          (row-major A)
// the FP64 residual of the refined solve.  The convergence test of that solve
// (max |r| <= tol max |psi|) needs both maxima over all rows: every workgroup leaves its own
// in chk[block] (max |r|; a NaN residual counts as infinite) and chk[grid + block] (max
// |psi|), and the next kernel on the stream (k_base_stage) takes the decision.  (One atomic
// maximum per wave on two shared words took 10 us of this launch's 23.)
//  Rows N..Np-1 of Gphi are zero.  Dynamic LDS: 4 N complex.  A workgroup
// takes `rows` consecutive rows (a multiple of 4; grid ceil(Np / rows)).
// -------------------------------------------------------------------------------------
// The entries of a wave's rows come from memory once; with two rows a wave (8 per
// workgroup) and rows of at most 1024 entries both rows are in flight before the
// transforms, which do not need them.
// -------------------------------------------------------------------------------------
template <int NF>
__global__ __launch_bounds__(WW_NT) void k_base_dtn(const double* __restrict__ mu, const double* __restrict__ psi,
                                                    const double* __restrict__ Gmr, const double* __restrict__ Ar,
                                                    int Np, const cplx* __restrict__ tw, int N,
                                                    double* __restrict__ Gphi,
                                                    double* __restrict__ chk, int rows) {
  constexpr int PT = FftSz<NF>::PT;
  constexpr int NR = 4 * PT;               // entries of a row per lane, N <= 64 NR
  constexpr int PRE = NR <= 16 ? 2 : 1;    // rows in flight
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* tws = lds + 2 * N;
  double* xs = reinterpret_cast<double*>(lds + 3 * N);   // mu (N doubles)
  double* gs = xs + N;                                   // gamma (N doubles)
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  double gv[PRE][NR], av[PRE][NR];
  auto load_row = [&](int b, int row) {   // clamped, unconditional loads
    const int rr = row < N ? row : N - 1;
    const double* gr = Gmr + (size_t)rr * Np;
    const double* ar = Ar + (size_t)rr * Np;
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int j = lane + 64 * m;
      const int jj = j < N ? j : N - 1;
      gv[b][m] = gr[jj];
      av[b][m] = ar[jj];
    }
  };
  const int row0 = blockIdx.x * rows + wv;
#pragma unroll
  for (int b = 0; b < PRE; ++b)
    if (b == 0 || rows > 4) load_row(b, row0 + 4 * b);
  const FftPlan P = make_plan(N);
  load_twiddles<PT>(tws, tw, N);
  {
    double va[PT];
    gload(va, mu, N);
    pin(va);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tidx(m);
      if (t < N) {
        Z[t] = cmk(va[m], 0.0);
        xs[t] = va[m];
      }
    }
  }
  FftSz<NF>::run(Z, W, tws, P, -1, tid, true);
  for (int t = tid; t < N; t += WW_NT) {
    const int k = wavenum(t, N);
    const double hk = (k == 0 || 2 * k == N || 2 * k == -N) ? 0.0 : 0.5 * fabs((double)k);
    // Z holds the spectrum of the real signal mu: gamma_hat = i k mu_hat, (H gamma / 2)_hat
    // = |k| mu_hat / 2; both real signals travel as one complex signal
    W[t] = pack_pair(sym_deriv(Z[t], k, N), cscale(Z[t], hk));
  }
  FftSz<NF>::run(W, Z, tws, P, +1, tid, true);
  for (int t = tid; t < N; t += WW_NT) gs[t] = W[t].x;
  __syncthreads();
  double mr = 0.0, mb = 0.0;
  for (int q0 = 0; q0 < rows / 4; q0 += PRE) {
#pragma unroll
    for (int b = 0; b < PRE; ++b) {
      const int q = q0 + b, row = row0 + 4 * q;
      if (q >= rows / 4 || row >= Np) break;
      if (q >= PRE) load_row(b, row);
      if (row >= N) {
        if (lane == 0) Gphi[row] = 0.0;
        continue;
      }
      double s0 = 0.0, s1 = 0.0, t0 = 0.0, t1 = 0.0;
#pragma unroll
      for (int m = 0; m < NR; m += 2) {
        const int j0 = lane + 64 * m, j1 = j0 + 64;
        if (j0 < N) {
          s0 = fma(gv[b][m], gs[j0], s0);
          t0 = fma(av[b][m], xs[j0], t0);
        }
        if (j1 < N) {
          s1 = fma(gv[b][m + 1], gs[j1], s1);
          t1 = fma(av[b][m + 1], xs[j1], t1);
        }
      }
      double s = s0 + s1, t = t0 + t1;
      for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_down(s, off, 64);
        t += __shfl_down(t, off, 64);
      }
      if (lane == 0) {
        Gphi[row] = W[row].y + s;
        const double r = psi[row] - t;
        mr = fmax(mr, fabs(r));
        if (r != r) mr = INFINITY;
        mb = fmax(mb, fabs(psi[row]));
      }
    }
  }
  __syncthreads();   // the transform buffer is free: the waves' maxima
  double* red = reinterpret_cast<double*>(Z);
  if (lane == 0) {
    red[wv] = mr;
    red[4 + wv] = mb;
  }
  __syncthreads();
  if (tid < 2) {
    const double* m = red + 4 * tid;
    chk[tid * gridDim.x + blockIdx.x] = fmax(fmax(m[0], m[1]), fmax(m[2], m[3]));
  }
}

// The convergence test of a lagged-factor solve from the n maxima of |r| and of |psi| left by
// k_base_dtn, by one wave.
__device__ __forceinline__ void lagged_check(const double* __restrict__ chk, int n, double tol,
                                             int* __restrict__ status, int flag) {
  const int lane = threadIdx.x & 63;
  double mr = 0.0, mb = 0.0;
  for (int i = lane; i < n; i += 64) {
    mr = fmax(mr, chk[i]);
    mb = fmax(mb, chk[n + i]);
  }
  for (int off = 32; off > 0; off >>= 1) {
    mr = fmax(mr, __shfl_xor(mr, off));
    mb = fmax(mb, __shfl_xor(mb, off));
  }
  if (lane == 0 && !(mr <= tol * mb)) atomicOr(status, flag);
}

// -------------------------------------------------------------------------------------
// Base right-hand side (Sec. 2.1 eq. (ww), (uv:from:G)), one workgroup:
//   u = (varphi' - eta_x G phi)/(1 + eta_x^2),  v = (eta_x varphi' + G phi)/(1 + eta_x^2)
//   eta_t = G phi
//   varphi_t = P[v eta_t - u^2/2 - v^2/2 - g eta + tau d/dx(eta_x/sqrt(1 + eta_x^2))]
// both filtered; u, v, (1 + eta_x^2)^{3/2} are kept for the variational columns.
// -------------------------------------------------------------------------------------
// One workgroup of two teams: the transforms of (eta_t, undifferentiated terms) and of the
// tension term run side by side (without tension there is none).  Dynamic LDS: 5 N complex.
template <int NF>
__global__ __launch_bounds__(PREP_NT) void k_base_rhs(const double* __restrict__ Ys, const double* __restrict__ Gphi,
                                                      double* __restrict__ aux, int nmax, double* __restrict__ Kout,
                                                      const cplx* __restrict__ tw, const double* __restrict__ sig,
                                                      int N, double g, double tau) {
  constexpr int PT = FftSz<NF>::PT;
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* S = lds + 2 * N;
  cplx* X = lds + 3 * N;
  cplx* tws = lds + 4 * N;
  const FftPlan P = make_plan(N);
  const int tid = threadIdx.x & 255, team = threadIdx.x >> 8;
  load_twiddles<(PT + 1) / 2>(tws, tw, N);
  double exv[PT];
  gload(exv, aux + AUX_EX * nmax, N, tid);
  if (team == 0) {
    double psv[PT], Gv[PT], etv[PT];
    gload(psv, aux + AUX_PHS * nmax, N, tid);
    gload(Gv, Gphi, N, tid);
    gload(etv, Ys, N, tid);
    pin(exv);
    pin(psv);
    pin(Gv);
    pin(etv);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) {
        const double ex = exv[m], ps = psv[m], G = Gv[m];
        const double den = 1.0 + ex * ex;
        const double u = (ps - ex * G) / den;
        const double v = (ex * ps + G) / den;
        aux[AUX_U * nmax + t] = u;
        aux[AUX_V * nmax + t] = v;
        aux[AUX_W3 * nmax + t] = den * sqrt(den);
        Z[t] = cmk(G, v * G - 0.5 * u * u - 0.5 * v * v - g * etv[m]);
      }
    }
  } else {
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) S[t] = cmk(tau * exv[m] / sqrt(1.0 + exv[m] * exv[m]), 0.0);
    }
  }
  FftSz<NF>::run(team ? S : Z, team ? X : W, tws, P, -1, tid, team == 0 || tau != 0.0);
  for (int t = threadIdx.x; t < N; t += PREP_NT) {
    cplx A, C, F = cmk(0.0, 0.0), dummy;
    split_pair(Z, t, N, A, C);
    if (tau != 0.0) split_pair(S, t, N, F, dummy);
    const int k = wavenum(t, N);
    const double sg = sig[t];
    cplx et = cscale(A, sg);
    cplx pt = (k == 0) ? cmk(0.0, 0.0) : cscale(cadd(C, sym_deriv(F, k, N)), sg);
    W[t] = pack_pair(et, pt);
  }
  FftSz<NF>::run(W, Z, tws, P, +1, tid, team == 0);
  for (int t = threadIdx.x; t < N; t += PREP_NT) {
    Kout[t] = W[t].x;
    Kout[N + t] = W[t].y;
  }
}

// -------------------------------------------------------------------------------------
// The right-hand side of stage s and the prep of the next stage state in one workgroup, on
// the march's critical path: the base column of a lagged-factor march is kept in spectral
// form.  The slope's spectrum K_s^ (of eta_t + i varphi_t, filtered) goes to the stage
// slot, the next stage state's spectrum is
//   Y^ = y^ + sum_{j <= s} w_j K_j^       (w: a row of the tableau times dt)
// or, at the end of a step (end = 1, w = b dt), y^ <- S_F Y^ with the filter symbol, and
// three inverse transforms give eta + i varphi, eta_x + i eta_xx and varphi'.  Bound by
// latency (one compute unit): three teams run the two forward transforms and then the
// three inverse ones side by side, and the terms j < s of the combination are summed
// while the forward transforms run.  One transform after the other, with the combination
// and the forward transform of the stage state in physical space, the same work took 24.5
// us at N = 1024 (27.8 us in the march, and 50 us at the end of a step in three
// launches); so: 11.7 us alone and 13.7 us in the march, at the end of a step too.
// MAP: on the mapped grid (the right-hand side of eq. (ww) with x-derivatives (1/E)
// d/dalpha, G phi / E and the E-weighted zero mean).  Dynamic LDS: 7 N complex, or 4 N
// (transforms in place) where 7 N does not fit.
// -------------------------------------------------------------------------------------
#define STAGE_NT 768
struct StageArgs {
  const double* Gphi;          // (1/2) H gamma + Gm gamma
  double* aux_cur;             // per-point quantities of stage s (in) and of the next (out)
  double* aux_next;
  double* Ys;                  // base stage state: eta of stage s (in), the next state (out)
  double* y;                   // base state in physical space (written at the end of a step)
  cplx* yhat;                  // its spectrum
  double* K;                   // stage slots (stride kstride doubles): spectra in the base column
  size_t kstride;
  const double* w;             // s + 1 weights
  const double* chk;           // the maxima of the lagged solve's test (nchk workgroups)
  int* status;
  const cplx* tw;
  const double* sig;
  const double* mesh;          // MAP: mesh tables
  double* rhs0;
  double chk_tol, g, tau, hsurf;
  int nchk, s, end, check, nmax, N, Np, inplace;
};

template <int NF, int MAP>
__global__ __launch_bounds__(STAGE_NT) void k_base_stage(StageArgs q) {
  constexpr int PT = FftSz<NF>::PT;
  extern __shared__ cplx lds[];
  __shared__ double red[4];
  const int N = q.N, nmax = q.nmax;
  const int tid = threadIdx.x & 255, team = threadIdx.x >> 8;
  cplx* B[3] = {lds, lds + N, lds + 2 * N};
  cplx* tws = lds + 3 * N;
  cplx* buf = lds + team * N;
  cplx* scr = q.inplace ? buf : lds + (4 + team) * N;
  cplx* const Yb = B[2];   // the next state's spectrum: team 2's buffer
  const FftPlan P = make_plan(N);
  const int done = q.status[1];   // steps completed before this one
  load_twiddles<(PT + 2) / 3>(tws, q.tw, N);
  cplx acc[PT];   // team 2: y^ + sum over the earlier slopes
  double Gv[PT];
  if (team == 0) {
    double exv[PT], psv[PT], etv[PT], iv[PT];
    gload(exv, q.aux_cur + AUX_EX * nmax, N, tid);
    gload(psv, q.aux_cur + AUX_PHS * nmax, N, tid);
    gload(Gv, q.Gphi, N, tid);
    gload(etv, q.Ys, N, tid);
    if (MAP) gload(iv, q.mesh + mesh_einv(nmax), N, tid);
    pin(exv);
    pin(psv);
    pin(Gv);
    pin(etv);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      double ex = exv[m], ps = psv[m];
      if (MAP) {
        ex *= iv[m];
        ps *= iv[m];
        Gv[m] *= iv[m];
      }
      const double G = Gv[m];
      const double den = 1.0 + ex * ex;
      const double u = (ps - ex * G) / den;
      const double v = (ex * ps + G) / den;
      if (t < N) {
        q.aux_cur[AUX_U * nmax + t] = u;
        q.aux_cur[AUX_V * nmax + t] = v;
        q.aux_cur[AUX_W3 * nmax + t] = den * sqrt(den);
        B[0][t] = cmk(G, v * G - 0.5 * u * u - 0.5 * v * v - q.g * etv[m]);
      }
    }
  } else if (team == 1) {
    if (q.tau != 0.0) {
      double exv[PT], iv[PT];
      gload(exv, q.aux_cur + AUX_EX * nmax, N, tid);
      if (MAP) gload(iv, q.mesh + mesh_einv(nmax), N, tid);
#pragma unroll
      for (int m = 0; m < PT; ++m) {
        const int t = tid + WW_NT * m;
        const double ex = MAP ? exv[m] * iv[m] : exv[m];
        if (t < N) B[1][t] = cmk(q.tau * ex / sqrt(1.0 + ex * ex), 0.0);
      }
    }
  } else {
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      acc[m] = q.yhat[t < N ? t : N - 1];
    }
    for (int j = 0; j < q.s; ++j) {
      const double w = q.w[j];
      const cplx* Kj = reinterpret_cast<const cplx*>(q.K + (size_t)j * q.kstride);
      cplx kv[PT];
#pragma unroll
      for (int m = 0; m < PT; ++m) {
        const int t = tid + WW_NT * m;
        kv[m] = Kj[t < N ? t : N - 1];
      }
#pragma unroll
      for (int m = 0; m < PT; ++m) acc[m] = cmk(fma(w, kv[m].x, acc[m].x), fma(w, kv[m].y, acc[m].y));
    }
    if (tid < 64) lagged_check(q.chk, q.nchk, q.chk_tol, q.status, 32);
  }
  if constexpr (MAP) {
    // the tension term's derivative and the E-weighted mean, in physical space
    if (q.tau != 0.0) {
      FftSz<NF>::run(buf, scr, tws, P, -1, tid, team == 1);
      if (team == 1)
        for (int t = tid; t < N; t += WW_NT) buf[t] = sym_deriv(buf[t], wavenum(t, N), N);
      FftSz<NF>::run(buf, scr, tws, P, +1, tid, team == 1);
    }
    double sum = 0.0, pre[PT];
    if (team == 0) {
      double ew[PT], iv[PT];
      gload(ew, q.mesh + mesh_e(nmax), N, tid);
      gload(iv, q.mesh + mesh_einv(nmax), N, tid);
#pragma unroll
      for (int m = 0; m < PT; ++m) {
        const int t = tid + WW_NT * m;
        pre[m] = 0.0;
        if (t < N) {
          pre[m] = B[0][t].y;
          if (q.tau != 0.0) pre[m] += B[1][t].x * iv[m];
          sum += ew[m] * pre[m];
        }
      }
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_down(sum, off, 64);
      if ((tid & 63) == 0) red[tid >> 6] = sum;
    }
    __syncthreads();
    if (team == 0) {
      const double mean = (((red[0] + red[1]) + red[2]) + red[3]) / (double)N;
#pragma unroll
      for (int m = 0; m < PT; ++m) {
        const int t = tid + WW_NT * m;
        if (t < N) B[0][t].y = pre[m] - mean;
      }
    }
    FftSz<NF>::run(buf, scr, tws, P, -1, tid, team == 0);
  } else {
    FftSz<NF>::run(buf, scr, tws, P, -1, tid, team == 0 || (team == 1 && q.tau != 0.0));
  }
  if (team == 2) {
    const double w = q.w[q.s];
    cplx* Ks = reinterpret_cast<cplx*>(q.K + (size_t)q.s * q.kstride);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) {
        const double sg = q.sig[t];
        const int k = wavenum(t, N);
        cplx ks;
        if (MAP) {
          ks = cscale(B[0][t], sg);
        } else {
          cplx A, C, F = cmk(0.0, 0.0), dummy;
          split_pair(B[0], t, N, A, C);
          if (q.tau != 0.0) split_pair(B[1], t, N, F, dummy);
          const cplx pt = (k == 0) ? cmk(0.0, 0.0) : cscale(cadd(C, sym_deriv(F, k, N)), sg);
          ks = pack_pair(cscale(A, sg), pt);
        }
        Ks[t] = ks;
        cplx Y = cmk(fma(w, ks.x, acc[m].x), fma(w, ks.y, acc[m].y));
        if (q.end) {
          Y = cscale(Y, sg);
          q.yhat[t] = Y;
        }
        Yb[t] = Y;
      }
    }
  }
  __syncthreads();
  // the three spectra: eta + i varphi, eta_x + i eta_xx, varphi' (team 2 replaces Yb by its
  // own after everyone has read it)
  {
    cplx own[PT];
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) {
        if (team == 0) {
          own[m] = Yb[t];
        } else {
          cplx E, F;
          split_pair(Yb, t, N, E, F);
          const int k = wavenum(t, N);
          const cplx d = sym_deriv(team == 1 ? E : F, k, N);
          own[m] = team == 1 ? pack_pair(d, sym_deriv(d, k, N)) : d;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) buf[t] = own[m];
    }
  }
  FftSz<NF>::run(buf, scr, tws, P, +1, tid, true);
  bool bad = false, bed = false;
  for (int t = tid; t < N; t += WW_NT) {
    const cplx z = buf[t];
    if (team == 0) {
      q.Ys[t] = z.x;
      q.Ys[N + t] = z.y;
      q.rhs0[t] = z.y;
      if (q.end) {
        q.y[t] = z.x;
        q.y[N + t] = z.y;
      }
      const double sh = z.x + q.hsurf;
      q.aux_next[AUX_EP * nmax + t] = exp(sh);
      q.aux_next[AUX_EM * nmax + t] = exp(-sh);
      bad |= !isfinite(z.x) || !isfinite(z.y);
      bed |= q.hsurf > 0.0 && sh <= 0.0;
    } else if (team == 1) {
      q.aux_next[AUX_EX * nmax + t] = z.x;
      q.aux_next[AUX_EXX * nmax + t] = z.y;
    } else {
      q.aux_next[AUX_PHS * nmax + t] = z.x;
    }
  }
  for (int i = N + (int)threadIdx.x; i < q.Np; i += STAGE_NT) q.rhs0[i] = 0.0;
  if (q.check && (bad || bed)) flag_state(q.status, bad, bed, q.end ? (done + 1) * 16 : done * 16 + q.s + 1);
  if (q.end && threadIdx.x == 0) q.status[1] = done + 1;
}

// -------------------------------------------------------------------------------------
// Column stage values and Dirichlet data of the variational columns (App. B, (l4)):
//   Ydot_s = ydot + sum_{j<s} a_sj dt kdot_j,  psidot = phidot - phi_y etadot
// Psi column c-1 (ld Np, rows N..Np-1 zero) for state column c = 1..M.
// -------------------------------------------------------------------------------------
__global__ void k_col_pre(const double* __restrict__ y, const double* __restrict__ K, double* __restrict__ Ys,
                          const double* __restrict__ coef, int stage, size_t kstride,
                          const double* __restrict__ aux, int nmax, double* __restrict__ Psi, int Np, int N, int M) {
  const int n2 = 2 * N;
  const size_t tot = (size_t)Np * M;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < tot; idx += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(idx / Np) + 1;
    const int i = (int)(idx - (size_t)(c - 1) * Np);
    if (i >= N) {
      Psi[idx] = 0.0;
      continue;
    }
    const size_t oe = (size_t)c * n2 + i, op = oe + N;
    const double e = stage_combine(y[oe], K, kstride, oe, coef, stage);
    const double p = stage_combine(y[op], K, kstride, op, coef, stage);
    Ys[oe] = e;
    Ys[op] = p;
    Psi[idx] = p - aux[AUX_V * nmax + i] * e;
  }
}

// -------------------------------------------------------------------------------------
// Variational right-hand side, one workgroup per column (App. B (l5a), (l6), (l6a)):
//   etadot_t = G psidot - d(etadot u)
//   phidot_t = P[-d(etadot u v) - u d psidot + v G psidot - g etadot
//               + tau d(d etadot / (1 + eta_x^2)^{3/2})]
// both filtered.  Spectral derivatives: pass 1 gives d psidot and d etadot; pass 2
// transforms the four real signals G psidot, etadot u, (undifferentiated terms of
// phidot_t) and (differentiated terms of phidot_t) and combines them spectrally.
// -------------------------------------------------------------------------------------
// Two teams: the two transforms of pass 2 run side by side.  Dynamic LDS: 5 N complex.
template <int NF>
__global__ __launch_bounds__(PREP_NT) void k_col_rhs(const double* __restrict__ Ys, const double* __restrict__ Gpsi,
                                                     int Np, const double* __restrict__ aux, int nmax,
                                                     double* __restrict__ Kout, const cplx* __restrict__ tw,
                                                     const double* __restrict__ sig, int N, double g, double tau) {
  constexpr int PT = FftSz<NF>::PT;
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* S = lds + 2 * N;
  cplx* X = lds + 3 * N;
  cplx* tws = lds + 4 * N;
  const FftPlan P = make_plan(N);
  const int tid = threadIdx.x & 255, team = threadIdx.x >> 8;
  load_twiddles<(PT + 1) / 2>(tws, tw, N);
  const int c = blockIdx.x + 1;
  const double* ye = Ys + (size_t)c * 2 * N;
  // pass 1: d psidot, d etadot
  double ev[PT], vv[PT];
  gload(ev, ye, N, tid);
  gload(vv, aux + AUX_V * nmax, N, tid);
  if (team == 0) {
    double pv[PT];
    gload(pv, ye + N, N, tid);
    pin(ev);
    pin(pv);
    pin(vv);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tid + WW_NT * m;
      if (t < N) Z[t] = cmk(pv[m] - vv[m] * ev[m], ev[m]);
    }
  }
  double uv[PT], gv[PT], wv[PT];   // in flight during pass 1
  gload(uv, aux + AUX_U * nmax, N, tid);
  gload(gv, Gpsi + (size_t)(c - 1) * Np, N, tid);
  gload(wv, aux + AUX_W3 * nmax, N, tid);
  pin(uv);
  pin(gv);
  pin(wv);
  FftSz<NF>::run(Z, W, tws, P, -1, tid, team == 0);
  for (int t = threadIdx.x; t < N; t += PREP_NT) {
    // i k times the spectrum of psidot + i etadot (both real, the multiplier odd)
    W[t] = sym_deriv(Z[t], wavenum(t, N), N);
  }
  FftSz<NF>::run(W, Z, tws, P, +1, tid, team == 0);
  // pass 2
#pragma unroll
  for (int m = 0; m < PT; ++m) {
    const int t = tid + WW_NT * m;
    if (t < N) {
      const double e = ev[m], u = uv[m], v = vv[m], G = gv[m];
      const double dpsi = W[t].x, deta = W[t].y;
      if (team == 0) Z[t] = cmk(G, e * u);
      else S[t] = cmk(-u * dpsi + v * G - g * e, -e * u * v + tau * deta / wv[m]);
    }
  }
  FftSz<NF>::run(team ? S : Z, team ? X : W, tws, P, -1, tid, true);
  for (int t = threadIdx.x; t < N; t += PREP_NT) {
    cplx A, B, C, F;
    split_pair(Z, t, N, A, B);
    split_pair(S, t, N, C, F);
    const int k = wavenum(t, N);
    const double sg = sig[t];
    cplx et = cscale(csub(A, sym_deriv(B, k, N)), sg);
    cplx pt = (k == 0) ? cmk(0.0, 0.0) : cscale(cadd(C, sym_deriv(F, k, N)), sg);
    W[t] = pack_pair(et, pt);
  }
  FftSz<NF>::run(W, Z, tws, P, +1, tid, team == 0);
  double* ko = Kout + (size_t)c * 2 * N;
  for (int t = threadIdx.x; t < N; t += PREP_NT) {
    ko[t] = W[t].x;
    ko[N + t] = W[t].y;
  }
}

// -------------------------------------------------------------------------------------
// End of step, one workgroup per state column: y <- S_F[y + sum_s b_s dt k_s]
// (the filter is applied to the solution after every step, Sec. 2.2).
// -------------------------------------------------------------------------------------
template <int NF>
__global__ __launch_bounds__(WW_NT) void k_step_end(double* __restrict__ y, const double* __restrict__ K,
                                                    size_t kstride, int nst, const double* __restrict__ coef,
                                                    const cplx* __restrict__ tw, const double* __restrict__ sig,
                                                    int N, int c0, int* __restrict__ status) {
  constexpr int PT = FftSz<NF>::PT;
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* tws = lds + 2 * N;
  const FftPlan P = make_plan(N);
  load_twiddles<PT>(tws, tw, N);
  const int c = c0 + blockIdx.x;
  double* yc = y + (size_t)c * 2 * N;
  const int tid = threadIdx.x;
  {
    double ev[PT], pv[PT];
    stage_combine_vec(ev, y + (size_t)c * 2 * N, K + (size_t)c * 2 * N, kstride, 0, coef + COEF_B, nst, N);
    stage_combine_vec(pv, y + (size_t)c * 2 * N, K + (size_t)c * 2 * N, kstride, N, coef + COEF_B, nst, N);
    pin(ev);
    pin(pv);
#pragma unroll
    for (int m = 0; m < PT; ++m) {
      const int t = tidx(m);
      if (t < N) Z[t] = cmk(ev[m], pv[m]);
    }
  }
  FftSz<NF>::run(Z, W, tws, P, -1, tid, true);
  for (int t = tid; t < N; t += WW_NT) Z[t] = cscale(Z[t], sig[t]);
  FftSz<NF>::run(Z, W, tws, P, +1, tid, true);
  for (int t = tid; t < N; t += WW_NT) {
    yc[t] = Z[t].x;
    yc[N + t] = Z[t].y;
  }
  if (status && c == 0 && tid == 0) status[1] += 1;   // steps completed (with the base column)
}

// status word of a call: bits, step counter, first failing 16 step + stage
__global__ void k_status_reset(int* __restrict__ status) {
  if (threadIdx.x == 0) {
    status[0] = 0;
    status[1] = 0;
    status[2] = 0x7fffffff;
    // status[4..7]: the two maxima of a double-double solve's residual test
    status[4] = status[5] = status[6] = status[7] = 0;
  }
}

// -------------------------------------------------------------------------------------
// Outputs (eq. (f:phi), (Jik), (dfdT)): r = w varphi(T/4), J = w phidot(T/4),
// drdT = w varphi_t(T/4)/4, f = r.r/2, w = 1/sqrt(N).
// -------------------------------------------------------------------------------------
__global__ void k_outputs(const double* __restrict__ y, const double* __restrict__ kT, double* __restrict__ r,
                          double* __restrict__ J, double* __restrict__ drdT, int N, int M) {
  const double w = 1.0 / sqrt((double)N);
  const size_t tot = (size_t)N * (M + 1);
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < tot; idx += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(idx / N);
    const int i = (int)(idx - (size_t)c * N);
    const double v = w * y[(size_t)c * 2 * N + N + i];
    if (c == 0) {
      r[i] = v;
      if (drdT && kT) drdT[i] = 0.25 * w * kT[N + i];
    } else if (J) {
      J[(size_t)(c - 1) * N + i] = v;
    }
  }
}

// f = r.r / 2 and, when d is given, df/dT = r.d (Sec. 3.2 eq. (dfdT) with d = dr/dT)
// into f[1]: one workgroup, FP64 wavefront reductions in a fixed order
__global__ __launch_bounds__(WW_NT) void k_objective(const double* __restrict__ r, int N, double* __restrict__ f,
                                                     const double* __restrict__ d) {
  __shared__ double red[2][WW_NT / 64];
  double s = 0.0, t = 0.0;
  for (int i = threadIdx.x; i < N; i += WW_NT) {
    s += r[i] * r[i];
    if (d) t += r[i] * d[i];
  }
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_down(s, off, 64);
    t += __shfl_down(t, off, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = s;
    red[1][threadIdx.x >> 6] = t;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
    for (int w = 0; w < WW_NT / 64; ++w) {
      a += red[0][w];
      b += red[1][w];
    }
    f[0] = 0.5 * a;
    if (d) f[1] = b;
  }
}

// copy between a dense N x R array (ld N) and a padded Np x R array (ld Np)
__global__ void k_pad_copy(const double* __restrict__ src, int lds_, double* __restrict__ dst, int ldd,
                           int nrows_src, int nrows_dst, int R) {
  const size_t tot = (size_t)nrows_dst * R;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < tot; idx += (size_t)gridDim.x * blockDim.x) {
    const int c = (int)(idx / nrows_dst);
    const int i = (int)(idx - (size_t)c * nrows_dst);
    dst[(size_t)c * ldd + i] = (i < nrows_src) ? src[(size_t)c * lds_ + i] : 0.0;
  }
}

// non-finite scan of the state (failure detection): flag bit 2
__global__ void k_check_finite(const double* __restrict__ y, size_t n, int* __restrict__ status) {
  bool bad = false;
  for (size_t idx = blockIdx.x * (size_t)blockDim.x + threadIdx.x; idx < n; idx += (size_t)gridDim.x * blockDim.x)
    if (!isfinite(y[idx])) bad = true;
  if (bad) atomicOr(status, 2);
}

// =====================================================================================
// Discrete adjoint (Sec. 3.2 and App. B, discrete form): the exact transpose of the
// tangent march above.  For one right-hand-side operator L = S_F DF(Y) of a stage,
//   psidot = phidot - v etadot,  G = (H/2 + Gm) D A^{-1} psidot,
//   etadot_t = G - D(u etadot),
//   phidot_t = P[-D(u v etadot) - u D psidot + v G - g etadot + tau D(w3^{-1} D etadot)],
// the transpose, with D^T = -D, H^T = -H, P^T = P, S_F^T = S_F, is, for adjoint data
// (alpha, beta) of (etadot_t, phidot_t):
//   a = S_F alpha,  b = P S_F beta,  gt = a + v b,
//   psit = A^{-T} D (H gt / 2 - Gm^T gt) + D(u b),
//   etat = u D a + u v D b - g b + tau D(w3^{-1} D b) - v psit,   phit = psit.
// A^{-T} and Gm^T are products with the stored row-major inverse and Gm, transposed.
// =====================================================================================

// adjoint stage, part 1 (one workgroup):  kappa = wb * mu + sum_{i > s} wa_i upsilon_i
// (the stage weights come from coef), then the spectral pieces of the transpose.
// Outputs (ld Np where noted): gt (Np, zero padded), hd = D(H gt / 2), e1, q.
__global__ __launch_bounds__(WW_NT) void k_adj_pre(const double* __restrict__ mu, const double* __restrict__ ups,
                                                   size_t ustride, const double* __restrict__ coef, int stage,
                                                   int nst, const double* __restrict__ saux, const cplx* __restrict__ tw,
                                                   const double* __restrict__ sig, int N, int Np, double g, double tau,
                                                   double* __restrict__ gt, double* __restrict__ hd,
                                                   double* __restrict__ e1, double* __restrict__ q) {
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* S = lds + 2 * N;
  cplx* tws = lds + 3 * N;
  const FftPlan P = make_plan(N);
  load_twiddles(tws, tw, N);
  const int tid = threadIdx.x;
  const double* u = saux;
  const double* v = saux + N;
  const double* w3 = saux + 2 * N;
  // kappa_s = b_s dt mu + sum_{i > s} a_is dt upsilon_i
  const double wb = coef[COEF_B + stage];
  for (int t = tid; t < 2 * N; t += WW_NT) {
    double kv = wb * mu[t];
    for (int i = stage + 1; i < nst; ++i) kv += coef[i * 16 + stage] * ups[(size_t)i * ustride + t];
    if (t < N) Z[t].x = kv;
    else Z[t - N].y = kv;
  }
  fft_lds(Z, W, tws, P, -1);
  for (int t = tid; t < N; t += WW_NT) {
    cplx Al, Be;
    split_pair(Z, t, N, Al, Be);
    const int k = wavenum(t, N);
    const double sg = sig[t];
    cplx a = cscale(Al, sg);
    cplx b = (k == 0) ? cmk(0.0, 0.0) : cscale(Be, sg);
    W[t] = pack_pair(a, b);
    S[t] = pack_pair(sym_deriv(a, k, N), sym_deriv(b, k, N));
  }
  fft_lds(W, Z, tws, P, +1);   // a + i b
  fft_lds(S, Z, tws, P, +1);   // D a + i D b
  // physical: gt = a + v b ; f1 = D b / w3 ; f2 = u b   (kept in registers between passes)
  double av[NPT], bv[NPT], dav[NPT], dbv[NPT];
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    const int t = tclamp(m, N);
    av[m] = W[t].x;
    bv[m] = W[t].y;
    dav[m] = S[t].x;
    dbv[m] = S[t].y;
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    const int t = tidx(m);
    if (t < N) {
      const double gg = av[m] + v[t] * bv[m];
      Z[t] = cmk(gg, dbv[m] / w3[t]);
      S[t] = cmk(u[t] * bv[m], 0.0);
      gt[t] = gg;
    }
  }
  for (int t = N + tid; t < Np; t += WW_NT) gt[t] = 0.0;
  fft_lds(Z, W, tws, P, -1);
  fft_lds(S, W, tws, P, -1);
  {
    // split_pair reads the mirrored bin N - t of S, which another thread (or this
    // thread's next m) would overwrite: read everything first, write after a barrier
    cplx wo[NPT], so[NPT];
#pragma unroll
    for (int m = 0; m < NPT; ++m) {
      const int t = tclamp(m, N);
      cplx Gh, F1, F2, dm;
      split_pair(Z, t, N, Gh, F1);
      split_pair(S, t, N, F2, dm);
      const int k = wavenum(t, N);
      // D(H gt / 2): symbol (i k)(-i sgn k)/2 = |k|/2, zero at Nyquist
      const double hk = (2 * k == N || 2 * k == -N) ? 0.0 : 0.5 * fabs((double)k);
      wo[m] = pack_pair(cscale(Gh, hk), sym_deriv(F1, k, N));
      so[m] = sym_deriv(F2, k, N);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NPT; ++m) {
      const int t = tidx(m);
      if (t < N) {
        W[t] = wo[m];
        S[t] = so[m];
      }
    }
  }
  fft_lds(W, Z, tws, P, +1);   // D(H gt/2) + i D f1
  fft_lds(S, Z, tws, P, +1);   // D f2
#pragma unroll
  for (int m = 0; m < NPT; ++m) {
    const int t = tidx(m);
    if (t < N) {
      const double uu = u[t], vv = v[t];
      hd[t] = W[t].x;
      e1[t] = uu * dav[m] + uu * vv * dbv[m] - g * bv[m] + tau * W[t].y;
      q[t] = S[t].x;
    }
  }
}

// adjoint stage, part 2 (one workgroup): zeta = hd - D(g2), g2 = Gm^T gt (ld Np);
// zeta padded with zeros to Np.
__global__ __launch_bounds__(WW_NT) void k_adj_mid(const double* __restrict__ g2, const double* __restrict__ hd,
                                                   const cplx* __restrict__ tw, int N, int Np,
                                                   double* __restrict__ zeta) {
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* tws = lds + 2 * N;
  const FftPlan P = make_plan(N);
  load_twiddles(tws, tw, N);
  for (int t = threadIdx.x; t < N; t += WW_NT) Z[t] = cmk(g2[t], 0.0);
  fft_lds(Z, W, tws, P, -1);
  for (int t = threadIdx.x; t < N; t += WW_NT) Z[t] = sym_deriv(Z[t], wavenum(t, N), N);
  fft_lds(Z, W, tws, P, +1);
  for (int t = threadIdx.x; t < Np; t += WW_NT) zeta[t] = (t < N) ? hd[t] - Z[t].x : 0.0;
}

// y = M^T x for one vector, M row-major Np x Np: a workgroup forms 16 outputs (128 B of
// every row), each lane a column and every 32nd row from its own, eight loads in flight; the
// partial sums are added in a fixed order (lane groups, then waves).  Bound by the reads of
// M; 16 columns per workgroup keep Np / 16 workgroups on the chip.
#define GTV_NT 512
__global__ __launch_bounds__(GTV_NT) void k_gemv_tr(const double* __restrict__ M, int Np, const double* __restrict__ x,
                                                    double* __restrict__ y) {
  __shared__ double part[GTV_NT / 64][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = blockIdx.x * 16 + (lane & 15);
  const int r0 = w * 4 + (lane >> 4);
  double s0 = 0.0, s1 = 0.0;
  // Np is a multiple of 64: an even number of 32-row steps
  for (int j = r0; j < Np; j += 64) {
    s0 = fma(M[(size_t)j * Np + i], x[j], s0);
    s1 = fma(M[(size_t)(j + 32) * Np + i], x[j + 32], s1);
  }
  double s = s0 + s1;
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  if (lane < 16) part[w][lane] = s;
  __syncthreads();
  if (threadIdx.x < 16) {
    double t = part[0][threadIdx.x];
    for (int q = 1; q < GTV_NT / 64; ++q) t += part[q][threadIdx.x];
    y[i] = t;
  }
}

// adjoint stage, part 3: psit = y + q;  upsilon = (e1 - v psit, psit)
__global__ void k_adj_post(const double* __restrict__ yv, const double* __restrict__ q, const double* __restrict__ e1,
                           const double* __restrict__ saux, int N, double* __restrict__ ups) {
  const double* v = saux + N;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < N; t += gridDim.x * blockDim.x) {
    const double ps = yv[t] + q[t];
    ups[t] = e1[t] - v[t] * ps;
    ups[N + t] = ps;
  }
}

// adjoint of the end of a step: lambda_n = mu + sum_s upsilon_s, then (for the step
// before) mu = S_F lambda.  One workgroup; first = 1 starts from lambda (no upsilon).
__global__ __launch_bounds__(WW_NT) void k_adj_step(double* __restrict__ lam, double* __restrict__ mu,
                                                    const double* __restrict__ ups, size_t ustride, int nst,
                                                    int first, const cplx* __restrict__ tw,
                                                    const double* __restrict__ sig, int N) {
  extern __shared__ cplx lds[];
  cplx* Z = lds;
  cplx* W = lds + N;
  cplx* tws = lds + 2 * N;
  const FftPlan P = make_plan(N);
  load_twiddles(tws, tw, N);
  for (int t = threadIdx.x; t < 2 * N; t += WW_NT) {
    double l = first ? lam[t] : mu[t];
    if (!first)
      for (int s = 0; s < nst; ++s) l += ups[(size_t)s * ustride + t];
    lam[t] = l;
    if (t < N) Z[t].x = l;
    else Z[t - N].y = l;
  }
  fft_lds(Z, W, tws, P, -1);
  for (int t = threadIdx.x; t < N; t += WW_NT) Z[t] = cscale(Z[t], sig[t]);
  fft_lds(Z, W, tws, P, +1);
  for (int t = threadIdx.x; t < N; t += WW_NT) {
    mu[t] = Z[t].x;
    mu[N + t] = Z[t].y;
  }
}

// gradient: grad_k = <basis_k, lambda_0>  (one wave per parameter)
__global__ __launch_bounds__(WW_NT) void k_adj_grad(const double* __restrict__ basis, const double* __restrict__ lam,
                                                    int N, int M, double* __restrict__ grad) {
  const int k = (blockIdx.x * WW_NT + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (k >= M) return;
  const double* bk = basis + (size_t)k * 2 * N;
  double s = 0.0;
  for (int t = lane; t < 2 * N; t += 64) s = fma(bk[t], lam[t], s);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) grad[k] = s;
}

// lambda at T/4: (0, w r)
__global__ void k_adj_seed(const double* __restrict__ r, int N, double* __restrict__ lam) {
  const double w = 1.0 / sqrt((double)N);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < 2 * N; t += gridDim.x * blockDim.x)
    lam[t] = (t < N) ? 0.0 : w * r[t - N];
}

// copy of the stage's u, v, (1 + eta_x^2)^{3/2} for the reverse sweep
__global__ void k_save_aux(const double* __restrict__ aux, int nmax, int N, double* __restrict__ saux) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < N; t += gridDim.x * blockDim.x) {
    saux[t] = aux[AUX_U * nmax + t];
    saux[N + t] = aux[AUX_V * nmax + t];
    saux[2 * N + t] = aux[AUX_W3 * nmax + t];
  }
}

// -------------------------------------------------------------------------------------
// Convergence test of a mixed-precision solve (one workgroup per column): with the
// FP64 residual r = B - A X of the final X, max|r| <= tol * max|B| over the N rows
// (a relative residual, which bounds the normwise backward error); a column that
// fails, or a NaN, sets status bit 4 (reported as WW_EREFINE).
// -------------------------------------------------------------------------------------
template <int NT>
__device__ inline void refine_check_col(const double* __restrict__ rc, const double* __restrict__ bc, int N,
                                        double tol, int* __restrict__ status, int flag, double* red) {
  double *rr = red, *rb = red + NT / 64;   // red: LDS of NT / 32 doubles, free again after the next barrier
  double mr = 0.0, mb = 0.0;
  for (int i = threadIdx.x; i < N; i += NT) {
    mr = fmax(mr, fabs(rc[i]));
    mb = fmax(mb, fabs(bc[i]));
    if (rc[i] != rc[i]) mr = INFINITY;
  }
  for (int off = 32; off > 0; off >>= 1) {
    mr = fmax(mr, __shfl_xor(mr, off));
    mb = fmax(mb, __shfl_xor(mb, off));
  }
  if ((threadIdx.x & 63) == 0) {
    rr[threadIdx.x >> 6] = mr;
    rb[threadIdx.x >> 6] = mb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < NT / 64; ++w) {
      mr = fmax(mr, rr[w]);
      mb = fmax(mb, rb[w]);
    }
    if (!(mr <= tol * mb)) atomicOr(status, flag);
  }
}

__global__ __launch_bounds__(WW_NT) void k_refine_check(const double* __restrict__ r, const double* __restrict__ B,
                                                        int Np, int N, double tol, int* __restrict__ status,
                                                        int flag) {
  __shared__ double red[WW_NT / 32];
  refine_check_col<WW_NT>(r + (size_t)blockIdx.x * Np, B + (size_t)blockIdx.x * Np, N, tol, status, flag, red);
}

// -------------------------------------------------------------------------------------
// Measurement stamp (not part of the method): one thread reads the GPU's constant-rate
// wall clock.  which = 0 keeps the start tick of a slot; which = 1 adds the ticks since
// that start to the slot's running sum and counts the interval.  Slots are
// [start, sum, count]; a slot is only touched by work on one stream, in order.
// -------------------------------------------------------------------------------------
__global__ void k_stamp(unsigned long long* __restrict__ st, int slot, int which) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const unsigned long long t = (unsigned long long)wall_clock64();
  unsigned long long* s = st + 3 * (size_t)slot;
  if (which == 0) {
    s[0] = t;
  } else {
    s[1] += t - s[0];
    s[2] += 1;
  }
}
