// Explicit inverse of the stage matrix A by block Gauss-Jordan elimination (Sec. 3.3:
// one factorisation of I/2 + K per stage), 64 x 64 blocks, no pivoting (A is diagonally
// dominant; a pivot guard reports violations), for one matrix or a group of up to four
// that share every launch.
#pragma once
#include "ww_kernels.hpp"

// -------------------------------------------------------------------------------------
// The method, on a matrix B of nb x nb blocks, step k = 0 .. nb - 1, D_k = B_kk^{-1}:
//   B_ij <- B_ij - (B_ik D_k) B_kj     (i, j != k)
//   B_ik <- -B_ik D_k,   B_kj <- D_k B_kj,   B_kk <- D_k,
// after which B holds the inverse: 2 N^3 flops in nb steps whose tiles are independent,
// nothing left to multiply afterwards.  A step reads one buffer and writes another (the
// panels it reads are overwritten by its own results): the matrix itself, then two
// scratch buffers in turn, the last step the destination.
//
// Orientation: a row-major array is the column-major transpose, and the inverse of the
// transpose is the transpose of the inverse.  The kernels index column-major arrays
// throughout, so a row-major A gives its inverse row-major.
//
// Launch per step (k_gj_step): task 0 of every matrix forms the next diagonal block
//   B_{k+1,k+1} - (B_{k+1,k} D_k) B_{k,k+1}  and inverts it (D_{k+1}: the critical path),
// the other tasks are strips of at most `strip` tiles of one block row: the row's left
// factor once, then each tile.  The chain of nb dependent diagonal inverses bounds the
// sequence up to N = 1024 (the tiles of a step fill the CUs beside it), the matrix units
// and the tile traffic above.
//
// Band layout (what makes a tile product chain without LDS round trips): wave w owns
// rows 16 w .. 16 w + 15 of a tile; lane (cl = lane & 15, rq = lane >> 4) holds in
// x[4 J + i] the entry (16 w + cl, 16 J + Mfma<T>::row(i, rq)).  That is the result
// layout of an MFMA that computes the transposed product, and at the same time its
// second operand's layout: a left factor formed by one product feeds the next from
// registers, column-major tiles load and store 16 consecutive rows per lane group, and
// only the right factors pass through LDS (one barrier per tile, double-buffered).
// -------------------------------------------------------------------------------------
#define GJ_GMAX 4           // matrices of a group
#define GJ_STRIP_MAX 16     // largest blu_strip (a strip task takes at most twice as many tiles)
#define GJ_LD 66            // pitch of a right factor in LDS, stored by columns: conflict-free reads and writes
#define GJ_TILE (64 * GJ_LD)
#define GJ_BLD 18           // pitch of the 16-row bands of the diagonal inverse (16-byte aligned in FP64)
#define GJ_SCR (2 * 64 * GJ_BLD + 2 * 16 * GJ_BLD)
static_assert(GJ_SCR <= GJ_TILE, "the diagonal inverse's scratch must fit in one LDS tile");

template <typename T>
struct GjGroup {
  const T* S0[GJ_GMAX];    // the matrix
  T* W0[GJ_GMAX];          // scratch: results of the even steps
  T* W1[GJ_GMAX];          // ... of the odd steps
  T* Mr[GJ_GMAX];          // the inverse (results of the last step)
  T* Dinv[GJ_GMAX];        // nb x 4096, D_k column-major
  float* Mr32[GJ_GMAX];    // optional FP32 copy of the inverse (null: none)
  int* status;
  double pivguard;
  int Np, count, strip;
};
// one matrix of the group: selects among kernel arguments, field by field (selecting
// through an index would copy the argument block into per-lane scratch memory)
#define GJ_SEL(g, f, m) ((m) == 0 ? g.f[0] : (m) == 1 ? g.f[1] : (m) == 2 ? g.f[2] : g.f[3])

template <typename T>
__device__ __forceinline__ size_t gj_tile(int Np, int i, int j) {
  return (size_t)j * WW_TB * Np + (size_t)i * WW_TB;
}

// column-major 64 x 64 tile (leading dimension ld) <-> band layout.  Every address is a
// wave-uniform pointer (of the entry's column) plus one 32-bit offset per lane, so that
// the sixteen accesses of a lane share one address register.
template <typename T>
__device__ __forceinline__ unsigned band_off(int ld) {
  const int lane = threadIdx.x & 63;
  return (unsigned)(Mfma<T>::rowl(lane >> 4) * ld + (threadIdx.x >> 6) * 16 + (lane & 15));
}
template <typename T>
__device__ __forceinline__ void band_load(T (&x)[16], const T* __restrict__ G, int ld) {
  const unsigned off = band_off<T>(ld);
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[4 * J + i] = (G + (size_t)(16 * J + Mfma<T>::rowc(i)) * ld)[off];
}
template <typename T, typename S>
__device__ __forceinline__ void band_store(const T (&x)[16], S* __restrict__ G, int ld) {
  const unsigned off = band_off<T>(ld);
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int i = 0; i < 4; ++i) (G + (size_t)(16 * J + Mfma<T>::rowc(i)) * ld)[off] = (S)x[4 * J + i];
}
// column-major tile into registers (thread t: entries t + 256 m), then into LDS by columns
template <typename T>
__device__ __forceinline__ void rf_fetch(T (&v)[16], const T* __restrict__ G, int ld) {
  const unsigned off = (unsigned)((threadIdx.x >> 6) * ld + (threadIdx.x & 63));
#pragma unroll
  for (int m = 0; m < 16; ++m) v[m] = (G + (size_t)(4 * m) * ld)[off];
}
template <typename T>
__device__ __forceinline__ void rf_put(T* S, const T (&v)[16]) {
#pragma unroll
  for (int m = 0; m < 16; ++m) S[((threadIdx.x >> 6) + 4 * m) * GJ_LD + (threadIdx.x & 63)] = v[m];
}

// acc += L R for the wave's band: L in band layout (registers), R in LDS by columns
template <typename T>
__device__ __forceinline__ void band_mfma(T (&acc)[16], const T (&l)[16], const T* S) {
  typedef typename Mfma<T>::V V;
  const int lane = threadIdx.x & 63, cl = lane & 15, rq = lane >> 4;
  V v[4];
#pragma unroll
  for (int J = 0; J < 4; ++J) v[J] = V{acc[4 * J], acc[4 * J + 1], acc[4 * J + 2], acc[4 * J + 3]};
#pragma unroll
  for (int Q = 0; Q < 4; ++Q) {
    T a[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int J = 0; J < 4; ++J) a[i][J] = S[(16 * J + cl) * GJ_LD + 16 * Q + Mfma<T>::row(i, rq)];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int J = 0; J < 4; ++J) v[J] = Mfma<T>::step(a[i][J], l[4 * Q + i], v[J]);
  }
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[4 * J + i] = v[J][i];
}

// A tile of a matrix behind a buffer descriptor: with on = false its loads give zero and its
// stores are dropped, without memory traffic and without a branch
typedef unsigned gj_u2 __attribute__((ext_vector_type(2)));
template <typename T>
struct TileBuf {
  __amdgpu_buffer_rsrc_t r;
  int ld;
  __device__ TileBuf(const T* p, int ld_, bool on)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, on ? 64 * ld_ * (int)sizeof(T) : 0, 0x00027000)),
        ld(ld_) {}
  // entry e of this lane's band (band_load), of its share of the columns (rf_fetch)
  __device__ int band_at(int e) const { return (16 * (e >> 2) + Mfma<T>::rowc(e & 3)) * ld * (int)sizeof(T); }
  __device__ int rf_at(int m) const { return 4 * m * ld * (int)sizeof(T); }
  __device__ T get(int voff, int soff) const {
    if constexpr (sizeof(T) == 8) {
      const gj_u2 u = __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0);
      return __builtin_bit_cast(T, u);
    } else {
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
    }
  }
  __device__ void put(T v, int voff, int soff) const {
    if constexpr (sizeof(T) == 8)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(gj_u2, v), r, voff, soff, 0);
    else
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
  }
};

// band_mfma with memory operations in between: bg(s), s = 0 .. 31, after every second matrix
// instruction.  A load holds the wave's issue for about 72 cycles when the four waves send
// theirs together, a matrix instruction occupies its unit for 64: 32 loads in front of the
// product cost 2300 cycles and 16 stores behind it 800 beside its own 4300.  The empty
// asm statements keep that order (matrix instructions have no order of their own).
template <typename T, typename Bg>
__device__ __forceinline__ void band_mfma_bg(T (&acc)[16], const T (&l)[16], const T* S, Bg bg) {
  typedef typename Mfma<T>::V V;
  const int lane = threadIdx.x & 63, cl = lane & 15, rq = lane >> 4;
  V v[4];
#pragma unroll
  for (int J = 0; J < 4; ++J) v[J] = V{acc[4 * J], acc[4 * J + 1], acc[4 * J + 2], acc[4 * J + 3]};
  T a[2][4];
  auto rd = [&](int g) {   // operands of group g = 4 Q + i
#pragma unroll
    for (int J = 0; J < 4; ++J) a[g & 1][J] = S[(16 * J + cl) * GJ_LD + 16 * (g >> 2) + Mfma<T>::row(g & 3, rq)];
  };
  rd(0);
#pragma unroll
  for (int g = 0; g < 16; ++g) {
    if (g < 15) rd(g + 1);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v[2 * h] = Mfma<T>::step(a[g & 1][2 * h], l[g], v[2 * h]);
      v[2 * h + 1] = Mfma<T>::step(a[g & 1][2 * h + 1], l[g], v[2 * h + 1]);
      asm volatile("" : "+v"(v[2 * h]), "+v"(v[2 * h + 1]));
      bg(2 * g + h);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[4 * J + i] = v[J][i];
}

// -------------------------------------------------------------------------------------
// Gauss-Jordan inverse of a 16 x 16 block by one wave, without pivoting, in the MFMA
// result layout (lane: column cl = lane & 15, rows Mfma<T>::row(i, lane >> 4)).  For pivot
// p every entry follows one rule,  a_rc <- a_rc - kap_r rho_c,
//   rho_c = a_pc / a_pp (c != p),  rho_p = 1 + 1/a_pp,
//   kap_r = a_rp (r != p),         kap_p = a_pp - 1,
// which yields A_QQ - a_Qp a_pQ / a_pp, a_pQ / a_pp, -a_Qp / a_pp and 1/a_pp on the four
// parts.  The chain of pivots bounds it: the entries of the next pivot's row are updated
// first, carried to the other three lane groups by lane swaps (no LDS), and its pivot,
// reciprocal (hardware estimate, one third-order correction) and row factors follow while
// the other rows are updated.
// -------------------------------------------------------------------------------------
__device__ __forceinline__ double recip(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  const float e = fmaf(-x, r, 1.0f);
  return fmaf(r, e, r);
}
// value of lane n of the wave (a scalar)
__device__ __forceinline__ double lane_read(double x, int n) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, n);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), n);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float lane_read(float x, int n) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), n));
}
// lane group g (16 lanes) of v copied to all four groups; a4 = 4 (lane & 15)
__device__ __forceinline__ double grp_bcast(double v, int g, int a4) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(a4 + 64 * g, (int)(unsigned)u);
  const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute(a4 + 64 * g, (int)(unsigned)(u >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float grp_bcast(float v, int g, int a4) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(a4 + 64 * g, __float_as_int(v)));
}
// pivot P: prow is the lane's entry of row P, piv the pivot, ip its reciprocal; then those
// of P + 1.  bg(P) issues work of the caller that does not depend on the block.
template <int P, typename T, typename Bg>
__device__ __forceinline__ void leaf_pivot(typename Mfma<T>::V& x, T prow, T piv, T ip, T& minpiv, int lane, int a4,
                                           Bg& bg) {
  constexpr int E = Mfma<T>::row_elem(P), G = Mfma<T>::row_grp(P);
  minpiv = fmin(minpiv, fabs(piv));
  // rho_p = (a_pp + 1) / a_pp: the row's entry plus 1 in the pivot's lane
  const T nrho = -((prow + ((lane & 15) == P ? T(1) : T(0))) * ip);
  T kap[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) kap[i] = row_bcast(x[i], P);
  kap[E] -= (lane >> 4) == G ? T(1) : T(0);
  if constexpr (P < 15) {
    constexpr int E1 = Mfma<T>::row_elem(P + 1), G1 = Mfma<T>::row_grp(P + 1);
    x[E1] = fma(kap[E1], nrho, x[E1]);
    prow = grp_bcast(x[E1], G1, a4);
    piv = lane_read(x[E1], 16 * G1 + P + 1);
    bg(P);
    ip = recip(piv);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i != E1) x[i] = fma(kap[i], nrho, x[i]);
    leaf_pivot<P + 1, T>(x, prow, piv, ip, minpiv, lane, a4, bg);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = fma(kap[i], nrho, x[i]);
  }
}
template <typename T, typename Bg>
__device__ __forceinline__ void leaf_gj16(typename Mfma<T>::V& x, T& minpiv, Bg bg) {
  // the lane number is opaque to the compiler here: it would otherwise keep the sixteen
  // lane masks of the pivots in registers over the block loop
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int a4 = 4 * (lane & 15);
  const T prow = grp_bcast(x[0], 0, a4);   // row 0: element 0 of lane group 0
  const T piv = lane_read(x[0], 0);
  leaf_pivot<0, T>(x, prow, piv, recip(piv), minpiv, lane, a4, bg);
}

// -------------------------------------------------------------------------------------
// In-place inverse of a 64 x 64 tile in band layout (wave w: rows 16 w ..): Gauss-Jordan
// over 16 x 16 blocks.  Step P: wave P inverts its diagonal block (D) and publishes D and
// its band; after the one barrier of the step wave P replaces its blocks by D B_PJ, every
// other wave forms L = B_wP D and updates B_wJ <- B_wJ - L B_PJ, B_wP <- -L.  The chain of
// the four diagonal blocks is the critical path: every wave updates the next pivot's
// column block first, and wave P + 1 issues its remaining products between the pivots of
// its own block.  The blocks rotate through the registers (v[q] holds column block
// (P + q) mod 4), so that the loop over P stays rolled: one copy of the code, which
// matters because a cold instruction cache costs more than the rotation.  The pivots are
// those of the scalar elimination.  scr: GJ_SCR elements of LDS.  Every wave returns the
// smallest |pivot| of the block it inverted.
// Measured (clock stamps, FP64, one workgroup): 9.3 us with the leaf's rows carried by lane
// swaps and the products after the barrier, 8.0 us with LDS permutes, and with the
// deferred products as here 8.0 us (the FP64 matrix instructions and the vector FP64 operations of
// the leaf take turns, so hiding one behind the other gains little).
// -------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T gj64(T (&x)[16], T* scr) {
  typedef typename Mfma<T>::V V;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int cl = lane & 15, rq = lane >> 4;
  const V zero = V{T(0), T(0), T(0), T(0)};
  V v[4];
#pragma unroll
  for (int J = 0; J < 4; ++J) v[J] = V{x[4 * J], x[4 * J + 1], x[4 * J + 2], x[4 * J + 3]};
  T minpiv = T(1e30);
  T a[3][4] = {}, d[4] = {};   // (none pending before the first block)
#pragma unroll 1
  for (int P = 0; P < 4; ++P) {
    // band P and D by columns, the rows of a column in the order in which a lane reads
    // them: row(i, rq) at 4 rq + i, so that its four operands are two 16-byte reads
    T* pub = scr + (P & 1) * 64 * GJ_BLD;
    T* dt = scr + 2 * 64 * GJ_BLD + (P & 1) * 16 * GJ_BLD;
    if (w == P) {
      V y = v[0];
      // the transposed block (the band layout) in registers; the products that wave P
      // deferred in the step before: blocks P + 1 and P + 2
      leaf_gj16<T>(y, minpiv, [&](int p) {
        if (p < 8) v[1 + (p & 1)] = Mfma<T>::step(a[1 + (p & 1)][p >> 1], d[p >> 1], v[1 + (p & 1)]);
      });
      const int pc = 4 * Mfma<T>::row_grp(cl) + Mfma<T>::row_elem(cl);   // place of row cl
#pragma unroll
      for (int i = 0; i < 4; ++i) dt[Mfma<T>::row(i, rq) * GJ_BLD + pc] = y[i];
#pragma unroll
      for (int q = 1; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) pub[(16 * ((P + q) & 3) + Mfma<T>::row(i, rq)) * GJ_BLD + pc] = v[q][i];
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = y[i];   // D[cl][k]
    }
    __syncthreads();
    T dn[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) dn[i] = dt[cl * GJ_BLD + 4 * rq + i];
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) a[q][i] = pub[(16 * ((P + 1 + q) & 3) + cl) * GJ_BLD + 4 * rq + i];
    if (w == P) {
#pragma unroll
      for (int q = 1; q < 4; ++q) v[q] = zero;
    } else {
      // L = B_wP D, transposed product: the result layout is the operand layout below
      V l0 = zero, l1 = zero;   // two chains
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        l0 = Mfma<T>::step(dn[i], v[0][i], l0);
        l1 = Mfma<T>::step(dn[i + 1], v[0][i + 1], l1);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = -(l0[i] + l1[i]);
    }
    {
      V u = zero;
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        v[1] = Mfma<T>::step(a[0][i], d[i], v[1]);
        u = Mfma<T>::step(a[0][i + 1], d[i + 1], u);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) v[1][i] += u[i];
    }
    if (w != P + 1) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 1; q < 3; ++q) v[1 + q] = Mfma<T>::step(a[q][i], d[i], v[1 + q]);
    }
    v[0] = v[1];
    v[1] = v[2];
    v[2] = v[3];
    v[3] = V{d[0], d[1], d[2], d[3]};   // column block P
  }
#pragma unroll
  for (int J = 0; J < 4; ++J)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[4 * J + i] = v[J][i];
  return minpiv;
}

// The pivot guard of an inverted diagonal block (status bit 1), x: an entry of the inverse.
// A NaN pivot passes the minimum unseen, but leaves no finite entry in its block's inverse
// (bit 128): the matrix is not finite, unless a small pivot did that, which read_status
// decides (a pivot of zero leaves NaN behind too, for the redo with row interchanges to
// mend).  FP64 only: entries beyond FP32's range fail the refinement test of the mixed
// form, which is redone in FP64.
template <typename T>
__device__ __forceinline__ void gj_guard(T minpiv, T x, double guard, int* __restrict__ status) {
  if ((threadIdx.x & 63) == 0 && !((double)minpiv >= guard)) atomicOr(status, 1);
  if (sizeof(T) == 8 && !isfinite(x)) atomicOr(status, 128);
}

// D_0 (and, for a single block, the inverse itself)
template <typename T>
__global__ __launch_bounds__(WW_NT) void k_gj_init(GjGroup<T> g) {
  __shared__ __attribute__((aligned(16))) T scr[GJ_SCR];
  const int m = blockIdx.x;
  T x[16];
  band_load<T>(x, GJ_SEL(g, S0, m), g.Np);
  const T mp = gj64<T>(x, scr);
  gj_guard<T>(mp, x[0], g.pivguard, g.status);
  band_store<T, T>(x, GJ_SEL(g, Dinv, m), 64);
  if (g.Np == WW_TB) {
    band_store<T, T>(x, GJ_SEL(g, Mr, m), g.Np);
    float* m32 = GJ_SEL(g, Mr32, m);
    if (m32) band_store<T, float>(x, m32, g.Np);
  }
}

// tasks of step k, per matrix
__host__ __device__ inline int gj_step_tasks(int nb, int k, int strip) {
  return nb * ((nb + strip - 1) / strip) + (k + 1 < nb ? 1 : 0);
}

// Measured per step (FP64, alone on the device), with the memory operations of a tile between
// its matrix instructions against in front of and behind them: N 1024, one matrix 15.0 us
// (15.6), two 16.2 (18.0), four 21.4 (26.1); N 2048 20.8 (25.6); a strip's tile 2.2 us (3.4;
// its matrix instructions 1.7).  Below that the critical task is the step: 13.8 us at N = 512
// (14.3), 8 of them gj64 and 3.5 its two products.
template <typename T>
__global__ __launch_bounds__(WW_NT, 2) void k_gj_step(GjGroup<T> g, int k) {
  extern __shared__ __attribute__((aligned(16))) double sm_raw[];
  T* const sm = reinterpret_cast<T*>(sm_raw);   // two right-factor tiles
  const int Np = g.Np, nb = Np / WW_TB, nstr = (nb + g.strip - 1) / g.strip;
  const bool last = k + 1 == nb;
  // block / count: the critical tasks (the next diagonal block of every matrix) come first
  const int m = blockIdx.x % g.count;
  int q = blockIdx.x / g.count;
  const T* src = k == 0 ? GJ_SEL(g, S0, m) : (k & 1) ? GJ_SEL(g, W0, m) : GJ_SEL(g, W1, m);
  T* dst = last ? GJ_SEL(g, Mr, m) : (k & 1) ? GJ_SEL(g, W1, m) : GJ_SEL(g, W0, m);
  T* Dinv = GJ_SEL(g, Dinv, m);
  const T* Dk = Dinv + (size_t)k * 4096;
  // this lane's byte offsets in a tile: its band, its share of the columns
  const int bdo = (int)(band_off<T>(Np) * sizeof(T));
  const int rfo = (int)(((threadIdx.x >> 6) * Np + (threadIdx.x & 63)) * sizeof(T));
  if (!last) {
    if (q == 0) {
      T l[16], c[16], vd[16], vr[16];
      rf_fetch<T>(vd, Dk, 64);
      band_load<T>(l, src + gj_tile<T>(Np, k + 1, k), Np);
      const TileBuf<T> tr(src + gj_tile<T>(Np, k, k + 1), Np, true), tc(src + gj_tile<T>(Np, k + 1, k + 1), Np, true);
      rf_put<T>(sm, vd);
      __syncthreads();
      T a[16] = {};
      band_mfma_bg<T>(a, l, sm, [&](int s) {   // L = B_{k+1,k} D_k
        if (s < 16) vr[s] = tr.get(rfo, tr.rf_at(s));
        else c[s - 16] = tc.get(bdo, tc.band_at(s - 16));
      });
#pragma unroll
      for (int e = 0; e < 16; ++e) a[e] = -a[e];
      rf_put<T>(sm + GJ_TILE, vr);
      __syncthreads();
      band_mfma<T>(c, a, sm + GJ_TILE);
      // (the inverse's scratch is the first tile, which every wave has left before the barrier above)
      const T mp = gj64<T>(c, sm);
      gj_guard<T>(mp, c[0], g.pivguard, g.status);
      band_store<T, T>(c, Dinv + (size_t)(k + 1) * 4096, 64);
      return;
    }
    q -= 1;
  }
  const int i = q / nstr, p0 = (q - i * nstr) * g.strip, p1 = min(nb, p0 + g.strip);
  float* m32 = last ? GJ_SEL(g, Mr32, m) : nullptr;
  // the next tile of the strip that needs a product (nb: none); the tile that the
  // critical task inverts is not stored
  auto next = [&](int j) {
    while (j < p1 && (j == k || (j == k + 1 && i == k + 1))) ++j;
    return j;
  };
  // the tiles j of row k and of row i (which row k's own strips do not take: zero)
  T l[16], vr[16], cn[16];
  auto rowk = [&](int j) { return TileBuf<T>(src + gj_tile<T>(Np, k, min(j, nb - 1)), Np, j < p1); };
  auto rowi = [&](int j) { return TileBuf<T>(src + gj_tile<T>(Np, i, min(j, nb - 1)), Np, j < p1 && i != k); };
  int j = next(p0);
  {
    const TileBuf<T> tr = rowk(j), tc = rowi(j);
    auto fetch = [&](int s) {
      if (s < 16) vr[s] = tr.get(rfo, tr.rf_at(s));
      else cn[s - 16] = tc.get(bdo, tc.band_at(s - 16));
    };
    if (i == k) {
      band_load<T>(l, Dk, 64);
#pragma unroll
      for (int s = 0; s < 32; ++s) fetch(s);
    } else {
      T b[16], vd[16];
      rf_fetch<T>(vd, Dk, 64);
      band_load<T>(b, src + gj_tile<T>(Np, i, k), Np);
      rf_put<T>(sm, vd);
      __syncthreads();
#pragma unroll
      for (int e = 0; e < 16; ++e) l[e] = T(0);
      band_mfma_bg<T>(l, b, sm, fetch);
#pragma unroll
      for (int e = 0; e < 16; ++e) l[e] = -l[e];
    }
  }
  if (p0 <= k && k < p1) {   // column k: -B_ik D_k, and D_k itself
    band_store<T, T>(l, dst + gj_tile<T>(Np, i, k), Np);
    if (m32) band_store<T, float>(l, m32 + gj_tile<T>(Np, i, k), Np);
  }
  // per tile: the next tile's loads and the stores of the tile before ride in its product
  T c[16], cs[16];
  int js = p1;   // tile of cs (p1: none)
  for (int buf = 1; j < p1; buf ^= 1) {
    T* S = sm + buf * GJ_TILE;
    rf_put<T>(S, vr);
#pragma unroll
    for (int e = 0; e < 16; ++e) c[e] = cn[e];
    __syncthreads();   // the tile is complete; every wave is done with the product before
    const int jn = next(j + 1);
    const TileBuf<T> tr = rowk(jn), tc = rowi(jn), ts(dst + gj_tile<T>(Np, i, min(js, nb - 1)), Np, js < p1);
    band_mfma_bg<T>(c, l, S, [&](int s) {
      if (s < 16) vr[s] = tr.get(rfo, tr.rf_at(s));
      else cn[s - 16] = tc.get(bdo, tc.band_at(s - 16));
      if (s % 2 == 0) ts.put(cs[s / 2], bdo, ts.band_at(s / 2));
    });
    if (m32) band_store<T, float>(c, m32 + gj_tile<T>(Np, i, j), Np);
#pragma unroll
    for (int e = 0; e < 16; ++e) cs[e] = c[e];
    js = j;
    j = jn;
  }
  if (js < p1) band_store<T, T>(cs, dst + gj_tile<T>(Np, i, js), Np);
}
