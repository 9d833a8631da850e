// Pieces of the 4D hop shared by the stencil kernels: spin projection and
// reconstruction, the colour product, register fences and the workgroup's
// place in the traversal.
#pragma once

#include "dev_common.h"
#include "kernels.h"

namespace mdwf {

// ---------------------------------------------------------------------------
// spin projection.  h = spins 0,1 of (1 + SIG g_mu) psi; with w = U h the
// spins 2,3 of the result follow from w (chiral DeGrand-Rossi basis):
//   x: r2 = -SIG i w1, r3 = -SIG i w0     y: r2 =  SIG w1, r3 = -SIG w0
//   z: r2 = -SIG i w0, r3 =  SIG i w1     t: r2 =  SIG w0, r3 =  SIG w1
// ---------------------------------------------------------------------------
template <class R> __device__ __forceinline__ Cplx<R> add(Cplx<R> a, Cplx<R> b) { return {a.re + b.re, a.im + b.im}; }
template <class R> __device__ __forceinline__ Cplx<R> sub(Cplx<R> a, Cplx<R> b) { return {a.re - b.re, a.im - b.im}; }
// a + sg * i * b
template <class R> __device__ __forceinline__ Cplx<R> addi(Cplx<R> a, Cplx<R> b, int sg) {
  return sg > 0 ? Cplx<R>{a.re - b.im, a.im + b.re} : Cplx<R>{a.re + b.im, a.im - b.re};
}

// the same operations on packed 16-bit (re, im) pairs, each result rounded
// once to the storage format
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x2 add(f16x2 a, f16x2 b) { return a + b; }
__device__ __forceinline__ f16x2 sub(f16x2 a, f16x2 b) { return a - b; }
__device__ __forceinline__ f16x2 addi(f16x2 a, f16x2 b, int sg) {
  return sg > 0 ? a + f16x2{-b.y, b.x} : a + f16x2{b.y, -b.x};
}
__device__ __forceinline__ bf16x2 add(bf16x2 a, bf16x2 b) { return a + b; }
__device__ __forceinline__ bf16x2 sub(bf16x2 a, bf16x2 b) { return a - b; }
__device__ __forceinline__ bf16x2 addi(bf16x2 a, bf16x2 b, int sg) {
  return sg > 0 ? a + bf16x2{-b.y, b.x} : a + bf16x2{b.y, -b.x};
}

template <int MU, int SIG, class C>
__device__ __forceinline__ void project(const C p[4][3], C h[2][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if constexpr (MU == 0) {  // g_x psi = (i p3, i p2, -i p1, -i p0)
      h[0][c] = addi(p[0][c], p[3][c], SIG);
      h[1][c] = addi(p[1][c], p[2][c], SIG);
    } else if constexpr (MU == 1) {  // g_y psi = (-p3, p2, p1, -p0)
      h[0][c] = SIG > 0 ? sub(p[0][c], p[3][c]) : add(p[0][c], p[3][c]);
      h[1][c] = SIG > 0 ? add(p[1][c], p[2][c]) : sub(p[1][c], p[2][c]);
    } else if constexpr (MU == 2) {  // g_z psi = (i p2, -i p3, -i p0, i p1)
      h[0][c] = addi(p[0][c], p[2][c], SIG);
      h[1][c] = addi(p[1][c], p[3][c], -SIG);
    } else {  // g_t psi = (p2, p3, p0, p1)
      h[0][c] = SIG > 0 ? add(p[0][c], p[2][c]) : sub(p[0][c], p[2][c]);
      h[1][c] = SIG > 0 ? add(p[1][c], p[3][c]) : sub(p[1][c], p[3][c]);
    }
  }
}

template <int MU, int SIG, class R>
__device__ __forceinline__ void accumulate(Cplx<R> acc[4][3], const Cplx<R> w[2][3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    acc[0][c] = add(acc[0][c], w[0][c]);
    acc[1][c] = add(acc[1][c], w[1][c]);
    if constexpr (MU == 0) {
      acc[2][c] = addi(acc[2][c], w[1][c], -SIG);
      acc[3][c] = addi(acc[3][c], w[0][c], -SIG);
    } else if constexpr (MU == 1) {
      acc[2][c] = SIG > 0 ? add(acc[2][c], w[1][c]) : sub(acc[2][c], w[1][c]);
      acc[3][c] = SIG > 0 ? sub(acc[3][c], w[0][c]) : add(acc[3][c], w[0][c]);
    } else if constexpr (MU == 2) {
      acc[2][c] = addi(acc[2][c], w[0][c], -SIG);
      acc[3][c] = addi(acc[3][c], w[1][c], SIG);
    } else {
      acc[2][c] = SIG > 0 ? add(acc[2][c], w[0][c]) : sub(acc[2][c], w[0][c]);
      acc[3][c] = SIG > 0 ? add(acc[3][c], w[1][c]) : sub(acc[3][c], w[1][c]);
    }
  }
}

__device__ __forceinline__ float fma_r(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_r(double a, double b, double c) { return fma(a, b, c); }

// acc += sc * (spin reconstruction of w): the accumulate above with the
// neighbour's per-site scale applied in the sum
template <int MU, int SIG, class R>
__device__ __forceinline__ void accumulate_scaled(Cplx<R> acc[4][3], const Cplx<R> w[2][3], R sc) {
  const R ps = SIG > 0 ? sc : -sc;  // +SIG*sc
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    acc[0][c] = {fma_r(sc, w[0][c].re, acc[0][c].re), fma_r(sc, w[0][c].im, acc[0][c].im)};
    acc[1][c] = {fma_r(sc, w[1][c].re, acc[1][c].re), fma_r(sc, w[1][c].im, acc[1][c].im)};
    if constexpr (MU == 0) {  // acc2 += -SIG i w1, acc3 += -SIG i w0
      acc[2][c] = {fma_r(ps, w[1][c].im, acc[2][c].re), fma_r(-ps, w[1][c].re, acc[2][c].im)};
      acc[3][c] = {fma_r(ps, w[0][c].im, acc[3][c].re), fma_r(-ps, w[0][c].re, acc[3][c].im)};
    } else if constexpr (MU == 1) {  // acc2 += SIG w1, acc3 -= SIG w0
      acc[2][c] = {fma_r(ps, w[1][c].re, acc[2][c].re), fma_r(ps, w[1][c].im, acc[2][c].im)};
      acc[3][c] = {fma_r(-ps, w[0][c].re, acc[3][c].re), fma_r(-ps, w[0][c].im, acc[3][c].im)};
    } else if constexpr (MU == 2) {  // acc2 += -SIG i w0, acc3 += SIG i w1
      acc[2][c] = {fma_r(ps, w[0][c].im, acc[2][c].re), fma_r(-ps, w[0][c].re, acc[2][c].im)};
      acc[3][c] = {fma_r(-ps, w[1][c].im, acc[3][c].re), fma_r(ps, w[1][c].re, acc[3][c].im)};
    } else {  // acc2 += SIG w0, acc3 += SIG w1
      acc[2][c] = {fma_r(ps, w[0][c].re, acc[2][c].re), fma_r(ps, w[0][c].im, acc[2][c].im)};
      acc[3][c] = {fma_r(ps, w[1][c].re, acc[3][c].re), fma_r(ps, w[1][c].im, acc[3][c].im)};
    }
  }
}

// w = U h (fwd) or U^dag h (bwd), two colour vectors.  Each row is one
// multiply-add chain per real and imaginary part (4 FMAs per complex product
// after the first), not products rounded and then added.
template <bool ADJ, class R>
__device__ __forceinline__ void colour_mul(const Cplx<R> U[3][3], const Cplx<R> h[2][3], Cplx<R> w[2][3]) {
#pragma unroll
  for (int k = 0; k < 2; ++k) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      R re = 0, im = 0;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Cplx<R> u = ADJ ? U[b][a] : U[a][b];
        const Cplx<R> x = h[k][b];
        if (b == 0) {
          re = u.re * x.re;
          im = u.re * x.im;
        } else {
          re = u.re * x.re + re;
          im = u.re * x.im + im;
        }
        if constexpr (ADJ) {  // conj(u) x
          re = u.im * x.im + re;
          im = im - u.im * x.re;
        } else {
          re = re - u.im * x.im;
          im = u.im * x.re + im;
        }
      }
      w[k][a] = {re, im};
    }
  }
}

// ---------------------------------------------------------------------------
// Packed 16-bit hop (F16 and BF16 storage).  A neighbour's 12 complex numbers
// stay in their stored (re, im) 16-bit pairs; the spin projection is formed on
// the pairs (its sum rounded once to the storage format) and the colour
// product uses dot2 instructions, whose 16 x 16-bit products are exact in FP32
// and are summed in FP32.  The neighbour's per-site scale enters in the FP32
// accumulation.  The staged link of a direction is V = U (forward) or U^dag
// (backward), with the antiperiodic sign, as two pairs per entry:
// (Re V, -Im V) and (Im V, Re V), so Re(V h) and Im(V h) are plain dot2 sums.
// ---------------------------------------------------------------------------

template <int P> struct Packed {
  static constexpr bool enabled = false;
};
template <> struct Packed<F16> {
  static constexpr bool enabled = true;
  using T2 = f16x2;
  static __device__ __forceinline__ float dot(T2 a, T2 b, float c) { return __builtin_amdgcn_fdot2(a, b, c, false); }
  // the first product of a chain: the three-operand form with a zero addend
  // (the builtin becomes a register clear plus the accumulating form)
  static __device__ __forceinline__ float dot0(T2 a, T2 b) {
    float r;
    asm("v_dot2_f32_f16 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
    return r;
  }
  static __device__ __forceinline__ T2 make(float re, float im) { return T2{(_Float16)re, (_Float16)im}; }
};
template <> struct Packed<BF16> {
  static constexpr bool enabled = true;
  using T2 = bf16x2;
  static __device__ __forceinline__ float dot(T2 a, T2 b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(a, b, c, false);
  }
  static __device__ __forceinline__ float dot0(T2 a, T2 b) {
    float r;
    asm("v_dot2_f32_bf16 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
    return r;
  }
  static __device__ __forceinline__ T2 make(float re, float im) { return T2{(__bf16)re, (__bf16)im}; }
};

// Compiler fence that also pins the accumulator: the arithmetic of one
// direction must be finished before the next direction's loads are issued,
// so at most one neighbour's spinor and link are live in registers.
template <class R>
__device__ __forceinline__ void pin_acc(Cplx<R> acc[4][3]) {
#pragma unroll
  for (int a = 0; a < 4; ++a)
    asm volatile("" : "+v"(acc[a][0].re), "+v"(acc[a][0].im), "+v"(acc[a][1].re), "+v"(acc[a][1].im),
                 "+v"(acc[a][2].re), "+v"(acc[a][2].im) : : "memory");
}

// Compiler fence after a batch's loads: every loaded register passes through
// an empty asm, so no load of the batch can sink below it and no arithmetic
// of the batch can rise above it.
template <class T, int N> __device__ __forceinline__ void pin_regs(T (&v)[N]) {
#pragma unroll
  for (int k = 0; k + 3 < N; k += 4) asm volatile("" : "+v"(v[k]), "+v"(v[k + 1]), "+v"(v[k + 2]), "+v"(v[k + 3]) : : "memory");
  if constexpr (N % 4 != 0) {
#pragma unroll
    for (int k = N - N % 4; k < N; ++k) asm volatile("" : "+v"(v[k]) : : "memory");
  }
}

// First site of workgroup q.  order_bt = 0: consecutive workgroups take
// consecutive ranges of cb (t is the slowest index, so a site's t-neighbours
// are a whole time slice away in the access stream).  order_bt = Bt > 0 (Bt
// divides Lt): the lattice is cut into order_yb bands of Ly/order_yb y-rows
// (the band's xy-rectangle holds a whole number of workgroups); inside a band
// the (z, t) rectangles are visited in blocks of Bt time slices, z inside a
// block, t fastest.  The z- and t-neighbour rectangles of a rectangle are then
// at most Bt rectangles away in the access stream, and a narrower band keeps
// that distance (in bytes) inside the XCD's L2.  Sites inside a rectangle stay
// consecutive (same reduction tiles).
__device__ __forceinline__ int block_first_site(const DslashArgs& A, int q, int CB) {
  if (A.order_bt <= 0) return q * CB;
  const Geom& g = A.g;
  const int rows = A.rows, bpp = A.bpp;  // y-rows of a band, workgroups per rectangle
  int r = div_by(q, bpp, A.m_bpp);
  const int k = q - r * bpp;
  const int r1 = div_by(r, A.order_bt, A.m_bt);
  const int tt = r - r1 * A.order_bt;
  const int r2 = div_by(r1, g.Lz, A.m_lz);
  const int z = r1 - r2 * g.Lz;
  const int ntb = A.ntb;
  const int yb = div_by(r2, ntb, A.m_ntb);
  const int t = (r2 - yb * ntb) * A.order_bt + tt;
  return ((t * g.Lz + z) * g.Ly + yb * rows) * g.Lxh + k * CB;
}

// What a workgroup reads of its right-hand side's tables and CG state, loaded
// together at the start of the kernel: there the loads are scalar and overlap
// the link stage; behind the first barrier each would be a vector load and one
// more memory latency in the chain (about a microsecond of the 7-17 us a launch
// takes on a small lattice).
struct SlotIO {
  char *in, *aux, *out, *r, *x, *p, *p2;
  double alpha, alpha_prev;
  int active, phase;
};
// AUX: the launch may have an aux field; R, X: it may update r, x
template <bool AUX, bool R, bool X> __device__ __forceinline__ SlotIO slot_io(const DslashArgs& A, int slot) {
  char *in = A.in[slot], *out = nullptr, *aux = nullptr, *r = nullptr, *x = nullptr, *p = nullptr, *p2 = nullptr;
  double alpha = 0, alpha_prev = 0;
  int active = 1, phase = 0;
  if (A.active != nullptr) active = A.active[(size_t)slot * A.active_stride];
  if (!R) out = A.out[slot];
  if (AUX) aux = A.aux[slot];
  if (AUX && !R && A.cg_update == 4) {  // aux is p, which alternates
    p2 = A.cg_p2[slot];
    phase = A.cg_st[slot].phase;
  }
  if (R || (X && A.cg_update == 3)) {
    phase = A.cg_st[slot].phase;
    alpha = A.cg_st[slot].alpha;
    alpha_prev = A.cg_st[slot].alpha_prev;
  }
  if (R) r = A.cg_r[slot];
  if (X && (A.cg_update == 1 || A.cg_update == 3)) {
    x = A.cg_x[slot];
    p = A.cg_p[slot];
    p2 = A.cg_p2[slot];
  }
  if (AUX && !R && phase != 0) aux = p2;
  return SlotIO{in, aux, out, r, x, p, p2, alpha, alpha_prev, active, phase};
}

// (RHS slot, site block) of logical workgroup lb in the launch's RHS order.
// The XCD remap hands XCD k the logical range [k, k + 1) * gridDim.x / 8, so
// order 2 keeps one eighth of the site blocks on each XCD and walks its RHS
// one after another there: one RHS's neighbour planes at a time in that L2.
__device__ __forceinline__ void block_slot(const DslashArgs& A, int lb, int& slot, int& blk) {
  if (A.rhs_order == 1) {
    slot = div_by(lb, A.nblk, A.m_nblk);
    blk = lb - slot * A.nblk;
  } else if (A.rhs_order == 2) {
    // nblk % 8 == 0, so the grid holds exactly nslots * nblk workgroups and
    // blockIdx.x is (place in the XCD's range) * 8 + XCD
    const int per = A.nblk >> 3;  // site blocks per XCD
    const int k = blockIdx.x & 7, j = blockIdx.x >> 3;
    slot = div_by(j, per, A.m_per);
    blk = k * per + (j - slot * per);
  } else {
    blk = div_by(lb, A.nslots, A.m_nslots);
    slot = lb - blk * A.nslots;
  }
}

}  // namespace mdwf
