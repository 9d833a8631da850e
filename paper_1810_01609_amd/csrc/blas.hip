// Fused BLAS-1 updates and deterministic FP64 reductions of the CG solver.
//
// The paper ("Performance Measurement Method", Linear Solver Performance)
// counts 50-100 flops per site for these operations, i.e. they are purely
// bandwidth bound, and does every reduction in double precision.  Here each
// thread owns one site of one slice, the updates are fused so each vector is
// read and written once, and every reduction accumulates in FP64 with a
// fixed summation tree (DPP moves within each 16-lane row, shuffles across
// the four rows of a wavefront, then LDS across wavefronts, then one
// workgroup per right-hand side over the block partials), so results are
// bitwise reproducible.
#include "dev_common.h"
#include "kernels.h"

namespace mdwf {

// Sum over a 256-thread block in a fixed order; valid in thread 0.
__device__ __forceinline__ double block_sum_256(double v) {
  __shared__ double red[kBlasThreads / 64];
  v = row_sum16(v);
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kBlasThreads / 64; ++w) t += red[w];
  return t;
}

// Threads are laid over the stored units (16 places each) of one half-field:
// consecutive threads touch consecutive memory whatever the layout, and a
// field gives 16 x units threads rather than one per 4D site, which keeps
// small lattices from walking L5 dependent loads.
__device__ __forceinline__ int blas_units(const Geom& g) { return ((g.Vh + 15) >> 4) * g.L5; }
// whether a place holds a site (the last tile of a ragged lattice is padded)
__device__ __forceinline__ bool holds_site(const Geom& g, int unit, int at) {
  const int u = unit - ((g.Vh - 1) >> 4) * g.L5;
  if (u < 0) return true;
  int in, s;
  place_site(u, at, g.L5, in, s);
  return ((g.Vh - 1) & ~15) + in < g.Vh;
}

// A workgroup's threads over whole fifth-dimension columns: `tiles` 16-site
// tiles, one thread per site and slice in the order of the stored units.
struct ColumnThread {
  int s, in, tl;  // slice, site in the tile, tile of the workgroup
  bool valid;
  Place at;
};
__device__ __forceinline__ ColumnThread column_thread(const Geom& g, int tiles) {
  const int ul = threadIdx.x >> 4, at = threadIdx.x & 15;
  ColumnThread t;
  t.tl = ul / g.L5;
  const int u = ul - t.tl * g.L5;
  const int tile = blockIdx.x * tiles + t.tl;
  place_site(u, at, g.L5, t.in, t.s);
  t.valid = tile * 16 + t.in < g.Vh;
  t.at = Place{(size_t)tile * g.L5 + u, at};
  return t;
}

// out = M_phi v on the workgroup's columns: (M_phi v)_s = b5 v_s + c5 (P5 v)_s,
// P5 taking spins 0,1 from slice s - 1 and spins 2,3 from slice s + 1, the wall
// hop carrying -mq.  The neighbouring slices' halves pass through LDS (both
// halves at once in FP32; FP64 takes them one after the other).
template <class R> constexpr bool kPhiBoth = sizeof(R) == 4;
template <class R> constexpr int kPhiRow = kPhiBoth<R> ? 24 : 12;
template <class R> constexpr int kPhiSlice = 16 * kPhiRow<R> + 4;  // the 4 spread a quad's rows over the banks
template <class R>
__device__ __forceinline__ void column_mphi(void* smem, const ColumnThread& t, int L5, const Coef5& c, const R v[24],
                                            R out[24]) {
  const R b5 = (R)c.b5, c5 = (R)c.c5, wall = (R)(-c.c5 * c.mq);
  const int s = t.s;
  R* lds = reinterpret_cast<R*>(smem) + (size_t)t.tl * L5 * kPhiSlice<R>;
  const int up = s == 0 ? L5 - 1 : s - 1, dn = s == L5 - 1 ? 0 : s + 1;
  const R cu = s == 0 ? wall : c5, cd = s == L5 - 1 ? wall : c5;
  R* mine = lds + s * kPhiSlice<R> + t.in * kPhiRow<R>;
  const R* ru = lds + up * kPhiSlice<R> + t.in * kPhiRow<R>;
  const R* rd = lds + dn * kPhiSlice<R> + t.in * kPhiRow<R> + (kPhiBoth<R> ? 12 : 0);
#pragma unroll
  for (int k = 0; k < kPhiRow<R>; ++k) mine[k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 12; ++k) out[k] = b5 * v[k] + cu * ru[k];
  if constexpr (!kPhiBoth<R>) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 12; ++k) mine[k] = v[12 + k];
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) out[12 + k] = b5 * v[12 + k] + cd * rd[k];
}

// p' = r + beta p, and pt = M_phi p': the input of the first stencil launch of
// the next iteration, which then needs no fifth-dimension prologue on its eight
// neighbours.  The direction alternates between two fields, so that x can be
// updated with two of them at once.
template <int PS>
__global__ __launch_bounds__(512) void k_cg_p(BlasArgs A, int tiles) {
  using RS = typename PrecTraits<PS>::Real;
  extern __shared__ __align__(16) unsigned char smem[];
  const int slot = blockIdx.y;
  // everything of the slot in one burst of scalar loads
  char *pa = A.a[slot], *pb = A.b[slot], *pc = A.c[slot], *pd = A.d[slot];
  const Coef5 coef = A.coef[slot];
  int active = 1, phase = 1;
  double b = A.ca;
  if (A.st != nullptr) {
    active = A.st[slot].active;
    phase = A.st[slot].phase;
    b = A.st[slot].beta;
  }
  if (!active) return;
  const RS beta = (RS)b;
  const bool fresh = A.st == nullptr && A.ca == 0.0;  // p' = r
  const char* from = phase != 0 ? pa : pd;
  char* to = phase != 0 ? pd : pa;
  const ColumnThread t = column_thread(A.g, tiles);
  const FieldDesc f{A.g.Vh, A.g.L5};
  RS cur[24], out[24];
#pragma unroll
  for (int k = 0; k < 24; ++k) cur[k] = 0;
  if (t.valid) {
    RS rv[24];
    if (!fresh) SpinorAt<PS>::load(from, f, t.at, cur);
    SpinorAt<PS>::load(pb, f, t.at, rv);
#pragma unroll
    for (int k = 0; k < 24; ++k) cur[k] = rv[k] + beta * cur[k];
    SpinorAt<PS>::store(to, f, t.at, cur, A.nt_store);
  }
  column_mphi<RS>(smem, t, A.g.L5, coef, cur, out);
  if (t.valid) SpinorAt<PS>::store(pc, f, t.at, out, A.nt_store);
}

// The streaming part of a reliable update in one pass: fold the solution
// increment into the FP64 solution, and form what the two M^ launches of the
// residual read (z = eta^ - xh as their xpay term, M_phi xh as their input).
// Bound by memory: 5 FP64 fields and x read and written.  It replaces a copy,
// two xpays, a clearing pass and a fifth-dimension pass, and the FP64 M^ of the
// update needs no M_phi prologue: the FP64 work of a 16^3 x 32 x 12 solve of 12
// RHS (12 updates each) went from 151 to 124 ms.
template <int PS>
__global__ __launch_bounds__(512) void k_update(BlasArgs A, int tiles) {
  using RS = typename PrecTraits<PS>::Real;
  extern __shared__ __align__(16) unsigned char smem[];
  const int slot = blockIdx.y;
  const ColumnThread t = column_thread(A.g, tiles);
  const FieldDesc f{A.g.Vh, A.g.L5};
  const bool has_x = !A.a.empty(), has_p = !A.f.empty();
  double xh[24], out[24];
#pragma unroll
  for (int k = 0; k < 24; ++k) xh[k] = 0;
  if (t.valid) {
    SpinorAt<F64>::load(A.b[slot], f, t.at, xh);
    if (has_x || has_p) {
      constexpr int PX = PS == F64 ? F64 : F32;
      RS x[24];  // the arithmetic type of the inner iteration is the type of x
#pragma unroll
      for (int k = 0; k < 24; ++k) x[k] = 0;
      if constexpr (PS == F64) {
#pragma unroll
        for (int k = 0; k < 24; ++k) x[k] = xh[k];
      } else {
        if (has_x) SpinorAt<PX>::load(A.a[slot], f, t.at, x);
      }
      if (has_p) {
        RS p[24];
        SpinorAt<PS>::load(A.f[slot], f, t.at, p);
        const RS alpha = (RS)A.ca;
#pragma unroll
        for (int k = 0; k < 24; ++k) x[k] += alpha * p[k];
      }
      if constexpr (PS == F64) {
#pragma unroll
        for (int k = 0; k < 24; ++k) xh[k] = x[k];
      } else {
#pragma unroll
        for (int k = 0; k < 24; ++k) {
          xh[k] += (double)x[k];
          x[k] = 0;
        }
        SpinorAt<PX>::store(A.a[slot], f, t.at, x, A.nt_store);
      }
      SpinorAt<F64>::store(A.b[slot], f, t.at, xh, A.nt_store);
    }
    SpinorAt<F64>::load(A.c[slot], f, t.at, out);
#pragma unroll
    for (int k = 0; k < 24; ++k) out[k] -= xh[k];
    SpinorAt<F64>::store(A.d[slot], f, t.at, out, A.nt_store);
  }
  column_mphi<double>(smem, t, A.g.L5, A.coef[slot], xh, out);
  if (t.valid) SpinorAt<F64>::store(A.e[slot], f, t.at, out, A.nt_store);
}

template <int PO>
__global__ __launch_bounds__(kBlasThreads) void k_round(BlasArgs A) {
  using RO = typename PrecTraits<PO>::Real;
  const int slot = blockIdx.y;
  const int idx = blockIdx.x * kBlasThreads + threadIdx.x;
  const int unit = idx >> 4, at = idx & 15;
  const FieldDesc f{A.g.Vh, A.g.L5};
  double loc = 0;
  if (unit < blas_units(A.g) && holds_site(A.g, unit, at)) {
    const Place pl{(size_t)unit, at};
    double iv[24];
    RO ov[24];
    SpinorAt<F64>::load(A.a[slot], f, pl, iv);
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      ov[k] = (RO)iv[k];
      loc += iv[k] * iv[k];
    }
    SpinorAt<PO>::store(A.b[slot], f, pl, ov);
  }
  const double t = block_sum_256(loc);
  if (threadIdx.x == 0) A.partials[(size_t)slot * A.nblk + blockIdx.x] = t;
}

template <int P>
__global__ __launch_bounds__(kBlasThreads) void k_norm_diff(BlasArgs A) {
  using R = typename PrecTraits<P>::Real;
  const int slot = blockIdx.y;
  const int idx = blockIdx.x * kBlasThreads + threadIdx.x;
  const int unit = idx >> 4, at = idx & 15;
  const FieldDesc f{A.g.Vh, A.g.L5};
  double loc = 0;
  if (unit < blas_units(A.g) && holds_site(A.g, unit, at)) {
    const Place pl{(size_t)unit, at};
    R av[24], bv[24];
    SpinorAt<P>::load(A.a[slot], f, pl, av);
    if (A.b[slot] != nullptr) {
      SpinorAt<P>::load(A.b[slot], f, pl, bv);
#pragma unroll
      for (int k = 0; k < 24; ++k) av[k] -= bv[k];
    }
#pragma unroll
    for (int k = 0; k < 24; ++k) loc += (double)av[k] * (double)av[k];
  }
  const double t = block_sum_256(loc);
  if (threadIdx.x == 0) A.partials[(size_t)slot * A.nblk + blockIdx.x] = t;
}

int blas_nblk(const Geom& g) {
  return (int)(((size_t)((g.Vh + 15) / 16) * g.L5 * 16 + kBlasThreads - 1) / kBlasThreads);
}

static dim3 blas_grid(BlasArgs& A) {
  A.nblk = blas_nblk(A.g);
  return dim3(A.nblk, A.nslots);
}


// Workgroups of whole columns: at least 256 threads' worth of 16-site tiles.
template <class R> struct ColumnLaunch {
  dim3 grid, block;
  int tiles;
  size_t lds;
  ColumnLaunch(const Geom& g, int nslots) {
    const int column = 16 * g.L5;
    tiles = column >= 256 ? 1 : 256 / column;
    grid = dim3(((g.Vh + 15) / 16 + tiles - 1) / tiles, nslots);
    block = dim3(tiles * column);
    lds = (size_t)tiles * g.L5 * kPhiSlice<R> * sizeof(R);
  }
};

template <int PS> static hipError_t cg_p_launch(const BlasArgs& A, hipStream_t st) {
  const ColumnLaunch<typename PrecTraits<PS>::Real> L(A.g, A.nslots);
  launch_k(k_cg_p<PS>, L.grid, L.block, L.lds, st, A, L.tiles);
  return hipGetLastError();
}

hipError_t blas_update(BlasArgs A, int ps, hipStream_t st) {
  const ColumnLaunch<double> L(A.g, A.nslots);
  // an increment needs a field to go to
  if (ps == F64 ? !A.a.empty() : A.a.empty() && !A.f.empty()) return hipErrorInvalidValue;
  switch (ps) {
    case F64: launch_k(k_update<F64>, L.grid, L.block, L.lds, st, A, L.tiles); break;
    case F32: launch_k(k_update<F32>, L.grid, L.block, L.lds, st, A, L.tiles); break;
    case F16: launch_k(k_update<F16>, L.grid, L.block, L.lds, st, A, L.tiles); break;
    case BF16: launch_k(k_update<BF16>, L.grid, L.block, L.lds, st, A, L.tiles); break;
    case I16: launch_k(k_update<I16>, L.grid, L.block, L.lds, st, A, L.tiles); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t blas_cg_p(BlasArgs A, int ps, hipStream_t st) {
  switch (ps) {
    case F64: return cg_p_launch<F64>(A, st);
    case F32: return cg_p_launch<F32>(A, st);
    case F16: return cg_p_launch<F16>(A, st);
    case BF16: return cg_p_launch<BF16>(A, st);
    case I16: return cg_p_launch<I16>(A, st);
  }
  return hipErrorInvalidValue;
}

hipError_t blas_round(BlasArgs A, int pout, hipStream_t st) {
  const dim3 grid = blas_grid(A);
  const dim3 blk(kBlasThreads);
  switch (pout) {
    case F64: launch_k(k_round<F64>, grid, blk, 0, st, A); break;
    case F32: launch_k(k_round<F32>, grid, blk, 0, st, A); break;
    case F16: launch_k(k_round<F16>, grid, blk, 0, st, A); break;
    case BF16: launch_k(k_round<BF16>, grid, blk, 0, st, A); break;
    case I16: launch_k(k_round<I16>, grid, blk, 0, st, A); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t blas_norm_diff(BlasArgs A, int p, hipStream_t st) {
  const dim3 grid = blas_grid(A);
  const dim3 blk(kBlasThreads);
  switch (p) {
    case F64: launch_k(k_norm_diff<F64>, grid, blk, 0, st, A); break;
    case F32: launch_k(k_norm_diff<F32>, grid, blk, 0, st, A); break;
    case F16: launch_k(k_norm_diff<F16>, grid, blk, 0, st, A); break;
    case BF16: launch_k(k_norm_diff<BF16>, grid, blk, 0, st, A); break;
    case I16: launch_k(k_norm_diff<I16>, grid, blk, 0, st, A); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// STREAM-style copy, the achievable-bandwidth reference the stencil's HBM
// figures are read against: each thread moves four 16-byte vectors, one per
// 256-thread stride (every wavefront access is 1 KB contiguous), with
// non-temporal loads and stores (nothing is re-read).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_copy16(const uint4* src, uint4* dst, size_t n) {
  const size_t base = (size_t)blockIdx.x * 1024 + threadIdx.x;
  v4u a[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const size_t i = base + 256 * (size_t)j;
    if (i < n) a[j] = __builtin_nontemporal_load((const MDWF_GLOBAL v4u*)(src + i));
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const size_t i = base + 256 * (size_t)j;
    if (i < n) __builtin_nontemporal_store(a[j], (MDWF_GLOBAL v4u*)(dst + i));
  }
}

hipError_t copy16(const void* src, void* dst, size_t n16, hipStream_t st) {
  if (n16 == 0) return hipErrorInvalidValue;
  const size_t blocks = (n16 + 1023) / 1024;
  if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
  launch_k(k_copy16, dim3((unsigned)blocks), dim3(256), 0, st, static_cast<const uint4*>(src), static_cast<uint4*>(dst),
           n16);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// scalar kernels: one 1024-thread workgroup per right-hand side
// ---------------------------------------------------------------------------
constexpr int kScalarThreads = 1024;

// Sum of one slot's n partials in a fixed order (four independent strided
// accumulators per thread, then a fixed tree); valid in thread 0.
__device__ __forceinline__ double slot_sum(const double* partials, int n, int slot) {
  const double* q = partials + (size_t)slot * n;
  constexpr int T = kScalarThreads;
  double v0 = 0, v1 = 0, v2 = 0, v3 = 0;
  int j = threadIdx.x;
  for (; j + 3 * T < n; j += 4 * T) {
    v0 += q[j];
    v1 += q[j + T];
    v2 += q[j + 2 * T];
    v3 += q[j + 3 * T];
  }
  for (; j < n; j += T) v0 += q[j];
  double v = (v0 + v1) + (v2 + v3);
  __shared__ double red[T / 64];
  v = row_sum16(v);
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < T / 64; ++w) t += red[w];
  return t;
}

__global__ __launch_bounds__(kScalarThreads) void k_reduce(const double* partials, int n, double* out) {
  const double t = slot_sum(partials, n, blockIdx.x);
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}

__device__ __forceinline__ bool finite_d(double v) { return v == v && v - v == 0.0; }

__global__ __launch_bounds__(kScalarThreads) void k_cg_alpha(CGState* S, const double* partials, int n) {
  const int slot = blockIdx.x;
  if (!S[slot].active) return;
  const double pq = slot_sum(partials, n, slot);
  if (threadIdx.x == 0) {
    CGState& s = S[slot];
    s.pq = pq;
    if (!finite_d(pq)) {
      s.flags |= CG_FLAG_NAN | CG_FLAG_ALPHA;
      s.active = 0;
    } else if (!(pq > 0.0)) {
      s.flags |= CG_FLAG_BREAKDOWN | CG_FLAG_ALPHA;
      s.active = 0;
    } else {
      s.alpha_prev = s.alpha;
      s.alpha = s.rho / pq;
    }
  }
}

__global__ __launch_bounds__(kScalarThreads) void k_cg_beta(CGState* S, const double* partials, int n) {
  const int slot = blockIdx.x;
  if (!S[slot].active) return;
  const double rr = slot_sum(partials, n, slot);
  if (threadIdx.x == 0) {
    CGState& s = S[slot];
    s.iters += 1;
    s.rho_new = rr;
    const double rn = sqrt(rr);
    if (!finite_d(rr)) {
      s.flags |= CG_FLAG_NAN;
      s.active = 0;
    } else if (rr <= s.tol2 || (s.delta > 0.0 && rn < s.delta * s.rmax)) {
      // converged in the inner precision, or the residual fell by delta:
      // the host recomputes the FP64 residual (reliable update)
      s.flags |= CG_FLAG_UPDATE;
      s.active = 0;
    } else if (s.iters >= s.max_iter) {
      s.flags |= CG_FLAG_MAXIT | CG_FLAG_UPDATE;
      s.active = 0;
    } else {
      s.beta = rr / s.rho;
      s.rho = rr;
      s.phase ^= 1;  // the next direction goes to the other field; a frozen RHS keeps its phase
      if (rn > s.rmax) s.rmax = rn;
    }
  }
}

hipError_t scalar_reduce(const double* partials, int n, int nslots, double* out, hipStream_t st) {
  launch_k(k_reduce, dim3(nslots), dim3(kScalarThreads), 0, st, partials, n, out);
  return hipGetLastError();
}
hipError_t scalar_cg_alpha(CGState* S, const double* partials, int n, int nslots, hipStream_t st) {
  launch_k(k_cg_alpha, dim3(nslots), dim3(kScalarThreads), 0, st, S, partials, n);
  return hipGetLastError();
}
hipError_t scalar_cg_beta(CGState* S, const double* partials, int n, int nslots, hipStream_t st) {
  launch_k(k_cg_beta, dim3(nslots), dim3(kScalarThreads), 0, st, S, partials, n);
  return hipGetLastError();
}

}  // namespace mdwf
