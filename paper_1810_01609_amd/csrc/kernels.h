// Launch interface of the libmdwf HIP kernels (internal to the library).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "dev_common.h"

namespace mdwf {

// Kernel-time profiling without marker packets: while a profiled library
// call is in flight on this thread, the first kernel it launches carries the
// start event and every kernel it launches records the stop event, both
// inside the dispatch itself.
struct LaunchTiming {
  hipEvent_t start = nullptr, stop = nullptr;
  int launches = 0;
};
LaunchTiming& launch_timing();

// A failed launch is left in the runtime's last-error state: every caller
// returns hipGetLastError() after its launches.
template <class F, class... Args>
inline void launch_k(F kernel, dim3 grid, dim3 block, size_t smem, hipStream_t st, Args... args) {
  LaunchTiming& t = launch_timing();
  hipEvent_t e0 = (t.stop != nullptr && t.launches == 0) ? t.start : nullptr;
  hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)smem, st, e0, t.stop, 0u, args...);
  if (t.stop != nullptr) ++t.launches;
}

// Fifth-dimension chains applied to whole columns of a site.
enum Chain : int {
  CH_NONE = 0,
  CH_M5INV = 1,
  CH_M5INV_DAG = 2,
  CH_MPHI = 3,
  CH_MPHI_DAG = 4,
  CH_M5 = 5,
  CH_M5_DAG = 6,
  CH_MPHI_M5INV = 7,        // M_phi M5^-1
  CH_MPHIDAG_M5INVDAG = 8,  // M_phi^T M5^-T
};

// Term added to coef_y * (chained hop result).
enum AuxMode : int {
  AUX_NONE = 0,
  AUX_PLAIN = 1,  // + aux
  AUX_M5 = 2,     // + M5 aux
  AUX_M5DAG = 3,  // + M5^T aux
};

// out = c2( coef_y * c1( H (or H^dag) [M_phi] in ) + auxterm )
// with an optional |.|^2 reduction of the value before c2.
struct DslashArgs {
  Geom g;
  int out_par;
  const char* gauge;       // gauge field of this precision
  PtrTab in;               // [nslots] input half-fields (parity 1-out_par; out_par if no hop)
  PtrTab aux;              // [nslots] or empty
  PtrTab out;              // [nslots]
  CoefTab coef;             // [nslots]
  const int* active;       // nullptr or active flag of slot i at active[i*active_stride]
  int active_stride;
  double* partials;        // [nslots][ntiles] (16-site tiles) when reduce
  int ntiles;
  int nslots;
  int nblk;                // filled by the launcher
  int cb_log2;             // filled by the launcher
  int lds_chain_bytes;     // filled by the launcher: offset of the reduction area
  int lds_stage_off;       // filled by the launcher
  int stage;               // 1: stage neighbour indices and links in LDS once per workgroup
  int order_bt;            // > 0: blocked (z, t) plane traversal with Bt time slices per block
  int order_yb;            // with order_bt > 0: the xy-plane is cut into order_yb bands of Ly/order_yb rows
  int nt_store;            // 1: the launch's field stores are streaming (non-temporal)
  // Order of (RHS, site block) over the workgroups of a multi-RHS launch:
  // 0 = the RHS of one site block consecutive; 1 = RHS by RHS over the whole
  // grid; 2 = each XCD's eighth of the site blocks, RHS by RHS inside it
  // (needs nblk % 8 == 0; the launcher falls back to 0 otherwise).
  int rhs_order;
  // filled by the launcher: y-rows of a band, workgroups per rectangle, Lt / Bt
  // and the multiply-high magic (0: divide) of division by workgroups per rectangle, Bt, Lz, Lt / Bt, slots,
  // site blocks, site blocks per XCD
  int rows, bpp, ntb;
  uint32_t m_bpp, m_bt, m_lz, m_ntb, m_nslots, m_nblk, m_per;
  int split_mask;          // bit mu: hops across the mu boundary come from halo buffers (skipped here)
  int c1, c2, aux_mode, reduce;
  int pro;                 // 1: M_phi on the input of the hop (16-bit storage, no CG update)
  double coef_y;
  // CG update fused into the epilogue.  cg_update = 1: with q the combined
  // value, r -= alpha q, and the reduction takes |r|^2; q and `out` are not
  // written; and x += alpha_prev p + alpha p2 where the state's phase is 1.  2:
  // the same without x (r -= alpha q only).  3: `out` is written as usual, and
  // the update of x is applied on the launch's (checkerboard index, slice)
  // pairs of x and p (fields of the other parity).  4: no update; aux is p, or
  // p2 in phase 1.  x is FP64 for an FP64 kernel, FP32 otherwise.
  int cg_update;
  PtrTab cg_x;
  PtrTab cg_r;
  PtrTab cg_p, cg_p2;
  const CGState* cg_st;
};

// The quad form of the stencil (dslash_quad.hip): whether it takes a launch,
// its LDS, and the launch itself (dslash_launch chooses).
bool dslash_quad_ok(const DslashArgs& A, int prec, bool hop, bool dag);
size_t dslash_quad_lds_bytes(int prec, int CB, int L5);
hipError_t dslash_quad_launch(const DslashArgs& A, int prec, bool dag, int threads, int grid, hipStream_t st);

hipError_t dslash_launch(DslashArgs A, int prec, bool hop, bool dag, int cb_log2, hipStream_t st);
// The traversal a launch of CB-site workgroups actually takes (invalid Bt or
// band counts fall back to the linear order / one band).
void clamp_traversal(const Geom& g, int CB, int& bt, int& yb);

// ---- domain decomposition, rehearsed on one GPU ---------------------------
// A rank owning a block of the lattice computes the hop in three steps: pack
// the faces its neighbours need (spin-projected half spinors, the backward
// ones already multiplied by U^dag), the interior hop with every hop across a
// split boundary left out (dslash5_kernel with split_mask), and the exterior
// update adding the received faces.  Face kind k = 2 mu + fb: fb = 0 holds
// (1 - g_mu) psi of the sites with x_mu = 0 (needed by the neighbour below as
// its forward term), fb = 1 holds U_mu^dag (1 + g_mu) psi of the sites with
// x_mu = L_mu - 1.  Layout per kind: [s][12 reals][face site], face sites of
// one parity indexed by the lexicographic index of the other three
// coordinates divided by two.
struct DDArgs {
  Geom g;
  int out_par;           // parity of the hop's output sites
  int split_mask;
  const char* gauge;
  // [nslots], in device memory always (a pointer by value made the packing and
  // the exterior step, which read them in scratch and in a loop, 5 us longer)
  char* const* in;       // input half-fields (parity 1 - out_par)
  char* const* out;      // output half-fields (updated in place by the exterior step)
  char* const* send;     // packed faces
  char* const* recv;     // faces received from the neighbours
  int nslots;
  size_t face_off[8];    // byte offset of face kind k inside a slot's buffer
  int face_n[4];         // sites of one parity on a face orthogonal to mu
};
hipError_t dd_pack(const DDArgs& A, int prec, hipStream_t st);
hipError_t dd_exterior(const DDArgs& A, int prec, hipStream_t st);
size_t dslash_lds_bytes(const DslashArgs& A, int prec, int cb_log2, bool hop, bool dag);
int dslash_max_threads(int prec);

// ---- BLAS-1 / reductions (one thread per site and slice) -------------------
struct BlasArgs {
  Geom g;
  PtrTab a;   // [nslots]
  PtrTab b;
  PtrTab c;
  PtrTab d;
  PtrTab e, f;
  CGState* st;      // [nslots] (CG kernels)
  double* partials; // [nslots][nblk]
  int nblk;         // filled by launcher
  int nslots;
  double ca;        // beta of blas_cg_p without a CG state, alpha of blas_update
  CoefTab coef;    // [nslots] (k_cg_p, k_update)
  int nt_store;      // streaming stores
};
constexpr int kBlasThreads = 256;

// CG: p' = r + beta p and pt = M_phi p'.   b=r c=pt, coef.  beta, the active
// flag and the phase come from the CG state: in phase 1 p is a and p' goes to
// d, in phase 0 the other way round.  Without a state (st null) p' goes to d,
// beta is A.ca, and p (a) is not read where that is zero.
hipError_t blas_cg_p(BlasArgs A, int ps, hipStream_t st);
// Start of a reliable update, FP64 xh, eta^, z and pt, x of precision px:
//   x += ca p, xh += x, x = 0, z = eta^ - xh, pt = M_phi xh
// with p in precision ps (an empty table: x is complete).  The plain FP64 solver
// has no x of its own (an empty table): xh += ca p.
// a=x b=xh c=eta^ d=z e=pt f=p, coef
hipError_t blas_update(BlasArgs A, int ps, hipStream_t st);
// b = a rounded from FP64 to precision pout; partials of |a|^2
hipError_t blas_round(BlasArgs A, int pout, hipStream_t st);
// partials of |a - b|^2 (|a|^2 where b's entry is null).  both precision p
hipError_t blas_norm_diff(BlasArgs A, int p, hipStream_t st);
int blas_nblk(const Geom& g);
// STREAM-style copy of n16 16-byte vectors (achievable-bandwidth reference)
hipError_t copy16(const void* src, void* dst, size_t n16, hipStream_t st);

// ---- scalar kernels (one workgroup per slot, fixed summation order) -------
// out[i] = sum_j partials[i*n + j]
hipError_t scalar_reduce(const double* partials, int n, int nslots, double* out, hipStream_t st);
// alpha = rho / <p,Ap>, with breakdown / NaN checks
hipError_t scalar_cg_alpha(CGState* st_, const double* partials, int n, int nslots, hipStream_t st);
// rho_new = |r|^2; freeze for the host or form beta
hipError_t scalar_cg_beta(CGState* st_, const double* partials, int n, int nslots, hipStream_t st);

// ---- layout, precision, sources --------------------------------------------
// user complex128 full field [s][t][z][y][x][spin][col] -> half-fields of
// precision p (an empty table: that parity is not wanted)
hipError_t layout_user_to_half(const Geom& g, const PtrTab& user, const PtrTab& even, const PtrTab& odd, int p,
                               int nslots, hipStream_t st);
// one parity of it, as half and phi = M_phi of it (FP64 and FP32)
hipError_t layout_user_to_half_phi(const Geom& g, const PtrTab& user, const PtrTab& half, const PtrTab& phi,
                                   const CoefTab& coef, int par, int p, int nslots, hipStream_t st);
// half-fields of precision p (a null entry: zeros) -> user field, both parities
hipError_t layout_half_to_user(const Geom& g, const PtrTab& even, const PtrTab& odd, const PtrTab& user, int p,
                               int nslots, hipStream_t st);
// user gauge complex128 [t][z][y][x][mu][3][3] (device) -> internal 12-real, prec p
hipError_t layout_gauge(const Geom& g, const double* user, char* out, int p, hipStream_t st);
hipError_t fill_zero(void* ptr, size_t bytes, hipStream_t st);
hipError_t source_point(const Geom& g, double* eta, const int x0[4], int spin, int colour, hipStream_t st);
hipError_t source_z2(const Geom& g, double* eta, uint64_t seed, int rhs_index, hipStream_t st);
// Feynman-Hellmann sequential source, user layouts, nrhs fields back to back
hipError_t propagator_4d(const Geom& g, int nrhs, const double* psi, double* q, hipStream_t st);
hipError_t current_source(const Geom& g, int nrhs, int mask, const double* q, double* eta, hipStream_t st);
// physical 4D-propagator source: eta = (beta + hc H) inject'(Gamma_mask xi), inject' = P+ on slice 0,
// P- on slice L5-1; gauge64 the FP64 internal gauge field
hipError_t source_physical(const Geom& g, int nrhs, int mask, const char* gauge64, const double* xi, double* eta,
                           double beta, double hc, hipStream_t st);

}  // namespace mdwf
