// Layout, precision and source kernels: user complex128 fields <-> internal
// half-fields, gauge compression to 12 reals, point and Z2 sources.
#include "dev_common.h"
#include "hop.h"
#include "kernels.h"

namespace mdwf {

__device__ __forceinline__ int lex_index(const Geom& g, int par, int cb) {
  int x, y, z, t;
  site_coords(g, par, cb, x, y, z, t);
  return ((t * g.Lz + z) * g.Ly + y) * g.Lx + x;
}

// ---------------------------------------------------------------------------
// User fields <-> half-fields.  The 16 sites of a tile of both parities are 32
// consecutive user sites (cb = lexicographic index / 2), 6 KB per slice, so a
// workgroup streams whole runs of the user field, 16 bytes per lane, and hands
// them over in LDS to the lanes that own a (site, slice).  Reading a spinor per
// lane instead (192 bytes apart) fetched every line several times.  Bound by
// memory latency more than by bandwidth (one burst of loads per wavefront), so
// the rows in LDS have the field's arithmetic type, not the user's FP64: that
// holds 24 wavefronts per CU instead of 12.  At 32^3 x 64, L5 = 12, one parity in and
// both out: FP16 787 + 1029 us (806 + 1739 with FP64 rows; a lane per spinor
// took 2 x 1220 out on 24^3 x 64 x 16 of two RHS, now 1135), FP32 874 + 1107.
// ---------------------------------------------------------------------------
constexpr int kRowU = 13;        // complex numbers per site in LDS: 12 and one of padding
template <class R> using Vec2 = R __attribute__((ext_vector_type(2)));
constexpr int kConvThreads = 128;

// parity bit of x of the site with index cb: its lexicographic index is
// 2 cb + (bit ^ parity)
__device__ __forceinline__ int row_bit(const Geom& g, int cb) {
  int x, y, z, t;
  site_coords(g, 0, cb, x, y, z, t);
  return (y + z + t) & 1;
}

// site and slice of a lane in a wavefront of 16 sites x 4 slices, in the order
// of the stored units
__device__ __forceinline__ void conv_lane(int L5, int lane, int& in, int& sq) {
  const bool q = quad_layout(L5);
  in = q ? lane >> 2 : lane & 15;
  sq = q ? lane & 3 : lane >> 4;
}

// BOTH: half-fields of both parities, 4 slices per workgroup, wavefront p
// converts parity p.  Otherwise parity par only, 8 slices per workgroup.
template <int P, bool BOTH>
__global__ __launch_bounds__(kConvThreads) void k_user_to_half(Geom g, PtrTab user, PtrTab even, PtrTab odd,
                                                               int par) {
  using R = typename PrecTraits<P>::Real;
  constexpr int S = BOTH ? 4 : 8, W = BOTH ? 32 : 16;  // slices, user sites per slice
  __shared__ __align__(16) Vec2<R> row[S * W * kRowU];
  __shared__ int bit[16];
  const int tid = threadIdx.x, tile = blockIdx.x, s0 = blockIdx.y * S, slot = blockIdx.z;
  const size_t V4 = (size_t)g.Vh * 2;
  const int ns = min(S, g.L5 - s0), nw = min(W, (int)(V4 - (size_t)tile * 32) / (BOTH ? 1 : 2));
  if (tid < 16) bit[tid] = row_bit(g, tile * 16 + tid);
  __syncthreads();
  const v2d* u = reinterpret_cast<const v2d*>(user[slot]);
#pragma unroll
  for (int j = 0; j < S * W * 12 / kConvThreads; ++j) {
    const int e = tid + j * kConvThreads;
    const int l = e / 12, k = e - l * 12;  // (slice, site), component
    const int sl = l / W, i = l % W;
    if (sl < ns && i < nw) {
      const size_t site = (size_t)tile * 32 + (BOTH ? i : 2 * i + (bit[i] ^ par));
      const v2d d = ldg<v2d>(u + ((size_t)(s0 + sl) * V4 + site) * 12 + k);
      row[l * kRowU + k] = Vec2<R>{(R)d.x, (R)d.y};
    }
  }
  __syncthreads();
  const int wave = tid >> 6;
  int in, sq;
  conv_lane(g.L5, tid & 63, in, sq);
  const int sl = BOTH ? sq : 4 * wave + sq, p = BOTH ? wave : par;
  const int cb = tile * 16 + in;
  if (sl >= ns || cb >= g.Vh) return;
  const Vec2<R>* r = row + (sl * W + (BOTH ? 2 * in + (bit[in] ^ p) : in)) * kRowU;
  R v[24];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    v[2 * k] = r[k].x;
    v[2 * k + 1] = r[k].y;
  }
  SpinorIO<P>::store(p == 0 ? even[slot] : odd[slot], FieldDesc{g.Vh, g.L5}, cb, s0 + sl, v);
}

// One parity with M_phi applied: whole columns of a 16-site tile per
// workgroup, so that slices s - 1 and s + 1 are in LDS beside s; M_phi is
// formed in the field's arithmetic from values rounded to that arithmetic.  The
// hop then reads a field that already holds M_phi psi; forming it on each of its
// eight neighbours took a 32^3 x 64 x 12 hop from 700 to 1310 us in FP32, against
// one more half-field written here.  FP64 and FP32: 16-bit storage would round
// M_phi psi.
template <int P>
__global__ __launch_bounds__(512) void k_user_to_half_phi(Geom g, PtrTab user, PtrTab half, PtrTab phi,
                                                          CoefTab coef, int par) {
  using R = typename PrecTraits<P>::Real;
  extern __shared__ __align__(16) unsigned char smem[];
  Vec2<R>* row = reinterpret_cast<Vec2<R>*>(smem);
  __shared__ int bit[16];
  const int tid = threadIdx.x, tile = blockIdx.x, slot = blockIdx.y;
  const int L5 = g.L5, nthr = 16 * L5;  // = blockDim.x: one thread per site and slice
  const size_t V4 = (size_t)g.Vh * 2;
  const int nw = min(16, g.Vh - tile * 16);
  if (tid < 16) bit[tid] = row_bit(g, tile * 16 + tid);
  __syncthreads();
  const v2d* u = reinterpret_cast<const v2d*>(user[slot]);
#pragma unroll
  for (int j = 0; j < 12; ++j) {
    const int e = tid + j * nthr;
    const int l = e / 12, k = e - l * 12;
    const int s = l >> 4, i = l & 15;
    if (i < nw) {
      const v2d d = ldg<v2d>(u + ((size_t)s * V4 + (size_t)tile * 32 + 2 * i + (bit[i] ^ par)) * 12 + k);
      row[l * kRowU + k] = Vec2<R>{(R)d.x, (R)d.y};
    }
  }
  __syncthreads();
  int in, s;
  place_site(tid >> 4, tid & 15, L5, in, s);
  if (in >= nw) return;
  const Place at{(size_t)tile * L5 + (tid >> 4), tid & 15};
  const FieldDesc f{g.Vh, L5};
  const Vec2<R>* r = row + (s * 16 + in) * kRowU;
  R v[24];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    v[2 * k] = r[k].x;
    v[2 * k + 1] = r[k].y;
  }
  SpinorAt<P>::store(half[slot], f, at, v);
  const Coef5 c = coef[slot];
  const R b5 = (R)c.b5, c5 = (R)c.c5, wall = (R)(-c.c5 * c.mq);
  const R cu = s == 0 ? wall : c5, cd = s == L5 - 1 ? wall : c5;
  const Vec2<R>* ru = row + ((s == 0 ? L5 - 1 : s - 1) * 16 + in) * kRowU;
  const Vec2<R>* rd = row + ((s == L5 - 1 ? 0 : s + 1) * 16 + in) * kRowU;
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const Vec2<R> d = r[k], o = k < 6 ? ru[k] : rd[k];
    const R w = k < 6 ? cu : cd;
    v[2 * k] = b5 * d.x + w * o.x;
    v[2 * k + 1] = b5 * d.y + w * o.y;
  }
  SpinorAt<P>::store(phi[slot], f, at, v);
}

// Both parities of 4 slices per workgroup; a null half-field writes zeros.
template <int P>
__global__ __launch_bounds__(kConvThreads) void k_half_to_user(Geom g, PtrTab even, PtrTab odd, PtrTab user,
                                                               bool nt) {
  using R = typename PrecTraits<P>::Real;
  constexpr int S = 4, W = 32;
  __shared__ __align__(16) Vec2<R> row[S * W * kRowU];
  const int tid = threadIdx.x, tile = blockIdx.x, s0 = blockIdx.y * S, slot = blockIdx.z;
  const size_t V4 = (size_t)g.Vh * 2;
  const int ns = min(S, g.L5 - s0), nw = min(W, (int)(V4 - (size_t)tile * 32));
  const int p = tid >> 6;
  int in, sq;
  conv_lane(g.L5, tid & 63, in, sq);
  const int cb = tile * 16 + in;
  if (sq < ns && cb < g.Vh) {
    const char* half = p == 0 ? even[slot] : odd[slot];
    R v[24];
    if (half != nullptr) {
      SpinorIO<P>::load(half, FieldDesc{g.Vh, g.L5}, cb, s0 + sq, v);
    } else {
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = 0;
    }
    Vec2<R>* r = row + (sq * W + 2 * in + (row_bit(g, cb) ^ p)) * kRowU;
#pragma unroll
    for (int k = 0; k < 12; ++k) r[k] = Vec2<R>{v[2 * k], v[2 * k + 1]};
  }
  __syncthreads();
  v2d* u = reinterpret_cast<v2d*>(user[slot]);
#pragma unroll
  for (int j = 0; j < S * W * 12 / kConvThreads; ++j) {
    const int e = tid + j * kConvThreads;
    const int l = e / 12, k = e - l * 12;
    const int sl = l / W, i = l % W;
    if (sl < ns && i < nw) {
      const Vec2<R> d = row[l * kRowU + k];
      stg<v2d>(u + ((size_t)(s0 + sl) * V4 + (size_t)tile * 32 + i) * 12 + k, v2d{(double)d.x, (double)d.y}, nt);
    }
  }
}

template <int P>
__global__ __launch_bounds__(256) void k_gauge(Geom g, const double* user, char* out) {
  const int cb = blockIdx.x * 256 + threadIdx.x;
  const int mu = blockIdx.y;
  const int par = blockIdx.z;
  if (cb >= g.Vh) return;
  const int i4 = lex_index(g, par, cb);
  const double* u = user + ((size_t)i4 * 4 + mu) * 18;  // rows 0,1 = 12 doubles
  if constexpr (P == F64) {
    double2* o = reinterpret_cast<double2*>(out) + link_index(par, mu, 0, cb, g.Vh, 6);
#pragma unroll
    for (int k = 0; k < 6; ++k) o[(size_t)k * kSiteTile] = make_double2(u[2 * k], u[2 * k + 1]);
  } else if constexpr (P == F32) {
    float4* o = reinterpret_cast<float4*>(out) + link_index(par, mu, 0, cb, g.Vh, 3);
#pragma unroll
    for (int k = 0; k < 3; ++k)
      o[(size_t)k * kSiteTile] = make_float4((float)u[4 * k], (float)u[4 * k + 1], (float)u[4 * k + 2], (float)u[4 * k + 3]);
  } else {
    uint2* o = reinterpret_cast<uint2*>(out) + link_index(par, mu, 0, cb, g.Vh, 3);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      uint2 q;
      q.x = pack2<P>((float)u[4 * k], (float)u[4 * k + 1]);
      q.y = pack2<P>((float)u[4 * k + 2], (float)u[4 * k + 3]);
      o[(size_t)k * kSiteTile] = q;
    }
  }
}

__global__ __launch_bounds__(256) void k_fill_zero(uint4* p, size_t n16) {
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}
__global__ void k_fill_zero_tail(unsigned char* p, size_t n) {
  if (threadIdx.x < n) p[threadIdx.x] = 0;
}

// one thread writes the wall entries of a unit 4D point source: in the chiral
// basis P+ keeps spins 0,1 (slice L5-1), P- keeps spins 2,3 (slice 0)
__global__ void k_source_point(Geom g, double* eta, int x, int y, int z, int t, int spin, int colour) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const size_t V4 = (size_t)g.Vh * 2;
  const size_t i4 = (size_t)((t * g.Lz + z) * g.Ly + y) * g.Lx + x;
  const int s = spin < 2 ? g.L5 - 1 : 0;
  eta[(((size_t)s * V4 + i4) * 12 + spin * 3 + colour) * 2] = 1.0;
}

// SplitMix64 (Steele, Lea, Flood 2014): output number k of the generator
// seeded with `seed`.
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t k) {
  uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void k_source_z2(Geom g, double* eta, uint64_t seed, int rhs) {
  const size_t V4 = (size_t)g.Vh * 2;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;  // (i4*4 + spin)*3 + colour
  if (idx >= V4 * 12) return;
  const size_t i4 = idx / 12;
  const int sc = (int)(idx % 12);
  const int spin = sc / 3;
  const uint64_t z = splitmix64(seed, (uint64_t)rhs * V4 * 12 + idx);
  const double r = 0.70710678118654752440;
  const double re = (z & 1) ? -r : r;
  const double im = (z & 2) ? -r : r;
  const int s = spin < 2 ? g.L5 - 1 : 0;
  double2* e = reinterpret_cast<double2*>(eta);
  e[((size_t)s * V4 + i4) * 12 + sc] = make_double2(re, im);
}

// ---------------------------------------------------------------------------
// Feynman-Hellmann sequential source (user layouts, FP64).
// 4D quark field read off the walls: q = P- psi_0 + P+ psi_{L5-1}; in the
// chiral basis spins 0,1 come from slice L5-1 and spins 2,3 from slice 0.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_propagator_4d(Geom g, const double2* psi, double2* q) {
  const size_t V4 = (size_t)g.Vh * 2;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;  // i4 * 12 + spin * 3 + colour
  const size_t r = blockIdx.y;
  if (idx >= V4 * 12) return;
  const int spin = (int)(idx % 12) / 3;
  const int s = spin < 2 ? g.L5 - 1 : 0;
  q[r * V4 * 12 + idx] = psi[(r * g.L5 + s) * V4 * 12 + idx];
}

// eta = wall injection of Gamma q: Gamma is a signed permutation in the
// chiral basis, row a of Gamma q = i^phase[a] q[perm[a]]; eta_0 takes the P-
// spins (2,3), eta_{L5-1} the P+ spins (0,1), every other slice is zero.
struct SpinPerm {
  int perm[4];
  int phase[4];  // power of i
};

__global__ __launch_bounds__(256) void k_current_source(Geom g, SpinPerm G, const double2* q, double2* eta) {
  const size_t V4 = (size_t)g.Vh * 2;
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;  // i4 * 12 + spin * 3 + colour
  const int s = blockIdx.y;
  const size_t r = blockIdx.z;
  if (idx >= V4 * 12) return;
  const size_t i4 = idx / 12;
  const int spin = (int)(idx % 12) / 3;
  const int colour = (int)(idx % 3);
  const bool wall = (s == 0 && spin >= 2) || (s == g.L5 - 1 && spin < 2);
  double2 v = make_double2(0.0, 0.0);
  if (wall) {
    const double2 x = q[r * V4 * 12 + i4 * 12 + G.perm[spin] * 3 + colour];
    switch (G.phase[spin] & 3) {
      case 0: v = x; break;
      case 1: v = make_double2(-x.y, x.x); break;   // i x
      case 2: v = make_double2(-x.x, -x.y); break;  // -x
      default: v = make_double2(x.y, -x.x); break;  // -i x
    }
  }
  eta[(r * g.L5 + s) * V4 * 12 + idx] = v;
}

// The gamma matrices (chiral DeGrand-Rossi basis, mu = x, y, z, t) as signed
// permutations: row a of g_mu has its one entry i^ph[mu][a] in column col[mu][a].
static const int kGammaCol[4][4] = {{3, 2, 1, 0}, {3, 2, 1, 0}, {2, 3, 0, 1}, {2, 3, 0, 1}};
static const int kGammaPh[4][4] = {{1, 1, 3, 3}, {2, 0, 0, 2}, {1, 3, 3, 1}, {0, 0, 0, 0}};

// Gamma = g_x^b0 g_y^b1 g_z^b2 g_t^b3 for mask = b0 + 2 b1 + 4 b2 + 8 b3.
// (A B) has row a in column colB[colA[a]] with phase phA[a] + phB[colA[a]].
static SpinPerm gamma_perm(int mask) {
  SpinPerm G;
  for (int a = 0; a < 4; ++a) {
    G.perm[a] = a;
    G.phase[a] = 0;
  }
  for (int mu = 0; mu < 4; ++mu) {
    if (!((mask >> mu) & 1)) continue;
    SpinPerm P;
    for (int a = 0; a < 4; ++a) {
      const int j = G.perm[a];
      P.perm[a] = kGammaCol[mu][j];
      P.phase[a] = (G.phase[a] + kGammaPh[mu][j]) & 3;
    }
    G = P;
  }
  return G;
}

// ---------------------------------------------------------------------------
// Source of the physical 4D propagator of the Moebius action: the 4D field
// Gamma xi enters on the walls of the opposite chirality to the read-out
// (P+ on slice 0, P- on slice L5-1) and is multiplied by the 4D factor
// (1 - c5 D_W) = beta + (c5/2) H, beta = 1 - c5 (4 - M5), that turns the
// Moebius operator into its Shamir-like form.  FP64, user layouts.
//
// The zeros of the inner slices are a plain clearing pass at the memory's rate;
// a workgroup hops 64 sites, wavefront w on wall w (one chirality of Gamma xi,
// two colour vectors per link), and hands its rows to coalesced stores through
// LDS.  The hop is bound by L1 accesses (xi is read 192 bytes apart) and by
// latency at three wavefronts per SIMD.  Twelve sources on 16^3 x 32, L5 = 12:
// 510 + 658 us (3233 with one thread per site that wrote its 12 slices 192 bytes
// at a time and kept both walls in scratch memory; the writes alone take 615 us
// at the copy kernel's rate).
// ---------------------------------------------------------------------------
// i^ph x, without branches
__device__ __forceinline__ Cplx<double> times_i_pow(v2d x, int ph) {
  const double re = (ph & 1) ? x.y : x.x, im = (ph & 1) ? x.x : x.y;
  const uint64_t fr = (uint64_t)((ph ^ (ph >> 1)) & 1) << 63, fi = (uint64_t)((ph >> 1) & 1) << 63;
  return {__builtin_bit_cast(double, __builtin_bit_cast(uint64_t, re) ^ fr),
          __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, im) ^ fi)};
}

// the spins of P_w Gamma xi at site i4 (w = 0: spins 0,1; w = 1: spins 2,3)
template <int W>
__device__ __forceinline__ void chi_at(const double2* x, size_t i4, const SpinPerm& G, Cplx<double> v[2][3]) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      v[k][c] = times_i_pow(ldg<v2d>(x + i4 * 12 + G.perm[2 * W + k] * 3 + c), G.phase[2 * W + k] & 3);
}

// acc += sc (1 + SIG g_mu) of the field whose spins of chirality W are w and
// whose others are zero
template <int W, int MU, int SIG>
__device__ __forceinline__ void accumulate_wall(Cplx<double> acc[4][3], const Cplx<double> w[2][3], double sc) {
  if constexpr (W == 0) {
    accumulate_scaled<MU, SIG>(acc, w, sc);
  } else {
    const double ps = SIG > 0 ? sc : -sc;  // +SIG*sc
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      acc[2][c] = {fma(sc, w[0][c].re, acc[2][c].re), fma(sc, w[0][c].im, acc[2][c].im)};
      acc[3][c] = {fma(sc, w[1][c].re, acc[3][c].re), fma(sc, w[1][c].im, acc[3][c].im)};
      if constexpr (MU == 0) {  // acc0 += SIG i w1, acc1 += SIG i w0
        acc[0][c] = {fma(-ps, w[1][c].im, acc[0][c].re), fma(ps, w[1][c].re, acc[0][c].im)};
        acc[1][c] = {fma(-ps, w[0][c].im, acc[1][c].re), fma(ps, w[0][c].re, acc[1][c].im)};
      } else if constexpr (MU == 1) {  // acc0 -= SIG w1, acc1 += SIG w0
        acc[0][c] = {fma(-ps, w[1][c].re, acc[0][c].re), fma(-ps, w[1][c].im, acc[0][c].im)};
        acc[1][c] = {fma(ps, w[0][c].re, acc[1][c].re), fma(ps, w[0][c].im, acc[1][c].im)};
      } else if constexpr (MU == 2) {  // acc0 += SIG i w0, acc1 -= SIG i w1
        acc[0][c] = {fma(-ps, w[0][c].im, acc[0][c].re), fma(ps, w[0][c].re, acc[0][c].im)};
        acc[1][c] = {fma(ps, w[1][c].im, acc[1][c].re), fma(-ps, w[1][c].re, acc[1][c].im)};
      } else {  // acc0 += SIG w0, acc1 += SIG w1
        acc[0][c] = {fma(ps, w[0][c].re, acc[0][c].re), fma(ps, w[0][c].im, acc[0][c].im)};
        acc[1][c] = {fma(ps, w[1][c].re, acc[1][c].re), fma(ps, w[1][c].im, acc[1][c].im)};
      }
    }
  }
}

// w = U h or U^dag h, two colour vectors.  Each complex product is rounded
// before it joins the sum, which keeps the sources 1 to 3 % closer to the exact
// ones than colour_mul's chain of multiply-adds does (1.75e-16 against 1.77e-16
// at b5, c5 = 1.5, 0.5); the chain took 647 us for the hop below.
template <bool ADJ>
__device__ __forceinline__ void colour_mul_sum(const Cplx<double> U[3][3], const Cplx<double> h[2][3],
                                               Cplx<double> w[2][3]) {
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double re = 0, im = 0;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const Cplx<double> u = ADJ ? Cplx<double>{U[b][a].re, -U[b][a].im} : U[a][b];
        const Cplx<double> x = h[k][b];
        re += fma(u.re, x.re, -(u.im * x.im));
        im += fma(u.im, x.re, u.re * x.im);
      }
      w[k][a] = {re, im};
    }
}

template <int W, int D>
__device__ __forceinline__ void source_hop(const Geom& g, const SpinPerm& G, const char* gauge, const double2* x,
                                           const int X[4], int par, int cb, double hc, Cplx<double> acc[4][3]) {
  constexpr int MU = D / 2, FB = D % 2, SG = FB == 0 ? -1 : +1;  // (1 - g_mu) forward, (1 + g_mu) backward
  const int Lmu = MU == 0 ? g.Lx : MU == 1 ? g.Ly : MU == 2 ? g.Lz : g.Lt;
  int Y[4] = {X[0], X[1], X[2], X[3]};
  Y[MU] = FB == 0 ? (X[MU] + 1 == Lmu ? 0 : X[MU] + 1) : (X[MU] == 0 ? Lmu : X[MU]) - 1;
  const bool flip = MU == 3 && g.tap && X[3] == (FB == 0 ? g.Lt - 1 : 0);
  const size_t j4 = (((size_t)Y[3] * g.Lz + Y[2]) * g.Ly + Y[1]) * g.Lx + Y[0];
  Cplx<double> U[3][3], v[2][3], w[2][3];
  // forward: U_mu(x) on the site's own parity; backward: U_mu(x - mu)^dag
  LinkIO<F64>::load(gauge, g.Vh, FB == 0 ? par : 1 - par, MU, FB == 0 ? cb : (int)(j4 >> 1), U);
  chi_at<W>(x, j4, G, v);
  colour_mul_sum<FB == 1>(U, v, w);
  accumulate_wall<W, MU, SG>(acc, w, flip ? -hc : hc);
  pin_acc(acc);  // one neighbour at a time in registers
}

template <int W>
__device__ __forceinline__ void source_site(const Geom& g, const SpinPerm& G, const char* gauge, const double2* x,
                                            size_t i4, double beta, double hc, Cplx<double> out[12]) {
  int X[4];
  size_t rem = i4;
  X[0] = (int)(rem % g.Lx); rem /= g.Lx;
  X[1] = (int)(rem % g.Ly); rem /= g.Ly;
  X[2] = (int)(rem % g.Lz); rem /= g.Lz;
  X[3] = (int)rem;
  const int par = (X[0] + X[1] + X[2] + X[3]) & 1, cb = (int)(i4 >> 1);
  Cplx<double> acc[4][3], v[2][3];
  chi_at<W>(x, i4, G, v);
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    acc[2 * W + k / 3][k % 3] = {beta * v[k / 3][k % 3].re, beta * v[k / 3][k % 3].im};
    acc[2 - 2 * W + k / 3][k % 3] = {0, 0};
  }
  pin_acc(acc);
  source_hop<W, 0>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 1>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 2>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 3>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 4>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 5>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 6>(g, G, gauge, x, X, par, cb, hc, acc);
  source_hop<W, 7>(g, G, gauge, x, X, par, cb, hc, acc);
#pragma unroll
  for (int k = 0; k < 12; ++k) out[k] = acc[k / 3][k % 3];
}

constexpr int kSitesBlock = 64;      // sites of a workgroup
constexpr int kSourceThreads = 128;  // two wavefronts: its sites on each wall

__global__ __launch_bounds__(kSourceThreads) void k_source_physical(Geom g, SpinPerm G, const char* gauge,
                                                                    const double2* xi, double2* eta, double beta,
                                                                    double hc) {
  __shared__ __align__(16) v2d row[2 * kSitesBlock * kRowU];
  const size_t V4 = (size_t)g.Vh * 2, r = blockIdx.y;
  const int tid = threadIdx.x;
  double2* e = eta + r * g.L5 * V4 * 12;
  const size_t site0 = (size_t)blockIdx.x * kSitesBlock;
  const size_t i4 = site0 + (tid & 63);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  Cplx<double> out[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) out[k] = {0, 0};
  if (i4 < V4) {
    const double2* x = xi + r * V4 * 12;
    if (w == 0) source_site<0>(g, G, gauge, x, i4, beta, hc, out);
    else source_site<1>(g, G, gauge, x, i4, beta, hc, out);
  }
  // wall 0 goes to slice 0, wall 1 to slice L5 - 1: one row of LDS per site and
  // wall, the walls added where they share the slice
  v2d* mine = row + tid * kRowU;
#pragma unroll
  for (int k = 0; k < 12; ++k) mine[k] = v2d{out[k].re, out[k].im};
  __syncthreads();
  const int walls = g.L5 == 1 ? 1 : 2;
#pragma unroll
  for (int j = 0; j < 2 * kSitesBlock * 12 / kSourceThreads; ++j) {
    const int el = tid + j * kSourceThreads;
    const int l = el / 12, k = el - l * 12;  // (wall, site), component
    const int wl = l >> 6, i = l & 63;
    if (wl >= walls || site0 + i >= V4) continue;
    v2d v = row[l * kRowU + k];
    if (walls == 1) v += row[(kSitesBlock + i) * kRowU + k];
    stg<v2d>(e + ((size_t)(wl == 0 ? 0 : g.L5 - 1) * V4 + site0 + i) * 12 + k, v);
  }
}

// Clears n 16-byte vectors at the same place of every right-hand side.
__global__ __launch_bounds__(256) void k_clear(uint4* p, size_t n, size_t stride, bool nt) {
  const size_t first = (size_t)blockIdx.x * 2048 + threadIdx.x;
  uint4* q = p + blockIdx.y * stride;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (first + 256 * j < n) stg<v4u>(q + first + 256 * j, v4u{0, 0, 0, 0}, nt);
}

hipError_t propagator_4d(const Geom& g, int nrhs, const double* psi, double* q, hipStream_t st) {
  const size_t n = (size_t)g.Vh * 2 * 12;
  const dim3 grid((unsigned)((n + 255) / 256), (unsigned)nrhs), blk(256);
  launch_k(k_propagator_4d, grid, blk, 0, st, g, reinterpret_cast<const double2*>(psi),
           reinterpret_cast<double2*>(q));
  return hipGetLastError();
}

hipError_t current_source(const Geom& g, int nrhs, int mask, const double* q, double* eta, hipStream_t st) {
  const size_t n = (size_t)g.Vh * 2 * 12;
  const dim3 grid((unsigned)((n + 255) / 256), (unsigned)g.L5, (unsigned)nrhs), blk(256);
  launch_k(k_current_source, grid, blk, 0, st, g, gamma_perm(mask), reinterpret_cast<const double2*>(q),
           reinterpret_cast<double2*>(eta));
  return hipGetLastError();
}

hipError_t source_physical(const Geom& g, int nrhs, int mask, const char* gauge64, const double* xi, double* eta,
                           double beta, double hc, hipStream_t st) {
  const size_t V4 = (size_t)g.Vh * 2;
  if (g.L5 > 2) {  // the inner slices
    const size_t n = (size_t)(g.L5 - 2) * V4 * 12;
    const bool nt = (double)nrhs * V4 * g.L5 * 192 > 256e6;  // beyond the MALL: streamed
    launch_k(k_clear, dim3((unsigned)((n + 2047) / 2048), (unsigned)nrhs), dim3(256), 0, st,
             reinterpret_cast<uint4*>(eta) + V4 * 12, n, (size_t)g.L5 * V4 * 12, nt);
  }
  launch_k(k_source_physical, dim3((unsigned)((V4 + kSitesBlock - 1) / kSitesBlock), (unsigned)nrhs),
           dim3(kSourceThreads), 0, st, g, gamma_perm(mask), gauge64, reinterpret_cast<const double2*>(xi),
           reinterpret_cast<double2*>(eta), beta, hc);
  return hipGetLastError();
}

template <int P>
static hipError_t user_to_half(const Geom& g, const PtrTab& user, const PtrTab& even, const PtrTab& odd, int nslots,
                               hipStream_t st) {
  const unsigned tiles = (g.Vh + 15) / 16;
  if (!even.empty() && !odd.empty())
    launch_k(k_user_to_half<P, true>, dim3(tiles, (g.L5 + 3) / 4, nslots), dim3(kConvThreads), 0, st, g, user, even,
             odd, 0);
  else
    launch_k(k_user_to_half<P, false>, dim3(tiles, (g.L5 + 7) / 8, nslots), dim3(kConvThreads), 0, st, g, user, even,
             odd, !even.empty() ? 0 : 1);
  return hipGetLastError();
}

hipError_t layout_user_to_half(const Geom& g, const PtrTab& user, const PtrTab& even, const PtrTab& odd, int p,
                               int nslots, hipStream_t st) {
  if (even.empty() && odd.empty()) return hipErrorInvalidValue;
  switch (p) {
    case F64: return user_to_half<F64>(g, user, even, odd, nslots, st);
    case F32: return user_to_half<F32>(g, user, even, odd, nslots, st);
    case F16: return user_to_half<F16>(g, user, even, odd, nslots, st);
    case BF16: return user_to_half<BF16>(g, user, even, odd, nslots, st);
    case I16: return user_to_half<I16>(g, user, even, odd, nslots, st);
  }
  return hipErrorInvalidValue;
}

template <int P>
static hipError_t user_to_half_phi(const Geom& g, const PtrTab& user, const PtrTab& half, const PtrTab& phi,
                                   const CoefTab& coef, int par, int nslots, hipStream_t st) {
  const size_t lds = (size_t)16 * g.L5 * kRowU * 2 * sizeof(typename PrecTraits<P>::Real);
  auto k = k_user_to_half_phi<P>;
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
  }
  launch_k(k, dim3((g.Vh + 15) / 16, nslots), dim3(16 * g.L5), lds, st, g, user, half, phi, coef, par);
  return hipGetLastError();
}

hipError_t layout_user_to_half_phi(const Geom& g, const PtrTab& user, const PtrTab& half, const PtrTab& phi,
                                   const CoefTab& coef, int par, int p, int nslots, hipStream_t st) {
  switch (p) {
    case F64: return user_to_half_phi<F64>(g, user, half, phi, coef, par, nslots, st);
    case F32: return user_to_half_phi<F32>(g, user, half, phi, coef, par, nslots, st);
  }
  return hipErrorInvalidValue;
}

hipError_t layout_half_to_user(const Geom& g, const PtrTab& even, const PtrTab& odd, const PtrTab& user, int p,
                               int nslots, hipStream_t st) {
  const dim3 grid((g.Vh + 15) / 16, (g.L5 + 3) / 4, nslots), blk(kConvThreads);
  // user fields beyond the 256 MB MALL are streamed past the caches
  const bool nt = (double)nslots * g.Vh * 2 * g.L5 * 192 > 256e6;
  switch (p) {
    case F64: launch_k(k_half_to_user<F64>, grid, blk, 0, st, g, even, odd, user, nt); break;
    case F32: launch_k(k_half_to_user<F32>, grid, blk, 0, st, g, even, odd, user, nt); break;
    case F16: launch_k(k_half_to_user<F16>, grid, blk, 0, st, g, even, odd, user, nt); break;
    case BF16: launch_k(k_half_to_user<BF16>, grid, blk, 0, st, g, even, odd, user, nt); break;
    case I16: launch_k(k_half_to_user<I16>, grid, blk, 0, st, g, even, odd, user, nt); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t layout_gauge(const Geom& g, const double* user, char* out, int p, hipStream_t st) {
  const dim3 grid((g.Vh + 255) / 256, 4, 2), blk(256);
  switch (p) {
    case F64: launch_k(k_gauge<F64>, grid, blk, 0, st, g, user, out); break;
    case F32: launch_k(k_gauge<F32>, grid, blk, 0, st, g, user, out); break;
    case F16: launch_k(k_gauge<F16>, grid, blk, 0, st, g, user, out); break;
    case BF16: launch_k(k_gauge<BF16>, grid, blk, 0, st, g, user, out); break;
    case I16: launch_k(k_gauge<I16>, grid, blk, 0, st, g, user, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t fill_zero(void* ptr, size_t bytes, hipStream_t st) {
  const size_t n16 = bytes / 16;
  if (n16 > 0) {
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    launch_k(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, st, reinterpret_cast<uint4*>(ptr), n16);
  }
  const size_t tail = bytes - n16 * 16;
  if (tail > 0)
    launch_k(k_fill_zero_tail, dim3(1), dim3(16), 0, st,
                       reinterpret_cast<unsigned char*>(ptr) + n16 * 16, tail);
  return hipGetLastError();
}

hipError_t source_point(const Geom& g, double* eta, const int x0[4], int spin, int colour, hipStream_t st) {
  const size_t bytes = (size_t)g.Vh * 2 * g.L5 * 12 * 16;
  hipError_t e = fill_zero(eta, bytes, st);
  if (e != hipSuccess) return e;
  launch_k(k_source_point, dim3(1), dim3(64), 0, st, g, eta, x0[0], x0[1], x0[2], x0[3], spin, colour);
  return hipGetLastError();
}

hipError_t source_z2(const Geom& g, double* eta, uint64_t seed, int rhs_index, hipStream_t st) {
  const size_t V4 = (size_t)g.Vh * 2;
  const size_t bytes = V4 * g.L5 * 12 * 16;
  hipError_t e = fill_zero(eta, bytes, st);
  if (e != hipSuccess) return e;
  const size_t n = V4 * 12;
  launch_k(k_source_z2, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g, eta, seed, rhs_index);
  return hipGetLastError();
}

}  // namespace mdwf
