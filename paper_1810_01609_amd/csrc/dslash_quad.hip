// The fused stencil for fifth dimensions of a multiple of four slices, 32- and
// 16-bit storage: the hop launches of dslash5_kernel with the work of a site
// laid over quads of lanes.
//
// A wavefront owns 16 consecutive sites x 4 consecutive slices, lane
// 4 * site + (slice & 3); a site's L5 / 4 wavefronts form one workgroup (times
// CB / 16 tiles).  Four lanes of a quad therefore share a site and its links,
// and hold neighbouring slices:
//  * the colour product of 16-bit storage runs on the matrix cores.  A quad is
//    one block of the 16-block 4x4x4 MFMA: A = rows of the site's link as a
//    real 6 x 6 matrix (one row per lane), B = the four lanes' projected
//    colour vectors, D = the four lanes' products, every lane's own;
//  * the fifth-dimension operators run in registers.  M5^-1 is the recurrence
//    S_i = x_i - kappa S_{i-1}: two DPP steps inside the quad, then one
//    exchange of the wavefronts' last values through LDS (which also carries
//    the -mq wall), so a chain costs one barrier and no column ever passes
//    through LDS;
//  * a neighbour is addressed by a 32-bit byte offset staged in LDS, on a
//    uniform base that holds the wavefront's slices.
//
// What bounds it (32^3 x 64, L5 = 12, the plain hop; dslash5_kernel took 465 us
// in FP16 and 791 in FP32): the reads of the eight neighbours on their way from
// L2 to L1.  FP16 makes 502 accesses of 64 bytes to the L1 per wavefront and takes 442 us, FP32
// 897 and 786 us, FP64 (dslash5_kernel) 1794 and 1664 us: 0.37 accesses per
// clock and CU (0.40 with 12 RHS), 11-12 TB/s out of the L2.  The times follow
// the accesses (FP16 : FP32 0.56 both) and not what misses the L2 (0.46), nor
// the arithmetic: int16 issues 1393 VALU instructions per wavefront where FP16
// issues 574 and takes 459 us.  With lanes on
// 16 sites of one slice (256 contiguous bytes per 16 lanes) replaced by a quad
// reading 64-byte pieces of four slices the same kernel took 680 us, which is
// why the fields are stored quad by quad (dev_common.h).  Fewer or more
// neighbours in flight per lane (1, 4, 8) and 3-7 waves per SIMD were no
// faster; FP16 at 6 waves spills (+12 %).
#include "dev_common.h"
#include "hop.h"
#include "kernels.h"

namespace mdwf {

namespace {

// ---------------------------------------------------------------------------
// storage: 16-byte groups per site and slice, and the place of a lane's own
// site inside its wavefront's 16 sites x 4 slices
// ---------------------------------------------------------------------------
template <int P> constexpr int kGroups = P == F32 ? 6 : 3;
template <int P> constexpr int kSliceBytes = kGroups<P> * 16 * kSiteTile;  // one slice of a tile
constexpr bool is16(int p) { return p == F16 || p == BF16 || p == I16; }

template <class T> __device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

// A load or store at (uniform base) + (32-bit lane offset) + constant.
template <class V> __device__ __forceinline__ V ldo(const char* base, uint32_t off, int imm) {
  return *(const MDWF_GLOBAL V*)((const MDWF_GLOBAL char*)(base) + (size_t)off + imm);
}
template <class V> __device__ __forceinline__ void sto(char* base, uint32_t off, int imm, V v, bool nt) {
  MDWF_GLOBAL V* p = (MDWF_GLOBAL V*)((MDWF_GLOBAL char*)(base) + (size_t)off + imm);
  if (nt) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// One spinor as it is stored.
template <int P> struct Raw {
  v4u g[kGroups<P>];
  float sc;
};

// Bases of one half-field for this wavefront: its data and its scales, both
// at tile 0 and slice 4 w.
struct Base {
  char* d;
  char* s;
};
template <int P> __device__ __forceinline__ Base field_base(char* field, const Geom& g, int w) {
  char* p = uniform_ptr(field);
  Base b;
  b.d = p + (size_t)w * 4 * kSliceBytes<P>;
  b.s = p;
  if constexpr (is16(P)) b.s = p + half_scale_offset(g.L5, g.Vh) + (size_t)w * 4 * 4 * kSiteTile;
  return b;
}
// the same moved to tile `tile`
template <int P> __device__ __forceinline__ Base at_tile(Base b, int tile, int L5) {
  b.d += (size_t)tile * L5 * kSliceBytes<P>;
  b.s += (size_t)tile * L5 * 4 * kSiteTile;
  return b;
}

template <int P> __device__ __forceinline__ void load_raw(const Base& b, uint32_t off, uint32_t soff, Raw<P>& r) {
  if constexpr (is16(P)) r.sc = ldo<float>(b.s, soff, 0);
#pragma unroll
  for (int k = 0; k < kGroups<P>; ++k) r.g[k] = ldo<v4u>(b.d, off, k * 16 * kSiteTile);
}
template <int P> __device__ __forceinline__ void pin_raw(Raw<P>& r) {
#pragma unroll
  for (int k = 0; k < kGroups<P>; ++k) asm volatile("" : "+v"(r.g[k]) : : "memory");
  if constexpr (is16(P)) asm volatile("" : "+v"(r.sc) : : "memory");
}
// one stored group: 4 (FP32) or 8 reals
template <int P> __device__ __forceinline__ void unpack_group(const v4u& g, float sc, float* v) {
  const uint32_t w[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if constexpr (P == F32) {
      v[j] = __uint_as_float(w[j]);
    } else if constexpr (P == I16) {
      const float scq = sc * (1.0f / 32767.0f);
      v[2 * j] = (float)(int16_t)(uint16_t)(w[j] & 0xffffu) * scq;
      v[2 * j + 1] = (float)(int16_t)(uint16_t)(w[j] >> 16) * scq;
    } else {
      float a, b;
      unpack2<P>(w[j], a, b);
      v[2 * j] = a * sc;
      v[2 * j + 1] = b * sc;
    }
  }
}
template <int P> __device__ __forceinline__ void unpack(const Raw<P>& r, float v[24]) {
#pragma unroll
  for (int k = 0; k < kGroups<P>; ++k) unpack_group<P>(r.g[k], r.sc, v + k * (24 / kGroups<P>));
}
template <int P>
__device__ __forceinline__ void store_own(const Base& b, uint32_t off, uint32_t soff, const float v[24], bool nt) {
  if constexpr (P == F32) {
#pragma unroll
    for (int k = 0; k < 6; ++k)
      sto<v4f>(b.d, off, k * 16 * kSiteTile, v4f{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]}, nt);
  } else {
    // as SpinorIO16::store
    float m = 0.f;
#pragma unroll
    for (int k = 0; k < 24; ++k) m = fmaxf(m, fabsf(v[k]));
    const bool keep = m >= kMinNormalF32;
    const float inv = keep ? 1.0f / m : 0.f;
    if (!keep) m = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float* w = v + 8 * k;
      sto<v4u>(b.d, off, k * 16 * kSiteTile,
               v4u{pack2<P>(w[0] * inv, w[1] * inv), pack2<P>(w[2] * inv, w[3] * inv), pack2<P>(w[4] * inv, w[5] * inv),
                   pack2<P>(w[6] * inv, w[7] * inv)},
               nt);
    }
    sto<float>(b.s, soff, 0, m, nt);
  }
}

// ---------------------------------------------------------------------------
// Stage: neighbour offsets and links of the workgroup's sites in LDS.
//   neighbours: per site 8 x (data offset, scale offset), rows of 18 words
//   links, 16-bit storage (matrix cores): per direction the real 6 x 6 matrix
//     of V = U or U^+ (antiperiodic sign included): row 2a = (Re V_ab, -Im V_ab),
//     row 2a + 1 = (Im V_ab, Re V_ab), one 16-bit pair per b, three pairs and a
//     zero word per row; site rows of 208 words (16-byte reads, no conflicts)
//   links, other storage: per direction the 18 reals of U, 20 words; site rows
//     of 164 words
// ---------------------------------------------------------------------------
constexpr int kNbrRow = 18;
template <int P> constexpr int kLinkDir = Packed<P>::enabled ? 24 : 20;
template <int P> constexpr int kLinkRow = Packed<P>::enabled ? 208 : 164;
constexpr int kTotRow = 24;

template <int P> constexpr size_t stage_bytes(int CB) { return (size_t)CB * (kNbrRow + kLinkRow<P>) * 4; }
constexpr size_t totals_bytes(int CB, int L5) { return (size_t)CB * (L5 / 4) * kTotRow * 4; }
// one area of wavefront totals (a second chain's totals overlay the stage,
// which is dead once the first chain's barrier has passed), and the partial
// sums of the reduction
template <int P> constexpr size_t lds_bytes(int CB, int L5) {
  return stage_bytes<P>(CB) + totals_bytes(CB, L5) + (size_t)(CB / 16) * (L5 / 4) * 8;
}

template <int P>
__device__ __forceinline__ void fill_stage(const DslashArgs& A, uint32_t* nbr, uint32_t* lnk, int CB, int cb_log2,
                                           int cb0, int tid, int nthr) {
  const Geom& g = A.g;
  for (int task = tid; task < CB * 8; task += nthr) {
    const int cbl = task & (CB - 1);
    const int dir = task >> cb_log2;
    const int cb = cb0 + cbl;
    int nb = 0;
    float r[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) r[k] = 0;
    bool flip = false;
    if (cb < g.Vh) {
      int X[4];
      site_coords(g, A.out_par, cb, X[0], X[1], X[2], X[3]);
      const int mu = dir & 3;
      const int Lmu = mu == 0 ? g.Lx : mu == 1 ? g.Ly : mu == 2 ? g.Lz : g.Lt;
      const int xm = mu == 0 ? X[0] : mu == 1 ? X[1] : mu == 2 ? X[2] : X[3];
      const bool fwd = dir < 4;
      const int xn = fwd ? (xm + 1 == Lmu ? 0 : xm + 1) : (xm == 0 ? Lmu : xm) - 1;
      flip = mu == 3 && g.tap && xm == (fwd ? Lmu - 1 : 0);
      nb = cb_index(g, mu == 0 ? xn : X[0], mu == 1 ? xn : X[1], mu == 2 ? xn : X[2], mu == 3 ? xn : X[3]);
      LinkIO<P>::load_raw(A.gauge, g.Vh, fwd ? A.out_par : 1 - A.out_par, mu, fwd ? cb : nb, r);
    }
    Cplx<float> U[3][3];
    link_from_raw(r, U);
    const float sg = flip ? -1.f : 1.f;
    const uint32_t tile = (uint32_t)nb / kSiteTile, in = (uint32_t)nb % kSiteTile;
    nbr[cbl * kNbrRow + 2 * dir] = (tile * (uint32_t)g.L5 + in / 4) * kSliceBytes<P> + in % 4 * 64;
    nbr[cbl * kNbrRow + 2 * dir + 1] = (tile * (uint32_t)g.L5 + in / 4) * (4 * kSiteTile) + in % 4 * 16;
    uint32_t* row = lnk + cbl * kLinkRow<P> + dir * kLinkDir<P>;
    if constexpr (Packed<P>::enabled) {
      using K = Packed<P>;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        v4u re{0, 0, 0, 0}, im{0, 0, 0, 0};
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          const Cplx<float> u = dir < 4 ? U[a][b] : Cplx<float>{U[b][a].re, -U[b][a].im};
          const float vr = sg * u.re, vi = sg * u.im;
          re[b] = __builtin_bit_cast(uint32_t, K::make(vr, -vi));
          im[b] = __builtin_bit_cast(uint32_t, K::make(vi, vr));
        }
        *reinterpret_cast<v4u*>(row + 8 * a) = re;
        *reinterpret_cast<v4u*>(row + 8 * a + 4) = im;
      }
    } else {
      float* fr = reinterpret_cast<float*>(row);
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        fr[2 * k] = sg * U[k / 3][k % 3].re;
        fr[2 * k + 1] = sg * U[k / 3][k % 3].im;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// the hop
// ---------------------------------------------------------------------------
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// D += A B for the quad's block: a = this lane's row of the link matrix (four
// of its columns), b = this lane's colour vector (the same four components)
template <int P> __device__ __forceinline__ v4f mfma4(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1, v4f c) {
  const v2u a{a0, a1}, b{b0, b1};
  if constexpr (P == F16)
    return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}

template <int P, bool DAG, int D>
__device__ __forceinline__ void hop_compute(const uint32_t* lnk, int q, const Raw<P>& n, Cplx<float> acc[4][3]) {
  constexpr int MU = D / 2, FB = D % 2;
  constexpr int DIR = MU + 4 * FB;
  constexpr int SG = (FB == 0) == DAG ? +1 : -1;  // projector 1 + SG g_mu
  Cplx<float> w[2][3];
  if constexpr (Packed<P>::enabled) {
    using T2 = typename Packed<P>::T2;
    T2 psi[4][3], h[2][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) psi[k / 3][k % 3] = __builtin_bit_cast(T2, (uint32_t)n.g[k / 4][k % 4]);
    project<MU, SG>(psi, h);
    const v4u r0 = *reinterpret_cast<const v4u*>(lnk + DIR * kLinkDir<P> + 4 * q);
    const v4u r1 = *reinterpret_cast<const v4u*>(lnk + DIR * kLinkDir<P> + 16 + 4 * (q & 1));
    v4f d[2][2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t h0 = __builtin_bit_cast(uint32_t, h[k][0]), h1 = __builtin_bit_cast(uint32_t, h[k][1]);
      d[k][0] = mfma4<P>(r0.x, r0.y, h0, h1, v4f{0, 0, 0, 0});
      d[k][1] = mfma4<P>(r1.x, r1.y, h0, h1, v4f{0, 0, 0, 0});
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t h2 = __builtin_bit_cast(uint32_t, h[k][2]);
      d[k][0] = mfma4<P>(r0.z, r0.w, h2, 0u, d[k][0]);
      d[k][1] = mfma4<P>(r1.z, r1.w, h2, 0u, d[k][1]);
      w[k][0] = {d[k][0].x, d[k][0].y};
      w[k][1] = {d[k][0].z, d[k][0].w};
      w[k][2] = {d[k][1].x, d[k][1].y};
    }
    accumulate_scaled<MU, SG>(acc, w, n.sc);
  } else {
    Cplx<float> U[3][3], psi[4][3], h[2][3];
    const float* row = reinterpret_cast<const float*>(lnk) + DIR * kLinkDir<P>;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const v4f u = *reinterpret_cast<const v4f*>(row + 4 * k);
      U[2 * k / 3][2 * k % 3] = {u.x, u.y};
      U[(2 * k + 1) / 3][(2 * k + 1) % 3] = {u.z, u.w};
    }
    const float2 u8 = *reinterpret_cast<const float2*>(row + 16);
    U[2][2] = {u8.x, u8.y};
    if constexpr (P == I16) {  // unscaled integers, the scale joins the accumulation
#pragma unroll
      for (int k = 0; k < 12; ++k) {
        const uint32_t v = n.g[k / 4][k % 4];
        psi[k / 3][k % 3] = {(float)(int16_t)(uint16_t)(v & 0xffffu), (float)(int16_t)(uint16_t)(v >> 16)};
      }
    } else {
#pragma unroll
      for (int k = 0; k < 12; ++k)
        psi[k / 3][k % 3] = {__uint_as_float(n.g[k / 2][2 * (k % 2)]), __uint_as_float(n.g[k / 2][2 * (k % 2) + 1])};
    }
    project<MU, SG>(psi, h);
    colour_mul<FB == 1>(U, h, w);
    if constexpr (P == I16) accumulate_scaled<MU, SG>(acc, w, n.sc * (1.0f / 32767.0f));
    else accumulate<MU, SG>(acc, w);
  }
}

// Neighbours loaded together per thread.
constexpr int kQuadBatch = 2;

template <int P, bool DAG, int D, int END, int B0> struct HopRun {
  static __device__ __forceinline__ void load(const Base& in, const uint32_t* nbr, uint32_t lo, uint32_t ls, Raw<P>* n) {
    if constexpr (D < END) {
      constexpr int DIR = D / 2 + 4 * (D % 2);
      const uint2 o = *reinterpret_cast<const uint2*>(nbr + 2 * DIR);
      load_raw<P>(in, o.x + lo, o.y + ls, n[D - B0]);
      HopRun<P, DAG, D + 1, END, B0>::load(in, nbr, lo, ls, n);
    }
  }
  static __device__ __forceinline__ void compute(const uint32_t* lnk, int q, const Raw<P>* n, Cplx<float> acc[4][3]) {
    if constexpr (D < END) {
      hop_compute<P, DAG, D>(lnk, q, n[D - B0], acc);
      HopRun<P, DAG, D + 1, END, B0>::compute(lnk, q, n, acc);
    }
  }
};

template <int P, bool DAG, int NB, int B0>
__device__ __forceinline__ void hop_all(const Base& in, const uint32_t* nbr, const uint32_t* lnk, int q, uint32_t lo,
                                        uint32_t ls, Cplx<float> acc[4][3]) {
  if constexpr (B0 < 8) {
    Raw<P> n[NB];
    HopRun<P, DAG, B0, B0 + NB, B0>::load(in, nbr, lo, ls, n);
#pragma unroll
    for (int j = 0; j < NB; ++j) pin_raw<P>(n[j]);
    HopRun<P, DAG, B0, B0 + NB, B0>::compute(lnk, q, n, acc);
    pin_acc(acc);
    hop_all<P, DAG, NB, B0 + NB>(in, nbr, lnk, q, lo, ls, acc);
  }
}

// ---------------------------------------------------------------------------
// fifth-dimension chains over the quad
// ---------------------------------------------------------------------------
// Multiply-adds whose first factor comes from another lane of the quad
// (v_fmac_f32_dpp; the compiler keeps a separate move for each).  A DPP source
// must not have been written by the two preceding VALU instructions: each
// block starts with the two wait states, and inside a block a register is read
// at least five instructions after it was written.

// Two steps of the recurrence on six columns, in place: v += k1 * (one slice
// back), then v += k2 * (two slices back).  "Back" is slice s - 1 for columns
// walked upwards (LOWER), s + 1 for the others; the quad's ends read
// themselves with a zero coefficient.
template <bool LOWER> __device__ __forceinline__ void quad_scan6(float* v, float k1, float k2) {
  if constexpr (LOWER)
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %6 quad_perm:[0,0,1,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %1, %6 quad_perm:[0,0,1,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %2, %6 quad_perm:[0,0,1,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %3, %6 quad_perm:[0,0,1,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %4, %4, %6 quad_perm:[0,0,1,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %5, %5, %6 quad_perm:[0,0,1,2] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %0, %7 quad_perm:[0,0,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %1, %7 quad_perm:[0,0,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %2, %7 quad_perm:[0,0,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %3, %7 quad_perm:[0,0,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %4, %4, %7 quad_perm:[0,0,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %5, %5, %7 quad_perm:[0,0,0,1] row_mask:0xf bank_mask:0xf"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5])
        : "v"(k1), "v"(k2));
  else
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %0, %6 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %1, %6 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %2, %6 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %3, %6 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %4, %4, %6 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %5, %5, %6 quad_perm:[1,2,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %0, %7 quad_perm:[2,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %1, %1, %7 quad_perm:[2,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %2, %2, %7 quad_perm:[2,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %3, %7 quad_perm:[2,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %4, %4, %7 quad_perm:[2,3,3,3] row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %5, %5, %7 quad_perm:[2,3,3,3] row_mask:0xf bank_mask:0xf"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5])
        : "v"(k1), "v"(k2));
}

// o[i] += k * perm(x[i]), i < 6
#define MDWF_QUAD_FMA6(PERM, o, x, k)                                                                            \
  asm("s_nop 1\n\t"                                                                                              \
      "v_fmac_f32_dpp %0, %6, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                             \
      "v_fmac_f32_dpp %1, %7, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                             \
      "v_fmac_f32_dpp %2, %8, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                             \
      "v_fmac_f32_dpp %3, %9, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                             \
      "v_fmac_f32_dpp %4, %10, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                            \
      "v_fmac_f32_dpp %5, %11, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf"                                \
      : "+v"((o)[0]), "+v"((o)[1]), "+v"((o)[2]), "+v"((o)[3]), "+v"((o)[4]), "+v"((o)[5])                       \
      : "v"((x)[0]), "v"((x)[1]), "v"((x)[2]), "v"((x)[3]), "v"((x)[4]), "v"((x)[5]), "v"(k))

// o[i] = k * perm(x[i]), i < 6
#define MDWF_QUAD_MUL6(PERM, o, x, k)                                                                            \
  asm("s_nop 1\n\t"                                                                                              \
      "v_mul_f32_dpp %0, %6, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                              \
      "v_mul_f32_dpp %1, %7, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                              \
      "v_mul_f32_dpp %2, %8, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                              \
      "v_mul_f32_dpp %3, %9, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                              \
      "v_mul_f32_dpp %4, %10, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf\n\t"                             \
      "v_mul_f32_dpp %5, %11, %12 quad_perm:" PERM " row_mask:0xf bank_mask:0xf"                                 \
      : "=&v"((o)[0]), "=&v"((o)[1]), "=&v"((o)[2]), "=&v"((o)[3]), "=&v"((o)[4]), "=&v"((o)[5])                 \
      : "v"((x)[0]), "v"((x)[1]), "v"((x)[2]), "v"((x)[3]), "v"((x)[4]), "v"((x)[5]), "v"(k))

// o = or += coefficient times the slice before along the walk (LOWER columns
// 0..11 of o and x are walked upwards, LC the first of them)
template <int LC> __device__ __forceinline__ void quad_back_mul(float o[24], const float x[24], float l, float u) {
  constexpr int UC = 12 - LC;
  MDWF_QUAD_MUL6("[0,0,1,2]", o + LC, x + LC, l);
  MDWF_QUAD_MUL6("[0,0,1,2]", o + LC + 6, x + LC + 6, l);
  MDWF_QUAD_MUL6("[1,2,3,3]", o + UC, x + UC, u);
  MDWF_QUAD_MUL6("[1,2,3,3]", o + UC + 6, x + UC + 6, u);
}
template <int LC> __device__ __forceinline__ void quad_back_fma(float o[24], const float x[24], float l, float u) {
  constexpr int UC = 12 - LC;
  MDWF_QUAD_FMA6("[0,0,1,2]", o + LC, x + LC, l);
  MDWF_QUAD_FMA6("[0,0,1,2]", o + LC + 6, x + LC + 6, l);
  MDWF_QUAD_FMA6("[1,2,3,3]", o + UC, x + UC, u);
  MDWF_QUAD_FMA6("[1,2,3,3]", o + UC + 6, x + UC + 6, u);
}
// the same two slices back
template <int LC> __device__ __forceinline__ void quad_back2_fma(float o[24], const float x[24], float l, float u) {
  constexpr int UC = 12 - LC;
  MDWF_QUAD_FMA6("[0,0,0,1]", o + LC, x + LC, l);
  MDWF_QUAD_FMA6("[0,0,0,1]", o + LC + 6, x + LC + 6, l);
  MDWF_QUAD_FMA6("[2,3,3,3]", o + UC, x + UC, u);
  MDWF_QUAD_FMA6("[2,3,3,3]", o + UC + 6, x + UC + 6, u);
}
// o += coefficient times E, of which lane j holds reals 6j .. 6j + 5
template <int LC> __device__ __forceinline__ void quad_share_fma(float o[24], const float E[6], float l, float u) {
  MDWF_QUAD_FMA6("[0,0,0,0]", o, E, LC == 0 ? l : u);
  MDWF_QUAD_FMA6("[1,1,1,1]", o + 6, E, LC == 0 ? l : u);
  MDWF_QUAD_FMA6("[2,2,2,2]", o + 12, E, LC == 0 ? u : l);
  MDWF_QUAD_FMA6("[3,3,3,3]", o + 18, E, LC == 0 ? u : l);
}

struct QuadPos {
  int q;       // lane's slice inside the quad
  int w, nw;   // wavefront's place along the fifth dimension, and how many
  int site;    // 0..15
  float* tot;  // [w][site][24] of this 16-site tile
};

// The last values along the walk, for the next wavefront: lane 3 holds those of
// the lower columns, lane 0 those of the upper ones.
template <bool DAG> __device__ __forceinline__ void put_ends(const float v[24], const QuadPos& Q) {
  float* t = Q.tot + ((size_t)Q.w * 16 + Q.site) * kTotRow;
  constexpr int lo = DAG ? 12 : 0, up = DAG ? 0 : 12;
  if (Q.q == 3) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *reinterpret_cast<v4f*>(t + lo + 4 * k) = v4f{v[lo + 4 * k], v[lo + 4 * k + 1], v[lo + 4 * k + 2], v[lo + 4 * k + 3]};
  }
  if (Q.q == 0) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      *reinterpret_cast<v4f*>(t + up + 4 * k) = v4f{v[up + 4 * k], v[up + 4 * k + 1], v[up + 4 * k + 2], v[up + 4 * k + 3]};
  }
}

// v_i = add_i + v_{i-1} along the walk, with v_{-1} = -mq v_{L5-1}.  DAG
// exchanges the walk directions of the two chiralities (spins 0,1: reals 0..11;
// 2,3: 12..23).  The lane at a quad's end takes its neighbour from LDS and no
// other lane multiplies it, so a slice that is not finite reaches the slices
// next to it and no more.
template <bool DAG>
__device__ __forceinline__ void quad_shift(float v[24], const float add[24], const QuadPos& Q, float mq) {
  constexpr int lc = DAG ? 12 : 0, uc = 12 - lc;  // first lower and upper real
  put_ends<DAG>(v, Q);
  float u[24];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    u[lc + k] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v[lc + k]), 0x90, 0xf, 0xf, false));  // [0,0,1,2]
    u[uc + k] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v[uc + k]), 0xf9, 0xf, 0xf, false));  // [1,2,3,3]
  }
  __syncthreads();
  const bool fl = Q.w == 0, fu = Q.w == Q.nw - 1;  // the walk's first wavefront
  const float* t = Q.tot + Q.site * kTotRow;
  float wl = 1.f, wu = 1.f;
  if (Q.q == 0) {
    const float* x = t + (size_t)(fl ? Q.nw - 1 : Q.w - 1) * 16 * kTotRow + lc;
    wl = fl ? -mq : 1.f;
#pragma unroll
    for (int k = 0; k < 12; ++k) u[lc + k] = x[k];
  }
  if (Q.q == 3) {
    const float* x = t + (size_t)(fu ? 0 : Q.w + 1) * 16 * kTotRow + uc;
    wu = fu ? -mq : 1.f;
#pragma unroll
    for (int k = 0; k < 12; ++k) u[uc + k] = x[k];
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    v[lc + k] = fmaf(wl, u[lc + k], add[lc + k]);
    v[uc + k] = fmaf(wu, u[uc + k], add[uc + k]);
  }
}

// Walks the columns of v: y = the recurrence S_i = x_i - kappa S_{i-1} (alpha
// M5 y without the wall), then
//   out_i = add_i + t0 y_i, or with SHIFT t0 y_i + t1 y_{i-1},
// where y includes the wall (y_{-1} = -mq y_{L5-1}).
// In the quad S takes two steps; the wavefronts' last values T_w then give
// every wavefront the value E before its first slice,
//   E_w = sum_{w' < w} k4^(w-1-w') T_w' - mq/c k4^w sum_w' k4^(nw-1-w') T_w'
// (k4 = kappa^4, c = 1 + mq (-kappa)^L5), and y_i = S_i + (-kappa)^(i+1) E.
// Each lane forms E of six of the 24 reals and the quad shares them by DPP.
//
// CAREFUL (32-bit storage) sums everything the recurrence adds to x first, so
// that the result is x times its coefficient plus that, rounded once at full
// size (twice with add or SHIFT); the plain form rounds S twice, the product
// with t0 and the term in E, each at full size.  16-bit storage, whose own
// rounding is 1e3 times larger, saves the registers and some 90 instructions.
// FP32 M^+M^ on 32^3 x 64 x 12: 8.8e-8 from 64 bits and 6.92 ms, plain 1.03e-7
// and 6.95 ms (columns in LDS, as the general kernel did then: 9.7e-8).
template <bool SHIFT, bool DAG, bool CAREFUL>
__device__ __forceinline__ void quad_solve(float v[24], const float* add, const QuadPos& Q, float kappa, float mq,
                                           float inv_c, float t0, float t1, float ia = 1.f) {
  constexpr int lc = DAG ? 12 : 0, uc = 12 - lc;  // first lower and upper real
  const int pl = Q.q, pu = 3 - Q.q;  // place along the walk
  const float nk = -kappa, k2 = kappa * kappa;
  const float l1 = pl >= 1 ? nk : 0.f, l2 = pl >= 2 ? k2 : 0.f;
  const float u1 = pu >= 1 ? nk : 0.f, u2 = pu >= 2 ? k2 : 0.f;
  const float lt = pl >= 1 ? t1 : 0.f, ut = pu >= 1 ? t1 : 0.f;
  // what needs no neighbour wavefront goes before the barrier: S, and of the
  // result c (CAREFUL) or all but the terms in E
  float out[24];
  if constexpr (CAREFUL) {
    quad_back_mul<lc>(out, v, l1, u1);
    float S[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) S[k] = v[k] + out[k];
    quad_back2_fma<lc>(out, S, l2, u2);
#pragma unroll
    for (int k = 0; k < 24; ++k) S[k] = v[k] + out[k];
    put_ends<DAG>(S, Q);
  } else {
    quad_scan6<true>(v + lc, l1, l2);
    quad_scan6<true>(v + lc + 6, l1, l2);
    quad_scan6<false>(v + uc, u1, u2);
    quad_scan6<false>(v + uc + 6, u1, u2);
    put_ends<DAG>(v, Q);
#pragma unroll
    for (int k = 0; k < 24; ++k) out[k] = add == nullptr ? t0 * v[k] : fmaf(t0, v[k], add[k]);
    if constexpr (SHIFT) quad_back_fma<lc>(out, v, lt, ut);
  }
  __syncthreads();
  // E of reals 6q .. 6q+5
  const bool lower6 = (Q.q < 2) != DAG;
  const int wl = lower6 ? Q.w : Q.nw - 1 - Q.w;  // place along these reals' walk
  const float* t = Q.tot + Q.site * kTotRow + 6 * Q.q;
  float E[6] = {0, 0, 0, 0, 0, 0};
  {
    const float k4 = k2 * k2;
    float wall = -mq * inv_c;
    for (int j = 0; j < wl; ++j) wall *= k4;
    float carry = 1.f;
    for (int o = Q.nw - 1; o >= 0; --o) {
      const float c = wall + (o < wl ? carry : 0.f);
      const float* x = t + (size_t)(lower6 ? o : Q.nw - 1 - o) * 16 * kTotRow;
      const float2 a = *reinterpret_cast<const float2*>(x), b = *reinterpret_cast<const float2*>(x + 2),
                   d = *reinterpret_cast<const float2*>(x + 4);
      E[0] = fmaf(c, a.x, E[0]);
      E[1] = fmaf(c, a.y, E[1]);
      E[2] = fmaf(c, b.x, E[2]);
      E[3] = fmaf(c, b.y, E[3]);
      E[4] = fmaf(c, d.x, E[4]);
      E[5] = fmaf(c, d.y, E[5]);
      wall *= k4;
      carry = o < wl ? carry * k4 : carry;
    }
  }
  const float k3 = nk * k2, k4 = k2 * k2;
  const float pw[5] = {1.f, nk, k2, k3, k4};
  auto pick = [&](int p, int d) {  // (-kappa)^(p + d)
    return p == 0 ? pw[d] : p == 1 ? pw[1 + d] : p == 2 ? pw[2 + d] : pw[3 + d];
  };
  if constexpr (CAREFUL) {
    quad_share_fma<lc>(out, E, pick(pl, 1), pick(pu, 1));
    if constexpr (SHIFT) {  // of ia y; y_{i-1} is the lane before, or E
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fmaf(ia, v[k], ia * out[k]);
      quad_back_mul<lc>(out, v, lt, ut);
      const float te = ia * t1;
      quad_share_fma<lc>(out, E, pl == 0 ? te : 0.f, pu == 0 ? te : 0.f);
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fmaf(t0, v[k], out[k]);
    } else if (add == nullptr) {
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fmaf(t0, v[k], t0 * out[k]);
    } else {
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fmaf(t0, v[k] + out[k], add[k]);
    }
  } else {
    // y_i = S_i + (-kappa)^(i+1) E enters out_i with t0, y_{i-1} with t1
    float el = t0 * pick(pl, 1), eu = t0 * pick(pu, 1);
    if constexpr (SHIFT) {
      el = fmaf(t1, pick(pl, 0), el);
      eu = fmaf(t1, pick(pu, 0), eu);
    }
    quad_share_fma<lc>(out, E, el, eu);
#pragma unroll
    for (int k = 0; k < 24; ++k) v[k] = out[k];
  }
}

// Fixed-order FP64 sum over a wavefront: DPP rows, then across the rows.
__device__ __forceinline__ double wave_sum(double v) {
  v = row_sum16(v);
  v += __shfl_xor(v, 16);
  v += __shfl_xor(v, 32);
  return v;
}

// What a launch computes after the hop h (see DslashArgs for the operators).
enum QuadProg : int {
  QP_HOP = 0,   // h
  QP_A1 = 1,    // M_phi M5^-1 h
  QP_A2 = 2,    // aux + coef_y M5^-1 h
  QP_A2C = 3,   // M5^-T (aux + coef_y M5^-1 h)
  QP_B1 = 4,    // M_phi^T M5^-T h
  QP_B2 = 5,    // M5^T aux + coef_y M_phi^T h
  QP_B2C = 6,   // the same into r -= alpha (.) instead of out
  QP_D = 7,     // M5 aux + coef_y h (32-bit storage: with 16 bits M_phi is a prologue of the general kernel)
  QP_PRE = 8,   // M5^-1 (aux + coef_y h) (likewise)
};
constexpr bool prog_dag(int p) { return p == QP_B1 || p == QP_B2 || p == QP_B2C; }

constexpr int kQuadThreads = 1024;
// Resident waves per SIMD the register allocation must leave room for.
template <int P> constexpr int kQuadWaves = is16(P) ? 5 : 4;

template <int P, int PROG, bool DAG>
__global__ __launch_bounds__(kQuadThreads) __attribute__((amdgpu_waves_per_eu(kQuadWaves<P>))) void dslash_quad_kernel(
    DslashArgs A) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int CB = 1 << A.cb_log2;
  const int L5 = A.g.L5, nw = L5 >> 2;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  if (lb >= A.nslots * A.nblk) return;
  int slot, blk;
  block_slot(A, lb, slot, blk);
  constexpr bool kAux = PROG != QP_HOP && PROG != QP_A1 && PROG != QP_B1;
  const SlotIO io = slot_io<kAux, PROG == QP_B2C, PROG == QP_B1 || PROG == QP_B2C>(A, slot);
  const int cb0 = block_first_site(A, blk, CB);
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sub = wave / nw;  // 16-site tile of the workgroup
  const int w = wave - sub * nw;
  const int lane = tid & 63, site = lane >> 2, q = lane & 3;
  const int cbl = sub * 16 + site;
  const int tile = __builtin_amdgcn_readfirstlane((cb0 >> 4) + sub);
  const bool valid = cb0 + cbl < A.g.Vh;
  const uint32_t lo = q * 16, ls = q * 4;  // the lane's slice
  const uint32_t oo = (lane >> 4) * kSliceBytes<P> + (lane & 15) * 16, os = lane * 4;  // its own site and slice
  const Coef5 cf = A.coef[slot];
  const float mq = (float)cf.mq;

  uint32_t* nbr = reinterpret_cast<uint32_t*>(smem + CB * kLinkRow<P> * 4);
  uint32_t* lnk = reinterpret_cast<uint32_t*>(smem);
  float* tot = reinterpret_cast<float*>(smem + stage_bytes<P>(CB));
  double* red = reinterpret_cast<double*>(smem + stage_bytes<P>(CB) + totals_bytes(CB, L5));
  const size_t tot_tile = (size_t)sub * nw * 16 * kTotRow;

  fill_stage<P>(A, nbr, lnk, CB, A.cb_log2, cb0, tid, nthr);
  if (io.active == 0) return;  // after the stage: its loads do not wait for the flag
  __syncthreads();

  float v[24];
  {
    Cplx<float> acc[4][3];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) acc[a][b] = {0, 0};
    const Base in = field_base<P>(io.in, A.g, w);
    hop_all<P, DAG, kQuadBatch, 0>(in, nbr + cbl * kNbrRow, lnk + cbl * kLinkRow<P>, q, lo, ls, acc);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      v[2 * k] = acc[k / 3][k % 3].re;
      v[2 * k + 1] = acc[k / 3][k % 3].im;
    }
  }

  // a lane of a ragged tile's tail works on padding: its own site of the
  // last tile is allocated, so its reads stay inside the field
  const QuadPos Q{q, w, nw, site, tot + tot_tile};
  const float kappa = (float)cf.kappa, inv_c = (float)cf.inv_c;
  constexpr bool kCareful = P == F32;
  // M_phi M5^-1 and its transpose: coefficients rounded to FP32 once
  const float ia = (float)cf.inv_alpha;
  const float b5a = (float)(kCareful ? cf.b5 : cf.b5 * cf.inv_alpha), c5a = (float)(kCareful ? cf.c5 : cf.c5 * cf.inv_alpha);
  const bool in_tile = tile < ((A.g.Vh + 15) >> 4);
  if constexpr (PROG == QP_A1) {
    quad_solve<true, false, kCareful>(v, nullptr, Q, kappa, mq, inv_c, b5a, c5a, ia);
  } else if constexpr (PROG == QP_B1) {
    quad_solve<true, true, kCareful>(v, nullptr, Q, kappa, mq, inv_c, b5a, c5a, ia);
  } else if constexpr (PROG == QP_A2 || PROG == QP_A2C) {
    Raw<P> ar{};
    if (in_tile) load_raw<P>(at_tile<P>(field_base<P>(io.aux, A.g, w), tile, L5), oo, os, ar);
    float aux[24];
    unpack<P>(ar, aux);
    quad_solve<false, false, kCareful>(v, aux, Q, kappa, mq, inv_c, (float)(A.coef_y * cf.inv_alpha), 0.f);
  } else if constexpr (PROG == QP_B2 || PROG == QP_B2C) {
    // M5^T aux + coef_y M_phi^T h = (alpha aux + coef_y b5 h) + shift(beta aux + coef_y c5 h)
    Raw<P> ar{};
    if (in_tile) load_raw<P>(at_tile<P>(field_base<P>(io.aux, A.g, w), tile, L5), oo, os, ar);
    float aux[24], add[24];
    unpack<P>(ar, aux);
    const float al = (float)cf.alpha, be = (float)cf.beta;
    const float b5y = (float)(A.coef_y * cf.b5), c5y = (float)(A.coef_y * cf.c5);
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      add[k] = kCareful ? b5y * v[k] : fmaf(al, aux[k], b5y * v[k]);
      v[k] = fmaf(be, aux[k], c5y * v[k]);
    }
    quad_shift<true>(v, add, Q, mq);
    if constexpr (kCareful) {  // the largest term last
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fmaf(al, aux[k], v[k]);
    }
  } else if constexpr (PROG == QP_D || PROG == QP_PRE) {
    Raw<P> ar{};
    if (in_tile) load_raw<P>(at_tile<P>(field_base<P>(io.aux, A.g, w), tile, L5), oo, os, ar);
    float aux[24], add[24];
    unpack<P>(ar, aux);
    const float al = (float)cf.alpha, be = (float)cf.beta, cy = (float)A.coef_y;
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      add[k] = PROG == QP_D ? cy * v[k] : aux[k] + cy * v[k];
      v[k] = PROG == QP_D ? be * aux[k] : add[k];
    }
    if constexpr (PROG == QP_D) {
      quad_shift<false>(v, add, Q, mq);
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = fmaf(al, aux[k], v[k]);
    } else quad_solve<false, false, kCareful>(v, nullptr, Q, kappa, mq, inv_c, (float)cf.inv_alpha, 0.f);
  }

  if constexpr (PROG == QP_B2C) {
    if (valid) {
      const float alpha = (float)io.alpha;
      const Base rb = at_tile<P>(field_base<P>(io.r, A.g, w), tile, L5);
      Raw<P> rr;
      load_raw<P>(rb, oo, os, rr);
      float rv[24];
      unpack<P>(rr, rv);
#pragma unroll
      for (int k = 0; k < 24; ++k) v[k] = rv[k] - alpha * v[k];
      store_own<P>(rb, oo, os, v, A.nt_store);
    }
  }

  if (A.reduce) {
    // 24 squares per thread in FP32, everything above in FP64, one sum per
    // wavefront; the tile's wavefronts are added in order, so the partial of a
    // tile does not depend on the workgroup's width
    float lr = 0;
#pragma unroll
    for (int k = 0; k < 24; ++k) lr += v[k] * v[k];
    const double sum = wave_sum(valid ? (double)lr : 0.0);
    if (lane == 0) red[wave] = sum;
    __syncthreads();
    if (w == 0 && lane == 0 && in_tile) {
      double s = 0;
      for (int k = 0; k < nw; ++k) s += red[wave + k];
      A.partials[(size_t)slot * A.ntiles + tile] = s;
    }
  }

  if constexpr (PROG == QP_A2C) {
    QuadPos Q2 = Q;
    Q2.tot = reinterpret_cast<float*>(smem) + tot_tile;  // over the stage, dead since the first chain's barrier
    quad_solve<false, true, kCareful>(v, nullptr, Q2, kappa, mq, inv_c, (float)cf.inv_alpha, 0.f);
  }
  if constexpr (PROG != QP_B2C) {
    if (valid) store_own<P>(at_tile<P>(field_base<P>(io.out, A.g, w), tile, L5), oo, os, v, A.nt_store);
  }
  if ((PROG == QP_B1 && A.cg_update == 3) || (PROG == QP_B2C && A.cg_update == 1)) {
    if (valid && io.phase != 0) {  // x += alpha_prev p + alpha p2
      const float a0 = (float)io.alpha_prev, a1 = (float)io.alpha;
      const Base b0 = at_tile<P>(field_base<P>(io.p, A.g, w), tile, L5);
      const Base b1 = at_tile<P>(field_base<P>(io.p2, A.g, w), tile, L5);
      const Base xb = at_tile<F32>(field_base<F32>(io.x, A.g, w), tile, L5);
      const uint32_t xo = (lane >> 4) * kSliceBytes<F32> + (lane & 15) * 16;
      // group by group: a few registers at a time
      Raw<P> r0, r1;
      if constexpr (is16(P)) {
        r0.sc = ldo<float>(b0.s, os, 0);
        r1.sc = ldo<float>(b1.s, os, 0);
      }
#pragma unroll
      for (int k = 0; k < kGroups<P>; ++k) {
        constexpr int N = 24 / kGroups<P>;
        float p0[N], p1[N];
        unpack_group<P>(ldo<v4u>(b0.d, oo, k * 16 * kSiteTile), r0.sc, p0);
        unpack_group<P>(ldo<v4u>(b1.d, oo, k * 16 * kSiteTile), r1.sc, p1);
#pragma unroll
        for (int j = 0; j < N / 4; ++j) {
          const int imm = (k * (N / 4) + j) * 16 * kSiteTile;
          v4f x = ldo<v4f>(xb.d, xo, imm);
#pragma unroll
          for (int i = 0; i < 4; ++i) x[i] = (x[i] + a0 * p0[4 * j + i]) + a1 * p1[4 * j + i];
          sto<v4f>(xb.d, xo, imm, x, A.nt_store);
        }
      }
    }
  }
}

template <int P, int PROG, bool DAG>
hipError_t launch_q(const DslashArgs& A, int threads, int grid, hipStream_t st) {
  const size_t smem = lds_bytes<P>(1 << A.cb_log2, A.g.L5);
  auto k = dslash_quad_kernel<P, PROG, DAG>;
  if (smem > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
  }
  launch_k(k, dim3(grid), dim3(threads), smem, st, A);
  return hipGetLastError();
}

// the program of a launch, or -1 where it has none here
int quad_prog(const DslashArgs& A, bool dag) {
  if (!dag) {
    if (A.cg_update != 0 && !(A.cg_update == 4 && A.c1 == CH_M5INV)) return -1;
    if (A.c1 == CH_NONE && A.c2 == CH_NONE && A.aux_mode == AUX_NONE && A.coef_y == 1.0) return QP_HOP;
    if (A.c1 == CH_MPHI_M5INV && A.c2 == CH_NONE && A.aux_mode == AUX_NONE && A.coef_y == 1.0) return QP_A1;
    if (A.c1 == CH_M5INV && A.aux_mode == AUX_PLAIN && (A.c2 == CH_NONE || A.c2 == CH_M5INV_DAG))
      return A.c2 == CH_NONE ? QP_A2 : QP_A2C;
    if (A.c1 == CH_NONE && A.c2 == CH_NONE && A.aux_mode == AUX_M5) return QP_D;
    if (A.c1 == CH_NONE && A.c2 == CH_M5INV && A.aux_mode == AUX_PLAIN) return QP_PRE;
    return -1;
  }
  if (A.c2 != CH_NONE) return -1;
  if (A.c1 == CH_NONE && A.aux_mode == AUX_NONE && A.coef_y == 1.0 && A.cg_update == 0) return QP_HOP;
  if (A.c1 == CH_MPHIDAG_M5INVDAG && A.aux_mode == AUX_NONE && A.coef_y == 1.0 && (A.cg_update == 0 || A.cg_update == 3))
    return QP_B1;
  if (A.c1 == CH_MPHI_DAG && A.aux_mode == AUX_M5DAG) return A.cg_update == 0 ? QP_B2 : A.cg_update <= 2 ? QP_B2C : -1;
  return -1;
}

template <int P> hipError_t launch_qp(const DslashArgs& A, bool dag, int threads, int grid, hipStream_t st) {
  switch (quad_prog(A, dag)) {
    case QP_HOP: return dag ? launch_q<P, QP_HOP, true>(A, threads, grid, st) : launch_q<P, QP_HOP, false>(A, threads, grid, st);
    case QP_A1: return launch_q<P, QP_A1, false>(A, threads, grid, st);
    case QP_A2: return launch_q<P, QP_A2, false>(A, threads, grid, st);
    case QP_A2C: return launch_q<P, QP_A2C, false>(A, threads, grid, st);
    case QP_B1: return launch_q<P, QP_B1, true>(A, threads, grid, st);
    case QP_B2: return launch_q<P, QP_B2, true>(A, threads, grid, st);
    case QP_B2C: return launch_q<P, QP_B2C, true>(A, threads, grid, st);
    case QP_D:
      if constexpr (P == F32) return launch_q<P, QP_D, false>(A, threads, grid, st);
      break;
    case QP_PRE:
      if constexpr (P == F32) return launch_q<P, QP_PRE, false>(A, threads, grid, st);
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace

// The launches this kernel takes: the staged hop without the split and without
// the M_phi prologue, 32- and 16-bit storage, L5 a multiple of 4, neighbour offsets
// that fit 32 bits (fields under 4 GB), and a second chain's totals that fit
// the stage they overlay (all but L5 = 32 of FP32 and int16).
bool dslash_quad_ok(const DslashArgs& A, int prec, bool hop, bool dag) {
  if (!hop || A.pro || !A.stage || A.split_mask != 0 || prec == F64 || A.g.L5 % 4 != 0 || kSiteTile != 16) return false;
  if (spinor_field_bytes(prec, A.g.L5, A.g.Vh) >= ((size_t)1 << 32)) return false;
  const size_t stage = prec == F32 || prec == I16 ? stage_bytes<F32>(16) : stage_bytes<F16>(16);
  if (totals_bytes(16, A.g.L5) > stage) return false;
  const int prog = quad_prog(A, dag);
  return prog >= 0 && (prec == F32 || (prog != QP_D && prog != QP_PRE));
}

size_t dslash_quad_lds_bytes(int prec, int CB, int L5) {
  return prec == F32 || prec == I16 ? lds_bytes<F32>(CB, L5) : lds_bytes<F16>(CB, L5);
}

hipError_t dslash_quad_launch(const DslashArgs& A, int prec, bool dag, int threads, int grid, hipStream_t st) {
  switch (prec) {
    case F32: return launch_qp<F32>(A, dag, threads, grid, st);
    case F16: return launch_qp<F16>(A, dag, threads, grid, st);
    case BF16: return launch_qp<BF16>(A, dag, threads, grid, st);
    case I16: return launch_qp<I16>(A, dag, threads, grid, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace mdwf
