// mdwf_dslash: the operators of the even-odd preconditioned Moebius
// domain-wall system, each built from the fused stencil kernel.
#include <cstring>
#include <mutex>

#include "internal.h"

using namespace mdwf;

namespace mdwf {

// The programs that compose the operators (see DslashArgs); the inputs of the
// first three hold M_phi of the field already (the conversion from the user
// layout, the CG's p-update and the reliable update write it), or the hop
// applies it (with_phi: mdwf_dslash on 16-bit storage, where a stored M_phi psi
// would round it to 16 bits before the projection):
//   D    : M5 aux - 1/2 H in                          (aux M5, coef -1/2)
//   A1   : t_o = M_phi M5^-1 H_oe in_e                (c1 M_phi M5^-1)
//   PRE  : out = M5^-1 (aux + 1/2 H in)               (aux, c2 M5^-1)
//   D^+  : M5^T aux - 1/2 M_phi^T H^+ in              (DAG, c1 M_phi^T, aux M5^T)
//   A2   : u = aux - 1/4 M5^-1 H_eo t_o, out M5^-T u  (c1 M5^-1, aux, c2 M5^-T)
//   B1   : w_o = M_phi^T M5^-T H^+_oe v_e             (DAG, c1 M_phi^T M5^-T)
//   B2   : q = M5^T v - 1/4 M_phi^T H^+_eo w_o        (DAG, c1 M_phi^T, aux M5^T)
// so that M^ p = A2 without c2, and M^+ y = B2(B1(M5^-T y)).
Prog prog_D(int par) { return Prog{true, false, CH_NONE, CH_NONE, AUX_M5, 0, -0.5, par}; }
Prog prog_Ddag(int par) { return Prog{true, true, CH_MPHI_DAG, CH_NONE, AUX_M5DAG, 0, -0.5, par}; }
Prog prog_A1() { return Prog{true, false, CH_MPHI_M5INV, CH_NONE, AUX_NONE, 0, 1.0, 1}; }
Prog prog_A2(bool with_c2, bool reduce) {
  return Prog{true, false, CH_M5INV, with_c2 ? CH_M5INV_DAG : CH_NONE, AUX_PLAIN, reduce ? 1 : 0, -0.25, 0};
}
Prog prog_B1() { return Prog{true, true, CH_MPHIDAG_M5INVDAG, CH_NONE, AUX_NONE, 0, 1.0, 1}; }
Prog prog_B2() { return Prog{true, true, CH_MPHI_DAG, CH_NONE, AUX_M5DAG, 0, -0.25, 0}; }
Prog prog_PRE(int par) { return Prog{true, false, CH_NONE, CH_M5INV, AUX_PLAIN, 0, 0.5, par}; }
static Prog with_phi(Prog p) {
  p.pro = true;
  return p;
}
Prog prog_HOP(int par, bool dag) { return Prog{true, dag, CH_NONE, CH_NONE, AUX_NONE, 0, 1.0, par}; }
Prog prog_5D(int chain) { return Prog{false, false, chain, CH_NONE, AUX_NONE, 0, 1.0, 0}; }

}  // namespace mdwf

// Argument checks shared by mdwf_dslash and its no-allocation variant.
static mdwf_status dslash_check(mdwf_ctx* c, const char* who, const mdwf_gauge* g, const mdwf_action* act,
                                int32_t op, int32_t prec, int32_t nrhs, const void* in, void* out) {
  std::string msg;
  if (check_action_msg(act, msg) != MDWF_OK) return set_err(c, MDWF_EINVAL, "%s: %s", who, msg.c_str());
  if (g == nullptr || in == nullptr || out == nullptr) return set_err(c, MDWF_EINVAL, "%s: NULL argument", who);
  for (int m = 0; m < 4; ++m)
    if (g->L[m] != act->L[m]) return set_err(c, MDWF_EINVAL, "%s: gauge lattice differs from the action's", who);
  if (prec < MDWF_F64 || prec > MDWF_I16) return set_err(c, MDWF_EINVAL, "%s: bad precision", who);
  if (g->data[prec] == nullptr)
    return set_err(c, MDWF_EINVAL, "%s: gauge field was not loaded in precision %d", who, prec);
  if (op < MDWF_OP_D || op > MDWF_OP_PREP) return set_err(c, MDWF_EINVAL, "%s: bad operator %d", who, op);
  if (nrhs < 1) return set_err(c, MDWF_EINVAL, "%s: nrhs must be >= 1", who);
  const Geom geom = make_geom(act);
  const size_t ub = (size_t)geom.Vh * 2 * geom.L5 * 12 * 16;  // user bytes per RHS
  const char* ib = static_cast<const char*>(in);
  const char* ob = static_cast<const char*>(out);
  if (ib < ob + ub * nrhs && ob < ib + ub * nrhs) return set_err(c, MDWF_EINVAL, "%s: in and out overlap", who);
  return MDWF_OK;
}

// The device tables one operator application reads: user fields, the five
// internal half-fields per RHS (in_e, in_o, out_e, out_o, temporary), a table
// of null pointers (a zero parity) and the per-RHS coefficients.
struct DslashTables {
  PtrTab UIN, UOUT, IE, IO, OE, OO, T, NUL;
  CoefTab coef;
};

static mdwf_status dslash_body(mdwf_ctx* c, const mdwf_gauge* g, const Geom& geom, int32_t op, int32_t prec,
                               int32_t nrhs, const DslashTables& t);

extern "C" mdwf_status mdwf_dslash(mdwf_ctx* c, const mdwf_gauge* g, const mdwf_action* act, int32_t op,
                                   int32_t prec, int32_t nrhs, const void* in, void* out) {
  if (c == nullptr) return MDWF_EINVAL;
  mdwf_status st = dslash_check(c, "mdwf_dslash", g, act, op, prec, nrhs, in, out);
  if (st != MDWF_OK) return st;
  const Geom geom = make_geom(act);
  const size_t ub = (size_t)geom.Vh * 2 * geom.L5 * 12 * 16;  // user bytes per RHS
  const char* ib = static_cast<const char*>(in);
  char* ob = static_cast<char*>(out);
  (void)hipSetDevice(c->device);
  reset_tables(c);
  const size_t fb = round_up(spinor_field_bytes(prec, geom.L5, geom.Vh), 256);
  st = ensure(c, c->dws, fb * 5 * nrhs);
  if (st != MDWF_OK) return st;
  const Coef5 coef = make_coef(act);
  std::vector<std::vector<const void*>> p(8, std::vector<const void*>(nrhs, nullptr));
  char* w = static_cast<char*>(c->dws.p);
  for (int r = 0; r < nrhs; ++r) {
    p[0][r] = ib + ub * r;
    p[1][r] = ob + ub * r;
    for (int k = 0; k < 5; ++k) p[2 + k][r] = w + fb * (5 * r + k);
  }
  LaunchTables lt;
  if (!make_tables(c, p, {coef}, lt))
    return set_err(c, MDWF_EHIP, "mdwf_dslash: table upload failed");
  const DslashTables t{lt.tab[0], lt.tab[1], lt.tab[2], lt.tab[3], lt.tab[4], lt.tab[5], lt.tab[6], lt.tab[7], lt.coef};
  return dslash_body(c, g, geom, op, prec, nrhs, t);
}

static mdwf_status dslash_body(mdwf_ctx* c, const mdwf_gauge* g, const Geom& geom, int32_t op, int32_t prec,
                               int32_t nrhs, const DslashTables& t) {
  const PtrTab& UIN = t.UIN;
  const PtrTab& UOUT = t.UOUT;
  const PtrTab& IE = t.IE;
  const PtrTab& IO = t.IO;
  const PtrTab& OE = t.OE;
  const PtrTab& OO = t.OO;
  const PtrTab& T = t.T;
  const PtrTab& NUL = t.NUL;
  const CoefTab& coef = t.coef;
  const int cls = prec == MDWF_F64 ? MDWF_PROF_DSLASH_F64 : MDWF_PROF_DSLASH_INNER;
  const bool pro = prec != MDWF_F64 && prec != MDWF_F32;  // M_phi in the hop, not in a stored field
  hipError_t e = hipSuccess;
  hipEvent_t ev;
  auto conv_in = [&](const PtrTab& even, const PtrTab& odd) {
    if (e != hipSuccess) return;
    prof_begin(c, &ev);
    e = layout_user_to_half(geom, UIN, even, odd, prec, nrhs, c->stream);
    prof_end(c, MDWF_PROF_OTHER, 0, ev);
  };
  // one parity, and M_phi of it
  auto conv_phi = [&](int par, const PtrTab& half, const PtrTab& phi) {
    if (e != hipSuccess) return;
    prof_begin(c, &ev);
    e = layout_user_to_half_phi(geom, UIN, half, phi, coef, par, prec, nrhs, c->stream);
    prof_end(c, MDWF_PROF_OTHER, 0, ev);
  };
  auto run = [&](const Prog& p, const PtrTab& i, const PtrTab& a, const PtrTab& o) {
    if (e != hipSuccess) return;
    e = run_prog(c, g, geom, prec, p, i, a, o, coef, nrhs, nullptr, 0, nullptr, 0, cls, i != o && a != o);
  };
  // IE = the even half, T = M_phi M5^-1 H_oe M_phi of it
  auto mhat_first = [&]() {
    if (pro) {
      conv_in(IE, PtrTab());
      run(with_phi(prog_A1()), IE, PtrTab(), T);
    } else {
      conv_phi(0, IE, IO);
      run(prog_A1(), IO, PtrTab(), T);
    }
  };
  PtrTab res_e = NUL, res_o = NUL;
  switch (op) {
    case MDWF_OP_D:
      if (pro) {
        conv_in(IE, IO);
        run(with_phi(prog_D(0)), IO, IE, OE);
        run(with_phi(prog_D(1)), IE, IO, OO);
        res_e = OE;
        res_o = OO;
        break;
      }
      conv_phi(1, IO, T);
      conv_phi(0, IE, OO);
      run(prog_D(0), T, IE, OE);
      run(prog_D(1), OO, IO, T);
      res_e = OE;
      res_o = T;
      break;
    case MDWF_OP_DDAG:
      conv_in(IE, IO);
      run(prog_Ddag(0), IO, IE, OE);
      run(prog_Ddag(1), IE, IO, OO);
      res_e = OE;
      res_o = OO;
      break;
    case MDWF_OP_MHAT:
      mhat_first();
      run(prog_A2(false, false), T, IE, OE);
      res_e = OE;
      break;
    case MDWF_OP_MHATDAG:
      conv_in(IE, PtrTab());
      run(prog_5D(CH_M5INV_DAG), IE, PtrTab(), OO);
      run(prog_B1(), OO, PtrTab(), T);
      run(prog_B2(), T, OO, OE);
      res_e = OE;
      break;
    case MDWF_OP_NORMAL:
      mhat_first();
      run(prog_A2(true, false), T, IE, OO);
      run(prog_B1(), OO, PtrTab(), T);
      run(prog_B2(), T, OO, OE);
      res_e = OE;
      break;
    case MDWF_OP_HOP_EO:
      conv_in(PtrTab(), IO);
      run(prog_HOP(0, false), IO, PtrTab(), OE);
      res_e = OE;
      break;
    case MDWF_OP_HOP_OE:
      conv_in(IE, PtrTab());
      run(prog_HOP(1, false), IE, PtrTab(), OO);
      res_o = OO;
      break;
    case MDWF_OP_HOP:
    case MDWF_OP_HOPDAG: {
      conv_in(IE, IO);
      const bool dg = op == MDWF_OP_HOPDAG;
      run(prog_HOP(0, dg), IO, PtrTab(), OE);
      run(prog_HOP(1, dg), IE, PtrTab(), OO);
      res_e = OE;
      res_o = OO;
      break;
    }
    case MDWF_OP_M5:
    case MDWF_OP_M5INV:
    case MDWF_OP_MPHI: {
      conv_in(IE, IO);
      const int ch = op == MDWF_OP_M5 ? CH_M5 : op == MDWF_OP_M5INV ? CH_M5INV : CH_MPHI;
      run(prog_5D(ch), IE, PtrTab(), OE);
      run(prog_5D(ch), IO, PtrTab(), OO);
      res_e = OE;
      res_o = OO;
      break;
    }
    case MDWF_OP_PREP:
      conv_in(IE, IO);
      run(prog_5D(pro ? CH_M5INV : CH_MPHI_M5INV), IO, PtrTab(), T);
      run(pro ? with_phi(prog_PRE(0)) : prog_PRE(0), T, IE, OE);
      res_e = OE;
      break;
    default:
      return set_err(c, MDWF_EINVAL, "mdwf_dslash: bad operator");
  }
  if (e == hipSuccess) {
    prof_begin(c, &ev);
    e = layout_half_to_user(geom, res_e, res_o, UOUT, prec, nrhs, c->stream);
    prof_end(c, MDWF_PROF_OTHER, 0, ev);
  }
  return hip_err(c, e, "mdwf_dslash");
}

// ---------------------------------------------------------------------------
// mdwf_dslash without allocation, for callers that cannot allocate: the
// pointer tables, the coefficients and the five internal half-fields per RHS
// live in `scratch`, one fixed array per GPU that the library holds for the
// life of the process.  Host code never names the array's symbol as an
// address: each device's address comes from hipGetSymbolAddress, taken once
// per device when a context is created on it.
// ---------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)256 << 20;  // 256 MiB per GPU
constexpr size_t kScratchTableBytes = (size_t)64 << 10;
constexpr int kScratchMaxRhs = 16;
constexpr int kScratchMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kScratchMaxDevices] = {};
static hipError_t g_scratch_err[kScratchMaxDevices] = {};

// With `device` current: fetch this device's address of `scratch` (once).
void mdwf::scratch_init(int device) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (device < 0 || device >= kScratchMaxDevices || g_scratch_ptr[device] != nullptr) return;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  g_scratch_err[device] = e;
  if (e == hipSuccess) g_scratch_ptr[device] = p;
}

static void* scratch_ptr(int device, hipError_t& err) {
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (device < 0 || device >= kScratchMaxDevices) {
    err = hipErrorInvalidDevice;
    return nullptr;
  }
  err = g_scratch_ptr[device] != nullptr ? hipSuccess : g_scratch_err[device];
  if (g_scratch_ptr[device] == nullptr && err == hipSuccess) err = hipErrorNotInitialized;
  return g_scratch_ptr[device];
}

// The tables travel by value in the kernel arguments and are written into the
// scratch by one small kernel on the caller's stream (no host-to-device copy).
struct ScratchTables {
  const char* ptr[8][kScratchMaxRhs];
  Coef5 coef[kScratchMaxRhs];
};
static_assert(sizeof(ScratchTables) <= 3072, "kernel argument size");
static_assert(8 * kScratchMaxRhs * sizeof(void*) + kScratchMaxRhs * sizeof(Coef5) <= kScratchTableBytes, "tables");

__global__ __launch_bounds__(256) void k_put_tables(ScratchTables t, char* dst) {
  const char** tab = reinterpret_cast<const char**>(dst);
  for (int i = threadIdx.x; i < 8 * kScratchMaxRhs; i += blockDim.x) tab[i] = t.ptr[i / kScratchMaxRhs][i % kScratchMaxRhs];
  Coef5* cf = reinterpret_cast<Coef5*>(dst + 8 * kScratchMaxRhs * sizeof(void*));
  for (int i = threadIdx.x; i < kScratchMaxRhs; i += blockDim.x) cf[i] = t.coef[i];
}

extern "C" mdwf_status mdwf_dslash_noalloc(mdwf_ctx* c, const mdwf_gauge* g, const mdwf_action* act, int32_t op,
                                           int32_t prec, int32_t nrhs, const void* in, void* out) {
  if (c == nullptr) return MDWF_EINVAL;
  mdwf_status st = dslash_check(c, "mdwf_dslash_noalloc", g, act, op, prec, nrhs, in, out);
  if (st != MDWF_OK) return st;
  if (nrhs > kScratchMaxRhs)
    return set_err(c, MDWF_EINVAL, "mdwf_dslash_noalloc: nrhs %d exceeds the maximum of %d", nrhs, kScratchMaxRhs);
  const Geom geom = make_geom(act);
  const size_t ub = (size_t)geom.Vh * 2 * geom.L5 * 12 * 16;
  const size_t fb = round_up(spinor_field_bytes(prec, geom.L5, geom.Vh), 256);
  const size_t need = kScratchTableBytes + fb * 5 * (size_t)nrhs;
  if (need > kScratchBytes)
    return set_err(c, MDWF_EINVAL, "mdwf_dslash_noalloc: needs %zu bytes of scratch, more than the %zu it holds", need,
                   kScratchBytes);
  (void)hipSetDevice(c->device);
  hipError_t e = hipSuccess;
  char* base = static_cast<char*>(scratch_ptr(c->device, e));
  if (base == nullptr) return hip_err(c, e, "mdwf_dslash_noalloc: scratch address");
  const char* ib = static_cast<const char*>(in);
  const char* ob = static_cast<const char*>(out);
  char* w = base + kScratchTableBytes;
  const Coef5 coef = make_coef(act);
  DslashTables d;
  if (nrhs == 1) {  // the pointers travel in the launches
    d = DslashTables{PtrTab::single(ib), PtrTab::single(ob), PtrTab::single(w), PtrTab::single(w + fb),
                     PtrTab::single(w + fb * 2), PtrTab::single(w + fb * 3), PtrTab::single(w + fb * 4), PtrTab(),
                     CoefTab::single(coef)};
  } else {
    ScratchTables t{};
    for (int r = 0; r < nrhs; ++r) {
      t.ptr[0][r] = ib + ub * r;
      t.ptr[1][r] = ob + ub * r;
      for (int k = 0; k < 5; ++k) t.ptr[2 + k][r] = w + fb * (5 * r + k);
      t.ptr[7][r] = nullptr;
      t.coef[r] = coef;
    }
    launch_k(k_put_tables, dim3(1), dim3(256), 0, c->stream, t, base);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_err(c, e, "mdwf_dslash_noalloc: table kernel");
    char* const* tab = reinterpret_cast<char* const*>(base);
    PtrTab p[8];
    for (int k = 0; k < 8; ++k) p[k] = PtrTab(tab + k * kScratchMaxRhs);
    d = DslashTables{p[0], p[1], p[2], p[3], p[4], p[5], p[6], p[7],
                     CoefTab(reinterpret_cast<const Coef5*>(base + 8 * kScratchMaxRhs * sizeof(void*)))};
  }
  // kernel timing would create HIP events: it is left off for this call
  const int prof = c->prof;
  c->prof = 0;
  st = dslash_body(c, g, geom, op, prec, nrhs, d);
  c->prof = prof;
  return st;
}

// The hop H_eo computed the way one rank of a domain-decomposed run computes
// it, with the lattice as its own neighbour in every split dimension: pack the
// faces, run the interior hop without the hops across split boundaries, and
// add those from the faces.  The faces are read back from the packing buffer
// itself (the exchange between ranks is the one step one GPU cannot show).
extern "C" mdwf_status mdwf_hop_split(mdwf_ctx* c, const mdwf_gauge* g, const mdwf_action* act, int32_t prec,
                                      int32_t split_mask, int32_t nrhs, const void* in, void* out,
                                      double* phase_ms) {
  if (c == nullptr) return MDWF_EINVAL;
  std::string msg;
  if (check_action_msg(act, msg) != MDWF_OK) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: %s", msg.c_str());
  if (split_mask < 0 || split_mask > 15) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: split_mask must be in [0, 15]");
  for (int m = 0; m < 4; ++m)
    if (((split_mask >> m) & 1) && act->L[m] % 2 != 0)
      return set_err(c, MDWF_EINVAL, "mdwf_hop_split: a split dimension needs an even extent");
  if ((split_mask & 1) && act->L[1] % 2 != 0)
    return set_err(c, MDWF_EINVAL, "mdwf_hop_split: splitting x needs an even Ly (face indexing)");
  if (g == nullptr || in == nullptr || out == nullptr) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: NULL argument");
  for (int m = 0; m < 4; ++m)
    if (g->L[m] != act->L[m]) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: gauge lattice differs from the action's");
  if (prec < MDWF_F64 || prec > MDWF_I16) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: bad precision");
  if (g->data[prec] == nullptr)
    return set_err(c, MDWF_EINVAL, "mdwf_hop_split: gauge field was not loaded in precision %d", prec);
  if (nrhs < 1) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: nrhs must be >= 1");
  {
    const char* e = getenv("MDWF_STAGE");
    if (split_mask != 0 && e != nullptr && e[0] == '0')
      return set_err(c, MDWF_EINVAL, "mdwf_hop_split: the split interior needs the staged stencil (MDWF_STAGE=0)");
  }
  const Geom geom = make_geom(act);
  const size_t ub = (size_t)geom.Vh * 2 * geom.L5 * 12 * 16;
  const char* ib = static_cast<const char*>(in);
  char* ob = static_cast<char*>(out);
  if (ib < ob + ub * nrhs && ob < ib + ub * nrhs) return set_err(c, MDWF_EINVAL, "mdwf_hop_split: in and out overlap");
  (void)hipSetDevice(c->device);
  reset_tables(c);
  DDArgs D{};
  D.g = geom;
  D.out_par = 0;
  D.split_mask = split_mask;
  D.gauge = static_cast<const char*>(g->data[prec]);
  D.nslots = nrhs;
  const int Ls[4] = {geom.Lx, geom.Ly, geom.Lz, geom.Lt};
  const size_t rb = prec == MDWF_F64 ? 8 : 4;
  size_t hb = 0;  // face buffer bytes per RHS
  for (int m = 0; m < 4; ++m) {
    D.face_n[m] = (int)((size_t)geom.Vh * 2 / Ls[m] / 2);
    for (int fb = 0; fb < 2; ++fb) {
      D.face_off[2 * m + fb] = hb;
      if ((split_mask >> m) & 1) hb += round_up((size_t)D.face_n[m] * geom.L5 * 12 * rb, 256);
    }
  }
  const size_t fb = round_up(spinor_field_bytes(prec, geom.L5, geom.Vh), 256);
  const size_t hb_r = round_up(hb, 256);
  mdwf_status st = ensure(c, c->dws, (fb * 2 + hb_r) * nrhs);
  if (st != MDWF_OK) return st;
  const Coef5 coef = make_coef(act);
  std::vector<const void*> uin(nrhs), uout(nrhs), io(nrhs), oe(nrhs), hal(nrhs), nul(nrhs, nullptr);
  char* w = static_cast<char*>(c->dws.p);
  for (int r = 0; r < nrhs; ++r) {
    uin[r] = ib + ub * r;
    uout[r] = ob + ub * r;
    io[r] = w + (fb * 2 + hb_r) * r;
    oe[r] = w + (fb * 2 + hb_r) * r + fb;
    hal[r] = w + (fb * 2 + hb_r) * r + 2 * fb;
  }
  LaunchTables lt;
  if (!make_tables(c, {uin, uout, io, oe, hal, nul}, {coef}, lt, true))
    return set_err(c, MDWF_EHIP, "mdwf_hop_split: table upload failed");
  const PtrTab &UIN = lt.tab[0], &UOUT = lt.tab[1], &IO = lt.tab[2], &OE = lt.tab[3], &HAL = lt.tab[4], &NUL = lt.tab[5];
  D.in = IO.t;
  D.out = OE.t;
  D.send = HAL.t;
  D.recv = HAL.t;  // every split neighbour is the lattice itself
  const int cls = prec == MDWF_F64 ? MDWF_PROF_DSLASH_F64 : MDWF_PROF_DSLASH_INNER;
  hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
  if (phase_ms != nullptr)
    for (auto& x : ev) (void)hipEventCreate(&x);
  hipError_t e = layout_user_to_half(geom, UIN, PtrTab(), IO, prec, nrhs, c->stream);
  if (e == hipSuccess && ev[0]) e = hipEventRecord(ev[0], c->stream);
  if (e == hipSuccess && split_mask != 0) e = dd_pack(D, prec, c->stream);
  if (e == hipSuccess && ev[1]) e = hipEventRecord(ev[1], c->stream);
  if (e == hipSuccess) {
    Prog p = prog_HOP(0, false);
    p.split = split_mask;
    e = run_prog(c, g, geom, prec, p, IO, PtrTab(), OE, lt.coef, nrhs, nullptr, 0, nullptr, 0, cls, false);
  }
  if (e == hipSuccess && ev[2]) e = hipEventRecord(ev[2], c->stream);
  if (e == hipSuccess && split_mask != 0) e = dd_exterior(D, prec, c->stream);
  if (e == hipSuccess && ev[3]) e = hipEventRecord(ev[3], c->stream);
  if (e == hipSuccess) e = layout_half_to_user(geom, OE, NUL, UOUT, prec, nrhs, c->stream);
  if (phase_ms != nullptr) {
    if (e == hipSuccess) e = hipEventSynchronize(ev[3]);
    for (int k = 0; k < 3; ++k) {
      float ms = 0;
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, ev[k], ev[k + 1]);
      phase_ms[k] = ms;
    }
    for (auto& x : ev) (void)hipEventDestroy(x);
  }
  return hip_err(c, e, "mdwf_hop_split");
}
