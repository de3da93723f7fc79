// Host runtime of the mu-mode library: contexts, prepared operators,
// argument validation and dispatch of the mode-product kernels.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <map>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include <mutex>

#include "../../include/mumode.h"
#include "mm_internal.h"

// Device memory of gpe_strang_step_noalloc: the FP16X2 running-bound slots
// (3 x SMAX_SLOT words) and the max-abs pass's partial maxima, in a
// file-scope array each GPU holds for the life of the process, so that call
// allocates nothing.  Host code never uses the array's name as an address:
// the device address comes from hipGetSymbolAddress, once per device.
constexpr int NOALLOC_SCRATCH_WORDS = 3 * mm::SMAX_SLOT + 1024;
static __device__ __align__(256) uint32_t scratch[NOALLOC_SCRATCH_WORDS];

struct mm_op_s {
  int64_t rows = 0, cols = 0;
  int cplx = 0;
  mm_prec prec = MM_PREC_FP64;
  int lay = 0;                   // layout of prep: mm::KPrec or mm::KLayout code
  double* dev_master = nullptr;  // FP64 master on the device, ld = rows
  void* prep = nullptr;          // fragment-order operator (own complexity)
  int KBT = 0, MFT = 0;
  int a_exp = 0;                 // FP16X2: the pieces represent L * 2^-a_exp
  double log2_norm = 0.0;        // log2 of a bound of ||L||_2, sqrt(||L||_1 ||L||_inf)
  int res_id = 0;                // resident layout: prep holds L - I though the master does not
  int res_c4 = 0;                // resident layout: four-product form
  int idsplit = 0;               // the master and pieces hold L - I; products add the input back
  void* prep_c = nullptr;        // real master promoted to complex (lazily)
  int KBT_c = 0, MFT_c = 0;
  double* dev_master_c = nullptr;
  // three-product (Gauss) preparation of a complex split operator: Re L, Im L
  // and Re L + Im L (none for real operators or the identity split)
  void* prep_g = nullptr;
  int JBT_g = 0, MFT_g = 0;
  int a_exp_g = 0;               // FP16X2: scale chosen from max(|Re|, |Im|, |Re + Im|)
};

struct mm_ctx_s {
  int device = 0;
  std::string err;
  std::vector<mm_op> ops;
  void* ws = nullptr;            // ping-pong buffer for products that cannot run in place
  size_t ws_bytes = 0;
  bool ws_user = false;          // ws belongs to the caller (mm_set_workspace)
  // autotuned tile class per problem shape: key (precision, complex, load
  // path, real rows Mr, real columns Kr, fibres F) -> (class, microseconds)
  std::map<std::array<int64_t, 6>, std::pair<int, double>> tune;
  int force_cls = -1;            // set while the autotuner times a class
  std::string tune_path;         // tune cache file (mm_create), "" if none
  std::array<int64_t, 6> last_key{};   // tune key of the last planned product
  bool small_run = true;         // several steps of a mode per launch (FP64 / FP32 expsteps)
  // in-call monitor (MM_OPT_MONITOR_EVERY): sum |T|^2 every mon_every steps
  // of mumode_expstep / gpe_strang_step, kept on the device until the call ends
  int mon_every = 0;
  // MM_OPT_FP16X2_CHAIN: an expstep / GPE call on the tensor the previous
  // such call ended with continues its FP16X2 running bound
  bool keep_chain = false;
  double* mon_dev = nullptr;
  size_t mon_cap = 0;
  std::vector<int> mon_steps;
  std::vector<double> mon_vals;
  double* red_partial = nullptr;
  double* red_result = nullptr;
  double* host_result = nullptr; // pinned
  // FP16X2 state bounds: three slots of SMAX_WORDS words rotate along a
  // chain of products (launch k reads slot k % 3, raises (k + 1) % 3,
  // clears (k + 2) % 3); words [3 SMAX_SLOT, + norm_partials()) are the
  // max-abs pass's partial maxima.  chain_end is the
  // output of the chain's last launch: a product whose input is anything
  // else (or the first one of an API call) starts a new chain with a
  // max-abs pass over its input.
  uint32_t* smax = nullptr;
  uint32_t* smax_static = nullptr;  // device address of `scratch` on this context's device
  const void* chain_end = nullptr;
  int sidx = 0;
  // device matrix exponential scratch: X, T, W (complex FP64 n x n each),
  // the prepared X / T, column sums
  double* ex_buf = nullptr;
  size_t ex_bytes = 0;
  void* ex_prep = nullptr;
  size_t ex_prep_bytes = 0;
  // mumode_magnus_step: generators and diagonals (device, pinned staging),
  // prepared exponentials of a block of steps, one exponential above EXPM_MAX_N
  void* mg_buf = nullptr;
  void* mg_stage = nullptr;
  void* mg_prep = nullptr;
  double* mg_exp = nullptr;
  size_t mg_bytes = 0, mg_stage_bytes = 0, mg_prep_bytes = 0, mg_exp_bytes = 0;
  size_t ex_failed = SIZE_MAX, mg_prep_failed = SIZE_MAX;   // see grow_units
  // operators re-prepared every step (ho_strang_step), a block of steps of all modes
  void* step_prep = nullptr;
  size_t step_prep_bytes = 0, step_prep_failed = SIZE_MAX;   // see grow_units
  // ho_strang_step: per mode, the collapsed propagator Psi diag(exp(-i tau
  // (k + 1/2))) Phi (FP64 complex master on the device) for the operators,
  // tau and precision of the last call that formed it
  struct HoMode {
    mm_op phi = nullptr, psi = nullptr;
    double tau = 0.0;
    int prec = -1;
    double* master = nullptr;
    size_t master_bytes = 0;
    double off = -1.0, all = 0.0;   // FP32: ||L - I||_F^2, ||L||_F^2 of the collapsed propagator (-1: not known)
    mm_op_s op;
  };
  HoMode ho[MM_MAXD];
  double* x2 = nullptr;          // squared node coordinates, MM_MAXD * 4096 doubles
  double* x2_stage = nullptr;    // pinned staging of x2
  hipEvent_t x2_ev = nullptr;    // the last upload from x2_stage
  std::vector<double> x2_nodes[MM_MAXD];   // nodes of the last upload, per mode
  // vortex_strang_step: inverse dual-cell widths per mode (device, MM_MAXD *
  // 4096 doubles), uploaded from pinned staging when the weights change
  double* winv = nullptr;
  double* winv_stage = nullptr;
  hipEvent_t winv_ev = nullptr;
  std::vector<double> winv_w[MM_MAXD];
  // batched integrator: work items of the last batch signature, its
  // launch groups and the captured per-step graph
  struct BatchGroup { mm::ModePlan plan; int ida, offset, count; size_t lds; };
  mm::BatchItem* bitems = nullptr;
  size_t bitems_cap = 0;
  mm::ResArgs* rargs = nullptr;   // resident-tile products of the batch and their tiles
  mm::ResItem* ritems = nullptr;
  size_t rargs_cap = 0, ritems_cap = 0;
  std::vector<BatchGroup> bgroups;
  std::vector<uint64_t> bsig;
  hipGraph_t bgraph = nullptr;
  hipGraphExec_t bexec = nullptr;
  // tile class of the batched step's products per (mode, complex), chosen by
  // mm_autotune_batched (-1: the planner's choice)
  int batch_cls[MM_MAXD][2] = {{-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}};
  hipStream_t cap_stream = nullptr;
  // optional per-launch timing (mm_profile_begin / mm_profile_end)
  bool profiling = false;
  struct Rec { int kind; hipEvent_t a, b; };
  std::vector<Rec> recs;
};

namespace {

std::string g_create_err;

// Device address of `scratch` per device, looked up once per device with
// that device current.
std::mutex g_scratch_mu;
std::map<int, uint32_t*> g_scratch_addr;

hipError_t scratch_address(int device, uint32_t** out) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  auto it = g_scratch_addr.find(device);
  if (it != g_scratch_addr.end()) {
    *out = it->second;
    return hipSuccess;
  }
  void* p = nullptr;
  hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_addr[device] = (uint32_t*)p;
  *out = (uint32_t*)p;
  return hipSuccess;
}

mm_status fail(mm_ctx ctx, mm_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (ctx) ctx->err = buf;
  else g_create_err = buf;
  // (a failed allocation's error is reported here, not by the next launch)
  if (st == MM_ERR_NOMEM) (void)hipGetLastError();
  return st;
}

#define HIPCHK(ctx, call)                                                              \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess)                                                              \
      return fail(ctx, MM_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e_));    \
  } while (0)

int kprec(mm_prec p) {
  switch (p) {
    case MM_PREC_FP64: return mm::KP_F64;
    case MM_PREC_FP32: return mm::KP_F32;
    case MM_PREC_SPLIT_BF16X3: return mm::KP_BF16X3;
    case MM_PREC_SPLIT_FP16X2: return mm::KP_FP16X2;
    default: return mm::KP_BF16;
  }
}

// Layout an operator of this shape is prepared in: the resident-tile kernels'
// for FP64 and FP32 up to their longest side, else the precision's own.
int op_layout(mm_prec p, int64_t rows, int64_t cols, int cplx) {
  if (mm::res_fits(rows, cols, cplx)) {
    if (p == MM_PREC_FP64) return mm::KY_RES64;
    if (p == MM_PREC_FP32) return mm::KY_RES32;
  }
  return kprec(p);
}
bool is_res(int lay) { return lay == mm::KY_RES64 || lay == mm::KY_RES32; }
void layout_blocks(int lay, int64_t rows, int64_t cols, int cplx, int* KBT, int* MFT) {
  if (is_res(lay)) mm::res_blocks(lay, rows, cols, cplx, KBT, MFT);
  else mm::op_blocks(lay, (cplx ? 2 : 1) * rows, (cplx ? 2 : 1) * cols, KBT, MFT);
}

bool is_complex(mm_dtype t) { return t == MM_C64 || t == MM_C128; }
bool is_f64(mm_dtype t) { return t == MM_R64 || t == MM_C128; }
size_t dsize(mm_dtype t) { return t == MM_R32 ? 4 : (t == MM_C128 ? 16 : 8); }

int64_t numel(const mm_tensor* T) {
  int64_t n = 1;
  for (int k = 0; k < T->d; ++k) n *= T->dims[k];
  return n;
}

mm_status check_tensor(mm_ctx ctx, const mm_tensor* T, const char* name) {
  if (!T) return fail(ctx, MM_ERR_ARG, "%s is NULL", name);
  if (T->d < 1 || T->d > MM_MAXD) return fail(ctx, MM_ERR_SHAPE, "%s: d = %d outside [1, %d]", name, T->d, MM_MAXD);
  for (int k = 0; k < T->d; ++k)
    if (T->dims[k] <= 0) return fail(ctx, MM_ERR_SHAPE, "%s: dims[%d] = %lld <= 0", name, k, (long long)T->dims[k]);
  if (T->dtype < MM_R32 || T->dtype > MM_C128) return fail(ctx, MM_ERR_ARG, "%s: bad dtype", name);
  if (!T->data) return fail(ctx, MM_ERR_ARG, "%s: data is NULL", name);
  if (((uintptr_t)T->data) & 15) return fail(ctx, MM_ERR_ALIGN, "%s: data not 16-byte aligned", name);
  if (numel(T) > ((int64_t)1 << 40)) return fail(ctx, MM_ERR_SHAPE, "%s: too many entries", name);
  return MM_OK;
}

bool overlap(const mm_tensor* A, const mm_tensor* B) {
  const char* a0 = (const char*)A->data;
  const char* a1 = a0 + numel(A) * dsize(A->dtype);
  const char* b0 = (const char*)B->data;
  const char* b1 = b0 + numel(B) * dsize(B->dtype);
  return a0 < b1 && b0 < a1;
}

mm_status check_op_dtype(mm_ctx ctx, mm_op L, mm_dtype t) {
  if (L->cplx && !is_complex(t)) return fail(ctx, MM_ERR_DTYPE, "complex operator on a real tensor");
  const bool want64 = L->prec == MM_PREC_FP64;
  if (want64 != is_f64(t))
    return fail(ctx, MM_ERR_DTYPE, "operator precision %d does not match tensor dtype %d", (int)L->prec, (int)t);
  return MM_OK;
}

// Prepare (or reuse) the fragment-order operator for a given complexity.
mm_status ensure_prepared(mm_ctx ctx, mm_op L, bool cplx, hipStream_t s, void** prep, int* KBT, int* MFT) {
  const int kp = kprec(L->prec);
  const int64_t Mr = cplx ? 2 * L->rows : L->rows;
  const int64_t Kr = cplx ? 2 * L->cols : L->cols;
  int kbt = 0, mft = 0;
  mm::op_blocks(kp, Mr, Kr, &kbt, &mft);
  if (cplx == (bool)L->cplx) {
    *prep = L->prep;
    *KBT = L->KBT;
    *MFT = L->MFT;
    return MM_OK;
  }
  // real operator acting on a complex state: promote to complex once
  if (!L->prep_c) {
    const size_t nn = (size_t)L->rows * L->cols;
    std::vector<double> host(nn), cm(2 * nn, 0.0);
    HIPCHK(ctx, hipMemcpy(host.data(), L->dev_master, nn * sizeof(double), hipMemcpyDeviceToHost));
    for (size_t e = 0; e < nn; ++e) cm[2 * e] = host[e];
    HIPCHK(ctx, hipMalloc((void**)&L->dev_master_c, 2 * nn * sizeof(double)));
    HIPCHK(ctx, hipMemcpy(L->dev_master_c, cm.data(), 2 * nn * sizeof(double), hipMemcpyHostToDevice));
    HIPCHK(ctx, hipMalloc(&L->prep_c, mm::prepared_bytes(kp, kbt, mft)));
    HIPCHK(ctx, mm::launch_prepare(kp, 1, L->dev_master_c, L->rows, L->cols, L->rows, mm::PhaseScale(),
                                   L->prep_c, kbt, mft, s, L->a_exp));
    L->KBT_c = kbt;
    L->MFT_c = mft;
  }
  *prep = L->prep_c;
  *KBT = L->KBT_c;
  *MFT = L->MFT_c;
  return MM_OK;
}

// Launch through `fn(start, stop)`, with events stamped by the dispatch and a
// record of `kind` while profiling.
template <typename F>
mm_status timed_launch(mm_ctx ctx, int kind, F&& fn) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (ctx->profiling) {
    HIPCHK(ctx, hipEventCreate(&e0));
    HIPCHK(ctx, hipEventCreate(&e1));
  }
  HIPCHK(ctx, fn(e0, e1));
  if (ctx->profiling) ctx->recs.push_back({kind, e0, e1});
  return MM_OK;
}

mm::ResForm res_form(const mm_op_s* L, mm_dtype dt) {
  return L->cplx ? (L->res_c4 ? mm::RF_C4 : mm::RF_C3) : (is_complex(dt) ? mm::RF_RC : mm::RF_RR);
}

// Arguments of a resident-tile product (launch shape still open).
mm::ResArgs res_args(const void* in, void* out, const int64_t* dims, int d, mm_dtype dt, const mm_op_s* L, int mu,
                     double s_pre, double s_post) {
  mm::ResArgs r = {};
  int64_t P = 1, Q = 1;
  for (int k = 0; k < mu - 1; ++k) P *= dims[k];
  for (int k = mu; k < d; ++k) Q *= dims[k];
  r.in = in;
  r.out = out;
  r.A = L->prep;
  r.P = P;
  r.F = P * Q;
  r.n = (int)dims[mu - 1];
  r.m = (int)L->rows;
  r.MFT = L->MFT;
  r.nsteps = 1;
  r.idadd = (L->idsplit || L->res_id) ? 1 : 0;
  if (is_complex(dt)) {
    r.s_pre = s_pre;
    r.s_post = s_post;
  }
  return r;
}

// One mode product out = in x_mu L on a tensor with dims `dims` (input dims),
// optional fused phases.  `in` and `out` may be equal when the plan covers
// all rows in one workgroup (checked by the caller through *in_place_ok).
mm_status run_mode(mm_ctx ctx, const void* in, void* out, const int64_t* dims, int d, mm_dtype dt,
                   mm_op L, int mu, double s_pre, double s_post, hipStream_t s, mm::ModePlan* plan_out,
                   bool dry, const void* prep_override = nullptr, bool batch = false,
                   int nsteps = 1, const double* winv = nullptr) {
  // A real operator on a complex state (with no fused phase) acts on the
  // (re, im) planes separately: the state is then the real tensor
  // (2, n_1, ..., n_d) and mode mu its mode mu + 1, i.e. two real fibres per
  // complex one (half the MFMA work of the complex block form, and no
  // promoted copy of the operator).
  const bool rview = !L->cplx && is_complex(dt) && !batch && s_pre == 0.0 && s_post == 0.0 && !prep_override;
  const bool cplx = is_complex(dt) && !rview;
  mm::ModeArgs a;
  int64_t P = rview ? 2 : 1, Q = 1;
  for (int k = 0; k < mu - 1; ++k) P *= dims[k];
  for (int k = mu; k < d; ++k) Q *= dims[k];
  a.in = in;
  a.out = out;
  a.A = nullptr;
  a.P = P;
  a.Q = Q;
  a.F = P * Q;
  a.n = (int)dims[mu - 1];
  a.m = (int)L->rows;
  a.Kr = (cplx ? 2 : 1) * a.n;
  a.Mr = (cplx ? 2 : 1) * a.m;
  a.s_pre = s_pre;
  a.s_post = s_post;
  a.smax_in = nullptr;
  a.smax_out = nullptr;
  a.smax_clr = nullptr;
  a.a_exp = L->a_exp;
  a.idadd = L->idsplit;
  a.rview = rview ? 1 : 0;
  const bool kcontig = (P == 1) && (a.Kr % 8 == 0);
  const bool fcontig = (P % 4 == 0);
  const bool pair = !kcontig && !cplx && P == 2 && a.Kr % 8 == 0;   // as the planner decides
  const int load = kcontig ? mm::KL_KCONTIG : (pair ? mm::KL_PAIR : (fcontig ? mm::KL_FCONTIG : mm::KL_GENERIC));
  // tune key: (precision, complex, load path, rows, columns, fibres); a
  // complex product with the fused prologue phase has its own entry (load
  // path + 8) and falls back to the plain one
  const bool pro_key = cplx && s_pre != 0.0;
  ctx->last_key = {(int64_t)kprec(L->prec), cplx ? 1 : 0, load + (pro_key ? 8 : 0), a.Mr, a.Kr, a.F};
  int force = ctx->force_cls;
  if (force < 0 && !ctx->tune.empty()) {
    auto it = ctx->tune.find(ctx->last_key);
    if (it == ctx->tune.end() && pro_key) {
      std::array<int64_t, 6> plain = ctx->last_key;
      plain[2] = load;
      it = ctx->tune.find(plain);
    }
    if (it != ctx->tune.end()) force = it->second.first;
  }
  mm::VortexW vw = {};
  if (winv && is_complex(dt)) {
    vw.winv = winv;
    vw.wd = d;
    vw.wmu = mu - 1;
    for (int k = 0; k < d; ++k) vw.wdims[k] = dims[k];
  }
  if (is_res(L->lay)) {
    // resident-tile kernel: the complex entries themselves are the fibres'
    // entries (no real view), any P
    mm::ResArgs r = res_args(in, out, dims, d, dt, L, mu, s_pre, s_post);
    if (prep_override) r.A = prep_override;
    r.nsteps = nsteps;
    r.w = vw;
    mm::ModePlan plan = {};
    plan.prec = kprec(L->prec);
    plan.cplx = cplx ? 1 : 0;
    plan.load = load;
    plan.pro = (cplx && s_pre != 0.0) ? 1 : 0;
    plan.epi = (cplx && s_post != 0.0) ? 1 : 0;
    plan.covers_all_rows = true;
    plan.res = 1;
    mm::res_plan(plan.prec, res_form(L, dt), plan.pro || plan.epi, force, &r, &plan.rp);
    plan.cls = force >= 0 ? std::min(force, 3) : plan.rp.mf - 1;
    plan.grid_x = plan.rp.grid_x;
    plan.grid_y = plan.rp.grid_y;
    plan.threads = plan.rp.threads;
    if (plan_out) *plan_out = plan;
    if (dry) return MM_OK;
    const int kind = plan.prec * 1000 + plan.cplx * 100 + plan.load * 10 + plan.pro * 2 + plan.epi;
    return timed_launch(ctx, kind, [&](hipEvent_t e0, hipEvent_t e1) { return mm::launch_res(plan.rp, r, s, e0, e1); });
  }
  // three-product kernels: complex operator with its Gauss preparation,
  // single-tensor products, whole staging tiles of 8 entries
  const bool gauss_ok = L->prep_g && cplx && !batch && !prep_override && a.n % 8 == 0;
  mm::ModePlan plan;
  if (!mm::plan_mode(a, kprec(L->prec), cplx ? 1 : 0, s_pre != 0.0, s_post != 0.0, fcontig, kcontig, &plan, batch,
                     force, gauss_ok))
    return fail(ctx, MM_ERR_UNSUPPORTED, "no kernel plan for this shape");
  // batched work items run in place, so each must own all rows of its
  // fibres: a tuned class that splits the rows gives way to the built-in one
  if (batch && !plan.covers_all_rows && force >= 0 &&
      !mm::plan_mode(a, kprec(L->prec), cplx ? 1 : 0, s_pre != 0.0, s_post != 0.0, fcontig, kcontig, &plan, batch,
                     -1))
    return fail(ctx, MM_ERR_UNSUPPORTED, "no kernel plan for this shape");
  if (plan.gauss) {
    a.A = L->prep_g;
    a.KBT = L->JBT_g;
    a.MFT = L->MFT_g;
    a.a_exp = L->a_exp_g;
  } else if (prep_override) {
    a.A = prep_override;
    a.KBT = L->KBT;
    a.MFT = L->MFT;
  } else if (!dry) {
    void* prep = nullptr;
    int KBT = 0, MFT = 0;
    mm_status st = ensure_prepared(ctx, L, cplx, s, &prep, &KBT, &MFT);
    if (st != MM_OK) return st;
    a.A = prep;
    a.KBT = KBT;
    a.MFT = MFT;
  } else {
    mm::op_blocks(kprec(L->prec), a.Mr, a.Kr, &a.KBT, &a.MFT);
  }
  if (plan_out) *plan_out = plan;
  if (dry) return MM_OK;
  if (plan.prec == mm::KP_FP16X2) {
    if (in != ctx->chain_end) {
      int64_t count = is_complex(dt) ? 2 : 1;
      for (int k = 0; k < d; ++k) count *= dims[k];
      HIPCHK(ctx, mm::launch_maxabs((const float*)in, count, ctx->smax + 3 * mm::SMAX_SLOT, ctx->smax, s));
      ctx->sidx = 0;
    }
    a.smax_in = ctx->smax + mm::SMAX_SLOT * ctx->sidx;
    a.smax_out = ctx->smax + mm::SMAX_SLOT * ((ctx->sidx + 1) % 3);
    a.smax_clr = ctx->smax + mm::SMAX_SLOT * ((ctx->sidx + 2) % 3);
    ctx->sidx = (ctx->sidx + 1) % 3;
    ctx->chain_end = out;
  }
  const int kind = plan.prec * 1000 + plan.cplx * 100 + plan.load * 10 + plan.pro * 2 + plan.epi;
  return timed_launch(ctx, kind, [&](hipEvent_t e0, hipEvent_t e1) { return mm::launch_mode(plan, a, s, e0, e1, &vw); });
}

mm_status ensure_ws(mm_ctx ctx, size_t bytes) {
  if (ctx->ws_bytes >= bytes) return MM_OK;
  if (ctx->ws_user)
    return fail(ctx, MM_ERR_NOMEM, "caller workspace of %zu bytes, %zu needed", ctx->ws_bytes, bytes);
  if (ctx->ws) {
    HIPCHK(ctx, hipDeviceSynchronize());
    HIPCHK(ctx, hipFree(ctx->ws));
    ctx->ws = nullptr;
    ctx->ws_bytes = 0;
  }
  if (hipMalloc(&ctx->ws, bytes) != hipSuccess) return fail(ctx, MM_ERR_NOMEM, "workspace of %zu bytes", bytes);
  ctx->ws_bytes = bytes;
  return MM_OK;
}

// Host array into a device buffer owned by the context, grown as needed.
template <typename V>
mm_status upload(mm_ctx ctx, V** dev, size_t* cap, const std::vector<V>& host) {
  if (host.size() > *cap) {
    if (*dev) {
      HIPCHK(ctx, hipDeviceSynchronize());
      HIPCHK(ctx, hipFree(*dev));
      *dev = nullptr;
      *cap = 0;
    }
    if (hipMalloc((void**)dev, host.size() * sizeof(V)) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "batch work items");
    *cap = host.size();
  }
  if (!host.empty()) HIPCHK(ctx, hipMemcpy(*dev, host.data(), host.size() * sizeof(V), hipMemcpyHostToDevice));
  return MM_OK;
}

// Relative MFMA time of one batched tile.
int64_t res_tile_cost(const mm::ResArgs& a, int kind) {
  const int form = kind / 10, mf = kind % 10;
  if (kind >= mm::RES_KIND_NF2) return (int64_t)a.n * mf * a.NRB * 2;
  return (int64_t)a.n * mf * a.NRB * (form == mm::RF_C4 ? 4 : (form == mm::RF_C3 ? 3 : (form == mm::RF_RC ? 2 : 1)));
}

// Drop the captured batch graph and its signature: its work items hold
// prepared-operator addresses and tile classes, so it must be rebuilt after
// an operator is destroyed or the tile choice changes.
void batch_invalidate(mm_ctx ctx) {
  if (!ctx->bexec && !ctx->bgraph && ctx->bsig.empty()) return;
  hipDeviceSynchronize();
  if (ctx->bexec) hipGraphExecDestroy(ctx->bexec);
  if (ctx->bgraph) hipGraphDestroy(ctx->bgraph);
  ctx->bexec = nullptr;
  ctx->bgraph = nullptr;
  ctx->bsig.clear();
}

// Tucker sweep over the modes with per-mode ops (square), in place on T.
// first_pre / last_post: phase coefficients fused into the first / last
// applied product (0 = none).
// winv: the phases are the vortex problem's (resident-tile kernels only).
mm_status sweep(mm_ctx ctx, mm_tensor* T, const mm_op* E, double first_pre, double last_post, hipStream_t s,
                const double* winv = nullptr) {
  int first = -1, last = -1;
  for (int k = 0; k < T->d; ++k)
    if (E[k]) {
      if (first < 0) first = k;
      last = k;
    }
  if (first < 0) return MM_OK;
  const size_t bytes = (size_t)numel(T) * dsize(T->dtype);
  void* cur = T->data;
  for (int k = first; k <= last; ++k) {
    if (!E[k]) continue;
    mm::ModePlan plan;
    mm_status st = run_mode(ctx, cur, cur, T->dims, T->d, T->dtype, E[k], k + 1, k == first ? first_pre : 0.0,
                            k == last ? last_post : 0.0, s, &plan, true);
    if (st != MM_OK) return st;
    void* dst = cur;
    if (!plan.covers_all_rows) {
      st = ensure_ws(ctx, bytes);
      if (st != MM_OK) return st;
      dst = (cur == T->data) ? ctx->ws : T->data;
    }
    st = run_mode(ctx, cur, dst, T->dims, T->d, T->dtype, E[k], k + 1, k == first ? first_pre : 0.0,
                  k == last ? last_post : 0.0, s, nullptr, false, nullptr, false, 1, winv);
    if (st != MM_OK) return st;
    cur = dst;
  }
  if (cur != T->data) {
    HIPCHK(ctx, hipMemcpyAsync(T->data, cur, bytes, hipMemcpyDeviceToDevice, s));
    if (ctx->chain_end == cur) ctx->chain_end = T->data;
  }
  return MM_OK;
}

// Grow a device buffer owned by the context.
mm_status grow(mm_ctx ctx, void** p, size_t* have, size_t need) {
  if (*have >= need) return MM_OK;
  if (*p) {
    HIPCHK(ctx, hipDeviceSynchronize());
    HIPCHK(ctx, hipFree(*p));
    *p = nullptr;
    *have = 0;
  }
  if (hipMalloc(p, need) != hipSuccess) return fail(ctx, MM_ERR_NOMEM, "scratch of %zu bytes", need);
  *have = need;
  return MM_OK;
}

// Grow a buffer to `fixed` bytes and *units blocks of `unit` bytes, or to as
// many blocks as there is memory for, `least` at the least (*units is lowered).
// *failed keeps the smallest size that could not be had, which later calls do
// not try again: a buffer that is large enough for the fewer blocks stays.
mm_status grow_units(mm_ctx ctx, void** p, size_t* have, size_t* failed, size_t fixed, size_t unit, int* units,
                     int least) {
  auto bytes = [&]() { return fixed + unit * (size_t)*units; };
  while (*units > least && bytes() > *have && bytes() >= *failed) *units = std::max(least, *units / 2);
  for (;;) {
    const mm_status st = grow(ctx, p, have, bytes());
    if (st != MM_ERR_NOMEM || *units <= least) return st;
    *failed = std::min(*failed, bytes());
    *units = std::max(least, *units / 2);
  }
}

// Form of a complex resident operator whose caller prepares it per step: L - I
// where ||L - I||_F < 1.22 ||L||_F is known, else L itself, which FP32 takes in
// four products (the rule and the errors of mm_op_prepare_ex; FP64 keeps three
// products on L, whose error there is that of the block form within 8 %).
void set_form(mm_op_s* o, bool near) {
  const bool f32 = o->prec == MM_PREC_FP32;
  o->res_id = f32 && near ? 1 : 0;
  o->res_c4 = f32 && !near ? 1 : 0;
}

// A throw-away operator record for products with a device-resident FP64
// master that is prepared by the caller (prep_override of run_mode).
mm_op_s scratch_op(int n, mm_prec prec, int a_exp) {
  mm_op_s o;
  o.rows = o.cols = n;
  o.cplx = 1;
  o.prec = prec;
  o.a_exp = a_exp;
  o.lay = op_layout(prec, n, n, 1);
  set_form(&o, false);
  layout_blocks(o.lay, n, n, 1, &o.KBT, &o.MFT);
  return o;
}

// Squarings that scale fa = |f| ||A + g diag d||_1 to at most 1.
mm_status expm_squarings(mm_ctx ctx, double fa, int* q) {
  *q = 0;
  if (!std::isfinite(fa)) return fail(ctx, MM_ERR_NONFINITE, "matrix holds NaN / Inf");
  if (fa > 1.0) *q = (int)std::ceil(std::log2(fa));
  if (*q > 1000) return fail(ctx, MM_ERR_ARG, "exponent argument too large (norm %g)", fa);
  return MM_OK;
}

// Buffers of one exponential of an n x n matrix; keep: also the result's.
mm_status expm_buffers(mm_ctx ctx, int n, bool keep) {
  const size_t mat = sizeof(double) * 2 * (size_t)n * n;
  mm_status st = grow(ctx, (void**)&ctx->ex_buf, &ctx->ex_bytes,
                      std::max(mm::expm_batch_bytes(n, 1), 6 * mat) + sizeof(double) * n);
  if (st == MM_OK && n > mm::EXPM_MAX_N) {
    const mm_op_s op = scratch_op(n, MM_PREC_FP64, 0);
    st = grow(ctx, &ctx->ex_prep, &ctx->ex_prep_bytes, 2 * mm::prepared_bytes(op.lay, op.KBT, op.MFT));
  }
  if (st == MM_OK && keep) st = grow(ctx, (void**)&ctx->mg_exp, &ctx->mg_exp_bytes, mat);
  return st;
}

// out = exp(f (A + g diag(d))) for a complex n x n FP64 matrix A on the
// device (d real, nullable), by scaling and squaring of the Taylor
// polynomial: X = f (A + g diag d) / 2^q with ||X||_1 <= 1, the degree-18
// Taylor polynomial (truncation <= e/19! < 2.2e-17) evaluated by the
// Paterson-Stockmeyer scheme with blocks of four terms (X^2, X^3, X^4, then
// Horner in X^4: 7 matrix products instead of 18), then q squarings.  Up to
// EXPM_MAX_N rows it is a batch of one (kern_expm.hip), above every matrix
// product is a mode-1 product of the FP64 MFMA kernel.  bound: an upper bound
// of ||A + g diag d||_1 known to the caller, or < 0 to compute it here
// (synchronises s).
mm_status expm_device(mm_ctx ctx, int n, const double* A, const double* d, double gr, double gi, double fr,
                      double fi, double bound, double* out, hipStream_t s) {
  const size_t mat = (size_t)n * n * 2;
  const bool small = n <= mm::EXPM_MAX_N;
  mm_status st = expm_buffers(ctx, n, false);
  if (st != MM_OK) return st;
  double* cs = ctx->ex_buf + 6 * mat;
  if (bound < 0) {
    HIPCHK(ctx, mm::launch_expm_colsum(A, n, d, gr, gi, cs, s));
    std::vector<double> h(n);
    HIPCHK(ctx, hipMemcpyAsync(h.data(), cs, sizeof(double) * n, hipMemcpyDeviceToHost, s));
    HIPCHK(ctx, hipStreamSynchronize(s));
    bound = 0.0;
    for (double v : h) bound = std::max(bound, v);
  }
  int q = 0;
  if ((st = expm_squarings(ctx, std::hypot(fr, fi) * bound, &q)) != MM_OK) return st;
  if (small) {
    mm::ExpmBatch b = {};
    b.n = n;
    b.nb = 1;
    b.q = q;
    b.j[0] = {A, d, gr, gi, fr, fi, nullptr, 0, 0};
    double* r = nullptr;
    HIPCHK(ctx, mm::launch_expm_batch(b, ctx->ex_buf, &r, s));
    HIPCHK(ctx, hipMemcpyAsync(out, r, sizeof(double) * mat, hipMemcpyDeviceToDevice, s));
    return MM_OK;
  }
  mm_op_s op = scratch_op(n, MM_PREC_FP64, 0);
  const size_t pb = mm::prepared_bytes(op.lay, op.KBT, op.MFT);
  double* X = ctx->ex_buf;
  double* X2 = X + mat;
  double* X3 = X2 + mat;
  double* Y = X3 + mat;     // X^4
  double* P = Y + mat;
  double* W = P + mat;
  void* prepX = ctx->ex_prep;
  void* prepY = (char*)ctx->ex_prep + pb;
  const double sc = std::ldexp(1.0, -q);
  const int64_t dims[2] = {n, n};
  // a product of two n x n matrices has only n fibres: where the default
  // FP64 tile would leave most CUs idle (fewer than 128 workgroups), the
  // one-wave tile of class 3 (32 real rows x 16 fibres) runs it
  const bool few = (int64_t)((n + 31) / 32) * ((2 * (int64_t)n + 511) / 512) < 128;
  auto mul = [&](const void* prep, const double* in, double* o) {
    const int keep = ctx->force_cls;
    if (few) ctx->force_cls = 3;
    mm_status r = run_mode(ctx, in, o, dims, 2, MM_C128, &op, 1, 0, 0, s, nullptr, false, prep);
    ctx->force_cls = keep;
    return r;
  };
  HIPCHK(ctx, mm::launch_expm_generator(A, n, d, gr, gi, fr * sc, fi * sc, X, s));
  HIPCHK(ctx, mm::launch_prepare(op.lay, 1, X, n, n, n, mm::PhaseScale(), prepX, op.KBT, op.MFT, s));
  if ((st = mul(prepX, X, X2)) != MM_OK) return st;
  if ((st = mul(prepX, X2, X3)) != MM_OK) return st;
  if ((st = mul(prepX, X3, Y)) != MM_OK) return st;
  HIPCHK(ctx, mm::launch_prepare(op.lay, 1, Y, n, n, n, mm::PhaseScale(), prepY, op.KBT, op.MFT, s));
  // coefficients 1/k!, k = 0..18, in blocks B_j = sum_i c_{4j+i} X^i
  double c[20] = {0};
  c[0] = 1.0;
  for (int k = 1; k <= 18; ++k) c[k] = c[k - 1] / k;
  HIPCHK(ctx, mm::launch_expm_ps(P, nullptr, X, X2, X3, n, c + 16, s));
  for (int j = 3; j >= 0; --j) {
    if ((st = mul(prepY, P, W)) != MM_OK) return st;   // P X^4 (polynomials in X commute)
    HIPCHK(ctx, mm::launch_expm_ps(P, W, X, X2, X3, n, c + 4 * j, s));
  }
  double* T = P;
  for (int r = 0; r < q; ++r) {
    HIPCHK(ctx, mm::launch_prepare(op.lay, 1, T, n, n, n, mm::PhaseScale(), prepX, op.KBT, op.MFT, s));
    if ((st = mul(prepX, T, W)) != MM_OK) return st;
    std::swap(T, W);
  }
  HIPCHK(ctx, hipMemcpyAsync(out, T, sizeof(double) * mat, hipMemcpyDeviceToDevice, s));
  return MM_OK;
}

// In-call monitor: FP64 sum |T|^2 after `step` steps into the next slot of
// the device log (no host synchronisation until monitor_end).
mm_status monitor_begin(mm_ctx ctx, int nsteps) {
  ctx->mon_steps.clear();
  ctx->mon_vals.clear();
  if (ctx->mon_every <= 0 || nsteps <= 0) return MM_OK;
  const size_t need = (size_t)(nsteps / ctx->mon_every + 2);
  if (ctx->mon_cap < need) {
    if (ctx->mon_dev) {
      HIPCHK(ctx, hipDeviceSynchronize());
      HIPCHK(ctx, hipFree(ctx->mon_dev));
      ctx->mon_dev = nullptr;
      ctx->mon_cap = 0;
    }
    if (hipMalloc((void**)&ctx->mon_dev, sizeof(double) * need) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "monitor log");
    ctx->mon_cap = need;
  }
  return MM_OK;
}

mm_status monitor_point(mm_ctx ctx, const mm_tensor* T, int step, hipStream_t s) {
  const size_t k = ctx->mon_steps.size();
  if (k >= ctx->mon_cap) return MM_OK;
  const int64_t count = numel(T) * (is_complex(T->dtype) ? 2 : 1);
  HIPCHK(ctx, mm::launch_reduce(mm::RED_SQ, T->data, nullptr, count, is_f64(T->dtype) ? 1 : 0, ctx->red_partial,
                                ctx->mon_dev + k, s));
  ctx->mon_steps.push_back(step);
  return MM_OK;
}

mm_status monitor_end(mm_ctx ctx, hipStream_t s) {
  const size_t k = ctx->mon_steps.size();
  if (k == 0) return MM_OK;
  ctx->mon_vals.resize(k);
  HIPCHK(ctx, hipMemcpyAsync(ctx->mon_vals.data(), ctx->mon_dev, sizeof(double) * k, hipMemcpyDeviceToHost, s));
  HIPCHK(ctx, hipStreamSynchronize(s));
  for (size_t i = 0; i < k; ++i)
    if (!std::isfinite(ctx->mon_vals[i]))
      return fail(ctx, MM_ERR_NONFINITE, "sum |T|^2 is not finite after step %d", ctx->mon_steps[i]);
  return MM_OK;
}

// Several steps of an expstep whose operators all run on the resident-tile
// kernels: one launch per mode.
// *used = false (and nothing launched) when the problem does not qualify.
mm_status fused_expstep(mm_ctx ctx, mm_tensor* T, const mm_op* E, int nsteps, hipStream_t s, bool* used) {
  *used = false;
  // every operator on the resident-tile kernels: all steps of one mode run in
  // one launch, the fibre tile staying in LDS between them (products along
  // different modes commute, Section 2, so the modes' steps may be reordered)
  double growth = 0.0;
  bool any = false, tiny = (size_t)numel(T) * dsize(T->dtype) <= ((size_t)2 << 20);
  for (int k = 0; k < T->d; ++k) {
    if (!E[k]) continue;
    if (!is_res(E[k]->lay)) return MM_OK;
    any = true;
    growth += std::max(0.0, E[k]->log2_norm);
    tiny = tiny && (E[k]->cplx ? 2 : 1) * E[k]->rows <= 128 && (E[k]->cplx || !is_complex(T->dtype)) && !E[k]->idsplit;
  }
  if (!any) return MM_OK;
  // steps per launch: reordered, a mode's steps may raise the state before
  // another mode's lower it again; the modes' norm bounds keep that within
  // 2^20 (FP32; exponent range 2^127) or 2^200 (FP64)
  const double room = is_f64(T->dtype) ? 200.0 : 20.0;
  // and a launch short however many steps the call has (256 products of n = 256
  // FP64 on 65536 fibres: 0.1 s)
  const int blk = std::min(growth * nsteps <= room ? nsteps : (int)(room / growth), 256);
  if (blk < 2) return MM_OK;
  // a state of at most 2 MiB with modes of at most 128 real rows is recorded
  // as one whole run (kind 91: 2-D real FP64, both modes at most 64 long),
  // larger ones launch by launch
  const bool prof = ctx->profiling;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (prof && tiny) {
    HIPCHK(ctx, hipEventCreate(&e0));
    HIPCHK(ctx, hipEventCreate(&e1));
    HIPCHK(ctx, hipEventRecord(e0, s));
    ctx->profiling = false;
  }
  mm_status st = MM_OK;
  for (int it = 0; it < nsteps && st == MM_OK; it += blk)
    for (int k = 0; k < T->d && st == MM_OK; ++k)
      if (E[k])
        st = run_mode(ctx, T->data, T->data, T->dims, T->d, T->dtype, E[k], k + 1, 0, 0, s, nullptr, false, nullptr,
                      false, std::min(blk, nsteps - it));
  ctx->profiling = prof;
  if (st != MM_OK) return st;
  if (prof && tiny) {
    HIPCHK(ctx, hipEventRecord(e1, s));
    const bool d2 = T->d == 2 && T->dtype == MM_R64 && T->dims[0] <= 64 && T->dims[1] <= 64;
    ctx->recs.push_back({(is_f64(T->dtype) ? mm::KP_F64 : mm::KP_F32) * 1000 + (is_complex(T->dtype) ? 100 : 0) +
                             (d2 ? 91 : 90), e0, e1});
  }
  *used = true;
  return MM_OK;
}

}  // namespace

extern "C" {

const char* mm_version(void) { return "mumode-gfx950 0.1"; }

const char* mm_status_string(mm_status s) {
  switch (s) {
    case MM_OK: return "ok";
    case MM_ERR_ARG: return "invalid argument";
    case MM_ERR_SHAPE: return "invalid shape";
    case MM_ERR_DTYPE: return "dtype / precision mismatch";
    case MM_ERR_ALIGN: return "misaligned data";
    case MM_ERR_NOMEM: return "out of device memory";
    case MM_ERR_HIP: return "HIP runtime error";
    case MM_ERR_UNSUPPORTED: return "unsupported";
    case MM_ERR_NONFINITE: return "non-finite value";
    case MM_ERR_NODEVICE: return "no gfx950 device";
  }
  return "unknown status";
}

const char* mm_last_error(mm_ctx ctx) { return ctx ? ctx->err.c_str() : g_create_err.c_str(); }

mm_status mm_create(mm_ctx* out, int device, const char* tune_cache_path) {
  if (!out) return fail(nullptr, MM_ERR_ARG, "out is NULL");
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count <= 0)
    return fail(nullptr, MM_ERR_NODEVICE, "no HIP device visible");
  if (device < 0 || device >= count) return fail(nullptr, MM_ERR_NODEVICE, "device %d of %d", device, count);
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return fail(nullptr, MM_ERR_NODEVICE, "device properties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(nullptr, MM_ERR_NODEVICE, "device %d is %s, not gfx950", device, prop.gcnArchName);
  if (hipSetDevice(device) != hipSuccess) return fail(nullptr, MM_ERR_HIP, "hipSetDevice");
  mm_ctx c = new mm_ctx_s;
  c->device = device;
  if (hipMalloc((void**)&c->red_partial, sizeof(double) * mm::norm_partials()) != hipSuccess ||
      hipMalloc((void**)&c->red_result, sizeof(double) * 4) != hipSuccess ||
      hipMalloc((void**)&c->smax, sizeof(uint32_t) * (3 * mm::SMAX_SLOT + mm::norm_partials())) != hipSuccess ||
      hipHostMalloc((void**)&c->host_result, sizeof(double) * 4, hipHostMallocDefault) != hipSuccess) {
    delete c;
    return fail(nullptr, MM_ERR_NOMEM, "context buffers");
  }
  {
    const hipError_t e = scratch_address(device, &c->smax_static);
    if (e != hipSuccess) {
      mm_destroy(c);
      return fail(nullptr, MM_ERR_HIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
    }
  }
  if (tune_cache_path) {
    c->tune_path = tune_cache_path;
    if (FILE* f = std::fopen(tune_cache_path, "r")) {
      std::fclose(f);
      if (mm_tune_load(c, tune_cache_path) != MM_OK) {
        const std::string why = c->err;
        mm_destroy(c);
        return fail(nullptr, MM_ERR_ARG, "tune cache: %s", why.c_str());
      }
    }
  }
  *out = c;
  return MM_OK;
}

mm_status mm_op_destroy(mm_ctx ctx, mm_op op) {
  if (!ctx || !op) return MM_ERR_ARG;
  auto it = std::find(ctx->ops.begin(), ctx->ops.end(), op);
  if (it == ctx->ops.end()) return fail(ctx, MM_ERR_ARG, "operator not owned by this context");
  ctx->ops.erase(it);
  hipSetDevice(ctx->device);
  batch_invalidate(ctx);
  for (int k = 0; k < MM_MAXD; ++k)
    if (ctx->ho[k].phi == op || ctx->ho[k].psi == op) ctx->ho[k].phi = ctx->ho[k].psi = nullptr;
  hipDeviceSynchronize();
  if (op->dev_master) hipFree(op->dev_master);
  if (op->prep) hipFree(op->prep);
  if (op->prep_c) hipFree(op->prep_c);
  if (op->prep_g) hipFree(op->prep_g);
  if (op->dev_master_c) hipFree(op->dev_master_c);
  delete op;
  return MM_OK;
}

mm_status mm_destroy(mm_ctx ctx) {
  if (!ctx) return MM_OK;
  hipSetDevice(ctx->device);
  hipDeviceSynchronize();
  while (!ctx->ops.empty()) mm_op_destroy(ctx, ctx->ops.back());
  for (auto& r : ctx->recs) {
    hipEventDestroy(r.a);
    hipEventDestroy(r.b);
  }
  if (ctx->ws && !ctx->ws_user) hipFree(ctx->ws);
  if (ctx->step_prep) hipFree(ctx->step_prep);
  if (ctx->x2) hipFree(ctx->x2);
  if (ctx->x2_stage) hipHostFree(ctx->x2_stage);
  if (ctx->x2_ev) hipEventDestroy(ctx->x2_ev);
  if (ctx->winv) hipFree(ctx->winv);
  if (ctx->winv_stage) hipHostFree(ctx->winv_stage);
  if (ctx->winv_ev) hipEventDestroy(ctx->winv_ev);
  for (int k = 0; k < MM_MAXD; ++k)
    if (ctx->ho[k].master) hipFree(ctx->ho[k].master);
  if (ctx->bexec) hipGraphExecDestroy(ctx->bexec);
  if (ctx->bgraph) hipGraphDestroy(ctx->bgraph);
  if (ctx->bitems) hipFree(ctx->bitems);
  if (ctx->rargs) hipFree(ctx->rargs);
  if (ctx->ritems) hipFree(ctx->ritems);
  if (ctx->cap_stream) hipStreamDestroy(ctx->cap_stream);
  if (ctx->red_partial) hipFree(ctx->red_partial);
  if (ctx->red_result) hipFree(ctx->red_result);
  if (ctx->smax) hipFree(ctx->smax);
  if (ctx->mon_dev) hipFree(ctx->mon_dev);
  if (ctx->ex_buf) hipFree(ctx->ex_buf);
  if (ctx->ex_prep) hipFree(ctx->ex_prep);
  if (ctx->mg_buf) hipFree(ctx->mg_buf);
  if (ctx->mg_stage) hipHostFree(ctx->mg_stage);
  if (ctx->mg_prep) hipFree(ctx->mg_prep);
  if (ctx->mg_exp) hipFree(ctx->mg_exp);
  if (ctx->host_result) hipHostFree(ctx->host_result);
  delete ctx;
  return MM_OK;
}

mm_status mm_op_prepare(mm_ctx ctx, const mm_matrix* M, mm_prec prec, mm_op* out) {
  return mm_op_prepare_ex(ctx, M, prec, 0u, out);
}

mm_status mm_op_prepare_ex(mm_ctx ctx, const mm_matrix* M, mm_prec prec, unsigned flags, mm_op* out) {
  if (!ctx) return MM_ERR_ARG;
  if (!M || !out || !M->data) return fail(ctx, MM_ERR_ARG, "NULL matrix or output");
  *out = nullptr;
  if (flags & ~(unsigned)MM_OP_IDENTITY_SPLIT) return fail(ctx, MM_ERR_ARG, "unknown operator flags 0x%x", flags);
  const bool idsplit = (flags & MM_OP_IDENTITY_SPLIT) != 0;
  if (idsplit && M->rows != M->cols) return fail(ctx, MM_ERR_SHAPE, "identity split needs a square operator");
  if (M->dtype != MM_R64 && M->dtype != MM_C128) return fail(ctx, MM_ERR_DTYPE, "master must be MM_R64 or MM_C128");
  if (prec < MM_PREC_FP64 || prec > MM_PREC_BF16) return fail(ctx, MM_ERR_ARG, "bad precision");
  if (M->rows < 1 || M->cols < 1 || M->rows > 4096 || M->cols > 4096)
    return fail(ctx, MM_ERR_SHAPE, "operator %lld x %lld outside [1, 4096]", (long long)M->rows, (long long)M->cols);
  if (M->ld < M->rows) return fail(ctx, MM_ERR_SHAPE, "ld < rows");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  const int cplx = M->dtype == MM_C128;
  const int comps = cplx ? 2 : 1;
  // compact host copy (ld = rows)
  std::vector<double> host((size_t)M->rows * M->cols * comps);
  if (M->on_device) {
    std::vector<double> full((size_t)M->ld * M->cols * comps);
    HIPCHK(ctx, hipMemcpy(full.data(), M->data, full.size() * sizeof(double), hipMemcpyDeviceToHost));
    for (int64_t j = 0; j < M->cols; ++j)
      std::memcpy(&host[(size_t)j * M->rows * comps], &full[(size_t)j * M->ld * comps], sizeof(double) * M->rows * comps);
  } else {
    const double* src = (const double*)M->data;
    for (int64_t j = 0; j < M->cols; ++j)
      std::memcpy(&host[(size_t)j * M->rows * comps], src + (size_t)j * M->ld * comps, sizeof(double) * M->rows * comps);
  }
  for (double v : host)
    if (!std::isfinite(v)) return fail(ctx, MM_ERR_NONFINITE, "operator holds NaN / Inf");
  std::vector<double> rsum(M->rows, 0.0);
  double cmax = 0.0;
  for (int64_t j = 0; j < M->cols; ++j) {
    double c = 0.0;
    for (int64_t i = 0; i < M->rows; ++i) {
      const double* v = &host[((size_t)j * M->rows + i) * comps];
      const double m = cplx ? std::sqrt(v[0] * v[0] + v[1] * v[1]) : std::fabs(v[0]);
      c += m;
      rsum[i] += m;
    }
    cmax = std::max(cmax, c);
  }
  // Form of a complex operator on the resident-tile kernels.  Square ones with
  // ||L - I||_F < 1.22 ||L||_F run on L - I in three products and add the
  // input back; others run as they are, FP32 in four products (so do FP32
  // operators that the caller keeps as L - I further from it).  Why: the third
  // product rounds at the size of |x + y|, where the block form rounds at that
  // of its result.  Relative L2 errors in FP32 against 64 bits (block form /
  // three products on L / on L - I), by the ratio of the norms: GPE n = 100,
  // four steps, ratio 0.05: 4.2e-7 / 6.3e-7 / 1.5e-7; vortex n = 99, five
  // steps, 1.01: 4.6e-7 / 5.8e-7 / 3.1e-7; free Schroedinger, two steps,
  // n = 200, 1.09: 4.0e-7 / 4.2e-7 / 2.9e-7, n = 256, 1.44: 3.2e-7 / 3.9e-7 /
  // 4.0e-7.  Those are the problems' own states; on white noise L - I rounds at
  // its own norm whatever the state, so the error passes the block form's from
  // a ratio of about 0.85 on (one product: 0.34 of it at 0.28, 0.7 at 0.68, 1.03
  // to 1.3 at 1.02, 1.2 to 1.57 at 1.2), while on smooth states it stays at 0.3
  // to 0.8 of it.  Four products are at 0.99 to 1.02 of the block form on both.
  // FP64 keeps three products there too: against extended precision, random
  // unitary operators of 32 to 256 rows, 1.0 to 1.08 of the block form's 2.7e-16
  // to 7.5e-16, and half of it on L - I near the identity.
  bool res_id = false, res_c4 = false;
  if (cplx && is_res(op_layout(prec, M->rows, M->cols, cplx))) {
    bool near = false;
    if (M->rows == M->cols) {
      double all = 0.0, off = 0.0;
      for (int64_t j = 0; j < M->cols; ++j)
        for (int64_t i = 0; i < M->rows; ++i) {
          const double* v = &host[((size_t)j * M->rows + i) * 2];
          const double dr = i == j ? v[0] - 1.0 : v[0];
          all += v[0] * v[0] + v[1] * v[1];
          off += dr * dr + v[1] * v[1];
        }
      near = off < 1.5 * all;
    }
    res_id = near && !idsplit;
    res_c4 = prec == MM_PREC_FP32 && !near;
  }
  const double rmax = *std::max_element(rsum.begin(), rsum.end());
  if (idsplit)   // L - I in FP64: the products carry only the departure from identity
    for (int64_t i = 0; i < M->rows; ++i) host[((size_t)i * M->rows + i) * comps] -= 1.0;
  double amax = 0.0;
  for (double v : host) amax = std::max(amax, std::fabs(v));
  mm_op op = new mm_op_s;
  op->rows = M->rows;
  op->cols = M->cols;
  op->cplx = cplx;
  op->prec = prec;
  op->idsplit = idsplit ? 1 : 0;
  op->res_id = res_id ? 1 : 0;
  op->res_c4 = res_c4 ? 1 : 0;
  op->log2_norm = (cmax > 0.0 && rmax > 0.0) ? 0.5 * (std::log2(cmax) + std::log2(rmax)) : 0.0;
  op->a_exp = prec == MM_PREC_SPLIT_FP16X2 ? mm::fp16x2_op_exp(amax) : 0;
  const int kp = kprec(prec);
  op->lay = op_layout(prec, M->rows, M->cols, cplx);
  layout_blocks(op->lay, M->rows, M->cols, cplx, &op->KBT, &op->MFT);
  // the three-product form of a complex split operator is prepared with it
  // (no product call allocates): Re L, Im L and Re L + Im L
  const bool gauss = cplx && !idsplit && (kp == mm::KP_FP16X2 || kp == mm::KP_BF16X3);
  if (gauss) {
    double gmax = 0.0;
    for (size_t e = 0; e + 1 < host.size(); e += 2)
      gmax = std::max(gmax, std::max(std::fabs(host[e]), std::max(std::fabs(host[e + 1]), std::fabs(host[e] + host[e + 1]))));
    op->a_exp_g = kp == mm::KP_FP16X2 ? mm::fp16x2_op_exp(gmax) : 0;
    mm::gauss_blocks(op->rows, op->cols, &op->JBT_g, &op->MFT_g);
  }
  if (hipMalloc((void**)&op->dev_master, host.size() * sizeof(double)) != hipSuccess ||
      hipMalloc(&op->prep, mm::prepared_bytes(op->lay, op->KBT, op->MFT)) != hipSuccess ||
      (gauss && hipMalloc(&op->prep_g, mm::gauss_prepared_bytes(kp, op->JBT_g, op->MFT_g)) != hipSuccess)) {
    if (op->dev_master) hipFree(op->dev_master);
    if (op->prep) hipFree(op->prep);
    delete op;
    return fail(ctx, MM_ERR_NOMEM, "operator buffers");
  }
  ctx->ops.push_back(op);
  HIPCHK(ctx, hipMemcpy(op->dev_master, host.data(), host.size() * sizeof(double), hipMemcpyHostToDevice));
  mm::PhaseScale ph;
  ph.minus_id = op->res_id;
  HIPCHK(ctx, mm::launch_prepare(op->lay, cplx, op->dev_master, op->rows, op->cols, op->rows, ph,
                                 op->prep, op->KBT, op->MFT, 0, op->a_exp));
  if (gauss)
    HIPCHK(ctx, mm::launch_prepare_gauss(kp, op->dev_master, op->rows, op->cols, op->rows, op->prep_g, op->JBT_g,
                                         op->MFT_g, op->a_exp_g, 0));
  HIPCHK(ctx, hipDeviceSynchronize());
  *out = op;
  return MM_OK;
}

mm_status mm_op_flags(mm_op op, unsigned* flags) {
  if (!op || !flags) return MM_ERR_ARG;
  *flags = op->idsplit ? (unsigned)MM_OP_IDENTITY_SPLIT : 0u;
  return MM_OK;
}

mm_status mm_op_info(mm_op op, int64_t* rows, int64_t* cols, int* is_complex_, mm_prec* prec) {
  if (!op) return MM_ERR_ARG;
  if (rows) *rows = op->rows;
  if (cols) *cols = op->cols;
  if (is_complex_) *is_complex_ = op->cplx;
  if (prec) *prec = op->prec;
  return MM_OK;
}

mm_status mumode_apply(mm_ctx ctx, mm_tensor* out, const mm_tensor* T, mm_op L, int mu, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, T, "T");
  if (st != MM_OK) return st;
  st = check_tensor(ctx, out, "out");
  if (st != MM_OK) return st;
  if (!L) return fail(ctx, MM_ERR_ARG, "operator is NULL");
  if (mu < 1 || mu > T->d) return fail(ctx, MM_ERR_SHAPE, "mu = %d outside [1, %d]", mu, T->d);
  if (L->cols != T->dims[mu - 1])
    return fail(ctx, MM_ERR_SHAPE, "operator has %lld columns, n_mu = %lld", (long long)L->cols, (long long)T->dims[mu - 1]);
  if (out->d != T->d || out->dtype != T->dtype) return fail(ctx, MM_ERR_SHAPE, "out must have T's order and dtype");
  for (int k = 0; k < T->d; ++k) {
    const int64_t want = (k == mu - 1) ? L->rows : T->dims[k];
    if (out->dims[k] != want) return fail(ctx, MM_ERR_SHAPE, "out dims[%d] = %lld, expected %lld", k, (long long)out->dims[k], (long long)want);
  }
  st = check_op_dtype(ctx, L, T->dtype);
  if (st != MM_OK) return st;
  if (overlap(out, T)) return fail(ctx, MM_ERR_ARG, "out overlaps T");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  return run_mode(ctx, T->data, out->data, T->dims, T->d, T->dtype, L, mu, 0, 0, (hipStream_t)stream, nullptr, false);
}

mm_status mumode_expstep(mm_ctx ctx, mm_tensor* T, const mm_op* E, int nsteps, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  ctx->mon_steps.clear();
  ctx->mon_vals.clear();
  mm_status st = check_tensor(ctx, T, "T");
  if (st != MM_OK) return st;
  if (!E) return fail(ctx, MM_ERR_ARG, "E is NULL");
  if (nsteps < 0) return fail(ctx, MM_ERR_ARG, "nsteps < 0");
  for (int k = 0; k < T->d; ++k) {
    if (!E[k]) continue;
    if (E[k]->rows != E[k]->cols || E[k]->cols != T->dims[k])
      return fail(ctx, MM_ERR_SHAPE, "E[%d] must be %lld x %lld", k, (long long)T->dims[k], (long long)T->dims[k]);
    st = check_op_dtype(ctx, E[k], T->dtype);
    if (st != MM_OK) return st;
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  if (!ctx->keep_chain || T->data != ctx->chain_end) ctx->chain_end = nullptr;
  if (ctx->small_run && nsteps >= 2 && ctx->mon_every <= 0) {
    bool used = false;
    st = fused_expstep(ctx, T, E, nsteps, (hipStream_t)stream, &used);
    if (st != MM_OK || used) return st;
  }
  st = monitor_begin(ctx, nsteps);
  if (st != MM_OK) return st;
  for (int it = 0; it < nsteps; ++it) {
    st = sweep(ctx, T, E, 0.0, 0.0, (hipStream_t)stream);
    if (st != MM_OK) return st;
    if (ctx->mon_every > 0 && ((it + 1) % ctx->mon_every == 0 || it + 1 == nsteps)) {
      st = monitor_point(ctx, T, it + 1, (hipStream_t)stream);
      if (st != MM_OK) return st;
    }
  }
  return monitor_end(ctx, (hipStream_t)stream);
}

mm_status mumode_transform(mm_ctx ctx, mm_tensor* out, const mm_tensor* in, const mm_op* Phi, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, in, "in");
  if (st != MM_OK) return st;
  st = check_tensor(ctx, out, "out");
  if (st != MM_OK) return st;
  if (!Phi) return fail(ctx, MM_ERR_ARG, "Phi is NULL");
  if (out->d != in->d || out->dtype != in->dtype) return fail(ctx, MM_ERR_SHAPE, "out must have in's order and dtype");
  for (int k = 0; k < in->d; ++k) {
    if (Phi[k]) {
      if (Phi[k]->cols != in->dims[k]) return fail(ctx, MM_ERR_SHAPE, "Phi[%d] has %lld columns, expected %lld", k, (long long)Phi[k]->cols, (long long)in->dims[k]);
      st = check_op_dtype(ctx, Phi[k], in->dtype);
      if (st != MM_OK) return st;
    }
    const int64_t want = Phi[k] ? Phi[k]->rows : in->dims[k];
    if (out->dims[k] != want) return fail(ctx, MM_ERR_SHAPE, "out dims[%d] = %lld, expected %lld", k, (long long)out->dims[k], (long long)want);
  }
  if (overlap(out, in)) return fail(ctx, MM_ERR_ARG, "out overlaps in");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  // chain of rectangular products: in -> A -> B -> ... -> out, where the
  // intermediate tensors live in the workspace (two halves) and the last
  // product writes out.
  int last = -1, count = 0;
  for (int k = 0; k < in->d; ++k)
    if (Phi[k]) {
      last = k;
      ++count;
    }
  const size_t es = dsize(in->dtype);
  if (count == 0) {
    HIPCHK(ctx, hipMemcpyAsync(out->data, in->data, (size_t)numel(in) * es, hipMemcpyDeviceToDevice, s));
    return MM_OK;
  }
  // largest intermediate
  int64_t dims[MM_MAXD];
  for (int k = 0; k < in->d; ++k) dims[k] = in->dims[k];
  size_t maxb = 0;
  for (int k = 0; k < in->d; ++k) {
    if (!Phi[k]) continue;
    dims[k] = Phi[k]->rows;
    int64_t n = 1;
    for (int q = 0; q < in->d; ++q) n *= dims[q];
    maxb = std::max(maxb, (size_t)n * es);
  }
  const size_t half = (maxb + 255) / 256 * 256;
  if (count > 1) {
    st = ensure_ws(ctx, 2 * half);
    if (st != MM_OK) return st;
  }
  for (int k = 0; k < in->d; ++k) dims[k] = in->dims[k];
  const void* cur = in->data;
  int pp = 0;
  for (int k = 0; k < in->d; ++k) {
    if (!Phi[k]) continue;
    void* dst = (k == last) ? out->data : (void*)((char*)ctx->ws + pp * half);
    st = run_mode(ctx, cur, dst, dims, in->d, in->dtype, Phi[k], k + 1, 0, 0, s, nullptr, false);
    if (st != MM_OK) return st;
    dims[k] = Phi[k]->rows;
    cur = dst;
    pp ^= 1;
  }
  return MM_OK;
}

namespace {

mm_status gpe_strang_impl(mm_ctx ctx, mm_tensor* psi, const mm_op* E, double tau, double beta, int nsteps,
                          hipStream_t s, bool noalloc) {
  if (!ctx) return MM_ERR_ARG;
  ctx->mon_steps.clear();
  ctx->mon_vals.clear();
  mm_status st = check_tensor(ctx, psi, "psi");
  if (st != MM_OK) return st;
  if (!is_complex(psi->dtype)) return fail(ctx, MM_ERR_DTYPE, "psi must be complex");
  if (!E) return fail(ctx, MM_ERR_ARG, "E is NULL");
  if (nsteps < 0) return fail(ctx, MM_ERR_ARG, "nsteps < 0");
  if (!std::isfinite(tau) || !std::isfinite(beta)) return fail(ctx, MM_ERR_ARG, "tau / beta not finite");
  for (int k = 0; k < psi->d; ++k) {
    if (!E[k]) return fail(ctx, MM_ERR_ARG, "E[%d] is NULL", k);
    if (E[k]->rows != E[k]->cols || E[k]->cols != psi->dims[k])
      return fail(ctx, MM_ERR_SHAPE, "E[%d] must be %lld x %lld", k, (long long)psi->dims[k], (long long)psi->dims[k]);
    st = check_op_dtype(ctx, E[k], psi->dtype);
    if (st != MM_OK) return st;
    if (noalloc && !E[k]->cplx)
      return fail(ctx, MM_ERR_UNSUPPORTED, "E[%d] is real: the allocation-free step takes complex operators", k);
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  if (noalloc || !ctx->keep_chain || psi->data != ctx->chain_end) ctx->chain_end = nullptr;
  const double half = 0.5 * tau * beta, full = tau * beta;
  if (noalloc) {
    // every product must run in place (no workspace), i.e. its plan must
    // give one workgroup all rows of its fibres; checked for each plan the
    // sweeps below use (phase in the first product, in the last one only on
    // the last step)
    for (int k = 0; k < psi->d; ++k)
      for (int lastep = 0; lastep < 2; ++lastep) {
        mm::ModePlan plan;
        const double pre = k == 0 ? half : 0.0;
        const double post = (k == psi->d - 1 && lastep) ? half : 0.0;
        st = run_mode(ctx, psi->data, psi->data, psi->dims, psi->d, psi->dtype, E[k], k + 1, pre, post, s, &plan,
                      true);
        if (st != MM_OK) return st;
        if (!plan.covers_all_rows)
          return fail(ctx, MM_ERR_SHAPE,
                      "n_%d = %lld: the allocation-free step runs every product in place, which needs "
                      "n_mu <= 256", k + 1, (long long)psi->dims[k]);
      }
  }
  // merged steps: N(tau/2) [L N(tau)]^(nsteps-1) L N(tau/2); each N(tau)
  // between steps is fused into the staging of the next step's first product
  // (where it overlaps MFMA work), the last N(tau/2) into the final epilogue
  if (!noalloc) {
    st = monitor_begin(ctx, nsteps);
    if (st != MM_OK) return st;
  }
  for (int it = 0; it < nsteps; ++it) {
    const double pre = (it == 0) ? half : full;
    const double post = (it + 1 < nsteps) ? 0.0 : half;
    st = sweep(ctx, psi, E, pre, post, s);
    if (st != MM_OK) return st;
    // the phase flows keep |psi|, so the mass between merged steps is the
    // mass after the step
    if (!noalloc && ctx->mon_every > 0 && ((it + 1) % ctx->mon_every == 0 || it + 1 == nsteps)) {
      st = monitor_point(ctx, psi, it + 1, s);
      if (st != MM_OK) return st;
    }
  }
  return noalloc ? MM_OK : monitor_end(ctx, s);
}

}  // namespace

mm_status gpe_strang_step(mm_ctx ctx, mm_tensor* psi, const mm_op* E, double tau, double beta, int nsteps,
                          mm_stream stream) {
  return gpe_strang_impl(ctx, psi, E, tau, beta, nsteps, (hipStream_t)stream, false);
}

mm_status gpe_strang_step_noalloc(mm_ctx ctx, mm_tensor* psi, const mm_op* E, double tau, double beta, int nsteps,
                                  mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  if (3 * mm::SMAX_SLOT + mm::norm_partials() > NOALLOC_SCRATCH_WORDS)
    return fail(ctx, MM_ERR_UNSUPPORTED, "scratch array smaller than the FP16X2 bound slots and partials");
  // the running-bound slots and max-abs partials of the FP16X2 products come
  // from `scratch` (every chain starts with the max-abs pass, which writes
  // all of them, so nothing needs clearing); no monitor, no per-launch events
  uint32_t* own = ctx->smax;
  const bool prof = ctx->profiling;
  ctx->smax = ctx->smax_static;
  ctx->profiling = false;
  const mm_status st = gpe_strang_impl(ctx, psi, E, tau, beta, nsteps, (hipStream_t)stream, true);
  ctx->smax = own;
  ctx->profiling = prof;
  ctx->chain_end = nullptr;
  return st;
}

mm_status ho_strang_step(mm_ctx ctx, mm_tensor* psi, const mm_op* Phi_fwd, const mm_op* Psi_bwd,
                         const double* const* nodes, double t0, double tau, double eps, int nsteps, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, psi, "psi");
  if (st != MM_OK) return st;
  if (!is_complex(psi->dtype)) return fail(ctx, MM_ERR_DTYPE, "psi must be complex");
  if (!Phi_fwd || !Psi_bwd || !nodes) return fail(ctx, MM_ERR_ARG, "Phi_fwd / Psi_bwd / nodes is NULL");
  if (nsteps < 0) return fail(ctx, MM_ERR_ARG, "nsteps < 0");
  if (!std::isfinite(t0) || !std::isfinite(tau) || !std::isfinite(eps)) return fail(ctx, MM_ERR_ARG, "t0 / tau / eps not finite");
  for (int k = 0; k < psi->d; ++k) {
    const mm_op F = Phi_fwd[k], B = Psi_bwd[k];
    if (!F || !B || !nodes[k]) return fail(ctx, MM_ERR_ARG, "Phi_fwd[%d] / Psi_bwd[%d] / nodes[%d] is NULL", k, k, k);
    if (F->cplx || B->cplx) return fail(ctx, MM_ERR_DTYPE, "Phi_fwd[%d] / Psi_bwd[%d] must be real", k, k);
    if (F->idsplit || B->idsplit)
      return fail(ctx, MM_ERR_ARG, "Phi_fwd[%d] / Psi_bwd[%d]: prepared with the identity split", k, k);
    if (F->prec != B->prec) return fail(ctx, MM_ERR_DTYPE, "Phi_fwd[%d] and Psi_bwd[%d] differ in precision", k, k);
    if (F->cols != psi->dims[k] || B->rows != psi->dims[k] || F->rows != B->cols || F->rows > F->cols)
      return fail(ctx, MM_ERR_SHAPE, "mode %d: Phi_fwd must be K x %lld and Psi_bwd %lld x K, K <= %lld", k + 1,
                  (long long)psi->dims[k], (long long)psi->dims[k], (long long)psi->dims[k]);
    st = check_op_dtype(ctx, F, psi->dtype);
    if (st != MM_OK) return st;
    for (int64_t i = 0; i < psi->dims[k]; ++i)
      if (!std::isfinite(nodes[k][i])) return fail(ctx, MM_ERR_ARG, "nodes[%d] holds NaN / Inf", k);
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  // the collapsed propagators of this tau, formed on the device once per
  // (operators, tau, precision)
  for (int k = 0; k < psi->d; ++k) {
    mm_ctx_s::HoMode& H = ctx->ho[k];
    const mm_op F = Phi_fwd[k], B = Psi_bwd[k];
    if (H.phi == F && H.psi == B && H.tau == tau && H.prec == (int)F->prec) continue;
    const int n = (int)psi->dims[k];
    // (a formation that fails leaves none: the master may be gone)
    H.phi = H.psi = nullptr;
    st = grow(ctx, (void**)&H.master, &H.master_bytes, sizeof(double) * 2 * (size_t)n * n);
    if (st != MM_OK) return st;
    HIPCHK(ctx, mm::launch_hermite_collapse(F->dev_master, B->dev_master, n, (int)F->rows, tau, H.master, s));
    H.op = scratch_op(n, F->prec, 0);
    H.op.dev_master = H.master;
    if (F->prec == MM_PREC_SPLIT_FP16X2) {
      // operator scale from the largest entry (one read-back per formation)
      std::vector<double> h((size_t)2 * n * n);
      HIPCHK(ctx, hipMemcpyAsync(h.data(), H.master, h.size() * sizeof(double), hipMemcpyDeviceToHost, s));
      HIPCHK(ctx, hipStreamSynchronize(s));
      double amax = 0.0;
      for (double v : h) amax = std::max(amax, std::fabs(v));
      H.op.a_exp = mm::fp16x2_op_exp(amax);
    }
    H.off = -1.0;
    if (H.op.lay == mm::KY_RES32) {
      // distance from the identity, for the form of its products (one read-back
      // per formation; a formation under capture goes without)
      hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
      HIPCHK(ctx, hipStreamIsCapturing(s, &cap));
      if (cap == hipStreamCaptureStatusNone) {
        HIPCHK(ctx, mm::launch_identity_norms(H.master, n, ctx->red_result, s));
        HIPCHK(ctx, hipMemcpyAsync(ctx->host_result, ctx->red_result, 2 * sizeof(double), hipMemcpyDeviceToHost, s));
        HIPCHK(ctx, hipStreamSynchronize(s));
        H.off = ctx->host_result[0];
        H.all = ctx->host_result[1];
      }
    }
    H.phi = F;
    H.psi = B;
    H.tau = tau;
    H.prec = (int)F->prec;
  }
  // with the potential's phases, at most theta = eps min(tau / 4, 1) max x^2 on
  // rows and on columns: ||P L P - I|| <= ||L - I|| + 2 theta ||L||
  for (int k = 0; k < psi->d; ++k) {
    const mm_ctx_s::HoMode& H = ctx->ho[k];
    double x2 = 0.0;
    for (int64_t i = 0; i < psi->dims[k]; ++i) x2 = std::max(x2, nodes[k][i] * nodes[k][i]);
    const double theta = std::fabs(eps) * std::min(0.25 * std::fabs(tau), 1.0) * x2;
    set_form(&ctx->ho[k].op, H.off >= 0.0 && std::sqrt(H.off) + 2.0 * theta * std::sqrt(H.all) < std::sqrt(1.5 * H.all));
  }
  // squared node coordinates, uploaded when the nodes change (from pinned
  // staging, once the previous upload from it has completed)
  if (!ctx->x2) {
    if (hipMalloc((void**)&ctx->x2, sizeof(double) * MM_MAXD * 4096) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "node buffer");
    if (hipHostMalloc((void**)&ctx->x2_stage, sizeof(double) * MM_MAXD * 4096, hipHostMallocDefault) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "node staging");
    HIPCHK(ctx, hipEventCreateWithFlags(&ctx->x2_ev, hipEventDisableTiming));
  }
  bool changed = false;
  for (int k = 0; k < psi->d && !changed; ++k)
    changed = ctx->x2_nodes[k].size() != (size_t)psi->dims[k] ||
              std::memcmp(ctx->x2_nodes[k].data(), nodes[k], sizeof(double) * psi->dims[k]) != 0;
  if (changed) {
    HIPCHK(ctx, hipEventSynchronize(ctx->x2_ev));
    for (int k = 0; k < MM_MAXD; ++k) ctx->x2_nodes[k].clear();
    for (int k = 0; k < psi->d; ++k) {
      ctx->x2_nodes[k].assign(nodes[k], nodes[k] + psi->dims[k]);
      for (int64_t i = 0; i < psi->dims[k]; ++i) ctx->x2_stage[(size_t)k * 4096 + i] = nodes[k][i] * nodes[k][i];
    }
    HIPCHK(ctx, hipMemcpyAsync(ctx->x2, ctx->x2_stage, sizeof(double) * psi->d * 4096, hipMemcpyHostToDevice, s));
    HIPCHK(ctx, hipEventRecord(ctx->x2_ev, s));
  }
  // per-step operators, prepared for blocks of up to 32 steps (and at most
  // 64 MiB) in one launch per precision, so no preparation sits between the
  // products of a step; without the time-dependent potential (eps = 0) they
  // are the same every step and are prepared once
  size_t need[MM_MAXD];
  size_t per_step = 0;
  for (int k = 0; k < psi->d; ++k) {
    const mm_op_s& L = ctx->ho[k].op;
    need[k] = (mm::prepared_bytes(L.lay, L.KBT, L.MFT) + 255) / 256 * 256;
    per_step += need[k];
  }
  int blk = eps != 0.0 ? 32 : 1;
  while (blk > 1 && per_step * blk > ((size_t)64 << 20)) blk /= 2;
  // (the buffers hold a whole block from the first call on: growing them for
  // a call of more steps costs 1 ms of waiting, freeing and allocating, as
  // much as 17 steps at n = 128; where there is no room for one, they hold
  // this call's steps)
  st = grow_units(ctx, &ctx->step_prep, &ctx->step_prep_bytes, &ctx->step_prep_failed, 0, per_step, &blk,
                  std::min(blk, std::max(nsteps, 1)));
  if (st != MM_OK) return st;
  char* prep_of[MM_MAXD];   // step j of mode k: prep_of[k] + j * need[k]
  for (int k = 0; k < psi->d; ++k)
    prep_of[k] = k == 0 ? (char*)ctx->step_prep : prep_of[k - 1] + need[k - 1] * blk;
  auto prepare_block = [&](int it0, int steps) -> mm_status {
    // one launch per operator layout
    bool done[MM_MAXD] = {false};
    for (int k0 = 0; k0 < psi->d; ++k0) {
      if (done[k0]) continue;
      mm::StepPrep p;
      p.steps = steps;
      p.t0 = t0 + it0 * tau;
      p.tau = tau;
      p.eps = eps;
      for (int k = k0; k < psi->d && p.modes < mm::MAX_STEP_MODES; ++k) {
        if (done[k] || ctx->ho[k].op.lay != ctx->ho[k0].op.lay) continue;
        const mm_op_s& L = ctx->ho[k].op;
        mm::StepPrepMode& m = p.m[p.modes++];
        m.master = L.dev_master;
        m.n = L.rows;
        m.x2 = ctx->x2 + (size_t)k * 4096;
        m.out = prep_of[k];
        m.stride = need[k];
        m.KBT = L.KBT;
        m.MFT = L.MFT;
        m.a_exp = L.a_exp;
        m.minus_id = L.res_id;
        done[k] = true;
      }
      HIPCHK(ctx, mm::launch_prepare_steps(ctx->ho[k0].op.lay, p, s));
    }
    return MM_OK;
  };
  const size_t bytes = (size_t)numel(psi) * dsize(psi->dtype);
  int blk0 = 0;   // first step of the prepared block
  for (int it = 0; it < nsteps; ++it) {
    if (it == 0 || (eps != 0.0 && it - blk0 >= blk)) {
      blk0 = it;
      st = prepare_block(it, eps != 0.0 ? std::min(blk, nsteps - it) : 1);
      if (st != MM_OK) return st;
    }
    const size_t sidx = eps != 0.0 ? (size_t)(it - blk0) : 0;
    void* cur = psi->data;
    for (int k = 0; k < psi->d; ++k) {
      mm_op_s* L = &ctx->ho[k].op;
      const void* prep = prep_of[k] + sidx * need[k];
      mm::ModePlan plan;
      st = run_mode(ctx, cur, cur, psi->dims, psi->d, psi->dtype, L, k + 1, 0, 0, s, &plan, true);
      if (st != MM_OK) return st;
      void* dst = cur;
      if (!plan.covers_all_rows) {
        st = ensure_ws(ctx, bytes);
        if (st != MM_OK) return st;
        dst = (cur == psi->data) ? ctx->ws : psi->data;
      }
      st = run_mode(ctx, cur, dst, psi->dims, psi->d, psi->dtype, L, k + 1, 0, 0, s, nullptr, false, prep);
      if (st != MM_OK) return st;
      cur = dst;
    }
    if (cur != psi->data) {
      HIPCHK(ctx, hipMemcpyAsync(psi->data, cur, bytes, hipMemcpyDeviceToDevice, s));
      if (ctx->chain_end == cur) ctx->chain_end = psi->data;
    }
  }
  return MM_OK;
}

mm_status vortex_strang_step(mm_ctx ctx, mm_tensor* v, const mm_op* E, const double* const* w, double tau, int nsteps,
                             mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, v, "v");
  if (st != MM_OK) return st;
  if (!is_complex(v->dtype)) return fail(ctx, MM_ERR_DTYPE, "v must be complex");
  if (!E || !w) return fail(ctx, MM_ERR_ARG, "E / w is NULL");
  if (nsteps < 0) return fail(ctx, MM_ERR_ARG, "nsteps < 0");
  if (!std::isfinite(tau)) return fail(ctx, MM_ERR_ARG, "tau not finite");
  for (int k = 0; k < v->d; ++k) {
    if (!E[k] || !w[k]) return fail(ctx, MM_ERR_ARG, "E[%d] / w[%d] is NULL", k, k);
    if (E[k]->rows != E[k]->cols || E[k]->cols != v->dims[k])
      return fail(ctx, MM_ERR_SHAPE, "E[%d] must be %lld x %lld", k, (long long)v->dims[k], (long long)v->dims[k]);
    if (v->dims[k] > 4096) return fail(ctx, MM_ERR_SHAPE, "n_%d > 4096", k + 1);
    st = check_op_dtype(ctx, E[k], v->dtype);
    if (st != MM_OK) return st;
    for (int64_t i = 0; i < v->dims[k]; ++i)
      if (!(w[k][i] > 0.0) || !std::isfinite(w[k][i])) return fail(ctx, MM_ERR_ARG, "w[%d][%lld] not a positive width", k, (long long)i);
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  if (nsteps == 0) return MM_OK;
  if (!ctx->winv) {
    if (hipMalloc((void**)&ctx->winv, sizeof(double) * MM_MAXD * 4096) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "weight buffer");
    if (hipHostMalloc((void**)&ctx->winv_stage, sizeof(double) * MM_MAXD * 4096, hipHostMallocDefault) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "weight staging");
    HIPCHK(ctx, hipEventCreateWithFlags(&ctx->winv_ev, hipEventDisableTiming));
  }
  bool changed = false;
  for (int k = 0; k < v->d && !changed; ++k)
    changed = ctx->winv_w[k].size() != (size_t)v->dims[k] ||
              std::memcmp(ctx->winv_w[k].data(), w[k], sizeof(double) * v->dims[k]) != 0;
  if (changed) {
    HIPCHK(ctx, hipEventSynchronize(ctx->winv_ev));
    for (int k = 0; k < MM_MAXD; ++k) ctx->winv_w[k].clear();
    for (int k = 0; k < v->d; ++k) {
      ctx->winv_w[k].assign(w[k], w[k] + v->dims[k]);
      for (int64_t i = 0; i < v->dims[k]; ++i) ctx->winv_stage[(size_t)k * 4096 + i] = 1.0 / w[k][i];
    }
    HIPCHK(ctx, hipMemcpyAsync(ctx->winv, ctx->winv_stage, sizeof(double) * v->d * 4096, hipMemcpyHostToDevice, s));
    HIPCHK(ctx, hipEventRecord(ctx->winv_ev, s));
  }
  const int f64 = is_f64(v->dtype) ? 1 : 0;
  // merged steps N(tau/2) [L N(tau)]^(nsteps-1) L N(tau/2): N keeps |v|, so
  // adjacent half steps compose.  The resident-tile kernels apply each N while
  // they stage the next step's first product, the last one as they write the
  // results (n = 81 FP64: 58.5 us per step against 61.6 with a pass of its
  // own); the others make one pass over the state for each (its coefficient
  // depends on the position through W^-1).  FP16X2: a rotation
  // raises a component by at most sqrt(2), which the state scale's headroom
  // covers (as for the fused prologue phase), so the running bound of the
  // last product carries over the pass to the next step's first product
  bool fused = true;
  for (int k = 0; k < v->d && fused; k += std::max(1, v->d - 1)) {
    mm::ModePlan plan;
    st = run_mode(ctx, v->data, v->data, v->dims, v->d, v->dtype, E[k], k + 1, k == 0 ? tau : 0.0,
                  k == v->d - 1 ? tau : 0.0, s, &plan, true);
    if (st != MM_OK) return st;
    fused = plan.res || plan.rs;
  }
  if (fused) {
    for (int it = 0; it < nsteps; ++it) {
      st = sweep(ctx, v, E, it == 0 ? 0.5 * tau : tau, it + 1 < nsteps ? 0.0 : 0.5 * tau, s, ctx->winv);
      if (st != MM_OK) return st;
    }
    ctx->chain_end = nullptr;
    return MM_OK;
  }
  HIPCHK(ctx, mm::launch_vortex_phase(v->data, f64, v->d, v->dims, ctx->winv, 0.5 * tau, s));
  for (int it = 0; it < nsteps; ++it) {
    st = sweep(ctx, v, E, 0.0, 0.0, s);
    if (st != MM_OK) return st;
    HIPCHK(ctx, mm::launch_vortex_phase(v->data, f64, v->d, v->dims, ctx->winv, it + 1 < nsteps ? tau : 0.5 * tau, s));
  }
  ctx->chain_end = nullptr;
  return MM_OK;
}

mm_status mumode_expstep_batched(mm_ctx ctx, int count, mm_tensor* const* T, const mm_op* const* E, int nsteps,
                                 mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  if (count < 0 || nsteps < 0) return fail(ctx, MM_ERR_ARG, "count / nsteps < 0");
  if (count == 0 || nsteps == 0) return MM_OK;
  if (!T || !E) return fail(ctx, MM_ERR_ARG, "T / E is NULL");
  mm_status st;
  for (int i = 0; i < count; ++i) {
    char nm[32];
    snprintf(nm, sizeof nm, "T[%d]", i);
    st = check_tensor(ctx, T[i], nm);
    if (st != MM_OK) return st;
    if (!E[i]) return fail(ctx, MM_ERR_ARG, "E[%d] is NULL", i);
    for (int k = 0; k < T[i]->d; ++k) {
      mm_op L = E[i][k];
      if (!L) continue;
      if (L->rows != L->cols || L->cols != T[i]->dims[k])
        return fail(ctx, MM_ERR_SHAPE, "E[%d][%d] must be %lld x %lld", i, k, (long long)T[i]->dims[k], (long long)T[i]->dims[k]);
      st = check_op_dtype(ctx, L, T[i]->dtype);
      if (st != MM_OK) return st;
      if (L->prec == MM_PREC_SPLIT_FP16X2)
        return fail(ctx, MM_ERR_UNSUPPORTED, "E[%d][%d]: the batched step has no FP16X2 kernels "
                                             "(a state bound per instance would be needed)", i, k);
    }
    for (int j = 0; j < i; ++j)
      if (overlap(T[i], T[j])) return fail(ctx, MM_ERR_ARG, "T[%d] overlaps T[%d]", i, j);
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  // signature of the batch: tensors and operators
  std::vector<uint64_t> sig;
  sig.push_back((uint64_t)count);
  for (int i = 0; i < count; ++i) {
    sig.push_back((uint64_t)(uintptr_t)T[i]->data);
    sig.push_back((uint64_t)T[i]->d * 16 + (uint64_t)T[i]->dtype);
    for (int k = 0; k < T[i]->d; ++k) {
      const mm_op L = E[i][k];
      sig.push_back((uint64_t)T[i]->dims[k]);
      sig.push_back((uint64_t)(uintptr_t)L);
      sig.push_back(L ? (uint64_t)L->prec : ~(uint64_t)0);
      sig.push_back(L ? (uint64_t)(uintptr_t)L->prep : 0);
    }
  }
  if (sig != ctx->bsig || !ctx->bexec) {
    // build the work items: per mode, one group per kernel (precision,
    // complexity, load path, tile class); every product runs in place
    std::vector<mm::BatchItem> items;
    std::vector<mm::ResArgs> rargs;
    std::vector<mm::ResItem> ritems;
    std::vector<mm_ctx_s::BatchGroup> groups;
    for (int k = 0; k < MM_MAXD; ++k) {
      std::vector<mm::ResItem> byres[2];   // FP64, FP32: one entry per instance (tile: its tile count)
      size_t lds[2] = {0, 0};
      std::vector<std::pair<uint64_t, std::vector<mm::BatchItem>>> byk;
      std::vector<mm::ModePlan> plans;
      for (int i = 0; i < count; ++i) {
        if (k >= T[i]->d || !E[i][k]) continue;
        mm_op L = E[i][k];
        mm::ModePlan plan;
        const int forced = ctx->batch_cls[k][is_complex(T[i]->dtype) ? 1 : 0];
        const int keep_force = ctx->force_cls;
        if (forced >= 0) ctx->force_cls = forced;
        st = run_mode(ctx, T[i]->data, T[i]->data, T[i]->dims, T[i]->d, T[i]->dtype, L, k + 1, 0, 0, s, &plan, true,
                      nullptr, true);
        ctx->force_cls = keep_force;
        if (st != MM_OK) return st;
        if (!plan.covers_all_rows || plan.load == mm::KL_GENERIC || (is_complex(T[i]->dtype) && T[i]->dims[k] > 256))
          return fail(ctx, MM_ERR_UNSUPPORTED, "batched step needs n_mu <= 256 (complex) / 512 (real) and "
                                               "aligned fibres (instance %d, mode %d)", i, k + 1);
        if (is_res(L->lay)) {
          const int w = L->lay == mm::KY_RES64 ? 0 : 1;
          mm::ResArgs a = res_args(T[i]->data, T[i]->data, T[i]->dims, T[i]->d, T[i]->dtype, L, k + 1, 0, 0);
          int kind = 0;
          int64_t tiles = 0;
          size_t need = 0;
          mm::res_batch_plan(w ? mm::KP_F32 : mm::KP_F64, res_form(L, T[i]->dtype), &a, &kind, &tiles, &need);
          lds[w] = std::max(lds[w], need);
          byres[w].push_back(mm::ResItem{(int)rargs.size(), kind, tiles});
          rargs.push_back(a);
          continue;
        }
        void* prep = nullptr;
        int KBT = 0, MFT = 0;
        st = ensure_prepared(ctx, L, is_complex(T[i]->dtype), s, &prep, &KBT, &MFT);
        if (st != MM_OK) return st;
        mm::ModeArgs a;
        int64_t P = 1, Q = 1;
        for (int q = 0; q < k; ++q) P *= T[i]->dims[q];
        for (int q = k + 1; q < T[i]->d; ++q) Q *= T[i]->dims[q];
        const bool cplx = is_complex(T[i]->dtype);
        a.in = T[i]->data;
        a.out = T[i]->data;
        a.A = prep;
        a.P = P;
        a.Q = Q;
        a.F = P * Q;
        a.n = (int)T[i]->dims[k];
        a.m = (int)L->rows;
        a.Kr = (cplx ? 2 : 1) * a.n;
        a.Mr = (cplx ? 2 : 1) * a.m;
        a.KBT = KBT;
        a.MFT = MFT;
        a.s_pre = 0.0;
        a.s_post = 0.0;
        a.smax_in = nullptr;
        a.smax_out = nullptr;
        a.smax_clr = nullptr;
        a.a_exp = 0;
        a.idadd = L->idsplit;
        a.rview = 0;
        // one merged launch per (mode, precision, identity split); the item's
        // kind selects its tile code
        const uint64_t key = (uint64_t)plan.prec * 2 + (L->idsplit ? 1 : 0);
        const int kind = plan.cplx * 100 + plan.load * 10 + plan.cls;
        size_t g = 0;
        while (g < byk.size() && byk[g].first != key) ++g;
        if (g == byk.size()) {
          byk.push_back({key, {}});
          plans.push_back(plan);
        }
        for (int tx = 0; tx < plan.grid_x; ++tx) byk[g].second.push_back(mm::BatchItem{a, tx, 0, kind});
      }
      for (size_t g = 0; g < byk.size(); ++g) {
        // longest tiles first (work ~ K x M of the instance's product), so the
        // launch does not end on a few large tiles started last; the items
        // are independent, so the order changes no result
        std::stable_sort(byk[g].second.begin(), byk[g].second.end(),
                         [](const mm::BatchItem& x, const mm::BatchItem& y) {
                           return (int64_t)x.a.Kr * x.a.Mr > (int64_t)y.a.Kr * y.a.Mr;
                         });
        groups.push_back({plans[g], (int)(byk[g].first & 1), (int)items.size(), (int)byk[g].second.size(), 0});
        items.insert(items.end(), byk[g].second.begin(), byk[g].second.end());
      }
      for (int w = 0; w < 2; ++w) {
        if (byres[w].empty()) continue;
        std::stable_sort(byres[w].begin(), byres[w].end(), [&](const mm::ResItem& x, const mm::ResItem& y) {
          return res_tile_cost(rargs[x.arg], x.kind) > res_tile_cost(rargs[y.arg], y.kind);
        });
        mm::ModePlan plan = {};
        plan.res = 1;
        plan.prec = w ? mm::KP_F32 : mm::KP_F64;
        const size_t first = ritems.size();
        for (const mm::ResItem& x : byres[w])
          for (int64_t tx = 0; tx < x.tile; ++tx) ritems.push_back(mm::ResItem{x.arg, x.kind, tx});
        groups.push_back({plan, 0, (int)first, (int)(ritems.size() - first), lds[w]});
      }
    }
    HIPCHK(ctx, hipStreamSynchronize(s));
    // the captured step reads the lists that the uploads overwrite or free: it
    // goes first, so that no later call can match a rebuild that failed
    batch_invalidate(ctx);
    if ((st = upload(ctx, &ctx->bitems, &ctx->bitems_cap, items)) != MM_OK ||
        (st = upload(ctx, &ctx->rargs, &ctx->rargs_cap, rargs)) != MM_OK ||
        (st = upload(ctx, &ctx->ritems, &ctx->ritems_cap, ritems)) != MM_OK)
      return st;
    ctx->bgroups = groups;
    // capture one step (all modes, all groups) as a graph
    if (!ctx->cap_stream) HIPCHK(ctx, hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking));
    HIPCHK(ctx, hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeThreadLocal));
    hipError_t le = hipSuccess;
    for (const auto& g : ctx->bgroups) {
      if (g.plan.res)
        le = g.plan.prec == mm::KP_F64
                 ? mm::launch_res_batch_f64(ctx->rargs, ctx->ritems + g.offset, g.count, g.lds, ctx->cap_stream)
                 : mm::launch_res_batch_f32(ctx->rargs, ctx->ritems + g.offset, g.count, g.lds, ctx->cap_stream);
      else
        le = mm::launch_mode_batch_merged(g.plan.prec, g.ida, ctx->bitems + g.offset, g.count, ctx->cap_stream);
      if (le != hipSuccess) break;
    }
    hipGraph_t graph = nullptr;
    hipError_t ce = hipStreamEndCapture(ctx->cap_stream, &graph);
    if (le != hipSuccess || ce != hipSuccess) {
      if (graph) hipGraphDestroy(graph);
      return fail(ctx, MM_ERR_HIP, "graph capture failed: %s", hipGetErrorString(le != hipSuccess ? le : ce));
    }
    ctx->bgraph = graph;
    HIPCHK(ctx, hipGraphInstantiate(&ctx->bexec, ctx->bgraph, nullptr, nullptr, 0));
    ctx->bsig = sig;
  }
  for (int it = 0; it < nsteps; ++it) HIPCHK(ctx, hipGraphLaunch(ctx->bexec, s));
  return MM_OK;
}

mm_status mm_energy_gpe(mm_ctx ctx, const mm_tensor* psi, const mm_op* H, double beta, double cell,
                        double* host_out, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, psi, "psi");
  if (st != MM_OK) return st;
  if (!is_complex(psi->dtype)) return fail(ctx, MM_ERR_DTYPE, "psi must be complex");
  if (!H || !host_out) return fail(ctx, MM_ERR_ARG, "H / host_out is NULL");
  for (int k = 0; k < psi->d; ++k) {
    if (!H[k]) return fail(ctx, MM_ERR_ARG, "H[%d] is NULL", k);
    if (H[k]->rows != H[k]->cols || H[k]->cols != psi->dims[k])
      return fail(ctx, MM_ERR_SHAPE, "H[%d] must be %lld x %lld", k, (long long)psi->dims[k], (long long)psi->dims[k]);
    st = check_op_dtype(ctx, H[k], psi->dtype);
    if (st != MM_OK) return st;
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  const size_t bytes = (size_t)numel(psi) * dsize(psi->dtype);
  st = ensure_ws(ctx, bytes);
  if (st != MM_OK) return st;
  const int64_t count = numel(psi);
  const int f64 = is_f64(psi->dtype) ? 1 : 0;
  double total = 0.0;
  for (int k = 0; k < psi->d; ++k) {
    st = run_mode(ctx, psi->data, ctx->ws, psi->dims, psi->d, psi->dtype, H[k], k + 1, 0, 0, s, nullptr, false);
    if (st != MM_OK) return st;
    HIPCHK(ctx, mm::launch_reduce(mm::RED_DOT_RE, psi->data, ctx->ws, count, f64, ctx->red_partial, ctx->red_result, s));
    HIPCHK(ctx, hipMemcpyAsync(ctx->host_result, ctx->red_result, sizeof(double), hipMemcpyDeviceToHost, s));
    HIPCHK(ctx, hipStreamSynchronize(s));
    total += ctx->host_result[0];
  }
  HIPCHK(ctx, mm::launch_reduce(mm::RED_ABS4, psi->data, nullptr, count, f64, ctx->red_partial, ctx->red_result, s));
  HIPCHK(ctx, hipMemcpyAsync(ctx->host_result, ctx->red_result, sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHK(ctx, hipStreamSynchronize(s));
  const double e = cell * (total + 0.5 * beta * ctx->host_result[0]);
  *host_out = e;
  if (!std::isfinite(e)) return fail(ctx, MM_ERR_NONFINITE, "energy is not finite");
  return MM_OK;
}

mm_status mm_profile_begin(mm_ctx ctx) {
  if (!ctx) return MM_ERR_ARG;
  for (auto& r : ctx->recs) {
    hipEventDestroy(r.a);
    hipEventDestroy(r.b);
  }
  ctx->recs.clear();
  ctx->profiling = true;
  return MM_OK;
}

mm_status mm_profile_end(mm_ctx ctx, int max_records, int* count, int* kinds, double* ms) {
  if (!ctx || !count) return MM_ERR_ARG;
  ctx->profiling = false;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  int n = 0;
  for (auto& r : ctx->recs) {
    HIPCHK(ctx, hipEventSynchronize(r.b));
    if (n < max_records && kinds && ms) {
      float t = 0.f;
      HIPCHK(ctx, hipEventElapsedTime(&t, r.a, r.b));
      kinds[n] = r.kind;
      ms[n] = t;
    }
    ++n;
  }
  for (auto& r : ctx->recs) {
    hipEventDestroy(r.a);
    hipEventDestroy(r.b);
  }
  ctx->recs.clear();
  *count = n;
  return MM_OK;
}

mm_status mm_norm2(mm_ctx ctx, const mm_tensor* T, double cell, double* host_out, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, T, "T");
  if (st != MM_OK) return st;
  if (!host_out) return fail(ctx, MM_ERR_ARG, "host_out is NULL");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  const int64_t count = numel(T) * (is_complex(T->dtype) ? 2 : 1);
  HIPCHK(ctx, mm::launch_reduce(mm::RED_SQ, T->data, nullptr, count, is_f64(T->dtype) ? 1 : 0, ctx->red_partial,
                                ctx->red_result, s));
  HIPCHK(ctx, hipMemcpyAsync(ctx->host_result, ctx->red_result, sizeof(double), hipMemcpyDeviceToHost, s));
  HIPCHK(ctx, hipStreamSynchronize(s));
  const double v = ctx->host_result[0] * cell;
  *host_out = v;
  if (!std::isfinite(v)) return fail(ctx, MM_ERR_NONFINITE, "norm is not finite");
  return MM_OK;
}

mm_status mm_set_workspace(mm_ctx ctx, void* dev_ptr, size_t bytes) {
  if (!ctx) return MM_ERR_ARG;
  if (dev_ptr && ((uintptr_t)dev_ptr & 255)) return fail(ctx, MM_ERR_ALIGN, "workspace not 256-byte aligned");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  HIPCHK(ctx, hipDeviceSynchronize());
  if (ctx->ws && !ctx->ws_user) HIPCHK(ctx, hipFree(ctx->ws));
  ctx->ws = dev_ptr;
  ctx->ws_bytes = dev_ptr ? bytes : 0;
  ctx->ws_user = dev_ptr != nullptr;
  return MM_OK;
}

mm_status mm_autotune(mm_ctx ctx, const mm_tensor* T, const mm_op* E, int budget_ms, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, T, "T");
  if (st != MM_OK) return st;
  if (!E) return fail(ctx, MM_ERR_ARG, "E is NULL");
  if (budget_ms < 1) budget_ms = 1;
  for (int k = 0; k < T->d; ++k) {
    if (!E[k]) continue;
    if (E[k]->cols != T->dims[k])
      return fail(ctx, MM_ERR_SHAPE, "E[%d] has %lld columns, n_%d = %lld", k, (long long)E[k]->cols, k + 1,
                  (long long)T->dims[k]);
    st = check_op_dtype(ctx, E[k], T->dtype);
    if (st != MM_OK) return st;
  }
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  const bool cplx = is_complex(T->dtype);
  int modes = 0;
  for (int k = 0; k < T->d; ++k) modes += E[k] ? 1 : 0;
  if (modes == 0) return MM_OK;
  hipEvent_t e0, e1;
  HIPCHK(ctx, hipEventCreate(&e0));
  HIPCHK(ctx, hipEventCreate(&e1));
  struct Ev {
    hipEvent_t a, b;
    ~Ev() { hipEventDestroy(a); hipEventDestroy(b); }
  } guard{e0, e1};
  const double per_mode_ms = (double)budget_ms / modes;
  for (int k = 0; k < T->d; ++k) {
    mm_op L = E[k];
    if (!L) continue;
    // product of mode k+1 of T, out of place into the workspace
    int64_t odims[MM_MAXD];
    for (int q = 0; q < T->d; ++q) odims[q] = T->dims[q];
    odims[k] = L->rows;
    int64_t onum = 1;
    for (int q = 0; q < T->d; ++q) onum *= odims[q];
    st = ensure_ws(ctx, (size_t)onum * dsize(T->dtype));
    if (st != MM_OK) return st;
    const int kp = kprec(L->prec);
    const int ncls = mm::num_classes(kp);
    std::vector<int> cands;
    for (int c = 0; c < ncls; ++c) {
      mm::ModePlan plan;
      ctx->force_cls = c;
      st = run_mode(ctx, T->data, ctx->ws, T->dims, T->d, T->dtype, L, k + 1, 0, 0, s, &plan, true);
      ctx->force_cls = -1;
      if (st == MM_OK && plan.cls == c) cands.push_back(c);
    }
    // unaligned fibres of a split product: only the gather of class 0 and
    // class 6 exist, and the built-in rule separates them
    if ((kp == mm::KP_BF16X3 || kp == mm::KP_FP16X2) && cands.size() > 1) {
      mm::ModePlan plan;
      st = run_mode(ctx, T->data, ctx->ws, T->dims, T->d, T->dtype, L, k + 1, 0, 0, s, &plan, true);
      if (st == MM_OK && plan.load == mm::KL_GENERIC) cands = {plan.cls};
    }
    if (cands.empty()) continue;
    // complex products with a complex operator are timed a second time with
    // the fused prologue phase (the first product of a Gross-Pitaevskii
    // step): the phase adds VALU work to the staging, which changes which
    // tile shape is fastest, so that choice is recorded under its own key
    const bool with_pro = cplx && L->cplx;
    const double per_cand_ms = per_mode_ms / cands.size() / (with_pro ? 2 : 1);
    std::array<int64_t, 6> key{};
    for (int pass = 0; pass < (with_pro ? 2 : 1); ++pass) {
      const double s_pre = pass ? 1e-3 : 0.0;
      // (the resident-tile kernels finish the phase before their products
      // start: the plain choice stands)
      if (pass && is_res(L->lay)) cands = {ctx->tune[key].first};
      int best = -1;
      double best_ms = 0.0;
      for (int c : cands) {
        ctx->force_cls = c;
        mm::ModePlan plan;
        if (pass) {   // classes without instances that carry the phase
          st = run_mode(ctx, T->data, ctx->ws, T->dims, T->d, T->dtype, L, k + 1, s_pre, 0, s, &plan, true);
          if (st != MM_OK || plan.cls != c) {
            ctx->err.clear();
            ctx->force_cls = -1;
            st = MM_OK;
            continue;
          }
        }
        // first launch: warm-up (and, for FP16X2, the bound of T in slot 0)
        ctx->chain_end = nullptr;
        st = run_mode(ctx, T->data, ctx->ws, T->dims, T->d, T->dtype, L, k + 1, s_pre, 0, s, &plan, false);
        if (st == MM_OK) {
          key = ctx->last_key;
          HIPCHK(ctx, hipEventRecord(e0, s));
          ctx->chain_end = T->data;
          ctx->sidx = 0;
          st = run_mode(ctx, T->data, ctx->ws, T->dims, T->d, T->dtype, L, k + 1, s_pre, 0, s, nullptr, false);
          HIPCHK(ctx, hipEventRecord(e1, s));
        }
        if (st != MM_OK) {
          ctx->force_cls = -1;
          return st;
        }
        HIPCHK(ctx, hipEventSynchronize(e1));
        float t1 = 0.f;
        HIPCHK(ctx, hipEventElapsedTime(&t1, e0, e1));
        int reps = (int)std::min(20.0, std::max(2.0, per_cand_ms / std::max(1e-3, (double)t1)));
        HIPCHK(ctx, hipEventRecord(e0, s));
        for (int r = 0; r < reps && st == MM_OK; ++r) {
          ctx->chain_end = T->data;   // every repetition reads the bound of T (slot 0)
          ctx->sidx = 0;
          st = run_mode(ctx, T->data, ctx->ws, T->dims, T->d, T->dtype, L, k + 1, s_pre, 0, s, nullptr, false);
        }
        HIPCHK(ctx, hipEventRecord(e1, s));
        ctx->force_cls = -1;
        if (st != MM_OK) return st;
        HIPCHK(ctx, hipEventSynchronize(e1));
        float tr = 0.f;
        HIPCHK(ctx, hipEventElapsedTime(&tr, e0, e1));
        const double avg = (double)tr / reps;
        if (best < 0 || avg < best_ms) {
          best = c;
          best_ms = avg;
        }
      }
      if (best >= 0) ctx->tune[key] = {best, best_ms * 1e3};
    }
  }
  batch_invalidate(ctx);
  ctx->chain_end = nullptr;
  if (!ctx->tune_path.empty()) return mm_tune_save(ctx, ctx->tune_path.c_str());
  return MM_OK;
}

mm_status mm_autotune_batched(mm_ctx ctx, int count, mm_tensor* const* T, const mm_op* const* E, int budget_ms,
                              mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  if (count <= 0) return MM_OK;
  hipStream_t s = (hipStream_t)stream;
  // the (mode, complex) groups present in the batch
  bool present[MM_MAXD][2] = {};
  for (int i = 0; i < count; ++i) {
    if (!T || !T[i] || !E || !E[i]) return fail(ctx, MM_ERR_ARG, "T / E entry %d is NULL", i);
    for (int k = 0; k < T[i]->d && k < MM_MAXD; ++k)
      // the resident-tile kernels take their shape from the operator alone
      if (E[i][k] && !is_res(E[i][k]->lay)) present[k][is_complex(T[i]->dtype) ? 1 : 0] = true;
  }
  for (int k = 0; k < MM_MAXD; ++k) ctx->batch_cls[k][0] = ctx->batch_cls[k][1] = -1;
  batch_invalidate(ctx);
  hipEvent_t e0, e1;
  HIPCHK(ctx, hipEventCreate(&e0));
  HIPCHK(ctx, hipEventCreate(&e1));
  struct Ev {
    hipEvent_t a, b;
    ~Ev() { hipEventDestroy(a); hipEventDestroy(b); }
  } guard{e0, e1};
  // one captured step per candidate: a warm-up replay, then reps timed replays
  auto time_step = [&](double* ms) -> mm_status {
    mm_status st = mumode_expstep_batched(ctx, count, T, E, 1, stream);
    if (st != MM_OK) return st;
    HIPCHK(ctx, hipEventRecord(e0, s));
    st = mumode_expstep_batched(ctx, count, T, E, 1, stream);
    if (st != MM_OK) return st;
    HIPCHK(ctx, hipEventRecord(e1, s));
    HIPCHK(ctx, hipEventSynchronize(e1));
    float t1 = 0.f;
    HIPCHK(ctx, hipEventElapsedTime(&t1, e0, e1));
    const int reps = (int)std::min(10.0, std::max(2.0, (double)budget_ms / 24.0 / std::max(1e-3, (double)t1)));
    HIPCHK(ctx, hipEventRecord(e0, s));
    st = mumode_expstep_batched(ctx, count, T, E, reps, stream);
    if (st != MM_OK) return st;
    HIPCHK(ctx, hipEventRecord(e1, s));
    HIPCHK(ctx, hipEventSynchronize(e1));
    float tr = 0.f;
    HIPCHK(ctx, hipEventElapsedTime(&tr, e0, e1));
    *ms = (double)tr / reps;
    return MM_OK;
  };
  double best_ms = 0.0;
  mm_status st = time_step(&best_ms);
  if (st != MM_OK) return st;
  // coordinate descent over the groups: each group's class in turn, the
  // others held at their current choice
  for (int k = 0; k < MM_MAXD; ++k)
    for (int c = 0; c < 2; ++c) {
      if (!present[k][c]) continue;
      int best = -1;
      for (int cls = 0; cls <= 2; ++cls) {
        ctx->batch_cls[k][c] = cls;
        batch_invalidate(ctx);
        double ms = 0.0;
        st = time_step(&ms);
        if (st == MM_ERR_UNSUPPORTED) {
          ctx->err.clear();
          continue;
        }
        if (st != MM_OK) {
          ctx->batch_cls[k][c] = best;
          batch_invalidate(ctx);
          return st;
        }
        if (ms < best_ms) {
          best_ms = ms;
          best = cls;
        }
      }
      ctx->batch_cls[k][c] = best;
      batch_invalidate(ctx);
    }
  return MM_OK;
}

mm_status mm_autotune_batched_get(mm_ctx ctx, int mode, int is_complex_, int* cls) {
  if (!ctx || !cls || mode < 1 || mode > MM_MAXD || is_complex_ < 0 || is_complex_ > 1) return MM_ERR_ARG;
  *cls = ctx->batch_cls[mode - 1][is_complex_];
  return MM_OK;
}

mm_status mm_tune_count(mm_ctx ctx, int* count) {
  if (!ctx || !count) return MM_ERR_ARG;
  *count = (int)ctx->tune.size();
  return MM_OK;
}

mm_status mm_tune_get(mm_ctx ctx, int index, int64_t* key6, int* cls, double* us) {
  if (!ctx || index < 0 || index >= (int)ctx->tune.size()) return MM_ERR_ARG;
  auto it = ctx->tune.begin();
  std::advance(it, index);
  if (key6)
    for (int q = 0; q < 6; ++q) key6[q] = it->first[q];
  if (cls) *cls = it->second.first;
  if (us) *us = it->second.second;
  return MM_OK;
}

mm_status mm_tune_clear(mm_ctx ctx) {
  if (!ctx) return MM_ERR_ARG;
  batch_invalidate(ctx);
  ctx->tune.clear();
  for (int k = 0; k < MM_MAXD; ++k) ctx->batch_cls[k][0] = ctx->batch_cls[k][1] = -1;
  return MM_OK;
}

mm_status mm_tune_save(mm_ctx ctx, const char* path) {
  if (!ctx || !path) return MM_ERR_ARG;
  FILE* f = std::fopen(path, "w");
  if (!f) return fail(ctx, MM_ERR_ARG, "cannot write %s", path);
  std::fprintf(f, "mumode-tune 2\n");
  for (const auto& e : ctx->tune)
    std::fprintf(f, "%lld %lld %lld %lld %lld %lld %d %.3f\n", (long long)e.first[0], (long long)e.first[1],
                 (long long)e.first[2], (long long)e.first[3], (long long)e.first[4], (long long)e.first[5],
                 e.second.first, e.second.second);
  const bool ok = std::fclose(f) == 0;
  return ok ? MM_OK : fail(ctx, MM_ERR_ARG, "write of %s failed", path);
}

mm_status mm_tune_load(mm_ctx ctx, const char* path) {
  if (!ctx || !path) return MM_ERR_ARG;
  FILE* f = std::fopen(path, "r");
  if (!f) return fail(ctx, MM_ERR_ARG, "cannot read %s", path);
  char head[32] = {0};
  int ver = 0;
  if (std::fscanf(f, "%31s %d", head, &ver) != 2 || std::strcmp(head, "mumode-tune") != 0 || (ver != 1 && ver != 2)) {
    std::fclose(f);
    return fail(ctx, MM_ERR_ARG, "%s is not a tune file", path);
  }
  std::map<std::array<int64_t, 6>, std::pair<int, double>> t;
  long long k[6];
  int c;
  double us;
  int n;
  while ((n = std::fscanf(f, "%lld %lld %lld %lld %lld %lld %d %lf", &k[0], &k[1], &k[2], &k[3], &k[4], &k[5], &c,
                          &us)) == 8) {
    if (k[0] < 0 || k[0] > mm::KP_BF16 || c < 0 || c >= mm::num_classes((int)k[0])) {
      std::fclose(f);
      return fail(ctx, MM_ERR_ARG, "%s: bad entry", path);
    }
    // Version 1 was also written when FP64 and FP32 products of the resident-
    // tile kernels' sizes ran on the chunked tiles, whose class numbers are other
    // shapes (class 2, the fastest then for 128 real FP64 rows at 16.6 us, would
    // be three fragments per wave, 19.3 us; the built-in choice takes 14.9)
    const bool f64 = k[0] == mm::KP_F64, f32 = k[0] == mm::KP_F32;
    if (ver == 1 && (f64 || f32) && k[3] <= 512 && k[4] <= 512) continue;
    t[{k[0], k[1], k[2], k[3], k[4], k[5]}] = {c, us};
  }
  const bool eof = n == EOF;
  std::fclose(f);
  if (!eof) return fail(ctx, MM_ERR_ARG, "%s: malformed line", path);
  batch_invalidate(ctx);
  for (const auto& e : t) ctx->tune[e.first] = e.second;
  return MM_OK;
}

mm_status mm_expm_device(mm_ctx ctx, int n, const double* A, double c_re, double c_im, double* out,
                         mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  if (!A || !out) return fail(ctx, MM_ERR_ARG, "A / out is NULL");
  if (n < 1 || n > 4096) return fail(ctx, MM_ERR_SHAPE, "n = %d outside [1, 4096]", n);
  if (((uintptr_t)A & 15) || ((uintptr_t)out & 15)) return fail(ctx, MM_ERR_ALIGN, "A / out not 16-byte aligned");
  if (!std::isfinite(c_re) || !std::isfinite(c_im)) return fail(ctx, MM_ERR_ARG, "c not finite");
  const char* a0 = (const char*)A;
  const char* o0 = (const char*)out;
  const size_t bytes = sizeof(double) * 2 * (size_t)n * n;
  if (a0 < o0 + bytes && o0 < a0 + bytes) return fail(ctx, MM_ERR_ARG, "out overlaps A");
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  return expm_device(ctx, n, A, nullptr, 0.0, 0.0, c_re, c_im, -1.0, out, (hipStream_t)stream);
}

mm_status mumode_magnus_step(mm_ctx ctx, mm_tensor* T, const mm_matrix* B, const double* const* dg, const double* g,
                             double tau, int nsteps, mm_prec prec, mm_stream stream) {
  if (!ctx) return MM_ERR_ARG;
  mm_status st = check_tensor(ctx, T, "T");
  if (st != MM_OK) return st;
  if (!is_complex(T->dtype)) return fail(ctx, MM_ERR_DTYPE, "T must be complex");
  if (!B) return fail(ctx, MM_ERR_ARG, "B is NULL");
  if (nsteps < 0) return fail(ctx, MM_ERR_ARG, "nsteps < 0");
  if (!std::isfinite(tau)) return fail(ctx, MM_ERR_ARG, "tau not finite");
  if (prec < MM_PREC_FP64 || prec > MM_PREC_BF16) return fail(ctx, MM_ERR_ARG, "bad precision");
  if ((prec == MM_PREC_FP64) != is_f64(T->dtype))
    return fail(ctx, MM_ERR_DTYPE, "precision %d does not match tensor dtype %d", (int)prec, (int)T->dtype);
  const int d = T->d;
  bool any_t = false;
  for (int k = 0; k < d; ++k) {
    if (!B[k].data) continue;
    if (B[k].rows != T->dims[k] || B[k].cols != T->dims[k])
      return fail(ctx, MM_ERR_SHAPE, "B[%d] must be %lld x %lld", k, (long long)T->dims[k], (long long)T->dims[k]);
    if (B[k].dtype != MM_C128 && B[k].dtype != MM_R64) return fail(ctx, MM_ERR_DTYPE, "B[%d] must be MM_C128 or MM_R64", k);
    if (B[k].ld < B[k].rows) return fail(ctx, MM_ERR_SHAPE, "B[%d]: ld < rows", k);
    if (dg && dg[k]) any_t = true;
  }
  if (any_t && !g) return fail(ctx, MM_ERR_ARG, "g is NULL but a mode has a time-dependent part");
  if (nsteps == 0) return MM_OK;
  HIPCHK(ctx, hipSetDevice(ctx->device));
  ctx->chain_end = nullptr;
  hipStream_t s = (hipStream_t)stream;
  // per-mode state: FP64 complex master and diagonal on the device, the
  // prepared exponentials of a block of steps
  struct Mode {
    int n = 0;
    size_t Boff = 0, doff = 0, poff = 0, pb = 0;   // byte offsets in mg_buf / mg_prep, bytes of one operator
    bool on = false, timed = false;
    double bnorm = 0.0, dmax = 0.0;
    // Gershgorin discs of the Hermitian part (B + B^H)/2: centres Re b_ii,
    // radii sum_{j != i} |b_ij + conj(b_ji)| / 2
    std::vector<double> hc, hr;
    std::vector<int> aexp;   // FP16X2 scale of each prepared exponential
    // FP32: squared Frobenius norms of B and of its Hermitian part without the
    // diagonal; whether each prepared exponential is one less the identity
    double foff = 0.0, hoff = 0.0;
    std::vector<char> near;
    mm_op_s op;
  };
  std::vector<Mode> modes(d);
  // the buffers below belong to the context: nothing of this call may still
  // run when it returns, also when it fails
  struct Guard {
    ~Guard() { hipDeviceSynchronize(); }
  } guard;
  size_t need = 0;
  auto reserve = [&](size_t bytes) {
    const size_t at = need;
    need += (bytes + 255) / 256 * 256;
    return at;
  };
  for (int k = 0; k < d; ++k) {
    if (!B[k].data) continue;
    Mode& M = modes[k];
    M.on = true;
    M.n = (int)T->dims[k];
    M.timed = dg && dg[k];
    M.Boff = reserve(sizeof(double) * 2 * (size_t)M.n * M.n);
    if (M.timed) M.doff = reserve(sizeof(double) * M.n);
    M.op = scratch_op(M.n, prec, 0);
    M.pb = (mm::prepared_bytes(M.op.lay, M.op.KBT, M.op.MFT) + 255) / 256 * 256;
  }
  if ((st = grow(ctx, &ctx->mg_buf, &ctx->mg_bytes, need)) != MM_OK) return st;
  if (ctx->mg_stage_bytes < need) {
    if (ctx->mg_stage) HIPCHK(ctx, hipHostFree(ctx->mg_stage));
    ctx->mg_stage = nullptr;
    ctx->mg_stage_bytes = 0;
    if (hipHostMalloc(&ctx->mg_stage, need, hipHostMallocDefault) != hipSuccess)
      return fail(ctx, MM_ERR_NOMEM, "staging of %zu bytes", need);
    ctx->mg_stage_bytes = need;
  }
  for (int k = 0; k < d; ++k) {
    Mode& M = modes[k];
    if (!M.on) continue;
    const int n = M.n;
    const int comps = B[k].dtype == MM_C128 ? 2 : 1;
    std::vector<double> full;
    const double* src = (const double*)B[k].data;
    if (B[k].on_device) {
      full.resize((size_t)B[k].ld * n * comps);
      HIPCHK(ctx, hipMemcpy(full.data(), src, full.size() * sizeof(double), hipMemcpyDeviceToHost));
      src = full.data();
    }
    double* host = (double*)((char*)ctx->mg_stage + M.Boff);
    double check = 0.0;
    for (int j = 0; j < n; ++j) {
      const double* col = src + (size_t)j * B[k].ld * comps;
      double* o = host + 2 * (size_t)j * n;
      double sum = 0.0;
      for (int i = 0; i < n; ++i) {
        const double re = col[(size_t)i * comps], im = comps == 2 ? col[(size_t)i * 2 + 1] : 0.0;
        o[2 * i] = re;
        o[2 * i + 1] = im;
        check += 0.0 * re + 0.0 * im;   // NaN as soon as one entry is not finite
        sum += std::sqrt(re * re + im * im);
      }
      if (!std::isfinite(sum)) {        // squares out of range
        sum = 0.0;
        for (int i = 0; i < n; ++i) sum += std::hypot(o[2 * i], o[2 * i + 1]);
      }
      M.bnorm = std::max(M.bnorm, sum);
    }
    if (check != 0.0) return fail(ctx, MM_ERR_NONFINITE, "B[%d] holds NaN / Inf", k);
    if (is_res(M.op.lay) && prec == MM_PREC_FP32)
      for (int j = 0; j < n; ++j)
        for (int i = 0; i < j; ++i) {
          const double *a = host + 2 * ((size_t)j * n + i), *b = host + 2 * ((size_t)i * n + j);
          const double re = a[0] + b[0], im = a[1] - b[1];
          M.foff += a[0] * a[0] + a[1] * a[1] + b[0] * b[0] + b[1] * b[1];
          M.hoff += 0.5 * (re * re + im * im);
        }
    if (prec == MM_PREC_SPLIT_FP16X2) {
      M.hc.assign(n, 0.0);
      M.hr.assign(n, 0.0);
      for (int i = 0; i < n; ++i) {
        M.hc[i] = host[2 * ((size_t)i * n + i)];
        for (int j = 0; j < n; ++j) {
          if (j == i) continue;
          const double re = host[2 * ((size_t)j * n + i)] + host[2 * ((size_t)i * n + j)];
          const double im = host[2 * ((size_t)j * n + i) + 1] - host[2 * ((size_t)i * n + j) + 1];
          M.hr[i] += 0.5 * std::hypot(re, im);
        }
      }
    }
    if (M.timed) {
      double* dd = (double*)((char*)ctx->mg_stage + M.doff);
      for (int i = 0; i < n; ++i) {
        if (!std::isfinite(dg[k][i])) return fail(ctx, MM_ERR_NONFINITE, "d[%d] holds NaN / Inf", k);
        dd[i] = dg[k][i];
        M.dmax = std::max(M.dmax, std::fabs(dg[k][i]));
      }
    }
  }
  if (need) HIPCHK(ctx, hipMemcpyAsync(ctx->mg_buf, ctx->mg_stage, need, hipMemcpyHostToDevice, s));
  // the exponentials of a block of steps are formed together, ahead of its
  // products (at most 256 MiB of prepared operators)
  size_t fixed = 0, per_step = 0;
  for (const Mode& M : modes)
    if (M.on) (M.timed ? per_step : fixed) += M.pb;
  int blk = per_step ? std::min(nsteps, 32) : nsteps;
  while (per_step && blk > 1 && per_step * blk > ((size_t)256 << 20)) blk /= 2;
  {
    // one exponential's buffers first: a block takes what is left
    for (const Mode& M : modes)
      if (M.on && (st = expm_buffers(ctx, M.n, M.n > mm::EXPM_MAX_N)) != MM_OK) return st;
    st = grow_units(ctx, &ctx->mg_prep, &ctx->mg_prep_bytes, &ctx->mg_prep_failed, fixed, per_step, &blk,
                    per_step ? 1 : blk);
    if (st != MM_OK) return st;
    size_t at = 0;
    for (Mode& M : modes)
      if (M.on) {
        M.poff = at;
        at += M.pb * (M.timed ? (size_t)blk : 1);
      }
  }
  const size_t bytes = (size_t)numel(T) * dsize(T->dtype);
  for (int it0 = 0; it0 < nsteps; it0 += blk) {
    const int cnt = std::min(blk, nsteps - it0);
    // jobs of one size, layout and number of squarings run as one batch
    mm::ExpmBatch batch = {};
    const mm_op_s* bop = nullptr;
    auto flush = [&]() -> mm_status {
      if (batch.nb == 0) return MM_OK;
      int units = batch.nb;   // as many at a time as there is memory for
      mm_status r = grow_units(ctx, (void**)&ctx->ex_buf, &ctx->ex_bytes, &ctx->ex_failed,
                               sizeof(double) * batch.n, mm::expm_batch_bytes(batch.n, 1), &units, 1);
      if (r != MM_OK) return r;
      for (int j0 = 0; j0 < batch.nb; j0 += units) {
        mm::ExpmBatch part = batch;
        part.nb = std::min(units, batch.nb - j0);
        std::copy(batch.j + j0, batch.j + j0 + part.nb, part.j);
        double* e = nullptr;
        HIPCHK(ctx, mm::launch_expm_batch(part, ctx->ex_buf, &e, s));
        HIPCHK(ctx, mm::launch_prepare_jobs(bop->lay, part, e, bop->KBT, bop->MFT, s));
      }
      batch.nb = 0;
      return MM_OK;
    };
    for (int k = 0; k < d; ++k) {
      Mode& M = modes[k];
      if (!M.on || (!M.timed && it0 > 0)) continue;
      for (int j = 0; j < (M.timed ? cnt : 1); ++j) {
        // E_k = exp(tau (B_k + g diag d_k)) at the midpoint of step it0 + j
        double gr = 0.0, gi = 0.0;
        if (M.timed) {
          gr = g[2 * ((size_t)(it0 + j) * d + k)];
          gi = g[2 * ((size_t)(it0 + j) * d + k) + 1];
          if (!std::isfinite(gr) || !std::isfinite(gi)) return fail(ctx, MM_ERR_NONFINITE, "g not finite");
        }
        const double bound = M.bnorm + std::hypot(gr, gi) * M.dmax;
        // FP16X2 operator scale from a bound of max |E_ij|: |E_ij| <= ||E||_2
        // <= exp(tau mu(A)) with mu the logarithmic 2-norm, the largest
        // eigenvalue of the Hermitian part of A = B + g diag(d) (that part is
        // (B + B^H)/2 + Re(g) diag(d)), bounded by its Gershgorin discs; for
        // tau < 0 the same with -A.  For a skew-Hermitian (unitary-flow)
        // generator the bound is 1, the true size of the entries.
        int a_exp = 0;
        if (prec == MM_PREC_SPLIT_FP16X2) {
          double mu = -HUGE_VAL;
          const double sg = tau >= 0.0 ? 1.0 : -1.0;
          for (int i = 0; i < M.n; ++i) {
            const double c = M.hc[i] + (M.timed ? gr * dg[k][i] : 0.0);
            mu = std::max(mu, sg * c + M.hr[i]);
          }
          a_exp = mm::fp16x2_op_exp(std::exp(std::min(700.0, std::fabs(tau) * mu)));
        }
        // FP32 form: with A = tau (B + g diag(d)) and H its Hermitian part,
        // ||e^A - I||_F <= ||A||_F e^||H|| and ||e^A||_F >= sqrt(n) e^-||H||
        bool near = false;
        if (is_res(M.op.lay) && prec == MM_PREC_FP32) {
          const double* host = (const double*)((const char*)ctx->mg_stage + M.Boff);
          double f = M.foff, h = M.hoff;
          for (int i = 0; i < M.n; ++i) {
            const double* b = host + 2 * ((size_t)i * M.n + i);
            const double di = M.timed ? dg[k][i] : 0.0;
            const double re = b[0] + gr * di, im = b[1] + gi * di;
            f += re * re + im * im;
            h += re * re;
          }
          near = std::fabs(tau) * std::sqrt(f) * std::exp(2.0 * std::fabs(tau) * std::sqrt(h)) <
                 std::sqrt(1.5 * M.n);
        }
        if ((int)M.aexp.size() <= j) M.aexp.resize(j + 1);
        if ((int)M.near.size() <= j) M.near.resize(j + 1);
        M.aexp[j] = a_exp;
        M.near[j] = near;
        const double* A = (const double*)((char*)ctx->mg_buf + M.Boff);
        const double* dd = M.timed ? (const double*)((char*)ctx->mg_buf + M.doff) : nullptr;
        void* out = (char*)ctx->mg_prep + M.poff + (size_t)j * M.pb;
        if (M.n > mm::EXPM_MAX_N) {
          st = expm_device(ctx, M.n, A, dd, gr, gi, tau, 0.0, bound, ctx->mg_exp, s);
          if (st != MM_OK) return st;
          HIPCHK(ctx, mm::launch_prepare(M.op.lay, 1, ctx->mg_exp, M.n, M.n, M.n, mm::PhaseScale(), out, M.op.KBT,
                                         M.op.MFT, s, a_exp));
          continue;
        }
        int q = 0;
        if ((st = expm_squarings(ctx, std::fabs(tau) * bound, &q)) != MM_OK) return st;
        const int cap = (int)std::max<size_t>(1, std::min<size_t>(mm::MAX_EXPM, ((size_t)64 << 20) / mm::expm_batch_bytes(M.n, 1)));
        if (batch.nb && (batch.n != M.n || batch.q != q || bop->lay != M.op.lay || batch.nb >= cap))
          if ((st = flush()) != MM_OK) return st;
        batch.n = M.n;
        batch.q = q;
        bop = &M.op;
        batch.j[batch.nb++] = {A, dd, gr, gi, tau, 0.0, out, a_exp, near};
      }
    }
    if ((st = flush()) != MM_OK) return st;
    for (int it = it0; it < it0 + cnt; ++it) {
      void* cur = T->data;
      for (int k = 0; k < d; ++k) {
        Mode& M = modes[k];
        if (!M.on) continue;
        const int j = M.timed ? it - it0 : 0;
        const void* P = (char*)ctx->mg_prep + M.poff + (size_t)j * M.pb;
        M.op.a_exp = M.aexp[j];
        set_form(&M.op, M.near[j]);
        mm::ModePlan plan;
        st = run_mode(ctx, cur, cur, T->dims, d, T->dtype, &M.op, k + 1, 0, 0, s, &plan, true, P);
        if (st != MM_OK) return st;
        void* dst = cur;
        if (!plan.covers_all_rows) {
          st = ensure_ws(ctx, bytes);
          if (st != MM_OK) return st;
          dst = (cur == T->data) ? ctx->ws : T->data;
        }
        st = run_mode(ctx, cur, dst, T->dims, d, T->dtype, &M.op, k + 1, 0, 0, s, nullptr, false, P);
        if (st != MM_OK) return st;
        cur = dst;
      }
      if (cur != T->data) {
        HIPCHK(ctx, hipMemcpyAsync(T->data, cur, bytes, hipMemcpyDeviceToDevice, s));
        if (ctx->chain_end == cur) ctx->chain_end = T->data;
      }
    }
  }
  return MM_OK;
}

mm_status mm_set_option(mm_ctx ctx, int option, int64_t value) {
  if (!ctx) return MM_ERR_ARG;
  switch (option) {
    case MM_OPT_SMALL_RUN:
      ctx->small_run = value != 0;
      return MM_OK;
    case MM_OPT_MONITOR_EVERY:
      if (value < 0 || value > (1 << 30)) return fail(ctx, MM_ERR_ARG, "monitor interval %lld", (long long)value);
      ctx->mon_every = (int)value;
      return MM_OK;
    case MM_OPT_FP16X2_CHAIN:
      if (value != 0 && value != 1) return fail(ctx, MM_ERR_ARG, "MM_OPT_FP16X2_CHAIN takes 0 or 1");
      ctx->keep_chain = value != 0;
      ctx->chain_end = nullptr;
      return MM_OK;
    default:
      return fail(ctx, MM_ERR_ARG, "unknown option %d", option);
  }
}

mm_status mm_monitor_log(mm_ctx ctx, int max_records, int* count, int* steps, double* sums) {
  if (!ctx || !count) return MM_ERR_ARG;
  const int k = (int)ctx->mon_vals.size();
  for (int i = 0; i < k && i < max_records; ++i) {
    if (steps) steps[i] = ctx->mon_steps[i];
    if (sums) sums[i] = ctx->mon_vals[i];
  }
  *count = k;
  return MM_OK;
}

}  // extern "C"
