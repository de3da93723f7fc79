// Internal interface between the host runtime (mumode_runtime.cpp) and the
// HIP kernels (mode_kernels.hip).  Not part of the public C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mm {

enum KPrec { KP_F64 = 0, KP_F32 = 1, KP_BF16X3 = 2, KP_FP16X2 = 3, KP_BF16 = 4 };
// Operator layouts: the precision codes above name the fragment order of the
// chunked kernels (mode_tile.h); these two are the layouts of the resident-
// tile kernels (resident.h).  KBT counts 16-byte units along K, MFT 16-row
// fragments.
enum KLayout { KY_RES64 = 5, KY_RES32 = 6 };
// Fibre load paths: KCONTIG fibres contiguous (mu = 1, P = 1); FCONTIG
// fibres interleaved with P % 4 == 0 (16-byte loads along P); GENERIC any
// P (gather); PAIR P == 2, pairs of fibres interleaved (a real operator on
// the (re, im) planes of a complex state along mode 1: each 16-byte load
// holds two fibres' consecutive entries).
enum KLoad { KL_KCONTIG = 0, KL_FCONTIG = 1, KL_GENERIC = 2, KL_PAIR = 3 };

// Geometry of the MFMA fragment a precision uses: M rows and K values per
// fragment, K values each lane holds, operator pieces per value (FP16X2
// keeps three: hi * 2^11, hi, lo; see mode_tile.h).
// KPAD / MPAD: the prepared operator's K-blocks and M-fragments are padded
// (with zeros) to multiples of these, so that every tile shape reads whole
// chunks and whole row tiles.
struct FragGeom {
  int MB, NB, KB, KPL, NPC, KPAD, MPAD;
};
FragGeom frag_geom(int prec);
// Padded K-block and M-fragment counts of a prepared operator with Mr real
// rows and Kr real columns.
void op_blocks(int prec, int64_t Mr, int64_t Kr, int* KBT, int* MFT);
// 16-byte units along K and 16-row fragments of a resident-layout operator.
void res_blocks(int lay, int64_t rows, int64_t cols, int cplx, int* KU, int* MFT);

// Arguments of one mu-mode product launch (real-GEMM view, see
// mode_kernels.hip).  Complex tensors: P, Q, n, m count complex entries.
// Words per running-bound slot: the workgroups of a launch spread their
// atomic maxima over this many words, so they do not all queue on one, and the
// words lie 256 bytes apart: in one cache line they queue all the same, at the
// end of every launch (real operator on 128 x 16384 complex fibres 15.9 -> 12.6
// us; 32 words of 128 bytes 14.5, the readers fetch four times the lines).
constexpr int SMAX_WORDS = 8;
constexpr int SMAX_STRIDE = 64;
constexpr int SMAX_SLOT = SMAX_WORDS * SMAX_STRIDE;

struct ModeArgs {
  const void* in;
  void* out;
  const void* A;       // operator in fragment order (mm_prepare_operator)
  int64_t P, Q, F;     // fibres: F = P*Q, entry (p, j, q) at p + P*(j + n*q)
  int n, m;            // mode length of input / output
  int Kr, Mr;          // real-GEMM K and M (2n, 2m when complex)
  int KBT, MFT;        // padded K-blocks and M-fragments of the prepared operator
  double s_pre;        // prologue phase: psi *= exp(-i s_pre |psi|^2) (0: off)
  double s_post;       // epilogue phase, same form
  // FP16X2 only: running bound of the state.  Each slot is SMAX_WORDS words,
  // SMAX_STRIDE apart; their maximum in smax_in is the float bits of max
  // |component| of `in`; the launch raises smax_out (workgroup tile_x the word
  // tile_x % SMAX_WORDS) to that of `out` and clears smax_clr (the slot the
  // launch before it read).  The operator pieces represent L * 2^-a_exp.
  const uint32_t* smax_in;
  uint32_t* smax_out;
  uint32_t* smax_clr;
  int a_exp;
  // identity split: the operator pieces hold L - I (square L) and the
  // epilogue adds the input entry at the same position back in FP32 (after
  // the prologue phase when there is one)
  int idadd;
  int rview;           // real operator on the (re, im) planes of a complex state
};

// Per-workgroup work item of a batched launch.
struct BatchItem {
  ModeArgs a;
  int64_t tile_x;
  int tile_y;
  int kind;            // complex * 100 + load path * 10 + tile class (0..2)
};

typedef void (*KernFn)(ModeArgs);
typedef void (*BatchFn)(const BatchItem*);

// Workgroup tile shape: WM x WN waves, each with WMF x WNF MFMA fragments,
// KCH K-blocks per LDS chunk.
struct TileShape {
  int WMF, WNF, WM, WN, KCH, OCC;
};

// Kernel tables, one per precision (kern_<prec>.hip).  cls selects the tile
// shape (0 default; 1, 2 regrouped waves for operators with at most 256 / 128
// real rows; 3..6 alternative split shapes).  nullptr if no instance exists.
KernFn pick_kernel_f64(int cplx, int ld, int pro, int epi, int cls, int full, int ida);
KernFn pick_kernel_f32(int cplx, int ld, int pro, int epi, int cls, int full, int ida);
KernFn pick_kernel_bf16x3(int cplx, int ld, int pro, int epi, int cls, int full, int ida);
KernFn pick_kernel_fp16x2(int cplx, int ld, int pro, int epi, int cls, int full, int ida);
KernFn pick_kernel_bf16(int cplx, int ld, int pro, int epi, int cls, int full, int ida);
bool batch_kind_f64(int cplx, int ld, int cls);
bool batch_kind_f32(int cplx, int ld, int cls);
bool batch_kind_bf16x3(int cplx, int ld, int cls);
bool batch_kind_fp16x2(int cplx, int ld, int cls);
bool batch_kind_bf16(int cplx, int ld, int cls);
bool tile_shape_f64(int cls, TileShape* out);
bool tile_shape_f32(int cls, TileShape* out);
bool tile_shape_bf16x3(int cls, TileShape* out);
bool tile_shape_fp16x2(int cls, TileShape* out);
bool tile_shape_bf16(int cls, TileShape* out);

bool tile_shape(int prec, int cls, TileShape* out);

// Three-product (Gauss) complex split kernels (kern_<prec>_g.hip), tile
// classes 8 and 9 of BF16X3 and FP16X2: complex operator and state,
// contiguous or strided fibres, operator prepared by launch_prepare_gauss.
KernFn pick_gauss_bf16x3(int ld, int pro, int epi, int cls, int full);
KernFn pick_gauss_fp16x2(int ld, int pro, int epi, int cls, int full);
bool gauss_shape_bf16x3(int cls, TileShape* out);
bool gauss_shape_fp16x2(int cls, TileShape* out);
inline bool is_gauss_class(int cls) { return cls == 8 || cls == 9; }
// Padded complex K-blocks (16 columns, a multiple of 4) and complex-row
// fragments (32 rows, a multiple of 8) of a three-product operator.
void gauss_blocks(int64_t rows, int64_t cols, int* JBT, int* MFT);
size_t gauss_prepared_bytes(int prec, int JBT, int MFT);
// master: complex FP64, column-major with leading dimension ld.
hipError_t launch_prepare_gauss(int prec, const double* master, int64_t rows, int64_t cols, int64_t ld, void* out,
                                int JBT, int MFT, int a_exp, hipStream_t s);

// Merged batched launch: one kernel per precision runs work items of every
// kind (complex / real, contiguous / strided fibres, tile class 0..2; all
// 256 threads), so every instance tile of one mode goes in a single launch.
BatchFn pick_batch_merged_bf16x3();
BatchFn pick_batch_merged_bf16();
BatchFn pick_batch_merged_bf16x3_ida();
BatchFn pick_batch_merged_bf16_ida();
// ida: the items' operators carry the identity split (a.idadd set on all)
hipError_t launch_mode_batch_merged(int prec, int ida, const BatchItem* items, int count, hipStream_t s);

// Resident-tile kernels (kern_res_<prec>.hip), FP64 and FP32: one launch
// applies an operator of at most 256 complex / 512 real rows and columns to
// every fibre, with the whole fibre tile in LDS (resident.h).
// operator x state: complex x complex in three or four real products, real x
// complex, real x real
enum ResForm { RF_C3 = 0, RF_RC = 1, RF_RR = 2, RF_C4 = 3 };
// Position-dependent phase exp((i s/2)(1 - W^-1 |v|^2)) in place of the Gross-
// Pitaevskii one: W^-1 = prod_j winv[j * 4096 + i_j] over the wd modes of
// lengths wdims; wmu is the (0-based) mode of the product.  winv null: none.
struct VortexW {
  const double* winv;
  int wd, wmu;
  int64_t wdims[6];
};
struct ResArgs {
  const void* in;
  void* out;
  const void* A;         // operator in the KY_RES layout of its precision
  int64_t P, F;          // fibre (p, q), q = f / P: entry j at p + P * (j + n * q)
  int n, m;              // entries of an input / output fibre
  int MFT;               // 16-row fragments of the prepared operator (padded)
  int WM, WN;            // waves along rows and fibres
  int NRB;               // row blocks a workgroup works through (1 when nsteps > 1)
  int nsteps;            // products applied to the resident tile (square operators; 1 otherwise)
  int idadd;             // the operator holds L - I: add the input back
  double s_pre, s_post;  // phase coefficients (0: none)
  VortexW w;
};
// Longest operator side of the resident kernels.
inline bool res_fits(int64_t rows, int64_t cols, int cplx) {
  const int64_t lim = cplx ? 256 : 512;
  return rows <= lim && cols <= lim;
}
// LDS of a workgroup.
constexpr size_t MAX_LDS = 160 * 1024;
// LDS rows of a tile: whole operator units and one K-block that is read ahead.
inline int res_lds_rows(int n) { return (n + 15) / 16 * 16 + 4; }
struct ResPlan {
  int prec, form, mf, nf, ph, threads;
  int grid_x, grid_y;    // tile y * grid_x + x; those past the last fibre have nothing to do
  int run;               // 32 or 64 rows: the operator stays in registers over the products (0: no)
  size_t lds;
};
// Launch shape of one product (fills a.WM / a.WN).  cls: tile class chosen by
// the tuner (MF = cls + 1 fragments per wave), -1 for the built-in rule.
void res_plan(int prec, int form, bool ph, int cls, ResArgs* a, ResPlan* p);
hipError_t launch_res(const ResPlan& p, const ResArgs& a, hipStream_t s, hipEvent_t start = nullptr,
                      hipEvent_t stop = nullptr);
hipError_t launch_res_f64(const ResPlan& p, const ResArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop);
hipError_t launch_res_f32(const ResPlan& p, const ResArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop);
// Batched form: work item i runs tile `tile` of args[arg] with the tile code
// kind = form * 10 + MF (4 waves, NF = 1), or RES_KIND_NF2 + MF for real fibres
// with NF = 2; res_batch_plan fills WM, WN, NRB.
constexpr int RES_KIND_NF2 = 100;
void res_batch_plan(int prec, int form, ResArgs* a, int* kind, int64_t* tiles, size_t* lds);
struct ResItem {
  int arg, kind;
  int64_t tile;
};
hipError_t launch_res_batch_f64(const ResArgs* args, const ResItem* items, int count, size_t lds, hipStream_t s);
hipError_t launch_res_batch_f32(const ResArgs* args, const ResItem* items, int count, size_t lds, hipStream_t s);

// Per-launch plan chosen by the runtime.
struct ModePlan {
  int prec, cplx, load, pro, epi;
  int cls;             // tile shape class
  int grid_x, grid_y, threads;
  int nt;              // fibres per workgroup
  int mt_rows;         // real rows covered by one workgroup (multiple of MB)
  bool covers_all_rows;
  int full;            // every tile complete and output offsets fit 32 bits
  int gauss;           // three-product kernel: the operator's Gauss preparation
  int rs = 0;          // resident-tile split kernel (class 6): N-fragments per tile
  int rs_form = 0;     // RsForm
  size_t rs_lds = 0;
  int res = 0;         // resident-tile kernel (FP64 / FP32; rp is its launch shape)
  ResPlan rp;
};

// Resident-tile kernels of the split products (rsplit.h), tile class 6 of FP16X2
// and BF16X3: operators of at most 512 real rows and columns.
constexpr int RS_CLASS = 6;
enum RsForm { RS_CC = 0, RS_RC = 1, RS_RR = 2 };   // operator x fibres: complex or real
bool rs_plan(const ModeArgs& a, int prec, int cplx, ModePlan* plan);
hipError_t launch_rsplit_fp16x2(const ModePlan& p, const ModeArgs& a, const VortexW& w, hipStream_t s, hipEvent_t start,
                                hipEvent_t stop);
hipError_t launch_rsplit_bf16x3(const ModePlan& p, const ModeArgs& a, const VortexW& w, hipStream_t s, hipEvent_t start,
                                hipEvent_t stop);

// Fill `plan` for the given problem; returns false if no kernel fits.
// batch: plan for the batched work-list kernel (tile classes 0..2 only).
// force_cls >= 0: use that tile class if an instance exists for the problem
// (the autotuner's choice), else fall back to the built-in choice.
bool plan_mode(const ModeArgs& a, int prec, int cplx, bool want_pro, bool want_epi,
               bool fcontig_ok, bool kcontig_ok, ModePlan* plan, bool batch = false, int force_cls = -1,
               bool gauss_ok = false);
// Number of tile classes of a precision (classes 0 .. n-1).
int num_classes(int prec);
// start / stop (optional): events recorded by the launch itself; w: vortex
// phase (class 6 only)
hipError_t launch_mode(const ModePlan& plan, const ModeArgs& a, hipStream_t s, hipEvent_t start = nullptr,
                       hipEvent_t stop = nullptr, const VortexW* w = nullptr);
// Optional diagonal phase scaling of a complex master before conversion:
// L'[i,j] = exp(-i rc rx2[i]) L[i,j] exp(-i cc cx2[j]); rx2 / cx2 are device
// arrays (null = no factor).
struct PhaseScale {
  const double* rx2 = nullptr;
  double rc = 0.0;
  const double* cx2 = nullptr;
  double cc = 0.0;
  int minus_id = 0;   // resident layouts: prepare L - I (products add the input back)
};

// The collapsed harmonic-oscillator propagators of `steps` consecutive steps
// of the time-dependent splitting, for up to 6 modes of one precision, in
// one launch: step s, entry e gets the diagonal phase factors
// exp(-i ca x_i^2) on its rows and exp(-i cb x_j^2) on its columns, where
// cb and ca are the potential's flows over the step's two halves,
// (eps/2)(cos t - cos(t + tau/2)) and (eps/2)(cos(t + tau/2) - cos(t + tau))
// with t = t0 + s tau, formed on the device.
constexpr int MAX_STEP_MODES = 6;
struct StepPrepMode {
  const double* master = nullptr;   // complex FP64, n x n, ld = n
  int64_t n = 0;
  const double* x2 = nullptr;       // squared nodes of the mode
  char* out = nullptr;              // step s at out + s * stride
  size_t stride = 0;
  int KBT = 0, MFT = 0, a_exp = 0;
  int minus_id = 0;                 // resident layouts: prepare L - I
};
struct StepPrep {
  StepPrepMode m[MAX_STEP_MODES];
  int modes = 0, steps = 0;
  double t0 = 0.0, tau = 0.0, eps = 0.0;
};
hipError_t launch_prepare_steps(int prec, const StepPrep& p, hipStream_t s);

// Convert an FP64 master (device, column-major, ld) into fragment order.
// a_exp (FP16X2 only): the pieces represent master * 2^-a_exp.
hipError_t launch_prepare(int prec, int cplx, const double* master, int64_t rows, int64_t cols,
                          int64_t ld, PhaseScale ph, void* out, int KBT, int MFT, hipStream_t s,
                          int a_exp = 0);
// Scale exponent of an operator whose largest |real component| is amax:
// the scaled entries stay below 16 (so hi * 2^11 stays below 2^15).
int fp16x2_op_exp(double amax);
// Device matrix exponential helpers (complex FP64, column-major interleaved,
// n x n): X = f (A + g diag(d)) (d real, nullable); T = I + f W (W null:
// T = I); out[j] = sum_i |(A + g diag(d))_ij|.
hipError_t launch_expm_generator(const double* A, int n, const double* d, double gr, double gi, double fr, double fi,
                                 double* X, hipStream_t s);
hipError_t launch_expm_colsum(const double* A, int n, const double* d, double gr, double gi, double* out,
                              hipStream_t s);
// P = W + c[0] I + c[1] X + c[2] X2 + c[3] X3 (W nullable)
hipError_t launch_expm_ps(double* P, const double* W, const double* X, const double* X2, const double* X3, int n,
                          const double* c, hipStream_t s);
// Exponentials exp(f (A + g diag(d))) of up to MAX_EXPM matrices of one size
// n <= EXPM_MAX_N with a common number q of squarings (kern_expm.hip); buf:
// expm_batch_bytes(n, nb).  *result: job z's exponential at z * n * n entries.
constexpr int MAX_EXPM = 32;
constexpr int EXPM_MAX_N = 256;
struct ExpmJob {
  const double* A;
  const double* d;         // nullable
  double gr, gi, fr, fi;
  void* out;               // prepared operator of launch_prepare_jobs
  int a_exp;
  int minus_id;            // resident layouts: prepare the exponential - I
};
struct ExpmBatch {
  int n, nb, q;
  ExpmJob j[MAX_EXPM];
};
size_t expm_batch_bytes(int n, int nb);
hipError_t launch_expm_batch(const ExpmBatch& b, double* buf, double** result, hipStream_t s);
// Prepare the batch's exponentials (layout lay, KBT x MFT blocks) into the jobs' outs.
hipError_t launch_prepare_jobs(int lay, const ExpmBatch& b, const double* exps, int KBT, int MFT, hipStream_t s);
// out = Psi diag(exp(-i tau (k + 1/2))) Phi (Phi: K x m, Psi: m x K, real
// FP64 device masters with ld = rows; out: m x m complex FP64 interleaved).
hipError_t launch_hermite_collapse(const double* Phi, const double* Psi, int m, int K, double tau, double* out,
                                   hipStream_t s);
// out[0] = ||L - I||_F^2, out[1] = ||L||_F^2 of a complex FP64 n x n matrix
// (column-major, interleaved).
hipError_t launch_identity_norms(const double* L, int n, double* out, hipStream_t s);
// Exact nonlinear flow of the Section 4.5 vortex problem over time s on a
// complex state (interleaved, d modes, column-major): v <- exp((i s/2)(1 -
// W^-1 |v|^2)) v with W^-1 = prod_k winv[k * 4096 + i_k] (device array).
hipError_t launch_vortex_phase(void* v, int is_f64, int d, const int64_t* dims, const double* winv, double s,
                               hipStream_t st);
// FP16X2 chain start: slots[0] = float bits of max |x_k| over `count` floats,
// slots[1] = slots[2] = 0.  partial: >= norm_partials() words.
hipError_t launch_maxabs(const float* x, int64_t count, uint32_t* partial, uint32_t* slots, hipStream_t s);
size_t prepared_bytes(int prec, int KBT, int MFT);

// Two-pass deterministic FP64 reductions (fp32 or fp64 data):
//   RED_SQ     sum x_k^2 over `count` scalars of x
//   RED_DOT_RE sum Re(conj(x_k) y_k) over `count` complex entries
//   RED_ABS4   sum |x_k|^4 over `count` complex entries
// partial: device buffer of >= norm_partials() doubles.
enum RedKind { RED_SQ = 0, RED_DOT_RE = 1, RED_ABS4 = 2 };
int norm_partials();
hipError_t launch_reduce(int kind, const void* x, const void* y, int64_t count, int is_f64,
                         double* partial, double* result, hipStream_t s);

}  // namespace mm
