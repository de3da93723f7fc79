// The library's host side on a machine without a GPU: this program defines the
// HIP runtime calls that libmumode.so makes (an executable's symbols come
// before those of the libraries it loads), with device memory as host memory
// under a budget and kernels that do nothing, and runs one scenario, named by
// its first argument.  Launches are refused where the hardware refuses them:
// more LDS than a workgroup has, 2^32 threads along a grid dimension.  A
// failed expectation is printed and makes the exit status 1.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "mm_internal.h"
#include "mumode.h"

namespace {

struct {
  size_t budget = (size_t)1 << 40, used = 0;
  long fail_at = -1;                 // index of the hipMalloc that fails from here on (-1: none)
  long mallocs = 0, frees = 0, launches = 0;
  struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;
  hipError_t last = hipSuccess;      // what hipGetLastError reports once
  std::map<void*, size_t> live;
  std::map<const void*, int> max_lds;
  long next_graph = 1;
  std::set<long> execs;              // instantiated graphs
  std::vector<long> graph_launches;  // graphs launched, in order
} rt;

int g_failed = 0;
#define EXPECT(cond, ...)                          \
  do {                                             \
    if (!(cond)) {                                 \
      if (++g_failed <= 20) {                      \
        printf("%s:%d: %s: ", __FILE__, __LINE__, #cond); \
        printf(__VA_ARGS__);                       \
        printf("\n");                              \
      }                                            \
    }                                              \
  } while (0)

hipError_t check_launch(const void* fn, dim3 grid, dim3 block, size_t lds) {
  ++rt.launches;
  const size_t allowed = rt.max_lds.count(fn) ? (size_t)rt.max_lds[fn] : 65536;
  if (lds > allowed || block.x * block.y * block.z > 1024 || grid.x == 0 || grid.y == 0 || grid.z == 0)
    return rt.last = hipErrorInvalidValue;
  if ((uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32 || (uint64_t)grid.z * block.z >> 32)
    return rt.last = hipErrorInvalidConfiguration;
  return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t bytes) {
  const long i = rt.mallocs++;
  if ((rt.fail_at >= 0 && i >= rt.fail_at) || rt.used + bytes > rt.budget) return rt.last = hipErrorOutOfMemory;
  *p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
  rt.live[*p] = bytes;
  rt.used += bytes;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  ++rt.frees;
  if (!rt.live.count(p)) return hipErrorInvalidValue;
  rt.used -= rt.live[p];
  rt.live.erase(p);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { *p = std::calloc(1, bytes); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static char scratch[65536];
  *p = scratch;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() {
  const hipError_t e = rt.last;
  rt.last = hipSuccess;
  return e;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)0x10; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  *c = hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)0x20; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)0x20; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* fn, hipFuncAttribute, int bytes) {
  if (bytes > 160 * 1024) return hipErrorInvalidValue;
  rt.max_lds[fn] = bytes;
  return hipSuccess;
}
// the launch configuration between a launch statement and its stub
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  rt.config = {grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
  *grid = rt.config.grid;
  *block = rt.config.block;
  *lds = rt.config.lds;
  *s = rt.config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void**, size_t lds, hipStream_t) {
  return check_launch(fn, grid, block, lds);
}
hipError_t hipExtLaunchKernel(const void* fn, dim3 grid, dim3 block, void**, size_t lds, hipStream_t, hipEvent_t,
                              hipEvent_t, int) {
  return check_launch(fn, grid, block, lds);
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = (hipGraph_t)(uintptr_t)rt.next_graph++;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)g;
  rt.execs.insert((long)(uintptr_t)g);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  if (!rt.execs.count((long)(uintptr_t)e)) return hipErrorInvalidValue;
  rt.graph_launches.push_back((long)(uintptr_t)e);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { rt.execs.erase((long)(uintptr_t)e); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
}

namespace {

mm_ctx open_ctx() {
  mm_ctx c = nullptr;
  EXPECT(mm_create(&c, 0, nullptr) == MM_OK, "%s", mm_last_error(nullptr));
  return c;
}

// Operator with pseudo-random entries of size 1 / cols.
mm_op make_op(mm_ctx c, int64_t rows, int64_t cols, bool cplx, mm_prec prec) {
  std::vector<double> v((size_t)rows * cols * (cplx ? 2 : 1));
  uint32_t x = 12345;
  for (double& e : v) e = ((int32_t)(x = x * 1664525u + 1013904223u)) / 2147483648.0 / (double)cols;
  mm_matrix m = {rows, cols, rows, cplx ? MM_C128 : MM_R64, v.data(), 0};
  mm_op op = nullptr;
  EXPECT(mm_op_prepare(c, &m, prec, &op) == MM_OK, "%s", mm_last_error(c));
  return op;
}

// A tensor at an address that nothing here reads (the kernels do nothing).
mm_tensor tensor(std::vector<int64_t> dims, mm_dtype dt, uintptr_t at = (uintptr_t)1 << 40) {
  mm_tensor T = {};
  T.d = (int)dims.size();
  for (int k = 0; k < T.d; ++k) T.dims[k] = dims[k];
  T.dtype = dt;
  T.data = (void*)at;
  return T;
}

// A rebuild of the batched step that fails part way leaves no captured graph
// behind: its work items may be freed or overwritten by then.
void batch_failed_rebuild() {
  for (int at = 0; at < 3; ++at) {
    mm_ctx c = open_ctx();
    mm_tensor A = tensor({16, 16}, MM_R32), B1 = tensor({64, 512, 16}, MM_R32, (uintptr_t)2 << 40),
              B2 = tensor({64, 512, 16}, MM_R32, (uintptr_t)3 << 40), B3 = tensor({64, 64}, MM_R32, (uintptr_t)4 << 40);
    mm_op a = make_op(c, 16, 16, false, MM_PREC_FP32), b = make_op(c, 64, 64, false, MM_PREC_FP32),
          s = make_op(c, 64, 64, false, MM_PREC_SPLIT_BF16X3), as = make_op(c, 16, 16, false, MM_PREC_SPLIT_BF16X3);
    mm_op Ea[MM_MAXD] = {a, as}, Eb[MM_MAXD] = {b}, Es[MM_MAXD] = {s, s};
    mm_tensor* Ta[1] = {&A};
    const mm_op* Eas[1] = {Ea};
    mm_tensor* Tb[3] = {&B1, &B2, &B3};
    const mm_op* Ebs[3] = {Eb, Eb, Es};
    EXPECT(mumode_expstep_batched(c, 1, Ta, Eas, 1, nullptr) == MM_OK, "%s", mm_last_error(c));
    rt.fail_at = rt.mallocs + at;    // the at-th list that has to grow
    EXPECT(mumode_expstep_batched(c, 3, Tb, Ebs, 1, nullptr) == MM_ERR_NOMEM, "upload %d", at);
    rt.fail_at = -1;
    const size_t before = rt.graph_launches.size();
    const long built = rt.next_graph;
    EXPECT(mumode_expstep_batched(c, 1, Ta, Eas, 1, nullptr) == MM_OK, "%s", mm_last_error(c));
    EXPECT(rt.graph_launches.size() == before + 1 && rt.graph_launches.back() >= built,
           "graph %ld captured before the failed rebuild (upload %d)", rt.graph_launches.back(), at);
    mm_destroy(c);
  }
}

// Launch shapes of the resident-tile products over all rows, columns and forms
// that they take, for few to very many fibres and every forced tile class.
template <typename Check>
void for_all_plans(Check&& check) {
  const int64_t fibres[] = {1, 100, 8191, 16384, 40000, 65537, 359000000, ((int64_t)1 << 30) + 1};
  for (int prec : {(int)mm::KP_F64, (int)mm::KP_F32})
    for (int form : {(int)mm::RF_C3, (int)mm::RF_RC, (int)mm::RF_RR, (int)mm::RF_C4}) {
      if (form == mm::RF_C4 && prec == mm::KP_F64) continue;
      const int lim = form == mm::RF_C3 || form == mm::RF_C4 ? 256 : 512;
      for (int m = 1; m <= lim; ++m)
        for (int n = 1; n <= lim; n += n < 64 ? 1 : 3)
          for (int64_t F : fibres)
            for (int cls = -1; cls < 4; ++cls) {
              mm::ResArgs a = {};
              a.n = n;
              a.m = m;
              a.P = 1;
              a.F = F;
              a.nsteps = 1;
              mm::ResPlan p = {};
              mm::res_plan(prec, form, false, cls, &a, &p);
              check(a, p);
              if (m == n) {
                a.nsteps = 5;
                mm::res_plan(prec, form, false, cls, &a, &p);
                check(a, p);
              }
            }
    }
}

void resident_plans_fit() {
  for_all_plans([](const mm::ResArgs& a, const mm::ResPlan& p) {
    const char* what = "prec %d form %d m %d n %d F %lld: lds %zu threads %d MF %d NF %d WM %d WN %d";
#define WHAT what, p.prec, p.form, a.m, a.n, (long long)a.F, p.lds, p.threads, p.mf, p.nf, a.WM, a.WN
    const size_t es = (p.prec == mm::KP_F64 ? 8 : 4) * (p.form == mm::RF_RR ? 1 : 2);
    const int nt = 16 * p.nf * a.WN;
    EXPECT(p.lds <= 160 * 1024, WHAT);
    EXPECT(p.threads == 64 * a.WM * a.WN && p.threads <= (p.run ? 256 : (p.mf == 1 ? 1024 : 512)), WHAT);
    if (p.run) EXPECT(p.lds == 2 * p.run * 17 * es && a.n <= p.run && a.WM * 16 >= a.m, WHAT);
    else EXPECT(p.lds >= (size_t)(a.n + 4) * (nt + 1) * es && a.WM * p.mf * 16 * a.NRB >= a.m, WHAT);
    EXPECT(p.mf >= 1 && p.mf <= 4 && (p.nf == 1 || (p.nf == 2 && p.form == mm::RF_RR)), WHAT);
    EXPECT((int64_t)p.grid_x * p.grid_y * nt >= a.F && (int64_t)(p.grid_x - 1) * p.grid_y * nt < a.F, WHAT);
    EXPECT((int64_t)p.grid_x * p.threads < (int64_t)1 << 32 && p.grid_y < 65536, WHAT);
  });
}

// Flat operators through the public calls, at the sizes of real transforms.
void flat_operators() {
  struct { int64_t m, n; bool cplx; mm_dtype dt; mm_prec prec; } cases[] = {
      {16, 200, false, MM_C128, MM_PREC_FP64}, {16, 256, true, MM_C128, MM_PREC_FP64},
      {16, 256, false, MM_R64, MM_PREC_FP64},  {32, 512, false, MM_C128, MM_PREC_FP64},
      {16, 512, false, MM_C64, MM_PREC_FP32},  {1, 145, true, MM_C128, MM_PREC_FP64}};
  mm_ctx c = open_ctx();
  for (const auto& t : cases) {
    mm_op L = make_op(c, t.m, t.n, t.cplx, t.prec);
    for (int mu = 1; mu <= 2; ++mu) {
      const std::vector<int64_t> in = mu == 1 ? std::vector<int64_t>{t.n, 256, 300} : std::vector<int64_t>{300, t.n, 256};
      std::vector<int64_t> out = in;
      out[mu - 1] = t.m;
      mm_tensor T = tensor(in, t.dt), O = tensor(out, t.dt, (uintptr_t)2 << 40);
      EXPECT(mumode_apply(c, &O, &T, L, mu, nullptr) == MM_OK, "%lld x %lld mode %d: %s", (long long)t.m,
             (long long)t.n, mu, mm_last_error(c));
      mm_op Phi[MM_MAXD] = {mu == 1 ? L : nullptr, mu == 2 ? L : nullptr};
      EXPECT(mumode_transform(c, &O, &T, Phi, nullptr) == MM_OK, "%s", mm_last_error(c));
      EXPECT(mm_autotune(c, &T, Phi, 1, nullptr) == MM_OK, "%s", mm_last_error(c));
    }
  }
  mm_destroy(c);
}

// States of 10^9 fibres and more: more threads than one grid dimension takes.
void very_many_fibres() {
  struct { std::vector<int64_t> dims; int mu; mm_dtype dt; mm_prec prec; bool cplx; } cases[] = {
      {{33, 19000, 19000}, 1, MM_C64, MM_PREC_FP32, true},   {{33, 19000, 19000}, 1, MM_C128, MM_PREC_FP64, true},
      {{32768, 1, 32769}, 2, MM_C64, MM_PREC_FP32, false},   {{2, 65536, 65536}, 1, MM_R32, MM_PREC_FP32, false},
      {{40, 16384, 32768}, 1, MM_R32, MM_PREC_FP32, false}};
  mm_ctx c = open_ctx();
  for (const auto& t : cases) {
    mm_tensor T = tensor(t.dims, t.dt);
    mm_op E[MM_MAXD] = {};
    E[t.mu - 1] = make_op(c, t.dims[t.mu - 1], t.dims[t.mu - 1], t.cplx, t.prec);
    for (int nsteps = 1; nsteps <= 2; ++nsteps)
      EXPECT(mumode_expstep(c, &T, E, nsteps, nullptr) == MM_OK, "%lld entries: %s", (long long)t.dims[t.mu - 1],
             mm_last_error(c));
  }
  mm_destroy(c);
}

struct Oscillator {
  mm_op F[MM_MAXD], B[MM_MAXD];
  std::vector<double> x;
  const double* nodes[MM_MAXD];
  mm_tensor T;
};
Oscillator oscillator(mm_ctx c, int64_t n, mm_prec prec) {
  Oscillator o = {};
  for (int k = 0; k < 3; ++k) {
    o.F[k] = make_op(c, n, n, false, prec);
    o.B[k] = make_op(c, n, n, false, prec);
  }
  o.x.resize(n);
  for (int64_t i = 0; i < n; ++i) o.x[i] = 0.1 * (double)i;
  o.T = tensor({n, n, n}, prec == MM_PREC_FP64 ? MM_C128 : MM_C64);
  return o;
}
mm_status step(mm_ctx c, Oscillator& o, int nsteps) {
  for (int k = 0; k < 3; ++k) o.nodes[k] = o.x.data();
  return ho_strang_step(c, &o.T, o.F, o.B, o.nodes, 0.1, 0.02, 0.1, nsteps, nullptr);
}

// The oscillator step where a whole block of step operators does not fit: the
// call's own steps do, for all modes together, and a buffer that holds them
// stays from call to call.
void oscillator_little_memory() {
  mm_ctx c = open_ctx();
  Oscillator o = oscillator(c, 128, MM_PREC_FP64);
  const size_t before = rt.used;
  EXPECT(step(c, o, 2) == MM_OK, "%s", mm_last_error(c));
  const size_t whole = rt.used - before;   // formation, nodes, a block of steps
  mm_destroy(c);
  c = open_ctx();
  o = oscillator(c, 128, MM_PREC_FP64);
  rt.budget = rt.used + whole / 3;
  EXPECT(step(c, o, 2) == MM_OK, "%s", mm_last_error(c));
  const long mallocs = rt.mallocs, frees = rt.frees;
  for (int i = 0; i < 3; ++i) EXPECT(step(c, o, 2) == MM_OK, "%s", mm_last_error(c));
  EXPECT(rt.mallocs == mallocs && rt.frees == frees, "%ld allocations, %ld frees in repeated calls",
         rt.mallocs - mallocs, rt.frees - frees);
  EXPECT(step(c, o, 3) == MM_OK, "%s", mm_last_error(c));
  mm_destroy(c);
}

// A formation that runs out of memory is not taken for the one before.
void oscillator_failed_formation() {
  mm_ctx c = open_ctx();
  Oscillator a = oscillator(c, 32, MM_PREC_FP64), b = oscillator(c, 96, MM_PREC_FP64);
  long n = rt.launches;
  EXPECT(step(c, a, 1) == MM_OK, "%s", mm_last_error(c));
  const long first = rt.launches - n;
  rt.fail_at = rt.mallocs;
  EXPECT(step(c, b, 1) == MM_ERR_NOMEM, "no failure");
  rt.fail_at = -1;
  n = rt.launches;
  EXPECT(step(c, a, 1) == MM_OK, "%s", mm_last_error(c));
  EXPECT(rt.launches - n >= first - 2, "%ld launches, %ld with all three modes formed", rt.launches - n, first);
  mm_destroy(c);
}

// The midpoint step where one step's operators and exponentials fit but not a
// block of them.
void midpoint_little_memory() {
  const int64_t n = 128;
  std::vector<double> g(2 * n * n), d(n, 1.0), coef(2 * 32 * 3, 0.5);
  for (size_t i = 0; i < g.size(); ++i) g[i] = 1e-3 * (double)(i % 7);
  const mm_matrix m = {n, n, n, MM_C128, g.data(), 0};
  const mm_matrix B[3] = {m, m, m};
  const double* dd[3] = {d.data(), d.data(), d.data()};
  for (mm_prec prec : {MM_PREC_FP64, MM_PREC_FP32, MM_PREC_SPLIT_BF16X3}) {
    rt.budget = (size_t)1 << 40;
    mm_ctx c = open_ctx();
    mm_tensor T = tensor({n, n, n}, prec == MM_PREC_FP64 ? MM_C128 : MM_C64);
    // per mode: the generator (16 n^2), one prepared operator and one
    // exponential with its five helpers (96 n^2)
    rt.budget = rt.used + (size_t)3 * 16 * n * n + (size_t)3 * 32 * n * n + (size_t)96 * n * n + (1 << 20);
    EXPECT(mumode_magnus_step(c, &T, B, dd, coef.data(), 0.1, 32, prec, nullptr) == MM_OK, "precision %d: %s", (int)prec,
           mm_last_error(c));
    const long mallocs = rt.mallocs, frees = rt.frees;
    EXPECT(mumode_magnus_step(c, &T, B, dd, coef.data(), 0.1, 32, prec, nullptr) == MM_OK, "%s", mm_last_error(c));
    EXPECT(rt.mallocs == mallocs && rt.frees == frees, "precision %d: %ld allocations, %ld frees in a repeated call",
           (int)prec, rt.mallocs - mallocs, rt.frees - frees);
    mm_destroy(c);
  }
}

// Steps of a mode per launch are bounded, also where nothing grows.
void steps_per_launch() {
  mm_ctx c = open_ctx();
  for (int64_t n : {48, 200}) {
    mm_op L = make_op(c, n, n, true, MM_PREC_FP64);   // norm below one
    mm_tensor T = tensor({n, n}, MM_C128);
    mm_op E[MM_MAXD] = {L, L};
    const long before = rt.launches;
    EXPECT(mumode_expstep(c, &T, E, 1000000, nullptr) == MM_OK, "%s", mm_last_error(c));
    EXPECT(rt.launches - before >= 2 * 1000000 / 256, "%ld launches for two modes of 10^6 steps", rt.launches - before);
  }
  mm_destroy(c);
}

// Tune files: of the first version, entries of FP64 / FP32 products that now run
// on the resident tiles are left out; what is written is read back whole.
void tune_file_versions() {
  const char* path = "tune_versions.txt";
  const char* entries = "0 0 1 128 128 16384 2 16.6\n1 1 0 512 512 4096 0 1.0\n0 0 1 600 600 900 1 9.0\n"
                        "3 1 0 256 256 16384 6 1.0\n";
  for (int version = 1; version <= 2; ++version) {
    FILE* f = std::fopen(path, "w");
    std::fprintf(f, "mumode-tune %d\n%s", version, entries);
    std::fclose(f);
    mm_ctx c = open_ctx();
    EXPECT(mm_tune_load(c, path) == MM_OK, "%s", mm_last_error(c));
    int n = 0, again = 0;
    mm_tune_count(c, &n);
    EXPECT(n == (version == 1 ? 2 : 4), "version %d: %d entries", version, n);
    EXPECT(mm_tune_save(c, path) == MM_OK && mm_tune_clear(c) == MM_OK && mm_tune_load(c, path) == MM_OK, "%s",
           mm_last_error(c));
    mm_tune_count(c, &again);
    EXPECT(again == n, "%d of %d entries read back", again, n);
    mm_destroy(c);
    std::remove(path);
  }
}

}  // namespace

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> scenarios = {
      {"batch_failed_rebuild", batch_failed_rebuild},
      {"resident_plans_fit", resident_plans_fit},
      {"flat_operators", flat_operators},
      {"very_many_fibres", very_many_fibres},
      {"oscillator_little_memory", oscillator_little_memory},
      {"oscillator_failed_formation", oscillator_failed_formation},
      {"midpoint_little_memory", midpoint_little_memory},
      {"tune_file_versions", tune_file_versions},
      {"steps_per_launch", steps_per_launch},
  };
  const auto it = scenarios.find(argc > 1 ? argv[1] : "");
  if (it == scenarios.end()) return 2;
  it->second();
  if (g_failed) printf("%d expectations failed\n", g_failed);
  return g_failed ? 1 : 0;
}
