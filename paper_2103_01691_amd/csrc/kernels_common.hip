// Operator preparation, FP64 reductions and the host-side planning and
// dispatch of the mu-mode product kernels (tables in kern_<prec>.hip).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>

#include "mode_tile.h"

namespace mm {
namespace {

// -------------------------------------------------------- preparation -----

// The stored pieces of one operator value x at out[base] (piece p at
// base + p * 64 * KPL).
template <int PR>
__device__ __forceinline__ void put_pieces(typename Tr<PR>::pc* __restrict__ out, int64_t base, double x,
                                           int a_exp) {
  constexpr int KPL = Tr<PR>::KPL, NPC = Tr<PR>::NPS;
  if constexpr (PR == KP_F64) {
    out[base] = x;
  } else if constexpr (PR == KP_F32) {
    out[base] = (float)x;
  } else if constexpr (PR == KP_FP16X2) {
    // stored pieces (h 2^11, l) of x 2^-a_exp = h + 2^-11 l; the residual
    // is exact in FP64.  h 2^11 multiplies both state pieces, l the high
    // one.
    const double xs = ldexp(x, -a_exp);
    const _Float16 h = (_Float16)(float)xs;
    const _Float16 l = (_Float16)(float)((xs - (double)h) * 2048.0);
    out[base] = (_Float16)((float)h * 2048.0f);
    out[base + (int64_t)64 * KPL] = l;
  } else {
    double r = x;
#pragma unroll
    for (int p = 0; p < NPC; ++p) {
      __bf16 h = (__bf16)(float)r;
      out[base + (int64_t)p * 64 * KPL] = h;
      r = r - (double)(float)h;
    }
  }
}

// One fragment slot s = (kb, mf, lane) of the prepared operator.
template <int PR>
__device__ __forceinline__ void prepare_slot(int64_t s, const double* __restrict__ master, int64_t rows,
                                             int64_t cols, int64_t ld, int cplx, const PhaseScale& ph,
                                             void* __restrict__ outv, int KBT, int MFT, int a_exp) {
  typedef Tr<PR> T;
  typedef typename T::pc pc;
  constexpr int MB = T::MB, KB = T::KB, KPL = T::KPL, NPC = T::NPS;
  const int64_t slots = (int64_t)KBT * MFT * 64;   // (kb, mf, lane)
  if (s >= slots) return;
  const int lane = (int)(s % 64);
  const int64_t t = s / 64;
  const int mf = (int)(t % MFT);
  const int kb = (int)(t / MFT);
  const int64_t Mr = cplx ? 2 * rows : rows;
  const int64_t Kr = cplx ? 2 * cols : cols;
  pc* out = (pc*)outv;
  // physical fragment row -> logical row of the real block operator; the
  // FP64 16x16 accumulator layout puts row lane/16 + 4r in register r, so
  // its complex rows are permuted to keep (re, im) pairs in one lane
  const int rho = lane % MB;
  const int row = (PR == KP_F64 && cplx) ? 2 * (mf * 8 + (rho % 4) + 4 * (rho / 8)) + ((rho / 4) % 2)
                                         : mf * MB + rho;
  for (int e = 0; e < KPL; ++e) {
    const int kap = kb * KB + KPL * (lane / MB) + e;
    double x = 0.0;
    if (row < Mr && kap < Kr) {
      if (cplx) {
        const int64_t i = row / 2, j = kap / 2;
        const int cr = row & 1, ck = kap & 1;
        double re = master[2 * (i + j * ld)], im = master[2 * (i + j * ld) + 1];
        // L'[i,j] = exp(-i rc rx2[i]) L[i,j] exp(-i cc cx2[j])
        double th = 0.0;
        if (ph.rx2) th += ph.rc * ph.rx2[i];
        if (ph.cx2) th += ph.cc * ph.cx2[j];
        if (th != 0.0) {
          double sn, cs;
          sincos(th, &sn, &cs);
          const double r2 = re * cs + im * sn;
          im = im * cs - re * sn;
          re = r2;
        }
        x = (cr == ck) ? re : (cr == 0 ? -im : im);
      } else {
        x = master[row + kap * ld];
      }
    }
    const int64_t base = (((int64_t)kb * MFT + mf) * NPC) * 64 * KPL + lane * KPL + e;
    put_pieces<PR>(out, base, x, a_exp);
  }
}

// One lane slot s = (unit, fragment, lane) of the resident layout: 16 bytes of
// operator entries, UK K-blocks of 4 columns ((re, im) pairs when complex).
// Lane l holds row l % 16 of its 16-row fragment and column l / 16 of each
// K-block; the FP64 accumulator keeps physical row l / 16 + 4 r in register r,
// so its rows are permuted to give every lane four consecutive rows, as the
// FP32 accumulator does.
template <typename S>
__device__ __forceinline__ void prepare_res_slot(int64_t s, const double* __restrict__ master, int64_t rows,
                                                 int64_t cols, int64_t ld, int cplx, const PhaseScale& ph,
                                                 void* __restrict__ outv, int KU, int MFT) {
  if (s >= (int64_t)KU * MFT * 64) return;
  const int lane = (int)(s % 64);
  const int64_t t = s / 64;
  const int mf = (int)(t % MFT);
  const int64_t ku = t / MFT;
  const int rho = lane % 16;
  const int64_t i = (int64_t)mf * 16 + (sizeof(S) == 8 ? 4 * (rho % 4) + rho / 4 : rho);
  const int comps = cplx ? 2 : 1;
  const int UK = 16 / (int)(sizeof(S) * comps);
  S* out = (S*)outv + s * (16 / sizeof(S));
  for (int u = 0; u < UK; ++u) {
    const int64_t j = (ku * UK + u) * 4 + lane / 16;
    double re = 0.0, im = 0.0;
    if (i < rows && j < cols) {
      if (cplx) {
        re = master[2 * (i + j * ld)];
        im = master[2 * (i + j * ld) + 1];
        double th = 0.0;
        if (ph.rx2) th += ph.rc * ph.rx2[i];
        if (ph.cx2) th += ph.cc * ph.cx2[j];
        if (th != 0.0) {
          double sn, cs;
          sincos(th, &sn, &cs);
          const double r2 = re * cs + im * sn;
          im = im * cs - re * sn;
          re = r2;
        }
      } else {
        re = master[i + j * ld];
      }
    }
    if (ph.minus_id && i == j && i < rows && j < cols) re -= 1.0;
    out[u * comps] = (S)re;
    if (cplx) out[u * comps + 1] = (S)im;
  }
}

// Three-product (Gauss) preparation: slot ((jb * 3 + t) * MFT + mf, lane)
// holds 8 columns of complex row mf * 32 + lane % 32 of Re L (t = 0), Im L
// (t = 1) or Re L + Im L (t = 2), formed in FP64.
template <int PR>
__global__ void prepare_gauss_kernel(const double* __restrict__ master, int64_t rows, int64_t cols, int64_t ld,
                                     void* __restrict__ outv, int JBT, int MFT, int a_exp) {
  typedef typename Tr<PR>::pc pc;
  constexpr int NPC = Tr<PR>::NPS;
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= (int64_t)JBT * 3 * MFT * 64) return;
  const int lane = (int)(s % 64);
  const int64_t t = s / 64;
  const int mf = (int)(t % MFT);
  const int64_t kbg = t / MFT;
  const int ty = (int)(kbg % 3);
  const int64_t jb = kbg / 3;
  const int64_t i = (int64_t)mf * 32 + lane % 32;
  pc* out = (pc*)outv;
  for (int e = 0; e < 8; ++e) {
    const int64_t j = jb * 16 + 8 * (lane / 32) + e;
    double x = 0.0;
    if (i < rows && j < cols) {
      const double re = master[2 * (i + j * ld)], im = master[2 * (i + j * ld) + 1];
      x = ty == 0 ? re : (ty == 1 ? im : re + im);
    }
    put_pieces<PR>(out, ((kbg * MFT + mf) * NPC) * 64 * 8 + lane * 8 + e, x, a_exp);
  }
}

// One slot of any operator layout (KPrec or KLayout code LY).
template <int LY>
__device__ __forceinline__ void prepare_any(int64_t s, const double* __restrict__ master, int64_t rows, int64_t cols,
                                            int64_t ld, int cplx, const PhaseScale& ph, void* __restrict__ outv,
                                            int KBT, int MFT, int a_exp) {
  if constexpr (LY == KY_RES64) prepare_res_slot<double>(s, master, rows, cols, ld, cplx, ph, outv, KBT, MFT);
  else if constexpr (LY == KY_RES32) prepare_res_slot<float>(s, master, rows, cols, ld, cplx, ph, outv, KBT, MFT);
  else prepare_slot<LY>(s, master, rows, cols, ld, cplx, ph, outv, KBT, MFT, a_exp);
}

template <int PR>
__global__ void prepare_kernel(const double* __restrict__ master, int64_t rows, int64_t cols,
                               int64_t ld, int cplx, PhaseScale ph, void* __restrict__ outv, int KBT,
                               int MFT, int a_exp) {
  prepare_any<PR>((int64_t)blockIdx.x * blockDim.x + threadIdx.x, master, rows, cols, ld, cplx, ph, outv, KBT,
                  MFT, a_exp);
}

// The operators of a batch of matrix exponentials (blockIdx.y: job).
template <int LY>
__global__ void prepare_jobs_kernel(ExpmBatch b, const double* __restrict__ exps, int KBT, int MFT) {
  const ExpmJob& j = b.j[blockIdx.y];
  PhaseScale ph;
  ph.minus_id = j.minus_id;
  prepare_any<LY>((int64_t)blockIdx.x * blockDim.x + threadIdx.x, exps + (int64_t)blockIdx.y * b.n * b.n * 2, b.n, b.n,
                  b.n, 1, ph, j.out, KBT, MFT, j.a_exp);
}

// Per-step operators of the time-dependent harmonic-oscillator splitting
// (blockIdx.y = step * modes + entry).
template <int PR>
__global__ void prepare_steps_kernel(StepPrep p) {
  const int e = (int)(blockIdx.y % p.modes);
  const int st = (int)(blockIdx.y / p.modes);
  const StepPrepMode& m = p.m[e];
  const double t = p.t0 + st * p.tau;
  const double th = t + 0.5 * p.tau;
  PhaseScale ph;
  ph.rx2 = m.x2;
  ph.cx2 = m.x2;
  ph.minus_id = m.minus_id;
  ph.cc = 0.5 * p.eps * (cos(t) - cos(th));           // first half step: columns
  ph.rc = 0.5 * p.eps * (cos(th) - cos(t + p.tau));   // second half step: rows
  prepare_any<PR>((int64_t)blockIdx.x * blockDim.x + threadIdx.x, m.master, m.n, m.n, m.n, 1, ph,
                  m.out + (size_t)st * m.stride, m.KBT, m.MFT, m.a_exp);
}

// ------------------------------------------------------------- norm2 ------

constexpr int NORM_BLOCKS = 1024;
constexpr int NORM_THREADS = 256;

template <typename S, int KIND>
__global__ __launch_bounds__(NORM_THREADS) void reduce_partial_kernel(const S* __restrict__ x,
                                                                      const S* __restrict__ y,
                                                                      int64_t count,
                                                                      double* __restrict__ partial) {
  __shared__ double red[NORM_THREADS];
  double acc = 0.0;
  const int64_t stride = (int64_t)gridDim.x * NORM_THREADS;
  int64_t start = (int64_t)blockIdx.x * NORM_THREADS + threadIdx.x;
  if constexpr (KIND == RED_SQ) {
    // 16-byte loads (the state is 16-byte aligned), then the scalar tail
    constexpr int VN = 16 / sizeof(S);
    typedef S vecS __attribute__((ext_vector_type(VN)));
    const int64_t countv = count / VN;
    const vecS* __restrict__ xv = (const vecS*)x;
    for (int64_t i = start; i < countv; i += stride) {
      const vecS v = xv[i];
#pragma unroll
      for (int e = 0; e < VN; ++e) acc += (double)v[e] * (double)v[e];
    }
    start += VN * countv;
  }
  for (int64_t i = start; i < count; i += stride) {
    if constexpr (KIND == RED_SQ) {
      const double v = (double)x[i];
      acc += v * v;
    } else if constexpr (KIND == RED_DOT_RE) {
      acc += (double)x[2 * i] * (double)y[2 * i] + (double)x[2 * i + 1] * (double)y[2 * i + 1];
    } else {
      const double a2 = (double)x[2 * i] * (double)x[2 * i] + (double)x[2 * i + 1] * (double)x[2 * i + 1];
      acc += a2 * a2;
    }
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = NORM_THREADS / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(NORM_THREADS) void norm_final_kernel(const double* __restrict__ partial,
                                                                  int nparts,
                                                                  double* __restrict__ result) {
  __shared__ double red[NORM_THREADS];
  double acc = 0.0;
  for (int i = threadIdx.x; i < nparts; i += NORM_THREADS) acc += partial[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = NORM_THREADS / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) result[0] = red[0];
}

// ------------------------------------------------------------ maxabs ------

// Bound of the state for the FP16X2 products: max |x_k| as float bits
// (non-negative floats order like their bit patterns; NaN bits order above
// every finite value).
__global__ __launch_bounds__(NORM_THREADS) void maxabs_partial_kernel(const float* __restrict__ x,
                                                                      int64_t count,
                                                                      uint32_t* __restrict__ partial) {
  __shared__ uint32_t red[NORM_THREADS];
  uint32_t m = 0;
  // 16-byte loads (the state is 16-byte aligned), four in flight per thread,
  // then the scalar tail
  const int64_t count4 = count / 4;
  const f32x4* __restrict__ x4 = (const f32x4*)x;
  const int64_t stride = (int64_t)gridDim.x * NORM_THREADS;
  int64_t i = (int64_t)blockIdx.x * NORM_THREADS + threadIdx.x;
  for (; i + 3 * stride < count4; i += 4 * stride) {
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = x4[i + u * stride];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) m = max(m, __float_as_uint(fabsf(v[u][e])));
  }
  for (; i < count4; i += stride) {
    const f32x4 v = x4[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) m = max(m, __float_as_uint(fabsf(v[e])));
  }
  for (int64_t t = 4 * count4 + (int64_t)blockIdx.x * NORM_THREADS + threadIdx.x; t < count; t += stride)
    m = max(m, __float_as_uint(fabsf(x[t])));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = NORM_THREADS / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(NORM_THREADS) void maxabs_final_kernel(const uint32_t* __restrict__ partial,
                                                                    int nparts, uint32_t* __restrict__ slots) {
  __shared__ uint32_t red[NORM_THREADS];
  uint32_t m = 0;
  for (int i = threadIdx.x; i < nparts; i += NORM_THREADS) m = max(m, partial[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int w = NORM_THREADS / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = max(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  // slot 0 gets the bound (word 0; its other words and slots 1, 2 cleared)
  for (int i = threadIdx.x; i < 3 * SMAX_WORDS; i += NORM_THREADS) slots[i * SMAX_STRIDE] = i == 0 ? red[0] : 0u;
}

// ||L - I||_F^2 and ||L||_F^2 (one workgroup)
__global__ __launch_bounds__(NORM_THREADS) void identity_norms_kernel(const double* __restrict__ L, int n,
                                                                      double* __restrict__ out) {
  __shared__ double red[2][NORM_THREADS];
  double off = 0.0, all = 0.0;
  for (int e = threadIdx.x; e < n * n; e += NORM_THREADS) {
    const double re = L[2 * e], im = L[2 * e + 1];
    const double dr = e % n == e / n ? re - 1.0 : re;
    off += dr * dr + im * im;
    all += re * re + im * im;
  }
  red[0][threadIdx.x] = off;
  red[1][threadIdx.x] = all;
  __syncthreads();
  for (int w = NORM_THREADS / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 2; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 2) out[threadIdx.x] = red[threadIdx.x][0];
}

// ------------------------------------------------------ device expm ------
// Helpers of the device matrix exponential (complex FP64, column-major,
// interleaved (re, im), n x n, leading dimension n).

// X = f (A + g diag(d)) with complex f, g; d real (nullable)
__global__ void expm_generator_kernel(const double* __restrict__ A, int n, const double* __restrict__ d,
                                      double gr, double gi, double fr, double fi, double* __restrict__ X) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int i = (int)(e % n), j = (int)(e / n);
  double re = A[2 * e], im = A[2 * e + 1];
  if (d && i == j) {
    re += gr * d[i];
    im += gi * d[i];
  }
  X[2 * e] = fr * re - fi * im;
  X[2 * e + 1] = fr * im + fi * re;
}

// P = W + c0 I + c1 X + c2 X2 + c3 X3 (W nullable): one Paterson-Stockmeyer
// block of the Taylor polynomial
__global__ void expm_ps_kernel(double* __restrict__ P, const double* __restrict__ W, const double* __restrict__ X,
                               const double* __restrict__ X2, const double* __restrict__ X3, int n, double c0,
                               double c1, double c2, double c3) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int i = (int)(e % n), j = (int)(e / n);
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int64_t k = 2 * e + c;
    double v = (W ? W[k] : 0.0) + c1 * X[k] + c2 * X2[k] + c3 * X3[k];
    if (c == 0 && i == j) v += c0;
    P[k] = v;
  }
}

// per-column sum of |A_ij| (1-norm = max over columns)
__global__ void expm_colsum_kernel(const double* __restrict__ A, int n, const double* __restrict__ d, double gr,
                                   double gi, double* __restrict__ out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  double s = 0.0;
  for (int i = 0; i < n; ++i) {
    const int64_t e = (int64_t)j * n + i;
    double re = A[2 * e], im = A[2 * e + 1];
    if (d && i == j) {
      re += gr * d[i];
      im += gi * d[i];
    }
    s += sqrt(re * re + im * im);
  }
  out[j] = s;
}

// Collapsed exact harmonic-oscillator propagator in nodal Hermite space:
// out[i, l] = sum_k Psi[i, k] exp(-i tau (k + 1/2)) Phi[k, l] (complex FP64,
// column-major interleaved, m x m); Phi is K x m, Psi m x K, real, ld = rows.
// One thread per entry; the phase of coefficient k is that mode's exact
// flow under the oscillator (phi_k has energy k + 1/2).
__global__ void hermite_collapse_kernel(const double* __restrict__ Phi, const double* __restrict__ Psi, int m,
                                        int K, double tau, double* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)m * m) return;
  const int i = (int)(e % m);
  const int l = (int)(e / m);
  double re = 0.0, im = 0.0;
  for (int k = 0; k < K; ++k) {
    double sn, cs;
    sincos(tau * (k + 0.5), &sn, &cs);
    const double v = Psi[i + (int64_t)k * m] * Phi[k + (int64_t)l * K];
    re += v * cs;
    im -= v * sn;
  }
  out[2 * e] = re;
  out[2 * e + 1] = im;
}

// Exact flow over time s of the nonlinear part of the Section 4.5 vortex
// problem in the symmetrised variable v = W^(1/2) u:
// v <- exp((i s / 2)(1 - W^-1 |v|^2)) v, W^-1 the product over the modes of
// the inverse dual-cell widths winv[k * 4096 + i_k].  |v| is constant along
// the flow.  One thread per entry (grid-stride); FP32 states take the angle
// and its sine / cosine in FP32 (the library's own reduction and series),
// FP64 states in FP64.
struct Dims6 {
  int64_t n[6];
};
template <typename T>
__global__ __launch_bounds__(256) void vortex_phase_kernel(T* __restrict__ v, int64_t count, int d, Dims6 dims,
                                                           const double* __restrict__ winv, double s) {
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < count; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t r = e;
    double wi = 1.0;
    for (int k = 0; k < d; ++k) {
      const int64_t i = r % dims.n[k];
      r /= dims.n[k];
      wi *= winv[(int64_t)k * 4096 + i];
    }
    T re = v[2 * e], im = v[2 * e + 1];
    const T th = (T)(0.5 * s) * ((T)1 - (T)wi * (re * re + im * im));
    T sn, cs;
    if constexpr (sizeof(T) == 8) sincos(th, &sn, &cs);
    else sincos_f32<false>(th, &sn, &cs);
    v[2 * e] = re * cs - im * sn;
    v[2 * e + 1] = im * cs + re * sn;
  }
}

// ---------------------------------------------------------- host side -----

KernFn pick_kernel_any(int prec, int cplx, int ld, int pro, int epi, int cls, int full = 0, int ida = 0) {
  switch (prec) {
    case KP_F64: return pick_kernel_f64(cplx, ld, pro, epi, cls, full, ida);
    case KP_F32: return pick_kernel_f32(cplx, ld, pro, epi, cls, full, ida);
    case KP_BF16X3: return pick_kernel_bf16x3(cplx, ld, pro, epi, cls, full, ida);
    case KP_FP16X2: return pick_kernel_fp16x2(cplx, ld, pro, epi, cls, full, ida);
    default: return pick_kernel_bf16(cplx, ld, pro, epi, cls, full, ida);
  }
}

bool batch_kind_any(int prec, int cplx, int ld, int cls) {
  switch (prec) {
    case KP_F64: return batch_kind_f64(cplx, ld, cls);
    case KP_F32: return batch_kind_f32(cplx, ld, cls);
    case KP_BF16X3: return batch_kind_bf16x3(cplx, ld, cls);
    case KP_FP16X2: return batch_kind_fp16x2(cplx, ld, cls);
    default: return batch_kind_bf16(cplx, ld, cls);
  }
}

}  // namespace

bool tile_shape(int prec, int cls, TileShape* out) {
  switch (prec) {
    case KP_F64: return tile_shape_f64(cls, out);
    case KP_F32: return tile_shape_f32(cls, out);
    case KP_BF16X3: return tile_shape_bf16x3(cls, out);
    case KP_FP16X2: return tile_shape_fp16x2(cls, out);
    default: return tile_shape_bf16(cls, out);
  }
}

FragGeom frag_geom(int prec) {
  switch (prec) {
    case KP_F64: return {16, 16, 4, 1, 1, 8, 32};
    case KP_F32: return {32, 32, 2, 1, 1, 32, 16};
    case KP_BF16X3: return {32, 32, 16, 8, 3, 4, 16};
    case KP_FP16X2: return {32, 32, 16, 8, 2, 4, 16};
    default: return {32, 32, 16, 8, 1, 4, 16};
  }
}

void op_blocks(int prec, int64_t Mr, int64_t Kr, int* KBT, int* MFT) {
  FragGeom g = frag_geom(prec);
  const int64_t kb = (Kr + g.KB - 1) / g.KB;
  const int64_t mf = (Mr + g.MB - 1) / g.MB;
  *KBT = (int)((kb + g.KPAD - 1) / g.KPAD * g.KPAD);
  *MFT = (int)((mf + g.MPAD - 1) / g.MPAD * g.MPAD);
}

void res_blocks(int lay, int64_t rows, int64_t cols, int cplx, int* KU, int* MFT) {
  const int uk = 16 / ((lay == KY_RES64 ? 8 : 4) * (cplx ? 2 : 1));
  // padding that no wave of at most 4 fragments and no ring of 4 units (from
  // any unit of the last chunk) reads past
  *KU = (int)(((cols + 3) / 4 + uk - 1) / uk) + 4;
  *MFT = (int)((rows + 15) / 16) + 3;
}

size_t prepared_bytes(int prec, int KBT, int MFT) {
  if (prec == KY_RES64 || prec == KY_RES32) return (size_t)KBT * MFT * 64 * 16;
  FragGeom g = frag_geom(prec);
  size_t elems = (size_t)KBT * MFT * g.NPC * 64 * g.KPL;
  size_t es = prec == KP_F64 ? 8 : prec == KP_F32 ? 4 : 2;
  return elems * es;
}

int num_classes(int prec) {
  return (prec == KP_BF16X3 || prec == KP_FP16X2) ? 11 : ((prec == KP_F64 || prec == KP_F32) ? 4 : 3);
}

// A launch takes fewer than 2^32 threads along x, which tiles of 16 fibres reach
// on states that fit the memory (33 complex rows: 3.6e8 fibres, 94 GB in FP32).
static void res_grid(int64_t tiles, ResPlan* p) {
  const int64_t most = 0xffffffffll / p->threads;
  p->grid_y = (int)((tiles + most - 1) / most);
  p->grid_x = (int)((tiles + p->grid_y - 1) / p->grid_y);
}

// Fragments per wave (MF) by the operator's rows: one up to 80 rows (four or
// five waves share the tile; two would make an odd fifth fragment a whole
// padded one: us, modes 1 / 2 of n = 72, one against two, FP64 complex 9.9 /
// 10.2 against 12.3 / 11.4, FP32 7.7 / 7.9 against 9.1 / 8.6, real 4.7 / 4.9
// against 5.4 / 5.1), two or three up to 256 (at most eight waves, 128
// registers or fewer, so four waves fit each SIMD; three where it divides the
// nine to twelve fragments: FP64 n = 168 102 / 98 against 132 / 132), four
// above (real operators of up to 512 rows).  Short operators put several 16-fibre groups
// in one workgroup, unless that would leave fewer than two workgroups per CU.
void res_plan(int prec, int form, bool ph, int cls, ResArgs* a, ResPlan* p) {
  const int frags = (a->m + 15) / 16;
  const int es = (prec == KP_F64 ? 8 : 4) * (form == RF_RR ? 1 : 2);
  p->run = 0;
  if (a->nsteps > 1 && a->n <= 64) {
    p->run = a->n <= 32 ? 32 : 64;
    p->prec = prec;
    p->form = form;
    p->mf = p->nf = 1;
    p->ph = 0;
    a->WM = frags;
    a->WN = a->NRB = 1;
    p->threads = 64 * frags;
    res_grid((a->F + 15) / 16, p);
    p->lds = (size_t)2 * p->run * 17 * es;
    return;
  }
  int mf = cls >= 0 ? std::min(cls, 3) + 1
                    : (frags <= 5 ? 1 : (frags <= 8 ? 2 : (frags <= 12 ? 3 : (frags <= 16 ? 2 : 4))));
  while (mf < 4 && (frags + mf - 1) / mf > (mf == 1 ? 16 : 8)) ++mf;
  p->prec = prec;
  p->form = form;
  p->mf = mf;
  p->ph = ph ? 1 : 0;
  a->WM = (frags + mf - 1) / mf;
  a->WN = a->WM == 1 ? 4 : (a->WM == 2 ? 2 : 1);
  p->nf = (form == RF_RR && a->n <= 256 && a->F >= 16384) ? 2 : 1;
  while (a->WN > 1 && (a->F + 16 * p->nf * a->WN - 1) / (16 * p->nf * a->WN) < 512) a->WN /= 2;
  a->NRB = 1;
  // an operator of few rows and long columns: the tile holds the columns
  auto lds = [&]() { return (size_t)res_lds_rows(a->n) * (16 * p->nf * a->WN + 1) * es; };
  while (a->WN > 1 && lds() > MAX_LDS) a->WN /= 2;
  if (lds() > MAX_LDS) p->nf = 1;
  const int nt = 16 * p->nf * a->WN;
  p->threads = 64 * a->WM * a->WN;
  res_grid((a->F + nt - 1) / nt, p);
  p->lds = lds();
}

// Four waves for every item of a batch: WM of them along the rows.
void res_batch_plan(int prec, int form, ResArgs* a, int* kind, int64_t* tiles, size_t* lds) {
  const int frags = (a->m + 15) / 16;
  a->WM = frags <= 1 ? 1 : (frags <= 2 ? 2 : 4);
  a->WN = 4 / a->WM;
  // at most three fragments per wave (and so 128 registers in FP32, four waves
  // per SIMD), the rows in as many passes as that takes
  a->NRB = (frags + 11) / 12;
  const int mf = (frags + a->WM * a->NRB - 1) / (a->WM * a->NRB);
  // real fibres: half the operator traffic per fibre, which they would wait for
  const int nf = form == RF_RR && frags > 2 ? 2 : 1;
  *kind = nf == 2 ? RES_KIND_NF2 + mf : form * 10 + mf;
  const int nt = 16 * nf * a->WN;
  *tiles = (a->F + nt - 1) / nt;
  *lds = (size_t)res_lds_rows(a->n) * (nt + 1) * (prec == KP_F64 ? 8 : 4) * (form == RF_RR ? 1 : 2);
}

hipError_t launch_res(const ResPlan& p, const ResArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
  return p.prec == KP_F64 ? launch_res_f64(p, a, s, start, stop) : launch_res_f32(p, a, s, start, stop);
}

void gauss_blocks(int64_t rows, int64_t cols, int* JBT, int* MFT) {
  *JBT = (int)(((cols + 15) / 16 + 3) / 4 * 4);
  *MFT = (int)(((rows + 31) / 32 + 7) / 8 * 8);
}

size_t gauss_prepared_bytes(int prec, int JBT, int MFT) {
  const int npc = prec == KP_BF16X3 ? 3 : 2;
  return (size_t)JBT * 3 * MFT * npc * 64 * 8 * 2;
}

hipError_t launch_prepare_gauss(int prec, const double* master, int64_t rows, int64_t cols, int64_t ld, void* out,
                                int JBT, int MFT, int a_exp, hipStream_t s) {
  const int64_t slots = (int64_t)JBT * 3 * MFT * 64;
  const dim3 grid((unsigned)((slots + 255) / 256));
  if (prec == KP_FP16X2)
    hipLaunchKernelGGL(prepare_gauss_kernel<KP_FP16X2>, grid, dim3(256), 0, s, master, rows, cols, ld, out, JBT, MFT,
                       a_exp);
  else if (prec == KP_BF16X3)
    hipLaunchKernelGGL(prepare_gauss_kernel<KP_BF16X3>, grid, dim3(256), 0, s, master, rows, cols, ld, out, JBT, MFT,
                       a_exp);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

bool rs_plan(const ModeArgs& a, int prec, int cplx, ModePlan* plan) {
  if (a.Mr > 512 || a.Kr > 512) return false;
  const int kb = (a.Kr + 15) / 16;
  const int npb = prec == KP_BF16X3 ? 3 : 2;
  const int form = cplx ? RS_CC : (a.rview ? RS_RC : RS_RR);
  auto lds = [&](int nf) { return (size_t)kb * nf * npb * 1024; };
  const bool two = lds(2) <= MAX_LDS && (prec != KP_BF16X3 || a.Mr <= 256);
  // 64 fibres per tile, 32 where that would leave CUs without one or not fit
  // the 160 KiB of LDS; the two planes of 32 complex fibres for RC
  const int nf = form == RS_RC ? 2 : (two && a.F >= 64 * 200 ? 2 : 1);
  if (form == RS_RC && !two) return false;
  *plan = ModePlan{};
  plan->cls = RS_CLASS;
  plan->rs = nf;
  plan->rs_form = form;
  plan->rs_lds = std::max<size_t>(lds(nf), 256);
  plan->nt = 32 * nf;
  plan->mt_rows = 512;
  plan->grid_x = (int)((a.F + 32 * nf - 1) / (32 * nf));
  plan->grid_y = 1;
  plan->threads = 64 * ((a.Mr + 31) / 32);
  plan->covers_all_rows = true;
  return plan->grid_x > 0;
}

namespace {
// Whether the built-in choice for a split product is class 6: operators of up
// to 400 real rows and columns.  Complex ones (200 entries): unaligned fibres, which the other classes gather entry by entry
// (FP16X2, mode 1 / 2, us, against class 0): n = 81 9.6 / 9.5 (15.7 / 15.6),
// 141 30 / 30 (42 / 39), 181 50 / 48 (62 / 49); aligned ones (mode 2, class 6 /
// best other built-in choice): n = 48 6.1 / 9.3, 64 7.0 / 9.4, 128 17.0 / 16.8,
// 192 60 / 73; BF16X3 64 5.3 / 9.8, 192 80 / 109.  Above, its 32- and 64-fibre
// tiles stream the operator too often (mode 2, n = 211 80 / 72 unaligned, 224
// 103 / 81, 256 138 / 106).  Real ones (mode 1 / 2, us, class 6 against the
// fastest other class), FP16X2 on complex fibres: n = 64 7.0 / 9.1 (9.2 / 9.1),
// 81 9.4 / 9.8 (17.2 / 17.1), 128 15.9 / 16.1 (19.4 / 15.9), 256 74 / 83
// (129 / 110), 400 509 / 492 (660 / 570); on real fibres 256 46 / 49 (73 / 59),
// 400 262 / 276 (337 / 283), 500 611 / 586 (888 / 519); BF16X3 on real fibres
// 256 69 / 77 (89 / 76), 350 273 / 276 (366 / 291), 400 444 / 436 (457 / 413):
// there the line is at 352 rows.
bool rs_rule(const ModeArgs& a, int prec, int cplx) {
  const int most = !cplx && prec == KP_BF16X3 ? 352 : 400;
  return a.Mr <= most && a.Kr <= most;
}
}  // namespace

bool plan_mode(const ModeArgs& a, int prec, int cplx, bool want_pro, bool want_epi, bool fcontig_ok,
               bool kcontig_ok, ModePlan* plan, bool batch, int force_cls, bool gauss_ok) {
  FragGeom g = frag_geom(prec);
  // two interleaved real fibres (P == 2), 16-byte aligned runs of 8 rows
  const bool pair_ok = !kcontig_ok && !cplx && a.P == 2 && a.Kr % 8 == 0;
  const int load = kcontig_ok ? KL_KCONTIG : (pair_ok ? KL_PAIR : (fcontig_ok ? KL_FCONTIG : KL_GENERIC));
  const int pro = (want_pro && cplx) ? 1 : 0;
  const int epi = (want_epi && cplx) ? 1 : 0;
  TileShape t0;
  if (!tile_shape(prec, 0, &t0)) return false;
  int cls = 0;
  const int rw = t0.WMF * g.MB;                      // rows per wave
  const bool split = prec == KP_BF16X3 || prec == KP_FP16X2;
  TileShape tf;
  // three-product classes only where the caller has the operator's Gauss
  // preparation (complex operator and state, no batch, no identity split)
  if (is_gauss_class(force_cls) && !(gauss_ok && cplx && !batch && (load == KL_KCONTIG || load == KL_FCONTIG)))
    force_cls = -1;
  // the prepared operator's K-blocks must make whole LDS chunks of the class
  // (three-product classes: their own padding, a multiple of every chunk)
  int kbt = 0, mft = 0;
  op_blocks(prec, a.Mr, a.Kr, &kbt, &mft);
  // resident-tile split kernel (class 6): any stride, at most 512 real rows
  // and columns
  if (split && !batch && (force_cls == RS_CLASS || (force_cls < 0 && rs_rule(a, prec, cplx))) &&
      rs_plan(a, prec, cplx, plan)) {
    plan->prec = prec;
    plan->cplx = cplx;
    plan->load = load;
    plan->pro = pro;
    plan->epi = epi;
    return true;
  }
  if (force_cls >= 0 && tile_shape(prec, force_cls, &tf) && (is_gauss_class(force_cls) || kbt % tf.KCH == 0) &&
      (batch ? batch_kind_any(prec, cplx, load, force_cls)
             : pick_kernel_any(prec, cplx, load, pro, epi, force_cls) != nullptr)) {
    cls = force_cls;
  } else if (!batch && split && cplx && load != KL_GENERIC && a.Mr > 2 * rw) {
    cls = 4;   // 4 x 128 rows, 128 fibres, 2 K-blocks per chunk: fastest for 256-long complex modes
  } else if (!pro && !epi && load != KL_GENERIC) {
    if (a.Mr <= rw) cls = 2;
    else if (a.Mr <= 2 * rw) cls = 1;
  }
  TileShape t;
  if (!tile_shape(prec, cls, &t)) return false;
  plan->prec = prec;
  plan->cplx = cplx;
  plan->load = load;
  plan->pro = pro;
  plan->epi = epi;
  plan->cls = cls;
  plan->gauss = is_gauss_class(cls) ? 1 : 0;
  plan->nt = t.WN * t.WNF * g.NB;
  plan->threads = 64 * t.WM * t.WN;
  plan->mt_rows = t.WM * t.WMF * g.MB;
  plan->grid_x = (int)((a.F + plan->nt - 1) / plan->nt);
  const int mfr = (a.Mr + g.MB - 1) / g.MB;          // fragments holding real rows
  plan->grid_y = (mfr + t.WM * t.WMF - 1) / (t.WM * t.WMF);
  plan->covers_all_rows = plan->grid_y == 1;
  {
    const int64_t out_bytes = (int64_t)a.Mr * a.F * (prec == KP_F64 ? 8 : 4);
    plan->full = (a.F % plan->nt == 0 && a.Mr % plan->mt_rows == 0 && out_bytes < ((int64_t)1 << 32) &&
                  load != KL_GENERIC && (cls == 0 || cls >= 3))
                     ? 1
                     : 0;
  }
  if (batch) return plan->grid_x > 0 && batch_kind_any(prec, cplx, load, cls);
  return plan->grid_x > 0 && pick_kernel_any(prec, cplx, load, pro, epi, cls) != nullptr;
}

hipError_t launch_mode(const ModePlan& p, const ModeArgs& a, hipStream_t s, hipEvent_t start, hipEvent_t stop,
                       const VortexW* w) {
  if (p.rs)
    return p.prec == KP_FP16X2 ? launch_rsplit_fp16x2(p, a, w ? *w : VortexW{}, s, start, stop)
                               : launch_rsplit_bf16x3(p, a, w ? *w : VortexW{}, s, start, stop);
  KernFn fn = pick_kernel_any(p.prec, p.cplx, p.load, p.pro, p.epi, p.cls, p.full, a.idadd ? 1 : 0);
  if (!fn) return hipErrorInvalidDeviceFunction;
  dim3 grid(p.grid_x, p.grid_y, 1);
  if (start || stop) {
    // events stamped by the kernel's own dispatch (no separate marker
    // packets between launches): the kernel's execution time
    hipExtLaunchKernelGGL(fn, grid, dim3(p.threads), 0, s, start, stop, 0, a);
  } else {
    hipLaunchKernelGGL(fn, grid, dim3(p.threads), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_mode_batch_merged(int prec, int ida, const BatchItem* items, int count, hipStream_t s) {
  BatchFn fn = nullptr;
  switch (prec) {
    case KP_BF16X3: fn = ida ? pick_batch_merged_bf16x3_ida() : pick_batch_merged_bf16x3(); break;
    case KP_BF16: fn = ida ? pick_batch_merged_bf16_ida() : pick_batch_merged_bf16(); break;
    default: return hipErrorInvalidDeviceFunction;
  }
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(fn, dim3(count), dim3(256), 0, s, items);
  return hipGetLastError();
}

hipError_t launch_prepare_steps(int prec, const StepPrep& p, hipStream_t s) {
  if (p.modes < 1 || p.modes > MAX_STEP_MODES || p.steps < 1) return hipErrorInvalidValue;
  int64_t slots = 0;
  for (int k = 0; k < p.modes; ++k) slots = std::max(slots, (int64_t)p.m[k].KBT * p.m[k].MFT * 64);
  const dim3 grid((unsigned)((slots + 255) / 256), (unsigned)(p.modes * p.steps));
  switch (prec) {
    case KP_F64: hipLaunchKernelGGL(prepare_steps_kernel<KP_F64>, grid, dim3(256), 0, s, p); break;
    case KP_F32: hipLaunchKernelGGL(prepare_steps_kernel<KP_F32>, grid, dim3(256), 0, s, p); break;
    case KP_BF16X3: hipLaunchKernelGGL(prepare_steps_kernel<KP_BF16X3>, grid, dim3(256), 0, s, p); break;
    case KP_FP16X2: hipLaunchKernelGGL(prepare_steps_kernel<KP_FP16X2>, grid, dim3(256), 0, s, p); break;
    case KY_RES64: hipLaunchKernelGGL(prepare_steps_kernel<KY_RES64>, grid, dim3(256), 0, s, p); break;
    case KY_RES32: hipLaunchKernelGGL(prepare_steps_kernel<KY_RES32>, grid, dim3(256), 0, s, p); break;
    default: hipLaunchKernelGGL(prepare_steps_kernel<KP_BF16>, grid, dim3(256), 0, s, p); break;
  }
  return hipGetLastError();
}

hipError_t launch_prepare_jobs(int lay, const ExpmBatch& b, const double* exps, int KBT, int MFT, hipStream_t s) {
  if (b.nb < 1 || b.nb > MAX_EXPM) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(((int64_t)KBT * MFT * 64 + 255) / 256), (unsigned)b.nb);
  switch (lay) {
#define MM_PJ(L_) \
  case L_: hipLaunchKernelGGL(prepare_jobs_kernel<L_>, grid, dim3(256), 0, s, b, exps, KBT, MFT); break;
    MM_PJ(KP_F64) MM_PJ(KP_F32) MM_PJ(KP_BF16X3) MM_PJ(KP_FP16X2) MM_PJ(KP_BF16) MM_PJ(KY_RES64) MM_PJ(KY_RES32)
#undef MM_PJ
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prepare(int prec, int cplx, const double* master, int64_t rows, int64_t cols,
                          int64_t ld, PhaseScale ph, void* out, int KBT, int MFT, hipStream_t s,
                          int a_exp) {
  const int64_t slots = (int64_t)KBT * MFT * 64;
  const int threads = 256;
  const int blocks = (int)((slots + threads - 1) / threads);
  switch (prec) {
    case KP_F64:
      hipLaunchKernelGGL(prepare_kernel<KP_F64>, dim3(blocks), dim3(threads), 0, s, master, rows,
                         cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
    case KP_F32:
      hipLaunchKernelGGL(prepare_kernel<KP_F32>, dim3(blocks), dim3(threads), 0, s, master, rows,
                         cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
    case KP_BF16X3:
      hipLaunchKernelGGL(prepare_kernel<KP_BF16X3>, dim3(blocks), dim3(threads), 0, s, master,
                         rows, cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
    case KY_RES64:
      hipLaunchKernelGGL(prepare_kernel<KY_RES64>, dim3(blocks), dim3(threads), 0, s, master, rows,
                         cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
    case KY_RES32:
      hipLaunchKernelGGL(prepare_kernel<KY_RES32>, dim3(blocks), dim3(threads), 0, s, master, rows,
                         cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
    case KP_FP16X2:
      hipLaunchKernelGGL(prepare_kernel<KP_FP16X2>, dim3(blocks), dim3(threads), 0, s, master,
                         rows, cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
    default:
      hipLaunchKernelGGL(prepare_kernel<KP_BF16>, dim3(blocks), dim3(threads), 0, s, master, rows,
                         cols, ld, cplx, ph, out, KBT, MFT, a_exp);
      break;
  }
  return hipGetLastError();
}

int norm_partials() { return NORM_BLOCKS; }

hipError_t launch_expm_generator(const double* A, int n, const double* d, double gr, double gi, double fr, double fi,
                                 double* X, hipStream_t s) {
  const int64_t nn = (int64_t)n * n;
  hipLaunchKernelGGL(expm_generator_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, A, n, d, gr, gi, fr,
                     fi, X);
  return hipGetLastError();
}

hipError_t launch_expm_ps(double* P, const double* W, const double* X, const double* X2, const double* X3, int n,
                          const double* c, hipStream_t s) {
  const int64_t nn = (int64_t)n * n;
  hipLaunchKernelGGL(expm_ps_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, P, W, X, X2, X3, n, c[0],
                     c[1], c[2], c[3]);
  return hipGetLastError();
}

hipError_t launch_expm_colsum(const double* A, int n, const double* d, double gr, double gi, double* out,
                              hipStream_t s) {
  hipLaunchKernelGGL(expm_colsum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, A, n, d, gr, gi, out);
  return hipGetLastError();
}

int fp16x2_op_exp(double amax) {
  if (!(amax > 0.0) || !std::isfinite(amax)) return 0;
  int e = 0;
  std::frexp(amax, &e);   // amax in [2^(e-1), 2^e)
  return e - 4;           // amax 2^-a_exp in [8, 16)
}

hipError_t launch_hermite_collapse(const double* Phi, const double* Psi, int m, int K, double tau, double* out,
                                  hipStream_t s) {
  const int64_t n = (int64_t)m * m;
  hipLaunchKernelGGL(hermite_collapse_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, Phi, Psi, m, K, tau,
                     out);
  return hipGetLastError();
}

hipError_t launch_identity_norms(const double* L, int n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(identity_norms_kernel, dim3(1), dim3(NORM_THREADS), 0, s, L, n, out);
  return hipGetLastError();
}

hipError_t launch_vortex_phase(void* v, int is_f64, int d, const int64_t* dims, const double* winv, double s,
                               hipStream_t st) {
  Dims6 D;
  int64_t count = 1;
  for (int k = 0; k < 6; ++k) D.n[k] = k < d ? dims[k] : 1;
  for (int k = 0; k < d; ++k) count *= dims[k];
  const int64_t blocks = std::min<int64_t>((count + 255) / 256, 8192);
  if (is_f64)
    hipLaunchKernelGGL(vortex_phase_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, st, (double*)v, count, d, D,
                       winv, s);
  else
    hipLaunchKernelGGL(vortex_phase_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, (float*)v, count, d, D,
                       winv, s);
  return hipGetLastError();
}

hipError_t launch_maxabs(const float* x, int64_t count, uint32_t* partial, uint32_t* slots, hipStream_t s) {
  hipLaunchKernelGGL(maxabs_partial_kernel, dim3(NORM_BLOCKS), dim3(NORM_THREADS), 0, s, x, count, partial);
  hipLaunchKernelGGL(maxabs_final_kernel, dim3(1), dim3(NORM_THREADS), 0, s, partial, NORM_BLOCKS, slots);
  return hipGetLastError();
}

template <typename S>
void reduce_dispatch(int kind, const void* x, const void* y, int64_t count, double* partial, hipStream_t s) {
  const S* xs = (const S*)x;
  const S* ys = (const S*)y;
  switch (kind) {
    case RED_SQ:
      hipLaunchKernelGGL((reduce_partial_kernel<S, RED_SQ>), dim3(NORM_BLOCKS), dim3(NORM_THREADS), 0, s, xs, ys,
                         count, partial);
      break;
    case RED_DOT_RE:
      hipLaunchKernelGGL((reduce_partial_kernel<S, RED_DOT_RE>), dim3(NORM_BLOCKS), dim3(NORM_THREADS), 0, s, xs,
                         ys, count, partial);
      break;
    default:
      hipLaunchKernelGGL((reduce_partial_kernel<S, RED_ABS4>), dim3(NORM_BLOCKS), dim3(NORM_THREADS), 0, s, xs,
                         ys, count, partial);
      break;
  }
}

hipError_t launch_reduce(int kind, const void* x, const void* y, int64_t count, int is_f64, double* partial,
                         double* result, hipStream_t s) {
  if (is_f64) reduce_dispatch<double>(kind, x, y, count, partial, s);
  else reduce_dispatch<float>(kind, x, y, count, partial, s);
  hipLaunchKernelGGL(norm_final_kernel, dim3(1), dim3(NORM_THREADS), 0, s, partial, NORM_BLOCKS, result);
  return hipGetLastError();
}

}  // namespace mm
