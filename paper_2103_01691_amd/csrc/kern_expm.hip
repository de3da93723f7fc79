// Device matrix exponentials of several complex FP64 matrices of one size at
// a time (column-major, interleaved, n x n, n <= 256): X = f (A + g diag(d)),
// the degree-18 Taylor polynomial by the Paterson-Stockmeyer scheme (blocks of
// four terms, Horner in X^4), q squarings.
//
// The exponentials of a splitting run are independent of each other (every
// step's generator is known in advance) but each is a chain of ~12 small
// products, so what bounds them is the launches and each product's latency,
// not its flops (128 x 128 complex: 17 Mflop).  Hence one launch per stage for
// the whole batch, the elementwise combinations in the products' epilogues,
// operands read straight from the column-major matrices (no operator
// preparation), and the K range of every 16 x 16 output tile split over a
// workgroup's four waves, which meet in LDS.  Four midpoint steps of n = 128
// FP64 (six exponentials, twelve state products of 37 us): 621 us per call,
// 1646 with one exponential at a time, an operator preparation before and a
// combination kernel after every product, and buffers allocated per call.
#include "mode_tile.h"

namespace mm {
namespace {

// X = f 2^-q (A + g diag(d)) for every job (blockIdx.y)
__global__ void expm_jobs_generator_kernel(ExpmBatch b, double* __restrict__ X) {
  const int64_t nn = (int64_t)b.n * b.n;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nn) return;
  const ExpmJob& j = b.j[blockIdx.y];
  const int i = (int)(e % b.n);
  double re = j.A[2 * e], im = j.A[2 * e + 1];
  if (j.d && i == (int)(e / b.n)) {
    re += j.gr * j.d[i];
    im += j.gi * j.d[i];
  }
  const double sc = ldexp(1.0, -b.q);
  const double fr = j.fr * sc, fi = j.fi * sc;
  f64x2* x = (f64x2*)X + blockIdx.y * nn + e;
  *x = f64x2{fr * re - fi * im, fr * im + fi * re};
}

// One product C = A B per matrix of up to two batches (blockIdx.z = pair * nb
// + matrix), with the Taylor combination of its stage:
//   EP_P0      also P = c0 I + c1 X + c2 C (the product is X^2)
//   EP_HORNER  C = A B + c0 I + c1 X + c2 X2 + c3 X3
enum { EP_NONE = 0, EP_P0 = 1, EP_HORNER = 2 };
struct ExpmGemm {
  const f64x2 *A[2], *B[2];
  f64x2* C[2];
  const f64x2 *X, *X2, *X3;
  f64x2* P;
  double c[4];
  int n, nb, ep;
};

__global__ __launch_bounds__(256) void expm_gemm_kernel(ExpmGemm a) {
  __shared__ double part[4][8][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, c = lane & 15;
  const int pair = blockIdx.z / a.nb;
  const int n = a.n;
  const int64_t off = (int64_t)(blockIdx.z % a.nb) * n * n;
  const int i0 = blockIdx.x * 16, j0 = blockIdx.y * 16;
  const f64x2* A = a.A[pair] + off + min(i0 + c, n - 1);
  const f64x2* B = a.B[pair] + off + (int64_t)min(j0 + c, n - 1) * n;
  f64x4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
  const int KB = (n + 3) / 4;
  for (int kb = wave; kb < KB; kb += 16) {
    f64x2 x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = (kb + 4 * u) * 4 + g;
      x[u] = y[u] = f64x2{0, 0};
      if (k < n) {
        x[u] = A[(int64_t)k * n];
        y[u] = B[k];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      mfma(re, x[u][0], y[u][0]);
      mfma(im, x[u][0], y[u][1]);
      mfma(re, -x[u][1], y[u][1]);
      mfma(im, x[u][1], y[u][0]);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    part[wave][2 * r][lane] = re[r];
    part[wave][2 * r + 1][lane] = im[r];
  }
  __syncthreads();
  // accumulator register r holds row g + 4 r; wave r sums and stores it
  const int i = i0 + g + 4 * wave, j = j0 + c;
  if (i >= n || j >= n) return;
  f64x2 v = {0, 0};
#pragma unroll
  for (int w = 0; w < 4; ++w) v += f64x2{part[w][2 * wave][lane], part[w][2 * wave + 1][lane]};
  const int64_t e = off + i + (int64_t)j * n;
  const double one = i == j ? a.c[0] : 0.0;
  if (a.ep == EP_HORNER) {
    v += a.c[1] * a.X[e] + a.c[2] * a.X2[e] + a.c[3] * a.X3[e];
    v[0] += one;
  } else if (a.ep == EP_P0) {
    f64x2 p = a.c[1] * a.X[e] + a.c[2] * v;
    p[0] += one;
    a.P[e] = p;
  }
  a.C[pair][e] = v;
}

}  // namespace

size_t expm_batch_bytes(int n, int nb) { return (size_t)6 * nb * n * n * 2 * sizeof(double); }

hipError_t launch_expm_batch(const ExpmBatch& b, double* buf, double** result, hipStream_t s) {
  const int64_t nn = (int64_t)b.n * b.n;
  const int64_t all = nn * b.nb;
  f64x2* X = (f64x2*)buf;
  f64x2 *X2 = X + all, *X3 = X2 + all, *Y = X3 + all, *P = Y + all, *W = P + all;
  hipLaunchKernelGGL(expm_jobs_generator_kernel, dim3((unsigned)((nn + 255) / 256), b.nb), dim3(256), 0, s, b, buf);
  double c[20] = {0};
  c[0] = 1.0;
  for (int k = 1; k <= 18; ++k) c[k] = c[k - 1] / k;
  const unsigned t = (unsigned)((b.n + 15) / 16);
  ExpmGemm g = {};
  g.n = b.n;
  g.nb = b.nb;
  g.X = X;
  g.X2 = X2;
  g.X3 = X3;
  g.P = P;
  auto run = [&](int pairs) {
    hipLaunchKernelGGL(expm_gemm_kernel, dim3(t, t, (unsigned)(pairs * b.nb)), dim3(256), 0, s, g);
  };
  auto set = [&](int k, const f64x2* A, const f64x2* B, f64x2* C) {
    g.A[k] = A;
    g.B[k] = B;
    g.C[k] = C;
  };
  // X^2 and the first block c16 I + c17 X + c18 X^2
  g.ep = EP_P0;
  for (int k = 0; k < 3; ++k) g.c[k] = c[16 + k];
  set(0, X, X, X2);
  run(1);
  // X^3 = X X^2 and X^4 = X^2 X^2 together
  g.ep = EP_NONE;
  set(0, X, X2, X3);
  set(1, X2, X2, Y);
  run(2);
  // Horner in X^4 (polynomials in X commute)
  g.ep = EP_HORNER;
  for (int j = 3; j >= 0; --j) {
    for (int k = 0; k < 4; ++k) g.c[k] = c[4 * j + k];
    set(0, Y, P, W);
    run(1);
    f64x2* tmp = P;
    P = W;
    W = tmp;
  }
  g.ep = EP_NONE;
  for (int r = 0; r < b.q; ++r) {
    set(0, P, P, W);
    run(1);
    f64x2* tmp = P;
    P = W;
    W = tmp;
  }
  *result = (double*)P;
  return hipGetLastError();
}

}  // namespace mm
