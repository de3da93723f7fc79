// mu-mode products in FP64 and FP32 with the whole fibre tile resident in LDS.
//
// One workgroup owns NT = 16 WN NF consecutive fibres of the [P, n, Q] view
// and all m output rows of them.  The fibres' n entries are staged into LDS
// once, in the state's own format (no chunk loop: every load of the tile is
// in flight together and the MFMA loop has no barrier in it); the WM x WN
// waves then split rows and fibres, each streaming its rows of the prepared
// operator from L2 through a register ring.  Entry layouts are the same for
// contiguous and strided fibres, so any P (odd ones too) takes the same path.
//
// What bounds it.  v_mfma_f64_16x16x4 takes 64 cycles and
// v_mfma_f32_16x16x4 32 (2048 flops each), so these precisions are bound by
// the matrix unit for every mode longer than ~32: the operator costs
// 16 bytes per lane and 16-row fragment against 3 x 64 (3 x 32) cycles of
// MFMAs, 21 bytes per cycle and CU of the 64 the L1 delivers.  What the
// shape has to avoid is padding and idle matrix units, hence 16-row
// fragments (81 complex rows run as 96, not 128 or 256) and tiles small
// enough for two to eight independent workgroups per CU, whose loads and
// stores overlap the others' MFMAs.
//
// Forms.  C3: complex operator A + iB on complex fibres x + iy in three real
// products T1 = A x, T2 = B y, T3 = (A + B)(x + y), Re = T1 - T2,
// Im = T3 - (T1 + T2): a quarter less MFMA work than the 2 x 2 block form and
// half as long an accumulation chain per product.  x + y and A + B are formed
// in registers from the rounded values, so T3's operator is consistent with
// T1's and T2's.  T3 rounds at the size of |x + y| where the block form rounds
// at that of its result; products on L - I (below) more than make up for it
// (the operator choice in mm_op_prepare_ex has the measured errors).  C4: the
// block form, Re = A x - B y and Im = A y + B x in four products, for FP32
// operators far from the identity.  RC: real operator on complex fibres, two
// products.  RR: real fibres.
//
// The tile stays in LDS until the results are written, so the identity add
// (operators prepared as L - I) reads its input there, with the prologue
// phase already applied.
#pragma once
#include "mode_tile.h"

namespace mm {

template <int PR> struct RTr;
template <> struct RTr<KP_F64> {
  typedef double st;
  typedef double st2 __attribute__((ext_vector_type(2)));
  typedef double unit __attribute__((ext_vector_type(2)));   // 16 bytes of a lane's operator entries
  typedef f64x4 acc;
};
template <> struct RTr<KP_F32> {
  typedef float st;
  typedef float st2 __attribute__((ext_vector_type(2)));
  typedef float unit __attribute__((ext_vector_type(4)));
  typedef f32x4 acc;
};

__device__ __forceinline__ void rmfma(f64x4& c, double a, double b) {
  c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ void rmfma(f32x4& c, float a, float b) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Split fibre index fg into (p, q) of the [P, n, Q] view; 32-bit division
// where the fibre count allows it.
__device__ __forceinline__ void fibre_pq(int64_t fg, int64_t P, int64_t F, int64_t* p, int64_t* q) {
  if (F <= 0x7fffffff) {
    const uint32_t u = (uint32_t)fg / (uint32_t)P;
    *q = u;
    *p = (uint32_t)fg - u * (uint32_t)P;
  } else {
    *q = fg / P;
    *p = fg - *q * P;
  }
}

// Inverse cell weight of fibre (p, q) without the factor of mode v.wmu.
__device__ __forceinline__ double fibre_weight(const VortexW& v, int64_t p, int64_t q) {
  double w = 1.0;
  for (int j = 0; j < v.wd; ++j) {
    if (j == v.wmu) continue;
    int64_t& r = j < v.wmu ? p : q;
    const int64_t i = r % v.wdims[j];
    r /= v.wdims[j];
    w *= v.winv[(int64_t)j * 4096 + i];
  }
  return w;
}

// v <- exp((i s / 2)(1 - wi |v|^2)) v
template <typename T>
__device__ __forceinline__ void vortex_phase(T& re, T& im, T hs, T wi) {
  const T th = hs * ((T)1 - wi * (re * re + im * im));
  T sn, cs;
  if constexpr (sizeof(T) == 8) sincos(th, &sn, &cs);
  else sincos_f32<false>(th, &sn, &cs);
  const T r = re * cs - im * sn;
  im = im * cs + re * sn;
  re = r;
}

// Stage the NT fibres from f0 (rows 0 .. K4 - 1, zero from row n on and for
// fibres past the last one): put(row, fibre, entry, weight of the fibre).
template <typename ent, bool PH, typename Put>
__device__ __forceinline__ void res_stage(const ResArgs& a, int64_t f0, int nthr, int NT, int K4, Put&& put) {
  constexpr int U = 8;   // loads in flight per thread
  const int tid = threadIdx.x;
  const int n = a.n;
  const ent* in = (const ent*)a.in;
  if (a.P == 1) {
    // contiguous fibres: 16 lanes along K
    const int kk = tid & 15;
    for (int f = tid >> 4; f < NT; f += nthr >> 4) {
      const int64_t fg = f0 + f;
      const bool ok = fg < a.F;
      const ent* src = in + (ok ? fg * n : 0);
      double wf = 0.0;
      if constexpr (PH) {
        if (a.w.winv && ok) wf = fibre_weight(a.w, 0, fg);
      }
      for (int k0 = kk; k0 < K4; k0 += 16 * U) {
        ent v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          v[u] = ent{};
          if (ok && k0 + 16 * u < n) v[u] = src[k0 + 16 * u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (k0 + 16 * u < K4) put(k0 + 16 * u, f, v[u], wf);
      }
    }
  } else {
    // strided fibres: lanes along the fibres
    const int sh = 31 - __clz(NT);
    const int f = tid & (NT - 1);
    const int kstep = nthr >> sh;
    const int64_t fg = f0 + f;
    const bool ok = fg < a.F;
    int64_t p = 0, q = 0;
    if (ok) fibre_pq(fg, a.P, a.F, &p, &q);
    double wf = 0.0;
    if constexpr (PH) {
      if (a.w.winv && ok) wf = fibre_weight(a.w, p, q);
    }
    const ent* src = in + (p + a.P * (int64_t)n * q);
    for (int k0 = tid >> sh; k0 < K4; k0 += kstep * U) {
      ent v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u] = ent{};
        if (ok && k0 + kstep * u < n) v[u] = src[(int64_t)(k0 + kstep * u) * a.P];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + kstep * u < K4) put(k0 + kstep * u, f, v[u], wf);
    }
  }
}

// The MFMAs of K-block u of operator unit au on fibre entries x.
template <int FORM, typename acc_t, int NP, typename unit, typename ent>
__device__ __forceinline__ void res_mac(acc_t (&acc)[NP], const unit& au, int u, const ent& x) {
  if constexpr (FORM == RF_C3) {
    rmfma(acc[0], au[2 * u], x[0]);
    rmfma(acc[1], au[2 * u + 1], x[1]);
    rmfma(acc[2], au[2 * u] + au[2 * u + 1], x[0] + x[1]);
  } else if constexpr (FORM == RF_C4) {
    rmfma(acc[0], au[2 * u], x[0]);
    rmfma(acc[1], au[2 * u], x[1]);
    rmfma(acc[0], -au[2 * u + 1], x[1]);
    rmfma(acc[1], au[2 * u + 1], x[0]);
  } else if constexpr (FORM == RF_RC) {
    rmfma(acc[0], au[u], x[0]);
    rmfma(acc[1], au[u], x[1]);
  } else {
    rmfma(acc[0], au[u], x);
  }
}
// The output entry of accumulator register r (logical row 4 g + r of the
// fragment in both precisions: the FP64 rows are permuted at preparation).
template <int FORM, typename ent, typename acc_t, int NP>
__device__ __forceinline__ ent res_out(const acc_t (&acc)[NP], int r) {
  if constexpr (FORM == RF_C3) return ent{acc[0][r] - acc[1][r], acc[2][r] - (acc[0][r] + acc[1][r])};
  else if constexpr (NP == 2) return ent{acc[0][r], acc[1][r]};
  else return acc[0][r];
}

// One tile: fibres [tile * NT, + NT), all rows, in NRB blocks of WM * MF
// fragments of 16 rows, one after the other.
// FORM: RF_C3, RF_C4, RF_RC, RF_RR.  PH: the instance carries the phases.  lds:
// res_lds_rows(n) rows of NT + 1 entries.
template <int PR, int FORM, int MF, int NF, bool PH>
__device__ __forceinline__ void res_tile(const ResArgs& a, int64_t tile, void* lds) {
  typedef RTr<PR> T;
  typedef typename T::st st;
  typedef typename T::st2 st2;
  typedef typename T::unit unit;
  typedef typename T::acc acc_t;
  constexpr bool CX = FORM != RF_RR;                 // complex entries
  constexpr bool AC = FORM == RF_C3 || FORM == RF_C4;   // complex operator
  typedef typename std::conditional<CX, st2, st>::type ent;
  constexpr int NP = FORM == RF_C3 ? 3 : (CX ? 2 : 1);   // accumulators per output fragment
  constexpr int UK = (int)(16 / ((AC ? 2 : 1) * sizeof(st)));       // K-blocks per operator unit
  constexpr int D = UK == 4 ? 2 : (MF == 1 ? 4 : (MF == 2 && sizeof(st) == 4 ? 3 : 2));   // operator ring depth in units

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave % a.WM, wn = wave / a.WM;
  const int nthr = 64 * a.WM * a.WN;
  const int NT = 16 * NF * a.WN;
  const int ld = NT + 1;
  const int K4 = (a.n + 4 * UK - 1) / (4 * UK) * (4 * UK);   // rows of whole units, zero from n on
  const int64_t f0 = tile * NT;
  ent* L = (ent*)lds;
  const int n = a.n;

  // operator: fragment mf0 + i, unit ku at Ap + i * 64 + ku * ustride (the
  // prepared operator is padded by MF - 1 fragments and D units)
  const int64_t ustride = (int64_t)a.MFT * 64;
  const int KU = K4 / (4 * UK);
  int mf0 = 0;                           // first row fragment of this wave
  const unit* __restrict__ Ap = nullptr;
  unit ring[D][MF];
  auto preload = [&](int rb) {
    mf0 = (rb * a.WM + wm) * MF;
    Ap = (const unit*)a.A + (int64_t)min(mf0, a.MFT - MF) * 64 + lane;
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
      for (int i = 0; i < MF; ++i) ring[d][i] = Ap[i * 64];
      Ap += ustride;
    }
  };

  if constexpr (!PH) preload(0);         // (with phases their registers come first)

  res_stage<ent, PH>(a, f0, nthr, NT, K4, [&](int k, int f, ent v, double wf) {
    if constexpr (PH) {
      if (a.s_pre != 0.0) {
        st re = v[0], im = v[1];
        if (a.w.winv) vortex_phase<st>(re, im, (st)(0.5 * a.s_pre), (st)(wf * a.w.winv[(int64_t)a.w.wmu * 4096 + min(k, n - 1)]));
        else phase<st>(re, im, (st)a.s_pre);
        v = st2{re, im};
      }
    }
    L[k * ld + f] = v;
  });
  __syncthreads();

  // ---------------------------------------------------------------- product
  const int g = lane >> 4, c = lane & 15;
  const int fl0 = wn * 16 * NF + c;      // this lane's fibre in N-fragment 0
  acc_t acc[MF][NF][NP];
  const ent* const Lb = L + g * ld + fl0;
  ent b[2][NF];
  // one product of the tile: fibre entries one K-block ahead from LDS,
  // operator units D ahead from L2
  auto product = [&]() {
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j)
#pragma unroll
        for (int t = 0; t < NP; ++t) acc[i][j][t] = acc_t{0, 0, 0, 0};
    if (mf0 * 16 >= a.m) return;         // a wave past the last row only stages
    const ent* Lk = Lb;
#pragma unroll
    for (int j = 0; j < NF; ++j) b[0][j] = Lk[16 * j];
    for (int ku0 = 0; ku0 < KU; ku0 += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        if (d == 0 || ku0 + d < KU) {
#pragma unroll
          for (int u = 0; u < UK; ++u) {
            const int s = (d * UK + u) & 1;
            // (the four rows after the tile's last are allocated, not used)
            Lk += 4 * ld;
#pragma unroll
            for (int j = 0; j < NF; ++j) b[s ^ 1][j] = Lk[16 * j];
            __builtin_amdgcn_sched_barrier(0);
            const ent(&x)[NF] = b[s];
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
              for (int j = 0; j < NF; ++j) res_mac<FORM>(acc[i][j], ring[d][i], u, x[j]);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int i = 0; i < MF; ++i) ring[d][i] = Ap[i * 64];
          Ap += ustride;
        }
      }
      if constexpr ((D * UK) % 2 == 1) {
#pragma unroll
        for (int j = 0; j < NF; ++j) b[0][j] = b[1][j];
      }
    }
  };
  auto result = [&](int i, int j, int r, int row) -> ent {
    ent y = res_out<FORM, ent>(acc[i][j], r);
    if (a.idadd) y += L[row * ld + fl0 + 16 * j];
    return y;
  };

  for (int rb = 0; rb < a.NRB; ++rb) {
    if (PH || rb > 0) preload(rb);
    for (int s = 1;; ++s) {
      product();
      if (s >= a.nsteps) break;
      // repeated products of a square operator: the result replaces the tile
      // (each lane reads, for the identity add, only the entries it rewrites)
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (mf0 + i) * 16 + 4 * g + r;
          if (row < n) {
#pragma unroll
            for (int j = 0; j < NF; ++j) L[row * ld + fl0 + 16 * j] = result(i, j, r, row);
          }
        }
      preload(0);
      __syncthreads();
    }

    // --------------------------------------------------------------- epilogue
    ent* out = (ent*)a.out;
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      const int64_t fg = f0 + fl0 + 16 * j;
      if (fg >= a.F) continue;
      int64_t p = 0, q = fg;
      if (a.P != 1) fibre_pq(fg, a.P, a.F, &p, &q);
      ent* dst = out + (p + a.P * (int64_t)a.m * q);
      double wf = 0.0;
      if constexpr (PH) {
        if (a.w.winv && a.s_post != 0.0) wf = fibre_weight(a.w, p, q);
      }
#pragma unroll
      for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = (mf0 + i) * 16 + 4 * g + r;
          if (row < a.m) {
            ent y = result(i, j, r, row);
            if constexpr (PH) {
              if (a.s_post != 0.0) {
                st re = y[0], im = y[1];
                if (a.w.winv) vortex_phase<st>(re, im, (st)(0.5 * a.s_post), (st)(wf * a.w.winv[(int64_t)a.w.wmu * 4096 + row]));
                else phase<st>(re, im, (st)a.s_post);
                y = st2{re, im};
              }
            }
            dst[(int64_t)row * a.P] = y;
          }
        }
    }
  }
}

// nsteps products of one square operator of at most KR rows on a tile of 16
// fibres, one wave per 16 rows, the operator in registers and the tile
// ping-ponging between two LDS buffers (one barrier per product).  Such runs
// leave one wave per SIMD, so a product is latency: its KR / 4 K-blocks are
// fully unrolled with the padding in place (no branch between them), all LDS
// reads run ahead of the first MFMA, and even and odd K-blocks accumulate
// apart, so that consecutive MFMAs do not wait for each other.  us per call,
// 20 steps: 2-D heat 64 x 64 FP64 36 (101 with the state and both operators in
// one workgroup's LDS, 52 through res_tile), n = 64 C3 FP32 87 (108 through
// res_tile).
template <int PR, int FORM, int KR>
__device__ __forceinline__ void res_run_tile(const ResArgs& a, int64_t tile, void* lds) {
  typedef RTr<PR> T;
  typedef typename T::st st;
  typedef typename T::st2 st2;
  typedef typename T::unit unit;
  typedef typename T::acc acc_t;
  constexpr bool CX = FORM != RF_RR;
  constexpr bool AC = FORM == RF_C3 || FORM == RF_C4;
  typedef typename std::conditional<CX, st2, st>::type ent;
  constexpr int NP = FORM == RF_C3 ? 3 : (CX ? 2 : 1);
  constexpr int UK = (int)(16 / ((AC ? 2 : 1) * sizeof(st)));
  constexpr int KUM = KR / (4 * UK);
  constexpr int ld = 17;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // row fragment
  const int n = a.n;
  const int KU = (n + 4 * UK - 1) / (4 * UK);
  const int64_t f0 = tile * 16;
  ent* cur = (ent*)lds;
  ent* nxt = cur + KR * ld;
  unit op[KUM];
#pragma unroll
  for (int ku = 0; ku < KUM; ++ku) {
    op[ku] = unit{};
    if (ku < KU) op[ku] = ((const unit*)a.A)[((int64_t)ku * a.MFT + wave) * 64 + lane];
  }
  res_stage<ent, false>(a, f0, 64 * a.WM, 16, KR, [&](int k, int f, ent v, double) {
    cur[k * ld + f] = v;
    if (k >= n) nxt[k * ld + f] = v;     // the padding rows of both buffers are zero
  });
  __syncthreads();
  const int g = lane >> 4, c = lane & 15;
  const int row0 = 16 * wave + 4 * g;
  for (int s = 1;; ++s) {
    acc_t acc[2][NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) acc[0][t] = acc[1][t] = acc_t{0, 0, 0, 0};
    const ent* Lk = cur + g * ld + c;
    ent b[KR / 4];
#pragma unroll
    for (int kb = 0; kb < KR / 4; ++kb) b[kb] = Lk[4 * kb * ld];
    __builtin_amdgcn_sched_barrier(0);   // every read is issued before the first MFMA waits
#pragma unroll
    for (int kb = 0; kb < KR / 4; ++kb) res_mac<FORM>(acc[kb & 1], op[kb / UK], kb % UK, b[kb]);
#pragma unroll
    for (int t = 0; t < NP; ++t) acc[0][t] += acc[1][t];
    ent y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      y[r] = res_out<FORM, ent>(acc[0], r);
      if (a.idadd) y[r] += cur[min(row0 + r, n - 1) * ld + c];
    }
    if (s >= a.nsteps) {
      const int64_t fg = f0 + c;
      if (fg < a.F) {
        int64_t p = 0, q = fg;
        if (a.P != 1) fibre_pq(fg, a.P, a.F, &p, &q);
        ent* dst = (ent*)a.out + (p + a.P * (int64_t)n * q);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row0 + r < n) dst[(int64_t)(row0 + r) * a.P] = y[r];
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (row0 + r < n) nxt[(row0 + r) * ld + c] = y[r];
    __syncthreads();
    ent* t = cur;
    cur = nxt;
    nxt = t;
  }
}

}  // namespace mm
