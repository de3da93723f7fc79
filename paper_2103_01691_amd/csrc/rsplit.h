// Split-precision products (FP16X2, BF16X3) with the whole fibre tile resident
// in LDS: tile class 6 of both precisions.  Forms: CC, complex operator on
// complex fibres as the real block operator; RC, real operator on complex
// fibres (their real and imaginary parts are two real fibres of one tile); RR,
// real operator on real fibres.
//
// One workgroup owns 32 NF consecutive CC or RR fibres (16 NF RC ones) and all
// rows: it loads their entries once (all loads in flight together), splits them
// into pieces and writes them to LDS in MFMA operand order; one wave per 32
// real rows then runs the K loop without a barrier, the operator streaming from
// L2 through a register ring.  The real block form and the prepared operator
// are those of mode_tile.h.
//
// Why.  At 32 cycles per v_mfma_f32_32x32x16 the products of modes up to ~200
// entries are bound by memory and latency (n = 141: 3.8 us of MFMAs, 8.5 us
// of HBM traffic), and the chunked tiles of mode_tile.h cover 128, 256 or 512
// rows (282 rows run as 512), read unaligned fibres entry by entry with a
// division per entry and wait for HBM once per chunk.  Here rows are padded to
// 32, any stride P takes the same loads (8 bytes per row and fibre, 16 along
// contiguous fibres), and the tile waits for HBM once.  64 fibres per tile
// keep the operator's L2 traffic (16 n^2 bytes per tile) at 41 bytes per cycle
// and CU; 32 are used where 64 would leave CUs without a tile or exceed LDS.
// Real operators do half the work per value, so memory and the single wait for
// it bind them further up: FP16X2 on 256 x 65536 complex fibres 129 -> 74 us
// (268 MB: 3.6 TB/s), 81 x 6561 17.2 -> 9.4, BF16X3 192 77 -> 51.
#pragma once
#include "resident.h"

namespace mm {

template <int PR, int FORM, int NF, bool PH>
__device__ __forceinline__ void rsplit_tile(const ModeArgs& a, const VortexW& vw, int64_t tile,
                                            typename Tr<PR>::pc* __restrict__ lds) {
  typedef Tr<PR> T;
  typedef typename T::pc pc;
  typedef typename T::afrag afrag;
  typedef Prods<PR> PP;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  constexpr int NPA = T::NPA, NPB = T::NPB;
  constexpr bool F16 = PR == KP_FP16X2;
  constexpr bool CC = FORM == RS_CC, RC = FORM == RS_RC;
  typedef typename std::conditional<FORM == RS_RR, float, f32x2>::type ent;
  typedef f32x4 f32x4w __attribute__((aligned(4)));
  constexpr int EPU = CC ? 4 : 8;         // entries of a staging unit
  constexpr int VPU = RC ? 16 : 8;        // its values
  constexpr int NT = RC ? 16 * NF : 32 * NF;   // fibres of entries
  constexpr int BLK = 512;                // pieces per (K-block, N-fragment, piece) block
  constexpr int D = 4;                    // operator ring depth in K-blocks
  constexpr int U = RC || (PR == KP_BF16X3 && NF == 1) ? 2 : 4;   // staging units in flight per thread

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // 32-row fragment
  const int nthr = blockDim.x;
  const int n = a.n;
  const int KB = ((CC ? 2 : 1) * n + 15) / 16;
  const int64_t P = RC ? a.P / 2 : a.P, F = RC ? a.F / 2 : a.F;   // (RC: a is the real view)
  const int64_t f0 = tile * NT;
  const float s_pre = (float)a.s_pre;

  int s_exp = 0;
  if constexpr (F16) {
    uint32_t bits = 0;
#pragma unroll
    for (int w = 0; w < SMAX_WORDS; ++w) bits = max(bits, a.smax_in[w * SMAX_STRIDE]);
    s_exp = fp16x2_state_exp(bits);
    if (tile == 0 && tid < SMAX_WORDS) a.smax_clr[tid * SMAX_STRIDE] = 0u;
  }

  // operator fragments of K-block kb for this wave
  const afrag* __restrict__ Aw = (const afrag*)a.A + (int64_t)wave * NPA * 64 + lane;
  const int64_t kstride = (int64_t)a.MFT * NPA * 64;
  afrag ring[D][NPA];
  auto load_a = [&](int kb, afrag (&dst)[NPA]) {
    const afrag* s = Aw + min(kb, a.KBT - 1) * kstride;
#pragma unroll
    for (int p = 0; p < NPA; ++p) dst[p] = s[p * 64];
  };
  if constexpr (!PH) {
#pragma unroll
    for (int d = 0; d < D; ++d) load_a(d, ring[d]);
  }

  // ---------------------------------------------------------------- staging
  // A unit is EPU consecutive entries of one fibre: one MFMA lane slot (8 real
  // K values), or two (RC: the real and the imaginary parts, N-fragments 2 j
  // and 2 j + 1).  Contiguous fibres have the lanes along K, strided ones along
  // the fibres.
  const bool contig = P == 1;
  const int KG = 2 * KB;                  // units per fibre
  const int units = KG * NT;
  auto unit_at = [&](int e, int& kg, int& f) {
    if (contig) {
      f = e / KG;
      kg = e - f * KG;
    } else {
      f = e & (NT - 1);
      kg = e / NT;
    }
  };
  // strided: the workgroup is a multiple of NT threads, so a thread keeps its fibre
  int64_t p0 = 0, q0 = min(f0 + (tid & (NT - 1)), F - 1);
  if (!contig) fibre_pq(q0, P, F, &p0, &q0);
  for (int e0 = tid; e0 < units; e0 += nthr * U) {
    float v[U][VPU];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * nthr;
      int kg, f;
      unit_at(e, kg, f);
      const int64_t fg = f0 + f;
      const bool ok = e < units && fg < F;
      const int64_t p = p0, q = contig ? (ok ? fg : 0) : q0;
      const ent* src = (const ent*)a.in + (p + P * (int64_t)n * q);
      const int j0 = EPU * kg;
#pragma unroll
      for (int r = 0; r < VPU; ++r) v[u][r] = 0.0f;
      if (contig && ok && j0 + EPU <= n) {
        // (entries are 8- or 4-byte aligned; the loads need no more)
#pragma unroll
        for (int w = 0; w < VPU / 4; ++w) {
          const f32x4w x = *(const f32x4w*)((const float*)(src + j0) + 4 * w);
#pragma unroll
          for (int r = 0; r < 4; ++r) v[u][4 * w + r] = x[r];
        }
      } else if (ok) {
#pragma unroll
        for (int r = 0; r < EPU; ++r)
          if (j0 + r < n) {
            const ent x = src[(int64_t)(j0 + r) * P];
            if constexpr (FORM == RS_RR) {
              v[u][r] = x;
            } else {
              v[u][2 * r] = x[0];
              v[u][2 * r + 1] = x[1];
            }
          }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * nthr;
      if (e >= units) break;
      int kg, f;
      unit_at(e, kg, f);
      if constexpr (PH) {
        if (a.s_pre != 0.0) {
          double wf = 0.0;
          if (vw.winv) wf = fibre_weight(vw, p0, contig ? min(f0 + f, F - 1) : q0);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (vw.winv)
              vortex_phase<float>(v[u][2 * r], v[u][2 * r + 1], (float)(0.5 * a.s_pre),
                                  (float)(wf * vw.winv[(int64_t)vw.wmu * 4096 + min(4 * kg + r, n - 1)]));
            else
              phase<float>(v[u][2 * r], v[u][2 * r + 1], s_pre);
          }
        }
      }
      const int kb = kg >> 1, g = kg & 1, nn = f % 32;
#pragma unroll
      for (int h = 0; h < (RC ? 2 : 1); ++h) {
        const int nf = RC ? 2 * (f / 32) + h : f / 32;
        pc pieces[8][NPB];
#pragma unroll
        for (int r = 0; r < 8; r += 2) {
          const float x0 = v[u][RC ? 2 * r + h : r], x1 = v[u][RC ? 2 * r + 2 + h : r + 1];
          if constexpr (F16) {
            split_f16x2(x0, x1, s_exp, pieces[r], pieces[r + 1]);
          } else {
            split_bf16<NPB>(x0, pieces[r]);
            split_bf16<NPB>(x1, pieces[r + 1]);
          }
        }
#pragma unroll
        for (int p = 0; p < NPB; ++p) {
          afrag w;
#pragma unroll
          for (int r = 0; r < 8; ++r) w[r] = pieces[r][p];
          *(afrag*)(lds + ((kb * NF + nf) * NPB + p) * BLK + (g * 32 + swz(nn, kb, g)) * 8) = w;
        }
      }
    }
  }
  if constexpr (PH) {
#pragma unroll
    for (int d = 0; d < D; ++d) load_a(d, ring[d]);
  }
  __syncthreads();

  // ---------------------------------------------------------------- product
  f32x16 acc[NF];
#pragma unroll
  for (int j = 0; j < NF; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.0f;
  const int g = lane / 32, nn = lane % 32;
  auto read_b = [&](int kb, afrag (&dst)[NF][NPB]) {
#pragma unroll
    for (int p = 0; p < NPB; ++p)
#pragma unroll
      for (int j = 0; j < NF; ++j)
        dst[j][p] = *(const afrag*)(lds + ((kb * NF + j) * NPB + p) * BLK + (g * 32 + swz(nn, kb, g)) * 8);
  };
  afrag b[2][NF][NPB];
  read_b(0, b[0]);
  for (int kb0 = 0; kb0 < KB; kb0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      if (d == 0 || kb0 + d < KB) {
        read_b(min(kb0 + d + 1, KB - 1), b[(d + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < PP::N; ++k)
#pragma unroll
          for (int j = 0; j < NF; ++j) mfma(acc[j], ring[d][PP::a(k)], b[d & 1][j][PP::b(k)]);
        __builtin_amdgcn_sched_barrier(0);
        load_a(kb0 + d + D, ring[d]);
      }
    }
  }

  // --------------------------------------------------------------- epilogue
  // register 4 qd + r holds real row 8 qd + 4 (lane / 32) + r of the fragment:
  // two complex entries per quad (CC), four real ones (RR), or the real and
  // imaginary parts of four in two fragments (RC)
  const int o_exp = s_exp + a.a_exp - 11;
  float vmax = 0.0f;
  const bool weigh = PH && vw.winv && (a.s_post != 0.0 || (a.idadd && a.s_pre != 0.0));
  constexpr int EPQ = CC ? 2 : 4;         // entries of a quad
#pragma unroll
  for (int j = 0; j < NF; j += (RC ? 2 : 1)) {
    const int64_t fg = f0 + (RC ? j / 2 : j) * 32 + nn;
    if (fg >= F) continue;
    int64_t p = 0, q = fg;
    if (!contig) fibre_pq(fg, P, F, &p, &q);
    const int64_t base = p + P * (int64_t)a.m * q;
    double wf = 0.0;
    if constexpr (PH) {
      if (weigh) wf = fibre_weight(vw, p, q);
    }
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      const int e0 = wave * (CC ? 16 : 32) + (CC ? 4 : 8) * qd + EPQ * g;
      constexpr int VPE = FORM == RS_RR ? 1 : 2;
      float w[EPQ * VPE];
#pragma unroll
      for (int r = 0; r < EPQ * VPE; ++r) {
        w[r] = RC ? acc[j + (r & 1)][4 * qd + r / 2] : acc[j][4 * qd + r];
        if constexpr (F16) w[r] = ldexpf(w[r], o_exp);
      }
#pragma unroll
      for (int h = 0; h < EPQ; ++h) {
        const int ie = e0 + h;
        if (ie >= a.m) {
#pragma unroll
          for (int r = 0; r < VPE; ++r) w[VPE * h + r] = 0.0f;
          continue;
        }
        float wk = 0.0f;
        if constexpr (PH) {
          if (weigh) wk = (float)(wf * vw.winv[(int64_t)vw.wmu * 4096 + ie]);
        }
        if (a.idadd) {
          const ent x = ((const ent*)a.in)[base + (int64_t)ie * P];
          if constexpr (FORM == RS_RR) {
            w[h] += x;
          } else {
            float re = x[0], im = x[1];
            if constexpr (PH) {
              if (a.s_pre != 0.0) {
                if (vw.winv) vortex_phase<float>(re, im, (float)(0.5 * a.s_pre), wk);
                else phase<float>(re, im, s_pre);
              }
            }
            w[2 * h] += re;
            w[2 * h + 1] += im;
          }
        }
        if constexpr (PH) {
          if (a.s_post != 0.0) {
            if (vw.winv) vortex_phase<float>(w[2 * h], w[2 * h + 1], (float)(0.5 * a.s_post), wk);
            else phase<float>(w[2 * h], w[2 * h + 1], (float)a.s_post);
          }
        }
        if constexpr (F16) {
#pragma unroll
          for (int r = 0; r < VPE; ++r) vmax = fmaxf(vmax, fabsf(w[VPE * h + r]));
        }
      }
      ent* dst = (ent*)a.out + base + (int64_t)e0 * P;
      if (contig && e0 + EPQ <= a.m) {
#pragma unroll
        for (int r = 0; r < EPQ * VPE; r += 4)
          *(f32x4w*)((float*)dst + r) = f32x4{w[r], w[r + 1], w[r + 2], w[r + 3]};
      } else {
#pragma unroll
        for (int h = 0; h < EPQ; ++h)
          if (e0 + h < a.m) {
            if constexpr (FORM == RS_RR) dst[h * P] = w[h];
            else dst[h * P] = f32x2{w[2 * h], w[2 * h + 1]};
          }
      }
    }
  }
  if constexpr (F16) {
    // running bound of the results (mode_tile.h): waves meet in LDS, one
    // atomic per workgroup
    uint32_t mb = __float_as_uint(vmax);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mb = max(mb, (uint32_t)__shfl_xor((int)mb, o));
    __syncthreads();
    uint32_t* wmx = (uint32_t*)lds;
    if (lane == 0) wmx[wave] = mb;
    __syncthreads();
    if (tid == 0) {
      uint32_t m = 0;
      for (int w = 0; w < nthr / 64; ++w) m = max(m, wmx[w]);
      atomicMax(a.smax_out + (int)(tile % SMAX_WORDS) * SMAX_STRIDE, m);
    }
  }
}

}  // namespace mm
