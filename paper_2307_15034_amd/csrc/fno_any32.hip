// Truncated transforms of fp32 planes of any extents (Nb >= 8, up to 64
// last-axis and 128 leading-axis modes), v_mfma_f32_16x16x4_f32.
//
// As plain DFT products the fp32 transforms would be bound by the matrix cores
// (157 TFLOP/s: 128 x 128 with 32 x 32 modes, 2048 planes, 55 us of them against
// 33 us of memory traffic), so an even axis is folded first:
// e^{-2 pi i k (n + N/2) / N} = (-1)^k e^{-2 pi i k n / N}, so even
// frequencies need only u[n] + u[n + N/2] and odd ones only their difference,
// over half the length (radix 2, in fp32).  FB folds the last axis (modes
// in the order even, odd), FA the leading one: a wave's two row tiles are then
// rows r and r + Na/2.  Odd axes are taken whole.
//
// As in the fp16 kernels for any extents, the last axis goes in segments of 64
// (32 with more than 32 modes) columns of one table held in LDS, the accumulators
// (in the inverse the rows of V) rotated in fp32 between segments; 1 to 8 waves
// share a plane, and a plane's rows are shared by several work-groups where
// planes are few.  A wave's next segment is in flight while one is multiplied.
//
// 2048 planes of 128 x 128, 32 x 32 modes: forward 130 -> 70 us, inverse 125 ->
// 64 us against the generic kernels (tables from L2, no radix 2, nothing in
// flight); 32 planes of 512 x 512, 42 x 35 modes: 478 -> 57 and 436 -> 57 us.
// Folded, neither limit is reached alone: the matrix cores are busy 36 and 37% of
// the time (61 and 67 TFLOP/s) at 2.4 and 3.0 TB/s, and the waves wait for a
// quarter and two fifths of theirs: the two steps of a plane follow one another,
// with one work-group on a compute unit.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "fno_device.h"
#include "fno_routes.h"

namespace fno {

namespace {

typedef MM<float> MF;
constexpr int F3_NW = 8;  // waves per work-group

__device__ __forceinline__ f4 as_f4(const u32x4& v) {
  f4 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

// the four values of v moved down by t (1..3, the same on every lane)
__device__ __forceinline__ f4 shift_down4(const f4& v, int t) {
  f4 r = {t == 1 ? v[1] : t == 2 ? v[2] : v[3], t == 1 ? v[2] : t == 2 ? v[3] : 0.0f,
          t == 1 ? v[3] : 0.0f, 0.0f};
  return r;
}

__device__ __forceinline__ void sync_group(int wpp) {
  if (wpp > 1) __syncthreads();
  else wave_lds_sync();
}

size_t f3_r2c_lds(int nct, int lw) {
  const int kbp = nct * 8;
  return (size_t)2 * kbp * (any32_nf(kbp) + 4) * 4 +
         (size_t)(F3_NW >> lw) * 2 * kbp * ((32 << lw) + 4) * 4;
}

size_t f3_c2r_lds(int nct, int lw, int kap) {
  const int kbp = nct * 8;
  return (size_t)any32_nf(kbp) * (2 * kbp + 4) * 4 + (size_t)kbp * 8 +
         (size_t)(F3_NW >> lw) * 2 * kbp * (kap + 4) * 4;
}

}  // namespace

// ---------------------------------------------------------------------------
// Forward.  a.twS [2 Kbp][64], a.segph [Kbp] (modes in tile order), a.cB and
// a.sB [Kap16][Nap] (slots in tile order, zero past the rows).
// ---------------------------------------------------------------------------
template <int NCT, bool FA, bool FB>
__global__ __launch_bounds__(F3_NW * 64, 2) void r2c_any32_kernel(R2CArgs a) {
  constexpr int NW = F3_NW, KBP = NCT * 8, NTB = NCT / 2, NTBC = FB ? NTB / 2 : NTB;
  constexpr int NL = FB ? 2 : 1, RB = FA ? 16 : 32;
  constexpr int F3_NF = any32_nf(KBP), F3_NK = F3_NF / 16, F3_LDT = F3_NF + 4;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int wpp = 1 << a.lw, grp = wave >> a.lw, j = wave & (wpp - 1), ngrp = NW >> a.lw;
  const int LDY = wpp * 32 + 4;
  float* sT = reinterpret_cast<float*>(smem);
  float* sY = sT + 2 * KBP * F3_LDT + grp * (2 * KBP * LDY);
  float* sE = sT + 2 * KBP * F3_LDT + ngrp * (2 * KBP * LDY);  // step-B tables (tab_lds)
  const int LDE = a.Nap + 4;

  const int Nh = FB ? a.Nb / 2 : a.Nb, NhA = FA ? a.Na / 2 : a.Na;
  const int nblk = (NhA + RB - 1) / RB, nseg = (Nh + F3_NF - 1) / F3_NF;
  const int nch = (nblk + wpp - 1) >> a.lw;
  const int cpp = (nch + a.parts - 1) / a.parts;  // chunks of this work-group (a.parts > 1)
  const int ch0 = (int)(blockIdx.x % a.parts) * cpp, ch1 = min(nch, ch0 + cpp);
  const int tail = Nh & 3;
  const int64_t plane_bytes = (int64_t)a.Na * a.Nb * 4;
  const int64_t step = (int64_t)(gridDim.x / a.parts) * ngrp;
  const int64_t trips = (a.planes + step - 1) / step;
  auto plane_of = [&](int64_t t) { return (int64_t)(blockIdx.x / a.parts) * ngrp + t * step + grp; };

  // k-step k of segment sg: lane holds row (tile u), columns h Nh + 64 sg +
  // 16 k + 4 g .. + 4
  struct Rows {
    __amdgpu_buffer_rsrc_t rs;
    int ro;
  };
  const int ustep = (FA ? NhA : 16) * a.Nb * 4;
  auto rows_of = [&](int64_t p, int b) {
    const bool ok = p < a.planes && b < nblk;
    const PlaneRef pr = plane_ref_at(a.in, ok ? p * plane_bytes : 0, ok ? plane_bytes : 0);
    const int row = RB * b + r16;
    return Rows{pr.rs, (row < NhA ? row * a.Nb * 4 : PLANE_OOB) + pr.off};
  };
  auto load = [&](const Rows& r, int sg, int k, u32x4 (&v)[F3_NK][2][NL]) {
    const int col = sg * F3_NF + k * 16 + g * 4;
    const int co = col + 4 <= Nh ? col * 4 : (col < Nh ? (Nh - 4) * 4 : PLANE_OOB / 2);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int h = 0; h < NL; ++h)
        v[k][u][h] = __builtin_amdgcn_raw_buffer_load_b128(r.rs, r.ro + co + u * ustep + h * Nh * 4,
                                                           0, 0);
  };
  u32x4 nxt[F3_NK][2][NL];
  {
    const Rows r = rows_of(plane_of(0), ch0 * wpp + j);
#pragma unroll
    for (int k = 0; k < F3_NK; ++k) load(r, nseg - 1, k, nxt);
  }
  stage_pieces<NW * 64, 2>(
      2 * KBP * (F3_NF / 4), [&](int i) { return reinterpret_cast<const u32x4*>(a.twS) + i; },
      [&](int i) {
        return reinterpret_cast<u32x4*>(sT + i / (F3_NF / 4) * F3_LDT + (i % (F3_NF / 4)) * 4);
      });
  if (a.tab_lds) {
    const int cpr = a.Nap / 4, n = a.Kap16 * cpr;  // both tables: rows r, Kap16 + r
    stage_pieces<NW * 64, 8>(
        2 * n,
        [&](int i) { return reinterpret_cast<const u32x4*>(i < n ? a.cB : a.sB) + (i < n ? i : i - n); },
        [&](int i) { return reinterpret_cast<u32x4*>(sE + i / cpr * LDE + (i % cpr) * 4); });
  }
  f2 om[NTB];
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) om[tb] = reinterpret_cast<const f2*>(a.segph)[tb * 16 + r16];
  __syncthreads();

  // step B as in the fp16 kernel: spectrum row tiles ta = j % q + q i, column
  // tiles tb0 + tbs * jj; several chunks only with all waves on one plane
  const int nta = a.Kap16 >> 4;
  int ntap = 1;
  while (ntap < nta) ntap *= 2;
  const int q = min(wpp, ntap), tb0 = j / q, tbs = wpp / q;
  f4 zr[NTB], zi[NTB];

  for (int64_t t = 0; t < trips; ++t) {
    const int64_t p = plane_of(t);
    const int64_t pn = t + 1 < trips ? plane_of(t + 1) : a.planes;
#pragma nounroll
    for (int ch = ch0; ch < ch1; ++ch) {
      const int b = ch * wpp + j;
      f4 acc[2][NCT];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) acc[u][ct] = f4zero();
#pragma nounroll
      for (int sg = nseg - 1; sg >= 0; --sg) {
        if (sg < nseg - 1) {
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) rotate(acc[u][tb], acc[u][NTB + tb], om[tb]);
        }
        const int ktail = tail && sg == nseg - 1 ? (Nh - sg * F3_NF) / 16 : -1;
        const bool same = sg > 0, chn = ch + 1 < ch1;
        const Rows rn = rows_of(same || chn ? p : pn, same ? b : (chn ? b + wpp : ch0 * wpp + j));
        const int sn = same ? sg - 1 : nseg - 1;
#pragma unroll
        for (int k = 0; k < F3_NK; ++k) {
          f4 x[2][NL], af[2][NL];
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < NL; ++h) {
              x[u][h] = as_f4(nxt[k][u][h]);
              if (k == ktail) {
                const f4 v = shift_down4(x[u][h], 4 - tail);
                const bool part = g == (Nh & 15) / 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[u][h][e] = part ? v[e] : x[u][h][e];
              }
            }
          load(rn, sn, k, nxt);
          if (a.act) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int h = 0; h < NL; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[u][h][e] = preact_f32(x[u][h][e], a.act, a.clip);
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            if constexpr (FB) {
              af[u][0] = x[u][0] + x[u][1];
              af[u][1] = x[u][0] - x[u][1];
            } else {
              af[u][0] = x[u][0];
            }
          }
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) {
            const int cls = (ct % NTB) / NTBC;
            const f4 bf = MF::ld(sT + (ct * 16 + r16) * F3_LDT + k * 16 + g * 4);
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u][ct] = MF::mma(af[u][cls], bf, acc[u][ct]);
          }
          __builtin_amdgcn_sched_barrier(0);  // bound the hoisting of LDS reads (registers)
        }
      }
      // columns of Y: FA the sums of rows r and r + Na/2, then the differences
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        float* d = sY + (ct * 16 + r16) * LDY + 4 * g;
        const f4 y0 = acc[0][ct] * a.scaleA, y1 = acc[1][ct] * a.scaleA;
        if (FA) {
          *reinterpret_cast<f4*>(d + j * 16) = y0 + y1;
          *reinterpret_cast<f4*>(d + wpp * 16 + j * 16) = y0 - y1;
        } else {
          *reinterpret_cast<f4*>(d + j * 32) = y0;
          *reinterpret_cast<f4*>(d + j * 32 + 16) = y1;
        }
      }
      sync_group(wpp);

      const int nb = min(wpp, nblk - ch * wpp);
      // ct, st: the row tile's rows of the tables
      auto row_tile = [&](int ta, const float* ct, const float* st, f4 (&ar_)[NTB], f4 (&ai_)[NTB]) {
        const int ca = FA && 2 * ta >= nta ? wpp * 16 : 0;  // differences: odd slots
        const float* y = sY + r16 * LDY + ca + g * 4;
        for (int ks = 0; ks < nb * (RB / 16); ++ks) {
          const f4 cf = MF::ld(ct + ks * 16), sf = MF::ld(st + ks * 16);
          const f4 nsf = MF::neg(sf);
#pragma unroll
          for (int jj = 0; jj < NTB; ++jj) {
            const int tb = tb0 + jj * tbs;
            if (tb >= NTB) break;
            const f4 yr = MF::ld(y + tb * 16 * LDY + ks * 16);
            const f4 yi = MF::ld(y + (KBP + tb * 16) * LDY + ks * 16);
            ar_[jj] = MF::mma(cf, yr, ar_[jj]);
            ar_[jj] = MF::mma(sf, yi, ar_[jj]);
            ai_[jj] = MF::mma(cf, yi, ai_[jj]);
            ai_[jj] = MF::mma(nsf, yr, ai_[jj]);
          }
        }
      };
      auto store = [&](int ta, const f4 (&ar_)[NTB], const f4 (&ai_)[NTB]) {
        if (p >= a.planes) return;
        const bool sums = a.parts > 1;  // this part's sums, to be added in order
        f2* out = sums ? reinterpret_cast<f2*>(a.part) + (int64_t)blockIdx.x * a.Ka * a.Kb
                       : reinterpret_cast<f2*>(a.out) + p * (int64_t)a.Ka * a.Kb;
        const float sc = sums ? 1.0f : a.scaleB;
#pragma unroll
        for (int jj = 0; jj < NTB; ++jj) {
          const int tb = tb0 + jj * tbs;
          const int t_b = FB ? 2 * (tb % NTBC * 16 + r16) + tb / NTBC : tb * 16 + r16;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int s = ta * 16 + 4 * g + i, nsl = a.Kap16 / 2;
            const int t_a = FA ? 2 * (s < nsl ? s : s - nsl) + (s < nsl ? 0 : 1) : s;
            if (tb < NTB && t_a < a.Ka && t_b < a.Kb)
              out[t_a * a.Kb + t_b] = f2{ar_[jj][i] * sc, ai_[jj][i] * sc};
          }
        }
      };
      // (planes of several chunks: all eight waves, one row tile each at most)
      for (int ta = j % q; ta < nta; ta += q) {
        if (ch == ch0) {
#pragma unroll
          for (int jj = 0; jj < NTB; ++jj) zr[jj] = zi[jj] = f4zero();
        }
        const int er = ta * 16 + r16, eo = ch * wpp * RB + g * 4;
        if (a.tab_lds) {
          const float* e = sE + er * LDE + eo;
          row_tile(ta, e, e + a.Kap16 * LDE, zr, zi);
        } else {
          const int64_t o = (int64_t)er * a.Nap + eo;
          row_tile(ta, reinterpret_cast<const float*>(a.cB) + o,
                   reinterpret_cast<const float*>(a.sB) + o, zr, zi);
        }
        if (ch == ch1 - 1) store(ta, zr, zi);
      }
      sync_group(wpp);  // Y read before the next chunk's
    }
  }
}

// ---------------------------------------------------------------------------
// Inverse.  a.twS [64][2 Kbp] (row m: cos, then -sin, modes in tile order),
// a.cI and a.sI [rows][Kap] (slots in class order: FA even ones, then odd).
// V(r) = E + O and V(r + Na/2) = E - O, then y[m] = e + o and y[m + Nb/2] = e - o.
// The D registers of step B' (four consecutive modes of a row) are the B
// operand of step A' as they are.
// ---------------------------------------------------------------------------
template <int NCT, bool FA, bool FB>
__global__ __launch_bounds__(F3_NW * 64, 2) void c2r_any32_kernel(C2RArgs a) {
  constexpr int NW = F3_NW, KBP = NCT * 8, NTB = NCT / 2, NTBC = FB ? NTB / 2 : NTB;
  constexpr int NL = FB ? 2 : 1, RB = FA ? 16 : 32, LDT = 2 * KBP + 4;
  constexpr int F3_NF = any32_nf(KBP);
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int wpp = 1 << a.lw, grp = wave >> a.lw, j = wave & (wpp - 1), ngrp = NW >> a.lw;
  const int LDZ = a.Kap + 4, Kah = FA ? a.Kap / 2 : a.Kap;
  float* sT = reinterpret_cast<float*>(smem);         // [64][LDT]
  f2* sW = reinterpret_cast<f2*>(sT + F3_NF * LDT);   // [KBP] segment phases
  float* zt = reinterpret_cast<float*>(sW + KBP) + grp * (2 * KBP * LDZ);  // [2 KBP][LDZ]
  float* sE = reinterpret_cast<float*>(sW + KBP) + ngrp * (2 * KBP * LDZ);  // (tab_lds)
  const int LDE = a.Kap + 4;

  const int Nh = FB ? a.Nb / 2 : a.Nb, NhA = FA ? a.Na / 2 : a.Na;
  const int nblk = (NhA + RB - 1) / RB, nseg = (Nh + F3_NF - 1) / F3_NF;
  const int bpp = ((nblk + wpp - 1) / wpp + a.parts - 1) / a.parts * wpp;
  const int b0 = (int)(blockIdx.x % a.parts) * bpp, b1 = min(nblk, b0 + bpp);
  const int64_t plane = (int64_t)a.Na * a.Nb;
  const int spec = a.Ka * a.Kb;
  const int gt = tid - grp * wpp * 64, gn = wpp * 64;
  const int64_t step = (int64_t)(gridDim.x / a.parts) * ngrp;
  const int64_t trips = (a.planes + step - 1) / step;
  auto plane_of = [&](int64_t t) { return (int64_t)(blockIdx.x / a.parts) * ngrp + t * step + grp; };

  // spectrum of plane p into zt[mode | KBP + mode][slot], in tile order; the
  // padding stays zero
  constexpr int ZQ = 8;  // values of the next spectrum in flight per thread
  auto ldz = [&](int64_t p, f2 (&v)[ZQ]) {
    const f2* z = reinterpret_cast<const f2*>(a.in) + (p < a.planes ? p : 0) * spec;
#pragma unroll
    for (int e = 0; e < ZQ; ++e) v[e] = z[min(gt + e * gn, spec - 1)];
  };
  auto put = [&](int i, const f2& v) {
    const int ta = i / a.Kb, tb = i - ta * a.Kb;
    const int row = FB ? (tb & 1) * NTBC * 16 + (tb >> 1) : tb;
    const int col = FA ? (ta & 1) * Kah + (ta >> 1) : ta;
    zt[row * LDZ + col] = v[0];
    zt[(KBP + row) * LDZ + col] = v[1];
  };
  auto stz = [&](int64_t p, const f2 (&v)[ZQ]) {
    if (p >= a.planes) return;
#pragma unroll
    for (int e = 0; e < ZQ; ++e)
      if (gt + e * gn < spec) put(gt + e * gn, v[e]);
    const f2* z = reinterpret_cast<const f2*>(a.in) + p * spec;
    for (int i = gt + ZQ * gn; i < spec; i += gn) put(i, z[i]);
  };

  f2 zn[ZQ];
  ldz(plane_of(0), zn);
  stage_pieces<NW * 64, 2>(
      F3_NF * (2 * KBP / 4), [&](int i) { return reinterpret_cast<const u32x4*>(a.twS) + i; },
      [&](int i) {
        return reinterpret_cast<u32x4*>(sT + i / (2 * KBP / 4) * LDT + (i % (2 * KBP / 4)) * 4);
      });
  for (int i = tid; i < KBP; i += NW * 64) sW[i] = reinterpret_cast<const f2*>(a.segph)[i];
  if (a.tab_lds) {
    const int cpr = a.Kap / 4, n = NhA * cpr;  // both tables: rows r, NhA + r
    stage_pieces<NW * 64, 8>(
        2 * n,
        [&](int i) { return reinterpret_cast<const u32x4*>(i < n ? a.cI : a.sI) + (i < n ? i : i - n); },
        [&](int i) { return reinterpret_cast<u32x4*>(sE + i / cpr * LDE + (i % cpr) * 4); });
  }
  for (int i = gt; i < 2 * KBP * LDZ / 4; i += gn)
    reinterpret_cast<u32x4*>(zt)[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  stz(plane_of(0), zn);
  __syncthreads();

  for (int64_t t = 0; t < trips; ++t) {
    const int64_t p = plane_of(t);
    const int64_t pn = t + 1 < trips ? plane_of(t + 1) : a.planes;
    ldz(pn, zn);
    float* y = reinterpret_cast<float*>(a.out) + (p < a.planes ? p : 0) * plane;
    const float* x = a.epilogue ? reinterpret_cast<const float*>(a.x) + (p < a.planes ? p : 0) * plane
                                : nullptr;
#pragma nounroll
    for (int b = b0 + j; b < b1; b += wpp) {
      // ---- step B' ----
      f4 vr[2][NTB], vi[2][NTB];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) vr[u][tb] = vi[u][tb] = f4zero();
      for (int k = 0; k < Kah; k += 16) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          // FA: u is the slot class; otherwise the row tile
          const int row = min(RB * b + (FA ? 0 : 16 * u) + r16, NhA - 1);
          const int co = (FA ? u * Kah : 0) + k + g * 4;
          f4 cf, sf;
          if (a.tab_lds) {
            cf = MF::ld(sE + row * LDE + co);
            sf = MF::ld(sE + (NhA + row) * LDE + co);
          } else {
            cf = MF::ld(reinterpret_cast<const float*>(a.cI) + (int64_t)row * a.Kap + co);
            sf = MF::ld(reinterpret_cast<const float*>(a.sI) + (int64_t)row * a.Kap + co);
          }
          const f4 nsf = MF::neg(sf);
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) {
            const f4 zr = MF::ld(zt + (tb * 16 + r16) * LDZ + co);
            const f4 zi = MF::ld(zt + (KBP + tb * 16 + r16) * LDZ + co);
            vr[u][tb] = MF::mma(zr, cf, vr[u][tb]);
            vr[u][tb] = MF::mma(zi, nsf, vr[u][tb]);
            vi[u][tb] = MF::mma(zr, sf, vi[u][tb]);
            vi[u][tb] = MF::mma(zi, cf, vi[u][tb]);
          }
        }
      }
      if (FA) {
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
          const f4 er = vr[0][tb], ei = vi[0][tb];
          vr[0][tb] = er + vr[1][tb];
          vi[0][tb] = ei + vi[1][tb];
          vr[1][tb] = er - vr[1][tb];
          vi[1][tb] = ei - vi[1][tb];
        }
      }
      // ---- step A', segment by segment ----
#pragma nounroll
      for (int sg = 0; sg < nseg; ++sg) {
        if (sg > 0) {
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) {
            const f4* w = reinterpret_cast<const f4*>(sW + tb * 16 + 4 * g);
            const f4 w0 = w[0], w1 = w[1];
            const f4 oc = {w0[0], w0[2], w1[0], w1[2]}, os = {w0[1], w0[3], w1[1], w1[3]};
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const float re = vr[u][tb][i], im = vi[u][tb][i];
                vr[u][tb][i] = fmaf(-im, os[i], re * oc[i]);
                vi[u][tb][i] = fmaf(re, os[i], im * oc[i]);
              }
          }
        }
#pragma unroll
        for (int c = 0; c < F3_NF / 16; ++c) {
          const int m = sg * F3_NF + c * 16 + 4 * g;  // this lane's first column
          if (sg * F3_NF + c * 16 >= Nh) break;
          f4 acc[2][NL];
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < NL; ++h) acc[u][h] = f4zero();
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) {
            const float* tp = sT + (c * 16 + r16) * LDT + tb * 16 + 4 * g;
            const f4 tc = MF::ld(tp), ts = MF::ld(tp + KBP);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              acc[u][tb / NTBC] = MF::mma(tc, vr[u][tb], acc[u][tb / NTBC]);
              acc[u][tb / NTBC] = MF::mma(ts, vi[u][tb], acc[u][tb / NTBC]);
            }
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int rr = RB * b + (FA ? 0 : 16 * u) + r16;
            if (rr >= NhA || m >= Nh || p >= a.planes) continue;
            const int64_t row = (int64_t)(rr + (FA ? u * NhA : 0)) * a.Nb;
#pragma unroll
            for (int h = 0; h < NL; ++h) {
              f4 v = !FB ? acc[u][0] : h == 0 ? acc[u][0] + acc[u][NL - 1] : acc[u][0] - acc[u][NL - 1];
              v = v * a.scale;
              const int64_t o = row + h * Nh + m;
              if (m + 4 <= Nh) {
                if (a.epilogue) {
                  f4 xv;
                  __builtin_memcpy(&xv, __builtin_assume_aligned(x + o, 4), 16);
#pragma unroll
                  for (int e = 0; e < 4; ++e) v[e] *= preact_grad_f32(xv[e], a.act, a.clip);
                }
                __builtin_memcpy(__builtin_assume_aligned(y + o, 4), &v, 16);
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (m + e < Nh)
                    y[o + e] = v[e] * (a.epilogue ? preact_grad_f32(x[o + e], a.act, a.clip) : 1.0f);
              }
            }
          }
        }
      }
    }
    sync_group(wpp);  // every wave is done with this spectrum
    stz(pn, zn);
    sync_group(wpp);
  }
}

// Spectrum of plane p from its parts' sums, as launch_part_sum in fp16.
__global__ __launch_bounds__(256) void part_sum32_kernel(const f2* part, f2* out, int parts,
                                                         int64_t K, int64_t n, float scale) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t p = i / K, k = i - p * K;
  const f2* src = part + p * parts * K + k;
  f2 v = src[0];
  for (int s = 1; s < parts; ++s) v += src[s * K];
  out[i] = v * scale;
}

hipError_t launch_part_sum32(const void* part, void* out, int parts, int64_t planes, int64_t K,
                             float scale, hipStream_t s) {
  const int64_t n = planes * K;
  hipLaunchKernelGGL(part_sum32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const f2*>(part), reinterpret_cast<f2*>(out), parts, K, n,
                     scale);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// blocks of 32 rows (16 pairs of folded ones) of a plane
static int f3_blocks(int Na, bool fold) { return fold ? (Na / 2 + 15) / 16 : (Na + 31) / 32; }

#define FNO_F3_DISPATCH(KERN, NCTV)                                                       \
  switch ((a.foldA ? 2 : 0) + (a.foldB ? 1 : 0)) {                                        \
    case 0: return go(KERN<NCTV, false, false>);                                          \
    case 1: return go(KERN<NCTV, false, true>);                                           \
    case 2: return go(KERN<NCTV, true, false>);                                           \
    default: return go(KERN<NCTV, true, true>);                                           \
  }

hipError_t launch_r2c_any32(const R2CArgs& a_in, int nct, int num_cu, hipStream_t s) {
  R2CArgs a = a_in;
  if (a.Nb < 8 || (int64_t)a.Na * a.Nb * 4 >= (PLANE_OOB >> 1) || a.Kap16 > 128)
    return hipErrorNotSupported;
  a.lw = share_waves_log2(f3_blocks(a.Na, a.foldA), a.planes, num_cu);
  while (a.lw < 3 && f3_r2c_lds(nct, a.lw) > 160 * 1024) ++a.lw;
  size_t lds = f3_r2c_lds(nct, a.lw);
  if (lds > 160 * 1024) return hipErrorNotSupported;
  const size_t tab = (size_t)2 * a.Kap16 * (a.Nap + 4) * 4;
  a.tab_lds = lds + tab <= 160 * 1024;
  if (a.tab_lds) lds += tab;
  const int64_t ngrp = F3_NW >> a.lw;
  const int per_cu = lds <= 80 * 1024 ? 2 : 1;
  const int grid = a.parts > 1 ? (int)(a.planes * a.parts)
                               : (int)std::min<int64_t>((a.planes + ngrp - 1) / ngrp,
                                                        (int64_t)per_cu * num_cu);
  if (a.parts > 1 && ngrp != 1) return hipErrorNotSupported;
  auto go = [&](void (*k)(R2CArgs)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(grid), dim3(F3_NW * 64), lds, s, a);
    return hipGetLastError();
  };
  if (nct == 2 && !a.foldB) return a.foldA ? go(r2c_any32_kernel<2, true, false>)
                                           : go(r2c_any32_kernel<2, false, false>);
  if (nct == 4) FNO_F3_DISPATCH(r2c_any32_kernel, 4)
  if (nct == 8) FNO_F3_DISPATCH(r2c_any32_kernel, 8)
  return hipErrorNotSupported;
}

hipError_t launch_c2r_any32(const C2RArgs& a_in, int nct, int num_cu, hipStream_t s) {
  C2RArgs a = a_in;
  if (a.Nb < 8 || (int64_t)a.Na * a.Nb * 4 >= (PLANE_OOB >> 1) || a.Kap > 128)
    return hipErrorNotSupported;
  a.lw = share_waves_log2(f3_blocks(a.Na, a.foldA), a.planes, num_cu);
  while (a.lw < 3 && f3_c2r_lds(nct, a.lw, a.Kap) > 160 * 1024) ++a.lw;
  size_t lds = f3_c2r_lds(nct, a.lw, a.Kap);
  if (lds > 160 * 1024) return hipErrorNotSupported;
  const size_t tab = (size_t)2 * (a.foldA ? a.Na / 2 : a.Na) * (a.Kap + 4) * 4;
  a.tab_lds = lds + tab <= 160 * 1024;
  if (a.tab_lds) lds += tab;
  const int64_t ngrp = F3_NW >> a.lw;
  const int per_cu = lds <= 80 * 1024 ? 2 : 1;
  if (a.parts > 1 && ngrp != 1) return hipErrorNotSupported;
  const int grid = a.parts > 1 ? (int)(a.planes * a.parts)
                               : (int)std::min<int64_t>((a.planes + ngrp - 1) / ngrp,
                                                        (int64_t)per_cu * num_cu);
  auto go = [&](void (*k)(C2RArgs)) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(grid), dim3(F3_NW * 64), lds, s, a);
    return hipGetLastError();
  };
  if (nct == 2 && !a.foldB) return a.foldA ? go(c2r_any32_kernel<2, true, false>)
                                           : go(c2r_any32_kernel<2, false, false>);
  if (nct == 4) FNO_F3_DISPATCH(c2r_any32_kernel, 4)
  if (nct == 8) FNO_F3_DISPATCH(c2r_any32_kernel, 8)
  return hipErrorNotSupported;
}
#undef FNO_F3_DISPATCH

}  // namespace fno
