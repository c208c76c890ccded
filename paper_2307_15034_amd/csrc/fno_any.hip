// Truncated transforms of fp16 planes of any extents (Nb >= 8, up to 64
// last-axis and 128 leading-axis modes): odd and ragged grids, row lengths
// that are not a multiple of eight or of a tile, mode counts that are not a
// multiple of four.
//
// Both axes are DFT-by-MFMA products over the retained modes, as in the
// other plane kernels.  What is particular here:
//   - the last axis is taken in segments of NF = 128 (64) columns.  With
//     n = NF s + m, e^{-2 pi i k n / Nb} = w_k^s e^{-2 pi i k m / Nb},
//     w_k = e^{-2 pi i k NF / Nb}, so one table of NF columns, held in LDS
//     for the whole kernel, serves every row length; the accumulators are
//     rotated by w_k in fp32 between segments (Horner, last segment first),
//     so nothing is rounded that a single long product would not round.  No
//     twiddle is loaded again and no barrier is needed inside the product.
//   - rows may start at any two-byte address (16-byte accesses at their own
//     alignment); the last partial eight of a row are read from Nb - 8 on and
//     shifted down.
//   - a wave takes 32 rows at a time; 1, 2, 4 or 8 waves share a plane, so
//     small planes keep all eight waves of a work-group busy.
// The next segment of a wave's rows (the next unit of x in the inverse) is in
// flight while one is multiplied.  512 planes of 241 x 241, 40 x 20 modes: forward
// 25 us, with tanh 28, inverse 28, with tanh' 45, at 2.5 to 3.8 TB/s of traffic
// (reads of such rows alone run at 4.2); the matrix cores are busy 5 to 8% of the
// time, so what is left is the latency of the rows and the table lookups and
// exponentials of tanh and tanh' (waits 38 to 45% of the waves' cycles, vector
// instructions 17 to 28% with them against 6 to 18 without).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "fno_device.h"
#include "fno_routes.h"

namespace fno {

namespace {

typedef MM<_Float16> MH;
constexpr int AN_NW = 8;    // waves per work-group
constexpr int AN_LDO = 72;  // inverse: staging row stride (fp16; fp32 with the epilogue)

// LDS bytes of the inverse's staging rows of one wave
constexpr size_t an_ob_bytes(bool epi) { return (size_t)16 * AN_LDO * (epi ? 4 : 2); }

__device__ __forceinline__ void group_sync(int wpp) {
  if (wpp > 1) __syncthreads();
  else wave_lds_sync();
}

size_t any_r2c_lds(int nct, int nk, int lw, bool pre, int sat) {
  const int kbp = nct * 8, wpp = 1 << lw;
  return (pre ? (size_t)lutn_bytes(sat) : 0) + (size_t)2 * kbp * (nk * 32 + 8) * 2 +
         (size_t)(AN_NW >> lw) * 2 * kbp * (wpp * 32 + 8) * 2;
}

size_t any_c2r_lds(int nct, int nk, int lw, int kap, bool epi) {
  const int kbp = nct * 8;
  return (size_t)nk * 32 * (2 * kbp + 8) * 2 + (size_t)kbp * 8 + (size_t)(AN_NW >> lw) * 2 * 2 * kbp * (kap + 8) * 2 +
         AN_NW * an_ob_bytes(epi);
}

}  // namespace

// ---------------------------------------------------------------------------
// Forward: plane [Na][Nb] -> spectrum [Ka][Kb].
// ---------------------------------------------------------------------------
template <int NCT, int NK, bool PRE, bool SHARE>
__global__ __launch_bounds__(AN_NW * 64, NCT <= 4 ? 4 : 2) void r2c_any_kernel(R2CArgs a) {
  constexpr int KBP = NCT * 8, NTB = NCT / 2, NF = NK * 32, LDT = NF + 8;
  extern __shared__ __align__(16) unsigned char smem[];  // the table at LDS byte 0
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int wpp = 1 << a.lw, grp = wave >> a.lw, j = wave & (wpp - 1), ngrp = AN_NW >> a.lw;
  const int LDY = wpp * 32 + 8;
  _Float16* lut = reinterpret_cast<_Float16*>(smem);
  _Float16* sT = reinterpret_cast<_Float16*>(smem + (PRE ? lutn_bytes(a.lut_sat) : 0));
  _Float16* sY = sT + 2 * KBP * LDT + grp * (2 * KBP * LDY);  // [2 KBP][LDY] of this plane
  _Float16* sE = sT + 2 * KBP * LDT + ngrp * (2 * KBP * LDY); // step-B tables (tab_lds)
  const int LDE = a.NaC + 8;
  const uint32_t s2 = (uint32_t)a.lut_sat * 2u * 0x10001u;

  const int nblk = (a.Na + 31) / 32, nseg = (a.Nb + NF - 1) / NF;
  const int nch = (nblk + wpp - 1) >> a.lw;  // chunks of a plane (1 unless wpp is 8)
  // SHARE: the chunks of a plane are shared by a.parts work-groups, which have
  // one plane each (too few planes): this one's chunks
  const int parts = SHARE ? a.parts : 1;
  const int cpp = (nch + parts - 1) / parts;
  const int part = SHARE ? (int)(blockIdx.x % parts) : 0;
  const int ch0 = part * cpp, ch1 = SHARE ? min(nch, ch0 + cpp) : nch;
  const int tail = a.Nb & 7;
  const int64_t plane_bytes = (int64_t)a.Na * a.Nb * 2;
  const int64_t trips =
      SHARE ? 1
            : (a.planes + (int64_t)gridDim.x * ngrp - 1) / ((int64_t)gridDim.x * ngrp);
  auto plane_of = [&](int64_t t) {
    return SHARE ? (int64_t)(blockIdx.x / parts)
                 : ((int64_t)blockIdx.x + t * gridDim.x) * ngrp + grp;
  };

  // k-step k of segment sg of a row block: lane holds rows 32 b + 16 u + r16,
  // columns NF sg + 32 k + 8 g .. + 8
  struct Rows {
    __amdgpu_buffer_rsrc_t rs;
    int ro;
  };
  auto rows_of = [&](int64_t p, int b) {
    const bool ok = p < a.planes && b < nblk;
    const PlaneRef pr = plane_ref_at(a.in, ok ? p * plane_bytes : 0, ok ? plane_bytes : 0);
    return Rows{pr.rs, (32 * b + r16) * a.Nb * 2 + pr.off};
  };
  auto load = [&](const Rows& r, int sg, int k, u32x4 (&v)[2][NK]) {
    const int col = sg * NF + k * 32 + g * 8;
    const int co = col + 8 <= a.Nb ? col * 2 : (col < a.Nb ? (a.Nb - 8) * 2 : PLANE_OOB);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      v[u][k] = __builtin_amdgcn_raw_buffer_load_b128(r.rs, r.ro + co + u * 32 * a.Nb, 0, 0);
  };
  u32x4 nxt[2][NK];
  {
    const Rows r = rows_of(plane_of(0), ch0 * wpp + j);
#pragma unroll
    for (int k = 0; k < NK; ++k) load(r, nseg - 1, k, nxt);
  }

  if (PRE) stage_lutn<AN_NW * 64>(lut, a.lut, a.lut_sat);
  stage_pieces<AN_NW * 64, 2>(
      2 * KBP * (NF / 8), [&](int i) { return reinterpret_cast<const u32x4*>(a.twS) + i; },
      [&](int i) {
        return reinterpret_cast<u32x4*>(sT + i / (NF / 8) * LDT + (i % (NF / 8)) * 8);
      });
  if (a.tab_lds) {
    const int cpr = a.NaC / 8, n = a.Kap16 * cpr;  // both tables: rows r, Kap16 + r
    stage_pieces<AN_NW * 64, 8>(
        2 * n,
        [&](int i) { return reinterpret_cast<const u32x4*>(i < n ? a.cBc : a.sBc) + (i < n ? i : i - n); },
        [&](int i) { return reinterpret_cast<u32x4*>(sE + i / cpr * LDE + (i % cpr) * 8); });
  }
  f2 om[NTB];  // w_k of this lane's modes
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) om[tb] = reinterpret_cast<const f2*>(a.segph)[tb * 16 + r16];
  __syncthreads();

  // step B: wave j of a plane takes spectrum row tiles ta = j % q + q i and
  // column tiles tb0 + tbs * jj.  Planes of several chunks have wpp = 8 and
  // one row tile per wave, whose accumulators carry over the chunks.
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
      // (a wave without a block walks the same segments with empty loads: the
      // waits stay the same on every path)
#pragma nounroll
      for (int sg = nseg - 1; sg >= 0; --sg) {
        if (sg < nseg - 1) {
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int tb = 0; tb < NTB; ++tb) rotate(acc[u][tb], acc[u][NTB + tb], om[tb]);
        }
        // the k-step that holds the row's last partial eight, if there is one
        const int ktail = tail && sg == nseg - 1 ? (a.Nb - sg * NF) / 32 : -1;
        // the next segment (of the next chunk or plane at the end), requested
        // k-step by k-step as this one's registers are used up
        const bool same = sg > 0, chn = ch + 1 < ch1;
        const Rows rn = rows_of(same || chn ? p : pn, same ? b : (chn ? b + wpp : j));
        const int sn = same ? sg - 1 : nseg - 1;
#pragma unroll
        for (int k = 0; k < NK; ++k) {
          h8 af[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            u32x4 w = nxt[u][k];
            if (k == ktail) {
              const bool part = g == (a.Nb & 31) / 8;
              const u32x4 v = shift_down(w, 8 - tail);
#pragma unroll
              for (int e = 0; e < 4; ++e) w[e] = part ? v[e] : w[e];
            }
            if (PRE) lutn_odd4(w, s2);
            af[u] = w_as_h8(w);
          }
          load(rn, sn, k, nxt);
#pragma unroll
          for (int ct = 0; ct < NCT; ++ct) {
            const h8 bf = MH::ld(sT + (ct * 16 + r16) * LDT + k * 32 + g * 8);
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u][ct] = MH::mma(af[u], bf, acc[u][ct]);
          }
          __builtin_amdgcn_sched_barrier(0);  // bound the hoisting of LDS reads (registers)
        }
      }
      // columns of Y, rows in the order of the tables: slots 8 g + e of block
      // j hold rows 4 g + e (e < 4) and 16 + 4 g + e - 4
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) {
        h8 y;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          y[i] = to_h(acc[0][ct][i] * a.scaleA);
          y[4 + i] = to_h(acc[1][ct][i] * a.scaleA);
        }
        *reinterpret_cast<h8*>(sY + (ct * 16 + r16) * LDY + j * 32 + g * 8) = y;
      }
      group_sync(wpp);

      const int nb = min(wpp, nblk - ch * wpp);
      for (int ta = j % q; ta < nta; ta += q) {
        if (ch == ch0) {
#pragma unroll
          for (int jj = 0; jj < NTB; ++jj) zr[jj] = zi[jj] = f4zero();
        }
        const int er = (ta * 16 + r16);
        auto products = [&](int kb, const h8& cf, const h8& sf) {
          const h8 nsf = MH::neg(sf);
#pragma unroll
          for (int jj = 0; jj < NTB; ++jj) {
            const int tb = tb0 + jj * tbs;
            if (tb >= NTB) break;
            const h8 ar = MH::ld(sY + (tb * 16 + r16) * LDY + kb * 32 + g * 8);
            const h8 ai = MH::ld(sY + (KBP + tb * 16 + r16) * LDY + kb * 32 + g * 8);
            zr[jj] = MH::mma(cf, ar, zr[jj]);
            zr[jj] = MH::mma(sf, ai, zr[jj]);
            zi[jj] = MH::mma(cf, ai, zi[jj]);
            zi[jj] = MH::mma(nsf, ar, zi[jj]);
          }
        };
        if (a.tab_lds) {
          for (int kb = 0; kb < nb; ++kb) {
            const _Float16* e = sE + er * LDE + (ch * wpp + kb) * 32 + g * 8;
            products(kb, MH::ld(e), MH::ld(e + a.Kap16 * LDE));
          }
        } else {
          const int64_t eo = (int64_t)er * a.NaC + ch * wpp * 32 + g * 8;
          const _Float16* cb = reinterpret_cast<const _Float16*>(a.cBc) + eo;
          const _Float16* sb = reinterpret_cast<const _Float16*>(a.sBc) + eo;
          for (int kb = 0; kb < nb; ++kb) products(kb, MH::ld(cb + kb * 32), MH::ld(sb + kb * 32));
        }
        if (SHARE && ch == ch1 - 1) {
          // this part's sums, unscaled in fp32, to be added in order
          f2* sum = reinterpret_cast<f2*>(a.part) + (int64_t)blockIdx.x * a.Ka * a.Kb;
#pragma unroll
          for (int jj = 0; jj < NTB; ++jj) {
            const int t_b = (tb0 + jj * tbs) * 16 + r16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int t_a = ta * 16 + 4 * g + i;
              if (t_a < a.Ka && t_b < a.Kb) sum[t_a * a.Kb + t_b] = f2{zr[jj][i], zi[jj][i]};
            }
          }
        } else if (ch == ch1 - 1 && p < a.planes) {
          _Float16* out = reinterpret_cast<_Float16*>(a.out) + p * (int64_t)a.Ka * a.Kb * 2;
#pragma unroll
          for (int jj = 0; jj < NTB; ++jj) {
            const int t_b = (tb0 + jj * tbs) * 16 + r16;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int t_a = ta * 16 + 4 * g + i;
              if (t_a < a.Ka && t_b < a.Kb)
                store_pair<_Float16>(out + ((int64_t)t_a * a.Kb + t_b) * 2, zr[jj][i] * a.scaleB,
                                     zi[jj][i] * a.scaleB);
            }
          }
        }
      }
      group_sync(wpp);  // Y read before the next chunk's
    }
  }
}

// ---------------------------------------------------------------------------
// Inverse: spectrum [Ka][Kb] -> plane [Na][Nb], y = scale * sum Re(Z e^{+i
// theta}), times f'(x) with the epilogue.  A wave takes 32 rows: step B'
// gives V^T[kb][row] in fp32 accumulators, which are rotated by conj(w_k)
// from segment to segment and rounded to fp16 once per segment as the
// operand of step A', whose table rows are permuted so that a lane holds 16
// consecutive outputs of a row.  They pass, 64 columns at a time, through the
// wave's LDS buffer (as fp16, or with the epilogue as fp32) so that eight
// lanes store, and read x of, 128 consecutive bytes of a row.  f' is evaluated
// in fp32.
// ---------------------------------------------------------------------------
template <int NCT, int NK, bool EPI, bool SHARE>
__global__ __launch_bounds__(AN_NW * 64, 2) void c2r_any_kernel(C2RArgs a) {
  constexpr int KBP = NCT * 8, NTB = NCT / 2, NF = NK * 32, NKV = NCT / 2;
  constexpr int LDT = 2 * KBP + 8, NU = NF / 64;
  constexpr int ZQ = 4;  // 16-byte pieces of the next spectrum in flight per thread
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  const int wpp = 1 << a.lw, grp = wave >> a.lw, j = wave & (wpp - 1), ngrp = AN_NW >> a.lw;
  const int LDZ = a.Kap + 8, zsize = 2 * KBP * LDZ;
  _Float16* sT = reinterpret_cast<_Float16*>(smem);             // [NF][LDT]
  f2* sW = reinterpret_cast<f2*>(sT + NF * LDT);                // [KBP] segment phases
  _Float16* sZ = sT + NF * LDT + 4 * KBP;                       // [ngrp][2][2 KBP][LDZ]
  // [16][AN_LDO] of this wave: fp16 results, or fp32 products with the epilogue
  _Float16* ob = sZ + ngrp * 2 * zsize + wave * (an_ob_bytes(EPI) / 2);
  _Float16* sE = sZ + ngrp * 2 * zsize + AN_NW * (an_ob_bytes(EPI) / 2);  // (tab_lds)
  const int LDE = a.Kap + 8;

  const int nblk = (a.Na + 31) / 32, nseg = (a.Nb + NF - 1) / NF;
  const int nkz = a.Kap / 32;
  const int tail = a.Nb & 7;
  const bool nt = a.Nb % 64 == 0;  // rows of whole 128-byte lines
  const int64_t plane_bytes = (int64_t)a.Na * a.Nb * 2;
  const int spec = a.Ka * a.Kb;  // complex values of a spectrum plane
  const int gt = tid - grp * wpp * 64, gn = wpp * 64;  // thread in the group that shares a plane
  // SHARE: the row blocks of a plane are shared by a.parts work-groups, as in
  // the forward: this one's blocks b0 + j + wpp i below b1
  const int parts = SHARE ? a.parts : 1;
  const int bpp = ((nblk + wpp - 1) / wpp + parts - 1) / parts * wpp;
  const int b0 = SHARE ? (int)(blockIdx.x % parts) * bpp : 0;
  const int b1 = SHARE ? min(nblk, b0 + bpp) : nblk;
  const int64_t trips =
      SHARE ? 1
            : (a.planes + (int64_t)gridDim.x * ngrp - 1) / ((int64_t)gridDim.x * ngrp);
  auto plane_of = [&](int64_t t) {
    return SHARE ? (int64_t)(blockIdx.x / parts)
                 : ((int64_t)blockIdx.x + t * gridDim.x) * ngrp + grp;
  };

  // spectrum of plane p, transposed into ZT[kb | KBP + kb][ka]; the padding
  // stays zero (every plane writes the same positions)
  auto ldz1 = [&](const PlaneRef& pr, int i) {
    return __builtin_amdgcn_raw_buffer_load_b128(pr.rs, (4 * i < spec ? i * 16 : PLANE_OOB) + pr.off,
                                                 0, 0);
  };
  auto zref = [&](int64_t p) {
    const bool ok = p < a.planes;
    return plane_ref_at(a.in, ok ? p * spec * 4 : 0, ok ? (int64_t)spec * 4 : 0);
  };
  auto stz1 = [&](_Float16* zt, int i, const u32x4& v) {
    int ka = 4 * i / a.Kb, kb = 4 * i - ka * a.Kb;
    const h8 h = w_as_h8(v);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (4 * i + e < spec) {
        zt[kb * LDZ + ka] = h[2 * e];
        zt[(KBP + kb) * LDZ + ka] = h[2 * e + 1];
      }
      if (++kb == a.Kb) {
        kb = 0;
        ++ka;
      }
    }
  };
  auto ldz = [&](int64_t p, u32x4 (&v)[ZQ]) {
    const PlaneRef pr = zref(p);
#pragma unroll
    for (int e = 0; e < ZQ; ++e) v[e] = ldz1(pr, gt + e * gn);
  };
  auto stz = [&](int64_t p, _Float16* zt, const u32x4 (&v)[ZQ]) {
#pragma unroll
    for (int e = 0; e < ZQ; ++e) stz1(zt, gt + e * gn, v[e]);
    if (4 * ZQ * gn < spec) {  // the rest of a large spectrum of few waves
      const PlaneRef pr = zref(p);
      for (int i = gt + ZQ * gn; 4 * i < spec; i += gn) stz1(zt, i, ldz1(pr, i));
    }
  };

  // x of unit (row block b, columns 64 c) in the row layout of the stores: row
  // lane / 8 + 8 h of row tile u, eight columns at (lane % 8) * 8
  const int nun = (a.Nb + 63) / 64;  // units of a row block
  const int rr = lane >> 3, c8 = (lane & 7) * 8;
  auto ldx = [&](int64_t p, int b, int c, u32x4 (&v)[2][2]) {
    if (!EPI) return;
    const bool ok = p < a.planes && b < nblk;
    const PlaneRef pr = plane_ref_at(a.x, ok ? p * plane_bytes : 0, ok ? plane_bytes : 0);
    const int col = c * 64 + c8;
    const int co = col + 8 <= a.Nb ? col * 2 : (col < a.Nb ? (a.Nb - 8) * 2 : PLANE_OOB);
    const int ro = (32 * b + rr) * a.Nb * 2 + co + pr.off;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        v[u][h] = __builtin_amdgcn_raw_buffer_load_b128(pr.rs, ro + (16 * u + 8 * h) * a.Nb * 2, 0, 0);
  };

  u32x4 zn[ZQ], xn[2][2];
  ldz(plane_of(0), zn);
  ldx(plane_of(0), b0 + j, 0, xn);
  stage_pieces<AN_NW * 64, 2>(
      NF * (2 * KBP / 8), [&](int i) { return reinterpret_cast<const u32x4*>(a.twS) + i; },
      [&](int i) {
        return reinterpret_cast<u32x4*>(sT + i / (2 * KBP / 8) * LDT + (i % (2 * KBP / 8)) * 8);
      });
  if (a.tab_lds) {
    const int cpr = a.Kap / 8, n = a.Na * cpr;  // both tables: rows r, Na + r
    stage_pieces<AN_NW * 64, 8>(
        2 * n,
        [&](int i) { return reinterpret_cast<const u32x4*>(i < n ? a.cI : a.sI) + (i < n ? i : i - n); },
        [&](int i) { return reinterpret_cast<u32x4*>(sE + i / cpr * LDE + (i % cpr) * 8); });
  }
  for (int i = tid; i < ngrp * 2 * zsize / 2; i += AN_NW * 64) reinterpret_cast<u32*>(sZ)[i] = 0;
  for (int i = tid; i < KBP; i += AN_NW * 64) sW[i] = reinterpret_cast<const f2*>(a.segph)[i];
  __syncthreads();  // padding cleared
  stz(plane_of(0), sZ + grp * 2 * zsize, zn);
  __syncthreads();

  for (int64_t t = 0; t < trips; ++t) {
    const int64_t p = plane_of(t);
    const int64_t pn = t + 1 < trips ? plane_of(t + 1) : a.planes;
    const _Float16* zt = sZ + (grp * 2 + (int)(t & 1)) * zsize;
    ldz(pn, zn);
    const PlaneRef py = plane_ref_at(a.out, p < a.planes ? p * plane_bytes : 0,
                                     p < a.planes ? plane_bytes : 0);
#pragma nounroll
    for (int b = b0 + j; b < b1; b += wpp) {
      // ---- step B' ----
      f4 vr[2][NTB], vi[2][NTB];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) vr[u][tb] = vi[u][tb] = f4zero();
      auto products = [&](int k, const h8 (&cf)[2], const h8 (&sf)[2]) {
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
          const h8 zr = MH::ld(zt + (tb * 16 + r16) * LDZ + k * 32 + g * 8);
          const h8 zi = MH::ld(zt + (KBP + tb * 16 + r16) * LDZ + k * 32 + g * 8);
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            vr[u][tb] = MH::mma(zr, cf[u], vr[u][tb]);
            vr[u][tb] = MH::mma(zi, MH::neg(sf[u]), vr[u][tb]);
            vi[u][tb] = MH::mma(zr, sf[u], vi[u][tb]);
            vi[u][tb] = MH::mma(zi, cf[u], vi[u][tb]);
          }
        }
      };
      int row[2];  // rows past the plane are never stored
#pragma unroll
      for (int u = 0; u < 2; ++u) row[u] = min(32 * b + 16 * u + r16, a.Na - 1);
      for (int k = 0; k < nkz; ++k) {
        h8 cf[2], sf[2];
        if (a.tab_lds) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const _Float16* e = sE + row[u] * LDE + k * 32 + g * 8;
            cf[u] = MH::ld(e);
            sf[u] = MH::ld(e + a.Na * LDE);
          }
        } else {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int64_t eo = (int64_t)row[u] * a.Kap + k * 32 + g * 8;
            cf[u] = MH::ld(reinterpret_cast<const _Float16*>(a.cI) + eo);
            sf[u] = MH::ld(reinterpret_cast<const _Float16*>(a.sI) + eo);
          }
        }
        products(k, cf, sf);
      }
      // ---- step A', segment by segment ----
#pragma nounroll
      for (int sg = 0; sg < nseg; ++sg) {
        if (sg > 0) {
          // times conj(w_k) of the modes 16 tb + 4 g + i (read again each
          // time: held in registers they spill)
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
        // k-step ks of step A': tiles 2 ks and 2 ks + 1 of (Re tiles, Im tiles)
        h8 vf[2][NKV];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int ks = 0; ks < NKV; ++ks)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
              const int pi = 2 * ks + hh;
              const f4 src = pi < NTB ? vr[u][pi % NTB] : vi[u][pi % NTB];
#pragma unroll
              for (int i = 0; i < 4; ++i) vf[u][ks][4 * hh + i] = to_h(src[i]);
            }
#pragma unroll
        for (int un = 0; un < NU; ++un) {
          const int c = sg * NU + un;
          if (c >= nun) break;
          u32x4 xv[2][2];
          if (EPI) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
              for (int h = 0; h < 2; ++h) xv[u][h] = xn[u][h];
            const bool same = c + 1 < nun, blk = b + wpp < b1;
            ldx(same || blk ? p : pn, same ? b : (blk ? b + wpp : b0 + j), same ? c + 1 : 0, xn);
          }
          f4 acc[2][4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            acc[0][q] = acc[1][q] = f4zero();
#pragma unroll
            for (int ks = 0; ks < NKV; ++ks) {
              const h8 tf = MH::ld(sT + (un * 64 + q * 16 + r16) * LDT + ks * 32 + g * 8);
#pragma unroll
              for (int u = 0; u < 2; ++u) acc[u][q] = MH::mma(tf, vf[u][ks], acc[u][q]);
            }
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            // D (rows of the table permuted): lane holds row r16, columns
            // 16 g + 4 q + i
            const int col = c * 64 + c8;
            u32x4 w[2];
            if (EPI) {
              float* of = reinterpret_cast<float*>(ob);
#pragma unroll
              for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f4*>(of + r16 * AN_LDO + 16 * g + 4 * q) = acc[u][q] * a.scale;
              wave_lds_sync();
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                u32x4 x = xv[u][h];
                if (tail && col < a.Nb && col + 8 > a.Nb) x = shift_down(x, 8 - tail);
                float v[8];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                  const f4 t = *reinterpret_cast<const f4*>(of + (rr + 8 * h) * AN_LDO + c8 + 4 * q);
#pragma unroll
                  for (int e = 0; e < 4; ++e) v[4 * q + e] = t[e];
                }
                mul_preact_grad8(v, w_as_h8(x), a.act, a.clip);
                h8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = to_h(v[e]);
                __builtin_memcpy(&w[h], &o, 16);
              }
            } else {
#pragma unroll
              for (int h = 0; h < 2; ++h) {
                h8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = to_h(acc[u][2 * h + e / 4][e % 4] * a.scale);
                *reinterpret_cast<h8*>(ob + r16 * AN_LDO + 16 * g + 8 * h) = o;
              }
              wave_lds_sync();
#pragma unroll
              for (int h = 0; h < 2; ++h)
                w[h] = *reinterpret_cast<const u32x4*>(ob + (rr + 8 * h) * AN_LDO + c8);
            }
            wave_lds_sync();
#pragma unroll
            for (int h = 0; h < 2; ++h)
              store_tail8(py, (32 * b + 16 * u + 8 * h + rr) * a.Nb, col, a.Nb, nt, w[h]);
          }
        }
      }
    }
    if (t + 1 < trips) stz(pn, sZ + (grp * 2 + (int)((t + 1) & 1)) * zsize, zn);
    group_sync(wpp);
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Spectrum of plane p from the sums of its parts, [planes][parts][K] in fp32:
// added in order, scaled and rounded once.
__global__ __launch_bounds__(256) void part_sum_kernel(const f2* part, h2* out, int parts,
                                                       int64_t K, int64_t n, float scale) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t p = i / K, k = i - p * K;
  const f2* src = part + p * parts * K + k;
  f2 v = src[0];
  for (int s = 1; s < parts; ++s) v += src[s * K];
  out[i] = h2{to_h(v[0] * scale), to_h(v[1] * scale)};
}

hipError_t launch_part_sum(const void* part, void* out, int parts, int64_t planes, int64_t K,
                           float scale, hipStream_t s) {
  const int64_t n = planes * K;
  hipLaunchKernelGGL(part_sum_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const f2*>(part), reinterpret_cast<h2*>(out), parts, K, n,
                     scale);
  return hipGetLastError();
}

// columns of a segment, in k-steps: 128 unless the row is that short
int any_nk(int Nb) { return Nb <= 64 ? 2 : 4; }

hipError_t launch_r2c_any(const R2CArgs& a_in, int nct, int num_cu, hipStream_t s) {
  R2CArgs a = a_in;
  if (!any_extents_fit(a.Na, a.Nb) || a.Kap16 > 128) return hipErrorNotSupported;
  const int nk = any_nk(a.Nb);
  a.lw = share_waves_log2((a.Na + 31) / 32, a.planes, num_cu);
  const bool pre = a.do_tanh != 0;
  size_t lds = any_r2c_lds(nct, nk, a.lw, pre, a.lut_sat);
  const size_t tab = (size_t)2 * a.Kap16 * (a.NaC + 8) * 2;
  // step-B tables in LDS where they fit beside as many work-groups per CU
  const int per_cu = nct <= 4 && lds <= 80 * 1024 ? 2 : 1;
  a.tab_lds = lds + tab <= (size_t)160 * 1024 / per_cu;
  if (a.tab_lds) lds += tab;
  if (lds > 160 * 1024) return hipErrorNotSupported;
  const int64_t ngrp = AN_NW >> a.lw;
  const int grid = a.parts > 1 ? (int)a.planes * a.parts
                               : (int)std::min<int64_t>((a.planes + ngrp - 1) / ngrp,
                                                        (int64_t)per_cu * num_cu);
#define FNO_ANY_F(N, K)                                                                   \
  if (nct == N && nk == K) {                                                              \
    auto k = a.parts > 1 ? (pre ? r2c_any_kernel<N, K, true, true>                        \
                                : r2c_any_kernel<N, K, false, true>)                      \
                         : (pre ? r2c_any_kernel<N, K, true, false>                       \
                                : r2c_any_kernel<N, K, false, false>);                    \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),                  \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    if (e != hipSuccess) return e;                                                        \
    hipLaunchKernelGGL(k, dim3(grid), dim3(AN_NW * 64), lds, s, a);                       \
    return hipGetLastError();                                                             \
  }
  FNO_ANY_F(2, 2) FNO_ANY_F(2, 4) FNO_ANY_F(4, 2) FNO_ANY_F(4, 4) FNO_ANY_F(8, 2) FNO_ANY_F(8, 4)
#undef FNO_ANY_F
  return hipErrorNotSupported;
}

hipError_t launch_c2r_any(const C2RArgs& a_in, int nct, int num_cu, hipStream_t s) {
  C2RArgs a = a_in;
  if (!any_extents_fit(a.Na, a.Nb) || a.Kap > 128) return hipErrorNotSupported;
  const int nk = any_nk(a.Nb);
  a.lw = share_waves_log2((a.Na + 31) / 32, a.planes, num_cu);
  while (a.lw < 3 && any_c2r_lds(nct, nk, a.lw, a.Kap, a.epilogue != 0) > 160 * 1024) ++a.lw;
  size_t lds = any_c2r_lds(nct, nk, a.lw, a.Kap, a.epilogue != 0);
  const size_t tab = (size_t)2 * a.Na * (a.Kap + 8) * 2;
  a.tab_lds = lds + tab <= (size_t)160 * 1024;
  if (a.tab_lds) lds += tab;
  if (lds > 160 * 1024) return hipErrorNotSupported;
  const int64_t ngrp = AN_NW >> a.lw;
  const int grid = a.parts > 1 ? (int)a.planes * a.parts
                               : (int)std::min<int64_t>((a.planes + ngrp - 1) / ngrp, num_cu);
#define FNO_ANY_I(N, K)                                                                   \
  if (nct == N && nk == K) {                                                              \
    auto k = a.parts > 1 ? (a.epilogue ? c2r_any_kernel<N, K, true, true>                 \
                                       : c2r_any_kernel<N, K, false, true>)               \
                         : (a.epilogue ? c2r_any_kernel<N, K, true, false>                \
                                       : c2r_any_kernel<N, K, false, false>);             \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),                  \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    if (e != hipSuccess) return e;                                                        \
    hipLaunchKernelGGL(k, dim3(grid), dim3(AN_NW * 64), lds, s, a);                       \
    return hipGetLastError();                                                             \
  }
  FNO_ANY_I(2, 2) FNO_ANY_I(2, 4) FNO_ANY_I(4, 2) FNO_ANY_I(4, 4) FNO_ANY_I(8, 2) FNO_ANY_I(8, 4)
#undef FNO_ANY_I
  return hipErrorNotSupported;
}

}  // namespace fno
