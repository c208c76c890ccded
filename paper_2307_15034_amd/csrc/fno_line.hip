// Truncated transforms of one-dimensional fp16 signals (ndim 1), any length
// of eight or more.
//
// The plane kernels see a 1-D signal as a plane of one row: one row tile in
// sixteen carries data and a work-group walks the whole signal alone
// (2048 signals of 8192 points: 947 us forward, 732 us inverse, 0.04 TB/s).
// Here both directions are laid out for what bounds them, the stream of
// samples:
//
//   forward  a signal is read as rows of 128 consecutive samples, 32 rows
//            (one block, 8 KiB) at a time.  With n = 128 r + m,
//              X[k] = sum_r e^{-2 pi i k 128 r / N} sum_m x[n] e^{-2 pi i k m / N},
//            so one small table (128 columns, in LDS for every block of every
//            signal) serves any N on the matrix cores, and the phases of the
//            rows are applied in fp32: blocks by rotating the accumulators
//            between them (Horner), rows once at the end.  The sums stay in
//            fp32 until the one rounding of X.
//   inverse  y[s][n] = sum_k Z[s][k] T[k][n] is a product with a long table;
//            a work-group keeps 128 columns of it in LDS and walks the signals,
//            so the table is read once and the outputs stream.
//
// The same sizes now: forward 10.9 us (3.1 TB/s), with tanh 13.4 us (the table
// lookups); inverse 9.7 us (3.8 TB/s), with tanh' 14.7 us (4.8 TB/s of x and gx;
// tanh' in fp32 arithmetic, as in the plane kernels for these shapes).  The
// matrix cores are busy 4 to 5% of the time; the waves wait for 43 to 62% of
// theirs.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "fno_device.h"

namespace fno {

namespace {

typedef MM<_Float16> MH;
constexpr int LN_NW = 8;     // waves per work-group
constexpr int LN_ROW = 128;  // samples per row
constexpr int LN_BLK = 32 * LN_ROW;
constexpr int LN_LDT = LN_ROW + 8;
constexpr int LN_CW = 128;   // inverse: output columns per work-group
constexpr int LN_LDO = 68;   // inverse: transpose buffer row stride (floats)

// LDS of the forward kernel: pre-activation table, twiddles, row phases,
// partial results of the waves that share a signal
size_t line_r2c_lds(int nct, bool pre, int sat) {
  const int kbp = nct * 8;
  return (pre ? (size_t)lutn_bytes(sat) : 0) + (size_t)2 * kbp * LN_LDT * 2 +
         (size_t)32 * kbp * 8 + (size_t)LN_NW * kbp * 8;
}

size_t line_c2r_lds(int nkv) {
  return (size_t)LN_CW * (nkv * 32 + 8) * 2 + (size_t)LN_NW * 16 * LN_LDO * 4;
}

}  // namespace

// ---------------------------------------------------------------------------
// Forward.  wpp = 1 << lw waves share a signal (block b goes to wave b % wpp)
// when there are too few signals to give every SIMD two waves of its own.
// ---------------------------------------------------------------------------
template <int NCT, bool PRE>
__global__ __launch_bounds__(LN_NW * 64, NCT <= 4 ? 2 : 1) void r2c_line_kernel(LineArgs a) {
  constexpr int KBP = NCT * 8, NTB = NCT / 2;
  extern __shared__ __align__(16) unsigned char smem[];  // the table at LDS byte 0
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  _Float16* lut = reinterpret_cast<_Float16*>(smem);
  _Float16* sT = reinterpret_cast<_Float16*>(smem + (PRE ? lutn_bytes(a.lut_sat) : 0));
  f2* sR = reinterpret_cast<f2*>(sT + 2 * KBP * LN_LDT);  // [32][KBP]
  f2* red = sR + 32 * KBP;                                // [LN_NW][KBP]
  const f2* blk = reinterpret_cast<const f2*>(a.blkph);
  const uint32_t s2 = (uint32_t)a.lut_sat * 2u * 0x10001u;

  const int wpp = 1 << a.lw, grp = wave >> a.lw, j = wave & (wpp - 1), ngrp = LN_NW >> a.lw;
  const int nblk = (a.N + LN_BLK - 1) / LN_BLK;
  const int nbw = (nblk - j + wpp - 1) >> a.lw;  // blocks of this wave (wpp <= nblk)
  const int tail = a.N & 7;
  const int64_t trips = (a.planes + (int64_t)gridDim.x * ngrp - 1) / ((int64_t)gridDim.x * ngrp);
  auto signal = [&](int64_t t) { return ((int64_t)blockIdx.x + t * gridDim.x) * ngrp + grp; };

  // block b of signal p: lane holds rows 32 b + 16 u + r16, samples 32 k + 8 g
  // .. + 8 of the row; past the signal zero, the last partial eight read from
  // N - 8 on and shifted down when used
  auto load = [&](int64_t p, int b, u32x4 (&v)[2][4]) {
    const bool ok = p < a.planes;
    const PlaneRef pr = plane_ref(a.in, ok ? p : 0, ok ? (int64_t)a.N * 2 : 0);
    int n0 = b * LN_BLK + r16 * LN_ROW + g * 8;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int n = n0 + u * 16 * LN_ROW + k * 32;
        const int vo = n + 8 <= a.N ? n : (n < a.N ? a.N - 8 : PLANE_OOB / 2);
        v[u][k] = __builtin_amdgcn_raw_buffer_load_b128(pr.rs, vo * 2 + pr.off, 0, 0);
      }
  };
  u32x4 nxt[2][4];
  load(signal(0), j + (nbw - 1) * wpp, nxt);

  if (PRE) stage_lutn<LN_NW * 64>(lut, a.lut, a.lut_sat);
  stage_pieces<LN_NW * 64, 2>(
      2 * KBP * (LN_ROW / 8), [&](int i) { return reinterpret_cast<const u32x4*>(a.tw) + i; },
      [&](int i) {
        return reinterpret_cast<u32x4*>(sT + i / (LN_ROW / 8) * LN_LDT + (i % (LN_ROW / 8)) * 8);
      });
  stage_pieces<LN_NW * 64, 1>(
      16 * KBP, [&](int i) { return reinterpret_cast<const u32x4*>(a.rowph) + i; },
      [&](int i) { return reinterpret_cast<u32x4*>(sR) + i; });
  // rotation between this wave's blocks, and the phase of its first block
  f2 om[NTB], ph[NTB];
#pragma unroll
  for (int tb = 0; tb < NTB; ++tb) {
    om[tb] = blk[wpp * KBP + tb * 16 + r16];
    ph[tb] = blk[j * KBP + tb * 16 + r16];
  }
  __syncthreads();

  for (int64_t t = 0; t < trips; ++t) {
    const int64_t p = signal(t);
    f4 acc[2][NCT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct) acc[u][ct] = f4zero();
#pragma nounroll
    for (int bi = nbw - 1; bi >= 0; --bi) {
      const int b = j + bi * wpp;
      u32x4 cur[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) cur[u][k] = nxt[u][k];
      if (bi > 0) load(p, b - wpp, nxt);
      else load(t + 1 < trips ? signal(t + 1) : a.planes, j + (nbw - 1) * wpp, nxt);
      if (tail && b == nblk - 1) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int n = b * LN_BLK + (16 * u + r16) * LN_ROW + k * 32 + g * 8;
            const u32x4 w = shift_down(cur[u][k], 8 - tail);
            const bool part = n < a.N && n + 8 > a.N;
#pragma unroll
            for (int e = 0; e < 4; ++e) cur[u][k][e] = part ? w[e] : cur[u][k][e];
          }
      }
      if (bi < nbw - 1) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) rotate(acc[u][tb], acc[u][NTB + tb], om[tb]);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        h8 af[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          u32x4 w = cur[u][k];
          if (PRE) lutn_odd4(w, s2);
          af[u] = w_as_h8(w);
        }
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
          const h8 bf = MH::ld(sT + (ct * 16 + r16) * LN_LDT + k * 32 + g * 8);
#pragma unroll
          for (int u = 0; u < 2; ++u) acc[u][ct] = MH::mma(af[u], bf, acc[u][ct]);
        }
      }
    }
    // rows: lane holds rows 16 u + 4 g + i of the mode tb * 16 + r16
    float xr[NTB], xi[NTB];
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb) {
      float sr = 0.0f, si = 0.0f;
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f2 c = sR[(16 * u + 4 * g + i) * KBP + tb * 16 + r16];
          const float yr = acc[u][tb][i], yi = acc[u][NTB + tb][i];
          sr = fmaf(yi, c[1], fmaf(yr, c[0], sr));
          si = fmaf(-yr, c[1], fmaf(yi, c[0], si));
        }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        sr += __shfl_xor(sr, o, 64);
        si += __shfl_xor(si, o, 64);
      }
      xr[tb] = (sr * ph[tb][0] + si * ph[tb][1]) * a.scale;
      xi[tb] = (si * ph[tb][0] - sr * ph[tb][1]) * a.scale;
    }
    _Float16* out = reinterpret_cast<_Float16*>(a.out) + p * a.Kb * 2;
    if (wpp == 1) {
      if (p < a.planes && g == 0) {
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
          if (tb * 16 + r16 < a.Kb) store_pair<_Float16>(out + (tb * 16 + r16) * 2, xr[tb], xi[tb]);
      }
    } else {
      if (g == 0) {
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) red[wave * KBP + tb * 16 + r16] = f2{xr[tb], xi[tb]};
      }
      __syncthreads();
      if (p < a.planes && j == 0) {
        for (int k = lane; k < a.Kb; k += 64) {
          f2 v = red[wave * KBP + k];
          for (int w = 1; w < wpp; ++w) v += red[(wave + w) * KBP + k];
          store_pair<_Float16>(out + k * 2, v[0], v[1]);
        }
      }
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------
// Inverse: y[s][n] = scale * sum_k Re(Z[s][k] e^{+2 pi i k n / N}), times
// f'(x) with the epilogue.  The contraction index of a k-step runs over the
// interleaved (re, im) pairs of the spectrum as they lie in memory (table
// columns 2 k and 2 k + 1: cos and -sin).  A wave takes 16 signals x 64
// columns at a time; the result passes through its fp32 LDS buffer so that
// eight lanes write (and read x of) 128 consecutive bytes of a signal.
// ---------------------------------------------------------------------------
template <int NKV, bool EPI>
__global__ __launch_bounds__(LN_NW * 64, 2) void c2r_line_kernel(LineArgs a) {
  constexpr int LDT = NKV * 32 + 8;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g = lane >> 4;
  _Float16* sT = reinterpret_cast<_Float16*>(smem);  // [LN_CW][LDT]
  float* ob = reinterpret_cast<float*>(smem + LN_CW * LDT * 2) + wave * 16 * LN_LDO;
  const int nsl = (a.N + LN_CW - 1) / LN_CW;
  const int sl = blockIdx.x % nsl, rg = blockIdx.x / nsl;
  const int m0 = sl * LN_CW;
  const int nrt = (int)((a.planes + 15) / 16);
  const int rt0 = rg * a.rtg, nt = 2 * (min(nrt, rt0 + a.rtg) - rt0);  // (tile, half) tasks
  const int tail = a.N & 7;
  const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<void*>(a.in), (short)0, (int)(a.planes * a.Kb * 4), 0x00020000);

  auto ldz = [&](int task, u32x4 (&v)[NKV]) {
    const int s = (rt0 + (task >> 1)) * 16 + r16;
#pragma unroll
    for (int k = 0; k < NKV; ++k) {
      const int t = k * 16 + g * 4;
      const int vo = task < nt && s < a.planes && t < a.Kb ? (s * a.Kb + t) * 4 : PLANE_OOB;
      v[k] = __builtin_amdgcn_raw_buffer_load_b128(rz, vo, 0, 0);
    }
  };
  // x and y of a task in the row layout: signal lane / 8 + 8 h, eight columns
  // at (lane % 8) * 8
  const int64_t tile_bytes = (int64_t)16 * a.N * 2;
  auto tile_ref = [&](const void* base, int task) {
    const int rt = task < nt ? rt0 + (task >> 1) : nrt;
    const int64_t first = (int64_t)rt * 16;
    const int rows = (int)max((int64_t)0, min((int64_t)16, a.planes - first));
    return plane_ref_at(base, rows > 0 ? rt * tile_bytes : 0, (int64_t)rows * a.N * 2);
  };
  auto ldx = [&](int task, u32x4 (&v)[2]) {
    if (!EPI) return;
    const PlaneRef pr = tile_ref(a.x, task);
    const int col = m0 + (task & 1) * 64 + (lane & 7) * 8;
    const int cl = col + 8 <= a.N ? col : (col < a.N ? a.N - 8 : PLANE_OOB / 2);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int vo = cl >= PLANE_OOB / 2 ? PLANE_OOB : (((lane >> 3) + 8 * h) * a.N + cl) * 2;
      v[h] = __builtin_amdgcn_raw_buffer_load_b128(pr.rs, vo + pr.off, 0, 0);
    }
  };

  u32x4 zn[NKV], xn[2];
  ldz(wave, zn);
  ldx(wave, xn);
  stage_pieces<LN_NW * 64, NKV>(
      LN_CW * NKV * 4,
      [&](int i) { return reinterpret_cast<const u32x4*>(a.tw) + (int64_t)m0 * NKV * 4 + i; },
      [&](int i) {
        return reinterpret_cast<u32x4*>(sT + i / (NKV * 4) * LDT + (i % (NKV * 4)) * 8);
      });
  __syncthreads();

#pragma nounroll
  for (int task = wave; task < nt; task += LN_NW) {
    h8 zf[NKV];
    u32x4 xv[2];
#pragma unroll
    for (int k = 0; k < NKV; ++k) {
      u32x4 v = zn[k];
      // modes past Kb belong to the next signal
      const int t = k * 16 + g * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = t + e < a.Kb ? v[e] : 0u;
      zf[k] = w_as_h8(v);
    }
    if (EPI) {
      xv[0] = xn[0];
      xv[1] = xn[1];
    }
    ldz(task + LN_NW, zn);
    ldx(task + LN_NW, xn);
    const _Float16* tb = sT + ((task & 1) * 64 + r16) * LDT + g * 8;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      f4 acc = f4zero();
#pragma unroll
      for (int k = 0; k < NKV; ++k) acc = MH::mma(MH::ld(tb + c * 16 * LDT + k * 32), zf[k], acc);
      // D: lane holds signal r16, columns c * 16 + 4 g + i
      *reinterpret_cast<f4*>(ob + r16 * LN_LDO + c * 16 + 4 * g) = acc * a.scale;
    }
    wave_lds_sync();
    float v[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f4 w = *reinterpret_cast<const f4*>(ob + ((lane >> 3) + 8 * h) * LN_LDO +
                                                  (lane & 7) * 8 + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[h][4 * q + e] = w[e];
      }
    wave_lds_sync();
    const PlaneRef py = tile_ref(a.out, task);
    const int col = m0 + (task & 1) * 64 + (lane & 7) * 8;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = ((lane >> 3) + 8 * h) * a.N;
      if (EPI) {
        u32x4 w = xv[h];
        if (tail && col < a.N && col + 8 > a.N) w = shift_down(w, 8 - tail);
        mul_preact_grad8(v[h], w_as_h8(w), a.act, a.clip);
      }
      h8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = to_h(v[h][e]);
      u32x4 w;
      __builtin_memcpy(&w, &o, 16);
      store_tail8(py, row, col, a.N, a.N % 64 == 0, w);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_r2c_line(const LineArgs& a_in, int nct, int num_cu, hipStream_t s) {
  LineArgs a = a_in;
  if (a.N < 8 || a.planes < 1) return hipErrorNotSupported;
  const bool pre = a.act != ACT_NONE;
  const size_t lds = line_r2c_lds(nct, pre, a.lut_sat);
  if (lds > 160 * 1024) return hipErrorNotSupported;
  // share a signal among more waves while that still leaves SIMDs with fewer
  // than two waves and every wave has a block
  const int nblk = (a.N + LN_BLK - 1) / LN_BLK;
  a.lw = 0;
  while (a.lw < 3 && (2 << a.lw) <= nblk && (a.planes << a.lw) < (int64_t)8 * num_cu) ++a.lw;
  const int64_t ngrp = LN_NW >> a.lw;
  const int per_cu = nct <= 4 && lds <= 80 * 1024 ? 2 : 1;
  const int grid = (int)std::min<int64_t>((a.planes + ngrp - 1) / ngrp, (int64_t)per_cu * num_cu);
#define FNO_LINE_F(N)                                                                     \
  if (nct == N) {                                                                         \
    auto k = pre ? r2c_line_kernel<N, true> : r2c_line_kernel<N, false>;                  \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),                  \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    if (e != hipSuccess) return e;                                                        \
    hipLaunchKernelGGL(k, dim3(grid), dim3(LN_NW * 64), lds, s, a);                       \
    return hipGetLastError();                                                             \
  }
  FNO_LINE_F(2) FNO_LINE_F(4) FNO_LINE_F(8) FNO_LINE_F(16)
#undef FNO_LINE_F
  return hipErrorNotSupported;
}

hipError_t launch_c2r_line(const LineArgs& a_in, int nkv, int num_cu, hipStream_t s) {
  LineArgs a = a_in;
  if (a.N < 8 || a.planes < 1 || a.planes * a.Kb * 4 >= (int64_t)PLANE_OOB)
    return hipErrorNotSupported;
  const size_t lds = line_c2r_lds(nkv);
  const int nsl = (a.N + LN_CW - 1) / LN_CW;
  const int nrt = (int)((a.planes + 15) / 16);
  // row groups: two work-groups per compute unit in all, at least four row
  // tiles (one task per wave) each
  int ng = std::max(1, std::min((2 * num_cu + nsl - 1) / nsl, (nrt + 3) / 4));
  a.rtg = (nrt + ng - 1) / ng;
  ng = (nrt + a.rtg - 1) / a.rtg;
#define FNO_LINE_I(N)                                                                     \
  if (nkv == N) {                                                                         \
    auto k = a.x ? c2r_line_kernel<N, true> : c2r_line_kernel<N, false>;                  \
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),                  \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); \
    if (e != hipSuccess) return e;                                                        \
    hipLaunchKernelGGL(k, dim3(nsl * ng), dim3(LN_NW * 64), lds, s, a);                   \
    return hipGetLastError();                                                             \
  }
  FNO_LINE_I(1) FNO_LINE_I(2) FNO_LINE_I(4) FNO_LINE_I(8)
#undef FNO_LINE_I
  return hipErrorNotSupported;
}

}  // namespace fno
