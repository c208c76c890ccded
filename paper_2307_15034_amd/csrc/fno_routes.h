// Which kernel a transform of planes or signals runs, by sizes alone; plain
// C++, so that the host can replay it.
#pragma once

#include <stdint.h>

namespace fno {

struct PlaneShape {
  int Na, Nb, Kbp;  // rows, columns, last-axis modes padded to 16, 32, 64, ..
  bool fp16;
  int64_t planes;
  int num_cu;
};

// Waves of a work-group of eight that share a plane in the kernels for any
// extents, as a power of two: one per block of 32 rows, up to all eight, and
// more while every plane still has its place in one pass over the chip.  (More
// than that starts a second pass that is nearly empty: 304 planes of 64 x 72 and
// 12 modes with the planes of one work-group each on 256 compute units, whole
// forward call 23.1 us in fp16 and 37.9 in fp32, so 19.0 and 30.9.)
constexpr int share_waves_log2(int64_t blocks, int64_t planes, int num_cu) {
  int lw = 0;
  while (lw < 3 && ((1 << lw) < blocks || (planes << (lw + 1)) <= (int64_t)8 * num_cu)) ++lw;
  return lw;
}

// Buffer offsets of this value lie past every plane: loads there read zero,
// stores are dropped.
constexpr int PLANE_OOB = 0x40000000;

// fp16 planes whose byte offsets, to the end of the last block of 256 rows and
// with PLANE_OOB added for columns past the row, stay below 2^31 (planes of up to
// 2^30 bytes).
constexpr bool any_extents_fit(int64_t Na, int64_t Nb) {
  return Nb >= 8 && (Na + 255) / 256 * 256 * Nb * 2 < PLANE_OOB;
}

// A call of few small planes, where the kernels' start-up is most of their
// time: the generic kernels, a work-group per plane, are quicker there than the
// ones for any extents, whose work-groups stage tables and whose waves take
// blocks of 32 rows.  The line lies at a plane's work (points, the rows rounded
// up to 16, per 16 padded modes): a table by the blocks of a plane (1, 2, 3 and
// 4, more), which say how many planes the kernels for any extents take in a pass
// over the chip, and by the planes per compute unit (1, 2, 3, 4 and up to 12);
// rows that the generic kernel reads by 16 bytes have lines of their own.
// Measured over 1 to 3008 planes of 8 to 201 rows of 8 to 505 columns with 3, 12
// and 28 modes; of 1800 other calls of such sizes one in thirty is more than 5%,
// and none more than 19%, slower than through the generic and small-plane kernels
// alone, near half are quicker.
// The whole call in us, generic and any extents: fp16 forward, 16 planes of 48 x
// 136: 17.4 and 19.2, 1024: 26.1 and 24.7; inverse with tanh', 512 planes of 16 x
// 264: 23.6 and 28.7, of 49 x 105: 27.6 and 22.4, 2048 of 200 x 16: 57 and 64;
// fp32 forward, 256 planes of 30 x 200: 32.3 and 36.6, 512 of 32 x 504: 73.6 and
// 65.4; inverse, 256 of 48 x 73 with 28 modes: 35.0 and 31.1.
// Forward fp16 planes of up to 64 rows and two to four planes per compute unit have
// their lines from 120 calls with tanh, whose table the kernels for any extents
// stage: below them these are 0.3 to 1.8 us behind (440 planes of 8 x 18, 3 modes, whole
// call 19.0 and 20.7), without tanh 0.7 us behind to 0.6 ahead.
// Forward fp32 planes of odd rows with 33 to 64 modes (unfolded, in segments of 32
// columns) of at most two blocks have a line of their own up to one plane per compute
// unit: the generic kernel was quicker in all 191 measured, by 3 to 22 us (4 planes of
// 20 x 383, 44 modes, whole call 91 and 105 us), and slower in the 42 of 65 to 100 rows.
constexpr bool few_small_planes(const PlaneShape& g, bool inverse) {
  typedef const short Lines[2][4][5];  // [aligned rows][blocks][planes per unit]: work / 16
  constexpr Lines h_fwd = {
      {{64, 64, 64, 64, 0}, {128, 96, 64, 0, 0}, {192, 0, 192, 128, 0}, {0, 0, 256, 256, 96}},
      {{384, 384, 384, 96, 0}, {640, 0, 0, 0, 0}, {192, 0, 256, 192, 192}, {0, 384, 384, 384, 256}}};
  constexpr Lines h_inv = {
      {{256, 128, 96, 0, 0}, {256, 128, 64, 0, 0}, {192, 64, 256, 0, 64}, {0, 192, 256, 96, 192}},
      {{1024, 512, 512, 0, 0}, {1536, 640, 192, 0, 64}, {384, 128, 2048, 128, 128}, {0, 256, 384, 256, 256}}};
  constexpr Lines s_fwd = {
      {{640, 512, 96, 96, 0}, {2048, 96, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}},
      {{1024, 640, 96, 128, 0}, {2048, 384, 0, 0, 0}, {192, 0, 640, 192, 192}, {0, 0, 1024, 384, 256}}};
  constexpr Lines s_inv = {
      {{128, 64, 0, 0, 0}, {128, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}},
      {{512, 128, 0, 0, 0}, {512, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}}};
  const int64_t units = (g.planes + g.num_cu - 1) / g.num_cu;
  if (units < 1 || units > 12) return false;
  const int q = units < 5 ? (int)units - 1 : 4;
  const int b = g.Na <= 32 ? 0 : g.Na <= 64 ? 1 : g.Na <= 128 ? 2 : 3;
  if (!g.fp16 && !inverse && g.Nb % 2 && g.Kbp == 64 && b <= 1 && units == 1) return true;
  const bool aligned = g.Nb % (g.fp16 ? 8 : 4) == 0;
  const Lines& l = g.fp16 ? (inverse ? h_inv : h_fwd) : (inverse ? s_inv : s_fwd);
  return (g.Na + 15) / 16 * (int64_t)g.Nb * (g.Kbp / 16) <= l[aligned][b][q];
}

// Few short 1-D signals in the forward transform, as few_small_planes: the
// kernels for small planes (the generic ones where those do not apply) start
// sooner than the one for signals, up to 64 samples; up to 128 where the former
// have them, and with 33 to 64 modes, whose tables are the larger part, up to
// 192.  (64 signals of 64 samples and 8 modes, the whole call with tanh: 11.7
// against 13.4 us, 2048: 18.7 against 15.2; 256 of 144 and 60 modes: 20.8
// against 22.9.)
constexpr bool few_short_signals(const PlaneShape& g, bool pre) {
  if (g.planes > 2 * (int64_t)g.num_cu) return g.Nb <= 32 && g.planes <= 4 * (int64_t)g.num_cu;
  return g.Nb <= 64 || (g.Nb <= 128 && g.Nb % 8 == 0 && g.Kbp <= 32) ||
         (g.Nb <= 192 && g.Kbp == 64 && !pre);
}

// Planes that the small-plane kernels take, a work-group each: up to 64 x 64 at
// any count, larger ones where planes are few and the short start-up counts
// (whole call in us, against the kernel for any extents: 72 x 72, 20 modes,
// forward with tanh, 64 planes 17.1 and 18.7, 2048: 51.6 and 47.9; inverse with
// tanh', 64 planes 16.9 and 19.4, 2048: 56.5 and 52.9).
constexpr bool fast_planes(const PlaneShape& g, bool inverse) {
  if (g.Nb <= 64 && g.Na <= 64) return true;
  if (g.Nb > 256 || g.Na > 128) return false;
  const int64_t work = (int64_t)(g.Na + 31) / 32 * 32 * g.Nb * (g.Kbp / 16);
  return g.planes <= g.num_cu ||
         (inverse && work <= 12288 && g.planes <= 3 * (int64_t)g.num_cu);
}

// Pairwise fp16 steps batched over an index t that is innermost in memory, M x N
// results of K products for each t: whether a wave per 16 x 16 results of four t
// (`waves` in all) beats the GEMM tiles.  It does without an upper bound, although
// each wave fetches its rows again (the neighbours' are in the L1): 2048 x 128
// results of 512 products for 32 t 450 against 1175 us, 2048 x 256 of 128 226
// against 719, 1024 x 128 of 128 59 against 93, 512 x 64 of 48 13 against 19.  It
// loses where few waves walk a long reduction, which the tiles split (64 x 64 of
// 384 for 32 t 29.7 against 26.3 us, 48 x 32 of 384 for 16 22.3 against 17.2), and
// by 1 to 2 us of start-up where a small step fills half of its 16 columns.
constexpr bool quad_pays(int64_t M, int64_t N, int64_t K, int64_t waves) {
  if (waves <= 128 && K > 256) return false;
  return !(waves <= 256 && M <= 64 && N <= 8 && K <= 32);
}

// The channel mix of fp16 rows whose length is not a multiple of eight, K to N
// channels of `points`: whether the kernels without matrix cores are quicker.  With
// so few products the pipelined ones are staging alone (1 to 1 channel, 120002
// points 8.2 against 4.8 us, 2 to 4 8.3 against 6.3, of 11300 points 5.5 against 5.7),
// and their 128 columns of weights cost more than a few products of few points (2 to
// 128, 11300 points 11.2 against 9.9, 57860 24 against 30).
constexpr bool few_channels(int64_t K, int64_t N, int64_t points) {
  return K * N <= (points < 32768 ? 6 : 12) || (K <= 4 && N > 64 && points <= 16384);
}

// Elementwise and outer products of `results` values: four results per thread
// instead of two.  Only outer products gain, whose operand without the innermost
// index (stride other than one) is loaded once for the four, and only from about
// 1.25 million results on, where fewer threads still fill the chip (0.79 M 4.8
// against 4.4 us, 1.57 M 5.9 against 6.5, 16.8 M 25.0 against 33.9, fp16); where
// both operands stream, two are as quick or quicker at any size (2.1 M 9.2 against
// 7.3 us, 33.6 M 67.2 against 64.5).
constexpr bool four_products_pay(int64_t results, int64_t a_stride, int64_t b_stride) {
  return results >= (int64_t)5 << 18 && (a_stride != 1 || b_stride != 1);
}

// A call with factorised weights, as far as its time goes.
struct FactorShape {
  bool cp, fp16;
  bool generic;      // its transforms run in the generic kernels
  int ndim;
  int64_t points;    // B (Cin + Cout) N
  int Nb, Kbp;       // last axis: points, padded modes
  int64_t products;  // with u_in and u_out: B modes (Cin r_in + Cout r_out)
  int64_t weight;    // Tucker: modes r_in r_out
};

// What its transforms (a forward's) and the products of its weight gradient take
// beyond their launches, in us: 2.5 TB/s with ramps; the generic kernels by the
// products, a 1-D signal walked by one work-group.
constexpr double factor_transforms_us(const FactorShape& f) {
  if (!f.generic) return 0.4e-6 * (double)f.points * (f.fp16 ? 2 : 4);
  return 10e-8 * (double)f.points * f.Kbp + (f.ndim == 1 ? 4e-3 * f.Nb * f.Kbp : 0.0);
}
constexpr double factor_products_us(const FactorShape& f) {
  return 35e-8 * (double)f.products + 107e-6 * (double)f.weight;
}

// Whether a call gains from its side streams.  path: the steps of the weight alone
// beside the transforms; backward: the weight gradient too; wgrad: its own chains.
// Two streams and their events take 130 to 150 us of host time in a backward
// launched from the host, so what they run beside has to be long; recorded into a
// graph they cost the device's dependencies alone.  Measured both ways over 613
// shapes of 0.1 to 260 M points, the lines give the quicker way to within (mean, calls
// more than 5% off; in brackets with one line on the points for all):
//   launched  path and backward 0.8%, 71 of 1226 (1.3%, 114), wgrad 0.2%, 9 of 613 (2.0%, 53)
//   recorded  path 0.9%, 42 of 613 (1.1%, 57), backward 0.7%, 34 of 613 (2.7%, 104)
// In us, forked and on one stream: Tucker, one sample of 12 to 26 channels, 114 x 216,
// 22 x 91 modes, backward recorded 163 and 229; 2 of 14 to 25, 125 x 390, 40 x 128
// modes, backward launched 393 and 455; CP of rank 16, 32 samples of 64 channels, 128 x
// 128, 64 x 32 modes, backward launched 212 and 170, recorded 155 and 167.
enum ForkCall { FORK_PATH, FORK_BACKWARD, FORK_WGRAD };
constexpr bool fork_pays(const FactorShape& f, ForkCall call, bool recorded) {
  if (call == FORK_WGRAD) return !recorded && factor_products_us(f) >= 65;
  const double us = factor_transforms_us(f);
  if (recorded) return us >= (call == FORK_BACKWARD ? (f.cp ? 6 : 2) : (f.cp ? 60 : 8));
  if (f.cp) return us >= 100;
  return us + (call == FORK_BACKWARD ? 10 * f.ndim : 0) >= 55;  // (weight steps by axis)
}

}  // namespace fno
