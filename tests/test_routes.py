"""The rules that choose how a transform is laid out and which kernel it runs,
replayed on the host from the plain header that the library compiles."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2307_15034_amd", "csrc")


def replay(tmp_path, body):
    """Compiles and runs `body` (statements that return non-zero on a fault)."""
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text('#include <cstdio>\n#include <initializer_list>\n#include "fno_routes.h"\n'
                   "using namespace fno;\nint main() {\n" + body + "\n}\n")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[:2000]


def test_waves_that_share_a_plane(tmp_path):
    """Never fewer waves than blocks (up to the eight), more only while the
    planes' work-groups still run in one pass."""
    replay(tmp_path, """
  int bad = 0;
  for (int cu : {256, 304})
    for (int blocks = 1; blocks <= 20; ++blocks)
      for (int planes = 1; planes <= 6000; ++planes) {
        const int lw = share_waves_log2(blocks, planes, cu);
        int need = 0;
        while (need < 3 && (1 << need) < blocks) ++need;
        const int groups = (planes + (8 >> lw) - 1) / (8 >> lw);
        const bool ok = lw >= need && lw <= 3 && (lw == need || groups <= cu) &&
                        (lw == 3 || (planes << (lw + 1)) > 8 * cu);
        if (!ok && ++bad < 5) std::printf("blocks %d planes %d: %d\\n", blocks, planes, lw);
      }
  return bad != 0;""")


def test_few_planes_and_signals(tmp_path):
    """Calls on either side of the lines, as measured on 256 compute units
    ({rows, columns, padded modes, fp16, planes, compute units})."""
    replay(tmp_path, """
  int bad = 0;
  auto expect = [&](const char* what, bool got, bool want) {
    if (got != want) ++bad, std::printf("%s: %d\\n", what, got);
  };
  // the small-plane kernels: any count up to 64 x 64, few larger planes
  for (bool inverse : {false, true}) {
    expect("72 x 72, 64", fast_planes({72, 72, 32, true, 64, 256}, inverse), true);
    expect("128 x 72, 16", fast_planes({128, 72, 32, true, 16, 256}, inverse), true);
    expect("72 x 72, 2048", fast_planes({72, 72, 32, true, 2048, 256}, inverse), false);
    expect("64 x 64, 8192", fast_planes({64, 64, 16, true, 8192, 256}, inverse), true);
    expect("129 x 64, 16", fast_planes({129, 64, 16, true, 16, 256}, inverse), false);
  }
  // the generic kernels against those for any extents
  expect("48 x 136, 16", few_small_planes({48, 136, 16, true, 16, 256}, false), true);
  expect("48 x 136, 1024", few_small_planes({48, 136, 16, true, 1024, 256}, false), false);
  expect("16 x 264, 512", few_small_planes({16, 264, 16, true, 512, 256}, true), true);
  expect("49 x 105, 512", few_small_planes({49, 105, 16, true, 512, 256}, true), false);
  expect("200 x 16, 2048", few_small_planes({200, 16, 16, true, 2048, 256}, true), true);
  expect("241 x 241, 512", few_small_planes({241, 241, 32, true, 512, 256}, false), false);
  expect("fp32 30 x 200, 256", few_small_planes({30, 200, 16, false, 256, 256}, false), true);
  expect("fp32 32 x 504, 512", few_small_planes({32, 504, 16, false, 512, 256}, false), false);
  expect("fp32 48 x 73, 256", few_small_planes({48, 73, 32, false, 256, 256}, true), false);
  expect("fp32 128 x 128, 2048", few_small_planes({128, 128, 32, false, 2048, 256}, true), false);
  expect("8 x 18, 440", few_small_planes({8, 18, 16, true, 440, 256}, false), true);
  expect("8 x 18, 1100", few_small_planes({8, 18, 16, true, 1100, 256}, false), false);
  expect("20 x 60, 600", few_small_planes({20, 60, 32, true, 600, 256}, false), false);
  expect("fp32 20 x 383, 4", few_small_planes({20, 383, 64, false, 4, 256}, false), true);
  expect("fp32 64 x 187, 256", few_small_planes({64, 187, 64, false, 256, 256}, false), true);
  expect("fp32 64 x 187, 257", few_small_planes({64, 187, 64, false, 257, 256}, false), false);
  expect("fp32 20 x 386, 4", few_small_planes({20, 386, 64, false, 4, 256}, false), false);
  expect("fp32 70 x 383, 4", few_small_planes({70, 383, 64, false, 4, 256}, false), false);
  expect("fp32 20 x 383, 4, inverse", few_small_planes({20, 383, 64, false, 4, 256}, true), false);
  // no count of planes leaves the tables
  for (long planes : {1L, 256L, 257L, 1024L, 1025L, 3072L, 3073L, 1L << 31})
    for (int rows : {1, 32, 33, 64, 65, 128, 129, 65536})
      for (int half = 0; half < 2; ++half)
        if (planes > 3072) expect("many", few_small_planes({rows, 8, 16, half > 0, planes, 256}, half > 0), false);
        else (void)few_small_planes({rows, 65536, 128, half > 0, planes, 256}, true);
  // 1-D signals
  expect("64, 64", few_short_signals({1, 64, 16, true, 64, 256}, true), true);
  expect("64, 2048", few_short_signals({1, 64, 16, true, 2048, 256}, true), false);
  expect("144, 60 modes", few_short_signals({1, 144, 64, true, 256, 256}, false), true);
  expect("144, 60 modes, tanh", few_short_signals({1, 144, 64, true, 256, 256}, true), false);
  expect("8192", few_short_signals({1, 8192, 32, true, 1, 256}, false), false);
  return bad != 0;""")


def test_planes_of_any_extents_fit_their_offsets(tmp_path):
    """Accepted planes: every offset below 2^31 and none of a column past the
    row inside the plane; refused only where that does not hold for the planes
    of whole 256-row blocks."""
    replay(tmp_path, """
  int bad = 0;
  for (int64_t na : {2LL, 100LL, 255LL, 256LL, 257LL, 8191LL, 16384LL, 16640LL, 32768LL, 65536LL})
    for (int64_t nb = 8; nb <= 65536; nb = nb < 64 ? nb + 1 : nb + 121) {
      const bool fit = any_extents_fit(na, nb);
      const int64_t rows = (na + 255) / 256 * 256, plane = na * nb * 2;
      const int64_t last = (rows - 1) * nb * 2 + 15;  // a lane's row, the alignment rest
      const bool safe = last + PLANE_OOB < (int64_t)1 << 31 && plane <= PLANE_OOB;
      if ((fit && !safe) || (na % 256 == 0 && fit != (plane < (int64_t)1 << 30)))
        ++bad, std::printf("%lld x %lld: %d\\n", (long long)na, (long long)nb, fit);
    }
  return bad != 0;""")


def test_batched_steps(tmp_path):
    """Steps on either side of the line as measured (results, products, t)."""
    replay(tmp_path, """
  int bad = 0;
  auto expect = [&](int M, int N, int K, int t, bool want) {
    const long waves = (long)((M + 15) / 16) * ((N + 15) / 16) * (t / 4);
    if (quad_pays(M, N, K, waves) != want) ++bad, std::printf("%d %d %d %d\\n", M, N, K, t);
  };
  expect(48, 32, 384, 16, false);
  expect(64, 64, 384, 32, false);
  expect(32, 4, 8, 192, false);
  expect(48, 8, 32, 192, false);
  expect(2048, 128, 512, 32, true);
  expect(128, 32, 12, 2048, true);
  expect(256, 128, 384, 12, true);
  expect(64, 32, 48, 16, true);
  expect(32, 8, 128, 192, true);
  expect(512, 8, 48, 32, true);
  return bad != 0;""")


def test_products_per_thread(tmp_path):
    replay(tmp_path, """
  int bad = 0;
  bad += four_products_pay(262144, 1, 0) || four_products_pay(786432, 1, 0);
  bad += !four_products_pay(1572864, 1, 0) || !four_products_pay(16777216, 0, 1);
  bad += !four_products_pay(8388608, 1, 8);
  bad += four_products_pay(2097152, 1, 1) || four_products_pay(33554432, 1, 1);
  return bad;""")


def test_forks_of_factorised_calls(tmp_path):
    """Calls on either side of the lines as measured: each way in us, forked and
    on one stream."""
    replay(tmp_path, """
  int bad = 0;
  auto expect = [&](bool cp, bool fp16, bool gen, int nd, long pts, int nb, int kbp, long modes,
                    int b, int ci, int co, int r0, int r1, ForkCall call, bool rec, bool want) {
    FactorShape f{cp, fp16, gen, nd, pts * b * (ci + co), nb, kbp,
                  modes * b * (ci * r0 + co * r1), cp ? 0 : modes * r0 * r1};
    if (fork_pays(f, call, rec) != want)
      ++bad, std::printf("%d %d %d %d %d\\n", nd, nb, (int)modes, (int)call, rec);
  };
  // 114 x 216, 22 x 91 modes, rank 9 x 8: recorded 163, 229
  expect(0, 1, 1, 2, 114 * 216, 216, 128, 2002, 1, 12, 26, 9, 8, FORK_BACKWARD, 1, true);
  // 175 x 46, 100 x 14 modes, rank 3 x 34: recorded 142, 196, launched 249, 199
  expect(0, 1, 0, 2, 175 * 46, 46, 16, 1400, 4, 26, 114, 3, 34, FORK_BACKWARD, 1, true);
  expect(0, 1, 0, 2, 175 * 46, 46, 16, 1400, 4, 26, 114, 3, 34, FORK_BACKWARD, 0, false);
  // 965 points in fp32, 25 modes, rank 22 x 8: recorded 198, 248, launched 239, 264
  expect(0, 0, 1, 1, 965, 965, 32, 25, 5, 35, 118, 22, 8, FORK_BACKWARD, 1, true);
  expect(0, 0, 1, 1, 965, 965, 32, 25, 5, 35, 118, 22, 8, FORK_BACKWARD, 0, true);
  // 125 x 390, 40 x 128 modes, rank 21 x 5: launched 393, 455; weight gradient 167, 141
  expect(0, 1, 1, 2, 125 * 390, 390, 128, 5120, 2, 25, 14, 21, 5, FORK_BACKWARD, 0, true);
  expect(0, 1, 1, 2, 125 * 390, 390, 128, 5120, 2, 25, 14, 21, 5, FORK_WGRAD, 0, false);
  // 128 x 128, 64 x 32 modes, CP rank 16, 32 samples of 64 channels: launched 212, 170,
  // recorded 155, 167; weight gradient 125, 78
  expect(1, 1, 0, 2, 128 * 128, 128, 32, 2048, 32, 64, 64, 16, 16, FORK_BACKWARD, 0, false);
  expect(1, 1, 0, 2, 128 * 128, 128, 32, 2048, 32, 64, 64, 16, 16, FORK_BACKWARD, 1, true);
  expect(1, 1, 0, 2, 128 * 128, 128, 32, 2048, 32, 64, 64, 16, 16, FORK_WGRAD, 0, false);
  // 256 x 256, 64 x 32 modes, rank 13 x 13, 16 samples of 128 channels: launched 374, 472,
  // recorded 342, 469; forward 227, 242
  for (bool rec : {false, true}) {
    expect(0, 1, 0, 2, 65536, 256, 32, 2048, 16, 128, 128, 13, 13, FORK_BACKWARD, rec, true);
    expect(0, 1, 0, 2, 65536, 256, 32, 2048, 16, 128, 128, 13, 13, FORK_PATH, rec, true);
  }
  // 8 x 160, 6 x 70 modes, 10 samples of 26 to 24 channels (the recorded calls of the
  // GPU test of graphs)
  for (bool cp : {false, true}) {
    expect(cp, 1, 1, 2, 1280, 160, 128, 420, 10, 26, 24, 8, 6, FORK_BACKWARD, 1, true);
    expect(cp, 1, 1, 2, 1280, 160, 128, 420, 10, 26, 24, 8, 6, FORK_PATH, 1, !cp);
    expect(cp, 1, 1, 2, 1280, 160, 128, 420, 10, 26, 24, 8, 6, FORK_BACKWARD, 0, false);
  }
  // few points: on one stream
  for (ForkCall c : {FORK_PATH, FORK_BACKWARD, FORK_WGRAD})
    for (bool rec : {false, true}) {
      expect(0, 1, 0, 1, 256, 256, 16, 16, 8, 16, 16, 4, 4, c, rec, false);
      expect(1, 1, 0, 2, 64 * 64, 64, 16, 512, 2, 16, 16, 8, 8, c, rec, false);
    }
  return bad;""")


def test_mixes_of_few_channels(tmp_path):
    """As measured: channels in and out, points."""
    replay(tmp_path, """
  int bad = 0;
  bad += !few_channels(1, 1, 120002) + !few_channels(1, 1, 116) + !few_channels(2, 4, 120002);
  bad += !few_channels(2, 128, 11300) + !few_channels(4, 128, 2408) + !few_channels(3, 2, 57860);
  bad += few_channels(2, 128, 57860) + few_channels(8, 20, 116) + few_channels(4, 4, 11300);
  bad += few_channels(1, 64, 120002) + few_channels(64, 64, 2450) + few_channels(6, 64, 2408);
  return bad;""")
