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
