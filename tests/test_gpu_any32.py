"""GPU parity of the fp32 plane transforms for any extents (even axes folded,
last axis in segments, 1 to 8 waves per plane, planes shared by several
work-groups) against the float64 oracle at their edges."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import fno_oracle as O  # noqa: E402

if torch.cuda.is_available():
    from tests import gpu_util as U

CASES = [
    # (n, modes, B, Cin, Cout)
    ((5, 8), (2, 3), 40, 30, 28),       # odd rows, one piece
    ((6, 9), (3, 5), 60, 20, 18),       # folded rows, odd columns, a wave per plane
    ((34, 38), (17, 18), 20, 20, 15),   # both folded: 17 row pairs, 19 columns a half
    ((33, 130), (8, 33), 9, 30, 29),    # second segment of a half holds one column
    ((64, 66), (32, 34), 10, 26, 26),   # every mode retained, four mode tiles
    ((70, 33), (24, 17), 2, 3, 3),      # 24 slots a class (two tiles of 16)
    ((257, 64), (6, 20), 1, 2, 2),      # second chunk holds one row
    ((600, 131), (64, 64), 1, 2, 2),    # folded rows over two chunks, 128 slots
    ((1030, 40), (5, 6), 1, 3, 3),      # few planes: five parts
    ((512, 512), (21, 35), 1, 3, 2),    # two parts, folded, 64-mode tiles
    ((128, 128), (32, 32), 2, 20, 17),
    ((20, 24), (4, 5), 18, 120, 58),    # several planes per wave
    ((7, 20, 36), (2, 5, 18), 10, 15, 15),  # 3-D
]


@pytest.mark.parametrize("mode", ["fp32", "fp32_tanh", "fp32_clip:1.5"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_any32_parity(case, mode):
    n, m, bt, ci, co = CASES[case]
    U.say(f"any32 case {case}: n={n} modes={m} B={bt} C={ci}->{co} {mode}")
    x, w, gy = synth.random_dense_case(600 + case, bt, ci, co, n, m, np.float32)
    layer = U.make_layer(n, m, bt, ci, co, mode)
    y, gx, gw = U.run_all(layer, x, w, gy)
    wc = U.cplx(w)
    for name, a, b in (("y", y, O.fwd(x, wc, n, m, mode)),
                       ("gx", gx, O.bwd_data(x, wc, gy, n, m, mode)),
                       ("gW", U.cplx(gw), O.bwd_weight(x, gy, n, m, mode))):
        # 32-bit sums of a few hundred terms: well inside the gate of 1e-5
        assert U.rel(a, b) <= 2e-6, (name, U.rel(a, b))
    U.check_routes(layer, x, w, gy, "r2c_any32_kernel", "c2r_any32_kernel")


def test_any32_nonfinite_stays_in_its_plane():
    n, m = (130, 137), (3, 5)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((3, 1) + n).astype(np.float32)
    x[1, 0, 0, 0] = x[1, 0, -1, -1] = np.nan
    w = np.zeros((1, 1, 2 * m[0], m[1], 2), np.float32)
    w[..., 0] = 1.0
    layer = U.make_layer(n, m, 3, 1, 1, "fp32")
    gy = rng.standard_normal((3, 1) + n).astype(np.float32)
    y, _, _ = U.run_all(layer, x, w, gy)
    U.check_routes(layer, x, w, gy, "r2c_any32_kernel", "c2r_any32_kernel")
    assert np.isnan(y[1]).all() and np.isfinite(y[[0, 2]]).all()
