"""GPU parity of the 1-D fp16 transforms (signals read as rows of 128 samples
in blocks of 4096; waves share a signal when there are few) against the
float64 oracle, at the edges of rows, blocks, 16-byte pieces and mode tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import fno_oracle as O  # noqa: E402

if torch.cuda.is_available():
    from tests import gpu_util as U

CASES = [
    # (N, modes, B, Cin, Cout)
    (8, 3, 60, 20, 18),        # one 16-byte piece
    (9, 5, 60, 20, 18),        # every second signal starts off a 4-byte address
    (127, 64, 30, 18, 18),     # one partial row, four mode tiles, all modes
    (257, 17, 3, 5, 7),        # third row holds one sample
    (1000, 1, 2, 17, 18),      # more than one 16-signal tile, one mode
    (4096, 32, 2, 9, 9),       # exactly one block
    (4101, 33, 1, 3, 3),       # second block holds five samples
    (8192, 32, 3, 40, 48),     # more signals than two waves per SIMD share out
    (33001, 100, 1, 3, 2),     # nine blocks over eight waves, widest mode tile
    (65536, 20, 1, 2, 2),      # the longest signal
]


@pytest.mark.parametrize("mode", ["fp16_tanh", "fp16", "fp16_clip:1.5"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_line_parity(case, mode):
    n, m, bt, ci, co = CASES[case]
    U.say(f"line case {case}: N={n} modes={m} B={bt} C={ci}->{co} {mode}")
    x, w, gy = synth.random_dense_case(700 + case, bt, ci, co, (n,), (m,), np.float16)
    layer = U.make_layer((n,), (m,), bt, ci, co, mode)
    y, gx, gw = U.run_all(layer, x, w, gy)
    wc = U.cplx(w)
    ry = O.fwd(x, wc, (n,), (m,), mode)
    rgx = O.bwd_data(x, wc, gy, (n,), (m,), mode)
    rgw = O.bwd_weight(x, gy, (n,), (m,), mode)
    for name, a, b in (("y", y, ry), ("gx", gx, rgx), ("gW", U.cplx(gw), rgw)):
        assert U.rel(a, b) <= U.TOL[mode], (name, U.rel(a, b))
    U.check_routes(layer, x, w, gy, "r2c_line_kernel", "c2r_line_kernel")


def test_line_nonfinite_stays_in_its_signal():
    """A NaN spoils its own signal's spectrum only (rows are read across
    16-byte pieces that neighbouring signals share)."""
    n, m = 2051, 9
    rng = np.random.default_rng(3)
    x = rng.standard_normal((4, 1, n)).astype(np.float16)  # one channel: no mixing
    x[1, 0, 0] = np.nan
    x[1, 0, n - 1] = np.nan
    w = np.zeros((1, 1, m, 2), np.float16)
    w[..., 0] = 1.0
    layer = U.make_layer((n,), (m,), 4, 1, 1, "fp16_tanh")
    y, gx, _ = U.run_all(layer, x, w, rng.standard_normal((4, 1, n)).astype(np.float16))
    assert np.isnan(y[1]).all()
    assert np.isfinite(y[[0, 2, 3]]).all()
    bad = np.argwhere(~np.isfinite(gx))
    assert bad.tolist() == [[1, 0, 0], [1, 0, n - 1]]
