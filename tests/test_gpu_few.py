"""GPU parity of calls with few planes or signals, which keep the kernels that
start soonest (the small-plane ones up to 128 x 256, the generic ones), against
the float64 oracle; each case names the kernels that it is about."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

import synth  # noqa: E402
from oracle import fno_oracle as O  # noqa: E402

if torch.cuda.is_available():
    from tests import gpu_util as U

CASES = [
    # (n, modes, B, Cin, Cout, storage, forward kernel, inverse kernel)
    ((72, 72), (10, 20), 2, 3, 4, "fp16", "r2c_fast_kernel<4, 4, 8>", "c2r_fast_kernel<4, 8, 2, 1"),
    ((72, 72), (10, 18), 2, 16, 8, "fp16", "r2c_fast_kernel<4, 4, 8>", None),
    ((40, 72), (6, 12), 1, 3, 3, "fp16", None, "c2r_fast_kernel<2, 4, 2, 1"),
    ((64, 128), (12, 5), 1, 4, 3, "fp16", "r2c_fast_kernel<2, 4, 4>", None),
    ((104, 96), (7, 11), 1, 4, 3, "fp16", "r2c_fast_kernel<2, 4, 8>", None),
    ((33, 120), (7, 19), 1, 4, 3, "fp16", "r2c_fast_kernel<4, 4, 4>", None),
    ((64, 256), (10, 18), 1, 3, 2, "fp16", "r2c_fast_kernel<4, 8, 4>", None),
    ((100, 104), (9, 24), 1, 3, 3, "fp16", None, "c2r_fast_kernel<4, 8, 2, 1"),
    ((100, 104), (17, 24), 1, 3, 3, "fp16", None, "c2r_fast_kernel<4, 8, 2, 2"),
    ((128, 104), (7, 35), 2, 3, 3, "fp16", "r2c_fast_kernel<8, 4, 8>", None),
    ((128, 80), (3, 12), 20, 16, 16, "fp16", None, None),     # 320 planes: past the forward's line
    ((16, 264), (8, 5), 16, 16, 16, "fp16", None, "c2r_plane_kernel"),
    ((15, 43), (5, 5), 1, 16, 16, "fp16", "r2c_plane_kernel", "c2r_plane_kernel"),
    ((24, 24), (4, 5), 2, 16, 16, "fp32", "r2c_plane_kernel", "c2r_plane_kernel"),
    ((30, 200), (3, 5), 1, 16, 16, "fp32", "r2c_plane_kernel", None),
    ((19, 131), (4, 35), 1, 4, 3, "fp32", "r2c_plane_kernel", "c2r_any32_kernel"),
    ((64, 129), (10, 64), 2, 3, 3, "fp32", "r2c_plane_kernel", "c2r_any32_kernel"),
    ((64,), (5,), 2, 16, 16, "fp16", "r2c_fast_kernel<2, 2, 4>", "c2r_line_kernel"),
    ((128,), (18,), 2, 16, 16, "fp16", "r2c_fast_kernel<4, 4, 4>", "c2r_line_kernel"),
    ((50,), (7,), 2, 16, 16, "fp16", "r2c_plane_kernel", "c2r_line_kernel"),
]


@pytest.mark.parametrize("act", ["tanh", "none"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_few(case, act):
    n, m, bt, ci, co, store, fwd, inv = CASES[case]
    mode = {"fp16tanh": "fp16_tanh", "fp16none": "fp16", "fp32tanh": "fp32_tanh",
            "fp32none": "fp32"}[store + act]
    U.say(f"few case {case}: n={n} modes={m} B={bt} C={ci}->{co} {mode}")
    npdt = np.float16 if store == "fp16" else np.float32
    x, w, gy = synth.random_dense_case(1100 + case, bt, ci, co, n, m, npdt)
    layer = U.make_layer(n, m, bt, ci, co, mode)
    y, gx, gw = U.run_all(layer, x, w, gy)
    wc = U.cplx(w)
    for name, a, b in (("y", y, O.fwd(x, wc, n, m, mode)),
                       ("gx", gx, O.bwd_data(x, wc, gy, n, m, mode)),
                       ("gW", U.cplx(gw), O.bwd_weight(x, gy, n, m, mode))):
        assert U.rel(a, b) <= U.TOL[mode], (name, U.rel(a, b))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        U.check_routes(layer, x, w, gy, fwd, inv)
