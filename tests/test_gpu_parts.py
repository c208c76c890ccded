"""GPU parity of the fp16 plane transforms where several work-groups share a
plane's rows (large planes, fewer than half as many as compute units): against
the float64 oracle, and against the call whose output lies in its input's
memory (one work-group per plane then)."""
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
    ((512, 256), (20, 20), 2, 3, 3),     # radix-2 kernels, two parts of one chunk
    ((1024, 512), (64, 64), 1, 2, 2),    # four parts, 128-column blocks in the inverse
    ((768, 256), (8, 12), 1, 30, 30),    # three chunks: three parts
    ((2048, 256), (8, 12), 3, 14, 14),   # eight chunks, 42 planes: four parts of two chunks
    ((257, 257), (6, 6), 1, 3, 3),       # any extents: the second part holds one row
    ((1300, 40), (64, 20), 1, 50, 50),   # six chunks, 50 planes: parts of two chunks
    ((520, 300), (50, 30), 2, 2, 2),     # three chunks of any extents
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_parts_parity(case):
    n, m, bt, ci, co = CASES[case]
    U.say(f"parts case {case}: n={n} modes={m} B={bt} C={ci}->{co}")
    x, w, gy = synth.random_dense_case(900 + case, bt, ci, co, n, m, np.float16)
    layer = U.make_layer(n, m, bt, ci, co, "fp16_tanh")
    y, gx, gw = U.run_all(layer, x, w, gy)
    wc = U.cplx(w)
    for name, a, b in (("y", y, O.fwd(x, wc, n, m, "fp16_tanh")),
                       ("gx", gx, O.bwd_data(x, wc, gy, n, m, "fp16_tanh")),
                       ("gW", U.cplx(gw), O.bwd_weight(x, gy, n, m, "fp16_tanh"))):
        assert U.rel(a, b) <= U.TOL["fp16_tanh"], (name, U.rel(a, b))
    names = U.kernels(lambda: layer.fwd(U.dev(x), U.dev(w)))
    assert not names or any("part_sum_kernel" in k for k in names), names
    # the combined backward, with and without the cached spectrum
    xd, wd, gyd = U.dev(x), U.dev(w), U.dev(gy)
    xh = layer.spectrum_buffer(0)
    layer.fwd(xd, wd, x_hat=xh)
    for cache in (xh, None):
        gx2, gw2 = layer.bwd(xd, wd, gyd, x_hat=cache)
        assert U.rel(U.host(gx2), gx.astype(np.float64)) <= 1e-3
        assert U.rel(U.host(gw2), gw.astype(np.float64)) <= 1e-3
    # outputs in the inputs' memory: the transforms take no memory of the output
    yin = xd.clone()
    layer.fwd(yin, wd, y=yin)
    assert U.rel(U.host(yin), y.astype(np.float64)) <= 1e-3
    gin = gyd.clone()
    layer.bwd_data(xd, wd, gin, gx=gin)
    assert U.rel(U.host(gin), gx.astype(np.float64)) <= 1e-3
