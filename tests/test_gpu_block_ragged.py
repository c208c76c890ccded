"""GPU parity of the fp16 block epilogue on channel rows that are not a
multiple of eight points (16-byte accesses at any two-byte address), at the
edges of pieces and of 64-point tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

from oracle import fno_oracle as O  # noqa: E402
import synth  # noqa: E402
from tests import gpu_util as U  # noqa: E402
from paper_2307_15034_amd import binding as B  # noqa: E402
from paper_2307_15034_amd.layer import BlockEpilogue  # noqa: E402

CASES = [
    # (points, B, Cin, Cout, residual)
    (7, 3, 4, 4, True),        # fewer than one piece: generic kernels
    (9, 3, 5, 6, False),       # last piece holds one point
    (63, 2, 16, 16, True),     # one tile, last piece holds seven
    (65, 2, 17, 30, False),    # second tile holds one point
    (129, 3, 33, 64, False),   # odd channel counts, two output tiles per wave
    (1225, 4, 128, 128, True),
    (4097, 2, 64, 64, True),
    (301, 3, 1, 1, True),      # few channels: the kernels without matrix cores
    (301, 2, 2, 128, False),   # forward so, data gradient pipelined
    (301, 2, 128, 2, False),   # and the other way round
    # skip weights whose rows are not a multiple of eight, aligned points
    (248, 12, 20, 128, False),  # pieces run over rows, 320 of them
    (64, 2, 1, 1, True),        # less than one piece
    (72, 3, 3, 5, False),       # one piece and seven values
    (128, 2, 127, 127, True),   # 16129 values: eight pieces a thread
    (128, 2, 121, 8, False),    # one direction by rows, the other by runs
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_ragged_epilogue(case):
    pts, bt, ci, co, res = CASES[case]
    U.say(f"ragged epilogue {case}: points={pts} B={bt} {ci}->{co}")
    grid = (pts,)
    epi = BlockEpilogue(grid, bt, ci, co, B.FNO_PREC_FP16_TANH, B.FNO_EPI_ACT_GELU, res)
    x, y, w, b, g = synth.random_block_case(300 + case, bt, ci, co, grid, np.float16)
    gxs = synth.random_block_case(400 + case, bt, ci, ci, grid, np.float16)[0]
    xd, yd, wd, bd, gd, gxsd = (U.dev(t) for t in (x, y, w, b, g, gxs))
    out, z = epi.fwd(xd, yd, wd, bd)
    gz, gw, gb = epi.bwd_weight(xd, z, gd)
    gx = epi.bwd_data(gz, wd, gxsd, gd if res else None)
    gx_in = epi.bwd_data(gz, wd, gxsd, gd if res else None, gx=gxsd)  # in place
    torch.cuda.synchronize()
    assert torch.equal(gx, gx_in)
    act = O.EPI_ACT_GELU
    r_out, r_z = O.block_epilogue_fwd(x, y, w, b, act, res)
    r_gz, r_gx, r_gw, r_gb = O.block_epilogue_bwd(x, r_z, g, w, act, res)
    for name, got, ref in (("out", out, r_out), ("z", z, r_z), ("g_z", gz, r_gz),
                           ("gx", gx, r_gx + gxs.astype(np.float64)), ("g_w", gw, r_gw),
                           ("g_b", gb, r_gb)):
        r = U.rel(U.host(got), ref)
        assert np.isfinite(r) and r <= U.TOL["fp16_tanh"], (name, r)
