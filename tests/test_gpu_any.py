"""GPU parity of the fp16 plane transforms for any extents (rows at any
two-byte address, last axis in segments, 1 to 8 waves per plane) against the
float64 oracle, at the edges of segments, row blocks, chunks, mode tiles and
16-byte pieces."""
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
    ((5, 12), (2, 3), 60, 20, 18),      # two pieces per row, eight planes per work-group
    ((33, 9), (3, 5), 40, 20, 20),      # second row block holds one row; Nyquist-free odd rows
    ((64, 63), (17, 7), 26, 20, 20),    # two waves per plane, 34 leading slots
    ((65, 65), (8, 33), 1, 4, 3),       # second segment holds one column, four mode tiles
    ((127, 129), (24, 17), 3, 3, 4),    # four waves, 48 leading slots (three tiles)
    ((129, 127), (40, 21), 1, 3, 3),    # eight waves, 80 leading slots (five tiles)
    ((256, 131), (64, 13), 1, 2, 2),    # all eight row blocks, 128 leading slots
    ((257, 257), (6, 64), 1, 2, 2),     # second chunk holds one row, four mode tiles
    ((300, 250), (50, 30), 1, 2, 3),    # two chunks, rows on 4-byte addresses
    ((700, 44), (64, 22), 1, 2, 2),     # three chunks, tables too large for LDS
    ((20, 1001), (5, 6), 2, 3, 3),      # eight segments, the last of 105 columns
    ((241, 241), (20, 20), 3, 60, 50),  # more planes than work-groups
    ((31, 41), (9, 11), 18, 120, 60),   # one wave per plane, several planes per wave
    ((7, 21, 35), (2, 5, 9), 10, 12, 12),  # 3-D
]


@pytest.mark.parametrize("mode", ["fp16_tanh", "fp16", "fp16_clip:1.5"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_any_parity(case, mode):
    n, m, bt, ci, co = CASES[case]
    U.say(f"any case {case}: n={n} modes={m} B={bt} C={ci}->{co} {mode}")
    x, w, gy = synth.random_dense_case(800 + case, bt, ci, co, n, m, np.float16)
    layer = U.make_layer(n, m, bt, ci, co, mode)
    y, gx, gw = U.run_all(layer, x, w, gy)
    wc = U.cplx(w)
    ry = O.fwd(x, wc, n, m, mode)
    rgx = O.bwd_data(x, wc, gy, n, m, mode)
    rgw = O.bwd_weight(x, gy, n, m, mode)
    for name, a, b in (("y", y, ry), ("gx", gx, rgx), ("gW", U.cplx(gw), rgw)):
        assert U.rel(a, b) <= U.TOL[mode], (name, U.rel(a, b))
    U.check_routes(layer, x, w, gy, "r2c_any_kernel", "c2r_any_kernel")


@pytest.mark.parametrize("n", [(65, 81), (130, 137)])
def test_any_nonfinite_stays_in_its_plane(n):
    """NaN and inf in one plane (its first and last samples share 16-byte
    pieces and 4-byte words with the neighbouring planes) leave the others
    finite; tanh of inf is finite."""
    m = (3, 5)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((4, 1) + n).astype(np.float16)  # one channel: no mixing
    x[1, 0, 0, 0] = x[1, 0, -1, -1] = np.nan
    x[3, 0, 0, 0] = x[3, 0, -1, -1] = np.inf
    w = np.zeros((1, 1, 2 * m[0], m[1], 2), np.float16)
    w[..., 0] = 1.0
    gy = rng.standard_normal((4, 1) + n).astype(np.float16)
    layer = U.make_layer(n, m, 4, 1, 1, "fp16_tanh")
    y, gx, _ = U.run_all(layer, x, w, gy)
    U.check_routes(layer, x, w, gy, "r2c_any_kernel", "c2r_any_kernel")
    assert np.isnan(y[1]).all() and np.isfinite(y[[0, 2, 3]]).all()
    assert np.argwhere(~np.isfinite(gx)).tolist() == [[1, 0, 0, 0], [1, 0, n[0] - 1, n[1] - 1]]
    y, _, _ = U.run_all(U.make_layer(n, m, 4, 1, 1, "fp16"), x, w, gy)
    assert np.isfinite(y[[0, 2]]).all() and not np.isfinite(y[[1, 3]]).any()


def test_any_planes_of_more_than_half_a_gibibyte():
    """Offsets past 2^29 bytes, an odd mode count and a row length that the
    radix-2 kernels do not take: the spectrum against float64 products over the
    whole plane, the inverse and its tanh' epilogue on sampled rows."""
    n, m = (16640, 16512), (3, 18)  # 549 MB a plane
    U.say(f"any large plane: n={n} modes={m}")
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((1, 1) + n, device="cuda", generator=g).half()
    for j in range(2):  # low modes well above the rounding of the stored spectrum
        ph = 2 * np.pi / n[j] * torch.arange(n[j], device="cuda", dtype=torch.float64)
        x += (torch.cos(ph) + torch.sin(2 * ph)).half().reshape((-1, 1) if j == 0 else (-1,))
    gy = torch.randn((1, 1) + n, device="cuda", generator=g).half()
    w = torch.zeros((1, 1, 2 * m[0], m[1], 2), device="cuda").half()
    w[..., 0] = 1.0
    layer = U.make_layer(n, m, 1, 1, 1, "fp16_tanh")
    xh, gh = layer.spectrum_buffer(0), layer.spectrum_buffer(1)
    y = layer.fwd(x, w, x_hat=xh)
    gx = layer.bwd_data(x, w, gy, gy_hat=gh)
    torch.cuda.synchronize()

    def dft(k, length):
        p = (k[:, None] * torch.arange(length, device="cuda")) % length
        return torch.polar(torch.ones((), device="cuda", dtype=torch.float64),
                           p.double() * (-2 * np.pi / length))

    ka = torch.tensor([0, 1, 2, n[0] - 3, n[0] - 2, n[0] - 1], device="cuda")
    fa, fb = dft(ka, n[0]), dft(torch.arange(m[1], device="cuda"), n[1])

    def spectrum(v):
        t = torch.stack([v @ fb.real.T.contiguous(), v @ fb.imag.T.contiguous()])
        return fa @ torch.complex(t[0], t[1])

    def check(name, got, ref):
        r = float(torch.linalg.vector_norm(got - ref) / torch.linalg.vector_norm(ref))
        U.say(f"  {name}: rel_l2 {r:.2e}")
        assert r <= U.TOL["fp16_tanh"], name

    def stored(h):
        return torch.view_as_complex(h.view(torch.float16).reshape(2 * m[0], m[1], 2).double())

    check("x_hat", stored(xh), spectrum(torch.tanh(x[0, 0].double())) / (n[0] * n[1]))
    check("gy_hat", stored(gh), spectrum(gy[0, 0].double()) / (n[0] * n[1]) ** 0.5)
    rows = torch.tensor([0, 1, 8191, 8192, 12345, n[0] - 2, n[0] - 1], device="cuda")
    c = torch.tensor([1.0] + [2.0] * (m[1] - 1), device="cuda", dtype=torch.float64)

    def inverse(z):
        t = fa[:, rows].T.conj() @ (z * c)
        return (t @ fb.conj()).real

    check("y", y[0, 0, rows].double(), inverse(stored(xh)))
    dt = 1 - torch.tanh(x[0, 0, rows].double()) ** 2
    check("gx", gx[0, 0, rows].double(), inverse(stored(gh)) * dt / (n[0] * n[1]) ** 0.5)
    gyd = gy.cpu().numpy()
    U.check_routes(layer, x.cpu().numpy(), w.cpu().numpy(), gyd, "r2c_any_kernel", "c2r_any_kernel")
