"""GPU parity of the pairwise steps of factorised weights at their edges: steps
batched over the last mode axis (four modes per wave, tiles of 16, contraction
steps of 16 and 32), GEMM stages that end in a partial stage, the fused CP
weight-gradient kernels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from oracle import fno_oracle as O  # noqa: E402

if torch.cuda.is_available():
    from tests import gpu_util as U

CASES = [
    # (n, modes, B, Cin, Cout, R), paths for min_result
    ((32, 32), (8, 12), 32, 36, 20, 17),   # b i x y, x i o y: K = 36 (partial step), M = 32
    ((64, 40), (16, 16), 16, 64, 64, 9),   # the same, whole tiles
    ((20, 10), (4, 4), 40, 36, 36, 5),     # b x r y from i r x y: 5 of 16 columns, K = 5
    ((128, 64), (32, 32), 17, 64, 64, 16),  # i r y and o r x factors, 17 samples
    ((32, 32), (8, 11), 32, 36, 20, 17),   # 11 modes: no quads, GEMM tiles
    ((300,), (61,), 3, 20, 9, 6),          # one axis: a single row of 61 modes
    ((140, 8), (64, 3), 2, 5, 6, 4),       # 128 rows of 3 columns
    ((10, 140), (3, 64), 5, 5, 6, 3),      # 6 rows of 64 columns
    ((6, 10, 12), (2, 3, 4), 2, 3, 2, 5),  # three axes
]


@pytest.mark.parametrize("policy", ["min_result", "min_net"])
@pytest.mark.parametrize("prec", ["fp32", "fp16_tanh"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_cp_steps(case, prec, policy):
    n, modes, bt, ci, co, r = CASES[case]
    _, npdt, oprec = U.prec_codes(prec)
    U.say(f"cp steps {case}: n={n} modes={modes} B={bt} C={ci}->{co} R={r} {prec} {policy}")
    rng = np.random.default_rng(np.random.SeedSequence([4000 + case]))
    d = len(n)
    kd = tuple(2 * m if j < d - 1 else m for j, m in enumerate(modes))

    def cpx(shape):
        return (rng.standard_normal(tuple(shape) + (2,)) * 0.5).astype(npdt)

    w = {"core": cpx((r,)), "u_in": cpx((ci, r)), "u_out": cpx((co, r)),
         "u_mode": [cpx((kd[j], r)) for j in range(d)]}
    x = rng.standard_normal((bt, ci) + n).astype(npdt)
    gy = rng.standard_normal((bt, co) + n).astype(npdt)
    layer = U.make_layer(n, modes, bt, ci, co, prec, policy=0 if policy == "min_result" else 1,
                         cp_rank=r)
    y, gx, gw = U.run_all(layer, x, w, gy)
    lam, u_in, u_out = U.cplx(w["core"]), U.cplx(w["u_in"]), U.cplx(w["u_out"])
    u_mode = [U.cplx(u) for u in w["u_mode"]]
    args = (lam, u_in, u_out, u_mode)
    g_lam, g_in, g_out, g_mode = O.cp_bwd_weight(x, gy, *args, n, modes, oprec)
    gwc = U.gw_complex(gw)
    pairs = [("y", y, O.cp_fwd(x, *args, n, modes, oprec, policy)),
             ("gx", gx, O.cp_bwd_data(x, *args, gy, n, modes, oprec, policy)),
             ("g_lambda", gwc["core"], g_lam), ("g_u_in", gwc["u_in"], g_in),
             ("g_u_out", gwc["u_out"], g_out)]
    pairs += [(f"g_u_mode{j}", gwc["u_mode"][j], g_mode[j]) for j in range(d)]
    for name, got, ref in pairs:
        e = U.rel(got, ref)
        U.say(f"  {name}: rel_l2 = {e:.3e} (tol {U.TOL[prec]:.0e})")
        assert np.isfinite(e) and e <= U.TOL[prec], name


TUCKER = [
    # (n, modes, B, Cin, Cout, ranks, a kernel that a call of it runs: its names)
    # 12 contracted elements of 64 rows: the last quad of a stage lies past them
    ((32, 32), (8, 12), 4, 36, 64, (8, 12, 5, 3), ("pair_gemm_kernel<64, 64, 2, true, true, 16>",)),
    ((32, 32), (8, 12), 5, 36, 64, (20, 24, 4, 4), ("pair_quad_kernel<32>",)),
    # outer products of more than 1.3 million results: four per thread
    ((64, 64), (32, 32), 2, 128, 128, (13, 13, 6, 3),
     ("pair_ew_kernel<4", "pair_ew_kernelILi4")),
]


@pytest.mark.parametrize("policy", ["min_result", "min_net"])
@pytest.mark.parametrize("prec", ["fp32", "fp16_tanh"])
@pytest.mark.parametrize("case", range(len(TUCKER)))
def test_tucker_steps(case, prec, policy):
    n, modes, bt, ci, co, rank, kernel = TUCKER[case]
    _, npdt, oprec = U.prec_codes(prec)
    U.say(f"tucker steps {case}: n={n} modes={modes} B={bt} C={ci}->{co} R={rank} {prec} {policy}")
    rng = np.random.default_rng(np.random.SeedSequence([4100 + case]))
    kd = (2 * modes[0], modes[1])

    def cpx(shape):
        return (rng.standard_normal(tuple(shape) + (2,)) * 0.3).astype(npdt)

    w = {"core": cpx(rank), "u_in": cpx((ci, rank[0])), "u_out": cpx((co, rank[1])),
         "u_mode": [cpx((k, r)) for k, r in zip(kd, rank[2:])]}
    x = rng.standard_normal((bt, ci) + n).astype(npdt)
    gy = rng.standard_normal((bt, co) + n).astype(npdt)
    layer = U.make_layer(n, modes, bt, ci, co, prec, policy=0 if policy == "min_result" else 1,
                         tucker_rank=rank)
    y, gx, gw = U.run_all(layer, x, w, gy)
    args = (U.cplx(w["core"]), U.cplx(w["u_in"]), U.cplx(w["u_out"]),
            [U.cplx(u) for u in w["u_mode"]])
    g_core, g_in, g_out, g_mode = O.tucker_bwd_weight(x, gy, *args, n, modes, oprec)
    gwc = U.gw_complex(gw)
    pairs = [("y", y, O.tucker_fwd(x, *args, n, modes, oprec, policy)),
             ("gx", gx, O.tucker_bwd_data(x, *args, gy, n, modes, oprec, policy)),
             ("g_core", gwc["core"], g_core), ("g_u_in", gwc["u_in"], g_in),
             ("g_u_out", gwc["u_out"], g_out)]
    pairs += [(f"g_u_mode{j}", gwc["u_mode"][j], g_mode[j]) for j in range(2)]
    for name, got, ref in pairs:
        e = U.rel(got, ref)
        U.say(f"  {name}: rel_l2 = {e:.3e} (tol {U.TOL[prec]:.0e})")
        assert np.isfinite(e) and e <= U.TOL[prec], name
    if prec == "fp16_tanh" and policy == "min_result":
        xd, gyd = U.dev(x), U.dev(gy)
        wd = {k: [U.dev(u) for u in v] if isinstance(v, list) else U.dev(v) for k, v in w.items()}
        names = U.kernels(lambda: (layer.fwd(xd, wd), layer.bwd(xd, wd, gyd)))
        U.say(" ".join(names))
        assert not names or any(q in k for k in names for q in kernel), names
