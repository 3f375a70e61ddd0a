"""The deposit's tile by the columns that a block spans (few particles per
cell), against the FP64 oracle: cell-sorted sets of 1 to 12 particles per cell
on both sides of the rule, whose blocks wrap from one theta row to the next or
reach over both axes and the radial edges, the same sets with some order lost,
and blocks too wide for any tile.  The same for the Gauss residual's charge
pass.  Fused and separate, double precision to the bars of test_gpu_parity.py; single precision against the double-precision
deposit of the same moves, to 200 roundings of a plane's largest value (a
node takes that many additions at most)."""
import numpy as np
import pytest

from test_gpu_parity import G, assert_fields, assert_particles, down, pair, up, wl  # noqa: F401

pytestmark = pytest.mark.gpu


def _state(O, prm, w, ppc, kind, seed):
    n_r, n_th = prm.n_r, prm.n_th
    F = O.fields_init_wald(prm, w.B0)
    P = O.particles_init(prm, int(n_r * n_th * ppc) // 2, 0, 1.0, 0, seed)
    g = np.random.default_rng(seed)
    if kind == "edges":  # the cells beside the axes and the radial edges
        k = len(P["tag"])
        P["i1"][: k // 4] = np.where(g.random(k // 4) < 0.5, 0, n_r - 1)
        P["i2"][k // 4: k // 2] = np.where(g.random(k // 2 - k // 4) < 0.5, 0, n_th - 1)
    order = np.argsort(P["i1"].astype(np.int64) * n_th + P["i2"], kind="stable")
    if kind == "moved":  # neighbours a few slots apart, one in twenty anywhere
        key = np.arange(len(order)) + g.normal(scale=20.0, size=len(order))
        far = g.random(len(order)) < 0.05
        key[far] = g.uniform(0, len(order), far.sum())
        order = order[np.argsort(key)]
    P = {q: np.ascontiguousarray(v[order]) for q, v in P.items()}
    P["tag"][::9] = 0  # dead slots among them
    return F, P


@pytest.mark.parametrize("kind", ["sorted", "edges", "moved"])
@pytest.mark.parametrize("n_r,n_th,ppc", [(12, 512, 0.3), (24, 200, 1), (16, 150, 2), (24, 40, 2), (20, 64, 3.3),
                                         (9, 9, 4), (24, 33, 10.9), (24, 33, 12)])
def test_sparse_deposit(O, G, n_r, n_th, ppc, kind):
    w = wl("c2_512").scaled(n_r, n_th)
    prm, ctx = pair(O, G, w, charge_scale=0.3)
    F, P = _state(O, prm, w, ppc, kind, 3)
    F_f, P_f = up({"F": F})["F"], up(P)
    F32, P32 = up({"F": F})["F"].float(), {q: (v.float() if v.is_floating_point() else v) for q, v in up(P).items()}
    O.push(prm, F, P)
    F_d, P_d = up({"F": F})["F"], up(P)
    O.deposit(prm, F, P)
    ctx.push_deposit(F_f, P_f)
    ctx.deposit(P_d, F_d)
    assert_particles(prm, P, down(P_f), what="fused", prev=False)
    assert_fields(F, F_f.cpu().numpy(), range(18, 21), what="fused J")
    assert_fields(F, F_d.cpu().numpy(), range(18, 21), what="J")

    c32 = G.Context(w.a, w.M, w.r_min, w.r_max, n_r, n_th, dt=ctx.dt, charge_scale=0.3, precision=G.GRPIC_FP32)
    A, B = c32.new_fields(), c32.new_fields()
    A[:33] = F32
    B[:33] = F32
    Q = {q: v.clone() for q, v in P32.items()}
    c32.push_deposit(A, P32)
    c32.push(B, Q)
    c32.deposit(Q, B)
    ref = up({"F": np.zeros_like(F)})["F"]
    ctx.deposit({q: (v.double() if v.is_floating_point() else v) for q, v in Q.items()}, ref)
    for c in range(18, 21):
        scale = ref[c].abs().max().item()
        for name, X in (("fused", A), ("separate", B)):
            assert (X[c].double() - ref[c]).abs().max().item() <= 200 * 2.0 ** -24 * scale, (name, c)


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("kind", ["sorted", "edges", "moved"])
@pytest.mark.parametrize("n_r,n_th,ppc", [(12, 800, 0.3), (16, 400, 1), (16, 150, 2), (24, 40, 2), (9, 9, 4), (24, 33, 6),
                                         (24, 33, 12)])
def test_sparse_charge(O, G, n_r, n_th, ppc, kind, fp32):
    w = wl("c1_64").scaled(n_r, n_th)
    prm, ctx = pair(O, G, w, charge_scale=0.03, precision=G.GRPIC_FP32 if fp32 else G.GRPIC_FP64)
    F, P = _state(O, prm, w, ppc, kind, 5)
    F[:3] = 0.0  # (the residual is then the charge)
    if fp32:  # (the oracle sees the rounded offsets)
        P = {q: (v.astype(np.float32).astype(np.float64) if v.dtype == np.float64 else v) for q, v in P.items()}
    res, mx, scale = O.gauss_residual(prm, F, P)
    Fg = ctx.new_fields()
    Pg = {q: (v.to(ctx.dtype) if v.is_floating_point() else v) for q, v in up(P).items()}
    d = ctx.diagnostics(Fg, Pg, w.B0, gauss_plane=True)
    err = np.abs(d["gauss_res"].double().cpu().numpy() - res).max()
    assert err <= (200 * 2.0 ** -24 if fp32 else 1e-12) * max(scale, np.abs(res).max())
