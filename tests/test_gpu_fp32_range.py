"""Range of the single-precision particle update: momenta up to gamma^2 of the
type's largest value, at any radius, and photons of any energy, against the
double-precision update of the same (rounded) state.  The bars are those of
one single-precision step: 3e-6 cells, 1e-5 of a momentum."""
import numpy as np
import pytest

from test_gpu_parity import G, down, pair, up, wl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma,tag", [(3.0, 1), (1e8, 1), (1e13, 1), (1e17, 2), (1e-12, 7), (1e-6, 7), (1e17, 7)])
@pytest.mark.parametrize("n", [48, 512])
def test_range_of_momenta(O, G, n, gamma, tag):
    w = wl("c5_4096", n, n_absorb=6)  # r up to 200
    rng = np.random.default_rng(1)
    prm, c64 = pair(O, G, w, charge_scale=0.1, n_filter=0)
    c32 = G.Context(w.a, w.M, w.r_min, w.r_max, n, n, dt=c64.dt, charge_scale=0.1, n_absorb=6, precision=G.GRPIC_FP32)
    P = O.particles_init(prm, 2000, 0, 1.0, 0, 3)
    k = len(P["tag"])
    s = rng.normal(size=(3, k))
    dxi, dth = np.log(w.r_max / w.r_min) / n, np.pi / n
    r = w.r_min * np.exp((P["i1"] + P["dx1"]) * dxi)
    th = (P["i2"] + P["dx2"]) * dth
    s *= gamma / np.sqrt((s ** 2).sum(axis=0))
    P["u1"], P["u2"], P["u3"] = s[0] * r * dxi, s[1] * r * dth, s[2] * r * np.sin(th)
    P["tag"][:] = tag
    P32 = {q: (v.astype(np.float32) if v.dtype == np.float64 else v) for q, v in P.items()}
    P64 = {q: (v.astype(np.float64) if v.dtype == np.float32 else v) for q, v in P32.items()}

    def run(ctx, S, fused):
        F, Q = ctx.new_fields(), up(S)
        ctx.push_deposit(F, Q) if fused else (ctx.push(F, Q), ctx.deposit(Q, F))
        return F[18:21].double().cpu().numpy(), down(Q)

    for fused in (False, True):
        J64, A = run(c64, P64, fused)
        J32, B = run(c32, P32, fused)
        far = (P["i2"] >= 2) & (P["i2"] < n - 2)  # (beside the axes a step amplifies the rounding of the angle)
        assert (B["tag"] != 0x40).all() and (A["tag"] != 0x40).all()
        for q in ("1", "2"):
            x = np.abs((A["i" + q] - B["i" + q]) + (A["dx" + q] - B["dx" + q].astype(float)))
            assert x[far].max() <= 3e-6, q
        scale = gamma * np.stack([r * dxi, r * dth, r * np.sin(th)])
        for c, q in enumerate(("u1", "u2", "u3")):
            assert (np.abs(A[q] - B[q]) / scale[c])[far].max() <= 1e-5, q
        if tag != 7:
            assert np.isfinite(J32).all()
            for c in range(3):
                assert np.abs(J32[c] - J64[c]).max() <= 1e-4 * np.abs(J64[c]).max(), c
