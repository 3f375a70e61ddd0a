"""The horizon rows of the field stages (rows i <= n_f take row n_f + 1, the
planes before the update are kept whole) on either side of the rule that
writes them in the updates or in a launch of their own: against the FP64
oracle to the bars of test_gpu_parity.py, and, in both precisions, as exact
copies of their row."""
import numpy as np
import pytest

from test_gpu_parity import G, assert_fields, pair, up, wl  # noqa: F401

pytestmark = pytest.mark.gpu


def _state(O, prm, w):
    F = O.fields_init_wald(prm, w.B0)
    g = np.random.default_rng(0)
    F[:12] *= 1 + 0.1 * g.normal(size=F[:12].shape)
    F[18:24] = 0.01 * g.normal(size=F[18:24].shape)
    return F


# (1449 x 1448: a plane of 2^21 points)
@pytest.mark.parametrize("n_r,n_th,n_f", [(40, 56, 4), (40, 56, 5), (33, 70, 17), (1449, 1448, 5)])
def test_horizon_rows(O, G, n_r, n_th, n_f):
    w = wl("c1_64").scaled(n_r, n_th)
    prm, ctx = pair(O, G, w, charge_scale=0.05, n_filter=n_f, n_absorb=6)
    F = _state(O, prm, w)
    for stage in (0, 1):
        Fg = up({"F": F})["F"]
        O.field_advance(prm, F, stage)
        ctx.field_advance(Fg, stage)
        assert_fields(F, Fg.cpu().numpy(), range(0, 24), what=f"stage {stage}")


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n_f", [0, 4, 5, 17])
def test_horizon_rows_are_copies(O, G, n_f, fp32):
    w = wl("c1_64").scaled(40, 56)
    prm, ctx = pair(O, G, w, charge_scale=0.05, n_filter=n_f, n_absorb=6,
                    precision=G.GRPIC_FP32 if fp32 else G.GRPIC_FP64)
    F = ctx.new_fields()
    F[:33] = up({"F": _state(O, prm, w)})["F"]
    D, B, D0, B0 = (slice(k, k + 3) for k in (0, 3, 6, 9))
    edge = prm.ng + n_f + 1  # (the row as a plane index)

    def rows_are_copies(planes):
        for p in F[planes].cpu().numpy():
            np.testing.assert_array_equal(p[:edge], np.broadcast_to(p[edge], p[:edge].shape))

    ctx.field_advance(F, 0)
    rows_are_copies(B0)
    before = F[0:6].clone()
    ctx.field_advance(F, 1)
    rows_are_copies(D)
    rows_are_copies(B)
    np.testing.assert_array_equal(F[D0].cpu().numpy(), before[0:3].cpu().numpy())
    np.testing.assert_array_equal(F[B0].cpu().numpy(), before[3:6].cpu().numpy())
    if fp32:  # the compensation of D and B, columns that belong to a component only
        for p in F[33:39].cpu().numpy():
            q = p[:, prm.ng:prm.ng + w.n_th]
            np.testing.assert_array_equal(q[:edge], np.broadcast_to(q[edge], q[:edge].shape))
