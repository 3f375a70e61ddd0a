"""Moves at the limit of what the deposit can represent, in the fused pass: an
offset of exactly 1 plus a displacement of the largest number below 1 is a
move of two cells after rounding, which neither the deposit's tile nor the
planes beyond the outer edge have room for.  Such a slot stays live and
deposits nothing, as in the separate deposit."""
import math

import numpy as np
import pytest

from test_gpu_parity import G, down, up  # noqa: F401

pytestmark = pytest.mark.gpu

N_R = N_TH = 16
R_MIN, R_MAX = 1.0, 2.0


def _slots(O, prm, rows, width, n, rng):
    """n slots per row at offset 1 of the cell, moving outwards in flat space by 1 cell to a relative `width`."""
    k = np.repeat(rows, n).astype(np.int32)
    P = O.new_particles(len(k))
    P["i1"][:] = P["i1p"][:] = k
    P["dx1"][:] = P["dx1p"][:] = 1.0
    P["i2"][:] = P["i2p"][:] = N_TH // 2
    P["dx2"][:] = P["dx2p"][:] = 0.25
    P["w"][:] = 1.0
    P["tag"][:] = 1
    F = np.zeros((33,) + (N_R + 4, N_TH + 4))
    lo, hi = np.zeros(len(rows)), np.full(len(rows), 10.0)
    for _ in range(80):  # the momentum of a displacement of 1, row by row
        mid = 0.5 * (lo + hi)
        Q = {q: v[::n].copy() for q, v in P.items()}
        Q["u1"][:] = mid
        O.push(prm, F, Q)
        far = (Q["i1"] - rows - 1) + Q["dx1"] > 1.0
        hi, lo = np.where(far, mid, hi), np.where(far, lo, mid)
    P["u1"][:] = np.repeat(0.5 * (lo + hi), n) * (1.0 + width * rng.uniform(-1.0, 1.0, len(k)))
    P["u3"][:] = math.sqrt(width) * rng.uniform(0.0, 1.0, len(k))
    return F, P


@pytest.mark.parametrize("ranked", [False, True])
@pytest.mark.parametrize("fp32", [False, True])
def test_moves_of_two_cells_deposit_nothing(O, G, fp32, ranked):
    dt = 0.125  # a power of two: dt v takes the value below 1 in both precisions
    ctx = G.Context(0.0, 0.0, R_MIN, R_MAX, N_R, N_TH, dt=dt, charge_scale=0.1,
                    precision=G.GRPIC_FP32 if fp32 else G.GRPIC_FP64)
    prm = O.Params.make(0.0, 0.0, R_MIN, R_MAX, N_R, N_TH, dt, charge_scale=0.1)
    rows = np.arange(1, N_R)  # (the displacements of some rows step over the value below 1)
    F, P = _slots(O, prm, rows, 4e-6 if fp32 else 4e-14, 8000, np.random.default_rng(3))
    if fp32:
        P = {q: (v.astype(np.float32) if v.dtype == np.float64 else v) for q, v in P.items()}

    def run(S):
        Fg, Pg = ctx.new_fields(), up(S)
        ctx.push_deposit(Fg, Pg, ranked=ranked)
        return Fg.double().cpu().numpy(), down(Pg)

    F1, P1 = run(P)
    two = (P1["i1"] - P["i1"] == 2) & (P1["tag"] != 0x40)  # (0x40: a displacement of 1 or more)
    assert 0 < two.sum() < len(two) // 4
    Q = {q: v.copy() for q, v in P.items()}
    Q["tag"][two] = 0
    F2, _ = run(Q)
    for c in range(F1.shape[0]):  # (atomics: the order of a node's additions varies)
        if 18 <= c < 21:
            assert np.abs(F1[c] - F2[c]).max() <= (1e-5 if fp32 else 1e-12) * np.abs(F2[c]).max(), c
        else:
            assert not F1[c].any(), c
