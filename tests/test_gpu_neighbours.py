"""A particle's update depends on its own state only: pushed beside particles
of the cells next to the axes, and beside none, it ends in the same bits.  On
the grids of each form of r, sin and cos (64^2 the long series, 512^2 the short
ones and, on the quasi-spherical map, theirs, 24^2 the library functions)."""
import dataclasses

import numpy as np
import pytest

from test_gpu_parity import G, down, pair, up, wl  # noqa: F401

pytestmark = pytest.mark.gpu

KEYS = ("tag", "i1", "i2", "dx1", "dx2", "u1", "u2", "u3", "phi")


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("n,r0,h0", [(24, 0.0, 0.0), (64, 0.0, 0.0), (512, 0.0, 0.0), (512, 0.5, 0.3)])
def test_neighbours_change_nothing(O, G, n, r0, h0, fp32, fused):
    w = dataclasses.replace(wl("c6_monopole", n), n_absorb=0)
    prm, ctx = pair(O, G, w, charge_scale=0.1, r0=r0, h0=h0, precision=G.GRPIC_FP32 if fp32 else G.GRPIC_FP64)
    P = O.particles_init(prm, 4000, 0, 1.0, 0, 5)
    if fp32:
        P = {q: (v.astype(np.float32) if v.dtype == np.float64 else v) for q, v in P.items()}
    axis = np.arange(len(P["tag"])) % 7 == 3  # every seventh slot: next to an axis, or empty
    P["i2"][axis] = np.where(np.arange(axis.sum()) % 2, 0, n - 1)
    alone = {q: v.copy() for q, v in P.items()}
    alone["tag"][axis] = 0

    def run(S):
        F, Q = ctx.new_fields(), up(S)
        ctx.fields_init_monopole(F, w.B0)
        ctx.push_deposit(F, Q) if fused else ctx.push(F, Q)
        return down(Q)

    A, B = run(P), run(alone)
    for q in KEYS:
        np.testing.assert_array_equal(A[q][~axis], B[q][~axis], err_msg=q)
