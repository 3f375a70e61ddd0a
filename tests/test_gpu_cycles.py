"""The separate push beyond 32 iterations ends when its implicit iterations
alternate between two values, with the one that the full count would end on.
The fused pass runs the full count, so both must agree bit for bit, at even and
odd counts; and some particles must be in such a cycle (their results at two
consecutive counts differ), or the test would show nothing."""
import dataclasses

import numpy as np
import pytest

from test_gpu_parity import G, down, pair, up, wl  # noqa: F401

pytestmark = pytest.mark.gpu

KEYS = ("tag", "i1", "i2", "dx1", "dx2", "u1", "u2", "u3", "phi")


@pytest.mark.parametrize("n,r0,h0", [(24, 0.0, 0.0), (64, 0.0, 0.0), (256, 0.0, 0.0), (512, 0.5, 0.3)])
def test_cycles_end_on_the_same_iterate(O, G, n, r0, h0):
    w = dataclasses.replace(wl("c6_monopole", n), n_absorb=0)
    last = {}
    for n_iter in (32, 33, 34, 41, 199, 200):
        prm, ctx = pair(O, G, dataclasses.replace(w, n_iter=n_iter), charge_scale=0.1, r0=r0, h0=h0)
        P = O.particles_init(prm, 20000, 0, 1.0, 0, 5)
        F = ctx.new_fields()
        ctx.fields_init_monopole(F, w.B0)
        A, B = up(P), up(P)
        ctx.push(F, A)
        ctx.push_deposit(F, B)
        A, B = down(A), down(B)
        for q in KEYS:
            np.testing.assert_array_equal(A[q], B[q], err_msg=f"n_iter {n_iter} {q}")
        last[n_iter] = A
    for q in ("u1", "u2"):
        assert (last[199][q] != last[200][q]).any(), q
    assert (last[199]["dx1"] != last[200]["dx1"]).any()
