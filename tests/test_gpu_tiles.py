"""The edges of the particle kernels' blocks, tiles and iteration counts
against the FP64 oracle, to the bars of test_gpu_parity.py (1e-12 of a
plane's largest value; the particle bars of assert_particles) and of
test_gpu_adjoint.py (1e-9 of a particle's gradient):

  - deposits of blocks that end in every place (a lane, a wavefront, a block
    more or less), of slots in random order (most particles outside the tile
    around the block's anchor cell), of a block whose first or whose second
    wavefront is empty, and of particles that crowd into one cell;
  - the Gauss residual's charge pass at the ends of its blocks;
  - pushes whose number of iterations lies on either side of the form that
    stops a cycle of two values, even and odd;
  - the quasi-spherical map on grids of the library and the short-series form;
  - gradients of pushes whose iterations stop long before they converge.
"""
import dataclasses

import numpy as np
import pytest

from test_gpu_adjoint import gpu_gradients, setup
from test_gpu_parity import G, _state, assert_fields, assert_particles, down, pair, up, wl  # noqa: F401

pytestmark = pytest.mark.gpu


def _slots(P, n, kind, rng):
    """n of the set's particles, shuffled (`random`), with an empty wavefront
    (`first`, `second`), or crowded into the cell of the first (`crowd`)."""
    k = rng.permutation(len(P["tag"]))[:n]
    Q = {q: np.ascontiguousarray(v[k]) for q, v in P.items()}
    if kind == "first":
        Q["tag"][:64] = 0
    if kind == "second":
        Q["tag"][64:128] = 0
    if kind == "crowd":
        for q in ("i1", "i2", "i1p", "i2p"):
            Q[q][:] = Q[q][0]
    return Q


@pytest.mark.parametrize("kind", ["random", "first", "second", "crowd"])
@pytest.mark.parametrize("n", [1, 63, 65, 127, 128, 129, 1000])
def test_deposits_at_block_and_tile_edges(O, G, n, kind):
    w = wl("c2_512", 40)
    prm, ctx = pair(O, G, w, charge_scale=0.3)
    F, P = _state(O, prm, w, n_pairs=2000)
    P = _slots(P, n, kind, np.random.default_rng(n))
    F_f, P_f = up({"F": F})["F"], up(P)
    O.push(prm, F, P)
    F_d, P_d = up({"F": F})["F"], up(P)
    O.deposit(prm, F, P)
    ctx.push_deposit(F_f, P_f)
    ctx.deposit(P_d, F_d)
    assert_particles(prm, P, down(P_f), what="fused", prev=False)
    assert_fields(F, F_f.cpu().numpy(), range(18, 21), what="fused J")
    assert_fields(F, F_d.cpu().numpy(), range(18, 21), what="J")


@pytest.mark.parametrize("n", [1, 255, 256, 257, 1000])
def test_charge_at_block_edges(O, G, n):
    w = wl("c1_64", 40)
    prm, ctx = pair(O, G, w, charge_scale=0.03)
    F, P = _state(O, prm, w, n_pairs=2000)
    P = _slots(P, n, "first" if n % 2 else "random", np.random.default_rng(n))
    d = ctx.diagnostics(up({"F": F})["F"], up(P), w.B0, gauss_plane=True)
    res, mx, scale = O.gauss_residual(prm, F, P)
    assert np.abs(d["gauss_res"].cpu().numpy() - res).max() <= 1e-12 * scale


@pytest.mark.parametrize("n_iter", [1, 2, 15, 16, 17, 18, 41, 200])
def test_push_iteration_counts(O, G, n_iter):
    w = dataclasses.replace(wl("c1_64", 48), n_iter=n_iter)
    prm, ctx = pair(O, G, w)
    F, P = _state(O, prm, w, n_pairs=3000)
    Fg, Pg = up({"F": F})["F"], up(P)
    O.push(prm, F, P)
    ctx.push(Fg, Pg)
    assert_particles(prm, P, down(Pg), what=f"n_iter {n_iter}")


@pytest.mark.parametrize("n", [48, 192, 384, 512])
def test_general_map_forms(O, G, n):
    w = dataclasses.replace(wl("c6_monopole", n), n_absorb=min(16, n // 8))
    prm, ctx = pair(O, G, w, charge_scale=0.3, r0=0.5, h0=0.3)
    F = O.fields_init_monopole(prm, w.B0)
    P = O.particles_init(prm, 4000, 0, w.T, 0, 5)
    P["i2"][:200], P["i2"][200:400] = 0, n - 1  # the cells beside the axes
    F_f, P_f = up({"F": F})["F"], up(P)
    O.push(prm, F, P)
    O.deposit(prm, F, P)
    ctx.push_deposit(F_f, P_f)
    assert_particles(prm, P, down(P_f), what=f"map {n}", prev=False)
    assert_fields(F, F_f.cpu().numpy(), range(18, 21), what=f"map J {n}")


@pytest.mark.parametrize("n_iter", [1, 3, 17, 40])
def test_adjoint_of_unconverged_iterations(O, G, n_iter):
    import torch
    import oracle.adjoint as A
    w, _, F1, P = setup(O, G, 24, 200)
    w = dataclasses.replace(w, n_iter=n_iter)
    ctx = G.Context(w.a, w.M, w.r_min, w.r_max, w.n_r, w.n_th, cfl=w.cfl, n_iter=n_iter, small_angle=w.small_angle)
    _, gu, gB0, _, _ = gpu_gradients(w, ctx, F1, P, 4, every=3)
    prm = O.Params.make(w.a, w.M, w.r_min, w.r_max, w.n_r, w.n_th, ctx.dt, n_iter=n_iter)
    st = A.state_from({k: v.cpu().numpy() for k, v in P.items()})
    _, gu_o, gB0_o, _ = A.gradients(prm, torch.from_numpy(O.fields_init_wald(prm, 1.0)), w.B0, st, 4)
    go = gu_o.numpy()
    err = np.abs(gu.cpu().numpy() - go).max(axis=1) / (np.abs(go).max(axis=1) + 1e-300)
    assert np.quantile(err, 0.99) <= 1e-9
    assert abs(gB0 - gB0_o) <= 1e-9 * abs(gB0_o)
