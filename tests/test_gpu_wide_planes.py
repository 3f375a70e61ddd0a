"""Planes beyond the 32-bit offsets of the field gather: 2^24 rows of 28 columns
(4.3 GB a plane in double precision).  Particles in the outermost rows, in
fields that are zero elsewhere, are pushed and deposited as on a grid that has
those rows alone (the same spacings up to the rounding of the radii; bars of a
double- and of a single-precision step)."""
import ctypes
import math

import numpy as np
import pytest

from test_gpu_parity import G, down, up  # noqa: F401

pytestmark = pytest.mark.gpu

N_R, N_TH, ROWS = 1 << 24, 28, 64
R_MIN, R_MAX = 1.2, 20.0


def _sets(G, ctx, fp32, planes):
    """A field set of nine planes (D, B0, J); the others, which no push reads, share the first."""
    shape = (9,) + tuple(ctx.shape)
    import torch
    F = torch.zeros(shape, dtype=ctx.dtype, device="cuda")
    F[:6, -ROWS - 2:] = planes.to(ctx.dtype)
    f = G.Fields()
    at = {"D": 0, "B0": 3, "J": 6}
    step = F[0].numel() * F.element_size()
    for name, _ in G.Fields._fields_:
        for c in range(3):
            getattr(f, name)[c] = F.data_ptr() + (at.get(name, -1 * c) + c) * step
    return F, f


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("fp32", [False, True])
def test_rows_far_behind_32_bit_offsets(G, fp32, fused):
    import torch
    prec = G.GRPIC_FP32 if fp32 else G.GRPIC_FP64
    dxi = math.log(R_MAX / R_MIN) / N_R
    first = R_MIN * math.exp((N_R - ROWS) * dxi)
    dt = 0.4 * dxi * first
    far = G.Context(0.9, 1.0, R_MIN, R_MAX, N_R, N_TH, dt=dt, charge_scale=0.1, precision=prec)
    near = G.Context(0.9, 1.0, first, R_MAX, ROWS, N_TH, dt=dt, charge_scale=0.1, precision=prec)
    g = torch.Generator(device="cuda").manual_seed(1)
    planes = torch.randn((6, ROWS + 2, N_TH + 4), dtype=torch.float64, device="cuda", generator=g)
    rng = np.random.default_rng(2)
    n = 5000
    T = np.float32 if fp32 else np.float64
    P = {"i1": rng.integers(4, ROWS - 2, n).astype(np.int32), "i2": rng.integers(0, N_TH, n).astype(np.int32)}
    P.update({q: rng.random(n).astype(T) for q in ("dx1", "dx2")})
    P.update({q: (s * rng.normal(size=n)).astype(T) for q, s in (("u1", 20 * dxi), ("u2", 20 * math.pi / N_TH), ("u3", 5.0))})
    P.update({"w": np.ones(n, T), "phi": np.zeros(n, T), "tag": rng.integers(1, 3, n).astype(np.uint8)})
    P.update({q: P[q[:-1]].copy() for q in ("i1p", "i2p", "dx1p", "dx2p")})

    def run(ctx, shift):
        S = {q: v.copy() for q, v in P.items()}
        S["i1"] += shift
        S["i1p"] += shift
        F, f = _sets(G, ctx, fp32, planes)
        Q = up(S)
        p, s = ctypes.byref(ctx._particles(Q)), G._stream()
        calls = [(G._lib.grpic_push_deposit, (f, p))] if fused else [(G._lib.grpic_push, (f, p)), (G._lib.grpic_deposit, (p, f))]
        for fn, (a, b) in calls:
            a, b = (ctypes.byref(v) if isinstance(v, G.Fields) else v for v in (a, b))
            assert fn(ctx._h, a, b, s) == 0
        torch.cuda.synchronize()
        Q = down(Q)
        Q["i1"] -= shift
        J = F[6:, -ROWS - 4:].double().cpu().numpy()
        del F
        torch.cuda.empty_cache()
        return Q, J

    A, JA = run(far, N_R - ROWS)
    B, JB = run(near, 0)
    tol = 1e-5 if fp32 else 1e-9
    assert np.abs(B["i1"] - P["i1"] + B["dx1"] - P["dx1"]).max() > 0.05  # they do move
    assert np.abs((B["u1"] - P["u1"]) / dxi).max() > 1e-7                 # and feel the fields
    np.testing.assert_array_equal(A["tag"], B["tag"])
    for q in ("1", "2"):
        x = (A["i" + q] - B["i" + q]) + (A["dx" + q].astype(np.float64) - B["dx" + q])
        assert np.abs(x).max() <= tol, q
    for q in ("u1", "u2", "u3"):
        assert np.abs(A[q] - B[q]).max() <= tol * np.abs(B[q]).max(), q
    for c in range(3):
        assert np.abs(JA[c] - JB[c]).max() <= 20 * tol * np.abs(JB[c]).max(), c
