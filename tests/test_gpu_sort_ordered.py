"""The cell sort in single precision on both sides of the size from which the
scatter orders each block's particles in LDS (2^21 slots), with a partial last
block, on slots in random order (a block's particles go everywhere) and on
slots that moved by a cell or two, with emptied and leaving slots.  The oracle
is a stable sort of the rows on the CPU: a sort moves bits, so cells, live
count and the particles of each cell agree exactly, and the slots behind are
empty."""
import numpy as np
import pytest

from test_gpu_sort_ranked import COLS, G, _rows  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", ["random", "near"])
@pytest.mark.parametrize("n", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1025])
def test_sort_in_single_precision(G, n, order):
    import torch
    n_r, n_th = 96, 57
    c = G.Context(0.9, 1.0, 1.2, 20.0, n_r, n_th, precision=G.GRPIC_FP32)
    g = np.random.default_rng(n)
    i1, i2 = (g.integers(0, m, n) for m in (n_r, n_th))
    if order == "near":
        k = np.argsort(i1 * n_th + i2, kind="stable")
        i1 = np.clip(i1[k] + g.integers(-1, 2, n), 0, n_r - 1)
        i2 = np.clip(i2[k] + g.integers(-2, 3, n), 0, n_th - 1)
    rows = {"i1": i1.astype(np.int32), "i2": i2.astype(np.int32)}
    rows.update({q: g.standard_normal(n).astype(np.float32) for q in ("dx1", "dx2", "u1", "u2", "u3", "w", "phi")})
    rows["tag"] = g.integers(1, 3, n).astype(np.uint8)
    rows["tag"][::13] = 0
    rows["tag"][5::101] |= 0x80  # leaving slots are not carried
    P, Q = c.new_particles(n), c.new_particles(n)
    for q in COLS:
        P[q].copy_(torch.from_numpy(rows[q]))
        Q[q].fill_(1)  # the destination holds an earlier set
    live = c.sort(P, Q, count=True)
    keep = (rows["tag"] != 0) & (rows["tag"] < 0x80)
    assert live == keep.sum()
    cell = (Q["i1"][:live].long() * n_th + Q["i2"][:live].long()).cpu().numpy()
    assert (np.diff(cell) >= 0).all()
    assert not (Q["tag"][live:] != 0).any()
    got = _rows(Q, live)
    want = _rows({q: torch.from_numpy(rows[q][keep]) for q in COLS}, live)
    for q in COLS:
        np.testing.assert_array_equal(got[q].view(np.uint8), want[q].view(np.uint8), err_msg=q)
