"""The posterior export at the edges of its rounds of 64 pixels per store and
128 per wave step: every entry of the caller's buffer is written (it starts as
NaN) and nothing past its end."""
import sys
from ctypes import c_void_p

import numpy as np
import pytest
import torch

from paper_1612_08792_amd import _lib
from paper_1612_08792_amd.gmmsp import GMMSP

pytestmark = pytest.mark.gpu

# cells of 1, 64, 65, 128, 129 and 784 pixels, one-pixel-wide and one-pixel-high
# cells, remainder columns and rows
SHAPES = [((7, 5), (1, 1)), ((24, 16), (8, 8)), ((40, 26), (13, 5)), ((33, 48), (16, 8)),
          ((130, 10), (43, 3)), ((90, 61), (28, 28)), ((5, 200), (1, 70)), ((200, 3), (70, 1))]


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("size,v", SHAPES)
def test_export_writes_every_entry(size, v, mode):
    W, H = size
    print("export", size, v, "cov_mode", mode, flush=True)
    sys.stdout.flush()
    dev = torch.device("cuda:0")
    m = GMMSP([(W, H)], v=v, device=dev, cov_mode=mode)
    rng = np.random.default_rng(W * 1000 + H)
    x = torch.from_numpy(rng.uniform(0, 60, W * H * m.channels).astype(np.float32)).to(dev)
    m.init_seeds(x)
    buf = torch.full((9 * W * H + 64,), float("nan"), dtype=torch.float32, device=dev)
    _lib.check(_lib.lib().gmmsp_export_responsibilities(
        m.handle, c_void_p(x.data_ptr()), c_void_p(buf.data_ptr()), c_void_p(m._stream())))
    R = buf.cpu().numpy()
    assert np.all(np.isnan(R[9 * W * H:]))
    R = R[:9 * W * H].reshape(H, W, 9).astype(np.float64)
    assert np.all(np.isfinite(R)) and np.all(R >= 0)
    # nine rounded quotients, a reciprocal within 1 ulp and the sum's own rounding
    assert np.abs(R.sum(-1) - 1).max() <= 12 * 2.0 ** -23
    # candidates outside the seed grid have posterior 0
    g = m.grids[0]
    cx, cy = np.arange(W) // g.vx, np.arange(H) // g.vy
    for s in range(9):
        kx, ky = cx + s % 3 - 1, cy + s // 3 - 1
        out = ~(((ky >= 0) & (ky < g.ny))[:, None] & ((kx >= 0) & (kx < g.nx))[None, :])
        assert np.all(R[..., s][out] == 0)
    # the public call returns the same values
    assert np.array_equal(m.export_responsibilities(x).cpu().numpy().reshape(H, W, 9), R.astype(np.float32))


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("size,v", [((61, 45), (4, 4)), ((91, 57), (13, 5)), ((150, 131), (28, 27)),
                                    ((230, 171), (57, 57)), ((5, 200), (1, 70))])
def test_shared_cells_match_one_wave(size, v, mode):
    """Up to 4096 cells the four waves of a block share a cell, beyond a wave has
    one: labels, L and posteriors of an image by itself are bit for bit those of the
    same image in a batch of more than 4096 cells."""
    W, H = size
    print("shared cells", size, v, "cov_mode", mode, flush=True)
    dev = torch.device("cuda:0")
    m = GMMSP([(W, H)], v=v, device=dev, cov_mode=mode)
    g = m.grids[0]
    n = 4096 // (g.ncx * g.ncy) + 1
    M = GMMSP([(W, H)] * n, v=v, device=dev, cov_mode=mode)
    rng = np.random.default_rng(W * 1000 + H)
    x = torch.from_numpy(rng.uniform(0, 60, W * H * m.channels).astype(np.float32)).to(dev)
    got = []
    for h, data in ((m, x), (M, x.repeat(n))):
        h.init_seeds(data)
        h.em_iterate(data, 2)
        labels, ll = h.label(data)
        got.append((labels.cpu().numpy(), np.asarray(ll), h.export_responsibilities(data).cpu().numpy()))
    (l1, ll1, r1), (l2, ll2, r2) = got
    r1, r2 = r1.reshape(1, -1), r2.reshape(n, -1)
    assert np.array_equal(l2.reshape(n, -1), np.repeat(l1.reshape(1, -1), n, 0))
    assert np.array_equal(ll2, np.repeat(ll1, n)) and np.isfinite(ll1).all()
    assert np.array_equal(r2, np.repeat(r1, n, 0))


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("size,v", [((95, 57), (19, 19)), ((40, 31), (10, 10)), ((84, 60), (28, 27))])
def test_shared_cells_on_both_sides_of_the_rule(size, v, mode):
    """Whether four waves share a cell depends on the cells of the batch and on the rounds
    of 128 pixels (64 in the other models) of a cell: the largest batch that shares
    them and the next give every image the labels, L and posteriors of its own."""
    W, H = size
    dev = torch.device("cuda:0")
    m = GMMSP([(W, H)], v=v, device=dev, cov_mode=mode)
    g = m.grids[0]
    per = g.ncx * g.ncy
    rounds = -(-(W * H // per) // (128 if mode == 0 else 64))
    n = min(682 * rounds, 4097) // per
    rng = np.random.default_rng(W * 1000 + H)
    x = torch.from_numpy(rng.uniform(0, 60, W * H * m.channels).astype(np.float32)).to(dev)
    got = []
    for k in (1, n - 1, n, n + 1):
        print("shared cells", size, v, "cov_mode", mode, "batch of", k, flush=True)
        h, data = GMMSP([(W, H)] * k, v=v, device=dev, cov_mode=mode), x.repeat(k)
        h.init_seeds(data)
        labels, ll = h.label(data)
        got.append((labels.cpu().numpy().reshape(k, -1), np.asarray(ll),
                    h.export_responsibilities(data).cpu().numpy().reshape(k, -1)))
    for labels, ll, R in got[1:]:
        assert np.array_equal(labels, np.broadcast_to(got[0][0], labels.shape))
        assert np.array_equal(ll, np.broadcast_to(got[0][1], ll.shape))
        assert np.array_equal(R, np.broadcast_to(got[0][2], R.shape))
