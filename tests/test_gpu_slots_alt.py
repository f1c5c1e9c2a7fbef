"""The slot-lane statistics pass of the 3x3 colour block, the full 5x5 Sigma and
grayscale images at every shape it is built for (cells 1 to 56 pixels wide), the
pixel-lane pass of wider cells, and the two forms of their gather."""
import sys

import numpy as np
import pytest
import torch

import synth
from oracle import gmm_oracle as O
from paper_1612_08792_amd.gmmsp import GMMSP

pytestmark = pytest.mark.gpu
TEAM_MAX = 16384     # superpixels up to which 16 lanes share a superpixel


def rows_of(theta, mode):
    return O.theta_to_rows3(theta) if mode == 1 else O.theta_to_rows_mode(theta, mode)


def image_of(im, mode):
    lab = im.lab.numpy()
    return np.ascontiguousarray(lab[..., 0]) if mode == 3 else lab


def errors(rows, theta, mode):
    """Means in the oracle's standard deviations, blocks by relative Frobenius error."""
    dim = 3 if mode == 3 else 5
    S = np.zeros((len(rows), dim, dim))
    idx = [(i, j) for b in O.blocks(mode) for i in b for j in b if i <= j]
    for k, (i, j) in enumerate(idx):
        S[:, i, j] = S[:, j, i] = rows[:, dim + k]
    var = np.diagonal(theta.sigma, axis1=1, axis2=2)
    out = [np.abs((rows[:, :dim] - theta.mu) / np.sqrt(var)).max()]
    for b in O.blocks(mode):
        ix = np.ix_(range(len(S)), b, b)
        d = (S[ix] - theta.sigma[ix]).reshape(len(S), -1)
        out.append((np.linalg.norm(d, axis=1) / np.linalg.norm(theta.sigma[ix].reshape(len(S), -1), axis=1)).max())
    return out


# one v per columns-per-lane value and both ends of it; 56 is the widest slot-lane
# cell, 57 the narrowest pixel-lane one; remainder columns and rows in each image
@pytest.mark.parametrize("v", [2, 7, 8, 14, 15, 21, 22, 28, 29, 32, 33, 35, 36, 42, 43, 49, 50, 56, 57])
@pytest.mark.parametrize("mode", [1, 2, 3])
def test_one_step_at_every_shape(mode, v):
    W, H = 3 * v + max(1, v // 3), 2 * v + max(1, v // 2)
    print("one step, cov_mode", mode, "v", v, flush=True)
    sys.stdout.flush()
    im = synth.voronoi_lab(W, H, 5, 4.0, 100 + v, 4)
    g = O.make_grid(W, H, vx=v, vy=v)
    p = O.Params(cov_mode=mode)
    res = O.run_em(image_of(im, mode), g, p, max_iters=2)
    dev = torch.device("cuda:0")
    m = GMMSP([(W, H)], v=v, device=dev, cov_mode=mode)
    x = torch.from_numpy(image_of(im, mode)).reshape(-1).contiguous().to(dev)
    m.set_params(rows_of(res["theta"], mode))
    m.em_iterate(x, 1)
    assert m.ll_history(0)[0] == pytest.approx(res["ll_final"], rel=1e-7)
    th1 = O.mstep(res["z"], g, res["R"], res["pos"], res["theta"], p)
    e = errors(m.get_params(), th1, mode)
    assert max(e) <= 1e-5, e       # the one-step tolerance of every model


@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("W,H,v", [(60, 41, 12), (9, 10, 9), (95, 64, 5), (250, 130, 60)])
def test_team_gather_equals_one_thread(W, H, v, mode):
    dev = torch.device("cuda:0")
    im = synth.voronoi_lab(W, H, 6, 4.0, 11, 4)
    n = TEAM_MAX // ((W // v) * (H // v)) + 1
    if n * W * H > 4e7:
        n = int(4e7 / (W * H))      # the widest cells stay with the team in both
    print("gather", W, H, v, "cov_mode", mode, "batch of", n, flush=True)
    x1 = torch.from_numpy(image_of(im, mode)).reshape(-1).contiguous().to(dev)
    out = []
    for k in (1, n):
        x = x1.repeat(k)
        m = GMMSP([(W, H)] * k, v=v, device=dev, cov_mode=mode)
        m.init_seeds(x)
        rows = m.get_params()
        rows[:, :2].reshape(k, -1, 2)[:, 0] += 4000.0    # the first seed far away: no mass
        m.set_params(rows)
        m.em_iterate(x, 5)
        out.append(m.get_params().reshape(k, -1, m.theta_row))
    assert np.isfinite(out[0]).all()
    for k in (0, n // 2, n - 1):
        assert np.array_equal(out[1][k], out[0][0])


def wave_sums(feats):
    """FP32 sums of the rows of feats (n, k), a list of factors each, as a wave takes them
    with one pixel per lane: lane l adds rows l, l + 64, ..., then the lanes pairwise."""
    f = np.float32
    acc = np.zeros((64, len(feats)), f)
    n = len(feats[0][0])
    for s in range(0, n, 64):
        k = min(64, n - s)
        for j, ab in enumerate(feats):
            a = ab[0][s:s + k].astype(np.float64)
            b = ab[1][s:s + k].astype(np.float64) if len(ab) > 1 else 1.0
            acc[:k, j] = (a * b + acc[:k, j]).astype(f)      # a fused multiply-add
    while len(acc) > 1:
        acc = (acc[:len(acc) // 2] + acc[len(acc) // 2:]).astype(f)
    return acc[0].astype(np.float64)


def moments(sums, n, nc, cross):
    """Means and covariances of the colours, and of x and y with them, from the sums of
    d, d d (upper triangle), x d, y d and the exact means of x and y."""
    m = sums[:nc] / n
    out, j = list(m), nc
    for a in range(nc):
        for b in range(a, nc):
            out.append(sums[j] / n - m[a] * m[b])
            j += 1
    for c in cross:
        for a in range(nc):
            out.append(sums[j] / n - c * m[a])
            j += 1
    return np.array(out)


# one cell, so every posterior is 1 and what is left is the error of the sums
@pytest.mark.parametrize("w,h", [(7, 64), (12, 12), (24, 24), (35, 35), (56, 56), (56, 600)])
@pytest.mark.parametrize("mode", [1, 2, 3])
def test_sums_as_accurate_as_one_pixel_per_lane(mode, w, h):
    """RMS error of the colour moments against FP64 over four images, each in units of its
    standard deviations: at most 1.5 x that of a wave's sums with one pixel per lane (the
    reciprocal is good to an ulp; 36 errors scatter by a tenth)."""
    f = np.float32
    dev = torch.device("cuda:0")
    nc = 1 if mode == 3 else 3
    got, ref = [], []
    for seed in range(4):
        print("sums", w, h, "cov_mode", mode, "seed", seed, flush=True)
        rng = np.random.default_rng(100 * seed + w)
        mix = np.array([[1, .5, .2], [0, 1, .3], [0, 0, 1]])
        z = (np.array([80., 50., -55.]) + rng.normal(0, 5, (h * w, 3)) @ mix).astype(f)[:, :nc]
        mean = np.array([81.3, 49.1, -54.2], f)[:nc]
        cov = (np.eye(3) * 64 + 30)[:nc, :nc]
        dim = 2 + nc
        S = np.zeros((dim, dim))
        S[0, 0], S[1, 1] = w * w, h * h
        S[2:, 2:] = cov
        idx = [(i, j) for b in O.blocks(mode) for i in b for j in b if i <= j]
        row = np.concatenate([[w / 2, h / 2], mean.astype(np.float64), [S[i, j] for i, j in idx], [w * h]])
        m = GMMSP([(w, h)], v=(w, h), device=dev, cov_mode=mode)
        assert m.n_superpixels == 1
        m.set_params(row[None])
        m.em_iterate(torch.from_numpy(z.ravel().copy()).to(dev), 1)
        r = m.get_params()[0]
        n = w * h
        x, y = (np.arange(n) % w).astype(f), (np.arange(n) // w).astype(f)
        cross = (x.mean(dtype=np.float64), y.mean(dtype=np.float64)) if mode == 2 else ()
        d = (z - mean).astype(f)
        R = rng.uniform(0.5, 1.0, n).astype(f)
        R = (R * (f(1) / R).astype(f)).astype(f)             # e / sum of one candidate
        Rd = (R[:, None] * d).astype(f)
        feats = [(Rd[:, a],) for a in range(nc)] + [(Rd[:, a], d[:, b]) for a in range(nc) for b in range(a, nc)]
        feats += [(p, Rd[:, a]) for p in ((x, y) if mode == 2 else ()) for a in range(nc)]
        D = z.astype(np.float64) - mean
        exact = [D[:, a].sum() for a in range(nc)]
        exact += [(D[:, a] * D[:, b]).sum() for a in range(nc) for b in range(a, nc)]
        exact += [(p * D[:, a]).sum() for p in ((x, y) if mode == 2 else ()) for a in range(nc)]
        want = moments(np.array(exact), n, nc, cross)
        lane = moments(wave_sums(feats), n, nc, cross)
        C = np.zeros((dim, dim))
        for k, (i, j) in enumerate(idx):
            C[i, j] = C[j, i] = r[dim + k]
        mine = list(r[2:dim] - mean) + [C[2 + a, 2 + b] for a in range(nc) for b in range(a, nc)]
        mine += [C[p, 2 + a] for p in ((0, 1) if mode == 2 else ()) for a in range(nc)]
        sd = D.std(axis=0)
        unit = list(sd) + [sd[a] * sd[b] for a in range(nc) for b in range(a, nc)]
        unit += [p.std(dtype=np.float64) * s for p in ((x, y) if mode == 2 else ()) for s in sd]
        got.append((np.array(mine) - want) / unit)
        ref.append((lane - want) / unit)
    got, ref = np.array(got), np.array(ref)
    for part in (slice(0, nc), slice(nc, None)):             # means, covariances
        a, b = np.sqrt((got[:, part] ** 2).mean()), np.sqrt((ref[:, part] ** 2).mean())
        print("rms", a, "one pixel per lane", b, flush=True)
        assert a <= 1.5 * b


@pytest.mark.parametrize("mode", [1, 2, 3])
def test_constant_colours_stay_exact(mode):
    """Colours equal to the seeds': every difference is 0, so the means keep their value."""
    W, H = 61, 47
    c = np.array([80.3, 50.7, -55.1], np.float32)[:1 if mode == 3 else 3]
    dev = torch.device("cuda:0")
    m = GMMSP([(W, H)], v=12, device=dev, cov_mode=mode)
    x = torch.from_numpy(np.tile(c, W * H)).to(dev)
    m.init_seeds(x)
    m.em_iterate(x, 3)
    assert np.array_equal(m.get_params()[:, 2:2 + len(c)], np.broadcast_to(c.astype(np.float64), (m.n_superpixels, len(c))))


# cells of several groups of 32 rows: the FP64 totals, and the LDS that they share with 1/sum
@pytest.mark.parametrize("vx,vy", [(7, 33), (9, 80), (21, 64), (30, 70), (33, 65), (56, 100)])
@pytest.mark.parametrize("mode", [1, 2, 3])
def test_one_step_of_tall_cells(mode, vx, vy):
    W, H = 3 * vx + max(1, vx // 3), 2 * vy + 7
    print("tall cells, cov_mode", mode, vx, vy, flush=True)
    im = synth.voronoi_lab(W, H, 5, 4.0, 100 + vx, 4)
    g = O.make_grid(W, H, vx=vx, vy=vy)
    p = O.Params(cov_mode=mode)
    res = O.run_em(image_of(im, mode), g, p, max_iters=2)
    dev = torch.device("cuda:0")
    m = GMMSP([(W, H)], v=(vx, vy), device=dev, cov_mode=mode)
    x = torch.from_numpy(image_of(im, mode)).reshape(-1).contiguous().to(dev)
    m.set_params(rows_of(res["theta"], mode))
    m.em_iterate(x, 1)
    assert m.ll_history(0)[0] == pytest.approx(res["ll_final"], rel=1e-7)
    th1 = O.mstep(res["z"], g, res["R"], res["pos"], res["theta"], p)
    e = errors(m.get_params(), th1, mode)
    assert max(e) <= 1e-5, e       # the one-step tolerance of every model


# narrow cells on both sides of the rule by which the pixel-lane pass takes them, alone and
# beside wider ones, which set the columns per lane of the whole batch
@pytest.mark.parametrize("cells", [[(2, 33)], [(2, 64)], [(3, 48)], [(3, 64)], [(8, 300)],
                                   [(9, 9), (50, 50)], [(9, 9), (14, 14)], [(5, 70), (56, 20), (3, 3)]])
@pytest.mark.parametrize("mode", [1, 2, 3])
def test_one_step_of_narrow_and_mixed_cells(mode, cells):
    p = O.Params(cov_mode=mode)
    sizes, xs, rows, want = [], [], [], []
    for b, (vx, vy) in enumerate(cells):
        W, H = 3 * vx + max(1, vx // 3), 2 * vy + max(1, vy // 3)
        print("narrow cells, cov_mode", mode, vx, vy, flush=True)
        im = synth.voronoi_lab(W, H, 5, 4.0, 200 + vx, 4)
        g = O.make_grid(W, H, vx=vx, vy=vy)
        res = O.run_em(image_of(im, mode), g, p, max_iters=2)
        sizes.append((W, H))
        xs.append(torch.from_numpy(image_of(im, mode)).reshape(-1))
        rows.append(rows_of(res["theta"], mode))
        want.append((res["ll_final"], O.mstep(res["z"], g, res["R"], res["pos"], res["theta"], p)))
    dev = torch.device("cuda:0")
    m = GMMSP(sizes, v=list(cells), device=dev, cov_mode=mode)
    m.set_params(np.concatenate(rows))
    m.em_iterate(torch.cat(xs).contiguous().to(dev), 1)
    got = m.get_params()
    for b, (ll, th1) in enumerate(want):
        assert m.ll_history(b)[0] == pytest.approx(ll, rel=1e-7)
        e = errors(got[m.sp_slice(b)], th1, mode)
        assert max(e) <= 1e-5, (b, e)       # the one-step tolerance of every model


@pytest.mark.parametrize("mode", [1, 2, 3])
def test_gather_forms_of_wide_cells(mode):
    """Cells wider than the slot-lane pass takes: the statistics of the pixel-lane pass
    through both forms of the gather."""
    W, H, v = 120, 7, (57, 3)
    dev = torch.device("cuda:0")
    im = synth.voronoi_lab(W, H, 4, 4.0, 12, 4)
    x1 = torch.from_numpy(image_of(im, mode)).reshape(-1).contiguous().to(dev)
    n = TEAM_MAX // 4 + 1
    out = []
    for k in (1, n):
        print("gather of wide cells, cov_mode", mode, "batch of", k, flush=True)
        x = x1.repeat(k)
        m = GMMSP([(W, H)] * k, v=v, device=dev, cov_mode=mode)
        assert (m.n_superpixels <= TEAM_MAX) == (k == 1)
        m.init_seeds(x)
        rows = m.get_params()
        rows[:, :2].reshape(k, -1, 2)[:, 0] += 4000.0    # the first seed far away: no mass
        m.set_params(rows)
        m.em_iterate(x, 5)
        out.append(m.get_params().reshape(k, -1, m.theta_row))
    assert np.isfinite(out[0]).all()
    for k in (0, n // 2, n - 1):
        assert np.array_equal(out[1][k], out[0][0])
