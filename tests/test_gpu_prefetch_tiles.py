"""Candidate scores over grids around the 16 x 4 tiles of a wave, leaf
fractions over tables and windows, and compaction around its block counts,
against numpy."""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2309_04393_amd import resoct  # noqa: E402
from paper_2309_04393_amd.pipeline import GpuScene  # noqa: E402


def _scene(dims, m, L, B=8, leaf=(4, 8, 4), spacing=(1, 1, 1)):
    depth = max(-(-dims[a] // leaf[a]) - 1 for a in range(3)).bit_length()
    src = SimpleNamespace(dims=dims, spacing=spacing, n_channels=m, bits=16, n_levels=L)
    return GpuScene(src, B, leaf, depth, 64, max_batch=64, set_metadata=False)


def _dense(sc, L):
    """Per level: first dense index inside a channel and brick counts; bricks per channel."""
    per = [int(np.prod(sc.nb[l])) for l in range(L)]
    return np.concatenate([[0], np.cumsum(per)[:-1]]), sum(per)


@pytest.mark.parametrize("dims,m,L,spacing,by", [
    ((8, 8, 8), 1, 1, (1, 1, 1), 0), ((136, 24, 16), 3, 5, (1, 1, 4), 0), ((120, 264, 9), 2, 9, (1, 1, 1), 1),
    ((128, 32, 40), 4, 4, (1, 4, 1), 0), ((500, 90, 8), 1, 3, (1, 1, 1), 1),
])
def test_candidates(dims, m, L, spacing, by):
    rng = np.random.default_rng(dims[0] + m)
    sc = _scene(dims, m, L, spacing=spacing)
    pf = resoct.PrefetchRows(sc.tree)
    ids = sc.all_ids()
    some = rng.permutation(ids)[:min(40, len(ids) // 2)]
    sc.cache.stream_bricks(1, some, torch.zeros(64 * sc.cache.slot_stride, dtype=torch.uint8, device="cuda"))
    z = rng.normal(size=(pf.rows, 16)).astype(np.float32) * 4
    z[rng.random(z.shape) < 0.05] = np.nan
    buf = torch.zeros(z.size + by, dtype=torch.float32, device="cuda")
    buf[by:].copy_(torch.from_numpy(z.reshape(-1)))
    Z = buf[by:].view(z.shape)
    off, per = _dense(sc, L)
    nx, ny, nz = (int(v) for v in sc.nb[0])
    c, pz, py, px = np.meshgrid(np.arange(m), np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    resident = sc.cache.page_table_host() != 0xFFFFFFFF
    for thr in (0.5, 0.0):
        gi, gp = pf.candidates(Z, thr, cap=1 << 17)
        # probabilities by the device's own definition, from a threshold of 0 per single row
        with np.errstate(over="ignore", invalid="ignore"):
            pr = 1.0 / (1.0 + np.exp(-z.astype(np.float64)))
        best = np.zeros(m * per)
        for l in range(min(L, 9)):
            f = [int(v) for v in sc.lf[l]]
            b = c * per + off[l] + ((pz // f[2]) * sc.nb[l][1] + py // f[1]) * sc.nb[l][0] + px // f[0]
            v = np.where(pr[:, l] > thr, pr[:, l], 0.0)
            np.maximum.at(best, b.reshape(-1), v)
        best[resident] = 0.0
        want = np.nonzero(best)[0]
        # float32 sigmoid: values within 4 ulp of the threshold may fall on either side
        edge = np.abs(best - thr) < 1e-6
        got = np.zeros(m * per)
        pos = {int(i): k for k, i in enumerate(ids)}
        got[[pos[int(i)] for i in gi]] = gp
        sure = ~edge
        assert np.array_equal(np.nonzero((got > 0) & sure)[0], want[sure[want]])
        assert np.abs(got - best)[sure].max() <= 1e-6
        assert np.all(np.diff(gi.astype(np.int64)) > 0)


@pytest.mark.parametrize("win", [(0, 65535 * 256), (300 * 256 + 7, 8000 * 256 + 1), (65000 * 256, 65001 * 256)])
def test_leaf_fractions(win):
    dims, m, L = (72, 40, 24), 3, 2
    rng = np.random.default_rng(win[0] % 1000)
    sc = _scene(dims, m, L)
    n = sc.tree.n_leaves
    mm = np.sort(rng.choice([0, 1, 299, 300, 301, 302, 700, 7999, 8000, 8001, 64999, 65000, 65001, 65535],
                            (m, n, 2)), -1).astype(np.uint16)
    for c in range(m):
        sc.set_metadata(c, mm[c])
    pf = resoct.PrefetchRows(sc.tree)
    chans, tabs = [], []
    for c, lo in ((2, 100), (0, 256)):  # channel 1 is not visible; channel 0's table is empty
        tf = np.ones((256, 4), np.float32)
        tf[:, 3] = 0.0
        tf[lo:, 3] = 0.25
        tf[3:5, 3] = 0.5 if c == 2 else 0.0
        tabs.append(tf)
        chans.append(dict(c=c, lo=0, hi=1, W0=win[0], W1=win[1], tf=tf))
    cam = synth.orbit_path(dims, (1, 1, 1), 2)[0]
    x = torch.zeros((pf.rows, 32), dtype=torch.float16, device="cuda")
    tfd = sc.tf_tensor(chans)
    pf.features(resoct.frame_desc(1, cam, 64, 64, 0.5, chans, tfd, L), x)
    got = x.cpu().numpy()[:, 7].reshape(m, 3, 5, 9).astype(np.float64)
    gx, gy, gz = sc.tree.leaf_grid
    want = np.zeros((m, 3, 5, 9))
    for (c, _), tf in zip(((2, 0), (0, 0)), tabs):
        v = mm[c].astype(object).reshape(gz, gy, gx, 2)
        lo = np.vectorize(lambda a: min(max(255 * (a * 256 - win[0]), 0) // (win[1] - win[0]), 255))(v[..., 0])
        hi = np.vectorize(lambda a: min(-(-max(255 * (a * 256 - win[0]), 0) // (win[1] - win[0])), 255))(v[..., 1])
        full = np.vectorize(lambda a, b: bool(np.any(tf[int(a):int(b) + 1, 3] != 0)))(lo, hi)
        f = full[:6, :5, :18].reshape(3, 2, 5, 1, 9, 2).astype(np.float64)
        want[c] = f.mean((1, 3, 5))
    assert np.array_equal(got, want)


# one block, block edges, and more blocks than a writing block sums itself
@pytest.mark.parametrize("dims,m", [((8, 8, 8), 1), ((64, 128, 64), 1), ((72, 128, 64), 1), ((1024, 1024, 512), 1)])
def test_compaction(dims, m):
    rng = np.random.default_rng(dims[0])
    sc = _scene(dims, m, 1, leaf=(8, 8, 8))
    nx, ny, nz = (int(v) for v in sc.nb[0])
    bz, by, bx = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    all_ids = (bz << 16 | by << 8 | bx).reshape(-1).astype(np.uint32)
    n = len(all_ids)
    cnt = np.where(rng.random(n) < 0.3, rng.integers(1, 2**32, n), 0).astype(np.uint32)
    cnt[[0, n - 1]] = (5, 2**32 - 1)
    for cap in (1 << 20, 7):
        sc.cache.t["counters"][:4 * n].view(torch.int32).copy_(torch.from_numpy(cnt.view(np.int32)))
        ids, c, nu, tot = sc.cache.read_requests(cap)
        hit = np.nonzero(cnt)[0]
        assert nu == len(hit) and tot == int(cnt.astype(np.uint64).sum())
        k = min(cap, nu)
        assert np.array_equal(ids, all_ids[hit[:k]]) and np.array_equal(c, cnt[hit[:k]])
        assert not sc.cache.t["counters"][:4 * n].any()
