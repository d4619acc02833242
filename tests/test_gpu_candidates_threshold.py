"""Candidates at a threshold of zero: no resident brick and no brick whose
rows are all NaN comes back; and compaction on both sides of the number of
blocks up to which a writing block sums the counts before it itself."""
from __future__ import annotations

import numpy as np
import pytest

from tests.test_gpu_prefetch_tiles import _dense, _scene, resoct, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,m,L", [((136, 24, 16), 3, 5), ((120, 264, 9), 2, 9), ((8, 8, 8), 1, 1)])
@pytest.mark.parametrize("thr", [0.0, 0.25])
def test_no_spurious_candidates(dims, m, L, thr):
    rng = np.random.default_rng(dims[0] + m + L)
    sc = _scene(dims, m, L)
    pf = resoct.PrefetchRows(sc.tree)
    ids = sc.all_ids()
    some = rng.permutation(ids)[:min(60, len(ids) // 2)]
    sc.cache.stream_bricks(1, some, torch.zeros(64 * sc.cache.slot_stride, dtype=torch.uint8, device="cuda"))
    z = rng.normal(size=(pf.rows, 16)).astype(np.float32) * 2  # probabilities well above 0 in float32
    z[rng.random(z.shape) < 0.6] = np.nan
    gi, gp = pf.candidates(torch.from_numpy(z).cuda(), thr, cap=1 << 17)
    off, per = _dense(sc, L)
    nx, ny, nz = (int(v) for v in sc.nb[0])
    c, pz, py, px = np.meshgrid(np.arange(m), np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    resident = sc.cache.page_table_host() != 0xFFFFFFFF
    with np.errstate(invalid="ignore"):
        pr = 1.0 / (1.0 + np.exp(-z.astype(np.float64)))
    best = np.zeros(m * per)
    for l in range(min(L, 9)):
        f = [int(v) for v in sc.lf[l]]
        b = c * per + off[l] + ((pz // f[2]) * sc.nb[l][1] + py // f[1]) * sc.nb[l][0] + px // f[0]
        np.maximum.at(best, b.reshape(-1), np.where(pr[:, l] > thr, pr[:, l], 0.0))
    best[resident] = 0.0
    pos = {int(i): k for k, i in enumerate(ids)}
    at = np.array([pos[int(i)] for i in gi], np.int64)
    assert not resident[at].any()
    got = np.zeros(m * per)
    got[at] = gp
    # a float32 sigmoid is within 1e-6 of the exact one: only rows that near to the threshold may differ
    near = (best > 0) & (np.abs(best - thr) < 1e-6)
    assert np.array_equal((got > 0)[~near], (best > 0)[~near])
    assert len(at) == 0 or np.abs(got - best)[~near].max() <= 1e-6


@pytest.mark.parametrize("dims", [(1024, 1024, 512), (1024, 1024, 520), (1024, 1024, 1000)])
def test_compaction_past_the_direct_blocks(dims):
    rng = np.random.default_rng(dims[2])
    sc = _scene(dims, 1, 1, leaf=(8, 8, 8))
    nx, ny, nz = (int(v) for v in sc.nb[0])
    bz, by, bx = np.meshgrid(np.arange(nz), np.arange(ny), np.arange(nx), indexing="ij")
    all_ids = (bz << 16 | by << 8 | bx).reshape(-1).astype(np.uint32)
    n = len(all_ids)
    assert (n > 1024 * 1024) == (dims[2] > 512)
    cnt = np.where(rng.random(n) < 0.4, rng.integers(1, 2**32, n), 0).astype(np.uint32)
    cnt[[0, n - 1]] = (3, 2**32 - 1)
    hit = np.nonzero(cnt)[0]
    for read, cap in ((sc.cache.read_requests, 1 << 21), (sc.cache.read_requests, 1000),
                      (sc.cache.read_requests_noalloc, resoct.NOALLOC_MAX_PAIRS)):
        sc.cache.t["counters"][:4 * n].view(torch.int32).copy_(torch.from_numpy(cnt.view(np.int32)))
        ids, c, nu, tot = read(cap)
        assert nu == len(hit) and tot == int(cnt.astype(np.uint64).sum())
        k = min(cap, nu)
        assert np.array_equal(ids, all_ids[hit[:k]]) and np.array_equal(c, cnt[hit[:k]])
        assert not sc.cache.t["counters"][:4 * n].any()
