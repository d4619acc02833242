"""Lists longer than the tree's scratch holds: a residency update of more than
261,120 bricks and leaf metadata from more than 20,164 bricks, which take
several launches each."""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import pytest

from paper_2309_04393_amd.pipeline import GpuScene

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def _scene(dims, m, L, depth, n_slots):
    src = SimpleNamespace(dims=dims, spacing=(1, 1, 1), n_channels=m, bits=8, n_levels=L)
    return GpuScene(src, 8, (8, 8, 8), depth, n_slots, max_batch=8192, set_metadata=False)


@pytest.mark.parametrize("n", [261120, 261121, 270000])
def test_residency_update(n):
    dims, L = (512, 504, 1040), 3
    sc = _scene(dims, 1, L, 8, 280000)
    rng = np.random.default_rng(n)
    ids = rng.permutation(sc.all_ids())
    staged = torch.zeros(8192 * sc.cache.slot_stride, dtype=torch.uint8, device="cuda")
    for a in range(0, n, 8192):
        part = ids[a:min(a + 8192, n)]
        assert np.all(sc.cache.stream_bricks(1, part, staged) == 1)
    sc.tree.update_residency()
    masks = sc.tree.masks()
    # a leaf is a level-0 brick: its bit of level l is the residency of the brick that holds it
    res = sc.cache.page_table_host() != 0xFFFFFFFF
    gx, gy, gz = sc.tree.leaf_grid
    want = np.zeros((gz, gy, gx), np.uint16)
    at = 0
    for l in range(L):
        nx, ny, nz = (int(v) for v in sc.nb[l])
        r = res[at:at + nx * ny * nz].reshape(nz, ny, nx)
        at += nx * ny * nz
        full = np.zeros((gz >> l, gy >> l, gx >> l), bool)
        full[:nz, :ny, :nx] = r[:gz >> l, :gy >> l, :gx >> l]
        want |= np.kron(full, np.ones((1 << l, 1 << l, 1 << l), bool)).astype(np.uint16) << l
    leaves = masks[len(masks) - sc.tree.n_leaves:, 0].reshape(gz, gy, gx)
    assert np.array_equal(leaves, want)
    sc.tree.rebuild_residency()
    assert np.array_equal(sc.tree.masks(), masks)


def test_metadata_from_bricks():
    dims, m, L = (256, 248, 136), 2, 3
    sc = _scene(dims, m, L, 5, 60000)
    g = torch.Generator(device="cuda").manual_seed(4)
    ids = np.random.default_rng(6).permutation(sc.all_ids())
    assert len(ids) > 20164
    staged = torch.randint(0, 256, (8192 * sc.cache.slot_stride,), dtype=torch.uint8, device="cuda", generator=g)
    for a in range(0, len(ids), 8192):
        assert np.all(sc.cache.stream_bricks(1, ids[a:a + 8192], staged) == 1)
    got = []
    level = (ids >> 24) % L
    for parts in ([ids], [p for l in range(L - 1, -1, -1) for p in np.array_split(ids[level == l], 5)]):
        for c in range(m):
            sc.tree.set_leaf_unknown(c)
        for p in parts:
            sc.tree.leaf_metadata_from_bricks(p)
        torch.cuda.synchronize()
        got.append((sc.tree.meta(), sc.tree.leaf_levels()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert (got[0][1] == 0).any()
