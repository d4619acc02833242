"""The tree's level kernels (metadata reduction, residency propagation)
against the oracle over channel counts and tree shapes."""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import pytest

import oracle
from paper_2309_04393_amd.pipeline import GpuScene
from tests.helpers import leaf_grid

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def _scene(dims, m, B, leaf, depth, n_slots, max_batch, n_levels=2, bits=16):
    src = SimpleNamespace(dims=dims, spacing=(1, 1, 1), n_channels=m, bits=bits, n_levels=n_levels)
    return GpuScene(src, B, leaf, depth, n_slots, max_batch=max_batch, set_metadata=False)


# channels that are no power of two, axes that stop splitting, trees of one
# and two levels, leaf ranges that are not 4-byte aligned
@pytest.mark.parametrize("dims,m,leaf,depth,shift", [
    ((16, 16, 16), 1, (16, 16, 16), 0, 1), ((32, 16, 16), 3, (16, 16, 16), 1, 0), ((200, 72, 8), 5, (4, 8, 4), 6, 1),
    ((16, 130, 60), 2, (2, 4, 2), 6, 0), ((256, 256, 40), 7, (4, 4, 4), 6, 0),
])
def test_tree_levels(dims, m, leaf, depth, shift):
    rng = np.random.default_rng(depth + m)
    B, L = 16, 3
    sc = _scene(dims, m, B, leaf, depth, 4096, 4096, n_levels=L)
    V = oracle.make_volume(dims, (1, 1, 1), m, 16, B, L, leaf, depth)
    n = sc.tree.n_leaves
    lg = leaf_grid(dims, leaf, depth)
    mm = np.sort(rng.integers(0, 65536, (m, n, 2)), -1).astype(np.uint16)
    for c in range(m):
        buf = torch.zeros(2 * n + 1, dtype=torch.int16, device="cuda")
        buf[shift:shift + 2 * n].copy_(torch.from_numpy(mm[c].reshape(-1).view(np.int16)))
        sc.tree.set_leaf_metadata(c, buf[shift:shift + 2 * n].view(torch.uint16))
        torch.cuda.synchronize()
    assert int(np.prod(lg)) == n
    assert np.array_equal(sc.tree.meta(), oracle.meta_all(V, mm))
    assert np.all(sc.tree.leaf_levels() == 0)
    sim = oracle.CacheSim(V, 4096)
    ids = rng.permutation(sc.all_ids())
    staged = torch.zeros(4096 * sc.cache.slot_stride, dtype=torch.uint8, device="cuda")
    for f, part in enumerate((ids[:1], ids[:len(ids) // 3], ids[len(ids) // 4:len(ids) // 2], ids), 1):
        part = part[:4096]
        flags = sc.cache.stream_bricks(f, part, staged)
        want, _, _ = sim.stream(f, sim.dense_of(part))
        assert np.array_equal(flags, want)
        sc.tree.update_residency()
        masks = sc.tree.masks()
        assert np.array_equal(masks, oracle.masks(V, sim.res_slot))
    sc.tree.rebuild_residency()
    assert np.array_equal(sc.tree.masks(), masks)
