"""Updates of the tree return once their work is queued: the caller's host work
overlaps them.  The list that such a call sends outlives the call, the next
call's list waits for it, and a stream under capture is refused with nothing
changed."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2309_04393_amd import resoct  # noqa: E402

M, L = 16, 9


@pytest.fixture(scope="module")
def big():
    """A tree of 8.4 million leaves; a brick of the coarsest level covers them all."""
    vol = resoct.Volume((8192, 8192, 192), (1.0, 1.0, 3.0), M, 2, 32, L)
    cache = resoct.Cache(vol, 64, 64)
    tree = resoct.Octree(cache, (16, 16, 8), 9)
    staged = cache.staging(64)
    staged.zero_()
    top = np.array([vol.encode(c, L - 1, (0, 0, 0)) for c in range(M)], np.uint32)
    fine = np.array([vol.encode(c, 0, (k, 0, 0)) for c in range(M) for k in range(4)], np.uint32)
    return vol, cache, tree, staged, top, fine


def test_calls_return_before_their_work_is_done(big):
    vol, cache, tree, staged, top, fine = big
    s = torch.cuda.current_stream()
    busy_update, busy_meta = [], []
    for i in range(5):
        cache.stream_bricks(10 * i + 1, fine, staged)  # all 64 slots: evicts the coarse bricks
        cache.stream_bricks(10 * i + 2, top, staged)
        s.synchronize()
        tree.update_residency()
        busy_update.append(not s.query())
        s.synchronize()
        for c in range(2):
            tree.set_leaf_unknown(c)
        s.synchronize()
        tree.leaf_metadata_from_bricks(top[:2])
        busy_meta.append(not s.query())
    s.synchronize()
    assert any(busy_update) and any(busy_meta), (busy_update, busy_meta)
    root_mask = tree.t["node_mask"][:2 * M].view(torch.int16).cpu().numpy()
    root_meta = tree.t["node_meta"][:4 * M].view(torch.int32).cpu().numpy()
    assert (root_mask & (1 << (L - 1))).all()
    assert (root_meta[:2] == 0).all()  # zero voxels, which were unknown before


def test_lists_of_calls_in_a_row(big):
    """Twelve updates queued behind one another without a wait give what a
    rebuild gives."""
    vol, cache, tree, staged, top, fine = big
    rng = np.random.default_rng(3)
    for i in range(12):
        ids = np.array([vol.encode(int(rng.integers(M)), int(l), (0, 0, 0)) for l in rng.integers(0, L, 20)], np.uint32)
        cache.stream_bricks(100 + i, ids, staged)
        tree.update_residency()
        cache.stream_bricks(100 + i, ids, staged)  # resident now: stamps only
    a = tree.masks()
    tree.rebuild_residency()
    torch.cuda.synchronize()
    assert np.array_equal(a, tree.masks())


def test_capture_is_refused(big):
    vol, cache, tree, staged, top, fine = big
    cache.stream_bricks(1000, fine[:8], staged)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    x = torch.zeros(8, device="cuda")
    with torch.cuda.stream(s):
        g.capture_begin(capture_error_mode="thread_local")
        x.add_(1.0)
        errs = []
        for call in (lambda: tree.update_residency(stream=s), lambda: tree.leaf_metadata_from_bricks(fine[:8], stream=s),
                     lambda: cache.stream_bricks(1001, fine[:8], staged, stream=s)):
            with pytest.raises(resoct.ResoctError) as e:
                call()
            errs.append(e.value.code)
        g.capture_end()
    assert errs == [-5] * 3  # RO_E_STATE
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
    assert (x == 3).all()
    tree.update_residency()
    a = tree.masks()
    tree.rebuild_residency()
    torch.cuda.synchronize()
    assert np.array_equal(a, tree.masks())
