"""The LRU select against numpy over key ranges and slot counts at the edges
of its passes."""
from __future__ import annotations

from types import SimpleNamespace

import numpy as np
import pytest

from paper_2309_04393_amd.pipeline import GpuScene

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

FREE = 0xFFFFFFFF


def _scene(dims, m, B, leaf, depth, n_slots, max_batch, n_levels=2, bits=16):
    src = SimpleNamespace(dims=dims, spacing=(1, 1, 1), n_channels=m, bits=bits, n_levels=n_levels)
    return GpuScene(src, B, leaf, depth, n_slots, max_batch=max_batch, set_metadata=False)


def _words(t, n):
    return t[:4 * n].view(torch.int32).cpu().numpy().view(np.uint32)


# slots, slots filled, batch, stamps: all eligible slots ranked without a
# pass; passes over few and over all 64 key bits; fewer eligible than asked.
@pytest.mark.parametrize("S,filled,batch,stamps", [
    (1, 1, 3, "few"), (65, 30, 64, "few"), (4097, 4097, 1, "few"), (4098, 4098, 1, "few"), (9001, 9001, 2048, "few"),
    (9001, 9001, 37, "wide"), (9001, 3000, 2048, "wide"), (9001, 9001, 2049, "one"), (12000, 12000, 1, "wide"),
    (12000, 11900, 300, "current"), (9001, 9001, 100, "all current"),
    (12000, 12000, 7, "far"), (12000, 11990, 2000, "far"),
])
def test_lru_select(S, filled, batch, stamps):
    rng = np.random.default_rng(S + batch)
    sc = _scene((256, 256, 128), 2, 8, (8, 8, 8), 5, S, 4096)
    ids = rng.permutation(sc.all_ids())
    staged = torch.randint(0, 256, (4096 * sc.cache.slot_stride,), dtype=torch.uint8, device="cuda")
    for a in range(0, filled, 4096):
        assert np.all(sc.cache.stream_bricks(1, ids[a:min(a + 4096, filled)], staged) == 1)
    frame = 77
    st = {"few": lambda: rng.integers(1, 5, S), "wide": lambda: rng.integers(0, 2**32 - 1, S),
          "one": lambda: np.full(S, 9), "current": lambda: np.where(rng.random(S) < 0.98, frame, 5),
          "far": lambda: np.where(np.arange(S) == 3, 2**32 - 2, 5),  # undecided after the three passes
          "all current": lambda: np.full(S, frame)}[stamps]().astype(np.uint32)
    st[st == frame] = frame if stamps.endswith("current") else 1
    sq = rng.permutation(np.unique(rng.integers(0, 2**32 if stamps == "wide" else 2**20, 4 * S)))[:S].astype(np.uint32)
    sc.cache.t["stamps"][:4 * S].view(torch.int32).copy_(torch.from_numpy(st.view(np.int32)))
    sc.cache.t["seqs"][:4 * S].view(torch.int32).copy_(torch.from_numpy(sq.view(np.int32)))
    brick = _words(sc.cache.t["slot_brick"], S)
    key = ((st.astype(np.uint64) + 1) << np.uint64(32)) | sq
    key = np.where(brick == FREE, np.arange(S, dtype=np.uint64), key)
    ok = (brick == FREE) | (st != frame)
    victims = np.argsort(np.where(ok, key, np.uint64(2**64 - 1)), kind="stable")[:min(batch, int(ok.sum()))]
    new = ids[filled:filled + batch]
    call = np.concatenate([new, new[:2]])  # repeats of listed bricks change nothing
    flags = sc.cache.stream_bricks(frame, call, staged)
    k = len(victims)
    assert np.array_equal(flags, np.concatenate([np.arange(len(new)) < k, np.full(len(call) - len(new), 2)]))
    pt = sc.cache.page_table_host()
    pos = {int(b): i for i, b in enumerate(sc.all_ids())}
    assert np.array_equal(pt[[pos[int(b)] for b in new[:k]]], victims)
    assert np.array_equal(_words(sc.cache.t["page_table"], len(pt)), pt)
    inv = np.full(S, FREE, np.uint32)
    inv[pt[pt != FREE]] = np.nonzero(pt != FREE)[0]
    assert np.array_equal(_words(sc.cache.t["slot_brick"], S), inv)
    w = sc.cache.slot_stride
    slots = sc.cache.t["slots"].view(-1, w)
    for i in {0, k // 2, k - 1} if k else ():
        assert torch.equal(slots[int(victims[i])], staged[i * w:(i + 1) * w])
