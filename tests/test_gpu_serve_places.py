"""Batches whose requests have more places for workgroups than the chip has
compute units, requests of one unit between and behind large ones, and rays
that end at their first samples, against the frame kernel."""
from __future__ import annotations

import numpy as np
import pytest

from tests.test_gpu_serve import Rig, _same, resoct, scene, torch  # noqa: F401
from tests.test_gpu_serve_units import _reqs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [(640, 480)] * 8, [(1, 1), (2, 3), (700, 500), (4, 4)] + [(640, 360)] * 8 + [(1, 1)] * 3, [(1601, 901)],
])
@pytest.mark.parametrize("haze", [False, True])
def test_places(scene, sizes, haze):  # noqa: F811
    reqs = _reqs(scene.src, sizes)
    if haze:
        for r in reqs:
            for c in r["chans"]:
                c["tf"] = c["tf"].copy()
                c["tf"][:, 3] = 0.6
    rig = Rig(scene, reqs)
    ref, st_ref = rig.frame_kernel()
    rig.stats.zero_()
    srv = resoct.Server(scene.tree, max_requests=64, max_tiles=1024)
    n = len(sizes)
    sets = [[rig.out(k) for k in range(n)] for _ in range(3)]
    torch.cuda.synchronize()
    tickets = [srv.launch([rig.fd(k, stats=i == 0) for k in range(n)], outs) for i, outs in enumerate(sets)]
    for t, outs in zip(tickets, sets):
        srv.wait(t)
        assert all(srv.request_done(t, k) for k in range(n)), "completion flags not posted"
        for k in range(n):
            _same(rig.image(k, outs[k]), ref[k], f"{k}")
    assert np.array_equal(rig.stats.cpu().numpy()[:, :5], st_ref[:, :5])
