"""Batches at the edges of the serving kernel's requests: as many as a server
takes, smaller than a workgroup's waves, one among large ones, and a batch
behind another that is still in flight."""
from __future__ import annotations

import numpy as np
import pytest

import synth
from tests.test_gpu_serve import N_CH, Rig, _chans, _same, resoct, scene, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _reqs(src, sizes):
    cams = synth.orbit_path(src.dims, src.spacing, len(sizes), az_step_deg=11.0)
    out = []
    for k, (W, H) in enumerate(sizes):
        cam = dict(cams[k])
        cam["tx"] = cam["ty"] * W / H
        out.append(dict(W=W, H=H, cam=cam, chans=_chans(range(1 + k % N_CH), k), frame=2 + k))
    return out


@pytest.mark.parametrize("sizes", [
    [(1, 1)], [(1 + k % 9, 1 + k % 5) for k in range(64)], [(256, 160), (1, 1), (3, 200)],
    [(33, 1)] * 7 + [(320, 240)] + [(1, 65)] * 3,
])
@pytest.mark.parametrize("graph", [False, True])
def test_batches(scene, sizes, graph):  # noqa: F811
    rig = Rig(scene, _reqs(scene.src, sizes))
    ref, st_ref = rig.frame_kernel()
    rig.stats.zero_()
    srv = resoct.Server(scene.tree, max_requests=64, max_tiles=64)
    n = len(sizes)
    sets = [[rig.out(k) for k in range(n)] for _ in range(3)]
    torch.cuda.synchronize()
    tickets = [srv.launch([rig.fd(k, stats=i == 0) for k in range(n)], outs, graph=graph) for i, outs in enumerate(sets)]
    for t, outs in zip(tickets, sets):
        srv.wait(t)
        assert all(srv.request_done(t, k) for k in range(n)), "completion flags not posted"
        for k in range(n):
            _same(rig.image(k, outs[k]), ref[k], f"{k}")
    assert np.array_equal(rig.stats.cpu().numpy()[:, :5], st_ref[:, :5])
