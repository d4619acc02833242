"""Frames around the sizes at which a workgroup takes two and four units at
once (8 and 32 units of 4 x 4 pixels per wave of a 256-CU chip), with ragged
edges and cameras that miss the volume, look along its axes or stand inside
it, against the oracle: image, requests, usage."""
from __future__ import annotations

import itertools

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_gpu_render import Pair  # noqa: E402


@pytest.fixture(scope="module")
def pair():
    src = synth.BlobVolume((40, 33, 29), n_channels=2, bits=16, n_levels=3, seed=5, n_blobs=12, spacing=(1, 1, 1.5))
    p = Pair(src, 16, (8, 8, 8), 3, n_slots=100, start_level=1)
    ids = p.gpu.all_ids()
    p.upload(0, ids[np.random.default_rng(2).random(len(ids)) < 0.7])
    p.check_masks()
    return p


FRAMES = itertools.count(1)


def _haze():
    t = synth.tf_hue(0.4, 0.3)
    t[:, 3] += 0.5  # a ray ends at its first samples
    return t


@pytest.mark.parametrize("W,H", [(640, 607), (637, 609), (1280, 1183), (1251, 1249)])
@pytest.mark.parametrize("view", ["outside", "away", "axis", "inside"])
def test_batches(pair, W, H, view):
    centre = (20.0, 16.0, 21.0)
    centre = (20.0, 16.0, 21.0)
    if view == "axis":
        cam = synth.camera_ortho((20.0, 16.0, -4.0), (0, 0, 1), (0, 1, 0), 25.0 * W / H, 25.0)
    else:
        eye = (21.0, 15.0, 20.0) if view == "inside" else (75.0, -31.0, 54.0)
        at = {"outside": centre, "away": (150.0, -80.0, 90.0), "inside": (40.0, 30.0, 0.0)}[view]
        cam = synth.camera_persp(eye, at, (0, 0, 1), 38.0, W / H)
    chans = [dict(c=0, lo=0, hi=2, W0=0, W1=65535 * 256, tf=_haze() if view == "outside" else synth.tf_hue(0.1, 0.3)),
             dict(c=1, lo=0, hi=2, W0=0, W1=65535 * 256, tf=synth.tf_hue(0.6, 0.2))]
    if view in ("axis", "inside"):
        # samples lie on voxel boundaries (every second one along the axis, the
        # first one of an eye at a voxel's corner), so the oracle calls the
        # pixels ambiguous: compared with the diagnostic kernel, which renders
        # with one lane per ray
        f, g = next(FRAMES), next(FRAMES)
        a = pair.gpu.render(f, cam, W, H, 1.0, chans, lod_bias=1.5)["rgba"].cpu().numpy().copy()
        ids, cnt, _, tot = pair.gpu.cache.read_requests(1 << 20)
        b = pair.gpu.render(g, cam, W, H, 1.0, chans, lod_bias=1.5, aov=True)["rgba"].cpu().numpy()
        ids1, cnt1, _, tot1 = pair.gpu.cache.read_requests(1 << 20)
        assert np.abs(a - b).max() <= 2.0 ** -22  # two units in the last place of values up to one
        assert tot == tot1 > 0 and np.array_equal(ids, ids1) and np.array_equal(cnt, cnt1)
        u, n = pair.gpu.cache.read_usage(f)
        v, m = pair.gpu.cache.read_usage(g)
        assert n == 0 and m > 0  # the later frame stamped the same slots again
        return
    res = pair.frame(next(FRAMES), cam, W, H, 1.0, chans, lod_bias=1.5)
    pair.check_frame(res, f"{view}-{W}x{H}")
