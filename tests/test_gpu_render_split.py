"""Frames so small that a wave takes a part of a unit's pixels (units of 4 x 4
in 32 x 32 tiles, whole tiles of them: 64, 128, 192, 256, 384 and 576 units
are handed out in 16, 8, 4, 4, 2 and 1 parts), against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.test_gpu_render import Pair  # noqa: E402
from tests.test_gpu_render_units import _tf  # noqa: E402


@pytest.fixture(scope="module")
def pair():
    src = synth.BlobVolume((40, 33, 29), n_channels=3, bits=16, n_levels=3, seed=9, n_blobs=12, spacing=(1, 1, 1))
    p = Pair(src, 16, (8, 8, 8), 3, n_slots=200, start_level=1)
    ids = p.gpu.all_ids()
    p.upload(0, ids[np.random.default_rng(5).random(len(ids)) < 0.6])
    p.check_masks()
    return p


@pytest.mark.parametrize("frame,W,H", [(1, 1, 1), (2, 32, 32), (3, 33, 7), (4, 70, 20), (5, 64, 33), (6, 65, 40), (7, 90, 96)])
def test_parts_of_units(pair, frame, W, H):
    src = pair.src
    cam = dict(synth.orbit_path(src.dims, src.spacing, 9)[frame])
    cam["tx"] = cam["ty"] * W / H
    W0, W1 = synth.window_fx(0.05 * 65535, 65535)
    chans = [dict(c=c, lo=0, hi=2, W0=W0, W1=W1, tf=_tf(k, c)) for c, k in ((2, "one"), (0, "gaps"), (1, "ramp"))]
    pair.check_frame(pair.frame(frame, cam, W, H, 0.5, chans), f"split-{W}x{H}")
