"""Per-channel sampling rates where bricks are missing: the samples of a ray
differ in the channels that take part, and their misses go through the wave's
table of sums.  Requests (bricks and counts), usage and image against the
oracle, with more missing bricks than the table has entries, with none
resident, and with samples that a ray's end leaves untaken."""
from __future__ import annotations

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2309_04393_amd import resoct  # noqa: E402
from tests.test_gpu_render import Pair  # noqa: E402


@pytest.mark.parametrize("m,resident,opacity,W,H", [
    (5, 0.3, 0.2, 67, 41), (16, 0.5, 0.1, 33, 65), (2, 0.0, 0.3, 40, 40), (4, 0.6, 1.0, 96, 30), (1, 0.4, 0.5, 5, 3),
])
def test_rates_misses(m, resident, opacity, W, H):
    src = synth.BlobVolume((70, 61, 45), n_channels=m, bits=16, n_levels=4, seed=11 + m, n_blobs=30,
                           spacing=(1, 1, 1))
    p = Pair(src, 8, (4, 4, 4), 5, n_slots=6000, max_batch=4096, start_level=1)
    ids = p.gpu.all_ids()
    pick = ids[np.random.default_rng(m).random(len(ids)) < resident][:5000]
    if len(pick):
        for s in range(0, len(pick), 4096):
            p.upload(0, pick[s:s + 4096])
    p.check_masks()
    chans = [dict(c=c, lo=min(c % 4, 2), hi=3, W0=0, W1=65535 * 256, tf=synth.tf_hue(c / m, opacity))
             for c in range(m)]
    cam = synth.camera_persp((120.3, -47.1, 71.7), (35.2, 30.4, 22.3), (0, 0, 1), 40.0, W / H)
    flags = resoct.RENDER_ADAPTIVE_STEP | resoct.RENDER_CHANNEL_RATES
    res = p.frame(1, cam, W, H, 0.5, chans, lod_bias=1.3, flags=flags)
    p.check_frame(res, f"rates-{m}-{resident}")
    assert W * H < 1000 or (res["tot"] > 0 and len(res["ids"]) > 32)
