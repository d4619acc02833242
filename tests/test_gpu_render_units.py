"""Frames at the edges of what the ray kernel splits: viewports around the
4 x 4-pixel units and 32 x 32 tiles, channel counts around the groups of
four and the lanes of a ray, transfer functions of one colour, of several
colours and with several zero runs (some across the 64-entry words of the
table scan), plain and adaptive, against the oracle: image, requests, usage."""
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


def _tf(kind, c):
    x = np.arange(256) / 255.0
    if kind == "one":
        return synth.tf_hue(0.13 * c, 0.3)
    if kind == "ramp":
        t = synth.tf_ramp()
        t[:, 3] *= 0.3
        return t
    # zero runs 0..63, 64+c..130, 190..193 and 255
    t = np.stack([x, 1 - x, np.full(256, 0.5), 0.2 + 0.3 * x], 1).astype(np.float32)
    for lo, hi in ((0, 63), (64 + c, 130), (190, 193), (255, 255)):
        t[lo:hi + 1, 3] = 0
    return t


@pytest.fixture(scope="module")
def volumes():
    return {(m, bits): synth.BlobVolume((40, 33, 29), n_channels=m, bits=bits, n_levels=3, seed=3 + m, n_blobs=12,
                                        spacing=(1, 1, 1))
            for m, bits in ((16, 8), (12, 16), (4, 16))}


@pytest.mark.parametrize("m,bits,vis,W,H,kind,adaptive", [
    (4, 16, (2,), 3, 5, "one", False),
    (4, 16, (0, 1, 2, 3), 17, 4, "gaps", False),
    (4, 16, (3, 0), 33, 15, "ramp", True),
    (12, 16, tuple(range(12)), 31, 33, "one", False),
    (12, 16, (11, 1, 5, 0, 7), 8, 9, "gaps", True),
    (12, 16, tuple(range(3, 12)), 20, 20, "ramp", False),
    (16, 8, tuple(range(16)), 37, 18, "one", True),
    (16, 8, tuple(range(15, 2, -1)), 16, 32, "gaps", False),
])
def test_units_channels_and_tables(volumes, m, bits, vis, W, H, kind, adaptive):
    src = volumes[m, bits]
    p = Pair(src, 16, (8, 8, 8), 3, n_slots=400, start_level=1)
    ids = p.gpu.all_ids()
    rng = np.random.default_rng(m * 100 + W)
    p.upload(0, ids[rng.random(len(ids)) < 0.6])
    p.check_masks()
    top = 255 if bits == 8 else 65535
    chans = [dict(c=c, lo=j % 2 if kind == "gaps" else 0, hi=2, W0=0, W1=top * 256, tf=_tf(kind, c))
             for j, c in enumerate(vis)]
    cam = synth.camera_persp((75.0, -31.0, 44.0), (20.0, 16.0, 14.0), (0, 0, 1), 38.0, W / H)
    for f, flags in ((1, resoct.RENDER_ADAPTIVE_STEP if adaptive else 0), (2, resoct.RENDER_NO_SKIP)):
        res = p.frame(f, cam, W, H, 0.5, chans, lod_bias=1.5, flags=flags)
        p.check_frame(res, f"units-{m}-{kind}-{W}x{H}-{flags}")
