"""The composite's reads of a row's two texels at once: images of one, two and three columns, taps inside, at and past every
edge, unaligned images, and the addressing of three taps over a large three-channel accumulation, against the oracle (1e-4,
the contract of the chromatic tests)."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height,channels", [(1, 5, 1), (2, 1, 3), (2, 300, 1), (3, 7, 3), (64, 33, 1), (2100, 2000, 3)])
def test_pairs(orc, width, height, channels):
    import torch
    import paper_2201_00094_amd as wt
    rng = np.random.default_rng(width + height)
    P = width * height
    spec = wt.FrameSpec(width, height, 3, channels)
    accum = rng.random((P, 8 if channels == 3 else 4), dtype=np.float32)
    image = rng.random((P, 3), dtype=np.float32)
    offset = (rng.uniform(-1.5, 1.5, (P, 2)) * min(width, 20)).astype(np.float32)
    offset[::3] = np.round(offset[::3])
    padded = torch.from_numpy(np.concatenate([np.zeros(1, np.float32), image.reshape(-1)])).cuda()
    for taps in (3, 5, 7, 9, 11, 63) if P < 100000 else (3,):
        say("case chromatic pairs", width, height, channels, taps)
        for shift in (False, True):
            im = padded[1:].view(P, 3) if shift else torch.from_numpy(image).cuda()  # 4 bytes off a 16-byte boundary
            out = wt.resolve_chromatic(spec, torch.from_numpy(accum).cuda(), im, torch.from_numpy(offset).cuda(), 0.7, taps)
            ref = orc.resolve_chromatic(width, height, accum[:, :3], accum[:, 3:4] if channels == 1 else accum[:, 4:7],
                                        image, offset, 0.7, taps, channels=channels)
            assert np.abs(out.cpu().double().numpy() - ref).max() <= 1e-4, taps
