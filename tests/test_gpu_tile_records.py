"""The tile kernel's record loops at the counts where they change form: tiles whose records are fewer than a batch, fill
the records a thread keeps between the build and the evaluation exactly, one more, and leave whole or half batches over.
One-tile and few-tile frames against the oracle at the parity contract (coefficients 1e-5 relative, composite 1e-4)."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu

COUNTS = [1, 63, 255, 257, 1023, 1025, 3073, 4095, 4097, 5121, 12287, 12289, 16383, 16385, 20481, 24577, 33001]


def _stream(rng, pixels, F, channels):
    pixel = rng.integers(0, pixels, F).astype(np.uint32)
    depth = rng.random(F, dtype=np.float32)
    alpha = (0.01 + 0.5 * rng.random((F, 3) if channels == 3 else F, dtype=np.float32)).astype(np.float32)
    return pixel, depth, alpha, rng.random((F, 3), dtype=np.float32)


@pytest.mark.parametrize("channels,tight,rank,dtype", [(1, False, 3, "f32"), (1, True, 4, "f32"), (3, False, 3, "f32"),
                                                       (3, True, 2, "f32"), (1, False, 1, "f32")])
def test_record_counts(orc, channels, tight, rank, dtype):
    import torch
    import paper_2201_00094_amd as wt
    W, H = 16, 12
    rng = np.random.default_rng(100 * rank + channels)
    spec = wt.FrameSpec(W, H, rank, channels, dtype, tight=tight)
    for F in COUNTS:
        say("case tile records", channels, tight, rank, F)
        pixel, depth, alpha, rgb = _stream(rng, W * H, F, channels)
        fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
        coeffs = spec.new_coeffs()
        out = wt.render(spec, fr, (0.2, 0.3, 0.4), wt.Workspace(spec, F), coeffs=coeffs)
        torch.cuda.synchronize()
        o = orc.resolve(W, H, rank, pixel, depth, alpha, rgb, bg=(0.2, 0.3, 0.4), channels=channels, tight=tight,
                        want=("coeffs", "out"))
        gc = coeffs.cpu().double().numpy()
        assert (gc[o["coeffs"] == 0] == 0).all()
        assert (np.abs(gc - o["coeffs"]) <= 1e-5 * np.abs(o["coeffs"])).all(), F
        assert np.abs(out.cpu().double().numpy() - o["out"]).max() <= 1e-4, F
