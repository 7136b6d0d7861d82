"""Ranks whose tiles hold coefficients instead of cells (M > 32): the record loops at the counts where they change form, with
tiles of many pixels and of one or two. Against the oracle at the parity contract (coefficients 1e-5 relative, composite and
accumulated colour 1e-4), and the accumulation of the evaluate pass."""
import numpy as np
import pytest

from gpu_helpers import accum_to_oracle_layout, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rank,channels,tight", [(5, 1, False), (5, 3, True), (8, 1, True), (8, 3, False), (10, 1, False),
                                                 (10, 3, True)])
def test_record_counts(orc, rank, channels, tight):
    import torch
    import paper_2201_00094_amd as wt
    W, H, bg = 3, 2, (0.2, 0.3, 0.4)
    rng = np.random.default_rng(10 * rank + channels)
    spec = wt.FrameSpec(W, H, rank, channels, tight=tight)
    for F in [1, 511, 513, 1023, 1025, 2049, 4097, 6143, 6145, 8193, 12301]:
        say("case high rank", rank, channels, tight, F)
        pixel = rng.integers(0, W * H, F).astype(np.uint32)
        pixel[: F // 2] = 4  # half of them in one pixel
        depth = rng.random(F, dtype=np.float32)
        alpha = (0.002 + 0.02 * rng.random((F, 3) if channels == 3 else F, dtype=np.float32)).astype(np.float32)
        rgb = rng.random((F, 3), dtype=np.float32)
        o = orc.resolve(W, H, rank, pixel, depth, alpha, rgb, bg=bg, channels=channels, tight=tight,
                        want=("coeffs", "accum", "suma", "out"))
        fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
        ws, coeffs, accum = wt.Workspace(spec, F), spec.new_coeffs(), spec.new_accum()
        out = wt.render(spec, fr, bg, ws, coeffs=coeffs)
        wt.evaluate(spec, fr, coeffs, accum, ws)
        torch.cuda.synchronize()
        gc = coeffs.cpu().double().numpy().reshape(o["coeffs"].shape)
        assert (gc[o["coeffs"] == 0] == 0).all(), F
        assert (np.abs(gc - o["coeffs"]) <= 1e-5 * np.abs(o["coeffs"])).all(), F
        assert np.abs(out.cpu().double().numpy() - o["out"]).max() <= 1e-4, F
        s, a = accum_to_oracle_layout(accum.cpu().double().numpy(), channels)
        assert np.abs(s - o["accum"].reshape(s.shape)).max() <= 1e-4, F
        assert np.abs(a - o["suma"].reshape(a.shape)).max() <= 1e-5 * max(1.0, np.abs(o["suma"]).max()), F
