"""Streams binned in one launch, in one part and several, where a tile holds most of the stream and where all do: against the
count and scatter of the same stream, which always take the general way. The same drop count; coefficients within 1e-5
relative and composites within 1e-5 (the order of FP64 sums differs, then FP32 rounding); gradients, which are zero for
fragments out of range or NaN, within 1e-4 of those of the same stream padded past the largest small one."""
import numpy as np
import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height,channels,where", [(1, 1, 1, "all"), (64, 64, 1, "corner"), (64, 64, 3, "end"),
                                                         (200, 100, 1, "sorted"), (64, 64, 3, "all")])
def test_parts_of_small_streams(width, height, channels, where):
    import torch
    import paper_2201_00094_amd as wt
    P, bg = width * height, (0.2, 0.3, 0.4)
    rng = np.random.default_rng(P + channels)
    spec = wt.FrameSpec(width, height, 3, channels)
    for F, shift in [(16383, 0), (16384, 1), (16385, 0), (16387, 2), (32768, 0), (32769, 0), (32771, 3), (40960, 0), (40961, 1), (40963, 0), (49151, 0), (65533, 1), (65536, 0)]:
        say("case small parts", width, height, channels, where, F, shift)
        pixel = rng.integers(0, P, F).astype(np.uint32)
        if where == "corner":
            pixel[rng.random(F) < 0.9] = 1
        elif where == "end":
            pixel[rng.random(F) < 0.9] = P - 1
        elif where == "sorted":
            pixel.sort()
        depth = rng.random(F, dtype=np.float32)
        alpha = (0.02 * rng.random((F, 3) if channels == 3 else F, dtype=np.float32)).astype(np.float32)
        rgb = rng.random((F, 3), dtype=np.float32)
        bad = [5, 16380, F - 1, 40]
        pixel[5], pixel[16380], pixel[F - 1] = P, 0xffffffff, P + 7
        depth[17], alpha.reshape(F, -1)[40, 0] = np.nan, np.nan
        t = [torch.from_numpy(a).cuda() for a in (pixel.view(np.int32), depth, alpha, rgb)]
        if shift:  # arrays that start off a 16-byte boundary
            t = [torch.cat([a.new_zeros((shift,) + a.shape[1:]), a])[shift:] for a in t]
        fr = wt.Fragments(*t)
        a, b = wt.Workspace(spec, F), wt.Workspace(spec, F)
        ca, cb = spec.new_coeffs(), spec.new_coeffs()
        oa = wt.render(spec, fr, bg, a, coeffs=ca)
        ob = torch.empty_like(oa)
        wt.bin_count(spec, fr, b)
        wt.bin_scatter(spec, fr, b)
        wt.render_binned(spec, b, bg, ob, coeffs=cb)
        assert wt.dropped_count(a) == wt.dropped_count(b) == 5
        assert (oa - ob).abs().max() <= 1e-5 and torch.allclose(ca, cb, rtol=1e-5, atol=0)
        # gradients: the stream as it is, and behind 70,000 fragments of no tile
        accum = spec.new_accum()
        wt.evaluate(spec, fr, ca, accum, a)
        g = torch.from_numpy(rng.standard_normal((P, 3)).astype(np.float32)).cuda()
        nan = float("nan")
        ga, gr = torch.full_like(t[2], nan), torch.full_like(t[3], nan)
        wt.backward(spec, fr, ca, accum, bg, g, a, ga, gr)
        n = 70000
        pad = [torch.cat([x.new_full((n,) + x.shape[1:], P if k == 0 else 0.5), x]) for k, x in enumerate(t)]
        big = wt.Workspace(spec, F + n)
        gb, grb = wt.backward(spec, wt.Fragments(*pad), ca, accum, bg, g, big)
        torch.cuda.synchronize()
        assert torch.isfinite(ga).all() and torch.isfinite(gr).all()
        assert not ga[bad].any() and not gr[bad].any()
        assert (ga - gb[n:]).abs().max() <= 1e-4 * max(1.0, float(gb.abs().max())) and (gr - grb[n:]).abs().max() <= 1e-4
