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


# Tiles of heights that are no power of two, last rows and columns cut, one and two binning levels (super-tiles of odd
# heights), small frames with small tiles: (width, height, rank, channels, tight, mean fragments per pixel)
SHAPES = [(70, 45, 3, 1, False, 9.0), (333, 201, 3, 3, False, 6.0), (640, 360, 4, 1, True, 3.0), (517, 1031, 2, 3, False, 2.0),
          (2100, 1701, 3, 3, False, 0.4), (1601, 1203, 4, 3, True, 0.5), (65, 16500, 3, 1, False, 0.6)]


@pytest.mark.parametrize("width,height,rank,channels,tight,mean", SHAPES)
def test_tile_shapes(orc, width, height, rank, channels, tight, mean):
    import torch
    import paper_2201_00094_amd as wt
    say("case tile shapes", width, height, rank, channels, tight)
    rng = np.random.default_rng(width)
    F = int(width * height * mean)
    pixel, depth, alpha, rgb = _stream(rng, width * height, F, channels)
    pixel[:2] = 0, width * height - 1
    spec = wt.FrameSpec(width, height, rank, channels, tight=tight)
    fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
    coeffs, ws = spec.new_coeffs(), wt.Workspace(spec, F)
    out = wt.render(spec, fr, (0.1, 0.2, 0.3), ws, coeffs=coeffs)
    torch.cuda.synchronize()
    assert wt.dropped_count(ws) == 0
    o = orc.resolve(width, height, rank, pixel, depth, alpha, rgb, bg=(0.1, 0.2, 0.3), channels=channels, tight=tight,
                    want=("coeffs", "out"))
    gc = coeffs.cpu().double().numpy()
    assert (gc[o["coeffs"] == 0] == 0).all()
    assert (np.abs(gc - o["coeffs"]) <= 1e-5 * np.abs(o["coeffs"])).all()
    assert np.abs(out.cpu().double().numpy() - o["out"]).max() <= 1e-4


@pytest.mark.parametrize("width,height,rank,channels", [(1700, 1401, 3, 3), (2203, 1703, 4, 1)])
def test_gradient_two_levels(orc, width, height, rank, channels):
    """Records that keep the stream index through super-tiles and the split (more than 8192 gradient tiles)."""
    import torch
    import paper_2201_00094_amd as wt
    say("case gradient two levels", width, height, rank, channels)
    rng = np.random.default_rng(height)
    F = width * height // 3
    pixel, depth, alpha, rgb = _stream(rng, width * height, F, channels)
    spec = wt.FrameSpec(width, height, rank, channels)
    fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
    ws, coeffs, accum = wt.Workspace(spec, F), spec.new_coeffs(), spec.new_accum()
    wt.build(spec, fr, coeffs, ws)
    wt.evaluate(spec, fr, coeffs, accum, ws)
    g = rng.standard_normal((width * height, 3)).astype(np.float32)
    ga, gr = wt.backward(spec, fr, coeffs, accum, (0.1, 0.2, 0.3), torch.from_numpy(g).cuda(), ws)
    torch.cuda.synchronize()
    oa, og = orc.backward(width, height, rank, pixel, depth, alpha, rgb, g, bg=(0.1, 0.2, 0.3), channels=channels)
    assert np.abs(ga.cpu().double().numpy().reshape(F, channels) - oa).max() <= 1e-3
    assert np.abs(gr.cpu().double().numpy() - og).max() <= 1e-4


@pytest.mark.parametrize("channels,tight,rank,dtype", [(1, False, 3, "f32"), (3, False, 3, "f16"), (1, True, 4, "f32"),
                                                       (3, False, 2, "e5b9g9r9"), (1, False, 5, "f32")])
def test_gradient_counts(orc, channels, tight, rank, dtype):
    """Gradients into arrays that hold NaN, at the counts where the record loops change form, with fragments that are in
    no tile (pixel out of range) or dropped in one (NaN depth or alpha): every element is written, theirs with zero."""
    import torch
    import paper_2201_00094_amd as wt
    W, H, bg = 16, 12, (0.2, 0.3, 0.4)
    rng = np.random.default_rng(7 * rank + channels)
    spec = wt.FrameSpec(W, H, rank, channels, dtype, tight=tight)
    for F in [9, 255, 1025, 2047, 4097, 8191, 8193, 12289, 16385, 20481, 33001]:
        say("case gradient counts", channels, tight, rank, dtype, F)
        pixel, depth, alpha, rgb = _stream(rng, W * H, F, channels)
        alpha *= np.float32(0.02)  # thousands of fragments per pixel
        pixel[F // 3], pixel[F - 1] = W * H, 0xfffffff0
        depth[F // 2] = np.nan
        alpha.reshape(F, -1)[1, channels - 1] = np.nan
        bad = np.zeros(F, bool)
        bad[[1, F // 3, F // 2, F - 1]] = True
        fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
        ws, coeffs, accum = wt.Workspace(spec, F), spec.new_coeffs(), spec.new_accum()
        wt.build(spec, fr, coeffs, ws)
        wt.evaluate(spec, fr, coeffs, accum, ws)
        g = rng.standard_normal((W * H, 3)).astype(np.float32)
        ga = torch.full((F,) if channels == 1 else (F, 3), float("nan"), device="cuda")
        gr = torch.full((F, 3), float("nan"), device="cuda")
        wt.backward(spec, fr, coeffs, accum, bg, torch.from_numpy(g).cuda(), ws, ga, gr)
        torch.cuda.synchronize()
        ga, gr = ga.cpu().double().numpy().reshape(F, channels), gr.cpu().double().numpy()
        assert (ga[bad] == 0).all() and (gr[bad] == 0).all(), F
        assert np.isfinite(ga).all() and np.isfinite(gr).all(), F
        assert wt.dropped_count(ws) == 4
        if dtype == "f32":  # the oracle's gradient is that of exact storage
            oa, og = orc.backward(W, H, rank, pixel, depth, alpha, rgb, g, bg=bg, channels=channels, tight=tight)
            scale = max(1.0, np.abs(oa).max())
            assert np.abs(ga - oa).max() <= 1e-3 * scale and np.abs(gr - og).max() <= 1e-4, F


@pytest.mark.parametrize("channels,rank,dtype", [(1, 3, "f32"), (3, 3, "f16"), (3, 2, "e5b9g9r9"), (1, 5, "bf16")])
def test_render_accum_matches_the_passes(orc, channels, rank, dtype):
    """The accumulation written by the one-pass render against evaluate's from the same coefficients (FP32 sums of FP64
    totals on both sides: 2e-6 relative), the padding words zero, composite and coefficients those of render."""
    import torch
    import paper_2201_00094_amd as wt
    from paper_2201_00094_amd.wt import render_accum
    W, H, bg, F = 53, 38, (0.2, 0.3, 0.4), 24000
    say("case render accum", channels, rank, dtype)
    rng = np.random.default_rng(rank)
    fr = wt.Fragments.from_numpy(*_stream(rng, W * H, F, channels))
    spec = wt.FrameSpec(W, H, rank, channels, dtype)
    ws = wt.Workspace(spec, F)
    nan = float("nan")
    out = torch.full((spec.pixels, 3), nan, device="cuda")
    accum = torch.full((spec.pixels, spec.accum_width), nan, device="cuda")
    coeffs = torch.full_like(spec.new_coeffs(), 7)
    render_accum(spec, fr, bg, ws, out, coeffs, accum)
    c2 = spec.new_coeffs()
    o2 = wt.render(spec, fr, bg, ws, coeffs=c2)
    a2 = spec.new_accum()
    wt.evaluate(spec, fr, coeffs, a2, ws)
    torch.cuda.synchronize()
    assert torch.allclose(coeffs.float(), c2.float(), rtol=1e-2 if dtype != "f32" else 1e-6, atol=1e-6)
    assert (out - o2).abs().max() <= 1e-5
    assert ((accum - a2).abs() <= 2e-6 * a2.abs().clamp(min=1e-3)).all()
    if channels == 3:
        assert (accum[:, 3] == 0).all() and (accum[:, 7] == 0).all()


@pytest.mark.parametrize("width,height,taps", [(1, 300, 5), (300, 1, 7), (1398102, 2, 5), (1398101, 2, 11), (129, 67, 3)])
def test_chromatic_addressing(orc, width, height, taps):
    """The composite's two addressing forms at their border (row pitch 12 x width at 2^24 bytes), one-pixel rows and
    columns, offsets past every edge: within 1e-4 of the oracle (the contract of the chromatic tests)."""
    import torch
    import paper_2201_00094_amd as wt
    say("case chromatic addressing", width, height, taps)
    rng = np.random.default_rng(width)
    P = width * height
    spec = wt.FrameSpec(width, height, 3)
    accum, image = rng.random((P, 4), dtype=np.float32), rng.random((P, 3), dtype=np.float32)
    offset = rng.uniform(-40, 40, (P, 2)).astype(np.float32)
    offset[:2] = (-1e6, 1e6), (3e9, -3e9)
    out = wt.resolve_chromatic(spec, *(torch.from_numpy(a).cuda() for a in (accum, image, offset)), 0.5, taps)
    ref = orc.resolve_chromatic(width, height, accum[:, :3], accum[:, 3:], image, offset, 0.5, taps)
    assert np.abs(out.cpu().double().numpy() - ref).max() <= 1e-4


@pytest.mark.parametrize("width,height,rank,channels", [(16, 12, 3, 1), (64, 64, 3, 3), (250, 130, 4, 1), (31, 700, 2, 3),
                                                        (9, 9, 6, 1)])
def test_small_streams_match_the_general_binning(width, height, rank, channels):
    """Streams binned in one launch against count + scatter of the same stream (which always take the general way), on
    both sides of the largest small stream, aligned and not, with fragments out of range and NaN: the same drop count,
    composites within 1e-5 (the order of FP64 sums differs, then FP32 rounding), gradients within 1e-4 of each other."""
    import torch
    import paper_2201_00094_amd as wt
    rng = np.random.default_rng(width + height)
    bg, P = (0.2, 0.3, 0.4), width * height
    spec = wt.FrameSpec(width, height, rank, channels)
    for F, shift in [(1, 0), (3, 1), (7, 0), (2048, 0), (4099, 1), (16384, 0), (65535, 2), (65536, 0), (65537, 0)]:
        say("case small streams", width, height, rank, channels, F, shift)
        pixel, depth, alpha, rgb = _stream(rng, P, F, channels)
        alpha *= np.float32(0.1)
        if F > 100:
            pixel[5], pixel[F - 1] = P, 0xffffffff
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
        assert wt.dropped_count(a) == wt.dropped_count(b) == (4 if F > 100 else 0)
        assert (oa - ob).abs().max() <= 1e-5 and torch.allclose(ca, cb, rtol=1e-5, atol=0)
        oc = torch.empty_like(oa)
        wt.render_binned(spec, a, bg, oc)  # the workspace serves later calls
        assert (oa - oc).abs().max() <= 1e-5
        with pytest.raises(ValueError):
            wt.bin_scatter(spec, fr, a)


# Both sides of every edge of the scatter that stays on its compute unit: whole and halved chunks (2048, with at most 512
# tiles), one or several of them per workgroup, a partial last chunk and a partial last group of four.
@pytest.mark.parametrize("width,height,rank,channels,F,shift", [
    (250, 130, 3, 1, 3, 0), (250, 130, 3, 1, 4, 1), (250, 130, 3, 1, 2047, 3), (250, 130, 3, 1, 2049, 1),
    (400, 300, 3, 1, 70001, 2), (250, 130, 3, 1, 1048579, 3), (250, 130, 4, 1, 1048575, 1), (250, 130, 2, 1, 5300003, 1),
    (1100, 900, 3, 1, 5, 1), (1100, 900, 3, 1, 4097, 2), (1100, 900, 4, 1, 300003, 3), (300, 200, 2, 3, 6291455, 1),
    (300, 200, 2, 3, 6291458, 1), (1366, 768, 3, 3, 6291459, 3), (2100, 1100, 3, 1, 300001, 1)])
def test_streamed_scatter(orc, width, height, rank, channels, F, shift):
    """Coefficients of one binning against the sum of builds of pieces that are binned in one launch: FP32 sums of at most
    106 pieces, each rounded once, so within 107 x 2^-24 < 1e-5 of each other; drop counts; gradients against the oracle
    (one fragment per pixel or fewer, so the bounds of the two-level gradients)."""
    import torch
    import paper_2201_00094_amd as wt
    say("case streamed scatter", width, height, rank, channels, F, shift)
    rng = np.random.default_rng(F)
    P = width * height
    pixel, depth, alpha, rgb = _stream(rng, P, F, channels)
    alpha *= np.float32(min(1.0, P / F))
    if F > 100:
        pixel[5], pixel[F - 1] = P, 0xffffffff
        depth[17], alpha.reshape(F, -1)[40, 0] = np.nan, np.nan
    t = [torch.from_numpy(a).cuda() for a in (pixel.view(np.int32), depth, alpha, rgb)]
    if shift:  # arrays that start off a 16-byte boundary
        t = [torch.cat([a.new_zeros((shift,) + a.shape[1:]), a])[shift:] for a in t]
    spec = wt.FrameSpec(width, height, rank, channels)
    fr = wt.Fragments(*t)
    ws, small = wt.Workspace(spec, F), wt.Workspace(spec, F)
    whole, parts = spec.new_coeffs(), spec.new_coeffs()
    wt.bin_count(spec, fr, ws)
    wt.bin_scatter(spec, fr, ws)
    wt.build_binned(spec, whole, ws)
    assert wt.dropped_count(ws) == (4 if F > 100 else 0)
    piece = max(50000 if P < 100000 else 16000, F // 105)  # (the longer ones are staged in rounds)
    for i in range(0, F, piece):
        wt.build(spec, wt.Fragments(*[a[i:i + piece] for a in t]), parts, small)
    assert torch.allclose(whole, parts, rtol=1e-5, atol=0)
    if F > P or F < 70001:
        return
    g = rng.standard_normal((P, 3)).astype(np.float32)
    accum = spec.new_accum()
    wt.evaluate(spec, fr, whole, accum, ws)
    ga, gr = wt.backward(spec, fr, whole, accum, (0.1, 0.2, 0.3), torch.from_numpy(g).cuda(), ws)
    torch.cuda.synchronize()
    ga, gr = ga.cpu().double().numpy().reshape(F, channels), gr.cpu().double().numpy()
    out = np.zeros(F, bool)
    out[[5, 17, 40, F - 1]] = True
    assert (ga[out] == 0).all() and (gr[out] == 0).all()
    oa, og = orc.backward(width, height, rank, pixel[~out], depth[~out], alpha[~out], rgb[~out], g, bg=(0.1, 0.2, 0.3),
                          channels=channels)
    assert np.abs(ga[~out] - oa).max() <= 1e-3
    assert np.abs(gr[~out] - og).max() <= 1e-4


@pytest.mark.parametrize("rank", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("width,height", [(1, 1), (37, 53), (333, 201)])
def test_packed_words_of_the_render(width, height, rank):
    """The words that a render packs are those that a build packs: the same FP64 sums (one thread, stream order), rounded
    to FP32 and packed by the same rule, so equal in every bit, for columns of every length and tiles cut by the frame;
    and a render that stores no words shows the same frame."""
    import torch
    import paper_2201_00094_amd as wt
    say("case packed words", width, height, rank)
    rng = np.random.default_rng(width + rank)
    F = 4 * width * height + 3
    spec = wt.FrameSpec(width, height, rank, 3, "e5b9g9r9", deterministic=True)
    fr = wt.Fragments.from_numpy(*_stream(rng, width * height, F, 3))
    ws, a, b = wt.Workspace(spec, F), spec.new_coeffs(), spec.new_coeffs()
    out = wt.render(spec, fr, (0.1, 0.2, 0.3), ws, coeffs=a)
    wt.build(spec, fr, b, ws)
    assert a.dtype == b.dtype and torch.equal(a, b) and bool((a != 0).any())
    assert torch.equal(out, wt.render(spec, fr, (0.1, 0.2, 0.3), ws))
