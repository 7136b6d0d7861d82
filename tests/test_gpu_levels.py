"""Binnings in one and in two levels at the sizes where they change, with the number of levels asserted. The capacity that a
refused call names tells it: a workspace holds half the records of a layout that keeps two copies of each."""
import ctypes as C
import re

import numpy as np
import pytest

import synth
from gpu_helpers import assert_close_abs, assert_coeffs, say

pytestmark = pytest.mark.gpu

BG = (0.1, 0.2, 0.3)


def _stream(rng, pixels, F, channels):
    pixel = rng.integers(0, pixels, F).astype(np.uint32)
    depth = rng.random(F, dtype=np.float32)
    alpha = (0.01 + 0.5 * rng.random((F, 3) if channels == 3 else F, dtype=np.float32)).astype(np.float32)
    return pixel, depth, alpha, rng.random((F, 3), dtype=np.float32)


def levels(spec, gradient=False):
    """Binning levels of a description (1 or 2), from the records that 64 GB hold. Validation only: nothing is enqueued."""
    from paper_2201_00094_amd import _lib
    lib, size, p = _lib.load(), 64 << 30, C.c_void_p(0x1000)
    frags = _lib.Fragments(_lib.WT_MAX_FRAGMENTS, 8, 8, 8, 8)
    if gradient:
        st = lib.wt_backward(C.byref(spec.c_desc()), C.byref(frags), p, p, _lib.bg3(BG), p, p, p, p, size, None)
    else:
        st = lib.wt_bin(C.byref(spec.c_desc()), C.byref(frags), p, size, None)
    assert st == _lib.WT_ERR_RANGE
    holds = int(re.search(r"holds (\d+) fragments", lib.wt_last_error().decode()).group(1))
    return round(size / (4 * (6 + spec.channels)) / holds)


def test_noalloc_past_two_levels():
    """A frame past two levels of its largest tiles, whose own tiles are binned in two: as many fragments as fit the static
    array twice, and more, which go in one level; composites within 1e-5 of render's (the order of FP64 sums differs)."""
    import torch
    import paper_2201_00094_amd as wt
    spec = wt.FrameSpec(398, 38445, 6, 3)
    assert levels(spec) == 2
    rng = np.random.default_rng(6)
    for F in (1000003, 5000001):
        say("case noalloc past two levels", F)
        fr = wt.Fragments.from_numpy(*_stream(rng, spec.pixels, F, 3))
        out = torch.full((spec.pixels, 3), float("nan"), device="cuda")
        wt.render_noalloc(spec, fr, BG, out)
        ref = wt.render(spec, fr, BG, wt.Workspace(spec, F))
        torch.cuda.synchronize()
        assert (out - ref).abs().max() <= 1e-5


@pytest.mark.parametrize("width,height,rank,channels,F,deterministic", [
    (2700, 1800, 4, 1, 1500001, False), (1, 600000, 3, 1, 900001, False), (3, 300000, 3, 3, 900001, False),
    (640, 640, 8, 1, 400001, False), (640, 640, 8, 1, 60001, True), (3, 300000, 3, 3, 60001, True)])
def test_two_levels(orc, width, height, rank, channels, F, deterministic):
    """Forward binnings in two levels, one and three channels, by the parallel scatter and split and by the serial one: about
    3,000 pixels with fragments and the first and last against the oracle at the parity contract, the others background."""
    import torch
    import paper_2201_00094_amd as wt
    say("case two levels", width, height, rank, channels, F, deterministic)
    P = width * height
    rng = np.random.default_rng(P + channels)
    pixel, depth, alpha, rgb = _stream(rng, P, F, channels)
    pixel[:2] = 0, P - 1
    spec = wt.FrameSpec(width, height, rank, channels, deterministic=deterministic)
    assert levels(spec) == 2
    fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
    ws, coeffs = wt.Workspace(spec, F), spec.new_coeffs()
    out = wt.render(spec, fr, BG, ws, coeffs=coeffs)
    torch.cuda.synchronize()
    assert wt.dropped_count(ws) == 0
    sel = np.unique(np.concatenate([[0, P - 1], pixel[rng.choice(F, 3000, replace=False)]]))
    keep = np.isin(pixel, sel)
    o = orc.resolve(sel.size, 1, rank, np.searchsorted(sel, pixel[keep]).astype(np.uint32), depth[keep], alpha[keep], rgb[keep],
                    bg=BG, channels=channels, want=("coeffs", "out"))
    at = torch.from_numpy(sel.astype(np.int64)).cuda()
    assert_coeffs(coeffs[at].cpu().double().numpy(), o["coeffs"])
    assert_close_abs(out[at].cpu().double().numpy(), o["out"], 1e-4)
    empty = torch.ones(P, dtype=torch.bool, device="cuda")
    empty[torch.from_numpy(pixel.astype(np.int64)).cuda()] = False
    assert bool((out[empty] == torch.tensor(BG, device="cuda")).all()) and not coeffs[empty].any()


@pytest.mark.parametrize("width,height,channels", [(896, 1024, 1), (240, 3824, 1), (448, 512, 3), (120, 1912, 3)])
def test_bins_of_a_short_chunk(orc, width, height, channels):
    """3,584 tiles, the most that are scattered in short chunks, and 3,585, at rank 5 (power-of-two tiles): three channels
    with just enough fragments for the streamed scatter. Against the oracle at the parity contract, about 2,000 pixels."""
    import torch
    import paper_2201_00094_amd as wt
    say("case bins of a short chunk", width, height, channels)
    P, F = width * height, 1000003 if channels == 1 else 6 * 256 * 4096 + 3
    rng = np.random.default_rng(P)
    pixel, depth, alpha, rgb = _stream(rng, P, F, channels)
    alpha *= np.float32(min(1.0, 2.0 * P / F))
    spec = wt.FrameSpec(width, height, 5, channels)
    fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
    ws, coeffs = wt.Workspace(spec, F), spec.new_coeffs()
    out = wt.render(spec, fr, BG, ws, coeffs=coeffs)
    torch.cuda.synchronize()
    assert wt.dropped_count(ws) == 0
    sel = np.unique(np.concatenate([[0, P - 1], rng.choice(P, 2000, replace=False)]))
    keep = np.isin(pixel, sel)
    o = orc.resolve(sel.size, 1, 5, np.searchsorted(sel, pixel[keep]).astype(np.uint32), depth[keep], alpha[keep], rgb[keep],
                    bg=BG, channels=channels, want=("coeffs", "out"))
    at = torch.from_numpy(sel.astype(np.int64)).cuda()
    assert_coeffs(coeffs[at].cpu().double().numpy(), o["coeffs"])
    assert_close_abs(out[at].cpu().double().numpy(), o["out"], 1e-4)


@pytest.mark.parametrize("width,height,channels", [(896, 512, 1), (240, 1912, 1), (448, 512, 3), (120, 1912, 3)])
def test_gradient_bins_of_a_short_chunk(orc, width, height, channels):
    """The same border for records that keep the stream index, against the oracle's gradient (the bounds of the two-level
    gradients)."""
    import torch
    import paper_2201_00094_amd as wt
    say("case gradient bins of a short chunk", width, height, channels)
    P, F = width * height, 700001
    rng = np.random.default_rng(P)
    pixel, depth, alpha, rgb = _stream(rng, P, F, channels)
    spec = wt.FrameSpec(width, height, 5, channels)
    fr = wt.Fragments.from_numpy(pixel, depth, alpha, rgb)
    ws, coeffs, accum = wt.Workspace(spec, F), spec.new_coeffs(), spec.new_accum()
    wt.build(spec, fr, coeffs, ws)
    wt.evaluate(spec, fr, coeffs, accum, ws)
    g = rng.standard_normal((P, 3)).astype(np.float32)
    ga, gr = wt.backward(spec, fr, coeffs, accum, BG, torch.from_numpy(g).cuda(), ws)
    torch.cuda.synchronize()
    oa, og = orc.backward(width, height, 5, pixel, depth, alpha, rgb, g, bg=BG, channels=channels)
    assert np.abs(ga.cpu().double().numpy().reshape(F, channels) - oa).max() <= 1e-3
    assert np.abs(gr.cpu().double().numpy() - og).max() <= 1e-4


def test_two_levels_past_2_31_fragments(orc):
    """Three visibility channels, 2^31 + 12,345 fragments over a 2600x1400 rank-3 frame, binned in two levels: record indices
    and offsets past 2^31 in the super-tiles and in the split. No drops, and 40 pixels with their whole lists of about 590
    fragments against the oracle. Skipped where the device has no room for the 237 GB this takes."""
    import torch
    import paper_2201_00094_amd as wt
    W, H, F = 2600, 1400, (1 << 31) + 12345
    P = W * H
    spec = wt.FrameSpec(W, H, 3, 3)
    assert levels(spec) == 2
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    need = 32 * F + wt.workspace_bytes(spec, F) + (3 * 16 * 4 + 12) * P + (8 << 30)
    if free < need:
        pytest.skip("needs %.0f GB of device memory, %.0f GB free" % (need / 1e9, free / 1e9))
    say("case two levels past 2^31: F", F)
    pixel, depth, alpha, rgb, A, B = synth.scrambled_stream(9, W, H, F, channels=3)
    torch.cuda.empty_cache()  # the generator's temporaries
    fr = wt.Fragments(pixel, depth, alpha, rgb)
    ws, coeffs = wt.Workspace(spec, F), spec.new_coeffs()
    out = wt.render(spec, fr, BG, ws, coeffs=coeffs)
    torch.cuda.synchronize()
    assert wt.dropped_count(ws) == 0
    rag = F % P
    firsts = np.unique(np.concatenate([[0, P - 1, rag - 1, rag, (F - 1) % P],
                                       np.random.default_rng(9).choice(P, 35, replace=False)]))
    sel = (A * firsts + B) % P
    lists = []
    for j, first in enumerate(firsts):
        idx = torch.arange(int(first), F, P, device="cuda")
        assert bool((pixel[idx] == int(sel[j])).all())
        lists.append((np.full(idx.numel(), j, np.uint32), depth[idx].cpu().numpy(), alpha[idx].cpu().numpy(),
                      rgb[idx].cpu().numpy()))
    mp, md, ma, mc = (np.concatenate([p[k] for p in lists]) for k in range(4))
    o = orc.resolve(len(lists), 1, 3, mp, md, ma, mc, bg=BG, channels=3, want=("coeffs", "out"))
    at = torch.from_numpy(sel).cuda()
    assert_coeffs(coeffs[at].cpu().double().numpy(), o["coeffs"])
    assert_close_abs(out[at].cpu().double().numpy(), o["out"], 1e-4)
    del pixel, depth, alpha, rgb, fr, ws, coeffs, out
    torch.cuda.empty_cache()
