"""Binnings in one and in two levels at the sizes where they change, with the number of levels asserted. The capacity that a
refused call names tells it: a workspace holds half the records of a layout that keeps two copies of each."""
import ctypes as C
import re

import numpy as np
import pytest

from gpu_helpers import say

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
