"""Frame geometry on the host (no GPU): the tiles, levels and tables that the library chooses for a description, compiled
for the host from its own sources."""
import ctypes as C
import os
import shutil
import subprocess

import pytest

from paper_2201_00094_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("geom") / "geom_check"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2201_00094_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", "geom_check.cpp"), "-o", str(exe)],
                          stderr=subprocess.DEVNULL)

    def run(name, *args):
        res = subprocess.run([str(exe), name, *(str(a) for a in args)], capture_output=True, text=True, timeout=300)
        assert res.returncode == 0 and "bad 0" in res.stdout, res.stdout
        return res.stdout
    return run


def test_frames_at_the_size_limits(check):
    """Descriptions of nearly 2^32 pixels in one row or column get tables for all their tiles; the few whose tiles cannot
    be numbered are refused (they ended the process with a division by zero)."""
    check("limits")
    lib = _lib.load()
    d = _lib.desc(1, (1 << 32) - 1, 10, 3)
    assert lib.wt_workspace_bytes(C.byref(d), 10) > 4 * ((1 << 32) - 1)
    frags, ws, bg = _lib.Fragments(10, 8, 8, 8, 8), C.c_void_p(0x1000), _lib.bg3((0, 0, 0))  # never dereferenced
    assert lib.wt_bin(C.byref(d), C.byref(frags), ws, 16, None) == _lib.WT_ERR_UNSUPPORTED
    assert lib.wt_backward(C.byref(d), C.byref(frags), ws, ws, bg, ws, ws, ws, ws, 16, None) == _lib.WT_ERR_UNSUPPORTED
    d = _lib.desc(1, (1 << 32) - 1, 9, 3)
    assert lib.wt_bin(C.byref(d), C.byref(frags), ws, 16, None) == _lib.WT_ERR_RANGE


def test_last_tile_of_any_frame(check):
    """A tile's rows past the frame stay outside it, also where row numbers would wrap at 2^32."""
    check("last_tile")


def test_scratch_takes_what_the_largest_tiles_take(check):
    """The fragments that wt_render_noalloc takes do not become fewer by the choice of tiles and binning levels."""
    check("scratch")


def test_tile_shape_search(check):
    """Every call makes its geometry anew, so the search of the tile shape is bounded; it finds what the full one finds."""
    check("shapes")


def test_frames_of_the_gpu_tests(check):
    """The binning levels and tiles that the GPU tests of them rely on: (width, height, rank, channels, flags, gradient)."""
    for frame in [(2700, 1800, 4, 1, 0, 0), (1, 600000, 3, 1, 0, 0), (3, 300000, 3, 3, 0, 0), (640, 640, 8, 1, 4, 0),
                  (3, 300000, 3, 3, 4, 0), (2600, 1400, 3, 3, 0, 0), (398, 38445, 6, 3, 0, 0), (1700, 1401, 3, 3, 0, 1),
                  (2203, 1703, 4, 1, 0, 1), (2100, 1701, 3, 3, 0, 0), (1601, 1203, 4, 3, 1, 0), (2000, 1100, 4, 3, 0, 0)]:
        assert "levels 2" in check("describe", *frame), frame
    for frame, tiles in [((896, 1024, 5, 1, 0, 0), 3584), ((240, 3824, 5, 1, 0, 0), 3585), ((448, 512, 5, 3, 0, 0), 3584),
                         ((120, 1912, 5, 3, 0, 0), 3585), ((896, 512, 5, 1, 0, 1), 3584), ((240, 1912, 5, 1, 0, 1), 3585),
                         ((448, 512, 5, 3, 0, 1), 3584), ((120, 1912, 5, 3, 0, 1), 3585)]:
        assert "tiles %d levels 1" % tiles in check("describe", *frame), frame


def test_rows_of_tiles(check):
    check("rows")
