"""The kernels' launch order, compiled for the host: every item goes to one XCD
once, and no XCD gets a one-sided share of what the items are part of."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from paper_2012_03325_amd import epb as E
from tests.test_abi import _Batch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2012_03325_amd", "csrc")

# prints the XCD of every item: in contiguous shares, or in the shading pass's chunks
PROBE = r"""
#include "tile_order.hpp"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv) {
    bool chunked = std::atoi(argv[1]) != 0;
    int total = std::atoi(argv[2]);
    unsigned char *owner = (unsigned char *)std::malloc(total);
    for (int i = 0; i < total; ++i) owner[i] = 255;
    for (int x = 0; x < epb::kNumXcd; ++x) {
        epb::XcdShare s = epb::xcd_share(x, total);
        for (int it = 0; it < s.count; ++it) {
            int g = chunked ? epb::xcd_chunk_item(x, it, total) : s.first + it;
            if (!chunked && g != epb::xcd_tile(it * epb::kNumXcd + x, total)) return 3;
            if (g < 0 || g >= total || owner[g] != 255) return 1;
            owner[g] = (unsigned char)x;
        }
    }
    return std::fwrite(owner, 1, total, stdout) == (size_t)total ? 0 : 2;
}
"""


@pytest.fixture(scope="module")
def owners(tmp_path_factory):
    d = tmp_path_factory.mktemp("order")
    (d / "probe.cpp").write_text(PROBE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", "/opt/rocm/include",
                    str(d / "probe.cpp"), "-o", str(d / "probe")], check=True)

    def run(chunked, total):
        r = subprocess.run([str(d / "probe"), str(int(chunked)), str(total)], capture_output=True)
        assert r.returncode == 0, f"an item twice, never or out of range ({total} items)"
        return np.frombuffer(r.stdout, np.uint8)
    return run


@pytest.mark.parametrize("total", [1, 7, 8, 63, 64, 65, 511, 512, 513, 1023, 1024, 1031, 1535, 1536, 8100, 65537])
def test_every_item_once(owners, total):
    for chunked in (0, 1):
        o = owners(chunked, total)
        assert (o < 8).all()
        counts = np.bincount(o, minlength=8)
        assert counts.max() - counts.min() <= 1


@pytest.mark.parametrize("views", [5, 12, 32, 64, 256])
@pytest.mark.parametrize("tiles", [64, 128, 192, 256, 320, 510, 512, 576, 1024])
def test_batch_of_equal_views(owners, views, tiles):
    """Every XCD takes each tile of the view about equally often (a contiguous share of L items
    holds a position of a view of T tiles floor(L / T) or ceil(L / T) times)."""
    o = owners(0, views * tiles).reshape(views, tiles)
    per = np.stack([(o == x).sum(0) for x in range(8)])
    assert per.max() - per.min() <= 1


@pytest.mark.parametrize("width", [1920, 2048, 3840, 4096, 6144, 8192, 10240, 16384])
@pytest.mark.parametrize("height", [1024, 2160, 4096])
def test_columns_of_an_image(owners, width, height):
    """In the shading pass's chunks every XCD gets about its eighth of each quarter of the columns.
    (1024 rows of 8192 pixels are 512 chunks, 16 of each quarter to an XCD: up to 4 more or less.)"""
    tx, ty = -(-width // 32), -(-height // 8)
    o = owners(1, tx * ty)
    quarter = np.arange(tx * ty) % tx * 4 // tx
    for x in range(8):
        share = np.bincount(quarter[o == x], minlength=4) / np.bincount(quarter) * 8
        assert (abs(share - 1) < 0.25).all(), (x, share)


@pytest.mark.parametrize("tiles,views", [(256, 256), (512, 64), (300, 100)])
def test_small_views_beside_a_large_one(owners, tiles, views):
    """In chunks an XCD's share of each quarter of the small views is about an eighth (a chunk of 64
    tiles is at least an eighth of such a view: 64 views of 512 tiles are 128 chunks of each quarter,
    16 of them an XCD's, up to 4 more or less)."""
    o = owners(1, 8192 + tiles * views)[8192:]
    quarter = np.arange(o.size) % tiles * 4 // tiles
    for x in range(8):
        share = np.bincount(quarter[o == x], minlength=4) / np.bincount(quarter) * 8
        assert (abs(share - 1) < 0.25).all(), (x, share)


# views of up to 4096 tiles of 32 x 8 pixels by contiguous shares, larger ones in chunks
@pytest.mark.parametrize("sizes,chunks", [([(256, 256)] * 16, 0), ([(320, 240)] * 8, 0), ([(64, 48)], 0),
                                          ([(256, 256)] * 8 + [(512, 512)], 0), ([(1280, 720)] * 3, 0),
                                          ([(2048, 512)], 0), ([(2048, 513)], 1), ([(1920, 1080)] * 2, 1),
                                          ([(1920, 1080), (1280, 720), (640, 480), (320, 240)] * 3, 1)])
def test_order_of_a_batch(sizes, chunks):
    """The shading stage's order in the table's header: never chunks in a grid that loops."""
    b = _Batch(sizes)
    for blocks_per_cu in (0, 1, 8):
        assert b.build(sched=E.epb_schedule(0, 0, 0, blocks_per_cu, 0, 0, 0)) == E.EPB_OK
        words = list(C.cast(b.table, C.POINTER(C.c_int32 * 37)).contents)
        assert words[36] == (chunks if blocks_per_cu == 0 else 0)
