"""How a pool launch, in HBM or over the link, splits its pieces over waves, emulated on the CPU (no GPU).

tests/cpp/pool_emu.cpp runs every wave and lane of a launch over the kernel's own walk and index maps
(mma_pool.h), with fixed shares and with claims, and checks bounds and that each destination byte is written
exactly once; the result is compared here with the oracle, in the piece and head-major layouts and both
directions.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import kv as okv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    out = str(tmp_path_factory.mktemp("pool") / "libpoolemu.so")
    cmd = [cxx, "-std=c++17", "-O1", "-g", "-shared", "-fPIC", "-Wall",
           f"-I{os.path.join(ROOT, 'paper_2512_16056_amd', 'csrc')}",
           os.path.join(ROOT, "tests", "cpp", "pool_emu.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    lib = ctypes.CDLL(out)
    f = lib.emu_pool
    f.restype = ctypes.c_int
    f.argtypes = ([ctypes.c_void_p, ctypes.c_uint64] * 2 + [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint32,
                  ctypes.c_uint64, ctypes.c_uint32] + [ctypes.c_int] * 4 + [ctypes.c_uint32] * 3)
    f.xp = lib.emu_pool_xp
    f.xp.restype = ctypes.c_int
    f.xp.argtypes = ([ctypes.c_void_p, ctypes.c_uint64] * 2 + [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint32,
                     ctypes.c_uint64, ctypes.c_uint32] + [ctypes.c_int] * 3 + [ctypes.c_uint32] * 3)
    f.div = lib.emu_div
    f.div.restype = ctypes.c_uint64
    f.div.argtypes = [ctypes.c_uint32] * 3
    f.last_counter = lib.emu_last_counter
    f.last_counter.restype = ctypes.c_uint32
    f.last_counter.argtypes = [ctypes.c_uint32, ctypes.c_int, ctypes.c_uint32]
    f.finish = lib.emu_finish
    f.finish.restype = ctypes.c_int
    f.finish.argtypes = [ctypes.c_void_p, ctypes.c_uint32, ctypes.c_int, ctypes.c_uint32]
    f.claims = lib.emu_noalloc_claims
    f.claims.restype = ctypes.c_int
    f.claims.argtypes = [ctypes.c_uint32] * 5
    f.long_spans = lib.emu_long_spans
    f.long_spans.argtypes = [ctypes.c_uint32, ctypes.c_uint64]
    return f


# tokens, heads, row bytes, layers, blocks: pieces of one unit, several to a row with lanes left over and
# a short last row, just over half a row, exactly one row, a row and a unit, many rows with a short last
# one; head rows that do and do not divide a wave's row
SHAPES = [(1, 1, 16, 1, 5), (3, 1, 80, 2, 7), (16, 1, 64, 3, 9), (11, 3, 16, 1, 4), (13, 5, 16, 1, 3), (16, 5, 160, 2, 4),
          (16, 4, 96, 3, 5), (16, 8, 64, 1, 3), (16, 8, 256, 2, 5), (16, 8, 272, 1, 3), (32, 8, 512, 1, 2),
          (7, 3, 1040, 1, 3), (16, 2, 2048, 1, 2)]


# workgroups over the link (0: in HBM) and whether their waves claim spans
@pytest.mark.parametrize("link,claims", [(0, 0), (1, 0), (2, 1), (24, 0), (24, 1)])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("layout", [okv.LAYOUT_PIECE, okv.LAYOUT_HND])
def test_pool_index_maps_match_oracle(emu, shape, layout, link, claims):
    B, H, R, L, n = shape
    piece, ppb, nb, slots = B * H * R, 2 * L, n + 3, n + 2
    geom = (B, H, R, 1)
    r = np.random.default_rng(B * 31 + H + R)
    pool = r.integers(0, 256, (slots, ppb * piece), dtype=np.uint8)
    cache = r.integers(0, 256, (L, 2, nb, piece), dtype=np.uint8)
    hs = r.permutation(slots)[:n].astype(np.int32)
    gb = np.sort(r.permutation(nb)[:n]).astype(np.int32)
    tab = hs.astype(np.uint64) | (gb.astype(np.uint64) << np.uint64(32))

    def run(p, c, to_paged):
        rc = emu(p.ctypes.data, p.nbytes, c.ctypes.data, c.nbytes, tab.ctypes.data, n, ppb, piece, nb, to_paged,
                 int(layout == okv.LAYOUT_HND), link, claims, B, H, R)
        assert rc == 0, rc

    got = cache.copy()
    run(pool.copy(), got, 1)
    for l in range(L):
        assert np.array_equal(got[l], okv.kv_fetch_layer(pool, cache[l], l, L, hs, gb, layout, geom)), l
    got = pool.copy()
    run(got, cache.copy(), 0)
    assert np.array_equal(got, okv.kv_offload(pool, list(cache), gb, hs, layout, geom))


# tokens, heads, head_dim, element bytes, layers, blocks: squares of 8 x 8 units and shapes they do not
# divide, pieces that share a row, each element size; value rows that go through a tile, the last ones short
XP_SHAPES = [(16, 8, 128, 2, 2, 4), (16, 1, 64, 2, 3, 9), (16, 5, 80, 2, 1, 3), (16, 4, 96, 1, 2, 5),
             (32, 2, 16, 1, 1, 6), (8, 3, 16, 2, 2, 5), (24, 1, 24, 2, 1, 3), (4, 8, 16, 4, 2, 3), (2, 5, 8, 8, 1, 7),
             (32, 8, 80, 1, 1, 3), (16, 8, 64, 4, 1, 2), (2, 5, 128, 8, 1, 2), (128, 2, 64, 2, 1, 2)]


# workgroups over the link (0: in HBM) and whether their waves claim spans
@pytest.mark.parametrize("link,claims", [(0, 0), (1, 0), (2, 1), (24, 0), (24, 1)])
@pytest.mark.parametrize("shape", XP_SHAPES)
def test_pool_xpacked_maps_match_oracle(emu, shape, link, claims):
    B, H, D, E, L, n = shape
    piece, nb, slots, geom = B * H * D * E, n + 3, n + 2, (B, H, D, E)
    r = np.random.default_rng(B * 31 + H + D)
    pool = r.integers(0, 256, (slots, 2 * L * piece), dtype=np.uint8)
    cache = r.integers(0, 256, (L, 2, nb, piece), dtype=np.uint8)
    hs = r.permutation(slots)[:n].astype(np.int32)
    gb = np.sort(r.permutation(nb)[:n]).astype(np.int32)
    tab = hs.astype(np.uint64) | (gb.astype(np.uint64) << np.uint64(32))

    def run(p, c, to_paged):
        rc = emu.xp(p.ctypes.data, p.nbytes, c.ctypes.data, c.nbytes, tab.ctypes.data, n, L, piece, nb, to_paged, link,
                    claims, B, H * D * E // 16, E)
        assert rc == 0, rc

    got = cache.copy()
    run(pool.copy(), got, 1)
    for l in range(L):
        assert np.array_equal(got[l], okv.kv_fetch_layer(pool, cache[l], l, L, hs, gb, okv.LAYOUT_XPACKED, geom)), l
    got = pool.copy()
    run(got, cache.copy(), 0)
    assert np.array_equal(got, okv.kv_offload(pool, list(cache), gb, hs, okv.LAYOUT_XPACKED, geom))


def test_division_by_reciprocal(emu):
    for d in [*range(1, 130), 255, 256, 257, 4095, 4096, 4097, 65521, 2 ** 28 - 1, 2 ** 28, 2 ** 31 + 1, 2 ** 32 - 1]:
        for first in {0, max(d - 500, 0), 2 ** 28 // d * d - min(500, 2 ** 28 // d * d), 2 ** 32 - 1000}:
            bad = emu.div(d, first, 1000)
            assert bad == 0, (d, bad - 1)


def test_finish_counters_keep_off_the_claims(emu):
    """Counter 1 holds the claims of a launch that has them; without claims 64 groups fit the counters."""
    for grid in [1, 15, 16, 31, 32, 33, 48, 96, 255, 256, 384]:
        assert emu.last_counter(grid, 1, 64) == 0, grid
    for grid, last in [(1, 0), (31, 0), (32, 2), (1024, 64), (16384, 64)]:
        assert emu.last_counter(grid, 0, 64) == last, grid


@pytest.mark.parametrize("grid", [1, 15, 16, 31, 32, 33, 48, 96, 384, 1024, 1025, 16384])
def test_finish_counters_are_reset_before_the_done_tag(emu, grid):
    """The done tag frees the launch's counters for another one: with each store of 0 held back until
    the workgroup that made it waits for it, none is outstanding when the last workgroup writes the tag."""
    r = np.random.default_rng(grid)
    for claims in (0, 1):
        for _ in range(3):
            order = r.permutation(grid).astype(np.uint32)
            rc = emu.finish(order.ctypes.data, grid, claims, 64)
            assert rc == 0, (grid, claims, rc)


@pytest.mark.parametrize("overlap", [1, 2, 16])
def test_noalloc_claims_after_calls_that_overlap(emu, overlap):
    """Fetches without allocations share their claim words: calls that overlapped, against the rule,
    leave none that makes a later call skip or repeat a span."""
    for seed in range(30):
        for before in (0, 5, 33):
            bad = emu.claims(before, overlap, 6, 40, seed)
            assert bad == 0, (seed, before, bad - 1)


def test_few_workgroups_over_the_link_take_long_spans(emu):
    for wgs, piece, want in [(3, 32768, 1), (11, 16384, 1), (12, 32768, 0), (24, 65536, 0), (3, 8192, 0), (0, 32768, 0)]:
        assert emu.long_spans(wgs, piece) == want, (wgs, piece)
