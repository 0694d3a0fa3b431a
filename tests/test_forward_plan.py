"""The forms that the layer outputs take by their sizes and the workspace they ask for, without a GPU: the header that the
library is built from, in a small C++ library of its own."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MIB = 1 << 20


class Plan:
    def __init__(self, lib):
        so = ctypes.CDLL(lib)
        i64, ptr = ctypes.c_int64, ctypes.POINTER
        for name, args in (("product_k_parts", [i64] * 6 + [ptr(ctypes.c_int), ptr(i64)]), ("compact_k_parts", [i64] * 6),
                           ("product_workspace", [i64, i64]),
                           ("compact_product_workspace", [i64, i64, ctypes.c_int, i64, i64, ctypes.c_int]),
                           ("compact_fills_tiles", [i64, i64]), ("product_streams", [i64, i64]), ("masks_by_list", [i64, i64, i64]),
                           ("list_pays", [i64] * 4)):
            fn = getattr(so, name)
            fn.argtypes = args
            fn.restype = i64 if name.endswith("workspace") else ctypes.c_int
            setattr(self, name, fn)

    def parts(self, pairs, experts, d_model, d_ff, m_tiles, dense=False):
        """(parts of K with m_tiles token tiles, the most parts and the workgroups that the call was planned for)"""
        least, most = (m_tiles, m_tiles) if dense else (-(-pairs // 256), pairs // 256 + min(pairs, experts))
        assert least <= m_tiles <= most
        most_parts, blocks = ctypes.c_int(), ctypes.c_int64()
        taken = self.product_k_parts(m_tiles, least, most, d_model, d_ff, pairs, ctypes.byref(most_parts), ctypes.byref(blocks))
        return taken, most_parts.value, blocks.value


@pytest.fixture(scope="session")
def plan(tmp_path_factory):
    return build_plan(tmp_path_factory.mktemp("plan"))


def build_plan(folder):
    gxx = shutil.which("g++") or "/opt/rocm/lib/llvm/bin/clang++"
    if not os.path.exists(gxx):
        pytest.skip("no C++ compiler")
    lib = os.path.join(str(folder), "forward_plan.so")
    res = subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "native", "forward_plan.cpp"), "-o", lib],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return Plan(lib)


SHAPES = [  # experts, top_k (0: dense), d_model, d_ff
    (8, 2, 4096, 14336), (64, 8, 3584, 2560), (64, 6, 2048, 1408), (1, 0, 3584, 20480), (2, 0, 2048, 2816), (4, 1, 256, 14336),
    (8, 2, 1024, 4096), (16, 2, 64, 960), (256, 8, 2048, 1024),
]
TOKENS = sorted({int(1.09 ** i) for i in range(115)} | {63, 64, 65, 255, 256, 257, 8192})


@pytest.mark.parametrize("experts,top_k,d_model,d_ff", SHAPES)
def test_no_smaller_batch_outgrows_the_workspace_of_a_larger_one(plan, experts, top_k, d_model, d_ff):
    """The parts of K change the size of the product rows the other way round from the batch (up to eight times them for a small
    one): the room made for a batch holds those of every smaller one, so that nothing is allocated after the largest.  Whatever
    number of token tiles the routing makes, its parts fit the room and the workgroups."""
    row, split, largest = 4 * d_model, 0, 0
    n_tiles = -(-d_model // 256)
    room = {"whole": 0, "compact": 0}
    for n in TOKENS:
        pairs = n * (top_k or experts)
        tiles = range(-(-pairs // 256), pairs // 256 + min(pairs, experts) + 1) if top_k else [experts * -(-n // 256)]
        for m in list(tiles)[:: max(1, len(tiles) // 12)] + [tiles[-1]]:
            parts, most, blocks = plan.parts(pairs, experts, d_model, d_ff, m, dense=not top_k)
            assert 1 <= parts <= most
            assert blocks % 8 == 0 and blocks // 8 >= -(-m * n_tiles // 8) * parts   # a die's share of the tiles, once per part
            assert parts == 1 or (parts * pairs * row < 256 * MIB and parts * 8 <= -(-d_ff // 64))
            assert not (most > 1 and plan.product_streams(pairs, d_model))
            split += parts > 1
            largest = max(largest, parts * pairs * row)
        room_now = plan.product_workspace(pairs * row, d_ff)
        assert room_now >= max(room["whole"], largest) and room_now <= max(pairs * row, 256 * MIB)
        room["whole"] = room_now
        # compacted: the streaming kernels' chunks of K below 65 tokens per expert, parts of K from there
        chunks = max(1, min(8, -(-d_ff // 3072)))
        tiled = plan.compact_fills_tiles(pairs, experts)
        assert tiled == (pairs // experts > 64)
        room_now = plan.compact_product_workspace(pairs, experts, tiled, row, d_ff, chunks)
        parts = plan.compact_k_parts(n, experts, top_k, 0, d_model, d_ff)
        assert parts == 1 or (parts * pairs * row < 256 * MIB and parts * 8 <= -(-d_ff // 64))
        assert room_now >= room["compact"] and room_now >= (parts if tiled else chunks) * pairs * row
        room["compact"] = room_now
    assert split or d_ff < 16 * 64                      # the shapes from 16 K tiles on do split at some size


def test_k_stays_whole_where_its_tiles_fill_the_rounds(plan):
    """The tiles of a die run on its 32 units: 250 parts of tiles are no single round where a die gets 35 of them.  Token tiles,
    pairs, experts, d_model, d_ff of second contractions that were slower in the parts of a guess, and of some that are fastest
    in parts."""
    for m_tiles, pairs, experts, d_model, d_ff, best in (
            (13, 2000, 8, 4096, 14336, {1}), (16, 3400, 8, 4096, 14336, {1}), (16, 3800, 8, 4096, 14336, {1}),
            (27, 6000, 8, 4096, 14336, {1}), (20, 4096, 8, 4096, 14336, {3}), (8, 800, 8, 4096, 14336, {2}),
            (47, 8192, 32, 512, 2048, {2}), (32, 4600, 24, 768, 2048, {2}), (17, 2703, 12, 2048, 4096, {1}), (5, 64, 5, 2560, 9000, {4}),
            (2, 300, 1, 3584, 20480, {6, 7, 8}), (3, 520, 1, 3584, 20480, {5}), (16, 4096, 1, 3584, 20480, {1}),
            (8, 1000, 8, 768, 3072, {4, 5, 6})):
        parts, _, _ = plan.parts(pairs, experts, d_model, d_ff, m_tiles)
        assert parts in best, (m_tiles, pairs, d_model, d_ff, parts)
    # no number of tiles that these pairs can make is better in parts: nothing is prepared for them
    assert plan.parts(9000, 8, 4096, 14336, 40)[1:] == (1, (9000 // 256 + 8) * 16)


def test_list_of_kept_micro_experts_where_it_leaves_enough_out(plan):
    """Token tiles, d_model, d_ff, pairs and the share pruned (in every expert alike) of masked calls: by list where that was
    faster when measured, everything computed where it was not (masks that keep nearly everything, few rounds of tiles)."""
    for m_tiles, d_model, d_ff, pairs, pruned, by_list in (
            (20, 4096, 14336, 4096, 0.0, False), (20, 4096, 14336, 4096, 0.02, False), (20, 4096, 14336, 4096, 0.2, True),
            (20, 4096, 14336, 4096, 0.4, True), (128, 2048, 1408, 24576, 0.05, False),
            (128, 2048, 1408, 24576, 0.3, True), (64, 3584, 2560, 5600, 0.1, False), (64, 3584, 2560, 5600, 0.25, True),
            (3, 3584, 20480, 600, 0.3, False), (3, 3584, 20480, 600, 0.6, True), (8, 4096, 14336, 800, 0.1, False),
            (8, 4096, 14336, 800, 0.15, True), (280, 3584, 2560, 65536, 0.05, False), (280, 3584, 2560, 65536, 0.2, True)):
        assert plan.masks_by_list(pairs, d_model, d_ff)
        tiles = lambda width: m_tiles * -(-width // 128)
        kept = d_ff - int(pruned * d_ff)
        zero_bytes = 2 * pairs * d_ff if pruned else 0
        got = plan.list_pays(tiles(kept), tiles(d_ff), -(-d_model // 64), zero_bytes)
        assert bool(got) == by_list, (m_tiles, d_model, d_ff, pairs, pruned)
