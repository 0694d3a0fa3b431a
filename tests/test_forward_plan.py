"""The forms that the layer outputs take by their sizes and the workspace they ask for, without a GPU: the header that the
library is built from, in a small C++ library of its own."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MIB = 1 << 20


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++") or "/opt/rocm/lib/llvm/bin/clang++"
    if not os.path.exists(gxx):
        pytest.skip("no C++ compiler")
    lib = str(tmp_path_factory.mktemp("plan") / "forward_plan.so")
    res = subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(ROOT, "tests", "native", "forward_plan.cpp"), "-o", lib],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    so = ctypes.CDLL(lib)
    i64 = ctypes.c_int64
    for name, args in (("expected_m_tiles", [i64, i64]), ("product_k_parts", [i64, i64, i64]), ("product_workspace", [i64, i64]),
                       ("compact_product_workspace", [i64, i64, ctypes.c_int, i64, i64, ctypes.c_int]),
                       ("compact_fills_tiles", [i64, i64]), ("product_streams", [i64, i64]), ("masks_by_list", [i64, i64, i64])):
        getattr(so, name).argtypes = args
        getattr(so, name).restype = i64 if name.startswith("expected") or name.endswith("workspace") else ctypes.c_int
    return so


SHAPES = [  # experts, top_k (0: dense), d_model, d_ff
    (8, 2, 4096, 14336), (64, 8, 3584, 2560), (64, 6, 2048, 1408), (1, 0, 3584, 20480), (2, 0, 2048, 2816), (4, 1, 256, 14336),
    (8, 2, 1024, 4096), (16, 2, 64, 960), (256, 8, 2048, 1024),
]
TOKENS = sorted({int(1.09 ** i) for i in range(115)} | {63, 64, 65, 255, 256, 257, 8192})


@pytest.mark.parametrize("experts,top_k,d_model,d_ff", SHAPES)
def test_no_smaller_batch_outgrows_the_workspace_of_a_larger_one(plan, experts, top_k, d_model, d_ff):
    """The parts of K change the size of the product rows the other way round from the batch (up to eight times them for a small
    one): the room made for a batch holds those of every smaller one, so that nothing is allocated after the largest."""
    row, split, largest = 4 * d_model, 0, 0
    room = {"whole": 0, "compact": 0}
    for n in TOKENS:
        pairs = n * (top_k or experts)
        tiles = (experts * -(-n // 256) if not top_k else plan.expected_m_tiles(pairs, experts)) * -(-d_model // 256)
        parts = plan.product_k_parts(tiles, d_ff, pairs * row)
        split += parts > 1
        largest = max(largest, parts * pairs * row)
        assert parts == 1 or (parts * pairs * row < 256 * MIB and parts * 8 <= -(-d_ff // 64))
        assert not (parts > 1 and plan.product_streams(pairs, d_model))
        room_now = plan.product_workspace(pairs * row, d_ff)
        assert room_now >= max(room["whole"], largest) and room_now <= max(pairs * row, 256 * MIB)
        room["whole"] = room_now
        # compacted: the streaming kernels' chunks of K below 65 tokens per expert, parts of K from there
        chunks = max(1, min(8, -(-d_ff // 3072)))
        tiled = plan.compact_fills_tiles(pairs, experts)
        assert tiled == (pairs // experts > 64)
        room_now = plan.compact_product_workspace(pairs, experts, tiled, row, d_ff, chunks)
        assert room_now >= room["compact"] and room_now >= (parts if tiled else chunks) * pairs * row
        room["compact"] = room_now
    assert split or d_ff < 16 * 64                      # the shapes from 16 K tiles on do split at some size
