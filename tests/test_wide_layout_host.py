"""Rows of the LDS slots that the 256 x 256 prefill kernel reads (csrc/wide_layout.h: plain C++, which the
kernel compiles too), without a GPU: every fragment read lies in its slot, also the ones that a narrow
or absent next tile has no use for, and the fragments that are used cover the tile without overlap."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2510_12357_amd", "csrc")


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    if cxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path_factory.mktemp("wide") / "wide_layout_check")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "wide_layout_check.cpp"), "-o", out], check=True)
    return subprocess.run([out], capture_output=True, text=True, check=True).stdout.splitlines()


@pytest.fixture(scope="module")
def reads(output):
    slot_rows, lds = map(int, output[0].split())
    rows = [line.split() for line in output[1:] if not line.startswith("k")]
    return slot_rows, lds, [(int(m), int(t), int(nb), int(w), op, int(f), int(r), int(at)) for m, t, nb, w, op, f, r, at in rows]


def test_every_fragment_read_lies_in_its_slot(reads):
    slot_rows, lds, rows = reads
    assert lds == 160 * 1024
    assert len(rows) == 2 * (5 + 2) * 4 * 4 * 2
    for m, t, nb, w, op, f, r, at in rows:
        assert 0 <= r and r + 32 <= slot_rows, (m, t, nb, w, op, f, r)
        assert at + 32 * 128 <= lds, (m, t, nb, w, op, f, at)


def test_used_fragments_cover_the_tile_once(reads):
    slot_rows, _, rows = reads
    for mode in (0, 1):
        for tall, nbs in ((1, (3, 4)), (0, (1, 2, 3, 4))):
            for nb in nbs:
                mine = [x for x in rows if x[:3] == (mode, tall, nb)]
                used = [0, 1, 2, 3] if tall else [0, 2 if mode else 1]
                a = {w: [x[6] for x in mine if x[3] == w and x[4] == "a" and x[5] < nb] for w in range(4)}
                b = {w: [x[6] for x in mine if x[3] == w and x[4] == "b" and x[5] in used] for w in range(4)}
                cells = sorted((i, j) for w in range(4) for i in a[w] for j in b[w])
                assert cells == sorted((i, j) for i in range(0, (2 if tall else 1) * nb * 32, 32) for j in range(0, slot_rows, 32))
                if mode:      # gate and up rows of the same outputs in one wave
                    for w in range(4):
                        assert {j + 128 for j in b[w] if j < 128} == {j for j in b[w] if j >= 128}


def test_load_offsets_stay_below_the_stated_size(output):
    """Chunk i of a tile is loaded at scalar offset 128 i, also where a short K has no such chunk; behind the
    last tile (K = 0) up to three more.  The size that the descriptor states covers the offset, and
    is not larger than the tensor unless that is shorter than the ring."""
    cursors = [list(map(int, line.split()[1:])) for line in output if line.startswith("k")]
    assert [c[0] for c in cursors] == list(range(0, 329, 8))
    for K, chunks, size in cursors:
        assert chunks == max(3, (K + 63) // 64)
        assert 128 * (chunks - 1) <= size, K
        assert size == max(2 * K, 3 * 128), K
