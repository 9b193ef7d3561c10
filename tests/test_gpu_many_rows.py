"""Requests of a MiB and more, where the planner chooses stores, word and rows per thread by row length and pitch:
both directions of shapes on either side of its lines, byte for byte against the C oracle, with the choice."""
import numpy as np
import pytest

import workloads as W
from workloads import BYTE, contiguous, hvector
from oracle import typemap_c as cc
from paper_2012_14363_amd import binding as tp

torch = pytest.importorskip("torch")

#: run, pitch, rows, typed offset, what the unpack plan says, what the pack plan says
SHAPES = [
    (12, 13, 90001, 5, "W=4 ux=1 ur=4 nt=3", "W=2 ux=1 ur=4"),      # rows share their lines
    (33, 63, 40000, 1, "W=8 ux=1 ur=1 nt=3", "W=16 ux=1 ur=4"),     # closer than half a line
    (33, 66, 40000, 1, "W=8 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (40, 191, 30000, 0, "W=8 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (40, 192, 30000, 0, "W=4 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (127, 150, 10000, 3, "W=16 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),  # they share lines, but are at most 4 MiB
    (127, 150, 34000, 3, "W=16 ux=1 ur=1 nt=3", "W=16 ux=1 ur=4"),
    (1, 8, 4200000, 3, "W=1 ux=1 ur=1 nt=7", "W=1 ux=1 ur=4"),      # eight times the run apart
    (1, 8, 4190000, 3, "W=1 ux=1 ur=4 nt=3", "W=1 ux=1 ur=4"),      # at most 4 MiB
    (7, 55, 600000, 3, "W=4 ux=1 ur=4 nt=3", "W=1 ux=1 ur=4"),      # not quite
    (7, 56, 600000, 3, "W=1 ux=1 ur=1 nt=7", "W=1 ux=1 ur=4"),
    (8, 128, 140000, 1, "W=1 ux=1 ur=1 nt=7", "W=2 ux=1 ur=4"),     # bytes: two rows to a line
    (31, 255, 40000, 1, "W=4 ux=1 ur=1 nt=7", "W=4 ux=1 ur=4"),
    (32, 257, 40000, 1, "W=2 ux=1 ur=1 nt=7", "W=4 ux=1 ur=4"),
    (17, 1023, 70000, 1, "W=2 ux=1 ur=1 nt=7", "W=4 ux=1 ur=4"),    # translations decide from 1 KiB on
    (17, 1024, 70000, 1, "W=4 ux=1 ur=1 nt=7", "W=4 ux=1 ur=4"),
    (128, 383, 9001, 1, "W=16 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),   # one or two lines at an odd address, below and from 384 on
    (256, 384, 9001, 1, "W=8 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (257, 385, 9001, 1, "W=16 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (1500, 1501, 2000, 1, "W=16 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (129, 512, 9001, 0, "W=8 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),
    (24, 600, 50000, 7, "W=2 ux=1 ur=1 nt=7", "W=4 ux=1 ur=4"),
    (12, 300, 90000, 7, "W=1 ux=1 ur=1 nt=7", "W=2 ux=1 ur=4"),
    (3, 64, 400001, 5, "W=1 ux=1 ur=1 nt=7", "W=1 ux=1 ur=4"),
    (64, 192, 20000, 64, "W=8 ux=1 ur=1 nt=7", "W=16 ux=1 ur=4"),   # whole 64-byte blocks
    (40, 4096, 27000, 0, "W=4 ux=1 ur=4 nt=3", "W=16 ux=1 ur=4"),   # a page apart
    (128, 512, 40000, 0, "W=16 ux=1 ur=1 nt=7", "W=16 ux=1 ur=1"),  # whole lines, more than 4 MiB
    (1024, 1024 + 30, 5000, 2, "W=16 ux=1 ur=1 nt=7", "W=16 ux=1 ur=1"),
    (1025, 1025 + 33, 5000, 2, "W=16 ux=1 ur=1 nt=3", "W=16 ux=1 ur=1"),
    (2408, 2648, 2000, 40, "W=16 ux=1 ur=1 nt=3", "W=16 ux=1 ur=1"),
    (5001, 6000, 1000, 0, "W=16 ux=2 ur=2 nt=3", "W=16 ux=2 ur=2"),  # 313 words: two-word tiles
    (9000, 9001, 600, 1, "W=16 ux=1 ur=1 nt=3", "W=16 ux=1 ur=1"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("run,pitch,rows,offset,unpack_plan,pack_plan", SHAPES)
def test_many_rows(run, pitch, rows, offset, unpack_plan, pack_plan):
    dev = torch.device("cuda:0")
    recipe = hvector(rows, 1, pitch, contiguous(run, BYTE))
    print("many rows", run, pitch, rows, offset, flush=True)
    h = tp.type_from_recipe(recipe)
    size, span = run * rows, rows * pitch + offset + 64
    typed_h, packed_h = W.random_bytes(run, span), W.random_bytes(pitch, size)
    typed, out = torch.from_numpy(typed_h).to(dev), torch.full((size + 3,), 0xEE, dtype=torch.uint8, device=dev)
    assert tp.pack(typed.data_ptr() + offset, 1, h, out, size + 3, 3) == size + 3
    assert pack_plan in tp.last_plan(), tp.last_plan()
    want = np.full(size + 3, 0xEE, np.uint8)
    cc.pack(typed_h, offset, 1, recipe, want, 3)
    assert np.array_equal(out.cpu().numpy(), want)
    packed = torch.from_numpy(packed_h).to(dev)
    assert tp.unpack(packed, size, 0, typed.data_ptr() + offset, 1, h) == size
    assert unpack_plan in tp.last_plan(), tp.last_plan()
    want = typed_h.copy()
    cc.unpack(packed_h, 0, want, offset, 1, recipe)
    assert np.array_equal(typed.cpu().numpy(), want)
    tp.type_free(h)


@pytest.mark.gpu
@pytest.mark.parametrize("elem", (1, 4, 12))
def test_unpack_of_two_interleaved_columns(elem):
    """Rows that lie between the rows of another outer index: four per thread, whatever the size."""
    dev = torch.device("cuda:0")
    rows = (5 << 20) // elem // 2 + 1
    recipe = hvector(2, 1, elem, hvector(rows, 1, 2 * elem, contiguous(elem, BYTE)))
    print("two columns", elem, rows, flush=True)
    h = tp.type_from_recipe(recipe)
    size = 2 * rows * elem
    typed_h, packed_h = W.random_bytes(elem, size + 8), W.random_bytes(rows, size)
    typed, packed = torch.from_numpy(typed_h).to(dev), torch.from_numpy(packed_h).to(dev)
    assert tp.unpack(packed, size, 0, typed.data_ptr() + 3, 1, h) == size
    assert "tile" in tp.last_plan() and " ux=1 ur=4 " in tp.last_plan(), tp.last_plan()
    want = typed_h.copy()
    cc.unpack(packed_h, 0, want, 3, 1, recipe)
    assert np.array_equal(typed.cpu().numpy(), want)
    tp.type_free(h)
