"""Transposing tiles that lie wholly inside their matrix (moved without a check per word) beside those cut at its edge:
one tile, whole tiles only, one element more or less, for every word width; byte for byte against the C oracle."""
import numpy as np
import pytest

import workloads as W
from workloads import BYTE, contiguous, hvector, vector
from oracle import typemap_c as cc
from paper_2012_14363_amd import binding as tp

torch = pytest.importorskip("torch")

EDGE = {1: 128, 2: 128, 4: 64, 8: 64, 16: 32}


@pytest.mark.gpu
@pytest.mark.parametrize("elem", sorted(EDGE))
@pytest.mark.parametrize("rows,cols", ((0, 0), (1, 0), (0, 1), (-1, 0), (0, -1)))
def test_whole_and_cut_tiles(elem, rows, cols):
    dev = torch.device("cuda:0")
    e = EDGE[elem]
    m, n = 2 * e + rows, 2 * e + cols
    recipe = hvector(n, 1, elem, vector(m, 1, n, contiguous(elem, BYTE)))
    print("whole tiles", elem, m, n, flush=True)
    h = tp.type_from_recipe(recipe)
    size = m * n * elem
    typed_h, packed_h = W.random_bytes(elem, size + 8), W.random_bytes(m, size)
    typed, out = torch.from_numpy(typed_h).to(dev), torch.full((size + 8,), 0xEE, dtype=torch.uint8, device=dev)
    assert tp.pack(typed.data_ptr() + 5, 1, h, out, size + 8, 3) == size + 3
    assert f"xpose W={elem} words=1 tile={e}x{e} " in tp.last_plan(), tp.last_plan()
    want = np.full(size + 8, 0xEE, np.uint8)
    cc.pack(typed_h, 5, 1, recipe, want, 3)
    assert np.array_equal(out.cpu().numpy(), want)
    packed = torch.from_numpy(packed_h).to(dev)
    assert tp.unpack(packed, size, 0, typed.data_ptr() + 5, 1, h) == size
    want = typed_h.copy()
    cc.unpack(packed_h, 0, want, 5, 1, recipe)
    assert np.array_equal(typed.cpu().numpy(), want)
    tp.type_free(h)
