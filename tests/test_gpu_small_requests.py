"""Synchronous calls of small requests, whose kernel tells the host itself that it is done: what the call has
written is there when it returns, for the host and for another stream, around the number of workgroups up to
which that holds (the last count here takes the other way)."""
import numpy as np
import pytest

import workloads as W
from workloads import BYTE, contiguous, hvector
from oracle import typemap_c as cc
from paper_2012_14363_amd import binding as tp

torch = pytest.importorskip("torch")

ROWS_PER_WORKGROUP = {False: 128, True: 16}   # pack: 16-byte words, four rows a thread; unpack: 8-byte words, one row


@pytest.mark.gpu
@pytest.mark.parametrize("workgroups", (1, 2, 255, 256, 257))
@pytest.mark.parametrize("unpack", (False, True))
def test_data_is_there_when_the_call_returns(workgroups, unpack):
    dev = torch.device("cuda:0")
    rows = ROWS_PER_WORKGROUP[unpack] * workgroups - 3
    recipe = hvector(rows, 1, 128, contiguous(100, BYTE))
    print("small request, workgroups", workgroups, "unpack", unpack, flush=True)
    h = tp.type_from_recipe(recipe)
    size, span = tp.type_size(h), rows * 128 + 64
    other = torch.cuda.Stream()
    for k in range(4):
        typed_h, packed_h = W.random_bytes(70 + k, span), W.random_bytes(80 + k, size)
        if not unpack:
            typed = torch.from_numpy(typed_h).to(dev)
            out = torch.full((size,), 0xEE, dtype=torch.uint8).pin_memory()
            torch.cuda.synchronize()
            assert tp.pack(typed.data_ptr() + 3, 1, h, out, size, 0) == size
            got = out.numpy().copy()
            want = np.full(size, 0xEE, np.uint8)
            cc.pack(typed_h, 3, 1, recipe, want, 0)
        else:
            packed = torch.from_numpy(packed_h).to(dev)
            typed = torch.from_numpy(typed_h).to(dev)
            torch.cuda.synchronize()
            assert tp.unpack(packed, size, 0, typed.data_ptr() + 3, 1, h) == size
            with torch.cuda.stream(other):
                got = typed.to("cpu").numpy()
            want = typed_h.copy()
            cc.unpack(packed_h, 0, want, 3, 1, recipe)
        assert f"blocks={workgroups} " in tp.last_plan() and tp.last_plan().count("\n") == 1, tp.last_plan()
        assert np.array_equal(got, want)
    tp.type_free(h)


@pytest.mark.gpu
@pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs a stream of another GPU")
def test_stream_of_another_gpu_than_the_current_one():
    other = torch.device("cuda:1")
    rows = 4 * ROWS_PER_WORKGROUP[False]
    recipe = hvector(rows, 1, 128, contiguous(100, BYTE))
    h = tp.type_from_recipe(recipe)
    size = tp.type_size(h)
    typed_h = W.random_bytes(90, rows * 128)
    with torch.cuda.device(other):
        typed, stream = torch.from_numpy(typed_h).to(other), torch.cuda.Stream()
        torch.cuda.synchronize()
    out = torch.full((size,), 0xEE, dtype=torch.uint8).pin_memory()
    with torch.cuda.device(0):
        assert tp.pack(typed, 1, h, out, size, 0, stream=stream) == size
    want = np.full(size, 0xEE, np.uint8)
    cc.pack(typed_h, 0, 1, recipe, want, 0)
    assert np.array_equal(out.numpy(), want)
    tp.type_free(h)
