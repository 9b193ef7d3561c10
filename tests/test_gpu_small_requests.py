"""Synchronous calls of small requests: what the call has written is there when it returns, for the host and for
another stream, and its stream is idle, around 256 workgroups (one for each CU)."""
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
@pytest.mark.parametrize("workgroups", (1, 256, 257))
@pytest.mark.parametrize("unpack", (False, True))
def test_the_stream_is_synchronized_when_the_call_returns(workgroups, unpack):
    """Work enqueued before the call is complete as well: an event recorded in front of it has happened, the stream
    has nothing left, and what an earlier enqueue-only call stored is there for the host and for another stream."""
    dev = torch.device("cuda:0")
    rows, many = ROWS_PER_WORKGROUP[unpack] * workgroups - 3, 1 << 16
    print("stream after a synchronous call, workgroups", workgroups, "unpack", unpack, flush=True)
    small, large = (tp.type_from_recipe(hvector(n, 1, 128, contiguous(100, BYTE))) for n in (rows, many))
    typed_h = W.random_bytes(60, many * 128)
    typed = torch.from_numpy(typed_h).to(dev)
    packed, target = torch.zeros(100 * rows, dtype=torch.uint8, device=dev), torch.zeros(128 * rows, dtype=torch.uint8, device=dev)
    want = np.zeros(100 * many, np.uint8)
    cc.pack(typed_h, 0, 1, hvector(many, 1, 128, contiguous(100, BYTE)), want, 0)
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for k in range(20):
        earlier = torch.zeros(100 * many, dtype=torch.uint8, device=dev)
        on_host = torch.zeros(100 * many, dtype=torch.uint8).pin_memory()
        torch.cuda.synchronize()
        before = torch.cuda.Event()
        with torch.cuda.stream(stream):
            assert tp.pack_async(typed, 1, large, on_host if k % 2 else earlier, 100 * many, 0) == 100 * many
            before.record()
            if unpack:
                tp.unpack(packed, 100 * rows, 0, target, 1, small)
            else:
                tp.pack(typed, 1, small, packed, 100 * rows, 0)
        assert before.query() and stream.query()
        with torch.cuda.stream(other):
            got = on_host.numpy() if k % 2 else earlier.to("cpu").numpy()
        assert np.array_equal(got, want)
    tp.type_free(small)
    tp.type_free(large)


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
