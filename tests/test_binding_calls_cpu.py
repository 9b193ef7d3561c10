"""What the pack and unpack calls take as arguments, as far as it can be told without a GPU: calls that move nothing
succeed, and calls the library refuses before it asks the device about memory."""
import ctypes

import pytest

from paper_2012_14363_amd import binding as tp

TP_ERR_COUNT, TP_ERR_TRUNCATE, TP_ERR_BUFFER = 2, 4, 5


def outcome(call, *args):
    """0, or the code the library refused the call with."""
    try:
        call(*args)
    except tp.TpError as e:
        return e.code
    return 0


def both(batch, size=8):
    """The outcomes of the four batched calls, which are to be one."""
    codes = {outcome(call, batch, 0, size, 0, 0) for call in (tp.pack_batch, tp.pack_batch_async)}
    codes |= {outcome(call, 0, size, 0, batch, 0) for call in (tp.unpack_batch, tp.unpack_batch_async)}
    assert len(codes) == 1
    return codes.pop()


def test_a_batch_is_read_as_it_stands_at_the_call():
    t = tp.PREDEFINED["BYTE"]
    batch = tp.Batch([0], [0], [t])
    assert both(batch) == 0
    batch.counts[0] = 4                         # in place
    assert both(batch) == TP_ERR_BUFFER
    batch.counts = (ctypes.c_int * 1)(16)       # another array
    assert both(batch) == TP_ERR_TRUNCATE
    batch.counts = (ctypes.c_int * 1)(-1)
    assert both(batch) == TP_ERR_COUNT
    batch.counts = (ctypes.c_int * 1)(0)
    assert both(batch) == 0
    batch.types = (ctypes.c_int32 * 1)(999)
    assert both(batch) != 0
    batch.n = 0
    assert both(batch) == 0
    batch.types = None                          # nothing to read
    assert both(batch) == 0
    batch.n = 1
    assert both(batch) != 0
    batch.types = (ctypes.c_int64 * 1)(t)       # not the type the library reads
    with pytest.raises(Exception) as e:
        tp.pack_batch(batch, 0, 8, 0, 0)
    assert not isinstance(e.value, tp.TpError)
    del batch.types
    with pytest.raises(AttributeError):
        tp.pack_batch(batch, 0, 8, 0, 0)


def test_anything_with_the_attributes_of_a_batch_is_one():
    class Mine:
        n, ptrs, counts, types = 1, (ctypes.c_void_p * 1)(0), (ctypes.c_int * 1)(4), (ctypes.c_int32 * 1)(tp.PREDEFINED["BYTE"])

    assert both(Mine()) == TP_ERR_BUFFER
    Mine.counts = (ctypes.c_int * 1)(0)
    assert both(Mine()) == 0


def test_ctypes_numbers_are_numbers():
    t = tp.PREDEFINED["BYTE"]

    class Names:
        _as_parameter_ = t

    for number in (t, ctypes.c_int32(t), Names(), ctypes.c_int(t)):
        assert outcome(tp.pack, 0, ctypes.c_int(4), number, 0, ctypes.c_int64(8), 0, 0) == TP_ERR_BUFFER
        assert outcome(tp.unpack_async, 0, ctypes.c_int64(2), 0, 0, 4, number, 0) == TP_ERR_TRUNCATE
        assert tp.pack_async(0, ctypes.c_int(0), number, 0, 8, 3, 0) == 3
    for wrong in (1.0, "1", None, ctypes.c_int16(1), ctypes.c_int64(1)):
        with pytest.raises(Exception) as e:
            tp.pack(0, wrong, t, 0, 8, 0, 0)
        assert not isinstance(e.value, tp.TpError)
