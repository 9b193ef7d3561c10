"""The work a program has this library do, as cases that can be timed and compared.

Every case is one pass through the public entry points of `paper_2012_14363_amd`: datatypes are built and
committed beforehand and kept, as an application keeps them; a pass is the pack and unpack calls alone.
Results are bytes (or whole grids of them), so every comparison is exact.

Families
  object    one strided 2D object of 64 B to 4 MiB, packed or unpacked by the synchronous calls: what a message
            layer does for a single small or medium message.  Latency counts.
  block     a box of a 3D array, a0 bytes x a1 rows x a2 planes, enqueued on the stream: strided columns, tiny runs,
            slabs with ragged rows, up to rows as long as whole pages and to 64 MiB of payload.
  halo      the ghost exchange of a cubic grid with itself (26 regions): one batched pack of the faces, edges and
            corners, one batched unpack into the ghost zones.
  messages  many objects of the four-level nested datatype, packed behind one another: as one call with an object
            count, or as a batch of separately addressed objects.
  matrix    a row-major matrix sent column by column (or received so), elements of 1 to 24 bytes; a thin matrix is
            the change between an array of records and one array per field.
  host      one object delivered to (or taken from) pinned host memory, for a transport that reads host memory.
"""
from __future__ import annotations

import itertools
import math

import torch

from paper_2012_14363_amd import binding as tp

BYTE, FLOAT, DOUBLE = ("named", "BYTE"), ("named", "FLOAT"), ("named", "DOUBLE")
MOST_TYPED = 4 << 30   # bytes of a drawn block's typed buffer
MOST_PACKED = 64 << 20  # bytes of a drawn block's packed stream


def listed():
    return [
        # the smallest call: a 2D vector, 64 runs of 8 B at 512-byte pitch
        {"name": "object_512B_pack", "family": "object", "op": "pack", "run": 8, "rows": 64, "pitch": 512, "offset": 0},
        # a medium message with rows that are no multiple of anything
        {"name": "object_300KB_unpack", "family": "object", "op": "unpack", "run": 100, "rows": 3001, "pitch": 512, "offset": 4},
        # the strided-block sweep at 64 MiB: columns of a few bytes out of 512-byte rows
        {"name": "block_8B_runs_pack", "family": "block", "op": "pack", "a0": 8, "a1": 512, "a2": 16384, "pitch": 512, "e1": 512, "offset": 0},
        {"name": "block_16B_runs_unpack", "family": "block", "op": "unpack", "a0": 16, "a1": 512, "a2": 8192, "pitch": 512, "e1": 512, "offset": 0},
        # tiny runs at an odd address, two to a memory line
        {"name": "tiny_3B_runs_unpack", "family": "block", "op": "unpack", "a0": 3, "a1": 1 << 24, "a2": 1, "pitch": 64, "e1": 1 << 24, "offset": 5},
        # a slab of a float64 field whose sizes are odd in every dimension
        {"name": "slab_ragged_unpack", "family": "block", "op": "unpack", "a0": 301 * 8, "a1": 157, "a2": 151, "pitch": 331 * 8, "e1": 167, "offset": 5 * 8},
        # a large local grid of a stencil code, and a small one
        {"name": "halo_512", "family": "halo", "n": 512, "r": 3, "double": True},
        {"name": "halo_64", "family": "halo", "n": 64, "r": 2, "double": True},
        # 1000 messages of 2 MiB, each with an address of its own
        {"name": "messages_1000_batch", "family": "messages", "objects": 1000, "batch": True},
        # a square float32 matrix by columns; records of six 4-byte fields put together from field arrays
        {"name": "matrix_4B_pack", "family": "matrix", "op": "pack", "rows": 4096, "cols": 4096, "elem": 4},
        {"name": "records_4B_unpack", "family": "matrix", "op": "unpack", "rows": 3000001, "cols": 6, "elem": 4},
        # the largest object of the latency figures, straight into pinned host memory
        {"name": "host_4MiB_pack", "family": "host", "op": "pack", "run": 256, "rows": 16384, "pitch": 512, "offset": 0},
    ]


def _log_int(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _pitch(rng, run):
    """Distance between rows of `run` bytes: a power of two (arrays with padded rows), or any."""
    if rng.random() < 0.5:
        p = 64 << rng.randrange(5)
        while p < run:
            p *= 2
        return p
    return run + _log_int(rng, 1, 2048)


def draw(rng):
    family = rng.choice(("object", "block", "block", "block", "halo", "messages", "matrix", "matrix", "host"))
    op = rng.choice(("pack", "unpack"))
    if family in ("object", "host"):
        size = _log_int(rng, 64, 4 << 20) if family == "object" else _log_int(rng, 1 << 10, 24 << 20)
        run = min(size, _log_int(rng, 1 if family == "object" else 16, 4096))
        pitch = _pitch(rng, run)
        return {"family": family, "op": op, "run": run, "rows": max(1, size // run), "pitch": pitch,
                "offset": rng.choice((0, rng.randrange(64)))}
    if family == "block":
        packed = _log_int(rng, 64 << 10, MOST_PACKED)
        a0 = _log_int(rng, 1, 8192)
        pitch = _pitch(rng, a0)
        rows = max(1, min(packed // a0, MOST_TYPED // pitch))
        a1 = _log_int(rng, 1, min(rows, 4096))
        e1 = a1 + rng.choice((0, _log_int(rng, 1, max(2, a1 // 4))))
        a2 = max(1, min(rows // a1, MOST_TYPED // (pitch * e1)))
        return {"family": family, "op": op, "a0": a0, "a1": a1, "a2": a2, "pitch": pitch, "e1": e1,
                "offset": rng.choice((0, rng.randrange(64)))}
    if family == "halo":
        return {"family": family, "n": _log_int(rng, 32, 512), "r": rng.randint(1, 3), "double": rng.random() < 0.6}
    if family == "messages":
        return {"family": family, "objects": _log_int(rng, 1, 999), "batch": rng.random() < 0.5}
    elem = rng.choice((1, 2, 4, 4, 8, 8, 12, 16, 24))
    total = _log_int(rng, 256 << 10, 128 << 20) // elem   # elements
    if rng.random() < 0.3:
        thin = rng.randint(2, 24)
        rows, cols = (thin, total // thin) if rng.random() < 0.5 else (total // thin, thin)
    else:
        rows = _log_int(rng, max(48, int(total ** 0.5) // 4), max(49, int(total ** 0.5) * 4))
        cols = total // rows
    return {"family": family, "op": op, "rows": rows, "cols": cols, "elem": elem}


# ------------------------------------------------------------------ datatypes
def _rows_type(run, rows, pitch):
    return ("hvector", rows, 1, pitch, ("contiguous", run, BYTE))


def _nested_type():
    """vector(4) of hvector(16) of an [8, 16, 64] float32 box at [3, 5, 0] of a [64, 64, 64] array."""
    box = ("subarray", (64, 64, 64), (8, 16, 64), (3, 5, 0), "C", FLOAT)
    return ("vector", 4, 1, 2, ("hvector", 16, 1, 8192, box))


def _halo_regions(n, r):
    """[(send box, ghost box)] of the 26 directions, a box being its (start, stop) in each dimension; what is sent
    towards d arrives in the ghost zone on the other side."""
    inner = {0: (r, n - r), -1: (r, 2 * r), 1: (n - 2 * r, n - r)}
    ghost = {0: (r, n - r), -1: (0, r), 1: (n - r, n)}
    return [([inner[c] for c in d], [ghost[-c] for c in d]) for d in itertools.product((-1, 0, 1), repeat=3) if any(d)]


def _box_type(n, box, elem):
    return ("subarray", (n, n, n), tuple(b - a for a, b in box), tuple(a for a, _ in box), "C", elem)


def _packed_bytes(case):
    f = case["family"]
    if f in ("object", "host"):
        return case["run"] * case["rows"]
    if f == "block":
        return case["a0"] * case["a1"] * case["a2"]
    if f == "halo":
        cells = sum(math.prod(b - a for a, b in send) for send, _ in _halo_regions(case["n"], case["r"]))
        return cells * (8 if case["double"] else 4)
    if f == "messages":
        return case["objects"] * (2 << 20)
    return case["rows"] * case["cols"] * case["elem"]


# ------------------------------------------------------------------ inputs
def _bytes(n, gen, pinned=False):
    """n random bytes, as a view of a buffer of whole 64-bit words (what `run` returns)."""
    words = torch.empty((n + 7) // 8, dtype=torch.int64, device="cuda").random_(generator=gen)
    if pinned:
        words = torch.empty(words.shape, dtype=torch.int64, pin_memory=True).copy_(words)
    return words


def _zeros(n, pinned=False):
    shape = ((n + 7) // 8,)
    if pinned:
        return torch.zeros(shape, dtype=torch.int64, pin_memory=True)
    return torch.zeros(shape, dtype=torch.int64, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    family, size = case["family"], _packed_bytes(case)
    state = {"case": case, "size": size}
    if family == "halo":
        n, elem, kind = case["n"], DOUBLE if case["double"] else FLOAT, torch.float64 if case["double"] else torch.float32
        grid = torch.empty((n, n, n), dtype=kind, device="cuda").uniform_(-1, 1, generator=gen)
        regions = _halo_regions(n, case["r"])
        send = [tp.type_from_recipe(_box_type(n, s, elem)) for s, _ in regions]
        ghost = [tp.type_from_recipe(_box_type(n, g, elem)) for _, g in regions]
        state.update(grid=grid, packed=torch.zeros(size // grid.element_size(), dtype=kind, device="cuda"),
                     send=tp.Batch([grid] * len(send), [1] * len(send), send),
                     ghost=tp.Batch([grid] * len(ghost), [1] * len(ghost), ghost))
        return state
    if family == "messages":
        t = tp.type_from_recipe(_nested_type())
        _, extent = tp.type_get_extent(t)
        k = case["objects"]
        state.update(type=t, typed=_bytes(k * extent, gen), packed=_zeros(size))
        if case["batch"]:
            base = state["typed"].data_ptr()
            state["batch"] = tp.Batch([base + i * extent for i in range(k)], [1] * k, [t] * k)
        return state
    if family == "matrix":
        rows, cols, elem = case["rows"], case["cols"], case["elem"]
        recipe = ("hvector", cols, 1, elem, ("hvector", rows, 1, cols * elem, ("contiguous", elem, BYTE)))
        span, offset = rows * cols * elem, 0
    elif family == "block":
        recipe = ("hvector", case["a2"], 1, case["pitch"] * case["e1"], _rows_type(case["a0"], case["a1"], case["pitch"]))
        offset = case["offset"]
        span = offset + case["a2"] * case["e1"] * case["pitch"]
    else:
        recipe = _rows_type(case["run"], case["rows"], case["pitch"])
        offset = case["offset"]
        span = offset + case["rows"] * case["pitch"]
    pinned = family == "host"
    unpack = case["op"] == "unpack"
    typed = _bytes(span, gen)
    packed = _bytes(size, gen, pinned) if unpack else _zeros(size, pinned)
    state.update(type=tp.type_from_recipe(recipe), typed=typed, packed=packed, origin=typed.view(torch.uint8)[offset:])
    return state


# ------------------------------------------------------------------ one pass
def run(state):
    case, size = state["case"], state["size"]
    family = case["family"]
    packed = state["packed"]
    if family == "halo":
        tp.pack_batch_async(state["send"], packed, size, 0)
        tp.unpack_batch_async(packed, size, 0, state["ghost"])
        return packed, state["grid"]
    if family == "messages":
        if case["batch"]:
            tp.pack_batch_async(state["batch"], packed, size, 0)
        else:
            tp.pack_async(state["typed"], case["objects"], state["type"], packed, size, 0)
        return packed
    t, origin = state["type"], state["origin"]
    if family == "host":
        if case["op"] == "pack":
            tp.pack_host(origin, 1, t, packed, size, 0)
            return packed
        tp.unpack_host(packed, size, 0, origin, 1, t)
        return state["typed"]
    if family == "object":
        pack, unpack = tp.pack, tp.unpack
    else:
        pack, unpack = tp.pack_async, tp.unpack_async
    if case["op"] == "pack":
        pack(origin, 1, t, packed, size, 0)
        return packed
    unpack(packed, size, 0, origin, 1, t)
    return state["typed"]


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    size = _packed_bytes(case)
    if case["family"] == "halo":
        return {"bytes": 4 * size, "flops": 0}   # packed and unpacked
    if case["family"] == "messages":
        # the nested type's boxes overlap: of the 128 runs of 4 KiB in each of its four parts 30 are distinct
        return {"bytes": size + case["objects"] * 4 * 30 * 4096, "flops": 0}
    return {"bytes": 2 * size, "flops": 0}


def tolerance(case):
    return "exact"   # bytes are moved, nothing is computed
