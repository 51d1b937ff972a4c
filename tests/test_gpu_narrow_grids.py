"""Streams whose tiles are more than a launch's grid may hold, byte for byte
against the oracle.  The limit is 2^24 workgroups, slabs of 128 GB; here the
library is the same sources built with a limit of 128 (tests/c/libdv_narrow.so,
made by __graft_entry__.build()), so that paged workgroups take several tiles one
after another and dense and split-key calls of many sequences fall back to 64 a
launch, and what is too wide even then is refused."""
import ctypes
import os

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2403_01876_amd import dv  # noqa: E402
from tests import gpu_util as G  # noqa: E402

PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "c", "libdv_narrow.so")
KINDS = {"dense": (dv.DV_DENSE, oracle.DENSE), "splitkey": (dv.DV_DENSE_KSPLIT, oracle.KSPLIT)}


@pytest.fixture(scope="module")
def lib():
    lib = ctypes.CDLL(PATH)
    for name in ("dv_stream_out_prompt", "dv_stream_in"):
        getattr(lib, name).argtypes = getattr(dv.lib, name).argtypes
    return lib


def run(lib, name, cache, L, t0, t1, wire, size):
    """One call over all layers on the current stream; its status."""
    args = [cache.ref, 0, 0, L, t0.ctypes.data, t1.ctypes.data, wire.data_ptr(), size]
    st = torch.cuda.current_stream().cuda_stream
    rc = lib.dv_stream_out_prompt(*args, None, st) if name == "out" else lib.dv_stream_in(*args, st)
    torch.cuda.synchronize()
    return rc


# heads, head_dim, elem_bytes, block_size, batch, tokens: lowest and highest
PAGED = {
    "two-tiles": (2, 128, 2, 16, 3, 900, 1400),
    "sixteen-tiles-whole-blocks": (4, 128, 2, 16, 5, 1500, 2000),
    "eight-tiles-straddling": (3, 80, 2, 8, 4, 1900, 2600),
    "small-blocks": (1, 8, 2, 5, 3, 40000, 60000),
    "a-hundred-sequences": (3, 72, 2, 8, 100, 20, 120),
}


@pytest.mark.parametrize("order", ["table", "pool"])
@pytest.mark.parametrize("shape", PAGED)
def test_paged_workgroups_of_several_tiles(oracle_lib, lib, shape, order):
    H, D, E, bs, B, lo, hi = PAGED[shape]
    L = 2
    r = np.random.default_rng(sorted(PAGED).index(shape))
    t0 = r.integers(0, bs, size=B).astype(np.int32)
    t1 = (t0 + r.integers(lo, hi + 1, size=B)).astype(np.int32)
    blocks = -(-t1 // bs) - t0 // bs
    s_blk = H * bs * D * E // 16
    maxb, nb = int(blocks.max()), int(blocks.sum())
    tiles = -(-nb * s_blk // 512) if order == "pool" else int((-(-blocks * s_blk // 512)).sum())
    assert tiles >= 128 > B
    bt = np.full((B, maxb), -1, np.int32)
    free = iter(r.permutation(nb))
    for b in range(B):
        bt[b, :blocks[b]] = [next(free) for _ in range(blocks[b])]
    lay = oracle.Layout(oracle.PAGED, L, H, D, B, elem_bytes=E, block_size=bs, num_blocks=nb,
                        block_table=bt)
    host = synth.fill_bytes(lay.storage_bytes(), 91)
    kw = dict(elem_bytes=E, block_size=bs, num_blocks=nb, max_blocks=maxb,
              block_tables=[G.to_dev(bt)])
    exp = oracle_lib.pack(lay, host, 0, L, t0, t1)
    if order == "table":
        c = dv.Cache(dv.DV_PAGED, L, H, D, B, [G.to_dev(host)], **kw)
        wire = G.dev_const(exp.nbytes + 32, 0x5C)
        assert run(lib, "out", c, L, t0, t1, wire, exp.nbytes) == dv.DV_OK
        assert G.host(wire)[:exp.nbytes].tobytes() == exp.tobytes()
        assert (G.host(wire)[exp.nbytes:] == 0x5C).all()
    recv = G.dev_const(lay.storage_bytes(), 0xA5)
    owner = G.dev_const(nb * 4, 0x7E)
    c = dv.Cache(dv.DV_PAGED, L, H, D, B, [recv],
                 block_owners=[owner] if order == "pool" else None, **kw)
    assert run(lib, "in", c, L, t0, t1, G.to_dev(exp), exp.nbytes) == dv.DV_OK
    want = np.full(lay.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.unpack(lay, want, 0, L, t0, t1, exp)
    assert G.host(recv)[: want.size].tobytes() == want.tobytes()
    if order == "pool":
        assert (G.host(owner).view(np.int32) == G.owner_map_expected(bt, nb, bs, t0, t1)).all()


@pytest.mark.parametrize("kind", KINDS)
def test_many_sequences_fall_back_to_64_a_launch(oracle_lib, lib, kind):
    """100 sequences of one or two tiles are too many for one launch; one
    sequence of 200 tiles is too many for any.  (Split-key starts that lie inside
    a line leave the first tile that much shorter.)"""
    L, H, D, E, B = 2, 1, 128, 2, 100
    r = np.random.default_rng(5)
    t0 = r.integers(0, 8, size=B).astype(np.int32)
    n = r.choice([32, 64] if kind == "dense" else [24, 56], size=B)
    assert int((-(-n // 32)).sum()) >= 128 > int((-(-n // 32))[:64].sum())
    t1 = (t0 + n).astype(np.int32)
    lay = oracle.Layout(KINDS[kind][1], L, H, D, B, seq_cap=80, elem_bytes=E)
    host = synth.fill_bytes(lay.storage_bytes(), 92)
    exp = oracle_lib.pack(lay, host, 0, L, t0, t1)
    c = dv.Cache(KINDS[kind][0], L, H, D, B, [G.to_dev(host)], max_seq=80)
    wire = G.dev_const(exp.nbytes, 0)
    assert run(lib, "out", c, L, t0, t1, wire, exp.nbytes) == dv.DV_OK
    assert G.host(wire).tobytes() == exp.tobytes()
    recv = G.dev_const(lay.storage_bytes(), 0xA5)
    c = dv.Cache(KINDS[kind][0], L, H, D, B, [recv], max_seq=80)
    assert run(lib, "in", c, L, t0, t1, wire, exp.nbytes) == dv.DV_OK
    want = np.full(lay.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.unpack(lay, want, 0, L, t0, t1, exp)
    assert G.host(recv)[: want.size].tobytes() == want.tobytes()

    S = 200 * 32
    big = G.dev_const(2 * H * S * D * E, 0x11)
    c = dv.Cache(KINDS[kind][0], 1, H, D, 1, [big], max_seq=S)
    wire = G.dev_const(2 * H * S * D * E, 0x22)
    z, n = np.zeros(1, np.int32), np.full(1, S, np.int32)
    assert run(lib, "out", c, 1, z, n, wire, wire.numel()) == dv.DV_ERR_HIP
    assert run(lib, "in", c, 1, z, n, wire, wire.numel()) == dv.DV_ERR_HIP
    assert bool((wire == 0x22).all()) and bool((big == 0x11).all())
