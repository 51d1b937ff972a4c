"""Dense streams on every side of the rules that pick their kernel, byte for byte
against the oracle: runs that fill tiles of 512 units well (tiles dealt in
eighths), fairly (tiles in the hardware's order on unpack, rows on pack, or the
tiles both ways where a token is one unit) and badly (rows both ways), runs one unit short of and past a tile, and batches of
up to 64, 256 and more sequences."""
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

# heads, head_dim, elem_bytes, batch, lowest and highest number of tokens
SHAPES = {
    "whole-tiles": (3, 128, 2, 5, 64, 64),
    "one-unit-past": (3, 8, 2, 5, 513, 513),
    "one-unit-short": (3, 8, 2, 5, 1023, 1023),
    "nine-tenths": (2, 80, 2, 9, 140, 150),
    "three-quarters": (5, 128, 2, 6, 40, 50),
    "half": (4, 256, 4, 7, 4, 13),
    "a-third": (2, 256, 4, 11, 0, 5),
    "past-64": (2, 128, 2, 80, 20, 70),
    "past-256": (1, 128, 2, 300, 0, 40),
    "with-one-unit-tokens": (3, 8, 2, 5, 720, 790),
}


@pytest.mark.parametrize("shape", SHAPES)
def test_dense_tiles(oracle_lib, shape):
    H, D, E, B, lo, hi = SHAPES[shape]
    L = 3
    r = np.random.default_rng(sorted(SHAPES).index(shape))
    n = r.integers(lo, hi + 1, size=B)
    n[B // 2] = hi  # past the short-run kernel's 256 units
    assert hi * D * E // 16 > 256
    t0 = r.integers(0, 20, size=B).astype(np.int32)
    t1 = (t0 + n).astype(np.int32)
    S = 20 + hi
    lay = oracle.Layout(oracle.DENSE, L, H, D, B, seq_cap=S, elem_bytes=E)
    host = synth.fill_bytes(lay.storage_bytes(), 61)
    src = dv.Cache(dv.DV_DENSE, L, H, D, B, [G.to_dev(host)], max_seq=S, elem_bytes=E)
    recv = G.dev_const(lay.storage_bytes(), 0xA5)
    dst = dv.Cache(dv.DV_DENSE, L, H, D, B, [recv], max_seq=S, elem_bytes=E)
    for l0, l1 in ((0, L), (1, 2)):
        size = dv.dv_packed_bytes(src, l0, l1, t0, t1)
        wire = G.dev_const(size + 32, 0x5C)
        recv.fill_(0xA5)
        dv.dv_stream_out_prompt(src, 0, l0, l1, t0, t1, wire, size)
        dv.dv_stream_in(dst, 0, l0, l1, t0, t1, wire, size)
        torch.cuda.synchronize()
        exp = oracle_lib.pack(lay, host, l0, l1, t0, t1)
        assert G.host(wire)[:size].tobytes() == exp.tobytes()
        assert (G.host(wire)[size:size + 32] == 0x5C).all()
        want = np.full(lay.storage_bytes(), 0xA5, np.uint8)
        oracle_lib.unpack(lay, want, l0, l1, t0, t1, exp)
        assert G.host(recv)[: want.size].tobytes() == want.tobytes()
