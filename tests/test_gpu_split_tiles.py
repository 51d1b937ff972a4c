"""Split-key streams of long runs at the edges of the kernel's tiles, byte for
byte against the oracle: every tile length (whole 128-byte lines of a key slab
in two units per lane, six or eight), runs of whole tiles, of one token more and
of one less, starts inside a line, runs that fill tiles badly (which go row by
row), and batches past 64 and 256 sequences."""
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


def check(oracle_lib, L, H, D, E, t0, n, whole_lines=False, shift=0):
    """``whole_lines``: a capacity of whole 128-byte lines (8 tokens of a group),
    the caches starting ``shift`` tokens past a line."""
    B = len(n)
    t0 = np.asarray(t0, np.int32)
    t1 = (t0 + n).astype(np.int32)
    S = int(t1.max()) + 3
    if whole_lines:
        S += -S % 8
    lay = oracle.Layout(oracle.KSPLIT, L, H, D, B, seq_cap=S, elem_bytes=E)
    host = synth.fill_bytes(lay.storage_bytes(), 51)
    moved = G.dev_const(lay.storage_bytes() + 16 * shift, 0)[16 * shift:]
    moved[:host.size] = G.to_dev(host)[:host.size]
    src = dv.Cache(dv.DV_DENSE_KSPLIT, L, H, D, B, [moved], max_seq=S, elem_bytes=E)
    recv = G.dev_const(lay.storage_bytes() + 16 * shift, 0xA5)[16 * shift:]
    dst = dv.Cache(dv.DV_DENSE_KSPLIT, L, H, D, B, [recv], max_seq=S, elem_bytes=E)
    size = dv.dv_packed_bytes(src, 0, L, t0, t1)
    wire = G.dev_const(size + 32, 0x5C)
    dv.dv_stream_out_prompt(src, 0, 0, L, t0, t1, wire, size)
    dv.dv_stream_in(dst, 0, 0, L, t0, t1, wire, size)
    torch.cuda.synchronize()
    exp = oracle_lib.pack(lay, host, 0, L, t0, t1)
    assert G.host(wire)[:size].tobytes() == exp.tobytes()
    assert (G.host(wire)[size:size + 32] == 0x5C).all()
    want = np.full(lay.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.unpack(lay, want, 0, L, t0, t1, exp)
    assert G.host(recv)[: want.size].tobytes() == want.tobytes()


@pytest.mark.parametrize("groups", [1, 2, 3, 5, 8, 10, 12, 13, 16, 17, 20, 22, 24, 25, 31, 32])
def test_split_tiles(oracle_lib, groups):
    two, six = 512 // groups & ~7, 1536 // groups & ~7
    tile = two if two * groups * 5 >= 4 * 512 else six  # tokens
    n = np.array([3 * tile, 4 * tile + 1, 4 * tile - 1, 0, 4 * tile])
    check(oracle_lib, 2, 3, 8 * groups, 2, [0, 1, 8, 2, 13], n)
    if groups >= 20:  # past 16 MB, where two units become eight on the way in
        eight = 2048 // groups & ~7
        n = np.array([3 * eight, eight // 2, eight + 1, 0, 2 * eight - 1])
        check(oracle_lib, 16, 3, 8 * groups, 2, [0, 1, 8, 2, 12], n)


@pytest.mark.parametrize("groups", [20, 32])
def test_split_tiles_of_eight_units_past_64_sequences(oracle_lib, groups):
    """20 and 22 MB into a capacity that is not whole lines: runs around one tile
    of eight units per lane and ragged ones, in one launch of 71 sequences."""
    r = np.random.default_rng(groups)
    eight = 2048 // groups & ~7
    n = r.integers(eight // 3, eight + 1, size=71)
    n[:6] = eight - 1, eight, eight + 1, 0, 2 * eight, 1
    t0 = r.integers(0, 9, size=71)
    t0[4] = 9  # then the capacity is 2 * eight + 12
    check(oracle_lib, 1, 7, 8 * groups, 2, t0, n)


@pytest.mark.parametrize("groups", [1, 5, 16, 24, 32])
@pytest.mark.parametrize("shift", [0, 3, 7])
def test_split_tiles_that_end_on_lines(oracle_lib, groups, shift):
    """Capacities of whole lines: starts at every place in a line, runs that end
    on a tile's last token, one past it and inside the shortened first tile."""
    two, six = 512 // groups & ~7, 1536 // groups & ~7
    tile = two if two * groups * 5 >= 4 * 512 else six  # tokens
    t0 = np.arange(12)
    lead = (t0 + shift) % 8
    ends = np.array([4, 4, 4, 3, 3, 3, 5, 5, 5, 4, 4, 4]) * tile + np.tile([-1, 0, 1], 4)
    n = ends - lead
    n[4], n[8] = 0, 2
    check(oracle_lib, 2, 2, 8 * groups, 2, t0, n, True, shift)


@pytest.mark.parametrize("whole_lines", [False, True])
def test_split_runs_of_few_tokens_in_a_large_stream(oracle_lib, whole_lines):
    """98 MB of 5-20 tokens, 32 groups: rows out, badly filled tiles in."""
    r = np.random.default_rng(4)
    n = r.integers(5, 21, size=40)
    check(oracle_lib, 4, 42, 256, 2, r.integers(0, 30, size=40), n, whole_lines, 5)


@pytest.mark.parametrize("B, lo, hi", [(7, 18, 40), (90, 20, 64), (300, 33, 64)])
def test_split_runs_of_few_tokens(oracle_lib, B, lo, hi):
    """32 groups of 16 bytes: tiles of 16 tokens, filled well and badly."""
    r = np.random.default_rng(B)
    n = r.integers(lo, hi + 1, size=B)
    check(oracle_lib, 2, 2, 256, 2, r.integers(0, 9, size=B), n)
    n = np.where(r.random(B) < 0.5, 1, 17)  # half-empty tiles: row by row
    check(oracle_lib, 2, 2, 256, 2, r.integers(0, 9, size=B), n)
