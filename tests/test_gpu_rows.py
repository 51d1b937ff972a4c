"""The short-run kernel where it can go wrong, byte for byte against the oracle:
even and ragged runs, one and two units per lane (on either side of 2^18 units
a launch), up to 64, up to 256 and more sequences with idle ones among them,
tokens of one unit and of many, one head, few and many sequences to a wave, and
every layout; both halves of a split-key cache in one launch, from a layer other
than the first."""
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

KINDS = {"dense": (dv.DV_DENSE, oracle.DENSE), "paged": (dv.DV_PAGED, oracle.PAGED),
         "splitkey": (dv.DV_DENSE_KSPLIT, oracle.KSPLIT)}
# layers, heads, head_dim, batch, tokens per active sequence (lowest, highest), share active
SHAPES = {
    "one-unit-rows": (2, 1, 8, 3, (1, 9), 1.0),
    "one-head-many-sequences": (2, 1, 8, 64, (2, 7), 0.7),
    "even-single": (3, 5, 64, 7, (1, 1), 1.0),
    "even-four": (3, 3, 80, 9, (4, 4), 0.6),
    "single-past-64": (2, 3, 64, 100, (1, 1), 0.8),
    "ragged-past-64": (2, 2, 64, 200, (1, 6), 0.8),
    "past-256": (2, 1, 128, 300, (1, 3), 0.9),
    "one-active": (2, 4, 128, 70, (5, 5), 0.0),
    "longest-runs": (2, 2, 256, 5, (7, 8), 1.0),
    "two-units-per-lane": (3, 24, 128, 30, (1, 16), 1.0),
    "two-units-past-64": (2, 16, 128, 130, (1, 16), 1.0),
    # sequences that a wave's 64 rows lie in: 40 to 45, four to six, eight to ten
    "wave-of-forty": (2, 1, 8, 64, (1, 2), 1.0),
    "wave-of-five": (2, 1, 8, 60, (11, 20), 1.0),
    "wave-of-nine": (2, 1, 8, 60, (6, 9), 1.0),
}


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape", SHAPES)
def test_short_runs(oracle_lib, shape, kind):
    L, H, D, B, (lo, hi), share = SHAPES[shape]
    E = 2
    r = np.random.default_rng(900 + sorted(SHAPES).index(shape))
    n = r.integers(lo, hi + 1, size=B)
    idle = r.random(B) >= share
    idle[B // 2] = False
    n[idle] = 0
    t0 = r.integers(0, 30, size=B).astype(np.int32)
    t1 = (t0 + n).astype(np.int32)
    units = int(n.sum()) * H * D * E // 16 * 2 * (L - 1)
    assert (units >= 1 << 18) == shape.startswith("two-units"), units
    cap = 30 + hi
    if kind == "paged":
        bs = 4
        bt, nb = synth.make_paged_tables(3, [cap] * B, bs, -(-cap // bs))
        lay = oracle.Layout(oracle.PAGED, L, H, D, B, elem_bytes=E, block_size=bs, num_blocks=nb,
                            block_table=bt)
        kw = dict(block_size=bs, num_blocks=nb, max_blocks=bt.shape[1],
                  block_tables=[G.to_dev(bt)])
    else:
        lay = oracle.Layout(KINDS[kind][1], L, H, D, B, seq_cap=cap, elem_bytes=E)
        kw = dict(max_seq=cap)
    host = synth.fill_bytes(lay.storage_bytes(), 41)
    src = dv.Cache(KINDS[kind][0], L, H, D, B, [G.to_dev(host)], **kw)
    recv = G.dev_const(lay.storage_bytes(), 0xA5)
    dst = dv.Cache(KINDS[kind][0], L, H, D, B, [recv], **kw)
    size = dv.dv_packed_bytes(src, 1, L, t0, t1)
    wire = G.dev_const(size + 32, 0x5C)
    dv.dv_stream_out_prompt(src, 0, 1, L, t0, t1, wire, size)
    dv.dv_stream_in(dst, 0, 1, L, t0, t1, wire, size)
    torch.cuda.synchronize()
    exp = oracle_lib.pack(lay, host, 1, L, t0, t1)
    assert G.host(wire)[:size].tobytes() == exp.tobytes()
    assert (G.host(wire)[size:size + 32] == 0x5C).all()
    want = np.full(lay.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.unpack(lay, want, 1, L, t0, t1, exp)
    assert G.host(recv)[: want.size].tobytes() == want.tobytes()
