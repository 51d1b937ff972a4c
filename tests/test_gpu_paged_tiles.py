"""Paged streams at the edges of the kernel's tiles, byte for byte against the
oracle: blocks smaller than a tile (several to a tile), blocks that tiles
straddle, blocks of whole tiles, ranges that cover just more and just less than
three quarters of their blocks (where tiles over whole blocks give way to the
rows of the range alone), unmapped table entries inside the ranges, and batches
past 64 and 256 sequences.  One case has tiles whose unit numbers pass 2^31."""
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

# heads, head_dim, elem_bytes, block_size, batch, (t0, n) drawn from these bounds
SHAPES = {
    "four-blocks-a-tile": (1, 128, 1, 16, 5, (0, 0), (40, 200)),
    "one-unit-blocks": (1, 8, 2, 1, 3, (0, 9), (257, 700)),
    "straddling-480": (3, 80, 2, 16, 4, (0, 40), (30, 90)),
    "straddling-960": (5, 96, 4, 8, 4, (0, 20), (12, 70)),
    "whole-tiles": (2, 256, 4, 64, 3, (0, 70), (70, 200)),
    "over-three-quarters": (2, 128, 2, 64, 3, (0, 0), (49, 49)),
    "under-three-quarters": (2, 128, 2, 64, 3, (0, 0), (47, 47)),
    "under-three-quarters-long-runs": (2, 128, 2, 128, 3, (70, 90), (70, 80)),
    "under-three-quarters-short-heads": (7, 64, 2, 64, 6, (3, 50), (33, 40)),
    "short-ranges-of-large-blocks": (1, 128, 4, 64, 41, (0, 9), (5, 23)),
    "seventy-sequences": (3, 64, 1, 8, 70, (0, 30), (0, 90)),
    "three-hundred-sequences": (2, 64, 1, 16, 300, (0, 10), (0, 70)),
}


def stream():
    return torch.cuda.current_stream()


@pytest.mark.parametrize("unmapped", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_paged_tiles(oracle_lib, shape, unmapped):
    H, D, E, bs, B, t0s, ns = SHAPES[shape]
    L = 2
    r = np.random.default_rng(sorted(SHAPES).index(shape))
    t0 = r.integers(t0s[0], t0s[1] + 1, size=B).astype(np.int32)
    n = r.integers(ns[0], ns[1] + 1, size=B)
    n[B - 1] = max(n[B - 1], 256 * 16 // (D * E) + 1)  # past the short-run kernel
    t1 = (t0 + n).astype(np.int32)
    maxb = -(-int(t1.max()) // bs) + 1
    bt, nb = synth.make_paged_tables(7, [int(t) for t in t1], bs, maxb)
    bt = np.where(bt < 0, -5, bt).astype(np.int32)
    if unmapped:
        bt[r.random(bt.shape) < 0.3] = -1
        bt[r.random(bt.shape) < 0.1] = nb + 3
    # The oracle works on a pool with one more block, which every unmapped
    # entry names.
    bad = (bt < 0) | (bt >= nb)
    ext = oracle.Layout(oracle.PAGED, L, H, D, B, elem_bytes=E, block_size=bs, num_blocks=nb + 1,
                        block_table=np.where(bad, nb, bt).astype(np.int32))
    blk = H * bs * D * E

    def extended(pool, fill):
        return np.concatenate([pool.reshape(2 * L, nb * blk),
                               np.full((2 * L, blk), fill, np.uint8)], axis=1).reshape(-1)

    host = synth.fill_bytes(2 * L * nb * blk, 31)
    kw = dict(elem_bytes=E, block_size=bs, num_blocks=nb, max_blocks=maxb,
              block_tables=[G.to_dev(bt)])
    src = dv.Cache(dv.DV_PAGED, L, H, D, B, [G.to_dev(host)], **kw)
    size = dv.dv_packed_bytes(src, 0, L, t0, t1)
    wire = G.dev_const(size + 32, 0x5C)
    dv.dv_stream_out_prompt(src, 0, 0, L, t0, t1, wire, size, stream())
    torch.cuda.synchronize()
    exp = oracle_lib.pack(ext, extended(host, 0x5C), 0, L, t0, t1)
    assert G.host(wire)[:size].tobytes() == exp.tobytes()
    assert (G.host(wire)[size:size + 32] == 0x5C).all()

    wire_h = synth.fill_bytes(size, 32)
    want = extended(np.full(2 * L * nb * blk, 0xA5, np.uint8), 0xA5)
    oracle_lib.unpack(ext, want, 0, L, t0, t1, wire_h)
    want = want.reshape(2 * L, (nb + 1) * blk)[:, : nb * blk].tobytes()
    for owners in (None, [G.dev_const(nb * 4, 0x7E)]):
        recv = G.dev_const(2 * L * nb * blk, 0xA5)
        dst = dv.Cache(dv.DV_PAGED, L, H, D, B, [recv], block_owners=owners, **kw)
        dv.dv_stream_in(dst, 0, 0, L, t0, t1, G.to_dev(wire_h), size, stream())
        torch.cuda.synchronize()
        assert G.host(recv)[: 2 * L * nb * blk].tobytes() == want, "pool order" if owners else "table"


@pytest.mark.parametrize("B, blocks", [(1, 1), (3, 64), (5, 65), (1, 192 * 64), (1, 192 * 64 + 1),
                                       (64, 193), (65, 30), (256, 128), (256, 129), (72, 256),
                                       (73, 256), (240, 128), (241, 128)])
def test_owner_map_one_launch_or_several(B, blocks):
    """The owner map of pools whose tables have chunks of 64 entries on either
    side of the counts up to which one launch builds it (192 for at most 64
    sequences, 288 up to 128, 480 from 193 on), with unmapped entries, ranges that start in
    later blocks and blocks that no entry names."""
    bs, H, D = 4, 1, 8
    r = np.random.default_rng(B * 1000 + blocks)
    nb = B * blocks + min(5, B * blocks // 2)  # most of the pool written: pool order
    bt = r.permutation(nb)[: B * blocks].reshape(B, blocks).astype(np.int32)
    bt[r.random(bt.shape) < 0.05] = -1
    t0 = r.integers(0, min(blocks, 3) * bs - bs + 1, size=B).astype(np.int32)
    t1 = np.full(B, blocks * bs, np.int32)
    t0[0] = 0
    E = 2 if blocks * bs > 256 else 512  # runs past the short-run kernel's 256 units
    pool = G.dev_const(2 * nb * H * bs * D * E, 0xA5)
    owner = torch.full((nb + 1,), 77, dtype=torch.int32, device=G.DEV)
    c = dv.Cache(dv.DV_PAGED, 1, H, D, B, [pool], elem_bytes=E, block_size=bs, num_blocks=nb,
                 max_blocks=blocks, block_tables=[G.to_dev(bt)], block_owners=[owner])
    size = dv.dv_packed_bytes(c, 0, 1, t0, t1)
    dv.dv_stream_in(c, 0, 0, 1, t0, t1, G.dev_const(size, 1), size, stream())
    torch.cuda.synchronize()
    got = G.host(owner)
    assert (got[:nb] == G.owner_map_expected(bt, nb, bs, t0, t1)).all() and got[nb] == 77


@pytest.mark.parametrize("H, D, E, bs", [(1, 8, 2, 64), (1, 8, 2, 127), (1, 8, 2, 128), (1, 8, 2, 129),
                                         (3, 64, 2, 16), (5, 80, 2, 8), (2, 72, 4, 30)])
@pytest.mark.parametrize("B", [64, 65, 200])
def test_pool_order_blocks_around_a_wave(oracle_lib, H, D, E, bs, B):
    """Pool order, blocks of a wave's 128 units, one less and one more, and larger
    ones that tiles straddle: a pool half again as large as what is written,
    ranges that start and end inside blocks, one sequence without tokens."""
    L, du = 2, D * E // 16
    r = np.random.default_rng(H * bs + B)
    t0 = r.integers(0, bs // 8 + 1, size=B).astype(np.int32)
    n = bs * r.integers(3, 8, size=B) - r.integers(0, bs // 8 + 1, size=B)
    n[1], n[B - 1] = 0, max(5 * bs, 256 // du + 1)
    t1 = (t0 + n).astype(np.int32)
    blocks = np.where(n > 0, -(-t1 // bs) - t0 // bs, 0)
    maxb, nb = int(-(-t1.max() // bs)), int(blocks.sum() * 3 // 2)
    assert 4 * n.sum() >= 3 * blocks.sum() * bs and 9 * blocks.sum() >= 5 * nb
    bt = np.full((B, maxb), -1, np.int32)
    free = iter(r.permutation(nb))
    for b in range(B):
        for j in range(t0[b] // bs, t0[b] // bs + blocks[b]):
            bt[b, j] = next(free)
    lay = oracle.Layout(oracle.PAGED, L, H, D, B, elem_bytes=E, block_size=bs, num_blocks=nb,
                        block_table=bt)
    recv = G.dev_const(lay.storage_bytes(), 0xA5)
    owner = G.dev_const(nb * 4, 0x7E)
    c = dv.Cache(dv.DV_PAGED, L, H, D, B, [recv], elem_bytes=E, block_size=bs, num_blocks=nb,
                 max_blocks=maxb, block_tables=[G.to_dev(bt)], block_owners=[owner])
    size = dv.dv_packed_bytes(c, 0, L, t0, t1)
    wire_h = synth.fill_bytes(size, 33)
    dv.dv_stream_in(c, 0, 0, L, t0, t1, G.to_dev(wire_h), size, stream())
    torch.cuda.synchronize()
    want = np.full(lay.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.unpack(lay, want, 0, L, t0, t1, wire_h)
    assert G.host(recv)[: want.size].tobytes() == want.tobytes()
    assert (G.host(owner).view(np.int32) == G.owner_map_expected(bt, nb, bs, t0, t1)).all()


def test_unit_numbers_past_2_31():
    """One sequence whose blocks hold 2^31 units of a slab, all but three of
    them unmapped: gather, scatter in table order, and scatter in pool order
    into a pool that large.  Mapped blocks compare with torch's own indexing;
    the buffers' other bytes are never touched."""
    free, _ = torch.cuda.mem_get_info()
    if free < 200 << 30:
        pytest.skip("needs 200 GiB of free device memory")
    L, H, D, E, bs, blocks = 1, 512, 512, 2, 256, 256
    n = bs * blocks
    slab = H * n * D * E  # bytes, 2^35
    wire = torch.empty(2 * slab, dtype=torch.uint8, device=G.DEV)
    w = wire.view(2, H, n, D * E)
    t1 = np.array([n], np.int32)
    mapped = {0: 1, 131: 0, 255: 2}  # logical block -> block of the small pool

    def table(m, nb):
        bt = np.full((1, blocks), -1, np.int32)
        for j, b in m.items():
            bt[0, j] = b
        return dict(block_size=bs, num_blocks=nb, max_blocks=blocks, block_tables=[G.to_dev(bt)])

    small = G.dev_filled(2 * 3 * H * bs * D * E, 5)
    s = small.view(2, 3, H, bs, D * E)
    c = dv.Cache(dv.DV_PAGED, L, H, D, 1, [small], **table(mapped, 3))
    assert dv.dv_stream_out_prompt(c, 0, 0, L, None, t1, wire, 2 * slab, stream()) == 2 * slab
    torch.cuda.synchronize()
    for j, b in mapped.items():
        assert torch.equal(w[:, :, j * bs:(j + 1) * bs], s[:, b]), f"gathered block {j}"
    recv = torch.zeros_like(small)
    c = dv.Cache(dv.DV_PAGED, L, H, D, 1, [recv], **table(mapped, 3))
    dv.dv_stream_in(c, 0, 0, L, None, t1, wire, 2 * slab, stream())
    torch.cuda.synchronize()
    assert torch.equal(recv, small), "scattered in table order"
    del recv
    large = torch.empty(2 * slab, dtype=torch.uint8, device=G.DEV)
    p = large.view(2, blocks, H, bs, D * E)
    places = {0: 255, 131: 77, 255: 0}
    owner = torch.empty(blocks, dtype=torch.int32, device=G.DEV)
    c = dv.Cache(dv.DV_PAGED, L, H, D, 1, [large], block_owners=[owner], **table(places, blocks))
    dv.dv_stream_in(c, 0, 0, L, None, t1, wire, 2 * slab, stream())
    torch.cuda.synchronize()
    assert owner[77].item() == 131 and owner[1].item() == -1
    for j, b in places.items():
        assert torch.equal(p[:, b], s[:, mapped[j]]), f"pool-order block {j}"
    del wire, large
    torch.cuda.empty_cache()
