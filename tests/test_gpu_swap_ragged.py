"""Swaps of ragged wide rows (one 3-D copy per sequence on the DMA engines),
byte for byte against the oracle: capacities that differ, ranges that start
anywhere, sequences without tokens, layer sub-ranges, odd head sizes, and the
same calls replayed from a HIP graph; a cache whose copies span more than 4 GB;
and slabs of 2 GB, which keep 2-D copies."""
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

# layers, (first, last) layer, heads, head_dim, elem_bytes, batch, slot and mirror capacity
SHAPES = {
    "even": (2, (0, 2), 3, 128, 2, 4, 600, 600),
    "odd-heads": (3, (1, 3), 5, 80, 2, 3, 700, 913),
    "narrower-mirror": (2, (0, 2), 2, 96, 4, 3, 401, 333),
    "one-sequence-ragged-start": (1, (0, 1), 1, 256, 2, 2, 300, 290),
}


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_ragged_wide_rows(oracle_lib, shape, captured):
    L, (l0, l1), H, D, E, B, S, M = SHAPES[shape]
    r = np.random.default_rng(sorted(SHAPES).index(shape))
    cap, tok = min(S, M), D * E
    t0 = r.integers(0, 20, size=B).astype(np.int32)
    t1 = np.array([r.integers(a, cap + 1) for a in t0], np.int32)
    t0[0], t1[0] = 3, cap  # rows of 64 KB and more
    t1[B - 1] = t0[B - 1] if B > 2 else t1[B - 1]  # a sequence without tokens
    assert (t1[0] - t0[0]) * tok >= 64 * 1024
    dl = oracle.Layout(oracle.DENSE, L, H, D, B, seq_cap=S, elem_bytes=E)
    hl = oracle.Layout(oracle.DENSE, L, H, D, B, seq_cap=M, elem_bytes=E)
    slot_h = synth.fill_bytes(dl.storage_bytes(), 71)
    slots = [G.to_dev(slot_h), G.dev_const(dl.storage_bytes(), 0xA5)]
    mirror = torch.full((hl.storage_bytes(),), 0x77, dtype=torch.uint8, pin_memory=True)
    d = dv.Cache(dv.DV_DENSE, L, H, D, B, slots, max_seq=S, elem_bytes=E)
    h = dv.Cache(dv.DV_DENSE, L, H, D, B, [mirror], max_seq=M, elem_bytes=E,
                 mem=dv.DV_MEM_HOST_PINNED)

    def swap():
        dv.dv_swap_out(d, 0, h, 0, l0, l1, t0, t1)
        dv.dv_swap_in(h, 0, d, 1, l0, l1, t0, t1)

    exp_host = np.full(hl.storage_bytes(), 0x77, np.uint8)
    oracle_lib.copy_ranges(dl, slot_h, hl, exp_host, l0, l1, t0, t1)
    exp_slot = np.full(dl.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.copy_ranges(hl, exp_host, dl, exp_slot, l0, l1, t0, t1)
    if captured:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            swap()
    for _ in range(3 if captured else 1):
        mirror.fill_(0x77)
        slots[1].fill_(0xA5)
        torch.cuda.synchronize()
        graph.replay() if captured else swap()
        torch.cuda.synchronize()
        assert mirror.numpy().tobytes() == exp_host.tobytes()
        assert G.host(slots[1]).tobytes() == exp_slot.tobytes()


def test_slabs_of_two_gigabytes():
    L, H, D, E, B, S = 1, 16, 128, 2, 2, 1 << 18
    row = D * E
    slot = torch.empty(2 * B * H * S * row // 8, dtype=torch.int64, device=G.DEV).random_()
    mirror = torch.empty(slot.numel(), dtype=torch.int64, pin_memory=True)
    back = torch.zeros_like(slot)
    d = dv.Cache(dv.DV_DENSE, L, H, D, B, [slot, back], max_seq=S)
    h = dv.Cache(dv.DV_DENSE, L, H, D, B, [mirror], max_seq=S, mem=dv.DV_MEM_HOST_PINNED)
    t0 = np.array([S - 300, 5], np.int32)
    t1 = np.array([S, 12], np.int32)
    dv.dv_swap_out(d, 0, h, 0, 0, L, t0, t1)
    dv.dv_swap_in(h, 0, d, 1, 0, L, t0, t1)
    torch.cuda.synchronize()
    a, b = (x.view(2, B, H, S, row // 8) for x in (slot, back))
    for s in range(B):
        assert torch.equal(a[:, s, :, t0[s]:t1[s]], b[:, s, :, t0[s]:t1[s]])
        b[:, s, :, t0[s]:t1[s]] = 0
    assert not bool(back.any()), "bytes outside the ranges changed"


def test_ragged_wide_rows_of_a_large_cache():
    """Slabs of 302 and 283 MB, 4.8 and 4.5 GB of cache and mirror with pitches of
    their own: every 3-D copy spans more than 4 GB.  The ranges arrive, in the
    mirror and back in a second slot, and nothing beside them changes."""
    L, H, D, E, B, S, M = 8, 72, 128, 2, 8, 2048, 1920
    w = D * E // 8  # int64 words per token
    assert 2 * L * B * H * min(S, M) * D * E > 1 << 32
    slot = torch.empty(2 * L * B * H * S * w, dtype=torch.int64, device=G.DEV).random_()
    back = torch.full_like(slot, 0x5A5A5A5A5A5A5A5A)
    mirror = torch.full((2 * L * B * H * M * w,), 0x3C3C3C3C3C3C3C3C, dtype=torch.int64,
                        pin_memory=True)
    d = dv.Cache(dv.DV_DENSE, L, H, D, B, [slot, back], max_seq=S)
    h = dv.Cache(dv.DV_DENSE, L, H, D, B, [mirror], max_seq=M, mem=dv.DV_MEM_HOST_PINNED)
    t0 = np.array([0, 7, 300, 1919, 0, 64, 900, 0], np.int32)
    t1 = np.array([1920, 411, 1501, 1920, 0, 700, 1900, 1], np.int32)
    l0 = 1  # the last layers
    dv.dv_swap_out(d, 0, h, 0, l0, L, t0, t1)
    dv.dv_swap_in(h, 0, d, 1, l0, L, t0, t1)
    torch.cuda.synchronize()
    host = mirror.to(G.DEV).view(2 * L, B, H, M, w)
    a, b = (x.view(2 * L, B, H, S, w) for x in (slot, back))
    for s in range(B):
        at = slice(int(t0[s]), int(t1[s]))
        assert torch.equal(host[2 * l0:, s, :, at], a[2 * l0:, s, :, at]), f"mirror, sequence {s}"
        assert torch.equal(b[2 * l0:, s, :, at], a[2 * l0:, s, :, at]), f"slot, sequence {s}"
        host[2 * l0:, s, :, at] = 0x3C3C3C3C3C3C3C3C
        b[2 * l0:, s, :, at] = 0x5A5A5A5A5A5A5A5A
    assert bool((host == 0x3C3C3C3C3C3C3C3C).all()), "mirror bytes outside the ranges changed"
    assert bool((back == 0x5A5A5A5A5A5A5A5A).all()), "slot bytes outside the ranges changed"
    del slot, back, mirror, host
    torch.cuda.empty_cache()


@pytest.mark.parametrize("B, hi", [(3, 9), (64, 1), (65, 5), (200, 1), (256, 3), (300, 4)])
def test_narrow_rows_of_many_sequences(oracle_lib, B, hi):
    """The copy kernel's launches of up to 64, up to 256 and more sequences, idle
    ones among them."""
    L, H, D, E, S, M = 2, 3, 80, 1, 40, 37
    r = np.random.default_rng(B)
    t0 = r.integers(0, M - hi, size=B).astype(np.int32)
    n = r.integers(0, hi + 1, size=B)
    n[B // 2] = hi
    t1 = (t0 + n).astype(np.int32)
    dl = oracle.Layout(oracle.DENSE, L, H, D, B, seq_cap=S, elem_bytes=E)
    hl = oracle.Layout(oracle.DENSE, L, H, D, B, seq_cap=M, elem_bytes=E)
    slot_h = synth.fill_bytes(dl.storage_bytes(), 81)
    slots = [G.to_dev(slot_h), G.dev_const(dl.storage_bytes(), 0xA5)]
    mirror = torch.full((hl.storage_bytes(),), 0x77, dtype=torch.uint8, pin_memory=True)
    d = dv.Cache(dv.DV_DENSE, L, H, D, B, slots, max_seq=S, elem_bytes=E)
    h = dv.Cache(dv.DV_DENSE, L, H, D, B, [mirror], max_seq=M, elem_bytes=E,
                 mem=dv.DV_MEM_HOST_PINNED)
    dv.dv_swap_out(d, 0, h, 0, 1, L, t0, t1)
    dv.dv_swap_in(h, 0, d, 1, 1, L, t0, t1)
    torch.cuda.synchronize()
    exp_host = np.full(hl.storage_bytes(), 0x77, np.uint8)
    oracle_lib.copy_ranges(dl, slot_h, hl, exp_host, 1, L, t0, t1)
    assert mirror.numpy().tobytes() == exp_host.tobytes()
    exp_slot = np.full(dl.storage_bytes(), 0xA5, np.uint8)
    oracle_lib.copy_ranges(hl, exp_host, dl, exp_slot, 1, L, t0, t1)
    assert G.host(slots[1])[: exp_slot.size].tobytes() == exp_slot.tobytes()
