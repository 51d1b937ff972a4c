"""Timing cases of the KV-cache streaming path, through the public calls.

Each case is one thing a serving or fault-tolerance loop does with the
library: a decode step's increment, a step that accepts several tokens, a
prompt streamed layer by layer, a whole cache replicated and restored, a paged
pool gathered and scattered, a microbatch swapped.  A pass runs both
directions, since a stream-out is always followed by the receiver's
stream-in, and a swap-out by a later swap-in.

Shapes are one pipeline stage's or one tensor-parallel shard's share of the
models the workloads in ``synth`` name; lengths are spread evenly over a
case's ``[len_lo, len_hi]`` and dealt to the sequences by the seed, so that a
case moves the same number of bytes for every seed.  Payloads are opaque
words to the library (bit copies): the caches are filled with random bits.

Keys of a case:
  op        "stream": stream-out then stream-in, over all layers at once;
            "layers": the same, one call per layer (as layers are computed);
            "swap":   swap-out to a pinned mirror, swap-in to a second slot
  kind      "dense", "splitkey" or "paged" (sender and receiver alike)
  layers, heads, head_dim, elem_bytes, batch   the cache's shape
  max_seq   token capacity of the dense kinds (paged: from the lengths)
  block     paged: tokens per block
  fill      paged: share of the receiver's pool that the call writes; the
            rest of the pool belongs to other sequences
  len_lo, len_hi   tokens that the sequences hold
  tokens    0: the pass moves each sequence's tokens [0, len); K > 0: it
            moves tokens [len, len + k_b), k_b spread over 1..K (a decode
            step: K = 1)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2403_01876_amd import dv


def _case(op, kind, layers, heads, head_dim, batch, len_lo, len_hi, tokens=0, elem_bytes=2,
          max_seq=0, block=0, fill=1.0, **name):
    return dict(name, op=op, kind=kind, layers=layers, heads=heads, head_dim=head_dim,
                elem_bytes=elem_bytes, batch=batch, max_seq=max_seq, block=block, fill=fill,
                len_lo=len_lo, len_hi=len_hi, tokens=tokens)


def listed():
    return [
        # The smallest stream: a tiny dense cache's 100-token prompt (two
        # layers, 410 KB), where launches and latency are all there is.
        _case("stream", "dense", 2, 4, 64, 2, 100, 100, max_seq=128, name="tiny_prompt"),
        # A decode step's increment on an OPT-13B stage: what runs after
        # every step of every microbatch when token streaming is on.
        _case("stream", "dense", 10, 40, 128, 8, 512, 1024, 1, max_seq=2048, name="dense_step"),
        # The same on an OPT-66B stage whose decoder kernels keep keys in
        # 16-byte groups along the token axis.
        _case("stream", "splitkey", 16, 72, 128, 8, 900, 1000, 1, max_seq=2048,
              name="splitkey_step"),
        # A decode step of a paged GQA serving batch of 256 requests.
        _case("stream", "paged", 20, 8, 128, 256, 64, 512, 1, block=16, name="paged_step"),
        # A speculative step: up to 8 accepted tokens per sequence, ragged.
        _case("stream", "paged", 20, 8, 128, 32, 128, 4096, 8, block=16,
              name="paged_multi_step"),
        # Prompts of an OPT-13B stage streamed layer by layer.
        _case("layers", "dense", 10, 40, 128, 8, 512, 1024, max_seq=2048,
              name="dense_prompt_layers"),
        # Fault-tolerance replica of a BLOOM-176B shard (14 of 112 heads) with
        # ragged lengths, and its restore.
        _case("stream", "dense", 10, 14, 128, 16, 64, 2048, max_seq=2048, name="dense_replica"),
        # Prompts of an OPT-13B stage in the split-key layout.
        _case("stream", "splitkey", 10, 40, 128, 8, 512, 1024, max_seq=2048,
              name="splitkey_prompt"),
        # LLaMA-2-70B paged prompts: gather, then scatter into another pool
        # that the call fills (recovery of a whole stage).
        _case("stream", "paged", 20, 8, 128, 32, 128, 4096, block=16, name="paged_prompt"),
        # The same model's tensor-parallel shard of one KV head with a 1-byte
        # cache, moved into a serving pool that other requests share.
        _case("stream", "paged", 80, 1, 128, 64, 128, 4096, elem_bytes=1, block=16, fill=0.4,
              name="paged_shard_1byte"),
        # A microbatch of an OPT-66B stage (two of its layers) through pinned
        # host memory and back.
        _case("swap", "dense", 2, 72, 128, 8, 1000, 1000, max_seq=1024, name="swap_microbatch"),
        # The part of a microbatch that one decode step changed, as the swap
        # scheduler moves it after each step.
        _case("swap", "dense", 16, 72, 128, 8, 200, 200, 1, max_seq=256, name="swap_update"),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], even over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["stream"] * 6 + ["layers", "swap"])
    kind = "dense" if op == "swap" else rng.choice(["dense", "paged", "paged", "splitkey"])
    # A third of the streams are prompts or replicas, the others steps of one
    # or of several tokens; layer-by-layer streams are prompts.
    tokens = 0 if op == "layers" else rng.choice([0, 1, _log_int(rng, 2, 64)])
    elem = rng.choice([1, 2, 2, 4])
    dim = rng.choice([64, 80, 96, 128, 128, 256])
    if kind == "splitkey" and dim * elem > 512:  # the layout's limit: 32 groups of 16 bytes
        dim = 128
    heads = _log_int(rng, 1, 72)
    batch = _log_int(rng, 1, 256 if tokens else 64)
    hi = _log_int(rng, 16, 4096)
    lo = max(1, int(hi * rng.uniform(0.05, 1.0)))
    layers = _log_int(rng, 2, 80)
    block = rng.choice([8, 16, 16, 32, 64]) if kind == "paged" else 0
    fill = rng.choice([1.0, 0.8, 0.4]) if kind == "paged" else 1.0
    cap = hi + tokens + rng.randint(0, hi)
    c = _case(op, kind, layers, heads, dim, batch, lo, hi, tokens, elem,
              0 if kind == "paged" else cap, block, fill)
    # Fewer layers, then fewer sequences, until the pass costs less than the
    # largest listed one and its caches fit.
    most_stored = (1 << 30) if op == "swap" else (8 << 30)
    most_moved = (1 << 29) if op == "swap" else (5 << 30)
    while _stored(c) > most_stored or work(c)["bytes"] > 2 * most_moved:
        if c["layers"] > 2:
            c["layers"] = max(2, c["layers"] // 2)
        elif c["batch"] > 1:
            c["batch"] //= 2
        else:
            c["heads"] = max(1, c["heads"] // 2)
    return c


def _spread(lo, hi, n):
    """n integers spread evenly over [lo, hi] (the middle for n = 1)."""
    return np.array([lo + ((hi - lo) * (2 * i + 1)) // (2 * n) for i in range(n)], dtype=np.int64)


def _ranges(case):
    """Per sequence: tokens held, and the moved range's first token and length."""
    lens = _spread(case["len_lo"], case["len_hi"], case["batch"])
    if case["tokens"] == 0:
        return lens, np.zeros_like(lens), lens
    k = _spread(1, case["tokens"] + 1, case["batch"]).clip(1, case["tokens"])
    return lens, lens, k[np.argsort((np.arange(case["batch"]) * 37) % 101, kind="stable")]


def _blocks(case):
    lens, _, n = _ranges(case)
    need = lens + (n if case["tokens"] else 0)
    return (need + case["block"] - 1) // case["block"]


def _pool_blocks(case):
    """Blocks of the sender's and of the receiver's pool."""
    nb = int(_blocks(case).sum())
    return nb, max(nb, int(nb / case["fill"]))


def _token_bytes(case):
    return case["layers"] * 2 * case["heads"] * case["head_dim"] * case["elem_bytes"]


def _stored(case):
    """Bytes of the larger cache."""
    if case["kind"] == "paged":
        return _token_bytes(case) * case["block"] * _pool_blocks(case)[1]
    return _token_bytes(case) * case["batch"] * case["max_seq"]


def work(case):
    """Every moved byte is read and written once by each of the pass's two
    directions; nothing is computed."""
    return {"bytes": 4 * _token_bytes(case) * int(_ranges(case)[2].sum()), "flops": 0}


def tolerance(case):
    return "exact"  # bit copies


_KINDS = {"dense": dv.DV_DENSE, "splitkey": dv.DV_DENSE_KSPLIT, "paged": dv.DV_PAGED}


def _bits(nbytes, gen):
    return torch.empty(nbytes // 8, dtype=torch.int64, device="cuda").random_(generator=gen)


def _zeros(nbytes, **where):
    return torch.zeros(nbytes // 8, dtype=torch.int64, **(where or {"device": "cuda"}))


def _table(blocks, pool, gen):
    """A block table over a random choice of the pool's blocks, -1 where unmapped."""
    perm = torch.randperm(pool, device="cuda", generator=gen).to(torch.int32)
    width = int(blocks.max())
    start = np.concatenate([[0], np.cumsum(blocks)[:-1]])
    col = torch.arange(width, device="cuda")[None, :]
    count = torch.tensor(blocks, device="cuda")[:, None]
    at = torch.tensor(start, device="cuda")[:, None] + col
    return torch.where(col < count, perm[at.clamp(max=pool - 1)],
                       torch.full((), -1, dtype=torch.int32, device="cuda")).contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    order = np.random.default_rng(seed).permutation(case["batch"])
    lens, first, n = (a[order] for a in _ranges(case))
    t0 = np.ascontiguousarray(first, dtype=np.int32)
    t1 = np.ascontiguousarray(first + n, dtype=np.int32)
    shape = (case["layers"], case["heads"], case["head_dim"], case["batch"])
    kind, eb = _KINDS[case["kind"]], case["elem_bytes"]
    s = {"op": case["op"], "layers": case["layers"], "t0": t0, "t1": t1,
         "single": case["tokens"] == 1}
    if case["op"] == "swap":
        size = _stored(case)
        slots = [_bits(size, gen), _zeros(size)]
        mirror = _zeros(size, pin_memory=True)
        s["slots"] = dv.Cache(kind, *shape, slots, max_seq=case["max_seq"], elem_bytes=eb)
        s["host"] = dv.Cache(kind, *shape, [mirror], max_seq=case["max_seq"], elem_bytes=eb,
                             mem=dv.DV_MEM_HOST_PINNED)
        s["out"] = {"mirror": mirror, "slot": slots[1]}
        return s
    if case["kind"] == "paged":
        blocks, pools = _blocks(case)[order], _pool_blocks(case)
        sizes = [_token_bytes(case) * case["block"] * p for p in pools]
        src, dst = _bits(sizes[0], gen), _zeros(sizes[1])
        tables = [_table(blocks, p, gen) for p in pools]
        owner = torch.empty(pools[1], dtype=torch.int32, device="cuda")
        width = int(blocks.max())
        s["src"] = dv.Cache(kind, *shape, [src], elem_bytes=eb, block_size=case["block"],
                            num_blocks=pools[0], max_blocks=width, block_tables=[tables[0]])
        s["dst"] = dv.Cache(kind, *shape, [dst], elem_bytes=eb, block_size=case["block"],
                            num_blocks=pools[1], max_blocks=width, block_tables=[tables[1]],
                            block_owners=[owner])
    else:
        src, dst = _bits(_stored(case), gen), _zeros(_stored(case))
        s["src"] = dv.Cache(kind, *shape, [src], max_seq=case["max_seq"], elem_bytes=eb)
        s["dst"] = dv.Cache(kind, *shape, [dst], max_seq=case["max_seq"], elem_bytes=eb)
    nbytes = dv.dv_packed_bytes(s["src"], 0, case["layers"], t0, t1)
    wire = _zeros(nbytes)
    s["wire"], s["bytes"], s["base"] = wire, nbytes, wire.data_ptr()
    s["out"] = {"wire": wire, "cache": dst}
    return s


def run(s):
    L, t0, t1 = s["layers"], s["t0"], s["t1"]
    if s["op"] == "swap":
        dv.dv_swap_out(s["slots"], 0, s["host"], 0, 0, L, t0, t1)
        dv.dv_swap_in(s["host"], 0, s["slots"], 1, 0, L, t0, t1)
    elif s["op"] == "layers":
        size = s["bytes"] // L
        for l in range(L):
            at = s["base"] + l * size
            dv.dv_stream_out_prompt(s["src"], 0, l, l + 1, t0, t1, at, size)
            dv.dv_stream_in(s["dst"], 0, l, l + 1, t0, t1, at, size)
    else:
        if s["single"]:
            n = dv.dv_stream_out_token(s["src"], 0, 0, L, t0, s["wire"], s["bytes"])
        else:
            n = dv.dv_stream_out_prompt(s["src"], 0, 0, L, t0, t1, s["wire"], s["bytes"])
        dv.dv_stream_in(s["dst"], 0, 0, L, t0, t1, s["wire"], n)
    return s["out"]
