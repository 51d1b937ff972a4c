"""Which kernels a call launches, without a GPU: the library's host code is
linked with launchers that write down what they are asked (tests/c/
dispatch_record.cpp) and called with made-up addresses, which nothing reads."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2403_01876_amd import dv

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CACHE, WIRE, TABLE, OWNER = 1 << 50, 1 << 52, 1 << 54, 1 << 55


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("dispatch") / "libdispatch.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", "-Werror",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "paper_2403_01876_amd", "csrc", "dv_api.cpp"),
                    os.path.join(ROOT, "tests", "c", "dispatch_record.cpp"),
                    "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-o", out], check=True, timeout=300)
    lib = ctypes.CDLL(out)
    for name in ("dv_packed_bytes", "dv_stream_out_prompt", "dv_stream_in",
                 "dv_stream_in_noalloc", "dv_swap_out"):
        getattr(lib, name).argtypes = getattr(dv.lib, name).argtypes
    lib.dispatch_record_take.restype = ctypes.c_char_p
    return lib


def paged(L, H, D, E, B, bs, nb, maxb, owner=True):
    return dv.Cache(dv.DV_PAGED, L, H, D, B, [CACHE], elem_bytes=E, block_size=bs, num_blocks=nb,
                    max_blocks=maxb, block_tables=[TABLE], block_owners=[OWNER] if owner else None)


def dense(L, H, D, E, B, S, kind=dv.DV_DENSE):
    return dv.Cache(kind, L, H, D, B, [CACHE], max_seq=S, elem_bytes=E)


def call(lib, name, cache, t0, t1, status=dv.DV_OK):
    """The launches of one call over all layers: a list of (kernel, fields)."""
    t0 = np.ascontiguousarray(t0, np.int32)
    t1 = np.ascontiguousarray(t1, np.int32)
    args = [cache.ref, 0, 0, cache.c.num_layers, t0.ctypes.data, t1.ctypes.data, WIRE, 1 << 62]
    lib.dispatch_record_take()
    if name == "out":
        got = lib.dv_stream_out_prompt(*args, None, None)
    else:
        got = getattr(lib, "dv_stream_in_noalloc" if name == "in_noalloc" else "dv_stream_in")(
            *args, None)
    assert got == status, (name, got)
    lines = lib.dispatch_record_take().decode().splitlines()
    return [(ln.split()[0], {k: int(v) for k, v in (f.split("=") for f in ln.split() if "=" in f)})
            for ln in lines]


def kernels(launches):
    return [name for name, _ in launches]


@pytest.mark.parametrize("name", ["in", "in_noalloc"])
def test_owner_map_is_built_where_pool_order_reads_it(lib, name):
    """Over random paged shapes and ranges the owner map is launched exactly
    when the pool-order kernel follows, and that is when the header says."""
    r = np.random.default_rng(3)
    seen = set()
    for _ in range(3000):
        H, D, E = int(r.integers(1, 9)), int(r.choice([16, 64, 128])), int(r.choice([1, 2, 4]))
        B, bs = int(r.choice([1, 3, 40, 64, 65, 256, 257])), int(r.choice([1, 4, 16, 64, 256]))
        n = r.integers(0, int(r.choice([2, 40, 300, 1500])) + 1, size=B)
        t0 = r.integers(0, int(r.choice([1, bs + 1, 4 * bs])), size=B)
        t1 = t0 + n
        blocks = int(np.where(n > 0, -(-t1 // bs) - t0 // bs, 0).sum())
        maxb = max(1, -(-int(t1.max()) // bs))
        nb = max(1, int(blocks / r.choice([1.0, 0.8, 0.56, 0.5, 0.3])))
        c = paged(2, H, D, E, B, bs, nb, maxb)
        ran = kernels(call(lib, name, c, t0, t1))
        want = (B <= 256 and n.max() * D * E // 16 > 256 and n.max() > 1 and
                9 * blocks >= 5 * nb and 4 * n.sum() >= 3 * blocks * bs)
        assert ("pool" in ran) == want, (ran, blocks, nb, bs, n.sum())
        built = [k for k in ran if k.startswith("owner")]
        assert bool(built) == want, ran
        if want:
            assert ran[-1] == "pool" and ran[:-1] == built
        seen.add((want, ran[-1] if ran else None))
    assert {(True, "pool"), (False, "rows"), (False, "table")} <= seen


@pytest.mark.parametrize("name", ["out", "in"])
@pytest.mark.parametrize("owner", [False, True])
def test_ranges_under_three_quarters_of_their_blocks_go_by_rows(lib, name, owner):
    """48 of 64 tokens stand for the table's (or the pool's) order, 47 for rows,
    whether rows fill tiles of their own well (16 heads) or not (one head); slabs
    of 2^31 units and more are past the row kernel and keep whole blocks."""
    whole = "pool" if owner and name == "in" else "table"
    for H in (1, 16):
        c = paged(2, H, 128, 2, 5, 64, 5, 1, owner)
        z = np.zeros(5, np.int32)
        assert kernels(call(lib, name, c, z, z + 48))[-1] == whole
        assert kernels(call(lib, name, c, z, z + 47)) == ["rows"]
        t0, t1 = z + 8, z + 50  # 42 tokens
        assert kernels(call(lib, name, c, t0, t1)) == ["rows"]
    big = paged(1, 1 << 16, 128, 2, 1, 4096, 1, 1, owner)  # 2^20 units a token
    assert kernels(call(lib, name, big, [0], [2047])) == ["rows"]
    assert kernels(call(lib, name, big, [0], [2048])) == ["table"]


@pytest.mark.parametrize("du, tile, odd_in", [(16, 32, 32), (20, 24, 96), (24, 64, 64), (32, 16, 64)])
def test_split_tiles_for_capacities_that_are_not_whole_lines(lib, du, tile, odd_in):
    """Tokens per tile: eight units per lane instead of two for a large stream-in
    of wide tokens into a capacity that is no multiple of 8, unless its runs
    leave more than two thirds of such tiles empty or just pass one."""
    z = np.zeros(3, np.int32)
    cases = [(2048, "out", 1000, tile, 40), (2048, "in", 1000, tile, 40),
             (2049, "out", 1000, tile, 40), (2049, "in", 1000, odd_in, 40)]
    if odd_in > tile:
        cases += [(2049, "in", (odd_in - 1) // 3, tile, 200), (2049, "in", -(-odd_in // 3), odd_in, 200),
                  (2049, "in", odd_in, odd_in, 200), (2049, "in", odd_in + 1, tile, 200),
                  (2049, "in", 6 * tile, tile, 200), (2049, "in", 6 * tile + 1, odd_in, 200)]
    for S, name, n, want, L in cases:
        c = dense(L, 64, 8 * du, 2, 3, S, dv.DV_DENSE_KSPLIT)
        ran = call(lib, name, c, z, z + n)
        assert kernels(ran) == ["split"] and ran[0][1]["tile"] == want, (S, name, n, ran)
    if odd_in > tile:  # 2^20 units, and fewer
        n = np.array([1000, 0, 0], np.int32)
        for H, want in ((-(-(1 << 20) // (2 * 1000 * du)), odd_in),
                        ((1 << 20) // (2 * 1000 * du), tile)):
            ran = call(lib, "in", dense(1, H, 8 * du, 2, 3, 2049, dv.DV_DENSE_KSPLIT), z, z + n)
            assert ran[0][1]["tile"] == want, (H, ran)


@pytest.mark.parametrize("du", [4, 8, 16, 32])
def test_large_split_key_stream_ins_of_short_runs_go_by_tiles(lib, du):
    """Runs that fill a tile three fifths: rows on the way out at every size, on
    the way in up to 100 million units times groups per token, and at every size
    for fewer than eight groups."""
    n = 512 // du * 3 // 5
    z = np.zeros(10, np.int32)
    most = 100_000_000 // (2 * 5 * 10 * n * du * du)  # layers
    for L in (most, most + 1):
        c = dense(L, 5, 8 * du, 2, 10, 96, dv.DV_DENSE_KSPLIT)
        assert kernels(call(lib, "out", c, z, z + n)) == ["split-rows"]
        by_rows = L == most or du < 8
        assert kernels(call(lib, "in", c, z, z + n)) == ["split-rows" if by_rows else "split"]


@pytest.mark.parametrize("du, L, line", [(1, 1, 70), (1, 40, 92), (4, 1, 92)])
def test_dense_runs_that_fill_tiles_badly_go_by_rows(lib, du, L, line):
    """Out: below 92 % of the tiles' units, for small streams of one-unit tokens
    below 70 %; in: below 45 %."""
    B = 100
    c = dense(L, 5, 16 * du, 1, B, 2048)
    tile = 512 // du
    z = np.zeros(B, np.int32)
    for percent in (46, 60, 69, 71, 91, 93):  # runs of two tiles, of one below the half
        tiles = 1 if percent < 52 else 2
        n = z + -(-tiles * tile * percent // 100)
        if percent == 46:  # below the short-run bound but for one run of two tiles
            n[0] = tile + 1
        full = int((-(-n * du // 512)).sum()) * 512
        assert call(lib, "out", c, z, z + n)[0][0] == (
            "rows" if 100 * n.sum() * du < line * full else "dense"), percent
        assert call(lib, "in", c, z, z + n)[0][0] == (
            "rows" if 100 * n.sum() * du < 45 * full else "dense"), percent
    n = np.where(np.arange(B) % 10, 1, tile)  # mostly empty tiles
    assert kernels(call(lib, "in", c, z, z + n)) == ["rows"]


def test_refusals_count_the_header_s_pieces(lib):
    """Over descriptors near the limit: refused exactly where 64 consecutive
    sequences hold 2^31 pieces, counted as the header counts them, and before
    anything is launched; what is launched fits 32 bits."""
    r = np.random.default_rng(11)
    seen = {True: 0, False: 0}
    for i in range(3000):
        kind = int(r.integers(0, 3))
        du = int(2 ** r.integers(0, 6))
        H = int(2 ** (r.uniform(17, 20) - np.log2(du)))
        B = int(r.choice([1, 64, 65, 130, 300]))
        n = np.minimum(r.integers(1, int(2 ** r.uniform(2, 16)) + 1, size=B), 1 << 16)
        n[r.random(B) < 0.2] = 0
        n[B // 2] = max(2, n[B // 2])
        t0 = r.integers(0, 20, size=B)
        bs = int(2 ** r.integers(0, 8))
        S = int((t0 + n).max())
        maxb = -(-S // bs)
        if kind == 0:
            c = dense(1, H, 8 * du, 2, B, S)
        elif kind == 1:
            c = paged(1, H, 8 * du, 2, B, bs, 1 << 20, maxb)
        else:
            c = dense(1, H, 8 * du, 2, B, S, dv.DV_DENSE_KSPLIT)
        if dv.lib.dv_cache_bytes(c.ref, None) != dv.DV_OK:
            continue
        small = n.max() * du <= 256

        def pieces(k, first):
            if small:
                return k * H * du
            if kind == 1:
                return ((first + k + bs - 1) // bs - first // bs) * ((H + 1) // 2) if k else 0
            return H * (-(-k * du // 512))

        refused = False
        for g in range(0, B, 64):
            k, first = n[g:g + 64].astype(object), t0[g:g + 64].astype(object)
            most = sum(pieces(a, b) for a, b in zip(k, first))
            if kind == 2 and not small:
                most = max(most, sum(H * (-(-a // 64)) for a in k))
            refused = refused or most >= 1 << 31
        seen[refused] += 1
        for name in ("out", "in"):
            ran = call(lib, name, c, t0, t0 + n, dv.DV_ERR_UNSUPPORTED if refused else dv.DV_OK)
            assert bool(ran) == (not refused)
            for kernel, f in ran:
                assert 0 < f.get("units", 1) < 1 << 31 and 0 < f.get("tiles", 1) < 3 << 30, (kernel, f)
                if kernel in ("table", "pool"):
                    assert f["tiles"] < 1 << 24
    assert min(seen.values()) > 100, seen


@pytest.mark.parametrize("B, most", [(1, 192), (64, 192), (65, 288), (128, 288), (150, 384), (256, 480)])
def test_owner_map_in_one_launch_up_to_96_chunks_for_each_it_saves(lib, B, most):
    """A chunk is 64 table entries of one sequence."""
    z = np.zeros(B, np.int32)
    for chunks in (most, most + 1):
        blocks = np.full(B, chunks // B) * 64  # of 16 tokens
        blocks[:chunks % B] += 64
        blocks = np.maximum(blocks - 63, 1)  # the last chunk of each holds one entry
        c = paged(1, 1, 512, 2, B, 16, int(blocks.sum()), int(blocks.max()))
        ran = call(lib, "in", c, z, z + 16 * blocks)
        if chunks == most:
            assert kernels(ran) == ["owner-map", "pool"] and ran[0][1]["chunks"] == chunks
        else:
            assert kernels(ran) == ["owner-clear"] + ["owner-build"] * (-(-B // 64)) + ["pool"]


@pytest.mark.parametrize("du, tile", [(8, 64), (12, 40), (16, 32), (24, 64), (32, 16)])
def test_large_split_key_stream_ins_that_leave_tiles_empty_go_by_rows(lib, du, tile):
    """Every run one tile, with as many tokens on average as the rule asks for,
    and one fewer in all."""
    B = 100
    z = np.zeros(B, np.int32)
    need = -(-(40 - du) * B * tile // 80)  # tokens of all sequences
    n = z + 1
    n[0] = tile  # past the short-run kernel
    for b in range(1, B):
        n[b] += min(tile - 1, max(0, need - int(n.sum())))
    assert int(n.sum()) >= need
    for less, want in ((0, "split"), (1, "split-rows")):
        m = n.copy()
        if less and int(m.sum()) != need:
            continue  # wide tokens: even runs of one token fill that much
        m[1] -= less
        c = dense(2000, 5, 8 * du, 2, B, 64, dv.DV_DENSE_KSPLIT)
        assert kernels(call(lib, "in", c, z, z + m)) == [want], (du, int(m.sum()), need)
        assert kernels(call(lib, "out", c, z, z + m)) == ["split-rows"]
