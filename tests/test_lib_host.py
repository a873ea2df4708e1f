"""Host-side checks of the C ABI: the library loads, exports every declared
symbol, and rejects bad arguments before touching the GPU."""
import ctypes
import os
import re

import pytest

import paper_2510_18830_amd as ms

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "msparse.h")


def declared():
    text = open(HEADER).read()
    return sorted(set(re.findall(r"\b(msparse_[a-z_]+)\s*\(", text)))


def test_exports_every_declared_symbol():
    so = ms.lib()
    names = declared()
    assert len(names) >= 11
    for n in names:
        assert hasattr(so, n), n


def test_strerror():
    L = ms.lib()
    assert L.msparse_strerror(0) == b"ok"
    assert L.msparse_strerror(-3) == b"index capacity too small"


def _bad(status_expected, fn, *args):
    st = fn(*args)
    assert st == status_expected, (st, ms.lib().msparse_last_error())


def test_validation_before_launch():
    L = ms.lib()
    d = ms.make_dims(1, 4096, 4, 2, 128)
    fake = ctypes.c_void_p(16)   # never dereferenced: validation fails first
    iv = ctypes.c_void_p(32)
    # bad head_dim / block / causal / N % 64 / GQA
    for field, val, st in (("head_dim", 96, -2), ("block", 128, -2), ("causal", 0, -2), ("seq_q", 4000, -2),
                           ("heads_kv", 3, -1)):
        dd = ms.make_dims(1, 4096, 4, 2, 128)
        setattr(dd, field, val)
        if field == "seq_q":
            dd.seq_k = val
        _bad(st, L.msparse_estimate, ctypes.byref(dd), fake, fake, 64, 10, 10, iv, iv, None, None, fake, 1 << 30,
             None)
    # budgets and last_q
    _bad(-1, L.msparse_estimate, ctypes.byref(d), fake, fake, 0, 10, 10, iv, iv, None, None, fake, 1 << 30, None)
    _bad(-1, L.msparse_estimate, ctypes.byref(d), fake, fake, 64, 0, 10, iv, iv, None, None, fake, 1 << 30, None)
    _bad(-1, L.msparse_estimate, ctypes.byref(d), fake, fake, 64, 10, 4097, iv, iv, None, None, fake, 1 << 30, None)
    _bad(-2, L.msparse_estimate, ctypes.byref(d), fake, fake, 65, 10, 10, iv, iv, None, None, fake, 1 << 30, None)
    _bad(-1, L.msparse_estimate, ctypes.byref(d), None, fake, 64, 10, 10, iv, iv, None, None, fake, 1 << 30, None)
    # workspace too small
    _bad(-4, L.msparse_estimate, ctypes.byref(d), fake, fake, 64, 10, 10, iv, iv, None, None, fake, 8, None)
    # ring descriptors
    r = ms.Ring(4, 4, 0, 0)
    _bad(-1, L.msparse_index_count, ctypes.byref(d), iv, 10, iv, 10, ctypes.byref(r), ctypes.byref(ctypes.c_int64()),
         ctypes.byref(ctypes.c_int64()), ctypes.byref(ctypes.c_int64()), fake, 1 << 30, None)
    r = ms.Ring(4, 1, 0, 7)
    _bad(-1, L.msparse_index_count, ctypes.byref(d), iv, 10, iv, 10, ctypes.byref(r), ctypes.byref(ctypes.c_int64()),
         ctypes.byref(ctypes.c_int64()), ctypes.byref(ctypes.c_int64()), fake, 1 << 30, None)
    # a null index
    _bad(-1, L.msparse_attn_fwd, ctypes.byref(d), fake, fake, fake, None, fake, fake, None, fake, 1 << 40, None)
    # fused forward + merge: a null index, a null accumulator, a bad head_dim
    _bad(-1, L.msparse_attn_fwd_merge, ctypes.byref(d), fake, fake, fake, None, fake, fake, None, 0, fake, 1 << 40,
         None)
    _bad(-1, L.msparse_attn_fwd_merge, ctypes.byref(d), fake, fake, fake, None, None, fake, None, 1, fake, 1 << 40,
         None)
    dd = ms.make_dims(1, 4096, 4, 2, 128)
    dd.head_dim = 96
    _bad(-2, L.msparse_attn_fwd_merge, ctypes.byref(dd), fake, fake, fake, None, fake, fake, None, 0, fake, 1 << 40,
         None)
    # tensors off 16-byte alignment (checked before the index and workspace)
    odd = ctypes.c_void_p(24)
    _bad(-1, L.msparse_attn_fwd, ctypes.byref(d), fake, odd, fake, None, fake, fake, None, fake, 1 << 40, None)
    _bad(-1, L.msparse_attn_fwd_merge, ctypes.byref(d), fake, fake, fake, None, odd, fake, None, 0, fake, 1 << 40,
         None)
    _bad(-1, L.msparse_attn_bwd, ctypes.byref(d), fake, fake, fake, fake, None, odd, fake, None, fake, fake, fake, 0,
         fake, 1 << 40, None)
    _bad(-1, L.msparse_estimate, ctypes.byref(d), odd, fake, 64, 10, 10, iv, iv, None, None, fake, 1 << 30, None)
    _bad(-1, L.msparse_merge_out_lse, ctypes.byref(d), fake, fake, fake, fake, odd, 0, None)
    assert "16-byte" in L.msparse_last_error().decode()


def test_index_capacity_needs_overflow_flag_or_bound():
    L = ms.lib()
    d = ms.make_dims(1, 4096, 1, 1, 64)
    fake = ctypes.c_void_p(16)
    x = ms.IndexStruct(fake, fake, 10, fake, fake, 10, fake, fake, fake, fake, 10, fake, fake, fake, None, 1)
    ws = L.msparse_index_workspace(ctypes.byref(d), 8, 8, None)
    assert ws > 0
    _bad(-3, L.msparse_build_index, ctypes.byref(d), fake, 8, fake, 8, None, ctypes.byref(x), fake, ws, None)


def test_workspace_queries_are_positive():
    L = ms.lib()
    d = ms.make_dims(1, 131072, 32, 8, 128)
    assert L.msparse_estimate_workspace(ctypes.byref(d), 64, 2048, 8192) >= 2 * 32 * 131072 * 4
    assert L.msparse_attn_bwd_workspace(ctypes.byref(d), 32 * 2048) >= 32 * 131072 * 4
    assert L.msparse_index_workspace(ctypes.byref(d), 2048, 8192, ctypes.byref(ms.Ring(8, 0, 3, 1))) > 0


def test_topp_validation_before_launch():
    L = ms.lib()
    d = ms.make_dims(1, 4096, 4, 2, 128)
    fake = ctypes.c_void_p(16)
    iv = ctypes.c_void_p(32)

    def call(p_v, p_s, kv=10, ks=10, cnt=iv, ws=1 << 30):
        return L.msparse_estimate_topp(ctypes.byref(d), fake, fake, 64, p_v, p_s, kv, ks, iv, iv, cnt, cnt, None,
                                       None, fake, ws, None)

    for p in (0.0, 1.0, -0.5, 1.5, float("nan")):
        _bad(-1, call, p, 0.5)
        _bad(-1, call, 0.5, p)
    _bad(-1, lambda: call(0.5, 0.5, cnt=None))
    _bad(-1, lambda: call(0.5, 0.5, kv=0))
    _bad(-1, lambda: call(0.5, 0.5, ks=4097))
    _bad(-4, lambda: call(0.5, 0.5, ws=8))
    assert L.msparse_estimate_topp_workspace(ctypes.byref(d), 64, 100, 100) == \
        L.msparse_estimate_workspace(ctypes.byref(d), 64, 100, 100)


def test_ring_shard_matches_oracle_schedule():
    from oracle import index as OI
    for W, inner in ((1, 0), (2, 0), (4, 2), (8, 4), (8, 2), (12, 3), (16, 16), (6, 1)):
        S = OI.ring_schedule(W, inner)
        for r in range(W):
            for t in range(W):
                assert ms.ring_shard(W, inner, r, t) == S[r, t], (W, inner, r, t)
    assert ms.ring_shard(8, 3, 0, 0) == -1 and ms.ring_shard(8, 4, 8, 0) == -1 and ms.ring_shard(8, 4, 0, -1) == -1


def test_ring_validation_before_launch():
    L = ms.lib()
    d = ms.make_dims(1, 8192, 2, 1, 128)
    fake = ctypes.c_void_p(16)
    iv = ctypes.c_void_p(32)
    # hierarchical inner must divide world
    r = ms.Ring(8, 1, 0, 0, 3)
    _bad(-1, L.msparse_index_count, ctypes.byref(d), iv, 10, iv, 10, ctypes.byref(r), ctypes.byref(ctypes.c_int64()),
         ctypes.byref(ctypes.c_int64()), ctypes.byref(ctypes.c_int64()), fake, 1 << 30, None)

    def work(world, layout, tiles=iv, ws=1 << 30):
        return L.msparse_ring_work(ctypes.byref(d), iv, 10, iv, 10, world, layout, tiles, iv, fake, ws, None)
    _bad(-1, lambda: work(0, 0))
    _bad(-1, lambda: work(8, 5))
    _bad(-1, lambda: work(8, 0, tiles=None))
    _bad(-2, lambda: work(3, 0))         # 128 blocks do not split into 3 shards
    _bad(-2, lambda: work(128, 1))       # zigzag needs 2 * 128 chunks
    _bad(-4, lambda: work(8, 0, ws=8))


def test_peak_probe_validation():
    L = ms.lib()
    fake = ctypes.c_void_p(16)
    for w, it, out in ((0, 16, fake), (9, 16, fake), (2, 0, fake), (2, 12, fake), (2, 16, None)):
        for rnd in (0, 1):
            assert L.msparse_mfma_peak_probe(w, it, rnd, out, None) == -1


def test_bwd_flags_validation():
    L = ms.lib()
    d = ms.make_dims(1, 4096, 4, 2, 128)
    fake = ctypes.c_void_p(16)
    idx = ms.IndexStruct()
    for f in ("blk_ptr", "blk_idx", "col_ptr", "col_idx", "kblk_ptr", "kblk_idx", "vcol_ptr", "vcol_idx", "diag_bits",
              "q_blk_global", "k_blk_global"):
        setattr(idx, f, 64)
    idx.blk_cap = idx.col_cap = idx.vcol_cap = 1
    idx.world = 1
    st = L.msparse_attn_bwd(ctypes.byref(d), fake, fake, fake, fake, None, fake, fake, ctypes.byref(idx), fake, fake,
                            fake, 4, fake, 1 << 40, None)
    assert st == -1, ms.lib().msparse_last_error()


def test_header_compiles_as_c_and_cpp():
    """include/msparse.h is a plain C header (C99 and C++)."""
    import shutil
    import subprocess
    hdr = os.path.join(os.path.dirname(__file__), "..", "include", "msparse.h")
    for cc, lang, std in (("gcc", "c", "-std=c99"), ("g++", "c++", "-std=c++17")):
        if shutil.which(cc) is None:
            pytest.skip(f"{cc} not installed")
        r = subprocess.run([cc, "-fsyntax-only", "-Wall", "-Werror", "-x", lang, std, hdr], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr


def _estimate_chunks(B, Hq, Hkv, N, d):
    """Key tiles per workgroup of the estimation passes, from the workspace that holds their partials."""
    up = lambda x: (x + 255) // 256 * 256
    BH, nb, ns = B * Hq, N // 64, (N + 16383) // 16384
    got = ms.lib().msparse_estimate_workspace(ctypes.byref(ms.make_dims(B, N, Hq, Hkv, d)), 64, 8, 8)
    hist = 2 * BH * 3 * 2048 if ns > 1 else 0
    rest = (2 * up(4 * BH * N) + up(4 * BH * 64) + up(4 * hist) + up(8 * hist) + up(8 * BH * N if ns > 1 else 0)
            + 3 * up(4 * 2 * BH * ns) + up(2 * BH * 3 * 24))
    fits = [t for t in (2, 4, 8, 16, 32) if rest + 3 * up(4 * BH * 64 * ((nb + t - 1) // t)) == got]
    assert len(fits) == 1, (got, rest, fits)
    return fits[0]


@pytest.mark.parametrize("B,Hq,Hkv,N,d,tiles", [
    # without GQA a share has two waves: four workgroups to a CU at head dim 64, three at 128
    (1, 16, 16, 65536, 64, 16), (1, 8, 8, 32768, 64, 4), (1, 32, 32, 16384, 64, 8), (1, 16, 16, 65536, 128, 8),
    # shares of two heads at head dim 64: four; of four heads: two
    (1, 16, 8, 65536, 64, 8), (1, 28, 4, 524288, 128, 32), (1, 32, 8, 131072, 128, 32), (1, 16, 2, 32768, 128, 4),
    # few heads: short chunks, but not so many that the combine takes longer
    (1, 1, 1, 4096, 64, 2), (1, 1, 1, 524288, 64, 8), (1, 1, 1, 524288, 128, 16)])
def test_estimate_chunks_by_resident_workgroups(B, Hq, Hkv, N, d, tiles):
    """The chunks that the passes measured fastest with, or within 5 % of it, over the sizes of
    their shares of heads."""
    assert _estimate_chunks(B, Hq, Hkv, N, d) == tiles


def test_bench_names_the_kernels_that_run():
    """bench.py's kernel names follow the launchers' rule for small grids."""
    import bench
    from synth import WORKLOADS
    text = open(os.path.join(os.path.dirname(HEADER), "..", "paper_2510_18830_amd", "csrc", "tiles.h")).read()
    for name, lines in (("kSplitFwdGrid", bench.SPLIT_FWD_GRID), ("kSplitDqGrid", bench.SPLIT_DQ_GRID)):
        m = re.search(rf"{name} = D == 64 \? (\d+) : (\d+);", text)
        assert lines == {64: int(m[1]), 128: int(m[2])}, name
    assert f"kSplitKeyGrid = {bench.SPLIT_KEY_GRID};" in text
    assert "return pairs <= kSplitKeyGrid && (pairs - 1) % 256 < 128;" in text
    names = {w: [bench.kernel_symbol(n, WORKLOADS[w]) for n in ("attn_fwd", "bwd_dq", "bwd_dkdv", "est_pass1")]
             for w in ("tiny_4k", "layer_32k", "layer_512k")}
    assert names["tiny_4k"] == ["attn_fwd_split_kernel<64>", "bwd_dq_split_kernel<64>",
                                "bwd_dkdv_rows_kernel<64, true>", "est_pass1_kernel<64>"]
    assert names["layer_32k"] == names["layer_512k"] == ["attn_fwd_kernel<128>", "bwd_dq_kernel<128>",
                                                         "bwd_dkdv_rows_kernel<128, false>", "est_pass1_kernel<128>"]
    wl = WORKLOADS["layer_32k"].resized(seq=64 * 39, heads_q=16, heads_kv=16)     # 320 pairs of key blocks
    assert bench.kernel_symbol("bwd_dkdv", wl) == "bwd_dkdv_rows_kernel<128, true>"


@pytest.mark.parametrize("BH,nb,world,k_v,k_s", [(200000, 1, 1, 8, 16), (100000, 2, 1, 16, 16), (1500, 1, 2, 4, 4),
                                                 (28, 8192, 1, 4096, 16384), (28, 1024, 8, 4096, 16384)])
def test_index_workspace_holds_the_lists_only(BH, nb, world, k_v, k_s):
    """The index workspace is the sum of its lists (bitmap, verticals, diagonals, prefix counts,
    counts, offsets): what the count pass needs besides lies in the place of one of them, so
    that calls which fit the fixed scratch of the allocation-free build keep fitting it."""
    up = lambda x: (x + 255) // 256 * 256
    ng = nb * world
    words = (ng + 31) // 32
    want = (up(4 * BH * 2 * ng) + up(4 * BH * k_v) + 2 * up(4 * BH) + up(4 * BH * ng) + up(4 * BH * words)
            + up(4 * BH * (words + 1)) + up(4 * BH * (ng + 1)) + up(4 * BH) + 3 * up(8 * BH * nb) + up(8 * BH)
            + 3 * up(8 * (BH * nb + 1)) + up(8 * (BH + 1)))
    dims, ring = ms.make_dims(1, 64 * nb, BH, BH, 64), ms.make_ring(world, world - 1, 0)
    assert ms.index_workspace_bytes(dims, k_v, k_s, ring) <= want
