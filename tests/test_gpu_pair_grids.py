"""The kernels that long layers run (two blocks per workgroup), at grids beyond the lines up
to which a workgroup takes one block: many heads of short sequences, sampled heads against the
fp64 oracle.  17 blocks make 9 pairs per head, one of them with a lone block."""
import math

import numpy as np
import pytest
import torch

import paper_2510_18830_amd as ms
from oracle import attn as OA
from oracle import index as OI
from synth import WORKLOADS, make_inputs
from tests.helpers import assert_close, assert_close_rows, assert_lse_close, inputs_f64
from tests.test_gpu_safety import _outlier_rows

pytestmark = pytest.mark.gpu

GRIDS = [(64, 100), (128, 52)]      # head dim, heads: 900 and 468 pairs of 17 blocks


def _workload(d, heads, seq):
    return WORKLOADS["layer_32k"].resized(seq=seq, heads_q=heads, heads_kv=heads, head_dim=d, k_v=60, k_s=120, n_vert=2)


def _lists(wl, seed):
    """Random lists per head; head 1 selects no key for its first block."""
    rng = np.random.default_rng(seed)
    N, H = wl.seq, wl.heads_q
    vi = np.stack([np.sort(rng.choice(N, wl.k_v, replace=False)) for _ in range(H)])
    si = np.stack([np.sort(rng.choice(N, wl.k_s, replace=False)) for _ in range(H)])
    si[:, 0] = 0
    si[1] = np.sort(rng.choice(np.arange(65, N), wl.k_s, replace=False))
    vi[1] = np.sort(rng.choice(np.arange(64, N), wl.k_v, replace=False))
    return vi[None].astype(np.int32), si[None].astype(np.int32)


def _one(f, names, h):
    return tuple(f[n][:, h:h + 1] for n in names)


@pytest.mark.parametrize("d,heads", GRIDS)
@pytest.mark.parametrize("outliers", [False, True])
def test_fwd_bwd_parity(gpu, d, heads, outliers):
    wl = _workload(d, heads, 1088)
    print(f"pair grids d{d} x {heads} outliers {outliers}", flush=True)
    x = _outlier_rows(wl, d, 3, 2) if outliers else make_inputs(wl, "cpu")
    f = inputs_f64(x)
    vi, si = _lists(wl, heads)
    dims = ms.make_dims(1, wl.seq, heads, heads, d)
    idx = ms.make_index(dims, torch.from_numpy(vi).to(gpu), torch.from_numpy(si).to(gpu))
    q, k, v, do = (x[n].to(gpu) for n in ("q", "k", "v", "do"))
    of = torch.empty(q.shape, dtype=torch.float32, device=gpu)
    out, lse = ms.attn_fwd(dims, q, k, v, idx, out_f32=of)
    dq, dk, dv = ms.attn_bwd(dims, q, k, v, out, do, lse, idx, out_f32=of)
    assert torch.equal(out, of.bfloat16())
    close = assert_close_rows if outliers else assert_close
    scale = 1 / math.sqrt(d)
    for h in (0, 1, heads - 1):
        ref = OI.Index(vi[:, h:h + 1], si[:, h:h + 1], wl.seq)
        ro, rl = OA.layer_fwd(*_one(f, ("q", "k", "v"), h), ref, scale)
        rg = OA.layer_bwd(*_one(f, ("q", "k", "v", "do"), h), ref, scale)
        assert_lse_close(lse[:, h:h + 1].cpu().numpy(), rl)
        for n, g, r in zip(("out", "dq", "dk", "dv"), (of, dq, dk, dv), (ro, *rg)):
            close(f"{n} head {h}", g[:, h:h + 1].cpu().numpy(), r)
    assert not of[:, 1, :64].any() and not dq[:, 1, :64].any() and bool(torch.isneginf(lse[:, 1, :64]).all())


@pytest.mark.parametrize("d,heads", GRIDS)
def test_overflowed_index_leaves_outputs_untouched(gpu, d, heads):
    wl = _workload(d, heads, 1088)
    x = make_inputs(wl, "cpu")
    vi, si = (torch.from_numpy(t).to(gpu) for t in _lists(wl, heads))
    dims = ms.make_dims(1, wl.seq, heads, heads, d)
    blk, col, vcol = ms.index_count(dims, vi, si)
    small = ms.alloc_index(dims, blk // 2, col // 2, vcol, gpu)
    ms.build_index(dims, vi, si, small)
    torch.cuda.synchronize()
    assert int(small["overflow"].item()) == 1
    q, k, v, do = (x[n].to(gpu) for n in ("q", "k", "v", "do"))
    rows = q.shape[:-1]
    t = {n: torch.full(s, 7.0, dtype=torch.bfloat16 if n == "out" else torch.float32, device=gpu)
         for n, s in (("out", q.shape), ("lse", rows), ("o32", q.shape), ("acc", q.shape), ("lacc", rows),
                      ("dq", q.shape), ("dk", k.shape), ("dv", v.shape))}
    ms.attn_fwd(dims, q, k, v, small, out=t["out"], lse=t["lse"], out_f32=t["o32"])
    ms.attn_fwd_merge(dims, q, k, v, small, t["acc"], t["lacc"], first=False)
    ms.attn_bwd(dims, q, k, v, t["out"], do, t["lse"], small, t["dq"], t["dk"], t["dv"], out_f32=t["o32"])
    torch.cuda.synchronize()
    for n, a in t.items():
        assert bool((a == 7.0).all()), n


@pytest.mark.parametrize("d,heads", GRIDS)
@pytest.mark.parametrize("layout", ["striped", "zigzag"])
def test_ring_merge(gpu, d, heads, layout):
    """Worker 1 of two at 2048 tokens: 8 pairs of blocks per head and step, merged in the
    forward's epilogue."""
    W, r = 2, 1
    wl = _workload(d, heads, 2048)
    x = make_inputs(wl, "cpu", with_do=False)
    f = inputs_f64(x, ("q", "k", "v"))
    vi, si = _lists(wl, heads + 1)
    tv, ts = torch.from_numpy(vi).to(gpu), torch.from_numpy(si).to(gpu)
    nb = wl.seq // 64
    local = lambda w: (OI.local_blocks(w, nb, W, layout)[:, None] * 64 + np.arange(64)[None]).reshape(-1)
    rows = local(r)
    dims = ms.make_dims(1, wl.seq // W, heads, heads, d)
    q = x["q"][:, :, torch.from_numpy(rows)].contiguous().to(gpu)
    acc = torch.empty(q.shape, dtype=torch.float32, device=gpu)
    lse = torch.empty(q.shape[:-1], dtype=torch.float32, device=gpu)
    out = torch.empty_like(q)
    for t in range(W):
        at = torch.from_numpy(local(ms.ring_shard(W, 0, r, t)))
        idx = ms.make_index(dims, tv, ts, ms.make_ring(W, r, t, layout))
        ms.attn_fwd_merge(dims, q, x["k"][:, :, at].contiguous().to(gpu), x["v"][:, :, at].contiguous().to(gpu), idx,
                          acc, lse, out if t == W - 1 else None, first=t == 0)
    assert torch.equal(out, acc.bfloat16())
    for h in (0, 1, heads - 1):
        ref = OI.Index(vi[:, h:h + 1], si[:, h:h + 1], wl.seq)
        ro, rl = OA.layer_fwd(*_one(f, ("q", "k", "v"), h), ref, 1 / math.sqrt(d), rows=rows)
        assert_close(f"out head {h}", acc[:, h:h + 1].cpu().numpy(), ro)
        assert_lse_close(lse[:, h:h + 1].cpu().numpy(), rl)


@pytest.mark.parametrize("d,heads", GRIDS)
def test_graph_replay(gpu, d, heads):
    wl = _workload(d, heads, 1088)
    dims = ms.make_dims(1, wl.seq, heads, heads, d)
    xs = [make_inputs(wl.resized(seed=wl.seed + i), "cpu") for i in range(2)]
    idx = ms.make_index(dims, *(torch.from_numpy(t).to(gpu) for t in _lists(wl, 3)))
    buf = {n: xs[0][n].to(gpu) for n in ("q", "k", "v", "do")}
    out = torch.empty_like(buf["q"])
    lse = torch.empty(buf["q"].shape[:-1], dtype=torch.float32, device=gpu)
    dq, dk, dv = (torch.empty(buf[n].shape, dtype=torch.float32, device=gpu) for n in ("q", "k", "v"))
    fws = ms._workspace(ms.attn_fwd_workspace_bytes(dims), gpu)
    bws = ms._workspace(ms.attn_bwd_workspace_bytes(dims, idx.struct.vcol_cap), gpu)

    def step(stream=None):
        ms.attn_fwd(dims, buf["q"], buf["k"], buf["v"], idx, out=out, lse=lse, workspace=fws, stream=stream)
        ms.attn_bwd(dims, buf["q"], buf["k"], buf["v"], out, buf["do"], lse, idx, dq, dk, dv, workspace=bws,
                    stream=stream)

    def load(x):
        for n in buf:
            buf[n].copy_(x[n].to(gpu))
        torch.cuda.synchronize()

    refs = []
    for x in xs:
        load(x)
        step()
        torch.cuda.synchronize()
        refs.append([t.clone() for t in (out, lse, dq, dk, dv)])
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        step(stream)
    for x, ref in zip(xs + xs[:1], refs + refs[:1]):
        load(x)
        graph.replay()
        torch.cuda.synchronize()
        for n, got, want in zip(("out", "lse", "dq", "dk", "dv"), (out, lse, dq, dk, dv), ref):
            assert torch.equal(got, want), n
