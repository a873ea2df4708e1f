"""Performance cases: what a user of the library has it do, with sizes, inputs and exact results.

A case is a dict of plain values.  Its ``kind`` names the calls of one pass:

  step      a training layer: estimate -> build_index -> attn_fwd -> attn_bwd
  prefill   a forward-only layer: estimate -> build_index -> attn_fwd
  estimate  pattern estimation with fixed budgets, scores returned
  topp      pattern estimation with the online top-p budgets
  index     build_index from lists in hand, whole sequence
  fwd       attn_fwd over an index in hand
  bwd       attn_bwd over an index and a forward result in hand
  ring      one ring worker's share: per step build_index and attn_fwd_merge, then per step attn_bwd

Inputs are seeded synthetic tensors with a planted vertical-slash structure: N(0, 1) draws, a rotary
band that raises the logits near the diagonal (``slash``), and outlier keys every query attends to.
Buffers, workspaces and indices are laid out once, as a training or serving loop keeps them.

``spread`` cases take lists with the verticals spread over the whole sequence and the slashes as a run
from the diagonal plus a few far ones (long documents with delimiters and sinks); the others take the
lists that the inputs themselves give, which mostly lie near the last queries.
"""
import math

import torch

import paper_2510_18830_amd as ms

LAST_Q = 64
FAR = 16  # far slashes of a spread list
DEV = "cuda"


def listed():
    return [
        # the smallest layer in use: one head at 4K tokens, where launches and latency count
        dict(name="step_4k", kind="step", B=1, Hq=1, Hkv=1, N=4096, d=64, k_v=128, k_s=256, slash=False),
        # an ordinary training layer: 32K tokens, GQA 8
        dict(name="step_32k", kind="step", B=1, Hq=16, Hkv=2, N=32768, d=128, k_v=1000, k_s=6096, slash=True),
        # the headline training layer: 512K tokens on one GPU
        dict(name="step_512k", kind="step", B=1, Hq=28, Hkv=4, N=524288, d=128, k_v=4096, k_s=16384, slash=True),
        # inference: sparse prefill of a 128K prompt
        dict(name="prefill_128k", kind="prefill", B=1, Hq=32, Hkv=8, N=131072, d=128, k_v=2048, k_s=8192, slash=True),
        # pattern estimation alone, as when the pattern is refreshed apart from the attention
        dict(name="estimate_512k", kind="estimate", B=1, Hq=28, Hkv=4, N=524288, d=128, k_v=4096, k_s=16384,
             slash=True),
        # estimation with the online top-p budget of a 128K layer
        dict(name="topp_128k", kind="topp", B=1, Hq=32, Hkv=8, N=131072, d=128, k_v=8192, k_s=16384, p=0.9,
             slash=True),
        # the index of a whole 512K sequence from lists in hand
        dict(name="index_512k", kind="index", B=1, Hq=28, Hkv=4, N=524288, d=128, k_v=4096, k_s=16384, slash=True),
        # a batch of short ragged sequences (an odd number of blocks) at head dim 64, spread verticals
        dict(name="fwd_b2_6k_d64", kind="fwd", B=2, Hq=8, Hkv=2, N=101 * 64, d=64, k_v=256, k_s=1024, spread=True,
             o32=False),
        # the backward of a 128K layer
        dict(name="bwd_128k", kind="bwd", B=1, Hq=32, Hkv=8, N=131072, d=128, k_v=2048, k_s=8192, slash=True, o32=True),
        # a backward with many gathered columns and an odd number of blocks
        dict(name="bwd_32k_cols", kind="bwd", B=1, Hq=16, Hkv=4, N=509 * 64, d=128, k_v=2048, k_s=4096, spread=True,
             o32=True),
        # a backward at head dim 64, no fp32 forward output kept
        dict(name="bwd_16k_d64", kind="bwd", B=1, Hq=12, Hkv=4, N=16384, d=64, k_v=512, k_s=2048, spread=True,
             o32=False),
        # worker 0 of a balanced 8-worker striped ring at 512K tokens, its 8 steps in sequence
        dict(name="ring_512k_w8", kind="ring", B=1, Hq=28, Hkv=4, N=524288, d=128, k_v=4096, k_s=16384, slash=True,
             world=8, rank=0, layout="striped", inner=0),
    ]


def draw(rng):
    kind = rng.choice(["step", "prefill", "estimate", "topp", "index", "fwd", "bwd", "ring"])
    top = 524288 if kind in ("estimate", "index", "topp", "ring") else 196608
    blocks = int(math.exp(rng.uniform(math.log(16), math.log(top // 64))))
    B = rng.choice([1, 1, 2]) if blocks < 1024 else 1
    Hq, Hkv = rng.choice([(1, 1), (4, 1), (8, 8), (8, 2), (12, 4), (16, 2), (28, 4), (32, 8)])
    d = rng.choice([64, 128, 128])
    c = dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, d=d)
    if kind == "ring":
        c["world"] = rng.choice([2, 4, 8])
        c["layout"] = rng.choice(["striped", "zigzag"])
        c["inner"] = rng.choice([0, 2])
        c["rank"] = rng.randrange(c["world"])
        blocks = max(2 * c["world"], blocks // (2 * c["world"]) * 2 * c["world"])
    c["N"] = N = 64 * blocks
    c["k_v"] = max(8, min(8192, int(N * math.exp(rng.uniform(math.log(1 / 128), math.log(1 / 12))))))
    c["k_s"] = max(64, min(16384, int(N * math.exp(rng.uniform(math.log(1 / 32), math.log(1 / 5))))))
    if kind == "topp":
        c["p"] = rng.choice([0.5, 0.8, 0.9, 0.95])
    if kind in ("fwd", "bwd", "index", "ring"):
        c["spread"] = rng.random() < 0.5
    if kind in ("fwd", "bwd"):
        c["o32"] = rng.random() < 0.5
    if not c.get("spread"):
        c["slash"] = rng.random() < 0.8
    return c


# ---------------------------------------------------------------- inputs
def _tensors(c, seed):
    """bf16 q, k, v, do of a case, from the seed alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    B, Hq, Hkv, N, d = c["B"], c["Hq"], c["Hkv"], c["N"], c["d"]
    G = Hq // Hkv
    slash = c.get("slash", True)
    bf = dict(dtype=torch.bfloat16, device=DEV)
    q, k, v, do = (torch.empty((B, h, N, d), **bf) for h in (Hq, Hkv, Hkv, Hq))
    theta = (4.0 * c["k_s"]) ** (-2.0 * torch.arange(d // 2, device=DEV, dtype=torch.float64) / d)
    keep = theta <= 2.0 / c["k_s"]
    keep[-1] = True
    pos = torch.arange(N, device=DEV, dtype=torch.float64)[:, None]
    cos, sin = (f(pos * theta[keep][None]).float() for f in (torch.cos, torch.sin))

    def draw():
        return torch.randn((N, d), generator=g, device=DEV)

    for b in range(B):
        for hk in range(Hkv):
            band = 0.0
            if slash:
                m = cos.shape[1]
                w = torch.randn(2 * m, generator=g, device=DEV)
                w = w / w.norm() * math.sqrt(8.0 * math.sqrt(d))
                band = torch.zeros((N, d), device=DEV)
                sel = torch.nonzero(keep).flatten()
                band[:, sel] = w[:m] * cos - w[m:] * sin
                band[:, sel + d // 2] = w[:m] * sin + w[m:] * cos
            u = torch.zeros(d, device=DEV)
            for h in range(hk * G, hk * G + G):
                x = draw()
                u += x.mean(0)
                q[b, h] = x + band
                do[b, h] = draw()
            x = draw() + band
            at = torch.randperm(N - LAST_Q, generator=g, device=DEV)[: 16 if N <= 4096 else 64]
            x[at] += 3.0 * math.sqrt(d) * u / u.norm()
            k[b, hk] = x
            v[b, hk] = draw()
    return q, k, v, do


def _scores(q, k, scale, dtype):
    """Vertical and slash scores of one head's last queries, plain torch."""
    L, N = q.shape[0], k.shape[0]
    z = (q.to(dtype) @ k.to(dtype).T) * scale
    row = torch.arange(N - L, N, device=z.device)[:, None]
    z.masked_fill_(torch.arange(N, device=z.device)[None] > row, -math.inf)
    p = torch.softmax(z, dim=1)
    skew = torch.zeros((L, N + L), dtype=dtype, device=z.device)
    skew[:, :N] = p.flip(1)
    return p.sum(0), skew.as_strided((L, N), (N + L - 1, 1), L - 1).sum(0)


def _top(score, k):
    """The k largest, lower index first among equal ones, ascending."""
    at = torch.sort(score, descending=True, stable=True).indices[:k]
    return torch.sort(at).values.to(torch.int32)


def _lists(c, seed, q, k, dtype=torch.float32):
    B, Hq, N = c["B"], c["Hq"], c["N"]
    G = Hq // c["Hkv"]
    k_v, k_s = c["k_v"], c["k_s"]
    vi = torch.empty((B, Hq, k_v), dtype=torch.int32, device=DEV)
    si = torch.empty((B, Hq, k_s), dtype=torch.int32, device=DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed + 1)
    for b in range(B):
        for h in range(Hq):
            if c.get("spread"):
                vi[b, h] = torch.sort(torch.randperm(N, generator=g, device=DEV)[:k_v]).values
                run = max(1, k_s - FAR)
                far = run + torch.randperm(N - run, generator=g, device=DEV)[: k_s - run]
                si[b, h] = torch.cat([torch.arange(run, device=DEV), torch.sort(far).values])
            else:
                v, s = _scores(q[b, h, N - LAST_Q:], k[b, h // G], 1 / math.sqrt(c["d"]), dtype)
                vi[b, h], si[b, h] = _top(v, k_v), _top(s, k_s)
    return vi, si


def _index(dims, vi, si, ring=None, room=1.0):
    """An index with the capacities that these lists need (times room)."""
    blk, col, vcol = ms.index_count(dims, vi, si, ring)
    return ms.alloc_index(dims, int(blk * room), int(col * room), vcol, DEV, ring.world if ring else 1)


def _roomy_index(c, dims, vi, si):
    """An index whose capacities follow from the sizes alone; entries past the lists stay 0."""
    blk, col, vcol = ms.index_count(dims, vi, si)
    BH, nb = c["B"] * c["Hq"], c["N"] // 64
    blk = max(blk, min(int(1.6 * BH * _tiles(c)[0]), BH * nb * (nb + 1) // 2))
    idx = ms.alloc_index(dims, blk, max(col, int(0.6 * BH * nb * c["k_v"])), vcol, DEV)
    for t in idx.tensors.values():
        t.zero_()
    return idx


def _shard(t, world, layout, rank):
    """The rows of one ring worker: 64-token blocks dealt striped or zigzag."""
    B, H, N, d = t.shape
    nb = N // 64
    x = t.view(B, H, nb, 64, d)
    if layout == "striped":
        x = x[:, :, rank::world]
    else:
        n = nb // (2 * world)
        a, z = rank * n, (2 * world - 1 - rank) * n
        x = torch.cat([x[:, :, a:a + n], x[:, :, z:z + n]], 2)
    return x.reshape(B, H, N // world, d).contiguous()


def prepare(case, seed):
    c, kind = case, case["kind"]
    B, Hq, Hkv, N, d = c["B"], c["Hq"], c["Hkv"], c["N"], c["d"]
    k_v, k_s = c["k_v"], c["k_s"]
    q, k, v, do = _tensors(c, seed)
    dims = ms.make_dims(B, N, Hq, Hkv, d)
    s = dict(c=c, q=q, k=k, v=v, do=do, dims=dims)
    f32, i32 = dict(dtype=torch.float32, device=DEV), dict(dtype=torch.int32, device=DEV)
    if kind in ("estimate", "topp"):
        s["v_score"], s["s_score"] = torch.empty((B, Hq, N), **f32), torch.empty((B, Hq, N), **f32)
        s["v_idx"], s["s_idx"] = torch.empty((B, Hq, k_v), **i32), torch.empty((B, Hq, k_s), **i32)
        del s["v"], s["do"]
        return s
    vi, si = _lists(c, seed, q, k)
    if kind == "ring":
        W, layout = c["world"], c["layout"]
        rings = [ms.make_ring(W, c["rank"], t, layout, c["inner"] if c["inner"] < W else 0) for t in range(W)]
        shards = [ms.ring_shard(W, rings[t].inner, c["rank"], t) for t in range(W)]
        s["dims"] = dims = ms.make_dims(B, N // W, Hq, Hkv, d)
        s["q"], s["do"] = _shard(q, W, layout, c["rank"]), _shard(do, W, layout, c["rank"])
        s["k"] = [_shard(k, W, layout, t) for t in shards]
        s["v"] = [_shard(v, W, layout, t) for t in shards]
        s["rings"] = rings
        s["idx"] = [_index(dims, vi, si, r) for r in rings]
        s["ws_i"] = ms._workspace(max(ms.index_workspace_bytes(dims, k_v, k_s, r) for r in rings), DEV)
        vcol = max(x.struct.vcol_cap for x in s["idx"])
        s["vi"], s["si"] = vi, si
        n = (B, Hkv, N // W, d)
        s["dk"], s["dv"] = [torch.empty(n, **f32) for _ in rings], [torch.empty(n, **f32) for _ in rings]
    else:
        s["vi"], s["si"] = vi, si
        # the layers select anew on each pass: room for lists that differ a little from these
        room = 1.05 if kind in ("step", "prefill") else 1.0
        s["idx"] = _roomy_index(c, dims, vi, si) if kind == "index" else _index(dims, vi, si, None, room)
        s["ws_i"] = ms._workspace(ms.index_workspace_bytes(dims, k_v, k_s), DEV)
        vcol = s["idx"].struct.vcol_cap
        s["dk"], s["dv"] = torch.empty((B, Hkv, N, d), **f32), torch.empty((B, Hkv, N, d), **f32)
    if kind == "index":
        for name in ("q", "k", "v", "do", "dk", "dv"):
            del s[name]
        return s
    shape = s["q"].shape
    s["out"] = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    s["lse"] = torch.empty(shape[:-1], **f32)
    s["o32"] = torch.empty(shape, **f32) if kind in ("step", "ring") or c.get("o32") else None
    s["ws_f"] = ms._workspace(ms.attn_fwd_workspace_bytes(dims), DEV)
    if kind in ("step", "bwd", "ring"):
        s["dq"] = torch.empty(shape, **f32)
        s["ws_b"] = ms._workspace(ms.attn_bwd_workspace_bytes(dims, vcol), DEV)
    else:
        del s["dk"], s["dv"], s["do"]
    if kind in ("fwd", "bwd"):
        ms.build_index(dims, vi, si, s["idx"], workspace=s["ws_i"])
    if kind == "bwd":
        ms.attn_fwd(dims, q, k, v, s["idx"], out=s["out"], lse=s["lse"], out_f32=s["o32"], workspace=s["ws_f"])
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    c, dims = s["c"], s["dims"]
    kind = c["kind"]
    if kind == "estimate":
        ms.estimate(dims, s["q"], s["k"], LAST_Q, c["k_v"], c["k_s"], s["v_idx"], s["s_idx"], s["v_score"],
                    s["s_score"])
        return {n: s[n] for n in ("v_idx", "s_idx", "v_score", "s_score")}
    if kind == "topp":
        vi, si, vc, sc = ms.estimate_topp(dims, s["q"], s["k"], LAST_Q, c["p"], c["p"], c["k_v"], c["k_s"],
                                          s["v_score"], s["s_score"])
        return dict(v_idx=vi, s_idx=si, v_cnt=vc, s_cnt=sc, v_score=s["v_score"], s_score=s["s_score"])
    if kind == "index":
        return dict(ms.build_index(dims, s["vi"], s["si"], s["idx"], workspace=s["ws_i"]).tensors)
    if kind == "ring":
        last = len(s["rings"]) - 1
        for t, ring in enumerate(s["rings"]):
            ms.build_index(dims, s["vi"], s["si"], s["idx"][t], ring, workspace=s["ws_i"])
            ms.attn_fwd_merge(dims, s["q"], s["k"][t], s["v"][t], s["idx"][t], s["o32"], s["lse"],
                              s["out"] if t == last else None, t == 0, workspace=s["ws_f"])
        for t in range(last + 1):
            ms.attn_bwd(dims, s["q"], s["k"][t], s["v"][t], s["out"], s["do"], s["lse"], s["idx"][t], s["dq"],
                        s["dk"][t], s["dv"][t], t > 0, s["o32"], workspace=s["ws_b"], reuse_qrows=t > 0)
        return dict(out=s["out"], lse=s["lse"], dq=s["dq"], dk=s["dk"], dv=s["dv"])
    if kind in ("step", "prefill"):
        vi, si = ms.estimate(dims, s["q"], s["k"], LAST_Q, c["k_v"], c["k_s"], s["vi"], s["si"])
        ms.build_index(dims, vi, si, s["idx"], workspace=s["ws_i"])
    if kind != "bwd":
        ms.attn_fwd(dims, s["q"], s["k"], s["v"], s["idx"], out=s["out"], lse=s["lse"], out_f32=s["o32"],
                    workspace=s["ws_f"])
    if kind in ("fwd", "prefill"):
        return dict(out=s["out"], lse=s["lse"], **({"o32": s["o32"]} if s["o32"] is not None else {}))
    ms.attn_bwd(dims, s["q"], s["k"], s["v"], s["out"], s["do"], s["lse"], s["idx"], s["dq"], s["dk"], s["dv"],
                out_f32=s["o32"], workspace=s["ws_b"])
    grads = dict(dq=s["dq"], dk=s["dk"], dv=s["dv"])
    return grads if kind == "bwd" else dict(out=s["out"], lse=s["lse"], **grads)


# ---------------------------------------------------------------- floors, tolerances
def _tiles(c):
    """Selected 64 x 64 tiles per head and their number of block-diagonals, nearly."""
    nb = c["N"] // 64
    if c.get("spread"):
        D = (c["k_s"] - FAR) / 64 + 1 + 2 * FAR
    elif c.get("slash"):
        D = 1.3 * c["k_s"] / 64 + 1     # a run, its ragged end and some far ones
    else:
        D = nb * (1 - math.exp(-2.0 * c["k_s"] / c["N"] * 64))   # random offsets
    D = min(nb, D)
    return D * nb - D * D / 2, D


def work(case):
    c, kind = case, case["kind"]
    BH, BK, N, d = c["B"] * c["Hq"], c["B"] * c["Hkv"], c["N"], c["d"]
    T, D = _tiles(c)
    nb = N // 64
    cols = c["k_v"] * nb / 2 * (1 - D / nb) if c.get("spread") else 0
    fwd = 4.0 * d * BH * (4096 * T + 64 * cols)
    qb, kb = 2.0 * BH * N * d, 2.0 * BK * N * d       # bytes of a bf16 query-side / key-side tensor
    lists = 4.0 * BH * (c["k_v"] + c["k_s"])
    index = 4.0 * BH * (2 * T + cols + c["k_v"]) + 8.0 * BH * 3 * nb
    est = dict(bytes=kb + 2.0 * BH * LAST_Q * d + lists, flops=2.0 * BH * LAST_Q * N * d)
    lse = 4.0 * BH * N
    if kind in ("estimate", "topp"):
        return dict(bytes=est["bytes"] + 8.0 * BH * N, flops=est["flops"])
    if kind == "index":
        return dict(bytes=lists + index, flops=0)
    o = qb + lse + (2 * qb if c.get("o32") else 0)
    if kind == "fwd":
        return dict(bytes=qb + 2 * kb + index + o, flops=fwd)
    if kind == "prefill":
        return dict(bytes=qb + 2 * kb + o, flops=fwd + est["flops"])
    if kind == "bwd":
        return dict(bytes=2 * qb + 2 * kb + index + o + 2 * qb + 4 * kb, flops=2.5 * fwd)
    if kind == "ring":
        W = c["world"]
        return dict(bytes=(2 * qb + qb + lse + 2 * qb) / W + 6 * kb + lists, flops=3.5 * fwd / W)
    return dict(bytes=2 * qb + 2 * kb + qb + lse + 2 * qb + 4 * kb, flops=3.5 * fwd + est["flops"])


def tolerance(case):
    """About four times the measured distance from the exact results: 5e-7 for the fp32 scores, 1.7e-3 for a
    bf16 output, 4.5e-4 for gradients with Delta from the fp32 output and 4.2e-3 from the bf16 one.  A layer
    that selects its own lists may also swap a slash at a tie, which moves one head's rows by some percent."""
    kind = case["kind"]
    if kind == "index":
        return "exact"
    if kind in ("estimate", "topp"):
        return {"rel": 2e-6, "differ": 0.01}
    if kind in ("step", "prefill"):
        return {"rel": 1.5e-2}
    if kind == "bwd":
        return {"rel": 2e-3 if case["o32"] else 1.7e-2}
    return {"rel": 7e-3}


# ---------------------------------------------------------------- exact results
def _attention(c, q, k, v, do, vi, si):
    """Dense masked attention of every head and its gradients, 64 bits, rows in chunks."""
    B, Hq, N, d = c["B"], c["Hq"], c["N"], c["d"]
    G = Hq // c["Hkv"]
    nb = N // 64
    scale = 1 / math.sqrt(d)
    f64 = dict(dtype=torch.float64, device=DEV)
    out, dq = torch.empty((B, Hq, N, d), **f64), torch.empty((B, Hq, N, d), **f64)
    lse = torch.empty((B, Hq, N), **f64)
    dk, dv = torch.zeros((B, c["Hkv"], N, d), **f64), torch.zeros((B, c["Hkv"], N, d), **f64)
    pos = torch.arange(N, device=DEV)
    rows = max(64, min(N, (1 << 26) // N // 64 * 64))
    for b in range(B):
        for h in range(Hq):
            kk, vv, qq, gg = (t[b, i].double() for t, i in ((k, h // G), (v, h // G), (q, h), (do, h)))
            diag = torch.zeros(nb + 1, dtype=torch.bool, device=DEV)
            sl = si[b, h].long()
            diag[sl // 64] = True
            diag[(sl + 63) // 64] = True
            vert = torch.zeros(N, dtype=torch.bool, device=DEV)
            vert[vi[b, h].long()] = True
            for r0 in range(0, N, rows):
                r1 = min(N, r0 + rows)
                n = pos[r0:r1, None]
                m = pos[None, :r1]
                seen = (diag[(n // 64 - m // 64).clamp(min=0)] | vert[None, :r1]) & (m <= n)
                z = (qq[r0:r1] @ kk[:r1].T * scale).masked_fill_(~seen, -math.inf)
                l = torch.logsumexp(z, 1)
                p = torch.where(seen, torch.exp(z - l[:, None]), 0.0)
                o = p @ vv[:r1]
                out[b, h, r0:r1], lse[b, h, r0:r1] = o, l
                if c["kind"] in ("fwd", "prefill"):
                    continue
                dz = p * (gg[r0:r1] @ vv[:r1].T - (gg[r0:r1] * o).sum(1, keepdim=True))
                dq[b, h, r0:r1] = scale * (dz @ kk[:r1])
                dk[b, h // G, :r1] += scale * (dz.T @ qq[r0:r1])
                dv[b, h // G, :r1] += p.T @ gg[r0:r1]
    return out, lse, dq, dk, dv


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "index":
        return None
    if kind in ("estimate", "topp"):
        q, k, _, _ = _tensors(c, seed)
        G = c["Hq"] // c["Hkv"]
        sc = [_scores(q[b, h, c["N"] - LAST_Q:], k[b, h // G], 1 / math.sqrt(c["d"]), torch.float64)
              for b in range(c["B"]) for h in range(c["Hq"])]
        shape = (c["B"], c["Hq"], c["N"])
        got = dict(v_idx=None, s_idx=None, v_score=torch.stack([x[0] for x in sc]).view(shape),
                   s_score=torch.stack([x[1] for x in sc]).view(shape))
        return got if kind == "estimate" else dict(got, v_cnt=None, s_cnt=None)
    if float(c["N"]) ** 2 * c["B"] * c["Hq"] > 2e10:
        return None
    q, k, v, do = _tensors(c, seed)
    vi, si = _lists(c, seed, q, k, torch.float32 if kind in ("fwd", "bwd", "ring") else torch.float64)
    out, lse, dq, dk, dv = _attention(c, q, k, v, do, vi, si)
    if kind in ("fwd", "prefill"):
        return dict(out=out, lse=lse, **({"o32": out} if c.get("o32") else {}))
    if kind == "ring":
        mine = [_shard(t, c["world"], c["layout"], c["rank"]) for t in (out, lse[..., None], dq)]
        return dict(out=mine[0], lse=mine[1][..., 0], dq=mine[2], dk=None, dv=None)
    grads = dict(dq=dq, dk=dk, dv=dv)
    return grads if kind == "bwd" else dict(out=out, lse=lse, **grads)
