"""The composition path's workloads as measurable cases.

A case is a dict of plain values: the operation, the cache's geometry and the
options of the call.  `prepare` makes on the GPU what a user's program holds
before the call (caches, fresh rows, offsets, outputs, workspaces), `run` is
one pass through the public entry points of the package, `exact` is the same
result in float64 from plain torch.

Operations (`op`):
  rebase   compose_rebase_k[_paged]: every stored key turned by its chunk's offset
  tokens   compose_rebase_k_tokens[_paged]: scalar re-basing, an offset per token
  select   score_deviation_topk[_paged]: deviation scores and the top-rho selection
  attend   selective_attend_scatter[_noalloc][_rope][_paged] of given selected rows
  compose  the whole chain: rebase, select, attention layer by layer

Geometry is Qwen2.5-VL-3B's (16 query / 2 KV heads, head dim 128, sections
16/24/24, base 1e6) in bf16 unless a case says otherwise; chunks are 2,048
tokens (8 x 16 x 16 patches) where the cache is not ragged.  In use a stored
key is a post-rotary activation and a fresh row is the same row recomputed
under its new context, so a fresh key is the stored key at its global
coordinate plus noise whose scale differs from token to token (log-normal).
"""
import math

import numpy as np
import torch

from paper_2607_19547_amd import binding as cs

GRID = (8, 16, 16)  # a chunk's patches (t, h, w)
BASE = 1.0e6
QWEN = dict(q_heads=16, kv_heads=2, dim=128, dtype="bf16")


def _case(op, tokens, chunks, layers=1, rho=0.0, ragged=False, paged=False, rope=False, call="layer", **geometry):
    c = dict(op=op, layers=layers, tokens=tokens, chunks=chunks, ragged=ragged, paged=paged, rope=rope, rho=rho,
             call=call)
    c.update(QWEN)
    c.update(geometry)
    return c


def listed():
    return [
        # The smallest composition (the "tiny" workload: 64 tokens, one layer,
        # float32, head dim 16): launches and latency, generic kernels.
        dict(_case("compose", 64, 2, rho=0.25, q_heads=4, kv_heads=2, dim=16, dtype="f32"), name="compose-tiny"),
        # Re-basing a short video's cache (8,192 tokens, 36 layers).
        dict(_case("rebase", 8192, 4, layers=36), name="rebase-8k"),
        # Re-basing a long video whose chunks stay in their own buffers, of
        # uneven lengths, the last one odd.
        dict(_case("rebase", 65501, 32, layers=36, ragged=True, paged=True), name="rebase-65k-paged"),
        # The scalar position policy (every token moves by its own offset).
        dict(_case("tokens", 65536, 32, layers=36), name="tokens-65k"),
        # Score and selection of the 65k-token composition.
        dict(_case("select", 65536, 32, layers=2, rho=0.1), name="select-65k"),
        # The same for an hour-long cache, with the larger repair fraction.
        dict(_case("select", 262144, 128, layers=2, rho=0.35), name="select-262k"),
        # One layer's repair on the headline cache: the dominant kernel.
        dict(_case("attend", 65536, 32, rho=0.1), name="layer-65k"),
        # Full later-chunk re-prefill (rho = 1) of one layer: the largest selection.
        dict(_case("attend", 32768, 16, rho=1.0), name="layer-32k-full"),
        # A small repair on chunk buffers with the rotary embedding fused in,
        # ragged chunks.
        dict(_case("attend", 32741, 16, rho=0.05, ragged=True, paged=True, rope=True), name="layer-32k-rope-paged"),
        # A float32 cache (fidelity runs at full precision) at model geometry.
        dict(_case("attend", 4096, 2, rho=0.25, dtype="f32"), name="layer-4k-f32"),
        # The whole composition of a short video: many small layer calls.
        dict(_case("compose", 8192, 4, layers=36, rho=0.1), name="compose-8k"),
        # The whole composition of a long video (65,536 tokens, 36 layers).
        dict(_case("compose", 65536, 32, layers=36, rho=0.1), name="compose-65k"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["rebase", "tokens", "select", "attend", "attend", "attend", "compose", "compose"])
    paged = rng.random() < 0.4
    ragged = rng.random() < 0.6
    # mostly model geometry; also other head counts, and float32 or another
    # head dim (the generic kernels)
    kind = rng.choice(["model", "model", "heads", "generic"])
    geometry = {}
    if kind == "heads":
        kv = rng.choice([1, 2, 4, 8])
        geometry = dict(kv_heads=kv, q_heads=kv * rng.choice([1, 2, 4, 8, 16]))
    elif kind == "generic":
        kv = rng.choice([1, 2, 3])
        geometry = dict(kv_heads=kv, q_heads=kv * rng.choice([1, 2, 4, 7]), dim=rng.choice([16, 64, 80, 128, 192]),
                        dtype=rng.choice(["f32", "f32", "bf16"]))
        if geometry["dim"] == 128:
            geometry["dtype"] = "f32"
    layers = rng.choice([1, 2, 4, 12, 36] if kind == "model" else [1, 2, 4, 12])
    rho = rng.choice([0.02, 0.05, 0.1, 0.2, 0.35, 0.5, 1.0])
    call = "layer"
    rope = False
    if op in ("rebase", "tokens"):
        top = 131072 if kind != "generic" else 32768
        tokens = _log_int(rng, 500, top)
    elif op == "select":
        layers, tokens = 2, _log_int(rng, 1000, 262144)
    elif op == "attend":
        layers = rng.choice([1, 1, 2, 4])
        tokens = _log_int(rng, 500, 65536 if kind != "generic" else 4096)
        if tokens > 16384 or kind == "generic":
            layers, rho = 1, min(rho, 0.35)
        rope = rng.random() < 0.3
        call = "batch" if layers > 1 and rng.random() < 0.5 else "layer"
        if call == "layer" and not paged and not rope and rng.random() < 0.25:
            call = "noalloc"
    else:
        tokens = _log_int(rng, 500, 32768 if kind != "generic" else 3000)
        rho = rng.choice([0.05, 0.1, 0.2, 0.35])
        if kind == "generic" or tokens > 12000:
            layers = min(layers, 2 if kind == "generic" else 4)
    if not ragged:
        tokens = max(256, tokens // 256 * 256)
    chunks = max(2, min(60, tokens // rng.choice([200, 700, 2048, 4096])))
    return _case(op, tokens, chunks, layers=layers, rho=rho, ragged=ragged, paged=paged, rope=rope, call=call,
                 **geometry)


# ------------------------------------------------------------------ geometry
def _mfma(case):
    return case["dtype"] == "bf16" and case["dim"] == 128


def _chunk_start(case):
    """Chunk starts: even chunks of whole 64-token blocks, or uneven ones (a
    paged bf16 cache keeps starts at multiples of 64); the last chunk takes
    what is left."""
    T, N = case["tokens"], case["chunks"]
    unit = 64 if case["paged"] and _mfma(case) else (1 if case["ragged"] else 32)
    w = np.array([4 + (5 * c) % 7 if case["ragged"] else 1 for c in range(N)], dtype=np.float64)
    start = [0]
    for c in range(1, N):
        s = int(T * w[:c].sum() / w.sum()) // unit * unit
        if s > start[-1]:
            start.append(s)
    return np.array(start + [T], dtype=np.int64)


def _sections(D):
    P = D // 2
    s0 = P // 4
    s1 = (P - s0) // 2
    return (s0, s1, P - s0 - s1)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _n_select(rho, n):
    return 0 if rho == 0 else min(n, math.ceil(rho * n - 1e-9))


def _sizes(case):
    start = _chunk_start(case)
    T, s1 = int(start[-1]), int(start[1])
    return start, T, s1, T - s1, _n_select(case["rho"], T - s1)


def _offsets(case, start):
    """(dt, dh, dw) per chunk: the timeline of consecutive chunks in a
    composition, any coordinate in a re-basing alone."""
    N = len(start) - 1
    off = np.zeros((N, 3), dtype=np.int32)
    if case["op"] == "rebase":
        r = np.random.RandomState(17 + N)
        off[:, 0] = r.randint(1, 100_001, size=N)
        off[:, 1:] = r.randint(-16, 17, size=(N, 2))
    else:
        off[:, 0] = 8 * np.arange(N)
    return off


def _local(start):
    """Local raster coordinates of every token, int32 [T, 3]."""
    j = np.concatenate([np.arange(b - a) for a, b in zip(start[:-1], start[1:])])
    _, h, w = GRID
    return np.stack([j // (h * w), (j // w) % h, j % w], axis=-1).astype(np.int32)


def _global(start, off):
    return _local(start) + np.repeat(off, np.diff(start), axis=0)


def _scalar_offsets(start):
    """Scalar re-basing: token j of the composed cache moves to (j, j, j)."""
    T = int(start[-1])
    return (np.arange(T, dtype=np.int32)[:, None] - _local(start)).astype(np.int32)


# ------------------------------------------------------------------ plain rotation
def _angles(case, moves):
    """cos and sin, float64 [T, D/2], of every token's move [T, 3]."""
    D = case["dim"]
    theta = BASE ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device="cuda") / D)
    axis = torch.repeat_interleave(torch.arange(3), torch.tensor(_sections(D))).cuda()
    phi = torch.from_numpy(np.ascontiguousarray(moves)).cuda().double()[:, axis] * theta
    return torch.cos(phi), torch.sin(phi)


def _rotate(x, cos, sin):
    """Rotary pairs (i, i + D/2) of x [..., T, D], in the tables' type."""
    a, b = x.to(cos.dtype).chunk(2, dim=-1)
    return torch.cat([a * cos - b * sin, a * sin + b * cos], dim=-1)


# ------------------------------------------------------------------ inputs
class _Draws:
    """The case's random tensors, from the seed alone (on the GPU)."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(1_000_003 * int(seed) + 11)

    def normal(self, shape, dtype):
        out = torch.empty(shape, dtype=dtype, device="cuda")
        for x in out:  # plane by plane: bounded float32 temporaries
            x.copy_(torch.randn(x.shape, generator=self.g, device="cuda"))
        return out

    def scales(self, n):
        return torch.randn(n, generator=self.g, device="cuda").exp_()

    def selection(self, n, k, s1):
        p = torch.randperm(n, generator=self.g, device="cuda")[:k]
        return (p.sort().values + s1).to(torch.int32)


def _fresh(draws, stored, scale, moved=None):
    """Recomputed rows of the later chunks: stored rows (re-based by `moved`)
    plus noise of the token's own scale."""
    out = torch.empty_like(stored, memory_format=torch.contiguous_format)
    for layer in range(stored.shape[0]):
        x = stored[layer].float() if moved is None else _rotate(stored[layer], *moved)
        z = torch.randn(x.shape, generator=draws.g, device="cuda")
        out[layer] = x + 0.1 * scale[:, None] * z
    return out


def _inputs(case, seed):
    """Everything the call reads, in the composed layout."""
    start, T, s1, n, k = _sizes(case)
    L, H, D, dt = case["layers"], case["kv_heads"], case["dim"], _dtype(case)
    d = _Draws(seed)
    x = {"k": d.normal((L, H, T, D), dt)}
    op = case["op"]
    if op == "select":
        layer = min(1, L - 1)
        x["kf"] = _fresh(d, x["k"][layer:layer + 1, :, s1:], d.scales(n))
    if op in ("attend", "compose"):
        x["v"] = d.normal((L, H, T, D), dt)
        x["q"] = d.normal((L, case["q_heads"], n, D), dt)
        scale = d.scales(n)
        moved = None
        if op == "compose":
            moves = np.repeat(_offsets(case, start), np.diff(start), axis=0)[s1:]
            moved = tuple(t.float() for t in _angles(case, moves))
        x["kf"] = _fresh(d, x["k"][:, :, s1:], scale, moved)
        x["vf"] = _fresh(d, x["v"][:, :, s1:], scale)
    if op == "attend":
        x["sel"] = d.selection(n, k, s1)
    return x


def _pages(case, x, start):
    """The cache as one buffer per chunk ([L][H][len][D] each, consecutive in
    one allocation) and the chunks' views of it."""
    L, H, _, D = x.shape
    flat = torch.empty(x.numel(), dtype=x.dtype, device="cuda")
    views = []
    for a, b in zip(start[:-1], start[1:]):
        v = flat[L * H * D * int(a):L * H * D * int(b)].view(L, H, int(b - a), D)
        v.copy_(x[:, :, int(a):int(b)])
        views.append(v)
    return flat, views


def _bytes(n):
    return torch.empty(max(1, n), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    start, T, s1, n, k = _sizes(case)
    L, Hq, D, dt = case["layers"], case["q_heads"], case["dim"], _dtype(case)
    geo = cs.Geo(L, Hq, case["kv_heads"], D, _sections(D), case["dtype"], start, BASE)
    x = _inputs(case, seed)
    s = {"case": case, "geo": geo, "k": x["k"], "n": n, "n_sel": k, "offsets": _offsets(case, start)}
    if "v" in x:
        s["v"] = x["v"]
    if case["paged"]:
        for name in ("k", "v"):
            if name in x:
                s[name], s[name + "_chunks"] = _pages(case, x.pop(name), start)
    for name in ("q", "kf", "vf", "sel"):
        if name in x:
            s[name] = x[name]
    op = case["op"]
    if op == "tokens":
        s["moves"] = torch.from_numpy(_scalar_offsets(start)).cuda()
    if op in ("select", "compose"):
        s["scores"] = torch.empty(n, dtype=torch.float32, device="cuda")
        s["sel"] = torch.empty(max(1, k), dtype=torch.int32, device="cuda")
    if op in ("attend", "compose"):
        s["out"] = torch.empty((L, Hq, k, D), dtype=dt, device="cuda")
        s["lse"] = torch.empty((L, Hq, k), dtype=torch.float32, device="cuda")
        per_call = L if case["call"] == "batch" else 1
        size = cs.selective_attend_scatter_rope_workspace if case["rope"] else cs.selective_attend_scatter_workspace
        s["ws"] = _bytes(size(geo, k, per_call))
        if case["rope"]:
            s["coords"] = torch.from_numpy(_global(start, s["offsets"])).cuda()
    return s


# ------------------------------------------------------------------ one pass
def _rebase(s):
    if "k_chunks" in s:
        cs.compose_rebase_k_paged(s["geo"], s["k_chunks"], s["offsets"])
    else:
        cs.compose_rebase_k(s["geo"], s["k"], s["offsets"])


def _select(s, k_fresh):
    layer = min(1, s["case"]["layers"] - 1)
    call, cache = (cs.score_deviation_topk_paged, s["k_chunks"]) if "k_chunks" in s else (cs.score_deviation_topk, s["k"])
    return call(s["geo"], cache, layer, k_fresh, s["case"]["rho"], s["scores"], s["sel"])


def _attend(s, n_sel):
    case, geo, L = s["case"], s["geo"], s["case"]["layers"]
    paged = "k_chunks" in s
    k, v = (s["k_chunks"], s["v_chunks"]) if paged else (s["k"], s["v"])
    step = L if case["call"] == "batch" else 1
    for a in range(0, L, step):
        if case["call"] == "noalloc":
            cs.selective_attend_scatter_noalloc(geo, k, v, a, a + step, s["sel"], n_sel, s["q"], s["kf"], s["vf"],
                                                s["out"], s["lse"])
        elif case["rope"]:
            f = cs.selective_attend_scatter_rope_paged if paged else cs.selective_attend_scatter_rope
            f(geo, k, v, a, a + step, s["sel"], n_sel, s["q"], s["kf"], s["vf"], s["coords"], s["out"], s["lse"],
              s["ws"])
        else:
            f = cs.selective_attend_scatter_paged if paged else cs.selective_attend_scatter
            f(geo, k, v, a, a + step, s["sel"], n_sel, s["q"], s["kf"], s["vf"], s["out"], s["lse"], s["ws"])


def run(s):
    op = s["case"]["op"]
    if op == "rebase":
        _rebase(s)
        return {"k": s["k"]}
    if op == "tokens":
        if "k_chunks" in s:
            cs.compose_rebase_k_tokens_paged(s["geo"], s["k_chunks"], s["moves"])
        else:
            cs.compose_rebase_k_tokens(s["geo"], s["k"], s["moves"])
        return {"k": s["k"]}
    if op == "select":
        n_sel = _select(s, s["kf"])
        return {"n_sel": n_sel, "scores": s["scores"], "sel": s["sel"]}
    if op == "attend":
        _attend(s, s["n_sel"])
        return {"k": s["k"], "v": s["v"], "out": s["out"], "lse": s["lse"]}
    _rebase(s)
    n_sel = _select(s, s["kf"][min(1, s["case"]["layers"] - 1)])
    _attend(s, n_sel)
    return {"n_sel": n_sel, "k": s["k"], "v": s["v"], "scores": s["scores"], "sel": s["sel"], "out": s["out"],
            "lse": s["lse"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    start, T, s1, n, k = _sizes(case)
    L, Hq, H, D = case["layers"], case["q_heads"], case["kv_heads"], case["dim"]
    e = 2 if case["dtype"] == "bf16" else 4
    op = case["op"]
    bytes_, flops = 0.0, 0.0
    if op in ("rebase", "tokens", "compose"):  # moved keys read and written; 6 flop per rotary pair
        moved = T if op != "compose" else n  # (a composition's first chunk stays where it is)
        bytes_ += 2.0 * L * H * moved * D * e + (12.0 * T if op == "tokens" else 0.0)
        flops += 3.0 * L * H * moved * D
    if op in ("select", "compose"):  # both keys of every candidate read; scores and indices written
        bytes_ += 2.0 * H * n * D * e + 4.0 * n + 4.0 * k
        flops += 3.0 * H * n * D
    if op in ("attend", "compose"):
        # the cache's other rows, the selected rows' fresh K, V and Q read; K and V rows and the results
        # written; two products over every visible key (the selection spreads evenly over the later chunks)
        bytes_ += L * (2.0 * H * (T - k) * D * e + 4.0 * H * k * D * e + 2.0 * Hq * k * D * e + 4.0 * Hq * k)
        flops += 4.0 * L * Hq * D * k * (s1 + T + 1) / 2.0
    return {"bytes": bytes_, "flops": flops}


# Relative errors: about four times what a pass shows against `exact` (re-based
# bf16 keys, one rounding of an exact value: 1.7e-3; a bf16 attention, which
# also rounds its probabilities: 2.3e-3; float32 attention over a few thousand
# keys: 1e-6; scores, float64 sums rounded once: 2.6e-8).
def tolerance(case):
    if case["op"] == "select":
        return {"rel": 1e-7, "max": 1e-6}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    if case["op"] in ("rebase", "tokens"):
        return {"rel": 7e-3, "max": 3e-2}
    return {"rel": 1e-2, "max": 2e-1}


# ------------------------------------------------------------------ float64 results
def _attend_exact(q, k, v, sel):
    """Causal attention of the selected rows, one query head, float64:
    q [n_sel, D], k and v [T, D], sel [n_sel] -> out [n_sel, D], lse [n_sel]."""
    D = q.shape[-1]
    out = torch.empty_like(q)
    lse = torch.empty(q.shape[0], dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // k.shape[0])
    kt = k.t().contiguous()
    pos = torch.arange(k.shape[0], device="cuda")
    for a in range(0, q.shape[0], step):
        t = sel[a:a + step].long()
        m = int(t[-1]) + 1
        sc = torch.mm(q[a:a + step], kt[:, :m]) / math.sqrt(D)
        sc.masked_fill_(pos[None, :m] > t[:, None], -math.inf)
        top = sc.amax(dim=1, keepdim=True)
        p = sc.sub_(top).exp_()
        tot = p.sum(dim=1, keepdim=True)
        out[a:a + step] = torch.mm(p, v[:m]) / tot
        lse[a:a + step] = (top + tot.log())[:, 0]
    return out, lse


def exact(case, seed):
    if case["op"] == "compose" and _mfma(case):
        return None  # its selection hangs on bf16 roundings; its steps are cases of their own
    start, T, s1, n, k = _sizes(case)
    dt = _dtype(case)
    op, D = case["op"], case["dim"]
    if work(case)["flops"] > 12e12:
        return None
    x = _inputs(case, seed)

    def laid(t):  # the composed cache in the layout that run() returns
        if not case["paged"]:
            return t
        return torch.cat([t[:, :, int(a):int(b)].reshape(-1) for a, b in zip(start[:-1], start[1:])])

    if op in ("rebase", "tokens"):
        moves = _scalar_offsets(start) if op == "tokens" else np.repeat(_offsets(case, start), np.diff(start), axis=0)
        cos, sin = _angles(case, moves)
        return {"k": laid(_rotate(x["k"], cos, sin))}
    res = {}
    if op == "compose":
        moves = np.repeat(_offsets(case, start), np.diff(start), axis=0)
        x["k"] = _rotate(x["k"], *_angles(case, moves)).to(dt)
        res["n_sel"] = None
    if op in ("select", "compose"):
        layer = min(1, case["layers"] - 1)
        kf = x["kf"][0] if op == "select" else x["kf"][layer]
        scores = (kf.double() - x["k"][layer, :, s1:].double()).square().sum(dim=(0, 2)).sqrt()
        res.update(scores=scores, sel=None)
        if op == "select":
            return dict(res, n_sel=None)
        x["sel"] = (torch.sort(scores.float(), descending=True, stable=True).indices[:k].sort().values + s1)
    sel = x["sel"].long()
    q, kf, vf = (x[name][:, :, sel - s1] for name in ("q", "kf", "vf"))
    if case["rope"]:  # rotated at the selected tokens' global coordinates and stored in the cache's type
        cos, sin = _angles(case, _global(start, _offsets(case, start))[sel.cpu().numpy()])
        q, kf = _rotate(q, cos, sin).to(dt), _rotate(kf, cos, sin).to(dt)
    x["k"][:, :, sel] = kf
    x["v"][:, :, sel] = vf
    L, Hq = case["layers"], case["q_heads"]
    group = Hq // case["kv_heads"]
    out = torch.empty((L, Hq, k, D), dtype=torch.float64, device="cuda")
    lse = torch.empty((L, Hq, k), dtype=torch.float64, device="cuda")
    for layer in range(L):
        for h in range(Hq):
            out[layer, h], lse[layer, h] = _attend_exact(q[layer, h].double(), x["k"][layer, h // group].double(),
                                                         x["v"][layer, h // group].double(), sel)
    res.update(k=laid(x["k"].double()), v=laid(x["v"].double()), out=out, lse=lse)
    return res
