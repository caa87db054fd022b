"""Runs of key pieces (the attention launch's items): the run descriptors in the
plan take every r-th piece of each row tile and cover its key tiles once, short
runs come last, and the outputs (one partial per run, none where a run is a whole
row tile) match float64 attention; fresh, kept and batched plans give the same
bits."""
import math

import numpy as np
import pytest

from tests.gpu_util import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

HDR = 32
# G, Hkv, T, n_sel, whole: about one item per CU, a few per CU, whole row tiles
CASES = [(8, 2, 32768, 1536, False), (4, 4, 16384, 1434, False), (1, 8, 12000, 1500, False), (16, 1, 40000, 2100, False),
         (32, 1, 9000, 1000, False), (8, 8, 3000, 2700, True), (32, 2, 4000, 2500, True)]


@pytest.fixture(scope="module", autouse=True)
def _gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")


def _reference(q, k, v, sel, h, g):
    t = sel.long()
    s = torch.mm(q[h].double(), k[h // g].double().t()) / math.sqrt(128)
    s.masked_fill_(torch.arange(k.shape[1], device="cuda")[None] > t[:, None], -math.inf)
    return torch.mm(torch.softmax(s, dim=1), v[h // g].double()), torch.logsumexp(s, dim=1)


@pytest.mark.parametrize("G,hkv,T,k,whole", CASES)
def test_runs_cover_every_piece_and_match(G, hkv, T, k, whole):
    from paper_2607_19547_amd import binding as b
    log(f"case runs G={G} Hkv={hkv} T={T} k={k}")
    cs1, L, hq, D = T // 16, 2, G * hkv, 128
    n = T - cs1
    geo = b.Geo(L, hq, hkv, D, (16, 24, 24), "bf16", np.array([0, cs1, T], np.int64))
    gen = torch.Generator(device="cuda").manual_seed(T + k)
    r = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(torch.bfloat16)
    K, V, Q, KF, VF = r(L, hkv, T, D), r(L, hkv, T, D), r(L, hq, n, D), r(L, hkv, n, D), r(L, hkv, n, D)
    sel = (torch.randperm(n, device="cuda", generator=gen)[:k].sort().values + cs1).to(torch.int32)
    out = torch.empty((L, hq, k, D), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty((L, hq, k), dtype=torch.float32, device="cuda")
    ws = torch.zeros(b.selective_attend_scatter_workspace(geo, k, L), dtype=torch.uint8, device="cuda")
    b.selective_attend_scatter(geo, K, V, 0, 1, sel, k, Q, KF, VF, out, lse, ws)
    torch.cuda.synchronize()
    plan = ws.view(torch.int32).cpu().numpy()
    hdr = plan[:HDR]
    S, per_q, rs, off, run, n_runs, ro = (int(hdr[i]) for i in (9, 12, 13, 14, 15, 25, 26))
    nt = int(hdr[17])
    nu, nsp = plan[HDR:HDR + nt], plan[HDR + nt:HDR + 2 * nt]
    assert run >= 2 and rs == run * S, "the case is one with runs of several pieces"
    assert (rs >= nu[0]) == whole
    pieces = plan[off:off + 4 * per_q].reshape(per_q, 4)
    runs = plan[ro:ro + 4 * n_runs].reshape(n_runs, 4)
    lead = sorted((int(i), int(y), int(z), int(min(z + rs, nu[i]))) for i, y, z, _ in pieces if (int(y) >> 16) % run == 0)
    assert sorted(tuple(map(int, x)) for x in runs) == lead and ro != off
    kvq = hkv // int(hdr[8])
    assert n_runs == sum(-(-int(p) // run) for p in nsp) * kvq
    covered = {}
    for i, y, z, e in lead:
        covered.setdefault((i, y & 0xffff), []).append((z, e))
    for (i, _), spans in covered.items():
        spans.sort()
        assert spans[0][0] == 0 and spans[-1][1] == nu[i] and all(x[1] == y[0] for x, y in zip(spans, spans[1:]))
    lens = [int(e - z) for _, _, z, e in runs]
    tail = lens if n_runs * int(hdr[8]) <= 512 else lens[n_runs - (n_runs + 3) // 4:]
    shift = 0
    while (rs >> shift) > 255:
        shift += 1
    assert all(min(x >> shift, 255) >= min(y >> shift, 255) for x, y in zip(tail, tail[1:])), "longest first"
    # the second layer keeps the plan; a batched call over both layers on a fresh workspace gives the same bits
    b.selective_attend_scatter(geo, K, V, 1, 2, sel, k, Q, KF, VF, out, lse, ws)
    out2, lse2 = torch.empty_like(out), torch.empty_like(lse)
    b.selective_attend_scatter(geo, K, V, 0, L, sel, k, Q, KF, VF, out2, lse2, torch.zeros_like(ws))
    torch.cuda.synchronize()
    assert int(ws.view(torch.int32)[24]) == 1 and torch.equal(out, out2) and torch.equal(lse, lse2)
    rows = sel.long() - cs1
    for layer, h in ((0, 0), (1, hq - 1)):
        o, l = _reference(Q[layer][:, rows], K[layer], V[layer], sel, h, G)
        err = float((out[layer, h].double() - o).norm() / o.norm())
        lerr = float((lse[layer, h].double() - l).abs().max())
        log(f"  run {run} x {S} tiles, {n_runs} items per queue: layer {layer} head {h} rel-L2 {err:.2e}, lse {lerr:.2e}")
        # bf16 probabilities and one bf16 rounding of the result: 2^-9 each at most, in the mean square below 3e-3
        assert err <= 5e-3 and lerr <= 1e-2


# Row tiles of 32 / G x 8 rows; short caches, so that every item is a whole row
# tile: just fewer items than the 256 workgroups (nothing is claimed), as many,
# and just more, with one queue per call, per KV head and per XCD.
@pytest.mark.parametrize("G,hkv,L,k", [(32, 1, 3, 680), (32, 1, 2, 1021), (32, 1, 3, 681), (32, 3, 1, 680), (32, 3, 1, 681),
                                       (32, 4, 1, 504), (32, 4, 1, 512), (32, 4, 1, 513), (32, 8, 1, 255), (32, 8, 1, 257),
                                       (16, 2, 1, 1020), (8, 2, 1, 33), (32, 1, 1, 1)])
def test_items_around_one_per_workgroup(G, hkv, L, k):
    from paper_2607_19547_amd import binding as b
    log(f"case one item each G={G} Hkv={hkv} L={L} k={k}")
    T, cs1, hq, D = 1024, 2, G * hkv, 128
    n = T - cs1
    geo = b.Geo(L, hq, hkv, D, (16, 24, 24), "bf16", np.array([0, cs1, T], np.int64))
    gen = torch.Generator(device="cuda").manual_seed(G * 1000 + k)
    r = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(torch.bfloat16)
    K, V, Q, KF, VF = r(L, hkv, T, D), r(L, hkv, T, D), r(L, hq, n, D), r(L, hkv, n, D), r(L, hkv, n, D)
    sel = (torch.randperm(n, device="cuda", generator=gen)[:k].sort().values + cs1).to(torch.int32)
    got = []
    for per in (1, L):  # a call per layer; one call
        k2, v2 = K.clone(), V.clone()
        out = torch.full((L, hq, k, D), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.zeros(b.selective_attend_scatter_workspace(geo, k, per), dtype=torch.uint8, device="cuda")
        for layer in range(0, L, per):
            b.selective_attend_scatter(geo, k2, v2, layer, layer + per, sel, k, Q, KF, VF, out, None, ws)
        got.append(out)
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])
    for layer in range(L):
        for h in (0, hq - 1):
            want, _ = _reference(Q[layer][:, sel.long() - cs1], k2[layer], v2[layer], sel, h, G)
            # bf16 probabilities and outputs: 2^-9 each, relative to the row
            err = (got[0][layer, h].double() - want).norm() / want.norm()
            assert err <= 5e-3, (layer, h, float(err))


# More items than workgroups in two, four and eight queues; short caches, so that
# every item is a whole row tile.
@pytest.mark.parametrize("G,hkv,L,k", [(32, 8, 1, 400), (32, 8, 3, 777), (16, 4, 2, 1000), (32, 2, 3, 1020)])
def test_workgroups_claim_only_where_positions_are_left(G, hkv, L, k):
    """Every position is taken once, and a workgroup that finds its queue empty
    leaves the other queues' counters alone unless they have positions left: one
    failed claim per workgroup on its own queue, and as many again for the rare
    claim that comes second (a claim on every queue would be nq per workgroup)."""
    from paper_2607_19547_amd import binding as b
    log(f"case claims G={G} Hkv={hkv} L={L} k={k}")
    T, cs1, hq, D = 1024, 2, G * hkv, 128
    n = T - cs1
    geo = b.Geo(L, hq, hkv, D, (16, 24, 24), "bf16", np.array([0, cs1, T], np.int64))
    gen = torch.Generator(device="cuda").manual_seed(G * 1000 + k)
    r = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(torch.bfloat16)
    K, V, Q, KF, VF = r(L, hkv, T, D), r(L, hkv, T, D), r(L, hq, n, D), r(L, hkv, n, D), r(L, hkv, n, D)
    sel = (torch.randperm(n, device="cuda", generator=gen)[:k].sort().values + cs1).to(torch.int32)
    out = torch.full((L, hq, k, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.zeros(b.selective_attend_scatter_workspace(geo, k, L), dtype=torch.uint8, device="cuda")
    b.selective_attend_scatter(geo, K, V, 0, L, sel, k, Q, KF, VF, out, None, ws)
    torch.cuda.synchronize()
    hdr = ws[:4 * HDR].view(torch.int32).tolist()
    nq, positions = hdr[8], hdr[25] * L
    assert nq * positions > 256, "the case is one with items left to claim"
    assert all(positions <= c for c in hdr[:nq])
    assert sum(hdr[:nq]) <= nq * positions + 2 * 256, hdr[:8]
    for layer in (0, L - 1):
        for h in (0, hq - 1):
            want, _ = _reference(Q[layer][:, sel.long() - cs1], K[layer], V[layer], sel, h, G)
            err = (out[layer, h].double() - want).norm() / want.norm()
            assert err <= 5e-3, (layer, h, float(err))  # bf16 probabilities and outputs: 2^-9 each


def _estimates(nu, S, hkv):
    """The plan's estimate of a layer launch, in key tiles, for runs of r = 1 .. 8
    pieces (float64; lengths in buckets of 2^shift as the plan counts them)."""
    nq = 8 if hkv % 8 == 0 else hkv if hkv in (1, 2, 4) else 1
    kvq, g, res = hkv // nq, 256 // nq, []
    for r in range(1, min(8, -(-nu[0] // S)) + 1):
        rs = min(r * S, nu[0])
        shift = 0
        while (rs >> shift) > 255:
            shift += 1
        lens = sorted((x for v in nu for x in [rs] * (v // rs) + [v % rs] * (v % rs > 0) for _ in range(kvq)), reverse=True)
        at = [min((((x >> shift) + 1) << shift) - 1, rs) for x in lens]
        n, full = len(lens), sum(v // rs for v in nu) * kvq
        rounds = min(full // g, (n - 1) // g) if n > 2 * g else 0
        mean = t = (sum(nu) * hkv + 7.0 * n * nq) / 256
        if n > 2 * g:
            last = nu[3 * len(nu) // 4] if kvq == 1 and rs == nu[0] <= 128 else rs
            t = max(1.05 * mean, (0.95 if kvq == 1 else 1.0) * (0.75 * mean + last + 7.0))
        if n - rounds * g <= 2 * g:
            at = at[rounds * g:]
            t = max(t, rounds * (rs + 7.0) + max([at[0] + 7.0] + [at[g - 1 - k] + at[g + k] + 14.0 for k in range(len(at) - g)]))
        res.append(t + 0.0065 * (n * nq // hkv - sum(v <= rs for v in nu)) * hkv)
    return res


# Whole row tiles of seven heads in one queue, and of two heads that fit an L2 or
# do not; items paired in one round and a bit, lengths beyond 255 tiles among them;
# a share per CU just above and below two pieces of 288 tiles.
@pytest.mark.parametrize("G,hkv,T,k", [(4, 7, 16384, 5376), (4, 7, 12288, 5760), (8, 2, 6000, 5625), (8, 2, 16384, 8192),
                                       (4, 8, 2048, 1920), (8, 8, 3000, 1000), (1, 8, 65536, 1000), (8, 1, 6000, 2000),
                                       (8, 2, 65536, 6349), (8, 2, 68000, 6375), (1, 16, 3000, 2800)])
def test_run_length_is_the_estimates_best(G, hkv, T, k):
    from paper_2607_19547_amd import binding as b
    log(f"case run length G={G} Hkv={hkv} T={T} k={k}")
    cs1, hq, D = T // 16, G * hkv, 128
    n = T - cs1
    geo = b.Geo(1, hq, hkv, D, (16, 24, 24), "bf16", np.array([0, cs1, T], np.int64))
    z = lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
    K, V, Q, KF, VF = z(1, hkv, T, D), z(1, hkv, T, D), z(1, hq, n, D), z(1, hkv, n, D), z(1, hkv, n, D)
    sel = np.sort(np.random.default_rng(T + k).choice(n, k, replace=False)) + cs1
    out = torch.empty((1, hq, k, D), dtype=torch.bfloat16, device="cuda")
    ws = torch.zeros(b.selective_attend_scatter_workspace(geo, k, 1), dtype=torch.uint8, device="cuda")
    b.selective_attend_scatter(geo, K, V, 0, 1, torch.from_numpy(sel.astype(np.int32)).cuda(), k, Q, KF, VF, out, None, ws)
    torch.cuda.synchronize()
    plan = ws.view(torch.int32).cpu().numpy()
    S, run, nt = int(plan[9]), int(plan[15]), int(plan[17])
    want = _estimates([int(v) for v in plan[HDR:HDR + nt]], S, hkv)
    log(f"  {nt} row tiles, S {S}, run {run}, estimates {[round(x, 1) for x in want]}")
    want[0] *= 0.99  # (runs of several pieces are taken where they gain 1%)
    assert want[run - 1] <= min(want) * (1 + 1e-5)  # (float32 sums of a few terms: 2^-22 each)


@pytest.mark.parametrize("where", ["descriptor", "count", "offset", "checksum"])
def test_damaged_runs_are_replanned(where):
    """The second pair of checksum words covers the runs: recomputed on the host, and
    a kept plan with one int of a run descriptor, the count of runs, the offset of
    their descriptors or the sum itself changed is made again, with the outputs
    of an undamaged one."""
    from paper_2607_19547_amd import binding as b
    log(f"case damaged runs: {where}")
    G, hkv, T, k, L, D = 1, 8, 12000, 1500, 2, 128
    cs1 = T // 16
    n, hq = T - cs1, G * hkv
    geo = b.Geo(L, hq, hkv, D, (16, 24, 24), "bf16", np.array([0, cs1, T], np.int64))
    gen = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(torch.bfloat16)
    K, V, Q, KF, VF = r(L, hkv, T, D), r(L, hkv, T, D), r(L, hq, n, D), r(L, hkv, n, D), r(L, hkv, n, D)
    sel = (torch.randperm(n, device="cuda", generator=gen)[:k].sort().values + cs1).to(torch.int32)
    out, lse = torch.zeros((L, hq, k, D), dtype=torch.bfloat16, device="cuda"), torch.zeros((L, hq, k), device="cuda")
    ws = torch.zeros(b.selective_attend_scatter_workspace(geo, k, 1), dtype=torch.uint8, device="cuda")
    call = lambda layer, o, l, w: b.selective_attend_scatter(geo, K, V, layer, layer + 1, sel, k, Q, KF, VF, o, l, w)
    call(0, out, lse, ws)
    torch.cuda.synchronize()
    plan = ws.view(torch.int32)
    host = plan.cpu().numpy()
    per_q, off, run, n_runs, ro = (int(host[i]) for i in (12, 14, 15, 25, 26))
    assert run >= 2 and ro != off, "the case is one with runs of several pieces"
    idx = np.concatenate([[25, 26], np.arange(ro, ro + 4 * n_runs)]).astype(np.uint64)
    v, m32 = host.view(np.uint32)[idx.astype(np.int64)].astype(np.uint64), np.uint64(0xFFFFFFFF)
    c1 = int(np.sum((v * (2 * idx + 1)) & m32) & m32)
    c2 = int(np.sum((((v ^ ((idx * 0x9E3779B9) & m32)) * 0x85EBCA6B) & m32) + idx) & m32)
    assert (c1, c2) == (int(np.uint32(host[27])), int(np.uint32(host[28])))
    call(1, out, lse, ws)
    torch.cuda.synchronize()
    assert int(plan[24]) == 1, "undamaged, the plan is kept"
    want_out, want_lse = out[1].clone(), lse[1].clone()
    if where == "descriptor":
        plan[ro + 4 * (n_runs // 2) + 3] -= 1  # a run that ends a key tile early
    elif where == "count":
        plan[25] -= 1
    elif where == "offset":
        plan[26] = off  # the piece descriptors, also within the plan
    else:
        plan[28] += 1
    out[1].zero_()
    lse[1].zero_()
    call(1, out, lse, ws)
    torch.cuda.synchronize()
    assert int(plan[24]) == 0, "made again"
    assert torch.equal(out[1], want_out) and torch.equal(lse[1], want_lse)
