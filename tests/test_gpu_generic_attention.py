"""The float32-arithmetic attention of every geometry outside the bf16 /
head_dim 128 kernels, against the float64 oracle: head dims at and between the
kernel's 32-element blocks, rows that end inside a 4-element chunk, group sizes
that do not divide a tile, caches shorter than one tile, and chunk buffers whose
boundaries fall inside tiles (bit-identical to the contiguous cache)."""
import numpy as np
import pytest

import oracle
from oracle import bf16 as obf
from tests.gpu_util import empty, log, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")


def _sections(D):
    P = D // 2
    return (P // 3, P // 3, P - 2 * (P // 3))


def _make(dtype, D, G, Hkv, lens, rho, seed=0):
    from paper_2607_19547_amd import binding as b
    cs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    T, cs1 = int(cs[-1]), int(cs[1])
    n = T - cs1
    rng = np.random.default_rng(seed)

    def draw(*shape):
        x = rng.standard_normal(shape, dtype=np.float32)
        return obf.encode(x) if dtype == "bf16" else x

    x = dict(K=draw(1, Hkv, T, D), V=draw(1, Hkv, T, D), Q=draw(1, Hkv * G, n, D), KF=draw(1, Hkv, n, D),
             VF=draw(1, Hkv, n, D))
    sel = np.sort(rng.choice(n, max(1, int(np.ceil(rho * n))), replace=False)).astype(np.int32) + cs1
    return b.Geo(1, Hkv * G, Hkv, D, _sections(D), dtype, cs), cs, x, sel


def _call(geo, cs, dtype, x, sel, paged):
    from paper_2607_19547_amd import binding as b
    K, V = to_dev(x["K"], dtype), to_dev(x["V"], dtype)
    Q, KF, VF = (to_dev(x[n], dtype) for n in ("Q", "KF", "VF"))
    S = torch.from_numpy(sel).cuda()
    k, D = len(sel), x["K"].shape[-1]
    out = empty((1, Q.shape[1], k, D), dtype)
    lse = torch.empty((1, Q.shape[1], k), dtype=torch.float32, device="cuda")
    if paged:
        Kc, Vc = ([t[:, :, a:e].contiguous() for a, e in zip(cs[:-1], cs[1:])] for t in (K, V))
        b.selective_attend_scatter_paged(geo, Kc, Vc, 0, 1, S, k, Q, KF, VF, out, lse)
    else:
        b.selective_attend_scatter(geo, K, V, 0, 1, S, k, Q, KF, VF, out, lse)
    torch.cuda.synchronize()
    return to_host(out, dtype)[0], lse.cpu().numpy()[0]


def _dec(a, dtype):
    return obf.decode(a).astype(np.float64) if dtype == "bf16" else a.astype(np.float64)


CASES = [
    ("f32", 2, 1, 1, (3, 7), 1.0),                  # one short tile, rows of half a chunk
    ("f32", 16, 2, 2, (32, 32), 0.25),
    ("bf16", 6, 3, 2, (31, 1, 33, 40), 0.5),        # rows end inside a chunk; a one-token chunk
    ("f32", 50, 5, 1, (64, 100, 37), 0.4),
    ("f32", 64, 7, 3, (33, 95, 201), 0.3),          # group size that divides no tile
    ("bf16", 80, 4, 2, (130, 31, 200), 0.2),
    ("f32", 96, 1, 2, (65, 300), 0.1),
    ("f32", 128, 8, 2, (517, 700, 900), 0.05),      # many key tiles per wavefront
    ("bf16", 128, 7, 1, (64, 128, 65), 0.5),        # bf16 / 128 with a group outside the bf16 kernels
    ("bf16", 192, 2, 1, (40, 300, 90), 0.5),
    ("f32", 194, 1, 1, (40, 300, 91), 0.5),
    ("f32", 256, 2, 2, (70, 140), 0.3),
    ("bf16", 258, 2, 1, (70, 141), 0.3),
    ("f32", 512, 4, 1, (50, 203), 0.3),
]


@pytest.mark.parametrize("dtype,D,G,Hkv,lens,rho", CASES)
def test_generic_attention_against_oracle(dtype, D, G, Hkv, lens, rho):
    log(f"case generic attention {dtype} D={D} G={G} Hkv={Hkv} lens={lens} rho={rho}")
    geo, cs, x, sel = _make(dtype, D, G, Hkv, lens, rho)
    cs1 = int(cs[1])
    out, lse = _call(geo, cs, dtype, x, sel, False)
    kp = oracle.attention.scatter_rows(_dec(x["K"][0], dtype), _dec(x["KF"][0], dtype), sel, cs1)
    vp = oracle.attention.scatter_rows(_dec(x["V"][0], dtype), _dec(x["VF"][0], dtype), sel, cs1)
    o_ref, lse_ref = oracle.attention.attend_rows(_dec(x["Q"][0], dtype), kp, vp, sel, cs1)
    # float32 sums of D products and of T weights: errors of a few 2^-24 per
    # term, growing with the square root of the count; a bf16 result adds its
    # own rounding (at most 2^-9, 1.2e-3 in the mean square)
    err = rel_l2(_dec(out, dtype), o_ref)
    lerr = float(np.max(np.abs(lse - lse_ref)))
    log(f"  rel-L2 {err:.2e}, lse {lerr:.2e}")
    assert err <= (2e-3 if dtype == "bf16" else 2e-6) and lerr <= 4e-6 * max(1.0, float(np.abs(lse_ref).max()))
    if not (dtype == "bf16" and D == 128 and any(c % 64 for c in cs[:-1])):
        out_p, lse_p = _call(geo, cs, dtype, x, sel, True)
        assert np.array_equal(out_p, out) and np.array_equal(lse_p, lse)


# Caches of one and of two key tiles, either side of where a wavefront takes one
# row (24, 40 and 64 tokens for D up to 128, 384 and beyond), and the instances
# for 10, 12 and 16 blocks of the head dimension.
@pytest.mark.parametrize("dtype,D,G,Hkv,lens", [("f32", 2, 3, 1, (1, 1)), ("f32", 128, 4, 1, (5, 19)), ("f32", 128, 4, 1, (5, 20)),
                                                ("bf16", 64, 3, 2, (1, 23)), ("f32", 130, 3, 2, (5, 35)), ("f32", 130, 3, 2, (5, 36)),
                                                ("bf16", 384, 2, 2, (20, 20)), ("bf16", 384, 2, 2, (20, 21)), ("f32", 512, 2, 2, (1, 63)),
                                                ("f32", 512, 2, 2, (1, 64)), ("bf16", 386, 7, 1, (16, 15, 33)), ("bf16", 386, 7, 1, (16, 15, 34)),
                                                ("bf16", 318, 2, 1, (30, 34)), ("f32", 322, 1, 2, (30, 93)), ("f32", 384, 2, 1, (70, 141))])
def test_short_caches_and_wide_rows(dtype, D, G, Hkv, lens):
    test_generic_attention_against_oracle(dtype, D, G, Hkv, lens, 0.6)


@pytest.mark.parametrize("dtype,D,G", [("f32", 128, 2), ("bf16", 64, 3), ("f32", 20, 1)])
def test_rows_do_not_see_later_non_finite_rows(dtype, D, G):
    """Cache rows after a row's token never reach it, whatever they hold; the rows
    that see an infinite value get exactly that."""
    log(f"case non-finite rows {dtype} D={D} G={G}")
    geo, cs, x, sel = _make(dtype, D, G, 1, (100, 100), 0.4, seed=3)
    free = [t for t in range(120, 199) if t not in set(sel.tolist())]
    t_inf, t_nan, t_k = free[4], free[20], free[-4]
    clean, clean_lse = _call(geo, cs, dtype, x, sel, False)
    inf = np.uint16(0x7f80) if dtype == "bf16" else np.float32(np.inf)
    nan = np.uint16(0x7fc0) if dtype == "bf16" else np.float32(np.nan)
    x["V"][0, 0, t_inf, 5] = inf
    x["V"][0, 0, t_nan, :] = nan
    x["K"][0, 0, t_k, :] = nan
    for paged in (False, True):
        out, lse = _call(geo, cs, dtype, x, sel, paged)
        got, want = _dec(out, dtype), _dec(clean, dtype)
        a, m, z = sel < t_inf, (sel > t_inf) & (sel < t_nan), sel > t_nan
        assert a.any() and m.any() and z.any()
        # (tiles are summed in the same order: the same bits)
        assert np.array_equal(out[:, a], clean[:, a]) and np.array_equal(lse[:, sel < t_k], clean_lse[:, sel < t_k])
        assert np.all(np.isposinf(got[:, m, 5])) and np.array_equal(np.delete(got[:, m], 5, 2), np.delete(want[:, m], 5, 2))
        assert np.all(np.isnan(got[:, z]))


@pytest.mark.parametrize("dtype,D,G", [("f32", 128, 2), ("bf16", 64, 3), ("f32", 258, 1), ("f32", 16, 4)])
def test_nan_scores_reach_the_log_sum_exp(dtype, D, G):
    """A query of NaN, and a tile of NaN keys that is all one wavefront sees: the
    rows' results and log-sum-exps are NaN, and every other row keeps its bits."""
    log(f"case NaN scores {dtype} D={D} G={G}")
    geo, cs, x, sel = _make(dtype, D, G, 1, (96, 160), 0.5, seed=5)
    cs1 = int(cs[1])
    clean, clean_lse = _call(geo, cs, dtype, x, sel, False)
    nan = np.uint16(0x7fc0) if dtype == "bf16" else np.float32(np.nan)
    q_nan = int(sel[3])
    assert q_nan < 128 and (sel >= 160).any() and (sel < 128).sum() > 4
    x["Q"][0, 0, q_nan - cs1, 0] = nan
    x["K"][0, 0, 128:160, :] = nan  # (32-key tiles, eight wavefronts: the fifth one's only tile)
    x["KF"][0, 0, 128 - cs1:160 - cs1, :] = nan
    for paged in (False, True):
        out, lse = _call(geo, cs, dtype, x, sel, paged)
        got = _dec(out, dtype)
        bad = np.zeros(lse.shape, bool)
        bad[:, sel >= 128] = True
        bad[0, sel == q_nan] = True
        assert np.isnan(lse[bad]).all(), lse[bad][~np.isnan(lse[bad])]
        assert np.isnan(got[bad]).all()
        assert np.array_equal(lse[~bad], clean_lse[~bad]) and np.array_equal(out[~bad], clean[~bad])
