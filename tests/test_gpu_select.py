"""The top-rho selection on scores of every shape that its kernels treat
differently, against the oracle's ranking of the same scores: candidate counts
at the edges of the ranked and the radix form, of a wavefront's groups and of
the shared compaction; scores that crowd into one first-digit bin (its list
overflows), that differ only in the last bits, and ties cut by index.  A cache
of zeros with fresh keys (s, 0) has the scores |s| exactly."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu(built_lib):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")


def _scores(kind, n, rng):
    if kind == "spread":
        return np.exp(rng.standard_normal(n))
    if kind == "equal":
        return np.full(n, 3.25)
    if kind == "few":  # heavy ties over four octaves
        return rng.choice([0.0, 0.5, 1.0, 1.5, 7.0], n)
    if kind == "close":  # one first-digit bin, every low digit
        return 1.0 + rng.integers(0, 1 << 20, n) * 2.0 ** -23
    return np.where(rng.random(n) < 0.5, 2.0 + rng.integers(0, 64, n) * 2.0 ** -22, np.exp(3 * rng.standard_normal(n)))


SIZES = [1, 3, 64, 65, 511, 512, 513, 1025, 4096, 4097, 8191, 16385, 65535, 65537, 200003]


@pytest.mark.parametrize("kind", ["spread", "equal", "few", "close", "mixed"])
@pytest.mark.parametrize("n", SIZES)
def test_selection_of_given_scores(n, kind):
    from paper_2607_19547_amd import binding as b
    log(f"case selection n={n} {kind}")
    cs1 = 5
    geo = b.Geo(1, 1, 1, 2, (1, 0, 0), "f32", [0, cs1, cs1 + n])
    want = _scores(kind, n, np.random.default_rng(n)).astype(np.float32)
    K = torch.zeros(1, 1, cs1 + n, 2, device="cuda")
    KF = torch.zeros(1, n, 2, device="cuda")
    KF[0, :, 0] = torch.from_numpy(want).cuda()
    buf = torch.empty(n + 1, dtype=torch.float32, device="cuda")
    for scores in (buf[:n], buf[1:]):  # (the second one is 4-byte aligned only)
        for k in sorted({1, min(2, n), (n + 9) // 10, (n + 1) // 2, max(1, n - 1), n}):
            sel = torch.full((k + 1,), -7, dtype=torch.int32, device="cuda")
            got = b.score_deviation_topk(geo, K, 0, KF, k / n, scores, sel)
            torch.cuda.synchronize()
            assert got == k
            assert np.array_equal(scores.cpu().numpy(), want)
            s = sel.cpu().numpy()
            assert s[k] == -7 and np.array_equal(s[:k], oracle.select.select_top(want, k, cs1)), k


@pytest.mark.parametrize("kind", ["spread", "equal", "close", "mixed"])
def test_selection_beyond_the_listed_band(kind):
    """More candidates than a band of the sample's width fits the list for: the
    histogram of every score from the start, or after the list overflows."""
    test_selection_of_given_scores(500_001, kind)
