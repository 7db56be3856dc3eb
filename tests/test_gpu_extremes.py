"""Transforms at the words that push their uncorrected sums furthest (needs an MI355X): all
words t - 1, half of them 0, 2^i-periodic patterns and random ones, on every ring degree
with a different number of column stages.  A polynomial times X^k is a known signed shift,
so both directions are checked exactly without another transform."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2312_04356_amd import Ct, Ctx, chain_primes  # noqa: E402


@pytest.mark.parametrize("log_n", [11, 12, 13, 14, 15, 16])
def test_extreme_words(log_n):
    N, level = 1 << log_n, 3
    q, p = chain_primes(log_n, 4, 2, 50, 48, 50)
    g = Ctx(log_n, q, p, 2.0 ** 40)
    rng = np.random.default_rng(5)
    k = np.arange(N)
    patterns = [np.ones(N, dtype=bool), k % 2 == 0, (k >> (log_n - 1)) == 0] + \
        [(k >> i) & 1 == 1 for i in range(0, log_n, 3)] + [rng.integers(0, 2, N) == 1]
    sh = N // 2 + 3
    for pat in patterns:
        x = np.stack([np.where(pat, t - 1, 0) for t in q]).astype(np.uint64)
        poly = np.stack([x, x[:, ::-1]])
        ct = Ct(g.to_device(poly), level)
        g.nj_to_eval(ct.data, level, 2)
        assert int(ct.data.min()) >= 0 and all(int(ct.data[:, i].max()) < t for i, t in enumerate(q))
        mono = np.zeros((level + 1, N), dtype=np.uint64)
        mono[:, sh] = 1
        md = g.to_device(mono)
        g.nj_to_eval(md, level, 1)
        out = g.empty_ct(level)
        g.nj_pmult(ct, md, out)
        for c in (ct, out):
            g.nj_to_coeff(c.data, level, 2)
        torch.cuda.synchronize()
        assert np.array_equal(g.to_host(ct.data).reshape(poly.shape), poly)
        want = np.roll(poly, sh, axis=-1)
        for i, t in enumerate(q):
            w = want[:, i, :sh]
            want[:, i, :sh] = np.where(w == 0, w, np.uint64(t) - w)
        assert np.array_equal(g.to_host(out.data).reshape(poly.shape), want)
