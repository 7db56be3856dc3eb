"""ModEval on the rings between N = 2^12 and 2^16 (needs an MI355X): the summed rescales of
its Chebyshev terms, with 2, 4 and 8 words per column, three key-switching digit sizes and
coefficient vectors that leave out single terms and whole baby-step sums, bit-exact against
the oracle's term-by-term evaluation."""
import numpy as np
import pytest

import oracle.bootstrap as B

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.boot_rig import SCALE, Rig  # noqa: E402


@pytest.mark.parametrize("log_n,n_q,n_p", [(13, 13, 4), (14, 14, 5), (15, 13, 8)])
def test_eval_mod_midsize(log_n, n_q, n_p):
    rig, K, r, lvl = Rig(log_n, n_q, n_p, 32), 16, 3, n_q - 1
    rng = np.random.default_rng(log_n)
    n, P = rig.N // 2, rig.q[0] / SCALE
    x, ct = rig.enc(rng.uniform(-1, 1, n) + P * rng.integers(-6, 7, n), lvl, SCALE, 21)
    full = B.cheb_coeffs(K, r)
    sparse = np.array(full)
    sparse[rng.permutation(64)[:20]] = 0.0
    sparse[16:24] = 0.0  # a baby-step sum without terms
    for coeffs in (full, sparse):
        want = rig.boot.eval_mod((x, lvl, SCALE), K, r, coeffs)
        out = rig.g.empty_ct(lvl - 11)
        rig.g.nj_eval_mod(ct, K, r, coeffs, out)
        assert out.level == want[1] and out.scale == want[2]
        assert np.array_equal(rig.coeff(out), want[0])
