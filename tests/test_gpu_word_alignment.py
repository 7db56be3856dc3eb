"""Ciphertexts and polynomials that start at an odd word (8-byte, not 16-byte aligned device
memory) against the same words at aligned addresses (needs an MI355X), on rings of one, two
and four tiles and the small ring, at one to four key-switching digits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2312_04356_amd import Ct, Ctx, chain_primes  # noqa: E402


def odd(t):
    """a copy of t that starts one word into its allocation"""
    buf = torch.zeros(t.numel() + 2, dtype=t.dtype, device=t.device)
    assert buf.data_ptr() % 16 == 0
    v = buf[1:1 + t.numel()].view(t.shape)
    v.copy_(t)
    return v


@pytest.mark.parametrize("log_n,alpha", [(11, 3), (12, 3), (13, 3), (14, 4)])
def test_odd_word_offsets(log_n, alpha):
    N = 1 << log_n
    q, p = chain_primes(log_n, 12, alpha, 50, 48, 50)
    c = Ctx(log_n, q, p, 2.0 ** 40)
    rng = np.random.default_rng(log_n)
    s = np.zeros(N, dtype=np.int8)
    s[rng.choice(N, 32, replace=False)] = 1
    c.nj_set_secret(s)
    c.nj_timing_keys(3)  # random residues in the place of keys
    for level in (1, 4, 11):
        x = c.to_device(np.stack([np.stack([rng.integers(0, t, N, dtype=np.uint64) for t in q[:level + 1]])
                                  for _ in range(2)]))
        plan = c.nj_plan_create_random(level, N // 64, list(range(6)), n1=3)
        plan.set_hoist(False)

        def calls(mk):
            a, r, v = (Ct(mk(x), level) for _ in range(3))
            h, y = (Ct(mk(torch.zeros_like(x[:, :level])), level - 1) for _ in range(2))
            c.nj_rotate(a, 3, r)
            c.nj_hmult(a, r, h)
            k0, k1 = mk(x[0]), mk(x[0])
            c.nj_keyswitch(a.data[1], level, 0, k0, k1)
            c.nj_conv2d_cins(plan, a, y)
            c.nj_to_coeff(v.data, level, 2)
            d = mk(x[0])
            c.nj_decrypt(a, d)
            torch.cuda.synchronize()
            return [t.clone() for t in (r.data, h.data, k0, k1, y.data, v.data, d)]

        for i, (w, g) in enumerate(zip(calls(lambda t: t.clone()), calls(odd))):
            assert torch.equal(w, g), "call %d at level %d" % (i, level)
