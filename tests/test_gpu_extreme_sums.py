"""Key switches, rescales and ModRaise at the words that push their uncorrected sums furthest,
and on rings of 31- to 40-bit primes, word for word against the oracle (needs an MI355X):
every scaled input of ModUp's and of ModDown's basis conversion q_a - 1 (up to 8 products of
50-bit primes in one sum), own limbs and key words t - 1 in every digit, and last limbs next to
the middle of their prime, where the centred lift changes sign."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2312_04356_amd import Ct, Ctx, chain_primes  # noqa: E402

G = 5  # the Galois element whose key is imported

RINGS = [  # log_n, n_q, alpha, bits of q_0, the other q_i, the p_i
    (11, 8, 8, 50, 50, 50),
    (12, 12, 3, 50, 50, 50),   # one tile, four digits
    (12, 16, 8, 50, 50, 50),
    (12, 8, 4, 33, 31, 40),
    (13, 16, 8, 50, 50, 50),
    (13, 12, 4, 40, 32, 36),
    (14, 32, 8, 50, 50, 50),   # four digits of 8
    (14, 10, 8, 50, 31, 50),   # ragged last digit, mixed sizes
    (15, 9, 8, 50, 50, 50),
    (16, 9, 8, 50, 50, 50),
    (16, 6, 2, 34, 34, 36),
]


def consts(values, N):
    """[limbs][N]: limb i with every coefficient values[i]"""
    return np.repeat(np.array(values, dtype=np.uint64)[:, None], N, 1)


def hat(primes, a, t):
    """(product of primes other than the a-th) mod t"""
    r = 1
    for b, p in enumerate(primes):
        if b != a:
            r = r * p % t
    return r


def cases(R, level, rng):
    """(name, polynomial [level+1][N], key [dnum][2][L+1+alpha][N]), coefficient form"""
    N, prs, al, dn, nq = R.n, R.key_primes(), R.alpha, R.n_digits(R.L), R.L + 1
    random = lambda: np.stack([np.stack([np.stack([rng.integers(0, t, N, dtype=np.uint64) for t in prs])  # noqa: E731
                                         for _ in range(2)]) for _ in range(dn)])
    # every input of ModUp's conversions q_a - 1
    top = []
    for i in range(level + 1):
        lo = i // al * al
        top.append((R.q[i] - 1) * hat(R.q[lo:min(lo + al, level + 1)], i - lo, R.q[i]) % R.q[i])
    yield "modup", consts(top, N), random()
    # the constant -1 as polynomial and keys: own limbs and key words t - 1, digits' words at
    # every step the same
    minus = np.zeros((len(prs), N), dtype=np.uint64)
    minus[:, 0] = [t - 1 for t in prs]
    yield "words", minus[:level + 1], np.broadcast_to(minus, (dn, 2, len(prs), N))
    # every input of ModDown's conversions p_k - 1: the polynomial has one coefficient, so its
    # extended digits are constants, which the first digit's key divides out
    d = np.zeros((level + 1, N), dtype=np.uint64)
    d[:, 0] = [rng.integers(1, t) for t in R.q[:level + 1]]
    ext, key = R.modup(level, d), random()
    key[1:, :, nq:] = 0
    for k, p in enumerate(R.p):
        c = int(ext[0, level + 1 + k, 0])
        assert c
        key[0, :, nq + k] = (p - 1) * hat(R.p, k, p) * pow(c, -1, p) % p
    yield "moddown", d, key


@pytest.mark.parametrize("log_n,n_q,alpha,b0,bq,bp", RINGS)
def test_extreme_sums(log_n, n_q, alpha, b0, bq, bp):
    O.set_threads(0)
    N, rng = 1 << log_n, np.random.default_rng(log_n + alpha)
    q, p = chain_primes(log_n, n_q, alpha, b0, bq, bp)
    R, c = O.Ring(N, q, p), Ctx(log_n, q, p, 2.0 ** 30)
    for level in sorted({min(alpha, n_q) - 1, n_q - 1}):
        for name, d, key in cases(R, level, rng):
            print("[extreme sums] N=2^%d %s level %d" % (log_n, name, level), flush=True)
            k = c.to_device(np.ascontiguousarray(key).reshape(-1, N))
            c.nj_ntt_limbs(k, list(range(n_q + alpha)) * (2 * c.dnum), False)
            c.nj_key_import(G, c.to_host(k).reshape(-1))
            x = c.to_device(d)
            c.nj_to_eval(x, level, 1)
            out = torch.empty((2, level + 1, N), dtype=torch.int64, device=c.device)
            c.nj_keyswitch(x, level, G, out[0], out[1])
            ct = c.empty_ct(level)  # the same switch with X -> X^G, c0 zero
            c.nj_apply_galois(Ct(torch.stack([torch.zeros_like(x), x]), level), G, ct)
            for t, dd in ((out, d), (ct.data, R.poly_automorph(level, d, G))):
                c.nj_to_coeff(t, level, 2)
                torch.cuda.synchronize()
                assert np.array_equal(c.to_host(t), np.stack(R.keyswitch(level, dd, key))), (name, level)
    ramp = np.arange(N)
    for level in (1, n_q - 1):
        ql, x = q[level], np.empty((2, level + 1, N), dtype=np.uint64)
        for i, t in enumerate(q[:level + 1]):
            x[0, i], x[1, i] = np.where(ramp % 3 == 0, t - 1, 0), np.where(ramp % 5 < 2, 0, t - 1)
        x[0, level] = np.where(ramp % 2 == 0, (ql - 1) // 2, (ql + 1) // 2)
        x[1, level] = np.where(ramp < N // 2, (ql + 1) // 2, (ql - 1) // 2)
        ct, out = Ct(c.to_device(x), level), c.empty_ct(level - 1)
        c.nj_to_eval(ct.data, level, 2)
        c.nj_rescale(ct, out)
        c.nj_to_coeff(out.data, level - 1, 2)
        torch.cuda.synchronize()
        assert np.array_equal(c.to_host(out.data), np.stack([R.rescale(level, x[z]) for z in (0, 1)])), level
    x = np.stack([np.where(ramp % 2 == 0, (q[0] - 1) // 2, (q[0] + 1) // 2),
                  np.where(ramp < N // 2, 0, q[0] - 1)]).astype(np.uint64).reshape(2, 1, N)
    ct, out = Ct(c.to_device(x), 0), c.empty_ct(n_q - 1)
    c.nj_to_eval(ct.data, 0, 2)
    c.nj_modraise(ct, n_q - 1, out)
    c.nj_to_coeff(out.data, n_q - 1, 2)
    torch.cuda.synchronize()
    assert np.array_equal(c.to_host(out.data), np.stack([R.modraise(x[z, 0]) for z in (0, 1)]))
