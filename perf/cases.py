"""What the library is timed on: the work a program that evaluates encrypted convolutions
has it do, from one rotation on the small ring to a batch of fused convs with CoeffToSlot
on the full one.

A case names a ring (log_n, n_q ciphertext primes, alpha special primes: the parameter
sets under synth/params and the rings between them that the tests run), an operation
(`op`) and its sizes.  A program keeps one context per ring with its switching keys and
its CoeffToSlot and StoC1 plans for as long as it lives; `ring()` does the same.  Weights,
images and ciphertexts are a state's own and come from its seed.

Outputs are residues modulo the ring's primes: whole numbers, to be equal word for word.
`exact` therefore has no value for any of them.
"""
import math

import numpy as np
import torch

from paper_2312_04356_amd import Ctx, chain_primes, nj_layer_masks

SCALE = 2.0 ** 40   # log_scale of every parameter set
H = 192             # nonzero entries of the secret
MODEVAL_K = 32      # range of the sine for that secret
BOUND = 16.0        # bound of a conv's output, folded into its weights and masks
RINGS = {12: (8, 2), 13: (12, 3), 14: (12, 4), 15: (12, 8), 16: (24, 8)}
FULL_SPLIT = (4, 8, 8)  # baby steps of the full ring's CoeffToSlot groups


# ------------------------------------------------------------------ the cases

def listed():
    small, mid, full = ({"log_n": n, "n_q": RINGS[n][0], "alpha": RINGS[n][1]} for n in (12, 14, 16))
    return [
        # one rotation on the smallest ring: the shortest call a program makes, all launches
        dict(small, name="rotate_n12", op="rotate", level=7, r=3),
        # the key switch everything else is built of, at the top level
        dict(full, name="rotate_n16_top", op="rotate", level=23, r=1),
        # a product with relinearisation halfway down ModEval (the last digit is ragged)
        dict(full, name="hmult_n16", op="hmult", level=13),
        # a fresh plaintext (mask, weight) transformed, multiplied in and rescaled
        dict(full, name="mask_n16", op="mask", level=18),
        # the client's side: c0 + c1 s and the inverse transform
        dict(full, name="decrypt_n16", op="decrypt", level=20),
        # Algorithm 1's conv of one layer in one ciphertext, 16 channels of 32x32 at level 1
        dict(full, name="conv_n16_l1", op="conv", level=1, w0=32, c=16, f=3, lazy=False),
        # a job's conv at its own level: 64 channels of 28x28
        dict(full, name="conv_n16_l15", op="conv", level=15, w0=28, c=64, f=3, lazy=True),
        # a layer wider than a ciphertext: 64 -> 64 channels of 56x56, 4 x 4 blocks
        dict(full, name="block_n16", op="block", level=1, w0=56, c_in=64, c_out=64, f=3),
        # conv + CoeffToSlot on a middle ring, every plan at its defaults
        dict(mid, name="step_n14", op="step", w0=16, c=16, f=3, lazy=False, split=False),
        # the benchmark's step
        dict(full, name="step_n16", op="step", w0=32, c=16, f=3, lazy=True, split=True),
        # a whole layer: conv, bootstrapping, masks, square, StoC1
        dict(full, name="layer_n16", op="layer", w0=32, c=16, f=3, masked=True, act=1),
        # a server's batch, one sub-batch of 8 and a remainder
        dict(full, name="batch_n16", op="batch", n=11, w0=32, c=16, f=3, lazy=True, split=True),
    ]


def draw(rng):
    """One more case: any ring, any level, any channel count and image width it can hold."""
    op = rng.choice(("rotate", "rotate", "hmult", "mask", "decrypt", "conv", "conv", "block", "step", "step", "layer",
                     "batch"))
    log_n = 16 if op == "layer" else rng.choice((12, 13, 14, 15, 16, 16, 16))
    n_q, alpha = RINGS[log_n]
    case = {"log_n": log_n, "n_q": n_q, "alpha": alpha, "op": op}
    if op in ("rotate", "hmult", "mask", "decrypt"):
        case["level"] = rng.randint(0 if op in ("rotate", "decrypt") else 1, n_q - 1)
        if op == "rotate":
            case["r"] = rng.choice((-1, 1)) * rng.randint(1, 64)
        return case
    f = rng.choice((1, 3, 3, 5))
    case["f"] = f
    # padded widths whose images leave 2..64 channels in a ciphertext
    W = rng.choice([w for w in (8, 16, 32, 64, 128) if 2 <= (1 << log_n) // (w * w) <= 64])
    w0 = rng.randint(W // 2 + 1, W - (f - 1) // 2)
    C = (1 << log_n) // (W * W)
    case["w0"] = w0
    if op == "block":
        case["level"] = rng.randint(1, 3)
        case["c_in"], case["c_out"] = rng.randint(C + 1, 3 * C), rng.randint(1, 3 * C)
        return case
    case["c"] = C if rng.random() < 0.7 else rng.randint(1, C)
    if op == "conv":
        case["level"] = rng.randint(1, n_q - 1)
        case["lazy"] = rng.random() < 0.5
    elif op == "layer":
        case["masked"], case["act"] = rng.random() < 0.5, rng.randint(0, 1)
    else:
        case["lazy"] = rng.random() < 0.5
        case["split"] = log_n == 16 and rng.random() < 0.5
        if op == "batch":
            case["n"] = rng.randint(2, 11)
    return case


# ----------------------------------------------- what a program keeps per ring

class _Ring:
    """A context with its secret, and the keys and plans made so far."""

    def __init__(self, log_n, n_q, alpha):
        self.log_n, self.N = log_n, 1 << log_n
        self.q, self.p = chain_primes(log_n, n_q, alpha, 50, 48, 50)
        self.ctx = Ctx(log_n, self.q, self.p, SCALE)
        rng = np.random.default_rng([log_n, n_q, alpha])
        s = np.zeros(self.N, dtype=np.int8)
        s[rng.choice(self.N, H, replace=False)] = rng.integers(0, 2, H) * 2 - 1
        self.ctx.nj_set_secret(s)
        self.made, self.plans = set(), {}
        self.groups = 2 if log_n == 12 else 3

    def keys(self, gs):
        """switching keys of the Galois elements gs (0: relinearisation)"""
        for g in gs:
            if g in self.made:
                continue
            rng = np.random.default_rng([self.log_n, 7, g])
            c = self.ctx
            a = np.stack([uniform(rng, self.q + self.p, self.N) for _ in range(c.dnum)])
            c.nj_gen_switch_key(g, a, np.stack([error(rng, self.N) for _ in range(c.dnum)]))
            self.made.add(g)

    def cts(self, lazy, split):
        key = ("cts", lazy, split)
        if key not in self.plans:
            c = self.ctx
            plan = c.nj_cts_plan_create_split(self.groups, FULL_SPLIT) if split else c.nj_cts_plan_create(self.groups)
            plan.set_lazy(lazy)
            self.keys(plan.galois())
            self.plans[key] = plan
        return self.plans[key]

    def stoc1(self, ell, level):
        key = ("stoc1", ell, level)
        if key not in self.plans:
            plan = self.ctx.nj_stoc1_plan_create(ell, 3, level)
            self.keys(plan.galois())
            self.plans[key] = plan
        return self.plans[key]


_RINGS = {}


def ring(case):
    key = (case["log_n"], case["n_q"], case["alpha"])
    if key not in _RINGS:
        _RINGS[key] = _Ring(*key)
    return _RINGS[key]


def uniform(rng, primes, n):
    return np.stack([rng.integers(0, q, n, dtype=np.uint64) for q in primes])


def error(rng, n):
    return np.rint(rng.normal(0.0, 3.24, n)).astype(np.int64)


def width(w0, f):
    W = 1
    while W < w0 + (f - 1) // 2:
        W *= 2
    return W


# --------------------------------------------------------------------- inputs

def encrypt(R, rng, coeffs, level, out=None):
    c = R.ctx
    m = torch.empty((level + 1, R.N), dtype=torch.int64, device=c.device)
    c.nj_upload_plain(coeffs, level, m)
    ct = c.empty_ct(level)
    if out is not None:
        ct.data = out
    return c.nj_encrypt_sk(m, level, uniform(rng, R.q[:level + 1], R.N), error(rng, R.N), SCALE, ct)


def message(R, rng, bound=1.0):
    """coefficients of a message bounded by `bound`"""
    return np.rint(rng.uniform(-bound, bound, R.N) * SCALE).astype(np.int64)


def image(R, rng, w0, W, channels):
    """real-CinS coefficients of `channels` images of w0 x w0 padded to W x W"""
    x = np.zeros((R.N // (W * W), W, W))
    x[:channels, :w0, :w0] = rng.uniform(-1, 1, (channels, w0, w0))
    return R.ctx.nj_encode_cins(x.reshape(x.shape[0], W * W), SCALE)


def conv_plan(R, rng, case, level=1, bound=1.0):
    c_in, c_out = case.get("c_in", case.get("c")), case.get("c_out", case.get("c"))
    f = case["f"]
    K = rng.uniform(-1, 1, (c_out, c_in, f, f))
    if bound > 1.0:  # outputs of rms 4 whatever the shape, a bound of 16 folded in
        K *= 12.0 / (f * math.sqrt(c_in) * bound)
    plan = R.ctx.nj_conv_plan_create_layer(case["w0"], K, level=level)
    if case.get("lazy"):
        plan.set_lazy(True)
    R.keys(plan.galois())
    return plan


def prepare(case, seed):
    R, rng = ring(case), np.random.default_rng([seed, 11])
    c, op = R.ctx, case["op"]
    st = {"op": op, "ctx": c, "case": case}
    if op in ("rotate", "hmult", "mask", "decrypt"):
        l = case["level"]
        st["x"] = encrypt(R, rng, message(R, rng), l)
        if op == "rotate":
            R.keys([c.nj_galois_elt(case["r"])])
            st["out"] = c.empty_ct(l)
        elif op == "hmult":
            R.keys([0])
            st["y"], st["out"] = encrypt(R, rng, message(R, rng), l), c.empty_ct(l - 1)
        elif op == "mask":
            st["m"] = torch.empty((l + 1, R.N), dtype=torch.int64, device=c.device)
            c.nj_upload_plain(c.nj_encode_slots(rng.uniform(-1, 1, R.N // 2) + 0j, float(R.q[l])), l, st["m"])
            st["pt"] = torch.empty_like(st["m"])
            st["prod"], st["out"] = c.empty_ct(l), c.empty_ct(l - 1)
        else:
            st["out"] = torch.empty((l + 1, R.N), dtype=torch.int64, device=c.device)
        return st
    W = width(case["w0"], case["f"])
    C = R.N // (W * W)
    if op == "block":
        l, bi, bo = case["level"], -(-case["c_in"] // C), -(-case["c_out"] // C)
        st["conv"] = conv_plan(R, rng, case, l)
        st["x"] = c.empty_batch(bi, l)
        for b in range(bi):
            ct = encrypt(R, rng, image(R, rng, case["w0"], W, min(C, case["c_in"] - b * C)), l, st["x"].data[b])
        st["x"].sync_from(ct)
        st["out"] = c.empty_batch(bo, l - 1)
        return st
    l = case.get("level", 1)
    st["conv"] = conv_plan(R, rng, case, l, BOUND if op == "layer" else 1.0)
    if op == "batch":
        n = case["n"]
        st["x"] = c.empty_batch(n, l)
        for z in range(n):
            ct = encrypt(R, rng, image(R, rng, case["w0"], W, case["c"]), l, st["x"].data[z])
        st["x"].sync_from(ct)
    else:
        st["x"] = encrypt(R, rng, image(R, rng, case["w0"], W, case["c"]), l)
    if op == "conv":
        st["out"] = c.empty_ct(l - 1)
        return st
    lo = c.L - R.groups
    if op == "layer":
        le = lo - 11  # after ModEval
        lp = le - (1 if case["masked"] else 0) - case["act"]
        st["cts"], st["stoc1"] = R.cts(True, True), R.stoc1(W * W // 2, lp)
        R.keys([0])
        st["masks"] = (None, None)
        if case["masked"]:
            st["masks"] = []
            for mask in nj_layer_masks(R.log_n, W, C, case["w0"]):
                t = torch.empty((le + 1, R.N), dtype=torch.int64, device=c.device)
                c.nj_upload_plain(c.nj_encode_slots(BOUND * mask + 0j, float(R.q[le])), le, t)
                c.nj_to_eval(t, le, 1)
                st["masks"].append(t)
        st["out"] = c.empty_ct(lp - 3)
        return st
    st["cts"] = R.cts(case["lazy"], case["split"])
    if op == "batch":
        st["y"], st["re"], st["im"] = (c.empty_batch(case["n"], k) for k in (0, lo, lo))
    else:
        st["y"], st["re"], st["im"] = (c.empty_ct(k) for k in (0, lo, lo))
    return st


# ------------------------------------------------------------------- one pass

def run(st):
    c, op, case = st["ctx"], st["op"], st["case"]
    if op == "rotate":
        return c.nj_rotate(st["x"], case["r"], st["out"]).data
    if op == "hmult":
        return c.nj_hmult(st["x"], st["y"], st["out"]).data
    if op == "mask":
        st["pt"].copy_(st["m"])  # the plaintext's coefficients are kept
        c.nj_to_eval(st["pt"], case["level"], 1)
        c.nj_pmult(st["x"], st["pt"], st["prod"])
        return c.nj_rescale(st["prod"], st["out"]).data
    if op == "decrypt":
        c.nj_decrypt(st["x"], st["out"])
        return st["out"]
    if op == "conv":
        return c.nj_conv2d_cins(st["conv"], st["x"], st["out"]).data
    if op == "block":
        return c.nj_conv2d_block(st["conv"], st["x"], st["out"]).data
    if op == "step":
        c.nj_conv2d_cins(st["conv"], st["x"], st["y"])
        c.nj_coeff_to_slot(st["cts"], st["y"], st["re"], st["im"])
    elif op == "batch":
        c.nj_conv2d_cins_batch(st["conv"], st["x"], case["n"], st["y"])
        c.nj_coeff_to_slot_batch(st["cts"], st["y"], case["n"], st["re"], st["im"])
    else:
        mre, mim = st["masks"]
        return c.nj_conv_act_layer(st["conv"], st["cts"], MODEVAL_K, 3, None, mre, mim, case["act"], st["stoc1"],
                                   st["x"], st["out"]).data
    return {"conv": st["y"].data, "re": st["re"].data, "im": st["im"].data}


def exact(case, seed):
    return None  # residues: whole numbers, equal word for word


# ----------------------------------------------------------------------- work

class _Count:
    """Words a pass has to read and write once each, and its modular multiply-adds."""

    def __init__(self, case):
        self.N, self.alpha, self.log_n = 1 << case["log_n"], case["alpha"], case["log_n"]
        self.words = self.muls = 0.0

    def io(self, limbs):
        self.words += limbs * self.N

    def ntt(self, limbs):
        self.muls += limbs * self.N * self.log_n / 2

    def key_switches(self, l, n, n_ct=1, keys=None, extend=None, reduce=None):
        """n key switches at level l of each of n_ct ciphertexts, `keys` distinct keys (n by
        default); `extend` polynomials are raised to the special primes and `reduce` pairs
        brought back (by default one each per key switch)"""
        d, ne, a = -(-(l + 1) // self.alpha), l + 1 + self.alpha, self.alpha
        extend, reduce = n if extend is None else extend, n if reduce is None else reduce
        self.io((n if keys is None else keys) * 2 * d * ne)
        self.muls += n_ct * n * 2 * d * ne * self.N
        self.ntt(n_ct * extend * (l + 1 + d * ne - (l + 1)))
        self.muls += n_ct * extend * (l + 1) * (ne - min(a, l + 1)) * self.N
        self.ntt(n_ct * reduce * 2 * (a + l + 1))
        self.muls += n_ct * reduce * 2 * a * (l + 1) * self.N

    def transform(self, l, diags, n1, n_ct=1, bi=1, bo=1):
        """a baby-step giant-step transform of `diags` diagonals per block: the baby steps
        share their raising, the giant steps their bringing back"""
        babies, giants = n1 - 1, -(-diags // n1) - 1
        self.io(bi * bo * diags * (l + 1))
        self.muls += n_ct * 2 * bi * bo * diags * (l + 1) * self.N
        if babies:
            self.key_switches(l, babies, n_ct * bi, extend=1)
        if giants:
            self.key_switches(l, giants, n_ct * bo, reduce=1)

    def rescale(self, l, n_ct=1):
        self.ntt(n_ct * 2 * (l + 1))
        self.muls += n_ct * 2 * l * self.N


def work(case):
    w, op, l = _Count(case), case["op"], case.get("level", 1)
    L, n = case["n_q"] - 1, case.get("n", 1)
    groups = 2 if case["log_n"] == 12 else 3
    if op == "rotate":
        w.io(4 * (l + 1))
        w.key_switches(l, 1)
    elif op == "hmult":
        w.io(4 * (l + 1) + 2 * l)
        w.muls += 4 * (l + 1) * w.N
        w.key_switches(l, 1)
        w.rescale(l)
    elif op == "mask":
        w.io(3 * (l + 1) + 2 * l)
        w.ntt(l + 1)
        w.muls += 2 * (l + 1) * w.N
        w.rescale(l)
    elif op == "decrypt":
        w.io(3 * (l + 1))
        w.muls += (l + 1) * w.N
        w.ntt(l + 1)
    else:
        W = width(case["w0"], case["f"])
        C = w.N // (W * W)
        bi, bo = -(-case.get("c_in", 1) // C), -(-case.get("c_out", 1) // C)
        w.io(n * (2 * bi * (l + 1) + 2 * bo * l))
        w.transform(l, C, math.isqrt(C - 1) + 1, n, bi, bo)
        w.rescale(l, n * bo)
    if op in ("step", "batch", "layer"):
        stages = case["log_n"] - 1
        for t in range(groups):
            k = stages * (t + 1) // groups - stages * t // groups
            diags = 2 ** k if t == 0 else 2 ** (k + 1) - 1
            w.transform(L - t, diags, math.isqrt(diags - 1) + 1, n)
            w.rescale(L - t, n)
        lo = L - groups
        w.ntt(n * 2 * (L + 2))
        w.key_switches(lo, 1, n)  # conjugation
        if op != "layer":
            w.io(n * 4 * (lo + 1))
    if op == "layer":  # two ModEvals of 19 products down 11 levels, one relinearisation key
        depths = [1, 2, 2, 3, 3, 3, 3, 4, 5] + [6, 6, 6, 6, 7, 7, 7] + [8, 9, 10]
        for i, d in enumerate(depths):
            w.key_switches(lo - d, 1, 2, keys=1 if i == 0 else 0)
            w.rescale(lo - d, 2)
        le = lo - 11
        if case["masked"]:
            w.io(2 * (le + 1))
            w.rescale(le, 2)
            le -= 1
        if case["act"]:
            w.key_switches(le, 1, 2, keys=0)
            w.rescale(le, 2)
            le -= 1
        stages = (W * W // 2).bit_length() - 1
        for t in range(3):
            k = stages * (t + 1) // 3 - stages * t // 3
            w.transform(le - t, 2 ** (k + 1) - 1, math.isqrt(2 ** (k + 1) - 2) + 1)
            w.rescale(le - t)
        w.io(2 * (le - 2))
    return {"bytes": 8.0 * w.words, "flops": 2.0 * w.muls}
