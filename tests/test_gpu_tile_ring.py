"""The ring of one 4096-word tile, whose key switches have kernels of their own (needs an
MI355X), word for word against the oracle: conv, CoeffToSlot with lazy and plain giant steps and
rotations at every level, for digits of 2 to 12 primes (one to six digits: with more than four,
or more than 8 primes in one, the general kernels run).  And decryption into separate memory
and in place of c1, on this ring and a larger one."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2312_04356_amd import Ct  # noqa: E402
from paper_2312_04356_amd.workload import GpuWorkload  # noqa: E402
from tests.midsize import mid_workload  # noqa: E402
from tests.oracle_workload import OracleWorkload  # noqa: E402
from tests.test_gpu_midsize import host_coeff, load  # noqa: E402


@pytest.mark.timeout(600)
@pytest.mark.parametrize("alpha,lazy", [(2, True), (3, True), (3, False), (4, False), (6, True), (8, True), (8, False),
                                        (12, True)])
def test_step_parity_one_tile(alpha, lazy):
    O.set_threads(0)
    name = mid_workload(12, alpha)
    print("[tile ring] alpha=%d lazy=%s" % (alpha, lazy), flush=True)
    o, g = OracleWorkload(name, with_cts=True), GpuWorkload(name, with_cts=True, lazy=lazy)
    gctx = g.ctx
    load(gctx, g.conv_plan, 0, o.conv_pts)
    for t, (_, pts) in enumerate(o.cts):
        load(gctx, g.cts_plan, t, pts)
    gs = g.galois_elements()
    g.make_keys(gs)
    o.make_keys(gs)
    m = o.ring.to_rns(o.input_plaintext(), 1)
    x_o, x_g = o.encrypt_input(1), g.encrypt_input(1, m_dev=gctx.to_device(m))
    y = gctx.empty_ct(0)
    gctx.nj_conv2d_cins(g.conv_plan, x_g, y)
    lvl = gctx.L - len(o.cts)
    re, im = gctx.empty_ct(lvl), gctx.empty_ct(lvl)
    gctx.nj_coeff_to_slot(g.cts_plan, y, re, im)
    torch.cuda.synchronize()
    y_o = o.ctx.conv2d_cins(x_o, o.conv_bsgs, o.conv_pts)
    assert np.array_equal(host_coeff(gctx, y), y_o), "conv output differs"
    w_re, w_im = o.ctx.coeff_to_slot(y_o, [p for p, _ in o.cts], [pts for _, pts in o.cts], lazy=lazy)
    assert np.array_equal(host_coeff(gctx, re), w_re) and np.array_equal(host_coeff(gctx, im), w_im)
    # one rotation per level: every digit count up to the ring's, the last digit of any size
    rot = next(r for r in range(1, g.N // 2) if pow(5, r, 2 * g.N) in gs)
    rng = np.random.default_rng(alpha)
    for level in range(gctx.L + 1):
        c = np.stack([np.stack([rng.integers(0, q, g.N, dtype=np.uint64) for q in g.q[:level + 1]]) for _ in range(2)])
        d = gctx.to_device(c)
        gctx.nj_to_eval(d, level, 2)
        out = gctx.empty_ct(level)
        gctx.nj_rotate(Ct(d, level), rot, out)
        assert np.array_equal(host_coeff(gctx, out), o.ctx.rotate(level, c, rot)), "level %d" % level


@pytest.mark.parametrize("log_n", [12, 13])
def test_decrypt_into_its_own_memory(log_n):
    g = GpuWorkload(mid_workload(log_n, 4), with_cts=False)
    gctx, N, level = g.ctx, g.N, 2
    rng = np.random.default_rng(log_n)
    c = np.stack([np.stack([rng.integers(0, q, N, dtype=np.uint64) for q in g.q[:level + 1]]) for _ in range(2)])
    d = gctx.to_device(c)
    gctx.nj_to_eval(d, level, 2)
    want = torch.empty((level + 1, N), dtype=torch.int64, device=gctx.device)
    gctx.nj_decrypt(Ct(d.clone(), level), want)
    gctx.nj_decrypt(Ct(d, level), d[1])  # the general kernels
    torch.cuda.synchronize()
    assert torch.equal(d[1], want)
