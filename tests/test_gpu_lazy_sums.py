"""Lazy giant steps whose c0 parts are summed inside the ModDown combine (up to 16 of them) or
in a pass of their own (more), word for word against the oracle's lazy evaluation, one
ciphertext and batches of 1, 3 and 11 (needs an MI355X): 32 or 64 diagonals split into 1 to
63 giant steps, odd and even, on the rings of one, two and four tiles."""
import numpy as np
import pytest

import oracle.plans as PL

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2312_04356_amd import Ct  # noqa: E402
from tests.midsize import mid_workload  # noqa: E402
from tests.test_gpu_conv_variants import Rig, host_coeff_batch  # noqa: E402


@pytest.mark.parametrize("log_n,w0,n1,giants,level", [(12, 6, 1, 63, 2), (12, 6, 4, 15, 5), (12, 6, 11, 5, 1),
                                                      (13, 14, 1, 31, 1), (13, 14, 2, 15, 4), (13, 14, 16, 1, 2),
                                                      (14, 14, 4, 15, 1), (14, 14, 22, 3, 3)])
def test_lazy_sums(log_n, w0, n1, giants, level):
    r, rng = Rig(mid_workload(log_n, 4), True), np.random.default_rng(log_n + n1)
    gctx, N, q = r.g.ctx, r.N, r.q
    W = PL.padded_width_taps(w0, PL.taps_same(np.ones((1, 1, 3, 3))))
    c = N // (W * W)
    plan = gctx.nj_conv_plan_create_taps(w0, c, c, PL.taps_same(rng.uniform(-1, 1, (c, c, 3, 3))), fuse=1, n1=n1,
                                         level=level)
    ell = plan.layout()[3]
    js = plan.offsets(0)
    oplan = PL.Bsgs(N // 2, ell, [j * ell for j in js], n1=n1)
    assert oplan.js == sorted(js) and sum(g != 0 for g in oplan.giants) == giants
    pts = {j: np.stack([rng.integers(0, q[i], N, dtype=np.uint64) for i in range(level + 1)]) for j in js}
    for idx, j in enumerate(js):
        gctx.nj_plan_set_diagonal(plan, 0, idx, pts[j])
    r.keys(plan.galois())
    plan.set_lazy(True)
    xs = rng.integers(0, q[0], (11, 2, 1, N), dtype=np.uint64)
    xs = np.concatenate([xs] + [rng.integers(0, q[i], (11, 2, 1, N), dtype=np.uint64) for i in range(1, level + 1)], 2)
    batch = gctx.empty_batch(11, level)
    batch.data.copy_(gctx.to_device(xs.reshape(-1, N)).view_as(batch.data))
    gctx.nj_to_eval(batch.data, level, 22)
    batch.scale = r.scale
    y = gctx.empty_ct(level)
    gctx.nj_plan_apply(plan, 0, Ct(batch.data[0], level), y, 1)
    want = r.o.ctx.bsgs(level, xs[0], oplan, pts, lazy=True)
    t = y.data.clone()
    gctx.nj_to_coeff(t, level, 2)
    torch.cuda.synchronize()
    assert np.array_equal(gctx.to_host(t), want)
    for n in (1, 3, 11):  # conv = transform and rescale
        out = gctx.empty_batch(n, level - 1)
        gctx.nj_conv2d_cins_batch(plan, batch, n, out)
        got = host_coeff_batch(gctx, out, n)
        for z in sorted({0, n - 1}):
            want = r.o.ctx.ct_rescale(level, r.o.ctx.bsgs(level, xs[z], oplan, pts, lazy=True))
            assert np.array_equal(got[z], want), "ciphertext %d of %d" % (z, n)
