"""nj_slot_activation of halves whose recorded scales differ within nj_combine's tolerance
(needs an MI355X): on the ring of one tile (N = 4096) each half keeps its own scale through
ModEval, and the call equals the chain of single calls word for word."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from tests.boot_rig import SCALE, Rig  # noqa: E402


@pytest.mark.parametrize("rel", [0.0, 2.0 ** -40, -2.0 ** -31])
def test_halves_at_slightly_different_scales(rel):
    rig = Rig()
    g, lo, n = rig.g, rig.g.L - 2, rig.N // 2
    rng, P = np.random.default_rng(3), rig.q[0] / SCALE
    re, im = (rig.enc(rng.uniform(-1, 1, n) + P * rng.integers(-6, 7, n), lo, SCALE, sub)[1] for sub in (31, 32))
    im.scale = SCALE * (1.0 + rel)
    stoc1 = g.nj_stoc1_plan_create(512, 3, lo - 11)
    for gl in stoc1.galois():
        rig.key(gl)
    out = g.empty_ct(lo - 14)
    g.nj_slot_activation(16, 3, None, None, None, 0, stoc1, re, im, out)
    er, ei, z, y = (g.empty_ct(l) for l in (lo - 11, lo - 11, lo - 11, lo - 14))
    g.nj_eval_mod(re, 16, 3, None, er)
    g.nj_eval_mod(im, 16, 3, None, ei)
    assert (ei.scale == er.scale) == (rel == 0.0)
    g.nj_combine(er, ei, z)
    g.nj_stoc1(stoc1, z, y)
    torch.cuda.synchronize()
    assert out.level == y.level and out.scale == y.scale
    assert torch.equal(out.data, y.data)
