"""The continuous machine's register-lean sum-product (one box-plus at a time,
packed partner words): every degree and launch shape that takes it, clamps on
both sides of the short folds, with and without skipped steps, against the oracle."""
import numpy as np
import pytest

from paper_2609_38139_amd import codes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("a GPU test ran without a visible GPU")
    from paper_2609_38139_amd import laim
    laim.lib()
    return laim


@pytest.mark.parametrize("q,clamp", [(0.05, 1000.0), (9e-5, 1000.0), (9e-5, 8.5)])
@pytest.mark.parametrize("name,cpt,p", [("bb:6x6", 4, 0.06), ("bb:12x6", 4, 0.04), ("toric2d:10", 8, 0.06),
                                        ("toric3d_point:4", 4, 0.03), ("toric3d_membrane:3", 4, 0.04)])
def test_against_the_oracle(L, orc, name, cpt, p, q, clamp):
    import torch
    code = codes.by_name(name)
    dc = L.Code(code, 0)
    kw = dict(bp="sumproduct", q=q, clamp=clamp, dt=0.01, t_max=4.0, seed=7)
    e0 = (np.random.default_rng(5).random((9, code.n)) < p).astype(np.uint8)
    o = orc.ctm_decode(code, orc.ContinuousParams(**kw), e0, shot0=2, nthreads=8)
    for skip in (True, False):
        print(f"[ctm] {name} cpt={cpt} q={q} clamp={clamp} skip={skip}", flush=True)
        g = L.decode_continuous(dc, L.ContinuousParams(skip_fixed=skip, **kw), torch.from_numpy(e0).cuda(), shot0=2,
                                checks_per_thread=cpt)
        for k in ("z", "s", "tclr"):
            assert np.array_equal(g[k].cpu().numpy(), o[k]), (k, skip)
        assert np.array_equal(g["counts"].cpu().numpy(), np.stack([o["events"], o["moves"]], axis=1)), skip
