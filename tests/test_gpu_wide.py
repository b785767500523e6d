"""The wide form: regular codes too large for the resident form, one block per
shot with its messages in LDS and past its end in device memory.

AUTO takes it; the stream form is the general path it is compared with, bit
for bit, over every option it accepts, and the oracle checks both on a few
shots. The codes put the end of the LDS after the last message (membrane L = 12,
toric L = 72 bicycle), inside the code (the others), in a ragged last tile of
checks, and need 16- and 32-bit word tables.
"""
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


_codes = {}


def dcode(L, name):
    if name not in _codes:
        spec = codes.bivariate_bicycle(66, 67) if name == "bb:66x67" else codes.by_name(name)
        if name.startswith("bb"):
            spec.logicals = codes.CSR.from_rows(0, spec.n, [])  # not needed, and slow to find
        _codes[name] = (spec, L.Code(spec, 0))
    return _codes[name]


CODES = ["toric3d_membrane:12", "toric3d_membrane:15", "toric3d_point:19", "toric3d_point:23", "toric2d:113", "bb:66x67"]
OPTIONS = [dict(), dict(skip_fixed=False, iters=3), dict(conflict="xor", move="multi"), dict(iters=1, rounds=9),
           dict(iters=2, rounds=6), dict(iters=0), dict(retire=False, evidence=False), dict(rounds=0),
           dict(alpha=1.25, clamp=6.0), dict(bp="sumproduct", iters=5), dict(bp="sumproduct", iters=4, conflict="xor")]


@pytest.mark.parametrize("name", CODES)
def test_against_the_stream_form_and_the_oracle(L, orc, name):
    import torch
    spec, dc = dcode(L, name)
    q = 0.125 if "membrane" in name else 0.05
    for k, opt in enumerate(OPTIONS):
        kw = dict(dict(rounds=4, iters=9, seed=3), **opt)
        P = L.DecodeParams(q=q, **kw)
        S = 3
        e0 = L.sample_noise(dc, 0.004 + 0.004 * (k % 3), 7 + k, 0, S)
        print(f"[wide] {name} {opt}", flush=True)
        with pytest.raises(L.LaimError):  # (so AUTO is the wide form)
            L.decode_rounds(dc, P, e0, form="resident")
        a = L.decode_rounds(dc, P, e0, shot0=5, want_beliefs=True, want_sweeps=True, want_fail=True)
        b = L.decode_rounds(dc, P, e0, shot0=5, want_beliefs=True, want_sweeps=True, want_fail=True, form="stream")
        for key in ("z", "s", "tclr", "fail", "sweeps"):
            assert torch.equal(a[key], b[key]), (opt, key)
        assert torch.equal(a["L"].view(torch.int32), b["L"].view(torch.int32)), opt
        if k in (0, 9) and spec.m < 7000:
            okw = {x: v for x, v in kw.items() if x != "skip_fixed"}
            o = orc.decode(spec, orc.DecodeParams(q=q, **okw), e0.cpu().numpy(), shot0=5, want_beliefs=True)
            for key in ("z", "s", "tclr"):
                assert np.array_equal(a[key].cpu().numpy(), o[key]), (opt, key)
            assert np.array_equal(a["L"].cpu().numpy().view(np.uint32), o["L"].view(np.uint32)), opt


@pytest.mark.parametrize("name,shots", [("toric3d_membrane:12", 1), ("toric3d_membrane:12", 700), ("toric3d_point:19", 300)])
def test_queue_plan_and_capture(L, name, shots):
    """More shots than compute units (the queue), one shot, and the same items
    in a replayed plan; shots that freeze and shots that run every round."""
    import torch
    spec, dc = dcode(L, name)
    P = L.DecodeParams(q=0.125 if "membrane" in name else 0.05, rounds=12, seed=9)
    e0 = L.sample_noise(dc, 0.02, 1, 0, shots)
    a = L.decode_rounds(dc, P, e0, want_fail=True)
    b = L.decode_rounds(dc, P, e0, want_fail=True, form="stream")
    plan = L.BatchPlan([{"code": dc, "params": P, "e0": e0}])
    for key in ("z", "s", "tclr", "fail"):
        assert torch.equal(a[key], b[key]), key
    for _ in range(3):
        o = plan.launch()[0]
        torch.cuda.synchronize()
        for key in ("z", "s", "tclr", "fail"):
            assert torch.equal(o[key], b[key]), key
        for key in ("z", "s", "tclr", "fail"):
            o[key].fill_(77)


def test_online_from_a_start_syndrome(L):
    import torch
    spec, dc = dcode(L, "toric2d:113")
    plan = L.OnlinePlan(dc, L.OnlineParams(rounds_total=1, window=1, commit=1, p=0.01, p_meas=0.01))
    P = L.DecodeParams(rounds=5, iters=8, seed=4)
    e = L.sample_noise(dc, 0.01, 4, 0, 2)
    eps = torch.zeros((2, 1, dc.m), dtype=torch.uint8, device="cuda")
    o = plan.decode(P, 2, e_in=e.view(2, 1, dc.n), eps_in=eps)
    ref = L.decode_rounds(dc, P, e, form="stream")
    assert torch.equal(o["z"], ref["z"])
