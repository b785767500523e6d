"""The form and shape a decode runs, as the library reports them: the wide form
where the codes of the wide tests expect it, small and full batches of the
resident one, and the errors of the decode call itself."""
import ctypes as C

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


def dcode(L, name):
    spec = codes.bivariate_bicycle(66, 67) if name == "bb:66x67" else codes.by_name(name)
    if name.startswith("bb:66"):
        spec.logicals = codes.CSR.from_rows(0, spec.n, [])  # not needed, and slow to find
    return L.Code(spec, 0)


def test_struct_layout(L):
    assert C.sizeof(L.LaunchInfo) == 24
    assert [getattr(L.LaunchInfo, f[0]).offset for f in L.LaunchInfo._fields_] == [0, 4, 8, 12, 16, 20]


@pytest.mark.parametrize("name", ["toric3d_membrane:12", "toric3d_membrane:15", "toric3d_point:19", "toric3d_point:23",
                                  "toric2d:113", "bb:66x67"])
def test_larger_regular_codes_run_wide(L, name):
    code = dcode(L, name)
    for kw, form in [({}, "wide"), (dict(bp="sumproduct"), "wide"), (dict(conflict="xor", move="multi"), "wide"),
                     (dict(skip_fixed=False), "wide"), (dict(alpha=1.25), "stream"),
                     (dict(conflict="sequential"), "stream")]:
        P = L.DecodeParams(**kw)
        for n in (1, 3, 700):
            got = code.launch_shape(P, n)
            assert got == dict(form=form, threads_per_shot=0, checks_per_thread=0, shots_per_block=0,
                               lanes_per_check=0, tiled=False), (kw, n)
            assert code.launch_shape(P, n, "stream")["form"] == "stream"
        with pytest.raises(L.LaimError) as e:
            code.launch_shape(P, 3, "resident")
        assert e.value.status == L.EUNSUP


@pytest.mark.parametrize("name,bp", [("toric2d:32", "minsum"), ("toric2d:16", "sumproduct"), ("bb:12x6", "sumproduct"),
                                     ("bb:12x6", "minsum"), ("rep:101", "minsum"), ("toric3d_point:8", "minsum")])
def test_resident_shapes(L, name, bp):
    code = dcode(L, name)
    P = L.DecodeParams(bp=bp)
    full = code.launch_shape(P, 1 << 30)
    assert full["form"] == "resident"
    assert {k: full[k] for k in ("threads_per_shot", "checks_per_thread", "shots_per_block")} == code.resident_cfg(bp)
    var = code.resident_variant(P)
    assert (full["checks_per_thread"], full["tiled"]) == (var["checks_per_thread"], var["tiled"])
    one = code.launch_shape(P, 1)
    assert one["form"] == "resident" and one["shots_per_block"] == 1 and one["checks_per_thread"] <= 2
    for s in (full, one):
        lanes = s["lanes_per_check"]
        assert lanes == (2 if bp == "sumproduct" and (name != "toric2d:16" or s is one) else 1)
        assert s["threads_per_shot"] // lanes * s["checks_per_thread"] >= code.m
        assert s["threads_per_shot"] * s["shots_per_block"] <= 1024
    cfg = {"checks_per_thread": 1, "shots_per_block": 2} if code.m <= 512 else {"checks_per_thread": 2}
    assert code.launch_shape(P, 5, cfg=cfg)["checks_per_thread"] == cfg["checks_per_thread"]


def test_errors_are_those_of_the_decode(L):
    code = dcode(L, "toric2d:8")
    for P, n, kw, status in [(L.DecodeParams(), -1, {}, L.EINVAL), (L.DecodeParams(q=1.5), 4, {}, L.EINVAL),
                             (L.DecodeParams(alpha=1.25), 4, dict(form="resident"), L.EUNSUP),
                             (L.DecodeParams(), 4, dict(cfg={"shots_per_block": 31, "threads_per_shot": 64}), L.EINVAL)]:
        with pytest.raises(L.LaimError) as e:
            code.launch_shape(P, n, **kw)
        assert e.value.status == status
