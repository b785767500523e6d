"""The built-in launch shape over the batch sizes where it changes.

The rule takes fewer checks per thread for a batch too small to fill the
device (one block per shot group and no shot queue while every group has a
block of its own), and the shape never changes a result: each batch is
compared bit for bit with the same shots under an explicit shape, and the
smallest with the oracle.
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


# (code, an explicit shape to compare with)
CASES = [("toric2d:8", (8, 8)), ("toric2d:13", (169, 1)), ("toric2d:21", (221, 2)), ("bb:6x6", (36, 1)),
         ("bb:12x6", (36, 2)), ("toric3d_point:5", (63, 2)), ("toric3d_membrane:4", (192, 1)), ("rep:101", (51, 2)),
         ("rep:9", (9, 1))]


@pytest.mark.parametrize("conflict", ["or", "sequential"])
@pytest.mark.parametrize("bp", ["minsum", "sumproduct"])
@pytest.mark.parametrize("name,shape", CASES)
def test_results_do_not_depend_on_the_batch_size(L, orc, name, shape, bp, conflict):
    import torch
    spec = codes.by_name(name)
    dc = L.Code(spec, 0)
    q = 0.125 if "membrane" in name else 0.05
    P = L.DecodeParams(bp=bp, q=q, rounds=8, conflict=conflict, seed=5)
    cfg = {"threads_per_shot": shape[0], "checks_per_thread": shape[1], "shots_per_block": 1}
    e0 = L.sample_noise(dc, 0.05, 3, 0, 4500)
    ref = L.decode_rounds(dc, P, e0, cfg=cfg, want_beliefs=True, want_fail=True)
    o = orc.decode(spec, orc.DecodeParams(bp=bp, q=q, rounds=8, conflict=conflict, seed=5), e0[:40].cpu().numpy(),
                   want_beliefs=True)
    for k in ("z", "s", "tclr"):
        assert np.array_equal(ref[k][:40].cpu().numpy(), o[k]), k
    for S in (1, 2, 7, 255, 256, 257, 1024, 1500, 4500):
        print(f"[shape] {name} {bp} {conflict} shots={S}", flush=True)
        g = L.decode_rounds(dc, P, e0[:S].contiguous(), want_beliefs=True, want_fail=True)
        for k in ("z", "s", "tclr", "fail"):
            assert torch.equal(g[k], ref[k][:S]), (S, k)
        assert torch.equal(g["L"].view(torch.int32), ref["L"][:S].view(torch.int32)), S


@pytest.mark.parametrize("cpt", [1, 2, 4])
@pytest.mark.parametrize("name", ["toric2d:6", "toric2d:9", "bb:6x6", "toric3d_point:3", "toric3d_membrane:3"])
def test_two_threads_per_check(L, orc, name, cpt):
    """The pair kernels against the oracle, bit for bit: pairs that end inside a
    wavefront, padding checks, several shots per block, every conflict rule and
    priors on both sides of the short folds."""
    import torch
    spec = codes.by_name(name)
    if cpt == 4 and name.startswith("bb"):
        pytest.skip("not compiled for (6, 3)")
    dc = L.Code(spec, 0)
    nt = 2 * -(-spec.m // cpt)
    e0 = (np.random.default_rng(2).random((61, spec.n)) < 0.05).astype(np.uint8)
    for spb in (1, 3):
        for k, (conflict, move) in enumerate([("or", "single"), ("xor", "multi"), ("sequential", "single")]):
            for q in (0.05, 9e-5, 0.5):
                P = dict(bp="sumproduct", q=q, rounds=4, iters=9, conflict=conflict, move=move, seed=k)
                cfg = {"threads_per_shot": nt, "checks_per_thread": cpt, "shots_per_block": spb}
                print(f"[pairs] {name} {cfg} {P}", flush=True)
                g = L.decode_rounds(dc, L.DecodeParams(**P), torch.from_numpy(e0).cuda(), cfg=cfg, want_beliefs=True,
                                    want_fail=True)
                o = orc.decode(spec, orc.DecodeParams(**P), e0, want_beliefs=True)
                for key in ("z", "s", "tclr"):
                    assert np.array_equal(g[key].cpu().numpy(), o[key]), (spb, conflict, q, key)
                assert np.array_equal(g["L"].cpu().numpy().view(np.uint32), o["L"].view(np.uint32)), (spb, conflict, q)
                assert np.array_equal(g["fail"].cpu().numpy(), orc.logical_failure(spec, e0, o["z"]))


@pytest.mark.parametrize("name", ["rep:51", "toric2d:4", "toric2d:8", "toric2d:12", "toric2d:16",
                                  "toric3d_point:4", "toric3d_membrane:4"])
def test_small_codes_in_large_batches(L, name):
    """Min-sum on small codes: several shots per block and part wavefronts by the built-in
    rule, on either side of the batch sizes where it changes, against one shot per block."""
    import torch
    spec = codes.by_name(name)
    dc = L.Code(spec, 0)
    P = L.DecodeParams(bp="minsum", q=0.125 if "membrane" in name else 0.05, rounds=6, seed=5)
    e0 = L.sample_noise(dc, 0.05, 3, 0, 40000)
    ref = L.decode_rounds(dc, P, e0, cfg={"checks_per_thread": 1, "shots_per_block": 1}, want_fail=True)
    for S in (8191, 8192, 16384, 32769, 40000):
        print(f"[shape] {name} shots={S}", flush=True)
        g = L.decode_rounds(dc, P, e0[:S].contiguous(), want_fail=True)
        for k in ("z", "s", "tclr", "fail"):
            assert torch.equal(g[k], ref[k][:S]), (S, k)
