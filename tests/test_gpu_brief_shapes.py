"""Decodes of at most two rounds: the shapes they take, and the stream form's results."""
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


# (code, rule, shots, (threads, checks per thread, lanes per check, shots per block))
@pytest.mark.parametrize("name,bp,shots,shape", [
    ("toric2d:8", "sumproduct", 2048, (128, 1, 2, 1)), ("toric2d:8", "sumproduct", 8192, (64, 1, 1, 4)),
    ("toric2d:18", "sumproduct", 8192, (162, 2, 1, 1)), ("toric2d:24", "sumproduct", 8191, (144, 4, 1, 1)),
    ("bb:12x6", "sumproduct", 1025, (72, 1, 1, 3)), ("toric3d_membrane:6", "minsum", 6001, (162, 4, 1, 1)),
    ("bb:30x30", "minsum", 4097, (225, 4, 1, 1)), ("toric2d:9", "minsum", 7993, (41, 2, 1, 6)),
    ("toric3d_point:5", "minsum", 8190, (63, 2, 1, 4)), ("toric3d_point:6", "minsum", 4095, (54, 4, 1, 1)),
    ("toric3d_point:6", "minsum", 8191, (54, 4, 1, 4)), ("toric2d:8", "minsum", 32769, (8, 8, 1, 16)),
    ("toric2d:16", "minsum", 8195, (32, 8, 1, 4))])
def test_short_decodes(L, name, bp, shots, shape):
    import torch
    code = L.Code(codes.by_name(name), 0)
    e0 = L.sample_noise(code, 0.03, 3, 0, shots)
    for rounds in (1, 2, 3):
        P = L.DecodeParams(bp=bp, q=0.125 if "membrane" in name else 0.05, rounds=rounds, seed=5)
        got = code.launch_shape(P, shots)
        got = tuple(got[k] for k in ("threads_per_shot", "checks_per_thread", "lanes_per_check", "shots_per_block"))
        assert rounds > 2 or got == shape, (rounds, got)
        print(f"[brief] {name} {bp} shots={shots} rounds={rounds}", flush=True)
        a = L.decode_rounds(code, P, e0, want_beliefs=True)
        b = L.decode_rounds(code, P, e0, want_beliefs=True, form="stream")
        torch.cuda.synchronize()
        for k in ("z", "s", "tclr", "L"):
            assert torch.equal(a[k], b[k]), (rounds, k)
