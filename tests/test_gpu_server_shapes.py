"""The server where its launch shape changes: more requests than the few-request
shape serves, several requests per block (full units, partial ones, and units
whose requests end in different rounds), requests that change shape between
their rounds, and results that find no room in pinned memory. Every request
equals its shot of a plain decode."""
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


def reference(L, code, P, e0, shot0):
    r = L.decode_rounds(code, P, e0, shot0=shot0, want_fail=True)
    return {k: r[k].cpu().numpy() for k in ("z", "s", "tclr", "fail")}


def run(L, srv, jobs, width):
    """jobs: (code, params, e0 row, shot id). width(step): requests advanced in
    that step. Returns results in the jobs' order, fetched as they finish."""
    tickets = {srv.submit(c, P, shot, e): k for k, (c, P, e, shot) in enumerate(jobs)}
    out, rounds, step = {}, {}, 0
    while len(out) < len(jobs):
        evs = srv.step(max_events=width(step))
        assert evs, "a step with resident requests reported nothing"
        step += 1
        for ev in evs:
            k = tickets[ev["ticket"]]
            assert ev["round"] == rounds.get(k, 0) + 1
            rounds[k] = ev["round"]
            if ev["done"]:
                out[k] = dict(srv.result(ev["ticket"]), fail=ev["fail"])
    return [out[k] for k in range(len(jobs))]


def check(got, refs):
    for k, (g, (ref, i)) in enumerate(zip(got, refs)):
        assert np.array_equal(g["z"], ref["z"][i]) and np.array_equal(g["s"], ref["s"][i]), k
        assert g["tclr"] == int(ref["tclr"][i]) and g["fail"] == int(ref["fail"][i]), k


@pytest.mark.parametrize("bp", ["minsum", "sumproduct"])
def test_more_requests_than_the_small_shape_serves(L, bp):
    """One wavefront per request in the small shape: 16 per compute unit is its
    limit. Steps of every request and of a few hundred alternate, so that the
    same requests run in both shapes in turn."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    mix = [("toric2d:8", 16 * cus + 300, 0.05), ("bb:6x6", 150, 0.02), ("rep:31", 101, 0.08)]
    jobs, refs = [], []
    for name, n, p in mix:
        code = L.Code(codes.by_name(name), 0)
        P = L.DecodeParams(bp=bp, rounds=7, iters=6, seed=3)
        e0 = L.sample_noise(code, p, 1, 40, n)
        ref = reference(L, code, P, e0, 40)
        rows = e0.cpu().numpy()
        jobs += [(code, P, rows[i], 40 + i) for i in range(n)]
        refs += [(ref, i) for i in range(n)]
    order = np.random.default_rng(0).permutation(len(jobs))
    jobs, refs = [jobs[k] for k in order], [refs[k] for k in order]
    srv = L.Server(0, 1 << 26, len(jobs))
    print(f"[server] {len(jobs)} requests, {bp}", flush=True)
    check(run(L, srv, jobs, lambda step: len(jobs) if step % 3 != 1 else 333), refs)
    st = srv.stats()
    assert st["resident"] == 0 and st["waiting"] == 0 and st["bytes"] == 0


@pytest.mark.parametrize("name,bp,cfg", [("toric2d:8", "minsum", (2, 5)), ("toric2d:9", "sumproduct", (1, 3)),
                                         ("toric2d:16", "minsum", (4, 16)), ("bb:12x6", "minsum", (1, 4)),
                                         ("toric3d_point:4", "sumproduct", (2, 7)), ("toric3d_membrane:3", "minsum", (1, 2)),
                                         ("rep:31", "minsum", (2, 16))])
@pytest.mark.parametrize("count", [1, 4, 63])
def test_several_requests_per_block(L, name, bp, cfg, count):
    code = L.Code(codes.by_name(name), 0)
    P = L.DecodeParams(bp=bp, q=0.125 if "membrane" in name else 0.05, rounds=6, seed=9)
    e0 = L.sample_noise(code, 0.04, 2, 0, count)
    ref = reference(L, code, P, e0, 0)
    rows = e0.cpu().numpy()
    code.set_resident_cfg(bp, {"checks_per_thread": cfg[0], "shots_per_block": cfg[1]})
    srv = L.Server(0, 1 << 24, 64)
    print(f"[server] {name} {bp} {cfg} x {count}", flush=True)
    # (a step of all and one of some: units that are full, partial and of requests in other rounds)
    got = run(L, srv, [(code, P, rows[i], i) for i in range(count)], lambda step: 64 if step % 2 == 0 else 7)
    check(got, [(ref, i) for i in range(count)])


def test_results_beyond_the_pinned_slab(L):
    """2,600 results of 6,912 bytes, none fetched before the last is done: 16 MiB
    hold 2,427 of them, the others are read back from the arena. Then a second
    batch finds room again."""
    code = L.Code(codes.by_name("toric2d:48"), 0)
    P = L.DecodeParams(rounds=2, iters=4, seed=5)
    n = 2600
    e0 = L.sample_noise(code, 0.01, 6, 0, n)
    ref = reference(L, code, P, e0, 0)
    rows = e0.cpu().numpy()
    srv = L.Server(0, 160 << 20, n)
    for turn in range(2):
        jobs = range(n) if turn == 0 else range(50)
        tickets = {srv.submit(code, P, i, rows[i]): i for i in jobs}
        fail = {}
        while len(fail) < len(tickets):
            for ev in srv.step():
                if ev["done"]:
                    fail[ev["ticket"]] = ev["fail"]
        got = [dict(srv.result(t), fail=fail[t]) for t in tickets]
        check(got, [(ref, i) for i in tickets.values()])
    assert srv.stats()["bytes"] == 0
