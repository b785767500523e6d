"""The work a user of the decoder has it do, as cases to be timed.

A case is a dict of plain values whose "kind" names a public path of
``paper_2609_38139_amd.laim``:

  decode      errors in hand -> z, s, t_clr, failure (one ``decode_rounds``)
  montecarlo  a logical-error-rate step: fresh noise, decode, failure test
  pipeline    the same as separate calls: noise, syndrome, decode, failure
  soft        plain BP: one round's sweeps, with the beliefs returned
  plan        one launch of a batched plan over several codes
  online      spacetime windows over noisy syndrome rounds
  continuous  the continuous-time machine
  bitcentric  the bit-centric machine on a repetition code
  serving     requests submitted to the server and stepped until all are done

``listed()`` holds the standing cases, ``draw(rng)`` gives more of the same
ranges, ``prepare`` makes a case's inputs on the GPU from a seed, ``run`` is
one pass, ``work`` the bytes and operations it cannot do without and
``exact`` the same results in 64 bits where the outputs are computed numbers.
"""
import math

import numpy as np
import torch

from paper_2609_38139_amd import codes, laim

# Codes of a batched plan or a serving mix: (code, rounds).
PLANS = {
    # bivariate-bicycle codes with toric codes, as in the bench's BB matrix
    "bb+toric2d": [("bb:6x6", 64), ("bb:12x6", 64), ("toric2d:16", 64), ("toric2d:32", 128)],
    # every resident family at once
    "families": [("toric2d:8", 64), ("toric3d_point:12", 48), ("toric3d_membrane:8", 32), ("bb:12x6", 64),
                 ("rep:101", 64)],
}
MIX = [("toric2d:16", 128), ("toric2d:32", 256), ("toric2d:48", 384), ("toric3d_point:12", 96),
       ("bb:12x6", 96)]


def prior(name):
    """Table S1's prior of a code's family."""
    return 0.125 if "membrane" in name else 0.05


def listed():
    return [
        # the smallest call: one shot of a small code, where latency counts
        {"name": "decode_toric8_one_shot", "kind": "decode", "code": "toric2d:8", "bp": "minsum", "p": 0.05,
         "shots": 1, "rounds": 64},
        # the bench's step: 2D toric L = 32, min-sum, 65,536 shots
        {"name": "mc_toric32_minsum", "kind": "montecarlo", "code": "toric2d:32", "bp": "minsum", "p": 0.05,
         "shots": 65536, "rounds": 128},
        # the paper's BP rule on the same code
        {"name": "mc_toric32_sumproduct", "kind": "montecarlo", "code": "toric2d:32", "bp": "sumproduct",
         "p": 0.05, "shots": 16384, "rounds": 128},
        # the [[144,12,12]] code with the paper's rule at a noise rate near its threshold
        {"name": "mc_bb144_sumproduct", "kind": "montecarlo", "code": "bb:12x6", "bp": "sumproduct", "p": 0.03,
         "shots": 65536, "rounds": 96},
        # an odd lattice and an odd batch, multi-qubit moves under XOR, each step a call of its own
        {"name": "pipeline_toric21_odd", "kind": "pipeline", "code": "toric2d:21", "bp": "minsum", "p": 0.04,
         "shots": 10007, "rounds": 84, "conflict": "xor", "move": "multi"},
        # beliefs of plain BP (20 sweeps), as a soft-output stage in front of another decoder
        {"name": "soft_point12_sumproduct", "kind": "soft", "code": "toric3d_point:12", "bp": "sumproduct",
         "p": 0.03, "shots": 4096, "rounds": 1},
        # a code too large for one compute unit's LDS: messages in HBM
        {"name": "mc_membrane16_stream", "kind": "montecarlo", "code": "toric3d_membrane:16", "bp": "minsum",
         "p": 0.03, "shots": 1024, "rounds": 64},
        # several code families and noise rates in one graph launch
        {"name": "plan_families", "kind": "plan", "plan": "families", "bp": "minsum", "p": 0.03, "shots": 8192},
        # online decoding: 16 noisy syndrome rounds, windows of 4 committing 2
        {"name": "online_toric16_sumproduct", "kind": "online", "code": "toric2d:16", "bp": "sumproduct",
         "p": 0.01, "shots": 8192, "rounds": 16, "rounds_total": 16, "window": 4, "commit": 2},
        # Algorithm 1 with Table S1's time step
        {"name": "continuous_toric32_minsum", "kind": "continuous", "code": "toric2d:32", "bp": "minsum",
         "p": 0.05, "shots": 4096, "t_max": 30.0},
        # the supplementary material's machine on the repetition code
        {"name": "bitcentric_rep101", "kind": "bitcentric", "code": "rep:101", "p": 0.3, "q": 0.1,
         "shots": 65536, "iters": 101},
        # the serving mix: 2D toric, 3D toric and bivariate-bicycle requests stepped together
        {"name": "serving_mix_64", "kind": "serving", "bp": "minsum", "p": 0.03, "shots": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _checks(name):
    fam, _, arg = name.partition(":")
    if fam == "bb":
        l, m = arg.split("x")
        return int(l) * int(m)
    k = int(arg)
    return {"toric2d": k * k, "toric3d_point": k ** 3, "toric3d_membrane": 3 * k ** 3, "rep": k}[fam]


def draw(rng):
    kind = rng.choice(["decode", "montecarlo", "montecarlo", "pipeline", "soft", "stream", "plan", "online",
                       "continuous", "bitcentric", "serving"])
    bp = rng.choice(["minsum", "sumproduct"])
    if kind == "stream":
        code = rng.choice(["toric3d_membrane:%d" % rng.randint(12, 16), "toric3d_point:%d" % rng.randint(22, 24)])
        return {"kind": "montecarlo", "code": code, "bp": "minsum", "p": round(rng.uniform(0.01, 0.03), 4),
                "shots": _log(rng, 32, 768), "rounds": 4 * int(code.split(":")[1])}
    if kind == "plan":
        return {"kind": "plan", "plan": rng.choice(sorted(PLANS)), "bp": "minsum",
                "p": round(rng.uniform(0.005, 0.04), 4), "shots": _log(rng, 16, 8192)}
    if kind == "online":
        L = rng.randint(6, 16)
        w = rng.randint(2, 4)
        return {"kind": "online", "code": "toric2d:%d" % L, "bp": bp, "p": round(rng.uniform(0.004, 0.012), 4),
                "shots": _log(rng, 16, 8192), "rounds": 16, "rounds_total": rng.randint(4, 16), "window": w,
                "commit": rng.randint(1, w - 1)}
    if kind == "continuous":
        L = rng.randint(8, 32)
        top = 4096 if bp == "minsum" else 512
        return {"kind": "continuous", "code": "toric2d:%d" % L, "bp": bp, "p": round(rng.uniform(0.02, 0.05), 4),
                "shots": _log(rng, 16, top), "t_max": float(rng.randint(10, 30))}
    if kind == "bitcentric":
        d = rng.randint(5, 128)
        return {"kind": "bitcentric", "code": "rep:%d" % d, "p": round(rng.uniform(0.05, 0.35), 4), "q": 0.1,
                "shots": _log(rng, 16, 65536), "iters": d}
    if kind == "serving":
        return {"kind": "serving", "bp": "minsum", "p": round(rng.uniform(0.01, 0.03), 4),
                "shots": rng.randint(4, 64)}
    code = rng.choice(["toric2d:%d" % rng.randint(4, 64), "toric2d:%d" % (8 * rng.randint(1, 5)),
                       "toric3d_point:%d" % rng.randint(4, 12), "toric3d_membrane:%d" % rng.randint(4, 8),
                       "bb:6x6", "bb:12x6", "rep:%d" % rng.randint(9, 201)])
    arg = code.split(":")[1]
    rounds = 96 if "x" in arg else (4 * int(arg) if not code.startswith("rep") else 64)
    p = round(rng.uniform(0.01, 0.04) if not code.startswith("toric2d") else rng.uniform(0.01, 0.06), 4)
    if code.startswith("bb"):
        p = round(rng.uniform(0.002, 0.03), 4)
    # shots times checks at most those of the listed cases of the same rule
    top = (1 << 26 if bp == "minsum" else 1 << 21) // _checks(code)
    shots = _log(rng, 1 if kind == "decode" else 64, max(128, min(top, 65536)))
    if kind == "soft":
        return {"kind": "soft", "code": code, "bp": "sumproduct", "p": p, "shots": min(shots, 4096), "rounds": 1}
    c = {"kind": kind, "code": code, "bp": bp, "p": p, "shots": shots, "rounds": rounds}
    if rng.random() < 0.4:
        c["conflict"] = rng.choice(["xor", "sequential"])
    if c.get("conflict") != "sequential" and rng.random() < 0.3:
        c["move"] = "multi"
    return c


def _params(case, name, rounds, seed):
    return laim.DecodeParams(bp=case["bp"], q=prior(name), rounds=rounds, seed=seed,
                             conflict=case.get("conflict", "or"), move=case.get("move", "single"))


def _errors(code, p, shots, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return (torch.rand((shots, code.n), generator=g, device="cuda") < p).to(torch.uint8)


def _outputs(code, shots):
    u8 = {"dtype": torch.uint8, "device": "cuda"}
    return {"z": torch.empty((shots, code.n), **u8), "s": torch.empty((shots, code.m), **u8),
            "tclr": torch.empty((shots,), dtype=torch.int32, device="cuda"),
            "fail": torch.empty((shots,), **u8), "L": None}


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "seed": seed}
    if kind == "serving":
        st["server"] = laim.Server(0, mem_budget=64 << 20, max_slots=256)
        st["mix"] = []
        for name, rounds in MIX:
            st["mix"].append((laim.Code(codes.by_name(name), 0), _params(case, name, rounds, seed)))
        return st
    if kind == "plan":
        items = []
        for k, (name, rounds) in enumerate(PLANS[case["plan"]]):
            code = laim.Code(codes.by_name(name), 0)
            # each code at the plan's noise rate and at half of it
            for h, p in enumerate((case["p"], case["p"] / 2)):
                items.append({"code": code, "params": _params(case, name, rounds, seed), "shot0": k << 32,
                              "e0": _errors(code, p, case["shots"], 1000 * seed + 2 * k + h)})
        st["plan"] = laim.BatchPlan(items)
        return st
    code = st["code"] = laim.Code(codes.by_name(case["code"]), 0)
    shots = case["shots"]
    st["shot0"] = (seed % 65521) << 20
    if kind == "online":
        st["plan"] = laim.OnlinePlan(code, laim.OnlineParams(case["rounds_total"], case["window"], case["commit"],
                                                             case["p"], case["p"]))
        st["params"] = _params(case, case["code"], case["rounds"], seed)
        n = max(256, st["plan"].workspace_bytes(st["params"], shots))
        st["ws"] = torch.empty((n,), dtype=torch.uint8, device="cuda")
        return st
    if kind in ("continuous", "bitcentric"):
        st["e0"] = _errors(code, case["p"], shots, seed)
        if kind == "continuous":
            st["params"] = laim.ContinuousParams(bp=case["bp"], q=prior(case["code"]), t_max=case["t_max"],
                                                 seed=seed)
        return st
    st["params"] = _params(case, case["code"], case["rounds"], seed)
    n = max(256, laim.workspace_bytes(code, st["params"], shots))
    st["ws"] = torch.empty((n,), dtype=torch.uint8, device="cuda")
    if kind in ("decode", "montecarlo"):
        st["out"] = _outputs(code, shots)
    if kind in ("montecarlo", "pipeline"):
        st["e0"] = torch.empty((shots, code.n), dtype=torch.uint8, device="cuda")
    else:
        st["e0"] = _errors(code, case["p"], shots, seed)
    return st


def run(st):
    case, kind, seed = st["case"], st["case"]["kind"], st["seed"]
    if kind == "serving":
        srv, order, res = st["server"], [], {}
        for i in range(case["shots"]):
            code, params = st["mix"][i % len(st["mix"])]
            order.append(srv.submit(code, params, seed * 1000 + i, None, case["p"]))
        while len(res) < len(order):
            for ev in srv.step():
                if ev["done"]:
                    res[ev["ticket"]] = (srv.result(ev["ticket"]), ev["fail"], ev["round"])
        r = [res[t] for t in order]
        return {"z": np.concatenate([x[0]["z"] for x in r]), "s": np.concatenate([x[0]["s"] for x in r]),
                "tclr": np.array([x[0]["tclr"] for x in r]), "fail": np.array([x[1] for x in r]),
                "rounds": np.array([x[2] for x in r])}
    if kind == "plan":
        return [{k: o[k] for k in ("z", "s", "tclr", "fail")} for o in st["plan"].launch()]
    code, shots = st["code"], case["shots"]
    if kind == "online":
        o = st["plan"].decode(st["params"], shots, shot0=st["shot0"], workspace=st["ws"])
        return {k: o[k] for k in ("z", "E", "fail", "cleared")}
    if kind == "continuous":
        o = laim.decode_continuous(code, st["params"], st["e0"], shot0=st["shot0"], want_fail=True)
        return {k: o[k] for k in ("z", "s", "tclr", "counts", "fail")}
    if kind == "bitcentric":
        o = laim.decode_bitcentric(code, case["q"], st["e0"], case["iters"], want_beliefs=True)
        return {k: o[k] for k in ("z", "iclr", "L")}
    if kind == "soft":
        o = laim.decode_rounds(code, st["params"], st["e0"], shot0=st["shot0"], want_beliefs=True,
                               workspace=st["ws"])
        return {k: o[k] for k in ("L", "z", "s", "tclr")}
    if kind == "pipeline":
        e0 = laim.sample_noise(code, case["p"], seed, st["shot0"], shots, out=st["e0"])
        s0 = laim.syndrome(code, e0)
        o = laim.decode_rounds(code, st["params"], e0, shot0=st["shot0"], workspace=st["ws"])
        fail = laim.logical_failure(code, e0, o["z"])
        return {"e0": e0, "s0": s0, "z": o["z"], "s": o["s"], "tclr": o["tclr"], "fail": fail}
    e0 = st["e0"]
    if kind == "montecarlo":
        laim.sample_noise(code, case["p"], seed, st["shot0"], shots, out=e0)
    o = laim.decode_rounds(code, st["params"], e0, shot0=st["shot0"], workspace=st["ws"], out=st["out"],
                           want_fail=True)
    out = {k: o[k] for k in ("z", "s", "tclr", "fail")}
    if kind == "montecarlo":
        out["e0"] = e0
    return out


# FP32 operations of one check in one BP sweep: the qubit-side sums, the
# sign and minimum (min-sum) or the prefix and suffix box-plus folds
# (sum-product, 62 operations a step), and the outputs' scales and signs.
def _check_ops(bp, dc, dv):
    q = dc * (dv - 1)
    if bp == "minsum":
        return q + (dc + 1) // 2 + 1 + dc * max(1, (dc - 1) // 2) + 2 * dc
    return q + 2 + 62 * 3 * max(0, dc - 2) + 3 * dc


def _shape(name):
    """(n, m, check degree, qubit degree) of a code."""
    m = _checks(name)
    fam = name.partition(":")[0]
    return {"toric2d": (2 * m, m, 4, 2), "toric3d_point": (3 * m, m, 6, 2), "toric3d_membrane": (m, m, 4, 4),
            "bb": (2 * m, m, 6, 3), "rep": (m, m, 2, 2)}[fam]


def work(case):
    """Inputs read once and outputs written once; of the operations the one
    round (its 20 sweeps) that every shot with a defect runs at the least --
    how many rounds follow depends on the errors."""
    kind = case["kind"]
    if kind in ("plan", "serving"):
        share = 1 if kind == "plan" else 1.0 / len(MIX)
        b = f = 0.0
        for name, _ in PLANS[case["plan"]] if kind == "plan" else MIX:
            n, m, dc, dv = _shape(name)
            k = case["shots"] * share * (2 if kind == "plan" else 1)
            b += k * (((2 if kind == "plan" else 1) * n) + m + 5)
            f += k * 20 * m * _check_ops(case["bp"], dc, dv)
        return {"bytes": b, "flops": f}
    n, m, dc, dv = _shape(case["code"])
    S = case["shots"]
    if kind == "bitcentric":  # one sum per message and one per belief, in every iteration
        return {"bytes": S * (2.0 * n + 4 + 8 * n), "flops": S * 3.0 * n * case["iters"]}
    ops = m * _check_ops(case["bp"], dc, dv)
    if kind == "online":
        windows = 1 + max(0, -(-(case["rounds_total"] - case["window"]) // case["commit"]))
        return {"bytes": S * (2.0 * n + 5), "flops": S * 20.0 * ops * case["window"] * windows}
    if kind == "continuous":  # 100 Euler steps are one relaxation time
        return {"bytes": S * (2.0 * n + m + 17), "flops": S * 100.0 * ops}
    b = 2.0 * n + m + 5
    if kind == "pipeline":
        b += m
    if kind == "soft":
        b += 4.0 * n
    return {"bytes": S * b, "flops": S * 20.0 * ops}


def _boxplus(a, b):
    s = torch.sign(a) * torch.sign(b)
    mn = torch.minimum(a.abs(), b.abs())
    c = torch.log1p(torch.exp(-(a.abs() + b.abs()))) - torch.log1p(torch.exp(-(a.abs() - b.abs()).abs()))
    return s * torch.clamp(mn + c, min=0.0)


def _exact_beliefs(spec, e0, q, clamp=1000.0, sweeps=20):
    """Sum-product flooding BP in float64 on a code whose checks all have one
    degree: beliefs after `sweeps` sweeps, messages starting at 0. A shot whose
    syndrome is clear at the start stops there, with the prior as its beliefs."""
    m, n = spec.m, spec.n
    nb = torch.as_tensor(spec.H.col.astype(np.int64), device=e0.device).view(m, -1)
    dc = nb.shape[1]
    pi = math.log(q / (1.0 - q))
    s = e0.to(torch.int64)[:, nb.reshape(-1)].view(-1, m, dc).sum(-1) & 1
    sign = (1 - 2 * ((s + dc) & 1)).to(torch.float64).unsqueeze(-1)
    mc = torch.zeros((e0.shape[0], m, dc), dtype=torch.float64, device=e0.device)
    L = None
    idx = nb.reshape(1, -1).expand(e0.shape[0], -1)
    for it in range(sweeps):
        if it == 0:
            x = torch.zeros_like(mc)
        else:
            x = torch.clamp(L.gather(1, idx).view_as(mc) - mc, -clamp, clamp)
        xs = [x[..., j] for j in range(dc)]
        pre, suf = [xs[0]], [xs[-1]]
        for j in range(1, dc - 1):
            pre.append(_boxplus(pre[-1], xs[j]))
            suf.append(_boxplus(xs[dc - 1 - j], suf[-1]))
        out = [suf[dc - 2]]
        for j in range(1, dc - 1):
            out.append(_boxplus(pre[j - 1], suf[dc - 2 - j]))
        out.append(pre[dc - 2])
        mc = torch.clamp(sign * torch.stack(out, -1), -clamp, clamp)
        L = torch.full((e0.shape[0], n), pi, dtype=torch.float64, device=e0.device)
        L.scatter_add_(1, idx, mc.reshape(e0.shape[0], -1))
    L = torch.where(s.any(1, keepdim=True), L, torch.full_like(L, pi))
    return torch.clamp(L, -clamp, clamp)


def _exact_bitcentric(d, q, e0, iters):
    """The bit-centric machine on the cycle of d bits (check c holds bits c
    and c + 1) as the supplementary material writes it, in float64."""
    pi0 = math.log(q / (1.0 - q))
    e = e0.to(torch.int64)
    S = e.shape[0]
    f64 = {"dtype": torch.float64, "device": e0.device}
    # messages of bit v with its check v ("own") and its check v - 1 ("prev")
    zero = torch.zeros((S, d), **f64)
    cv_own, cv_prev, vc_own, vc_prev = zero, zero, zero, zero
    pi = torch.full((S, d), pi0, **f64)
    s = e ^ e.roll(-1, 1)  # check c: bits c, c + 1
    z = torch.zeros_like(e)
    iclr = torch.where(s.any(1), -1, 0).to(torch.int32)
    L = pi.clone()
    for i in range(1, iters + 1):
        sg = (1 - 2 * s).to(torch.float64)
        n_cv_own = sg * vc_prev.roll(-1, 1)  # check v, from bit v + 1
        n_cv_prev = (sg * vc_own).roll(1, 1)  # check v - 1, from bit v - 1
        n_vc_own = pi + cv_prev
        n_vc_prev = pi + cv_own
        L = (pi + cv_prev) + cv_own  # ascending checks
        L[:, 0] = (pi[:, 0] + cv_own[:, 0]) + cv_prev[:, 0]
        f = (L > 0).to(torch.int64)
        z = z ^ f
        s = s ^ f ^ f.roll(-1, 1)
        t = (1 - 2 * f).to(torch.float64)
        pi, cv_own, cv_prev = t * pi, t * n_cv_own, t * n_cv_prev
        vc_own, vc_prev = t * n_vc_own, t * n_vc_prev
        iclr = torch.where((iclr < 0) & ~s.any(1), torch.full_like(iclr, i), iclr)
    return {"z": z.to(torch.uint8), "iclr": iclr, "L": L}


def exact(case, seed):
    if case["kind"] == "bitcentric":
        spec = codes.by_name(case["code"])
        return _exact_bitcentric(spec.n, case["q"], _errors(spec, case["p"], case["shots"], seed), case["iters"])
    if case["kind"] == "soft" and case["rounds"] == 1:
        spec = codes.by_name(case["code"])
        e0 = _errors(spec, case["p"], case["shots"], seed)
        step = max(1, (1 << 25) // spec.H.nnz)
        L = torch.cat([_exact_beliefs(spec, e0[a:a + step], prior(case["code"])) for a in range(0, case["shots"], step)])
        return {"L": L, "z": None, "s": None, "tclr": None}
    return None  # whole numbers, decided by 32-bit messages whose order of rounding is part of the method
