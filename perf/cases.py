"""The work this library is used for, as cases that can be timed.

A case is one call (or one short stream of calls) through the public binding `sa`: a one-shot
run on host buffers, a run of a prepared plan into device buffers, a batch of instances in one
launch, or a burst of requests to the server.  `listed()` names the cases, `draw()` gives others of
the same ranges, `prepare()` makes what a program holds before the call (instances, plan, batch,
server and output buffers; the instance and the annealing key both follow the seed), `run()` makes
one pass, `work()` counts what the path cannot do without.

States and energies are integers that follow the seed's random stream exactly, so two passes on
the same inputs return the same numbers.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

from paper_2511_17245_amd import inputs as I
from paper_2511_17245_amd import sa

RULES = ("metropolis", "heat_bath", "otm", "heat_bath_closed")
POLY_RULES = {"metropolis": sa.METROPOLIS, "heat_bath": sa.HEAT_BATH, "otm": sa.OPT_METROPOLIS,
              "heat_bath_closed": sa.HEAT_BATH_CLOSED}


def _plan_case(name, family, rule, sweeps, reads, **shape):
    return dict(name=name, call="plan", family=family, rule=rule, sweeps=sweeps, reads=reads, **shape)


def listed():
    return [
        # a first try from a notebook or a small sub-problem inside another solver: one call on
        # host buffers, where preparation, launches and copies are most of the time
        dict(name="oneshot_huio_n30", call="oneshot", family="huio", rule="heat_bath", sweeps=100, reads=8,
             n=30, lo=-7, hi=9, monomials=180, jmax=5),
        # the dense N = 100 problem with its given schedule, few reads: one dependent chain per read
        _plan_case("dense_n100_metropolis", "dense", "metropolis", 1000, 16, n=100, lo=0, hi=15, jmax=10,
                   given_beta=True),
        # the fully connected model of the paper's Figs. 1 and 3 at its sample count
        _plan_case("fc_n100_p2_u100_heat_bath", "fc", "heat_bath", 300, 1000, n=100, p=2, u=100),
        # the multilinear model of Figs. 2, 4, 6 and 8: a ring, long terms, few independent updates
        _plan_case("ml_n100_p10_u10_otm", "ml", "otm", 300, 100, n=100, p=10, u=10),
        # random-interaction realizations of Figs. 3, 5 and 7, all in one launch
        dict(name="ri_n100_p4_u100_batch", call="batch", family="ri", rule="heat_bath", sweeps=100, reads=100,
             problems=32, n=100, p=4, u=100, monomials=1000, graph=False),
        # the sparse N = 10^4 heat bath, the configuration the throughput is quoted on
        _plan_case("sparse_n10000_heat_bath", "sparse", "heat_bath", 2000, 256, n=10000, lo=-50, hi=50,
                   degree=8.0, jmax=10, hmax=20),
        # a sparse model whose variables come from different sources: ranges of 2 to 120 values
        _plan_case("sparse_n3001_mixed_heat_bath", "sparse", "heat_bath", 400, 96, n=3001, lo=-60, hi=59,
                   degree=8.0, jmax=10, hmax=20, mixed=True),
        # the higher-order N = 2000 problem under both rules it is measured with
        _plan_case("huio_n2000_otm", "huio", "otm", 300, 1024, n=2000, lo=0, hi=100, monomials=20000, jmax=5),
        _plan_case("huio_n2000_metropolis", "huio", "metropolis", 300, 1024, n=2000, lo=0, hi=100,
                   monomials=20000, jmax=5),
        # the widest request of the served mix: dense couplings, 2001 values per variable
        _plan_case("dense_n4096_w2001_heat_bath", "dense", "heat_bath", 20, 16, n=4096, lo=-1000, hi=1000, jmax=10),
        # many unrelated instances of uneven size, width and rule in one graph-replayed launch
        dict(name="mixed_batch_64", call="batch", family="mixed", rule="mixed", sweeps=200, reads=32, problems=64,
             n_min=50, n_max=5000, w_min=2, w_max=1000, graph=True),
        # a burst of requests to a running server: nine in ten higher-order, one in ten dense and wide
        dict(name="served_burst_20", call="serve", family="served", rule="mixed", sweeps=300, reads=16, requests=20,
             n=2000, monomials=20000, dense_n=2048, dense_sweeps=20),
    ]


def _logint(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def _sweeps(n, reads, chain=1.5e5, total=2.0e8):
    """Sweeps for an instance: bounded by one read's chain and by all reads' updates."""
    return max(3, min(1000, int(chain / n), int(total / (n * reads))))


def draw(rng):
    call = rng.choice(["oneshot", "dense", "dense", "fc", "ml", "ri", "sparse", "sparse", "huio", "huio", "wide",
                       "batch", "serve"])
    rule = rng.choice(RULES)
    reads = _logint(rng, 1, 1024)
    option = rng.choice(["", "", "", "resume", "trace"])
    if call == "oneshot":
        n = _logint(rng, 5, 300)
        w = _logint(rng, 2, 200)
        reads = _logint(rng, 1, 64)
        lo = -rng.randrange(0, w)
        return dict(call="oneshot", family="huio", rule=rule, sweeps=min(300, _sweeps(n, reads)), reads=reads, n=n,
                    lo=lo, hi=lo + w - 1, monomials=rng.randrange(2, 9) * n, jmax=5)
    if call == "dense":
        n = _logint(rng, 33, 900)
        w = _logint(rng, 2, 300)
        lo = -rng.randrange(0, w)
        return _plan_case_unnamed("dense", rule, _sweeps(n, reads), reads, option, n=n, lo=lo, hi=lo + w - 1,
                                  jmax=rng.choice([3, 10, 100, 5000]), given_beta=False)
    if call == "fc":
        n = rng.randrange(40, 201)
        p = rng.choice([1, 2, 2, 3, 4])
        return _plan_case_unnamed("fc", rule, min(300, _sweeps(n, reads)), reads, option, n=n, p=p,
                                  u=_logint(rng, 1, 1000 if p <= 2 else 100))
    if call == "ml":
        n = rng.randrange(40, 201)
        p = rng.randrange(2, 11)
        return _plan_case_unnamed("ml", rule, min(300, _sweeps(n, reads)), reads, option, n=n, p=p, u=_logint(rng, 1, 20))
    if call == "ri":
        n = rng.randrange(50, 201)
        reads = _logint(rng, 10, 100)
        problems = rng.randrange(2, 32)
        return dict(call="batch", family="ri", rule=rule, sweeps=min(200, _sweeps(n, reads * problems)), reads=reads,
                    problems=problems, n=n, p=rng.choice([2, 3, 4]), u=_logint(rng, 1, 1000), monomials=10 * n,
                    graph=rng.random() < 0.5)
    if call == "sparse":
        n = _logint(rng, 100, 20000)
        w = _logint(rng, 2, 128) if rng.random() < 0.8 else _logint(rng, 129, 3000)
        lo = -rng.randrange(0, w)
        return _plan_case_unnamed("sparse", rule, _sweeps(n, reads, 6.0e5, 1.0e9), reads, option, n=n, lo=lo,
                                  hi=lo + w - 1, degree=round(rng.uniform(2.0, 12.0), 1), jmax=10, hmax=20,
                                  mixed=rng.random() < 0.4)
    if call == "huio":
        n = _logint(rng, 60, 4000)
        w = _logint(rng, 2, 128) if rng.random() < 0.8 else _logint(rng, 129, 1000)
        lo = -rng.randrange(0, w)
        return _plan_case_unnamed("huio", rule, _sweeps(n, reads, 3.0e5, 4.0e8), reads, option, n=n, lo=lo,
                                  hi=lo + w - 1, monomials=rng.randrange(3, 13) * n, jmax=5)
    if call == "wide":
        n = _logint(rng, 300, 3000)
        reads = _logint(rng, 4, 64)
        w = _logint(rng, 300, 3000)
        return _plan_case_unnamed("dense", rng.choice(["heat_bath", "heat_bath_closed"]), max(3, 40000 // n), reads, "",
                                  n=n, lo=-(w // 2), hi=-(w // 2) + w - 1, jmax=10, given_beta=False)
    if call == "batch":
        problems = rng.randrange(4, 64)
        return dict(call="batch", family="mixed", rule="mixed", sweeps=rng.randrange(20, 150),
                    reads=_logint(rng, 4, 32), problems=problems, n_min=50, n_max=rng.randrange(500, 5000), w_min=2,
                    w_max=rng.randrange(100, 1000), graph=rng.random() < 0.5)
    return dict(call="serve", family="served", rule="mixed", sweeps=rng.randrange(50, 300),
                reads=rng.randrange(4, 17), requests=rng.randrange(3, 20), n=_logint(rng, 300, 2000),
                monomials=rng.randrange(2000, 20000), dense_n=rng.randrange(200, 1500), dense_sweeps=rng.randrange(5, 20))


def _plan_case_unnamed(family, rule, sweeps, reads, option, **shape):
    c = dict(call="plan", family=family, rule=rule, sweeps=sweeps, reads=reads, **shape)
    if option:
        c["option"] = option
    return c


def _rng(seed, *more):
    return np.random.Generator(np.random.PCG64([int(seed), *more]))


def _problem(c, rng):
    f = c["family"]
    if f == "huio":
        return I.random_huio(c["n"], c["monomials"], [2, 3, 4], c["lo"], c["hi"], c["jmax"], rng)
    if f == "dense":
        return I.dense_quio(c["n"], c["lo"], c["hi"], c["jmax"], c["jmax"], rng)
    if f == "sparse":
        p = I.erdos_renyi_quio(c["n"], min(c["degree"], c["n"] - 1.0), c["lo"], c["hi"], c["jmax"], c["hmax"], rng)
        if c.get("mixed"):  # every variable a range of its own inside the box
            w = np.exp(rng.uniform(math.log(2.0), math.log(c["hi"] - c["lo"] + 1.0), size=c["n"])).astype(np.int64)
            w = np.clip(w, 2, c["hi"] - c["lo"] + 1)
            p.lower = (c["lo"] + rng.integers(0, c["hi"] - c["lo"] + 2 - w)).astype(np.int32)
            p.upper = (p.lower + w - 1).astype(np.int32)
        return p
    if f == "fc":
        return I.fully_connected(c["n"], c["p"], c["u"])
    if f == "ml":
        return I.multilinear(c["n"], c["p"], c["u"])
    if f == "ri":
        return I.random_interaction(c["n"], c["p"], c["u"], c["monomials"], rng)
    raise ValueError(f)


def _mixed_items(c, seed):
    """The mixed batch's recipe: size and width log-uniform, pair graphs and higher-order monomials in
    turn, the rules in turn.  The sizes and widths do not follow the seed, so every seed costs the same."""
    shape = _rng(c["problems"], c["n_max"], c["w_max"])
    rng = _rng(seed, 1)
    out = []
    for i in range(c["problems"]):
        n = int(round(math.exp(shape.uniform(math.log(c["n_min"]), math.log(c["n_max"])))))
        w = int(round(math.exp(shape.uniform(math.log(c["w_min"]), math.log(c["w_max"])))))
        lo = -(w // 2)
        if i % 2 == 0:
            prob = I.erdos_renyi_quio(n, 8.0, lo, lo + w - 1, 10, 10, rng)
        else:
            prob = I.random_huio(n, 10 * n, [2, 3, 4], lo, lo + w - 1, 10, rng)
        out.append(I.Workload(prob, i % 3, c["sweeps"], c["reads"], 7 + seed, i))
    return out


def _served_items(c, seed):
    rng = _rng(seed, 2)
    out = []
    for i in range(c["requests"]):
        if i % 10 == 4:
            prob = I.dense_quio(c["dense_n"], -1000, 1000, 10, 10, rng)
            out.append(I.Workload(prob, sa.HEAT_BATH, c["dense_sweeps"], c["reads"], 11 + seed + i, i))
        else:
            prob = I.random_huio(c["n"], c["monomials"], [2, 3, 4], 0, 100, 5, rng)
            rule = sa.OPT_METROPOLIS if i % 2 == 0 else sa.METROPOLIS
            out.append(I.Workload(prob, rule, c["sweeps"], c["reads"], 11 + seed + i, i))
    return out


def prepare(case, seed):
    c = dict(case)
    s = types.SimpleNamespace(case=c, seed=1000003 * (int(seed) + 1))
    if c["call"] == "oneshot":
        s.problem = _problem(c, _rng(seed))
        return s
    if c["call"] == "plan":
        prob = _problem(c, _rng(seed))
        s.plan = sa.Plan(prob, POLY_RULES[c["rule"]])
        s.z = torch.empty((c["reads"], prob.n_vars), dtype=torch.int32, device="cuda")
        s.e = torch.empty(c["reads"], dtype=torch.int64, device="cuda")
        s.beta = I.cfg1_beta(c["sweeps"]) if c.get("given_beta") else None
        s.init = s.trace = None
        s.begin = 0
        if c.get("option") == "resume":  # the second half of a run, from states the caller holds
            s.begin = c["sweeps"] // 2
            z0 = _rng(seed, 3).integers(prob.lower, prob.upper.astype(np.int64) + 1, size=(c["reads"], prob.n_vars))
            s.init = torch.from_numpy(z0.astype(np.int32)).cuda()
        if c.get("option") == "trace":
            s.trace = torch.empty((c["reads"], c["sweeps"]), dtype=torch.int64, device="cuda")
        return s
    if c["call"] == "batch":
        if c["family"] == "mixed":
            items = _mixed_items(c, int(seed))
        else:
            rng = _rng(seed, 4)
            items = [I.Workload(_problem(c, rng), POLY_RULES[c["rule"]], c["sweeps"], c["reads"], s.seed, i)
                     for i in range(c["problems"])]
        s.batch = sa.Batch(items, use_graph=c["graph"])
        return s
    s.items = _served_items(c, int(seed))
    s.server = sa.Server()
    return s


def run(s):
    c = s.case
    if c["call"] == "oneshot":
        return sa.anneal(s.problem, POLY_RULES[c["rule"]], c["sweeps"], c["reads"], s.seed)
    if c["call"] == "plan":
        s.plan.run_device(c["sweeps"], c["reads"], s.seed, s.z, s.e, beta=s.beta,
                          stream=torch.cuda.current_stream().cuda_stream, sweep_begin=s.begin, init_states=s.init,
                          trace=s.trace)
        return (s.z, s.e) if s.trace is None else (s.z, s.e, s.trace)
    if c["call"] == "batch":
        s.batch.run()
        out = s.batch.results()
        return np.concatenate([z.ravel() for z, _ in out]), np.concatenate([e for _, e in out])
    tickets = [s.server.submit(w) for w in s.items]
    for t in tickets:
        s.server.wait(t)
    out = [s.server.result(t) for t in tickets]
    return np.concatenate([z.ravel() for z, _ in out]), np.concatenate([e for _, e in out])


def _family_work(family, c, n, reads, sweeps, rule, width, monomials=0):
    """Bytes: couplings, incidences and bounds once, outputs once.  Operations: per update two for every
    coupling or other factor of the variable's terms, and for the heat bath two per candidate value."""
    if family == "dense" or family == "fc":
        per_var, inst = 2.0 * n, n * n * (4.0 if c.get("jmax", 10) > 127 else 1.0)
    elif family == "sparse":
        per_var, inst = 2.0 * c.get("degree", 8.0), 8.0 * n * c.get("degree", 8.0)
    elif family == "ml":
        per_var, inst = 2.0 * c["p"] * c["p"], 4.0 * n * c["p"]
    else:
        d = c.get("p", 3.0)
        per_var, inst = 2.0 * d * d * monomials / n, 4.0 * (d + 1) * monomials
    if rule == "heat_bath":
        per_var += 2.0 * width
    return inst + 8.0 * n + reads * (4.0 * n + 8.0), per_var * float(n) * reads * sweeps


def work(case):
    c = dict(case)
    b = f = 0.0

    def add(*a, **k):
        nonlocal b, f
        x, y = _family_work(*a, **k)
        b += x
        f += y

    if c["call"] == "batch" and c["family"] == "mixed":
        shape = _rng(c["problems"], c["n_max"], c["w_max"])
        for i in range(c["problems"]):
            n = int(round(math.exp(shape.uniform(math.log(c["n_min"]), math.log(c["n_max"])))))
            w = int(round(math.exp(shape.uniform(math.log(c["w_min"]), math.log(c["w_max"])))))
            add("sparse" if i % 2 == 0 else "huio", {}, n, c["reads"], c["sweeps"], RULES[i % 3], w, 10 * n)
    elif c["call"] == "serve":
        for i in range(c["requests"]):
            if i % 10 == 4:
                add("dense", {}, c["dense_n"], c["reads"], c["dense_sweeps"], "heat_bath", 2001)
            else:
                add("huio", {}, c["n"], c["reads"], c["sweeps"], "metropolis", 101, c["monomials"])
    else:
        width = 2 * c["u"] + 1 if "u" in c else c["hi"] - c["lo"] + 1
        sweeps = c["sweeps"] - (c["sweeps"] // 2 if c.get("option") == "resume" else 0)
        for _ in range(c.get("problems", 1)):
            add(c["family"], c, c["n"], c["reads"], sweeps, c["rule"], width, c.get("monomials", 0))
        if c.get("option") == "trace":
            b += 8.0 * c["reads"] * c["sweeps"]
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """States drawn by a seeded stream and their integer energies: there is no real number to be near to."""
    return None
