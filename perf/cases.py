"""The work that is measured for speed: what a program does with the library
through its public entry points, over the range of sizes, coupling families,
precisions and options that it offers.

A case is a dict of plain values; `kind` says which calls one pass makes:

* ``block``     a context kept by the program is advanced by K steps and the
                best solution per run is read out (sbqa_step, sbqa_best): how a
                long anneal is followed block by block;
* ``solve``     one whole solve from host arrays: sbqa_create, all steps of the
                schedule, sbqa_best, sbqa_destroy;
* ``handover``  a state given by the program is advanced and taken back
                (sbqa_set_state, sbqa_step, sbqa_get_state): warm starts and
                checkpoints;
* ``energy``    energies of given configurations (sbqa_energy);
* ``serve``     a batch of requests of mixed size and density through a running
                server (sbqa_submit from a few client threads, sbqa_poll).

Coupling families: ``sk`` (dense +-1), ``gauss`` (dense N(0,1)), ``sidon``
(dense integers +-8, +-13, +-19, +-28), ``regular`` (random graph of degree d,
N(0,1) weights, fields N(0, 0.1^2)), ``cubic`` (periodic L^3 lattice, the same
weights and fields), ``heavy_hex`` (pairs and native three-body terms).
"""
from __future__ import annotations

import time
from concurrent.futures import ThreadPoolExecutor
from functools import lru_cache

import numpy as np
import torch

import paper_2604_01050_amd as sb
import sbqa_instances as inst

PRECISIONS = {"auto": sb.PREC_AUTO, "fp32": sb.PREC_FP32, "fp8": sb.PREC_FP8, "bf16x3": sb.PREC_BF16X3}
F_MODES = {"ternary": sb.F_TERNARY, "ballistic": sb.F_BALLISTIC}


def listed():
    return [
        # the smallest call: one all-to-all instance of 64 spins, solved whole
        dict(name="sk64_solve", kind="solve", family="sk", N=64, R=8, runs=4, K=1000, precision="auto", f="ternary"),
        # a dense +-1 instance of some hundred spins, an odd size, at the usual 16 x 8 replicas
        dict(name="sk_mid", kind="block", family="sk", N=601, R=16, runs=8, K=200, precision="auto", f="ternary"),
        # the large dense +-1 instance, default precision
        dict(name="sk_large", kind="block", family="sk", N=16384, R=16, runs=16, K=40, precision="auto", f="ternary"),
        # real couplings and a real-valued operand in split bf16, read out with float64 energies
        dict(name="gauss_split", kind="block", family="gauss", N=8192, R=16, runs=32, K=8, precision="bf16x3",
             f="ballistic"),
        # integer couplings, the best solution tracked along the way
        dict(name="sidon_tracked", kind="block", family="sidon", N=6000, R=16, runs=16, K=40, precision="auto",
             f="ternary", track=20),
        # the throughput workload: degree 6, 2048 replica columns, short blocks
        dict(name="sparse_block", kind="block", family="regular", N=4096, d=6, R=32, runs=64, K=20, f="ternary"),
        # an ordinary sparse instance solved whole with the default schedule
        dict(name="sparse_solve", kind="solve", family="regular", N=1000, d=3, R=16, runs=8, K=1000, f="ternary"),
        # a lattice far larger than the caches
        dict(name="cubic_block", kind="block", family="cubic", L=64, R=16, runs=8, K=20, f="ternary"),
        # native three-body terms
        dict(name="three_body", kind="block", family="heavy_hex", L=100, R=16, runs=8, K=50, f="ternary"),
        # mixed requests, half dense and half sparse
        dict(name="serve_mixed", kind="serve", requests=16, lo=256, hi=4096, R=16, runs=8, K=400),
        # energies of configurations from elsewhere
        dict(name="energies", kind="energy", family="gauss", N=3000, count=200),
        # a state handed in, advanced and taken back
        dict(name="handover", kind="handover", family="gauss", N=1500, R=10, runs=6, K=100, precision="fp32",
             f="ballistic"),
    ]


def _between(rng, lo, hi):
    """An integer in [lo, hi], spread evenly over the logarithm."""
    return int(min(hi, max(lo, round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    what = rng.choice(["dense", "dense", "dense", "sparse", "sparse", "sparse", "cubic", "heavy_hex", "solve",
                       "energy", "handover", "serve"])
    R, runs = rng.choice([4, 8, 10, 16, 16, 32]), _between(rng, 1, 16)
    if what == "dense":
        family, precision, f = rng.choice([("sk", "auto", "ternary"), ("sk", "fp8", "ternary"),
                                           ("sidon", "auto", "ternary"), ("gauss", "auto", "ternary"),
                                           ("gauss", "bf16x3", "ballistic")])
        case = dict(kind="block", family=family, N=_between(rng, 48, 6000), R=R, runs=runs, K=_between(rng, 10, 100),
                    precision=precision, f=f)
        if family != "gauss" and rng.random() < 0.25:
            case["track"] = max(5, case["K"] // 3)
        return case
    if what == "sparse":
        return dict(kind="block", family="regular", N=_between(rng, 200, 60000), d=rng.randint(3, 12), R=R, runs=runs,
                    K=_between(rng, 20, 200), f=rng.choice(["ternary", "ternary", "ternary", "ballistic"]))
    if what == "cubic":
        return dict(kind="block", family="cubic", L=rng.randint(10, 60), R=R, runs=rng.randint(1, 8),
                    K=_between(rng, 10, 40), f="ternary")
    if what == "heavy_hex":
        return dict(kind="block", family="heavy_hex", L=rng.randint(10, 100), R=R, runs=rng.randint(1, 8),
                    K=_between(rng, 10, 50), f="ternary")
    if what == "solve":
        if rng.random() < 0.5:
            return dict(kind="solve", family="sk", N=_between(rng, 16, 1200), R=R, runs=rng.randint(1, 8),
                        K=_between(rng, 100, 1000), precision="auto", f="ternary")
        return dict(kind="solve", family="regular", N=_between(rng, 100, 8000), d=rng.randint(3, 8), R=R,
                    runs=rng.randint(1, 8), K=_between(rng, 100, 1000), f="ternary")
    if what == "energy":
        family = rng.choice(["gauss", "sk", "regular"])
        case = dict(kind="energy", family=family, N=_between(rng, 100, 4000), count=_between(rng, 1, 300))
        if family == "regular":
            case.update(N=_between(rng, 100, 60000), d=rng.randint(3, 12))
        return case
    if what == "handover":
        return dict(kind="handover", family="gauss", N=_between(rng, 60, 1500), R=rng.choice([1, 4, 7, 10, 16]),
                    runs=rng.randint(1, 6), K=_between(rng, 10, 100), precision=rng.choice(["fp32", "bf16x3"]),
                    f="ballistic")
    return dict(kind="serve", requests=rng.randint(4, 16), lo=256, hi=_between(rng, 512, 4096), R=16, runs=8,
                K=_between(rng, 100, 400))


# ------------------------------------------------------------------ instances
def _dense(family, N, seed):
    """Symmetric float64 couplings with a zero diagonal (drawn on the GPU: a
    host draw of the largest takes longer than its solve)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if family == "gauss":
        A = torch.randn((N, N), generator=g, device="cuda", dtype=torch.float64)
    else:
        A = torch.randint(0, 2, (N, N), generator=g, device="cuda", dtype=torch.int8).to(torch.float64) * 2 - 1
        if family == "sidon":
            mag = torch.tensor(inst.SIDON28, device="cuda", dtype=torch.float64)
            A *= mag[torch.randint(0, 4, (N, N), generator=g, device="cuda", dtype=torch.uint8).to(torch.int32)]
    A.triu_(1)
    A += A.T.clone()
    return A.cpu().numpy()


def _graph(N, d, rng):
    """Edges of a random graph of degree at most d, d reached almost
    everywhere: d // 2 random Hamiltonian cycles, and one matching if d is odd."""
    parts = []
    for _ in range(d // 2):
        p = rng.permutation(N)
        parts.append(np.stack([p, np.roll(p, 1)], 1))
    if d % 2:
        p = rng.permutation(N)[: N // 2 * 2]
        parts.append(p.reshape(-1, 2))
    E = np.sort(np.concatenate(parts), axis=1).astype(np.int64)
    return np.unique(E, axis=0)


@lru_cache(maxsize=4)
def _heavy_hex_terms(L):
    """The pairs and triples of the L x L heavy-hexagon instance (its weights
    are drawn for each instance)."""
    N, pairs, _, triples, _ = inst.hubo_heavy_hex(L, L, 2301)
    return N, pairs, triples


def _instance(case, seed):
    """Keyword arguments of sbqa_create for the case's couplings and fields."""
    family = case["family"]
    rng = np.random.default_rng(seed)
    if family in ("sk", "gauss", "sidon"):
        out = dict(J=_dense(family, case["N"], seed))
        if family == "gauss":
            out["h"] = rng.standard_normal(case["N"]) * 0.1
        return out
    if family == "heavy_hex":
        N, pairs, triples = _heavy_hex_terms(case["L"])
        return dict(csr=inst.edges_to_csr(N, pairs, rng.standard_normal(len(pairs))), tri=triples,
                    K=rng.standard_normal(len(triples)))
    if family == "cubic":
        N, E = case["L"] ** 3, inst.cubic_lattice(case["L"])
    else:
        N, E = case["N"], _graph(case["N"], case["d"], rng)
    return dict(csr=inst.edges_to_csr(N, E, rng.standard_normal(len(E))), h=rng.standard_normal(N) * 0.1)


def _schedule(case, steps, seed):
    kw = dict(R=case["R"], runs=case["runs"], steps=steps, seed=seed, fmode=F_MODES[case.get("f", "ternary")],
              energy_every=case.get("track", 0))
    if "precision" in case:
        kw["precision"] = PRECISIONS[case["precision"]]
    return kw


def _long_schedule(case):
    """Steps of a context that is advanced block by block: enough blocks for a
    long session, the coupling table within 64 MB."""
    return int(min(case["K"] * 20000, (1 << 24) // case["runs"], 1 << 21))


LINEAR = dict(jp_kind=sb.JP_LINEAR, jp_start=0.5, jp_end=0.0)


def _sizes(case):
    """Sizes of a batch of requests, spread over the logarithm."""
    q = case["requests"]
    return np.exp(np.log(case["lo"]) + (np.arange(q) + 0.5) / q * np.log(case["hi"] / case["lo"])).astype(int)


def _requests(case, seed):
    """The batch, alternately dense +-1 and sparse, in mixed order."""
    rng = np.random.default_rng(seed)
    out = []
    for k, N in enumerate(_sizes(case)):
        N = int(N)
        if k % 2 == 0:
            item = dict(J=_dense("sk", N, seed + k), precision=sb.PREC_FP8)
        else:
            E = _graph(N, int(rng.integers(3, 13)), rng)
            item = dict(csr=inst.edges_to_csr(N, E, rng.standard_normal(len(E))))
        out.append(dict(item, R=case["R"], runs=case["runs"], steps=case["K"], seed=seed + k, **LINEAR))
    return [out[k] for k in np.random.default_rng(5001).permutation(len(out))]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return dict(case=case, server=sb.sbqa_server_create(8 << 30, 32), items=_requests(case, seed),
                    clients=ThreadPoolExecutor(max_workers=4))
    problem = _instance(case, seed)
    if kind == "solve":
        return dict(case=case, problem=problem, schedule=_schedule(case, case["K"], seed))
    if kind == "energy":
        N = len(problem["J"]) if "J" in problem else len(problem["csr"][0]) - 1
        return dict(case=case, context=sb.sbqa_create(**problem, R=1, runs=1, steps=1),
                    spins=inst.spins_pm1(case["count"], N, seed + 1))
    context = sb.sbqa_create(**problem, **_schedule(case, _long_schedule(case), seed), **LINEAR)
    state = dict(case=case, context=context)
    if kind == "handover":
        state["x"], state["y"] = inst.uniform_state(context.N, context.C, 0.1, seed + 1)
    sb.sbqa_sync(context)
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "block":
        sb.sbqa_step(state["context"], case["K"])
        return sb.sbqa_best(state["context"])
    if kind == "solve":
        context = sb.sbqa_create(**state["problem"], **state["schedule"])
        sb.sbqa_step(context, case["K"])
        best = sb.sbqa_best(context)
        sb.sbqa_destroy(context)
        return best
    if kind == "energy":
        return sb.sbqa_energy(state["context"], state["spins"])
    if kind == "handover":
        sb.sbqa_set_state(state["context"], state["x"], state["y"])
        sb.sbqa_step(state["context"], case["K"])
        return sb.sbqa_get_state(state["context"])
    server = state["server"]
    tickets = list(state["clients"].map(lambda item: sb.sbqa_submit(server, **item), state["items"]))
    done = {}
    while len(done) < len(tickets):
        for k, t in enumerate(tickets):
            if k not in done:
                r = sb.sbqa_poll(server, t)
                if r is not None:
                    done[k] = r[:2]
        time.sleep(0.0002)
    return [done[k] for k in range(len(tickets))]


# ----------------------------------------------------------------------- work
def _size(case):
    """(spins, coupling bytes, coupling terms) of the case's instance."""
    family = case["family"]
    if family in ("sk", "gauss", "sidon"):
        N = case["N"]
        return N, N * N * {"sk": 0.125, "sidon": 1, "gauss": 4}[family], N * N
    if family == "heavy_hex":
        N, pairs, triples = _heavy_hex_terms(case["L"])
        return N, 16 * len(pairs) + 36 * len(triples), 2 * len(pairs) + 6 * len(triples)
    N = case["L"] ** 3 if family == "cubic" else case["N"]
    nnz = N * (6 if family == "cubic" else case["d"])
    return N, 8 * nnz + 4 * N, nnz


def work(case):
    """The couplings once (in the form the contraction takes), the state read
    and written once, the results; two operations for each term of the coupling
    sum and 13 for each update."""
    if case["kind"] == "serve":
        sizes = _sizes(case).astype(np.float64)
        C = case["R"] * case["runs"]
        dense, sparse = sizes[::2], sizes[1::2]
        return {"bytes": float((dense ** 2).sum() / 8 + (sparse * 60).sum() + 16 * C * sizes.sum() + case["runs"] * sizes.sum()),
                "flops": float(case["K"] * C * (2 * (dense ** 2).sum() + 15 * sparse.sum() + 13 * sizes.sum()))}
    N, jbytes, terms = _size(case)
    if case["kind"] == "energy":
        jbytes = 8 * terms if case["family"] in ("sk", "gauss") else 12 * terms
        return {"bytes": jbytes + case["count"] * (N + 8.0), "flops": 2.0 * terms * case["count"]}
    C, K = case["R"] * case["runs"], case["K"]
    results = 8 * N * C if case["kind"] == "handover" else case["runs"] * (N + 8)
    return {"bytes": float(jbytes + 16 * N * C + results), "flops": float(K * C * (2 * terms + 13 * N))}


# ---------------------------------------------------------------------- exact
def exact(case, seed):
    """Energies and few-step states in float64; a whole anneal is chaotic (its
    end depends on every rounding on the way) and has no such value."""
    if case["kind"] == "energy":
        problem = _instance(case, seed)
        N = len(problem["J"]) if "J" in problem else len(problem["csr"][0]) - 1
        s = inst.spins_pm1(case["count"], N, seed + 1).astype(np.float64)
        h = problem.get("h")
        if "J" in problem:
            Js = s @ problem["J"]
        else:
            ptr, col, val = problem["csr"]
            rows = np.repeat(np.arange(N), np.diff(ptr))
            Js = np.zeros_like(s)
            for m in range(len(s)):
                Js[m] = np.bincount(rows, weights=val * s[m, col], minlength=N)
        return -0.5 * (s * Js).sum(1) - (s @ h if h is not None else 0.0)
    if case["kind"] != "handover":
        return None
    problem = _instance(case, seed)
    J, h = problem["J"], problem["h"]
    N, R, runs, S = len(J), case["R"], case["runs"], _long_schedule(case)
    x, y = (a.astype(np.float64) for a in inst.uniform_state(N, R * runs, 0.1, seed + 1))
    c0 = 0.5 / (np.sqrt(N) * np.sqrt((J * J).sum() / (N * (N - 1.0))))
    for n in range(case["K"]):
        ring = x.reshape(N, runs, R)
        ring = (np.roll(ring, 1, 2) + np.roll(ring, -1, 2)).reshape(N, -1)
        force = -(1.0 - n / S) / R * x + c0 / R * (J @ x + h[:, None]) + (0.5 - 0.5 * n / S) * ring
        y = y + 0.5 * force
        x = x + 0.5 / R * y
        wall = np.abs(x) > 1.0
        x[wall] = np.sign(x[wall])
        y[wall] = 0.0
    return x, y
