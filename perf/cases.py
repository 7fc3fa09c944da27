"""The work that users of this framework have it do, as cases that can be timed.

Every case is one pass through public entry points (GARun, GABatch, Server and
the C ABI's all-pairs relatedness call) over the shapes of this repository's
workloads, treatments, tests and benchmark: runs from one compute unit's worth
of agents to 16.8M, both selection modes, both mutation laws, the genome models,
the surface policies, both schedules, batched and served runs, and the
reconstruction step after a run. Inputs come from the seed alone.

A pass of a run case continues the run by `gens` generations and takes out what
such a program takes out: the whole population (a checkpoint, mean fitness) or
one genome per island (the paper's end-state sample).
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_2405_03605_amd import GABatch, GARun, load
from paper_2405_03605_amd.serve import Server
from paper_2405_03605_amd.workloads import ADAPTIVE, P33, batched_configs, run_config

RUN_FIELDS = ("width", "height", "pop", "sites", "k", "selection", "p32", "migration", "law",
              "p_ben32", "schedule", "model", "dbits", "policy")


def _run(name, gens, take, **kw):
    return {"name": name, "kind": "run", "gens": gens, "take": take, **kw}


def listed():
    return [
        # the smallest workload, the 8 x 8 quick start: latency of one tile
        _run("tiny_8x8x32", 1000, "state", width=8, height=8, pop=32, sites=64, k=2),
        # an odd grid of small islands, tournament 5 as in the paper: a parameter scan's run
        _run("odd_37x23x16", 500, "state", width=37, height=23, pop=16, sites=32, k=5),
        # the paper's treatment comparison at its smallest grid, 10,000 tips sampled
        _run("treatment_100x100x32", 1000, "sample", width=100, height=100, pop=32, sites=64,
             **ADAPTIVE),
        # the mid workload, 2.1M agents, held on the chip
        _run("mid_256x256x32", 5000, "state", width=256, height=256, pop=32, sites=32, k=2),
        # the paper-scale workload, 16.8M agents, streamed from HBM
        _run("paper_1024x512x32", 1000, "sample", width=1024, height=512, pop=32, sites=32, k=2),
        # a genome model with a string and the hybrid surface, large islands, too big for LDS
        _run("trap4_hybrid_300x200x64", 400, "sample", width=300, height=200, pop=64, sites=64,
             k=3, model=2, policy=2),
        # the paper's asynchronous exchange with its default pacing
        _run("async_512x256x32", 400, "sample", width=512, height=256, pop=32, sites=32, k=2,
             schedule=1),
        # the 64 uneven runs of the batched workload, sampled at the end
        {"name": "batch_64_runs", "kind": "batch", "runs": 64, "mix": 20240503, "gens": 1000},
        # a server draining a queue of uneven requests through fewer slots
        {"name": "served_queue", "kind": "serve", "requests": 24, "slots": 16, "mix": 20240504,
         "most_agents": 400000, "most_gens": 4000},
        # relatedness of the 10,000 sampled end-state genomes of a reconstruction
        {"name": "mrca_steady_10k", "kind": "mrca", "n": 10000, "sites": 32, "dbits": 1,
         "policy": 0, "kc": 5},
        # the same on the recency-proportional and the hybrid surfaces
        {"name": "mrca_tilted_10k", "kind": "mrca", "n": 10000, "sites": 32, "dbits": 1,
         "policy": 1, "kc": 5},
        {"name": "mrca_hybrid_4k", "kind": "mrca", "n": 4000, "sites": 64, "dbits": 1,
         "policy": 2, "kc": 5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["run"] * 7 + ["batch"] * 2 + ["serve"] + ["mrca"] * 3)
    if kind == "batch":
        return {"kind": "batch", "runs": rng.randint(3, 64), "mix": rng.randrange(1 << 20),
                "gens": rng.randint(100, 600)}
    if kind == "serve":
        return {"kind": "serve", "requests": rng.randint(6, 24), "slots": rng.randint(4, 24),
                "mix": rng.randrange(1 << 20), "most_agents": _log_int(rng, 2e4, 4e5),
                "most_gens": _log_int(rng, 500, 4000)}
    if kind == "mrca":
        sites, dbits, policy = rng.choice([(32, 1, 0), (64, 1, 0), (16, 4, 0), (8, 8, 0),
                                           (32, 1, 1), (64, 1, 1), (32, 2, 1), (64, 1, 2)])
        return {"kind": "mrca", "n": _log_int(rng, 200, 10000), "sites": sites, "dbits": dbits,
                "policy": policy, "kc": rng.randint(1, 8)}
    pop = rng.choice([8, 16, 32, 32, 64])
    islands = _log_int(rng, 2e3, 1.2e7) / pop
    aspect = math.exp(rng.uniform(-1.0, 1.0))
    width = min(2048, max(3, int(round(math.sqrt(islands) * aspect))))
    height = min(2048, max(3, int(round(islands / width))))
    agents = width * height * pop
    case = _run(None, 0, "sample" if agents > 400000 else rng.choice(["state", "sample"]),
                width=width, height=height, pop=pop, sites=rng.choice([32, 64]),
                k=rng.choice([2, 2, 3, 5, 5, 7]))
    del case["name"]
    case["gens"] = max(50, min(1000, int(2e9 / agents)))
    form = rng.randrange(8)
    if form == 0:
        case["selection"] = 0                        # neutral runs
    elif form == 1:
        case.update(ADAPTIVE, p32=P33)               # the paper's treatments
    elif form == 2:
        case["model"] = rng.choice([1, 2])           # OneMax, Trap-4
    elif form == 3:                                  # wider differentia, other policies
        case.update(rng.choice([{"sites": 16, "dbits": 4}, {"sites": 32, "dbits": 2},
                                {"sites": 32, "policy": 1}, {"sites": 64, "policy": 2}]))
    elif form == 4 and agents <= 4000000:
        case["schedule"] = 1                         # the asynchronous exchange, default pacing
    elif form == 5:
        case["migration"] = 0                        # the closed-islands control
    return case


# -- configurations of a case ---------------------------------------------------------------------

def _config(case, seed):
    return run_config(**{f: case[f] for f in RUN_FIELDS if f in case}, seed=seed & 0xFFFFFFFF)


def _batch_configs(case, seed):
    return [dict(c, seed=seed & 0xFFFFFFFF) for c in batched_configs(case["runs"], case["mix"])]


def _requests(case, seed):
    """Queued requests: agents log-uniform from 1,000, budgets log-uniform from 200."""
    rng = np.random.default_rng(case["mix"])
    out = []
    for r in range(case["requests"]):
        agents = math.exp(rng.uniform(math.log(1e3), math.log(case["most_agents"])))
        pop = int(rng.choice([8, 16, 32, 64]))
        islands = max(1, int(round(agents / pop)))
        width = int(math.ceil(math.sqrt(islands)))
        cfg = run_config(width=width, height=max(1, int(round(islands / width))), pop=pop,
                         sites=int(rng.choice([32, 64])), k=int(rng.integers(2, 9)),
                         selection=int(rng.integers(0, 2)), seed=seed & 0xFFFFFFFF,
                         run_id=1000 + r)
        gens = int(round(math.exp(rng.uniform(math.log(200), math.log(case["most_gens"])))))
        out.append((cfg, gens))
    return out


# -- the passes -----------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "run":
        return {"case": case, "run": GARun(_config(case, seed))}
    if kind == "batch":
        runs, batch = [GARun(c) for c in _batch_configs(case, seed)], GABatch()
        for r in runs:
            batch.add(r, 1 << 40)
        return {"case": case, "runs": runs, "batch": batch}
    if kind == "serve":
        return {"case": case, "server": Server(256 << 20, max_slots=case["slots"]),
                "requests": _requests(case, seed)}
    # surfaces sampled from the end of a run, on the GPU, and the call's buffers
    words, n = case["sites"] * case["dbits"] // 32, case["n"]
    run = GARun(run_config(width=128, height=128, pop=32, sites=case["sites"],
                           dbits=case["dbits"], policy=case["policy"], seed=seed & 0xFFFFFFFF))
    run.step(3000)
    ids = np.random.default_rng(seed).choice(run.agents, size=n, replace=False)
    _, T, D = run.extract(ids.astype(np.uint64))
    run.close()
    dev = torch.device("cuda", torch.cuda.current_device())
    return {"case": case,
            "T": torch.from_numpy(T.view(np.int32)).to(dev),
            "D": torch.from_numpy(D.view(np.int32).reshape(n, words)).to(dev),
            "workspace": torch.empty(load().ga_mrca_workspace_bytes(n), dtype=torch.uint8,
                                     device=dev),
            "L": torch.empty((n, n), dtype=torch.int32, device=dev),
            "U": torch.empty((n, n), dtype=torch.int32, device=dev)}


def _signed(a):
    return a.view(np.int64 if a.dtype.itemsize == 8 else np.int32)


def _taken(run, take):
    if take == "sample":
        ids, T, D = run.extract()
        return {"ids": _signed(ids), "T": _signed(T), "D": _signed(D)}
    got = run.read(outbox=bool(run.cfg["migration"]))
    out = {"f": got["f"], "T": _signed(got["T"]), "D": _signed(got["D"])}
    if "P" in got:
        out["P"] = _signed(got["P"])
    if "outbox" in got:
        out["outbox"] = {k: v if v.dtype.kind == "f" else v.astype(np.int64)
                         for k, v in got["outbox"].items()}
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "run":
        state["run"].step(case["gens"])
        return _taken(state["run"], case["take"])
    if kind == "batch":
        state["batch"].step(case["gens"])
        got = [r.extract() for r in state["runs"]]
        return {"T": np.concatenate([_signed(T) for _, T, _ in got]),
                "D": np.concatenate([_signed(D).reshape(-1) for _, _, D in got])}
    if kind == "serve":
        server = state["server"]
        reqs = [server.submit(cfg, gens) for cfg, gens in state["requests"]]
        server.drain()
        server.done.clear()
        return {"ids": np.concatenate([_signed(r.result[0]) for r in reqs]),
                "T": np.concatenate([_signed(r.result[1]) for r in reqs]),
                "D": np.concatenate([_signed(r.result[2]).reshape(-1) for r in reqs])}
    lib, ptr = load(), lambda t: ctypes.c_void_p(t.data_ptr())
    code = lib.ga_mrca_matrix_ex(
        ptr(state["T"]), ptr(state["D"]), case["n"], case["sites"], case["dbits"],
        case["policy"], case["kc"], ptr(state["workspace"]), state["workspace"].numel(),
        ptr(state["L"]), ptr(state["U"]),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    if code:
        raise RuntimeError(lib.ga_last_error().decode())
    return {"L": state["L"], "U": state["U"]}


# -- what a pass cannot do without ----------------------------------------------------------------

def _run_work(cfg, gens):
    """The state read and written once, and the 32-bit lane operations of its generations: a
    Philox block, k entrants and k - 1 comparisons, mutation and deposit per child; a block, four
    arrivals and an emission per island."""
    islands = cfg["width"] * cfg["height"]
    agents = islands * cfg["pop"]
    words = cfg["sites"] * cfg.get("dbits", 1) // 32 + (2 if cfg.get("model", 0) else 0)
    k = cfg["k"] if cfg["selection"] else 1
    state = agents * (8 + 4 * words) + islands * (12 + 4 * words)
    return 2 * state, gens * (agents * (40 + k + 3 * (k - 1) + 13) + islands * 50)


def work(case):
    kind = case["kind"]
    if kind == "mrca":
        n, words = case["n"], case["sites"] * case["dbits"] // 32
        return {"bytes": 8 * n * n + 4 * n * (1 + words), "flops": 10 * n * n}
    if kind == "run":
        parts = [(_config(case, 1), case["gens"])]
    elif kind == "batch":
        parts = [(c, case["gens"]) for c in _batch_configs(case, 1)]
    else:
        parts = _requests(case, 1)
    done = [_run_work(c, g) for c, g in parts]
    return {"bytes": sum(b for b, _ in done), "flops": sum(f for _, f in done)}


# -- the fitness of a run in 64 bits --------------------------------------------------------------

LOW = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors that hold 32-bit words."""
    for r in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((b >> 32) & LOW) ^ c1 ^ ((k0 + r * 0x9E3779B9) & LOW), b & LOW, \
            ((a >> 32) & LOW) ^ c3 ^ ((k1 + r * 0xBB67AE85) & LOW), a & LOW
    return c0, c1, c2, c3


def exact(case, seed):
    """The population's fitness after a run's first `gens` generations, in 64 bits (the discrete
    mutation law on the fitness-valued genome, whose sums are exact); everything else is whole."""
    if case["kind"] != "run" or case["take"] != "state":
        return None
    cfg = _config(case, seed)
    islands, pop, k = cfg["width"] * cfg["height"], cfg["pop"], cfg["k"]
    if cfg.get("law", 0) or cfg.get("model", 0) or islands * pop * case["gens"] > 1e9:
        return None
    dev = torch.device("cuda", torch.cuda.current_device())
    whole = lambda v: torch.as_tensor(v, dtype=torch.int64, device=dev)  # noqa: E731
    k0, k1, bits = cfg["seed"], cfg["run_id"], pop.bit_length() - 1
    isl, slots = torch.arange(islands, device=dev), torch.arange(pop, device=dev)
    x, y, W, H = isl % cfg["width"], isl // cfg["width"], cfg["width"], cfg["height"]
    near = [((y - 1) % H) * W + x, y * W + (x + 1) % W, ((y + 1) % H) * W + x, y * W + (x - 1) % W]
    f = torch.zeros((islands, pop), dtype=torch.float64, device=dev)
    sent = to = None
    for t in range(case["gens"]):
        mx, my, mz, _ = _philox(whole(0), isl, whole(t), whole(1), k0, k1)
        if cfg["migration"]:
            for q in range(4) if t else ():
                came = to[near[q]] == q ^ 2
                slot = (((mz >> (8 * q)) & 0xFF) >> (8 - bits)).unsqueeze(1)
                here = f.gather(1, slot).squeeze(1)
                f.scatter_(1, slot, torch.where(came, sent[near[q]], here).unsqueeze(1))
            sent = f.gather(1, (mx >> (32 - bits)).unsqueeze(1)).squeeze(1)
            to = my >> 30
        w = _philox(slots.unsqueeze(0), isl.unsqueeze(1), whole(t), whole(0), k0, k1)
        best = f.gather(1, (w[0] & 0xFF) >> (8 - bits))
        for m in range(1, k if cfg["selection"] else 1):
            got = f.gather(1, ((w[m // 4] >> (8 * (m % 4))) & 0xFF) >> (8 - bits))
            best = torch.where(got > best, got, best)
        step = ((((w[3] & 0x7FFFFFFF) * 10) >> 32) - 2).double() * 0.5
        f = torch.where(w[2] < cfg["p32"], best + step, best)
    out = {"f": f.reshape(-1), "T": None, "D": None}
    if cfg["migration"]:
        if cfg.get("schedule", 0) == 0:
            out["outbox"] = {"valid": None, "dir": None, "f": sent, "T": None, "D": None}
    return out
