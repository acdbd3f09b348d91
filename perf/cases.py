"""Cases for timing the sampler through its public entry points.

Each case is one call as a user's program makes it, into buffers that the
program keeps (the output tensor, a batch, a session), on the current stream:

  sample       dcs.sample: n distinct values of 1..N
  replacement  dcs.sample_replacement
  bernoulli    dcs.sample_bernoulli, p >= 2^-10 (single-precision skips)
  batch        dcs.Batch.run, graph replay, uneven instances (workloads.py's
               law with the tuning table's leaf sizes)
  online       dcs.Online.next: one run of consecutive parts of a session
  segments     dcs.sample_segments over an uneven universe
  gnm, gnp     dcs.sample_edges_gnm / dcs.sample_edges_gnp (p below 2^-10:
               double-precision skips)

Every output is a whole number that the library defines bit for bit, so there
is no value in floating point to compare it with (`exact` is None).
"""
import math

import torch

import paper_1610_05141_amd as dcs
from paper_1610_05141_amd import autotune, workloads


def listed():
    return [
        # the smallest request of the serving law: latency of one call
        {"name": "sample_256_of_1e6", "kind": "sample", "n": 256, "N": 1_000_000},
        # an ordinary call: a million indices (launches and the tree's chain count)
        {"name": "sample_2p20_of_2p32", "kind": "sample", "n": 1 << 20, "N": 1 << 32},
        # the benchmark's headline: large, sparse, power-of-two universe
        {"name": "sample_2p30_of_2p48", "kind": "sample", "n": 1 << 30, "N": 1 << 48},
        # large over a universe that is no power of two, as most are (the
        # total of the benchmark's uneven segments)
        {"name": "sample_2p28_of_odd", "kind": "sample", "n": 1 << 28,
         "N": 286_538_054_670_896},
        # dense: every second element (Algorithm B's leaves)
        {"name": "sample_2p29_of_2p30", "kind": "sample", "n": 1 << 29, "N": 1 << 30},
        # with replacement
        {"name": "replacement_2p28_of_2p40", "kind": "replacement", "n": 1 << 28,
         "N": 1 << 40},
        # Bernoulli sampling of a large table at one per cent
        {"name": "bernoulli_1pc_of_2p36", "kind": "bernoulli", "p": 0.01, "N": 1 << 36},
        # a thousand uneven requests in one replayed batch
        {"name": "batch_1024", "kind": "batch", "count": 1024},
        # streaming a large sample: 16 of 256 parts per call
        {"name": "online_16_of_256_parts", "kind": "online", "n": 1 << 30, "N": 1 << 48,
         "depth": 8, "run": 16},
        # one sample over 4096 shards of uneven sizes
        {"name": "segments_2p28_of_4096", "kind": "segments", "n": 1 << 28, "K": 4096},
        # random graphs: a fixed number of edges, and independent edges
        {"name": "gnm_2p28_edges", "kind": "gnm", "V": 1 << 26, "m": 1 << 28},
        {"name": "gnp_2p28_edges", "kind": "gnp", "V": 1 << 26, "p": 2.0 ** -23},
    ]


def _log2_uniform(rng, lo, hi):
    return int(2.0 ** rng.uniform(lo, hi))


def _universe(rng, n, dens_lo):
    """A universe of density log-uniform in [dens_lo, 1/2]; a power of two one
    time in four."""
    N = max(n, math.ceil(n / 10.0 ** rng.uniform(math.log10(dens_lo), math.log10(0.5))))
    return 1 << (N - 1).bit_length() if rng.random() < 0.25 else N


def draw(rng):
    kind = rng.choice(["sample", "sample", "sample", "replacement", "bernoulli", "batch",
                       "online", "segments", "gnm", "gnp"])
    if kind in ("sample", "replacement"):
        n = _log2_uniform(rng, 8, 28)
        return {"kind": kind, "n": n, "N": _universe(rng, n, 4e-6)}
    if kind == "bernoulli":
        p = 10.0 ** rng.uniform(-3.0, -0.5)
        return {"kind": kind, "p": p, "N": int(_log2_uniform(rng, 12, 28) / p)}
    if kind == "batch":
        return {"kind": kind, "count": _log2_uniform(rng, 4, 10)}
    if kind == "online":
        n = _log2_uniform(rng, 20, 28)
        depth = rng.randint(3, 8)
        return {"kind": kind, "n": n, "N": _universe(rng, n, 4e-6), "depth": depth,
                "run": 1 << rng.randint(0, depth)}
    if kind == "segments":
        return {"kind": kind, "n": _log2_uniform(rng, 14, 28), "K": _log2_uniform(rng, 2, 12)}
    V = _log2_uniform(rng, 14, 26)
    m = min(_log2_uniform(rng, 12, 27), V * (V - 1) // 4)
    if kind == "gnm":
        return {"kind": kind, "V": V, "m": m}
    # sparse graphs: an average degree of at most V / 1100 keeps p below 2^-10
    return {"kind": kind, "V": V, "p": min(m, V * V // 2200) / (V * (V - 1) / 2)}


def _out(n):
    """An output buffer; entries a call leaves unwritten stay zero."""
    return torch.zeros(n, dtype=torch.int64, device="cuda")


def _segment_lengths(case):
    return workloads.segment_lengths(case["K"], 16, 40)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "seed": seed}
    if kind in ("sample", "replacement"):
        s["out"] = _out(case["n"])
    elif kind == "bernoulli":
        s["out"] = _out(dcs.bernoulli_capacity_hint(case["p"], case["N"]))
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    elif kind == "batch":
        table = autotune.load_table()
        specs, off = [], 0
        for x in workloads.batched_instances(case["count"]):
            specs.append(dcs.InstanceSpec(n=x.n, N=x.N, seed=seed + x.seed, out_offset=off,
                                          n0=autotune.n0_for(x.n, x.N, table)))
            off += x.n
        s["batch"] = dcs.Batch(specs)
        s["out"] = _out(off)
        # a replayed graph is captured on a stream of the program's own
        s["stream"] = torch.cuda.Stream()
    elif kind == "online":
        runs = (1 << case["depth"]) // case["run"]
        mean = case["n"] // runs
        s["online"] = dcs.Online(case["n"], case["N"], seed, case["depth"])
        s["first"] = (seed % runs) * case["run"]
        # a streaming program's buffer: an eighth above a run's mean
        s["out"] = _out(min(case["n"], mean + mean // 8 + (1 << 16)))
    elif kind == "segments":
        s["lengths"] = _segment_lengths(case)
        s["out"] = _out(case["n"])
        s["count"] = torch.zeros(case["K"], dtype=torch.int64, device="cuda")
    elif kind == "gnm":
        s["out"] = torch.zeros((case["m"], 2), dtype=torch.int32, device="cuda")
    elif kind == "gnp":
        N = case["V"] * (case["V"] - 1) // 2
        s["out"] = torch.zeros((dcs.bernoulli_capacity_hint(case["p"], N), 2),
                               dtype=torch.int32, device="cuda")
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    return s


def run(state):
    case, seed, out = state["case"], state["seed"], state["out"]
    kind = case["kind"]
    if kind == "sample":
        return dcs.sample(case["n"], case["N"], seed, out=out)
    if kind == "replacement":
        return dcs.sample_replacement(case["n"], case["N"], seed, out=out)
    if kind == "bernoulli":
        return dcs.sample_bernoulli(case["p"], case["N"], seed, out=out, count=state["count"])
    if kind == "batch":
        own = state["stream"]
        own.wait_stream(torch.cuda.current_stream())
        state["batch"].run(out, use_graph=True, stream=own)
        torch.cuda.current_stream().wait_stream(own)
        return out
    if kind == "online":
        written = state["online"].next(state["first"], case["run"], out)
        return out, written
    if kind == "segments":
        return dcs.sample_segments(case["n"], state["lengths"], seed, out=out,
                                   counts=state["count"])
    if kind == "gnm":
        return dcs.sample_edges_gnm(case["V"], case["m"], seed, out=out)
    return dcs.sample_edges_gnp(case["V"], case["p"], seed, out=out, count=state["count"])


def work(case):
    """Every value of the sample written once (8 bytes, an edge's two vertex
    numbers too); segment sizes read and segment counts written."""
    kind = case["kind"]
    if kind in ("sample", "replacement"):
        values = case["n"]
    elif kind == "bernoulli":
        values = int(case["p"] * case["N"])
    elif kind == "batch":
        values = sum(x.n for x in workloads.batched_instances(case["count"]))
    elif kind == "online":
        values = max(1, (case["n"] >> case["depth"]) * case["run"])
    elif kind == "segments":
        values = case["n"] + 2 * case["K"]
    elif kind == "gnm":
        values = case["m"]
    else:
        values = int(case["p"] * (case["V"] * (case["V"] - 1) // 2))
    return {"bytes": 8 * values, "flops": 0}


def exact(case, seed):
    return None
