"""The work that a user of this library has it do, as cases that can be timed.

Every case goes through the public entry points of paper_1309_4349_amd.kk and
returns everything the calls produce: lattices, accepted counts, N_AB, cluster
histograms, observables.  Kinds:

  square    one L x L lattice swept through kk.Sim, then N_AB and the cluster
            histogram (the statistics the paper takes regularly) and the lattice
  series    one L x L lattice observed every few sweeps (kk.Sim.series)
  triangular, mpkk
            the paper's own lattice, class schedule and literal MPKK
  batch     many square replicas advanced together, a histogram of each
  tri_batch many triangular replicas advanced together
  server    simulation jobs submitted to the job server and served to the end
"""
import math

import numpy as np

from paper_1309_4349_amd import kk, workloads


def listed():
    return [
        # the smallest standing workload: 1000 sweeps of a 64 x 64 lattice, latency-bound
        {"name": "square 64 int8", "kind": "square", "L": 64, "layout": "int8", "composition": 0.5, "omega": 0.5,
         "sweeps": 1000},
        # the paper's headline size, one lattice at a time, a histogram every 1000 sweeps
        {"name": "square 400 int8", "kind": "square", "L": 400, "layout": "int8", "composition": 0.3, "omega": 0.9,
         "sweeps": 1000},
        # a mid-sized lattice that is no multiple of 32 (the int8 layout's reason to exist)
        {"name": "square 1036 int8", "kind": "square", "L": 1036, "layout": "int8", "composition": 0.5, "omega": 0.6,
         "sweeps": 500},
        # the large standing workload: 4096 x 4096 bit-packed just below demixing, a stretch of its 1e4 sweeps
        {"name": "square 4096 bits", "kind": "square", "L": 4096, "layout": "bitpacked", "composition": 0.5,
         "omega": 0.88, "sweeps": 2000},
        # time series of the observables: energy, sampled neighbours and cluster averages every 50 sweeps
        {"name": "series 2048 bits", "kind": "series", "L": 2048, "layout": "bitpacked", "composition": 0.5,
         "omega": 0.7, "every": 50, "count": 8},
        # the twelve runs of the paper's size (3 compositions x 4 omegas) together, a histogram of each per 1000 sweeps
        {"name": "batch grid 400 x 12", "kind": "batch", "table": "grid", "replicas": 12, "sweeps": 1000, "tune": True},
        # the replica table of uneven sides 64 .. 1024
        {"name": "batch table 256", "kind": "batch", "table": "mixed", "replicas": 256, "sweeps": 1000,
         "tune": False},
        # the paper's lattice at its own size: one 100 x 100 ring
        {"name": "triangular 100", "kind": "triangular", "L": 100, "H": 100, "composition": 0.5, "omega": 0.4,
         "sweeps": 1000},
        # and at the size of the large workload
        {"name": "triangular 4092", "kind": "triangular", "L": 4092, "H": 4092, "composition": 0.5, "omega": 0.88,
         "sweeps": 200},
        # the literal MPKK on the ring next to 400 x 400
        {"name": "mpkk 404 x 420", "kind": "mpkk", "L": 404, "H": 420, "composition": 0.5, "omega": 0.3,
         "sweeps": 500},
        # many runs of the paper's lattice together
        {"name": "tri batch 100 x 256", "kind": "tri_batch", "L": 100, "replicas": 256, "omega": 0.4, "sweeps": 1000},
        # a burst of served jobs, sides 128 .. 2048
        {"name": "server 24 jobs", "kind": "server", "jobs": 24, "scale": 0.05, "trace": 1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["square", "square", "square", "series", "triangular", "mpkk", "batch", "tri_batch", "server"])
    x, w = round(rng.uniform(0.2, 0.8), 3), round(rng.uniform(0.2, 1.4), 3)
    if kind in ("square", "series"):
        # sides 32 .. 4096; half of them whole words, half any multiple of 4; attraction between unlike types too
        layout = rng.choice(["int8", "bitpacked"])
        step = 32 if layout == "bitpacked" or rng.random() < 0.3 else 4
        L = max(32, min(4096, step * round(_log_int(rng, 32, 4096) / step)))
        if 2688 < L < 3972:  # these sides have no valid default tile
            L = 2688 if L < 3300 else 3972 if layout == "int8" else 4000
        if rng.random() < 0.15:
            w = -w
        c = {"kind": kind, "L": L, "layout": layout, "composition": x, "omega": w}
        if kind == "square":
            c["sweeps"] = max(50, min(1000, int(4e9 / L / L)))
        else:
            c["every"], c["count"] = rng.randint(1, 60), rng.randint(2, 8)
        return c
    if kind == "triangular":
        L, H = 8 * rng.randint(1, 20) + 4, 4 * rng.randint(3, 40)
        if rng.random() < 0.6:
            L = max(100, min(4092, 8 * round(_log_int(rng, 100, 4092) / 8) + 4))
            H = max(100, min(4092, 4 * round(L * rng.uniform(0.6, 1.2) / 4)))
        return {"kind": kind, "L": L, "H": H, "composition": x, "omega": w, "sweeps": max(50, min(1000, int(2e9 / L / H)))}
    if kind == "mpkk":
        L = 7 * round(_log_int(rng, 60, 4000) / 7) + rng.choice([3, 5])
        H = 7 * round(L * rng.uniform(0.7, 1.0) / 7)
        return {"kind": kind, "L": L, "H": H, "composition": x, "omega": w, "sweeps": max(30, min(500, int(8e8 / L / H)))}
    if kind == "batch":
        table = rng.choice(["grid", "mixed", "offgrid"])
        n = rng.randint(2, 12) if table == "grid" else rng.randint(16, 256)
        return {"kind": kind, "table": table, "replicas": n, "sweeps": rng.randint(100, 1000), "tune": False}
    if kind == "tri_batch":
        return {"kind": kind, "L": 8 * rng.randint(6, 25) + 4, "replicas": rng.randint(8, 256), "omega": w,
                "sweeps": rng.randint(50, 400)}
    return {"kind": "server", "jobs": rng.randint(4, 24), "scale": 0.02, "trace": rng.randint(2, 1000)}


def _batch_jobs(case, seed):
    n = case["replicas"]
    if case["table"] == "grid":
        jobs = workloads.grid_400(case["sweeps"])[:n]
    else:
        jobs = workloads.batch_replicas(n, case["sweeps"], offgrid=case["table"] == "offgrid")
    for i, j in enumerate(jobs):
        j.seed = workloads.job_seed(seed, i)
    return jobs


def _tri_jobs(case, seed):
    return [workloads.Job(case["L"], 0.3 + 0.4 * (i % 8) / 8, case["omega"], workloads.job_seed(seed, i),
                          case["sweeps"]) for i in range(case["replicas"])]


def _server_jobs(case, seed):
    # sizes, sweep counts and parameters belong to the case; the seeds of the runs are the input
    jobs = workloads.serving_trace(case["jobs"], sweep_scale=case["scale"], seed=workloads.MASTER_SEED ^ case["trace"])
    for i, j in enumerate(jobs):
        j.seed = workloads.job_seed(seed, i)
    return jobs


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind in ("square", "series"):
        s["sim"] = kk.Sim(case["L"], case["composition"], case["omega"], workloads.job_seed(seed, 0),
                          layout=case["layout"])
    elif kind in ("triangular", "mpkk"):
        s["sim"] = kk.Sim(case["L"], case["composition"], case["omega"], workloads.job_seed(seed, 0),
                          geometry="triangular", rows=case["H"], scheme="classes" if kind == "triangular" else "mpkk")
    elif kind == "batch":
        s["jobs"] = _batch_jobs(case, seed)
        s["batch"] = kk.Batch(s["jobs"])
        if case["tune"]:
            s["batch"].autotune()
    elif kind == "tri_batch":
        s["jobs"] = _tri_jobs(case, seed)
        s["batch"] = kk.TriBatch(s["jobs"])
    else:
        s["jobs"] = _server_jobs(case, seed)
        s["server"] = kk.Server(keep_lattice=True)
    return s


def _pairs(hist, sites):
    """A histogram as (size, count) rows, zeros after the last: k distinct sizes need k (k + 1) / 2 sites."""
    out = np.zeros((math.isqrt(2 * sites) + 1, 2), dtype=np.int64)
    out[:len(hist)] = hist
    return out


def _replicas(batch, n, hists):
    """What a program reads from a batch after a run: every replica's lattice and statistics."""
    lattices, scalars, pairs = [], [], []
    for i in range(n):
        sim = batch.sim(i)
        scalars.append((*sim.stats(), sim.energy()[0]))
        if hists:
            pairs.append(_pairs(sim.cluster_hist(1), sim.L * sim.H))
        lattices.append(sim.get_lattice().ravel())
    out = {"lattices": np.concatenate(lattices), "scalars": np.array(scalars, dtype=np.int64)}
    if hists:
        out["hists"] = np.concatenate(pairs)
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("square", "triangular", "mpkk"):
        sim = state["sim"]
        sim.sweep(case["sweeps"])
        n_unlike = sim.energy()[0]
        hist = _pairs(sim.cluster_hist(1), sim.L * sim.H)
        return {"n_unlike": n_unlike, "hist": hist, "stats": list(sim.stats()), "lattice": sim.get_lattice()}
    if kind == "series":
        sim = state["sim"]
        series = sim.series(case["every"], case["count"])
        return {"series": np.array([list(o.values()) for o in series], dtype=np.float64), "lattice": sim.get_lattice()}
    if kind == "batch":
        state["batch"].run()
        state["batch"].cluster_hists(1)
        return _replicas(state["batch"], case["replicas"], True)
    if kind == "tri_batch":
        state["batch"].run()
        return _replicas(state["batch"], case["replicas"], False)
    server = state["server"]
    ids = [server.submit(j) for j in state["jobs"]]
    done = {}
    while len(done) < len(ids):
        server.step()
        for r in server.poll():
            done[r["id"]] = r
    out = {"scalars": np.array([[done[i]["sweeps"], done[i]["accepted"], done[i]["n_unlike"]] for i in ids], np.int64),
           "hists": np.concatenate([_pairs(server.job_hist(i), j.sites) for i, j in zip(ids, state["jobs"])]),
           "lattices": [server.job_lattice(i) for i in ids]}
    for i in ids:
        server.release(i)
    return out


# 32-bit operations one attempt cannot do without (its share of the random
# words, the compare with the threshold, the bit-sliced or byte-wise decision)
_OPS = {"square": 12.22, "triangular": 76.0, "mpkk": 87.0}


def work(case):
    """A lattice is read and written once in its device layout and returned once as bytes; attempts are counted as
    the 32-bit operations above."""
    kind = case["kind"]
    if kind in ("square", "series"):
        n = case["L"] * case["L"]
        sweeps = case["sweeps"] if kind == "square" else case["every"] * case["count"]
        return {"bytes": n * (1 + (2 if case["layout"] == "int8" else 0.25)), "flops": n * sweeps * _OPS["square"]}
    if kind in ("triangular", "mpkk"):
        n = case["L"] * case["H"]
        return {"bytes": 3 * n, "flops": n * case["sweeps"] * _OPS[kind]}
    if kind == "tri_batch":
        n = case["L"] * case["L"] * case["replicas"]
        return {"bytes": 3 * n, "flops": n * case["sweeps"] * _OPS["triangular"]}
    jobs = _batch_jobs(case, 0) if kind == "batch" else _server_jobs(case, 0)
    lattice = sum(j.L * j.L * (1 + (2 if j.layout == "int8" else 0.25)) for j in jobs)
    return {"bytes": lattice, "flops": sum(j.attempts for j in jobs) * _OPS["square"]}
