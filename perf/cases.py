"""Workloads for timing the engine through its Python entry points.

Every case is work that a user of the library has it do, over the sizes of the repository's
workloads (workloads/, bench.py, tests/): ensembles of trajectories in the three state
precisions, from a few on a 3-qubit ring to 10^5; one batched launch over many
instances; a new instance taken from its couplings to its ground-state population; the
low spectrum of larger instances, by the dense and by the iterative eigensolver; the
gradient of the ground-state population, alone and inside one step of a schedule
optimisation.

    listed()             the fixed cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  engine, tables and buffers that a program holds before the call
    run(state)           one pass and its outputs
    work(case)           bytes and operations that one pass cannot do without
    exact(case, seed)    the spectrum cases' outputs by LAPACK in 64 bits

The seed draws the instance (fields, couplings, where there are any the control points)
and is the key of the trajectories' random streams.
"""
import math

import numpy as np
import torch

import workloads as W
from paper_1710_03431_amd import binding

BYTES = {"fp64": 8, "fp32": 4, "bf16": 4}   # Delta per element: BF16 runs hold it as a hi/lo pair


def listed():
    return [
        # the smallest call in use: a few trajectories on three qubits, results on the host (launch latency)
        dict(name="ring3_fp64", kind="ensemble", couplings="ring", qubits=3, levels=8, grid=101, traj=64,
             precision="fp64", call="run"),
        # the 4-qubit ring workload: the plain FP64 method, a chain of 1000 short steps
        dict(name="ring4_fp64", kind="ensemble", couplings="ring", qubits=4, levels=16, grid=1001, traj=1000,
             precision="fp64", call="run_into"),
        # the 8-qubit all-to-all workload at its full spectrum, in each state precision
        dict(name="a2a8_fp32", kind="ensemble", couplings="pm1", qubits=8, levels=256, grid=2000, traj=10000,
             precision="fp32", call="run_into"),
        dict(name="a2a8_fp64", kind="ensemble", couplings="pm1", qubits=8, levels=256, grid=2000, traj=10000,
             precision="fp64", call="run_into"),
        dict(name="a2a8_bf16", kind="ensemble", couplings="pm1", qubits=8, levels=256, grid=2000, traj=10000,
             precision="bf16", call="run_into"),
        # a large ensemble on a truncated spectrum of 32 levels, 500 grid points: bound by its jumps
        dict(name="levels32_fp32", kind="ensemble", couplings="pm1", qubits=8, levels=32, grid=500, traj=100000,
             precision="fp32", call="run_into"),
        # many small instances (6-8 qubits; 16, 32 or 64 levels) in one launch, as a benchmark set is scanned
        dict(name="batch24_bf16", kind="batch", instances=24, grid=500, traj=2048, precision="bf16"),
        # a new 8-qubit instance from its couplings to its population: eigensystem, tables, trajectories
        dict(name="new8_fp64", kind="new", couplings="ring", qubits=8, levels=256, grid=1000, traj=2000,
             precision="fp64"),
        # energies and decay rates of the 32 lowest levels of 10 qubits along the anneal (dense eigensolver)
        dict(name="spectrum10", kind="spectrum", couplings="ring", qubits=10, levels=32, grid=400),
        # the same beyond the dense solver's sizes (matrix-free iteration)
        dict(name="spectrum12", kind="spectrum", couplings="ring", qubits=12, levels=32, grid=60),
        # gradient of the final ground-state population for 8 + 8 control points and eta, full spectrum
        dict(name="gradient8_fp32", kind="gradient", qubits=8, controls=8, grid=500, traj=4096, precision="fp32"),
        # one step of a schedule optimisation through autograd: tables, trajectories, adjoint sweep
        dict(name="descent6_fp64", kind="descent", qubits=6, controls=8, grid=501, traj=2000, precision="fp64"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["ensemble"] * 4 + ["batch", "new", "spectrum", "gradient", "descent"])
    precision = rng.choice(["fp64", "fp32", "bf16"])
    if kind == "ensemble":
        qubits = rng.randint(3, 8)
        couplings = "ring" if qubits < 6 else rng.choice(["ring", "pm1"])
        levels = 1 << qubits
        if qubits >= 6 and rng.random() < 0.5:
            levels = rng.choice([16, 32, 64, rng.randint(10, 64)])
            levels = levels if levels + 16 <= 1 << qubits else 32
        grid = _log(rng, 100, 2000)
        # at most the work of the largest listed ensemble
        most = min(1e5, 1.9e7 * (256.0 / max(levels, 32)) ** 1.4 / grid)
        return dict(kind=kind, couplings=couplings, qubits=qubits, levels=levels, grid=grid,
                    traj=_log(rng, 50, max(60.0, most)), precision=precision,
                    call=rng.choice(["run", "run_into", "run_into"]))
    if kind == "batch":
        return dict(kind=kind, instances=rng.randint(3, 24), grid=_log(rng, 150, 500), traj=_log(rng, 200, 2048),
                    precision=precision)
    if kind == "new":
        qubits = rng.randint(3, 8)
        return dict(kind=kind, couplings="ring", qubits=qubits, levels=1 << qubits, grid=_log(rng, 100, 1000),
                    traj=_log(rng, 100, 2000), precision="fp64")
    if kind == "spectrum":
        qubits = rng.randint(8, 10)
        return dict(kind=kind, couplings="ring", qubits=qubits, levels=rng.randint(12, 48), grid=_log(rng, 50, 400))
    qubits = rng.randint(3, 6)
    return dict(kind=kind, qubits=qubits, controls=rng.randint(2, 16), grid=_log(rng, 100, 1000),
                traj=_log(rng, 100, 4096), precision=precision if kind == "gradient" and precision == "fp32" else "fp64")


# ------------------------------------------------------------------ instances ----
def _instance(case, seed):
    if case["couplings"] == "pm1":
        return W.pm1_all_to_all(case["qubits"], seed, n_grid=case["grid"], n_levels=case["levels"])
    return W.ring_instance(case["qubits"], seed, n_grid=case["grid"], n_levels=case["levels"])


def _controlled(case, seed):
    """A ring whose schedule is given by control points, off the linear one as in a search under way."""
    m = case["controls"]
    A, B = W.linear_schedule(m)
    rng = np.random.default_rng([seed, 1])
    A = A + 0.2 * rng.uniform(0.0, 1.0, m)
    B = B + 0.2 * rng.uniform(0.0, 1.0, m)
    return W.ring_instance(case["qubits"], seed, n_grid=case["grid"], t_f=300.0, eta=1e-3, A_ctrl=A, B_ctrl=B)


def _batch_instances(case, seed):
    """Instances as in workloads.config_batched, up to 8 qubits."""
    rng = np.random.default_rng([seed, 2])
    out = []
    for k in range(case["instances"]):
        qubits = int(rng.integers(6, 9))
        levels = int(rng.choice([16, 32, 64]))
        t_f = 1000.0 * 10.0 ** rng.uniform(0.0, 2.0)
        out.append(W.pm1_all_to_all(qubits, int(rng.integers(0, 2**31 - 1)), t_f=t_f, n_grid=case["grid"],
                                    n_levels=levels, n_traj=case["traj"], instance_id=k))
    return out


# -------------------------------------------------------------- prepare and run ----
def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case, seed=seed)
    if kind == "batch":
        engines, runs = [], []
        for inst in _batch_instances(case, seed):
            eng = binding.Engine(0)
            eng.set_instance(inst)
            eng.precompute(inst.n_grid, inst.levels)
            engines.append(eng)
            runs.append(dict(n_traj=inst.n_traj, seed=seed, instance_id=inst.instance_id))
        state["batch"] = binding.Batch(engines, runs, case["precision"])
        return state
    eng = state["engine"] = binding.Engine(0)
    if kind in ("gradient", "descent"):
        inst = state["instance"] = _controlled(case, seed)
        eng.set_instance(inst)
        if kind == "gradient":
            eng.precompute(inst.n_grid, inst.levels)
            return state
        for name, v in (("A", inst.A_ctrl), ("B", inst.B_ctrl), ("eta", inst.eta)):
            state[name] = torch.tensor(v, dtype=torch.float64, requires_grad=True)
        return state
    inst = state["instance"] = _instance(case, seed)
    if kind == "ensemble":
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, inst.levels)
        if case["call"] == "run_into":
            state["outs"] = eng.alloc_outputs(case["traj"])
    return state


def run(state):
    case, seed = state["case"], state["seed"]
    kind = case["kind"]
    if kind == "batch":
        batch = state["batch"]
        for o in batch.outs:   # totals and histograms accumulate over launches
            o["jump_totals"].zero_()
            o["net_hist"].zero_()
        batch.launch()
        return [{"pgs_sum": o["pgs_sum"], "jump_count": o["jump_count"]} for o in batch.outs]
    eng = state["engine"]
    if kind == "ensemble":
        if case["call"] == "run":
            res = eng.run(case["traj"], case["precision"], seed=seed, final_state=True)
            return {k: res[k] for k in ("pgs_sum", "pgs_sumsq", "jump_totals", "jump_count", "net_gs", "net_hist",
                                        "final_state")}
        outs = state["outs"]
        outs["jump_totals"].zero_()
        outs["net_hist"].zero_()
        eng.run_into(outs, case["traj"], case["precision"], seed=seed)
        return _outputs(outs)
    inst = state["instance"]
    if kind == "new":
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, inst.levels)
        res = eng.run(case["traj"], case["precision"], seed=seed)
        return {k: res[k] for k in ("pgs_sum", "pgs_sumsq", "jump_totals", "jump_count", "net_gs", "net_hist")}
    if kind == "spectrum":
        eng.set_instance(inst)
        eng.precompute(inst.n_grid, inst.levels)
        return eng.get_tables(("E", "gs", "Gamma"))
    if kind == "gradient":
        return eng.grad_pgs(case["traj"], case["precision"], seed=seed)
    A, B, eta = state["A"], state["B"], state["eta"]
    for p in (A, B, eta):
        p.grad = None
    value = binding.pgs(eng, A, B, eta, t_f=inst.t_f, omega_c=inst.omega_c, T=inst.T, n_grid=inst.n_grid,
                        n_levels=inst.levels, n_traj=case["traj"], precision=case["precision"], seed=seed)
    value.backward()
    return {"value": value.detach(), "A": A.grad, "B": B.grad, "eta": eta.grad}


def _outputs(o):
    return {k: o[k] for k in ("pgs_sum", "pgs_sumsq", "jump_totals", "jump_count", "net_gs", "net_hist")}


# ------------------------------------------------------------------------ work ----
def _ensemble_work(levels, grid, traj, precision, channels):
    """Delta, the phases and the rate rows of every grid point read once; the outputs written once."""
    n = levels
    size = BYTES[precision]
    return {"bytes": float(grid * (n * n * size + 2 * n * size + (3 * channels + 4) * n * 8) + 8 * traj + 16 * grid),
            "flops": float(traj * (grid - 1) * (4 * n * n + 10 * n))}


def _table_work(qubits, levels, grid):
    """Householder reduction, eigenvectors of the wanted levels, overlaps, matrix elements; tables written once."""
    N, n = 1 << qubits, levels
    per = 4.0 / 3.0 * N ** 3 + 2.0 * N * N * n + 2.0 * n * n * N * (1 + qubits)
    if N > 1024:   # products with the sparse H instead of the reduction: a filter of degree 10 on the block
        per = 10.0 * 2 * N * (qubits + 1) * (n + 16) + 2.0 * n * n * N * (1 + qubits)
    return {"bytes": float(grid * (1 + qubits) * n * n * 8), "flops": float(grid * per)}


def _sum(*parts):
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


def work(case):
    kind = case["kind"]
    if kind == "batch":
        return _sum(*[_ensemble_work(i.levels, i.n_grid, i.n_traj, case["precision"], i.n_qubits)
                      for i in _batch_instances(case, 1)])
    if kind == "ensemble":
        return _ensemble_work(case["levels"], case["grid"], case["traj"], case["precision"], case["qubits"])
    if kind == "spectrum":
        return _table_work(case["qubits"], case["levels"], case["grid"])
    n = 1 << case["qubits"]
    run_w = _ensemble_work(n, case["grid"], case["traj"], case["precision"], case["qubits"])
    if kind == "new":
        return _sum(_table_work(case["qubits"], n, case["grid"]), run_w)
    # adjoint sweep: the recorded states again, the adjoint moved back, the contraction with dO (three products)
    sweep = {"bytes": 2 * run_w["bytes"], "flops": float(case["traj"] * (case["grid"] - 1) * 12 * n * n)}
    if kind == "gradient":
        return _sum(run_w, sweep)
    return _sum(_table_work(case["qubits"], n, case["grid"]), run_w, sweep)


# ----------------------------------------------------------------------- exact ----
def exact(case, seed):
    """Energies and decay rates of the spectrum cases (Gamma_b = sum_i [sum_{a != b} gamma(e_b - e_a)
    z_i,ab^2 + gamma(0) z_i,bb^2] over the retained levels).  Trajectories follow their random draws jump
    by jump, one after another, and have no value of this kind that is quick to compute."""
    if case["kind"] != "spectrum":
        return None
    nq, n, M = case["qubits"], case["levels"], case["grid"]
    N = 1 << nq
    if M * float(N) ** 3 > 1.5e10:   # tens of seconds of LAPACK
        return None
    inst = _instance(case, seed)
    x = np.arange(N)
    sz = 1.0 - 2.0 * ((x[None, :] >> np.arange(nq)[:, None]) & 1)
    ez = inst.h @ sz
    for i in range(nq):
        for j in range(i + 1, nq):
            ez = ez + inst.J[i, j] * sz[i] * sz[j]
    hx = np.zeros((N, N))
    for q in range(nq):
        hx[x, x ^ (1 << q)] -= 1.0
    E, Gamma = np.zeros((M, n)), np.zeros((M, n))
    for g in range(M):
        s = g / (M - 1)
        H = inst.A_ctrl[0] * (1.0 - s) * hx + np.diag(inst.B_ctrl[-1] * s * ez)
        e, V = np.linalg.eigh(H)
        e, V = e[:n], V[:, :n]
        E[g] = e
        if g == 0:
            continue
        w = e[:, None] - e[None, :]   # w[b, a] = e_b - e_a
        den = -np.expm1(-w / inst.T)
        rate = np.full_like(w, 2.0 * math.pi * inst.eta * inst.T)
        off = ~np.eye(n, dtype=bool)
        rate[off] = 2.0 * math.pi * inst.eta * w[off] * np.exp(-np.abs(w[off]) / inst.omega_c) / den[off]
        z2 = sum(((V * sz[i][:, None]).T @ V) ** 2 for i in range(nq))
        Gamma[g] = (rate * z2).sum(axis=1)
    return {"E": E, "Gamma": Gamma, "gs": None}
