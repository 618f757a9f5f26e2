"""Performance cases of the batched checkpoint solver: what its users have it do.

A planner holds B candidate plans for one network, each plan a chain of L stages whose sizes are
counted in slots of a memory budget cut into M parts.  It fills the tables of all chains
(``ckpt_solve_batched``), picks a plan, walks the tables into operation lists and block indices and
checks the lists.  ``op`` names the path of a case:

  solve    the table fill alone, descriptors and tables resident on the device
  plan     one profile in bytes, cut into slots under ten budgets, solved, selected, walked, annotated, simulated
  readout  everything after the fill, on tables that are there already
  host     ``solve(batch)``: numpy arrays in, tables allocated, filled and checked

``mix`` names the stage mix (the recipes of workloads/chains.py with the sizes as shares of M):
uniform stages, attention/MLP pairs, one chain sharded 1/2/4/8 ways, four kinds of layers, and
lognormal times under a tight budget.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2302_02599_amd as amd

SWEEP = 10               # budgets base * (1 + 1/10)^n, n = 0..9
SLOT_BYTES = 1 << 20     # a slot of the smallest budget of the sweep
# smallest and largest activation as shares of M, smallest and largest abar / a
MIXES = {
    "uniform": (1 / 64, 4 / 64, 1.0, 3.0),
    "pairs": (4 / 512, 16 / 512, 2.0, 5.0),
    "sharded": (8 / 1024, 64 / 1024, 2.0, 5.0),
    "kinds": (8 / 2048, 64 / 2048, 1.0, 6.0),
    "lognormal": (5 / 4096, 158 / 4096, 1.0, 8.0),
}
KIND_TIMES = ((50, 200), (1000, 3000), (2000, 6000), (10, 40))  # embedding, attention, MLP, layernorm


def listed():
    def case(name, op, mix, L, M, B, extras=False):
        return {"name": name, "op": op, "mix": mix, "L": L, "M": M, "B": B, "extras": extras}

    return [
        # the smallest call: one short chain, a handful of stages; launches and latency
        case("tiny_chain", "solve", "uniform", 8, 64, 1),
        # one plan of a 12-layer transformer, a stage per attention or MLP block
        case("transformer_chain", "solve", "pairs", 24, 512, 1),
        # a few plans whose length and budget divide by nothing, with memory overheads and gradient sizes of their own
        case("ragged_plans", "solve", "kinds", 53, 777, 5, True),
        # many candidate plans of a short chain
        case("many_short_plans", "solve", "pairs", 13, 500, 200),
        # sixteen sharding candidates of a 24-layer transformer
        case("sharded_plans", "solve", "sharded", 48, 1024, 16),
        # a whole sweep of intra-op plans of a deep mixed network
        case("deep_batch", "solve", "kinds", 96, 2048, 64),
        # long chains under a tight budget, fine slots: the largest job
        case("long_batch", "solve", "lognormal", 192, 4096, 8),
        # a single plan of that network, re-solved on its own
        case("long_chain", "solve", "lognormal", 192, 4096, 1),
        # the longest chain the candidate byte allows, with overheads
        case("longest_chains", "solve", "kinds", 254, 1500, 3, True),
        # the planner's loop: one profile under ten budgets, from bytes to checked block indices
        case("budget_sweep", "plan", "pairs", 50, 500, SWEEP),
        # plans that live in host arrays, through the convenience call
        case("host_call", "host", "pairs", 24, 512, 10),
        # reading schedules out of large tables
        case("long_readout", "readout", "lognormal", 192, 4096, 8),
    ]


def _evals(L, M, B):
    return B * (M + 1) * (L * (L + 1) * (L + 2) // 6)


def _cells(L, M, B):
    return B * (M + 1) * (L * (L + 1) // 2)


def draw(rng):
    """One more case: chains of 6 to 254 stages, 64 to 4096 slots, 1 to 256 plans, nothing costlier than the largest listed."""
    def between(lo, hi):
        return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5))))))

    while True:
        op = rng.choice(("solve",) * 7 + ("plan", "host", "readout"))
        L, M = between(6, 254), between(64, 4096)
        B = SWEEP if op == "plan" else between(1, 16 if op == "host" else 256)
        if _evals(L, M, B) <= _evals(192, 4096, 8) and _cells(L, M, B) <= _cells(192, 4096, 8):
            return {"op": op, "mix": rng.choice(sorted(MIXES)), "L": L, "M": M, "B": B, "extras": rng.random() < 0.3}


def _chains(mix, L, M, B, extras, rng):
    """Host arrays of B chains: uf, ub [B, L], wa [B, L+1], wabar [B, L], and wdelta, of, ob or None."""
    lo, hi, r0, r1 = MIXES[mix]
    n = 1 if mix == "sharded" else B
    if mix == "uniform":
        uf = rng.integers(1, 1000, (n, L), endpoint=True)
    elif mix == "pairs":  # an attention stage, then an MLP stage of twice its time
        u = rng.integers(200, 1000, (n, (L + 1) // 2), endpoint=True)
        uf = np.stack([u, 2 * u], axis=2).reshape(n, -1)[:, :L]
    elif mix == "sharded":
        uf = rng.integers(100, 3000, (n, L), endpoint=True)
    elif mix == "kinds":
        kind = np.array(KIND_TIMES)[rng.integers(0, 4, (n, L))]
        uf = rng.integers(kind[..., 0], kind[..., 1], endpoint=True)
    else:
        uf = np.clip(np.rint(rng.lognormal(7.0, 1.0, (n, L))), 1, 20000).astype(np.int64)
    ub = 2 * uf + rng.integers(0, np.maximum(1, uf // 4), endpoint=True)
    x_lo = max(1, round(lo * M))
    wa = rng.integers(x_lo, max(x_lo, round(hi * M)), (n, L + 1), endpoint=True)
    wabar = np.ceil(wa[:, 1:] * rng.uniform(r0, r1, (n, L))).astype(np.int64)
    if mix == "sharded":  # plan b divides sizes and times by its shard factor and pays for communication
        k = np.array([(1, 2, 4, 8)[b % 4] for b in range(B)])[:, None]
        wa, wabar = -(-wa // k), -(-wabar // k)
        uf = -(-uf // k) + rng.integers(0, 50, (B, L), endpoint=True)
        ub = -(-ub // k) + rng.integers(0, 50, (B, L), endpoint=True)
    wabar = np.maximum(wabar, wa[:, 1:])
    wdelta = of = ob = None
    if extras:
        wdelta = np.maximum(1, wa + rng.integers(-x_lo, x_lo, (B, L + 1), endpoint=True))
        of = rng.integers(0, x_lo, (B, L), endpoint=True)
        ob = rng.integers(0, x_lo, (B, L), endpoint=True)
    arrays = dict(uf=uf, ub=ub, wa=wa, wabar=wabar, wdelta=wdelta, of=of, ob=ob)
    return {k: None if v is None else np.ascontiguousarray(v, dtype=np.int32) for k, v in arrays.items()}


def _up(a, dtype=np.int32):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a, dtype=dtype)).cuda()


def _tables(s):
    L, M, B = s.L, s.M, s.B
    shape = (B, amd.ckpt_table_rows(L), amd.ckpt_row_pitch(M))
    s.cost = torch.empty(shape, dtype=torch.int32, device="cuda")
    s.arg = torch.empty(shape, dtype=torch.uint8, device="cuda")
    s.workspace = torch.empty(amd.ckpt_workspace_bytes(L, M, B), dtype=torch.uint8, device="cuda")
    s.tables = (s.cost[:, :, :M + 1], s.arg[:, :, :M + 1])  # the columns after M are padding


def _readout_buffers(s):
    L, B = s.L, s.B
    i32 = dict(dtype=torch.int32, device="cuda")
    i64 = dict(dtype=torch.int64, device="cuda")
    s.choice = torch.zeros(2, **i32)
    s.cap = L * (L + 1) // 2 + L
    s.ops = torch.zeros((B, s.cap, 2), dtype=torch.uint8, device="cuda")
    s.n_ops = torch.zeros(B, **i32)
    s.walk = torch.empty(amd.ckpt_schedule_workspace_bytes(L, B), dtype=torch.uint8, device="cuda")
    s.blocks, s.n_blocks = torch.zeros((B, L), **i32), torch.zeros(B, **i32)
    s.time, s.peak, s.status = torch.zeros(B, **i64), torch.zeros(B, **i64), torch.zeros(B, **i32)


def prepare(case, seed):
    L, M, B, op = case["L"], case["M"], case["B"], case["op"]
    s = SimpleNamespace(op=op, L=L, M=M, B=B)
    host = _chains(case["mix"], L, M, 1 if op == "plan" else B, case["extras"], np.random.default_rng(seed))
    if op == "host":
        s.batch = SimpleNamespace(L=L, M=M, B=B, **host)
        amd.load_library()
        return s
    amd.ckpt_init()
    if op == "plan":  # sizes in bytes, counted in slots of the smallest budget, plus what a slot does not divide
        rng = np.random.default_rng([seed, 1])
        s.bytes = {k: _up(v[0] * np.int64(SLOT_BYTES) - rng.integers(0, SLOT_BYTES, v[0].shape) * (v[0] > 0), np.int64)
                   for k, v in host.items() if k not in ("uf", "ub") and v is not None}
        s.chains = {k: torch.zeros((B, v.shape[1]), dtype=torch.int32, device="cuda") if v is not None else None
                    for k, v in host.items()}
        for k in ("uf", "ub"):
            s.chains[k].copy_(_up(host[k]).expand(B, L))
        s.budgets = torch.zeros(B, dtype=torch.int64, device="cuda")
    else:
        s.chains = {k: _up(v) for k, v in host.items()}
    _tables(s)
    if op in ("plan", "readout"):
        _readout_buffers(s)
    if op == "readout":
        _solve(s)
    return s


def _solve(s):
    c = s.chains
    amd.ckpt_solve_batched(c["uf"], c["ub"], c["wa"], c["wabar"], s.L, s.M, s.B, s.cost, s.arg, s.workspace,
                           wdelta=c["wdelta"], of=c["of"], ob=c["ob"])
    return s.tables


def _readout(s):
    c, L, M, B = s.chains, s.L, s.M, s.B
    budget = M - c["wa"][:, 0]  # the chain's input is not counted in m
    budget = budget.contiguous()
    amd.ckpt_select_plan(s.cost, L, M, B, budget, s.choice)
    amd.ckpt_schedule_batched(s.arg, c["wa"], c["wabar"], L, M, B, budget, s.ops, s.cap, s.n_ops, s.walk)
    amd.ckpt_block_indices_batched(s.ops, s.cap, s.n_ops, L, B, s.blocks, s.n_blocks)
    amd.ckpt_simulate_batched(c["uf"], c["ub"], c["wa"], c["wabar"], L, B, s.ops, s.cap, s.n_ops, s.time, s.peak,
                              s.status, wdelta=c["wdelta"], of=c["of"], ob=c["ob"])
    return s.choice, s.ops, s.n_ops, s.blocks, s.n_blocks, s.time, s.peak, s.status


def run(s):
    if s.op == "solve":
        return _solve(s)
    if s.op == "host":
        sol = amd.solve(s.batch)
        return sol.cost[:, :, :s.M + 1], sol.arg[:, :, :s.M + 1]
    if s.op == "readout":
        return _readout(s)
    by, out = s.bytes, s.chains
    amd.ckpt_discretize_sweep(by["wa"], by["wabar"], s.M * SLOT_BYTES, 1, 10, s.B, s.L, s.M, out["wa"], out["wabar"],
                              bytes_wdelta=by.get("wdelta"), bytes_of=by.get("of"), bytes_ob=by.get("ob"),
                              wdelta=out["wdelta"], of=out["of"], ob=out["ob"], budgets_out=s.budgets)
    return (s.budgets,) + _solve(s) + _readout(s)


def work(case):
    """Descriptors read once; five bytes stored for each cell, one addition and one comparison for each candidate; a list
    of about three operations a stage walked, annotated and executed."""
    L, M, B, op = case["L"], case["M"], case["B"], case["op"]
    per_stage = 4 * (7 if case["extras"] else 4)
    got = {"bytes": B * L * per_stage, "flops": 0}
    if op != "readout":
        got["bytes"] += 5 * _cells(L, M, B)
        got["flops"] += 2 * _evals(L, M, B)
    if op in ("plan", "readout"):
        got["bytes"] += B * L * (3 * 2 + 3 + 4)
        got["flops"] += B * L * 3 * 4
    return got


def tolerance(case):
    """Whole numbers throughout: every cell, candidate, operation and sum is exact."""
    return "exact"
