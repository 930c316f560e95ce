"""Performance cases: what a user of the framework has it do, through its public entry points.

A case names a configuration of workloads.py and the largest sizes m, k, n of the
goal it is solved under: the lattice then holds every allowed size up to those.  The seed draws the
target's cost coefficients (and the Specs that are asked for).  Five operations:

  solve     fill and compress every lattice of the configuration into buffers the program keeps
            (binding.solve_lattices); the outputs are the dense tables and the number of boxes
  database  the same, and the compressed tables (both box lists of every lattice) taken to the host
            and appended to the database image that the program keeps there
  query     the costs and rewrites of `points` Specs out of a solved table (Table.query)
  lookup    the same out of the box lists alone (Table.query with compressed=True)
  program   the schedule of the goal Spec out of a solved table (Table.schedule)

All results are integers, so every comparison is exact.
"""
import math

import numpy as np
import torch

from paper_2505_01637_amd import binding as B
from paper_2505_01637_amd import workloads as W

LISTS = ("decisions", "costs")
PROGRAM_MOST = 128          # nodes of a program (a goal's program has a few dozen)
SCRATCH_MOST = 8 << 30      # bytes of scratch per lattice; smaller lattices get what suffices for any contents
LABEL = {1: "M", 2: "M", 3: "M", 4: "M", 5: "F", 6: "P", 7: "B", 9: "M", 10: "G", 11: "F", 12: "M"}   # the table that answers


def _case(name, op, config, m, k, n, points=0):
    case = {"op": op, "config": config, "m": m, "k": k, "n": n, "points": points}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest solve: a kernel author's inner loop over one small tile (two levels, all
        # sizes to 16, 32,768 Specs); launches, synchronisations and host work are what it costs
        _case("solve_tiny_tile", "solve", 1, 16, 16, 16),
        # the vector-matrix product of a language model's decoding step, 1 x 2048 x 16384, bf16
        # inputs and a weight matrix of either layout (92,160 Specs in a long chain of sizes)
        _case("solve_vecmat_bf16", "solve", 3, 1, 2048, 16384),
        # a Matmul of any size to 64, every integer (ragged tiles included): 16.8 M Specs
        _case("solve_matmul_all_sizes", "solve", 2, 64, 64, 64),
        # a batched Matmul with transposing Moves, a layout per operand: 23.7 M Specs
        _case("solve_batched_layouts", "solve", 4, 512, 512, 512),
        # the largest: Matmul -> bias add -> ReLU under a 2048-cube goal, three tables, 478 M Specs
        _case("solve_pipeline", "solve", 5, 2048, 2048, 2048),
        # peak-memory bounds as coordinates: 41 M Specs, all of them with an implementation to find
        _case("solve_memory_bounds", "solve", 7, 64, 64, 64),
        # Moves as Specs with packed layouts and the Matmul that reads their table: 84 M Specs
        _case("solve_packed_moves", "solve", 12, 32, 32, 32),
        # two Matmuls composed, as in an MLP or attention: 67 M Specs, a quarter of them admissible
        _case("solve_two_matmuls", "solve", 10, 128, 128, 128),
        # an ordinary layer of odd sizes, solved and stored: the box lists are what is kept on disk
        _case("database_pipeline_ragged", "database", 5, 100, 72, 56),
        # a scheduler that asks a solved table for many Specs at once (no multiple of any chunk)
        _case("query_points", "query", 4, 128, 128, 128, 100003),
        # the same for a database that was kept as boxes only
        _case("lookup_points_in_boxes", "lookup", 4, 128, 128, 128, 100003),
        # the program of one goal, rewrite by rewrite: single-Spec questions, latency alone
        _case("program_of_goal", "program", 5, 256, 256, 256),
    ]


def _log_uniform(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["solve"] * 6 + ["database", "query", "lookup", "program"])
    points = _log_uniform(rng, 1, 200000) if op in ("query", "lookup") else 0
    if op == "database":
        config, lo, hi = rng.choice([4, 5]), 12, 100
    elif op in ("query", "lookup"):
        config, lo, hi = rng.choice([4, 5]), 12, 128
    elif op == "program":
        config, lo, hi = 5, 16, 256
    else:
        config = rng.choice([1, 2, 3, 4, 5, 5, 6, 7, 9, 10, 11, 12])
        lo, hi = {1: (3, 16), 2: (5, 64), 3: (2, 2048), 4: (12, 512), 5: (12, 2048), 6: (5, 64), 7: (2, 64), 9: (5, 32),
                  10: (4, 128), 11: (12, 256), 12: (5, 32)}[config]
    m, k, n = (_log_uniform(rng, lo, hi) for _ in range(3))
    if config == 3:
        m, n = 1, _log_uniform(rng, 2, 16384)
    if config in (9, 10, 12):       # these read one table along several dimensions: one size list for all
        k = n = m
    return _case(None, op, config, m, k, n, points)


def _config(case, seed):
    """The configuration with its size lists cut at the case's m, k, n."""
    cfg = W.config(case["config"], seed=seed)
    most = (None, case["m"], case["k"], case["n"])
    for _, lat, _ in cfg["lattices"]:
        for d in (1, 2, 3):
            lat["sizes"][d] = [x for x in lat["sizes"][d] if x <= most[d]]
        if lat["kind"] == W.KIND_MATMUL_CHAIN:          # p, the dimension the two Matmuls share
            lat["sizes"][0] = [x for x in lat["sizes"][0] if x <= case["k"]]
    return cfg


def prepare(case, seed):
    cfg = _config(case, seed)
    target = B.Target(cfg["target"])
    device = torch.device("cuda", torch.cuda.current_device())
    buffers = {}
    for label, lat, _ in cfg["lattices"]:
        cost, arg, scratch = B.table_bytes(target, lat)
        buffers[label] = tuple(torch.empty(x, dtype=torch.uint8, device=device) for x in (cost, arg, min(scratch, SCRATCH_MOST)))
    state = {"op": case["op"], "target": target, "lattices": cfg["lattices"], "buffers": buffers, "tables": None, "image": {}}
    if case["op"] == "database":
        # room for the box lists: far fewer than Specs, except in small lattices
        for label, lat, _ in cfg["lattices"]:
            n = W.n_specs(cfg["target"], lat)
            room = n if n <= 1 << 20 else n // 4
            state["image"][label] = {name: np.zeros((room, B.BOX_DTYPE.itemsize // 8), dtype=np.int64) for name in LISTS}
    if case["op"] in ("solve", "database"):
        return state
    tables = B.solve_lattices(target, cfg["lattices"], buffers=buffers)
    tab = tables[LABEL[case["config"]]]
    state["tables"], state["table"] = tables, tab
    if case["op"] == "program":
        sizes = tab.lattice["sizes"]
        top = cfg["target"]["n_levels"] - 1
        state["goal"] = tab.coord_of_spec([s[-1] for s in sizes], [top] * 5, layouts=[0] * 5, dtypes=[0] * 5)
        return state
    # Specs that have an implementation, all over the table
    cost = buffers[LABEL[case["config"]]][0].view(torch.int64)
    finite = torch.nonzero(cost != -1).reshape(-1)
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    pick = finite[torch.randint(finite.numel(), (case["points"],), generator=gen, device=device)].cpu().numpy()
    state["specs"] = np.stack(np.unravel_index(pick, tab.extents), axis=1).astype(np.uint32)
    return state


def _tables(state):
    out = {}
    for label, tab in state["tables"].items():
        cost, arg, _ = state["buffers"][label]
        out[label] = {"cost": cost.view(torch.int64), "rewrite": arg.view(torch.int16),
                      "decision_boxes": int(tab.stats.n_decision_boxes), "cost_boxes": int(tab.stats.n_cost_boxes)}
    return out


def run(state):
    op = state["op"]
    if op in ("solve", "database"):
        state["tables"] = B.solve_lattices(state["target"], state["lattices"], buffers=state["buffers"])
        out = _tables(state)
        if op == "database":
            for label, tab in state["tables"].items():
                for which, name in enumerate(LISTS):
                    boxes = tab.boxes(which)
                    image = state["image"][label][name]
                    image[:len(boxes)] = boxes.view(np.int64).reshape(len(boxes), -1)
                    out[label][name] = image
        return out
    if op == "program":
        nodes = state["table"].schedule(state["goal"])
        # (table, rewrite, cost, children, coordinate) of every node
        out = np.zeros((PROGRAM_MOST, 20), dtype=np.int64)
        for i, (table, x, rewrite, cost, children) in enumerate(nodes):
            out[i, :4 + len(x)] = (table, rewrite, cost, children) + x
        return {"nodes": len(nodes), "program": out}
    cost, rewrite = state["table"].query(state["specs"], compressed=op == "lookup")
    return {"cost": cost.view(np.int64), "rewrite": rewrite.view(np.int16)}


def work(case):
    """Bytes: the dense tables written once (cost 8, rewrite 2 per Spec); for questions the
    coordinates read and the answers read from the table and written.  Nothing is floating point."""
    cfg = _config(case, 1)
    specs = sum(W.n_specs(cfg["target"], lat) for _, lat, _ in cfg["lattices"])
    if case["op"] in ("solve", "database"):
        return {"bytes": 10 * specs, "flops": 0}
    dims = max(len(W.coord_extents(cfg["target"], lat)) for _, lat, _ in cfg["lattices"])
    if case["op"] == "program":
        return {"bytes": 32 * (10 + 4 * dims), "flops": 0}
    return {"bytes": case["points"] * (4 * dims + 20), "flops": 0}


def tolerance(case):
    return "exact"
