"""The work a user has the solver do, as cases that can be timed and compared.

``listed()`` holds the named cases, ``draw(rng)`` more of the same ranges.  ``prepare`` makes
what a program has before the call (procedures, a context, a resident plan), ``run`` is one
pass through the public entry points and returns every output of the analysis, ``work`` what
such a pass cannot do without.

Procedures are structured control-flow graphs: a region of n blocks is a sequence (0.40), an
if (0.20), an if/else (0.15) or a loop (0.25, three in ten do-while) whose parts split the
remaining blocks uniformly; whole loops and then single statements become kernels until the
wanted share of the blocks is on the device; accesses are Bernoulli bits per (block, variable).
``shapes`` says how many different graphs a batch holds; its procedures take them in turn,
each with its own variables and accesses (which keeps making the inputs quick).  The edges of a
graph follow from the case, so that every seed's outputs have the same shapes; which blocks are
kernels, their ids where these are shuffled, the accesses and the boundaries follow from the seed.

The ``sweeps`` counters that some entry points return next to the results are left out: they
say how the solver went about it and depend on the schedule, not on the input alone.
"""
import math
import random
from dataclasses import dataclass
from typing import Optional

import numpy as np

import paper_2406_13881_amd as ompd
from paper_2406_13881_amd.resident import ResidentBatch

NORMAL, BACK, LOOP_ENTRY = 0, 1, 2
FLAGS = {"default": 0, "eager": ompd.F_PLACEMENT_EAGER, "lazy": ompd.F_PLACEMENT_LAZY,
         "refine": ompd.F_PLACEMENT_REFINE}
# what a compiler asks for: the placement and its labels
PLACED = ("ins_entry_h", "ins_entry_d", "ins_edge_h", "ins_edge_d", "var_kind", "after_dev", "before_dev")
EDGES_PER_BLOCK = 1.37   # of the graphs grown below, on average


# ---- the cases --------------------------------------------------------------------------------

def span(min_blocks, max_blocks, min_vars, max_vars):
    return dict(min_blocks=min_blocks, max_blocks=max_blocks, min_vars=min_vars, max_vars=max_vars)


def listed():
    one = dict(count=1, shapes=1, depth=3, dense=True, order="source", extras=False, placement="default")
    return [
        # one small function analysed again and again in a tool that keeps it resident: latency
        dict(one, name="resident_64x32", path="resident", **span(64, 64, 32, 32)),
        # the smallest call a program can make: one small function, host arrays in and out
        dict(one, name="host_64x32", path="host", **span(64, 64, 32, 32)),
        # one function of odd sizes with boundaries of its own, marked scalars and the refinement
        dict(one, name="resident_777x333_refine", path="resident", **span(777, 777, 333, 333),
             extras=True, placement="refine"),
        # a large function of the batch range on its own
        dict(one, name="resident_8000x1500", path="resident", **span(8000, 8000, 1500, 1500)),
        # the largest function: deep loops, few accesses
        dict(one, name="resident_16384x2048", path="resident", **span(16384, 16384, 2048, 2048),
             depth=6, dense=False),
        # a whole code base resident on the card, every size of function: throughput
        dict(one, name="batch_1024", path="resident", count=1024, shapes=256, **span(16, 8192, 32, 4096)),
        # very many small functions at once
        dict(one, name="batch_2048_small", path="resident", count=2048, shapes=512, **span(16, 160, 8, 96)),
        # functions whose block ids are in no order, with scalars and boundaries, pure lazy placement
        dict(one, name="batch_96_shuffled_lazy", path="resident", count=96, shapes=48, **span(150, 3000, 40, 1500),
             order="shuffled", extras=True, placement="lazy"),
        # a compiler that hands over a source file's functions in host arrays and wants the placement
        dict(one, name="host_batch_9", path="host_batch", count=9, shapes=9, **span(60, 2000, 20, 900)),
        # a caller that owns device buffers and may not allocate, eager placement
        dict(one, name="noalloc_1501x700_eager", path="noalloc", **span(1501, 1501, 700, 700),
             placement="eager"),
        # whole-program analysis: summaries bottom up, contexts top down
        dict(name="program_64", path="program", procs=64, min_blocks=32, max_blocks=512, globals=128, locals=16,
             calls=1.5),
        # requests in flight through the serving loop: submitted together, collected in order
        dict(one, name="serving_9", path="serving", count=9, shapes=3, **span(16384, 16384, 2048, 2048), depth=6,
             dense=False),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["one", "one", "batch", "batch", "small", "host", "host_batch", "noalloc", "program", "serving"])
    if kind == "program":
        lo = log_int(16, 100)
        return dict(path="program", procs=log_int(6, 60), min_blocks=lo, max_blocks=log_int(lo + 20, 500),
                    globals=log_int(20, 128), locals=rng.randint(1, 16), calls=round(rng.uniform(0.8, 1.5), 2))
    depth = rng.choice([1, 2, 3, 3, 4, 6])
    case = dict(path="resident", count=1, shapes=1, depth=depth, dense=rng.random() < 0.6,
                order="shuffled" if rng.random() < 0.25 else "source", extras=rng.random() < 0.4,
                placement=rng.choice(["default", "default", "refine", "lazy", "eager"]))
    if kind in ("one", "host", "noalloc"):
        b = log_int(16, 14000 if kind == "one" else 3000)
        v = log_int(8, 2048 if kind == "one" else 700)
        case.update(path="resident" if kind == "one" else kind, **span(b, b, v, v))
    elif kind == "small":
        n = log_int(200, 2000)
        case.update(count=n, shapes=min(n, 400), **span(16, log_int(40, 160), 8, log_int(20, 96)))
    elif kind == "serving":
        b, v = log_int(200, 12000), log_int(60, 1500)
        case.update(path="serving", count=rng.randint(2, 9), shapes=2, **span(b // 2, b, v // 2, v))
    else:
        lo, lv = log_int(16, 200), log_int(8, 200)
        if kind == "batch":
            n = log_int(4, 500)
            case.update(count=n, shapes=min(n, 64), **span(lo, log_int(lo * 2, 6000), lv, log_int(lv * 2, 3000)))
        else:
            n = rng.randint(2, 9)
            case.update(path=kind, count=n, shapes=n, **span(lo, log_int(lo * 2, 2000), lv, log_int(lv * 2, 900)))
    return case


# ---- procedures -------------------------------------------------------------------------------

@dataclass
class Procedure:
    """One procedure as the entry points take it."""
    n_blocks: int
    n_vars: int
    entry: int
    exit: int
    succ_ptr: np.ndarray
    succ_idx: np.ndarray
    edge_kind: np.ndarray
    space: np.ndarray
    R: np.ndarray
    W: np.ndarray
    entry_valid_h: Optional[np.ndarray] = None
    entry_valid_d: Optional[np.ndarray] = None
    exit_live_h: Optional[np.ndarray] = None
    exit_live_d: Optional[np.ndarray] = None
    scalar: Optional[np.ndarray] = None

    def boundary(self):
        m = mask(self.n_vars)
        z = np.zeros_like(m)
        return tuple(d if v is None else v for v, d in
                     ((self.entry_valid_h, m), (self.entry_valid_d, z), (self.exit_live_h, m), (self.exit_live_d, z)))


@dataclass
class Program:
    """A whole program as ``analyze_program`` takes it."""
    procs: list
    n_globals: int
    call_proc: np.ndarray
    call_block: np.ndarray
    callee: np.ndarray
    roots: list


def mask(n_vars):
    m = np.full((n_vars + 63) // 64, ~np.uint64(0), np.uint64)
    if n_vars % 64:
        m[-1] = np.uint64((1 << (n_vars % 64)) - 1)
    return m


def sizes(case):
    """(blocks, variables) of each procedure: spread over the logarithm of their ranges."""
    def spread(lo, hi, i, step):
        return int(round(lo * (hi / lo) ** ((0.5 + i * step) % 1.0)))
    k = case["shapes"]
    return [(spread(case["min_blocks"], case["max_blocks"], i % k, 0.6180339887498949),
             spread(case["min_vars"], case["max_vars"], i, 0.4142135623730951))
            for i in range(case["count"])]


def grow(n_user, depth, device, edges, seed):
    """A structured graph of n_user blocks between ENTRY (0) and EXIT (n_user + 1) in source
    order: (succ_ptr, succ_idx, edge_kind, space); the edges are a function of `edges` alone."""
    rnd = random.Random(edges).random
    src, dst, heads, loops, saved = [], [], set(), [], []
    pend, nxt = [0], 1
    todo = [("region", n_user, 0)]
    while todo:
        op, n, d = todo.pop()
        if op == "region":
            u = rnd() if n > 1 else 1.0
            loop = 0.75 <= u < 1.0 and d < depth and (n > 2 or u < 0.925)
            if n > 1 and (u < 0.40 or (u >= 0.75 and not loop) or (0.60 <= u < 0.75 and n < 3)):
                a = 1 + int(rnd() * (n - 1))
                todo += [("region", n - a, d), ("region", a, d)]
                continue
            b, nxt = nxt, nxt + 1
            src += pend
            dst += [b] * len(pend)
            pend = [b]
            if n == 1:
                continue
            if u < 0.60:
                todo += [("join", b, 0), ("region", n - 1, d)]
            elif u < 0.75:
                a = 1 + int(rnd() * (n - 2))
                todo += [("merge", 0, 0), ("region", n - 1 - a, d), ("else", b, 0), ("region", a, d)]
            elif u < 0.925 or n < 3:
                heads.add(b)
                todo += [("while", b, 0), ("region", n - 1, d + 1)]
            else:
                heads.add(b)
                todo += [("until", b, 0), ("region", n - 2, d + 1)]
        elif op == "join":
            pend = pend + [n]
        elif op == "else":
            saved.append(pend)
            pend = [n]
        elif op == "merge":
            pend = saved.pop() + pend
        elif op == "while":
            src += pend
            dst += [n] * len(pend)
            loops.append((n, nxt))
            pend = [n]
        else:
            b, nxt = nxt, nxt + 1
            src += pend + [b]
            dst += [b] * len(pend) + [n]
            loops.append((n, nxt))
            pend = [b]
    src += pend
    dst += [n_user + 1] * len(pend)
    src, dst = np.array(src, np.int64), np.array(dst, np.int64)
    head = np.zeros(n_user + 2, bool)
    head[list(heads)] = True
    kind = np.where(head[dst], np.where(src >= dst, BACK, LOOP_ENTRY), NORMAL)
    at = np.argsort(src, kind="stable")
    ptr = np.zeros(n_user + 3, np.int32)
    ptr[1:] = np.cumsum(np.bincount(src, minlength=n_user + 2))
    space = np.zeros(n_user + 2, np.uint8)
    want, got = int(device * n_user), 0
    random.Random(seed).shuffle(loops)
    for a, z in loops:
        if got + z - a <= want and not space[a:z].any():
            space[a:z] = 1
            got += z - a
    host = 1 + np.flatnonzero(space[1:-1] == 0)
    space[np.random.default_rng(seed).permutation(host)[:want - got]] = 1
    return ptr, dst[at].astype(np.int32), kind[at].astype(np.uint8), space


def shuffle_ids(graph, seed):
    """The same graph with its block ids permuted (ENTRY and EXIT keep theirs)."""
    ptr, idx, kind, space = graph
    nb = len(space)
    perm = np.arange(nb)
    perm[1:-1] = 1 + np.random.default_rng(seed).permutation(nb - 2)
    src = perm[np.repeat(np.arange(nb), np.diff(ptr))]
    at = np.argsort(src, kind="stable")
    new = np.zeros(nb + 1, np.int32)
    new[1:] = np.cumsum(np.bincount(src, minlength=nb))
    moved = np.zeros_like(space)
    moved[perm] = space
    return new, perm[idx][at].astype(np.int32), kind[at], moved


def bits(gen, shape, sixtyfourths):
    """Words of independent bits, each set with probability sixtyfourths / 64."""
    x = np.zeros(shape, np.uint64)
    n = x.size
    for i in range(6):
        r = gen.random_raw(n).reshape(shape)
        x = x | r if (sixtyfourths >> i) & 1 else x & r
    return x


def procedure(graph, n_vars, dense, extras, gen):
    ptr, idx, kind, space = graph
    nb, m = len(space), mask(n_vars)
    rw = []
    for p in (13, 6) if dense else (3, 1):   # reads 0.20 and writes 0.09, or 0.05 and 0.016
        x = bits(gen, (nb, len(m)), p) & m
        x[0] = x[nb - 1] = 0
        rw.append(x)
    g = Procedure(nb, n_vars, 0, nb - 1, ptr, idx, kind, space, *rw)
    if extras:
        g.entry_valid_h = bits(gen, m.shape, 48) & m
        g.entry_valid_d = (~g.entry_valid_h | bits(gen, m.shape, 16)) & m
        g.exit_live_h, g.exit_live_d = bits(gen, m.shape, 32) & m, bits(gen, m.shape, 8) & m
        g.scalar = bits(gen, m.shape, 20) & m
        only_read = g.scalar & bits(gen, m.shape, 32)   # half of the scalars are never written by a kernel
        g.W[space == 1] &= ~only_read
    return g


def procedures(case, seed):
    gen = np.random.SFC64(seed)
    of = sizes(case)
    device = 0.30 if case["dense"] else 0.40
    graphs = [grow(of[k][0], case["depth"], device, 10007 * case["count"] + k, seed * 1000003 + k)
              for k in range(case["shapes"])]
    if case["order"] == "shuffled":
        graphs = [shuffle_ids(g, seed + k) for k, g in enumerate(graphs)]
    return [procedure(graphs[i % len(graphs)], nv, case["dense"], case["extras"], gen)
            for i, (_, nv) in enumerate(of)]


def call_graph(case):
    """(procedure, callee) of every call site: callees have higher indices, but for a cycle of
    two in every sixteen procedures."""
    rnd = random.Random(case["procs"] * 7919 + case["globals"])
    n, sites = case["procs"], []
    for i in range(n - 1):
        for _ in range(min(3, int(case["calls"] + rnd.random()))):
            sites.append((i, rnd.randint(i + 1, n - 1)))
        if i % 16 == 7:
            sites += [(i, i + 1), (i + 1, i)]
    return sites


def program(case, seed):
    gen, sites = np.random.SFC64(seed), call_graph(case)
    lo, hi = case["min_blocks"], case["max_blocks"]
    procs, blocks = [], [0] * len(sites)
    for i in range(case["procs"]):
        n = int(round(lo * (hi / lo) ** ((0.5 + i * 0.6180339887498949) % 1.0)))
        graph = grow(n, 3, 0.30, 10007 * case["procs"] + i, seed * 1000003 + i)
        mine = [k for k, s in enumerate(sites) if s[0] == i]
        host = 1 + np.flatnonzero(graph[3][1:-1] == 0)   # a call is made from a host statement
        for k, b in zip(mine, np.random.default_rng(seed + i).permutation(host)):
            blocks[k] = int(b)
        procs.append(procedure(graph, case["globals"] + case["locals"], True, False, gen))
    called = {q for _, q in sites}
    return Program(procs, case["globals"], np.array([s[0] for s in sites], np.int32), np.array(blocks, np.int32),
                   np.array([s[1] for s in sites], np.int32),
                   [0] + [i for i in range(1, case["procs"]) if i not in called])


# ---- what a program has before the call, and the call -----------------------------------------

def prepare(case, seed):
    ctx = ompd.Context(0)
    state = {"path": case["path"], "ctx": ctx}
    if case["path"] == "program":
        state["program"] = program(case, seed)
        return state
    state["flags"] = FLAGS[case["placement"]]
    procs = procedures(case, seed)
    if case["path"] in ("resident", "noalloc"):
        state["batch"] = ResidentBatch(ctx, procs, flags=state["flags"])
    else:
        state["procs"] = procs
    return state


def run(state):
    ctx, path = state["ctx"], state["path"]
    if path == "resident":
        state["batch"].run()
        return dict(state["batch"].out)
    if path == "noalloc":
        b = state["batch"]
        ompd.analyze_device(ctx, b.dcfgs, b.dres, state["flags"], noalloc=True)
        return dict(b.out)
    if path == "host":
        got = ompd.analyze_cfg(ctx, state["procs"][0], state["flags"])
        return {k: got[k] for k in ompd.OUTPUTS}
    if path == "host_batch":
        got = ompd.analyze_batch(ctx, state["procs"], state["flags"], want=PLACED)
        return [{k: r[k] for k in PLACED} for r in got]
    if path == "serving":
        live = [ompd.submit(ctx, g, state["flags"], want=PLACED) for g in state["procs"]]
        if not all(r.admitted for r in live):
            raise RuntimeError("a request was not admitted")
        return [{k: v for k, v in r.wait().items() if k != "sweeps"} for r in live]
    got = ctx.analyze_program(state["program"], want=PLACED)
    out = {k: np.concatenate([r[k].ravel() for r in got["results"]]) for k in PLACED}
    out["boundaries"] = np.concatenate([x for b in got["boundaries"] for x in b])
    return dict(out, summaries=got["summaries"], demands=got["demands"])


def work(case):
    """R and W (and the graph) in, every requested output out, once, in the stored layout.  The
    arithmetic is bitwise, a handful of operations per 64 facts, and counts no flops."""
    def moved(nb, nv, want):
        wd, ne = (nv + 63) // 64, int(EDGES_PER_BLOCK * nb)
        rows, edges = 8 * nb * wd, 8 * ne * wd
        total = 2 * rows + 4 * (nb + 1) + 5 * ne + nb
        for k in want:
            total += edges if k.startswith("ins_edge") else nv if k == "var_kind" else nb if k.endswith("_dev") else rows
        return total

    if case["path"] != "program":
        want = PLACED if case["path"] in ("serving", "host_batch") else ompd.OUTPUTS
        return {"bytes": sum(moved(nb + 2, nv, want) for nb, nv in sizes(case)), "flops": 0}
    sites = call_graph(case)
    of = {}
    for k, (i, _) in enumerate(sites):
        of.setdefault(i, []).append(k)
    called = {q for _, q in sites}
    todo = [(i, ()) for i in range(case["procs"]) if i == 0 or i not in called]
    seen = set(todo)
    while todo:   # a context: a procedure and the last two call sites that led to it
        i, at = todo.pop()
        for k in of.get(i, []):
            c = (sites[k][1], (at + (k,))[-2:])
            if c not in seen:
                seen.add(c)
                todo.append(c)
    lo, hi = case["min_blocks"], case["max_blocks"]
    nv = case["globals"] + case["locals"]
    return {"bytes": sum(moved(2 + int(round(lo * (hi / lo) ** ((0.5 + i * 0.6180339887498949) % 1.0))), nv,
                               PLACED) for i, _ in seen), "flops": 0}


def exact(case, seed):
    """Every output is whole bits; there are no rounded numbers to hold against a wider type."""
    return None
