"""GPU parity of the strips with the oracle at the edges of their shapes: one to four words per
strip, CFGs on both sides of each wavefront count, blocks with fewer, as many and more edges than a
row of 16 lanes holds, long chains (a level per block) and wide levels, in launches that leave the
GPU idle and in launches that fill it, with and without a call's and a caller's options."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

KEYS = ("nu_h", "nu_d", "ave_h", "ave_d", "avf_h", "avf_d", "ins_entry_h", "ins_entry_d",
        "ins_edge_h", "ins_edge_d", "var_kind", "after_dev", "before_dev")


@pytest.fixture(scope="module")
def ctx():
    import paper_2406_13881_amd as ompd
    c = ompd.Context(0)
    yield c
    c.close()


def _blocks(rng, n, n_vars):
    out = [(0, [], [])]
    for _ in range(n):
        out.append((int(rng.random() < 0.4), sorted(set(rng.integers(0, n_vars, 5).tolist())) if n_vars else [],
                    sorted(set(rng.integers(0, n_vars, 2).tolist())) if n_vars else []))
    return out + [(0, [], [])]


def _fan(n, n_vars, seed):
    """A switch of n cases in a loop, so that two blocks have n edges and one has a BACK edge."""
    rng = np.random.default_rng(seed)
    join, ex = n + 2, n + 3
    edges = [(0, 1, 2)] + [(1, 2 + k, 0) for k in range(n)] + [(2 + k, join, 0) for k in range(n)]
    return synth.from_edges(_blocks(rng, n + 2, n_vars), edges + [(join, 1, 1), (join, ex, 0)], n_vars)[0]


def _chain(n, n_vars, seed):
    """n blocks in a row, a loop around every third pair: a level per block, a BACK edge at each distance."""
    rng = np.random.default_rng(seed)
    edges = [(b, b + 1, 2 if b % 3 == 0 and b + 2 <= n else 0) for b in range(n + 1)]
    edges += [(b + 2, b + 1, 1) for b in range(0, n - 1, 3)] + ([(n, 1, 1)] if n > 3 else [])
    return synth.from_edges(_blocks(rng, n, n_vars), edges, n_vars)[0]


def _cfgs(n_vars):
    out = [_fan(n, n_vars, 100 + n) for n in (1, 2, 15, 16, 17, 31, 33, 64, 65)]
    out += [_chain(n, n_vars, 200 + n) for n in (1, 6, 30, 31, 62, 63, 126, 198, 199, 254, 399)]
    out += [synth.permute_blocks(_chain(150, n_vars, 7), 8)[0], synth.random_dag(9, 90, n_vars, p_loop_entry=0.3)]
    return out


@pytest.mark.parametrize("copies", [1, 60])
@pytest.mark.parametrize("n_vars", [0, 1, 64, 65, 192, 193, 257, 449])
def test_strip_edges(ctx, n_vars, copies):
    cfgs = _cfgs(n_vars)
    want = [oracle.solve(c) for c in cfgs]
    print("strips: %d variables, %d copies" % (n_vars, copies), flush=True)
    got = ctx.analyze_batch(cfgs * copies)
    for i in range(len(cfgs) * copies):
        for k in KEYS:
            g, r = np.asarray(got[i][k]), np.asarray(want[i % len(cfgs)][k])
            assert np.array_equal(g, r.reshape(g.shape)), (i % len(cfgs), k)


@pytest.mark.parametrize("n_vars", [65, 193])
def test_strip_alone(ctx, n_vars):
    """Each CFG in a launch of its own (a row of lanes per word), also with a cap that its rounds stay under."""
    for i, cfg in enumerate(_cfgs(n_vars)):
        want = oracle.solve(cfg)
        for flags in (0, 1000 << 16):
            got = ctx.analyze_batch([cfg], flags=flags)[0]
            for k in KEYS:
                g = np.asarray(got[k])
                assert np.array_equal(g, np.asarray(want[k]).reshape(g.shape)), (i, flags, k)


def test_strip_sweeps_repeat(ctx):
    """The sweeps reported do not depend on which wavefront of a strip is ahead."""
    cfgs = [synth.c3_item(i) for i in range(8)] + [_chain(1500, 130, 3), _fan(40, 130, 4)]
    runs = [[r["sweeps"] for r in ctx.analyze_batch(cfgs)] for _ in range(6)]
    for again in runs[1:]:
        assert np.array_equal(np.asarray(runs[0]), np.asarray(again))


def _dense(n, n_edges, n_vars, seed):
    """A chain of n blocks; edges of every kind between blocks of its first half make it n_edges."""
    rng = np.random.default_rng(seed)
    edges = [(b, b + 1, 0) for b in range(n + 1)]
    a, b = rng.integers(1, n // 2, n_edges), rng.integers(1, n // 2, n_edges)
    edges += [(int(x), int(y), 1 if x >= y else 2 * int(k < 0.2)) for x, y, k in zip(a, b, rng.random(n_edges))]
    return synth.from_edges(_blocks(rng, n, n_vars), edges[:n_edges], n_vars)[0]


@pytest.mark.parametrize("n_edges", [65533, 65534, 65535, 65536, 70001, 140000])
def test_strip_many_edges(ctx, n_edges):
    """Edge entries that fit the 16 bits of a lane record and ones that do not, up to the largest 17-bit
    ones, with the refinement (whose backward sweep reads the copies of its edges) and without; all by
    level, alone and in a launch that fills the GPU."""
    import json
    import paper_2406_13881_amd as ompd
    from paper_2406_13881_amd.resident import ResidentBatch
    cfg = _dense(3000, n_edges, 70, n_edges)
    assert len(cfg.succ_idx) == n_edges
    for flags, placement in ((0, 0), (ompd.F_PLACEMENT_REFINE, oracle.PLACEMENT_REFINE)):
        want = oracle.solve(cfg, placement=placement)
        for copies in (1, 200):
            print("%d edges, flags %d, %d copies" % (n_edges, flags, copies), flush=True)
            rb = ResidentBatch(ctx, [cfg] * copies, flags=flags)
            assert json.loads(rb.plan.describe())["tiles"] == 0   # (of the walk)
            rb.run()
            assert (rb.plan.status() == 0).all()
            for i in {0, copies - 1}:
                got = rb.fetch(i)
                for k in KEYS:
                    g = np.asarray(got[k])
                    assert np.array_equal(g, np.asarray(want[k]).reshape(g.shape)), (flags, copies, i, k)
            rb.close()


@pytest.mark.parametrize("refine", [False, True])
def test_strip_sweep_cap(ctx, refine):
    """A cap counts the same sweeps by level as on the walk: a capped call reports the walk's, a cap of as
    many as the slowest phase needs finishes, one less stops; uncapped rounds are never fewer."""
    import paper_2406_13881_amd as ompd
    base = ompd.F_PLACEMENT_REFINE if refine else 0
    cfgs = [synth.c1(3), synth.c3_item(5, n_user=700, n_vars=300), synth.permute_blocks(synth.c1(4), 5)[0],
            _chain(400, 130, 3), _fan(40, 130, 4), _dense(300, 4000, 70, 5), synth.random_dag(9, 90, 70, p_loop_entry=0.3),
            synth.make_cfg(5_003, n_user=160, n_vars=90, max_loop_depth=6, device_frac=0.4, irr_loop_frac=0.2)]
    for i, cfg in enumerate(cfgs):
        need = ctx.analyze_cfg(cfg, flags=base | ompd.F_SCHED_WALK)["sweeps"]
        most = int(max(need))
        for flags in (base, base | ompd.F_SCHED_LEVEL):
            assert (ctx.analyze_cfg(cfg, flags=flags)["sweeps"] >= need).all(), i
            got = ctx.analyze_cfg(cfg, flags=flags | (most << 16))
            assert np.array_equal(got["sweeps"], need), (i, got["sweeps"], need)
            want = oracle.solve(cfg, placement=oracle.PLACEMENT_REFINE if refine else 0)
            for k in KEYS:
                g = np.asarray(got[k])
                assert np.array_equal(g, np.asarray(want[k]).reshape(g.shape)), (i, k)
            if most > 1:
                with pytest.raises(ompd.OmpdError) as e:
                    ctx.analyze_cfg(cfg, flags=flags | ((most - 1) << 16))
                assert e.value.code == ompd.OMPD_E_NOCONVERGE, i


@pytest.mark.parametrize("n_blocks,strips", [(0, 1), (1, 1), (25_000, 1), (32_000, 1), (32_001, 0)])
def test_strip_most_blocks(ctx, n_blocks, strips):
    """CFGs whose peel is the last that LDS holds (0: 8 bytes a block and 8 more), the first that global
    memory does (1), and the largest that the strips take; ids in order and shuffled."""
    import json
    from paper_2406_13881_amd.resident import ResidentBatch
    if n_blocks < 2:
        n_blocks += ctx.device_info()["lds_bytes"] // 8 - 1
    cfg = synth.make_cfg(n_blocks, n_user=n_blocks - 2, n_vars=70, max_loop_depth=4, device_frac=0.3,
                         irr_loop_frac=0.01, p_read=0.05, p_write=0.02)
    assert cfg.n_blocks == n_blocks
    cfgs = [cfg, synth.permute_blocks(cfg, 1)[0], _chain(n_blocks - 2, 70, 2)]
    print("%d blocks" % n_blocks, flush=True)
    rb = ResidentBatch(ctx, cfgs)
    assert json.loads(rb.plan.describe())["strip_cfgs"] == strips * len(cfgs)
    rb.run()
    assert (rb.plan.status() == 0).all()
    for i, c in enumerate(cfgs):
        got, want = rb.fetch(i), oracle.solve(c)
        for k in KEYS:
            g = np.asarray(got[k])
            assert np.array_equal(g, np.asarray(want[k]).reshape(g.shape)), (i, k)
    rb.close()


def test_strips_that_do_not_fit_their_scratch(ctx):
    """The allocation-free entry point and the serving loop solve by the walk what their memory holds
    only that way (the sweeps show it: the strips' rounds are more)."""
    import paper_2406_13881_amd as ompd
    from paper_2406_13881_amd.resident import ResidentBatch
    cfg = synth.c3_item(5, n_user=300, n_vars=32)
    walk = ctx.analyze_cfg(cfg, flags=ompd.F_SCHED_WALK)
    assert (ctx.analyze_cfg(cfg)["sweeps"] > walk["sweeps"]).any()

    def same(got, tag):
        for k in KEYS:
            g = np.asarray(got[k])
            assert np.array_equal(g, np.asarray(walk[k]).reshape(g.shape)), (tag, k)

    for copies, by_walk in ((100, False), (2000, True)):   # of 256 MiB
        rb = ResidentBatch(ctx, [cfg] * copies)
        sweeps = ompd.analyze_device(ctx, rb.dcfgs, rb.dres, 0, noalloc=True)
        assert (sweeps == walk["sweeps"]).all() == by_walk, copies
        for i in (0, copies - 1):
            same(rb.fetch(i), "no allocation, %d" % copies)
        rb.close()
    for budget in range(100 << 10, 4 << 20, 20 << 10):   # the least that admits the request holds its walk
        small = ompd.Context(0, budget)
        try:
            r = ompd.submit(small, cfg)
            if r.admitted:
                got = r.wait()
                assert np.array_equal(got["sweeps"], walk["sweeps"]), budget
                same(got, "serving, %d bytes" % budget)
                break
        finally:
            small.close()
    else:
        assert False, "no budget admitted the request"


def _wild(seed):
    """A random graph with nothing structured about it: edges of any kind in any direction (cycles
    without a BACK edge, BACK edges that go forward, repeated edges, self loops), ids shuffled, random
    boundaries, now and then marked scalars."""
    rng = np.random.default_rng(seed)
    n, nv = int(rng.integers(1, 160)), int(rng.choice([1, 31, 64, 65, 130, 260, 520]))
    edges = [(int(rng.integers(0, b)), b) for b in range(1, n + 1)]
    edges += [(b, int(rng.integers(b + 1, n + 2))) for b in range(1, n + 1)]
    extra = int(rng.integers(0, 1 + int(n * rng.choice([0.2, 1, 4]))))
    edges += [(int(a), int(b)) for a, b in zip(rng.integers(1, n + 1, extra), rng.integers(1, n + 1, extra))]
    kinds = [0 if b == n + 1 else int(rng.choice([0, 2])) if a == 0 else
             int(rng.choice([0, 0, 1, 2])) if a >= b else int(rng.choice([0, 0, 0, 0, 2, 1])) for a, b in edges]
    cfg = synth.from_edges(_blocks(rng, n, nv), [(a, b, k) for (a, b), k in zip(edges, kinds)], nv)[0]
    if rng.random() < 0.5:
        cfg = synth.permute_blocks(cfg, seed)[0]
    m = synth.var_mask(nv)
    word = lambda: rng.integers(0, 1 << 63, size=cfg.wd, dtype=np.uint64) & m
    if rng.random() < 0.5:
        cfg.entry_valid_d = word()
        cfg.entry_valid_h = (~cfg.entry_valid_d | word()) & m
        cfg.exit_live_h, cfg.exit_live_d = word(), word()
    if rng.random() < 0.4:
        synth.mark_scalars(cfg, seed)
    return cfg


@pytest.mark.parametrize("variant", ["DEFAULT", "EAGER", "LAZY", "REFINE"])
def test_strip_wild_graphs(ctx, variant):
    import paper_2406_13881_amd as ompd
    flag = 0 if variant == "DEFAULT" else getattr(ompd, "F_PLACEMENT_" + variant)
    cfgs = [_wild(1000 + s) for s in range(150)]
    want = [oracle.solve(c, placement=0 if variant == "DEFAULT" else getattr(oracle, "PLACEMENT_" + variant)) for c in cfgs]
    for copies, flags in ((1, flag), (4, flag), (1, flag | (3000 << 16))):   # room for every strip, queueing, one run each
        print("wild graphs: %s, %d copies, flags %x" % (variant, copies, flags), flush=True)
        got = ctx.analyze_batch(cfgs * copies, flags=flags)
        for i in range(len(cfgs) * copies):
            for k in KEYS + ("fp_clause",):
                g = np.asarray(got[i][k])
                assert np.array_equal(g, np.asarray(want[i % len(cfgs)][k]).reshape(g.shape)), (i % len(cfgs), copies, flags, k)


def test_strip_malformed(ctx):
    """What the walk refuses the strips refuse, and the CFGs beside it are solved."""
    import copy
    import paper_2406_13881_amd as ompd
    good = _chain(40, 70, 1)
    n = good.n_blocks

    def change(field, at, value):
        c = copy.deepcopy(good)
        getattr(c, field)[at] = value
        return c

    def edges(extra, blocks=None):
        rng = np.random.default_rng(3)
        base = [(b, b + 1, 0) for b in range(n - 1)]
        return synth.from_edges(_blocks(rng, n - 2, 70), base + extra if blocks is None else blocks, 70)[0]

    cut = [(b, b + 1, 0) for b in range(n - 1) if b != 20]
    bad = {"row start": change("succ_ptr", 0, 1), "row end": change("succ_ptr", n, 3), "rows out of order": change("succ_ptr", 7, 30),
           "successor": change("succ_idx", 5, n), "negative successor": change("succ_idx", 5, -1),
           "edge into ENTRY": change("succ_idx", 5, good.entry), "kind": change("edge_kind", 5, 3), "space": change("space", 5, 2),
           "ENTRY on the device": change("space", good.entry, 1), "padding": change("R", (5, 1), np.uint64(1) << np.uint64(63)),
           "ENTRY reads": change("R", (good.entry, 0), np.uint64(1)), "BACK out of ENTRY": change("edge_kind", 0, 1),
           "BACK into EXIT": change("edge_kind", list(good.succ_idx).index(good.exit), 1), "edge out of EXIT": edges([(n - 1, 5, 0)]),
           "no way in": edges(None, cut + [(20, 22, 0)]), "no way out": edges(None, cut + [(19, 21, 0)]),
           "cycle without a way in": edges(None, [e for e in cut if e[0] not in (19, 21)] + [(19, 22, 0), (20, 21, 0), (21, 20, 0), (21, 22, 0)]),
           "cycle without a way out": edges(None, [e for e in cut if e[0] not in (19, 21)] + [(19, 20, 0), (19, 22, 0), (20, 21, 0), (21, 20, 1)])}
    gap = copy.deepcopy(good)
    gap.entry_valid_h, gap.entry_valid_d = np.zeros(2, np.uint64), np.zeros(2, np.uint64)
    bad["variables valid nowhere"] = gap
    from paper_2406_13881_amd.resident import ResidentBatch
    want = oracle.solve(good)
    for copies in (1, 400):   # room for every strip, and not
        rb = ResidentBatch(ctx, [good] + list(bad.values()) + [good] * copies)
        rb.run()
        status = rb.plan.status()
        for i, name in enumerate(bad):
            assert status[1 + i] == ompd.OMPD_E_INVAL, (name, status[1 + i])
        for i in (0, 1 + len(bad), len(bad) + copies):
            assert status[i] == 0
            got = rb.fetch(i)
            for k in KEYS:
                g = np.asarray(got[k])
                assert np.array_equal(g, np.asarray(want[k]).reshape(g.shape)), (i, k)
        rb.close()
