"""CPU tests of the library's host code: libompd on a stand-in for the HIP runtime
(tests/cpp/hip_standin.cpp), which checks every copy against the allocations, bounds the device
memory, and counts kernels instead of running them.  Each test is a program of its own, so that the
stand-in is the only runtime in the process."""
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import sys
sys.modules["torch"] = None   # (it brings a HIP runtime of its own)
sys.path.insert(0, %r)
import ctypes, json
from types import SimpleNamespace
import numpy as np
import paper_2406_13881_amd as ompd
import synth
lib = ompd.lib()
hip = ctypes.CDLL("libamdhip64.so.7")
hip.standin_first.restype = hip.standin_events.restype = ctypes.c_char_p
hip.standin_live.restype = hip.standin_alloc_size.restype = ctypes.c_size_t
for f in ("launches", "items"):
    getattr(hip, "standin_" + f).argtypes = [ctypes.c_char_p]
    getattr(hip, "standin_" + f).restype = ctypes.c_long
hip.standin_allocs.restype = hip.standin_violations.restype = ctypes.c_long
hip.standin_budget.argtypes = [ctypes.c_size_t]
hip.standin_fail_alloc.argtypes = hip.standin_alloc_size.argtypes = [ctypes.c_long]

def on_device(a):
    p = ctypes.c_void_p()
    a = np.ascontiguousarray(a)
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(a.nbytes)) == 0
    assert hip.hipMemcpy(p, ctypes.c_void_p(a.ctypes.data), ctypes.c_size_t(a.nbytes), 1) == 0
    return p.value

def resident(ctx, cfgs, flags=0):
    # a plan of CFGs in device memory that asks for the map kinds and a label
    D, R = [], []
    for c in cfgs:
        D.append(ompd.DeviceCFG(n_blocks=c.n_blocks, n_edges=len(c.succ_idx), n_vars=c.n_vars, entry=c.entry, exit=c.exit,
                                succ_ptr=on_device(c.succ_ptr), succ_idx=on_device(c.succ_idx),
                                edge_kind=on_device(c.edge_kind), space=on_device(c.space),
                                read_bits=on_device(c.R), write_bits=on_device(c.W)))
        R.append(ompd.DeviceResult(var_kind=on_device(np.zeros(c.n_vars, np.uint8)),
                                   after_dev=on_device(np.zeros(c.n_blocks, np.uint8))))
    return ompd.Plan(ctx, D, R, flags)

def chain(n, n_vars, seed=1):
    rng = np.random.default_rng(seed)
    blocks = [(0, [], [])] + [(0, [int(rng.integers(0, n_vars))], []) for _ in range(n)] + [(0, [], [])]
    return synth.from_edges(blocks, [(b, b + 1, 0) for b in range(n + 1)], n_vars)[0]
""" % ROOT


@pytest.fixture(scope="module")
def standin(tmp_path_factory):
    out = tmp_path_factory.mktemp("hip")
    so = out / "libamdhip64.so.7"
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "cpp", "hip_standin.cpp"), "-Wl,-soname,libamdhip64.so.7",
                    "-o", str(so)], check=True)
    return str(out)


def run(standin, body):
    env = dict(os.environ, LD_LIBRARY_PATH=standin)
    code = PRELUDE + textwrap.dedent(body) + "\nassert hip.standin_violations() == 0, hip.standin_first()\n"
    p = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr


def test_calls_stay_inside_their_allocations_and_give_them_back(standin):
    run(standin, """
        ctx = ompd.Context(0, 256 << 20)
        ctx.analyze_batch([synth.c1(0), synth.c1(1), synth.c3_item(2)])
        ctx.analyze_program(synth.c4(20))
        r = ompd.submit(ctx, synth.c1(3))
        assert r.admitted
        r.wait()
        ctx.close()
        assert hip.standin_live() == 0, hip.standin_live()
    """)


def test_program_work_lists_larger_than_their_buffer(standin):
    """96 call sites in each of three procedures in a row give 96^3 call-table items of 80 bytes,
    more than the 64 MiB their buffers hold: every item still reaches the kernel, and no copy leaves
    an allocation."""
    run(standin, """
        n = 96
        procs = [chain(n, 2, seed) for seed in range(4)]
        prog = SimpleNamespace(procs=procs, n_globals=1, roots=[0],
                               call_proc=[p for p in range(3) for _ in range(n)],
                               call_block=[1 + k for _ in range(3) for k in range(n)],
                               callee=[p + 1 for p in range(3) for _ in range(n)])
        ctx = ompd.Context(0, 64 << 20)
        got = ctx.analyze_program(prog, want=("after_dev",))
        assert len(got["contexts"]) == 1 + n + 2 * n * n
        # the summaries' tables, then those of every context, in the liveness and in the validity system
        per_round = 3 * n + 2 * (n + n * n + n * n * n)
        assert hip.standin_items(b"k_calltab") == got["rounds"] * per_round, hip.standin_items(b"k_calltab")
        ctx.close()
    """)


def test_every_failed_allocation_is_reported_as_one(standin):
    """Each device allocation of a call fails in turn: the call succeeds all the same or returns
    OMPD_E_NOMEM, and gives back what it had."""
    run(standin, """
        cfgs, prog = [synth.c1(0), synth.c3_item(2)], synth.c4(12)
        ctx = ompd.Context(0, 64 << 20)
        for call in (lambda: ctx.analyze_batch(cfgs), lambda: ctx.analyze_program(prog)):
            before = hip.standin_allocs()
            call()
            n = hip.standin_allocs() - before
            for k in range(n):
                hip.standin_fail_alloc(k)
                try:
                    call()
                except ompd.OmpdError as e:
                    assert e.code == ompd.OMPD_E_NOMEM, (k, e)
                hip.standin_fail_alloc(-1)
                assert hip.standin_live() == 0, k
        ctx.close()
    """)


def test_kept_plans_give_way_to_the_next(standin):
    """A program in memory that holds its arena and any one of its batches, but not several: plans
    kept from earlier batches go before the next one takes a smaller layout (the walk's ingest would
    show it) or fails."""
    run(standin, """
        prog = synth.c4(60)
        ctx = ompd.Context(0, 64 << 20)
        first = hip.standin_allocs()
        ctx.analyze_program(prog)
        size = [hip.standin_alloc_size(k) for k in range(first, hip.standin_allocs())]
        assert hip.standin_launches(b"ompd_k_prep") == 0
        small = max(x for x in size if x < max(size[1:]) // 4)   # tables
        hip.standin_budget(size[0] + max(size[1:]) + 4 * small)   # size[0]: the arena
        ctx.analyze_program(prog)
        assert hip.standin_launches(b"ompd_k_prep") == 0
        ctx.close()
        assert hip.standin_live() == 0
    """)


def test_a_plan_that_cannot_be_reconfigured_stays_as_it_was(standin):
    """When an allocation of a reconfiguration fails the plan keeps its configuration and its tables,
    and still runs; a reconfiguration waits for the plan's last run before it changes anything."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        plan = resident(ctx, [synth.c1(0), synth.c3_item(2)])
        plan.run()
        was = plan.describe()
        for change in (lambda: plan.set_schedule([0] * 5), lambda: plan.configure(8192, 2), lambda: plan.split_kernels(False)):
            n = hip.standin_allocs()
            change()
            n = hip.standin_allocs() - n
            plan.set_schedule([-1] * 5)
            plan.split_kernels(True)
            plan.configure(0, 0)
            plan.run()
            for k in range(n):
                hip.standin_fail_alloc(k)
                try:
                    change()
                    assert False, "the allocation did not fail"
                except ompd.OmpdError as e:
                    assert e.code == ompd.OMPD_E_NOMEM, e
                hip.standin_fail_alloc(-1)
                assert plan.describe() == was, (was, plan.describe())
                plan.run()
        hip.standin_clear_events()
        plan.run()
        plan.set_schedule([0] * 5)
        events = hip.standin_events().decode().split()
        assert events[-2:] == ["sync", "memcpy"], events   # the descriptors, which the run reads
    """)


def test_per_tile_kernel_where_the_launch_fills_the_gpu(standin):
    """OMPD_F_TILE_KERNEL and a plan's split_kernels(False): the per-tile kernel runs on the walk,
    which a launch that leaves the GPU idle and a large CFG do not take unless the caller names it."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        small, big = synth.c1(0), chain(13000, 2)
        def kernels(f):
            hip.standin_clear_kernels()
            f()
            return [hip.standin_launches(k) > 0 for k in (b"k_solve", b"k_strip_b", b"k_post_avf")]
        T, W, L = ompd.F_TILE_KERNEL, ompd.F_SCHED_WALK, ompd.F_SCHED_LEVEL
        solve = lambda cfgs, flags: kernels(lambda: ctx.analyze_batch(cfgs, flags=flags, want=("after_dev",)))
        assert solve([small], T) == [False, True, False]
        assert solve([small], T | W) == [True, False, False]
        assert solve([small] * 300, T) == [True, False, False]
        assert solve([small] * 300, T | L) == [False, True, False]
        assert solve([small] * 300 + [big], T) == [False, True, True]   # both schedules: a kernel per phase
        assert solve([small] * 300, 0) == [False, True, False]
        plan = resident(ctx, [small] * 2)
        plan.split_kernels(False)
        assert kernels(plan.run) == [False, True, False]
    """)


def test_a_named_level_schedule_takes_the_shape_of_the_launch(standin):
    """Naming the schedule that a CFG takes anyway changes nothing: the wavefronts of its strips follow
    from the launch's load, whether the flags, the plan's buckets or the rule put it on the strips."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        for cfg, copies in ((synth.c1(0), 2), (synth.c1(0), 1500), (synth.c3_item(5, n_user=700, n_vars=500), 300)):
            plans = [resident(ctx, [cfg] * copies, flags) for flags in (0, 0, ompd.F_SCHED_LEVEL)]
            plans[1].set_schedule([1] * 5)
            shapes = []
            for p in plans:
                d = json.loads(p.describe())
                shapes.append({k: d[k] for k in ("level_tiles", "lds_level", "strip_launches", "level_cfgs")})
            assert shapes[0] == shapes[1] == shapes[2], (copies, shapes)
    """)


def test_autotuner_leaves_alone_what_has_no_effect(standin):
    """The launch configuration is the walk's: a plan of strips keeps the one it was given, and its
    schedules, once they are what the rule would choose, are not replaced by the rule's."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        plan = resident(ctx, [synth.c1(0), synth.c3_item(2)])
        plan.configure(8192, 3)
        plan.autotune()
        d = json.loads(plan.describe())
        assert (d["lds_bytes"], d["wg_per_cu"]) == (8192, 3), d
        walk = resident(ctx, [synth.c1(0)], ompd.F_SCHED_WALK)
        walk.autotune()
        d = json.loads(walk.describe())
        assert d["lds_bytes"] > 0, d
    """)


def test_describe_counts_the_cfgs_of_each_schedule(standin):
    """strip_cfgs is every CFG solved by level, also in a launch that fills the GPU."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        small = synth.c1(0)
        for copies, flags, sched, strips in ((2, 0, -1, 2), (1500, 0, -1, 1500), (2, ompd.F_SCHED_WALK, None, 0),
                                             (3, ompd.F_SCHED_LEVEL, None, 3), (3, 0, 0, 0)):
            plan = resident(ctx, [small] * copies, flags)
            if sched is not None:
                plan.set_schedule([sched] * 5)
            d = json.loads(plan.describe())
            assert d["strip_cfgs"] == strips and (d["tiles"] > 0) == (strips == 0), d
            assert (d["level_tiles"] > 0) == (strips > 0), d
    """)


def test_a_caller_that_names_the_walk_pays_for_the_walk(standin):
    """The strips' larger scratch is not reserved for a plan, an allocation-free call or a request that
    names the walk."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        cfg = synth.c3_item(5, n_user=3000, n_vars=64)
        W = ompd.F_SCHED_WALK
        nb, ne, words = cfg.n_blocks, len(cfg.succ_idx), 1
        # the walk's arrays (three pairs of block rows, a tile's four flag words, 20 words of records; three
        # edge rows and the predecessor lists) and the results not asked for (three pairs and an edge pair)
        most = 8 * (nb * ((6 + 6) * words + 4 + 20) + ne * ((3 + 2) * words + 1)) + 65536
        size = {f: json.loads(resident(ctx, [cfg], f).describe())["scratch_bytes"] for f in (0, W)}
        assert size[W] < most < size[0], (size, most)
        used = {}
        for f in (0, W):
            r = ompd.submit(ctx, cfg, flags=f)
            used[f] = ompd.serving_stats(ctx)["bytes_in_use"]
            r.wait()
        assert used[0] - used[W] > (size[0] - size[W]) // 4, (used, size)
        ctx.close()
    """)


def test_schedule_limits(standin):
    """Which CFGs the strips take: up to 32,000 blocks and 2^24 edges, however many words."""
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        at = on_device(np.zeros(64, np.uint8))   # (never read here)
        for blocks, edges, n_vars, strips in ((2, 1, 0, 1), (32000, 65534, 1, 1), (32000, 65535, 1, 1), (32001, 65534, 1, 0),
                                              (100, 1 << 24, 1, 1), (100, (1 << 24) + 1, 1, 0), (500, 700, 20000, 1)):
            g = ompd.DeviceCFG(n_blocks=blocks, n_edges=edges, n_vars=n_vars, entry=0, exit=blocks - 1, succ_ptr=at,
                               succ_idx=at, edge_kind=at, space=at, read_bits=at, write_bits=at)
            d = json.loads(ompd.Plan(ctx, [g], [ompd.DeviceResult(after_dev=at)]).describe())
            assert d["strip_cfgs"] == strips, (blocks, edges, d)
    """)


def test_plan_without_room_for_its_strips_takes_the_walk(standin):
    run(standin, """
        ctx = ompd.Context(0, 64 << 20)
        cfgs = [synth.c1(0)] * 50
        def walks():
            hip.standin_clear_kernels()
            ctx.analyze_batch(cfgs)
            return hip.standin_launches(b"ompd_k_prep") > 0
        before = hip.standin_allocs()
        assert not walks()
        hip.standin_fail_alloc(1)   # the plan's scratch, after the staging of inputs and outputs
        assert walks()
        hip.standin_fail_alloc(-1)
        assert not walks()
    """)
