"""The server's host code on the CPU (tests/host_server.py): how the calls of a
script go out, what a failed launch leaves behind, and that joined and single
calls do the same."""
import random

import numpy as np
import pytest

from paper_1611_06213_amd import ps
from tests import host_server as hs

F32, BF16 = ps.PS_F32, ps.PS_BF16
HEADLINE, LARGE = 138_357_544, 200_000_000   # parameters of VGG-16 and of the bf16 workload


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    return hs.build(str(tmp_path_factory.mktemp("host") / "libhost.so"))


@pytest.fixture
def lib(built, monkeypatch):
    monkeypatch.setattr(ps, "_lib", built)
    return built


class Memory:
    """`places` buffers of n values, each of room for fp32, in one array of
    2-byte units with finite values of either type."""

    def __init__(self, n, places, seed=0):
        self.step = 2 * n + 6
        vals = np.random.default_rng(seed).normal(0, 1e-2, places * self.step // 2 + 1)
        self.a = vals.astype(np.float32).view(np.uint16).copy()
        self.a[(self.a & 0x7F80) == 0x7F80] = 0x3C00
        self.base = self.a.ctypes.data

    def __getitem__(self, i):
        return i * self.step


def one_by_one(srv, ops, base):
    """The script's calls, each by itself: (status, calls made)."""
    for i, op in enumerate(ops):
        rc, _ = ps.ps_run(srv.h, hs.script([op], base))
        if rc != ps.PS_OK:
            return rc, i
    return ps.PS_OK, len(ops)


@pytest.mark.parametrize("seed", range(40))
def test_joined_calls_equal_single_ones(lib, seed):
    """Random scripts over buffers of one memory, refused calls among them: the
    same weights, memory, state, status and number of calls."""
    r = random.Random(seed)
    n, m = r.choice([1, 5, 33]), r.choice([0.0, 0.9])
    mode, skip = r.choice([ps.PS_QUEUE_FIFO, ps.PS_QUEUE_ROUND_ROBIN]), r.random() < 0.5
    depth = r.choice([4, 16])
    gdts = r.choice([[F32], [BF16], [F32, F32, BF16]])
    pdts = r.choice([[F32], [BF16], [F32, BF16]])
    mems = [Memory(n, 14, seed), Memory(n, 14, seed)]
    ops = []
    for _ in range(120):
        kind = r.choice(["push"] * 5 + ["apply", "apply", "sync", "pull", "pull", "apply_pull"])
        if kind == "push":   # (an odd place of bf16 gradients lies on no 4-byte boundary)
            dt = r.choice(gdts)
            ops.append((kind, r.randrange(3), mems[0][r.randrange(8)] + (r.random() < 0.1 and dt == BF16), dt))
        elif kind in ("apply", "sync"):
            ops.append((kind,))
        else:
            ops.append((kind, r.sample([mems[0][8 + i] for i in range(6)], r.randrange(4)), r.choice(pdts)))
    got = []
    for mem, run in zip(mems, (None, one_by_one)):
        srv = hs.Host(lib, n, momentum=m, depth=depth, skip=skip)
        if mode:
            assert ps.ps_set_queue_mode(srv.h, mode, 3) == 0
        at, log = 0, []
        while at < len(ops):   # a refused call is left out, the rest goes on
            rc, done = (run(srv, ops[at:], mem.base) if run
                        else ps.ps_run(srv.h, hs.script(ops[at:], mem.base)))
            log.append((rc, done))
            at += done + 1
        v = srv.v()
        got.append((log, srv.state(), srv.w().tobytes(), b"" if v is None else v.tobytes(), mem.a.tobytes()))
        srv.close()
    assert got[0] == got[1]


def pushes(mem, count, dt=F32, at=0):
    return [("push", j % 3, mem[at + j], dt) for j in range(count)]


def test_a_plan_does_not_depend_on_earlier_replicas(lib):
    """Joined synchronous steps without replicas are the same launch whatever
    type of replica was pulled before."""
    mem = Memory(9, 8)
    sync = pushes(mem, 1) + [("sync",)] + pushes(mem, 1, at=1) + [("sync",)]
    pull16 = pushes(mem, 1) + [("apply_pull", [mem[6]], BF16)]
    srv = hs.Host(lib, 9)
    for ops in (sync, sync + pull16):
        s = hs.script(ops, mem.base)
        rc, g = ps.ps_graph_create(srv.h, s)
        assert rc == 0
        for _ in range(2):
            assert ps.ps_graph_launch(srv.h, g) == 0, ps.ps_last_error()
            assert ps.ps_run(srv.h, hs.script(pull16, mem.base))[0] == 0
        ps.ps_graph_destroy(g)
    srv.close()


@pytest.mark.parametrize("fail,done", [(0, 1), (1, 129), (2, 257)])
def test_done_names_the_calls_before_a_failed_launch(lib, fail, done):
    """300 calls go out in launches of 64 gradients: `done` counts the calls
    before those of the launch that failed, not those of the first one."""
    mem = Memory(3, 1)
    srv = hs.Host(lib, 3)
    srv.clear(fail)
    assert ps.ps_run(srv.h, hs.script([*pushes(mem, 1), ("apply",)] * 150, mem.base)) == (ps.PS_EHIP, done)
    assert [(l.kind, l.k) for l in srv.launches()] == [(hs.APPLY, 64)] * fail
    srv.close()


def fail_script(mem):
    """Steps of either kind, replicas of two types, gradients of two: several
    joined launches and single ones."""
    ops = []
    for s in range(3):
        ops += pushes(mem, 2) + [("apply_pull", [mem[8], mem[9]], F32)]
        ops += pushes(mem, 1) + [("apply",), ("pull", [mem[8]], F32), ("pull", [mem[10]], BF16)]
        ops += pushes(mem, 3) + [("sync",)] + pushes(mem, 2, at=2) + [("sync",), ("pull", [mem[11]], F32)]
        ops += pushes(mem, 2, BF16, at=5) + [("apply",)] + pushes(mem, 1, at=3)   # one stays queued
    return ops


@pytest.mark.parametrize("mode", [ps.PS_QUEUE_FIFO, ps.PS_QUEUE_ROUND_ROBIN])
@pytest.mark.parametrize("skip", [True, False])
def test_after_a_failed_launch_only_the_calls_before_it_are_made(lib, mode, skip):
    """Whichever launch of a script fails: `done` calls are made, the server
    says and holds what those calls alone leave, and the script goes on from there
    to the same end."""
    def server(mem):
        srv = hs.Host(lib, 9, momentum=0.9, depth=8, skip=skip)
        if mode:
            assert ps.ps_set_queue_mode(srv.h, mode, 8) == 0
        return srv

    def all_of(srv, mem):
        return srv.state(), srv.w().tobytes(), srv.v().tobytes(), mem.a.tobytes()

    whole = Memory(9, 14)
    ops = fail_script(whole)
    srv = server(whole)
    srv.clear()
    assert ps.ps_run(srv.h, hs.script(ops, whole.base)) == (ps.PS_OK, len(ops))
    launches, end = len(srv.launches()), all_of(srv, whole)
    srv.close()
    assert launches > 8
    for fail in range(launches):
        mem, ref = Memory(9, 14), Memory(9, 14)
        a = server(mem)
        a.clear(fail)
        rc, done = ps.ps_run(a.h, hs.script(ops, mem.base))
        assert rc == ps.PS_EHIP and done < len(ops)
        got = all_of(a, mem)
        b = server(ref)
        assert one_by_one(b, ops[:done], ref.base) == (ps.PS_OK, done)
        assert got == all_of(b, ref), (fail, done)
        b.close()
        assert ps.ps_run(a.h, hs.script(ops[done:], mem.base)) == (ps.PS_OK, len(ops) - done)
        assert all_of(a, mem) == end, (fail, done)
        a.close()


@pytest.mark.parametrize("mode", [ps.PS_QUEUE_FIFO, ps.PS_QUEUE_ROUND_ROBIN])
def test_without_memory_no_gradient_is_lost_or_applied_twice(lib, mode):
    """Whichever allocation of a script throws: PS_ENOMEM, the gradients of the
    `done` calls are applied once each, and the rest of the script ends as it
    would have."""
    fail = 0
    while True:
        mem, ref = Memory(9, 14), Memory(9, 14)
        ops = fail_script(mem)
        a, b = (hs.Host(lib, 9, momentum=0.9, depth=8, skip=False) for _ in range(2))
        if mode:
            for s in (a, b):
                assert ps.ps_set_queue_mode(s.h, mode, 8) == 0
        s = hs.script(ops, mem.base)
        lib.host_fail_alloc(fail)
        rc, done = ps.ps_run(a.h, s)
        if lib.host_fail_alloc(-1) >= 0:   # there are no more
            assert rc == ps.PS_OK and fail > 50
            break
        assert (rc == ps.PS_ENOMEM and done < len(ops)) or (rc, done) == (ps.PS_OK, len(ops))
        assert one_by_one(b, ops[:done], ref.base) == (ps.PS_OK, done)
        assert a.w().tobytes() == b.w().tobytes() and a.v().tobytes() == b.v().tobytes(), fail
        assert ps.ps_timestamp(a.h) == ps.ps_timestamp(b.h), fail
        assert ps.ps_pending(a.h) == ps.ps_pending(b.h), fail
        assert ps.ps_run(a.h, hs.script(ops[done:], mem.base)) == (ps.PS_OK, len(ops) - done)
        assert one_by_one(b, ops[done:], ref.base) == (ps.PS_OK, len(ops) - done)
        assert a.w().tobytes() == b.w().tobytes() and mem.a.tobytes() == ref.a.tobytes(), fail
        a.close()
        b.close()
        fail += 1


@pytest.mark.parametrize("fail", range(4))
def test_a_replay_that_fails_half_way_counts_what_it_enqueued(lib, fail):
    """A replay of four kernels launched one by one, of which the fail-th fails:
    the server says and holds what the calls before that kernel leave, as ps_run
    of the script does when that launch fails (before the first one: nothing)."""
    got = []
    for graph in (False, True):
        mem = Memory(9, 14)
        ops = (pushes(mem, 2) + [("apply",), ("pull", [mem[8]], F32)] + pushes(mem, 2, BF16, at=4) +
               [("apply_pull", [mem[9], mem[10]], F32), ("pull", [mem[11]], BF16)] +
               pushes(mem, 1) + [("sync",)])
        srv = hs.Host(lib, 9, momentum=0.9)
        s = hs.script(ops, mem.base)
        if graph:
            rc, g = ps.ps_graph_create(srv.h, s)
            assert rc == 0 and len(srv.launches()) == 4
        srv.clear(fail)
        before = srv.state()
        assert (ps.ps_graph_launch(srv.h, g) if graph else ps.ps_run(srv.h, s)[0]) == ps.PS_EHIP
        assert len(srv.launches()) == fail
        got.append((srv.state(), srv.w().tobytes(), srv.v().tobytes(), mem.a.tobytes()))
        if fail == 0:   # (ps_run has made the pushes)
            got[-1] = (before if not graph else srv.state(), *got[-1][1:])
        if graph:
            ps.ps_graph_destroy(g)
        srv.close()
    assert got[0] == got[1]


def kinds(srv):
    return [l.kind for l in srv.launches()]


def test_looking_ahead_stops_at_any_count(lib):
    """Later pulls of absurd counts (refused when the script gets there) do not
    wrap round to few replicas: the step before them goes out by itself."""
    n = 10_000_000
    mem = Memory(4, 20)   # (nothing runs: only the places count)
    mem.step = 2 * n + 6
    ops = pushes(mem, 8) + [("apply",), ("pull", [mem[i] for i in range(8, 16)], F32)] + pushes(mem, 8)
    srv = hs.Host(lib, n, run=False)
    s = hs.script(ops, mem.base)
    for _ in range(2):
        s.pull([0], [mem.base], F32)
    s.apply()
    s.build()
    for i in (-2, -3):
        s.array[i].count = 2**31 - 1
    rc, done = ps.ps_run(srv.h, s)
    assert (rc, done) == (ps.PS_EINVAL, len(ops)) and kinds(srv) == [hs.APPLY, hs.PULL]
    srv.close()


def test_a_step_joins_no_empty_one(lib):
    """An apply with nothing queued is no step: the replicas before it are
    written as by a step alone (the fan-out here), unless gradients are left
    in the queues for it."""
    n = 10_000_000
    mem = Memory(4, 40)
    mem.step = 2 * n + 6
    step = [("apply",), ("pull", [mem[i] for i in range(16, 24)], F32)]
    srv = hs.Host(lib, n, run=False, skip=False)
    assert ps.ps_run(srv.h, hs.script(pushes(mem, 16) + step * 2, mem.base))[0] == 0
    assert kinds(srv) == [hs.APPLY, hs.PULL, hs.PULL]
    srv.clear()
    lib.host_reset(0)
    assert ps.ps_run(srv.h, hs.script((pushes(mem, 16) + step) * 2, mem.base))[0] == 0
    assert kinds(srv) == [hs.STEPS]
    srv.close()
    srv = hs.Host(lib, n, run=False, skip=False, depth=16)
    assert ps.ps_set_queue_mode(srv.h, ps.PS_QUEUE_ROUND_ROBIN, 16) == 0
    assert ps.ps_run(srv.h, hs.script(pushes(mem, 16) * 2 + step * 2, mem.base))[0] == 0
    assert kinds(srv) == [hs.STEPS]
    srv.close()


def test_settings_reach_the_steps_of_a_script(lib):
    """ps_set_fronts and the residency of ps_set_launch_shape hold for a joined
    launch too; a gradient group asked for leaves every step its own launch,
    whose loads it arranges."""
    n = 1_000_000
    mem = Memory(4, 16)
    mem.step = 2 * n + 6
    ops = []
    for s in range(2):
        ops += pushes(mem, 4, at=4 * s) + [("apply",), ("pull", [mem[8], mem[9]], F32)]
    for sync in (False, True):
        if sync:
            ops = [("sync",) if o == ("apply",) else o for o in ops]
        s = hs.script(ops, mem.base)
        srv = hs.Host(lib, n, momentum=0.9, run=False, skip=False)
        for f in (0, 3, -1):
            assert ps.ps_set_fronts(srv.h, f) == 0 and ps.ps_run(srv.h, s)[0] == 0
        for b in (0, 4, -1):
            assert ps.ps_set_launch_shape(srv.h, b, 0) == 0 and ps.ps_run(srv.h, s)[0] == 0
        steps = srv.launches()
        assert [l.kind for l in steps] == [hs.SYNC_STEPS if sync else hs.STEPS] * 6
        assert [l.fronts for l in steps] == [0, 3, 0, 0, 0, 0]
        assert [l.blocks for l in steps] == [steps[0].blocks] * 3 + [0, 4, steps[0].blocks]
        lib.host_reset(0)
        assert ps.ps_set_launch_shape(srv.h, -1, 12) == 0 and ps.ps_run(srv.h, s)[0] == 0
        first = [l for l in srv.launches() if l.kind != hs.PULL]
        assert [(l.kind, l.k, l.group) for l in first] == [(hs.SYNC if sync else hs.APPLY, 4, 12)] * 2
        srv.close()


@pytest.mark.parametrize("n,k,r,dt", [(HEADLINE, 16, 16, F32), (LARGE, 32, 32, BF16), (10_000_000, 16, 16, F32)])
@pytest.mark.parametrize("rule", ["apply", "sync", "fused"])
def test_steps_with_many_replicas_join_if_they_are_written_again(lib, n, k, r, dt, rule):
    """Steps that write the same replicas share launches; steps that write 16
    fp32 or 32 bf16 others each go out by themselves (measured slower joined),
    whatever call the replicas are pulled by."""
    steps = 128 // k
    mem = Memory(4, 64 + 64)
    mem.step = 2 * n + 6
    for other in (False, True):
        ops = []
        for s in range(steps):
            dsts = [mem[64 + (s * r * other + j) % 64] for j in range(r)]
            ops += pushes(mem, k, dt) + ([("apply_pull", dsts, dt)] if rule == "fused" else
                                         [(rule,), ("pull", dsts, dt)])
        srv = hs.Host(lib, n, momentum=0.9, run=False, skip=False)
        assert ps.ps_run(srv.h, hs.script(ops, mem.base))[0] == 0
        one = [hs.SYNC if rule == "sync" else hs.APPLY, hs.PULL]
        joined = hs.SYNC_STEPS if rule == "sync" else hs.STEPS
        assert kinds(srv) == (one * steps if other else [joined] * (steps * k // 64))
        srv.close()


def test_replicas_in_rotation_join(lib):
    """Two sets of replicas in turn: half of what the launch writes is written
    again in it."""
    mem = Memory(4, 100)
    mem.step = 2 * HEADLINE + 6
    ops = []
    for s in range(4):
        ops += pushes(mem, 16) + [("apply",), ("pull", [mem[64 + 16 * (s % 2) + j] for j in range(16)], F32)]
    srv = hs.Host(lib, HEADLINE, momentum=0.9, run=False, skip=False)
    assert ps.ps_run(srv.h, hs.script(ops, mem.base))[0] == 0
    assert [(l.kind, l.k, l.r) for l in srv.launches()] == [(hs.STEPS, 64, 64)]
    srv.close()


@pytest.mark.parametrize("m,pdt,fused", [(0.0, F32, False), (0.9, F32, True), (0.0, BF16, True)])
def test_a_script_writes_replicas_as_the_calls_do(lib, m, pdt, fused):
    """Four replicas of a single step of 8 bf16 gradients: from the apply, but
    not fp32 ones without momentum, as measured; by apply_pull and, in a script,
    by apply and pull."""
    mem = Memory(4, 16)
    mem.step = 2 * HEADLINE + 6
    dsts = [mem[8 + i] for i in range(4)]
    srv = hs.Host(lib, HEADLINE, momentum=m, run=False, skip=False)
    for ops in ([("apply_pull", dsts, pdt)], [("apply",), ("pull", dsts, pdt)]):
        lib.host_reset(0)
        assert ps.ps_run(srv.h, hs.script(pushes(mem, 8, BF16) + ops, mem.base))[0] == 0
        assert kinds(srv) == ([hs.APPLY] if fused else [hs.APPLY, hs.PULL])
    srv.close()


@pytest.mark.parametrize("error", [RuntimeError("not built"), ImportError("undefined symbol")])
def test_without_the_native_binding_the_python_route_serves(lib, monkeypatch, error):
    """ParameterServer needs the library alone; it says that its calls are
    slower."""
    torch = pytest.importorskip("torch")

    class Device:   # what the binding asks of a device tensor, over host memory
        is_cuda = True
        dtype = torch.float32

        def __init__(self, values):
            self.a = np.array(values, np.float32)
            self.numel, self.data_ptr = lambda: self.a.size, lambda: self.a.ctypes.data
            self.is_contiguous = lambda: True

    def missing():
        raise error
    lib.host_reset(1)
    with monkeypatch.context() as m, pytest.warns(RuntimeWarning, match=str(error)):
        m.setattr(ps, "load_binding", missing)
        srv = ps.ParameterServer(3, 0.5, queue_depth=2)
    g, d, e = Device([1, 2, 3]), Device([0] * 3), Device([0] * 3)
    assert srv.push(0, g) and srv.push(1, g) and not srv.push(2, g)
    srv.apply_pull([0], [d])
    srv.pull_many([1], [e])
    assert d.a.tolist() == e.a.tolist() == [-1, -2, -3] and srv.timestamp == 2 and not srv._pending
    srv.close()
