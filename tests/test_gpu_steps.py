"""Scripts whose steps go out in one launch (ps_run, HIP graphs), against a
plain replay of the same calls in numpy with the oracle's arithmetic: device
memory is one array, gradients are read from it and replicas written to it at
their place in the script. Bitwise."""
import random

import numpy as np
import pytest

from oracle import server as orc
from paper_1611_06213_amd import ps
from tests import parity

pytestmark = pytest.mark.gpu

F32, BF16 = ps.PS_F32, ps.PS_BF16


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    ps.load_library()
    return torch


def units(dt):   # 16-bit units of memory per value
    return 2 if dt == F32 else 1


class Replay:
    def __init__(self, n, lr, m, w0, mem):
        self.n, self.lr, self.m = n, lr, m
        self.w = w0.copy()
        self.v = np.zeros_like(self.w) if m else None
        self.mem = mem.copy()
        self.queue = []

    def run(self, ops):
        for op in ops:
            kind = op[0]
            if kind == "push":
                self.queue.append(op[2:])
            if kind in ("apply", "apply_pull"):
                for off, dt in self.queue:
                    g = self.mem[off:off + self.n * units(dt)].copy()
                    g = g.view(np.float32) if dt == F32 else g
                    orc.step(self.w, g, self.lr, self.v, self.m)
                self.queue = []
            if kind == "sync":
                gs = [self.mem[o:o + self.n * units(dt)].copy() for o, dt in self.queue]
                gs = [g.view(np.float32) if dt == F32 else g
                      for g, (_, dt) in zip(gs, self.queue)]
                if gs:
                    orc.ssgd_step(self.w, gs, self.lr, self.v, self.m)
                self.queue = []
            if kind in ("pull", "apply_pull"):
                for off in op[1]:
                    c = orc.pull_copy(self.w, op[2])
                    self.mem[off:off + self.n * units(op[2])] = c.view(np.uint16).ravel()


def script_of(ops, base):
    s = ps.OpScript()
    for op in ops:
        if op[0] == "push":
            s.push(op[1], base + 2 * op[2], op[3])
        elif op[0] == "apply":
            s.apply()
        elif op[0] == "sync":
            s.apply_sync()
        else:
            f = s.pull if op[0] == "pull" else s.apply_pull
            f(list(range(len(op[1]))), [base + 2 * o for o in op[1]], op[2])
    return s.build()


def compare(torch, n, m, ops, size, depth=64, seed=0, fusion=None, graph=False, skip=False,
            fronts=None):
    """Run ops by ps_run (and, with graph, twice more as a HIP graph) on the
    device and in the replay; memory, w and v must be the same bits."""
    rng = np.random.default_rng(seed)
    vals = rng.normal(0, 1e-2, (size + 1) // 2).astype(np.float32)
    mem = vals.view(np.uint16)[:size].copy()
    # every 16-bit unit is also a finite bf16 value
    mem[(mem & 0x7F80) == 0x7F80] = 0x3C00
    w0 = rng.normal(0, 0.05, n).astype(np.float32)
    stream = torch.cuda.Stream()
    dmem = torch.from_numpy(mem.view(np.int16)).cuda()
    dw0 = torch.from_numpy(w0).cuda()
    torch.cuda.synchronize()
    srv = ps.ParameterServer(n, 0.01, m, queue_depth=depth, stream=stream)
    srv.set_pull_skip(skip)
    if fusion is not None:
        srv.set_pull_fusion(fusion)
    if fronts is not None:
        srv.set_fronts(fronts)
    srv.set_weights(dw0)
    script = script_of(ops, dmem.data_ptr())
    ref = Replay(n, 0.01, m, w0, mem)

    def check(what):
        srv.sync()
        torch.cuda.synchronize()
        assert np.array_equal(dmem.cpu().numpy().view(np.uint16), ref.mem), what
        assert parity.bitwise(parity.np_bits(srv.weights_copy()), ref.w), what
        if m:
            assert parity.bitwise(parity.np_bits(srv.velocity_copy()), ref.v), what

    rc, done = ps.ps_run(srv.h, script)
    assert rc == ps.PS_OK and done == len(ops), ps.ps_last_error()
    ref.run(ops)
    check("run")
    if graph:
        g = srv.capture(script)
        for i in range(3):
            g.launch()
            if i == 1:   # the program's own work between replays
                assert ps.ps_run(srv.h, script)[0] == ps.PS_OK
                ref.run(ops)
            ref.run(ops)
            check(f"replay {i}")
        g.close()
    srv.close()


def regular(n, steps, k, r, learners, gdt, pdt, fused, align=8, apply="apply"):
    """steps x (k pushes, an apply, r pulls), buffers `align` 16-bit units apart
    from each other's ends."""
    def room(dt):
        return -(-(n * units(dt)) // align) * align + align
    grads = [i * room(gdt) for i in range(steps * k)]
    at = steps * k * room(gdt)
    reps = [at + i * room(pdt) for i in range(learners)]
    ops = []
    for s in range(steps):
        ops += [("push", j % 5, grads[s * k + j], gdt) for j in range(k)]
        dsts = [reps[(s * r + j) % learners] for j in range(r)]
        if fused:
            ops.append(("apply_pull", dsts, pdt))
        else:
            ops.append((apply,))
            if dsts:
                ops.append(("pull", dsts, pdt))
    return ops, at + learners * room(pdt)


@pytest.mark.parametrize("n", [1, 3, 8, 1025, 20011])
@pytest.mark.parametrize("k,r,learners,steps", [
    (1, 1, 4, 70),     # more steps than one launch takes; replicas repeat
    (1, 1, 64, 9),     # every replica once
    (3, 2, 2, 3), (4, 4, 4, 2),   # the compact argument block and just past it
    (7, 3, 5, 4), (8, 8, 8, 2), (16, 5, 7, 4), (17, 1, 1, 3),
    (32, 32, 32, 2),   # exactly full
    (33, 2, 2, 2), (64, 1, 1, 2),   # a second step never fits
    (2, 33, 33, 3),    # two steps' replicas never fit
    (5, 0, 1, 4),      # applies only
])
def test_steps(torch, n, k, r, learners, steps):
    i = 0
    for gdt, pdt in ((F32, F32), (BF16, BF16), (F32, BF16), (BF16, F32)):
        i += 1
        ops, size = regular(n, steps, k, r, learners, gdt, pdt, fused=i % 2 == 0)
        compare(torch, n, 0.9 if i < 3 else 0.0, ops, size, seed=n + i, graph=i == 2)


@pytest.mark.parametrize("n", [1, 9, 4099])
@pytest.mark.parametrize("k,r,learners,steps", [
    (1, 1, 4, 5), (3, 2, 2, 3), (4, 4, 4, 2), (7, 0, 1, 4), (8, 1, 1, 1), (5, 3, 7, 9),
    (17, 2, 5, 3), (32, 32, 32, 2), (40, 2, 2, 2), (16, 5, 5, 8)])
def test_synchronous_steps(torch, n, k, r, learners, steps):
    """Averaged steps in one launch; a step's gradients lie across load groups."""
    i = 0
    for gdt, pdt in ((F32, F32), (BF16, BF16), (F32, BF16), (BF16, F32)):
        i += 1
        ops, size = regular(n, steps, k, r, learners, gdt, pdt, fused=False, apply="sync")
        compare(torch, n, 0.9 if i % 2 else 0.0, ops, size, seed=n + i, graph=i == 1)
        if i == 1:   # both kinds of step in one script
            mixed = ops + [("apply",) if o[0] == "sync" else o for o in ops] + ops
            compare(torch, n, 0.9, mixed, size, seed=n)


@pytest.mark.parametrize("fronts", [None, 0, 2, 3])
@pytest.mark.parametrize("rule", ["apply", "sync"])
def test_steps_over_many_blocks(torch, rule, fronts):
    """More blocks than the chip holds at once, in every order of the sweep, with
    pulls that are skipped as current."""
    n = 1_300_003   # 1270 blocks of fp32 lanes, 635 of bf16 ones
    for gdt, pdt in ((F32, F32), (BF16, BF16)):
        ops, size = regular(n, 3, 4, 3, 4, gdt, pdt, fused=False, apply=rule)
        ops += [ops[-1], ops[-1]]   # (the learners hold these weights)
        compare(torch, n, 0.9, ops, size, skip=True, fronts=fronts, graph=fronts is None)


def test_steps_that_go_out_one_by_one(torch):
    """Each step writes eight other replicas of 24 MB: none joins another; where
    they write the same ones, all do."""
    n = 6_000_003
    for learners in (24, 8):
        ops, size = regular(n, 3, 8, 8, learners, F32, F32, fused=False)
        compare(torch, n, 0.0, ops, size, skip=True)


@pytest.mark.parametrize("align", [1, 2, 4])
def test_steps_element_aligned(torch, align):
    """Buffers on element boundaries only: fp32 from 4-byte, bf16 from 2- and
    4-byte ones."""
    for gdt, pdt in ((F32, F32), (BF16, BF16), (F32, BF16), (BF16, F32)):
        a = max(align, units(gdt), units(pdt))
        ops, size = regular(4099, 3, 5, 3, 4, gdt, pdt, fused=True, align=a)
        compare(torch, 4099, 0.9, ops, size, seed=align)


@pytest.mark.parametrize("k,r", [(1, 1), (5, 3), (16, 9)])
def test_steps_of_odd_bf16_gradients(torch, k, r):
    """Rows an odd number of bf16 values apart: steps whose gradients all lie
    on 4-byte boundaries join, the others keep the scalar kernels and write
    their replicas from the apply or by the fan-out."""
    for pdt in (F32, BF16):
        ops, size = regular(4098, 4, k, r, 16, BF16, pdt, fused=True, align=1 if pdt == BF16 else 2)
        ops = [(o[0], o[1], o[2] + (pdt == F32 and i % 2), o[3]) if o[0] == "push" else o
               for i, o in enumerate(ops)]
        compare(torch, 4098, 0.9, ops, size, seed=k, graph=True)


@pytest.mark.parametrize("fusion", [0, 1, 64])
def test_steps_with_a_fusion_limit(torch, fusion):
    ops, size = regular(5003, 5, 2, 2, 4, F32, F32, fused=True)
    compare(torch, 5003, 0.9, ops, size, fusion=fusion, graph=True)


@pytest.mark.parametrize("seed", range(12))
def test_random_scripts_over_shared_memory(torch, seed):
    """Pushes, applies, synchronous steps and pulls in random order over a few
    places of one memory that overlap, wholly and in part: a replica pushed as a
    gradient, pulled over a gradient already applied, pulled over another
    replica, both types at one place. (bf16 gradients only where no fp32 replica
    is written, whose low halves could be bf16 NaNs.)"""
    r = random.Random(seed)
    gdts, pdts = ([F32, F32, BF16], [BF16]) if seed % 2 else ([F32], [F32, F32, BF16])
    n = r.choice([5, 257, 4099])
    step = r.choice([2, 8, 2 * n])   # places overlap in part, or each twice its size apart
    places = [2 * i * step for i in range(6)]
    size = places[-1] + 2 * n + 64

    def clash(a, da, b, db):
        return a < b + n * units(db) and b < a + n * units(da)

    ops, pending = [], []
    for _ in range(60):
        kind = r.choice(["push"] * 4 + ["apply", "pull", "pull", "apply_pull", "sync"])
        if kind == "push" and len(pending) < 8:
            p = (r.choice(places), r.choice(gdts))
            pending.append(p)
            ops.append(("push", r.randrange(3), *p))
        elif kind == "apply":
            ops.append(("apply",))
            pending = []
        elif kind == "sync" and len({d for _, d in pending}) <= 1:
            ops.append(("sync",))
            pending = []
        elif kind in ("pull", "apply_pull"):
            dt = r.choice(pdts)
            dsts = []
            for p in r.sample(places, 3):   # a call's own replicas and pending gradients are apart
                if all(not clash(p, dt, q, dt) for q in dsts) and \
                        all(not clash(p, dt, q, d) for q, d in pending):
                    dsts.append(p)
            ops.append((kind, dsts, dt))
            if kind == "apply_pull":
                pending = []
    ops.append(("apply",))
    compare(torch, n, r.choice([0.0, 0.9]), ops, size, depth=8, seed=seed, graph=seed % 3 == 0)


def test_calls_before_a_refused_one_are_done(torch):
    """The queue is full at call 5: the step before it has run, `done` counts
    it, and the script goes on from there."""
    n = 1001
    ops, size = regular(n, 1, 2, 2, 2, F32, F32, fused=True)
    full = ops + [ops[0], ops[1], ops[0]] + ops[2:]
    mem = np.random.default_rng(3).normal(0, 1e-2, size // 2).astype(np.float32)
    dmem = torch.from_numpy(mem).cuda()
    w0 = torch.zeros(n, device="cuda")
    srv = ps.ParameterServer(n, 0.01, 0.9, queue_depth=2)
    srv.set_weights(w0)
    rc, done = ps.ps_run(srv.h, script_of(full, dmem.data_ptr()))
    assert (rc, done) == (ps.PS_EFULL, 5) and "full" in ps.ps_last_error()
    assert (srv.timestamp, srv.pending) == (2, 2)
    ref = Replay(n, 0.01, 0.9, w0.cpu().numpy(), mem.view(np.uint16))
    ref.run(ops)
    srv.sync()
    assert parity.bitwise(parity.np_bits(srv.weights_copy()), ref.w)
    assert np.array_equal(dmem.cpu().numpy().view(np.uint16), ref.mem)
    srv.apply_pending()
    ref.run([ops[0], ops[1], ("apply",)])
    assert parity.bitwise(parity.np_bits(srv.weights_copy()), ref.w)
    srv.close()
