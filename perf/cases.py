"""Timed cases: what a user of the parameter server has it do.

A case is one or more server steps. A step is `depth` pushes (round the
`learners` ids), one apply (asynchronous, or the averaged synchronous one) and
the pull of `pulls` learners into their replicas. The fields of a case:

  n         parameters
  depth     gradients folded per step (K)
  steps     steps of one pass
  learners  learner ids (and replica buffers)
  pulls     replicas refreshed per step
  grad      gradient type, "f32" or "bf16"
  pull      replica type
  momentum  0 or the heavy-ball factor
  rule      "async" (one step per gradient) or "sync" (the average as one)
  fused     True: one apply_pull call; False: apply, then pull_many
  buffers   "rows"   the server's own rows (alloc_rows)
            "torch"  a torch allocation per buffer
            "packed" the rows of one (count, n) torch tensor: for odd n most
                     of them lie on no 16-byte boundary
  via       "calls"  ParameterServer methods, one by one
            "script" a prepared OpScript run by ps_run
            "graph"  the same script captured once and replayed

Sizes are those of the workloads in workloads.py, of the smoke test and of
generic odd lengths. Results are specified to the bit (every product and sum
rounded on its own, oldest gradient first), so the tolerance is "exact".
"""
import torch

from paper_1611_06213_amd import ps, workloads

LR = {"async": 1e-3, "sync": 1e-2}
MAX_BYTES = 25e9   # a drawn case: at most the work and the buffers of the large listed ones
_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
_CODE = {"f32": ps.PS_F32, "bf16": ps.PS_BF16}
_BYTES = {"f32": 4, "bf16": 2}


def _case(name, n, depth, steps, learners, pulls, grad="f32", pull="f32", momentum=0.0,
          rule="async", fused=True, buffers="rows", via="calls"):
    return {"name": name, "n": n, "depth": depth, "steps": steps, "learners": learners,
            "pulls": pulls, "grad": grad, "pull": pull, "momentum": momentum, "rule": rule,
            "fused": fused, "buffers": buffers, "via": via}


def listed():
    c = workloads.CONFIGS
    return [
        # one learner's turn on a small model from Python, on the learners'
        # own tensors: call latency
        _case("tiny_calls", c["tiny"].n, 1, 1, 4, 1, buffers="torch"),
        # a whole schedule of such turns handed to the native executor, with
        # the pull a call of its own
        _case("tiny_script", c["tiny"].n, 1, 200, 4, 1, fused=False, via="script"),
        # one round of the learners replayed as a HIP graph
        _case("tiny_graph", c["tiny"].n, 1, 4, 4, 1, via="graph"),
        # a small model of odd length whose gradients are rows of one tensor
        _case("small_odd", 100_003, 8, 1, 4, 2, momentum=0.9, buffers="packed"),
        # bf16 gradients averaged over the learners, odd length
        _case("sync_bf16_odd", 4_000_037, 8, 1, 8, 8, grad="bf16", pull="bf16", momentum=0.9,
              rule="sync", fused=False, buffers="packed"),
        # Text-CNN: no momentum, the learners of the batch pull; some steps of
        # the schedule per native call
        _case("textcnn_script", c["textcnn"].n, 8, 8, 8, 5, via="script"),
        # one GPU's eighth of VGG-16 (an odd length), gradients packed
        _case("shard_packed", c["vgg16_shard8"].n, 32, 1, 16, 16, momentum=0.9,
              buffers="packed"),
        # AlexNet on the learners' own tensors
        _case("alexnet_torch", c["alexnet"].n, 16, 1, 16, 10, momentum=0.9, buffers="torch"),
        # VGG-16, the framework's flagship step, in the server's slots ...
        _case("vgg16_rows", c["vgg16"].n, 32, 1, 16, 16, momentum=0.9, fused=False),
        # ... and on the learners' own tensors
        _case("vgg16_torch", c["vgg16"].n, 32, 1, 16, 16, momentum=0.9, buffers="torch"),
        # VGG-16 as synchronous SGD over 16 learners
        _case("vgg16_sync", c["vgg16"].n, 16, 1, 16, 16, momentum=0.9, rule="sync", fused=False),
        # the largest vector: bf16 gradients and replicas, 32 learners
        _case("mixed_rows", c["mixed"].n, 32, 1, 32, 32, grad="bf16", pull="bf16", momentum=0.9),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    learners = rng.choice([1, 2, 4, 8, 16, 32])
    grad = rng.choice(["f32", "f32", "bf16"])
    rule = rng.choice(["async", "async", "async", "sync"])
    via = rng.choice(["calls", "calls", "script", "graph"])
    case = {
        "n": 4 * _log_int(rng, 12_500, 50_000_000) + rng.choice([0, 0, 1, 2, 3]),
        "depth": _log_int(rng, 1, 64),
        "steps": 1 if via == "calls" else _log_int(rng, 2, 64),
        "learners": learners,
        "pulls": rng.choice([0, 1, 1, learners, rng.randint(1, learners)]),
        "grad": grad,
        "pull": rng.choice(["f32", grad]),
        "momentum": rng.choice([0.0, 0.9]),
        "rule": rule,
        "fused": rule == "async" and rng.random() < 0.6,
        "buffers": rng.choice(["rows", "torch", "packed"]),
        "via": via,
    }
    # large vectors with few steps, many steps with small vectors
    case["steps"] = max(1, min(case["steps"], 256 // case["depth"]))
    while max(work(case)["bytes"], _resident(case)) > MAX_BYTES:
        case["n"] = case["n"] * 2 // 3
    return case


def _resident(case):
    n = case["n"]
    return n * (case["steps"] * case["depth"] * _BYTES[case["grad"]] + 8
                + case["learners"] * _BYTES[case["pull"]])


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _inputs(case, seed):
    """w0 and the gradients, one after the other (fp32 draws; a bf16 gradient
    is rounded from its draw), scaled as in workloads.py."""
    g = _gen(seed)
    n = case["n"]
    yield (torch.rand(n, generator=g, device="cuda") - 0.5) * 0.1
    for _ in range(case["steps"] * case["depth"]):
        yield torch.empty(n, device="cuda").normal_(0.0, 1e-3, generator=g)


def _buffers(srv, case, count, dtype):
    if case["buffers"] == "rows":
        out = srv.alloc_rows(count, dtype)
        for t in out:
            t.server = srv   # the rows live as long as the server
        return out
    if case["buffers"] == "packed":
        return list(torch.empty((count, case["n"]), dtype=dtype, device="cuda"))
    return [torch.empty(case["n"], dtype=dtype, device="cuda") for _ in range(count)]


def _plan(case):
    """Per step: the pushing learners in order, and the pulling ones."""
    k, l = case["depth"], case["learners"]
    return [([(s * k + j) % l for j in range(k)], [(s * k + j) % l for j in range(case["pulls"])])
            for s in range(case["steps"])]


class _State:
    def __init__(self, case, seed):
        self.case = case
        self.graph = None
        n = case["n"]
        if case["via"] == "graph":   # a graph needs a stream that can be captured
            self.stream = torch.cuda.Stream()
        else:
            self.stream = torch.cuda.current_stream()
        self.srv = srv = ps.ParameterServer(n, LR[case["rule"]], case["momentum"],
                                            queue_depth=case["depth"], stream=self.stream)
        inputs = _inputs(case, seed)
        w0 = next(inputs)
        self.grads = _buffers(srv, case, case["steps"] * case["depth"], _DTYPE[case["grad"]])
        for g, x in zip(self.grads, inputs):
            g.copy_(x)
        self.plan = _plan(case)
        self.replicas = (_buffers(srv, case, case["learners"], _DTYPE[case["pull"]])
                         if case["pulls"] else [])
        self.stream.wait_stream(torch.cuda.current_stream())
        srv.set_weights(w0)
        self.outputs = ps.rows_as_tensors([p for p in (ps.ps_weights(srv.h), ps.ps_velocity(srv.h))
                                           if p], n, torch.float32)
        for t in self.outputs:
            t.server = srv
        pulled = sorted({l for _, pl in self.plan for l in pl})
        self.outputs += [self.replicas[l] for l in pulled]
        if case["via"] != "calls":
            self.script = self._script()
        if case["via"] == "graph":
            self.graph = srv.capture(self.script)

    def _script(self):
        case = self.case
        gd, pd = _CODE[case["grad"]], _CODE[case["pull"]]
        s = ps.OpScript()
        grads = iter(self.grads)
        for pushers, pullers in self.plan:
            for l in pushers:
                s.push(l, next(grads).data_ptr(), gd)
            dsts = [self.replicas[l].data_ptr() for l in pullers]
            if case["fused"]:
                s.apply_pull(pullers, dsts, pd)
                continue
            if case["rule"] == "sync":
                s.apply_sync()
            else:
                s.apply()
            if pullers:
                s.pull(pullers, dsts, pd)
        return s.build()

    def __del__(self):
        if self.graph is not None:
            self.graph.close()


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    case, srv = state.case, state.srv
    if case["via"] == "graph":
        state.graph.launch()
        return state.outputs
    if case["via"] == "script":
        rc, _ = ps.ps_run(srv.h, state.script)
        if rc != ps.PS_OK:
            raise ps.PSError(rc, ps.ps_last_error())
        return state.outputs
    grads = iter(state.grads)
    for pushers, pullers in state.plan:
        for l in pushers:
            srv.push(l, next(grads))
        dsts = [state.replicas[l] for l in pullers]
        if case["fused"]:
            srv.apply_pull(pullers, dsts)
            continue
        if case["rule"] == "sync":
            srv.apply_sync()
        else:
            srv.apply_pending()
        if pullers:
            srv.pull_many(pullers, dsts)
    return state.outputs


def work(case):
    """Every gradient read once, w (and v) read and written once per pass, and
    every pulled replica written at its pull."""
    n, grads = case["n"], case["steps"] * case["depth"]
    mom = case["momentum"] != 0
    state = 16 if mom else 8
    pulled = case["steps"] * case["pulls"]
    return {"bytes": n * (grads * _BYTES[case["grad"]] + state + pulled * _BYTES[case["pull"]]),
            "flops": n * grads * ((4 if mom else 2) if case["rule"] == "async" else 1)}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The pass in 64 bits; a replica holds the weights of its learner's last
    pull."""
    lr, m = (float(torch.tensor(x, dtype=torch.float32)) for x in (LR[case["rule"]],
                                                                   case["momentum"]))
    inputs = _inputs(case, seed)
    w = next(inputs).double()
    v = torch.zeros_like(w)
    bf16 = case["grad"] == "bf16"
    seen = {}

    def step(g):
        if m:
            v.mul_(m).add_(g)
            w.sub_(v, alpha=lr)
        else:
            w.sub_(g, alpha=lr)

    for s, (pushers, pullers) in enumerate(_plan(case)):
        total = torch.zeros_like(w) if case["rule"] == "sync" else None
        for _ in pushers:
            x = next(inputs)
            g = (x.to(torch.bfloat16) if bf16 else x).double()
            if total is None:
                step(g)
            else:
                total.add_(g)
        if total is not None:
            step(total.div_(len(pushers)))
        if pullers:
            # one copy per step that some learner pulled last
            snap = w if s == case["steps"] - 1 else w.clone()
            for l in pullers:
                seen[l] = snap
    return [w] + ([v] if m else []) + [seen[l] for l in sorted(seen)]
