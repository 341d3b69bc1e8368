"""ParameterServer's per-step calls take their native route for plain device
tensors and the Python one for everything else; both do and refuse the same."""
import numpy as np
import pytest

from paper_1611_06213_amd import ps

pytestmark = pytest.mark.gpu

N = 1003


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    ps.load_library()
    return torch


def server(torch, depth=8, stream=True):
    srv = ps.ParameterServer(N, 0.5, 0.0, queue_depth=depth,
                             stream=torch.cuda.current_stream() if stream else None)
    srv.set_weights(torch.zeros(N, device="cuda"))
    return srv


def native_only(srv, monkeypatch):
    """Fail if a call leaves the native route."""
    def no(*a):
        raise AssertionError("not the native route")
    monkeypatch.setattr(srv, "_tensor", no)


@pytest.mark.parametrize("stream", [True, False])
@pytest.mark.parametrize("gdt", ["float32", "bfloat16"])
def test_native_route(torch, monkeypatch, gdt, stream):
    dt = getattr(torch, gdt)
    srv = server(torch, stream=stream)
    base = torch.ones(2 * N + 8, dtype=dt, device="cuda")
    grads = [base[:N], base[N + 1:2 * N + 1], torch.nn.Parameter(torch.ones(N, dtype=dt, device="cuda")),
             torch.ones(17, 59, dtype=dt, device="cuda")]
    assert N == 17 * 59
    d = torch.empty(3, N, dtype=dt, device="cuda")
    with monkeypatch.context() as m:
        native_only(srv, m)
        for l, g in enumerate(grads):
            assert srv.push(l, g)
        assert sum(map(len, srv._pending.values())) == 4
        srv.apply_pull(range(2), [d[0], d[1]])
        assert not srv._pending
        srv.pull_many((2,), (d[2],))
        srv.apply_pull([], [])
    assert srv.timestamp == 4 and srv.last_applied() == [] and srv.stats().pulls == 3
    assert bool((d == -2.0).all()) and bool((srv.weights_copy() == -2.0).all())
    srv.close()


def test_python_route_and_refusals(torch):
    class Sub(torch.Tensor):
        pass

    srv = server(torch, depth=2)
    ok = torch.ones(N, device="cuda")
    dst = torch.empty(N, device="cuda")
    for bad in (torch.ones(N), torch.ones(N + 1, device="cuda"),
                torch.ones(2 * N, device="cuda")[::2],
                torch.sparse_coo_tensor(torch.zeros(1, 1), torch.ones(1), (N,), device="cuda")):
        with pytest.raises((ValueError, RuntimeError)):
            srv.push(0, bad)
        with pytest.raises((ValueError, RuntimeError)):
            srv.pull_many([0], [bad])
    for bad in (ok.half(), ok.int()):
        with pytest.raises(TypeError):
            srv.push(0, bad)
        with pytest.raises(TypeError):
            srv.apply_pull([0], [bad])
    with pytest.raises(ValueError):
        srv.pull_many([0, 1], [dst])
    with pytest.raises(ValueError):
        srv.pull_many([0, 1], [dst, dst.bfloat16()])
    with pytest.raises(ps.PSError):
        srv.pull_many([0, 1], [dst, dst])                 # one buffer twice
    with pytest.raises(ps.PSError):
        srv.pull_many(list(range(65)), [dst] * 65)
    with pytest.raises(ps.PSError):
        srv.push(-1, ok)
    with pytest.raises(Exception):
        srv.push("0", ok)
    assert srv.pending == 0 and not srv._pending and srv.stats().pulls == 0
    assert srv.push(0, ok.as_subclass(Sub)) and srv.push(1, ok)
    assert not srv.push(2, ok)                            # full
    assert [len(q) for q in srv._pending.values()] == [1, 1]
    srv.apply_pull([np.int32(0)][:0], [])
    assert srv.timestamp == 2 and not srv._pending
    srv.pull_many([1], [dst.as_subclass(Sub)])
    assert bool((dst == -1.0).all())
    srv.close()
    with pytest.raises(ps.PSError):
        srv.push(0, ok)


def test_under_vmap_nothing_is_pushed(torch):
    srv = server(torch)
    with pytest.raises(Exception):
        torch.vmap(lambda g: srv.push(0, g) or g)(torch.ones(2, N, device="cuda"))
    assert srv.pending == 0
    srv.close()
