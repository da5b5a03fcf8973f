"""The calls that go through csrc/fastcall.cpp against the ctypes path (taken when a stream is passed): the same results, the
same refusals, the current stream.  Bytes and whole numbers: no tolerance."""
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu
N, k, E, D, H = 37, 4, 16, 4, 64


@pytest.fixture(scope="module")
def f():
    import paper_2512_22036_amd as f
    from paper_2512_22036_amd import binding
    f.load_library()
    assert binding._fast is not None
    return f


def tensors(f):
    import numpy as np
    A = torch.from_numpy(random_topk(np.random.default_rng(1), N, k, E)).cuda()
    g = torch.Generator(device="cuda").manual_seed(5)
    rows = lambda n, h, t=torch.bfloat16: torch.randn((n, h), generator=g, device="cuda").to(t)
    cap = N * min(k, D)
    return dict(A=A, x=rows(N, H), y=rows(N * k, H), w=torch.rand((N, k), generator=g, device="cuda"), xa=rows(N, 8, torch.float32),
                eb=torch.zeros((N * k, H), dtype=torch.bfloat16, device="cuda"), ea=torch.zeros((N * k, 8), device="cuda"),
                sb=torch.zeros((cap, H), dtype=torch.bfloat16, device="cuda"), sa=torch.zeros((cap, 8), device="cuda"),
                part=torch.zeros((cap, H), device="cuda"), out=torch.zeros((N, H), device="cuda"))


CALLS = {
    "plan": lambda f, L, t, **s: f.fusco_plan(L, t["A"], **s),
    "dispatch": lambda f, L, t, **s: f.fusco_dispatch(L, t["x"], t["eb"], **s),
    "dispatch planes": lambda f, L, t, **s: f.fusco_dispatch(L, t["x"], t["eb"], x_aux=t["xa"], expert_aux=t["ea"], **s),
    "dispatch wire": lambda f, L, t, **s: f.fusco_dispatch(L, t["x"], send_buf=t["sb"], flags=2, **s),
    "dispatch all": lambda f, L, t, **s: f.fusco_dispatch(L, t["x"], t["eb"], t["xa"], t["ea"], t["sb"], t["sa"], flags=3, **s),
    "dispatch two hop": lambda f, L, t, **s: f.fusco_dispatch(L, t["x"], t["eb"], send_buf=t["sb"], flags=4, **s),
    "dispatch unasked": lambda f, L, t, **s: f.fusco_dispatch(L, t["x"], t["eb"], send_buf=t["sb"], **s),
    "plan dispatch": lambda f, L, t, **s: f.fusco_plan_dispatch(L, t["A"], t["x"], t["eb"], **s),
    "plan dispatch planes": lambda f, L, t, **s: f.fusco_plan_dispatch(L, t["A"], t["x"], t["eb"], x_aux=t["xa"], expert_aux=t["ea"], **s),
    "combine": lambda f, L, t, **s: f.fusco_combine(L, t["y"], t["w"], t["out"], **s),
    "two hop": lambda f, L, t, **s: f.fusco_combine_two_hop(L, t["y"], t["w"], t["part"], t["out"], **s),
}


# the calls that csrc/fastcall.cpp makes itself; it leaves the others to ctypes
PLAIN = sorted(set(CALLS) - {"dispatch unasked"})


class Recorder:
    """Stands in for the module and notes what each of its calls returned: None where the call is left to ctypes."""

    def __init__(self, module):
        self.module, self.seen = module, []

    def __getattr__(self, name):
        def call(*args):
            rc = getattr(self.module, name)(*args)
            self.seen.append((name, rc))
            return rc
        return call


@pytest.fixture
def route(f, monkeypatch):
    from paper_2512_22036_amd import binding
    recorder = Recorder(binding._fast)
    monkeypatch.setattr(binding, "_fast", recorder)
    return recorder.seen


def run(f, name, t, **s):
    L = f.Layout(N, k, E, D)
    L.mem.zero_()
    if name != "plan" and not name.startswith("plan "):
        f.fusco_plan(L, t["A"], **s)
    CALLS[name](f, L, t, **s)
    return L.mem


@pytest.mark.parametrize("name", sorted(CALLS))
def test_same_as_ctypes(f, name, route):
    a, b = tensors(f), tensors(f)
    here = torch.cuda.current_stream()
    got = run(f, name, a)
    assert [rc for _, rc in route][-1] == (0 if name in PLAIN else None) and all(rc == 0 for _, rc in route[:-1]), route
    route.clear()
    assert torch.equal(got, run(f, name, b, stream=here))
    assert not route, "a call with a stream goes through ctypes"
    for key in a:
        assert torch.equal(a[key], b[key]), key
    # other kinds of tensor are accepted as they were
    c = {key: torch.nn.Parameter(v, requires_grad=False) for key, v in tensors(f).items()}
    run(f, name, c)
    for key in b:
        assert torch.equal(c[key].data, b[key]), key


def test_current_stream(f, route):
    """The calls go to the stream that is current: captured into a graph there, they do nothing before the graph runs."""
    t, want = tensors(f), tensors(f)
    for name in ("plan dispatch", "combine"):
        run(f, name, want)
    L = f.Layout(N, k, E, D)
    L.mem.zero_()
    calls = lambda: (f.fusco_plan_dispatch(L, t["A"], t["x"], t["eb"]), f.fusco_combine(L, t["y"], t["w"], t["out"]))
    torch.cuda.synchronize()
    route.clear()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        calls()
    assert [rc for _, rc in route] == [0, 0]
    torch.cuda.synchronize()
    assert not bool(t["out"].any()) and not bool(t["eb"].any()) and not bool(L.mem.any())
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(t["out"], want["out"]) and torch.equal(t["eb"], want["eb"])
        for key in ("out", "eb"):
            t[key].zero_()
        L.mem.zero_()
        calls()                                        # the same calls between the replays, on the default stream
        torch.cuda.synchronize()
        assert torch.equal(t["out"], want["out"]) and torch.equal(t["eb"], want["eb"])
        for key in ("out", "eb"):
            t[key].zero_()


BROKEN = [("A", lambda v: v.long()), ("A", lambda v: v[:-1]), ("A", lambda v: v.t().contiguous().t()), ("A", lambda v: v.cpu()),
          ("x", lambda v: v[:-1].contiguous()), ("x", lambda v: v[:, ::2]), ("x", lambda v: v.view(-1)), ("x", lambda v: v.cpu()),
          ("xa", lambda v: v[:-1]), ("ea", lambda v: v[:, :4].contiguous()), ("ea", lambda v: None), ("eb", lambda v: v[:-1]),
          ("eb", lambda v: v[:, :32].contiguous()), ("sb", lambda v: v[:-1]), ("sa", lambda v: v[:-1]), ("y", lambda v: v[:-1]),
          ("y", lambda v: v.half()), ("y", lambda v: v[:, :32].contiguous()), ("w", lambda v: v.double()), ("w", lambda v: v[:, :2].contiguous()),
          ("out", lambda v: v[:-1]), ("out", lambda v: v.half()), ("out", lambda v: v[:, :32].contiguous()), ("part", lambda v: v[:-1]),
          ("part", lambda v: v.bfloat16()), ("part", lambda v: v.int())]


@pytest.mark.parametrize("name", sorted(CALLS))
def test_same_refusals(f, name, route):
    L = f.Layout(N, k, E, D)
    t = tensors(f)
    f.fusco_plan(L, t["A"])
    refused = 0
    for key, change in BROKEN:
        b = dict(t)
        b[key] = change(t[key])
        said = []
        route.clear()
        for s in (dict(), dict(stream=torch.cuda.current_stream())):
            try:
                CALLS[name](f, L, b, **s)
                said.append(None)
            except (f.FuscoError, TypeError, AttributeError) as e:
                said.append((type(e), str(e)))
        assert said[0] == said[1], (key, said)
        assert len(route) == 1, route
        if said[0] is not None:
            assert route[0][1] != 0, (key, route)
        refused += said[0] is not None
    assert refused >= 4
