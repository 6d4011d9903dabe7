"""cqsa_forward_noalloc under stream capture: recorded calls stay out of the
order of the calls made outside the capture.  Every replay and every other call
is compared bit for bit with the same plan's eager result."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2604_20819_amd as cq
from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _state(i, L=None, H=2, d=64, **opts):
    L = L or 130 + 41 * i
    opts = dict(dict(depth=1, with_backward=True), **opts)
    ins = [x.cuda() for x in synth.make_inputs(70 + i, 1, L, H, d, "bf16", with_dO=True)]
    plan = cq.cqsa_plan(L, H, d, i % 2 == 0, 0, cq.make_opts(**opts))
    out = [torch.empty((1, L, H, d), dtype=torch.float32, device="cuda"),
           torch.empty((1, H, L), dtype=torch.float32, device="cuda")]
    return dict(plan=plan, ins=ins[:3], dO=ins[3], out=out, grads=[torch.empty_like(out[0]) for _ in range(3)])


def _eager(s, entry=cq.cqsa_forward, backward=False):
    for x in s["out"] + s["grads"]:
        x.fill_(float("nan"))
    entry(s["plan"], *s["ins"], *s["out"])
    if backward:
        cq.cqsa_backward(s["plan"], *s["ins"], *s["out"], s["dO"], *s["grads"])
    return s["out"] + (s["grads"] if backward else [])


def _want(s, backward=False):
    got = [x.clone() for x in _eager(s, backward=backward)]
    torch.cuda.synchronize()
    return got


def _same(got, want):
    torch.cuda.synchronize()
    return all(torch.equal(a, b) for a, b in zip(got, want))


def _replays(graph, states, want, between):
    """Three replays, each with eager work of the program between them."""
    for k in range(3):
        for s in states:
            for x in s["out"]:
                x.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        for s, w in zip(states, want):
            assert _same(s["out"], w), k
        between()


def test_calls_after_a_capture():
    """More plans than the image cache holds, through both entry points, after
    an eager and a captured no-allocation call; two streams forked inside the
    capture share the scratch and stay in order."""
    need_gpu()
    say("capture: two streams, then eager calls of 20 plans")
    caught = [_state(0, L=1500), _state(1, L=1100)]
    others = [_state(i) for i in range(20)]
    want_c, want_o = [_want(s) for s in caught], [_want(s, True) for s in others]
    for s, w in zip(caught, want_c):
        assert _same(_eager(s, cq.cqsa_forward_noalloc), w)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=one, capture_error_mode="relaxed"):
        cq.cqsa_forward_noalloc(caught[0]["plan"], *caught[0]["ins"], *caught[0]["out"])
        two.wait_stream(one)
        with torch.cuda.stream(two):
            cq.cqsa_forward_noalloc(caught[1]["plan"], *caught[1]["ins"], *caught[1]["out"])
        one.wait_stream(two)
    torch.cuda.synchronize()

    def eager():
        for k in range(2):
            for i, (s, w) in enumerate(zip(others, want_o)):
                noalloc = (i + k) % 3 == 0
                assert _same(_eager(s, cq.cqsa_forward_noalloc if noalloc else cq.cqsa_forward, not noalloc), w), (k, i)

    eager()
    _replays(graph, caught, want_c, eager)


@pytest.mark.parametrize("opts", [dict(depth=2, read_in_place=False, tasks_per_slot=4),  # staged, several groups
                                  dict(depth=1, tasks_per_slot=2)])                      # read in place, four groups
def test_calls_beside_an_open_capture(opts):
    """A capture of calls that use several streams outside capture stays open
    while 18 other plans (more than the image cache holds) run through every entry
    point on another stream, with the same library streams and events."""
    need_gpu()
    say(f"capture: open beside other calls, {opts}")
    caught = [_state(0, L=1500, **opts), _state(1, L=1100, **opts)]
    others = [_state(2 + i, **(opts if i % 2 else {})) for i in range(18)]
    want_c, want_o = [_want(s) for s in caught], [_want(s, True) for s in others]
    for s, w in zip(caught, want_c):
        assert _same(_eager(s, cq.cqsa_forward_noalloc), w)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    got = []
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=one, capture_error_mode="relaxed"):
        for k, s in enumerate(caught):
            cq.cqsa_forward_noalloc(s["plan"], *s["ins"], *s["out"])
            with torch.cuda.stream(two):
                for o in others[9 * k:9 * k + 9]:
                    _eager(o, cq.cqsa_forward_noalloc)
                    got.append(_eager(o, backward=True))
        two.synchronize()
    torch.cuda.synchronize()
    for i, (g, w) in enumerate(zip(got, want_o)):
        assert _same(g, w), i

    def eager():
        for o, w in zip(others, want_o):
            assert _same(_eager(o, backward=True), w)

    _replays(graph, caught, want_c, eager)


def test_new_plans_beside_a_capture_of_the_global_mode():
    """First calls on another stream upload their images without ending the capture."""
    need_gpu()
    say("capture: new plans beside a global capture")
    caught, first, second = _state(0), _state(1), _state(2)
    want = [_want(s, b) for s, b in ((caught, False), (first, False), (second, True))]
    big = _state(3, L=900)  # the ordinary workspace is large enough
    _eager(big, backward=True)
    _eager(caught, cq.cqsa_forward_noalloc)
    for s in (first, second):  # as new
        L, H, d = s["ins"][0].shape[1:]
        s["plan"] = cq.cqsa_plan(L, H, d, s["plan"].causal, 0, cq.make_opts(depth=1, with_backward=True))
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=one):
        cq.cqsa_forward_noalloc(caught["plan"], *caught["ins"], *caught["out"])
        with torch.cuda.stream(two):
            cq.cqsa_forward_noalloc(first["plan"], *first["ins"], *first["out"])
            cq.cqsa_forward(second["plan"], *second["ins"], *second["out"])
            cq.cqsa_backward(second["plan"], *second["ins"], *second["out"], second["dO"], *second["grads"])
    torch.cuda.synchronize()
    assert _same(first["out"], want[1]) and _same(second["out"] + second["grads"], want[2])
    _replays(graph, [caught], want[:1], lambda: _eager(first, cq.cqsa_forward_noalloc))


FIRST_CALL = """
import torch
import paper_2604_20819_amd as cq
L, H, d = 500, 2, 64
g = torch.Generator(device="cuda").manual_seed(3)
q, k, v = (torch.randn((1, L, H, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
O, LSE = torch.empty((1, L, H, d), device="cuda"), torch.empty((1, H, L), device="cuda")
plan = cq.cqsa_plan(L, H, d, True, 0, cq.make_opts(depth=1))
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):  # mode "global": allocations end such a capture
    cq.cqsa_forward_noalloc(plan, q, k, v, O, LSE)
got = []
for _ in range(3):
    O.fill_(float("nan"))
    LSE.fill_(float("nan"))
    graph.replay()
    got.append((O.clone(), LSE.clone()))
cq.cqsa_forward_noalloc(plan, q, k, v, O, LSE)
torch.cuda.synchronize()
assert all(torch.equal(a, O) and torch.equal(b, LSE) for a, b in got) and not O.isnan().any()
"""


def test_the_first_call_of_a_process_may_be_captured():
    """The device's set-up then runs while a capture is open."""
    need_gpu()
    say("capture: first call of a process")
    r = subprocess.run([sys.executable, "-c", FIRST_CALL], cwd=ROOT, timeout=90, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
