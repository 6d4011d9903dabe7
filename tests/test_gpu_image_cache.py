"""Plan images stay on the device between calls, 16 of them: calls of more
plans than that, in an order that evicts them, on two streams, through every
entry point, and through a plan made at a destroyed one's place, must find
their own image.  Every pass is compared bit for bit with the plan's first."""
import pytest
import torch

import paper_2604_20819_amd as cq
from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu


def _state(i):
    L, H, d, causal, depth = 120 + 37 * i, 1 + i % 2, 64, i % 3 == 0, (1, 0, 2)[i % 3]
    Q, K, V, dO = (x.cuda() for x in synth.make_inputs(40 + i, 1, L, H, d, "bf16", with_dO=True))
    plan = cq.cqsa_plan(L, H, d, causal, 0, cq.make_opts(depth=depth, with_backward=True))
    return dict(plan=plan, ins=(Q, K, V), dO=dO)


def _run(s, entry=cq.cqsa_forward, backward=True):
    Q = s["ins"][0]
    O = torch.empty(Q.shape, dtype=torch.float32, device="cuda")
    LSE = torch.empty((1, Q.shape[2], Q.shape[1]), dtype=torch.float32, device="cuda")
    entry(s["plan"], *s["ins"], O, LSE)
    if not backward:
        return [O, LSE]
    G = [torch.empty_like(O) for _ in range(3)]
    cq.cqsa_backward(s["plan"], *s["ins"], O, LSE, s["dO"], *G)
    return [O, LSE] + G


def test_every_call_finds_its_own_image():
    need_gpu()
    say("image cache: 22 plans, two streams")
    n = 22
    states = [_state(i) for i in range(n)]
    want = [_run(s) for s in states]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for step in (1, 5, 7):  # 1: always the one evicted longest ago
        got = []
        for k in range(2 * n):
            i = (k * step) % n
            with torch.cuda.stream(streams[k % 2]):
                got.append((i, _run(states[i], cq.cqsa_forward_noalloc if k % 3 == 2 else cq.cqsa_forward,
                                    backward=k % 4 != 1)))
        torch.cuda.synchronize()
        for i, g in got:
            assert all(torch.equal(a, b) for a, b in zip(g, want[i])), (step, i)


def test_a_new_plan_does_not_find_an_old_image():
    need_gpu()
    say("image cache: plans made and destroyed")
    for i in (0, 3, 6, 9, 0, 3):
        s = _state(i)
        first = _run(s)
        again = _run(s)
        cq.cqsa_release_workspace()
        after = _run(s)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) and torch.equal(a, c) for a, b, c in zip(first, again, after))
        # the undecomposed call does the same sums up to their order
        Q = s["ins"][0]
        ref = cq.cqsa_plan(Q.shape[1], Q.shape[2], Q.shape[3], s["plan"].causal, 0, cq.make_opts(depth=0))
        O, LSE = _run(dict(plan=ref, ins=s["ins"]), backward=False)
        assert ((O - first[0]).norm() / O.norm()).item() < 1e-3
        del s, ref


@pytest.mark.parametrize("L,depth", [(1, 0), (1, 1), (63, 0), (700, 1), (2111, 2), (6000, 2), (30000, 2)])
def test_images_of_every_size_arrive_whole(L, depth):
    """From one token to more than a slot's 64 KB (L = 30000: 49 tasks with 87 block records of 16 bytes
    each): a first call by each entry point against one in a caller's workspace, which copies its image there."""
    need_gpu()
    say(f"image cache: L={L} depth={depth}")
    Q, K, V = (x.cuda() for x in synth.make_inputs(7 + L, 1, L, 1, 32, "bf16"))
    mk = lambda: dict(plan=cq.cqsa_plan(L, 1, 32, True, 0, cq.make_opts(depth=depth)), ins=(Q, K, V))
    held = {}

    def alloc(n):
        t = torch.empty((n,), dtype=torch.uint8, device="cuda")
        held[t.data_ptr()] = t
        return t.data_ptr()

    cq.cqsa_set_allocator(alloc, lambda p: held.pop(p, None))
    try:
        want = _run(mk(), backward=False)
    finally:
        cq.cqsa_set_allocator(None, None)
    for entry in (cq.cqsa_forward, cq.cqsa_forward_noalloc):
        for s in (mk(), mk(), mk()):  # three uploads in a row, two buffers
            assert all(torch.equal(a, b) for a, b in zip(_run(s, entry, backward=False), want))


def test_new_plans_of_one_kind_do_not_wait_for_calls_of_the_other():
    """A no-allocation call of a new plan, made while ordinary calls of another
    stream run, ends before them: on one of several streams, as streams that
    share a hardware queue run in order whatever they wait for."""
    need_gpu()
    say("image cache: no-allocation calls beside long ordinary ones")
    L, H, d = 32768, 16, 128
    x = torch.randn((1, L, H, d), device="cuda").to(torch.bfloat16)
    O, LSE = torch.empty(x.shape, device="cuda"), torch.empty((1, H, L), device="cuda")
    long = cq.cqsa_plan(L, H, d, False, 0, cq.make_opts(depth=1))
    cq.cqsa_forward(long, x, x, x, O, LSE)
    small = [_state(i) for i in range(9)]
    _run(small[8], cq.cqsa_forward_noalloc, backward=False)
    torch.cuda.synchronize()
    main, streams = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(8)]
    ended_first = 0
    for s, one in zip(small, streams):
        with torch.cuda.stream(main):
            for _ in range(2):  # about 20 ms
                cq.cqsa_forward(long, x, x, x, O, LSE)
            end = main.record_event()
        with torch.cuda.stream(one):
            _run(s, cq.cqsa_forward_noalloc, backward=False)
        one.synchronize()
        ended_first += not end.query()
        torch.cuda.synchronize()
    assert ended_first > 0
