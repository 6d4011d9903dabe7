"""Forward and gradients of deep plans, whose merges search more segments than a
wave has lanes, against the float64 oracle with the other tests' bounds."""
import pytest

from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, say
from tests.test_gpu_backward import _check_grads, oracle_grads, run_fwd_bwd
from tests.test_gpu_forward import _check_vs_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,depth,causal", [(900, 3, False), (1003, 4, True)])
def test_merges_of_many_segments(L, depth, causal):
    need_gpu()
    H, d, dt = 2, 64, "bf16"
    Q, K, V, dO = synth.make_inputs(800 + L, 1, L, H, d, dt, with_dO=True)
    say(f"deep plan L={L} depth={depth} causal={causal}")
    O, LSE, dQ, dK, dV, plan = run_fwd_bwd(Q, K, V, dO, causal, depth=depth)[:6]
    # the last launch group's merge covers every segment
    ends = {x for t in range(plan.num_tasks) for g, n, _ in plan.task(t)["runs"] for x in (g, g + n)}
    assert len(ends | {0, L}) - 1 > 64
    _check_vs_oracle(O, LSE, Q, K, V, causal, dt)
    _check_grads((dQ, dK, dV), oracle_grads(Q, K, V, dO, causal), dt)
