"""Gradients at the edges of the backward kernels' tiles (32 and 64 queries, 64
keys, 128- and 256-row strips) at head dims of every form of the kernels (own or
compiler's order of the products, columns split evenly or not), against the
float64 oracle with the backward grid's bounds."""
import pytest

from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, say
from tests.test_gpu_backward import _check_grads, oracle_grads, run_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [31, 33, 65, 129, 257])
@pytest.mark.parametrize("d,dt,causal", [(32, "f16", False), (64, "bf16", True), (96, "f16", True), (128, "bf16", False),
                                         (160, "bf16", True), (192, "f16", False), (224, "f16", True),
                                         (256, "bf16", False)])
def test_tile_edges(d, dt, causal, L):
    need_gpu()
    Q, K, V, dO = synth.make_inputs(700 + L + d, 1, L, 2, d, dt, with_dO=True)
    want = oracle_grads(Q, K, V, dO, causal)
    for depth in (0, 1):
        say(f"bwd edges d={d} dt={dt} causal={causal} L={L} depth={depth}")
        got = run_fwd_bwd(Q, K, V, dO, causal, depth=depth)[2:5]
        _check_grads(got, want, dt)
