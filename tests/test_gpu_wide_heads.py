"""The hand-pipelined forward of d = 224 and 256 at the edges of its 64-key
tiles and 32-key blocks, and where a block cannot keep its row's shift: the
first block of a tile, the second only (the first already accumulated), or
both, each of which leaves the pipelined path at another point.  Float64
oracle; the element bound is the rounding of the weights to the input dtype,
u max|V| (u = 2^-8 bf16, 2^-11 fp16)."""
import pytest
import torch

from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, run_forward, say
from tests.test_gpu_forward import _check_vs_oracle

pytestmark = pytest.mark.gpu

U = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}


@pytest.mark.parametrize("L", [1, 31, 33, 64, 65, 127, 193, 513])
@pytest.mark.parametrize("d,dt,causal", [(224, "f16", False), (224, "bf16", True), (256, "bf16", False),
                                         (256, "f16", True)])
def test_tile_edges(d, dt, causal, L):
    need_gpu()
    Q, K, V = synth.make_inputs(300 + L + d, 1, L, 2, d, dt)
    for depth in (0, 1):
        say(f"wide heads d={d} dt={dt} causal={causal} L={L} depth={depth}")
        O, LSE, _ = run_forward(Q, K, V, causal, depth=depth)
        _check_vs_oracle(O, LSE, Q, K, V, causal, dt, atol=U[dt] * float(V.abs().max()))


@pytest.mark.parametrize("d", [224, 256])
@pytest.mark.parametrize("first", [0, 32])
@pytest.mark.parametrize("every", [32, 64, 192])
def test_blocks_that_leave_the_pipeline(d, first, every):
    """The scores climb by about 20 (log2) at key `first` and every `every`
    keys from there, past the 2^16 that a kept shift allows."""
    need_gpu()
    L = 640
    Q, K, V = synth.make_inputs(500 + every, 1, L, 1, d, "bf16")
    e = torch.ones(d, dtype=torch.float32) / d ** 0.5
    step = ((torch.arange(L) - first).clamp(min=-1).div(every, rounding_mode="floor") + 1).float() * 14.0 * d ** 0.5 / 3.0
    Q = (0.25 * Q.float() + 3.0 * e).to(Q.dtype)
    K = (0.25 * K.float() + step[None, :, None, None] * e).to(K.dtype)
    for causal in (False, True):
        say(f"climbing blocks d={d} first={first} every={every} causal={causal}")
        for depth in (0, 1):
            O, LSE, _ = run_forward(Q, K, V, causal, depth=depth)
            _check_vs_oracle(O, LSE, Q, K, V, causal, "bf16", atol=U["bf16"] * float(V.abs().max()))
