"""fp16 weights at the edge of their type.  The largest finite fp16 is 65504 and
65520 already rounds to infinity, so a tile may keep its row's shift only while
every weight stays below that.  Each row here meets, after keys of score 0,
keys whose score lies between log2(65520) and 16 above them, with every other
key far below: one weight alone decides.  Float64 oracle, finite results, the
element bound u max|V| of the rounded weights (u = 2^-11)."""
import math

import pytest
import torch

from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, run_forward, say
from tests.test_gpu_forward import _check_vs_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 64, 128, 192, 224, 256])
@pytest.mark.parametrize("first", [64 + 5, 64 + 37, 128])  # a tile's first block, its second, its first key
def test_weights_between_the_largest_fp16_and_two_to_the_16(d, first):
    need_gpu()
    L = 450
    Q, K, V = synth.make_inputs(1600 + d, 1, L, 2, d, "f16")
    score = math.log2(65528.0) * math.log(2.0) * math.sqrt(d)  # of q.k: (65520 + 65536) / 2
    hi = torch.tensor(score).half()
    Q.zero_()
    Q[..., 0], Q[..., 1] = 1.0, 2.0 ** -10
    K.zero_()
    K[:, 64:, :, 0] = -400.0
    K[:, first::128, :, 0] = hi
    K[:, first::128, :, 1] = (score - float(hi)) * 2.0 ** 10
    w = 2.0 ** ((synth.as_f64(Q)[0, 0, 0] @ synth.as_f64(K)[0, first, 0]) / math.sqrt(d) / math.log(2.0))
    assert 65520.0 < w < 65536.0
    for causal in (False, True):
        for depth in (0, 1):
            say(f"fp16 weights at the type's edge d={d} first={first} causal={causal} depth={depth}")
            O, LSE, _ = run_forward(Q, K, V, causal, depth=depth)
            _check_vs_oracle(O, LSE, Q, K, V, causal, "f16", atol=2.0 ** -11 * float(V.abs().max()))
