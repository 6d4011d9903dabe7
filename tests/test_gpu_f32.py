"""The fp32 forward at the edges of its 16-query groups, 32- and 128-query
work groups and 64-key tiles, at every dim layout (whole groups of 64 dims and
a last 32), against the float64 oracle.  Bounds: max |dO| <= 1e-5 and |dLSE| <=
1e-4 as for the fp32 exactness case; rel-L2 <= max(1e-6, u sqrt(n)), u = 2^-24
and n the keys of the longest sum: the partial sums of n independent terms grow
as sqrt(i), so the n roundings add up to about u n / sqrt(12) of a term against
a result of sqrt(n) terms, u sqrt(n / 12), and a factor 3.5 is left."""
import numpy as np
import pytest
import torch

from oracle import dense
from paper_2604_20819_amd import synth
from tests.gpu_util import need_gpu, rel_l2, run_forward, say

pytestmark = pytest.mark.gpu


def _check(O, LSE, Q, K, V, causal, n, rows=None):
    Of, LSEf = dense.attention_forward(synth.as_f64(Q), synth.as_f64(K), synth.as_f64(V), causal, rows=rows)
    Og, LSEg = O.double().numpy(), LSE.double().numpy()
    if rows is not None:
        Og = np.stack([Og[:, r, h] for h, r in enumerate(rows)], axis=2)
        LSEg = np.stack([LSEg[:, h, r] for h, r in enumerate(rows)], axis=1)
    err, rl, lerr = np.abs(Og - Of).max(), rel_l2(Og, Of), np.abs(LSEg - LSEf).max()
    say(f"max_abs={err:.3e} rel_l2={rl:.3e} lse_abs={lerr:.3e}")
    assert err <= 1e-5 and lerr <= 1e-4
    assert rl <= max(1e-6, 2.0 ** -24 * n ** 0.5)

@pytest.mark.parametrize("L", [1, 15, 17, 33, 64, 65, 129])
@pytest.mark.parametrize("d,causal", [(32, True), (64, False), (96, True), (224, False), (256, True)])
def test_short(d, causal, L):
    need_gpu()
    Q, K, V = synth.make_inputs(900 + L + d, 2, L, 3, d, "f32")
    for depth in (0, 1):
        say(f"f32 d={d} causal={causal} L={L} depth={depth}")
        O, LSE, _ = run_forward(Q, K, V, causal, depth=depth)
        _check(O, LSE, Q, K, V, causal, L)


@pytest.mark.parametrize("L,depth", [(1215, 1), (1280, 1), (3333, 0)])
@pytest.mark.parametrize("d,causal", [(32, False), (96, True), (160, False), (256, True)])
def test_wide_work_groups(d, causal, L, depth):
    """Calls of at least 1536 strips of 32 rows whose tasks hold 512 tokens
    or more run 128-query work groups; scores that climb along the keys also
    make them change their shift."""
    need_gpu()
    B, H = 2, 8
    Q, K, V = synth.make_inputs(77 + d, B, L, H, d, "f32")
    K = K + 0.02 * (torch.arange(L) // 64).float()[None, :, None, None]
    rows = synth.sample_rows(5, L, 96, H)
    say(f"f32 wide d={d} causal={causal} L={L} depth={depth}")
    O, LSE, plan = run_forward(Q, K, V, causal, depth=depth)
    lengths = [plan.task(t)["L_local"] for t in range(plan.num_tasks)]
    assert sum((n + 31) // 32 for n in lengths) * B * H >= 1536 and max(lengths) >= 512
    _check(O, LSE, Q, K, V, causal, max(lengths), rows=rows)


@pytest.mark.parametrize("L,H,rows", [(1001, 3, 32), (4100, 2, 128)])
def test_staged_launch_groups_keep_the_bits(L, H, rows):
    """One task, two or three, the planner's number and 32 per launch, gathered or read in place:
    work groups of the call's height in every launch, so every row is summed alike."""
    need_gpu()
    Q, K, V = synth.make_inputs(31, 2, L, H, 64, "f32")
    ref = run_forward(Q, K, V, True, depth=2)
    lengths = [ref[2].task(t)["L_local"] for t in range(ref[2].num_tasks)]
    wide = sum((n + 31) // 32 for n in lengths) * 2 * H >= 1536 and max(lengths) >= 512
    assert wide == (rows == 128)
    for tps in (0, 1, 2, 3, 32):
        say(f"f32 staged L={L} H={H} tasks_per_slot={tps}")
        O, LSE, _ = run_forward(Q, K, V, True, depth=2, read_in_place=False, tasks_per_slot=tps)
        assert torch.equal(O, ref[0]) and torch.equal(LSE, ref[1])
