"""GPU: the edges of the launch and dispatch rules (work splits, list
lengths, remainders), each against the CPU oracle or against the same
problem on another path."""
import numpy as np
import pytest

import apd_synth as S
import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_03571_amd as apd
    return apd.Context(0)


def _prob(inst):
    import paper_2403_03571_amd as apd
    return apd.Problem.from_instance(inst, "cuda:0")


@pytest.mark.parametrize("count", [1, 255, 257, 600])
def test_batch_work_list(ctx, count):
    """The list of active work over fewer, as many and more instances than a
    block has threads, instances leaving at different evaluations: each fit
    certified by the oracle's recount, and bit-identical to a batch of one."""
    insts = [S.custom(2, 2 + b % 7, (33 + 8 * (b % 5), 70), seed=b, sigma=0.3) for b in range(count)]
    probs = [_prob(i) for i in insts]
    ws, reps, status = ctx.apd_fit_weights_batched(probs, eps=0.05)
    assert status == "APD_OK" and len({r.evals for r in reps}) > (1 if count > 1 else 0)
    for b in {0, count // 2, count - 1}:
        one, rep, _ = ctx.apd_fit_weights_batched([probs[b]], eps=0.05)
        assert rep[0].evals == reps[b].evals
        np.testing.assert_array_equal(one[0].cpu().numpy(), ws[b].cpu().numpy())
        assert O.evaluate(insts[b], ws[b].cpu().numpy()).maxrel < 0.05
