"""The whole-network bf16 kernels against the bf16-rounding CPU oracle at the sizes where their dispatch and their tiles
change: widths one below, at and one above 32 and 64, the widest input, layer and head they take and one beyond (the
layered kernels), a single layer, batches around one and two groups of 16 rows, one, two and four groups per block, and
both weight-gradient tilings, with one slice of the batch and with several.

Tolerance 2e-2 of each tensor's largest entry, as for every bf16 update: both sides round operands to 8 significant bits
(2^-9 relative), and a value next to a rounding boundary may round to neighbouring bf16 numbers on the two sides
(2^-8 of one operand) wherever their fp32 and fp64 sums differ."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2502_20190_amd import synth
from paper_2502_20190_amd.synth import LIN

import test_gpu_learner as T
import test_gpu_ppo as P
from parity_util import plan_layers

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.fixture(scope="module")
def tj():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2502_20190_amd import binding

    binding.lib()
    return binding


@pytest.mark.parametrize("D,widths,A,B", [
    (1, (31,), 1, 1), (33, (32, 33), 2, 15), (64, (65, 63), 5, 17), (1024, (64,), 32, 33), (4, (), 3, 31),
    (77, (300, 300), 17, 1000), (250, (700, 700), 18, 130), (64, (100, 256, 40, 128), 18, 4100), (64, (128, 128), 33, 40),
    (1025, (64,), 2, 40)])
def test_q_learner(tj, orc, D, widths, A, B):
    layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=B, layers=layers, precision="bf16",
                 lr=1e-3, target_interval=2)
    g, o = T._pair(tj, orc, wl, seed=3)
    for step in range(2):                       # the second step also refreshes the target network
        T._step_both(tj, orc, g, o, wl, T._batch(wl, 50 + step, B), TOL, sync=step > 0)
    T._load_oracle_state_into_gpu(tj, orc, g, o)
    for n in (1, 2 * B):
        T._check_act(tj, orc, g, o, wl, T._batch(wl, 60, n)["obs"], 0.1, n, TOL)


@pytest.mark.parametrize("D,widths,A,B", [
    (1, (32,), 2, 1), (33, (65, 31), 3, 18), (1024, (1024,), 31, 33), (12, (512, 512), 18, 4130), (4, (64, 64), 2, 16400)])
def test_on_policy_learner(tj, orc, D, widths, A, B):
    g, o = P._pair(tj, orc, D, widths, A, "bf16", B, seed=5, lr=1e-3)
    for step in range(2):
        rows = P._batch(orc, o, D, A, 1 + B // 8, 8, 70 + step, "bf16", n=B)
        P._step_both(tj, orc, g, o, rows, TOL, sync=step > 0, precision="bf16")


# Networks whose groups of rows fill LDS to a few KB: the most that any of them takes per block
@pytest.mark.parametrize("D,widths,A,B,rows_per_block,on_policy", [
    (128, (160, 160, 160), 18, 4129, 32, False), (256, (64, 64), 18, 4100, 32, False), (128, (736, 736), 18, 4100, 32, True),
    (384, (64, 64), 18, 8210, 64, True)])
def test_rows_per_block_that_fill_lds(tj, orc, mlp_plan, D, widths, A, B, rows_per_block, on_policy):
    net = plan_layers(D, *widths, A + on_policy)
    assert mlp_plan.b16_fits(*net, 1 if on_policy else 3, B) and mlp_plan.b16_rows(*net, B, not on_policy, 1) == rows_per_block
    if on_policy:
        test_on_policy_learner(tj, orc, D, widths, A, B)
    else:
        test_q_learner(tj, orc, D, widths, A, B)


@pytest.mark.parametrize("D,widths,A,max_batch,batches", [
    (180, (215, 215), 3, 4177, (4090, 4177, 4082, 4080)), (187, (207,), 6, 8323, (8164, 8323, 40))])
@pytest.mark.parametrize("on_policy", [False, True])
def test_smaller_batches_of_a_larger_learner(tj, D, widths, A, max_batch, batches, on_policy):
    """Across the switch between the tilings, where a smaller batch may be cut into more slices than the largest one: the
    kernels see the batch only, so a learner made for it gives the same bits."""
    import torch

    if on_policy:
        layers = synth.ppo_layers(widths, A)
        theta = synth.xavier_init(layers, (D, 1, 1), 1)
        make = lambda n: tj.PpoLearner(D, widths, A, "bf16", n, theta)
    else:
        layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
        wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=max_batch, layers=layers, precision="bf16")
        theta, target = T._init_state(wl, 1)
        make = lambda n: tj.learner_for_workload(wl, theta, target, max_batch=n)
    large = make(max_batch)
    g = torch.Generator(device="cuda").manual_seed(2)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")
    for t, B in enumerate(batches):
        small = make(B)
        action = torch.randint(0, A, (B,), generator=g, device="cuda", dtype=torch.int32)
        if on_policy:
            rows = (randn(B, D), action, -1.0 + 0.1 * randn(B), randn(B), randn(B))
            step = lambda lrn: lrn.step(*rows)
        else:
            mb = tj.Minibatch(B, D, "f32")
            for f, v in (("obs", randn(B, D)), ("next_obs", randn(B, D)), ("action", action), ("reward", randn(B)),
                         ("done", (randn(B) > 1.5).to(torch.uint8))):
                getattr(mb, f).copy_(v.view(getattr(mb, f).shape))
            step = lambda lrn: lrn.step(mb)
        for which in (tj.TJ_STATE_PARAMS, tj.TJ_STATE_ADAM_M, tj.TJ_STATE_ADAM_V):
            small.set_state(which, large.get_state(which))
        assert tj.lib().tj_learner_set_step(small.h, t) == tj.TJ_OK
        if not on_policy:
            small.set_state(tj.TJ_STATE_TARGET, large.get_state(tj.TJ_STATE_TARGET))
        assert step(large) == step(small) == tj.TJ_OK
        torch.cuda.synchronize()
        assert torch.equal(large.stats, small.stats)
        for which in (tj.TJ_STATE_PARAMS, tj.TJ_STATE_ADAM_M, tj.TJ_STATE_ADAM_V, tj.TJ_STATE_GRADS):
            assert np.array_equal(large.get_state(which), small.get_state(which)), (B, which)
