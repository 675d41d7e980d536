"""The two-launch fp32 update against the CPU oracle at the sizes where its dispatch and its tiles change: widths one
below, at and one above 16 and 64, the widest input, layer and head it takes and one beyond (the layered kernels), a
network on either side of the rule for few rows, a single layer, batches that leave 1 to 3 rows of the last group of
four, and both weight-gradient tilings, with one slice of the batch and with several.

Tolerance 1e-4 of each tensor's largest entry: a contraction here adds at most 1024 terms (rows for the gradients: at
most 1500) in fp32, whose rounding is bounded by terms * 2^-24 of the sum of magnitudes, 9e-5 at the worst and a few
1e-6 when the roundings are independent; the batches are drawn clear of the ReLU kinks."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2502_20190_amd import synth
from paper_2502_20190_amd.synth import LIN

import test_gpu_learner as T
import test_gpu_ppo as P
from parity_util import plan_layers

pytestmark = pytest.mark.gpu
TOL = 1e-4


@pytest.fixture(scope="module")
def tj():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2502_20190_amd import binding

    binding.lib()
    return binding


@pytest.mark.parametrize("D,widths,A,B", [
    (1, (15,), 1, 1), (17, (16, 17), 2, 3), (16, (64, 63), 5, 130), (1024, (65,), 64, 66), (4, (), 3, 33),
    (300, (512, 512), 18, 257), (64, (128, 128, 128), 18, 1500), (20, (512,), 65, 40), (1025, (16,), 2, 9),
    (1024, (512,), 18, 128), (1024, (512,), 18, 129)])
def test_q_learner(tj, orc, D, widths, A, B):
    layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=B, layers=layers, precision="fp32",
                 lr=1e-3, target_interval=2)
    g, o = T._pair(tj, orc, wl, seed=3)
    for step in range(2):                       # the second step also refreshes the target network
        rows = T._batch_clear_of_kinks(o, wl, 50 + step, B)
        # weights whose gradient is near Adam's epsilon make the state itself incomparable at 1e-4
        T._step_both(tj, orc, g, o, wl, rows, TOL, check_state=False, sync=step > 0)
        T._check_compute_copies(tj, g, wl)
    T._load_oracle_state_into_gpu(tj, orc, g, o)
    for n in (1, min(2 * B, 5), 2 * B):
        T._check_act(tj, orc, g, o, wl, T._batch(wl, 60, n)["obs"], 0.1, n, TOL)


@pytest.mark.parametrize("D,widths,A,B", [
    (1, (16,), 2, 1), (4, (17, 64), 3, 7), (1024, (65,), 63, 66), (12, (512, 512), 18, 1029), (4, (256, 256), 2, 1500)])
def test_on_policy_learner(tj, orc, D, widths, A, B):
    g, o = P._pair(tj, orc, D, widths, A, "fp32", B, seed=5, lr=1e-3)
    for step in range(2):
        rows = P._batch(orc, o, D, A, 1 + B // 8, 8, 70 + step, "fp32", n=B)
        P._step_both(tj, orc, g, o, rows, TOL, sync=step > 0)
        P._check_compute_copies(tj, g, "fp32")


@pytest.mark.parametrize("on_policy", [False, True])
@pytest.mark.parametrize("D,widths,B", [(4, (16, 17), 8), (20, (33, 40, 29), 33), (5, (1, 3, 2), 3), (20, (33, 41, 29), 2050)])
def test_a_unit_switched_off_by_an_infinite_bias_leaves_the_rest_finite(tj, mlp_plan, D, widths, B, on_policy):
    """Biases lie behind their weight matrix, where the last chunk of a contraction over 17, 29 .. units ends: minus infinity is a
    unit that never fires, the same as a very large negative bias, bit for bit.  2050 rows: eight rows per block, on-policy sixteen."""
    if B > 2048:
        assert mlp_plan.f32_rows(*plan_layers(D, *widths, 4 if on_policy else 3), B, not on_policy, 1) == (16 if on_policy else 8)
    import torch

    A = 3
    layers = synth.ppo_layers(widths, A) if on_policy else tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    g = torch.Generator(device="cuda").manual_seed(4)
    randn = lambda *s: torch.randn(s, generator=g, device="cuda")
    obs, next_obs, a, b, c = randn(B, D), randn(B, D), -1.0 + 0.1 * randn(B), randn(B), randn(B)
    action = torch.zeros(B, dtype=torch.int32, device="cuda")
    got = []
    for off in (-np.inf, -1e30):
        theta = synth.xavier_init(layers, (D, 1, 1), 1)
        at = 0
        for i, (_, w, _, _, _) in enumerate(synth.layer_shapes(layers, (D, 1, 1))):
            at += int(np.prod(w))
            if i + 1 < len(layers):
                theta[at + w[0] // 2] = off
            at += w[0]
        if on_policy:
            lrn = tj.PpoLearner(D, widths, A, "fp32", B, theta)
            assert lrn.step(obs, action, a, b, c) == tj.TJ_OK
        else:
            wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=B, layers=layers, precision="fp32")
            lrn = tj.learner_for_workload(wl, theta, synth.xavier_init(layers, (D, 1, 1), 2))
            mb = tj.Minibatch(B, D, "f32")
            mb.obs.copy_(obs), mb.next_obs.copy_(next_obs), mb.action.copy_(action), mb.reward.copy_(b), mb.done.zero_()
            assert lrn.step(mb) == tj.TJ_OK
        torch.cuda.synchronize()
        got.append(lrn.get_state(tj.TJ_STATE_GRADS))
    assert np.isfinite(got[0]).all() and np.array_equal(*got)


@pytest.mark.parametrize("D,widths,A,batches", [(4, (16,), 2, (2049, 2048, 2063, 2064, 2100)), (20, (33, 70), 3, (4100, 2049, 2048, 2500))])
def test_small_networks_on_long_batches(tj, orc, D, widths, A, batches):
    """Both sides of the batch from which the gradient of every network comes in slices, the last of them empty or of a few rows, on
    one learner that has held longer batches before."""
    layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=max(batches), layers=layers, precision="fp32", lr=1e-3)
    g, o = T._pair(tj, orc, wl, seed=6)
    for step, B in enumerate(batches):
        T._step_both(tj, orc, g, o, wl, T._batch_clear_of_kinks(o, wl, 90 + step, B), TOL, check_state=False, sync=step > 0)
        T._check_compute_copies(tj, g, wl)


@pytest.mark.parametrize("D,widths,A,batches", [
    (4, (16,), 2, (1025, 1031, 1024)), (20, (33, 64, 5), 18, (1032, 1029)), (100, (128,), 7, (1027,)), (4, (16,), 2, (16384, 16381)),
    (4, (16,), 2, (16385, 1030))])
def test_q_learner_with_two_groups_of_rows_per_block(tj, orc, mlp_plan, D, widths, A, batches):
    """From 1025 rows on, narrow networks; partial groups, and both sides of the largest batch that these kernels take.  Roundings of a
    sum over 16 k rows: 16385 * 2^-24 = 1e-3 at the worst, some 128 * 2^-24 = 8e-6 where they are independent."""
    net = plan_layers(D, *widths, A)
    assert mlp_plan.f32_fits(*net, 3, max(batches)) == (max(batches) <= 16384)
    assert [mlp_plan.f32_rows(*net, B, 1, 1) for B in batches] == [8 if B > 1024 else 4 for B in batches]
    layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=max(batches), layers=layers, precision="fp32", lr=1e-3)
    g, o = T._pair(tj, orc, wl, seed=8)
    for step, B in enumerate(batches):
        T._step_both(tj, orc, g, o, wl, T._batch_clear_of_kinks(o, wl, 95 + step, B), TOL, check_state=False, sync=step > 0)
        T._check_compute_copies(tj, g, wl)


@pytest.mark.parametrize("D,widths,A", [(4, (16,), 2), (20, (33, 70, 29, 64, 5), 3), (70, (385,), 18), (17, (512, 40, 512, 400), 6),
                                        (1000, (512, 512), 33)])
def test_acting_on_many_observations(tj, orc, D, widths, A):
    """One, two and four groups of rows per block, whole and partial; deeper networks than the two layers that are kept."""
    layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=2500, layers=layers, precision="fp32")
    g, o = T._pair(tj, orc, wl, seed=7)
    for n in (1024, 1025, 2048, 2053, 4999):
        T._check_act(tj, orc, g, o, wl, T._batch(wl, 61, n)["obs"], 0.1, n, TOL)


@pytest.mark.parametrize("D,widths,A,B", [(20, (192, 320), 18, 70), (300, (257, 129, 64), 33, 1030), (65, (256, 255), 17, 9)])
def test_q_learner_at_the_edges_of_the_feature_tiles(tj, orc, D, widths, A, B):
    """Tiles of 16, 32 and 64 features (128 | 129 and 256 | 257 wide), steps of 64, 32 and 16 k with a remainder, one to three tiles of the
    head.  Tolerance as above: at most 1030 terms."""
    layers = tuple((LIN, w, 0, 0) for w in widths) + ((LIN, A, 0, 0),)
    wl = replace(synth.WORKLOADS["c2"], obs_shape=(D,), n_actions=A, batch=B, layers=layers, precision="fp32", lr=1e-3, target_interval=2)
    g, o = T._pair(tj, orc, wl, seed=9)
    for step in range(2):
        T._step_both(tj, orc, g, o, wl, T._batch_clear_of_kinks(o, wl, 97 + step, B), TOL, check_state=False, sync=step > 0)
        T._check_compute_copies(tj, g, wl)


@pytest.mark.parametrize("D,widths,A,B,rows_per_block", [
    (12, (129, 257), 18, 2101, 16), (5, (33, 448), 2, 2049, 16), (70, (64, 31, 96), 33, 4099, 16), (5, (33, 512), 2, 2049, 8)])
def test_on_policy_learner_with_sixteen_rows_per_block(tj, orc, mlp_plan, D, widths, A, B, rows_per_block):
    """From 2049 rows on: column tiles of 32 with a remainder, more tiles than waves (257 and 448 wide), contractions over fewer rows of a
    matrix than a step and over a remainder, a last block of 1 to 5 rows; and a network too wide for sixteen, which takes eight.
    Sums over 4099 rows: 4099 * 2^-24 = 2.4e-4 at the worst, some 64 * 2^-24 = 4e-6 where the roundings are independent."""
    net = plan_layers(D, *widths, A + 1)
    assert mlp_plan.f32_fits(*net, 1, B) and mlp_plan.f32_rows(*net, B, 0, 1) == rows_per_block
    g, o = P._pair(tj, orc, D, widths, A, "fp32", B, seed=5, lr=1e-3)
    for step in range(2):
        rows = P._batch(orc, o, D, A, 1 + B // 8, 8, 74 + step, "fp32", n=B)
        P._step_both(tj, orc, g, o, rows, TOL, sync=step > 0)
        P._check_compute_copies(tj, g, "fp32")
