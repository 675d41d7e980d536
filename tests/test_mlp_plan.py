"""The plan of the whole-network kernels, compiled for the CPU: what an update writes fits what its learner holds."""
import ctypes

import numpy as np
import pytest

from parity_util import plan_layers

def _random_nets():
    g = np.random.default_rng(0)
    nets = []
    for _ in range(60):
        depth = g.integers(1, 4)
        widths = [int(v) for v in np.exp(g.uniform(np.log(8), np.log(700), depth + 1))] + [int(g.integers(2, 33))]
        nets.append((widths, int(np.exp(g.uniform(np.log(64), np.log(20000))))))
    return nets


@pytest.mark.parametrize("widths,max_batch", [((180, 215, 215, 3), 4177), ((187, 207, 6), 8323)] + _random_nets())
def test_bf16_gradient_slices_of_every_smaller_batch_fit(mlp_plan, widths, max_batch):
    held, written = ctypes.c_int(), ctypes.c_int()
    mlp_plan.b16_slices(*plan_layers(*widths), max_batch, ctypes.byref(held), ctypes.byref(written))
    assert written.value == held.value, (widths, max_batch)


SIDES = list(range(1, 70)) + [127, 128, 129, 255, 257, 511, 512]


def test_fp32_row_kernel_loads_of_the_parameters_end_with_their_matrix(mlp_plan):
    """The backward pass reads W [out][in] itself, whole groups of 64 inputs: at most 63 floats behind it."""
    mlp_plan.f32_reach.restype = ctypes.c_long
    for fin in SIDES:
        for fout in SIDES:
            assert mlp_plan.f32_reach(fin, fout, fin) == (fout - 1) * fin + (fin + 63) // 64 * 64, (fin, fout)


def test_fp32_row_kernel_partial_sums_have_room_for_every_wave_that_multiplies(mlp_plan):
    mlp_plan.f32_active.restype = ctypes.c_uint
    held = ctypes.c_int()
    for rows in SIDES:
        for cols in SIDES:
            assert mlp_plan.f32_active(cols, rows, cols, ctypes.byref(held)) == (1 << held.value) - 1, (rows, cols)


# Updates of few rows whose weight stream through one block takes longer than a launch per layer (128 rows and fewer), and networks
# on the other side of each line: narrower, deeper for their width, longer batches, or small enough in LDS to act here
@pytest.mark.parametrize("widths,max_batch,here", [
    ((1024, 512, 18), 8, False), ((1024, 512, 18), 128, False), ((1024, 512, 18), 129, True), ((1024, 512, 18), 512, True),
    ((768, 512, 18), 32, False), ((896, 512, 512, 18), 64, False), ((768, 512, 512, 512, 18), 32, False),
    ((128, 512, 512, 512, 512, 18), 32, False), ((128, 512, 512, 512, 512, 18), 128, True),
    ((512, 512, 512, 512, 512, 512, 512, 18), 128, False), ((512, 512, 512, 512, 512, 512, 512, 18), 256, True),
    ((128,) + (448,) * 7 + (18,), 64, False), ((1024, 64, 18), 8, True), ((1024, 256, 18), 32, True), ((768,) + (64,) * 4 + (18,), 32, True),
    ((512, 512, 512, 512, 18), 32, True), ((256, 512, 512, 512, 18), 32, True), ((128, 256, 256, 18), 8, True)])
def test_fp32_q_learners_with_few_rows_run_where_an_update_is_faster(mlp_plan, widths, max_batch, here):
    assert mlp_plan.f32_fits(*plan_layers(*widths), 3, max_batch) == here


@pytest.mark.parametrize("widths,max_batch,here", [
    ((896,) + (256,) * 7 + (18,), 8192, True), ((896,) + (256,) * 7 + (18,), 16384, False), ((896,) + (256,) * 7 + (18,), 65536, False),
    ((896,) + (384,) * 7 + (18,), 16384, False), ((1024,) + (320,) * 6 + (18,), 16384, False),
    ((1024,) + (192,) * 6 + (18,), 16384, True), ((1024,) + (192,) * 6 + (18,), 32768, False), ((1024,) + (128,) * 6 + (3,), 32768, False),
    ((896,) + (64,) * 7 + (18,), 65536, True), ((1024,) + (256,) * 5 + (18,), 32768, True), ((512,) * 7 + (18,), 65536, True),
    ((4, 256, 256, 3), 65536, True)])
def test_fp32_on_policy_learners_with_long_batches_run_where_an_update_is_faster(mlp_plan, widths, max_batch, here):
    """Networks that fill LDS with four rows; shallower ones stay, whose acting here weighs more."""
    assert mlp_plan.f32_fits(*plan_layers(*widths), 1, max_batch) == here


def test_fp32_sixteen_rows_multiply_every_weight_once(mlp_plan):
    """The backward pass over W [rows][cols]: what it reads of the gradient and writes of the result stays inside their rows."""
    written, row, gradient = ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    for rows in SIDES:
        for cols in SIDES:
            read = mlp_plan.f32_back16_reach(rows, cols, ctypes.byref(written))
            mlp_plan.f32_pitches(*plan_layers(1, cols, rows), 4, ctypes.byref(row), ctypes.byref(gradient))
            assert rows <= read <= gradient.value and read <= (rows + 63) // 64 * 64, (rows, cols)   # zeros from `rows` on
            assert cols <= written.value <= row.value and written.value <= (cols + 63) // 64 * 64, (rows, cols)


def test_fp32_row_kernel_has_room_for_the_slices_of_every_head(mlp_plan):
    held = ctypes.c_int()
    for fin in SIDES + [1000, 1024]:
        for fout in range(1, 65):
            assert 0 < mlp_plan.f32_head_floats(fin, fout, ctypes.byref(held)) <= held.value, (fin, fout)
