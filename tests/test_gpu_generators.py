"""Generator kernels at the widths where their split into wavefront runs can go wrong, bit for bit against the oracle.

A wavefront takes runs of 512 columns of one row, of 256 columns of up to 16 rows in large matrices, or 256 elements over the rows' ends where
rows have at most 256 columns: the widths sit on and beside those edges, the row counts leave a last wavefront partly filled."""

import numpy as np
import pytest
import torch

from oracle import rng as orng
from paper_2403_11204_amd import api, datagen

pytestmark = pytest.mark.gpu


def bits(t):
    return t.to(torch.float32).cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("dim", [1, 2, 31, 32, 33, 63, 65, 255, 256, 257, 511, 512, 513, 1100])
@pytest.mark.parametrize("rows", [1, 5, 67])
def test_labels_inputs_and_weights(dim, rows):
    seed = (9 << 32) | (dim * 1000 + rows)
    for dist in (api.UNIFORM01, api.UNIFORM_PM1, api.NORMAL, api.BINARY_PM1):
        ref = orng.make_synthetic_labels(seed, rows, dim, dist, 2.5)
        assert np.array_equal(bits(api.make_synthetic_labels(seed, rows, dim, dist, 2.5)), ref.view(np.uint32))
        got16 = api.make_synthetic_labels(seed, rows, dim, dist, 2.5, api.BF16)
        assert np.array_equal(bits(got16), orng.round_to_bf16(ref).astype(np.float32).view(np.uint32))
    table = api.make_synthetic_labels(seed, 3, dim, api.NORMAL)
    y = datagen.balanced_classes(rows, 3)
    first = (1 << 32) - 2                    # the sample counter's low word wraps inside the batch
    ref = orng.make_segment_inputs(seed, table.cpu().numpy(), y, first, 0.05)
    yd = torch.from_numpy(y).cuda()
    assert np.array_equal(bits(api.make_segment_inputs(seed, table, yd, first, 0.05)), ref.view(np.uint32))
    assert np.array_equal(bits(api.make_segment_inputs(seed, table, yd, first, 0.05, api.BF16)),
                          orng.round_to_bf16(ref).astype(np.float32).view(np.uint32))
    seg = api.Segment([dim, rows], api.RELU_ALL, api.MSE_SIL, max_batch=4)
    seg.init(seed)
    W, b = seg.get_params(0)
    Wr, br = orng.init_weights(seed, 0, rows, dim)
    assert np.array_equal(bits(W), np.asarray(Wr, np.float32).view(np.uint32))
    assert np.array_equal(bits(b), np.asarray(br, np.float32).view(np.uint32))


# 16384 runs of 256 columns and more go 2 to 16 rows to a wavefront: a last one with fewer rows, a last run with one column, and the sample
# counter's low word wrapping inside a wavefront's rows.  Rows whose last run is mostly empty (257 columns) stay single
@pytest.mark.parametrize("rows,dim", [(12290, 257), (4099, 1025), (1537, 8192), (1031, 32769), (1029, 65600)])
def test_several_rows_per_wavefront(rows, dim):
    seed = (7 << 32) | dim
    assert np.array_equal(bits(api.make_synthetic_labels(seed, rows, dim, api.UNIFORM_PM1)),
                          orng.make_synthetic_labels(seed, rows, dim, api.UNIFORM_PM1).view(np.uint32))
    table = api.make_synthetic_labels(seed, 3, dim, api.NORMAL)
    y = datagen.balanced_classes(rows, 3)
    part = slice(rows - 70, rows)            # the oracle's share, from 35 rows before the wrap on
    first = (1 << 32) - rows + 35
    ref = orng.make_segment_inputs(seed, table.cpu().numpy(), y[part], first + part.start, 0.05)
    got = api.make_segment_inputs(seed, table, torch.from_numpy(y).cuda(), first, 0.05)
    assert np.array_equal(bits(got[part]), ref.view(np.uint32))
    again = api.make_segment_inputs(seed, table, torch.from_numpy(y[:64].copy()).cuda(), first, 0.05)      # one row per wavefront
    assert torch.equal(got[:64], again)
    if dim <= 8192:
        seg = api.Segment([dim - 1, rows], api.RELU_ALL, api.MSE_SIL, max_batch=4)      # a row of weights and its bias
        seg.init(seed)
        for tensor, ref in zip(seg.get_params(0), orng.init_weights(seed, 0, rows, dim - 1)):
            assert np.array_equal(bits(tensor), np.asarray(ref, np.float32).view(np.uint32))


@pytest.mark.parametrize("seed, j", [(20, 0x7FFFFF), (28, 0xFFFFFE)])
def test_normals_of_a_long_row(seed, j):
    """2^20 draws, among them one of ln(j 2^-24) whose significand is the largest below 1: the one quotient whose rounding rests on
    the reciprocal instruction itself (see tests/test_generator_rounding.py)."""
    dim = 1 << 20
    r0 = orng.philox4x32_10(np.arange(dim), 0, 0, 0, seed, 0)[0]
    assert np.count_nonzero((r0 >> np.uint32(8)) + np.uint32(1) == j) == 1
    ref = orng.make_synthetic_labels(seed, 1, dim, api.NORMAL)
    assert np.array_equal(bits(api.make_synthetic_labels(seed, 1, dim, api.NORMAL)), ref.view(np.uint32))
