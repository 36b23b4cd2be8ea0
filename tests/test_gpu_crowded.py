"""The matrix-core product at the edges of its steps: columns that do not fill a step of 64, token tiles
of one block, of two, of four and their remainders, rows that end inside a wavefront's 64, rows without codewords to
spare and rows of very different lengths next to each other."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_16795_amd as q
from paper_2310_16795_amd import device as dev
from paper_2310_16795_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [8, 24, 32, 56, 64, 72, 128, 200, 1000])
@pytest.mark.parametrize("minmax", [False, True])
def test_partial_steps_and_tiles(oracle_dict, cols, minmax):
    gpu = "cuda:0"
    rows = 70
    tern = np.concatenate([synth.ternary(51, 24, cols, 0.3), synth.ternary(52, 23, cols, 0.9), synth.ternary(53, 23, cols, 1.0)])
    tern = tern[np.random.default_rng(5).permutation(rows)]
    scale = None if minmax else synth.uniform_f16(54, (rows,), 0.01, 0.1)
    mm = synth.minmax_bf16(55, rows, 0.01, 0.1) if minmax else None
    codes, row_off = oracle.encode(oracle_dict, tern)
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    M = dev.DeviceMatrix(codes, row_off, scale, rows, cols, device=gpu, device_order_of=dd, minmax_bf16=mm)
    q.qmoe_set_tuning("mfma_min_tokens", 1)
    try:
        for batch in (1, 15, 17, 32, 33, 63, 64, 130):
            x = synth.normal_bf16(56 + batch, (batch, cols))
            y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device=gpu)
            q.qmoe_decode_matvec(dd.handle, M.desc, torch.from_numpy(x.view(np.int16).copy()).to(gpu), y)
            torch.cuda.synchronize()
            y_ref, bound = oracle.matvec(tern, scale, x, with_bound=True, minmax_bf16=mm)
            assert (np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= 1e-3 * bound + 1e-30).all(), batch
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        dd.close()


def _matvec(oracle_dict, tern, scale, mm, batches):
    """The matrix-core kernel's result for every batch, with its activations."""
    gpu, (rows, cols) = "cuda:0", tern.shape
    codes, row_off = oracle.encode(oracle_dict, tern)
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    M = dev.DeviceMatrix(codes, row_off, scale, rows, cols, device=gpu, device_order_of=dd, minmax_bf16=mm)
    q.qmoe_set_tuning("mfma_min_tokens", 1)
    try:
        for batch in batches:
            x = synth.normal_bf16(66 + batch, (batch, cols))
            y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device=gpu)
            q.qmoe_decode_matvec(dd.handle, M.desc, torch.from_numpy(x.view(np.int16).copy()).to(gpu), y)
            torch.cuda.synchronize()
            yield batch, x, y.cpu().numpy().astype(np.float64)
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        dd.close()


@pytest.mark.parametrize("cols", [512, 1000, 2080])
@pytest.mark.parametrize("minmax", [False, True])
def test_lanes_far_apart(oracle_dict, cols, minmax):
    """Rows that are dense in one half and nearly empty in the other, next to rows the other way round: lanes that run out of codewords
    next to lanes that are so far ahead that their next piece comes too early."""
    rows, half = 130, cols // 2 // 8 * 8
    dense, thin = synth.ternary(61, rows, cols, 0.2), synth.ternary(62, rows, cols, 0.985)
    tern = dense.copy()
    for r in range(rows):
        if r % 4 == 0:
            tern[r, :half] = thin[r, :half]
        elif r % 4 == 1:
            tern[r, half:] = thin[r, half:]
        elif r % 4 == 2:
            tern[r] = thin[r]
    scale = None if minmax else synth.uniform_f16(63, (rows,), 0.01, 0.1)
    mm = synth.minmax_bf16(64, rows, 0.01, 0.1) if minmax else None
    for batch, x, y in _matvec(oracle_dict, tern, scale, mm, (3, 20, 64, 65)):
        y_ref, bound = oracle.matvec(tern, scale, x, with_bound=True, minmax_bf16=mm)
        assert (np.abs(y - y_ref) <= 1e-3 * bound + 1e-30).all(), batch


@pytest.mark.parametrize("cols", [8, 64, 72, 200])
def test_unused_grid_point_is_not_read(oracle_dict, cols):
    """What stands behind a row's last codeword multiplies with zeros: an infinite grid point that the row does not use leaves its
    result alone (rows of negative weights only, rows of positive ones after them)."""
    rows = 70
    tern = -np.abs(synth.ternary(65, rows, cols, 0.6))
    tern[1::2] *= -1
    mm = synth.minmax_bf16(66, rows, 0.01, 0.1).copy()
    ref = mm.copy()
    mm[0::2, 1], mm[1::2, 0] = 0x7F80, 0xFF80  # w_max, w_min
    for batch, x, y in _matvec(oracle_dict, tern.astype(np.int8), None, mm, (5, 20, 32, 64, 100)):
        y_ref, bound = oracle.matvec(tern.astype(np.int8), None, x, with_bound=True, minmax_bf16=ref)
        assert (np.abs(y - y_ref) <= 1e-3 * bound + 1e-30).all(), batch


@pytest.mark.parametrize("batch", [5, 32, 64])
def test_grid_points_far_apart(oracle_dict, batch):
    """A row's small grid point keeps its share next to one that is 2^24 times as large: rows that use only the small one, with the large
    one there, come out as precise as a sum in float32 of the products (2^-24 a sum, in a chain of at most `cols` sums)."""
    rows, cols = 70, 520
    tern = -np.abs(synth.ternary(67, rows, cols, 0.6)).astype(np.int8)
    tern[1::2] *= -1
    mm = synth.minmax_bf16(68, rows, 0.01, 0.1).copy()
    mm[0::2, 1] += 24 << 7  # w_max of the rows of negative weights
    mm[1::2, 0] += 24 << 7  # w_min of the others
    for _, x, y in _matvec(oracle_dict, tern, None, mm, (batch,)):
        y_ref, bound = oracle.matvec(tern, None, x, with_bound=True, minmax_bf16=mm)
        assert (np.abs(y - y_ref) <= cols * 2.0 ** -24 * bound).all()


@pytest.mark.parametrize("ratio", [100.0, 2.0 ** 14])
def test_a_large_grid_point_leaves_the_other_signs_sum_alone(oracle_dict, ratio):
    """Rows of one sign but for two weights, whose grid point is far the larger and whose activations are as much smaller: it scales the
    rounding of their own sum only.  Products are exact in float32, so a row's error is below one rounding (2^-24) of sum |w x| for
    each of its weights."""
    rows, cols = 70, 6144
    tern = -np.abs(synth.ternary(69, rows, cols, 0.9)).astype(np.int8)
    for r in range(rows):
        tern[r, [r % 7, 8 + r % 5]] = 1
    tern[1::2] *= -1
    mm = synth.minmax_bf16(70, rows, 0.01, 0.1).view(np.uint16).copy().reshape(rows, 2)
    small = torch.from_numpy(mm[:, 0].astype(np.uint16).view(np.int16).copy()).view(torch.bfloat16)
    large = (-small.float() * ratio).to(torch.bfloat16)  # |w_max| of the rows whose two weights are positive, |w_min| of the others
    neg, pos = small.clone(), large.clone()
    neg[1::2], pos[1::2] = -large[1::2], -small[1::2]
    mm[:, 0], mm[:, 1] = neg.view(torch.int16).numpy().view(np.uint16), pos.view(torch.int16).numpy().view(np.uint16)
    gpu = "cuda:0"
    codes, row_off = oracle.encode(oracle_dict, tern)
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    M = dev.DeviceMatrix(codes, row_off, None, rows, cols, device=gpu, device_order_of=dd, minmax_bf16=mm)
    q.qmoe_set_tuning("mfma_min_tokens", 1)
    try:
        for batch in (5, 32, 64):
            x = torch.randn((batch, cols), generator=torch.Generator().manual_seed(71 + batch)).clamp(min=0)  # (one sign: no cancellation)
            x[:, :16] /= ratio
            x = x.to(torch.bfloat16).view(torch.int16)
            y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device=gpu)
            q.qmoe_decode_matvec(dd.handle, M.desc, x.to(gpu), y)
            torch.cuda.synchronize()
            y_ref, bound = oracle.matvec(tern, None, x.numpy().view(np.uint16), with_bound=True, minmax_bf16=mm)
            err = np.abs(y.cpu().numpy().astype(np.float64) - y_ref)
            print(batch, (err / bound).max())
            assert (err <= (tern != 0).sum(1) * 2.0 ** -24 * bound).all(), batch
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        dd.close()
