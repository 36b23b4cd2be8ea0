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


def _rounding(tern):
    """What float32 sums of a row's products, which are exact, may be off by, of sum |w x|: a rounding for each of them and a few for the
    scale."""
    return ((tern != 0).sum(1) + 4) * 2.0 ** -24


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
            assert (np.abs(y.cpu().numpy().astype(np.float64) - y_ref) <= _rounding(tern) * bound).all(), batch
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        dd.close()


def _matvec(oracle_dict, tern, scale, mm, batches, like_sizes=False):
    """The matrix-core kernel's result for every batch, with its activations (`like_sizes`: all between 1 and 2, of either sign)."""
    gpu, (rows, cols) = "cuda:0", tern.shape
    codes, row_off = oracle.encode(oracle_dict, tern)
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    M = dev.DeviceMatrix(codes, row_off, scale, rows, cols, device=gpu, device_order_of=dd, minmax_bf16=mm)
    q.qmoe_set_tuning("mfma_min_tokens", 1)
    try:
        for batch in batches:
            x = synth.normal_bf16(66 + batch, (batch, cols))
            if like_sizes:
                x = x & np.uint16(0x807F) | np.uint16(0x3F80)
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
    next to lanes that are so far ahead that their next piece comes too early.  The tolerance is below half of what any one weight adds, so
    that one that is lost, or there twice, shows."""
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
    mm = synth.minmax_bf16(64, rows, 0.06, 0.1) if minmax else None
    smallest = np.abs(synth.bf16_to_f64(mm)).min(1) if minmax else synth.f16_to_f64(scale)
    for batch, x, y in _matvec(oracle_dict, tern, scale, mm, (3, 20, 64, 65), like_sizes=True):
        y_ref, bound = oracle.matvec(tern, scale, x, with_bound=True, minmax_bf16=mm)
        tolerance = _rounding(tern) * bound
        assert (tolerance < 0.5 * smallest).all()  # (|x| is 1 or more)
        assert (np.abs(y - y_ref) <= tolerance).all(), batch


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
        assert (np.abs(y - y_ref) <= _rounding(tern) * bound).all(), batch


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


def _of_weights(tern, grid, x):
    """sum of w x over a row's weights only (no weight, no part), in float64: [tokens, rows]; `grid` float64 [rows, 2] (under -1, under +1)."""
    y = np.zeros((x.shape[0], tern.shape[0]))
    with np.errstate(invalid="ignore"):
        for r in range(tern.shape[0]):
            at = np.flatnonzero(tern[r])
            y[:, r] = (np.where(tern[r, at] > 0, grid[r, 1], grid[r, 0]) * x[:, at]).sum(1)
    return y


def _same(got, ref, tol):
    """Equal where the reference is infinite or no number, within the tolerance elsewhere."""
    odd = ~np.isfinite(ref)
    assert np.array_equal(got[odd], ref[odd], equal_nan=True)
    assert (np.abs(got[~odd] - ref[~odd]) <= np.broadcast_to(tol, ref.shape)[~odd]).all()
    return odd


@pytest.mark.parametrize("cols", [72, 1000])
@pytest.mark.parametrize("minmax", [False, True])
def test_activations_that_are_not_finite(oracle_dict, cols, minmax):
    """An infinite activation, or one that is no number, counts in the rows that have a weight there and in no others, and for its own
    token only; a sum of doubled weights that overflows is no infinity."""
    rows = 70
    tern = synth.ternary(81, rows, cols, 0.7)
    scale = None if minmax else synth.uniform_f16(82, (rows,), 0.01, 0.1)
    mm = synth.minmax_bf16(83, rows, 0.01, 0.1) if minmax else None
    grid = synth.bf16_to_f64(mm) if minmax else np.stack([-scale.view(np.float16), scale.view(np.float16)], 1).astype(np.float64)
    gpu = "cuda:0"
    codes, row_off = oracle.encode(oracle_dict, tern)
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    M = dev.DeviceMatrix(codes, row_off, scale, rows, cols, device=gpu, device_order_of=dd, minmax_bf16=mm)
    q.qmoe_set_tuning("mfma_min_tokens", 1)
    try:
        for batch in (1, 5, 17, 40, 64, 70):
            x = synth.normal_bf16(84 + batch, (batch, cols)).copy()
            x[0, 3] = 0x7F80                                 # +inf
            x[batch // 2, cols - 1] = 0xFF80                 # -inf
            x[batch - 1, 5], x[batch - 1, 6] = 0x7FC0, 0x7F80  # NaN, +inf
            y = torch.full((batch, rows), 7.0, dtype=torch.float32, device=gpu)
            q.qmoe_decode_matvec(dd.handle, M.desc, torch.from_numpy(x.view(np.int16)).to(gpu), y)
            torch.cuda.synchronize()
            xf = synth.bf16_to_f64(x).reshape(batch, cols)
            with np.errstate(invalid="ignore"):
                bound = _of_weights(np.abs(tern), np.abs(grid).max(1, keepdims=True).repeat(2, 1), np.abs(xf))
            odd = _same(y.cpu().numpy().astype(np.float64), _of_weights(tern, grid, xf), cols * 2.0 ** -24 * bound)
            assert odd.any() and not odd.all(), batch
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        dd.close()


@pytest.mark.parametrize("minmax", [False, True])
@pytest.mark.parametrize("n", [8, 30, 150])
def test_layers_of_activations_that_are_not_finite(oracle_dict, n, minmax):
    """The same in a layer: hidden vectors by blocks of tokens, results by gates.  A token whose first product meets an infinity in a
    few rows has finite results in the rows of the second product without a weight there."""
    gpu, E, d_model, d_ff = "cuda:0", 2, 136, 264
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    layer = dev.DeviceLayer(E, d_model, d_ff, gpu, minmax=minmax)
    tern, grid = {}, {}
    for e in range(E):
        for which, rows, cols in (("wi", d_ff, d_model), ("wo", d_model, d_ff)):
            t = synth.ternary(90 + 2 * e + (which == "wo"), rows, cols, 0.9)
            g = synth.minmax_bf16(95 + e, rows, 0.01, 0.1) if minmax else synth.uniform_f16(95 + e, (rows,), 0.01, 0.1)
            layer.set_expert(e, which, *oracle.encode(oracle_dict, t), g)
            tern[e, which] = t
            grid[e, which] = synth.bf16_to_f64(g) if minmax else np.stack([-g.view(np.float16), g.view(np.float16)], 1).astype(np.float64)
    layer.finalize(device_order_of=dd)
    idx = np.arange(n, dtype=np.int32) % E
    x = synth.normal_bf16(99, (n, d_model)).copy()
    x[0, 7], x[1, 0], x[n // 2, 135], x[n - 1, 64] = 0x7F80, 0xFF80, 0x7F80, 0xFF80
    gate = (0.5 + np.arange(n) % 3).astype(np.float32)
    y, ws = torch.empty((n, d_model), dtype=torch.float32, device=gpu), layer.workspace(n)
    q.qmoe_set_tuning("mfma_min_tokens", 1)
    try:
        layer.forward(dd, torch.from_numpy(x.view(np.int16)).to(gpu), torch.from_numpy(idx).to(gpu), y, ws, torch.from_numpy(gate).to(gpu))
        torch.cuda.synchronize()
        out = dev.read_workspace(ws, E, d_model, d_ff, n)
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        dd.close()
    assert out["counters"][7] > 0
    slot = np.empty(n, dtype=np.int64)
    slot[out["perm"][:n]] = np.arange(n)
    hidden = synth.bf16_to_f64(np.ascontiguousarray(out["hidden"][slot])).reshape(n, d_ff)
    for e in range(E):
        own = np.flatnonzero(idx == e)
        ref = np.maximum(_of_weights(tern[e, "wi"], grid[e, "wi"], synth.bf16_to_f64(x[own]).reshape(own.size, d_model)), 0.0)
        odd = _same(hidden[own], ref, 2.0 ** -8 * ref + 1e-5)  # (bf16)
        assert odd.any() and not odd.all()
        ref = _of_weights(tern[e, "wo"], grid[e, "wo"], hidden[own]) * gate[own, None]
        odd = _same(y.cpu().numpy().astype(np.float64)[own], ref, d_ff * 2.0 ** -24 * 3 * np.nansum(np.where(np.isfinite(hidden[own]), hidden[own], 0), 1)[:, None])
        assert odd.any() and not odd[odd.any(1)].all()
