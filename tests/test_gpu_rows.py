"""The kernel that shares a row between several lanes, against the oracle, at the edges of its branches: calls of
one item and of more items than workgroups, tiles of every size, the largest call that groups its tokens itself and
the smallest that does not, rows that no eight and no group of lanes divides, more columns than one round of staging."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_16795_amd as q
from paper_2310_16795_amd import device as dev
from paper_2310_16795_amd import synth
from test_gpu_parity import _build_layer, _check_layer, _check_product, _run_layer, _to_dev16, _upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.fail("the GPU tests need a GPU: the HIP path has no fallback")
    return "cuda:0"


@pytest.fixture(scope="module")
def ddict(gpu, oracle_dict):
    dd = dev.DeviceDict(q.qmoe_dict_from_words(oracle_dict.words), gpu)
    yield dd
    dd.close()


@pytest.fixture(autouse=True)
def always_this_kernel():
    q.qmoe_hook_set("rows", 1)
    yield
    q.qmoe_hook_set("rows", 0)


@pytest.mark.parametrize("minmax", [False, True])
@pytest.mark.parametrize("E,d_model,d_ff,T", [
    (3, 8, 20, 1),        # fewer rows than lanes, one piece per row
    (5, 30, 2, 9),        # two rows
    (40, 258, 130, 1),    # one item on the whole GPU
    (7, 520, 514, 33),    # rows that no eight divides
    (600, 72, 96, 512),   # more items than workgroups, the largest call that groups its tokens itself
    (600, 72, 96, 513),   # ... and the smallest that does not
    (1, 264, 136, 510),   # every tile on one expert
    (4, 64, 8400, 6),     # more columns than one round of staging
])
def test_layer_every_tile(gpu, ddict, oracle_dict, E, d_model, d_ff, T, minmax):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    if T > 8 and E > 4:
        idx[0], idx[T // 2] = -1, E    # tokens without an expert
        idx[1:8] = [2, 2, 2, 2, 3, 3, 3]
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, minmax=minmax)
    gate = np.random.default_rng(5).uniform(0.2, 1.0, T)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu, gate)
    valid = [t for t in range(T) if 0 <= idx[t] < E]
    tok_off, perm = oracle.dispatch(idx, E)
    assert np.array_equal(wsout["tok_off"], tok_off) and np.array_equal(wsout["perm"][:len(valid)], perm)
    assert wsout["counters"][0] == len(valid) and wsout["counters"][2] == len({int(idx[t]) for t in valid})
    covered = np.zeros(len(valid), dtype=int)
    for e, slot0, ntok, _ in wsout["items_wi"][:wsout["counters"][3]]:
        assert tok_off[e] <= slot0 and slot0 + ntok <= tok_off[e + 1]
        covered[slot0:slot0 + ntok] += 1
    n_items = wsout["counters"][3]
    assert (covered == 1).all() and np.array_equal(wsout["items_wi"][:n_items], wsout["items_wo"][:wsout["counters"][4]])
    _check_layer(w, idx, x, y, wsout, valid if len(valid) < 60 else valid[:30] + valid[-30:], gate, asym=minmax)
    assert not y[[t for t in range(T) if not 0 <= idx[t] < E]].any()
    y2, _ = _run_layer(layer, ddict, x, idx, gpu, gate)
    assert np.array_equal(y, y2)
    for tile in (1, 2, 8) if d_ff < 5000 else (1, 2):  # (8: the kernel keeps to four; a plan for eight tokens of 8400 columns does not fit the LDS)
        q.qmoe_set_tuning("token_tile", tile)
        try:
            yt, wst = _run_layer(layer, ddict, x, idx, gpu, gate)
        finally:
            q.qmoe_set_tuning("token_tile", 0)
        _check_layer(w, idx, x, yt, wst, valid[:20], gate, asym=minmax)


@pytest.mark.parametrize("rows,cols,p0,batch", [(1, 2, 0.5, 1), (3, 16, 0.9, 2), (9, 226, 0.8, 3), (2080, 6144, 0.9, 5),
                                                (4001, 130, 0.97, 37), (600, 2080, 0.0, 1), (50, 8194, 1.0, 4), (31, 12000, 0.9, 9)])
@pytest.mark.parametrize("minmax", [False, True])
def test_single_matrix(gpu, ddict, oracle_dict, rows, cols, p0, batch, minmax):
    tern = synth.ternary(rows + cols, rows, cols, p0)
    scale = None if minmax else synth.uniform_f16(1, (rows,), 0.01, 0.1)
    pairs = synth.minmax_bf16(2, rows, 0.01, 0.1) if minmax else None
    x = synth.normal_bf16(3, (batch, cols))
    M = _upload(oracle_dict, tern, scale, gpu, ddict, minmax=pairs)
    y = torch.full((batch, rows), float("nan"), dtype=torch.float32, device=gpu)
    q.qmoe_decode_matvec(ddict.handle, M.desc, _to_dev16(x, gpu), y)
    torch.cuda.synchronize()
    y_ref, bound = oracle.matvec(tern, scale, x, with_bound=True, minmax_bf16=pairs)
    _check_product(y.cpu().numpy(), y_ref, bound, f"{rows}x{cols}")


@pytest.mark.parametrize("T,d_model", [(1, 40), (33, 258), (512, 130), (511, 2050)])
@pytest.mark.parametrize("keep", [0, 5])
def test_tokens_without_an_expert(gpu, ddict, oracle_dict, T, d_model, keep):
    """Nearly all of a call's tokens, and all of them: zero rows, and the others as ever."""
    E = 6
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=96, n_tokens=T)
    x = w.tokens()
    idx = np.where(np.arange(T) % 2, -1, E).astype(np.int32)
    idx[::max(1, T // keep) if keep else T + 1] = 2
    if keep == 0:
        idx[0] = 2 ** 31 - 1
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict)
    print(f"{T} tokens of {d_model}, {keep}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    kept = [t for t in range(T) if idx[t] == 2]
    assert len(kept) <= 6 and wsout["counters"][0] == len(kept) and wsout["counters"][1] == T - len(kept)
    assert not y[[t for t in range(T) if idx[t] != 2]].any()  # (the output held NaN before the call)
    _check_layer(w, idx, x, y, wsout, kept)


@pytest.mark.parametrize("minmax", [False, True])
@pytest.mark.parametrize("E,d_model,d_ff,T,loaded_for", [
    (3, 8, 20, 1, 1),          # fewer rows than the layout's lanes
    (4, 258, 130, 9, 1),       # a row or two per lane, some lanes with one more
    (4, 200, 1030, 33, 1),     # two rows per lane, a few lanes with three
    (2, 520, 3002, 5, 4096),   # many rows per lane that the lanes do not divide
    (40, 258, 516, 1, 1),      # one item on the whole GPU
    (600, 72, 200, 512, 4096),  # more items than workgroups, tokens grouped inside the first product
    (600, 72, 200, 513, 1),    # ... and by the dispatch kernel
    (2, 64, 8400, 6, 1),       # more columns than one round of staging
])
def test_lane_interleaved_layers(gpu, ddict, oracle_dict, monkeypatch, E, d_model, d_ff, T, loaded_for, minmax):
    monkeypatch.setattr(dev.B, "qmoe_plan_row_layout", lambda *a: False)
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    if T > 8 and E > 4:
        idx[0], idx[T // 2] = -1, E
        idx[1:8] = [2, 2, 2, 2, 3, 3, 3]
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, minmax=minmax, lanes_for_tokens=loaded_for)
    assert layer.lanes["wi"] >= 64 and layer.lanes["wo"] >= 64
    gate = np.random.default_rng(5).uniform(0.2, 1.0, T)
    print(f"{layer.lanes} lanes", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu, gate)
    valid = [t for t in range(T) if 0 <= idx[t] < E]
    _check_layer(w, idx, x, y, wsout, valid if len(valid) < 60 else valid[:30] + valid[-30:], gate, asym=minmax)
    assert not y[[t for t in range(T) if not 0 <= idx[t] < E]].any()


@pytest.mark.parametrize("E,T", [(1, 64), (2, 63), (3, 65), (2048, 64), (2047, 1), (5000, 33), (300, 300), (1100, 512), (33, 2)])
@pytest.mark.parametrize("drop", [False, True])
def test_tokens_grouped_in_the_first_product(gpu, ddict, oracle_dict, E, T, drop):
    """Up to 64 tokens in one wavefront's registers, more by masks in LDS: the lists in the workspace are the ones the
    dispatch kernel writes, and the second product finds its shares."""
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=48, d_ff=80, n_tokens=T)
    x, rng = w.tokens(), np.random.default_rng(E + T)
    idx = np.minimum(rng.pareto(0.7, T).astype(np.int64), E - 1).astype(np.int32)
    idx[-(T // 3):] = E - 1
    if drop:
        idx[rng.integers(0, T, 1 + T // 4)] = np.int32(-1 if T % 2 else E)
    layer = dev.DeviceLayer(E, 48, 80, gpu)
    used = sorted({int(e) for e in idx if 0 <= e < E})
    for e in used:
        for which, tern, scale in (("wi", w.wi_ternary(e), w.wi_scale(e)), ("wo", w.wo_ternary(e), w.wo_scale(e))):
            layer.set_expert(e, which, *q.qmoe_encode_host(ddict.handle, tern), scale)
    layer.finalize(device_order_of=ddict)
    print(f"{E} experts, {T} tokens", flush=True)
    y, got = _run_layer(layer, ddict, x, idx, gpu)
    tok_off, perm = oracle.dispatch(idx, E)
    n = int(tok_off[-1])
    assert np.array_equal(got["tok_off"], tok_off) and np.array_equal(got["perm"][:n], perm)
    counts = np.diff(tok_off)
    assert list(got["counters"][:3]) == [n, T - n, int((counts > 0).sum())]
    tiles = [(e, int(tok_off[e]) + i, min(4, int(counts[e]) - i)) for e in used for i in range(0, int(counts[e]), 4)]
    expect = [t for k in ((3, 4), (2,), (1,)) for t in tiles if t[2] in k]
    for items, k in (("items_wi", 3), ("items_wo", 4)):
        assert got["counters"][k] == len(expect) and [tuple(r[:3]) for r in got[items][:len(expect)].tolist()] == expect
    assert list(got["counters"][10:14]) == [0] + [sum(t[2] in k for t in tiles) for k in ((3, 4), (2,), (1,))]
    _check_layer(w, idx, x, y, got, [t for t in range(T) if 0 <= idx[t] < E][:24])
    assert not y[[t for t in range(T) if not 0 <= idx[t] < E]].any()


# Uneven shares (nearly as many items as workgroups) of matrices whose rows no eight divides: a share's beginning may fall behind
# the last row of an item, and the wavefronts of that workgroup go on with the item after it, 16 and more lanes to a row.
@pytest.mark.parametrize("d_model,d_ff,pairs,singles", [(354, 2048, 0, 26), (394, 2048, 0, 44), (396, 4714, 17, 18), (2048, 468, 0, 26)])
@pytest.mark.parametrize("minmax", [False, True])
@pytest.mark.parametrize("lanes", [False, True])
def test_shares_that_begin_behind_an_item(gpu, ddict, oracle_dict, monkeypatch, d_model, d_ff, pairs, singles, minmax, lanes):
    if lanes:
        monkeypatch.setattr(dev.B, "qmoe_plan_row_layout", lambda *a: False)
    E, T = pairs + singles, 2 * pairs + singles
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    x = w.tokens()
    idx = np.concatenate([np.repeat(np.arange(pairs), 2), np.arange(pairs, E)]).astype(np.int32)
    layer = _build_layer(w, oracle_dict, gpu, "library", ddict.handle, order_of=ddict, minmax=minmax, lanes_for_tokens=T if lanes else 0)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    _check_layer(w, idx, x, y, wsout, list(range(T)), asym=minmax)


@pytest.mark.parametrize("minmax", [False, True])
@pytest.mark.parametrize("batch", [3, 7])
def test_three_tokens_like_four(gpu, ddict, oracle_dict, batch, minmax):
    """A tile of three tokens computes what it computes with a fourth token of zeros, infinities among the activations included."""
    rows, cols = 130, 600
    tern = synth.ternary(41, rows, cols, 0.7)
    scale = None if minmax else synth.uniform_f16(1, (rows,), 0.01, 0.1)
    pairs = synth.minmax_bf16(2, rows, 0.01, 0.1) if minmax else None
    x = synth.normal_bf16(3, (batch + 1, cols))
    x[batch - 1, [7, 301]] = 0x7F80
    x[batch] = 0
    M = _upload(oracle_dict, tern, scale, gpu, ddict, minmax=pairs)
    got = []
    for b in (batch, batch + 1):
        y = torch.empty((b, rows), dtype=torch.float32, device=gpu)
        q.qmoe_decode_matvec(ddict.handle, M.desc, _to_dev16(x[:b], gpu), y)
        torch.cuda.synchronize()
        got.append(y.cpu().numpy()[:batch])
    assert np.isinf(got[1]).any() and np.array_equal(got[0], got[1], equal_nan=True)
