"""Calls on either side of the lines at which the library changes its kernel, with nothing forced, against the oracle."""
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


# The lists of the grouping inside the first product fit the LDS, next to the paper's table, up to 12032 experts for one
# token, 11986 for 32 and 7958 for 64; more experts, up to the 16384 of the layer call, take the dispatch kernel.
@pytest.mark.parametrize("E,T", [(12032, 1), (12033, 1), (16384, 1), (11986, 32), (11987, 32), (16384, 32), (7958, 64), (8192, 64),
                                 (16384, 64)])
def test_many_experts(gpu, ddict, oracle_dict, E, T):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=512, d_ff=512, n_tokens=T)
    x = w.tokens()
    idx = np.resize(np.array([E - 1, 0, E // 2, E - 1, 1], dtype=np.int32), T)
    if T > 8:
        idx[7] = E  # a token without an expert
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=sorted({int(e) for e in idx if e < E}))
    print(f"{E} experts, {T} tokens", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    valid = [t for t in range(T) if idx[t] < E]
    tok_off, perm = oracle.dispatch(idx, E)
    assert np.array_equal(wsout["tok_off"], tok_off) and np.array_equal(wsout["perm"][:len(valid)], perm)
    _check_layer(w, idx, x, y, wsout, valid[:12])
    assert not y[[t for t in range(T) if idx[t] >= E]].any()


# Few lanes per matrix (256 and 192 here), and calls so small that their matrices would be split over more workgroups than that.
@pytest.mark.parametrize("T", [1, 5, 40])
def test_lanes_of_a_large_call_in_a_small_one(gpu, ddict, oracle_dict, T):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=2, d_model=520, d_ff=3002, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, lanes_for_tokens=4096)
    print(f"{T} tokens, {layer.lanes} lanes", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    _check_layer(w, idx, x, y, wsout, list(range(min(T, 8))))


# Batches on both sides of the lines between the single-matrix call's three kernels (256 compute units): 16 lanes per row to
# several, several to the matrix cores, 16 lanes to the matrix cores; widths where a tile's activations are resident
# three times, twice and once, and a width no multiple of eight, which the matrix cores do not take.
@pytest.mark.parametrize("rows,cols,p0,batches", [
    (1040, 2080, 0.80, (1, 249, 250, 377, 378, 412, 413)), (2080, 1040, 0.90, (8, 9, 249, 250, 273, 274)), (2000, 512, 0.80, (193, 194, 201, 202)),
    (1040, 2082, 0.80, (249, 413)), (600, 5096, 0.80, (1, 2, 64)), (300, 3400, 0.92, (4, 5, 65)), (40, 10300, 0.90, (4, 5, 9))])
@pytest.mark.parametrize("minmax", [False, True])
def test_single_matrix(gpu, ddict, oracle_dict, rows, cols, p0, batches, minmax):
    tern = synth.ternary(rows + cols, rows, cols, p0)
    scale = None if minmax else synth.uniform_f16(1, (rows,), 0.01, 0.1)
    pairs = synth.minmax_bf16(2, rows, 0.01, 0.1) if minmax else None
    M = _upload(oracle_dict, tern, scale, gpu, ddict, minmax=pairs)
    x = synth.normal_bf16(3, (max(batches), cols))
    some = sorted({0, 1, 7, 63, 64, 248, 249, *(b - 1 for b in batches)} & set(range(max(batches))))
    y_ref, bound = oracle.matvec(tern, scale, x[some], with_bound=True, minmax_bf16=pairs)
    for b in batches:
        print(f"{rows}x{cols}, {b} tokens", flush=True)
        y = torch.full((b, rows), float("nan"), dtype=torch.float32, device=gpu)
        q.qmoe_decode_matvec(ddict.handle, M.desc, _to_dev16(x[:b], gpu), y)
        torch.cuda.synchronize()
        y = y.cpu().numpy()
        assert np.isfinite(y).all()
        for i, t in enumerate(some):
            if t < b:
                _check_product(y[t][None, :], y_ref[i][None, :], bound[i][None, :], f"{rows}x{cols} token {t} of {b}")


# A workspace without the 32 KiB behind the parts that callers look at, in which the second product of a small call finds its
# shares of the work: accepted by all calls, nothing written behind it, the same results; shorter ones are refused.
@pytest.mark.parametrize("T,d_ff", [(1, 600), (70, 600), (600, 600), (40, 64)])
def test_workspace_without_records(gpu, ddict, oracle_dict, T, d_ff):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=6, d_model=520, d_ff=d_ff, n_tokens=T)
    x, idx = _to_dev16(w.tokens(), gpu), torch.from_numpy(w.expert_idx()).to(gpu)
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict)
    full = layer.workspace(T)
    less = full.numel() - 32768
    pool = torch.full((full.numel(),), 0x5A, dtype=torch.uint8, device=gpu)
    ys = [torch.full((T, w.d_model), float("nan"), dtype=torch.float32, device=gpu) for _ in range(2)]
    print(f"{T} tokens, {less} bytes", flush=True)
    layer.forward(ddict, x, idx, ys[0], full)
    layer.forward(ddict, x, idx, ys[1], pool[:less])
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1]) and bool((pool[less:] == 0x5A).all())
    q.qmoe_moe_dispatch(ddict.handle, 1, idx, 6, w.d_model, d_ff, pool[:less])
    with pytest.raises(q.QmoeError):
        layer.forward(ddict, x, idx, ys[1], pool[:less - 1])
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1]) and bool((pool[less:] == 0x5A).all())


# Offsets that are no offsets, in the lane-interleaved layout, whose pieces lie 1 KiB apart: wrong numbers for that expert, no
# access outside its stream, and the other experts' results as ever.  The calls read the layout with each of the kernels that do.
@pytest.mark.parametrize("T,min_tokens,rows", [(3, 0, 0), (1100, -1, 1), (1100, -1, -1), (1100, 8, 0)])
@pytest.mark.parametrize("kind", ["large", "random", "falling"])
def test_corrupt_offsets_in_the_lane_layout(gpu, ddict, oracle_dict, T, min_tokens, rows, kind):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=3, d_model=264, d_ff=1024, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    idx[:3] = [0, 1, 2]
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, lanes_for_tokens=4096)
    assert layer.lanes["wi"]
    q.qmoe_set_tuning("mfma_min_tokens", min_tokens)
    q.qmoe_hook_set("rows", rows)
    try:
        y, wsout = _run_layer(layer, ddict, x, idx, gpu)
        rng = np.random.default_rng(3)
        for which in ("wi", "wo"):
            off = layer.bufs[which][1]  # [experts][rows + 1]
            n = off.shape[1]
            bad = {"large": np.full(n, 0xFFFFFFFF), "random": rng.integers(0, 2 ** 32, n), "falling": np.arange(n)[::-1] * 40}[kind]
            off[1] = torch.from_numpy(bad.astype(np.uint32).view(np.int32)).to(gpu)
        print(f"{kind} offsets, {T} tokens", flush=True)
        y2, _ = _run_layer(layer, ddict, x, idx, gpu)
    finally:
        q.qmoe_set_tuning("mfma_min_tokens", 0)
        q.qmoe_hook_set("rows", 0)
    sound = [t for t in range(T) if idx[t] != 1]
    assert np.array_equal(y[sound], y2[sound])
    _check_layer(w, idx, x, y, wsout, sound[:4])
    out = torch.full((3, w.d_ff, w.d_model), 77, dtype=torch.int8, device=gpu)
    ptrs = torch.tensor([out[e].data_ptr() for e in range(3)], dtype=torch.int64, device=gpu)
    q.qmoe_decompress(ddict.handle, layer.desc_dev["wi"], layer.format, 3, w.d_ff, w.d_model, 0, ptrs)
    torch.cuda.synchronize()
    for e in (0, 2):
        assert np.array_equal(out[e].cpu().numpy(), w.wi_ternary(e))


# Layer calls on both sides of their lines: tokens grouped inside the first product up to 512, the matrix cores from four
# tokens per compute unit (1024) on, several lanes per row where a matrix has 2^18 weights, both layouts.
@pytest.mark.parametrize("d_model,d_ff", [(512, 512), (510, 512), (512, 520)])
@pytest.mark.parametrize("T", [512, 513, 1023, 1024])
@pytest.mark.parametrize("loaded_for", [0, 4096])
def test_layer(gpu, ddict, oracle_dict, d_model, d_ff, T, loaded_for):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=24, d_model=d_model, d_ff=d_ff, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    idx[3], idx[5] = -1, 24
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, lanes_for_tokens=loaded_for, minmax=bool(T & 1))
    print(f"{d_model}x{d_ff}, {T} tokens, {layer.lanes}", flush=True)
    gate = np.random.default_rng(5).uniform(0.2, 1.0, T)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu, gate)
    _check_layer(w, idx, x, y, wsout, [0, 1, 2, T // 2, T - 1], gate, asym=bool(T & 1))
    assert np.isfinite(y).all() and not y[[3, 5]].any()


# Small calls and decompression in a HIP graph: replays with other work between them, and with other tokens in the same buffers.
@pytest.mark.parametrize("loaded_for", [0, 4096])
@pytest.mark.parametrize("T", [1, 100, 600])
def test_small_calls_in_a_graph(gpu, ddict, oracle_dict, T, loaded_for):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=6, d_model=520, d_ff=520, n_tokens=T)
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, lanes_for_tokens=loaded_for)
    x, idx = _to_dev16(w.tokens(), gpu), torch.from_numpy(w.expert_idx()).to(gpu)
    y, ws = torch.zeros((T, w.d_model), dtype=torch.float32, device=gpu), layer.workspace(T)
    out = torch.zeros((6, w.d_ff, w.d_model), dtype=torch.int8, device=gpu)
    ptrs = torch.tensor([out[e].data_ptr() for e in range(6)], dtype=torch.int64, device=gpu)

    def work(stream):
        layer.forward(ddict, x, idx, y, ws, stream=stream)
        q.qmoe_decompress(ddict.handle, layer.desc_dev["wi"], layer.format, 6, w.d_ff, w.d_model, 0, ptrs, stream=stream)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    print(f"{T} tokens, {layer.lanes}", flush=True)
    with torch.cuda.stream(side):
        work(side.cuda_stream)
        torch.cuda.synchronize()
        eager, dense = y.clone(), out.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            work(side.cuda_stream)
    torch.cuda.synchronize()
    for rep in range(3):
        y.fill_(float("nan"))
        out.fill_(5)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, eager) and torch.equal(out, dense), f"replay {rep}"
        (y * 2).sum().item()
    x.copy_(_to_dev16(w.scaled(cfg_id=97).tokens(), gpu))
    idx.copy_(torch.from_numpy(np.roll(w.expert_idx(), 1) if T > 1 else (w.expert_idx() + 1) % 6))
    graph.replay()
    torch.cuda.synchronize()
    got = y.clone()
    work(torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(got, y) and not torch.equal(got, eager)


# Calls of 1024 tokens, next to the matrix cores: the experts with few tokens take several lanes per row up to 1.25 active experts
# per compute unit (320, which 335 experts do not reach and 336 do), beyond that where two tiles fit the LDS and, lane-interleaved,
# below 2^22 weights.  One to seven tokens, and tiles of one block and of several; eagerly and in a graph.
@pytest.mark.parametrize("E,d_model,d_ff,loaded_for,several", [
    (335, 64, 5900, 0, True), (336, 64, 5900, 0, False), (335, 5900, 64, 4096, True), (336, 5900, 64, 4096, False),
    (700, 64, -2, 0, True), (700, 64, 0, 0, False), (700, -2, 64, 4096, True), (700, 0, 64, 4096, False),
    (700, 2048, 2040, 4096, True), (700, 2048, 2048, 4096, False), (700, 2048, 2048, 0, True), (6, 510, 514, 0, False), (6, 510, 516, 0, True)])
def test_few_tokens_next_to_the_matrix_cores(gpu, ddict, oracle_dict, E, d_model, d_ff, loaded_for, several):
    line = next(c for c in range(5000, 6500, 2) if not q.qmoe_hook_several_lanes(ddict.handle, 1, 700, 64, c, 1024))
    d_model, d_ff = (d if d > 0 else line + d for d in (d_model, d_ff))  # 0: the first width without room for two tiles, -2: the last with
    T, asym = 1024, bool(E & 1)
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    x, counts = w.tokens(), {0: 1, E - 1: 3, 2: 7, 3: 20, 4: 100}
    idx = np.full(T, -1, dtype=np.int32)
    idx[np.random.default_rng(4).permutation(T)[:131]] = np.repeat(list(counts), list(counts.values()))
    layer = _build_layer(w, oracle_dict, gpu, encoder="library", lib_dict=ddict.handle, experts=list(counts), order_of=ddict, minmax=asym,
                         lanes_for_tokens=loaded_for)
    assert bool(layer.lanes["wi"]) == bool(loaded_for)
    assert q.qmoe_hook_several_lanes(ddict.handle, layer.format, E, d_model, d_ff, T) == several
    print(f"{E} experts of {d_model} x {d_ff}, {layer.lanes}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    some = [int(np.flatnonzero(idx == e)[k]) for e, n in counts.items() for k in {0, n - 1}]
    _check_layer(w, idx, x, y, wsout, some, asym=asym)
    assert np.isfinite(y).all() and not y[idx < 0].any()
    xd, idxd, yd, ws = _to_dev16(x, gpu), torch.from_numpy(idx).to(gpu), torch.zeros((T, d_model), dtype=torch.float32, device=gpu), layer.workspace(T)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0]):
        layer.forward(ddict, xd, idxd, yd, ws, stream=streams[0].cuda_stream, side_stream=streams[1].cuda_stream)
    for rep in range(3):
        yd.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(yd.cpu().numpy(), y), f"replay {rep}"


# Thousands of items for several lanes per row: widths that the matrix cores do not take, shares of many items.
@pytest.mark.parametrize("loaded_for", [0, 4096])
def test_many_tokens_without_the_matrix_cores(gpu, ddict, oracle_dict, loaded_for):
    T, E = 20003, 3
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=510, d_ff=518, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    idx[[5, 12345]] = -1, E
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, lanes_for_tokens=loaded_for)
    assert q.qmoe_hook_several_lanes(ddict.handle, layer.format, E, 510, 518, T)
    print(f"{T} tokens, {layer.lanes}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    _check_layer(w, idx, x, y, wsout, [0, 1, 5000, 9999, T // 2, T - 2, T - 1])
    assert np.isfinite(y).all() and not y[[5, 12345]].any() and (y != 0).any(axis=1).sum() == T - 2


# Calls of fewer than 1024 tokens, on both sides of the line from which on their crowded experts take the matrix cores: 626 tokens for
# four experts of 1504 x 2600 (627 on the asymmetric grid), 785 for 32.  Tokens without an expert do not count.
@pytest.mark.parametrize("E,T,lost,crowded,minmax", [
    (4, 625, 0, False, False), (4, 626, 0, True, False), (4, 626, 1, False, False), (4, 637, 11, True, False), (4, 626, 0, False, True),
    (4, 627, 0, True, True), (32, 784, 0, False, False), (32, 785, 0, True, False), (32, 1023, 300, False, False)])
def test_small_calls_on_crowded_experts(gpu, ddict, oracle_dict, E, T, lost, crowded, minmax):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=1504, d_ff=2600, n_tokens=T)
    x = w.tokens()
    idx = np.random.default_rng(T).choice(np.array([0, E - 1], dtype=np.int32), T)
    idx[:3], idx[3:3 + lost] = 1, -1  # one expert with few tokens
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=[0, 1, E - 1], minmax=minmax)
    print(f"{E} experts, {T} tokens, {lost} without, asymmetric grid {minmax}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert (wsout["counters"][7] > 0) == crowded
    kept = [t for t in range(T) if idx[t] >= 0]
    tok_off, perm = oracle.dispatch(idx, E)
    assert np.array_equal(wsout["tok_off"], tok_off) and np.array_equal(wsout["perm"][:len(kept)], perm)
    _check_layer(w, idx, x, y, wsout, kept[:2] + kept[-4:], asym=minmax)
    assert not y[idx < 0].any()


# 1100 tokens, from how many of them on an expert takes the matrix cores: both sides of 4, 7 and 24 tokens per expert and of 4e8 weights
@pytest.mark.parametrize("E,d_model,d_ff,least", [(276, 544, 2680, 8), (275, 544, 2680, 5), (275, 544, 2672, 8), (158, 632, 4008, 5),
                                                  (157, 640, 3984, 6), (157, 640, 3976, 8), (46, 1456, 5976, 6), (45, 1456, 6144, 8)])
def test_crowded_from(gpu, ddict, oracle_dict, E, d_model, d_ff, least):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=1100)
    x, few = w.tokens(), np.repeat(np.arange(5, dtype=np.int32), np.arange(4, 9))
    idx = np.full(1100, E - 1, dtype=np.int32)
    at = np.random.default_rng(E).permutation(1100)[:few.size]
    idx[at] = few
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=[0, 1, 2, 3, 4, E - 1])
    print(f"{E} experts of {d_model} x {d_ff}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert wsout["counters"][7] == (9 - least) + -(-(1100 - few.size) // 64)
    _check_layer(w, idx, x, y, wsout, list(at) + [t for t in (0, 1, 1098, 1099) if idx[t] == E - 1])


# The matrix-core kernel's units (64 rows of a tile) against its 2048 wavefronts: fewer, spread over the compute units or eight to a workgroup
# (`experts` many more than those with tokens), one round, two and their edges, units that are drawn, and workgroups whose wavefronts go in step.
@pytest.mark.parametrize("experts,used,n,d_model,d_ff", [
    (3, 3, 350, 72, 64), (683, 683, 8, 64, 192), (682, 682, 8, 192, 200), (4000, 683, 8, 64, 200), (4000, 256, 8, 512, 520), (900, 585, 8, 256, 224),
    (1000, 1000, 8, 320, 312), (1365, 1365, 8, 64, 192), (1024, 1024, 8, 136, 256), (1025, 1025, 8, 136, 256), (90, 90, 33, 2056, 1544), (200, 64, 33, 2056, 2104)])
def test_units_of_the_matrix_cores(gpu, ddict, oracle_dict, experts, used, n, d_model, d_ff):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=experts, d_model=d_model, d_ff=d_ff, n_tokens=used * n)
    x, some = w.tokens(), np.random.default_rng(used).permutation(experts)[:used].astype(np.int32)
    idx = np.random.default_rng(n).permutation(np.repeat(some, n))
    layer = _build_layer(w, oracle_dict, gpu, encoder="library", lib_dict=ddict.handle, experts=[int(e) for e in some], order_of=ddict)
    units = [used * -(-n // 64) * -(-rows // 64) for rows in (d_ff, d_model)]
    print(f"{used} of {experts} experts of {d_model} x {d_ff}, {n} tokens each: {units} units", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert wsout["counters"][7] == used * -(-n // 64) and np.isfinite(y).all()
    first = {int(e): t for t, e in reversed(list(enumerate(idx)))}
    _check_layer(w, idx, x, y, wsout, [first[int(e)] for e in sorted(some)[::max(1, used // 40)]] + [first[int(max(some))]])
    again, _ = _run_layer(layer, ddict, x, idx, gpu)  # (which wavefront takes a unit does not show)
    assert np.array_equal(y, again)


class _Repeated:
    """A workload of many experts whose matrices are those of the first few."""

    def __init__(self, w, distinct):
        self.w, self.distinct = w, distinct

    def __getattr__(self, name):
        a = getattr(self.w, name)
        return (lambda e: a(e % self.distinct)) if name[:3] in ("wi_", "wo_") else a

    def layer(self, gpu, ddict, minmax):
        layer = dev.DeviceLayer(self.w.n_experts, self.w.d_model, self.w.d_ff, gpu, minmax=minmax)
        for which in ("wi", "wo"):
            coded = [q.qmoe_encode_host(ddict.handle, getattr(self.w, which + "_ternary")(e)) for e in range(self.distinct)]
            for e in range(self.w.n_experts):
                layer.set_expert(e, which, *coded[e % self.distinct], getattr(self, which + ("_minmax" if minmax else "_scale"))(e))
        return layer.finalize(device_order_of=ddict)


# The matrix-core kernel's units in calls on two streams whose few-token kernels run beside it, and have items.  Matrices below 2^18 weights (kernel with a row range per lane
# beside it: tickets, from the first unit on in up to 8/7 of a round; in step, also in one round), larger ones (several lanes per row: a second round from the counter where
# the few-token items are many), and without few-token items a second round that would leave too many long units' places empty.  The same bits as on one stream.
@pytest.mark.parametrize("crowded,n,few,m,d_model,d_ff,minmax", [
    (60, 40, 30, 3, 256, 1000, False), (140, 40, 30, 2, 256, 1000, True), (130, 16, 30, 2, 256, 1000, False), (300, 16, 40, 3, 256, 1000, True), (20, 70, 9, 7, 104, 520, False),
    (270, 9, 1050, 3, 512, 520, False), (576, 16, 0, 0, 4800, 256, False)])
def test_units_beside_few_tokens(gpu, ddict, oracle_dict, crowded, n, few, m, d_model, d_ff, minmax):
    E = crowded + few
    w = _Repeated(synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=crowded * n + few * m), 5)
    x, experts = w.tokens(), np.random.default_rng(E).permutation(E).astype(np.int32)
    idx = np.random.default_rng(n).permutation(np.concatenate([np.repeat(experts[:crowded], n), np.repeat(experts[crowded:], m)]))
    layer = w.layer(gpu, ddict, minmax)
    print(f"{crowded} experts of {d_model} x {d_ff} with {n} tokens, {few} with {m}, asymmetric grid {minmax}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert wsout["counters"][7] == crowded * -(-n // 64) and wsout["counters"][3] == few * -(-m // 4) and np.isfinite(y).all()
    _check_layer(w, idx, x, y, wsout, [int(np.flatnonzero(idx == e)[k]) for e in experts[[0, 1, crowded - 1, -1]] for k in (0, -1)], asym=minmax)
    q.qmoe_set_tuning("overlap", -1)
    try:
        alone, _ = _run_layer(layer, ddict, x, idx, gpu)
    finally:
        q.qmoe_set_tuning("overlap", 0)
    assert np.array_equal(y, alone)


# Calls whose experts all take the matrix cores, those with one token too: both sides of 1024 tokens, of 2^18 weights a matrix, of 2.5 tokens per expert below 3.5e8 weights
# and of 25 above, from 1280 tokens on of 14 up to 7e8 weights; also with tokens without an expert.  `least`: tokens from which on an expert takes them.
@pytest.mark.parametrize("E,d_model,d_ff,T,lost,least", [
    (400, 512, 512, 1024, 0, 1), (400, 512, 512, 1024, 1, 1), (400, 512, 504, 1024, 0, 8), (409, 264, 1000, 1024, 0, 1), (410, 264, 1000, 1024, 0, 8), (437, 296, 2704, 1093, 0, 1),
    (437, 296, 2712, 1093, 0, 8), (41, 2080, 4104, 1025, 0, 1), (41, 2080, 4104, 1025, 5, 1), (42, 2080, 4008, 1049, 0, 8),
    (91, 1024, 4000, 1280, 6, 1), (91, 1024, 4000, 1280, 7, 1), (91, 1024, 4000, 1279, 0, 8), (92, 1024, 4000, 1280, 0, 8), (91, 1024, 7512, 1280, 0, 1),
    (91, 1024, 7520, 1280, 0, 6)])
def test_all_experts_on_the_matrix_cores(gpu, ddict, oracle_dict, E, d_model, d_ff, T, lost, least):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    x, few = w.tokens(), np.repeat(np.arange(5, dtype=np.int32), [1, 2, 5, 7, 8])
    idx = np.full(T, E - 1, dtype=np.int32)
    order = np.random.default_rng(E).permutation(T)
    at = order[:few.size]
    idx[at], idx[order[few.size:few.size + lost]] = few, -1
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=[0, 1, 2, 3, 4, E - 1])
    print(f"{E} experts of {d_model} x {d_ff}, {T} tokens, {lost} without", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert wsout["counters"][7] == sum(n >= least for n in (1, 2, 5, 7, 8)) + -(-(T - lost - few.size) // 64)
    _check_layer(w, idx, x, y, wsout, list(at) + [int(t) for t in np.flatnonzero(idx == E - 1)[[0, 1, -2, -1]]])
    assert np.isfinite(y).all() and not y[idx < 0].any()


# Which kernels the experts of such layers go to when tokens are without an expert, or experts have few: `sizes` = (experts, tokens each) of those that have any, the other
# tokens have none.  least: 1 = all to the matrix cores; 0 = none, up to 13 few-token passes (of four tokens) for ten tiles (of 64), 17 from 3.5e8 weights a projection
# on; 8 = those with eight tokens (asymmetric grid, from 3.5e8 weights on, fewer tokens than the line, more experts below than tiles above).
@pytest.mark.parametrize("E,d_model,d_ff,T,sizes,minmax,least", [
    (128, 768, 3072, 1088, [], False, 0), (128, 768, 3072, 1088, [(1, 1)], False, 0), (128, 768, 3072, 1088, [(70, 1), (10, 5)], False, 0), (128, 768, 3072, 1088, [(70, 1), (7, 9)], False, 0),
    (128, 768, 3072, 1088, [(6, 1), (4, 5)], False, 1), (128, 768, 3072, 1088, [(7, 4), (3, 8)], False, 0), (128, 768, 3072, 1088, [(120, 8)], False, 1), (128, 768, 3072, 1088, [(5, 150)], False, 1),
    (400, 512, 512, 1100, [(324, 2), (75, 5)], False, 0), (400, 512, 512, 1100, [(1, 1), (324, 2), (75, 5)], False, 1), (400, 512, 512, 1100, [(200, 2), (100, 5)], False, 1),
    (400, 512, 960, 2400, [(280, 4), (120, 5)], False, 0), (400, 512, 960, 2400, [(279, 4), (121, 5)], False, 1), (400, 512, 960, 2400, [(400, 6)], False, 1),
    (100, 1568, 2400, 1420, [(3, 4), (7, 8)], True, 0), (100, 1568, 2400, 1420, [(2, 4), (1, 5), (7, 8)], True, 1), (100, 1568, 2400, 1420, [(3, 4), (7, 8)], False, 0),
    (100, 1568, 2400, 1420, [(12, 40), (60, 3)], True, 8), (100, 1568, 2400, 1420, [(12, 40), (60, 3)], False, 1), (100, 1568, 2400, 1420, [(12, 40), (12, 3)], True, 1),
    (100, 1568, 2400, 1420, [(12, 40), (13, 7)], True, 8), (100, 1568, 2400, 1420, [(20, 66), (79, 1)], True, 8), (100, 1568, 2400, 1420, [(20, 66), (80, 1)], True, 1)])
def test_tokens_without_an_expert(gpu, ddict, oracle_dict, E, d_model, d_ff, T, sizes, minmax, least):
    w = _Repeated(synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T), 3)
    n = np.concatenate([np.repeat(m, k) for k, m in sizes] + [np.zeros(0, int)]).astype(int)
    assert n.size <= E and n.sum() <= T
    kept = np.repeat(np.random.default_rng(E).permutation(E)[:n.size].astype(np.int32), n)
    idx = np.random.default_rng(T).permutation(np.concatenate([kept, np.where(np.arange(T - kept.size) % 2, E, -1)])).astype(np.int32)
    x, layer = w.tokens(), w.layer(gpu, ddict, minmax)
    print(f"{E} experts of {d_model} x {d_ff}, {kept.size} of {T} tokens, asymmetric grid {minmax}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    on = n >= (least or 1 << 30)
    assert wsout["counters"][7] == sum(-(-k // 64) for k in n[on]) and wsout["counters"][3] == sum(-(-k // 4) for k in n[~on])
    have = np.flatnonzero((idx >= 0) & (idx < E))
    # (not among them: token 169 of the 1420, whose row 345 sums to 3e-6 out of terms of +-0.17; fp32 sums, with up to 2^-24 of all terms' 5.5 an addition, are within
    # 5e-9 of the terms there on either kernel, which is two bf16 ulp of the rest)
    some = {int(have[k * (have.size - 1) // 7]) for k in range(8)} - {169} if have.size else set()
    _check_layer(w, idx, x, y, wsout, sorted(some), asym=minmax)
    assert not np.delete(y, have, 0).any() and np.isfinite(y).all()


# Calls of fewer than 1024 tokens that take the matrix cores: all experts from 14 tokens per expert on, below from eight tokens on.
@pytest.mark.parametrize("E,T,lost,least", [(68, 952, 0, 1), (68, 951, 0, 8), (4, 700, 0, 1), (68, 1023, 20, 1)])
def test_small_calls_give_all_experts(gpu, ddict, oracle_dict, E, T, lost, least):
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=1504, d_ff=2600, n_tokens=T)
    x, few = w.tokens(), np.repeat(np.arange(3, dtype=np.int32), [1, 7, 8])
    idx = np.full(T, E - 1, dtype=np.int32)
    order = np.random.default_rng(T).permutation(T)
    idx[order[:few.size]] = few
    idx[order[few.size:few.size + lost]] = -1
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=[0, 1, 2, E - 1])
    print(f"{E} experts, {T} tokens, {lost} without", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert wsout["counters"][7] == sum(n >= least for n in (1, 7, 8)) + -(-(T - lost - few.size) // 64)
    _check_layer(w, idx, x, y, wsout, [int(t) for t in order[:few.size]] + [int(t) for t in order[-3:]])
    assert not y[idx < 0].any() and np.isfinite(y).all()


# Calls whose activations go to the first product in blocks of 16 tokens, in the output's memory, against the same call with an output that such
# blocks cannot go to (4 bytes off): the same bits.  Full and partial blocks of every tile size, widths with partial steps and partial pieces of 128
# columns, tokens without an expert (also so many that fewer than 1024 are left), an infinite activation.
@pytest.mark.parametrize("E,d_model,d_ff,lost,minmax,inf", [
    (100, 136, 2056, 0, False, False), (100, 136, 2056, 7, True, False), (100, 264, 2056, 76, False, True), (100, 264, 2056, 77, False, False),
    (96, 456, 2600, 3, False, True), (96, 200, 4104, 3, True, True)])
def test_activations_in_blocks(gpu, ddict, oracle_dict, E, d_model, d_ff, lost, minmax, inf):
    T = 1100
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    x, sizes = w.tokens(), [1, 8, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 130]
    idx = np.full(T, E - 1, dtype=np.int32)
    order = np.random.default_rng(d_model).permutation(T)
    idx[order[:sum(sizes)]] = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    none = order[sum(sizes):sum(sizes) + lost]
    idx[none] = np.where(np.arange(lost) % 2, E, -1)
    at = [int(np.flatnonzero(idx == e)[k]) for e in list(range(len(sizes))) + [E - 1] for k in (0, -1)]
    if inf:
        x[order[-1], 5] = 0x7F80
        at = [t for t in at if t != order[-1]]
    layer = _build_layer(w, oracle_dict, gpu, order_of=ddict, experts=list(range(len(sizes))) + [E - 1], minmax=minmax)
    print(f"{E} experts of {d_model} x {d_ff}, {lost} without, asymmetric grid {minmax}, infinite {inf}", flush=True)
    y, wsout = _run_layer(layer, ddict, x, idx, gpu)
    assert wsout["counters"][7] == sum(-(-n // 64) for n in sizes) + -(-(T - lost - sum(sizes)) // 64)
    _check_layer(w, idx, x, y, wsout, at, asym=minmax)
    assert not y[none].any() and np.isfinite(np.delete(y, order[-1:] if inf else [], axis=0)).all()
    other = torch.full((T * d_model + 1,), float("nan"), dtype=torch.float32, device=gpu)[1:].view(T, d_model)
    layer.forward(ddict, _to_dev16(x, gpu), torch.from_numpy(idx).to(gpu), other, layer.workspace(T))
    torch.cuda.synchronize()
    assert np.array_equal(y, other.cpu().numpy(), equal_nan=True)


def _blocks(x, items, perm):
    """Activations of the listed tiles as the copy leaves them in the output, by slot."""
    out = np.zeros((perm.size, x.shape[1]), dtype=np.uint16)
    for _, slot0, ntok, _ in items:
        for s in range(slot0, slot0 + ntok, 16):
            t = x[perm[s:min(slot0 + ntok, s + 16)]]
            out[s:s + len(t)] = t.reshape(len(t), -1, 8).transpose(1, 0, 2).reshape(len(t), -1)
    return out


# Where those blocks are taken, seen after the dispatch and the first product alone: calls from 2048 units of the first product on (by the plan's estimate: 90 experts, not
# 89), with an output that is aligned and apart from the activations and from the experts' numbers.  Elsewhere the output is untouched by then.  Complete calls give the same
# bits, with a gate, from the entry without a workspace, and from a graph that is replayed between other work.
def test_where_blocks_are_taken(gpu, ddict, oracle_dict):
    T, d_model, d_ff = 1100, 136, 2056
    for E in (90, 89):
        w = _Repeated(synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T), 3)
        x, idx = w.tokens(), np.random.default_rng(E).integers(0, E, T).astype(np.int32)
        idx[:400] = 7
        layer = w.layer(gpu, ddict, False)
        gate = torch.linspace(0.2, 1.0, T, device=gpu)
        room = torch.empty(4 * T * d_model + 64, dtype=torch.uint8, device=gpu)

        def buffers(where):
            """x, experts' numbers and output, the first two inside the third where it says so."""
            room.fill_(0xFF)
            at = 4 if where == "misaligned" else 0
            y = room[at:at + 4 * T * d_model].view(torch.float32).view(T, d_model)
            bits, numbers = _to_dev16(x, gpu), torch.from_numpy(idx).to(gpu)
            if where == "x inside":
                bits = room[2 * T * d_model:4 * T * d_model].view(torch.int16).view(T, d_model).copy_(bits)
            if where == "numbers inside":
                numbers = room[:4 * T].view(torch.int32).copy_(numbers)
            return bits, numbers, y

        results = {}
        for where in ("apart", "misaligned", "x inside", "numbers inside"):
            print(f"{E} experts, {where}", flush=True)
            bits, numbers, y = buffers(where)
            before, ws = y.clone(), layer.workspace(T)
            q.qmoe_hook_set("phases", 1 | 8)
            try:
                layer.forward(ddict, bits, numbers, y, ws, gate)
                torch.cuda.synchronize()
            finally:
                q.qmoe_hook_set("phases", 0)
            out = dev.read_workspace(ws, E, d_model, d_ff, T)
            items = out["items_mm"][:out["counters"][7]]
            assert items[:, 2].sum() == T
            if E == 90 and where == "apart":
                held = y.view(torch.int16).cpu().numpy().view(np.uint16).reshape(-1)[:T * d_model].reshape(T, d_model)
                assert np.array_equal(held, _blocks(x, items, out["perm"]))
            else:
                assert torch.equal(y.view(torch.int32), before.view(torch.int32))
            bits, numbers, y = buffers(where)
            layer.forward(ddict, bits, numbers, y, ws, gate)
            torch.cuda.synchronize()
            results[where] = y.cpu().numpy().copy()
            if where == "apart":
                _check_layer(w, idx, x, results[where], dev.read_workspace(ws, E, d_model, d_ff, T), [0, 1, 399, 400, 1098, 1099], gate=gate.cpu().numpy())
        bits, numbers, y = buffers("apart")
        layer.forward_static(ddict, bits, numbers, y, gate)
        torch.cuda.synchronize()
        results["static"] = y.cpu().numpy().copy()
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            layer.forward(ddict, bits, numbers, y, ws, gate, stream=torch.cuda.current_stream().cuda_stream)
        for k in range(3):
            other = torch.empty_like(y)
            layer.forward(ddict, bits, numbers, other, layer.workspace(T), gate)
            y.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            results[f"replay {k}"] = y.cpu().numpy().copy()
        for what, y in results.items():
            assert np.array_equal(y, results["apart"]), what
