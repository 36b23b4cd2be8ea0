"""Calls of the library on its CPU build (cpu_build.py), seeded: `python cases.py KIND SEED COUNT`.  Prints each call before it is made and
what came of it; the exit code is 1 when an access was out of range or a result wrong."""
import ctypes
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))
import oracle  # noqa: E402
import paper_2310_16795_amd as q  # noqa: E402
from paper_2310_16795_amd import synth  # noqa: E402

L = q.lib()
L.lanes_alloc.restype, L.lanes_alloc.argtypes = ctypes.c_void_p, [ctypes.c_size_t, ctypes.c_int, ctypes.c_size_t]
L.lanes_reports.restype = ctypes.c_long
P, N = ctypes.c_void_p, ctypes.c_int
L.lanes_tile_x.argtypes, L.lanes_dispatch.argtypes = [P, P, N, P, P, N, P, N], [P, N, N, *[P] * 8, N, N]
OD = oracle.Dictionary()
D = q.qmoe_dict_from_words(OD.words)


class Memory:
    """Device memory of a call: all of it with its end, or all with its start, next to what may not be touched."""

    def __init__(self, at_start):
        self.at_start = at_start
        assert L.qmoe_dict_upload(D, self.new(q.qmoe_dict_device_bytes(), 256), q.qmoe_dict_device_bytes(), None) == 0

    def new(self, n, align=4, fill=0xFF):
        p = L.lanes_alloc(n, self.at_start, align)
        ctypes.memset(p, fill, n)
        return p

    def put(self, a, align=None):
        a = np.ascontiguousarray(a)
        p = L.lanes_alloc(a.nbytes, self.at_start, align or a.dtype.itemsize)
        ctypes.memmove(p, a.ctypes.data, a.nbytes)
        return p


def read(p, n, dtype):
    return np.frombuffer((ctypes.c_char * (n * np.dtype(dtype).itemsize)).from_address(p), dtype=dtype).copy()


def matrix(m, rng, tern, scale, order, minmax, lanes, corrupt):
    """corrupt: 1 other codewords, 2 other row offsets, 3 both."""
    codes, off = oracle.encode(OD, tern)
    wave = None
    if lanes:
        codes, wave = q.qmoe_lane_layout_build(codes, off, tern.shape[0], lanes)
    held = np.zeros((codes.size + 7) // 8 * 8, dtype=np.uint16)
    held[:codes.size] = rng.integers(0, 65536, codes.size) if corrupt & 1 else codes
    off = off.astype(np.uint32)
    if corrupt & 2:
        at = rng.integers(0, off.size, max(1, off.size // 3))
        off[at] = rng.integers(0, 2 ** 32, at.size)
    at = m.put(held, 16)
    if order and not corrupt & 1:
        assert L.qmoe_codes_to_device_order(D, at, held.size, None) == 0
    s = m.put(scale, 4 if minmax else 2)
    return q.qmoe_matrix(at, m.put(off), None if minmax else s, *tern.shape, codes.size, order, s if minmax else None,
                         m.put(wave.astype(np.uint32)) if lanes else None, lanes, 0)


def layer(rng, i, corrupt):
    E, T = int(rng.choice([1, 2, 3, 7, 12])), int(np.exp(rng.uniform(0, np.log(20 if corrupt else 150))))
    d_model, d_ff = (2 * int(np.exp(rng.uniform(0, np.log(350)))) for _ in range(2))
    w = synth.WORKLOADS["switch_base128"].scaled(n_experts=E, d_model=d_model, d_ff=d_ff, n_tokens=T)
    idx, x = w.expert_idx(), w.tokens()
    if T > 10:
        idx[:T // 3] = rng.integers(0, E)
    if T > 5:
        idx[[1, T - 2]] = -1, E
    order, minmax = int(rng.integers(0, 2)), bool(rng.integers(0, 2))
    loaded_for = int(rng.choice([0, T, 4096])) if order else 0
    tuning = {"token_tile": int(rng.choice([0, 0, 1, 2, 8])), "lds_dict_entries": int(rng.choice([0, 0, 0, -1, 8192]))}
    hooks = {"rows": int(rng.choice([0, 1, -1])), "stage_out": int(rng.choice([0, 0, -1]))}
    print(f"layer {i}: {E} experts of {d_model} x {d_ff}, {T} tokens, order {order}, minmax {minmax}, loaded for {loaded_for}, {tuning}, {hooks}", flush=True)
    m = Memory(i % 2)
    lanes = [q.qmoe_plan_lanes(D, r, c, E, loaded_for) if loaded_for else 0 for r, c in ((d_ff, d_model), (d_model, d_ff))]
    descs = []
    for n, which in zip(lanes, ("wi", "wo")):
        scale = getattr(w, which + ("_minmax" if minmax else "_scale"))
        of = (q.qmoe_matrix * E)(*[matrix(m, rng, getattr(w, which + "_ternary")(e), scale(e), order, minmax, n, corrupt) for e in range(E)])
        descs.append(m.put(np.frombuffer(bytes(of), dtype=np.uint8), 64))
    fmt = order | (q.FORMAT_GRID_MINMAX if minmax else 0) | (q.format_lanes(*lanes) if loaded_for else 0)
    n_ws = q.qmoe_moe_layer_workspace(E, d_model, d_ff, T)
    ws, y = m.new(n_ws, 256), m.new(4 * T * d_model, 16)
    gate = rng.uniform(0.2, 1.0, T).astype(np.float32)
    for key, v in tuning.items():
        q.qmoe_set_tuning(key, v)
    for key, v in hooks.items():
        q.qmoe_hook_set(key, v)
    status = L.qmoe_moe_layer_forward(D, *descs, fmt, E, d_model, d_ff, m.put(x), m.put(idx), m.put(gate), T, y, ws, n_ws, None, None)
    assert status == 0, status
    if corrupt:
        return True
    out = read(y, T * d_model, np.float32).reshape(T, d_model)
    valid = [t for t in range(T) if 0 <= idx[t] < E]
    ref = oracle.moe_layer(w, idx, x, gate=gate, tokens=valid, asym=minmax)
    # (a hidden value on a rounding boundary may go the other way: 2^-8 of a term)
    return all((np.abs(out[t] - ref[t][0]) <= 2.0 ** -8 * np.abs(ref[t][2]) + 1e-30).all() for t in valid) and not np.delete(out, valid, 0).any()


def single(rng, i, corrupt):
    """One matrix: product, decoding, decompression."""
    kind = ("product", "decode", "decompress")[i % 3]
    rows, cols, p0 = int(np.exp(rng.uniform(0, 4.0 if corrupt else 5.5))), 2 * int(np.exp(rng.uniform(0, 6.3))), float(rng.choice([0.0, 0.5, 0.9, 0.97, 1.0]))
    order, minmax, lanes = int(rng.integers(0, 2)), bool(rng.integers(0, 2)), 0
    if kind == "decompress":
        cols, order, lanes = (cols + 7) // 8 * 8, 1, 64 * int(rng.choice([0, 1, 4]))
    batch, rows_hook = int(np.exp(rng.uniform(0, 3.0))), int(rng.choice([0, 1, -1]))
    print(f"{kind} {i}: {rows} x {cols}, {p0} zeros, order {order}, minmax {minmax}, {lanes} lanes, {batch} tokens, rows {rows_hook}", flush=True)
    tern = synth.ternary(int(rng.integers(1 << 20)), rows, cols, p0)
    scale = synth.minmax_bf16(2, rows, 0.01, 0.1) if minmax else synth.uniform_f16(1, (rows,), 0.01, 0.1)
    m = Memory(i // 3 % 2)
    M = matrix(m, rng, tern, scale, order, minmax, lanes, corrupt)
    if kind == "product":
        x, y = synth.normal_bf16(3, (batch, cols)), m.new(4 * batch * rows)
        q.qmoe_hook_set("rows", rows_hook)
        assert L.qmoe_decode_matvec(D, ctypes.byref(M), m.put(x), batch, y, None) == 0
        ref, bound = oracle.matvec(tern, None if minmax else scale, x, with_bound=True, minmax_bf16=scale if minmax else None)
        return corrupt or (np.abs(read(y, batch * rows, np.float32).reshape(batch, rows) - ref) <= 1e-3 * bound + 1e-30).all()
    if kind == "decode":
        out = [m.new(rows * cols, 1)]
        assert L.qmoe_decode_dense(D, ctypes.byref(M), out[0], 0, None) == 0
    else:
        out = [m.new(rows * cols, 16) for _ in range(3)]
        fmt = 1 | (q.FORMAT_GRID_MINMAX if minmax else 0) | (q.format_lanes(lanes, lanes) if lanes else 0)
        assert L.qmoe_decompress(D, m.put(np.frombuffer(bytes(M) * 3, dtype=np.uint8), 64), fmt, 3, rows, cols, 0, m.put(np.array(out, dtype=np.uint64)), None) == 0
    return corrupt or all(np.array_equal(read(o, rows * cols, np.int8).reshape(rows, cols), tern) for o in out)


def encode(rng, i, bad):
    """The device encoder; bad: a value that is none, or too little room."""
    rows, cols, p0 = int(np.exp(rng.uniform(0, 5.5))), 2 * int(np.exp(rng.uniform(0, 6.5))), float(rng.choice([0.0, 0.3, 0.6, 0.8, 0.9, 0.95, 0.98, 1.0]))
    a_round = int(rng.choice([0, 1, 64, 100]))  # rows
    print(f"encode {i}: {rows} x {cols}, {p0} zeros, {a_round} rows a round", flush=True)
    tern = synth.ternary(int(rng.integers(1 << 20)), rows, cols, p0)
    if i % 3 == 0:
        tern[::3] = synth.ternary(5, len(tern[::3]), cols, 0.4)
    codes, off = oracle.encode(OD, tern)
    room = max(1, codes.size // 2) if bad == 2 else codes.size
    if bad == 1:
        tern[rows // 2, cols // 3] = 5
    m = Memory(i % 2)
    q.qmoe_hook_set("encode_rows", a_round)
    at, at_off, status = m.new(2 * room, 2), m.new(4 * (rows + 1)), m.new(8)
    assert L.qmoe_encode_device(D, m.put(tern), rows, cols, at, room, at_off, status, None) == 0
    status = read(status, 2, np.int32).tolist()
    if bad:
        return status == [-3, rows // 2] if bad == 1 else status[0] == (-2 if codes.size > room else 0)
    return status == [0, 0] and np.array_equal(read(at_off, rows + 1, np.uint32), off) and np.array_equal(read(at, codes.size, np.uint16), codes)


def blocks(rng, i):
    """The copy of activations into blocks of 16 tokens."""
    cols, cus = int(rng.choice([8, 16, 120, 128, 136, 264])), int(rng.choice([1, 6]))
    sizes = rng.choice([1, 2, 15, 16, 17, 31, 33, 48, 63, 64], int(rng.integers(0, 6)))
    more, skipped = int(rng.integers(0, 9)), int(rng.integers(0, 5))  # tokens of no listed tile; slots of one, ahead of the others
    slots = int(sizes.sum()) + skipped
    T = slots + more
    print(f"blocks {i}: {sizes.tolist()} of {T} tokens, {cols} columns, {cus} compute units", flush=True)
    m = Memory(i % 2)
    x, perm = synth.normal_bf16(int(rng.integers(1 << 20)), (T + 1, cols))[:T], rng.permutation(T).astype(np.int32)
    at = skipped + np.concatenate([[0], np.cumsum(sizes)])[:len(sizes)].astype(int)
    items = np.array([[0, s, n, 0] for s, n in zip(at, sizes)], dtype=np.int32).reshape(-1, 4)
    order = rng.permutation(len(items))
    out = m.new(max(1, 2 * slots * cols), 16)
    assert L.lanes_tile_x(m.put(items[order]) if len(items) else None, m.put(np.array([len(items)], dtype=np.int32)), max(1, len(items)), m.put(perm[:max(1, slots)]), m.put(x, 16), cols, out, cus) == 0
    got, want = read(out, slots * cols, np.uint16).reshape(slots, cols), np.full((slots, cols), 0xFFFF, dtype=np.uint16)
    for s, n in zip(at, sizes):
        for b in range(0, n, 16):
            t = x[perm[s + b:s + min(n, b + 16)]]
            want[s + b:s + b + len(t)] = t.reshape(len(t), cols // 8, 8).transpose(1, 0, 2).reshape(len(t), cols)
    return np.array_equal(got, want)


def dispatch(rng, i):
    """The dispatch of calls whose experts may all take the matrix cores."""
    E, T = int(rng.choice([1, 5, 40, 130, 300])), int(np.exp(rng.uniform(0, np.log(1500))))
    idx = rng.integers(0, E, T)
    if rng.random() < 0.5:
        idx = np.minimum((E * rng.random(T) ** 4).astype(int), E - 1)
    idx[rng.random(T) < rng.choice([0.0, 0.1, 0.7, 1.0])] = rng.choice([-1, E, 1 << 30])
    idx = idx.astype(np.int32)
    n = np.bincount(idx[(idx >= 0) & (idx < E)], minlength=E)
    kept = int(n.sum())
    passes, tiles = int((-(-n // 4)).sum()), int((-(-n // 64)).sum())
    edge = 10 * passes // max(1, tiles)
    lines = [1, int(rng.choice([kept, kept + 1, 1, T])), int(rng.choice([5, 8])), int(rng.choice([0, kept, kept + 1, T + 1])), int(rng.choice([13, 17, edge, edge + 1])), int(rng.integers(0, 2))]
    least = lines[0] if kept >= lines[1] else lines[2]
    if kept < lines[3]:
        few, crowded = int(((n > 0) & (n < lines[2])).sum()), int((-(-n[n >= lines[2]] // 64)).sum())
        least = 1 << 30 if 10 * passes <= lines[4] * tiles else (lines[2] if lines[5] and kept < lines[1] and few > crowded else 1)
    print(f"dispatch {i}: {E} experts, {kept} of {T} tokens, lines {lines}", flush=True)
    m = Memory(i % 2)
    lists, off, perm, counters, y = [m.new(16 * T, 16) for _ in range(3)], m.new(4 * (E + 1)), m.new(4 * T), m.new(64), m.new(4 * T * 3)
    assert L.lanes_dispatch(m.put(idx), T, E, off, perm, counters, *lists, m.put(np.array(lines, dtype=np.int32)), y, 3, 160 << 10) == 0
    c, ref_off, ref_perm = read(counters, 16, np.int32), *oracle.dispatch(idx, E)
    right = np.array_equal(read(off, E + 1, np.int32), ref_off) and np.array_equal(read(perm, kept, np.int32), ref_perm)
    for list_at, count, tile, experts in ((lists[0], c[3], 4, n < least), (lists[1], c[4], 4, n < least), (lists[2], c[7], 64, n >= least)):
        got = read(list_at, 4 * count, np.int32).reshape(count, 4).tolist()
        right &= sorted(got) == [[e, ref_off[e] + b, min(tile, n[e] - b), 0] for e in np.flatnonzero(experts) for b in range(0, n[e], tile)]
    none = (idx < 0) | (idx >= E)
    return right and c[0] == kept and c[1] == none.sum() and not read(y, 3 * T, np.float32).reshape(T, 3)[none].any()


if __name__ == "__main__":
    kind, seed, count = sys.argv[1], int(sys.argv[2]), int(sys.argv[3])
    rng, ok = np.random.default_rng(seed), True
    for i in range(count):
        before = L.lanes_reports()
        right = {"layer": lambda: layer(rng, i, 0), "layer_corrupt": lambda: layer(rng, i, 1 + i % 3), "single": lambda: single(rng, i, 0),
                 "single_corrupt": lambda: single(rng, i, 1 + i % 4 % 3), "encode": lambda: encode(rng, i, i % 4 % 3),
                 "blocks": lambda: blocks(rng, i), "dispatch": lambda: dispatch(rng, i)}[kind]()
        out = L.lanes_reports() - before
        ok &= bool(right) and out == 0
        if not right or out:
            print(f"  -> right {bool(right)}, {out} accesses out of range", flush=True)
    print("done" if ok else "failed", flush=True)
    sys.exit(0 if ok else 1)
