"""Decompression at the edges of its groups and rings: widths around one group of columns and one ring, a row of one piece,
rows that no wavefront divides, all-zero and zero-free rows, both layouts, destinations at odd 16-byte offsets."""
import numpy as np
import pytest
import torch

import paper_2310_16795_amd as q
from paper_2310_16795_amd import device as dev
from paper_2310_16795_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,p0", [(1, 8, 0.9), (3, 248, 0.9), (5, 256, 0.0), (130, 264, 0.97), (67, 2048, 0.885), (65, 2056, 1.0),
                                          (9, 384, 0.9), (9, 392, 0.9), (2, 512, 0.0), (33, 1000, 0.9),
                                          (9, 20000, 0.9)])
@pytest.mark.parametrize("lanes", [0, 64, 192])
def test_edges(rows, cols, p0, lanes):
    gpu = "cuda:0"
    dd = dev.DeviceDict(device=gpu)
    tern = synth.ternary(rows * 7 + cols, rows, cols, p0)
    pairs = synth.minmax_bf16(5, rows, 0.01, 0.1)
    scale = synth.uniform_f16(6, (rows,), 0.01, 0.1)
    codes, off = q.qmoe_encode_host(dd.handle, tern)
    wave_off = None
    if lanes:
        codes, wave_off = q.qmoe_lane_layout_build(codes, off, rows, lanes)
    d_codes = torch.from_numpy(np.concatenate([codes, np.zeros(8, np.uint16)]).view(np.int16)).to(gpu)
    q.qmoe_codes_to_device_order(dd.handle, d_codes)
    keep = [torch.from_numpy(a.view(np.int32 if a.dtype.itemsize == 4 else np.int16).copy()).to(gpu)
            for a in (off.astype(np.uint32), scale, pairs, *([wave_off] if lanes else []))]
    desc = (q.qmoe_matrix * 2)()
    desc[1] = q.qmoe_matrix(d_codes.data_ptr(), keep[0].data_ptr(), keep[1].data_ptr(), rows, cols, int(codes.size), 1,
                            keep[2].data_ptr(), keep[3].data_ptr() if lanes else None, lanes, 0)
    d_desc = torch.from_numpy(np.frombuffer(bytes(desc), dtype=np.uint8).copy()).to(gpu)
    sb = (scale.view(np.float16).astype(np.float32).view(np.uint32))
    sb = ((sb + 0x7FFF + ((sb >> 16) & 1)) >> 16).astype(np.uint16)[:, None]
    want = {0: tern, 1: np.where(tern == 0, 0, np.where(tern > 0, sb, sb | 0x8000)).astype(np.uint16),
            2: np.where(tern == 0, 0, np.where(tern > 0, pairs[:, 1:2], pairs[:, 0:1])).astype(np.uint16)}
    for kind in (0, 1, 2):
        dt = torch.int8 if kind == 0 else torch.int16
        pool = torch.full((rows * cols + 400,), 77, dtype=dt, device=gpu)
        at = 24 * (2 if kind == 0 else 1)  # a multiple of 16 bytes that is none of a line
        ptrs = torch.tensor([0, pool.data_ptr() + at * pool.element_size()], dtype=torch.int64, device=gpu)
        fmt = q.FORMAT_DEVICE_ORDER | (q.FORMAT_GRID_MINMAX if kind == 2 else 0)
        print(f"{rows}x{cols} lanes {lanes} kind {kind}", flush=True)
        q.qmoe_decompress(dd.handle, d_desc, fmt, 2, rows, cols, min(kind, 1), ptrs)
        torch.cuda.synchronize()
        host = pool.cpu().numpy()
        got = host[at: at + rows * cols].reshape(rows, cols)
        assert np.array_equal(got if kind == 0 else got.view(np.uint16), want[kind])
        assert (host[:at] == 77).all() and (host[at + rows * cols:] == 77).all()
    dd.close()


@pytest.mark.parametrize("n_mats,rows,cols", [(1500, 24, 40), (1800, 20, 768), (1800, 20, 776), (70, 3, 400), (5000, 2, 8)])
@pytest.mark.parametrize("wanted", ["all", "some"])
def test_many_matrices(n_mats, rows, cols, wanted):
    """A wavefront goes from matrix to matrix through the ones that have a destination: many of them, none for hundreds in a row,
    rows that no unit divides, widths on both sides of the lines between eight and 32 lanes per row."""
    gpu, made = "cuda:0", 7
    dd = dev.DeviceDict(device=gpu)
    scale = synth.uniform_f16(6, (rows,), 0.01, 0.1)
    terns = [synth.ternary(40 + i, rows, cols, 0.85) for i in range(made)]
    mats = [dev.DeviceMatrix(*q.qmoe_encode_host(dd.handle, t), scale, rows, cols, device=gpu, device_order_of=dd) for t in terns]
    desc = (q.qmoe_matrix * n_mats)(*[mats[m % made].desc for m in range(n_mats)])
    rng = np.random.default_rng(n_mats)
    want = np.ones(n_mats, bool) if wanted == "all" else rng.random(n_mats) < 0.3
    if wanted == "some":
        want[n_mats // 5: n_mats // 2] = False
        want[-1] = True
    at = np.flatnonzero(want)
    out = torch.full((at.size + 1, rows, cols), 77, dtype=torch.int8, device=gpu)
    ptrs = np.zeros(n_mats, dtype=np.int64)
    ptrs[at] = out.data_ptr() + np.arange(at.size) * rows * cols
    d_desc = torch.from_numpy(np.frombuffer(bytes(desc), dtype=np.uint8).copy()).to(gpu)
    print(f"{n_mats} of {rows}x{cols}", flush=True)
    q.qmoe_decompress(dd.handle, d_desc, q.FORMAT_DEVICE_ORDER, n_mats, rows, cols, 0, torch.from_numpy(ptrs).to(gpu))
    torch.cuda.synchronize()
    host = out.cpu().numpy()
    assert np.array_equal(host[:-1], np.stack(terns)[at % made]) and (host[-1] == 77).all()
    dd.close()


@pytest.mark.parametrize("kind", [0, 1, 2])
def test_stream_past_its_width_spoils_no_other_row(kind):
    """Two matrices whose every row runs on to ten times the width they are described with, and two sound ones that the same
    wavefronts take after them: the sound ones come out whole."""
    gpu, rows, cols = "cuda:0", 4096, 64
    dd = dev.DeviceDict(device=gpu)
    long = synth.ternary(3, rows, 10 * cols, 0.9)
    sound = synth.ternary(4, rows, cols, 0.9)
    scale, pairs = synth.uniform_f16(6, (rows,), 0.01, 0.1), synth.minmax_bf16(5, rows, 0.01, 0.1)
    desc, keep = (q.qmoe_matrix * 4)(), []
    for i, tern in ((0, long), (2, sound)):
        codes, off = q.qmoe_encode_host(dd.handle, tern)
        M = dev.DeviceMatrix(codes, off, None if kind == 2 else scale, rows, cols, device=gpu, device_order_of=dd,
                             minmax_bf16=pairs if kind == 2 else None)
        desc[i] = desc[i + 1] = M.desc
        keep.append(M)
    d_desc = torch.from_numpy(np.frombuffer(bytes(desc), dtype=np.uint8).copy()).to(gpu)
    out = torch.full((6, rows, cols), 77, dtype=torch.int8 if kind == 0 else torch.int16, device=gpu)
    ptrs = torch.tensor([out[i].data_ptr() for i in range(1, 5)], dtype=torch.int64, device=gpu)
    print(f"kind {kind}", flush=True)
    q.qmoe_decompress(dd.handle, d_desc, q.FORMAT_DEVICE_ORDER | (q.FORMAT_GRID_MINMAX if kind == 2 else 0), 4, rows, cols, min(kind, 1),
                      ptrs)
    torch.cuda.synchronize()
    host = out.cpu().numpy()
    sb = scale.view(np.float16).astype(np.float32).view(np.uint32)
    sb = ((sb + 0x7FFF + ((sb >> 16) & 1)) >> 16).astype(np.uint16)[:, None]
    want = (sound if kind == 0 else
            np.where(sound == 0, 0, np.where(sound > 0, sb, sb | 0x8000)).astype(np.uint16) if kind == 1 else
            np.where(sound == 0, 0, np.where(sound > 0, pairs[:, 1:2], pairs[:, 0:1])).astype(np.uint16))
    for i in (3, 4):
        assert np.array_equal(host[i].view(want.dtype), want), i
    assert (host[0] == 77).all() and (host[5] == 77).all()
    dd.close()
