"""The wide kernel's layout (32x32x16 MFMA fragments and the stage table),
decoded on the host back to W * expand(mask), and the bounds its launches rely
on, over odd channel counts, strides, paddings and fused pools."""
import os

import numpy as np
import pytest
import torch

from paper_2007_09835_amd import build, rt3d

LDS_FIXED = 4 * 128 * 144 + 2 * (128 * 8 + 256 * 4)


@pytest.fixture(scope="module", autouse=True)
def built():
    build.build(force=False)


def _wide(info):
    raw = bytes(info.plan)[104:128]
    a_off = int(np.frombuffer(raw[:8], np.uint64)[0])
    bt, bh, bw, c16 = raw[8:12]
    hwp, hpp = (int(v) for v in np.frombuffer(raw[12:16], np.uint16))
    return a_off, bt, bh, bw, c16, hwp, hpp


@pytest.mark.parametrize("case", [
    # c_in, c_out, thw, k, stride, pad, g, keep (None: dense), pool, n
    (16, 32, (4, 7, 9), (3, 3, 3), (1, 1, 1), (1, 1, 1), (4, 4), 9, (1, 1, 1), 1),
    (40, 72, (5, 7, 6), (3, 3, 3), (2, 2, 2), (1, 1, 1), (4, 4), None, (1, 1, 1), 2),
    (21, 13, (3, 9, 11), (3, 3, 3), (1, 1, 1), (1, 1, 1), (4, 4), 7, (1, 1, 1), 1),
    (460, 33, (6, 5, 5), (3, 1, 1), (2, 1, 1), (1, 0, 0), (4, 4), 2, (1, 1, 1), 1),
    (64, 130, (4, 8, 8), (1, 3, 3), (1, 2, 2), (0, 1, 1), (8, 4), 4, (1, 2, 2), 32),
    (96, 64, (4, 6, 16), (3, 3, 3), (1, 1, 1), (1, 1, 1), (16, 4), 27, (2, 2, 2), 4),
    (48, 32, (3, 6, 6), (1, 1, 1), (1, 1, 1), (0, 0, 0), (4, 4), 0, (1, 1, 1), 1),
    (17, 64, (2, 20, 20), (1, 7, 7), (1, 1, 1), (0, 3, 3), (4, 4), 20, (1, 1, 1), 1),
])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_wide_layout_decodes_to_masked_weights(dt, case, monkeypatch):
    monkeypatch.delenv("RT3D_TUNE", raising=False)
    c_in, c_out, thw, k, stride, pad, g, keep, pool, n = case
    rng = np.random.default_rng(c_in * 1000 + c_out)
    w = torch.from_numpy(rng.standard_normal((c_out, c_in, *k)).astype(np.float32))
    w = w.to(torch.bfloat16 if dt == "bf16" else torch.float16)
    bits = w.view(torch.uint16).numpy().reshape(c_out, c_in, -1)
    ks = bits.shape[2]
    desc = rt3d.make_desc(n, c_in, c_out, thw, k, stride, pad, g, dt, pool=pool)
    if keep is None:
        blob, info = rt3d.rt3d_dense_pack(desc, w)
        want = bits
    else:
        mask = np.zeros((-(-c_out // g[0]), -(-c_in // g[1]), ks), np.uint8)
        for p in range(mask.shape[0]):
            for q in range(mask.shape[1]):
                mask[p, q, rng.choice(ks, keep, replace=False)] = 1
        blob, info = rt3d.rt3d_kgs_pack(desc, w, mask)
        full = np.repeat(np.repeat(mask, g[0], 0), g[1], 1)[:c_out, :c_in]
        want = np.where(full == 1, bits, 0)
    a_off, bt, bh, bw, c16, hwp, hpp = _wide(info)
    assert a_off > 0 and c16 > 0
    # weights: [32-filter row][step][lane][8], steps over chunks, positions, slices
    c16_total, frags = -(-c_in // 16), -(-(-(-c_out // 32)) // 2) * 2
    stot = ks * c16_total
    a = np.frombuffer(blob[a_off:a_off + frags * stot * 1024].tobytes(), np.uint16)
    a = a.reshape(frags, stot, 64, 8)
    got = np.zeros((frags * 32, c16_total * 16, ks), np.uint16)
    lane = np.arange(64)
    s = 0
    for c0 in range(0, c16_total, c16):
        for pos in range(ks):
            for sl in range(c0, min(c16_total, c0 + c16)):
                for e in range(8):
                    m = (np.arange(frags)[:, None] * 32 + (lane & 31)[None, :]).ravel()
                    c = np.tile(sl * 16 + 8 * (lane >> 5) + e, frags)
                    got[m, c, pos] = a[:, s, :, e].ravel()
                s += 1
    assert s == stot
    assert got[:c_out, :c_in].tobytes() == np.ascontiguousarray(want).astype(np.uint16).tobytes()
    assert not got[c_out:].any() and not got[:, c_in:].any()
    # geometry: the brick holds whole pooling windows and at most 128 slots, and
    # every voxel's every kernel tap lies inside a halo buffer
    assert bt % pool[0] == 0 and bh % pool[1] == 0 and bw % pool[2] == 0 and bt * bh * bw <= 128
    ht, hh, hw = ((b - 1) * st + kk for b, st, kk in zip((bt, bh, bw), stride, k))
    assert hwp >= hw and hpp >= hh * hwp
    row, rows = c16 * 32 + 16, ht * hpp
    assert 2 * rows * row + LDS_FIXED <= 160 * 1024 and rows * (row // 16) <= 11 * 256
    assert -(-ks * c16 // 4) <= 128
    last = ((ht - 1) * hpp + (hh - 1) * hwp + hw - 1) * row + c16 * 32
    assert last <= rows * row
    # stage table: every halo voxel's every piece exactly once, the rest padding
    tab_off = a_off + frags * stot * 1024
    tab = np.frombuffer(blob[tab_off:tab_off + rows * (row // 16) * 4].tobytes(), np.uint32)
    real = tab != 0xFFFFFFFF
    t, h, wv, p = (tab & 511)[real], ((tab >> 9) & 511)[real], ((tab >> 18) & 511)[real], (tab >> 27)[real]
    slot = np.nonzero(real)[0]
    assert np.array_equal(slot, ((t.astype(np.int64) * hpp + h * hwp + wv) * (2 * c16 + 1) + p))
    assert real.sum() == ht * hh * hw * 2 * c16
    assert t.max() < ht and h.max() < hh and wv.max() < hw and p.max() < 2 * c16


def test_wide_layout_is_left_out(monkeypatch):
    """fp32, 5 to 15 input channels and a tuning switch that names an
    item-kernel layout keep a blob without it."""
    def a_off(c_in, dt, tune=None, thw=(4, 8, 8)):
        if tune:
            monkeypatch.setenv("RT3D_TUNE", tune)
        else:
            monkeypatch.delenv("RT3D_TUNE", raising=False)
        d = rt3d.make_desc(1, c_in, 32, thw, dtype=dt)
        w = torch.zeros((32, c_in, 3, 3, 3), dtype={"f32": torch.float32, "bf16": torch.bfloat16}[dt])
        return _wide(rt3d.rt3d_dense_pack(d, w)[1])[0]
    assert a_off(32, "bf16") > 0
    assert a_off(32, "f32") == 0
    assert a_off(12, "bf16") == 0
    assert a_off(3, "bf16", thw=(4, 8, 44)) > 0       # the RGB kernel's weights
    assert a_off(3, "bf16", "small_mfw=1", thw=(4, 8, 44)) == 0
    for tune in ("wide=0", "slots=64", "dense_mfw=1", "cc=32"):
        assert a_off(32, "bf16", tune) == 0


@pytest.mark.parametrize("c_in,c_out,thw,dtype", [(64, 64, (4, 14, 14), "bf16"), (64, 64, (4, 14, 14), "f16")])
def test_small_layers_stay_in_one_launch(c_in, c_out, thw, dtype):
    """A layer that one item-kernel launch serves is not split for a gain
    smaller than a second launch: it asks for no workspace."""
    d = rt3d.make_desc(1, c_in, c_out, thw, (3, 3, 3), (1, 1, 1), (1, 1, 1), (4, 4), dtype)
    w = torch.zeros((c_out, c_in, 3, 3, 3), dtype={"bf16": torch.bfloat16, "f16": torch.float16}[dtype])
    _, info = rt3d.rt3d_dense_pack(d, w)
    assert _wide(info)[0] > 0                      # the layout is there
    assert rt3d.rt3d_conv3d_workspace_size(d, info) == 0
