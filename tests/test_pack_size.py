"""The size a pack is asked for, worked out without building the operand
streams, is the size of the blob: every kernel layout, dense and KGS."""
import numpy as np
import pytest
import torch

from paper_2007_09835_amd import build, rt3d

DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


@pytest.mark.parametrize("tune", [None, "kgs_map=1", "kgs_map=2", "kgs_f32=0", "kgs_f32=1", "wide=0"])
@pytest.mark.parametrize("c_in,c_out,thw,k,g,dt", [
    (3, 20, (4, 8, 44), (3, 3, 3), (4, 4), "bf16"), (3, 64, (4, 9, 9), (1, 7, 7), (4, 4), "f16"),
    (12, 32, (4, 8, 8), (3, 3, 3), (4, 4), "bf16"), (21, 37, (3, 7, 6), (3, 1, 1), (8, 4), "f16"),
    (64, 96, (4, 8, 8), (3, 3, 3), (4, 4), "bf16"), (48, 130, (2, 9, 9), (1, 1, 1), (16, 16), "bf16"),
    (40, 72, (3, 6, 6), (3, 3, 3), (4, 4), "f32")])
def test_pack_size_is_the_blob_s(c_in, c_out, thw, k, g, dt, tune, monkeypatch):
    build.build(force=False)
    if tune is None:
        monkeypatch.delenv("RT3D_TUNE", raising=False)
    else:
        monkeypatch.setenv("RT3D_TUNE", tune)
    rng = np.random.default_rng(c_in)
    d = rt3d.make_desc(2, c_in, c_out, thw, k, pad=tuple(v // 2 for v in k), g=g, dtype=dt)
    w = torch.from_numpy(rng.standard_normal((c_out, c_in, *k)).astype(np.float32)).to(DT[dt])
    mask = (rng.random((-(-c_out // g[0]), -(-c_in // g[1]), k[0] * k[1] * k[2])) < 0.4).astype(np.uint8)
    assert rt3d.rt3d_dense_pack_size(d) == rt3d.rt3d_dense_pack(d, w)[1].packed_bytes
    assert rt3d.rt3d_kgs_pack_size(d, mask) == rt3d.rt3d_kgs_pack(d, w, mask)[1].packed_bytes
