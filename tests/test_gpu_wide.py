"""The wide 16-bit kernel on every launch shape it has (one and two filter
rows per wave, one to four parts of the reduction, channel splits), at the
sizes where it can go wrong (each shape has over 128 filters, so that every
launch shape takes it): filters off the 32- and 4-filter grids, channel off the 16- and 8-channel grids (next to NaN channels), last chunks of
fewer steps than parts, bricks past the volume's edges, fused pools,
residuals, more tiles than workgroups.  Full comparison with the oracle,
every output within its own bound (harness.error_bound)."""
import numpy as np
import pytest
import torch

from harness import TOL, LayerCase, assert_within_bound, from_device_ndhwc, rel_l2, to_device_ndhwc
from paper_2007_09835_amd import build, rt3d, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def built():
    build.build(force=False)


SHAPES = {
    # n, c_in, c_out, thw, k, stride, pad, pool, residual, keep (None: dense)
    "edges": (1, 48, 136, (3, 9, 11), (3, 3, 3), (1, 1, 1), (1, 1, 1), (1, 1, 1), True, 9),
    "ragged": (1, 21, 133, (3, 7, 6), (3, 3, 3), (1, 1, 1), (1, 1, 1), (1, 1, 1), False, None),
    "half_slice": (2, 24, 160, (4, 6, 6), (1, 3, 3), (1, 2, 2), (0, 1, 1), (1, 1, 1), True, 4),
    "pool222": (2, 64, 144, (4, 10, 12), (3, 3, 3), (1, 1, 1), (1, 1, 1), (2, 2, 2), False, 9),
    "pool122_res": (1, 32, 131, (3, 8, 10), (3, 3, 3), (1, 1, 1), (1, 1, 1), (1, 2, 2), True, 13),
    "pointwise": (1, 144, 130, (2, 9, 9), (1, 1, 1), (1, 1, 1), (0, 0, 0), (1, 1, 1), False, None),
    "temporal": (1, 176, 192, (7, 5, 5), (3, 1, 1), (2, 1, 1), (1, 0, 0), (1, 1, 1), True, 2),
    # every halo column but the brick's own lies outside the clip in some wave
    "borders": (3, 40, 132, (2, 9, 9), (1, 3, 3), (1, 2, 2), (0, 1, 1), (1, 1, 1), False, 4),
    "many_tiles": (40, 16, 136, (4, 12, 12), (3, 3, 3), (1, 1, 1), (1, 1, 1), (1, 1, 1), False, 9),
}


def _case(name, dtype):
    n, c_in, c_out, thw, k, stride, pad, pool, res, keep = SHAPES[name]
    mask = None
    if keep is not None:
        mask = synth.kgs_mask(synth.rng_for("wide", name, "mask"), -(-c_out // 4), -(-c_in // 4),
                              k[0] * k[1] * k[2], keep)
    return LayerCase("wide-" + name, n, c_in, c_out, thw, k, stride, pad, dtype, mask, residual=res,
                     pool=pool)


def _run(case):
    """The layer on its input, widened to an 8-channel pitch whose extra
    channels are NaN when the channel count is ragged."""
    x = to_device_ndhwc(case.x_t)
    c_in = x.shape[-1]
    if c_in % 8:
        wide = torch.full((*x.shape[:-1], (c_in + 7) // 8 * 8 + 8), float("nan"), dtype=x.dtype, device=x.device)
        wide[..., 8:8 + c_in] = x
        res = None if case.res_t is None else to_device_ndhwc(case.res_t)
        return from_device_ndhwc(case.conv(wide, res, x_off=8))
    return case.run_gpu()


def _launch(case):
    """The launch that _run makes."""
    d = case.conv.desc_for(case.x_t.shape[0])
    if d.c_in % 8:
        d.x_c_total, d.x_c_off = (d.c_in + 7) // 8 * 8 + 8, 8
    return rt3d.rt3d_conv3d_launch_info(d, case.conv.info)


@pytest.mark.parametrize("tune", ["wide_fm=1,wide_wm=1", "wide_fm=1,wide_wm=2", "wide_fm=2,wide_wm=1",
                                  "wide_fm=2,wide_wm=2", "wide_fm=1,wide_wm=4", "wide_fm=2,wide_wm=4",
                                  "splits=2"])
@pytest.mark.parametrize("name", list(SHAPES))
def test_wide_launch_shapes(name, tune, monkeypatch):
    monkeypatch.setenv("RT3D_TUNE", "wide=1," + tune)
    dtype = "f16" if name in ("half_slice", "temporal") else "bf16"
    case = _case(name, dtype)
    shape = _launch(case)
    assert rt3d.KERNELS[shape.kernel] == "wide", (name, tune)
    for key, value in (kv.split("=") for kv in tune.split(",")):
        if key == "splits":   # (a layer of one channel chunk cannot split)
            chunks = -(-SHAPES[name][1] // shape.chunk)
            assert shape.splits == min(2, chunks) and (chunks > 1 or name == "many_tiles")
        else:
            assert {"wide_fm": shape.rows // 32, "wide_wm": shape.wm}[key] == int(value), (name, tune)
    got, ref = _run(case), case.oracle_full()
    err = rel_l2(got, ref)
    print(f"wide {name} {tune}: relL2={err:.3e}", flush=True)
    assert err <= TOL[dtype], (name, tune, err)
    assert_within_bound(got, ref, case.bound_full(ref), f"wide {name} {tune}")


def test_wide_and_item_kernels_take_the_same_blob(monkeypatch):
    """An input whose pitch is not a multiple of 8 channels runs on the item
    kernel, from the same blob, and both agree with the oracle."""
    monkeypatch.setenv("RT3D_TUNE", "wide=1")
    case = _case("edges", "bf16")
    ref = case.oracle_full()
    x = to_device_ndhwc(case.x_t)
    odd = torch.zeros((*x.shape[:-1], x.shape[-1] + 4), dtype=x.dtype, device=x.device)
    odd[..., :x.shape[-1]] = x
    res = to_device_ndhwc(case.res_t)
    for inp in (x, odd):
        got = from_device_ndhwc(case.conv(inp, res))
        assert rel_l2(got, ref) <= TOL["bf16"]
        assert_within_bound(got, ref, case.bound_full(ref), "wide/item")


@pytest.mark.parametrize("name", ["ragged", "edges", "pointwise"])
def test_wide_kernel_writes_its_channel_slice_only(name, monkeypatch):
    """A channel slice of a wider output, c_out on and off the 4-filter grid:
    the channels beside it stay as they are."""
    monkeypatch.setenv("RT3D_TUNE", "wide=1")
    case = _case(name, "bf16")
    assert rt3d.KERNELS[_launch(case).kernel] == "wide"
    x = to_device_ndhwc(case.x_t)
    if x.shape[-1] % 8:
        padded = torch.zeros((*x.shape[:-1], x.shape[-1] // 8 * 8 + 8), dtype=x.dtype, device=x.device)
        padded[..., :x.shape[-1]] = x
        x = padded
    res = None if case.res_t is None else to_device_ndhwc(case.res_t)
    y = case.conv(x, res)
    m = y.shape[-1]
    wide = torch.full((*y.shape[:-1], (m + 3) // 4 * 4 + 16), 7.0, dtype=y.dtype, device=y.device)
    case.conv(x, res, out=wide, c_off=8)
    assert torch.equal(wide[..., 8:8 + m], y)
    assert bool((wide[..., :8] == 7).all()) and bool((wide[..., 8 + m:] == 7).all())
