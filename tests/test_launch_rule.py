"""The launch a forward call makes, as rt3d_conv3d_launch_info reports it: what
a blob holds for the wide kernel changes nothing for the calls that stay on
the item kernel.  Host only (the planner's figures for 256 compute units)."""
import random

import pytest
import torch

from paper_2007_09835_amd import build, rt3d


@pytest.fixture(scope="module", autouse=True)
def built():
    build.build(force=False)


@pytest.fixture(autouse=True)
def no_tune(monkeypatch):
    monkeypatch.delenv("RT3D_TUNE", raising=False)


def pack(c_in, c_out, thw, k, n=1, dtype="bf16", **kw):
    d = rt3d.make_desc(n, c_in, c_out, thw, k, pad=tuple(v // 2 for v in k), dtype=dtype, **kw)
    w = torch.zeros((c_out, c_in, *k), dtype=torch.bfloat16 if dtype == "bf16" else torch.float16)
    return d, rt3d.rt3d_dense_pack(d, w)[1]


def shapes(count, seed):
    rng = random.Random(seed)
    fixed = [(576, 256, (4, 14, 14), (3, 1, 1), 1), (128, 288, (8, 28, 28), (1, 3, 3), 1)]
    for _ in range(count):
        k = rng.choice([(3, 3, 3), (1, 3, 3), (3, 1, 1), (1, 1, 1)])
        s = rng.choice([7, 14, 28])
        fixed.append((rng.randint(2, 40) * 8, rng.randint(2, 40) * 8, (rng.randint(2, 8), s, s), k,
                      rng.choice([1, 1, 2, 4, 8])))
    return fixed


def test_item_launch_does_not_depend_on_the_wide_section(monkeypatch):
    """With a pitch that the wide kernel cannot read, the launch is the one of
    a blob without the wide section, its workgroup order included."""
    for c_in, c_out, thw, k, n in shapes(40, 1):
        d, both = pack(c_in, c_out, thw, k, n)
        monkeypatch.setenv("RT3D_TUNE", "wide=0")
        _, alone = pack(c_in, c_out, thw, k, n)
        monkeypatch.delenv("RT3D_TUNE")
        d.x_c_total = c_in + 4
        assert both.packed_bytes > alone.packed_bytes
        a, b = (bytes(rt3d.rt3d_conv3d_launch_info(d, i)) for i in (both, alone))
        assert a == b, (c_in, c_out, thw, k, n)
        assert rt3d.rt3d_conv3d_launch_info(d, both).kernel == rt3d.KERNELS.index("item")


@pytest.mark.parametrize("c_in,c_out,thw,k", [(576, 256, (4, 14, 14), (3, 1, 1)), (216, 248, (5, 7, 7), (3, 1, 1)),
                                              (296, 80, (2, 28, 28), (1, 3, 3))])
def test_without_workspace_the_kernels_are_compared_as_they_run(c_in, c_out, thw, k):
    """A split item launch is no rival where there is no workspace for it: the
    item kernel would walk every channel chunk in one workgroup, which the wide
    kernel's four parts of the reduction beat."""
    d, info = pack(c_in, c_out, thw, k)
    split, whole = rt3d.rt3d_conv3d_launch_info(d, info), rt3d.rt3d_conv3d_launch_info(d, info, 0)
    assert split.kernel == rt3d.KERNELS.index("item") and split.splits > 1
    assert whole.kernel == rt3d.KERNELS.index("wide")
    assert whole.splits == 1 and whole.workspace_bytes == 0


def test_workspace_covers_every_input_pitch():
    """A layer's workspace is asked for before its input's pitch is known.
    Ragged channel counts run on the wide kernel only where the pitch is padded
    to 8 channels: the size without a pitch covers that launch too."""
    rng = random.Random(3)
    cases = [(500, 64, (2, 14, 14), (1, 3, 3), 4, 1)]
    for c_in, c_out, thw, k, n in shapes(60, 4):
        cases.append((c_in - rng.randint(1, 7) if c_in > 24 else 21, c_out, thw, k, n, rng.choice([1, n])))
    grew = 0
    for c_in, c_out, thw, k, n, run_n in cases:
        d, info = pack(c_in, c_out, thw, k, n)
        d.n = run_n
        asked = rt3d.rt3d_conv3d_workspace_size(d, info)
        for pitch, off in ((0, 0), (-(-c_in // 8) * 8, 0), (-(-c_in // 8) * 8 + 16, 8), (c_in + 1, 1)):
            d.x_c_total, d.x_c_off = pitch, off
            want = rt3d.rt3d_conv3d_launch_info(d, info)
            got = rt3d.rt3d_conv3d_launch_info(d, info, asked)
            assert bytes(want) == bytes(got), (c_in, c_out, thw, k, n, run_n, pitch)
            grew += want.kernel == rt3d.KERNELS.index("wide") and want.splits > 1
    assert grew > 5   # (split wide launches were among them)


def test_tuning_switches_do_not_bend_the_search(monkeypatch):
    """The search passes over shapes that its bound rules out: a call that a
    switch forces onto the wide kernel takes the shape of the free search."""
    wide = rt3d.KERNELS.index("wide")
    seen = 0
    for c_in, c_out, thw, k, n in shapes(60, 5):
        d, info = pack(c_in, c_out, thw, k, n)
        for ws in (0, 1 << 20, 2 ** 64 - 1):
            free = rt3d.rt3d_conv3d_launch_info(d, info, ws)
            monkeypatch.setenv("RT3D_TUNE", "wide=1")
            forced = rt3d.rt3d_conv3d_launch_info(d, info, ws)
            monkeypatch.delenv("RT3D_TUNE")
            assert forced.kernel == wide
            if free.kernel == wide:
                assert bytes(free) == bytes(forced), (c_in, c_out, thw, k, n, ws)
                seen += 1
    assert seen > 20


@pytest.mark.parametrize("c_in,c_out,thw,k", [(208, 224, (2, 14, 14), (1, 1, 1)), (224, 256, (4, 7, 7), (1, 1, 1)),
                                              (256, 16, (5, 7, 7), (1, 1, 1)), (336, 96, (2, 7, 7), (1, 1, 1))])
def test_smallest_pointwise_layers_stay_on_the_item_kernel(c_in, c_out, thw, k):
    """Calls of 8-9 us, where the wide kernel starts later than its model has
    it (7.5-8.9 us on the item kernel, 8.3-9.5 on the wide one)."""
    d, info = pack(c_in, c_out, thw, k)
    assert rt3d.rt3d_conv3d_launch_info(d, info).kernel == rt3d.KERNELS.index("item")


@pytest.mark.parametrize("thw,k,stride,pad,n,kernel", [
    ((8, 28, 28), (1, 7, 7), (1, 2, 2), (0, 3, 3), 1, "small"),    # 8 bricks of 14 steps
    ((16, 224, 224), (1, 7, 7), (1, 2, 2), (0, 3, 3), 1, "rgb"),
    ((8, 56, 12), (3, 3, 3), (1, 1, 1), (1, 1, 1), 1, "small"),    # 28 bricks of 9 steps
    ((4, 56, 36), (3, 3, 3), (1, 1, 1), (1, 1, 1), 2, "rgb"),      # 56
    ((3, 4, 12), (1, 3, 3), (1, 1, 1), (0, 1, 1), 1, "rgb")])
def test_few_bricks_of_many_steps_stay_on_the_small_channel_kernel(thw, k, stride, pad, n, kernel, monkeypatch):
    d = rt3d.make_desc(n, 3, 64, thw, k, stride, pad, dtype="bf16")
    _, info = rt3d.rt3d_dense_pack(d, torch.zeros((64, 3, *k), dtype=torch.bfloat16))
    assert rt3d.KERNELS[rt3d.rt3d_conv3d_launch_info(d, info).kernel] == kernel
    monkeypatch.setenv("RT3D_TUNE", "wide=1")
    assert rt3d.KERNELS[rt3d.rt3d_conv3d_launch_info(d, info).kernel] == "rgb"


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("c_in", [3, 12, 64, 512])
def test_an_empty_batch_needs_no_workspace(c_in, dtype):
    w = torch.zeros((64, c_in, 3, 3, 3), dtype={"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype])
    d = rt3d.make_desc(1, c_in, 64, (4, 8, 8), dtype=dtype)
    _, info = rt3d.rt3d_dense_pack(d, w)
    d.n = 0
    assert rt3d.rt3d_conv3d_workspace_size(d, info) == 0
    assert rt3d.rt3d_conv3d_launch_info(d, info).workspace_bytes == 0
