"""Max-pools large enough for the kernel that computes a run of outputs along
w per thread: against the same pool one clip at a time (a thread per output),
bit for bit, with infinities, the type's lowest value and NaN among the
inputs, and against torch where there is no NaN."""
import pytest
import torch

from paper_2007_09835_amd import build, layers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def built():
    build.build(force=False)


@pytest.mark.parametrize("n", [12, 56])           # runs of 4 and of 7
@pytest.mark.parametrize("w", [28, 30, 31, 33])   # remainders of both
@pytest.mark.parametrize("k,stride,pad", [((3, 3, 3), (1, 1, 1), (1, 1, 1)),
                                          ((3, 3, 3), (2, 2, 2), (1, 1, 1)),
                                          ((1, 3, 3), (1, 2, 2), (0, 1, 1)),
                                          ((1, 3, 3), (1, 1, 1), (0, 0, 0))])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_pool_runs(dtype, k, stride, pad, w, n):
    g = torch.Generator().manual_seed(w * 100 + n)
    c = 64 if dtype != "f32" else 32
    x = torch.randn((n, 4, 33, w, c), generator=g).to(layers.TORCH_DTYPES[dtype])
    flat = x.view(-1)
    special = torch.randint(0, flat.numel(), (flat.numel() // 50,), generator=g)
    flat[special[0::3]] = float("inf")
    flat[special[1::3]] = float("-inf")
    flat[special[2::3]] = torch.finfo(x.dtype).min
    xd = x.cuda()
    y = layers.maxpool3d(xd, k, stride, dtype, pad=pad)
    ref = torch.nn.functional.max_pool3d(x.float().permute(0, 4, 1, 2, 3), k, stride, pad)
    assert torch.equal(y.float().cpu().permute(0, 4, 1, 2, 3), ref)
    flat[special[0::4]] = float("nan")
    xd = x.cuda()
    y = layers.maxpool3d(xd, k, stride, dtype, pad=pad)
    bits = {2: torch.int16, 4: torch.int32}[y.element_size()]
    for i in (0, n // 2, n - 1):
        one = layers.maxpool3d(xd[i:i + 1].contiguous(), k, stride, dtype, pad=pad)
        a, b = y[i].view(bits), one[0].view(bits)
        same = (a == b) | (torch.isnan(y[i].float()) & torch.isnan(one[0].float()))
        assert bool(same.all())
