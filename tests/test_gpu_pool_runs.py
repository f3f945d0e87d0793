"""Max-pools large enough for the kernel that computes a run of outputs along
w per thread, runs of 4 and of 7 at either stride along w: against the same
pool one clip at a time (a thread per output), bit for bit but for the sign of
a zero, with infinities, the type's lowest value, zeros of both signs and NaN
among the inputs, and against torch where there is no NaN."""
import pytest
import torch

from paper_2007_09835_amd import build, layers

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def built():
    build.build(force=False)


def run_length(k, stride, n, out, vectors):
    """The library's rule: outputs per thread along w (0: a thread per output)."""
    if k[0] not in (1, 3) or k[1:] != (3, 3) or stride[2] not in (1, 2):
        return 0
    lines = n * out[0] * out[1] * vectors
    least = 98304 if k[0] == 1 and stride[2] == 2 else 65536
    for r in (7, 4):
        if lines * -(-out[2] // r) >= (262144 if r == 7 else least):
            return r
    return 0


WINDOWS = [((3, 3, 3), (1, 1, 1), (1, 1, 1)), ((3, 3, 3), (1, 1, 2), (1, 1, 1)),
           ((1, 3, 3), (1, 1, 2), (0, 1, 1)), ((1, 3, 3), (1, 1, 1), (0, 0, 0))]
# Runs of 7 of these take 120 million inputs; the stride along w is what a run sees.
STRIDED = [((3, 3, 3), (2, 2, 2), (1, 1, 1)), ((1, 3, 3), (1, 2, 2), (0, 1, 1))]


@pytest.mark.parametrize("w", [28, 30, 31, 33])   # remainders of both
@pytest.mark.parametrize("k,stride,pad,run", [(*c, r) for r in (4, 7) for c in WINDOWS] + [(*c, 4) for c in STRIDED])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_pool_runs(dtype, k, stride, pad, w, run):
    c = 64 if dtype != "f32" else 32
    t, h = 4, 33
    out = tuple((d + 2 * p - kk) // s + 1 for d, p, kk, s in zip((t, h, w), pad, k, stride))
    n = next(i for i in range(1, 4096) if run_length(k, stride, i, out, 8) == run)
    assert run_length(k, stride, 1, out, 8) == 0
    g = torch.Generator(device="cuda").manual_seed(w * 100 + run)
    x = torch.randn((n, t, h, w, c), generator=g, device="cuda").to(layers.TORCH_DTYPES[dtype])
    flat = x.view(-1)
    special = torch.randint(0, flat.numel(), (flat.numel() // 50,), generator=g, device="cuda")
    flat[special[0::3]] = float("inf")
    flat[special[1::3]] = float("-inf")
    flat[special[2::3]] = torch.finfo(x.dtype).min
    x[:, :, 10:16, 8:16] = -0.0                      # windows of zeros of both signs
    x[:, 1::2, 11:16:2, 9:16:3] = 0.0
    y = layers.maxpool3d(x, k, stride, dtype, pad=pad)
    ref = torch.nn.functional.max_pool3d(x.float().permute(0, 4, 1, 2, 3), k, stride, pad)
    assert torch.equal(y.float().permute(0, 4, 1, 2, 3), ref)   # (zeros compare equal)
    flat[special[0::4]] = float("nan")
    y = layers.maxpool3d(x, k, stride, dtype, pad=pad)
    bits = {2: torch.int16, 4: torch.int32}[y.element_size()]
    for i in (0, n // 2, n - 1):
        one = layers.maxpool3d(x[i:i + 1].contiguous(), k, stride, dtype, pad=pad)[0]
        same = (y[i].view(bits) == one.view(bits)) | ((y[i] == 0) & (one == 0)) | (y[i].isnan() & one.isnan())
        assert bool(same.all())
