"""The unit kernel of the penalty pass (KGS scope, four-channel groups of 4, 8
or 16 filters) at the edges of its rule, against the float64 oracle: short
last filter and channel groups, one to 343 positions, block widths of 64, 128
and 256 threads and units past one pass, both norms, in place.

Tolerances are those of the pass: 32-bit sums of at most 64 terms agree to
1e-5 relative L2 (64 * 2^-24 = 4e-6), proximal outputs to their type.
"""
import numpy as np
import pytest
import torch

from paper_2007_09835_amd import rt3d, synth
from test_gpu_reweight import check, run_gpu, weights

pytestmark = pytest.mark.gpu

CASES = [
    # c_out, c_in, k, g, dtype, norm: what it reaches
    (1, 1, (1, 1, 1), (4, 4), "f32", 2),        # one unit, one weight
    (7, 5, (3, 3, 3), (4, 4), "f32", 1),        # short row and channel groups, 64 threads
    (19, 9, (1, 3, 3), (8, 4), "bf16", 2),      # 8 filters
    (37, 30, (3, 1, 1), (16, 4), "f16", 1),     # 16 filters, last group of 5
    (16, 4, (7, 7, 7), (8, 4), "f32", 2),       # 343 units: a second pass of 256 threads
    (8, 8, (5, 5, 5), (8, 4), "bf16", 1),       # 125 units: 128 threads
    (512, 510, (3, 3, 3), (4, 4), "f32", 2),    # eight channel groups a block, the last one short
    (512, 512, (1, 3, 3), (4, 4), "bf16", 2),   # 72 units: 128 threads
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}k{''.join(map(str, c[2]))}g{c[3][0]}{c[4]}l{c[5]}"
                                             for c in CASES])
def test_unit_kernel_matches_oracle(case):
    c_out, c_in, k, g, dtype, norm = case
    print("unit kernel case", case, flush=True)
    desc = rt3d.make_group_desc(c_out, c_in, k, g, dtype, norm, 0)
    w_dev, w64 = weights("unit%dx%d" % (c_out, c_in), c_out, c_in, k, g, dtype)
    rng = synth.rng_for("reweight-unit", c_out, c_in)
    units = rt3d.rt3d_group_units(desc)
    pen = rng.uniform(0.5, 20.0, units).astype(np.float32).astype(np.float64)
    grad0 = rng.standard_normal(w64.shape).astype(np.float32)
    ushape = (-(-c_out // g[0]), -(-c_in // g[1]), k[0] * k[1] * k[2])
    args = dict(lam=0.02, eps=1e-4, tau=0.5, step=0.5, grad0=grad0)
    got = run_gpu(desc, w_dev, pen, **args)
    check(desc, w64, got, pen.reshape(ushape), dtype=dtype, **args)
    again = run_gpu(desc, w_dev, pen, in_place=True, **args)
    for key in got:
        assert np.array_equal(got[key], again[key]), key
