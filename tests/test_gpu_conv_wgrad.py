"""The weight gradient of the 3x3x3 convolution at the edges of its work split: one voxel,
rows that are no whole number of 4-voxel pieces, several runs per plane, rows longer than a
run (x staged as three row ranges), several z segments, and chunks of several samples.

The operands are exact in BF16 and the sums accumulate in FP32: with n products of magnitude
at most 1 per entry, the error against FP64 is below n 2^-24 (worst case); 1e-4 of the largest
entry covers it for these sizes, since random sums of n such products are of order sqrt(n) / 3
and their rounding errors add as sqrt(n) too."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import unet_oracle as U

pytestmark = pytest.mark.gpu

CASES = [  # B, (D, H, W), cin, cout
    (1, (1, 1, 1), 16, 16),
    (1, (2, 3, 5), 8, 32),
    (1, (3, 4, 6), 24, 16),
    (2, (3, 33, 21), 16, 32),
    (1, (5, 19, 68), 48, 16),
    (1, (2, 3, 401), 16, 16),
    (1, (1, 2, 1030), 32, 48),
    (1, (40, 6, 9), 16, 96),
    (140, (1, 2, 3), 64, 64),
]


@pytest.mark.parametrize("B,grid,cin,cout", CASES)
def test_weight_gradient_split(B, grid, cin, cout):
    import torch
    import paper_2308_09839_amd as q1
    print(f"\n[wgrad] B={B} grid={grid} cin={cin} cout={cout}", flush=True)

    def make(c, seed):
        n = B * int(np.prod(grid)) * c
        a = -1 + 2 * si.uniform(seed, si.STREAM_X, np.arange(n, dtype=np.uint64))
        return torch.from_numpy(a.reshape((B,) + grid + (c,)).astype(np.float32)).to(torch.bfloat16)

    x, gy = make(cin, 41), make(cout, 42)
    gw, gb = q1.q1_conv3d_backward_weight(x.cuda(), cin, gy.cuda(), cout)
    gw2, gb2 = q1.q1_conv3d_backward_weight(x.cuda(), cin, gy.cuda(), cout)
    assert torch.equal(gw, gw2) and torch.equal(gb, gb2)
    rw, rb = U.conv3d_backward_weight(x.double().numpy(), gy.double().numpy())
    for got, ref in ((gw, rw), (gb, rb)):
        err = np.max(np.abs(got.double().cpu().numpy() - ref)) / np.max(np.abs(ref))
        print(f"  max err {err:.2e}", flush=True)
        assert err < 1e-4
