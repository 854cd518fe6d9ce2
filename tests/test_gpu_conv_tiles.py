"""The 3x3x3 convolution at the edges of its tiles (8 x 8 x 4 voxels): one voxel, one past a
tile in each direction, partial tiles at every face, several channel chunks, and z marches of
more than one tile per workgroup with uneven segments.

Operands are exact in BF16; K <= 27 * 96 products accumulate in FP32, so the error against FP64
is of order sqrt(K) 2^-24 of the largest entry: 1e-4 leaves a factor above ten."""
import numpy as np
import pytest

import seeded_inputs as si
from oracle import unet_oracle as U

pytestmark = pytest.mark.gpu

CASES = [  # B, (D, H, W), cin, cout
    (1, (1, 1, 1), 8, 16),
    (1, (5, 9, 17), 16, 16),
    (2, (4, 8, 8), 48, 32),
    (1, (9, 7, 33), 96, 16),
    (64, (12, 16, 10), 16, 96),
    (50, (13, 9, 12), 32, 64),
]


def make(shape, seed):
    import torch
    a = -1 + 2 * si.uniform(seed, si.STREAM_X, np.arange(int(np.prod(shape)), dtype=np.uint64))
    return torch.from_numpy(a.reshape(shape).astype(np.float32)).to(torch.bfloat16)


def close(got, ref):
    err = np.max(np.abs(got.double().cpu().numpy() - ref)) / np.max(np.abs(ref))
    print(f"  max err {err:.2e}", flush=True)
    assert err < 1e-4


@pytest.mark.parametrize("B,grid,cin,cout", CASES)
def test_forward_and_adjoint_tiles(B, grid, cin, cout):
    import paper_2308_09839_amd as q1
    print(f"\n[conv] B={B} grid={grid} cin={cin} cout={cout}", flush=True)
    x, w = make((B,) + grid + (cin,), 51), make((27, cin, cout), 52)
    bias = make((cout + 1,), 53).float().cuda()[1:]  # 4-byte aligned only
    y = q1.q1_conv3d_forward(x.cuda(), cin, w.float().cuda(), cout, bias=bias)
    close(y, U.conv3d(x.double().numpy(), w.double().numpy(), bias.double().cpu().numpy()))
    if cin >= 16:
        gy = make((B,) + grid + (cout,), 54)
        gx = q1.q1_conv3d_backward_data(gy.cuda(), cout, w.float().cuda(), cin)
        close(gx, U.conv3d_backward_data(gy.double().numpy(), w.double().numpy()))
