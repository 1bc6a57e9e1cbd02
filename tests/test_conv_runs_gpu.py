"""3x3 layers whose patches are staged in runs of four pixels (float32, bfloat16 with tiles of 32 filters) or in pairs that begin at even
elements (bfloat16), where the loads are moved or cut: planes of a few pixels, rows shorter than a run, odd rows in even planes, odd
planes, channels that end inside a group, activations that begin at an odd element.  Exact arithmetic against the oracle (activations
in {-1, 0, +1}, alphas powers of two)."""
import numpy as np
import pytest
import torch

from oracle import tbn_oracle as orc
from paper_2407_12075_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, C, H, W, O, stride, pad, k
CASES = [
    (2, 16, 2, 2, 64, 1, 1, 2),       # a plane of one run
    (2, 17, 1, 4, 64, 1, 1, 2),
    (3, 24, 9, 1, 34, 1, 1, 1),       # rows of one pixel (float32)
    (2, 40, 5, 3, 34, 1, 1, 1),       # rows shorter than a run, an odd plane
    (1, 31, 10, 7, 66, 1, 1, 2),      # odd rows in an even plane; channels end inside a group
    (2, 16, 14, 13, 34, 1, 0, 1),     # no halo
    (1, 20, 7, 31, 40, 1, 2, 1),      # two pixels of halo, an odd plane
    (2, 64, 14, 14, 64, 1, 1, 4),     # a patch row is a whole number of runs: its LDS rows are one pixel longer
    (1, 33, 12, 30, 20, 1, 1, 2),     # tiles of 16 filters in bfloat16
    (2, 48, 9, 11, 70, 2, 1, 1),      # stride 2
    (1, 4200, 3, 5, 18, 1, 1, 2),     # float32: all bits of small activations
]


@pytest.fixture(scope="module")
def tbn():
    from paper_2407_12075_amd import tbn as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("dtype,off", [("f32", 0), ("f32", 1), ("bf16", 0), ("bf16", 1), ("bf16", 2)])
@pytest.mark.parametrize("N,C,H,W,O,stride,pad,k", CASES)
def test_staged_loads_exact(tbn, N, C, H, W, O, stride, pad, k, dtype, off):
    rng = np.random.default_rng(C * 1000 + O + off)
    p = O * C * 9 // k
    tile = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha = np.asarray([2.0 ** ((i % 5) - 2) for i in range(k)], dtype=np.float32)
    x = (rng.integers(-1, 2, size=(N, C, H, W)) * (rng.random((N, C, H, W)) < min(1.0, 1500 / (9 * C)))).astype(np.float32)
    ref = orc.conv2d_forward(x, tile, alpha, O, 3, 3, k, stride=(stride, stride), pad=(pad, pad)).astype(np.float32)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    if dtype == "bf16":
        ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    held = torch.full((x.size + off,), float("nan"), device="cuda", dtype=dt)   # `off` elements behind the allocation's first
    xd = held[off:].view(N, C, H, W).copy_(torch.from_numpy(x))
    y = tbn.tbn_conv2d_forward(xd, torch.from_numpy(tile.view(np.int32)).cuda(), torch.from_numpy(alpha).cuda(), O, 3, 3, k,
                               stride=(stride, stride), pad=(pad, pad))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(y.float().cpu().numpy(), ref)
