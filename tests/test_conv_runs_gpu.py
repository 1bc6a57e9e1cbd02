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

# N, C, H, W, O, stride, pad, k, and how float32 and bfloat16 patches are staged ("block": another kernel takes the layer)
CASES = [
    (2, 16, 2, 2, 64, 1, 1, 2, "block", "even-runs"),       # a plane of one run
    (16, 16, 2, 2, 256, 1, 1, 1, "runs", "even-runs"),
    (2, 17, 1, 4, 64, 1, 1, 2, "block", "even-runs"),
    (24, 17, 1, 4, 64, 1, 1, 4, "runs", "even-pairs"),
    (3, 24, 9, 1, 34, 1, 1, 1, "block", "block"),
    (24, 24, 9, 1, 34, 1, 1, 2, "runs", "block"),           # rows of one pixel (float32)
    (2, 40, 5, 3, 34, 1, 1, 1, "block", "runs"),            # rows shorter than a run, an odd plane
    (56, 40, 5, 3, 34, 1, 1, 1, "runs", "runs"),
    (1, 31, 10, 7, 66, 1, 1, 2, "block", "even-pairs"),     # odd rows in an even plane; channels end inside a group
    (60, 31, 10, 5, 66, 1, 1, 2, "runs", "even-runs"),
    (60, 31, 5, 10, 66, 1, 1, 1, "runs", "even-runs"),      # the patch's last row is one run and three pixels long
    (2, 16, 14, 13, 34, 1, 0, 1, "block", "even-runs"),     # no halo
    (20, 16, 14, 13, 34, 1, 0, 1, "runs", "even-runs"),
    (1, 20, 7, 31, 40, 1, 2, 1, "block", "runs"),           # two pixels of halo, an odd plane
    (8, 25, 7, 31, 40, 1, 2, 1, "runs", "runs"),            # one channel behind the first group
    (2, 64, 14, 14, 64, 1, 1, 4, "runs", "even-pairs"),     # a patch row is a whole number of runs: its LDS rows are one pixel longer
    (1, 33, 12, 30, 20, 1, 1, 2, "block", "even-pairs"),    # tiles of 16 filters in bfloat16
    (1, 33, 12, 30, 20, 1, 1, 4, "runs", "even-pairs"),
    (9, 47, 17, 18, 260, 1, 1, 2, "runs", "even-runs"),     # three chunks, the last one short of a channel
    (60, 12, 6, 9, 66, 1, 1, 2, "block", "even-runs"),      # the only chunk ends inside its second group
    (128, 17, 16, 16, 64, 1, 1, 1, "runs", "even-runs"),    # two filter tiles per wave, a last chunk of one channel
    (2, 48, 9, 11, 70, 2, 1, 1, "block", "pairs"),          # stride 2
    (36, 24, 8, 8, 64, 2, 1, 4, "runs", "even-pairs"),
    (1, 4200, 3, 5, 18, 1, 1, 2, "runs", "pairs"),          # float32: all bits of small activations
    (1, 4201, 3, 5, 18, 1, 1, 2, "runs", "pairs"),
]


@pytest.fixture(scope="module")
def tbn():
    from paper_2407_12075_amd import tbn as binding
    binding.lib()
    return binding


def _check_staging(tbn, layer, dtype, want):
    N, C, H, W, O, stride, pad, k = layer
    name = tbn.tbn_conv2d_forward_kernel(torch.float32 if dtype == "f32" else torch.bfloat16, N, C, H, W, O, 3, 3, k, (stride, stride), (pad, pad), k)
    assert name == want if want == "block" else f" staged={want}" in name and name.startswith("wave "), name


@pytest.mark.parametrize("dtype,off", [("f32", 0), ("f32", 1), ("bf16", 0), ("bf16", 1), ("bf16", 2)])
@pytest.mark.parametrize("N,C,H,W,O,stride,pad,k,f32,bf16", CASES)
def test_staged_loads_exact(tbn, N, C, H, W, O, stride, pad, k, f32, bf16, dtype, off):
    _check_staging(tbn, (N, C, H, W, O, stride, pad, k), dtype, f32 if dtype == "f32" else bf16)
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
