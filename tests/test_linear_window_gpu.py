"""The windowed form of the bfloat16 block kernel (row lengths in multiples of 8, tile starts inside rows) at the edges of its
blocks, rounds and tile pieces: exact arithmetic (activations in {-1, 0, +1}, alphas powers of two), so it has to equal the
oracle and the kernel with one thread per output bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tbn_oracle as orc
from paper_2407_12075_amd import workloads as wl

pytestmark = pytest.mark.gpu

# M, in, out, k, n_alpha
CASES = [
    (4000, 200, 1016, 1, 1),        # one pair of rounds, mostly padding; a last row block of 32, a last column block of 120
    (1200, 768, 3064, 3, 3),        # no padding; tile starts inside rows, two alphas there
    (1200, 264, 3064, 11, 1),       # windows that cross the tile's end, none repaired; eight elements in the second pair
    (6000, 280, 2560, 4, 4),        # tile of whole rows
    (16000, 1000, 1088, 1000, 1000),   # a tile start in nearly every row: alphas differ from column to column
    (1090, 744, 1600, 12, 12),      # an alpha per third of the distinct columns
    (2049, 3000, 3072, 9, 9),       # 136 blocks
    (12000, 2984, 2944, 4, 4),      # more blocks than CUs: stores under the next block
    (8192, 3000, 3072, 9, 9),       # two blocks per CU
    (8192, 3000, 3072, 9, 1),
]


@pytest.mark.parametrize("M,cin,cout,k,n_alpha", CASES)
def test_window_exact(M, cin, cout, k, n_alpha):
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, n_alpha) == "window"
    rng = np.random.default_rng(cin + k)
    p = cin * cout // k
    tile_ref = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile_ref[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha_ref = np.asarray([2.0 ** (i % 3 - 1) for i in range(n_alpha)], dtype=np.float32)
    # sums stay below 64 in magnitude, so that halves and doubles of them and of their parts are exact in bfloat16
    x = (rng.integers(-1, 2, size=(M, cin)) * (rng.random((M, cin)) < min(1.0, 60 / cin))).astype(np.float32)
    tile, alpha = torch.from_numpy(tile_ref.view(np.int32)).cuda(), torch.from_numpy(alpha_ref).cuda()
    xd = torch.from_numpy(x).cuda().bfloat16()
    for flags in (0, tbn.TBN_FLAG_RELU):
        y = tbn.tbn_linear_forward(xd, tile, alpha, cout, k, flags=flags)
        gen = tbn.tbn_linear_forward(xd, tile, alpha, cout, k, flags=flags | tbn.TBN_FLAG_FORCE_GENERIC)
        assert torch.equal(y, gen)
    rows = np.unique(np.concatenate([np.arange(0, M, 331), [127, 128, M - 1]]))
    ref = np.maximum(orc.linear_forward(x[rows], tile_ref, alpha_ref, cout, k).astype(np.float32), 0.0)
    ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    got = y[torch.from_numpy(rows).cuda()].float().cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {got.size} outputs differ, first at {tuple(bad[0])}"


def test_window_infinity_and_rows_behind_others():
    """An infinity stays in its own row of Y, also where it lies in the last elements of a row whose end is padded."""
    from paper_2407_12075_amd import tbn
    M, cin, cout, k = 6000, 744, 1600, 4
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(M, cin, generator=g, device="cuda").bfloat16()
    x[1, 0] = float("inf")       # right behind the end of row 0
    x[5999, cin - 1] = float("-inf")
    tile, alpha = tbn.tbn_pack_tile(torch.randn(cin * cout, generator=g, device="cuda"), k, k)
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, k) == "window"
    y = tbn.tbn_linear_forward(x, tile, alpha, cout, k)
    finite = torch.isfinite(y).all(dim=1)
    assert torch.isinf(y[1]).all() and torch.isinf(y[5999]).all()
    finite[1] = finite[5999] = True
    assert finite.all()
