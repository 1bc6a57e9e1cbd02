"""bfloat16 layers whose K is split among the waves of a 32-row workgroup, at the edges of the rules that choose the number of
columns per wave and of the shared epilogue.  Exact arithmetic (activations in {-1, 0, +1}, alphas powers of two): outputs equal
the oracle and the kernel with one thread per output bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tbn_oracle as orc
from paper_2407_12075_amd import workloads as wl

pytestmark = pytest.mark.gpu

# M, in, out, k, n_alpha
CASES = [
    (33, 1024, 1024 * 70, 70, 70),   # four slices of two chunks; replicas beyond the 64 whose alphas sit in lanes
    (100, 1536, 520, 1, 1),          # four slices of three chunks; last column tile of 8
    (2, 1024, 8192, 2, 2),           # few rows, over the decode kernel
    (16, 2048, 520, 1, 1),           # the smallest product there: 8320
    (65, 1024, 1040 * 8, 130, 1),    # replicas in three rounds of alphas, one alpha
    (17, 8192, 200, 5, 5),           # 40 distinct columns
    (512, 2048, 1024, 2, 1),         # 256 workgroups of one column tile per wave
    (513, 2048, 1024, 2, 2),         # 17 row tiles: two column tiles per wave
    (500, 2048, 3000, 3, 3),         # 1000 distinct columns: the second tile of the last group is cut
    (900, 1024, 2064, 2, 2),         # 29 x 33 tiles, two per wave, four slices
    (65, 4096, 1152, 9, 9),
]


@pytest.mark.parametrize("M,cin,cout,k,n_alpha", CASES)
def test_split_tiles_exact(M, cin, cout, k, n_alpha):
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, n_alpha) == "tile"
    rng = np.random.default_rng(cin + k + M)
    p = cin * cout // k
    tile_ref = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    alpha_ref = np.asarray([2.0 ** (i % 3 - 1) for i in range(n_alpha)], dtype=np.float32)
    # sums stay far below 256 in magnitude, so that halves and doubles of them are exact in bfloat16
    x = (rng.integers(-1, 2, size=(M, cin)) * (rng.random((M, cin)) < 60 / cin)).astype(np.float32)
    tile, alpha = torch.from_numpy(tile_ref.view(np.int32)).cuda(), torch.from_numpy(alpha_ref).cuda()
    xd = torch.from_numpy(x).cuda().bfloat16()
    for flags in (0, tbn.TBN_FLAG_RELU):
        y = tbn.tbn_linear_forward(xd, tile, alpha, cout, k, flags=flags)
        gen = tbn.tbn_linear_forward(xd, tile, alpha, cout, k, flags=flags | tbn.TBN_FLAG_FORCE_GENERIC)
        assert torch.equal(y, gen)
    rows = np.unique(np.concatenate([np.arange(0, M, 97), [M - 1]]))
    ref = np.maximum(orc.linear_forward(x[rows], tile_ref, alpha_ref, cout, k).astype(np.float32), 0.0)
    ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    got = y[torch.from_numpy(rows).cuda()].float().cpu().numpy()
    assert np.array_equal(got, ref)
