"""The bfloat16 kernel that keeps short rows in LDS, at the edges of its row blocks, column groups and chunks of K: exact
arithmetic (activations in {-1, 0, +1}, alphas powers of two), so it has to equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tbn_oracle as orc
from paper_2407_12075_amd import workloads as wl

pytestmark = pytest.mark.gpu

# M, in, out, k, n_alpha
CASES = [
    (9217, 8, 1000, 1, 1),       # one chunk, mostly padding; a last row block of one row; a last column group of 40
    (8190, 64, 4096, 2, 2),      # one whole chunk, two replicas
    (5100, 72, 2048, 1, 1),      # eight elements in the second chunk
    (4100, 136, 3080, 1, 1),     # windows at byte positions
    (3200, 256, 5000, 1, 1),     # four chunks: all of them formed ahead
    (3000, 264, 3104, 1, 1),     # five
    (2757, 576, 10320, 2, 2),    # nine chunks, two replicas
    (8100, 512, 4104, 1, 1),     # several passes per wave, a last one that not every wave has
]


@pytest.mark.parametrize("M,cin,cout,k,n_alpha", CASES)
def test_short_rows_exact(M, cin, cout, k, n_alpha):
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, n_alpha) == "short-rows"
    rng = np.random.default_rng(cin)
    p = cin * cout // k
    tile_ref = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile_ref[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha_ref = np.asarray([2.0 ** (i % 5 - 2) for i in range(n_alpha)], dtype=np.float32)
    x = rng.integers(-1, 2, size=(M, cin)).astype(np.float32)
    # the +-1 product of the distinct rows in float32 is exact; rows for the oracle: the ends of the row blocks and some between
    tile, alpha = torch.from_numpy(tile_ref.view(np.int32)).cuda(), torch.from_numpy(alpha_ref).cuda()
    y = tbn.tbn_linear_forward(torch.from_numpy(x).cuda().bfloat16(), tile, alpha, cout, k, flags=tbn.TBN_FLAG_RELU)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, M, 97), np.arange(127, M, 128), [M - 1]]))
    ref = np.maximum(orc.linear_forward(x[rows], tile_ref, alpha_ref, cout, k).astype(np.float32), 0.0)
    ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    got = y[torch.from_numpy(rows).cuda()].float().cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {got.size} outputs differ, first at {tuple(bad[0])}"
    # every row against the one-thread-per-output kernel
    gen = tbn.tbn_linear_forward(torch.from_numpy(x).cuda().bfloat16(), tile, alpha, cout, k, flags=tbn.TBN_FLAG_RELU | tbn.TBN_FLAG_FORCE_GENERIC)
    assert torch.equal(y, gen)
