"""The small-batch kernel where a wave's share of K changes: no, one, several blocks of 128 and a second round of them, and the calls
of at most 16 rows that it takes from the decode kernel.  Exact arithmetic (activations in {-1, 0, +1}, alphas powers of two), so it
has to equal the one-thread-per-output kernel bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# dtype, M, in, out, k, n_alpha, kernel
CASES = [
    ("bf16", 9, 8, 320, 2, 2, "small-batch"),          # one block, mostly padding
    ("bf16", 16, 1016, 328, 4, 4, "small-batch"),      # eight blocks, the last one cut
    ("bf16", 13, 1032, 96, 4, 1, "small-batch"),       # nine: one wave has two
    ("bf16", 12, 3072, 3072, 4, 4, "small-batch"),     # 24
    ("bf16", 5, 2048, 3072, 2, 1, "small-batch"),      # five rows, 16
    ("bf16", 33, 4104, 200, 5, 5, "small-batch"),      # 33: a second round for one wave; tile starts inside rows or not
    ("bf16", 40, 8200, 72, 3, 3, "small-batch"),       # a third
    ("f32", 10, 1024, 640, 16, 16, "small-batch"),
    ("f32", 8, 768, 2080, 4, 4, "small-batch"),
    ("f32", 17, 2056, 80, 5, 1, "small-batch"),        # 17 blocks: a second round for one wave
    ("f32", 21, 6200, 48, 3, 3, "small-batch"),
    ("bf16", 9, 1544, 64, 4, 4, "decode"),             # beyond the lines
    ("f32", 8, 776, 2080, 4, 4, "decode"),
    ("bf16", 4, 512, 4160, 2, 2, "decode"),
]


@pytest.mark.parametrize("dtype,M,cin,cout,k,n_alpha,kernel", CASES)
def test_small_batch_exact(dtype, M, cin, cout, k, n_alpha, kernel):
    from paper_2407_12075_amd import tbn
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    assert tbn.tbn_linear_forward_kernel(dt, M, cin, cout, k, n_alpha) == kernel
    rng = np.random.default_rng(cin + M)
    p = cin * cout // k
    tile = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha = np.asarray([2.0 ** (i % 5 - 2) for i in range(n_alpha)], dtype=np.float32)
    x = torch.from_numpy(rng.integers(-1, 2, size=(M, cin)).astype(np.float32)).cuda().to(dt)
    args = (x, torch.from_numpy(tile.view(np.int32)).cuda(), torch.from_numpy(alpha).cuda(), cout, k)
    assert torch.equal(tbn.tbn_linear_forward(*args), tbn.tbn_linear_forward(*args, flags=tbn.TBN_FLAG_FORCE_GENERIC))
