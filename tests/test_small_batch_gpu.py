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
    ("bf16", 33, 4104, 200, 5, 5, "small-batch"),      # 33: a second round for one wave
    ("bf16", 40, 8200, 72, 3, 3, "small-batch"),       # a third
    ("f32", 10, 1024, 640, 16, 16, "decode"),
    ("f32", 8, 768, 2080, 4, 4, "decode"),
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


# Tiles that end inside rows: windows that run past the tile's end anywhere in a row, an alpha per tile, the repair pass by this
# kernel's form for it (float32 from 512 elements on, bfloat16 up to 8 rows from 1408 on) or the direct kernel's, one round of loads or several.
@pytest.mark.parametrize("dtype,M,cin,cout,k", [
    ("bf16", 8, 4360, 330, 16), ("bf16", 3, 8456, 200, 16), ("bf16", 33, 8200, 90, 16), ("bf16", 64, 1448, 330, 16),
    ("f32", 17, 2056, 100, 16), ("f32", 5, 6200, 36, 16), ("f32", 64, 520, 250, 16), ("f32", 40, 136, 45, 8), ("f32", 9, 4104, 39, 24)])
def test_tile_starts_inside_rows_exact(dtype, M, cin, cout, k):
    from paper_2407_12075_amd import tbn
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    p = cin * cout // k
    assert cin * cout % k == 0 and p % cin != 0 and tbn.tbn_linear_forward_kernel(dt, M, cin, cout, k, k) == "small-batch"
    rng = np.random.default_rng(cin + M)
    tile = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha = torch.tensor([2.0 ** (i % 3 - 1) for i in range(k)], device="cuda")
    if dtype == "bf16":
        x = rng.integers(-1, 2, size=(M, cin))
    else:   # 16 whole numbers of 18 bits in a row, so that all three terms of the split count: sums below 2^22, in halves after the alphas below 2^24
        x = np.zeros((M, cin), dtype=np.int64)
        for r in x:
            r[rng.choice(cin, 16, replace=False)] = rng.integers(-(2 ** 18 - 1), 2 ** 18, size=16) | 1
        assert np.abs(x).sum(1).max() < 2 ** 22
    xd = torch.from_numpy(x.astype(np.float32)).cuda().to(dt)
    args = (xd, torch.from_numpy(tile.view(np.int32)).cuda(), alpha, cout, k)
    assert torch.equal(tbn.tbn_linear_forward(*args), tbn.tbn_linear_forward(*args, flags=tbn.TBN_FLAG_FORCE_GENERIC))


# float32 calls next to the bfloat16 ones that the small-batch kernel takes: its sums of three terms turn an infinity into a NaN
# and drop what lies below 2^-133, the decode and the direct kernel do neither
@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("M,cin,cout,k,kernel", [
    (5, 512, 3328, 4, "decode"), (8, 768, 2080, 4, "decode"), (12, 512, 2048, 4, "decode"), (16, 1024, 1024, 8, "decode"),
    (16, 1152, 4096, 4, "decode"), (17, 512, 512, 4, "direct"), (32, 1280, 1024, 4, "direct"), (64, 512, 1024, 4, "direct"),
    (128, 640, 512, 4, "direct"), (200, 1024, 1024, 8, "direct")])
def test_float32_infinities_nan_and_smallest_numbers(M, cin, cout, k, kernel, relu):
    from paper_2407_12075_amd import tbn
    rng = np.random.default_rng(M + cin)
    x = rng.integers(-999, 1000, size=(M, cin)).astype(np.float32)   # whole numbers: sums are exact in any order
    x[1::5] *= np.float32(2.0 ** -149)
    x[2::5, 7] = np.inf
    x[3::5, cin - 1] = -np.inf
    x[3::5, 100] = np.inf
    x[4::5, cin // 2] = np.nan
    tile = torch.from_numpy(rng.integers(0, 2 ** 32, size=cin * cout // k // 32, dtype=np.uint64).astype(np.uint32).view(np.int32)).cuda()
    alpha = torch.tensor([2.0 ** (i % 5 - 2) for i in range(k)], device="cuda")
    args = (torch.from_numpy(x).cuda(), tile, alpha, cout, k)
    y = tbn.tbn_linear_forward(*args, flags=int(relu))
    want = tbn.tbn_linear_forward(*args, flags=int(relu) | tbn.TBN_FLAG_FORCE_GENERIC)
    assert torch.isinf(want[2]).any() and (want[1] != 0).any()
    assert torch.equal(torch.isnan(y), torch.isnan(want)) and torch.equal(torch.nan_to_num(y, 3.0, posinf=torch.inf, neginf=-torch.inf),
                                                                         torch.nan_to_num(want, 3.0, posinf=torch.inf, neginf=-torch.inf))
    assert tbn.tbn_linear_forward_kernel(torch.float32, M, cin, cout, k, k) == kernel
