"""The windowed form of the bfloat16 block kernel (row lengths in multiples of 8, tile starts inside rows) at the edges of its
blocks, rounds and tile pieces: exact arithmetic (activations in {-1, 0, +1}, alphas powers of two), so it has to equal the
oracle and the kernel with one thread per output bit for bit."""
import collections
import math
import random

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
    # workgroups with three blocks at every ring phase and slot: 14, 16, 18, 20, 22 and 26 rounds (24 above), the last row block
    # of a few rows, tile starts in the first and in the last chunk of a row
    (4867, 1656, 2320, 9, 9),
    (22019, 1872, 392, 9, 9),
    (17412, 2088, 424, 9, 9),
    (13314, 2376, 536, 11, 11),
    (9730, 2600, 776, 13, 13),
    (11144, 3120, 648, 13, 13),
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


@pytest.mark.parametrize("seed", [1, 2])
def test_drawn_layers_in_both_forms(seed):
    """Rows in multiples of 8, on grids of at most a block per CU and on larger ones (the form whose workgroups walk blocks)."""
    from paper_2407_12075_amd import tbn
    rng = random.Random(seed)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    drawn = collections.Counter()
    while min(drawn[False], drawn[True]) < 20:
        large = drawn[True] < 20 and rng.random() < 0.5
        M = rng.randint(4000, 20000) if large else rng.randint(100, 5000)
        cin, cout, k = 8 * rng.randint(25, 420), 8 * rng.randint(8, 300), rng.choice([1, 2, 3, 4, 5, 6, 7, 9, 10, 12])
        if cin * cout % k or M * cin * cout > 3e10:
            continue
        p, n_alpha, flags = cin * cout // k, rng.choice([1, k]), rng.choice([0, tbn.TBN_FLAG_RELU])
        blocks = -(-M // 128) * -(-min(cout, p // math.gcd(p, cin)) // 128)
        if (blocks > cus) != large or tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, n_alpha, flags) != "window":
            continue
        drawn[large] += 1
        what = f"M={M} in={cin} out={cout} k={k} n_alpha={n_alpha} flags={flags} blocks={blocks}"
        print(what, flush=True)
        g = torch.Generator(device="cuda").manual_seed(M + cin)
        tile = torch.randint(-2 ** 31, 2 ** 31 - 1, ((p + 31) // 32,), device="cuda", dtype=torch.int32, generator=g)
        alpha = torch.tensor([2.0 ** (i % 3 - 1) for i in range(n_alpha)], device="cuda")
        # (as above: every partial sum that is rounded stays exact in bfloat16)
        keep = torch.rand(M, cin, device="cuda", generator=g) < 60 / cin
        x = ((torch.randint(-1, 2, (M, cin), device="cuda", generator=g)) * keep).bfloat16()
        y = tbn.tbn_linear_forward(x, tile, alpha, cout, k, flags=flags)
        gen = tbn.tbn_linear_forward(x, tile, alpha, cout, k, flags=flags | tbn.TBN_FLAG_FORCE_GENERIC)
        assert torch.equal(y, gen), what
    print(f"seed {seed}: {drawn[False]} layers with a block per workgroup, {drawn[True]} with several", flush=True)


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
