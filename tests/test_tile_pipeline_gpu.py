"""float32 layers whose tile holds whole weight rows, one wave per 32 batch rows: the loop over chunks of 64 elements, of which one or two are
on their way while one is multiplied, at every count where its beginning and end differ, for one to four column tiles per wave, K in one
slice or several (there one or two column tiles keep a plain loop), rows and columns that end inside a tile.  Exact arithmetic: half of the rows hold integers of 13 bits, whose sums
float32 holds, the other half one integer of 24 bits, which takes all three terms of the split.  Below, the kernel for any row length where
its workgroups of eight waves would need a second round of the CUs and take four waves, or one column tile instead of four."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tbn():
    from paper_2407_12075_amd import tbn as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("U", [32, 60, 96, 100, 256])
@pytest.mark.parametrize("chunks", [1, 2, 3, 4, 5, 6, 7, 11, 13, 14, 15, 17,   # K in one slice; two chunks on their way from 13 on
                                    8, 12, 16, 24, 28, 40])                    # four or eight slices of two, three, seven or five
def test_chunks_of_the_float32_loop(tbn, chunks, U):
    M, cin, k = 301, 64 * chunks, 2
    g = torch.Generator().manual_seed(chunks * 1000 + U)
    x = torch.randint(-4096, 4097, (M, cin), generator=g).double()
    x[1::2] = 0
    rows = torch.arange(1, M, 2)
    x[rows, (rows * 37) % cin] = (torch.randint(2 ** 22, 2 ** 23, (len(rows),), generator=g) * 2 + 1).double()
    words = torch.randint(-2 ** 31, 2 ** 31, (U * cin // 32,), generator=g).to(torch.int32)
    signs = ((words.view(-1, 1) >> torch.arange(32)) & 1).reshape(U, cin).double() * 2 - 1
    alpha = torch.tensor([0.5, -2.0])
    want = torch.cat([x @ signs.T * a for a in alpha.double()], 1).float()
    flags = tbn.TBN_FLAG_LARGE_BATCH
    assert tbn.tbn_linear_forward_kernel(torch.float32, M, cin, U * k, k, k, flags) == "tile"
    y = tbn.tbn_linear_forward(x.float().cuda(), words.cuda(), alpha.cuda(), U * k, k, flags=flags)
    assert torch.equal(y.cpu(), want)


@pytest.mark.parametrize("M,cin,U,k", [
    (8225, 65, 100, 2),       # 258 workgroups of four column tiles: one tile instead
    (8193, 768, 97, 1),       # twelve chunks, the most with one
    (8225, 772, 100, 1),      # thirteen: four tiles, four waves
    (611, 777, 1633, 1),      # 52 tiles of columns, the last one holds one
    (10977, 776, 72, 1),      # three tiles
    (8193, 300, 31, 2),       # 257 workgroups of one tile: four waves
    (3041, 1300, 100, 1),     # 384
])
def test_direct_kernel_in_two_rounds_of_workgroups(tbn, M, cin, U, k):
    g = torch.Generator().manual_seed(M + cin)
    x = torch.randint(-4096, 4097, (M, cin), generator=g).double()
    words = torch.randint(-2 ** 31, 2 ** 31, ((U * cin + 31) // 32,), generator=g).to(torch.int32)
    signs = ((words.view(-1, 1) >> torch.arange(32)) & 1).reshape(-1)[: U * cin].view(U, cin).double() * 2 - 1
    alpha = torch.tensor([0.5, -2.0])[:k]
    want = torch.cat([x @ signs.T * a for a in alpha.double()], 1).float()
    assert tbn.tbn_linear_forward_kernel(torch.float32, M, cin, U * k, k, k) == "direct"
    y = tbn.tbn_linear_forward(x.float().cuda(), words.cuda(), alpha.cuda(), U * k, k)
    assert torch.equal(y.cpu(), want)


@pytest.mark.parametrize("M,cin,U,part", [
    (2100, 20001, 100, 1024),     # 264 workgroups of one column tile, 128 in the part
    (3041, 13825, 400, 512),      # 384 of four column tiles, 208 of one
])
def test_long_rows_keep_the_sums_of_eight_waves(tbn, M, cin, U, part):
    """Rows of more than 13824 elements: more workgroups than CUs take no longer sums, whose error would be the larger, than fewer do."""
    g = torch.Generator(device="cuda").manual_seed(cin)
    x = torch.randn(M, cin, generator=g, device="cuda")
    words = torch.randint(-2 ** 31, 2 ** 31, ((U * cin + 31) // 32,), generator=g, device="cuda", dtype=torch.int64).int()
    one = torch.ones(1, device="cuda")
    assert all(tbn.tbn_linear_forward_kernel(torch.float32, m, cin, U, 1) == "direct" for m in (M, part))
    assert torch.equal(tbn.tbn_linear_forward(x, words, one, U, 1)[:part], tbn.tbn_linear_forward(x[:part], words, one, U, 1))
