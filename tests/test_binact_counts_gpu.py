"""Layers on sign bits whose products are formed from set bits and counts of them (sign bits out, long rows with real outputs), where they
can go wrong: one super-step, odd numbers of them, a last stage that is half a stage, blocks that end inside the last rows and columns,
words of the last column block, many replicas, scalars of either sign, zero and not a number.  Every output is one float32 product of a
scalar and an integer, so the one-thread-per-output kernel agrees bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tbn():
    from paper_2407_12075_amd import tbn as m
    m.lib()
    return m


def _layer(M, cin, U, k, seed, ones=0.5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    bits = lambda rows: torch.randint(-2 ** 31, 2 ** 31, (rows, cin // 32), generator=g, device="cuda", dtype=torch.int64).to(torch.int32)
    x, t = bits(M), bits(U)
    if ones != 0.5:      # rows of set bits only: the largest sums
        x[: M // 2] = -1
        t[: U // 2] = -1 if ones == 1.0 else 0
    alpha = torch.randn(k, generator=g, device="cuda")
    if k >= 4:
        alpha[1], alpha[2] = 0.0, float("nan")
    return x, t.reshape(-1), alpha


def _both(tbn, x, cin, t, alpha, out, k, flags, dtype):
    got = tbn.tbn_linear_forward_binact(x, cin, t, alpha, out, k, flags=flags, dtype=dtype)
    want = tbn.tbn_linear_forward_binact(x, cin, t, alpha, out, k, flags=flags | tbn.TBN_FLAG_FORCE_GENERIC, dtype=dtype)
    torch.cuda.synchronize()
    nan = torch.isnan(want)      # a product with a scalar that is no number: any NaN
    assert torch.equal(nan, torch.isnan(got))
    assert torch.equal(got.masked_fill(nan, 0), want.masked_fill(nan, 0))


@pytest.mark.parametrize("M,cin,U,k", [
    (2113, 256, 1056, 1),        # one super-step, the last column block holds one word, the last row block one row
    (2113, 512, 1056, 4),
    (2100, 768, 1120, 2),        # a stage and a half; three words in the last column block
    (1153, 1280, 2048, 1),
    (2050, 2304, 1088, 2),       # more than 512 blocks of 64 x 64
    (4097, 4096, 576, 17),       # sixteen super-steps, four and a half column blocks, 17 replicas
    (8200, 256, 288, 70),        # replicas past the 64th
])
def test_sign_bits_out(tbn, M, cin, U, k):
    x, t, alpha = _layer(M, cin, U, k, M + cin)
    assert tbn.tbn_linear_forward_binact_kernel(torch.float32, M, cin, U * k, k, k, tbn.TBN_FLAG_SIGN_OUT) == "matrix-core"
    _both(tbn, x, cin, t, alpha, U * k, k, tbn.TBN_FLAG_SIGN_OUT, torch.float32)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,cin,U,k,flags", [(6273, 2304, 1024, 1, 0), (6200, 2560, 960, 2, 1), (49160, 2816, 64, 4, 0)])
def test_long_rows_with_real_outputs(tbn, M, cin, U, k, flags, dtype):
    x, t, alpha = _layer(M, cin, U, k, M + cin)
    _both(tbn, x, cin, t, alpha, U * k, k, flags, dtype)


@pytest.mark.parametrize("ones", [0.0, 1.0])   # rows of set bits against rows without any, and against rows of set bits
def test_largest_sums(tbn, ones):
    M, cin, U = 2113, 65536, 1088
    x, t, alpha = _layer(M, cin, U, 2, cin, ones)
    _both(tbn, x, cin, t, alpha, 2 * U, 2, tbn.TBN_FLAG_SIGN_OUT, torch.float32)
    _both(tbn, x, cin, t, alpha, 2 * U, 2, 0, torch.float32)
