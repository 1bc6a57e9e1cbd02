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


def _counted(tbn, M, cin, U, k, flags, dtype=torch.float32):
    return tbn.lib().tbn_diag_binact_counted(tbn.TBN_F32 if dtype == torch.float32 else tbn.TBN_BF16, M, cin, U * k, k, k, flags) == 1


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
    assert _counted(tbn, M, cin, U, k, tbn.TBN_FLAG_SIGN_OUT)
    _both(tbn, x, cin, t, alpha, U * k, k, tbn.TBN_FLAG_SIGN_OUT, torch.float32)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,cin,U,k,flags", [(6273, 2304, 1024, 1, 0), (6200, 2560, 960, 2, 1), (49160, 2816, 64, 4, 0)])
def test_long_rows_with_real_outputs(tbn, M, cin, U, k, flags, dtype):
    x, t, alpha = _layer(M, cin, U, k, M + cin)
    assert _counted(tbn, M, cin, U, k, flags, dtype)
    _both(tbn, x, cin, t, alpha, U * k, k, flags, dtype)


@pytest.mark.parametrize("ones", [0.0, 1.0])   # rows of set bits against rows without any, and against rows of set bits
def test_largest_sums(tbn, ones):
    M, cin, U = 2113, 65536, 1088      # (real outputs: the 64 x 64 blocks, which do not count)
    x, t, alpha = _layer(M, cin, U, 2, cin, ones)
    assert _counted(tbn, M, cin, U, 2, tbn.TBN_FLAG_SIGN_OUT) and not _counted(tbn, M, cin, U, 2, 0)
    _both(tbn, x, cin, t, alpha, 2 * U, 2, tbn.TBN_FLAG_SIGN_OUT, torch.float32)
    _both(tbn, x, cin, t, alpha, 2 * U, 2, 0, torch.float32)
    M, cin, U = 49160, 8192, 64        # real outputs that are counted
    x, t, alpha = _layer(M, cin, U, 2, cin, ones)
    assert _counted(tbn, M, cin, U, 2, 0)
    _both(tbn, x, cin, t, alpha, 2 * U, 2, 0, torch.float32)


def _prefix_rows(n, cin, seed):
    """n rows whose first a[i] bits are set: a product of two of them is cin - 2 |a - b|."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    edges = torch.tensor([0, 1, 2, cin // 2 - 1, cin // 2, cin // 2 + 1, cin // 2 + 2, cin - 1, cin], device="cuda")
    a = torch.randint(0, cin + 1, (n,), generator=g, device="cuda")
    a[::2] = edges[torch.randint(0, len(edges), (len(a[::2]),), generator=g, device="cuda")]
    a[0], a[-1] = cin, 0
    rows = torch.empty(n, cin // 32, dtype=torch.int32, device="cuda")
    first = torch.arange(0, cin, 32, device="cuda")
    for i in range(0, n, 256):
        bits = (a[i:i + 256, None] - first).clamp_(0, 32)
        rows[i:i + 256] = ((1 << bits) - 1).to(torch.int32)     # (the low 32 bits of the number)
    return rows, a


@pytest.mark.parametrize("M,cin,U,counted", [
    (6145, 1 << 22, 1024, True),              # the longest rows that are counted: partial sums of up to 3.25 * 2^22
    (65, (1 << 22) + 256, 1024, False),       # one super-step more
])
def test_sums_at_the_longest_counted_rows(tbn, M, cin, U, counted):
    """Products of rows of set bits and of rows that differ in half of them, give or take one, whose signs show any error of the sums."""
    x, a = _prefix_rows(M, cin, 3)
    t, b = _prefix_rows(U, cin, 4)
    z = cin - 2 * (a[:, None] - b).abs()
    assert z.max() == cin and z.min() == -cin and all((z == v).any() for v in (-4, -2, 0, 2, 4))
    one = torch.ones(1, device="cuda")
    assert _counted(tbn, M, cin, U, 1, 0) == counted and _counted(tbn, M, cin, U, 1, tbn.TBN_FLAG_SIGN_OUT) == counted
    y = tbn.tbn_linear_forward_binact(x, cin, t.reshape(-1), one, U, 1, dtype=torch.float32)
    assert torch.equal(y, z.float())
    for alpha in (one, -one):
        words = tbn.tbn_linear_forward_binact(x, cin, t.reshape(-1), alpha, U, 1, flags=tbn.TBN_FLAG_SIGN_OUT)
        set_bits = (words[:, :, None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1
        assert torch.equal(set_bits.reshape(M, U) == 1, z * int(alpha.item()) > 0)
