"""The fully-connected kernel for any row length and alignment, at the edges of its chunks, row tiles and column tiles:
exact arithmetic (activations in {-1, 0, +1}, alphas powers of two: every output is one float32 number whatever the
order of the sums), so it has to equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tbn_oracle as orc
from paper_2407_12075_amd import workloads as wl

pytestmark = pytest.mark.gpu

# M, in, out, k, n_alpha, element offset of the activations
CASES = [
    (1, 1, 1, 1, 1, 0), (33, 3, 30, 2, 1, 1), (37, 5, 33, 1, 1, 0), (40, 7, 8, 8, 8, 3),       # rows shorter than a load
    (31, 63, 96, 3, 3, 0), (32, 65, 64, 2, 1, 0), (97, 127, 66, 2, 2, 1), (64, 129, 31, 1, 1, 0),   # edges of a chunk
    (1, 257, 1000, 4, 4, 0), (300, 301, 520, 8, 8, 0), (5, 4095, 4096, 8, 8, 0),
    (2500, 196, 384, 4, 1, 0),                       # one column tile per workgroup, four waves
    (4001, 91, 1024, 4, 1, 0),                       # more than 1024 tiles of 32 x 32: two or four column tiles
    (8200, 67, 1026, 2, 2, 0),                       # more than 4096: three or four column tiles, 513 columns
    (200, 4096, 128, 2, 1, 1), (130, 256, 72, 3, 3, 5),   # whole chunks at unaligned addresses
    # aligned rows that other kernels could take as well
    (500, 512, 512, 2, 1, 0), (64, 768, 2048, 4, 4, 0), (1000, 200, 500, 2, 1, 0), (200, 1024, 1024, 2, 1, 0),
    (817, 640, 952, 2, 2, 0), (700, 3840, 128, 2, 1, 0), (2000, 520, 608, 2, 1, 0),
    (1306, 256, 832, 1, 1, 0), (2500, 512, 832, 2, 2, 0),
]


def _signs(tile, n):
    """The first n entries of a tile as +1 / -1 in float32."""
    bits = np.unpackbits(tile.cpu().numpy().view(np.uint8), bitorder="little")[:n]
    return torch.from_numpy(bits.astype(np.float32) * 2 - 1).cuda()


@pytest.fixture(scope="module")
def tbn():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_12075_amd import tbn as binding
    binding.lib()
    return binding


def _at_offset(values, offset):
    """A device tensor of these values whose first element sits `offset` elements after a 256-byte boundary."""
    buf = torch.empty(values.numel() + offset, dtype=values.dtype, device="cuda")
    buf[offset:].copy_(values.reshape(-1))
    return buf[offset:].view(values.shape)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,cin,cout,k,n_alpha,offset", CASES)
def test_direct_exact(tbn, M, cin, cout, k, n_alpha, offset, dtype):
    rng = np.random.default_rng(M * 10000 + cin)
    p = cin * cout // k
    tile_ref = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile_ref[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha_ref = np.asarray([2.0 ** ((i % 5) - 2) for i in range(n_alpha)], dtype=np.float32)
    x = rng.integers(-1, 2, size=(M, cin)).astype(np.float32)
    ref = np.maximum(orc.linear_forward(x, tile_ref, alpha_ref, cout, k).astype(np.float32), 0.0)
    xd = torch.from_numpy(x)
    if dtype == "bf16":
        xd = xd.bfloat16()
        ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    xd = _at_offset(xd, offset)
    tile, alpha = torch.from_numpy(tile_ref.view(np.int32)).cuda(), torch.from_numpy(alpha_ref).cuda()
    y = _at_offset(torch.full((M, cout), 7.0, dtype=xd.dtype), offset)
    tbn.tbn_linear_forward(xd, tile, alpha, cout, k, y=y, flags=tbn.TBN_FLAG_RELU)
    torch.cuda.synchronize()
    got = y.float().cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {got.size} outputs differ, first at {tuple(bad[0])}: {got[tuple(bad[0])]} against {ref[tuple(bad[0])]}"


def test_direct_infinities_and_nan(tbn):
    """An infinity or a NaN reaches the outputs of its own row only, as in the one-thread-per-output kernel."""
    g = torch.Generator().manual_seed(1)
    for dt in (torch.float32, torch.bfloat16):
        x = torch.randn(70, 67, generator=g).to(dt)
        x[3, 5], x[8, 66], x[40, 0] = float("inf"), float("-inf"), float("nan")
        x[50, 1], x[50, 2] = float("inf"), float("inf")
        x = x.cuda()
        tile, alpha = tbn.tbn_pack_tile(torch.randn(67 * 64, generator=g).cuda(), 4)
        y = tbn.tbn_linear_forward(x, tile, alpha, 64, 4).float()
        ref = tbn.tbn_linear_forward(x, tile, alpha, 64, 4, flags=tbn.TBN_FLAG_FORCE_GENERIC).float()
        torch.cuda.synchronize()
        assert torch.equal(torch.isnan(y), torch.isnan(ref))
        assert torch.equal(torch.isinf(y), torch.isinf(ref)) and torch.equal(y[torch.isinf(y)], ref[torch.isinf(ref)])


@pytest.mark.parametrize("M,cin,cout,k,ends", [(300, 196, 384, 4, False), (37, 5, 64, 2, False), (2500, 1199, 1024, 2, False),
                                              (70, 264, 520, 11, True)])
def test_small_activations_keep_all_their_bits(tbn, M, cin, cout, k, ends):
    """Activations down to the smallest float32 numbers.  In float32 sums each of the `cin` additions is off by at most 2^-24
    of the partial sum (at most the sum of the magnitudes) or, among subnormal numbers, exact; alpha is 1, with tile ends
    a power of two, whose products of subnormal sums are rounded once more."""
    g = torch.Generator().manual_seed(cin)
    x0 = torch.randn(M, cin, generator=g)
    x0[1::3] *= torch.exp2(torch.randint(-20, 1, (1, cin), generator=g).float())   # rows of mixed magnitudes
    p = cin * cout // k
    tile = torch.randint(-2 ** 31, 2 ** 31, ((p + 31) // 32,), generator=g).int().cuda()
    alpha = torch.exp2((torch.arange(k) % 3 - 1).float()).cuda() if ends else torch.ones(1).cuda()
    sign = _signs(tile, p).double().repeat(k).view(cout, cin)
    scale = (alpha.double().repeat_interleave(p) if ends else torch.ones(cin * cout, device="cuda")).view(cout, cin)
    cols = torch.arange(cout, device="cuda")
    if ends:   # the columns of the repair pass: the other kernel's are not looked at here
        starts = torch.arange(1, k, device="cuda") * p
        cols = (starts // cin)[starts % cin != 0]
        assert len(cols) == k - 1
    else:
        assert tbn.tbn_linear_forward_kernel(torch.float32, M, cin, cout, k) == "direct"
    for e in (0, -90, -105, -112, -118, -124, -128, -134, -142):
        x = (x0.double() * 2.0 ** e).float().cuda()
        y = tbn.tbn_linear_forward(x, tile, alpha, cout, k)[:, cols].double()
        want = x.double() @ (sign * scale)[cols].t()
        bound = cin * 2.0 ** -24 * (x.double().abs() @ scale[cols].t().double()) + 3 * 2.0 ** -149
        worst = float(((y - want).abs() / bound).max())
        assert worst <= 1.0, (e, worst)
    if not ends:   # an infinity and small activations in the same row tile
        x = (x0.double() * 2.0 ** -118).float().cuda()
        want = tbn.tbn_linear_forward(x, tile, alpha, cout, k)
        x[2, 1] = float("inf")
        y = tbn.tbn_linear_forward(x, tile, alpha, cout, k)
        assert torch.isinf(y[2]).all() and torch.equal(torch.sign(y[2]), sign[:, 1].float())
        want[2] = y[2]
        assert torch.equal(y, want)


# tile starts inside rows, an alpha per tile: M, in, out, k
ENDS = [(33, 264, 520, 11), (1000, 3000, 3072, 9), (8, 1448, 330, 16), (9, 1448, 330, 16), (3, 512, 300, 16), (300, 776, 250, 20), (4100, 520, 250, 16), (64, 1000, 312, 16), (17, 1016, 123, 24), (40, 136, 45, 6), (700, 520, 1000, 64)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,cin,cout,k", ENDS)
def test_tile_starts_inside_rows_exact(tbn, M, cin, cout, k, dtype):
    n = cin * cout
    assert n % k == 0 and (n // k) % cin != 0
    p = n // k
    rng = np.random.default_rng(k)
    tile_ref = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile_ref[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha_ref = np.asarray([2.0 ** (i % 5 - 2) for i in range(k)], dtype=np.float32)
    x = rng.integers(-1, 2, size=(M, cin)).astype(np.float32)
    ref = orc.linear_forward(x, tile_ref, alpha_ref, cout, k).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    if dtype == "bf16":
        xd = xd.bfloat16()
        ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    y = tbn.tbn_linear_forward(xd, torch.from_numpy(tile_ref.view(np.int32)).cuda(), torch.from_numpy(alpha_ref).cuda(), cout, k)
    torch.cuda.synchronize()
    got = y.float().cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {got.size} outputs differ, first at {tuple(bad[0])}: {got[tuple(bad[0])]} against {ref[tuple(bad[0])]}"


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,cin,cout,k", [(70, 264, 520, 11), (8, 1448, 330, 16), (55, 776, 250, 20)])
def test_tile_starts_inside_rows_infinities_and_nan(tbn, M, cin, cout, k, dt):
    """An infinity on one side of a tile start leaves the other side's sum alone."""
    g = torch.Generator().manual_seed(3)
    tile, alpha = tbn.tbn_pack_tile(torch.randn(cin * cout, generator=g).cuda(), k, k)
    x = torch.randn(M, cin, generator=g)
    x[5, 7], x[6, cin - 1], x[M // 2, 100], x[1, 9] = float("inf"), float("-inf"), float("inf"), float("nan")
    x[M - 1, 0], x[M - 1, cin - 1] = float("inf"), float("inf")
    x = x.to(dt).cuda()
    starts = torch.arange(1, k, device="cuda") * (cin * cout // k)
    cols = (starts // cin)[starts % cin != 0]
    y = tbn.tbn_linear_forward(x, tile, alpha, cout, k)[:, cols].float()
    ref = tbn.tbn_linear_forward(x, tile, alpha, cout, k, flags=tbn.TBN_FLAG_FORCE_GENERIC)[:, cols].float()
    assert torch.isinf(ref).sum() >= 3 * len(cols)
    assert torch.equal(torch.isnan(y), torch.isnan(ref))
    assert torch.equal(torch.isinf(y), torch.isinf(ref)) and torch.equal(y[torch.isinf(y)], ref[torch.isinf(ref)])


def test_more_workgroups_than_a_grid_row_holds(tbn):
    """2^24 + 2 row tiles of four waves: more than 2^32 threads, which one grid dimension cannot count."""
    M, cin = (1 << 29) + 33, 3
    assert tbn.tbn_linear_forward_kernel(torch.float32, M, cin, 1, 1) == "direct"
    x = torch.empty(M, cin, device="cuda").random_(0, 3, generator=torch.Generator(device="cuda").manual_seed(1)).sub_(1)
    tile = torch.tensor([5], dtype=torch.int32, device="cuda")
    y = torch.full((M, 1), 7.0, device="cuda")
    tbn.tbn_linear_forward(x, tile, torch.ones(1, device="cuda"), 1, 1, y=y)
    want = (x * _signs(tile, cin)).sum(1, keepdim=True)   # integers: exact in any order
    assert torch.equal(y, want)


def test_repair_pass_with_more_workgroups_than_a_grid_row_holds(tbn):
    """29,132 row tiles x 288 groups of tile starts, eight waves each."""
    M, cin, cout, k = 932200, 144, 6144, 4608
    p = cin * cout // k
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.empty(M, cin, device="cuda").random_(0, 3, generator=g).sub_(1).bfloat16()
    tile = torch.randint(-2 ** 31, 2 ** 31, (p // 32,), generator=g, device="cuda", dtype=torch.int64).int()
    alpha = torch.exp2((torch.arange(k, device="cuda") % 5 - 2).float())
    y = tbn.tbn_linear_forward(x, tile, alpha, cout, k)
    for rows in (slice(0, 4000), slice(M - 20000, M)):
        want = tbn.tbn_linear_forward(x[rows], tile, alpha, cout, k, flags=tbn.TBN_FLAG_FORCE_GENERIC)
        assert torch.equal(y[rows], want)


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_rows_and_tiles_beyond_32_bit_offsets(tbn, dt):
    """Rows of 2^25 and more elements, tiles of 2^36 and more bits; integers, so that the sums are exact."""
    g = torch.Generator(device="cuda").manual_seed(4)
    for M, cin, U, k in ((33, (1 << 25) + 3, 2, 2), (2, (1 << 25) + 3, 2048, 1)):
        if dt == torch.bfloat16 and U > 2:
            continue
        cout, p = U * k, U * cin
        assert tbn.tbn_linear_forward_kernel(dt, M, cin, cout, k) == "direct"
        x = torch.empty(M, cin, device="cuda", dtype=dt).random_(0, 3, generator=g).sub_(1)
        tile = torch.empty((p + 31) // 32, dtype=torch.int32, device="cuda").random_(-2 ** 31, 2 ** 31 - 1, generator=g)
        y = tbn.tbn_linear_forward(x, tile, torch.ones(1, device="cuda"), cout, k).float()
        for u in {0, 1, U // 2 + 1, U - 1} & set(range(U)):
            first = u * cin
            words = tile[first // 32: (first + cin + 31) // 32]
            bits = ((words[:, None] >> torch.arange(32, device="cuda", dtype=torch.int32)) & 1).view(-1)[first % 32: first % 32 + cin]
            sign = bits.double() * 2 - 1
            for m in {0, 1, M - 1}:
                want = (x[m].double() @ sign).to(dt).float()
                assert torch.equal(y[m, u::U], want.repeat(k)), (m, u)
