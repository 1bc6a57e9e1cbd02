"""The convolution kernel with one wave per block of output pixels, at the edges of its blocks: exact arithmetic
(activations in {-1, 0, +1}, alphas powers of two: every output is one float32 number whatever the order of the sums),
so it has to equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tbn_oracle as orc
from paper_2407_12075_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, C, H, W, O, window, stride, pad, k, n_alpha
CASES = [
    (2, 9, 7, 7, 8, 3, 1, 1, 2, 2),          # 49 pixels in one block, a short chunk, fewer filters than a tile of 16
    (1, 33, 14, 14, 34, 3, 1, 1, 2, 2),      # 17 distinct filters, one channel in the second chunk
    (2, 64, 9, 65, 66, 3, 1, 1, 2, 1),       # 33 filters; 65 columns: a last column block of few pixels
    (1, 40, 5, 91, 16, 3, 1, 1, 1, 1),       # odd rows: bfloat16 stores at 2-byte alignment
    (3, 16, 13, 2, 64, 3, 1, 1, 64, 64),     # two columns (one pair of pixels), one distinct filter, 64 replicas
    (1, 12, 3, 3, 130, 3, 1, 1, 65, 65),     # more replicas than lanes
    (2, 48, 15, 17, 96, 3, 2, 1, 1, 1),      # stride 2, 96 filters: three tiles of 32
    (1, 128, 11, 13, 260, 3, (2, 1), (0, 2), 2, 2),   # 130 filters, unequal strides and paddings, 4 or 8 channel slices
    (1, 512, 4, 4, 32, 3, 1, 1, 1, 1),       # eight channel slices of several chunks
    (1, 64, 14, 14, 48, 3, 1, 1, 3, 3),      # whole filters
    (1, 32, 10, 12, 40, 3, 1, 1, 9, 9),      # tile ends inside filters: windows that wrap, repaired channels
    (1, 32, 10, 12, 40, 3, 1, 1, 9, 1),
    (2, 24, 8, 8, 6, 1, 1, 0, 2, 1),         # 1x1
    (2, 56, 15, 15, 70, 1, 2, 0, 2, 2),      # 1x1 with stride 2
    (1, 272, 9, 9, 128, 1, 1, 1, 1, 1),      # 1x1 with padding, 128 filters, a half chunk at the end
    (1, 64, 8, 24, 45, 1, 1, 0, 8, 8),       # 1x1, tile ends inside filters
]


@pytest.fixture(scope="module")
def tbn():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_12075_amd import tbn as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,C,H,W,O,ks,stride,pad,k,n_alpha", CASES)
def test_conv_wave_blocks_exact(tbn, N, C, H, W, O, ks, stride, pad, k, n_alpha, dtype):
    stride = stride if isinstance(stride, tuple) else (stride, stride)
    pad = pad if isinstance(pad, tuple) else (pad, pad)
    rng = np.random.default_rng(C * 1000 + O)
    p = O * C * ks * ks // k
    tile_ref = rng.integers(0, 2 ** 32, size=(p + 31) // 32, dtype=np.uint64).astype(np.uint32)
    if p % 32:
        tile_ref[-1] &= np.uint32((1 << (p % 32)) - 1)
    alpha_ref = np.asarray([2.0 ** ((i % 5) - 2) for i in range(n_alpha)], dtype=np.float32)
    x = rng.integers(-1, 2, size=(N, C, H, W)).astype(np.float32)
    ref = orc.conv2d_forward(x, tile_ref, alpha_ref, O, ks, ks, k, stride=stride, pad=pad).astype(np.float32)
    ref = np.maximum(ref, 0.0)
    xd = torch.from_numpy(x).cuda()
    if dtype == "bf16":
        xd = xd.bfloat16()
        ref = wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(ref)).reshape(ref.shape)
    y = tbn.tbn_conv2d_forward(xd, torch.from_numpy(tile_ref.view(np.int32)).cuda(), torch.from_numpy(alpha_ref).cuda(), O, ks, ks, k,
                               stride=stride, pad=pad, flags=tbn.TBN_FLAG_RELU)
    torch.cuda.synchronize()
    got = y.float().cpu().numpy()
    bad = np.argwhere(got != ref)
    assert bad.size == 0, f"{len(bad)} of {got.size} outputs differ, first at {tuple(bad[0])}: {got[tuple(bad[0])]} against {ref[tuple(bad[0])]}"


# Every instance of the kernel: dtype, N, C, H, W, O, window, stride, k, n_alpha, the plan (filter tiles per wave x filters per
# tile, pixels per wave, pixels of a patch in LDS; "all-bits": the instance for layers the block kernel does not take)
PLANS = [
    ("bf16", 1, 41, 4, 4, 18, 1, 2, 2, 2, "1x16 pixels=64 patch=129"),
    ("bf16", 1, 64, 4, 4, 17, 1, 2, 1, 1, "1x32 pixels=64 patch=129"),
    ("bf16", 64, 17, 16, 65, 140, 1, 1, 2, 2, "2x32 pixels=64 patch=129"),
    ("bf16", 96, 16, 46, 46, 130, 1, 2, 1, 1, "4x32 pixels=64 patch=129"),
    ("bf16", 1, 16, 4, 4, 18, 3, 2, 2, 1, "1x16 pixels=64 patch=128"),
    ("bf16", 1, 17, 4, 4, 17, 3, 2, 1, 1, "1x32 pixels=64 patch=128"),
    ("bf16", 1, 16, 9, 9, 9, 3, 2, 1, 1, "1x32 pixels=64 patch=256"),
    ("bf16", 1, 16, 15, 15, 17, 3, 2, 1, 1, "1x32 pixels=32 patch=256"),
    ("bf16", 64, 127, 4, 4, 140, 3, 2, 2, 2, "2x32 pixels=64 patch=128"),
    ("bf16", 64, 128, 9, 9, 70, 3, 2, 1, 1, "2x32 pixels=64 patch=256"),
    ("bf16", 64, 128, 15, 15, 34, 3, 2, 1, 1, "2x32 pixels=32 patch=256"),
    ("bf16", 64, 128, 4, 4, 260, 3, 2, 2, 2, "4x32 pixels=64 patch=128"),
    ("bf16", 64, 127, 9, 9, 130, 3, 2, 1, 1, "4x32 pixels=64 patch=256"),
    ("bf16", 64, 64, 15, 15, 130, 3, 2, 1, 1, "4x32 pixels=32 patch=256"),
    ("bf16", 128, 128, 4, 4, 99, 3, 2, 16, 1, "4x32 pixels=64 patch=128"),      # tile ends inside filters
    ("f32", 1, 64, 4, 4, 18, 1, 2, 2, 2, "1x32 pixels=64 patch=65"),
    ("f32", 64, 17, 16, 65, 140, 1, 1, 2, 2, "2x32 pixels=64 patch=65"),
    ("f32", 96, 16, 46, 46, 130, 1, 2, 1, 1, "4x32 pixels=64 patch=65"),
    ("f32", 1, 64, 4, 4, 18, 3, 2, 2, 2, "1x32 pixels=64 patch=100"),
    ("f32", 1, 64, 9, 9, 9, 3, 2, 1, 1, "1x32 pixels=64 patch=128"),
    ("f32", 2, 16, 3, 200, 9, 3, 2, 1, 1, "1x32 pixels=64 patch=192"),
    ("f32", 64, 17, 14, 14, 9, 3, 2, 1, 1, "1x32 pixels=32 patch=192"),
    ("f32", 64, 127, 4, 4, 140, 3, 2, 2, 2, "2x32 pixels=64 patch=100"),
    ("f32", 32, 64, 5, 130, 34, 3, 2, 1, 1, "2x32 pixels=64 patch=128"),
    ("f32", 64, 16, 5, 130, 70, 3, 2, 1, 1, "2x32 pixels=64 patch=192"),
    ("f32", 64, 128, 14, 14, 34, 3, 2, 1, 1, "2x32 pixels=32 patch=192"),
    ("f32", 64, 128, 4, 4, 70, 3, 2, 3, 1, "2x32 pixels=64 patch=100"),       # tile ends inside filters
    ("f32", 1, 4200, 4, 4, 18, 3, 2, 2, 2, "1x32 pixels=64 patch=100 all-bits"),
    ("f32", 1, 4200, 9, 9, 9, 3, 2, 1, 1, "1x32 pixels=64 patch=128 all-bits"),
    ("f32", 1, 16, 2, 4096, 40, 1, 1, 2, 2, "1x32 pixels=64 patch=65 all-bits"),
]


def _plan_matches(name, plan):
    fields = dict(f.split("=") for f in name.split()[1:] if "=" in f)
    want = plan.split()
    return name.startswith("wave ") and fields["filters"] == want[0] and all(f"{k}={fields[k]}" in want for k in ("pixels", "patch")) and \
        name.endswith("all-bits") == plan.endswith("all-bits")


@pytest.mark.parametrize("dtype,N,C,H,W,O,ks,stride,k,n_alpha,plan", PLANS)
def test_conv_wave_every_instance_exact(tbn, dtype, N, C, H, W, O, ks, stride, k, n_alpha, plan):
    """Exact arithmetic, against one thread per output.  Float32: integers of 20 bits, which take all three terms of the split, so
    few of them that no sum leaves 24 bits; bfloat16: integers of 8 bits."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    name = tbn.tbn_conv2d_forward_kernel(dt, N, C, H, W, O, ks, ks, k, (stride, stride), (ks // 2, ks // 2), n_alpha)
    assert _plan_matches(name, plan), name
    g = torch.Generator(device="cuda").manual_seed(O * C)
    F, p = C * ks * ks, O * C * ks * ks // k
    top = 2 ** 19 if dtype == "f32" else 255
    x = torch.randint(-top, top + 1, (N, C, H, W), generator=g, device="cuda").float()
    x *= torch.rand(x.shape, generator=g, device="cuda") < (6.0 / F if dtype == "f32" else 0.5)
    tile = torch.randint(-2 ** 31, 2 ** 31, ((p + 31) // 32,), generator=g, device="cuda", dtype=torch.int64).int()
    alpha = torch.exp2((torch.arange(n_alpha, device="cuda") % 5 - 2).float())
    args = (x.to(dt), tile, alpha, O, ks, ks, k)
    y = tbn.tbn_conv2d_forward(*args, stride=(stride, stride), pad=(ks // 2, ks // 2))
    ref = tbn.tbn_conv2d_forward(*args, stride=(stride, stride), pad=(ks // 2, ks // 2), flags=tbn.TBN_FLAG_FORCE_GENERIC)
    assert float(ref.float().abs().max()) < 2 ** 26 and ref.any()
    assert torch.equal(y, ref)


# float32: N, C, H, W, O, window, stride, pad, k
SPECIAL = [(2, 64, 14, 14, 64, 3, 1, 1, 4), (1, 40, 9, 65, 66, 3, 1, 1, 2), (2, 48, 15, 17, 96, 3, 2, 1, 1), (1, 272, 9, 9, 128, 1, 1, 0, 1),
           (1, 4200, 6, 6, 32, 3, 1, 1, 2)]   # the last one: more channels than tbn_conv_mfma.hip takes


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,C,H,W,O,kh,kw,k", [(1, 32, 10, 12, 40, 3, 3, 9), (2, 64, 9, 12, 45, 1, 1, 8), (2, 32, 14, 9, 34, 9, 1, 8),
                                              (3, 64, 20, 20, 64, 9, 1, 4), (1, 64, 9, 30, 33, 1, 9, 4)])
def test_conv_block_kernel_infinities_and_nan(tbn, N, C, H, W, O, kh, kw, k, dt):
    """The block kernel (windows of nine taps in a row) and the pass over channels whose filter contains a tile start."""
    g = torch.Generator().manual_seed(C + O)
    x = torch.randn(N, C, H, W, generator=g)
    x[0, 3, 0, 1], x[0, C - 1, H - 1, W - 1], x[N - 1, 9, 4, 4] = float("inf"), float("-inf"), float("nan")
    x = x.to(dt).cuda()
    tile, alpha = tbn.tbn_pack_tile(torch.randn(O * C * kh * kw, generator=g).cuda(), k, k)
    pad = ((kh - 1) // 2, (kw - 1) // 2)
    y = tbn.tbn_conv2d_forward(x, tile, alpha, O, kh, kw, k, pad=pad).float()
    ref = tbn.tbn_conv2d_forward(x, tile, alpha, O, kh, kw, k, pad=pad, flags=tbn.TBN_FLAG_FORCE_GENERIC).float()
    assert torch.isinf(ref).any() and torch.isnan(ref).any()
    assert torch.equal(torch.isnan(y), torch.isnan(ref))
    assert torch.equal(torch.isinf(y), torch.isinf(ref)) and torch.equal(y[torch.isinf(y)], ref[torch.isinf(ref)])


@pytest.mark.parametrize("N,C,H,W,O,ks,stride,pad,k", SPECIAL)
def test_conv_wave_infinities_and_nan(tbn, N, C, H, W, O, ks, stride, pad, k):
    """An infinity or a NaN reaches the outputs whose window holds it, as in the one-thread-per-output kernel."""
    g = torch.Generator().manual_seed(C)
    x = torch.randn(N, C, H, W, generator=g)
    x[0, 3, 0, 1], x[0, C - 1, H - 1, W - 1], x[N - 1, 9, 4, 4] = float("inf"), float("-inf"), float("nan")
    x[0, 1, 2, 5], x[0, 2, 2, 5] = float("inf"), float("inf")
    x = x.cuda()
    tile, alpha = tbn.tbn_pack_tile(torch.randn(O * C * ks * ks, generator=g).cuda(), k)
    y = tbn.tbn_conv2d_forward(x, tile, alpha, O, ks, ks, k, stride=(stride, stride), pad=(pad, pad))
    ref = tbn.tbn_conv2d_forward(x, tile, alpha, O, ks, ks, k, stride=(stride, stride), pad=(pad, pad), flags=tbn.TBN_FLAG_FORCE_GENERIC)
    assert torch.isinf(ref).any() and torch.isnan(ref).any()
    assert torch.equal(torch.isnan(y), torch.isnan(ref))
    assert torch.equal(torch.isinf(y), torch.isinf(ref)) and torch.equal(y[torch.isinf(y)], ref[torch.isinf(ref)])


@pytest.mark.parametrize("N,C,H,W,O,ks,stride,pad,k", [(1, 4200, 6, 6, 36, 3, 1, 1, 2), (1, 16, 2, 4096, 40, 1, 1, 0, 2),
                                                      (1, 4100, 5, 9, 24, 3, 2, 1, 9)])
def test_conv_small_activations_keep_all_their_bits(tbn, N, C, H, W, O, ks, stride, pad, k):
    """Layers that tbn_conv_mfma.hip does not take, activations down to the smallest float32 numbers.  In float32 sums each of
    the F additions is off by at most 2^-24 of the partial sum (at most the sum of the magnitudes) or, among subnormal
    numbers, exact."""
    g = torch.Generator().manual_seed(C)
    F, p = C * ks * ks, O * C * ks * ks // k
    x0 = torch.randn(N, C, H, W, generator=g, dtype=torch.float64)
    tile = torch.randint(-2 ** 31, 2 ** 31, ((p + 31) // 32,), generator=g).int()
    bits = np.unpackbits(tile.numpy().view(np.uint8), bitorder="little")[:p]
    sign = torch.from_numpy(bits.astype(np.float64) * 2 - 1).repeat(k).view(O, C, ks, ks)
    tile, alpha = tile.cuda(), torch.ones(1).cuda()
    for e in (0, -105, -112, -118, -126, -134):
        x = (x0 * 2.0 ** e).float()
        y = tbn.tbn_conv2d_forward(x.cuda(), tile, alpha, O, ks, ks, k, stride=(stride, stride), pad=(pad, pad)).double().cpu()
        want = torch.nn.functional.conv2d(x.double(), sign, stride=stride, padding=pad)
        bound = F * 2.0 ** -24 * torch.nn.functional.conv2d(x.double().abs(), sign.abs(), stride=stride, padding=pad) + 2.0 ** -149
        worst = float(((y - want).abs() / bound).max())
        assert worst <= 1.0, (e, worst)
