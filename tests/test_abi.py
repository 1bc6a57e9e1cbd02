"""CPU-side checks of the C ABI: the library loads, exports what include/tbn.h declares, and its
argument validation (which runs before any device call) reports the documented status codes."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "tbn.h")
LIB = os.path.join(ROOT, "paper_2407_12075_amd", "libtbn.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2407_12075_amd import build
        build.build(verbose=False)
    from paper_2407_12075_amd import tbn
    return tbn.lib()


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tbn_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_three_entry_points():
    syms = declared_symbols()
    for name in ("tbn_pack_tile", "tbn_linear_forward", "tbn_conv2d_forward", "tbn_tile_words", "tbn_last_error"):
        assert name in syms


def test_library_exports_every_declared_symbol(lib):
    for name in declared_symbols():
        assert hasattr(lib, name), f"libtbn.so does not export {name}"


def test_tile_words(lib):
    assert lib.tbn_tile_words(65536, 4) == 512
    assert lib.tbn_tile_words(784 * 128, 4) == 784          # 25,088 bits: the microcontroller MLP's first layer
    assert lib.tbn_tile_words(33, 1) == 2
    assert lib.tbn_tile_words(32, 1) == 1
    assert lib.tbn_tile_words(10, 3) == 0                    # k must divide n
    assert lib.tbn_tile_words(0, 1) == 0
    assert lib.tbn_tile_words(8, 0) == 0
    assert lib.tbn_tile_words(4096 * 4096, 8) == 65536


def test_pack_workspace_bytes(lib):
    assert lib.tbn_pack_workspace_bytes(10, 3, 1) == 0
    assert lib.tbn_pack_workspace_bytes(16, 4, 2) == 0
    need = lib.tbn_pack_workspace_bytes(4096 * 4096, 8, 8)
    assert need > 0 and need % 8 == 0


def _err(lib):
    return lib.tbn_last_error().decode()


def test_validation_status_codes(lib):
    p = ctypes.c_void_p
    fake = p(256)  # never dereferenced: validation fails first
    # NULL pointers
    assert lib.tbn_pack_tile(None, None, 16, 2, 1, fake, fake, fake, 1 << 20, None) == 1
    assert "NULL" in _err(lib)
    assert lib.tbn_linear_forward(None, fake, 0, 1, 4, 4, fake, 2, fake, 1, 0, None) == 1
    assert lib.tbn_conv2d_forward(fake, None, 0, 1, 1, 4, 4, 2, 3, 3, 1, 1, 0, 0, fake, 2, fake, 1, 0, None) == 1
    # n not divisible by k, n_alpha not in {1, k}
    assert lib.tbn_pack_tile(fake, None, 10, 3, 1, fake, fake, fake, 1 << 20, None) == 2
    assert "divisible" in _err(lib)
    assert lib.tbn_pack_tile(fake, None, 16, 4, 2, fake, fake, fake, 1 << 20, None) == 2
    assert lib.tbn_linear_forward(fake, fake, 0, 1, 5, 3, fake, 2, fake, 1, 0, None) == 2
    assert lib.tbn_linear_forward(fake, fake, 0, -1, 4, 4, fake, 2, fake, 1, 0, None) == 2
    assert lib.tbn_linear_forward(fake, fake, 0, 1, 0, 4, fake, 2, fake, 1, 0, None) == 2
    # kernel larger than the padded input
    assert lib.tbn_conv2d_forward(fake, fake, 0, 1, 1, 2, 2, 2, 5, 5, 1, 1, 0, 0, fake, 2, fake, 1, 0, None) == 2
    assert lib.tbn_conv2d_forward(fake, fake, 0, 1, 1, 4, 4, 2, 3, 3, 0, 1, 0, 0, fake, 2, fake, 1, 0, None) == 2
    # unknown dtype / flag
    assert lib.tbn_linear_forward(fake, fake, 7, 1, 4, 4, fake, 2, fake, 1, 0, None) == 3
    assert lib.tbn_linear_forward(fake, fake, 0, 1, 4, 4, fake, 2, fake, 1, 0x8000, None) == 3
    assert lib.tbn_conv2d_forward(fake, fake, 9, 1, 1, 4, 4, 2, 3, 3, 1, 1, 0, 0, fake, 2, fake, 1, 0, None) == 3
    # workspace too small / missing / misaligned
    assert lib.tbn_pack_tile(fake, None, 1 << 20, 2, 1, fake, fake, fake, 8, None) == 5
    assert lib.tbn_pack_tile(fake, None, 1 << 20, 2, 1, fake, fake, None, 1 << 30, None) == 5
    assert lib.tbn_pack_tile(fake, None, 1 << 20, 2, 1, fake, fake, p(260), 1 << 30, None) == 5
    # empty batch is legal and touches nothing
    assert lib.tbn_linear_forward(fake, fake, 0, 0, 4, 4, fake, 2, fake, 1, 0, None) == 0
    assert lib.tbn_conv2d_forward(fake, fake, 0, 0, 1, 4, 4, 2, 3, 3, 1, 1, 0, 0, fake, 2, fake, 1, 0, None) == 0


def test_column_tiled_entry_points_validate(lib):
    p = ctypes.c_void_p
    fake = p(256)
    assert lib.tbn_pack_coltile_workspace_bytes(16, 10, 4, 4) == 0       # k must divide in, not just out * in
    assert lib.tbn_pack_coltile_workspace_bytes(16, 12, 4, 4) > 0
    assert lib.tbn_linear_coltiled_workspace_bytes(1, 8, 64, 4) == 8 * 16 * 2 + 256
    assert lib.tbn_linear_coltiled_workspace_bytes(0, 3, 10, 5) == 256 + 256
    assert lib.tbn_linear_coltiled_workspace_bytes(0, 3, 10, 4) == 0
    assert lib.tbn_pack_coltile(None, None, 4, 8, 2, 1, fake, fake, fake, 1 << 20, None) == 1
    assert lib.tbn_pack_coltile(fake, None, 16, 10, 4, 4, fake, fake, fake, 1 << 20, None) == 2
    assert "column blocks" in _err(lib)
    assert lib.tbn_pack_coltile(fake, None, 16, 12, 4, 2, fake, fake, fake, 1 << 20, None) == 2
    assert lib.tbn_pack_coltile(fake, None, 1024, 1024, 2, 1, fake, fake, fake, 8, None) == 5
    assert lib.tbn_linear_coltiled_forward(None, fake, 0, 1, 8, 4, fake, 2, fake, 1, 0, fake, 1 << 20, None) == 1
    assert lib.tbn_linear_coltiled_forward(fake, fake, 0, 1, 10, 4, fake, 4, fake, 1, 0, fake, 1 << 20, None) == 2
    assert lib.tbn_linear_coltiled_forward(fake, fake, 0, 1, 8, 4, fake, 2, fake, 3, 0, fake, 1 << 20, None) == 2
    assert lib.tbn_linear_coltiled_forward(fake, fake, 5, 1, 8, 4, fake, 2, fake, 1, 0, fake, 1 << 20, None) == 3
    assert lib.tbn_linear_coltiled_forward(fake, fake, 0, 1, 8, 4, fake, 2, fake, 1, 0, fake, 16, None) == 5
    assert lib.tbn_linear_coltiled_forward(fake, fake, 0, 1, 8, 4, fake, 2, fake, 1, 0, p(264), 1 << 20, None) == 5
    assert lib.tbn_linear_coltiled_forward(fake, fake, 0, 1, 8, 4, fake, 2, fake, 1, 0, None, 1 << 20, None) == 5
    assert lib.tbn_linear_coltiled_forward(fake, fake, 0, 0, 8, 4, fake, 2, fake, 1, 0, fake, 1 << 20, None) == 0


def test_binding_refuses_host_tensors():
    import torch
    from paper_2407_12075_amd import tbn
    w = torch.zeros(16)
    with pytest.raises(ValueError):
        tbn.tbn_pack_tile(w, 2)


# Which kernel family serves which shape is host arithmetic (shapes, alignment, 256 CUs where there is no device):
# the table the design states, pinned here so that a change of a dispatch rule shows up without a GPU.
KERNEL_CHOICE = [
    # dtype, M, in, out, k, flags, x address, expected family
    ("bf16", 8192, 4096, 4096, 8, 0, 0, "block"),          # the metric shape
    ("bf16", 8192, 4096, 16384, 2, 0, 0, "block"),         # more blocks than CUs: the persistent form of the same kernel
    ("bf16", 4096, 4096, 4096, 8, 0, 0, "stream"),         # at most 128 blocks: 64-row half tiles
    ("bf16", 1024, 4096, 4096, 8, 0, 0, "tile"),           # mid batches: a wave per 32 rows
    ("bf16", 64, 4096, 4096, 8, 0, 0, "small-batch"),
    ("bf16", 16, 4096, 4096, 8, 0, 0, "decode"),
    ("bf16", 1, 4096, 4096, 8, 0, 0, "decode"),
    ("bf16", 16, 4096, 4096, 8, "TBN_FLAG_LARGE_BATCH", 0, "small-batch"),   # the flag keeps the decode kernel out
    ("bf16", 8192, 256, 16384, 4, 0, 0, "general"),        # rows of 256 on a large grid
    ("f32", 12608, 384, 1536, 4, 0, 0, "tile"),            # ViT MLP
    ("f32", 12608, 1536, 384, 4, 0, 0, "tile"),
    ("f32", 8192, 196, 384, 4, 0, 0, "direct"),            # row length no multiple of 8
    ("bf16", 8192, 2050, 1026, 2, 0, 0, "direct"),
    ("bf16", 8192, 4096, 4096, 8, 0, 2, "direct"),         # activations not 16-byte aligned
    ("f32", 64, 24, 10, 3, 0, 0, "generic"),               # tile of no whole rows, row length no multiple of 8
    ("bf16", 8192, 4096, 4096, 8, "TBN_FLAG_FORCE_GENERIC", 0, "generic"),
]


@pytest.mark.parametrize("dtype,M,cin,out,k,flags,x_ptr,expected", KERNEL_CHOICE)
def test_kernel_choice(lib, dtype, M, cin, out, k, flags, x_ptr, expected):
    import torch
    from paper_2407_12075_amd import tbn
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    if isinstance(flags, str):
        flags = getattr(tbn, flags)
    assert tbn.tbn_linear_forward_kernel(dt, M, cin, out, k, 1, flags, x_ptr=x_ptr) == expected


@pytest.mark.parametrize("M,cin,cout,k", [(4, 1024, 6656, 2), (16, 2048, 2048, 2), (13, 1024, 1664, 2)])
def test_flags_of_the_larger_kernels_leave_a_few_rows_to_the_decode_kernel(lib, M, cin, cout, k):
    """Without them the kernel with one wave per 32 rows takes these calls; they keep that one out, not the decode kernel."""
    import torch
    from paper_2407_12075_amd import tbn
    q = lambda flags: tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, 1, flags)
    assert q(0) == "tile"
    assert q(tbn.TBN_FLAG_BLOCK_KERNEL) == q(tbn.TBN_FLAG_STREAM_KERNEL) == "decode"


@pytest.mark.parametrize("M,cin,U,k,expected", [
    (16, 1536, 1192, 32, "tile"), (16, 1536, 1192, 33, "direct"),      # the direct kernel is the other choice
    (14, 3072, 2048, 48, "tile"), (14, 3072, 2048, 49, "direct"),
    (14, 8192, 2048, 96, "tile"), (14, 8192, 2048, 97, "direct"),
    (50, 6656, 2048, 96, "tile"), (50, 6656, 2048, 97, "direct"),
    (7, 4096, 2400, 100, "tile"),                                        # the small-batch kernel is
    (16, 1536, 1024, 64, "tile"), (16, 1536, 1024, 65, "decode"),
    (33, 1024, 1024, 70, "tile"),                                        # more rows: no limit
])
def test_many_replicas_of_a_few_rows(lib, M, cin, U, k, expected):
    import torch
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, U * k, k, 1) == expected


@pytest.mark.parametrize("M,cin,U,k,expected", [
    (64, 768, 256, 16, "small-batch"), (118, 768, 328, 17, "direct"), (118, 768, 328, 32, "direct"),
    (96, 1280, 96, 16, "small-batch"), (95, 1792, 16, 16, "direct"), (95, 1792, 16, 8, "small-batch"), (20, 2816, 1800, 16, "direct"),
    (14, 1280, 104, 16, "small-batch"), (14, 1536, 104, 9, "decode"), (14, 1536, 104, 8, "small-batch"),
])
def test_replicas_in_the_small_batch_kernel(lib, M, cin, U, k, expected):
    """Many replicas of a bfloat16 call stay with the direct and the decode kernel, which store them in wider pieces."""
    import torch
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, U * k, k, 1) == expected


# layers on sign bits with real outputs: the 64 x 64 blocks of the staged kernel end at 384 of them, with long rows at 2048
@pytest.mark.parametrize("dtype,M,cin,out,k,expected", [
    ("bf16", 8192, 4096, 4096, 8, "staged"), ("f32", 2048, 4096, 2048, 2, "staged"),
    ("bf16", 384, 3328, 4096, 1, "staged"),           # 384
    ("bf16", 1947, 3328, 3392, 1, "matrix-core"),     # 1643, one replica
    ("f32", 3406, 3840, 2048, 1, "matrix-core"),
    ("bf16", 2292, 3584, 12288, 4, "matrix-core"),
    ("f32", 2048, 3072, 7 * 1024, 7, "matrix-core"), ("f32", 2048, 3072, 8 * 1024, 8, "staged"),
    ("f32", 2048, 2816, 8 * 1024, 8, "matrix-core"),
    ("bf16", 1000, 3584, 8 * 1600, 8, "matrix-core"), ("bf16", 2300, 3584, 8 * 1024, 8, "staged"),   # a last round of 400 and of 64 in 512
])
def test_kernel_choice_of_layers_on_sign_bits(lib, dtype, M, cin, out, k, expected):
    import torch
    from paper_2407_12075_amd import tbn
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    assert tbn.tbn_linear_forward_binact_kernel(dt, M, cin, out, k, 1) == expected


# layers on sign bits: the form of the 128 x 128 blocks that counts set bits takes all sign bits out that the 64 x 64 blocks leave, and real
# outputs of long rows on more than 384 blocks, both up to rows of 2^22
@pytest.mark.parametrize("dtype,M,cin,U,k,flags,expected,counted", [
    ("f32", 1024, 1024, 1024, 2, 0x4000, "staged", 0), ("f32", 1025, 1024, 1024, 2, 0x4000, "matrix-core", 1),    # 256 and 272 blocks of 64 x 64
    ("f32", 2048, 1280, 1024, 2, 0x4000, "staged", 0), ("f32", 2049, 1280, 1024, 2, 0x4000, "matrix-core", 1),    # rows of more than 1024: 512 and 528
    ("f32", 2048, 1024, 992, 2, 0x4000, "staged", 0), ("f32", 2049, 1024, 992, 2, 0x4000, "matrix-core", 1),      # column blocks of 128 to fill
    ("f32", 449, 1024, 4096, 8, 0x4000, "staged", 0), ("f32", 448, 1024, 4096, 8, 0x4000, "matrix-core", 1),      # eight replicas, 8 - 13 blocks of 64 rows
    ("f32", 832, 768, 2048, 8, 0x4000, "staged", 0), ("f32", 833, 768, 2048, 8, 0x4000, "matrix-core", 1),
    ("f32", 640, 512, 2048, 8, 0x4000, "staged", 0), ("f32", 641, 512, 2048, 8, 0x4000, "matrix-core", 1),        # up to 10
    ("f32", 449, 1024, 4096, 7, 0x4000, "matrix-core", 1), ("f32", 449, 256, 4096, 8, 0x4000, "matrix-core", 1),
    ("f32", 513, 1024, 4096, 8, 0x4000, "matrix-core", 1),                                                        # 576
    ("f32", 4200, 1 << 22, 1024, 1, 0x4000, "matrix-core", 1), ("f32", 4200, (1 << 22) + 256, 1024, 1, 0x4000, "staged", 0),
    ("bf16", 6144, 2304, 1024, 1, 0, "matrix-core", 0), ("bf16", 6145, 2304, 1024, 1, 0, "matrix-core", 1),       # 384 and 392 blocks of 128 x 128
    ("bf16", 6145, 2048, 1024, 1, 0, "matrix-core", 0), ("f32", 6145, 2304, 1000, 1, 0, "matrix-core", 0),        # row length; rows of Y off the lines
    ("f32", 6145, 1 << 22, 1024, 1, 1, "matrix-core", 1), ("f32", 6145, (1 << 22) + 256, 1024, 1, 1, "staged", 0),
])
def test_counted_form_of_layers_on_sign_bits(lib, dtype, M, cin, U, k, flags, expected, counted):
    import torch
    from paper_2407_12075_amd import tbn
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    assert tbn.tbn_linear_forward_binact_kernel(dt, M, cin, U * k, k, k, flags) == expected
    assert tbn.lib().tbn_diag_binact_counted(tbn.TBN_F32 if dtype == "f32" else tbn.TBN_BF16, M, cin, U * k, k, k, flags) == counted
    assert tbn.lib().tbn_diag_binact_counted(tbn.TBN_F32, 0, cin, U * k, k, k, flags) == 0
    assert tbn.lib().tbn_diag_binact_counted(tbn.TBN_F32, M, cin, U * k, k, k + 1, flags) == 0


# bfloat16, rows in multiples of 8 that the general and the windowed kernel both take: M, in, out, k, n_alpha, expected
WINDOW_CHOICE = [
    (3141, 3608, 80, 11, 1, "general"),       # 17.6 tile starts among a block's rows
    (12804, 1560, 128, 3, 1, "general"),      # three
    (1300, 3000, 384, 9, 1, "general"),       # three, as ninths of more rows
    (1300, 3000, 408, 9, 1, "window"),        # 2.8
    (2288, 384, 408, 9, 1, "general"),        # two pairs of rounds: from one start on
    (1200, 264, 3064, 11, 1, "window"),
    (3851, 2072, 152, 7, 7, "general"),       # an alpha per tile copy: 5.9
    (3851, 2080, 152, 5, 5, "window"),        # 4.2
    (16000, 1000, 1088, 1000, 1000, "window"),   # rows of at most 1024
    (21113, 3512, 3552, 12, 1, "general"),    # larger grids: twelve replicas
    (17120, 3000, 3072, 3, 3, "general"),     # three, activations and outputs beyond 170 MB
    (8192, 3000, 3072, 9, 9, "window"),
    (9827, 1312, 1952, 1, 1, "general"),      # rows with a sixth of padding
    (12000, 2984, 2944, 4, 4, "window"),
]


@pytest.mark.parametrize("M,cin,cout,k,n_alpha,expected", WINDOW_CHOICE)
def test_windowed_kernel_leaves_what_the_general_kernel_does_faster(lib, M, cin, cout, k, n_alpha, expected):
    import torch
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, M, cin, cout, k, n_alpha) == expected


def test_kernel_choice_rejects_what_the_forward_call_rejects(lib):
    import torch
    from paper_2407_12075_amd import tbn
    assert tbn.tbn_linear_forward_kernel(torch.float32, 0, 8, 8, 2) == ""     # empty batch: nothing is launched
    assert tbn.tbn_linear_forward_kernel(torch.float32, 4, 4, 4, 3) == ""     # n not divisible by k
    assert tbn.tbn_linear_forward_kernel(torch.float32, 4, 4, 4, 2, n_alpha=3) == ""


def test_convolution_kernel_choice(lib):
    import torch
    from paper_2407_12075_amd import tbn
    q = tbn.tbn_conv2d_forward_kernel
    assert q(torch.float32, 128, 3, 32, 32, 64, 3, 3, 4, pad=(1, 1)) == "direct"            # up to 8 channels
    assert q(torch.float32, 128, 256, 14, 14, 256, 3, 3, 8, pad=(1, 1)).startswith("wave ")
    assert q(torch.bfloat16, 32, 64, 56, 56, 64, 1, 1, 4).startswith("wave ")
    assert q(torch.float32, 4, 64, 14, 14, 64, 9, 1, 4, pad=(4, 0)) == "block"              # nine taps, not 3x3
    assert q(torch.float32, 4, 64, 14, 14, 64, 5, 5, 4, pad=(2, 2)) == "direct"
    assert q(torch.float32, 4, 64, 14, 14, 64, 3, 3, 4, flags=tbn.TBN_FLAG_FORCE_GENERIC) == "generic"
    assert q(torch.float32, 4, 64, 14, 14, 64, 3, 3, 5) == ""                               # k does not divide n
    assert q(torch.float32, 0, 64, 14, 14, 64, 3, 3, 4) == ""


def test_convolution_plans_of_a_network_are_kept(lib):
    """The 1x1 and 3x3 layers of a 50-layer residual network, run in a loop: every plan is searched for once."""
    import torch
    from paper_2407_12075_amd import tbn
    layers, C = [], 64
    for mid, blocks, size in ((64, 3, 56), (128, 4, 28), (256, 6, 14), (512, 3, 7)):
        for b in range(blocks):
            s = 2 if b == 0 and mid > 64 else 1
            H = size * s
            layers += [(C, H, mid, 1, 1), (mid, H, mid, 3, s), (mid, size, 4 * mid, 1, 1)]
            if b == 0:
                layers.append((C, H, 4 * mid, 1, s))
            C = 4 * mid
    assert len(layers) == 52

    def one_pass():
        before = lib.tbn_diag_conv_plan_searches()
        for dt in (torch.float32, torch.bfloat16):
            for (c, h, o, ks, s) in layers:
                name = tbn.tbn_conv2d_forward_kernel(dt, 32, c, h, h, o, ks, ks, 4, stride=(s, s), pad=(ks // 2, ks // 2), n_alpha=4)
                assert name.startswith("wave ")
        return lib.tbn_diag_conv_plan_searches() - before

    assert one_pass() <= 2 * len(set(layers))
    assert one_pass() == 0


def test_binding_works_without_the_extension_module(lib, monkeypatch):
    import sys
    import paper_2407_12075_amd as package
    import torch
    from paper_2407_12075_amd import tbn
    monkeypatch.setitem(sys.modules, "paper_2407_12075_amd._tbn_host", None)   # importing it raises ImportError
    monkeypatch.delattr(package, "_tbn_host", raising=False)
    monkeypatch.setattr(tbn, "_lib", None)
    monkeypatch.setattr(tbn, "_host", None)
    with pytest.warns(UserWarning, match="_tbn_host"):
        assert tbn.lib() is not None
    assert tbn._host is None
    assert tbn.tbn_linear_forward_kernel(torch.bfloat16, 8192, 4096, 4096, 8) == "block"
    with pytest.raises(ValueError):
        tbn.tbn_pack_tile(torch.zeros(16), 2)


def test_library_is_built_where_the_extension_module_cannot_be(tmp_path, monkeypatch, capsys):
    from paper_2407_12075_amd import build
    monkeypatch.setattr(build, "HOST", str(tmp_path / "_tbn_host.so"))
    monkeypatch.setenv("PATH", str(tmp_path))   # no g++
    build._compile_host()
    assert not os.path.exists(build.HOST) and "not built" in capsys.readouterr().err
