"""The extension module that makes the binding's plain calls: the same results as the wrappers' own code, the caller's
stream, and None (so the wrapper's own code and its errors) for every other form of a call."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tbn():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_12075_amd import tbn as binding
    binding.lib()
    assert binding._host is not None
    return binding


def _layer(tbn, dt, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(40, 96, generator=g, device="cuda").to(dt)
    w = torch.randn(64 * 96, generator=g, device="cuda")
    return x, w


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
def test_same_results_as_the_wrappers_own_code(tbn, dt, monkeypatch):
    x, w = _layer(tbn, dt)
    img = x[:, :96].reshape(5, 12, 8, 8).contiguous()

    def calls():
        tile, alpha = tbn.tbn_pack_tile(w, 4, 4)
        ct, ca = tbn.tbn_pack_coltile(w.view(64, 96), 4, 4)
        bits = tbn.tbn_sign_pack(x)
        return [tile, alpha, tbn.tbn_linear_forward(x, tile, alpha, 64, 4, flags=tbn.TBN_FLAG_RELU),
                tbn.tbn_linear_forward(x[:0], tile, alpha, 64, 4),
                tbn.tbn_linear_coltiled_forward(x, ct, ca, 64, 4), bits,
                tbn.tbn_linear_forward_binact(bits, 96, tile, alpha, 64, 4, flags=tbn.TBN_FLAG_SIGN_OUT),
                tbn.tbn_linear_forward_binact(bits, 96, tile, alpha, 64, 4, dtype=dt),
                tbn.tbn_conv2d_forward(img, *tbn.tbn_pack_tile(w[:16 * 12 * 9], 4), 16, 3, 3, 4, stride=(2, 1), pad=(1, 0))]

    fast = calls()
    monkeypatch.setattr(tbn, "_host", None)
    slow = calls()
    torch.cuda.synchronize()
    for f, s in zip(fast, slow):
        assert f.dtype == s.dtype and f.shape == s.shape and f.device == s.device and not f.requires_grad
        assert torch.equal(f, s)


def test_other_forms_are_left_to_the_wrapper(tbn):
    x, w = _layer(tbn, torch.float32)
    tile, alpha = tbn.tbn_pack_tile(w, 4)
    h = tbn._host

    class Sub(torch.Tensor):
        pass

    assert h.linear_forward(x, tile, alpha, 64, 4, 0) is not None
    for bad in [(x.cpu(), tile, alpha, 64, 4, 0), (x.t(), tile, alpha, 64, 4, 0), (x[:, ::2], tile, alpha, 64, 4, 0),
                (x.half(), tile, alpha, 64, 4, 0), (x[0], tile, alpha, 64, 4, 0), (x.as_subclass(Sub), tile, alpha, 64, 4, 0),
                (x, tile[:-1], alpha, 64, 4, 0), (x, tile.cpu(), alpha, 64, 4, 0), (x, tile.float(), alpha, 64, 4, 0),
                (x, tile, alpha.double(), 64, 4, 0), (x, tile, alpha[:0], 64, 4, 0), (x, tile, alpha, 64.0, 4, 0),
                (x, tile, alpha, True, 4, 0), (x, tile, alpha, 64, 0, 0), (x, tile, alpha, 64, 5, 0), (x, tile, alpha, 64, 4, -1),
                (x, tile, alpha, 64, 1 << 70, 0), (None, tile, alpha, 64, 4, 0), (x, tile, alpha)]:
        assert h.linear_forward(*bad) is None
    assert h.pack_tile(w, 5, 1) is None and h.pack_tile(w, 4, 2) is None and h.sign_pack(x.cpu()) is None
    img = x[:4, :96].reshape(1, 6, 8, 8).contiguous()
    assert h.conv2d_forward(img, tile, alpha, 4, 9, 9, 4, (1, 1), (0, 0), 0) is None
    assert h.conv2d_forward(img, tile, alpha, 4, 3, 3, 4, [1, 1], (0, 0), 0) is None
    with pytest.raises(ValueError):
        tbn.tbn_linear_forward(x.t(), tile, alpha, 64, 4)
    with pytest.raises(tbn.TbnError):
        tbn.tbn_linear_forward(x, tile, alpha, 64, 4, flags=0x80000)
    from torch.utils._python_dispatch import TorchDispatchMode

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    with Mode():
        assert h.linear_forward(x, tile, alpha, 64, 4, 0) is None
    from torch.overrides import TorchFunctionMode
    seen = []

    class FunctionMode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func)
            return func(*args, **(kwargs or {}))

    with FunctionMode():
        assert h.linear_forward(x, tile, alpha, 64, 4, 0) is None
        tbn.tbn_linear_forward(x, tile, alpha, 64, 4)
    assert torch.empty in seen   # the wrapper's own allocation of the output
    torch.cuda.synchronize()


def test_streams_and_threads(tbn):
    x, w = _layer(tbn, torch.bfloat16)
    tile, alpha = tbn.tbn_pack_tile(w, 4)
    want = tbn.tbn_linear_forward(x, tile, alpha, 64, 4)
    torch.cuda.synchronize()
    got = [None] * 4

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            big = torch.full((2048, 2048), 0.5, device="cuda")
            x2 = x * (big @ big).flatten()[0].div(512.0).to(x.dtype)   # x again, written on this stream behind some work
            ys = [tbn.tbn_linear_forward(x2, tile, alpha, 64, 4) for _ in range(20)]
            s.synchronize()
        got[i] = all(torch.equal(y, want) for y in ys)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [True] * 4
