"""Performance cases: the calls a program that serves tiled-bit layers makes, through the package's public wrappers.

A case is a dict of plain values; its "op" names the path:

* ``linear``   -- one fully-connected layer, ``tbn_linear_forward``;
* ``mlp``      -- two of them, the first with the fused ReLU (a transformer's feed-forward block);
* ``conv``     -- one convolution, ``tbn_conv2d_forward``;
* ``coltiled`` -- one column-tiled layer, ``tbn_linear_coltiled_forward``;
* ``binact``   -- binary activations: ``tbn_sign_pack``, a layer that hands on sign bits, a layer with real outputs;
* ``pack``     -- ``tbn_pack_tile`` on a layer's real weights.

Sizes are those of ``workloads.py`` and ``bench.py`` (the paper's CNN, vision transformer, mixer and transformer layers).
Weights are N(0, 0.02) and activations N(0, 1); the tile and the scalars a program keeps come from the packing calls.
"""
from __future__ import annotations

import math

import torch

from paper_2407_12075_amd import tbn

_DT = {"f32": torch.float32, "bf16": torch.bfloat16}
_ESZ = {"f32": 4, "bf16": 2}


def listed():
    return [
        # one token of a decoder through a 4096 x 4096 projection: latency, launches, host work
        dict(name="linear_decode_b1", op="linear", dt="bf16", M=1, cin=4096, cout=4096, k=8, na=8),
        # a short prompt, a ragged number of tokens
        dict(name="linear_prompt_b300", op="linear", dt="bf16", M=300, cin=4096, cout=4096, k=8, na=8),
        # a large batch through the same projection: the layer the headline metric is quoted on
        dict(name="linear_batch_b8192", op="linear", dt="bf16", M=8192, cin=4096, cout=4096, k=8, na=8),
        # feed-forward up-projection with the mildest compression: the largest matrix product
        dict(name="linear_ffn_up_k2", op="linear", dt="bf16", M=8192, cin=4096, cout=16384, k=2, na=2),
        # tile ends inside weight rows and a row length that is no multiple of 32
        dict(name="linear_misaligned_k9", op="linear", dt="bf16", M=8192, cin=3000, cout=3072, k=9, na=9),
        # feed-forward block of a small vision transformer, 64 images of 197 tokens, float32
        dict(name="mlp_vit_f32", op="mlp", dt="f32", M=197 * 64, cin=384, hid=1536, cout=384, k=4, na=1),
        # token mixing over 196 patches, float32: a row length that is no multiple of 8
        dict(name="linear_mixer_196_f32", op="linear", dt="f32", M=8192, cin=196, cout=384, k=4, na=1),
        # ResNet-style 3x3 convolutions: deep layer with small maps in float32, early layer with large maps in bfloat16
        dict(name="conv_14x14_c256_f32", op="conv", dt="f32", N=128, C=256, H=14, W=14, O=256, ks=3, st=1, pd=1, k=8, na=1),
        dict(name="conv_56x56_c64_bf16", op="conv", dt="bf16", N=32, C=64, H=56, W=56, O=64, ks=3, st=1, pd=1, k=4, na=1),
        # the layout whose columns are tiled, at the headline layer's sizes
        dict(name="coltiled_b8192", op="coltiled", dt="bf16", M=8192, cin=4096, cout=4096, k=8, na=8),
        # binary activations: packing, a hidden layer, an output layer
        dict(name="binact_b8192", op="binact", dt="bf16", M=8192, cin=4096, hid=4096, cout=4096, k=8, na=8),
        # real weights to tile and scalars, after a training step or at load time
        dict(name="pack_4096", op="pack", cin=4096, cout=4096, k=8, na=8),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _round_to(v, m):
    return max(m, (v + m // 2) // m * m)


def _layer_size(rng, lo, hi):
    """A row length or a number of outputs: mostly multiples of 256, some of 8, down to 64."""
    v = _log_int(rng, lo, hi)
    return _round_to(v, 256) if v >= 192 and rng.random() < 0.65 else _round_to(v, 8)


def _draw_linear(rng):
    dt = rng.choice(["bf16", "bf16", "f32"])
    M = _log_int(rng, 1, 12608)
    kind = rng.random()
    if kind < 0.15:      # odd row lengths, tile of whole rows
        k = rng.choice([2, 4, 8])
        cin = rng.randrange(65, 1200)
        cout = k * rng.randrange(8, 1024 // k + 1)
        limit = 6e9
    elif kind < 0.35:    # tile ends inside rows
        cin = _round_to(rng.randrange(256, 3300), 8)
        cout = _round_to(rng.randrange(256, 3300), 8)
        k = rng.choice([k for k in (5, 6, 7, 9, 10, 12, 3, 16, 2, 4) if cin * cout % k == 0])
        limit = 7e10 if dt == "bf16" else 2.5e10
    else:
        cin, cout = _layer_size(rng, 64, 8192), _layer_size(rng, 64, 16384)
        k = rng.choice([2, 4, 4, 8, 8, 16] if cout % 16 == 0 else [2, 4, 4, 8])
        limit = 3e11 if dt == "bf16" else 8e10
    return dict(op="linear", dt=dt, M=M, cin=cin, cout=cout, k=k, na=rng.choice([1, k])), limit


def _draw_mlp(rng):
    dt = rng.choice(["bf16", "f32"])
    cin = _round_to(_log_int(rng, 128, 2048), 64)
    k = rng.choice([2, 4, 8])
    return dict(op="mlp", dt=dt, M=_log_int(rng, 16, 12608), cin=cin, hid=cin * rng.choice([2, 4]), cout=cin, k=k,
                na=rng.choice([1, k])), (1.5e11 if dt == "bf16" else 5e10)


def _draw_conv(rng):
    dt = rng.choice(["bf16", "f32"])
    k = rng.choice([2, 4, 4, 8])
    if rng.random() < 0.2:    # first layer on colour images
        C, O, ks, st = 3, rng.choice([32, 64]), rng.choice([3, 7]), rng.choice([1, 2])
        H, N, limit = _log_int(rng, 28, 224), _log_int(rng, 1, 64), 1e10
    else:
        C = rng.choice([16, 32, 48, 64, 96, 128, 160, 256, 512])
        O = rng.choice([32, 64, 96, 128, 256, 512])
        ks, st = rng.choice([(1, 1), (3, 1), (3, 1), (3, 2), (1, 2)])
        H, N, limit = _log_int(rng, 7, 112), _log_int(rng, 1, 128), 4e10
        if C >= 32 and C * O * ks * ks % 3 == 0 and rng.random() < 0.2:    # tile ends inside filters
            k, limit = 3, 2e10
    W = H if rng.random() < 0.7 else max(7, H - rng.randrange(1, 6))
    return dict(op="conv", dt=dt, N=N, C=C, H=H, W=W, O=O, ks=ks, st=st, pd=ks // 2, k=k, na=rng.choice([1, k])), limit


def _draw_coltiled(rng):
    dt = rng.choice(["bf16", "bf16", "f32"])
    k = rng.choice([2, 4, 8])
    cin = k * _round_to(_log_int(rng, 64, 1024), 64)
    return dict(op="coltiled", dt=dt, M=_log_int(rng, 1, 8192), cin=cin, cout=_layer_size(rng, 64, 8192), k=k,
                na=rng.choice([1, k])), (1e11 if dt == "bf16" else 3e10)


def _draw_binact(rng):
    k = rng.choice([2, 4, 8])
    cin, hid, cout = (_round_to(_log_int(rng, 256, 4096), 256) for _ in range(3))
    return dict(op="binact", dt=rng.choice(["bf16", "f32"]), M=_log_int(rng, 1, 8192), cin=cin, hid=hid, cout=cout, k=k,
                na=rng.choice([1, k])), 3e11


def _draw_pack(rng):
    k = rng.choice([2, 3, 4, 8, 16])
    n = k * _log_int(rng, 2000, 4000000)
    return dict(op="pack", cin=n, cout=1, k=k, na=rng.choice([1, k])), 1e9


def draw(rng):
    """One more case of the same ranges, at most as large as the largest listed one."""
    while True:
        make = rng.choice([_draw_linear, _draw_linear, _draw_linear, _draw_linear, _draw_mlp, _draw_conv, _draw_conv,
                           _draw_conv, _draw_coltiled, _draw_binact, _draw_pack])
        case, limit = make(rng)
        w = work(case)
        if w["flops"] <= limit and w["bytes"] <= 3e8:
            return case


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _acts(shape, dt, g):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(_DT[dt])


def _weights(n, g):
    return torch.randn(n, generator=g, device="cuda", dtype=torch.float32).mul_(0.02)


def prepare(case, seed):
    g = _gen(seed)
    op, s = case["op"], {"case": case}
    if op == "pack":
        s["w"] = _weights(case["cin"] * case["cout"], g)
    elif op == "conv":
        s["x"] = _acts((case["N"], case["C"], case["H"], case["W"]), case["dt"], g)
        s["w1"] = tbn.tbn_pack_tile(_weights(case["O"] * case["C"] * case["ks"] ** 2, g), case["k"], case["na"])
    elif op == "coltiled":
        s["x"] = _acts((case["M"], case["cin"]), case["dt"], g)
        s["w1"] = tbn.tbn_pack_coltile(_weights(case["cout"] * case["cin"], g).view(case["cout"], case["cin"]), case["k"], case["na"])
    else:
        s["x"] = _acts((case["M"], case["cin"]), case["dt"], g)
        sizes = [case["cin"], case["cout"]] if op == "linear" else [case["cin"], case["hid"], case["cout"]]
        for i, (a, b) in enumerate(zip(sizes, sizes[1:])):
            s[f"w{i + 1}"] = tbn.tbn_pack_tile(_weights(a * b, g), case["k"], case["na"])
    return s


def run(s):
    c = s["case"]
    op, k = c["op"], c["k"]
    if op == "linear":
        return tbn.tbn_linear_forward(s["x"], *s["w1"], c["cout"], k)
    if op == "mlp":
        h = tbn.tbn_linear_forward(s["x"], *s["w1"], c["hid"], k, flags=tbn.TBN_FLAG_RELU)
        return tbn.tbn_linear_forward(h, *s["w2"], c["cout"], k)
    if op == "conv":
        return tbn.tbn_conv2d_forward(s["x"], *s["w1"], c["O"], c["ks"], c["ks"], k, stride=(c["st"], c["st"]),
                                      pad=(c["pd"], c["pd"]))
    if op == "coltiled":
        return tbn.tbn_linear_coltiled_forward(s["x"], *s["w1"], c["cout"], k)
    if op == "binact":
        bits = tbn.tbn_sign_pack(s["x"])
        hbits = tbn.tbn_linear_forward_binact(bits, c["cin"], *s["w1"], c["hid"], k, flags=tbn.TBN_FLAG_SIGN_OUT)
        return hbits, tbn.tbn_linear_forward_binact(hbits, c["hid"], *s["w2"], c["cout"], k, dtype=_DT[c["dt"]])
    return tbn.tbn_pack_tile(s["w"], k, c["na"])


def _distinct(rows, row_len, k):
    """Distinct weight rows of the implicit (rows, row_len) weight: what has to be multiplied."""
    p = rows * row_len // k
    return min(rows, p // math.gcd(row_len, p))


def work(case):
    """Inputs read once, outputs written once; multiply-adds of the distinct weight rows."""
    op, k = case["op"], case["k"]
    if op == "pack":
        n = case["cin"] * case["cout"]
        return {"bytes": 4 * n + n // k / 8 + 4 * case["na"], "flops": 2 * n}
    e = _ESZ[case["dt"]]
    if op == "conv":
        F = case["C"] * case["ks"] ** 2
        Ho = (case["H"] + 2 * case["pd"] - case["ks"]) // case["st"] + 1
        Wo = (case["W"] + 2 * case["pd"] - case["ks"]) // case["st"] + 1
        return {"bytes": e * case["N"] * (case["C"] * case["H"] * case["W"] + case["O"] * Ho * Wo) + case["O"] * F / k / 8,
                "flops": 2 * case["N"] * Ho * Wo * F * _distinct(case["O"], F, k)}
    M, cin, cout = case["M"], case["cin"], case["cout"]
    if op == "linear":
        return {"bytes": e * M * (cin + cout) + cin * cout / k / 8, "flops": 2 * M * cin * _distinct(cout, cin, k)}
    if op == "coltiled":
        return {"bytes": e * M * (cin + cout) + cin * cout / k / 8, "flops": 2 * M * (cin // k) * cout}
    hid = case["hid"]
    flops = 2 * M * (cin * _distinct(hid, cin, k) + hid * _distinct(cout, hid, k))
    tiles = (cin * hid + hid * cout) / k / 8
    if op == "mlp":    # the hidden activations are the first layer's output and the second one's input
        return {"bytes": e * M * (cin + 2 * hid + cout) + tiles, "flops": flops}
    return {"bytes": e * M * (cin + cout) + M * (cin + hid) / 4 + tiles, "flops": flops}


def tolerance(case):
    op = case["op"]
    if op == "pack":         # tile bits are equal; scalars are float32 roundings of double sums
        return {"rel": 2e-7}
    if op == "binact":
        return "exact"
    if case["dt"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 1e-2 if op in ("coltiled", "mlp") else 7e-3}    # bfloat16 outputs; two roundings where a bfloat16 value lies between
