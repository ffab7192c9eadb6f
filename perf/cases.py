"""The calls by which the speed of this library is followed from change to change: what a program that uses
paper_2310_12109_amd.binding asks of it, over the range of sizes, element types and options such programs have.

Every case is one call (a training step: forward and gradients; a transform: there and back) on tensors that are in
device memory already.  Outputs and workspaces are the binding's own, as in a call without `out` and `ws`.

`listed()` are named points, `draw()` gives others of the same ranges: ragged lengths, odd batches, both gates or
none, every element type a path is used with.
"""
import math

import torch

from paper_2310_12109_amd import binding, costmodel

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}

# Monarch factors of a padded length, as the tests and the benchmark use them
TWO = {256: (16, 16), 512: (32, 16), 1024: (32, 32), 2048: (64, 32), 4096: (64, 64), 8192: (128, 64), 16384: (128, 128)}
THREE = {4096: (16, 16, 16), 8192: (32, 16, 16), 16384: (32, 32, 16), 32768: (32, 32, 32), 65536: (64, 32, 32),
         131072: (64, 64, 32), 262144: (64, 64, 64)}


def listed():
    return [
        # a single order-2 product on a handful of vectors: launch latency, the smallest call of the library
        dict(name="product_b16_f32_64", kind="product", dtype="f32", b=16, batch=64),
        # sequence mixer of an M2-BERT layer at 128 tokens: bidirectional, so the kernel has both halves of the circle
        dict(name="conv_bidirectional_128_bf16", kind="conv", dtype="bf16", B=32, H=768, n=128, klen=256, nfft=256, order=2,
             gates=3, causal=False),
        # the benchmark convolution: 8 sequences of 1024
        dict(name="conv_causal_1024_bf16", kind="conv", dtype="bf16", B=8, H=768, n=1024, klen=1024, nfft=2048, order=2, gates=3,
             causal=True),
        # long sequences, two factors of 128
        dict(name="conv_causal_8192_bf16", kind="conv", dtype="bf16", B=4, H=768, n=8192, klen=8192, nfft=16384, order=2, gates=3,
             causal=True),
        # one very long sequence, three factors of 64
        dict(name="conv_causal_131072_bf16", kind="conv", dtype="bf16", B=1, H=256, n=131072, klen=131072, nfft=262144, order=3,
             gates=3, causal=True),
        # the same operator in fp32 (evaluation, parity runs), length and batch that divide nothing
        dict(name="conv_causal_2004_f32", kind="conv", dtype="f32", B=7, H=384, n=2004, klen=2004, nfft=4096, order=2, gates=3,
             causal=True),
        # dimension mixer of an M2-BERT layer: 32 sequences of 128 tokens, 4 blocks
        dict(name="mlp_order1_4096_bf16", kind="mlp", dtype="bf16", tokens=4096, d=768, d_hidden=3072, nb=4, order=1),
        # dimension mixer at scale, order 2, 16 blocks
        dict(name="mlp_order2_65536_bf16", kind="mlp", dtype="bf16", tokens=65536, d=1024, d_hidden=4096, nb=16, order=2),
        # training step of the learned sequence mixer at N = 1024: forward and every gradient
        dict(name="mixer_training_1024_f32", kind="mixer_training", dtype="f32", B=16, H=768, b=32, gates=3),
        # the basic M2 layer, n = d = 1024
        dict(name="m2_layer_1024_bf16", kind="m2_layer", dtype="bf16", B=16, bn=32, bd=32),
        # the gated-convolution layer of the causal models: heads of 16 features, 48 heads
        dict(name="hyena_heads_1024_bf16", kind="hyena", dtype="bf16", B=8, n=1024, d=768, head_dim=16, taps=3),
        # the transforms on their own: real rows to a spectrum and back
        dict(name="fft_ifft_2048_bf16", kind="fft", dtype="bf16", rows=6144, nfft=2048, order=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_conv(rng):
    shape = rng.choice(["bidirectional", "causal", "causal", "causal", "long", "f32"])
    gates = rng.choice([0, 1, 2, 3, 3, 3])
    if shape == "long":     # one sequence per channel, three factors
        n = _log_int(rng, 1500, 131072)
        n -= n % 8 if rng.random() < 0.7 else 0
        nfft = min(v for v in THREE if v >= 2 * n)
        H = _log_int(rng, 2, max(2, min(256, 256 * 131072 // n)))
        return dict(kind="conv", dtype="bf16", B=1, H=H, n=n, klen=n, nfft=nfft, order=3, gates=gates, causal=True)
    dtype = "f32" if shape == "f32" else "bf16"
    n = _log_int(rng, 64, 4096 if shape == "f32" else 8192)
    n -= n % 8 if rng.random() < 0.7 else 0
    nfft = min(v for v in TWO if v >= 2 * n)
    if nfft == 2048 and dtype == "bf16" and rng.random() < 0.3:
        dtype = "f16"
    most = (8 * 768 * 1024 if shape == "f32" else 4 * 768 * 8192) // n
    H = rng.choice([64, 96, 256, 384, 500, 768, 1024])
    B = _log_int(rng, 1, max(1, min(64, most // H)))
    if shape == "bidirectional":
        return dict(kind="conv", dtype=dtype, B=B, H=H, n=n, klen=nfft, nfft=nfft, order=2, gates=gates, causal=False)
    klen = n if rng.random() < 0.8 else _log_int(rng, 1, n)
    return dict(kind="conv", dtype=dtype, B=B, H=H, n=n, klen=klen, nfft=nfft, order=2, gates=gates, causal=True)


def draw(rng):
    kind = rng.choice(["product", "conv", "conv", "conv", "mlp", "mlp", "mixer_training", "m2_layer", "hyena", "fft"])
    if kind == "conv":
        return _draw_conv(rng)
    if kind == "product":
        b = rng.choice([16, 16, 32, 64])
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), b=b, batch=_log_int(rng, 1, 2 ** 24 // (b * b)))
    if kind == "mlp":
        d, d_hidden, nb = rng.choice([(768, 3072, 4), (1024, 4096, 16), (512, 2048, 8), (1536, 6144, 8)])
        dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32"])
        tokens = _log_int(rng, 1, 2048 if dtype == "f32" else 65536 * 1024 // max(d, 1024) // (4 if d // nb > 64 else 1))
        return dict(kind=kind, dtype=dtype, tokens=tokens, d=d, d_hidden=d_hidden, nb=nb, order=rng.choice([1, 2]))
    if kind == "mixer_training":
        b = rng.choice([16, 32, 32, 64])
        H = rng.choice([64, 192, 250, 384, 768])
        most = 16 * 768 * 1024 // (b * b) // (4 if b == 64 else 1)
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), B=_log_int(rng, 1, max(1, most // H)), H=H, b=b, gates=rng.choice([0, 3, 3]))
    if kind == "m2_layer":
        bn, bd = rng.choice([(16, 16), (16, 32), (32, 16), (32, 32), (32, 32)])
        return dict(kind=kind, dtype=rng.choice(["f32", "bf16"]), B=_log_int(rng, 1, 16 * 1024 * 1024 // (bn * bn * bd * bd)), bn=bn, bd=bd)
    if kind == "hyena":
        head_dim = rng.choice([1, 1, 4, 16])
        dtype = rng.choice(["bf16", "bf16", "f32"])
        d = rng.choice([256, 384, 768])
        n = 8 * _log_int(rng, 16, 256)
        most = 8 * 1024 * 768 * 16 // (n * d * head_dim) // (8 if dtype == "f32" else 1)
        return dict(kind=kind, dtype=dtype, B=_log_int(rng, 1, max(1, min(64, most))), n=n, d=d, head_dim=head_dim, taps=rng.choice([2, 3, 4]))
    order = rng.choice([2, 2, 3])
    nfft = rng.choice([v for v in (TWO if order == 2 else THREE) if v <= 65536])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    return dict(kind="fft", dtype=dtype, rows=_log_int(rng, 1, 6144 * 2048 // nfft // (2 if dtype == "f32" else 1)), nfft=nfft, order=order)


def _factors(case):
    return (TWO if case["order"] == 2 else THREE)[case["nfft"]]


def prepare(case, seed):
    c, dt = case, DTYPES[case["dtype"]]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, scale=1.0):
        return (torch.randn(*shape, device="cuda", generator=gen) * scale).to(dt)

    def decaying(rows, length, circular=False):
        t = torch.arange(length, device="cuda", dtype=torch.float32)
        lag = torch.minimum(t, length - t) if circular else t
        return (torch.randn(rows, length, device="cuda", generator=gen) * torch.exp(-0.01 * lag)).to(dt)

    s = {"case": c}
    if c["kind"] == "product":
        b = c["b"]
        s.update(x=normal(c["batch"], b * b), R=normal(b, b, b, scale=b ** -0.5), L=normal(b, b, b, scale=b ** -0.5))
    elif c["kind"] == "conv":
        shape = (c["B"], c["H"], c["n"])
        s.update(u=normal(*shape), k=decaying(c["H"], c["klen"], not c["causal"]), factors=_factors(c),
                 g_in=normal(*shape) if c["gates"] & 1 else None, g_out=normal(*shape) if c["gates"] & 2 else None)
    elif c["kind"] == "mlp":
        d, dh, nb = c["d"], c["d_hidden"], c["nb"]
        s.update(x=normal(c["tokens"], d), b1=normal(dh, scale=0.02), b2=normal(d, scale=0.02), W1_L=None, W2_L=None)
        if c["order"] == 1:
            s.update(W1_R=normal(nb, dh // nb, d // nb, scale=0.02), W2_R=normal(nb, d // nb, dh // nb, scale=0.02))
        else:
            s.update(W1_R=normal(nb, d // nb, d // nb, scale=0.02), W1_L=normal(nb, dh // nb, d // nb, scale=0.02),
                     W2_R=normal(nb, d // nb, dh // nb, scale=0.02), W2_L=normal(nb, d // nb, d // nb, scale=0.02))
    elif c["kind"] == "mixer_training":
        b = c["b"]
        shape = (c["B"], c["H"], b * b)
        s.update(u=normal(*shape), K=normal(c["H"], b * b), dy=normal(*shape),
                 g_in=normal(*shape) if c["gates"] & 1 else None, g_out=normal(*shape) if c["gates"] & 2 else None,
                 matrices=[normal(b, b, b, scale=b ** -0.5) for _ in range(4)])
    elif c["kind"] == "m2_layer":
        bn, bd = c["bn"], c["bd"]
        n, d = bn * bn, bd * bd
        s.update(x=normal(c["B"], n, d), n_kernel=normal(d, n), d_kernel=normal(d), beta=normal(d, scale=0.1),
                 gamma=(1.0 + 0.1 * torch.randn(d, device="cuda", generator=gen)).to(dt),
                 seq=[normal(bn, bn, bn, scale=bn ** -0.5) for _ in range(4)], dim=[normal(bd, bd, bd, scale=bd ** -0.5) for _ in range(4)])
    elif c["kind"] == "hyena":
        d, n = c["d"], c["n"]
        s.update(u=normal(c["B"], n, d), W_in=normal(3 * d, d, scale=d ** -0.5), b_in=normal(3 * d, scale=0.1),
                 k_short=normal(3 * d, c["taps"], scale=c["taps"] ** -0.5), k_long=decaying(d // c["head_dim"], n),
                 W_out=normal(d, d, scale=d ** -0.5), b_out=normal(d, scale=0.1), factors=TWO[min(v for v in TWO if v >= 2 * n)])
    else:
        s.update(x=normal(c["rows"], c["nfft"]), factors=_factors(c))
    return s


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "product":
        return binding.monarch_matmul(s["x"], s["R"], s["L"])
    if c["kind"] == "conv":
        return binding.monarch_causal_conv(s["u"], s["k"], s["g_in"], s["g_out"], s["factors"], causal=c["causal"])
    if c["kind"] == "mlp":
        return binding.monarch_mlp(s["x"], s["W1_R"], s["W1_L"], s["b1"], s["W2_R"], s["W2_L"], s["b2"], c["nb"], c["order"], 2, c["d_hidden"])
    if c["kind"] == "mixer_training":
        y = binding.monarch_mixer(s["u"], s["K"], s["g_in"], s["g_out"], *s["matrices"])
        gradients = binding.monarch_mixer_backward(s["u"], s["K"], s["g_in"], s["g_out"], *s["matrices"], s["dy"])
        return dict(gradients, y=y)
    if c["kind"] == "m2_layer":
        return binding.monarch_m2_layer(s["x"], s["seq"], s["n_kernel"], s["dim"], s["d_kernel"], s["gamma"], s["beta"])
    if c["kind"] == "hyena":
        weights = (s["W_in"], s["b_in"], s["k_short"], s["k_long"], s["W_out"], s["b_out"])
        if c["head_dim"] == 1:
            return binding.monarch_hyena_layer(s["u"], *weights, s["factors"])
        return binding.monarch_hyena_heads_layer(s["u"], *weights, s["factors"], c["head_dim"])
    X = binding.monarch_fft(s["x"], s["factors"], True)
    return [X, binding.monarch_ifft(X, s["factors"], True, dtype=s["x"].dtype)]


def work(case):
    """Bytes: every input read once, every output written once.  Operations: the Monarch factors' own products (for the
    convolutions two real rows to a complex transform, the zero half and the dropped half not counted)."""
    c, es = case, 4 if case["dtype"] == "f32" else 2
    if c["kind"] == "product":
        N = c["b"] ** 2
        return {"bytes": (2 * c["batch"] * N + 2 * N * c["b"]) * es, "flops": 4.0 * c["batch"] * N * c["b"]}
    if c["kind"] == "conv":
        rows, gates = c["B"] * c["H"], bin(c["gates"]).count("1")
        return {"bytes": ((2 + gates) * rows * c["n"] + c["H"] * c["klen"]) * es,
                "flops": costmodel.conv_executed_flops(c["B"], c["H"], _factors(c))}
    if c["kind"] == "mlp":
        d, dh, nb, t = c["d"], c["d_hidden"], c["nb"], c["tokens"]
        weights = 2 * d * dh // nb + (2 * d * d // nb if c["order"] == 2 else 0)
        return {"bytes": (2 * t * d + weights + d + dh) * es, "flops": 2.0 * t * weights}
    if c["kind"] == "mixer_training":
        N, rows, gates = c["b"] ** 2, c["B"] * c["H"], bin(c["gates"]).count("1")
        # forward: u, gates, y; gradients: u, gates, dy, du and the gates' gradients; the backward call sees no intermediate
        # of the forward, so it forms the two products again
        act = (2 + gates) + (3 + 2 * gates)
        weights = 2 * (c["H"] * N + 4 * N * c["b"])
        return {"bytes": (act * rows * N + weights) * es + (c["H"] * N + 4 * N * c["b"]) * 4, "flops": 32.0 * rows * N * c["b"]}
    if c["kind"] == "m2_layer":
        n, d = c["bn"] ** 2, c["bd"] ** 2
        return {"bytes": (2 * c["B"] * n * d + n * d + 4 * n * c["bn"] + 4 * d * c["bd"]) * es,
                "flops": 8.0 * c["B"] * n * d * (c["bn"] + c["bd"])}
    if c["kind"] == "hyena":
        B, n, d, dh = c["B"], c["n"], c["d"], c["head_dim"]
        factors = TWO[min(v for v in TWO if v >= 2 * n)]
        return {"bytes": (2 * B * n * d + 4 * d * d + (d // dh) * n) * es,
                "flops": 8.0 * B * n * d * d + costmodel.conv_executed_flops(B * dh * dh, d // dh, factors)}
    elements = c["rows"] * c["nfft"]
    return {"bytes": elements * (2 * es + 2 * 8), "flops": 2 * 4.0 * elements * sum(_factors(c))}


def exact(case, seed):
    """What run() returns for these inputs, by torch's own 64-bit products and Fourier transforms."""
    c, s = case, prepare(case, seed)
    wide = lambda t: None if t is None else [wide(v) for v in t] if isinstance(t, list) else t.double()     # noqa: E731
    s = {name: wide(v) if isinstance(v, (torch.Tensor, list)) else v for name, v in s.items()}

    def product(x, R, L):
        """P L P R P x over the last axis: blocks of R take every nb-th element, blocks of L the row-major middle."""
        z = torch.einsum("krc,xck->xrk", R, x.reshape(-1, R.shape[2], R.shape[0]))
        w = torch.einsum("jlc,xjc->xlj", L, z.reshape(-1, L.shape[0], L.shape[2]))
        return w.reshape(*x.shape[:-1], -1)

    def conv(u, k, g_in, g_out, nfft):
        a = u if g_in is None else u * g_in
        y = torch.fft.irfft(torch.fft.rfft(a, nfft) * torch.fft.rfft(k, nfft), nfft)[..., :u.shape[-1]]
        return y if g_out is None else y * g_out

    if c["kind"] == "product":
        return product(s["x"], s["R"], s["L"])
    if c["kind"] == "conv":
        return conv(s["u"], s["k"], s["g_in"], s["g_out"], c["nfft"])
    if c["kind"] == "mlp":
        def layer(x, R, L):
            if L is None:
                return torch.einsum("krc,xkc->xkr", R, x.reshape(-1, R.shape[0], R.shape[2])).reshape(len(x), -1)
            return product(x, R, L)
        h = torch.nn.functional.gelu(layer(s["x"], s["W1_R"], s["W1_L"]) + s["b1"])
        return layer(h, s["W2_R"], s["W2_L"]) + s["b2"]
    if c["kind"] == "mixer_training":
        names = {"du": s["u"], "dK": s["K"], "dg_in": s["g_in"], "dg_out": s["g_out"]}
        names.update(zip(("dR1", "dL1", "dR2", "dL2"), s["matrices"]))
        leaves = {name: t.requires_grad_() for name, t in names.items() if t is not None}
        a = s["u"] if s["g_in"] is None else s["u"] * s["g_in"]
        y = product(s["K"] * product(a, *s["matrices"][:2]), *s["matrices"][2:])
        y = y if s["g_out"] is None else y * s["g_out"]
        found = dict(zip(leaves, torch.autograd.grad(y, list(leaves.values()), s["dy"])))
        return dict({name: found.get(name) for name in names}, y=y.detach())
    if c["kind"] == "m2_layer":
        mixed = product(torch.relu(s["n_kernel"] * product(s["x"].transpose(1, 2), *s["seq"][:2])), *s["seq"][2:]).transpose(1, 2)
        out = product(torch.relu(s["d_kernel"] * product(mixed, *s["dim"][:2])), *s["dim"][2:])
        return torch.nn.functional.layer_norm(out + mixed, (c["bd"] ** 2,), s["gamma"], s["beta"], 1e-5)
    if c["kind"] == "hyena":
        B, n, d, dh = c["B"], c["n"], c["d"], c["head_dim"]
        p = (s["u"] @ s["W_in"].T + s["b_in"]).transpose(1, 2)
        short = sum(torch.nn.functional.pad(p, (t, 0))[..., :n] * s["k_short"][:, t, None] for t in range(c["taps"]))
        x1, x2, v = short.reshape(B, 3, d // dh, dh, n).unbind(1)
        O = torch.zeros_like(v)
        for i in range(dh):     # the head's i-th feature gates all of its d_h inputs
            inner = conv((x2[:, :, i, None] * v).transpose(1, 2), s["k_long"], None, None, math.prod(s["factors"])).transpose(1, 2)
            O += x1[:, :, i, None] * inner
        return O.reshape(B, d, n).transpose(1, 2) @ s["W_out"].T + s["b_out"]
    X = torch.fft.ifft(s["x"], norm="forward")      # the + sign, unscaled
    return [torch.view_as_real(X.resolve_conj()), s["x"]]


# Largest relative errors seen against the same computation in fp64, over the listed cases and 70 drawn ones: fp32 3.7e-7
# (with the dense projections 1.0e-6); bf16 convolution 5.6e-3, gated-convolution layer 6.5e-3, transforms 4.5e-3, training
# 3.7e-3, MLP 2.5e-3, M2 layer 2.4e-3; fp16 MLP 8.9e-4.  Each bound is two to five times that.
_REL = {("f32", "hyena"): 4e-6, ("bf16", "conv"): 1.5e-2, ("bf16", "hyena"): 1.5e-2, ("bf16", "fft"): 1.2e-2,
        ("bf16", "mixer_training"): 1.2e-2, ("bf16", "mlp"): 8e-3, ("bf16", "m2_layer"): 8e-3, ("bf16", "product"): 7e-3,
        ("f16", "conv"): 2.5e-3, ("f16", "mlp"): 3.5e-3}


def tolerance(case):
    return {"rel": _REL.get((case["dtype"], case["kind"]), 2e-6)}
