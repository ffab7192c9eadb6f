"""GPU parity: monarch_causal_conv against the oracle's direct O(n^2) sum (Eq. 2 / Thm 3)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import TOL_BF16, TOL_F32, announce, dev, host, rel_l2
from paper_2310_12109_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    from paper_2310_12109_amd import binding
    return binding


def _run(mm, w, factors, bf16, causal=True):
    y = mm.monarch_causal_conv(dev(w["u"], bf16), dev(w["k"], bf16), dev(w["g_in"], bf16), dev(w["g_out"], bf16),
                               factors, causal=causal)
    return host(y)


def _oracle(w, nfft, causal=True):
    return oracle.causal_conv(w["u"], w["k"], w["g_in"], w["g_out"], nfft=nfft, causal=causal)


@pytest.mark.parametrize("factors", [(64, 32), (32, 64)])
@pytest.mark.parametrize("bf16", [False, True])
def test_config2_full_tensor(mm, factors, bf16):
    # B=8, H=768, n=1024 zero-padded to 2048: every output element against the direct sum.
    announce("conv c2", factors, "bf16" if bf16 else "fp32")
    c = workloads.CONFIGS["c2_conv"]
    w = workloads.conv_inputs(c["B"], c["H"], c["n"], c["seed"], gates="projected", bf16=bf16)
    y = _run(mm, w, factors, bf16)
    want = _oracle(w, 2048)
    assert rel_l2(y, want) <= (TOL_BF16 if bf16 else TOL_F32)
    # per-row check as well, so that one bad row cannot hide in the global norm
    num = np.linalg.norm((y - want).reshape(-1, c["n"]), axis=1)
    den = np.linalg.norm(want.reshape(-1, c["n"]), axis=1)
    assert (num / den).max() <= (2.5 * TOL_BF16 if bf16 else 5 * TOL_F32)


@pytest.mark.parametrize("bf16", [False, True])
def test_config3a_causal(mm, bf16):
    announce("conv c3a causal", "bf16" if bf16 else "fp32")
    c = workloads.CONFIGS["c3a_conv"]
    w = workloads.conv_inputs(c["B"], c["H"], c["n"], c["seed"], gates="normal", bf16=bf16)
    y = _run(mm, w, (16, 16), bf16)
    assert rel_l2(y, _oracle(w, 256)) <= (TOL_BF16 if bf16 else TOL_F32)


@pytest.mark.parametrize("bf16", [False, True])
def test_config3a_bidirectional(mm, bf16):
    # two-sided kernel of length nfft with negative lags wrapped to the end (causal = 0)
    announce("conv c3a bidirectional", "bf16" if bf16 else "fp32")
    c = workloads.CONFIGS["c3a_conv"]
    w = workloads.conv_inputs(4, c["H"], c["n"], c["seed"], gates="normal", bf16=bf16, two_sided_nfft=256)
    y = _run(mm, w, (16, 16), bf16, causal=False)
    assert rel_l2(y, _oracle(w, 256, causal=False)) <= (TOL_BF16 if bf16 else TOL_F32)


@pytest.mark.parametrize("B,H,n,klen,factors,gates", [
    (3, 5, 100, 37, (16, 16), "normal"),
    (1, 1, 1, 1, (2, 2), "none"),
    (2, 3, 50, 50, (10, 12), "normal"),
    (2, 3, 50, 21, (4, 5, 6), "normal"),
    (3, 2, 512, 512, (8, 8, 16), "none"),
    (5, 7, 1000, 1000, (64, 32), "normal"),
    (1, 2, 128, 128, (16, 32), "normal"),     # nfft = 4n
])
def test_ragged_shapes_fp32(mm, B, H, n, klen, factors, gates):
    announce("conv ragged", B, H, n, klen, factors, gates)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, seed=n + klen, gates=gates)
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    y = _run(mm, w, factors, False)
    assert rel_l2(y, _oracle(w, nfft)) <= TOL_F32


@pytest.mark.parametrize("B,H,n,klen,factors,gates", [
    (3, 5, 100, 37, (16, 16), "normal"),          # odd batch: the last row of each channel travels alone
    (1, 3, 128, 128, (16, 16), "normal"),         # B = 1
    (2, 3, 1000, 999, (32, 64), "none"),
    (5, 2, 2048, 2048, (64, 64), "normal"),
    (4, 3, 1024, 300, (128, 16), "normal"),
    (3, 2, 2000, 2000, (16, 16, 16), "normal"),   # three factors of a length that two are taken for
    (2, 2, 4096, 4096, (32, 16, 64), "normal"),   # nfft = 8n
    (1, 5, 1000, 999, (32, 64), "normal"),        # B = 1, klen odd; H odd
    (1, 4, 2048, 2048, (16, 16, 16), "normal"),
    (1, 5, 16384, 16000, (32, 32, 32), "normal"), # three factors, B = 1: neighbouring channels share a complex row, every chunk
                                                  # stage in one kernel; H odd: the last channel travels alone
    (1, 3, 8000, 5000, (16, 64, 32), "normal"),   # ... unequal chunk factors, nfft > 2n
    (1, 2, 30000, 30000, (64, 32, 32), "none"),
    (3, 3, 8192, 8000, (32, 32, 16), "normal"),   # B > 1: batch entries paired at a stride of H = 3 rows, odd B
    (2, 2, 12288, 12288, (64, 16, 32), "normal"), # three factors that end in no chunk: passes, nfft > 2n
    (1, 2, 3000, 17, (128, 64), "none"),          # short kernel, no gates
])
def test_ragged_shapes_bf16_matrix_core_passes(mm, B, H, n, klen, factors, gates):
    announce("conv bf16 ragged", B, H, n, klen, factors, gates)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, seed=n + klen + 1, gates=gates, bf16=True)
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    y = _run(mm, w, factors, True)
    want = _oracle(w, nfft)
    assert rel_l2(y, want) <= TOL_BF16
    num = np.linalg.norm((y - want).reshape(-1, n), axis=1)
    assert (num / np.linalg.norm(want.reshape(-1, n), axis=1)).max() <= 2.5 * TOL_BF16


def test_single_gate_and_bf16_odd_batch(mm):
    announce("conv one gate, odd B, bf16")
    w = workloads.conv_inputs(3, 4, 1024, seed=8, gates="normal", bf16=True)
    w["g_in"] = None
    y = _run(mm, w, (64, 32), True)
    assert rel_l2(y, _oracle(w, 2048)) <= TOL_BF16
    w2 = workloads.conv_inputs(3, 4, 1024, seed=8, gates="normal", bf16=True)
    w2["g_out"] = None
    y2 = _run(mm, w2, (64, 32), True)
    assert rel_l2(y2, _oracle(w2, 2048)) <= TOL_BF16


@pytest.mark.parametrize("n,klen", [(1000, 1000), (1024, 504), (512, 512), (1024, 1024)])
@pytest.mark.parametrize("gates", ["both", "in", "out", "none"])
def test_fused_64x32_bf16_short_rows_and_each_gate(mm, n, klen, gates):
    # the fused 64 x 32 kernel with rows or kernels shorter than 1024 (zero fill on load, stores past n skipped),
    # with and without each gate; B = 5 leaves the third wave with a lone row and the fourth without work
    announce("conv fused 64x32 bf16 short", n, klen, gates)
    B, H = 5, 6
    w = workloads.conv_inputs(B, H, n, seed=n + klen + len(gates), gates="normal", bf16=True)
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    if gates in ("out", "none"):
        w["g_in"] = None
    if gates in ("in", "none"):
        w["g_out"] = None
    y = _run(mm, w, (64, 32), True)
    want = _oracle(w, 2048)
    assert rel_l2(y, want) <= TOL_BF16
    num = np.linalg.norm((y - want).reshape(-1, n), axis=1)
    assert (num / np.linalg.norm(want.reshape(-1, n), axis=1)).max() <= 2.5 * TOL_BF16


@pytest.mark.parametrize("B", [9, 17, 24])
@pytest.mark.parametrize("n,klen", [(1024, 1024), (1000, 1000), (512, 512)])
def test_fused_64x32_bf16_many_batch_groups(mm, B, n, klen):
    # more than eight batch entries: several workgroups per channel (groups of four row pairs), odd tails
    announce("conv fused 64x32 bf16 groups", B, n, klen)
    H = 5
    w = workloads.conv_inputs(B, H, n, seed=B + n, gates="normal", bf16=True)
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    y = _run(mm, w, (64, 32), True)
    want = _oracle(w, 2048)
    assert rel_l2(y, want) <= TOL_BF16
    num = np.linalg.norm((y - want).reshape(-1, n), axis=1)
    assert (num / np.linalg.norm(want.reshape(-1, n), axis=1)).max() <= 2.5 * TOL_BF16


@pytest.mark.parametrize("B", [5, 9, 16])
@pytest.mark.parametrize("n,klen", [(1024, 1024), (1000, 500), (512, 512), (4, 4)])
@pytest.mark.parametrize("gates", ["both", "in", "out", "none"])
def test_fused_64x32_fp32(mm, B, n, klen, gates):
    # the fp32 fused 64 x 32 kernel: short rows and kernels, each gate combination, odd batch sizes (a lone last
    # row), more than one group of four row pairs per channel
    announce("conv fused 64x32 fp32", B, n, klen, gates)
    H = 3
    w = workloads.conv_inputs(B, H, n, seed=B + n + klen + len(gates), gates="normal")
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    if gates in ("out", "none"):
        w["g_in"] = None
    if gates in ("in", "none"):
        w["g_out"] = None
    y = _run(mm, w, (64, 32), False)
    want = _oracle(w, 2048)
    assert rel_l2(y, want) <= TOL_F32
    num = np.linalg.norm((y - want).reshape(-1, n), axis=1)
    assert (num / np.linalg.norm(want.reshape(-1, n), axis=1)).max() <= 2.5 * TOL_F32


@pytest.mark.parametrize("B,H,n,klen,gates", [
    (3, 5, 8192, 8192, "both"),     # odd batch: the last pair of every channel has one row
    (4, 3, 8000, 8000, "none"),     # rows that end inside a tile row
    (1, 4, 4096, 1000, "in"),       # one sequence per channel, short kernel
    (2, 300, 8192, 512, "out"),     # more channels than compute units: workgroups walk over several
    (6, 2, 128, 8, "both"),         # a single tile row of input
])
def test_fused_128x128_bf16(mm, B, H, n, klen, gates):
    # nfft = 16384 = 128 x 128 with rows of a multiple of 8 elements: the fused kernel (spectrum of k in registers,
    # row pairs through one LDS tile); every output against the direct sum
    announce("conv fused 128x128 bf16", B, H, n, klen, gates)
    w = workloads.conv_inputs(B, H, n, seed=B + H + n + klen, gates="normal", bf16=True)
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    if gates in ("out", "none"):
        w["g_in"] = None
    if gates in ("in", "none"):
        w["g_out"] = None
    y = _run(mm, w, (128, 128), True)
    want = _oracle(w, 16384)
    assert rel_l2(y, want) <= TOL_BF16
    num = np.linalg.norm((y - want).reshape(-1, n), axis=1)
    assert (num / np.linalg.norm(want.reshape(-1, n), axis=1)).max() <= 2.5 * TOL_BF16


def test_delta_kernel_and_causality(mm):
    announce("conv delta / causality")
    B, H, n = 2, 3, 1024
    w = workloads.conv_inputs(B, H, n, seed=5, gates="normal")
    k0 = np.zeros((H, n), dtype=np.float32); k0[:, 0] = 1.0
    w0 = dict(w, k=k0)
    y = _run(mm, w0, (64, 32), False)
    assert rel_l2(y, w["g_out"].astype(np.float64) * w["g_in"] * w["u"]) <= TOL_F32
    # Thm 3: changing u from t0 on leaves y before t0 unchanged (up to rounding on the GPU).
    t0 = 400
    w2 = dict(w, u=w["u"].copy())
    w2["u"][..., t0:] = np.random.default_rng(1).standard_normal((B, H, n - t0)).astype(np.float32)
    ya, yb = _run(mm, w, (64, 32), False), _run(mm, w2, (64, 32), False)
    assert rel_l2(ya[..., :t0], yb[..., :t0]) <= 2 * TOL_F32
    assert rel_l2(ya[..., t0:], yb[..., t0:]) > 1e-2


def test_empty_batch(mm):
    announce("conv empty")
    u = torch.empty((0, 4, 128), device="cuda")
    k = torch.zeros((4, 128), device="cuda")
    y = mm.monarch_causal_conv(u, k, None, None, (16, 16))
    assert y.shape == (0, 4, 128)


def _sampled_rows_check(mm, cfg, bf16, nrows, tol):
    c = workloads.CONFIGS[cfg]
    B, H, n, factors = c["B"], c["H"], c["n"], c["factors"]
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, c["seed"], gates=c["gates"], bf16=bf16)
    y = _run(mm, w, factors, bf16)
    rng = np.random.default_rng(0)
    rows = rng.choice(B * H, size=nrows, replace=False)
    rows[0] = 0; rows[-1] = B * H - 1
    worst = 0.0
    for r in rows:
        b, h = divmod(int(r), H)
        sub = {key: (None if w[key] is None else w[key][b:b + 1, h:h + 1]) for key in ("u", "g_in", "g_out")}
        want = oracle.causal_conv(sub["u"], w["k"][h:h + 1], sub["g_in"], sub["g_out"], nfft=nfft)
        worst = max(worst, rel_l2(y[b, h], want[0, 0]))
    assert worst <= tol
    # library screen over every row (not the oracle): float64 FFT convolution of the same inputs
    gi = 1.0 if w["g_in"] is None else w["g_in"].astype(np.float64)
    go = 1.0 if w["g_out"] is None else w["g_out"].astype(np.float64)
    ref = np.fft.irfft(np.fft.rfft(gi * w["u"], nfft) * np.fft.rfft(w["k"].astype(np.float64), nfft)[None], nfft)[..., :n] * go
    assert rel_l2(y, ref) <= tol


@pytest.mark.parametrize("bf16", [False, True])
def test_config4_sampled_rows(mm, bf16):
    # B=4, H=768, n=8192 padded to 16384 = 128x128: the oracle's direct sum on 16 seeded rows.
    announce("conv c4 sampled", "bf16" if bf16 else "fp32")
    _sampled_rows_check(mm, "c4_conv", bf16, 16, TOL_BF16 if bf16 else TOL_F32)


@pytest.mark.parametrize("bf16", [True])
def test_config5a_order3_sampled_rows(mm, bf16):
    # B=1, H=256, n=131072 padded to 262144 = 64^3: the oracle's direct sum on 2 seeded rows.
    announce("conv c5a sampled", "bf16" if bf16 else "fp32")
    _sampled_rows_check(mm, "c5a_conv", bf16, 2, TOL_BF16 if bf16 else TOL_F32)


# the fp32 kernel that holds a pair of rows in registers: every length it takes, one and several channels per workgroup with
# a remainder, odd n and klen, odd batches, n past half the transform, every gate combination, a two-sided kernel
@pytest.mark.parametrize("B,H,n,klen,factors,gates,causal", [
    (1, 1, 1, 1, (16, 16), "normal", True),
    (5, 17, 127, 128, (16, 16), "normal", False),
    (2, 9, 255, 2, (16, 16), "none", True),
    (3, 9, 251, 250, (32, 16), "normal", True),
    (4, 5, 509, 512, (8, 64), "in", False),
    (7, 5, 511, 511, (32, 32), "out", True),
    (2, 3, 1024, 1023, (64, 32), "normal", True),
    (3, 2, 1500, 549, (64, 32), "in", True),
    (5, 3, 2004, 2004, (64, 64), "normal", True),
    (2, 2, 4001, 96, (16, 16, 16), "out", True),
    (3, 2, 4096, 4096, (128, 64), "normal", True),
    (2, 2, 4097, 8192, (64, 128), "none", False),
])
def test_fp32_rows_in_registers(mm, B, H, n, klen, factors, gates, causal):
    announce("conv fp32 rows in registers", B, H, n, klen, factors, gates, causal)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, seed=n + klen, gates="none" if gates == "none" else "normal")
    w["k"] = np.random.default_rng(klen).standard_normal((H, klen)).astype(np.float32)
    if gates in ("in", "out"):
        w["g_out" if gates == "in" else "g_in"] = None
    # a transform of radix 2..32 steps in fp32: error about 2^-24 sqrt(log2 N), far below the bound of the fp32 paths
    assert rel_l2(_run(mm, w, factors, False, causal), _oracle(w, nfft, causal)) <= TOL_F32


# rows so short that most waves of a workgroup load nothing between the kernel's transform and the first pair's: a slot of
# several waves (lengths 2048 to 8192), its kernel long and short, more pairs than one per slot; every call the same bits
@pytest.mark.parametrize("factors", [(64, 32), (64, 64), (128, 64)])
@pytest.mark.parametrize("n,klen", [(1, 1), (1, 1024), (17, 17), (64, 1000)])
def test_fp32_short_rows_behind_the_kernel_spectrum(mm, factors, n, klen):
    announce("conv fp32 short rows", factors, n, klen)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(5, 600, n, seed=n + klen, gates="none")
    w["k"] = np.random.default_rng(klen).standard_normal((600, klen)).astype(np.float32)
    want = _oracle(w, nfft, False)
    first = _run(mm, w, factors, False, False)
    # Each row by itself, as a wrong spectrum of k is a wrong channel.  The transforms are accurate in the 2-norm, about
    # 2^-24 sqrt(log2 N) each: three of them are below 1e-6 of the largest |F k| times the norm of the rows that share a transform.
    gain = np.abs(np.fft.fft(w["k"].astype(np.float64), nfft)).max(axis=1)
    rows = np.linalg.norm(w["u"].astype(np.float64), axis=2)
    for b in range(5):
        pair = np.hypot(rows[b], rows[min(b ^ 1, 4)])
        assert (np.linalg.norm(first[b] - want[b], axis=1) <= 1e-6 * gain * pair).all(), b
    assert np.array_equal(first, _run(mm, w, factors, False, False))


# Splits of a length that no matrix-core pass takes keep the entries of a batch apart: a row beside one with an infinity, a NaN
# or values of 1e15 is what it is beside itself
@pytest.mark.parametrize("factors", [(8, 64), (8, 8, 16), (256, 8), (4, 1024), (2048, 4)])
def test_fp32_other_splits_keep_rows_apart(mm, factors):
    announce("conv fp32 rows apart", factors)
    nfft = int(np.prod(factors))
    n = nfft // 2 - 3
    w = workloads.conv_inputs(5, 6, n, seed=n, gates="normal")
    w["u"][1] = w["u"][0]
    w["g_in"][1], w["g_out"][1] = w["g_in"][0], w["g_out"][0]
    alone = _run(mm, {k: v if k == "k" else np.ascontiguousarray(v[:1]) for k, v in w.items()}, factors, False)
    assert rel_l2(alone, _oracle(w, nfft)[:1]) <= TOL_F32
    for strange in (np.inf, np.nan, 1e15):
        w["u"][1, :, n // 2] = strange
        y = _run(mm, w, factors, False)
        assert np.array_equal(y[:1], alone), strange
        assert np.isfinite(y[2:]).all()


# 16-bit tensors on the vector unit's transform: every length, rows of any length, all gates, a circular kernel, an odd batch.
# Inputs and products are fp32 there, so what is left is one rounding of the result: at most 2^-9 (bf16) or 2^-12 (fp16) of
# every entry, beside 1e-6 of the transforms.  Splits that no matrix-core pass takes, and fp16, keep the rows apart.
@pytest.mark.parametrize("B,H,n,klen,factors,gates,causal,dtype", [
    (1, 3, 256, 256, (16, 16), "normal", False, torch.bfloat16),
    (5, 9, 255, 200, (32, 16), "normal", True, torch.bfloat16),
    (2, 5, 512, 512, (16, 32), "in", False, torch.bfloat16),
    (3, 4, 503, 503, (32, 32), "out", True, torch.bfloat16),
    (3, 3, 1015, 1015, (64, 32), "normal", True, torch.bfloat16),
    (2, 3, 1016, 2048, (64, 32), "normal", False, torch.float16),
    (3, 3, 1001, 77, (64, 32), "none", True, torch.float16),
    (1, 4, 2047, 2047, (16, 16, 16), "normal", True, torch.bfloat16),
    (2, 3, 2048, 4096, (4, 1024), "normal", False, torch.bfloat16),
    (3, 2, 4095, 4095, (4, 2048), "normal", True, torch.float16),
    # two factors that are no chunk, with as many rows as send the others to the chunk kernels
    (2, 3072, 40, 40, (64, 16), "normal", True, torch.bfloat16),
    (3, 512, 48, 48, (128, 32), "normal", True, torch.bfloat16),
    (3, 4, 1000, 1000, (16, 128), "normal", True, torch.bfloat16),
])
def test_16_bit_rows_in_registers(mm, B, H, n, klen, factors, gates, causal, dtype):
    announce("conv 16-bit rows in registers", B, H, n, klen, factors, gates, causal, dtype)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, seed=n + klen, gates="none" if gates == "none" else "normal")
    w["k"] = np.random.default_rng(klen).standard_normal((H, klen)).astype(np.float32) / np.sqrt(klen)
    if gates in ("in", "out"):
        w["g_out" if gates == "in" else "g_in"] = None
    t = {name: None if v is None else torch.from_numpy(np.ascontiguousarray(v)).cuda().to(dtype) for name, v in w.items()}
    w = {name: None if v is None else v.float().cpu().numpy() for name, v in t.items()}
    y = host(mm.monarch_causal_conv(t["u"], t["k"], t["g_in"], t["g_out"], factors, causal=causal))
    want = _oracle(w, nfft, causal)
    assert rel_l2(y, want) <= (2.0 ** -9 if dtype == torch.bfloat16 else 2.0 ** -12) + 1e-6


# Rows that are no multiple of 8 elements go through the chunk kernels in unaligned pieces, the last one shifted into place: every
# remainder, rows that end with a chunk row or one element behind it, rows shorter than a piece, alone and in pairs
@pytest.mark.parametrize("B", [1, 2, 3])
@pytest.mark.parametrize("n,klen,factors", [
    (4095, 1, (128, 64)), (4089, 4090, (128, 64)), (2057, 2049, (128, 64)), (4090, 3, (64, 128)), (2051, 8, (32, 16, 16)),
    (4092, 15, (128, 64)), (8191, 16383, (128, 128)), (4097, 9, (128, 128)), (9, 5, (128, 64)), (7, 6, (128, 64)), (1, 7, (128, 128)),
    (8189, 8195, (32, 32, 16)),
])
def test_bf16_chunks_rows_of_any_length(mm, B, n, klen, factors):
    announce("conv bf16 chunks, any row length", B, n, klen, factors)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, 3, n, seed=n + klen, gates="normal", bf16=True)
    k = np.random.default_rng(klen).standard_normal((3, klen)) / np.sqrt(klen)
    w["k"] = torch.from_numpy(k).to(torch.bfloat16).float().numpy()
    guard = torch.full((B * 3 * n + 64,), 7.0, device="cuda", dtype=torch.bfloat16)   # nothing past the result is written
    y = host(mm.monarch_causal_conv(dev(w["u"], True), dev(w["k"], True), dev(w["g_in"], True), dev(w["g_out"], True), factors,
                                    causal=False, out=guard[:B * 3 * n].view(B, 3, n)))
    assert rel_l2(y, _oracle(w, nfft, False)) <= TOL_BF16
    assert (guard[B * 3 * n:] == 7.0).all()


# the chunk kernels where many rows take them: whole rows of 1024 and 4096 (short rows, so that the direct sum stays cheap), alone and in
# pairs of batch entries, rows of any length, past half the transform (4096); channels alone and in pairs on both sides of the
# line (three rows for each of 256 compute units), an odd number of them, ragged rows, kernels longer than the rows
@pytest.mark.parametrize("B,H,n,klen,factors", [
    (2, 3072, 40, 40, (32, 32)), (1, 3073, 48, 17, (32, 32)), (5, 1024, 8, 100, (32, 32)),
    (3, 512, 41, 9, (64, 64)), (3, 513, 48, 48, (64, 64)), (1, 1025, 39, 64, (64, 64)), (2, 512, 2051, 3, (64, 64)), (1, 1024, 64, 8, (64, 64)),
    (1, 768, 48, 48, (128, 64)), (1, 769, 48, 50, (128, 64)), (1, 1601, 64, 9, (128, 64)), (1, 770, 648, 5, (128, 64)), (1, 900, 47, 6, (128, 64)),
    (1, 1000, 48, 41, (128, 128)), (1, 1601, 56, 3, (128, 128)), (1, 769, 1160, 4, (128, 128)),
])
@pytest.mark.parametrize("gates", ["normal", "none"])
def test_bf16_chunks_many_rows(mm, B, H, n, klen, factors, gates):
    announce("conv bf16 chunks, many rows", B, H, n, klen, factors, gates)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, seed=n + klen + H, gates=gates, bf16=True)
    k = np.random.default_rng(klen).standard_normal((H, klen)) / np.sqrt(klen)
    w["k"] = torch.from_numpy(k).to(torch.bfloat16).float().numpy()
    y = _run(mm, w, factors, True, False)
    want = _oracle(w, nfft, False)
    assert rel_l2(y, want) <= TOL_BF16
    # every row by itself against the larger of the two that share a transform: one bf16 error of the transform is in both
    num, den = np.linalg.norm(y - want, axis=2), np.linalg.norm(want, axis=2)
    assert (num <= 2.5 * TOL_BF16 * den.max()).all()


# three factors beyond 16384: every chunk shape, batch entries in pairs (six launches), an odd batch, rows that end inside a row
# of a chunk; one sequence per channel in the shapes that have no fused middle
@pytest.mark.parametrize("B,H,n,klen,factors", [
    (3, 3, 700, 300, (32, 32, 32)), (2, 2, 16384, 900, (32, 32, 32)), (3, 2, 701, 65, (64, 64, 32)), (2, 3, 700, 300, (16, 32, 64)),
    (5, 2, 333, 77, (16, 64, 64)), (3, 3, 700, 300, (128, 16, 16)), (2, 3, 700, 300, (16, 128, 64)), (3, 2, 700, 300, (16, 64, 128)),
    (3, 2, 700, 300, (16, 128, 128)), (1, 1, 700, 300, (32, 32, 32)),
    (1, 3, 700, 300, (16, 128, 64)), (1, 4, 701, 33, (16, 64, 128)), (1, 3, 9000, 300, (16, 128, 128)),
])
def test_bf16_three_factor_chunks(mm, B, H, n, klen, factors):
    announce("conv bf16 chunks, three factors", B, H, n, klen, factors)
    nfft = int(np.prod(factors))
    w = workloads.conv_inputs(B, H, n, seed=n + klen, gates="normal", bf16=True)
    w["k"] = np.ascontiguousarray(w["k"][:, :klen])
    y = _run(mm, w, factors, True)
    want = _oracle(w, nfft)
    assert rel_l2(y, want) <= TOL_BF16
    num = np.linalg.norm((y - want).reshape(-1, n), axis=1)
    assert (num / np.linalg.norm(want.reshape(-1, n), axis=1)).max() <= 2.5 * TOL_BF16
