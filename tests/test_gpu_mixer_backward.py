"""GPU parity: monarch_mixer_backward (gradients of the gated sequence mixer, Sec. 3.2 Eq. 2) against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import TOL_BF16, TOL_F32, announce, dev, host, rel_l2
from oracle import layer
from paper_2310_12109_amd import workloads

pytestmark = pytest.mark.gpu

KEYS = ("u", "K", "g_in", "g_out", "R1", "L1", "R2", "L2")
GRADS = ("du", "dK", "dg_in", "dg_out", "dR1", "dL1", "dR2", "dL2")


@pytest.fixture(scope="module")
def mm():
    from paper_2310_12109_amd import binding
    return binding


def _check(mm, w, dy, tol, bf16=False):
    got = mm.monarch_mixer_backward(*(dev(w[k], bf16) for k in KEYS), dev(dy, bf16))
    want = layer.mixer_backward(*(w[k] for k in KEYS), dy)
    for name in GRADS:
        if want[name] is None:
            assert got[name] is None
            continue
        assert rel_l2(host(got[name]), want[name]) <= tol, name
    for name in ("dK", "dR1", "dL1", "dR2", "dL2"):
        assert got[name].dtype == torch.float32


def _dy(w, seed, bf16=False):
    dy = np.random.default_rng(seed).standard_normal(w["u"].shape).astype(np.float32)
    return workloads.round_to_bf16(dy) if bf16 else dy


@pytest.mark.parametrize("B,H", [(4, 16), (1, 1), (3, 7), (16, 96)])
def test_n256_fp32(mm, B, H):
    # the matrix-core kernels of the order-2 product and its gradients under the composition; ragged tiles
    announce("mixer backward fp32 b=16 B,H", B, H)
    w = workloads.mixer_inputs(B, H, 16, seed=B + H)
    _check(mm, w, _dy(w, 1), TOL_F32)


@pytest.mark.parametrize("gates", [(True, False), (False, True), (False, False)])
def test_n256_fp32_gates_absent(mm, gates):
    announce("mixer backward fp32 gates", gates)
    w = workloads.mixer_inputs(3, 11, 16, seed=7, gates=gates)
    _check(mm, w, _dy(w, 2), TOL_F32)


@pytest.mark.parametrize("b", [2, 3, 8, 32])
def test_other_block_sizes_fp32(mm, b):
    announce("mixer backward fp32 b", b)
    w = workloads.mixer_inputs(3, 5, b, seed=b)
    _check(mm, w, _dy(w, 3), TOL_F32)


@pytest.mark.parametrize("b,B,H", [(32, 5, 9), (64, 2, 5)])
def test_blocks_of_32_and_64_on_the_matrix_cores(mm, b, B, H):
    # N = 1024, 4096: the products and their gradients of the composition run in place on LDS tiles (fp32 MFMA);
    # 45 and 10 rows: ragged tiles of 16, 8 and 4 rows
    announce("mixer backward fp32 b, B, H", b, B, H)
    w = workloads.mixer_inputs(B, H, b, seed=b + B)
    _check(mm, w, _dy(w, 5), TOL_F32)


@pytest.mark.parametrize("b", [4, 16, 32])
def test_bf16(mm, b):
    # every intermediate row is rounded to bf16 between the kernels
    announce("mixer backward bf16 b", b)
    w = workloads.mixer_inputs(4, 9, b, seed=b, bf16=True)
    _check(mm, w, _dy(w, 4, bf16=True), TOL_BF16, bf16=True)


def test_empty_batch_clears_the_sums(mm):
    announce("mixer backward empty batch")
    w = workloads.mixer_inputs(1, 4, 16, seed=0)
    for k in ("u", "g_in", "g_out"):
        w[k] = w[k][:0]
    got = mm.monarch_mixer_backward(*(dev(w[k]) for k in KEYS), dev(w["u"]))
    torch.cuda.synchronize()
    assert got["du"].shape == (0, 4, 256)
    for name in ("dK", "dR1", "dL1", "dR2", "dL2"):
        assert float(got[name].abs().max()) == 0.0


def test_empty_batch_with_null_inputs_through_the_raw_abi(mm):
    # B = 0 through the C ABI with every input NULL (the header allows it): nothing may be read, and the sums that
    # were asked for come back cleared
    announce("mixer backward empty batch, NULL inputs, raw ABI")
    H, bs = 4, 16
    N = bs * bs
    outs = {name: torch.full((n,), 7.0, device="cuda") for name, n in
            (("dK", H * N), ("dR1", N * bs), ("dL1", N * bs), ("dR2", N * bs), ("dL2", N * bs))}
    lib = mm.raw()
    rc = lib.monarch_mixer_backward(None, None, None, None, None, None, None, None, None,
                                    None, outs["dK"].data_ptr(), None, None,
                                    outs["dR1"].data_ptr(), outs["dL1"].data_ptr(), outs["dR2"].data_ptr(), outs["dL2"].data_ptr(),
                                    0, H, bs, mm.F32, None, 0, torch.cuda.current_stream().cuda_stream)
    assert rc == 0, lib.monarch_last_error()
    torch.cuda.synchronize()
    for name, t in outs.items():
        assert float(t.abs().max()) == 0.0, name


@pytest.mark.parametrize("B,H,gates,bf16", [(1, 40, (True, True), False), (3, 11, (False, True), False), (16, 3, (True, False), False),
                                            (17, 2, (False, False), False), (37, 3, (True, True), True), (40, 128, (True, True), False)])
def test_blocks_of_32_channel_by_channel(mm, B, H, gates, bf16):
    # tiles of 16 rows in the order of the channels: channels that are a part of a tile, that end inside one and that take
    # several, a last tile of 1 to 15 rows, and (40 x 128) workgroups with more than one tile and channels shared by two
    announce("mixer backward b=32 B, H, gates, bf16", B, H, gates, bf16)
    w = workloads.mixer_inputs(B, H, 32, seed=B + H, gates=gates, bf16=bf16)
    _check(mm, w, _dy(w, 6, bf16), TOL_BF16 if bf16 else TOL_F32, bf16=bf16)


# dK is a sum over the sequences in a fixed order, also where workgroups share a channel: parts of it at the ends of two runs of
# tiles, and of whole runs (one channel, many tiles).  The same bits from every call, and a one in each row counted once
@pytest.mark.parametrize("B,H,bf16", [(40, 128, False), (40, 128, True), (20000, 1, False), (4100, 3, True), (1, 600, False)])
def test_blocks_of_32_kernel_gradient_repeats(mm, B, H, bf16):
    announce("mixer backward b=32, dK again and again", B, H, bf16)
    dt = torch.bfloat16 if bf16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(B)
    normal = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)     # noqa: E731
    u, dy, K = normal(B, H, 1024).to(dt), normal(B, H, 1024).to(dt), normal(H, 1024).to(dt)
    m = [(normal(32, 32, 32) * 32 ** -0.5).to(dt) for _ in range(4)]
    first = mm.monarch_mixer_backward(u, K, None, None, *m, dy)["dK"]
    for _ in range(12):
        assert torch.equal(mm.monarch_mixer_backward(u, K, None, None, *m, dy)["dK"], first)
    one = torch.eye(32, device="cuda").expand(32, 32, 32).contiguous().to(dt)     # all blocks the identity: y = K o u up to the order
    got = mm.monarch_mixer_backward(torch.ones_like(u), K, None, None, one, one, one, one, torch.ones_like(u))["dK"]
    assert torch.equal(got, torch.full_like(got, float(B)))


@pytest.mark.parametrize("asked", GRADS)
def test_blocks_of_32_one_output_alone(mm, asked):
    announce("mixer backward b=32, one output:", asked)
    w = workloads.mixer_inputs(5, 7, 32, seed=3)
    dy = _dy(w, 7)
    want = layer.mixer_backward(*(w[k] for k in KEYS), dy)[asked]
    t = [dev(w[k]) for k in KEYS] + [dev(dy)]
    out = torch.full(want.shape, 7.0, device="cuda")
    lib = mm.raw()
    ws = torch.empty(lib.monarch_mixer_backward_workspace_bytes(5, 7, 32, mm.F32), dtype=torch.uint8, device="cuda")
    rc = lib.monarch_mixer_backward(*(v.data_ptr() for v in t), *(out.data_ptr() if name == asked else None for name in GRADS),
                                    5, 7, 32, mm.F32, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0, lib.monarch_last_error()
    assert rel_l2(host(out), want) <= TOL_F32


# An infinite entry in each matrix, bf16 blocks of 32: every other entry is +-1/2 or +-1, so that all sums are exact and most
# values have no lower bf16 parts.  The transposed stages of dx; 16 rows: none repeated in a tile
@pytest.mark.parametrize("factor", ["R", "L"])
def test_infinite_bf16_weights_in_the_product_gradient(mm, factor):
    announce("matmul backward infinite weight", factor)
    b, batch = 32, 16
    g = torch.Generator().manual_seed(5)
    x, dy, R, L = (torch.tensor([-1.0, -0.5, 0.5, 1.0])[torch.randint(4, shape, generator=g)]
                   for shape in ((batch, b * b), (batch, b * b), (b, b, b), (b, b, b)))
    {"R": R, "L": L}[factor][3, 18, 5] = float("inf")
    got = mm.monarch_matmul_backward(*(t.bfloat16().cuda() for t in (x, R, L, dy)))
    mid = torch.einsum("krc,xck->xrk", R.double(), x.double().reshape(batch, b, b))
    d = dy.double().reshape(batch, b, b)      # [s][r]
    dmid = torch.einsum("jlc,xlj->xjc", L.double(), d)
    want = {"dx": torch.einsum("krc,xrk->xck", R.double(), dmid).reshape(batch, b * b),
            "dR": torch.einsum("xrk,xck->krc", dmid, x.double().reshape(batch, b, b)), "dL": torch.einsum("xlj,xjc->jlc", d, mid)}
    assert torch.isinf(want["dx"]).any()
    for name, t in zip(("dx", "dR", "dL"), got):
        w = want[name].to(t.dtype)
        assert torch.equal(torch.isnan(t.cpu()), torch.isnan(w)), name
        assert torch.equal(torch.nan_to_num(t.cpu(), nan=0.25, posinf=3e38, neginf=-3e38), torch.nan_to_num(w, nan=0.25, posinf=3e38, neginf=-3e38)), name
