"""GPU parity: monarch_matmul_backward (gradients of the order-2 Monarch product, Sec. 3.1) against the oracle."""
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


def _dy(batch, d_out, seed, bf16=False):
    dy = np.random.default_rng(seed).standard_normal((batch, d_out)).astype(np.float32)
    return workloads.round_to_bf16(dy) if bf16 else dy


def _check(mm, w, dy, tol, bf16=False):
    dx, dR, dL = mm.monarch_matmul_backward(dev(w["x"], bf16), dev(w["R"], bf16), dev(w["L"], bf16), dev(dy, bf16))
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    assert dR.dtype == torch.float32 and dL.dtype == torch.float32
    assert rel_l2(host(dx), wdx) <= tol
    assert rel_l2(host(dR), wdR) <= tol
    assert rel_l2(host(dL), wdL) <= tol


@pytest.mark.parametrize("batch", [64, 67, 1, 1000, 5000])
def test_config1_square_fp32(mm, batch):
    # several tiles, a ragged last tile, more tiles than workgroups (batch 5000)
    announce("matmul backward c1 fp32 batch", batch)
    w = workloads.monarch_matmul_inputs(batch=batch, b=16, seed=0)
    _check(mm, w, _dy(batch, 256, batch), TOL_F32)


def test_config1_more_tiles_than_workgroups(mm):
    # 1251 tiles of 16 vectors on at most 512 workgroups: every workgroup walks over several tiles and keeps its
    # share of dR, dL in registers across them; the last tile is ragged
    batch = 20011
    announce("matmul backward c1 fp32 batch", batch)
    w = workloads.monarch_matmul_inputs(batch=batch, b=16, seed=1)
    _check(mm, w, _dy(batch, 256, 2), TOL_F32)


@pytest.mark.parametrize("b", [2, 8, 32, 64])
def test_square_other_block_sizes(mm, b):
    announce("matmul backward square b", b)
    w = workloads.monarch_matmul_inputs(batch=19, b=b, seed=b)
    _check(mm, w, _dy(19, b * b, b), TOL_F32)


@pytest.mark.parametrize("shape", [(4, 3, 2, 2, 5, 6), (4, 192, 192, 4, 768, 192), (16, 64, 64, 16, 256, 64), (3, 7, 5, 7, 2, 3)])
def test_rectangular_fp32(mm, shape):
    announce("matmul backward rect", shape)
    nbR, r_out, r_in, nbL, l_out, l_in = shape
    w = workloads.monarch_matmul_rect_inputs(37, *shape, seed=11)
    _check(mm, w, _dy(37, nbL * l_out, 12), TOL_F32)


@pytest.mark.parametrize("batch", [1, 67, 5000, 20011])
def test_bf16_config1_shape_on_the_matrix_cores(mm, batch):
    # bf16 tensors through the fp32 MFMA kernel: ragged tiles, more tiles than workgroups; dx is rounded to bf16,
    # dR and dL are fp32 sums of products of bf16 values
    announce("matmul backward bf16 b=16 batch", batch)
    w = workloads.monarch_matmul_inputs(batch=batch, b=16, seed=batch, bf16=True)
    dy = _dy(batch, 256, batch + 1, bf16=True)
    dx, dR, dL = mm.monarch_matmul_backward(dev(w["x"], True), dev(w["R"], True), dev(w["L"], True), dev(dy, True))
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    assert dx.dtype == torch.bfloat16 and rel_l2(host(dx), wdx) <= TOL_BF16
    assert rel_l2(host(dR), wdR) <= 10 * TOL_F32 and rel_l2(host(dL), wdL) <= 10 * TOL_F32


@pytest.mark.parametrize("batch", [1, 16, 100, 9000])
@pytest.mark.parametrize("bf16", [False, True])
def test_blocks_of_32_on_the_matrix_cores(mm, batch, bf16):
    # N = 1024: both factors, their transposes and the factor gradients in place on two LDS tiles of 16 rows; ragged
    # last tile, and (batch 9000) more tiles than workgroups, so the sums stay in registers over several tiles
    announce("matmul backward b=32 batch", batch, "bf16" if bf16 else "fp32")
    w = workloads.monarch_matmul_inputs(batch=batch, b=32, seed=batch + 7, bf16=bf16)
    dy = _dy(batch, 1024, batch + 8, bf16=bf16)
    dx, dR, dL = mm.monarch_matmul_backward(dev(w["x"], bf16), dev(w["R"], bf16), dev(w["L"], bf16), dev(dy, bf16))
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    assert rel_l2(host(dx), wdx) <= (TOL_BF16 if bf16 else TOL_F32)
    assert rel_l2(host(dR), wdR) <= 10 * TOL_F32 and rel_l2(host(dL), wdL) <= 10 * TOL_F32


@pytest.mark.parametrize("batch", [1, 5, 100, 1500])
@pytest.mark.parametrize("bf16", [False, True])
def test_blocks_of_64_on_the_matrix_cores(mm, batch, bf16):
    # N = 4096: dx from one tile of eight rows; dL and dR from workgroups that each sum a group of 16 blocks over a slice
    # of the rows (tiles of four rows; batch 1500: several tiles per workgroup, ragged last tile)
    announce("matmul backward b=64 batch", batch, "bf16" if bf16 else "fp32")
    w = workloads.monarch_matmul_inputs(batch=batch, b=64, seed=batch + 9, bf16=bf16)
    dy = _dy(batch, 4096, batch + 10, bf16=bf16)
    dx, dR, dL = mm.monarch_matmul_backward(dev(w["x"], bf16), dev(w["R"], bf16), dev(w["L"], bf16), dev(dy, bf16))
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    assert rel_l2(host(dx), wdx) <= (TOL_BF16 if bf16 else TOL_F32)
    assert rel_l2(host(dR), wdR) <= 10 * TOL_F32 and rel_l2(host(dL), wdL) <= 10 * TOL_F32


def test_blocks_of_64_partial_outputs(mm):
    announce("matmul backward b=64 partial outputs")
    w = workloads.monarch_matmul_inputs(batch=21, b=64, seed=31)
    dy = _dy(21, 4096, 32)
    x, R, L, g = dev(w["x"]), dev(w["R"]), dev(w["L"]), dev(dy)
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dR=False, need_dL=False)
    assert dR is None and dL is None and rel_l2(host(dx), wdx) <= TOL_F32
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dx=False, need_dR=False)
    assert dx is None and dR is None and rel_l2(host(dL), wdL) <= TOL_F32
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dx=False, need_dL=False)
    assert dx is None and dL is None and rel_l2(host(dR), wdR) <= TOL_F32


def test_blocks_of_32_partial_outputs(mm):
    announce("matmul backward b=32 partial outputs")
    w = workloads.monarch_matmul_inputs(batch=50, b=32, seed=21)
    dy = _dy(50, 1024, 22)
    x, R, L, g = dev(w["x"]), dev(w["R"]), dev(w["L"]), dev(dy)
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dR=False, need_dL=False)
    assert dR is None and dL is None and rel_l2(host(dx), wdx) <= TOL_F32
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dx=False, need_dR=False)
    assert dx is None and dR is None and rel_l2(host(dL), wdL) <= TOL_F32
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dx=False, need_dL=False)
    assert dx is None and dL is None and rel_l2(host(dR), wdR) <= TOL_F32
    again = mm.monarch_matmul_backward(x, R, L, g)   # overwritten, not accumulated
    assert rel_l2(host(again[1]), wdR) <= TOL_F32 and rel_l2(host(again[2]), wdL) <= TOL_F32 and rel_l2(host(again[0]), wdx) <= TOL_F32


# one gradient alone has an instance of its own, two or three share one: one tile with a single row, a ragged one, several tiles
# per workgroup.  dx is the same sum in each (the same bits), dR and dL by atomic adds.
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("batch", [1, 37, 4100])
def test_blocks_of_32_every_set_of_gradients(mm, batch, bf16):
    announce("matmul backward b=32 sets of gradients", batch, bf16)
    w = workloads.monarch_matmul_inputs(batch=batch, b=32, seed=batch + 40, bf16=bf16)
    x, R, L, g = dev(w["x"], bf16), dev(w["R"], bf16), dev(w["L"], bf16), dev(_dy(batch, 1024, batch + 41, bf16=bf16), bf16)
    full = [host(t) for t in mm.monarch_matmul_backward(x, R, L, g)]
    for asked in range(1, 7):
        need = [bool(asked >> i & 1) for i in range(3)]
        got = mm.monarch_matmul_backward(x, R, L, g, *need)
        assert [t is not None for t in got] == need
        if need[0]:
            assert np.array_equal(host(got[0]), full[0])
        for i in (1, 2):
            if need[i]:
                assert rel_l2(host(got[i]), full[i]) <= TOL_F32


def test_bf16_inputs(mm):
    announce("matmul backward bf16")
    w = workloads.monarch_matmul_inputs(batch=130, b=16, seed=3, bf16=True)
    _check(mm, w, _dy(130, 256, 4, bf16=True), TOL_BF16, bf16=True)


def test_outputs_can_be_skipped_and_are_overwritten(mm):
    announce("matmul backward partial outputs")
    w = workloads.monarch_matmul_inputs(batch=40, b=16, seed=5)
    dy = _dy(40, 256, 6)
    x, R, L, g = dev(w["x"]), dev(w["R"]), dev(w["L"]), dev(dy)
    wdx, wdR, wdL = oracle.matmul_backward(w["x"], w["R"], w["L"], dy)
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dR=False, need_dL=False)
    assert dR is None and dL is None and rel_l2(host(dx), wdx) <= TOL_F32
    dx, dR, dL = mm.monarch_matmul_backward(x, R, L, g, need_dx=False)
    assert dx is None and rel_l2(host(dR), wdR) <= TOL_F32 and rel_l2(host(dL), wdL) <= TOL_F32
    # a second call into the same (non-zero) buffers gives the same result: overwritten, not accumulated
    again = mm.monarch_matmul_backward(x, R, L, g, need_dx=False)
    assert rel_l2(host(again[1]), wdR) <= TOL_F32


def test_identity_blocks_give_the_transposed_permutation_exactly(mm):
    announce("matmul backward identity")
    b = 16
    eye = np.broadcast_to(np.eye(b, dtype=np.float32), (b, b, b)).copy()
    x = np.random.default_rng(7).standard_normal((33, b * b)).astype(np.float32)
    dy = _dy(33, b * b, 8)
    dx, _, _ = mm.monarch_matmul_backward(dev(x), dev(eye), dev(eye), dev(dy), need_dR=False, need_dL=False)
    s = oracle.perm(b, b * b)
    want = np.zeros_like(dy)
    want[:, s] = dy
    assert np.array_equal(host(dx), want.astype(np.float64))


def test_empty_batch_gives_zero_parameter_gradients(mm):
    announce("matmul backward empty")
    w = workloads.monarch_matmul_inputs(batch=1, b=16, seed=0)
    x = torch.empty((0, 256), device="cuda")
    dx, dR, dL = mm.monarch_matmul_backward(x, dev(w["R"]), dev(w["L"]), torch.empty((0, 256), device="cuda"))
    assert dx.shape == (0, 256) and float(dR.abs().max()) == 0.0 and float(dL.abs().max()) == 0.0
