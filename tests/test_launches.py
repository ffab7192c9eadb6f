"""Which kernels a call launches, and with which operands it calls rocBLAS: the library's host code on stand-ins for the HIP runtime
(launches.py).  No GPU."""
import pytest

import launches


@pytest.fixture(scope="module")
def recorded(tmp_path_factory):
    so = launches.build(str(tmp_path_factory.mktemp("launches")))
    return lambda script: launches.record(so, script)


# bf16 splits into two factors that are no chunk of the chunk kernels, whose passes hold the spectrum of k in fp32, go to the kernel that
# is fp32 throughout, at any number of rows
def test_splits_whose_kernel_spectrum_is_fp32(recorded):
    got = recorded("""
result = []
for factors in [(16, 32), (32, 16), (16, 64), (64, 16), (16, 128), (128, 16), (32, 128), (128, 32)]:
    nfft = factors[0] * factors[1]
    for B, H in [(1, 1), (1, 4096), (2, 3), (5, 768), (2, 3072), (8, 1536)]:
        for n, klen in [(nfft // 2, nfft // 2), (40, 40), (41, 9), (nfft, nfft)]:
            result.append(calls.conv(B, H, n, klen, factors))
""")
    for kernels in got:
        assert len(kernels) == 1 and kernels[0].startswith("conv_kernel "), kernels


# one sequence per channel, two factors: channels alone up to three rounds of rows for every compute unit, in pairs beyond, at one line
@pytest.mark.parametrize("units", [256, 304, 64])
def test_channels_alone_or_in_pairs(recorded, units):
    got = recorded(f"""
calls.compute_units({units})
result = [[H, n, factors[1], calls.conv(1, H, n, klen, factors)] for factors, n, klen in
          [((128, 64), 4096, 4096), ((128, 64), 48, 8192), ((128, 64), 4095, 4095), ((128, 128), 8192, 16384), ((128, 128), 9, 9)]
          for H in list(range(1, 40)) + [{units} * r + d for r in range(1, 17) for d in (-1, 0, 1)]]
""")
    for H, n, f, kernels in got:
        if n % 8 == 0 and H > 3 * units:
            assert len(kernels) == 3 and kernels[2].startswith(f"fft2_lds_kernel 128 {f} 1 8 6"), (H, n, kernels)
        else:
            assert len(kernels) == 2 and kernels[1].startswith(f"fft2_lds_kernel 128 {f} 0 3 3"), (H, n, kernels)


# threads with a stream each: the products of a call go to its stream, though the threads share the device's rocBLAS handle
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_products_of_threads_go_to_their_own_streams(recorded, dtype):
    products, launched = recorded(f"""
import threading
def work(t):
    for _ in range(25):
        calls.hyena(2, 64, 8, 3, 64, (8, 16), 1, "{dtype}", base=GAP * (1 + 16 * t), stream=1000 + t)
threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
for t in threads: t.start()
for t in threads: t.join()
log = calls.log()
result = [[[int(line[5].split()[0]) // (16 * GAP), int(line[-1])] for line in log if line[0] == "product"],
          [int(line[-1]) for line in log if line[0] == "kernel"]]
""")
    assert len(products) >= 4 * 25 * 2
    assert all(stream == 1000 + thread for thread, stream in products)
    assert all(1000 <= stream < 1004 for stream in launched)


# what rocBLAS is asked to read and write lies inside the caller's tensors and scratch, to the last element, at the smallest and
# the largest calls; C is written by no two entries of a batch
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,n,d,factors,head_dim", [
    (1, 8, 8, (16, 16), 1), (3, 128, 48, (16, 16), 16), (8, 1024, 768, (64, 32), 16), (8, 1024, 768, (64, 32), 1), (64, 128, 768, (16, 16), 1),
    (4, 2048, 768, (64, 64), 16), (32, 1024, 768, (64, 32), 16), (64, 1536, 768, (64, 64), 1), (19, 1240, 384, (64, 64), 4),
])
def test_products_stay_inside_their_tensors(recorded, B, n, d, factors, head_dim, dtype):
    base, gap = 1 << 38, 1 << 38
    ws_bytes, log = recorded(f"""
ws = calls.hyena({B}, {n}, {d}, 3, {n}, {factors}, {head_dim}, "{dtype}", base={base}, gap={gap})
result = [ws, [line[1:] for line in calls.log() if line[0] == "product"]]
""")
    es = 4 if dtype == "f32" else 2
    size = dict(enumerate([B * n * d * es, 3 * d * d * es, 3 * d * es, 9 * d * es, d // head_dim * n * es, d * d * es, d * es, B * n * d * es, ws_bytes]))
    plain, written = 111, 0
    assert len(log) == (2 if dtype == "f32" else 4)
    for ops, mnk, *operands, batch, _type, _stream in log:
        (ta, tb), (m, cols, k), batch = map(int, ops.split()), map(int, mnk.split()), int(batch)
        shapes = [(m, k) if ta == plain else (k, m), (k, cols) if tb == plain else (cols, k), (m, cols)]
        for (rows, columns), operand in zip(shapes, operands):
            at, ld, stride = map(int, operand.split())
            assert ld >= rows and stride >= 0
            end = at + (stride * (batch - 1) + ld * (columns - 1) + rows) * es
            tensor = (at - base) // gap
            assert end <= base + gap * tensor + size[tensor], (operand, rows, columns)
        assert batch == 1 or stride >= ld * (columns - 1) + rows
        written += m * cols * batch
    assert written == 4 * B * n * d


# every convolution and transform finds its kernels, and every instance of the chunk kernels that is built is one that some call takes:
# all splits into two and three factors of 16 ... 128 and others, rows of every kind, few and many
def test_every_call_reaches_a_built_chunk_kernel_and_every_chunk_kernel_is_reached(recorded):
    unreached = recorded("""
import itertools
splits = [f for nf in (2, 3) for f in itertools.product((8, 16, 32, 64, 128, 256), repeat=nf)]
seen = set()
for f in splits:
    nfft = 1
    for v in f: nfft *= v
    if nfft > 1 << 18: continue
    for rows in (1, 3, 5000):
        for real in (0, 1):
            for inverse in (0, 1):
                seen.update(calls.fft(rows, f, "bf16", real, inverse))
    for B, H in ((1, 1), (1, 6), (1, 4000), (2, 3), (3, 3072)):
        for n, klen in ((nfft // 2, nfft // 2), (nfft // 2 - 3, nfft // 2 - 3), (nfft, nfft), (nfft // 2, 9), (7, 16), (nfft - 8, nfft - 5)):
            for gates in (0, 3):
                for dtype in ("bf16", "f16", "f32"):
                    seen.update(calls.conv(B, H, n, klen, f, dtype, gates=gates))
result = sorted(k for k in calls.built() if k.startswith(("fft2_lds_kernel", "conv3_middle_kernel")) and k not in seen)
""")
    assert unreached == []
