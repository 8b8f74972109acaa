"""GPU BFP16 quantiser / decoder vs the oracle: bit-exact (runs on an MI355X)."""
import numpy as np
import pytest

import oracle
import paper_2511_16041_amd as atb
import workloads
from helpers import bf16_tensor_bits, pack_a_bfp, unpack_a_bfp

pytestmark = pytest.mark.gpu


def _quantize_gpu(A):
    import torch
    At = torch.from_numpy(A).cuda()
    buf = atb.bfp16_quantize(At)
    torch.cuda.synchronize()
    M, K = A.shape
    lay = atb.bfp16_layout(M, K)
    return buf, unpack_a_bfp(buf.cpu().numpy(), M, K, lay)


@pytest.mark.parametrize("name,M,K", [("small256", 256, 256), ("ragged", 300, 264), ("ragged", 37, 4104),
                                      ("mlp", 129, 1024), ("small256", 1, 8), ("ragged", 5, 24)])
def test_quantizer_bit_exact(name, M, K):
    print(f"quantize {name} M={M} K={K}", flush=True)
    A, _ = workloads.make_inputs(workloads.CONFIGS[name], M=M, N=8, K=K)
    mant, expo = oracle.quantize(A)
    _, (gm, ge, pad) = _quantize_gpu(A)
    assert np.array_equal(ge, expo)
    assert np.array_equal(gm, mant)
    assert not pad.any()                       # mantissa padding is zero


def test_quantizer_special_blocks():
    """Zero blocks, ties, saturation to +-127, tiny and huge exponents."""
    rows = [
        [1.0, 0.5, -0.75, 2 ** -7, 1.5 * 2 ** -7, 255 / 128, -1.0, 0.0],
        [1.0, 1.5 / 64, 2.5 / 64, 3.5 / 64, -0.5 / 64, -1.5 / 64, 0.0, 0.0],
        [0.0, -0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0],
        [256.0, 1.0, -1.0, 1.9, 2.0, -3.0, 0.99, 0.0],
        [3.999, -3.999, 2.0, 0.03125, 0.0, 0.0, 0.0, 0.0],
        [3.0e38, -3.4e38, 1e38, 0, 0, 0, 0, 0],
        [1e-30, -3e-31, 2e-32, 0, 0, 0, 0, 1e-35],
        [1.17549435e-38, 1e-38, -1.2e-38, 0, 0, 0, 0, 0],          # around the smallest normal fp32
    ]
    A = np.array(rows, dtype=np.float32)
    A = np.concatenate([A, A[:, ::-1]], axis=1)                    # two blocks per row
    mant, expo = oracle.quantize(A)
    _, (gm, ge, _) = _quantize_gpu(A)
    assert np.array_equal(ge, expo) and np.array_equal(gm, mant)


def test_quantizer_row_pitch():
    import torch
    A, _ = workloads.make_inputs(workloads.CONFIGS["small256"], M=33, N=8, K=72)
    big = torch.zeros((33, 80), dtype=torch.float32, device="cuda")
    big[:, :72] = torch.from_numpy(A).cuda()
    buf = atb.bfp16_quantize(big[:, :72])                          # lda = 80
    torch.cuda.synchronize()
    gm, ge, _ = unpack_a_bfp(buf.cpu().numpy(), 33, 72, atb.bfp16_layout(33, 72))
    mant, expo = oracle.quantize(A)
    assert np.array_equal(ge, expo) and np.array_equal(gm, mant)


def test_decode_exact():
    import torch
    A, _ = workloads.make_inputs(workloads.CONFIGS["ragged"], M=70, N=8, K=264)
    mant, expo = oracle.quantize(A)
    buf, _ = _quantize_gpu(A)
    dec = atb.bfp16_decode(buf, 70, 264)
    torch.cuda.synchronize()
    got = oracle.bf16_to_double(bf16_tensor_bits(dec))
    assert np.array_equal(got, oracle.decode(mant, expo))


@pytest.mark.parametrize("M,K", [(3, 520), (4, 512), (6, 1032), (6150, 2056), (6145, 2048), (65533, 72), (65552, 256), (65537, 8)])
def test_quantizer_rows_per_workgroup(M, K):
    """Workgroups of 4 rows (small problems), of 8 (above 3072 of the small ones) and of 16 (many narrow rows), with whole and partial
    last ones."""
    print(f"quantize {(M, K)}", flush=True)
    A, _ = workloads.make_inputs(workloads.CONFIGS["ragged"], M=M, N=8, K=K)
    mant, expo = oracle.quantize(A)
    _, (gm, ge, pad) = _quantize_gpu(A)
    assert np.array_equal(ge, expo) and np.array_equal(gm, mant) and not pad.any()


@pytest.mark.parametrize("M,K", [(1, 8), (15, 64), (17, 264), (33, 320), (4101, 4160), (4101, 4168),
                                 (100003, 24), (3660, 1000), (3675, 1000), (7169, 512), (7169, 520), (4201, 8200), (8201, 6144), (8201, 6152)])
def test_decode_shapes(M, K):
    """Lane by lane (small and narrow), by panels of 16 rows x 4 panels (above 3.67 million values and from 512 columns) and of 8 rows
    (above 64 MiB): edges, tails of the last panel, and outputs above 96 MiB with whole and with shared 128-byte lines (the first are
    stored past the caches)."""
    import torch
    print(f"decode {(M, K)}", flush=True)
    rng = np.random.default_rng(4)
    mant = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
    expo = rng.integers(100, 160, size=(M, K // 8), dtype=np.uint8)
    dec = atb.bfp16_decode(torch.from_numpy(pack_a_bfp(mant, expo)).cuda(), M, K)
    torch.cuda.synchronize()
    want = np.ldexp(mant.astype(np.float32).reshape(M, -1, 8), expo.astype(np.int32)[:, :, None] - 133).reshape(M, K)
    assert np.array_equal(dec.float().cpu().numpy(), want)


def test_tall_matrices_fit_one_launch():
    """A launch takes fewer than 2^32 threads: 2^27 + 8 rows to quantise and 2^28 + 16 rows of one panel to decode need the forms
    with more rows, or blocks, per thread.  The rows repeat a pattern, so the first and the last of them say whether all were reached."""
    import torch
    M, K = 2 ** 27 + 8, 8
    print(f"quantize {(M, K)}", flush=True)
    rows = torch.randn((1024, K), device="cuda")
    x = rows.repeat(M // 1024 + 1, 1)[:M]
    buf = atb.bfp16_quantize(x)
    want = atb.bfp16_quantize(rows)
    lay, few = atb.bfp16_layout(M, K), atb.bfp16_layout(1024, K)
    man, exp = buf[:M * 64].view(M, 64), buf[lay.exp_off:lay.exp_off + M * 8].view(M, 8)
    wman, wexp = want[:1024 * 64].view(1024, 64), want[few.exp_off:few.exp_off + 1024 * 8].view(1024, 8)
    for first in (0, M // 2 // 1024 * 1024, M // 1024 * 1024 - 1024):
        assert torch.equal(man[first:first + 1024], wman) and torch.equal(exp[first:first + 1024], wexp)
    assert torch.equal(man[-8:], wman[:8]) and torch.equal(exp[-8:], wexp[:8])
    del x, buf, man, exp
    M, K = 2 ** 28 + 16, 64
    print(f"decode {(M, K)}", flush=True)
    lay = atb.bfp16_layout(M, K)
    buf = torch.zeros(lay.bytes, dtype=torch.uint8, device="cuda")
    man, exp = buf[:M * 64].view(M, 64), buf[lay.exp_off:lay.exp_off + M * 8].view(M, 8)
    man.view(torch.int64).copy_(torch.randint(-2 ** 62, 2 ** 62, (1, 8), device="cuda").expand(M, 8))
    exp.fill_(130)
    dec = atb.bfp16_decode(buf, M, K)
    want = man[:1].view(torch.int8).float() * 0.125
    for first in (0, M // 2, M - 4096):
        assert torch.equal(dec[first:first + 4096].float(), want.expand(4096, K))
    torch.cuda.synchronize()
    del buf, man, exp, dec
    torch.cuda.empty_cache()


def test_quantizer_rejects_bad_arguments():
    import ctypes
    import torch
    L = atb.lib()
    A = torch.zeros((4, 16), dtype=torch.float32, device="cuda")
    out = torch.zeros(atb.bfp16_bytes(4, 16), dtype=torch.uint8, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    assert L.atb_bfp16_quantize(p(A), 16, p(out), 4, 12, None) == 1      # K % 8
    assert L.atb_bfp16_quantize(p(A), 8, p(out), 4, 16, None) == 1       # lda < K
    assert L.atb_bfp16_quantize(None, 16, p(out), 4, 16, None) == 1
    assert L.atb_bfp16_quantize(ctypes.c_void_p(A.data_ptr() + 4), 16, p(out), 4, 16, None) == 1   # misaligned
