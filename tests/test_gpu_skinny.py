"""The streaming kernel for few rows (K > 1024; M <= 64, or one tile per CU) against the oracle: every row-block count, every tile width and
the edges of each, K tails, odd N, every storage format.  Exact (small-integer) inputs must give the oracle's bits,
since every order of the sums is then exact; random ones the GEMM tolerance (and half a mantissa step of a BFP16 C)."""
import numpy as np
import pytest

import oracle
import paper_2511_16041_amd as atb
import workloads
from helpers import bits_to_bf16_tensor, bf16_tensor_bits, pack_a_bfp, unpack_a_bfp

pytestmark = pytest.mark.gpu

# (M, N, K): 32, 64 and 128 columns per workgroup; M on both sides of a row block; N below, at and past a tile, odd, and
# not a multiple of 4; K of one panel past the threshold, with and without a tail
SHAPES = [(1, 2, 1032), (16, 32, 1088), (17, 33, 1032), (48, 34, 1096), (64, 264, 1024 + 64), (33, 1001, 1160), (64, 8191, 1032),
          (48, 8194, 1032), (49, 8264, 1032), (64, 16386, 1032), (16, 16448, 1096),
          # above 64 rows: 64 x 32 and 64 x 64 tiles, then (B row-major / transposed) 64 x 128 / 128 x 64
          (65, 72, 1032), (130, 2802, 1096), (260, 3400, 4104), (130, 4802, 1096), (260, 3400, 5640)]


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("b_format,c_format", [("bf16", "bf16"), ("bf16_t", "bf16"), ("bfp16", "bf16"), ("bf16", "bfp16"), ("bfp16", "bfp16")])
@pytest.mark.parametrize("shape", SHAPES)
def test_streaming_kernel(shape, b_format, c_format, exact):
    import torch
    M, N, K = shape
    if c_format == "bfp16" and N % 8 != 0:
        N = -(-N // 8) * 8
    print(f"skinny {(M, N, K)} B={b_format} C={c_format} exact={exact}", flush=True)
    if exact:
        A, Bb = workloads.small_integer_inputs(M, N, K, seed=21)
    else:
        A, Bb = workloads.make_inputs(workloads.CONFIGS["ragged"], M=M, N=N, K=K)
    mant, expo = oracle.quantize(A)
    A_dev = torch.from_numpy(pack_a_bfp(mant, expo)).cuda()
    if b_format == "bfp16":
        bm, be = oracle.quantize(np.ascontiguousarray(oracle.bf16_to_double(Bb).T.astype(np.float32)))
        Bb = np.ascontiguousarray(oracle.bfp16_as_bf16_bits(bm, be).T)
        B_dev = torch.from_numpy(pack_a_bfp(bm, be)).cuda()
    else:
        B_dev = bits_to_bf16_tensor(Bb, "cuda")
        if b_format == "bf16_t":
            B_dev = B_dev.t().contiguous()
    C_ref, T, S, _ = oracle.gemm(mant, expo, Bb, want_sum=True)
    tiles = (64, 128, 64, 256) if b_format == "bf16_t" else (32, 32, 256, 64)
    out = (torch.full((atb.bfp16_bytes(M, N),), 0xAB, dtype=torch.uint8, device="cuda") if c_format == "bfp16"
           else torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda"))
    g = atb.Gemm(M, N, K, *tiles, b_format=b_format, c_format=c_format)
    g.run(A_dev, B_dev, out)
    torch.cuda.synchronize()
    g.close()
    tol = oracle.tolerance(T)
    if c_format == "bfp16":
        cm, ce, pad = unpack_a_bfp(out.cpu().numpy(), M, N)
        assert not pad.any()
        if exact:
            rm, re_ = oracle.quantize(S.astype(np.float32))
            assert np.array_equal(cm, rm) and np.array_equal(ce, re_)
        err, tol = np.abs(oracle.decode(cm, ce) - S), tol + np.repeat(np.ldexp(1.0, ce.astype(np.int64) - 134), 8, axis=1)
    else:
        bits = bf16_tensor_bits(out)
        if exact:
            assert np.array_equal(bits, C_ref)
        err = np.abs(oracle.bf16_to_double(bits) - oracle.bf16_to_double(C_ref))
    assert not np.isnan(err).any() and not (err > tol).any(), f"worst ratio {np.max(err / tol):.3g}"
