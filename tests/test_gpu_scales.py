"""The streaming kernel's decode with B^T multiplies by 2^(E - 133), a denormal for E below 7: on exact inputs of the smallest, ordinary and the
largest exponents it gives the bits of the tile pipeline, which scales with ldexp."""
import numpy as np
import pytest

import oracle
import paper_2511_16041_amd as atb
import workloads
from helpers import bf16_tensor_bits, pack_a_bfp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b_format", ["bfp16", "bf16_t"])
@pytest.mark.parametrize("a_exp,b_exp", [(-133, 64), (-128, 40), (-120, 20), (0, 0), (60, -60), (118, -64)])
def test_exponents_at_the_ends_of_their_range(a_exp, b_exp, b_format):
    import torch
    M, N, K = 20, 264, 1096
    print(f"scales A 2^{a_exp} B 2^{b_exp} {b_format}", flush=True)
    A, Bb = workloads.small_integer_inputs(M, N, K, seed=41)
    A = np.ldexp(np.rint(A), a_exp).astype(np.float32)
    mant, expo = oracle.quantize(A)
    B = np.ldexp(oracle.bf16_to_double(Bb).T, b_exp).astype(np.float32)
    A_dev = torch.from_numpy(pack_a_bfp(mant, expo)).cuda()
    W = torch.from_numpy(np.ascontiguousarray(B)).cuda()
    bits = []
    for tiles, streams in (((64, 128, 64, 256) if b_format == "bf16_t" else (32, 32, 256, 64), True), ((64, 64, 64, 64), False)):
        fmt = b_format if streams or b_format == "bfp16" else "bf16"
        g = atb.Gemm(M, N, K, *tiles, b_format=fmt)
        assert g.streams() == streams
        B_dev = torch.from_numpy(pack_a_bfp(*oracle.quantize(B))).cuda() if fmt == "bfp16" else W.bfloat16() if fmt == "bf16_t" else W.t().contiguous().bfloat16()
        bits.append(bf16_tensor_bits(g.run(A_dev, B_dev)))
        torch.cuda.synchronize()
        g.close()
    assert np.array_equal(*bits)
    assert a_exp < -126 or bits[0].any()
