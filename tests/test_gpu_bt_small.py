"""B^T in bf16 on the pipeline: problems that run on 64 x 64 and 128 x 128 tiles in place of the ones that the plan names, on both sides of either
line, cut by M, N and K; and the named tiles themselves on problems just too large for those.  The bits are those of row-major B."""
import numpy as np
import pytest

import oracle
import paper_2511_16041_amd as atb
import workloads
from helpers import bf16_tensor_bits, bits_to_bf16_tensor, pack_a_bfp
from test_gpu_skinny import BT_TILES

pytestmark = pytest.mark.gpu
# (M, N, K) -> rows and columns of a workgroup's tile
SMALL = [((1, 1, 8), 64), ((65, 129, 72), 64), ((64, 64, 1024), 64), ((1023, 2047, 136), 64), ((32760, 3, 64), 64),
         ((1025, 2048, 200), 128), ((2048, 2047, 1024), 128), ((32700, 65, 72), 128), ((1300, 2600, 2056), 128), ((2000, 2000, 1288), 128)]
LARGE = [(2049, 2048, 136), (33000, 100, 72), (129, 16500, 264), (2100, 2100, 8)]


def _bits(shape, tiles, A_dev, B_dev, b_format):
    import torch
    g = atb.Gemm(*shape, *tiles, b_format=b_format)
    assert not g.streams()
    info, C = g.launch_info(), torch.full(shape[:2], float("nan"), dtype=torch.bfloat16, device="cuda")
    g.run(A_dev, B_dev, C)
    torch.cuda.synchronize()
    g.close()
    return bf16_tensor_bits(C), info


@pytest.mark.parametrize("shape,side", SMALL + [(s, 0) for s in LARGE])
def test_small_tiles_for_transposed_b(shape, side):
    import torch
    M, N, K = shape
    for exact in (True, False):
        A, Bb = workloads.small_integer_inputs(M, N, K, seed=51) if exact else workloads.make_inputs(workloads.CONFIGS["ragged"], M=M, N=N, K=K)
        mant, expo = oracle.quantize(A)
        A_dev = torch.from_numpy(pack_a_bfp(mant, expo)).cuda()
        B_dev = bits_to_bf16_tensor(Bb, "cuda")
        want, _ = _bits(shape, (32, 64, 64, 64), A_dev, B_dev, "bf16")
        if exact:
            assert np.array_equal(want, oracle.gemm(mant, expo, Bb)[0])
        Bt = B_dev.t().contiguous()
        for tiles in BT_TILES:
            print(f"B^T small {shape} tiles={tiles}", flush=True)
            got, info = _bits(shape, tiles, A_dev, Bt, "bf16_t")
            assert np.array_equal(got, want), tiles
            rows, cols = (side, side) if side else (tiles[1], tiles[3])
            assert info.workgroups == -(-(-(-M // rows) * -(-N // cols)) // 8) * 8
