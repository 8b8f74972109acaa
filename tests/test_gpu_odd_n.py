"""Odd N on the tile pipeline: B's last element, which its tile's request does not bring in, for every instance: its K-step the first of a
reduction, the second, the third and a later one, whole or of 8 rows, N below, at and past one and more tiles; and with several tiles of the last
column in one workgroup's walk.  Exact inputs; only the last column of A's last rows and of B's last row depends on nothing else."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_gemm import BIG, MID, SKINNY, SMALL, WIDE_K, _run

pytestmark = pytest.mark.gpu
EVERY = BIG + SMALL + MID + WIDE_K + SKINNY
PERSISTENT = [t for t in EVERY if t[1] * t[3] >= 256 * 256]


def _compare(M, N, K, tiles):
    A, Bb = workloads.small_integer_inputs(M, N, K, seed=33)
    A[:, K - 1] = 3.0 * (1 + np.arange(M) % 2)                 # the last product counts in every row
    Bb[K - 1, N - 1] = 0x4040                                  # 3.0
    mant, expo = oracle.quantize(A)
    C_ref, _, _ = oracle.gemm(mant, expo, Bb)
    assert np.array_equal(_run(mant, expo, Bb, tiles), C_ref)


@pytest.mark.parametrize("tiles", EVERY)
@pytest.mark.parametrize("N", [1, 63, 65, 255, 257, 391])
def test_last_element_of_b(tiles, N):
    for K in (8, 64, 72, 128, 136, 256, 264, 512, 520, 776):
        print(f"odd N last element {(70, N, K)} tiles={tiles}", flush=True)
        _compare(70, N, K, tiles)


@pytest.mark.parametrize("tiles", PERSISTENT)
@pytest.mark.parametrize("K", [64, 72, 136, 264])
def test_last_element_of_b_in_a_walk_of_several_tiles(tiles, K):
    print(f"odd N walk {(17000, 1281, K)} tiles={tiles}", flush=True)
    _compare(17000, 1281, K, tiles)                            # 402 tiles for 256 workgroups, 67 of them in the last column


@pytest.mark.parametrize("tiles", [(128, 128, 64, 128), (64, 128, 64, 128)])
@pytest.mark.parametrize("shape", [(2049, 2049, 1024), (16 * 128 + 1, 2177, 1032), (8200, 513, 1288), (3713, 1665, 1024)])
def test_128_row_tiles_run_as_wide_ones(tiles, shape):
    """Above one 128 x 128 tile per CU the 128 x 256 tiles run in their place, with the bits that any other instance gives."""
    import paper_2511_16041_amd as atb
    M, N, K = shape
    print(f"odd N wide {shape} tiles={tiles}", flush=True)
    plan = atb.Gemm(M, N, K, *tiles)
    assert plan.launch_info().workgroups == -(-(-(-M // 128) * -(-N // 256)) // 8) * 8
    plan.close()
    _compare(M, N, K, tiles)
    A, Bb = workloads.make_inputs(workloads.CONFIGS["ragged"], M=M, N=N, K=K)
    mant, expo = oracle.quantize(A)
    assert np.array_equal(_run(mant, expo, Bb, tiles), _run(mant, expo, Bb, (64, 64, 64, 64)))


@pytest.mark.parametrize("N", [1, 129, 391])
@pytest.mark.parametrize("tiles", [(64, 64, 128, 128), (128, 128, 64, 128)])
def test_third_b_buffer(tiles, N):
    """From K = 768 on these tiles have three buffers for B of odd N (128 x 128 up to one tile per CU): the last K-step in each of the three, whole or of
    8 rows."""
    import paper_2511_16041_amd as atb
    lds = {}
    for K in (760, 768, 776, 832, 896, 904, 1024, 1032, 1160, 1288):
        plan = atb.Gemm(150, N, K, *tiles)
        assert not plan.streams()
        lds[K] = plan.launch_info().lds_bytes
        plan.close()
        print(f"odd N third buffer {(150, N, K)} tiles={tiles}", flush=True)
        _compare(150, N, K, tiles)
    assert all(n - lds[760] == (0 if K < 768 else tiles[2] * tiles[3] * 2) for K, n in lds.items())
