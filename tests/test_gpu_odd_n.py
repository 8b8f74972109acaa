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


def _inputs(M, N, K):
    A, Bb = workloads.small_integer_inputs(M, N, K, seed=33)
    A[:, K - 1] = 3.0 * (1 + np.arange(M) % 2)                 # the last product counts in every row
    Bb[K - 1, N - 1] = 0x4040                                  # 3.0
    return A, Bb


def _compare(M, N, K, tiles):
    A, Bb = _inputs(M, N, K)
    mant, expo = oracle.quantize(A)
    C_ref, _, _ = oracle.gemm(mant, expo, Bb)
    assert np.array_equal(_run(mant, expo, Bb, tiles), C_ref)


@pytest.mark.parametrize("tiles", EVERY)
@pytest.mark.parametrize("N", [1, 63, 65, 255, 257, 391])
def test_last_element_of_b(tiles, N):
    for K in (8, 64, 72, 128, 136, 256, 264, 512, 520, 776):
        print(f"odd N last element {(70, N, K)} tiles={tiles}", flush=True)
        _compare(70, N, K, tiles)


def _walks(M, N, tiles):
    """Tiles and tiles of the last column in the walk of each workgroup of a persistent grid (one workgroup per CU; an XCD's run of tiles lies in
    patches of 2048 rows, walked column by column)."""
    import torch
    tm, tn = -(-M // tiles[1]), -(-N // tiles[3])
    per_xcd, group = -(-tm * tn // 8), 2048 // tiles[1]
    slots, out = min(per_xcd, torch.cuda.get_device_properties(0).multi_processor_count // 8), []
    for xcd in range(8):
        for first in range(slots):
            last = []
            for t in range(first, per_xcd, slots):
                if xcd * per_xcd + t < tm * tn:
                    band, at = divmod(xcd * per_xcd + t, group * tn)
                    last.append(at // min(group, tm - band * group) == tn - 1)
            out.append((len(last), sum(last)))
    return out


@pytest.mark.parametrize("K", [64, 72, 136, 264])
@pytest.mark.parametrize("shape,last", [((17000, 1281), 1), ((70001, 255), 2), ((132000, 255), 3), ((70000, 513), 2)])
def test_last_element_of_b_in_a_walk_of_several_tiles(shape, last, K):
    """Walks of two and more tiles: one of them in the last column (which is not always the first), and several."""
    (M, N), tiles = shape, PERSISTENT[0]
    walks = _walks(M, N, tiles)
    assert max(n for _, n in walks) >= last and (N < 256 or any(0 < n < t for t, n in walks))
    assert all((t[1], t[3]) == (256, 256) for t in PERSISTENT)
    A, Bb = _inputs(M, N, K)
    mant, expo = oracle.quantize(A)
    C_ref, _, _ = oracle.gemm(mant, expo, Bb)
    for tiles in PERSISTENT:
        print(f"odd N walk {(M, N, K)} tiles={tiles}", flush=True)
        assert np.array_equal(_run(mant, expo, Bb, tiles), C_ref), tiles


# (M, N, K), whether 128 x 256 tiles run: above one 128 x 128 tile per CU; two rounds of wide tiles that are well filled, and one and a bit; K too
# short; and N that the wide tiles pad to twice its width
WIDE = [((2049, 2049, 1024), True), ((16 * 128 + 1, 2177, 1032), True), ((8200, 513, 1288), True), ((3713, 1665, 1024), True),
        ((3073, 4097, 1032), True), ((3073, 2817, 1032), False), ((2048, 2047, 1032), False), ((2049, 2049, 1016), False), ((33000, 127, 1032), False)]


@pytest.mark.parametrize("tiles", [(128, 128, 64, 128), (64, 128, 64, 128)])
@pytest.mark.parametrize("shape,wide", WIDE)
def test_128_row_tiles_run_as_wide_ones(tiles, shape, wide):
    """Where the 128 x 256 tiles run in place of 128 x 128 ones, on both sides of each line: the bits that any other instance gives."""
    import paper_2511_16041_amd as atb
    M, N, K = shape
    print(f"odd N wide {shape} tiles={tiles}", flush=True)
    plan = atb.Gemm(M, N, K, *tiles)
    kernel, columns = plan.kernel(), 256 if wide else 128
    plan.close()
    assert kernel.tiles() == ((128, 128, 64, 256) if wide else tiles) and kernel.workgroups == -(-(-(-M // 128) * -(-N // columns)) // 8) * 8
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
