"""The streaming kernel for few rows (K > 1024; M <= 64, or one tile per CU) and the pipeline's instances on the long reductions that
stay with them, against the oracle.  The shapes reach every variant of the streaming kernel that the rules can choose (checked on the CPU in
test_abi_host.py), the edges of each, K tails, odd N and every storage format; each case asserts which kernel runs.  Exact
(small-integer) inputs must give the oracle's bits, since every order of the sums is then exact; random ones the GEMM tolerance (and
half a mantissa step of a BFP16 C)."""
import re

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
          (5, 1001, 1032), (48, 8194, 1032), (7, 8256, 1032), (20, 8256, 1032), (49, 8264, 1032), (64, 16386, 1032), (16, 16448, 1096),
          (20, 16448, 1032), (40, 16448, 1032),
          # above 64 rows: 64 x 32 and 64 x 64 tiles, then (B row-major / transposed) 64 x 128 / 128 x 64; many rows of few columns
          (65, 72, 1032), (130, 2802, 1096), (260, 3400, 4104), (130, 4802, 1096), (4130, 32, 1032)]
WIDE_AND_LONG = (50, 16386, 8192)            # bf16 B at 49 to 64 rows and 128 columns
COMBOS = [("bf16", "bf16"), ("bf16_t", "bf16"), ("bfp16", "bf16"), ("bf16", "bfp16"), ("bfp16", "bfp16")]
BOTH = ("bf16", "bfp16")
# {(shape, b_format): C formats} that the rules leave with the pipeline
PIPELINE = {((64, 264, 1088), "bf16"): BOTH, ((64, 8191, 1032), "bf16"): ("bfp16",), ((64, 16386, 1032), "bf16"): BOTH,
            ((64, 16386, 1032), "bfp16"): BOTH, ((65, 72, 1032), "bf16"): BOTH, ((130, 2802, 1096), "bf16"): BOTH,
            ((260, 3400, 4104), "bfp16"): BOTH, ((4130, 32, 1032), "bf16"): BOTH}
BT_TILES = [(256, 256, 64, 256), (128, 256, 64, 256), (64, 256, 64, 256), (128, 128, 64, 256), (64, 128, 64, 256)]


def columns(N, c_format):
    return -(-N // 8) * 8 if c_format == "bfp16" else N            # C in BFP16: whole blocks


def plan(shape, b_format, c_format):
    M, N, K = shape
    tiles = (64, 128, 64, 256) if b_format == "bf16_t" else (32, 32, 256, 64)
    return atb.Gemm(M, columns(N, c_format), K, *tiles, b_format=b_format, c_format=c_format)


def variants(log):
    """From what the library logs of plans as it makes them (ATB_LOG=1): the set of (form of B, rows and columns of a workgroup's tile,
    threads, panels in flight) of the streaming kernel that runs them."""
    out = set()
    for N, b, rest in re.findall(r"^atb_gemm_create: M=\d+ N=(\d+) .* b=(\S+) .* streaming: (.*)$", log, re.M):
        rows, cols, threads, depth = re.match(r"tile=(\d+)x(\d+) threads=(\d+) depth=(\d+) ", rest).groups()
        out.add(("bf16 odd" if b == "bf16" and int(N) % 2 else b, int(rows), int(cols), int(threads), int(depth)))
    return out


def _check(g, exact, seed=21):
    import torch
    M, N, K = g.shape
    b_format, c_format = g.b_format, g.c_format
    if exact:
        A, Bb = workloads.small_integer_inputs(M, N, K, seed=seed)
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
    out = (torch.full((atb.bfp16_bytes(M, N),), 0xAB, dtype=torch.uint8, device="cuda") if c_format == "bfp16"
           else torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda"))
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


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("b_format,c_format", COMBOS)
@pytest.mark.parametrize("shape", SHAPES)
def test_streaming_kernel(shape, b_format, c_format, exact):
    print(f"skinny {shape} B={b_format} C={c_format} exact={exact}", flush=True)
    g = plan(shape, b_format, c_format)
    assert g.streams() == (c_format not in PIPELINE.get((shape, b_format), ()))
    _check(g, exact)


TWO_PANELS = [(20, 8264, 1608), (48, 8264, 2048), (49, 8264, 1544), (66, 72, 1608), (129, 1032, 1992), (257, 2120, 1992)]


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("c_format", BOTH)
@pytest.mark.parametrize("shape", TWO_PANELS)
def test_two_panels_in_flight(shape, c_format, exact):
    """B in BFP16, four rounds of eight panels: 20 to 64 rows and more, 64 and 32 columns, the last round whole, of one panel (1544) or with a
    tail.  (That these plans have two panels in flight is checked in test_abi_host.py.)"""
    print(f"two panels {shape} C={c_format} exact={exact}", flush=True)
    g = plan(shape, "bfp16", c_format)
    assert g.streams() and g.launch_info().threads == 512 and (-(-shape[2] // 64) + 7) // 8 == 4
    _check(g, exact, seed=25)


def test_wide_and_long():
    print(f"skinny {WIDE_AND_LONG}", flush=True)
    g = plan(WIDE_AND_LONG, "bf16", "bf16")
    assert g.streams()
    _check(g, exact=True)


@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("shape,b_format,c_format", [
    ((50, 264, 1096), "bf16", "bf16"), ((64, 1030, 2056), "bf16", "bfp16"),                              # 49 to 64 rows, up to 8192 columns
    ((65, 72, 1032), "bf16", "bf16"), ((65, 75, 1288), "bf16", "bf16"), ((97, 301, 1544), "bf16", "bfp16"),   # few tiles, one nearly without rows; odd N
    ((193, 2304, 1160), "bfp16", "bf16"), ((193, 2304, 1672), "bfp16", "bfp16"), ((49, 16448, 1096), "bfp16", "bf16")])
@pytest.mark.parametrize("tiles", [(64, 64, 128, 128), (32, 64, 256, 64), (32, 32, 256, 64)])
def test_long_reductions_on_the_pipeline(tiles, shape, b_format, c_format, exact):
    """The instances that hand problems over to the streaming kernel, on K > 1024 problems that they keep."""
    M, N, K = shape
    print(f"pipeline {shape} tiles={tiles} B={b_format} C={c_format} exact={exact}", flush=True)
    g = atb.Gemm(M, columns(N, c_format), K, *tiles, b_format=b_format, c_format=c_format)
    assert not g.streams()
    _check(g, exact, seed=23)


def _bits(tiles, A, Bb, b_format="bf16"):
    """(result bits, threads of the streaming kernel or 0) of one plan."""
    import torch
    (M, K), N = A.shape, Bb.shape[1]
    B_dev = bits_to_bf16_tensor(Bb if b_format == "bf16" else np.ascontiguousarray(Bb.T), "cuda")
    g = atb.Gemm(M, N, K, *tiles, b_format=b_format)
    C = g.run(torch.from_numpy(pack_a_bfp(*oracle.quantize(A))).cuda(), B_dev)
    C2 = g.run(torch.from_numpy(pack_a_bfp(*oracle.quantize(A))).cuda(), B_dev)
    torch.cuda.synchronize()
    threads = g.launch_info().threads if g.streams() else 0
    g.close()
    bits = bf16_tensor_bits(C)
    assert np.array_equal(bits, bf16_tensor_bits(C2)), "two runs differ"
    return bits, threads


@pytest.mark.parametrize("K", [1024, 1096, 4104])
def test_equal_bits(K):
    """What holds of the bits: up to K = 1024 every plan of a problem agrees, B^T included, and a row of C does not depend on M.  Above, the
    plans that stay with the pipeline agree among themselves, and those that stream agree where the kernel has as many waves."""
    M, N = 48, 520
    print(f"equal bits K={K}", flush=True)
    A, Bb = workloads.make_inputs(workloads.CONFIGS["ragged"], M=M, N=N, K=K)
    seen = {}
    for rows in (M, 17):
        for tiles in atb.instances():
            for b_format in ("bf16", "bf16_t") if tiles in BT_TILES else ("bf16",):
                bits, threads = _bits(tiles, A[:rows], Bb, b_format)
                want = seen.setdefault(threads, bits)
                assert np.array_equal(bits, want[:rows]), f"{tiles} {b_format} M={rows} threads={threads}"
    assert set(seen) == ({0} if K <= 1024 else {0, 512})
