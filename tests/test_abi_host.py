"""CPU-only tests of libatb: the library loads, exports every symbol the header
declares, validates arguments without touching a device, lays BFP16 out as
documented, and its model / selector agree with the oracle of the paper's model."""
import ctypes

import numpy as np
import os
import re
import shutil
import subprocess
import sys
import sysconfig
import textwrap

import pytest

import paper_2511_16041_amd as atb
from oracle import model as om

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "atb.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(atb_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = atb.lib()
    names = _declared_symbols()
    assert len(names) >= 16
    for n in names:
        assert hasattr(L, n), n
    assert sorted(atb.EXPORTS) == names


def test_status_strings():
    L = atb.lib()
    seen = {L.atb_status_string(i) for i in range(7)}
    assert len(seen) == 7 and all(s for s in seen)
    assert L.atb_status_string(99) is not None


def test_instances_and_create_validation():
    inst = atb.instances()
    assert (256, 256, 64, 256) in inst and (64, 256, 64, 256) in inst and (32, 64, 64, 64) in inst
    for (a, c, k, n) in inst:
        assert c % a == 0 and k % 16 == 0
    L = atb.lib()
    h = ctypes.c_void_p()

    def create(M, N, K, *t):
        return L.atb_gemm_create(ctypes.byref(h), M, N, K, *t)

    assert create(256, 256, 256, 32, 64, 64, 64) == 0 and h.value
    wg, th, lds = ctypes.c_int64(), ctypes.c_int(), ctypes.c_int()
    assert L.atb_gemm_launch_info(h, ctypes.byref(wg), ctypes.byref(th), ctypes.byref(lds)) == 0
    assert wg.value == 16 and th.value in (128, 256, 512) and 0 < lds.value <= 160 * 1024
    L.atb_gemm_destroy(h)
    assert create(0, 256, 256, 32, 64, 64, 64) == 1 and not h.value          # M < 1
    assert create(256, 256, 252, 32, 64, 64, 64) == 1                         # K % 8
    assert create(256, 256, 256, 48, 64, 64, 64) == 2                         # T_MC % T_MA
    assert create(256, 256, 256, 64, 64, 32, 64) == 2                         # not compiled
    assert create(256, 256, 256, 512, 512, 64, 256) == 4                      # C tile > accumulators
    assert create(256, 256, 256, 256, 256, 512, 64) == 3                      # A + B > LDS
    assert create(256, 256, 256, 256, 256, 128, 256) == 3                     # T_K = 128 does not fit symmetric ...
    assert create(256, 256, 256, 32, 256, 128, 256) == 0 and h.value         # ... but fits at rho = 8
    L.atb_gemm_destroy(h)
    assert L.atb_gemm_create(None, 1, 1, 8, 32, 64, 64, 64) == 1
    assert L.atb_gemm_run(None, None, None, None, None) == 1
    L.atb_gemm_destroy(None)                                                  # no-op


def test_bfp16_layout():
    for (M, K) in [(256, 256), (3000, 4104), (1, 8), (7, 24)]:
        lay = atb.bfp16_layout(M, K)
        assert lay.panel_k == 64 and lay.panels == (K + 63) // 64
        assert lay.man_stride == M * 64 and lay.exp_stride == M * 8
        assert lay.exp_off % 256 == 0 and lay.exp_off >= lay.panels * lay.man_stride
        assert lay.bytes % 256 == 0 and lay.bytes >= lay.exp_off + lay.panels * lay.exp_stride
        assert atb.bfp16_bytes(M, K) == lay.bytes
    assert atb.bfp16_bytes(4, 12) == 0 and atb.bfp16_bytes(0, 8) == 0
    # 9 bytes per 8 elements, up to padding
    lay = atb.bfp16_layout(8192, 8192)
    assert lay.bytes == 8192 * 8192 * 9 // 8


def test_model_matches_oracle_in_paper_mode():
    hw = atb.hw_params("xdna2")
    assert hw.n_core == 32 and hw.array_rows == 4 and hw.array_cols == 8
    peak = om.peak_core_flops(512, 1.8e9)
    assert hw.peak_core_flops == pytest.approx(peak)
    cases = [(2048, 2048, 4096, 64, 64, 64, 128), (2048, 2048, 4480, 16, 64, 224, 64),
             (4096, 2048, 4096, 32, 128, 64, 128), (4096, 2048, 4096, 128, 128, 8, 128)]
    for (M, N, K, T_MA, T_MC, T_K, T_N) in cases:
        ch = atb.model_eval(M, N, K, T_MA, T_MC, T_K, T_N, hw)
        a, b, c = hw.a_bytes, hw.b_bytes, hw.c_bytes
        rho = T_MC // T_MA
        assert ch.rho == rho
        assert ch.ai_core == pytest.approx(om.ai_rho(T_MC, T_N, K, a, b, c), rel=1e-12)
        assert ch.ai == pytest.approx(om.ai_array(T_MC, T_N, K, a, b, c, 4, 8), rel=1e-12)
        assert ch.buffer_bytes == pytest.approx(om.buffer_bytes(T_MA, T_MC, T_K, T_N, a, b, c), rel=1e-12)
        em = om.eff_micro(T_K, hw.eta, hw.eps, hw.II)
        assert ch.eff_micro == pytest.approx(em, rel=1e-12)
        ec = om.eff_core(T_MC, T_K, T_N, rho, peak, em, hw.delta_cycles / hw.clock_hz)
        assert ch.eff_core == pytest.approx(ec, rel=1e-12)
        perf, mem, comp = om.perf_array(ch.ai, hw.bw_offchip, ec, peak, 32)
        assert ch.mem_bound == pytest.approx(mem, rel=1e-12)
        assert ch.compute_bound == pytest.approx(comp, rel=1e-12)
        assert ch.pred_flops == pytest.approx(perf, rel=1e-12)
        assert ch.feasible == int(ch.buffer_bytes <= 63 * 1024)
    # Table 2, Config 1, 128x64x128 rho=4: AI_array 410, memory bound 26.6 TFLOP/s
    ch = atb.model_eval(4096, 2048, 4096, 32, 128, 64, 128, hw)
    assert round(ch.ai) == 410 and ch.mem_bound / 1e12 == pytest.approx(26.6, abs=0.1)


def test_model_mi355x_mode_and_selector():
    hw = atb.hw_params("mi355x")
    assert hw.n_core == 256 and hw.buffer_bytes == 160 * 1024 and hw.acc_bytes == 256 * 1024
    assert hw.peak_core_flops * hw.n_core == pytest.approx(2.5e15)
    ch = atb.model_eval(8192, 8192, 8192, 64, 256, 64, 256)          # hw = NULL -> MI355X
    ch2 = atb.model_eval(8192, 8192, 8192, 64, 256, 64, 256, hw)
    assert ch.pred_flops == ch2.pred_flops and ch.feasible == 1
    assert ch.acc_bytes == 4 * 256 * 256
    # C lives in registers: the LDS term has no C share
    ab, bb = hw.a_buf_bytes, hw.b_buf_bytes
    assert ch.buffer_bytes == pytest.approx(2 * ab * 64 * 64 + 2 * bb * 64 * 256)
    # Eq. (15) ordering with the fill term switched off: at fixed C tile and T_K, larger rho lowers
    # the compute bound; the LDS footprint always shrinks with rho
    hw0 = atb.hw_params("mi355x")
    hw0.fill_cycles = 0.0
    prev = None
    for T_MA in (256, 128, 64, 32):
        c = atb.model_eval(8192, 8192, 8192, T_MA, 256, 64, 256, hw0)
        if prev is not None:
            assert c.eff_core < prev.eff_core and c.buffer_bytes < prev.buffer_bytes
        prev = c
    # with the fill term: T = T_mfma / Eff_micro + delta rho + fill / rho per K-step
    for T_MA in (256, 128, 64, 32):
        rho = 256 // T_MA
        c = atb.model_eval(8192, 8192, 8192, T_MA, 256, 64, 256, hw)
        t_mfma = 2.0 * 256 * 256 * 64 / hw.peak_core_flops
        t = t_mfma / c.eff_micro + (hw.delta_cycles * rho + hw.fill_cycles / rho) / hw.clock_hz
        assert c.eff_core == pytest.approx(t_mfma / t, rel=1e-12)
    # ATB makes T_K = 128 legal: 264 KiB of LDS symmetric, 146 KiB at rho = 8
    assert atb.model_eval(8192, 8192, 8192, 256, 256, 128, 256, hw).feasible == 0
    assert atb.model_eval(8192, 8192, 8192, 32, 256, 128, 256, hw).feasible == 1
    ranked = atb.select_tiles(8192, 8192, 8192)
    assert len(ranked) == len(atb.instances())
    assert ranked[0].feasible == 1 and ranked[0].T_MC == 256
    assert all(ranked[i].pred_flops >= ranked[i + 1].pred_flops
               for i in range(len(ranked) - 1) if ranked[i + 1].feasible)
    small = atb.select_tiles(256, 256, 256)
    assert small[0].T_MC <= 64                        # many small tiles beat one big tile on 256 CUs
    assert atb.lib().atb_select_tiles(0, 1, 8, None, None, 0, None) == 1


def test_create_fmt_validation():
    """Plans with B and/or C stored as BFP16: argument checks run on the host."""
    L = atb.lib()
    h = ctypes.c_void_p()

    def create(M, N, K, t, bf, cf):
        return L.atb_gemm_create_fmt(ctypes.byref(h), M, N, K, *t, bf, cf)

    assert create(512, 512, 256, (128, 256, 64, 256), 1, 1) == 0 and h.value
    L.atb_gemm_destroy(h)
    assert create(512, 512, 256, (128, 256, 64, 256), 0, 0) == 0 and h.value      # same as atb_gemm_create
    L.atb_gemm_destroy(h)
    assert create(512, 508, 256, (128, 256, 64, 256), 0, 1) == 1 and not h.value  # C in BFP16: N % 8 != 0
    assert create(512, 508, 256, (128, 256, 64, 256), 1, 0) == 0 and h.value      # B in BFP16 does not constrain N
    L.atb_gemm_destroy(h)
    assert create(512, 512, 256, (128, 256, 64, 256), 3, 0) == 1                  # unknown format
    assert create(512, 512, 256, (128, 256, 64, 256), 0, 2) == 1                  # "transposed" is a format of B only
    assert create(512, 508, 256, (128, 256, 64, 256), 2, 0) == 0 and h.value      # bf16 B handed over transposed
    L.atb_gemm_destroy(h)
    assert create(512, 512, 256, (128, 256, 64, 256), 2, 1) == 1                  # ... needs a bf16 C
    assert create(512, 512, 256, (64, 64, 64, 64), 2, 0) == 2                     # ... and one of the large tiles
    assert create(512, 512, 256, (32, 256, 128, 256), 2, 0) == 2
    assert create(64, 64, 1 << 23, (128, 256, 64, 256), 2, 0) == 1                # 2 T_N K >= 2^31
    assert create(512, 512, 256, (32, 256, 64, 256), 0, 1) == 2                   # instance without format variants
    assert create(512, 512, 256, (32, 256, 128, 256), 1, 1) == 2
    assert create(64, 512, 1024, (32, 64, 256, 64), 1, 0) == 0 and h.value           # the skinny-problem instances carry the variants
    L.atb_gemm_destroy(h)
    assert create(512, 512, 256, (64, 64, 64, 64), 1, 1) == 0 and h.value
    L.atb_gemm_destroy(h)


def test_selector_tracks_problem_size():
    """Few C tiles: smaller tiles fill the chip better (the N = 2048 shapes of the paper's Table 3)."""
    assert atb.select_tiles(8192, 8192, 8192)[0].T_MC == 256
    assert atb.select_tiles(4096, 2048, 4096)[0].T_MC == 128         # 128 x 256 and 128 x 128 tiles measure within 3 % of each other here
    assert atb.select_tiles(1024, 2048, 8192)[0].T_MC == 64
    assert atb.select_tiles(1024, 2048, 4096)[0].T_MC <= 128
    assert atb.select_tiles(1024, 2048, 4096)[0].T_N <= 128
    # a launch never beats its fixed cost, and predictions grow with the problem
    a = atb.select_tiles(256, 256, 256)[0].pred_flops
    b = atb.select_tiles(1024, 1024, 1024)[0].pred_flops
    c = atb.select_tiles(8192, 8192, 8192)[0].pred_flops
    assert a < b < c and a < 2.0 * 256 ** 3 / 6e-6


def test_microkernel_model_against_measurements():
    """The CDNA4 issue model (unit costs measured by csrc/microbench/unit_costs.hip) against the
    measured full-load throughput and MFMA-busy fraction of every compiled instance."""
    import os
    rows = []
    for line in open(os.path.join(os.path.dirname(__file__), "measured", "mi355x_instances.txt")):
        if line.startswith("#") or not line.strip():
            continue
        f = line.split()
        rows.append((tuple(int(x) for x in f[:4]), tuple(int(x) for x in f[4:8]), float(f[8]),
                     None if f[9] == "-" else float(f[9]), f[10]))
    inst = atb.instances()
    assert {r[0] for r in rows} == set(inst)
    for tiles, geom, tflops, busy, flag in rows:
        assert atb.instance_geometry(inst.index(tiles)) == geom
        m = atb.model_microkernel(*tiles, *geom)
        # components as documented in include/atb.h
        assert m.n_mfma == tiles[1] * tiles[3] * tiles[2] / 16384 and m.mfma_cycles == m.n_mfma * 8
        assert m.steady_cycles == pytest.approx(max(m.mfma_cycles, m.valu_cycles, m.lds_cycles, m.vmem_cycles) / 0.85)
        assert m.kstep_cycles == pytest.approx(m.steady_cycles + (tiles[1] // tiles[0]) * m.switch_cycles)
        assert m.mfma_util == pytest.approx(m.mfma_cycles / m.kstep_cycles) and 0 < m.mfma_util < 1
        if flag in ("ok", "loose"):
            assert abs(m.pred_flops / 1e12 / tflops - 1) < (0.15 if flag == "ok" else 0.25), (tiles, m.pred_flops / 1e12, tflops)
            if busy is not None:
                # workgroups that share a CU overlap more than the model's division by waves per SIMD grants them:
                # they run busier and at a lower clock than predicted (the throughput bound above still holds)
                assert abs(m.mfma_util - busy) < (0.10 if geom[2] == 1 else 0.15), (tiles, m.mfma_util, busy)
    # every large tile is limited by the VALU issue port (decode next to MFMAs), the small ones by the LDS
    big = atb.model_microkernel(128, 256, 64, 256, 2, 4, 1, 16)
    assert big.valu_cycles > big.mfma_cycles > big.lds_cycles * 0.9 and big.valu_cycles > big.lds_cycles
    small = atb.model_microkernel(64, 64, 64, 64, 2, 2, 4, 16)
    assert small.lds_cycles > small.valu_cycles > small.mfma_cycles
    L = atb.lib()
    assert L.atb_model_microkernel(128, 256, 64, 256, 2, 4, 1, 16, None) == 1
    mm = atb.MicroModel()
    assert L.atb_model_microkernel(96, 256, 64, 256, 2, 4, 1, 16, ctypes.byref(mm)) == 2      # rho not an integer
    assert L.atb_model_microkernel(128, 256, 64, 256, 3, 4, 1, 16, ctypes.byref(mm)) == 2     # bands do not divide


def test_host_packers_agree():
    """The binding's layout marshalling against the tests' own packer (written from include/atb.h)."""
    from helpers import pack_a_bfp, unpack_a_bfp
    rng = np.random.default_rng(0)
    for (M, K) in [(5, 8), (37, 72), (64, 64), (130, 200)]:
        mant = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
        expo = rng.integers(0, 255, size=(M, K // 8), dtype=np.uint8)
        a, b = pack_a_bfp(mant, expo), atb.bfp16_pack_host(mant, expo)
        assert np.array_equal(a, b)
        for unpack in (unpack_a_bfp, atb.bfp16_unpack_host):
            m2, e2, pad = unpack(a, M, K)
            assert np.array_equal(m2, mant) and np.array_equal(e2, expo) and not pad.any()


def test_create_rejects_sizes_beyond_32_bit_offsets():
    """The documented size limits: every operand below 2^31 elements, a B tile's byte offsets below 2^31."""
    import ctypes
    L = atb.lib()
    h = ctypes.c_void_p()
    def create(M, N, K, tiles=(128, 256, 64, 256)):
        return L.atb_gemm_create(ctypes.byref(h), M, N, K, *tiles)
    assert create(256, 32768, 32768) == 0                    # K * N = 2^30 elements: B is 2 GiB, allowed
    L.atb_gemm_destroy(h)
    assert create(256, 65536, 32768) == 1                    # K * N = 2^31
    assert create(65536, 32768, 64) == 1                     # M * N = 2^31
    assert create(32768, 256, 65536) == 1                    # M * K = 2^31
    assert create(64, (1 << 23) + 256, 64) == 1              # N > 2^23
    assert create(64, 1 << 23, 64, (32, 256, 128, 256)) == 1  # 2 N (T_K + 1) >= 2^31 with T_K = 128
    assert create(64, 1 << 23, 64, (128, 256, 64, 256)) == 0
    L.atb_gemm_destroy(h)


def test_selector_against_measured_sweep():
    """The selector's pick against a measured sweep of every instance over 20 problem shapes (large squares, the
    N = 2048 shapes of the paper's Table 3, skinny problems): within 5 % of the fastest instance on each, and the
    predicted throughput of the pick within 30 % of its measurement (20 % but for M = 16)."""
    import os
    inst = atb.instances()
    rows = [l.split() for l in open(os.path.join(os.path.dirname(__file__), "measured", "mi355x_shape_sweep.txt"))
            if l.strip() and not l.startswith("#")]
    assert len(rows) == 20
    for f in rows:
        M, N, K = (int(x) for x in f[:3])
        meas = [float(x) for x in f[3:]]
        assert len(meas) == len(inst)
        pick = atb.select_tiles(M, N, K)[0]
        got = meas[inst.index(pick.tiles())]
        assert got >= 0.95 * max(meas), ((M, N, K), pick.tiles(), got, inst[meas.index(max(meas))], max(meas))
        assert abs(pick.pred_flops / 1e12 / got - 1) < (0.30 if M < 32 else 0.20), ((M, N, K), pick.tiles(), pick.pred_flops / 1e12, got)


def test_plans_report_the_kernel_that_runs():
    """A plan that the streaming kernel takes says so, with that kernel's launch; the others report their instance's."""
    info = {i: None for i in atb.instances()}
    for tiles in info:
        g = atb.Gemm(256, 256, 256, *tiles)
        assert not g.streams()
        info[tiles] = g.launch_info()
        g.close()
    def plan(M, N, K, tiles, b="bf16", c="bf16"):
        g = atb.Gemm(M, N, K, *tiles, b_format=b, c_format=c)
        out = g.streams(), g.launch_info()
        g.close()
        return out
    # (M, N, K), tiles, b, c -> rows x columns of a workgroup's tile, waves
    for shape, tiles, b, c, rows, cols, waves in [
            ((16, 8192, 8192), (32, 32, 256, 64), "bf16", "bf16", 16, 32, 8), ((16, 8192, 8192), (64, 64, 128, 128), "bf16", "bf16", 16, 32, 8),
            ((64, 14336, 4096), (64, 64, 128, 128), "bfp16", "bf16", 64, 64, 8), ((16, 5001, 4096), (32, 32, 256, 64), "bf16", "bf16", 16, 32, 8),
            ((16, 2000, 4096), (32, 32, 256, 64), "bfp16", "bfp16", 16, 32, 16), ((128, 4096, 4096), (256, 256, 64, 256), "bf16_t", "bf16", 64, 32, 8),
            ((500, 4096, 14336), (64, 64, 128, 128), "bf16", "bf16", 64, 128, 4)]:
        M, N, K = shape
        streams, i = plan(M, N, K, tiles, b, c)
        n = -(-N // 64) * 64 if c == "bfp16" else N
        assert streams and i.threads == 64 * waves and i.lds_bytes == waves * 16 * (cols + 4) * 4
        assert i.workgroups == -(-(-(-M // rows) * -(-n // cols)) // 8) * 8
    for shape, tiles in [((16, 8192, 1024), (32, 32, 256, 64)), ((16, 8192, 8192), (32, 64, 64, 64)), ((8192, 8192, 8192), (64, 64, 128, 128))]:
        streams, i = plan(*shape, tiles)
        assert not streams and (i.threads, i.lds_bytes) == (info[tiles].threads, info[tiles].lds_bytes)
    assert atb.lib().atb_gemm_streams(None) == 0


def test_plans_name_the_tiles_that_run():
    """atb_gemm_kernel: the plan's factors, or those that run in their place, and all the LDS that a workgroup takes."""
    def kernel(shape, tiles, b="bf16", c="bf16"):
        g = atb.Gemm(*shape, *tiles, b_format=b, c_format=c)
        k, info = g.kernel(), g.launch_info()
        assert (k.streams, k.threads, k.workgroups) == (int(g.streams()), info.threads, info.workgroups)
        g.close()
        return k
    for tiles in atb.instances():
        k = kernel((256, 256, 256), tiles)
        assert k.tiles() == tiles and not k.streams and k.lds_bytes <= 160 * 1024
    wide, small, mid = (128, 128, 64, 256), (64, 64, 64, 64), (64, 128, 64, 128)
    for tiles in (mid, (128, 128, 64, 128)):
        assert kernel((1500, 3001, 2056), tiles).tiles() == wide                                   # odd N, many tiles
        assert kernel((1500, 3000, 2056), tiles).tiles() == tiles == kernel((51200, 65, 2056), tiles).tiles()
    for tiles in ((256, 256, 64, 256), (128, 128, 64, 256)):
        assert kernel((500, 500, 520), tiles, "bf16_t").tiles() == small and kernel((1500, 1500, 520), tiles, "bf16_t").tiles() == mid
        assert kernel((4096, 4096, 520), tiles, "bf16_t").tiles() == tiles == kernel((500, 500, 520), tiles).tiles()
    # LDS: a third B buffer for odd N, B in BFP16, panels of B in LDS (64 rows of row-major B), partial sums alone
    a, b = 2 * 64 * (128 * 2 + 16), 128 * 128 * 2
    assert kernel((600, 5001, 760), (64, 64, 128, 128)).lds_bytes == a + 2 * b and kernel((600, 5001, 1024), (64, 64, 128, 128)).lds_bytes == a + 3 * b
    assert kernel((600, 5000, 760), (64, 64, 128, 128), "bfp16").lds_bytes == a + 2 * 128 * (128 * 2 + 16)
    for shape, cols in (((1024, 2048, 4096), 128), ((64, 14336, 4096), 64)):
        k = kernel(shape, (64, 64, 128, 128))
        ring, panel_a, partial = 2 * 64 * cols * 2, 64 * 72, 64 * (cols + 4) * 4
        assert k.streams and k.tiles() == (64, 64, 64, cols) and k.lds_bytes == partial + 3 * ring + 4 * panel_a
    k = kernel((16, 8192, 8192), (32, 32, 256, 64))
    assert k.streams and k.tiles() == (16, 16, 64, 32) and k.lds_bytes == 8 * 16 * 36 * 4


def test_bfp16_bytes_refuses_floats_also_from_its_cache():
    assert atb.bfp16_bytes(24, 136) == atb.bfp16_layout(24, 136).bytes
    for bad in ((24.0, 136), (24, 136.0)):
        with pytest.raises(ctypes.ArgumentError):
            atb.bfp16_bytes(*bad)


def test_gpu_cases_reach_every_streaming_variant(monkeypatch, capfd):
    """The shapes of test_gpu_skinny.py go where that file says, and reach every variant that any problem is sent to and every one that is
    compiled (read from the library)."""
    import test_gpu_skinny as t
    from paper_2511_16041_amd import build
    from test_kernel_resources import READELF, kernels
    monkeypatch.setenv("ATB_LOG", "1")

    def logged(plans):
        capfd.readouterr()
        for g in plans:
            g.close()
        return t.variants(capfd.readouterr().err)

    def gpu_cases():
        for shape in t.SHAPES:
            for b, c in t.COMBOS:
                g = t.plan(shape, b, c)
                assert g.streams() == (c not in t.PIPELINE.get((shape, b), ())), (shape, b, c)
                yield g
        yield t.plan(t.WIDE_AND_LONG, "bf16", "bf16")

    def many_problems():
        for M in (1, 17, 33, 49, 65, 100, 128, 193, 256, 300, 512, 1000, 4100, 16384):
            for N in (32, 65, 200, 1024, 2050, 4096, 8001, 8194, 12288, 16384, 16448, 24001, 32768, 33000, 50000, 50257, 70000):
                for K in (1032, 1288, 1600, 2560, 4096, 5632, 8192, 14336):
                    if M * -(-N // 64) * 64 < 2 ** 31:
                        for b in ("bf16", "bf16_t", "bfp16"):
                            yield t.plan((M, N, K), b, "bf16")

    two = logged(t.plan(shape, "bfp16", c) for shape in t.TWO_PANELS for c in t.BOTH)
    assert {v[1:] for v in two} == {(32, 64, 512, 2), (48, 64, 512, 2), (64, 64, 512, 2), (64, 32, 512, 2)}
    reached = logged(gpu_cases()) | two
    sent = logged(many_problems())
    assert len(reached) == 47 and sent <= reached, sent - reached
    if os.path.exists(READELF):
        forms = ["bf16", "bf16_t", "bfp16", "bf16 odd"]            # template arguments: form of B, blocks of 16 rows, of 16 columns, waves, panels
        compiled = set()
        for name in kernels(build.ensure_built()):
            m = re.search(r"skinny_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d+)ELi(\d)E", name)
            if m:
                f, mb, nb, w, d = (int(x) for x in m.groups())
                compiled.add((forms[f], 16 * mb, 16 * nb, 64 * w, d))
        assert compiled == reached


def test_device_calls_refuse_host_tensors():
    """What the binding checks before any launch (no GPU is needed to be refused): in Python what quantise reads, the rest in the extension."""
    import torch
    g = atb.Gemm(8, 16, 64, 32, 64, 64, 64)
    a, b, c = torch.zeros(atb.bfp16_bytes(8, 64), dtype=torch.uint8), torch.zeros(64, 16, dtype=torch.bfloat16), torch.zeros(8, 16, dtype=torch.bfloat16)
    with pytest.raises(AssertionError):
        g.run(a, b, c)
    with pytest.raises(TypeError):
        g.run(a, b.float().numpy(), c)
    with pytest.raises(AssertionError):
        atb.bfp16_quantize(torch.zeros(8, 64))
    with pytest.raises(AssertionError):
        atb.bfp16_decode(a, 8, 64)
    g.close()


def _on_device(size, dtype, strides=None):
    """A tensor that says that it is on the GPU and has no memory: what is refused before a launch needs no GPU to be tested."""
    import torch

    class OnDevice(torch.Tensor):
        @staticmethod
        def __new__(cls):
            return torch.Tensor._make_wrapper_subclass(cls, size, strides=strides, dtype=dtype, device="cuda")

        @classmethod
        def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
            raise NotImplementedError(func)
    return OnDevice()


@pytest.mark.parametrize("b_format,c_format", [("bf16", "bf16"), ("bf16_t", "bf16"), ("bfp16", "bfp16")])
def test_run_refuses_operands_that_a_kernel_would_read_or_store_past(b_format, c_format):
    """C in pageable host memory, and buffers whose bytes are not in a row (strided, one element repeated)."""
    import torch
    M, N, K = 8, 16, 64
    g = atb.Gemm(M, N, K, 64, 128, 64, 256, b_format=b_format, c_format=c_format)
    def buffer(rows, cols, strides=None):
        return _on_device((atb.bfp16_bytes(rows, cols),), torch.uint8, strides)
    a = buffer(M, K)
    b = buffer(N, K) if b_format == "bfp16" else _on_device((K, N) if b_format == "bf16" else (N, K), torch.bfloat16)
    c = buffer(M, N) if c_format == "bfp16" else _on_device((M, N), torch.bfloat16)
    host = torch.zeros(c.shape, dtype=c.dtype)
    bad = [(a, b, host), (buffer(M, K, (2,)), b, c), (buffer(M, K, (0,)), b, c)]
    if b_format == "bfp16":
        bad += [(a, buffer(N, K, (2,)), c), (a, buffer(N, K, (0,)), c)]
    if c_format == "bfp16":
        bad += [(a, b, buffer(M, N, (2,))), (a, b, buffer(M, N, (0,)))]
    for args in bad:
        with pytest.raises(AssertionError):
            g.run(*args)
    g.close()


def test_quantise_and_decode_refuse_what_a_kernel_would_read_or_store_past():
    import torch
    M, K = 8, 64
    n = atb.bfp16_bytes(M, K)
    f32 = _on_device((M, K), torch.float32)
    for out in (torch.zeros(n, dtype=torch.uint8), _on_device((n - 1,), torch.uint8), _on_device((n,), torch.int8), _on_device((n,), torch.uint8, (2,))):
        with pytest.raises(AssertionError):
            atb.bfp16_quantize(f32, out=out)
    for a in (_on_device((n - 1,), torch.uint8), _on_device((n // 4 - 1,), torch.float32), _on_device((n,), torch.uint8, (2,)), _on_device((n,), torch.uint8, (0,))):
        with pytest.raises(AssertionError):
            atb.bfp16_decode(a, M, K)


def test_decode_keeps_the_type_of_an_allocation_failure():
    """A caller that frees memory and retries catches torch.OutOfMemoryError, which the allocation of the result raises."""
    import torch
    from torch.utils._python_dispatch import TorchDispatchMode

    class Full(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise torch.OutOfMemoryError("no room")
    a = _on_device((atb.bfp16_bytes(8, 64),), torch.uint8)
    with pytest.raises(torch.OutOfMemoryError, match="no room"), Full():
        atb.bfp16_decode(a, 8, 64)


def _package_copy(tmp_path):
    """The package as built, without the extension module, in a folder of its own."""
    for part in ("paper_2511_16041_amd", "include"):
        shutil.copytree(os.path.join(ROOT, part), tmp_path / part, ignore=shutil.ignore_patterns("_launch*.so", "_build", "__pycache__"))
    return tmp_path


def test_the_library_needs_no_torch(tmp_path):
    """The C ABI and the host-only calls load, and are not built again, where there is neither torch nor the extension module, and however
    new the extension module's source is."""
    root = _package_copy(tmp_path)
    os.utime(root / "paper_2511_16041_amd" / "csrc" / "atb_binding.cpp", (2 ** 31, 2 ** 31))
    code = textwrap.dedent("""
        import os, sys
        sys.modules["torch"] = None               # importing it raises ImportError
        os.environ["PATH"] = ""                   # no compiler to be found by name
        import paper_2511_16041_amd as atb
        atb._build.HIPCC = "/nonexistent/hipcc"
        assert atb.bfp16_bytes(8, 64) > 0 and atb.select_tiles(256, 256, 256)
        atb.Gemm(8, 16, 64, 32, 64, 64, 64).close()
        print("no-torch ok")
    """)
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "no-torch ok" in r.stdout, r.stdout + r.stderr


def test_the_extension_module_belongs_to_one_python_and_one_torch(monkeypatch):
    """Another torch does not load what was built against this one: it finds nothing built under its own name."""
    import torch
    from paper_2511_16041_amd import build
    here = build.ensure_binding()
    assert os.path.exists(here) and sysconfig.get_config_var("SOABI") in here and torch.__version__ in here
    monkeypatch.setattr(torch, "__version__", torch.__version__ + ".other")
    built = []
    monkeypatch.setattr(build, "build_binding", lambda verbose=False: built.append(build.binding_path()))
    assert build.ensure_binding() != here and built == [build.binding_path()]
