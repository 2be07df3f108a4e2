"""Host logic of bench.py (no GPU): the one-GPU refusal, the algorithmic bytes that
the roofline divides by the measured launch time, and the rule that HBM traffic from
the committed counters is reported only while the kernel code is the code they were
taken on."""
import shutil
import subprocess
import sys
from pathlib import Path

import numpy as np
import pytest

import bench
from paper_1710_09472_amd import lbm
from paper_1710_09472_amd import workloads as W

ROOT = Path(__file__).resolve().parents[1]


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, str(ROOT / "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       cwd=ROOT, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr and r.stdout == ""


def test_algorithmic_bytes():
    wl = W.throughput_2d(nx=64, ny=32)
    assert bench.algorithmic_bytes(wl, 9, 4) == 64 * 32 * 72
    assert bench.algorithmic_bytes(wl, 9, 2) == 64 * 32 * 36
    # obstacles: fluid nodes move their populations, every node has one byte of flag;
    # a porosity field adds 4 bytes per node
    wl = W.random_fields("D3V19", 10, 6, 5, seed=3, solid_fraction=0.2, soft=True)
    fluid = int((wl.mask == 0).sum())
    assert 0 < fluid < wl.N
    assert bench.algorithmic_bytes(wl, 19, 4) == fluid * 152 + wl.N + 4 * wl.N
    assert bench.wl_q(wl) == 19


def _copy_sources(tmp: Path) -> Path:
    dst = tmp / "paper_1710_09472_amd" / "csrc"
    dst.mkdir(parents=True)
    for name in ("lbm_device.h", "lbm_step_kernels.h", "lbm_kernels.hip", "lbm_thermal.hip"):
        shutil.copy(ROOT / "paper_1710_09472_amd" / "csrc" / name, dst / name)
    return dst


def test_code_hash_ignores_comments_not_code(tmp_path, monkeypatch):
    ref, ref_th = bench.kernel_code_hash(), bench.kernel_code_hash(thermal=True)
    src = _copy_sources(tmp_path)
    monkeypatch.setattr(bench, "ROOT", tmp_path)
    assert bench.kernel_code_hash() == ref
    f = src / "lbm_kernels.hip"
    f.write_text("// a comment line\n\n" + f.read_text().replace("\n", "  // trailing note\n", 1))
    assert bench.kernel_code_hash() == ref
    f.write_text(f.read_text() + "\nstatic int unused_marker = 0;\n")
    assert bench.kernel_code_hash() != ref
    # the thermal step's hash covers the device header and the thermal kernel file only
    assert bench.kernel_code_hash(thermal=True) == ref_th


def test_traffic_only_for_the_code_it_was_taken_on(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "PROFILE_DIR", tmp_path)
    tag = "k_step_D2V9_f32_throughput_2d"
    assert bench.traffic_from_profile(tag) is None  # no summary
    good = bench.kernel_code_hash()
    (tmp_path / f"{tag}_pmc.txt").write_text(f"hbm_bytes_per_launch: 1.25e+09\nkernel_code_sha256: {good}\n")
    assert np.isclose(bench.traffic_from_profile(tag), 1.25e9)
    (tmp_path / f"{tag}_pmc.txt").write_text("hbm_bytes_per_launch: 1.25e+09\nkernel_code_sha256: " + "0" * 64 + "\n")
    assert bench.traffic_from_profile(tag) is None


def test_oracle_blocks_equal_the_full_grid_oracle(oracle_lib):
    """The error figures of bench.py compare the GPU with the oracle on sampled blocks that the
    oracle recomputes on the windows of their dependence cones: on a grid the oracle runs
    whole, the blocks equal the full-grid run exactly (also where a window wraps around)."""
    wl = W.throughput_2d(nx=96, ny=80, seed=3)
    wl.u = 0.01 * np.random.default_rng(4).standard_normal((2, wl.N))
    steps, core = 12, 8
    centres = ((0, 0, 0), (90, 40, 0), (47, 79, 0))
    idx, rho_b, u_b = bench.oracle_blocks(wl, steps, core, centres)
    m = oracle_lib.OracleModel("D2V9", wl.nx, wl.ny, 1, tau=wl.tau)
    rho, u = m.moments(m.run(m.init_state(wl.rho, wl.u), steps))
    assert idx.size == len(centres) * core * core
    np.testing.assert_array_equal(rho_b, rho[idx])
    np.testing.assert_array_equal(u_b, u[:, idx])
    # the block of centre (90, 40) holds x = 90..95 and 0..1 (wrapped), y = 40..47
    b = idx[core * core:2 * core * core]
    assert set(b % wl.nx) == set(range(90, 96)) | {0, 1} and set(b // wl.nx) == set(range(40, 48))


def test_launch_plan_is_the_librarys():
    """The kernel and launch counts of a bench line are the library's own plan: remainder launches
    count (4096 x 4: 17 + 3 of 20 steps), and FP32 states of 4 GiB with solids take single steps."""
    wl = W.throughput_2d(nx=4096, ny=4)
    assert bench.launch_plan(wl, "f32", 20) == ("k_tile", 17, 2)
    assert bench.launch_plan(wl, "f32", 20, inplace=True) == ("k_step_aa_pull+k_step_aa_local", 1, 20)
    wl = W.throughput_2d(nx=16, ny=16)
    wl.nx, wl.ny = 12000, 10000  # (the plan takes the sizes alone)
    assert bench.launch_plan(wl, "f32", 20) == ("k_march", 5, 4)
    wl.mask = np.zeros(1, np.uint8)
    assert bench.launch_plan(wl, "f32", 20) == ("k_step", 1, 20)
    assert bench.launch_plan(wl, "f16", 21, "stochastic") == ("k_march", 5, 5)  # 4 of 5 steps, one of 1


def test_launch_plan_launches_and_errors():
    p3 = lbm.make_params("D3V19", 128, 128, 128)
    assert lbm.launch_plan(p3, 3) == ("k_step", 1, 3)  # launches of two steps come in pairs
    assert lbm.launch_plan(p3, 11) == ("k_march3", 2, 7)
    pt = lbm.make_params("D1V7", 1000, theta=0.25)
    assert [lbm.launch_plan(pt, n) for n in (1, 2, 9)] == [("k_thermal_step", 1, 1), ("k_thermal_step", 1, 2),
                                                         ("k_thermal_multi", 5, 3)]  # 5 + 3 + 1
    for bad in ((p3, 0, {}), (lbm.make_params("D2V9", 8, 8, tau=0.5), 1, {}), (pt, 1, {"solids": True})):
        with pytest.raises(lbm.LbmError):
            lbm.launch_plan(bad[0], bad[1], **bad[2])


def test_thin_grids_are_planned_by_their_shape():
    """Strips write 56 of 64 columns and walk rows, so grids of few columns or rows take tiles at any
    size (FP32 states of 4 GiB and more single steps, the tiles' offsets being 32 bits wide)."""
    def plan(nx, ny, **kw):
        return lbm.launch_plan(lbm.make_params("D2V9", nx, ny, **kw), 34)

    for nx, ny in ((9_000_000, 1), (4_500_000, 2), (1_200_000, 8), (1, 9_000_000), (4, 2_250_000), (8, 1_125_000)):
        assert plan(nx, ny) == ("k_tile", 17, 2), (nx, ny)
    for nx, ny in ((9, 1_000_000), (64, 140_625), (99, 90_000)):
        assert plan(nx, ny)[:2] == ("k_tile", 5), (nx, ny)
    for nx, ny in ((100, 90_000), (1_000_000, 9), (4096, 4096)):
        assert plan(nx, ny)[:2] == ("k_march", 5), (nx, ny)
    assert plan(120_000_000, 1) == plan(1, 120_000_000) == ("k_step", 1, 34)
    assert plan(120_000_000, 1, storage="bf16") == ("k_tile", 17, 2)


def test_two_step_launches_of_3d_grids_are_planned_by_their_shape():
    """k_march3 pays for whole blocks of 64 x 13 columns: narrow and flat grids, on which it measured
    slower than single steps, keep those; the grids it gains on keep it."""
    def kernel(nx, ny, nz, solids=False, porosity=False, **kw):
        return lbm.launch_plan(lbm.make_params("D3V19", nx, ny, nz, **kw), 8, solids, porosity)[0]

    E, bf16 = {"E": (1e-6, 0, 0)}, {"storage": "bf16"}
    for dims in ((512, 512, 2), (1024, 512, 1), (4096, 2048, 1), (8, 256, 256), (1, 1000, 520)):
        assert kernel(*dims) == kernel(*dims, solids=True) == kernel(*dims, solids=True, porosity=True) == "k_step"
    for dims in ((256, 128, 16), (32, 128, 128)):  # even or faster without solids only
        assert (kernel(*dims, **E), kernel(*dims, solids=True, **E)) == ("k_march3", "k_step")
    # solids with porosity: the instances that spill lose from about two slots per node
    assert kernel(256, 16, 2048, True, True) == kernel(96, 96, 96, True, True) == "k_step"
    assert kernel(256, 16, 2048, True, True, **E) == kernel(96, 96, 96, True, True, **E) == "k_march3"
    for dims in ((1024, 1024, 8), (512, 512, 32), (256, 16, 2048), (32, 512, 512)):
        assert kernel(*dims, **bf16) == "k_step"
    # 16 bits with solids: walls and ordinary obstacles leave the single step ahead where rows lie on lines
    walls = dict(solids=True, E=(1e-6, 0, 0), **bf16)
    assert kernel(256, 256, 128, **walls) == kernel(512, 26, 640, **walls) == kernel(200, 200, 210, **walls) == "k_step"
    assert kernel(128, 256, 256, slip=3, **bf16) == kernel(229, 181, 388, porosity=True, slip=3, **bf16) == "k_step"
    assert kernel(229, 181, 388, **walls) == kernel(63, 360, 368, porosity=True, **walls) == "k_march3"
    assert kernel(208, 16, 858, slip=1) == kernel(256, 32, 256, porosity=True, slip=3, B=(0, 0, 1e-3)) == "k_step"
    assert kernel(256, 32, 256, porosity=True, slip=3) == kernel(96, 96, 96, slip=3, **E) == "k_march3"
    for dims in ((128, 128, 128), (256, 128, 128), (96, 96, 96), (65, 128, 128), (24, 160, 160)):
        assert kernel(*dims, **E) == "k_march3"
    assert kernel(256, 128, 128, True, E=(1e-6, 0, 0), B=(0, 0, 1e-3)) == kernel(128, 128, 128, True, True) == "k_march3"
    assert kernel(128, 256, 256, **bf16) == kernel(128, 256, 256, True, **bf16) == "k_march3"


def test_ragged_16_bit_tiles_take_launches_that_pay():
    """Tiles that reach beyond the grid (73 rows in four tiles of 24) take five steps per launch or
    single ones with 16-bit storage and porosity, and with stochastic rounding and a field single ones."""
    def plan(nx, ny, steps, porosity=False, **kw):
        return lbm.launch_plan(lbm.make_params("D2V9", nx, ny, **kw), steps, porosity=porosity)

    sr, E = {"storage": "f16", "rounding": "stochastic"}, {"E": (1e-6, 0, 0)}
    for args in ((8241, 73, 13, True), (1000, 700, 13, True)):
        assert plan(*args) == ("k_tile", 5, 3)  # 5 + 5 + 3
    assert plan(8241, 73, 13, **sr) == plan(1000, 700, 13, True, **sr, **E) == plan(50, 8533, 13, True, **sr, **E) \
        == ("k_tile", 5, 3)
    assert plan(8241, 73, 13, True, **sr) == plan(8241, 73, 13, True, storage="bf16", **E) == ("k_tile", 5, 5)
    assert plan(8241, 73, 13, True, **sr, **E) == ("k_step", 1, 13)
    assert plan(8241, 73, 3, True, storage="bf16") == ("k_step", 1, 3)
    assert plan(8975, 29, 13, True, storage="f16", **E) == ("k_step", 1, 13)
