"""Every instance of the multi-step kernels (solids, porosity, forcing and slip chosen independently)
against single steps, bit for bit, on grids that are planned for the kernel (asserted), and captured
sequences of each kernel replayed."""
import pytest
import torch

from paper_1710_09472_amd import lbm

pytestmark = pytest.mark.gpu

FORMATS = [("f32", "nearest"), ("f16", "nearest"), ("bf16", "stochastic")]
FORCES = {"none": {}, "E": dict(E=(1e-5, -2e-5, 0.0)), "EB": dict(E=(1e-5, -2e-5, 0.0), B=(0.0, 0.0, 1e-3)),
          "shift": dict(E=(1e-5, -2e-5, 0.0), B=(0.0, 0.0, 1e-3), forcing="shift")}


def _sim(lattice, dims, storage, rounding, solids, soft, force, slip=0):
    g = torch.Generator(device="cuda").manual_seed(11)
    N = dims[0] * dims[1] * dims[2]
    D = 2 if lattice == "D2V9" else 3
    rand = lambda: torch.rand(N, device="cuda", generator=g)
    kw = dict(tau=0.7, storage=storage, dev_scale_log2=12 if storage == "f16" else 0, rounding=rounding, slip=slip)
    if solids:
        kw["mask"] = (rand() < 0.1).to(torch.uint8)
    if soft:
        kw["s"] = 0.3 * rand()
    sim = lbm.Simulation(lattice, *dims, **kw, **FORCES[force])
    sim.init(1.0 + 0.02 * (rand().double() - 0.5), 0.02 * torch.stack([rand().double() - 0.5 for _ in range(D)]))
    return sim


def _same_bits(kernel, steps, lattice, dims, storage, rounding, solids, soft, force, slip=0):
    one, many = (_sim(lattice, dims, storage, rounding, solids, soft, force, slip) for _ in range(2))
    assert lbm.launch_plan(many.params, steps, solids, soft)[0] == kernel
    for _ in range(steps):
        one.step(1)
    many.step(steps)
    assert torch.equal(one.export_f64(), many.export_f64(many.bufs[steps & 1]))


@pytest.mark.parametrize("storage,rounding", FORMATS)
@pytest.mark.parametrize("force", list(FORCES))
@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("solids,slip", [(False, 0), (True, 0), (False, lbm.SLIP_Y), (True, lbm.SLIP_Y)])
@pytest.mark.parametrize("kernel,dims", [("k_tile", (70, 45, 1)), ("k_march", (1121, 7141, 1))])
def test_2d_instances(kernel, dims, solids, slip, soft, force, storage, rounding):
    _same_bits(kernel, 8, "D2V9", dims, storage, rounding, solids, soft, force, slip)  # 7 + 1 or 1; 5 + 3


# FP32 grids around a block's 64 columns and 13 rows that fill the CUs
@pytest.mark.parametrize("force", list(FORCES))
@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("solids,slip", [(False, 0), (True, 0), (False, 3), (True, 3)])
@pytest.mark.parametrize("dims", [(63, 183, 200), (127, 209, 151)])
def test_3d_instances_f32(dims, solids, slip, soft, force):
    _same_bits("k_march3", 8, "D3V19", dims, "f32", "nearest", solids, soft, force, slip)


@pytest.mark.parametrize("storage,rounding", FORMATS[1:])
@pytest.mark.parametrize("force", list(FORCES))
@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("solids,slip", [(True, 0), (False, 3), (True, 3)])
def test_3d_instances_16_bit_with_solids(solids, slip, soft, force, storage, rounding):
    _same_bits("k_march3", 4, "D3V19", (127, 391, 162), storage, rounding, solids, soft, force, slip)


@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("force", ["none", "shift"])
@pytest.mark.parametrize("soft", [False, True])
def test_3d_instances_16_bit_open(soft, force, storage):
    _same_bits("k_march3", 8, "D3V19", (128, 129, 127), storage, "nearest", False, soft, force)


# the sides of the planning lines: the largest grids of single steps beside the smallest of k_march3
@pytest.mark.parametrize("kernel,dims", [("k_step", (64, 64, 121)), ("k_march3", (64, 64, 128)), ("k_march3", (67, 92, 154)),
                                         ("k_march3", (256, 8, 256)), ("k_step", (512, 512, 2))])
def test_3d_plan_lines(kernel, dims):
    _same_bits(kernel, 8, "D3V19", dims, "f32", "nearest", False, False, "E")


@pytest.mark.parametrize("kernel,lattice,dims", [("k_march", "D2V9", (1121, 7141, 1)), ("k_march3", "D3V19", (128, 65, 130)),
                                                 ("k_thermal_multi", "D1V7", (70001, 1, 1))])
def test_captured_steps_replay(kernel, lattice, dims):
    """A graph of an even number of steps advances the state on every replay, with eager work and
    synchronisations between replays; the first launch of an instance may be a captured one."""
    def make():
        if lattice != "D1V7":
            return _sim(lattice, dims, "f32", "nearest", True, False, "E")
        sim = lbm.Simulation("D1V7", *dims, tau=0.8, theta=0.25, mu=1.0)
        x = torch.arange(dims[0], device="cuda", dtype=torch.float64)
        sim.init(1.0 + 0.01 * torch.sin(0.1 * x), 0.01 * torch.cos(0.2 * x))
        return sim

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim, ref = make(), make()
        assert lbm.launch_plan(sim.params, 8, solids=lattice != "D1V7")[0] == kernel
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(8)
        for _ in range(4):
            graph.replay()
            for _ in range(8):
                ref.step(1)
            assert torch.equal(sim.export_f64(), ref.export_f64())
            torch.cuda.synchronize()
