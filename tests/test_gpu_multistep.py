"""Several D2V9 steps per launch (tiles on small grids, strips on large ones) against single
steps: lbm_step(n) gives bit for bit the state of n calls of lbm_step(1), in the same state
buffer, also when the launches are captured and replayed. Sizes at the kernels' edges: widths
around a strip (56 columns, 224 per block) and a tile, rows that wrap, grids narrower or
shorter than a tile, remainders of steps, on both sides of the line between the kernels."""
import pytest
import torch

from paper_1710_09472_amd import lbm

pytestmark = pytest.mark.gpu

# nx, ny: tiles (one block, ragged tiles, thin grids), larger grids of odd shapes (below 8 M nodes tiles
# as well; the strips' grids follow further down)
TILES = [(1, 1), (5, 3), (16, 16), (33, 18), (70, 9), (300, 5), (4, 131), (301, 290), (1000, 640)]
STRIPS = [(56, 24000), (223, 5900), (225, 5861), (1120, 1171), (65537, 21), (350000, 4)]


def _sim(nx, ny, storage, rounding, kind, seed=5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    N = nx * ny
    rand = lambda: torch.rand(N, device="cuda", generator=g)
    kw = dict(tau=0.7, storage=storage, dev_scale_log2=12 if storage == "f16" else 0, rounding=rounding)
    if kind != "open":
        kw["mask"] = (rand() < 0.15).to(torch.uint8)
    if kind == "soft":
        kw["s"] = 0.3 * rand()
    if kind in ("soft", "slip"):
        kw |= dict(E=(1e-5, -2e-5, 0.0), B=(0.0, 0.0, 1e-3), forcing="shift" if kind == "slip" else "source")
    if kind == "slip" and ny >= 3:
        kw["slip"] = lbm.SLIP_Y
    if kind == "walls":
        kw["E"] = (1e-5, 0.0, 0.0)
    sim = lbm.Simulation("D2V9", nx, ny, 1, **kw)
    rho = 1.0 + 0.02 * (rand().double() - 0.5)
    u = 0.02 * torch.stack([rand().double() - 0.5, rand().double() - 0.5])
    sim.init(rho, u)
    return sim


@pytest.mark.parametrize("kind", ["open", "walls", "soft", "slip"])
@pytest.mark.parametrize("storage,rounding", [("f32", "nearest"), ("f16", "nearest"), ("bf16", "stochastic")])
@pytest.mark.parametrize("nx,ny", TILES + STRIPS)
def test_same_bits_as_single_steps(nx, ny, storage, rounding, kind):
    for steps in (4, 23) if nx * ny < 655360 else (3, 9):
        one, many = (_sim(nx, ny, storage, rounding, kind) for _ in range(2))
        for _ in range(steps):
            one.step(1)
        many.step(steps)
        fa = one.export_f64()
        assert torch.equal(fa, many.export_f64()), steps
        # the state sits in the buffer that single steps leave it in
        assert torch.equal(fa, many.export_f64(many.bufs[steps & 1])), steps
        assert torch.equal(fa, one.export_f64(many.get_state())), steps
        one.step(1)
        many.step(1)
        assert torch.equal(one.export_f64(), many.export_f64()), steps


# strips in every storage format (N >= 8 M), tiles of each plan:
# 4 x 4, 8 x 8 and 20 x 18 nodes a block, exactly 256 of them, and one more along an axis
@pytest.mark.parametrize("kind", ["open", "walls", "soft", "slip"])
@pytest.mark.parametrize("storage,rounding", [("f32", "nearest"), ("f16", "nearest"), ("bf16", "stochastic")])
@pytest.mark.parametrize("nx,ny", [(225, 36001), (65537, 123), (350000, 23), (64, 64), (65, 64), (17, 45), (128, 128),
                                   (100, 129), (320, 288), (319, 271), (530, 501)])
def test_same_bits_on_larger_strips_and_each_plan(nx, ny, storage, rounding, kind):
    steps = 16 if nx * ny < 655360 else 8  # 9 + 7 or 7 + 7 + 1 + 1, 5 + 3
    one, many = (_sim(nx, ny, storage, rounding, kind) for _ in range(2))
    for _ in range(steps):
        one.step(1)
    many.step(steps)
    assert torch.equal(one.export_f64(), many.export_f64(many.bufs[0]))


# thin grids: tiles that span the short axis, of 32 nodes (256 and 257 of them along the long axis), longer
# ones and the longest a block holds, below and beyond 8 M nodes; few columns beyond 8 M nodes
@pytest.mark.parametrize("kind", ["open", "walls", "soft", "slip"])
@pytest.mark.parametrize("storage,rounding", [("f32", "nearest"), ("f16", "nearest"), ("bf16", "stochastic")])
@pytest.mark.parametrize("nx,ny", [(8192, 1), (8193, 1), (3, 8193), (300001, 1), (1, 300001), (40001, 3), (6, 40001),
                                   (20011, 7), (8, 99999), (8000003, 1), (4, 2000003), (1000003, 8), (99, 80809)])
def test_same_bits_on_thin_grids(nx, ny, storage, rounding, kind):
    one, many = (_sim(nx, ny, storage, rounding, kind) for _ in range(2))
    for _ in range(22):
        one.step(1)
    many.step(22)  # 17 + 5, or 5 + 5 + 5 + 5 + 1 + 1
    assert torch.equal(one.export_f64(), many.export_f64(many.bufs[0]))


@pytest.mark.parametrize("nx,ny", [(300, 290), (1120, 600)])
def test_captured_steps_replay(nx, ny):
    """A graph of an even number of steps advances the state on every replay."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        sim, ref = _sim(nx, ny, "f32", "nearest", "walls"), _sim(nx, ny, "f32", "nearest", "walls")
        sim.step(14)  # warm-up outside the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            sim.step(14)
        ref.step(14)
        for _ in range(3):
            graph.replay()
            ref.step(14)
            assert torch.equal(sim.export_f64(), ref.export_f64())
            torch.cuda.synchronize()


def _thermal(n, storage, order):
    g = torch.Generator(device="cuda").manual_seed(7)
    noise = lambda: 0.01 * (torch.rand(n, device="cuda", generator=g).double() - 0.5)
    sim = lbm.Simulation("D1V7", n, 1, 1, tau=0.8, theta=0.25, mu=1.0, storage=storage, order=order,
                         dev_scale_log2=17 if storage == "f16" else 0)
    k = lbm.compute_constants("D1V7", "fd", 0.25, 1.0)
    sim.init(1.0 + noise(), noise(), k["I2"] / k["I0"] * (1.0 + noise()))
    return sim


@pytest.mark.parametrize("storage,order", [("f32", 4), ("f16", 4), ("bf16", 3)])
@pytest.mark.parametrize("n", [1, 2, 7, 63, 479, 480, 481, 511, 513, 1920, 1923, 70001])
def test_thermal_same_bits_as_single_steps(n, storage, order):
    for steps in (3, 4, 23):
        one, many = _thermal(n, storage, order), _thermal(n, storage, order)
        for _ in range(steps):
            one.step(1)
        many.step(steps)
        fa = one.export_f64()
        assert torch.equal(fa, many.export_f64()), steps
        assert torch.equal(fa, many.export_f64(many.bufs[steps & 1])), steps


def _sim3(nx, ny, nz, storage, rounding, kind):
    g = torch.Generator(device="cuda").manual_seed(9)
    N = nx * ny * nz
    rand = lambda: torch.rand(N, device="cuda", generator=g)
    kw = dict(tau=0.7, storage=storage, dev_scale_log2=12 if storage == "f16" else 0, rounding=rounding)
    if kind != "open":
        kw["mask"] = (rand() < 0.12).to(torch.uint8)
    if kind == "soft":
        kw["s"] = 0.3 * rand()
    if kind in ("soft", "slip"):
        kw |= dict(E=(1e-5, -2e-5, 1e-5), B=(1e-3, 0.0, 1e-3), forcing="shift" if kind == "slip" else "source")
    if kind == "slip":
        kw["slip"] = (lbm.SLIP_Y if ny >= 3 else 0) | (lbm.SLIP_Z if nz >= 3 else 0)
    if kind == "walls":
        kw["E"] = (1e-5, 0.0, 0.0)
    sim = lbm.Simulation("D3V19", nx, ny, nz, **kw)
    sim.init(1.0 + 0.02 * (rand().double() - 0.5), 0.02 * torch.stack([rand().double() - 0.5 for _ in range(3)]))
    return sim


# 3D grids from the sizes at which two steps may share a launch (FP32: N >= 500000; 16 bits: N >= 2 M without
# solids and source term, N >= 8 M with solids): widths around a block's 64 columns, heights around its 13
# rows, thin axes (the thinnest are planned for single steps; test_gpu_multistep_instances.py asserts the
# kernel it runs)
LARGE3 = [(65, 14, 551), (63, 100, 80), (130, 27, 143), (3, 410, 409), (1, 1000, 501), (700, 751, 1), (1024, 2, 250),
          (250, 13, 155), (64, 26, 301)]


@pytest.mark.parametrize("nx,ny,nz,storage,rounding,kind",
                         [(*d, "f32", "nearest", k) for d in LARGE3 for k in ("open", "walls", "soft", "slip")]
                         + [(*d, st, "nearest", "open") for d in [(65, 250, 124), (130, 1027, 15)] for st in ("f16", "bf16")]
                         + [(*d, *st, k) for d in [(129, 250, 250), (64, 14, 8930)] for k in ("walls", "soft", "slip")
                            for st in (("f16", "stochastic"), ("bf16", "nearest"))])
def test_3d_two_steps_per_launch_same_bits(nx, ny, nz, storage, rounding, kind):
    one, many = (_sim3(nx, ny, nz, storage, rounding, kind) for _ in range(2))
    for _ in range(9):
        one.step(1)
    many.step(9)  # 4 launches of two, one of one
    fa = one.export_f64()
    assert torch.equal(fa, many.export_f64())
    assert torch.equal(fa, many.export_f64(many.bufs[1]))


@pytest.mark.parametrize("kind", ["open", "walls", "soft", "slip"])
@pytest.mark.parametrize("storage,rounding", [("f32", "nearest"), ("f16", "stochastic"), ("bf16", "nearest")])
@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1), (3, 2, 5), (64, 13, 9), (65, 14, 7), (63, 12, 3), (128, 26, 40),
                                      (70, 100, 33), (200, 11, 67)])
def test_3d_same_bits_as_single_steps(nx, ny, nz, storage, rounding, kind):
    for steps in (4, 11):
        one, many = (_sim3(nx, ny, nz, storage, rounding, kind) for _ in range(2))
        for _ in range(steps):
            one.step(1)
        many.step(steps)
        fa = one.export_f64()
        assert torch.equal(fa, many.export_f64()), steps
        assert torch.equal(fa, many.export_f64(many.bufs[steps & 1])), steps
        one.step(1)
        many.step(1)
        assert torch.equal(one.export_f64(), many.export_f64()), steps
