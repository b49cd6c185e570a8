"""Several BGK or channel steps in one pass (lbm_steps_*) against as many
single steps, value for value: the same arithmetic at every node, whatever
kernel a lattice's size selects."""
import ctypes

import pytest
import torch

from paper_2504_14494_amd import _lib, inputs, lbm

EINVAL = -1

# one workgroup (up to 1024 nodes), small and large tiles and the march, at the
# edges of their ranges, with partial tiles, strips and segments, and lattices
# narrower than a region
SIZES = [(1, 1), (4, 32), (1, 1024), (32, 32), (25, 41), (64, 64), (3, 700), (130, 63),
         (128, 256), (181, 182), (362, 361), (363, 363), (9, 15000), (512, 512), (835, 836),
         (1501, 503), (448, 1600), (449, 1700), (20, 40000), (1100, 2003)]


def _state(nx, ny, dtype):
    gen = torch.Generator(device="cuda").manual_seed(nx * 31 + ny)
    g = torch.randn((ny, 9, nx), generator=gen, device="cuda", dtype=torch.float64)
    return (3e-3 * g).to(dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_steps_at_once_equal_single_steps(nx, ny, dtype, walls):
    most = lbm.lbm_steps_max(nx, ny, dtype, walls)
    assert most >= 2
    one, many = ((lbm.lbm_step_channel, lbm.lbm_steps_channel) if walls else
                 (lbm.lbm_step_bgk, lbm.lbm_steps_bgk))
    args = (0.61, 1e-5) if walls else (0.61,)
    start = _state(nx, ny, dtype)
    a, b = start.clone(), torch.empty_like(start)
    for n in range(1, min(most, 9) + 1):
        one(a, b, *args)
        a, b = b, a
        out = torch.full_like(start, float("nan"))
        if n > 1:
            many(start, out, *args, n)
            assert torch.equal(out, a), f"{n} steps of {nx} x {ny}"


@pytest.mark.gpu
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("nx,ny", [(16, 16), (64, 48), (300, 200), (520, 520), (1501, 503)])
def test_lattice_runs_equal_single_steps(nx, ny, graph):
    """Any number of steps, split over launches and graphs, also from the
    second buffer."""
    lat, one = lbm.Lattice(nx, ny), lbm.Lattice(nx, ny)
    lat.load(_state(nx, ny, torch.float32))
    one.load(lat.a)
    for n in (1, 0, 7, 64 + 13, 128, 3):
        lat.step_bgk(0.7, n, graph=graph)
        for _ in range(n):
            one.step_bgk(0.7)
        assert lat.steps == one.steps
        assert torch.equal(lat.a, one.a), n


@pytest.mark.gpu
def test_blown_up_state_stays_not_finite_as_in_single_steps():
    start = _state(520, 300, torch.float32)
    start[100, 3, 200] = float("nan")
    start[7, 0, 0] = float("inf")
    out = torch.empty_like(start)
    lbm.lbm_steps_bgk(start, out, 0.6, 3)
    a, b = start, torch.empty_like(start)
    for _ in range(3):
        lbm.lbm_step_bgk(a, b, 0.6)
        a, b = b, torch.empty_like(a)
    assert torch.equal(torch.isnan(out), torch.isnan(a))
    assert torch.equal(out.nan_to_num(0.0), a.nan_to_num(0.0))


def test_most_steps_and_refusals_need_no_gpu():
    L = _lib.load()
    assert L.lbm_steps_max(0, 4, 0, 0) == 1
    for nx, ny in SIZES + [(8192, 8192), (100000, 7), (7, 100000)]:
        for f64 in (0, 1):
            for walls in (0, 1):
                assert L.lbm_steps_max(nx, ny, f64, walls) >= 2
    a, b = (ctypes.create_string_buffer(9 * 64 * 64 * 4) for _ in range(2))
    pa, pb = ctypes.addressof(a), ctypes.addressof(b)
    most = L.lbm_steps_max(64, 64, 0, 0)
    for n in (-1, 0, 1, most + 1):
        assert L.lbm_steps_bgk(pa, pb, 64, 64, 0.8, n, None) == EINVAL
    assert L.lbm_steps_bgk(None, pb, 64, 64, 0.8, 2, None) == EINVAL
    assert L.lbm_steps_bgk(pa, pa, 64, 64, 0.8, 2, None) == EINVAL
    assert L.lbm_steps_bgk(pa, pb, 64, 0, 0.8, 2, None) == EINVAL
    assert L.lbm_steps_bgk(pa, pb, 64, 64, 0.0, 2, None) == EINVAL
    assert L.lbm_steps_channel(pa, pb, 64, 64, 0.5, 1e-6, 2, None) == EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,dtype,captured", [
    (128, 128, torch.float32, True), (129, 128, torch.float32, False),
    (64, 128, torch.float64, True), (65, 128, torch.float64, False)])
def test_graph_is_taken_up_to_its_size(nx, ny, dtype, captured):
    start = torch.as_tensor(inputs.random_shifted_state((ny, 9, nx), 1e-3, 3), dtype=dtype)
    a, b = (lbm.Lattice(nx, ny, dtype).load(start) for _ in range(2))
    for n in (130, 64):
        a.step_bgk(0.7, n, graph=True)
        b.step_bgk(0.7, n)
    assert torch.equal(a.g, b.g) and a.steps == b.steps == 194
    assert bool(a._graphs) == captured
