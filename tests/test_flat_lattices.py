"""Several BGK or channel steps at once on lattices of few rows, whose regions
and halos are mostly rows that the lattice does not have: as many steps as pay,
and value for value the single steps for any number that a call takes."""
import pytest
import torch

from paper_2504_14494_amd import _lib, lbm

# tiles that fill the card (regions of the lattice's own rows), fewer rows than
# the halo; then the march
TILES = [(20001, 1), (60000, 1), (480001, 1), (30001, 2), (240001, 2), (40001, 3), (120001, 4),
         (10001, 12), (29999, 16), (20003, 23)]
MARCH = [(700001, 1), (350001, 2), (233335, 3), (175001, 4)]


@pytest.mark.parametrize("f64", [0, 1])
@pytest.mark.parametrize("walls", [0, 1])
def test_few_rows_take_few_steps_at_once(walls, f64):
    """A step of ny rows costs ny + 2 (nsteps - 1) of them: once the lattice fills
    the card, no more than ny + 1 steps, and single ones of one row."""
    L = _lib.load()
    assert L.lbm_steps_max(480001, 1, f64, walls) == 1
    for nx, ny in [(240001, 2), (160001, 3)] + MARCH:
        assert 2 <= L.lbm_steps_max(nx, ny, f64, walls) <= ny + 1, (nx, ny)
    for nx, ny in [(2000, 1), (8000, 1), (4000, 2), (5000, 4)]:  # their launches count
        assert L.lbm_steps_max(nx, ny, f64, walls) == 8


@pytest.mark.gpu
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("nx,ny", TILES + MARCH)
def test_steps_of_few_rows_equal_single_steps(nx, ny, dtype, walls):
    most = lbm.lbm_steps_max(nx, ny, dtype, walls)
    march = nx * ny >= (700000 if dtype == torch.float32 else 500000)
    taken = ((3 if dtype == torch.float64 else 4) if walls else 4) if march else (
        8 if nx * ny <= 131072 else 5)
    assert most <= taken
    one, many = ((lbm.lbm_step_channel, lbm.lbm_steps_channel) if walls else
                 (lbm.lbm_step_bgk, lbm.lbm_steps_bgk))
    args = (0.61, 1e-5) if walls else (0.61,)
    gen = torch.Generator(device="cuda").manual_seed(nx + ny)
    start = (3e-3 * torch.randn((ny, 9, nx), generator=gen, device="cuda",
                                dtype=torch.float64)).to(dtype)
    a, b = start.clone(), torch.empty_like(start)
    for n in range(1, taken + 1):
        one(a, b, *args)
        a, b = b, a
        if n > 1:
            out = torch.full_like(start, float("nan"))
            many(start, out, *args, n)
            assert torch.equal(out, a), f"{n} steps of {nx} x {ny}"


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(60000, 1), (120001, 2)])
def test_runs_of_few_rows_keep_their_graphs(nx, ny):
    lat, one = lbm.Lattice(nx, ny), lbm.Lattice(nx, ny)
    gen = torch.Generator(device="cuda").manual_seed(3)
    lat.load(3e-3 * torch.randn((ny, 9, nx), generator=gen, device="cuda"))
    one.load(lat.a)
    for n in (64 + 7, 128):
        lat.step_bgk(0.7, n, graph=True)
        for _ in range(n):
            one.step_bgk(0.7)
        assert torch.equal(lat.a, one.a) and lat.steps == one.steps
    assert lat._graphs
