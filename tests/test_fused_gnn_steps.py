"""Several gated corrected steps in one call (lbm_steps_gnn), which packs the weights
once, against as many single ones: message passing in the fused kernel, at its edge
and past it, and the per-node network (no rounds) within and past one workgroup."""
import pytest
import torch

from paper_2504_14494_amd import gnn, inputs

pytestmark = pytest.mark.gpu


def _setup(nx, ny, rounds, s_delta, trip):
    blob = inputs.gnn_blob(31, rounds, s_delta=s_delta)
    if trip:   # a head that drives populations negative at every step
        o, _ = inputs.blob_offsets(rounds)["bh"]
        blob[o + 1] += 50.0
        blob[o + 2] -= 50.0
    g = torch.as_tensor(inputs.random_shifted_state((ny, 9, nx), 1e-3, nx + 7 * ny), device="cuda")
    return torch.as_tensor(blob, device="cuda"), g


def _gate(g, threshold):
    return gnn.Fallback(g.numel() // 9 + float(g.double().sum()), threshold)


@pytest.mark.parametrize("nx,ny,rounds", [(1, 1, 1), (16, 4, 2), (17, 5, 1), (100, 60, 2), (128, 128, 2),
                                          (256, 129, 2), (64, 32, 3), (300, 211, 1), (16, 16, 0),
                                          (45, 23, 0), (128, 128, 0), (700, 301, 0)])
def test_several_steps_equal_single_ones(nx, ny, rounds):
    # every step kept, every step redone, some of each (a drift threshold at the
    # size of the steps' own rounding), and without the gate
    for s_delta, trip, threshold in ((1e-4, False, 1.0), (1.0, True, 1.0), (1e-4, False, 1e-8),
                                     (1e-4, False, None)):
        blob, start = _setup(nx, ny, rounds, s_delta, trip)
        one = None if threshold is None else _gate(start, threshold)
        a, b = start.clone(), torch.empty_like(start)
        for n in range(1, 7):
            if rounds:
                gnn.lbm_step_gnn(a, b, 0.7, blob, rounds, one)
            else:
                gnn.lbm_step_simple(a, b, 0.7, blob, one)
            a, b = b, a
            if n not in (1, 2, 5, 6):
                continue
            fb = None if threshold is None else _gate(start, threshold)
            s, d = start.clone(), torch.full_like(start, float("nan"))
            out = gnn.lbm_steps_gnn(s, d, 0.7, blob, n, rounds, fb)
            assert out is (d if n % 2 else s)
            assert torch.equal(out, a)
            assert torch.equal(d if out is s else s, b)
            if fb is not None:
                assert torch.equal(fb.flags, one.flags)
                assert torch.equal(fb.n_fallback, one.n_fallback)
                assert torch.equal(fb.mass, one.mass)


@pytest.mark.parametrize("rounds", [0, 2])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130])
def test_lattice_steps_with_and_without_a_graph(n, rounds):
    nx, ny = 48, 30
    blob, start = _setup(nx, ny, rounds, 1e-4, False)
    states = []
    for graph in (False, True):
        lat = gnn.GnnLattice(nx, ny, blob, rounds)
        lat.load(start)
        for _ in range(2):   # the second run replays what the first captured
            lat.step_gnn(0.7, n, graph=graph)
        states.append((lat.a.clone(), lat.fallback.mass.clone(), lat.steps))
    ref, tmp = start.clone(), torch.empty_like(start)
    fb = gnn.Fallback(0.0)
    lat = gnn.GnnLattice(nx, ny, blob, rounds)
    lat.load(start)
    fb.mass.copy_(lat.fallback.mass)
    for _ in range(2 * n):
        if rounds:
            gnn.lbm_step_gnn(ref, tmp, 0.7, blob, rounds, fb)
        else:
            gnn.lbm_step_simple(ref, tmp, 0.7, blob, fb)
        ref, tmp = tmp, ref
    for state, mass, steps in states:
        assert torch.equal(state, ref) and torch.equal(mass, fb.mass) and steps == 2 * n


def test_bad_step_count_is_rejected():
    blob, start = _setup(16, 4, 2, 1e-4, False)
    with pytest.raises(Exception, match="nsteps"):
        gnn.lbm_steps_gnn(start, torch.empty_like(start), 0.7, blob, 0)
