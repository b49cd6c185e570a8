"""Several gated steps of the per-node network in one call (lbm_steps_simple,
_channel) against as many single ones, and lattices that one workgroup holds
against the kernels of larger ones."""
import ctypes

import pytest
import torch

from paper_2504_14494_amd import _lib, gnn, inputs, lbm

SIZES = [(1, 1), (4, 32), (16, 8), (3, 43), (16, 16), (257, 1), (20, 25), (1, 512), (27, 19),
         (32, 32), (1024, 1)]


def _setup(nx, ny, s_delta=1e-4, trip=False):
    blob = inputs.gnn_blob(21, 0, s_delta=s_delta)
    if trip:   # a head that drives populations negative at every step
        o, _ = inputs.blob_offsets(0)["bh"]
        blob[o + 1] += 50.0
        blob[o + 2] -= 50.0
    g = torch.as_tensor(inputs.random_shifted_state((ny, 9, nx), 1e-3, nx + 7 * ny), device="cuda")
    return torch.as_tensor(blob, device="cuda"), g


def _gate(g, threshold):
    return gnn.Fallback(g.numel() // 9 + float(g.double().sum()), threshold)


def _single(walls, src, dst, blob, fb):
    if walls:
        return gnn.lbm_step_simple_channel(src, dst, 0.7, 1e-4, blob, fb)
    return gnn.lbm_step_simple(src, dst, 0.7, blob, fb)


def _several(walls, src, dst, blob, n, fb):
    if walls:
        return gnn.lbm_steps_simple_channel(src, dst, 0.7, 1e-4, blob, n, fb)
    return gnn.lbm_steps_simple(src, dst, 0.7, blob, n, fb)


@pytest.mark.gpu
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_several_steps_equal_single_ones(nx, ny, walls):
    # every step kept, every step redone, and some of each (a drift threshold
    # at the size of the steps' own rounding)
    for s_delta, trip, threshold in ((1e-4, False, 1.0), (1.0, True, 1.0), (1e-4, False, 1e-8)):
        blob, start = _setup(nx, ny, s_delta, trip)
        fb, one = _gate(start, threshold), _gate(start, threshold)
        a, b = start.clone(), torch.empty_like(start)
        for n in range(1, 8):
            _single(walls, a, b, blob, one)
            a, b = b, a
            if n in (1, 2, 7):
                fb = _gate(start, threshold)
                out = _several(walls, start, torch.full_like(start, float("nan")), blob, n, fb)
                assert torch.equal(out, a)
                assert fb.flags.item() == one.flags.item()
                assert fb.n_fallback.item() == one.n_fallback.item()
                assert abs(fb.mass.item() - one.mass.item()) <= 1e-13 * nx * ny
        if threshold == 1.0:
            assert one.n_fallback.item() == (7 if trip else 0)
        ungated = _several(walls, start, torch.empty_like(start), blob, 2, None)
        p, q = torch.empty_like(start), torch.empty_like(start)
        _single(walls, _single(walls, start, p, blob, None), q, blob, None)
        assert torch.equal(ungated, q)


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny", [(1, 1), (16, 8), (20, 25), (32, 32), (1024, 1)])
def test_one_workgroup_equals_the_collision_of_large_lattices(nx, ny):
    blob, start = _setup(nx, ny)
    fb = _gate(start, 1.0)
    out = gnn.lbm_step_simple(start, torch.empty_like(start), 0.7, blob, fb)
    tau = torch.full((1,), 0.7, device="cuda")
    ref, _ = gnn.simple_forward(lbm.lbm_stream(start)[None], tau, blob)
    assert torch.equal(out, ref[0]) and fb.n_fallback.item() == 0
    mass = nx * ny + out.double().sum().item()
    assert abs(fb.mass.item() - mass) <= 1e-9 * nx * ny   # FP32 sums per node
    fb = _gate(start, -1.0)
    out = gnn.lbm_step_simple(start, torch.empty_like(start), 0.7, blob, fb)
    assert torch.equal(out, lbm.lbm_step_bgk(start, torch.empty_like(start), 0.7))
    assert fb.flags.item() == 2 and fb.n_fallback.item() == 1
    assert abs(fb.mass.item() - nx * ny - out.double().sum().item()) <= 1e-13 * nx * ny
    fb = _gate(start, -1.0)
    out = gnn.lbm_step_simple_channel(start, torch.empty_like(start), 0.7, 1e-4, blob, fb)
    assert torch.equal(out, lbm.lbm_step_channel(start, torch.empty_like(start), 0.7, 1e-4))


@pytest.mark.gpu
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("nx,ny", [(4, 32), (32, 32), (33, 32)])
def test_lattice_runs_equal_single_steps(nx, ny, graph):
    blob, start = _setup(nx, ny)
    many, one = (gnn.GnnLattice(nx, ny, blob, 0).load(start) for _ in range(2))
    for n in (1, 70, 0, 5, 128):
        many.step_gnn(0.7, n, graph=graph)
        many.step_gnn_channel(0.7, 1e-4, n, graph=graph)
        for _ in range(n):
            one.step_gnn(0.7)
        for _ in range(n):
            one.step_gnn_channel(0.7, 1e-4)
        assert torch.equal(many.a, one.a) and many.steps == one.steps
        assert torch.equal(many.n_fallback, one.n_fallback)
        assert torch.equal(many.fallback.mass, one.fallback.mass)


def test_most_steps_and_refusals_need_no_gpu():
    L = _lib.load()
    assert L.lbm_steps_simple_max(32, 32) > 1 and L.lbm_steps_simple_max(33, 32) == 1
    assert L.lbm_steps_simple_max(0, 4) == 1
    buf = ctypes.create_string_buffer(9 * 40 * 40 * 4)
    out = ctypes.create_string_buffer(9 * 40 * 40 * 4)
    ws = ctypes.create_string_buffer(int(L.lbm_workspace_bytes(_lib.LBM_WS_SIMPLE, 1, 40, 40, 0)))
    par = ctypes.create_string_buffer(4 * int(L.gnn_blob_len(0)))
    p, o, w, b = (ctypes.addressof(v) for v in (buf, out, ws, par))
    for n, nx in ((0, 8), (-3, 8), (L.lbm_steps_simple_max(8, 8) + 1, 8), (2, 40)):
        assert L.lbm_steps_simple(p, o, nx, nx, 0.7, b, n, None, w, len(ws), None) == -1
        assert b"steps" in L.lbm_last_error()
    assert L.lbm_steps_simple(p, p, 8, 8, 0.7, b, 2, None, w, len(ws), None) == -1
    assert L.lbm_steps_simple_channel(p, o, 8, 8, 0.7, float("nan"), b, 2, None, w, len(ws),
                                      None) == -1
    assert L.lbm_steps_simple(p, o, 8, 8, 0.7, b, 2, None, None, 0, None) == -2
