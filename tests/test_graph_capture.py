"""What Lattice captures into a graph has run before, outside the capture."""
import pytest
import torch

from paper_2504_14494_amd import gnn, inputs, lbm

pytestmark = pytest.mark.gpu


def _watch(monkeypatch, module, names):
    calls = []

    def wrap(name):
        real = getattr(module, name)

        def call(*args):
            # arguments of one kind of call differ in its tensors only
            key = (name,) + tuple(x for x in args if isinstance(x, (int, float)))
            calls.append((key, torch.cuda.is_current_stream_capturing()))
            return real(*args)
        monkeypatch.setattr(module, name, call)
    for name in names:
        wrap(name)
    return calls


@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("nx,ny,dtype", [(64, 48, torch.float32), (40, 36, torch.float64),
                                         (60000, 1, torch.float32), (480001, 1, torch.float32)])
def test_captured_steps_have_been_warmed_up(monkeypatch, nx, ny, dtype, walls):
    calls = _watch(monkeypatch, lbm, ["lbm_step_bgk", "lbm_steps_bgk", "lbm_step_channel",
                                      "lbm_steps_channel"])
    lat = lbm.Lattice(nx, ny, dtype)
    lat.a.zero_()
    if walls:
        lat.step_channel(0.7, 1e-6, 64, graph=True)
    else:
        lat.step_bgk(0.7, 64, graph=True)
    assert lat._graphs
    captured = {key for key, inside in calls if inside}
    assert captured and captured <= {key for key, inside in calls if not inside}


@pytest.mark.parametrize("rounds", [2, 0])
def test_captured_corrected_steps_have_been_warmed_up(monkeypatch, rounds):
    names = ["lbm_step_gnn", "lbm_steps_gnn", "lbm_step_simple", "lbm_steps_simple"]
    calls = _watch(monkeypatch, gnn, names)
    blob = torch.as_tensor(inputs.gnn_blob(3, rounds, s_delta=1e-4), device="cuda")
    lat = gnn.GnnLattice(40, 36, blob, rounds)
    lat.a.zero_()
    lat.sync_mass()
    lat.step_gnn(0.7, 64, graph=True)
    assert lat._graphs
    assert {k[0] for k, inside in calls if inside} <= {k[0] for k, inside in calls if not inside}
