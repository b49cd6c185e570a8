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


CH = lbm.Lattice.GRAPH_CHUNK


def _bad(rounds, seed):
    """A head that makes every step fall back."""
    blob = inputs.gnn_blob(seed, rounds, s_delta=1.0)
    o, _ = inputs.blob_offsets(rounds)["bh"]
    blob[o + 1], blob[o + 2] = 50.0, -50.0
    return torch.as_tensor(blob, device="cuda")


def _replays(eager, graphed, advance, rounds=3, extra=5):
    """Graph runs equal eager ones, replay after replay, with eager work in between."""
    for r in range(rounds):
        advance(eager, CH + extra, False)
        advance(graphed, CH + extra, True)
        torch.cuda.synchronize()
        assert graphed._graphs and not eager._graphs
        assert torch.equal(eager.a, graphed.a), f"replay {r}"
        assert eager.steps == graphed.steps
        lbm.lbm_moments(graphed.a.float())
        torch.cuda.synchronize()


# (lattices of more than 1024 nodes: smaller ones take whole runs in one launch)
@pytest.mark.parametrize("nx,ny,dtype", [(40, 36, torch.float32), (24, 50, torch.float64)])
def test_captured_channel_steps_replay(nx, ny, dtype):
    a, b = (lbm.Lattice(nx, ny, dtype) for _ in range(2))
    for lat in (a, b):
        lat.a.zero_()
        lat.step_channel(0.8, 1e-5)            # from the second buffer
    _replays(a, b, lambda lat, n, gr: lat.step_channel(0.8, 1e-5, n, graph=gr))


def test_captured_steps_replay_from_the_second_buffer():
    a, b = (lbm.Lattice(41, 37).init(*inputs.tgv_velocity(41, 37, 0.03)) for _ in range(2))
    for lat in (a, b):
        lat.step_bgk(0.7)
    _replays(a, b, lambda lat, n, gr: lat.step_bgk(0.7, n, graph=gr), rounds=2, extra=0)
    _replays(a, b, lambda lat, n, gr: lat.step_bgk(0.7, n, graph=gr), rounds=2, extra=1)


def _corrected(walls, blob):
    lat = gnn.GnnLattice(40, 36, blob, 0)
    if walls:
        lat.a.zero_()
        lat.sync_mass()
    else:
        lat.init(*inputs.tgv_velocity(40, 36, 0.04))
    return lat


def _advance(walls):
    if walls:
        return lambda lat, n, gr: lat.step_gnn_channel(0.75, 2e-4, n, graph=gr)
    return lambda lat, n, gr: lat.step_gnn(0.7, n, graph=gr)


def _same_gate(a, b):
    for x, y in ((a.fallback.flags, b.fallback.flags), (a.fallback.mass, b.fallback.mass),
                 (a.n_fallback, b.n_fallback)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("walls", [False, True])
def test_captured_fallbacks_of_the_per_node_network_replay(walls, bad):
    blob = _bad(0, 6) if bad else torch.as_tensor(inputs.gnn_blob(6, 0, s_delta=1e-4),
                                                  device="cuda")
    a, b = (_corrected(walls, blob) for _ in range(2))
    _replays(a, b, _advance(walls), rounds=2, extra=3)
    _same_gate(a, b)
    assert (int(b.n_fallback.item()) == b.steps) == bad


@pytest.mark.parametrize("walls", [False, True])
def test_threshold_and_blob_of_the_per_node_network_choose_the_graph(walls):
    blob, other = (torch.as_tensor(inputs.gnn_blob(s, 0, s_delta=1e-4), device="cuda")
                   for s in (7, 8))
    a, b = (_corrected(walls, blob) for _ in range(2))
    _replays(a, b, _advance(walls), rounds=1, extra=0)
    before = int(b.n_fallback.item())
    for lat in (a, b):
        lat.fallback.threshold = -1.0           # every step falls back
    _replays(a, b, _advance(walls), rounds=1, extra=0)
    assert int(b.n_fallback.item()) == before + CH
    for lat in (a, b):
        lat.fallback.threshold = 1e-6
        lat.blob = other
    _replays(a, b, _advance(walls), rounds=1, extra=0)
    assert int(b.n_fallback.item()) == before + CH
    assert len(b._graphs) == 3
    _same_gate(a, b)


@pytest.mark.parametrize("kind", ["bgk", "channel", "simple", "simple_channel"])
def test_runs_in_one_launch_replay_in_a_graph_of_the_caller(kind):
    """Lattices of one workgroup: a caller's own graph of a whole run, which falls
    back in the per-node network's."""
    nx, ny, n = (32, 32, 70) if kind in ("bgk", "simple") else (7, 20, 70)
    blob, ws = _bad(0, 9), lbm.Workspace()
    gen = torch.Generator(device="cuda").manual_seed(4)
    start = 1e-3 * torch.randn((ny, 9, nx), generator=gen, device="cuda")

    def run(src, dst, fb):
        if kind == "bgk":
            lbm.lbm_steps_bgk(src, dst, 0.7, n)
        elif kind == "channel":
            lbm.lbm_steps_channel(src, dst, 0.7, 1e-5, n)
        elif kind == "simple":
            gnn.lbm_steps_simple(src, dst, 0.7, blob, n, fb, ws)
        else:
            gnn.lbm_steps_simple_channel(src, dst, 0.7, 1e-5, blob, n, fb, ws)

    a, b, c = start.clone(), torch.empty_like(start), torch.empty_like(start)
    gates = [gnn.Fallback(nx * ny) for _ in range(2)]
    run(a, b, gnn.Fallback(nx * ny))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(a, b, gates[0])
    for r in range(3):
        graph.replay()
        run(a, c, gates[1])
        torch.cuda.synchronize()
        assert torch.equal(b, c), f"replay {r}"
        a.copy_(b)
        lbm.lbm_moments(a)
        torch.cuda.synchronize()
    if kind.startswith("simple"):
        for x, y in ((gates[0].flags, gates[1].flags), (gates[0].mass, gates[1].mass),
                     (gates[0].n_fallback, gates[1].n_fallback)):
            assert torch.equal(x, y)
        assert int(gates[0].n_fallback.item()) == 3 * n
