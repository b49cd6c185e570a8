"""Backward pass of the per-node network (zero rounds) in one kernel, where its
walk over the nodes can go wrong: groups past the row end, chunks whose two
groups lie in different rows, an odd last chunk, lanes without a second chunk,
several turns per wave."""
import numpy as np
import pytest
import torch

from paper_2504_14494_amd import gnn, inputs

pytestmark = pytest.mark.gpu


def _grad(g, G, taus, blob):
    B, ny, _, nx = g.shape
    saved = torch.empty(gnn.saved_bytes(B, nx, ny, 0), dtype=torch.uint8, device="cuda")
    gnn.simple_forward(g, taus, blob, saved=saved)
    return gnn.gnn_backward(G, g, saved, taus, blob, 0)


def _state(shape, amp, seed):
    planes = inputs.random_shifted_state(shape, amp, seed)
    return planes, torch.as_tensor(inputs.planes_to_rows(planes), device="cuda")


# the bar of the other oracle comparisons: BF16 operands of the gradient products
@pytest.mark.parametrize("B,ny,nx", [(1, 1, 1), (3, 5, 17), (1, 9, 100), (2, 33, 48), (1, 2, 16)])
def test_matches_oracle_gradient(orc, B, ny, nx):
    g, gd = _state((B, 9, ny, nx), 4e-3, 300 + nx)
    G, Gd = _state((B, 9, ny, nx), 1.0, 400 + nx)
    taus = np.float32(0.6 + 0.1 * np.arange(B))
    blob = inputs.gnn_blob(12, 0, s_delta=1.0)
    got = _grad(gd, Gd, torch.as_tensor(taus, device="cuda"),
                torch.as_tensor(blob, device="cuda")).double().cpu().numpy()
    w = orc.lattice()[2][:, None, None]
    ref = orc.gnn_backward(g.astype(np.float64) + w[None], G.astype(np.float64),
                           taus.astype(np.float64), blob.astype(np.float64), 0, mode=1, act=1)
    assert np.linalg.norm(got - ref) <= 2e-2 * np.linalg.norm(ref)


# sums of up to 3e5 FP32 terms in another order
@pytest.mark.parametrize("B,ny,nx", [(40, 75, 100), (33, 64, 64), (5, 128, 512)])
def test_is_additive_over_lattices(B, ny, nx):
    _, g = _state((B, 9, ny, nx), 4e-3, 5)
    _, G = _state((B, 9, ny, nx), 1.0, 6)
    taus = torch.linspace(0.6, 0.9, B, device="cuda")
    blob = torch.as_tensor(inputs.gnn_blob(12, 0, s_delta=1.0), device="cuda")
    whole = _grad(g, G, taus, blob).double()
    parts = sum(_grad(g[b:b + 1].contiguous(), G[b:b + 1].contiguous(), taus[b:b + 1], blob).double()
                for b in range(B))
    assert float((whole - parts).norm() / parts.norm()) <= 1e-4
