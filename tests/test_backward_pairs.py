"""Backward pass of the message-passing network where its layout can go wrong:
the buffers between its kernels are laid out by groups of up to 16 columns, and
two waves share each partial gradient.  Row ends one column past, at and one
short of a group; chunks whose second group lies past the lattice; blocks with
pairs past the last chunk."""
import numpy as np
import pytest
import torch

from paper_2504_14494_amd import gnn, inputs

pytestmark = pytest.mark.gpu


def _inputs(B, ny, nx, R):
    g = inputs.random_shifted_state((B, 9, ny, nx), 4e-3, seed=500 + nx)
    G = inputs.random_shifted_state((B, 9, ny, nx), 1.0, seed=600 + nx)
    taus = np.float32(0.6 + 0.1 * np.arange(B))
    return g, G, taus, inputs.gnn_blob(13, R, s_delta=1.0)


def _device(g, G, taus, blob, R):
    B, _, ny, nx = g.shape
    gd, Gd = (torch.as_tensor(inputs.planes_to_rows(a), device="cuda") for a in (g, G))
    t, b = torch.as_tensor(taus, device="cuda"), torch.as_tensor(blob, device="cuda")
    saved = torch.empty(gnn.saved_bytes(B, nx, ny, R), dtype=torch.uint8, device="cuda")
    gnn.gnn_forward(gd, t, b, R, saved=saved)
    return lambda ws=None: gnn.gnn_backward(Gd, gd, saved, t, b, R, ws=ws)


# the bar of the other oracle comparisons: BF16 operands of the gradient products
@pytest.mark.parametrize("B,ny,nx,R", [(1, 3, 15, 1), (1, 5, 16, 2), (2, 3, 17, 1), (1, 7, 31, 1),
                                       (1, 2, 33, 3), (3, 3, 50, 1)])
def test_matches_oracle_gradient(orc, B, ny, nx, R):
    g, G, taus, blob = _inputs(B, ny, nx, R)
    got = _device(g, G, taus, blob, R)().double().cpu().numpy()
    w = orc.lattice()[2][:, None, None]
    ref = orc.gnn_backward(g.astype(np.float64) + w[None], G.astype(np.float64),
                           taus.astype(np.float64), blob.astype(np.float64), R, mode=1)
    assert np.linalg.norm(got - ref) <= 2e-2 * np.linalg.norm(ref)


class _Filled(gnn.Workspace):
    def get(self, nbytes):
        buf = super().get(nbytes)
        buf[: buf.numel() // 4 * 4].view(torch.float32).fill_(self.value)
        return buf


# nothing of the workspace is read before it is written, and every store holds
# what was computed: all runs give the same bits
@pytest.mark.parametrize("B,ny,nx,R", [(3, 37, 130, 1), (2, 5, 17, 3), (4, 9, 250, 2),
                                       (3, 40, 64, 2), (1, 1, 1, 1)])
def test_same_bits_whatever_the_workspace_held(B, ny, nx, R):
    grad = _device(*_inputs(B, ny, nx, R), R)
    ws = _Filled()
    ref = None
    for k in range(12):
        ws.value = (1e37, float("nan"), -3.0)[k % 3]
        got = grad(ws).clone()
        ref = got if ref is None else ref
        assert torch.equal(got, ref)
    assert bool(torch.isfinite(ref).all())
