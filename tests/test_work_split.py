"""How chunks of nodes are shared among waves changes no result: a batch whose
waves draw them two, three or four at a time gives each lattice, value for
value, what it gives alone (one chunk per wave)."""
import pytest
import torch

from paper_2504_14494_amd import gnn, inputs

pytestmark = pytest.mark.gpu


# chunks of 64 nodes: 150 rows x 1 or 2, batches of 20 to 120 lattices give
# the resident waves (three or four blocks of four per CU) from less than one
# to more than four chunks each
@pytest.mark.parametrize("rounds", [0, 2])
@pytest.mark.parametrize("batch,nx", [(20, 64), (63, 64), (90, 50), (40, 100), (60, 70), (120, 64)])
def test_batch_equals_its_lattices_alone(rounds, batch, nx):
    ny = 150
    blob = torch.as_tensor(inputs.gnn_blob(8, rounds, s_delta=1e-2), device="cuda")
    g = torch.as_tensor(inputs.random_shifted_state((batch, ny, 9, nx), 4e-3, seed=batch),
                        device="cuda")
    tau = torch.linspace(0.6, 0.9, batch, device="cuda")
    post, z = gnn.collide(g, tau, blob, rounds, want_z=True)
    saved = torch.empty(gnn.saved_bytes(batch, nx, ny, rounds), dtype=torch.uint8, device="cuda")
    kept, _ = gnn.collide(g, tau, blob, rounds, saved=saved)
    assert torch.equal(kept, post)
    for b in (0, 1, batch // 2, batch - 1):
        one, z1 = gnn.collide(g[b:b + 1].contiguous(), tau[b:b + 1], blob, rounds, want_z=True)
        assert torch.equal(one[0], post[b]) and torch.equal(z1[0], z[b]), b
