"""How the work of a collision is split changes no result: a batch whose waves
draw chunks of nodes two, three or four at a time, or that goes through memory
between its kernels, gives each lattice, value for value, what it gives alone
(one chunk per wave; the fused kernel of small lattices)."""
import pytest
import torch

from paper_2504_14494_amd import gnn, inputs, lbm

pytestmark = pytest.mark.gpu

W = torch.tensor([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4, dtype=torch.float32)[:, None].to(
    "cuda" if torch.cuda.is_available() else "cpu")


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


# batches of more than 512 tiles of 16 x 4 nodes take the kernels of large
# lattices, each of their lattices alone the fused one: tiny lattices that wrap
# onto themselves, whole tiles, one column or row past them
@pytest.mark.parametrize("rounds", [1, 2])
@pytest.mark.parametrize("batch,nx,ny", [(600, 1, 1), (600, 3, 2), (600, 16, 4), (200, 17, 5),
                                         (300, 15, 8), (90, 50, 9), (5, 128, 128)])
def test_small_lattices_alone_equal_a_large_batch(rounds, batch, nx, ny):
    blob = torch.as_tensor(inputs.gnn_blob(9, rounds, s_delta=1e-2), device="cuda")
    g = torch.as_tensor(inputs.random_shifted_state((batch, ny, 9, nx), 4e-3, seed=nx),
                        device="cuda")
    tau = torch.linspace(0.6, 0.9, batch, device="cuda")
    post, z = gnn.gnn_forward(g, tau, blob, rounds, want_z=True)
    for b in (0, batch - 1):
        one, z1 = gnn.gnn_forward(g[b:b + 1].contiguous(), tau[b:b + 1], blob, rounds, want_z=True)
        assert torch.equal(one[0], post[b]) and torch.equal(z1[0], z[b]), b
        # the same collision after streaming, with the gate: kept and recorded,
        # or redone with plain BGK where it leaves a negative population
        src, dst = g[b].contiguous(), torch.empty_like(g[b])
        mass = nx * ny + float(g[b].double().sum())
        fb = gnn.Fallback(mass, 1.0)
        t = float(tau[b])
        gnn.lbm_step_gnn(src, dst, t, blob, rounds, fb)
        ref, _ = gnn.gnn_forward(lbm.lbm_stream(src)[None], tau[b:b + 1], blob, rounds)
        kept = bool((ref[0] + W >= 0).all())
        want = ref[0] if kept else lbm.lbm_step_bgk(src, torch.empty_like(src), t)
        assert torch.equal(dst, want)
        assert fb.flags.item() == (0 if kept else 1) and fb.n_fallback.item() == (0 if kept else 1)
        assert abs(fb.mass.item() - nx * ny - dst.double().sum().item()) <= 1e-12 * nx * ny
        # and forced to fall back: the plain step, counted
        fb = gnn.Fallback(mass, -1.0)
        gnn.lbm_step_gnn(src, dst, t, blob, rounds, fb)
        assert torch.equal(dst, lbm.lbm_step_bgk(src, torch.empty_like(src), t))
        assert fb.flags.item() == (2 if kept else 3) and fb.n_fallback.item() == 1
