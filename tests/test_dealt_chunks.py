"""Which wave takes a chunk of 64 nodes: with few chunks per wave they are dealt
out in turn and nobody draws from the counters (their draws, one after the other,
took longer than the chunks); with more, waves draw them.  Same values either
way."""
import numpy as np
import pytest
import torch

from paper_2504_14494_amd import _lib, gnn, inputs, lbm

pytestmark = pytest.mark.gpu

CTRL_BYTES = 4 * 512     # the control words close the scratch
CHUNK_QUEUE, PARTS, STRIDE = 32, 8, 32


def _step(src, blob):
    ws = lbm.Workspace()
    out = gnn.lbm_step_simple(src, torch.full_like(src, float("nan")), 0.62, blob, ws=ws)
    n = _lib.load().lbm_workspace_bytes(_lib.LBM_WS_SIMPLE, 1, src.shape[2], src.shape[0], 0)
    words = ws.buf[n - CTRL_BYTES:n].view(torch.int32).cpu().numpy()
    return out, words[CHUNK_QUEUE:CHUNK_QUEUE + PARTS * STRIDE:STRIDE]


@pytest.mark.parametrize("nx,ny", [(2, 4000), (1, 8000), (130, 433), (65, 1777), (512, 512),
                                   (64, 15001)])
def test_few_chunks_per_wave_are_dealt(nx, ny):
    blob = torch.as_tensor(inputs.gnn_blob(3, 0, s_delta=1e-4), device="cuda")
    g = torch.as_tensor(inputs.random_shifted_state((ny, 9, nx), 3e-3, nx + ny).astype(np.float32),
                        device="cuda")
    out, draws = _step(g, blob)
    assert not draws.any(), draws
    # the same rows as one of several copies, enough for the waves to draw
    copies = -(-8 * 4096 // (ny * (-(-nx // 64))))
    many, draws = _step(g.repeat(copies, 1, 1), blob)
    assert draws.all(), draws
    assert torch.equal(many, out.repeat(copies, 1, 1))
