"""Bands of tiles that start a chunk further on each: every tile of a matrix is taken once, whatever its number of chunks.  Bars as everywhere:
errors and features 1e-5, clip indices the oracle's but for ties of 1e-9."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n_chunks,rows,unit_rows", [(6, 1100, 0), (7, 1100, 0), (8, 577, 0), (9, 1100, 0), (10, 1100, 0), (16, 1024, 0), (18, 640, 128), (22, 130, 0)])
def test_every_tile_once(windq, n_chunks, rows, unit_rows, dtype):
    G, K = 32, 5
    W = synth.weights_llm(rows, G * n_chunks, seed=rows + n_chunks, device=DEV, dtype=dtype)
    s = torch.exp(torch.randn(G * n_chunks, generator=torch.Generator().manual_seed(n_chunks)))
    s[::29] *= 20.0
    cg = synth.clip_grid(K)
    feat, err, clip, ref = (t.cpu().numpy() for t in windq.windq_features_fit_score(W, s.to(DEV), G, unit_rows, cg))
    Wn = W.float().cpu().numpy()
    o_err, o_clip, o_ref, table = O.fit_score_all_bits(Wn, s.numpy(), G, unit_rows, cg.numpy())
    assert (np.abs(err.astype(np.float64) - o_err) <= 1e-5 * o_err).all()
    assert (np.abs(ref.astype(np.float64) - o_ref) <= 1e-5 * o_ref).all()
    for u, b in zip(*np.nonzero(clip != o_clip)):
        assert table[u, b, clip[u, b]] <= table[u, b].min() * (1 + 1e-9)
    assert torch.equal(torch.from_numpy(feat), windq.windq_unit_features(W, s.to(DEV), G, unit_rows).cpu())
