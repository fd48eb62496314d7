"""Every tile of a matrix is taken once, whatever its number of chunks: in the matrix's order, and, where heavy columns may go first, in bands that start a chunk further
on each.  Bars as everywhere: errors and features 1e-5, clip indices the oracle's but for ties of 1e-9."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth
from test_gpu_heavy_first import both, same, scales

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


@pytest.mark.parametrize("steep", [True, False])
@pytest.mark.parametrize("n_chunks,rows,unit_rows", [(6, 64 * 342, 0), (8, 16384, 1024), (9, 64 * 228, 0), (10, 64 * 205 - 3, 0), (14, 64 * 147, 64 * 21), (22, 64 * 94, 0)])
def test_every_tile_once_turned(windq, n_chunks, rows, unit_rows, steep):
    """Matrices of 2048 tiles and a few, whose halves are below that and not turned."""
    G, K = 64, 40
    C = G * n_chunks
    W = synth.weights_llm(rows, C, seed=rows + n_chunks, device=DEV)
    s = scales(C, n_chunks) if steep else torch.ones(C, device=DEV)
    whole, parts, _ = both(windq, W, s, G, K, unit_rows, fused=True)
    same(whole, parts, W, s, G, synth.clip_grid(K), unit_rows)
