"""Heavy columns first only where the scales are steep in three quarters of a matrix's chunks (sixteen of them are looked at): the chunks' records
say which route was taken, and the results are those of the same columns in matrices too small for it."""
import pytest
import torch

from paper_2605_26660_amd import synth, workload
from test_gpu_heavy_first import both, same

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("R,n_chunks,G,K,steep,taken", [
    (8192, 16, 128, 20, 12, True), (8192, 16, 128, 20, 11, False), (4200, 32, 256, 16, 32, True), (16384, 8, 64, 40, 6, True),
    (16384, 8, 64, 40, 5, False), (16384, 9, 192, 17, 0, False)])
def test_route_by_steep_chunks(windq, R, n_chunks, G, K, steep, taken):
    W = synth.weights_llm(R, G * n_chunks, seed=R + K, device=DEV)
    s = torch.ones(n_chunks, G)
    g = torch.Generator().manual_seed(K)
    s[torch.randperm(n_chunks, generator=g)[:steep]] = torch.exp(1.5 * torch.randn(G, generator=g))
    s = s.reshape(-1).to(DEV)
    whole, parts, _ = both(windq, W, s, G, K)
    same(whole, parts, W, s, G, synth.clip_grid(K))
    cg = synth.clip_grid(K)
    ws = torch.empty(windq.workspace_bytes(windq.CALL_FIT_SCORE, windq.WINDQ_BF16, R, G * n_chunks, G, 0, K), dtype=torch.uint8, device=DEV)
    windq.windq_fit_score_all_bits(W, s, G, 0, cg, ws=ws)
    # a record per chunk, its count of columns below -1 where heavy columns went first
    records = workload.FitWorkspace(R, G * n_chunks, G, 0, K).listed_columns(ws)
    assert int((records < -1).sum()) == (steep if taken else 0)
