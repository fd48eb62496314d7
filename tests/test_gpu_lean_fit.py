"""fit+score of small matrices by themselves: a launch that leaves no candidate out, prepares nothing and scores nothing again.  Bars as
everywhere: errors 1e-5, clip indices the oracle's but for ties of 1e-9; and the bits of the same matrix in a launch that does all that."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth, workload

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("R,C,G,unit_rows,K", [
    (1, 8, 8, 0, 1), (63, 64, 32, 0, 20), (64, 128, 64, 0, 16), (65, 256, 128, 0, 64), (640, 512, 64, 64, 20), (2000, 96, 96, 0, 5),
    (1024, 512, 128, 0, 32), (4096, 64, 64, 0, 20), (130, 512, 512, 0, 20)])
def test_alone_and_beside_a_large_matrix(windq, R, C, G, unit_rows, K, dtype):
    W = synth.weights_llm(R, C, seed=R + K, device=DEV, dtype=dtype)
    g = torch.Generator().manual_seed(R)
    s = torch.exp(torch.randn(C, generator=g))
    s[::37] *= 30.0
    cg = synth.clip_grid(K)
    dt = windq.WINDQ_F32 if dtype == torch.float32 else windq.WINDQ_BF16
    ws = torch.full((windq.workspace_bytes(windq.CALL_FIT_SCORE, dt, R, C, G, unit_rows, K),), 255, dtype=torch.uint8, device=DEV)
    alone = windq.windq_fit_score_all_bits(W, s.to(DEV), G, unit_rows, cg, ws=ws)
    torch.cuda.synchronize()
    assert windq.windq_fit_score_rescored_units(ws, W, G, unit_rows, K) == 0          # (the workspace was not clear)
    rows = unit_rows or 64
    big = synth.weights_llm(rows * (3 if G < 64 else 1) * ((260 * 64 + rows - 1) // rows), G * (2 if G < 64 else 1), seed=2, device=DEV, dtype=dtype)
    sb = torch.exp(torch.randn(big.shape[1], generator=g)).to(DEV)
    both = windq.windq_fit_score_all_bits_batch([W, big], [s.to(DEV), sb], G, unit_rows, cg)
    assert all(torch.equal(a, b) for a, b in zip(alone, both[0]))
    feat = windq.windq_features_fit_score(W, s.to(DEV), G, unit_rows, cg)
    assert all(torch.equal(a, b) for a, b in zip(alone, feat[1:]))
    assert torch.equal(feat[0], windq.windq_unit_features(W, s.to(DEV), G, unit_rows))
    o_err, o_clip, o_ref, table = O.fit_score_all_bits(W.float().cpu().numpy(), s.numpy(), G, unit_rows, cg.numpy())
    g_err, g_clip = alone[0].double().cpu().numpy(), alone[1].cpu().numpy()
    bar = 1e-5 if min(R, unit_rows or R) >= 64 else 1e-4            # few rows: one weight may carry the error (include/windq.h)
    assert (np.abs(g_err - o_err) <= bar * o_err + 1e-30).all()
    for u, b in zip(*np.nonzero(g_clip != o_clip)):
        assert table[u, b, g_clip[u, b]] <= table[u, b].min() * (1 + 1e-9)


@pytest.mark.parametrize("R,C,G,K,lean", [(4096, 256, 64, 20, True), (4096, 512, 128, 20, False), (2100, 256, 256, 33, True), (2100, 512, 256, 33, False)])
def test_where_the_exact_route_ends(windq, R, C, G, K, lean):
    """Matrices in quarters whose work is that of a lean launch at most take every column on the exact 8-bit route, larger ones the short route for
    most of them; alone and in a batch the bits are the same on both sides, and within the bars."""
    W = synth.weights_llm(R, C, seed=R + K, device=DEV)
    s = torch.exp(torch.randn(C, generator=torch.Generator().manual_seed(R)))
    big, sb = synth.weights_llm(R, 4 * C, seed=2, device=DEV), torch.exp(torch.randn(4 * C, generator=torch.Generator().manual_seed(3))).to(DEV)
    cg = synth.clip_grid(K)
    alone = windq.windq_fit_score_all_bits(W, s.to(DEV), G, 0, cg)
    ws = [torch.empty(windq.workspace_bytes(windq.CALL_FIT_SCORE, windq.WINDQ_BF16, R, c, G, 0, K), dtype=torch.uint8, device=DEV) for c in (C, 4 * C)]
    both = windq.windq_fit_score_all_bits_batch([W, big], [s.to(DEV), sb], G, 0, cg, wss=ws)
    assert all(torch.equal(a, b) for a, b in zip(alone, both[0]))
    listed = workload.FitWorkspace(R, C, G, 0, K).listed_columns(ws[0])
    assert ((listed == -1) if lean else (listed >= 0)).all()
    o_err, o_clip, o_ref, table = O.fit_score_all_bits(W.float().cpu().numpy(), s.numpy(), G, 0, cg.numpy())
    g_err, g_clip = alone[0].double().cpu().numpy(), alone[1].cpu().numpy()
    assert (np.abs(g_err - o_err) <= 1e-5 * o_err).all()
    for u, b in zip(*np.nonzero(g_clip != o_clip)):
        assert table[u, b, g_clip[u, b]] <= table[u, b].min() * (1 + 1e-9)


def test_lean_call_with_features_makes_no_records(windq):
    """Nothing of a lean launch reads the chunks' records: the kernel that clears the features' counters leaves them as they were."""
    R, C, G, K = 512, 512, 64, 20
    W = synth.weights_llm(R, C, seed=1, device=DEV)
    s = torch.ones(C, device=DEV)
    at = windq.workspace_bytes(windq.CALL_UNIT_FEATURES, windq.WINDQ_BF16, R, C, G, 0, 1)
    ws = torch.full((windq.workspace_bytes(windq.CALL_FEATURES_FIT_SCORE, windq.WINDQ_BF16, R, C, G, 0, K),), 7, dtype=torch.uint8, device=DEV)
    got = windq.windq_features_fit_score(W, s, G, 0, synth.clip_grid(K), ws=ws)
    assert (workload.FitWorkspace(R, C, G, 0, K, at).listed_columns(ws) == 0x07070707).all()
    assert all(torch.equal(a, b) for a, b in zip(got, windq.windq_features_fit_score(W, s, G, 0, synth.clip_grid(K))))


@pytest.mark.parametrize("K", [20, 64])
def test_counted_work_of_a_lean_call(windq, K):
    """The benchmark counts the work of such a call as all of the definition's, whatever the workspace held before."""
    import bench
    R, C, G = 512, 512, 64
    mat = workload.Mat()
    mat.spec, mat.W, (mat.U, mat.R_u) = synth.MatrixSpec("linear", R, C, "h"), synth.weights_llm(R, C, seed=1, device=DEV), windq.n_units(R, C, G, 0)
    ws = torch.full((windq.workspace_bytes(windq.CALL_FEATURES_FIT_SCORE, windq.WINDQ_BF16, R, C, G, 0, K),), 0xEE, dtype=torch.uint8, device=DEV)
    windq.windq_features_fit_score(mat.W, torch.ones(C, device=DEV), G, 0, synth.clip_grid(K), ws=ws)
    flops, share = bench.executed_work(windq, torch, [mat], [ws], G, 0, K, True)
    assert share == 1.0 and abs(flops - bench.fit_score_flops_per_weight(K)) < 1e-9
