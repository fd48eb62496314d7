"""fit+score of large matrices, heavy columns first: a unit's candidates are scored on the columns that carry most of its error, and
only those that may still win on the others.  Whatever the data, the results are those of scoring everything: here
of the same columns in matrices too small for that route.  Bar: 1e-5 as everywhere (both routes are good to about 1e-6); a clip
index may differ where the errors are that close."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
TILES = 2048        # fewer 64-row tiles: scored in one piece


def scales(C, seed):
    g = torch.Generator().manual_seed(seed)
    s = torch.exp(torch.randn(C, generator=g))
    s[torch.randperm(C, generator=g)[:C // 64]] *= 30.0
    return s.to(DEV)


def both(windq, W, s, G, K, unit_rows=0, cg=None, fused=False):
    """(outputs, units scored a second time) by the matrix's own route, and the outputs of its parts."""
    R, C = W.shape
    cg = synth.clip_grid(K) if cg is None else cg
    call = windq.windq_features_fit_score if fused else windq.windq_fit_score_all_bits
    U, R_u = windq.n_units(R, C, G, unit_rows)
    per_chunk = R // R_u * ((R_u + 63) // 64)
    chunks = C // G
    assert per_chunk * chunks >= TILES and K * G >= 2560
    ws = torch.empty(windq.workspace_bytes(windq.CALL_FIT_SCORE, windq.WINDQ_BF16, R, C, G, unit_rows, K), dtype=torch.uint8, device=DEV)
    whole = call(W, s, G, unit_rows, cg) if fused else call(W, s, G, unit_rows, cg, ws=ws)
    torch.cuda.synchronize()
    listed = None if fused else windq.windq_fit_score_rescored_units(ws, W, G, unit_rows, K)
    at = [0] + [chunks * (i + 1) // 2 for i in range(2)]
    parts = []
    for a, b in zip(at, at[1:]):
        assert per_chunk * (b - a) < TILES
        parts.append(call(W[:, a * G:b * G], s[a * G:b * G].contiguous(), G, unit_rows, cg))
    rb = R // R_u
    join = [torch.cat([p[i].reshape(rb, b - a, *p[i].shape[1:]) for p, (a, b) in zip(parts, zip(at, at[1:]))], 1).reshape(U, *whole[i].shape[1:])
            for i in range(len(whole))]
    return whole, join, listed


def same(whole, parts):
    a, b = whole[-3].double().cpu().numpy(), parts[-3].double().cpu().numpy()
    assert np.array_equal(np.isnan(a), np.isnan(b))
    with np.errstate(invalid="ignore"):
        bad = ~(np.isnan(a) | (a == b) | (np.abs(a - b) <= 1e-5 * np.abs(b)))
    assert not bad.any(), (np.argwhere(bad)[:4], a[bad][:4], b[bad][:4])
    ci, cj = whole[-2].cpu().numpy(), parts[-2].cpu().numpy()
    with np.errstate(invalid="ignore"):
        tie = np.abs(a[:, :4] - b[:, :4]) <= 1e-6 * np.abs(b[:, :4])
    assert ((ci == cj) | tie).all(), np.argwhere(~((ci == cj) | tie))[:4]
    assert (ci != cj).mean() <= 0.01
    assert torch.allclose(whole[-1], parts[-1], rtol=1e-6, equal_nan=True)
    if len(whole) == 4:
        assert torch.equal(whole[0], parts[0])                # the features are not touched


@pytest.mark.parametrize("R,C,G,K,unit_rows", [
    (1024, 128 * 129, 128, 20, 0), (1031, 64 * 124, 64, 40, 0), (1150, 192 * 118, 192, 17, 0), (1100, 256 * 116, 256, 64, 0),
    (2048, 128 * 66, 128, 41, 1024), (4200, 128 * 32, 128, 20, 0), (1024, 256 * 130, 256, 16, 0)])
def test_same_as_small_matrices(windq, R, C, G, K, unit_rows):
    W = synth.weights_llm(R, C, seed=R + K, device=DEV)
    whole, parts, _ = both(windq, W, scales(C, K), G, K, unit_rows, fused=K % 2 == 0)
    same(whole, parts)


def test_grids_that_are_not_the_usual(windq):
    W = synth.weights_llm(1024, 128 * 130, seed=3, device=DEV)
    s = scales(W.shape[1], 4)
    for ratios in (np.linspace(0.05, 0.9, 24), np.linspace(0.9, 1.0, 20), np.linspace(0.97, 0.99, 33)):
        cg = torch.tensor(ratios, dtype=torch.float32)
        whole, parts, _ = both(windq, W, s, 128, len(cg), cg=cg)
        same(whole, parts)


def test_chunks_of_both_kinds(windq):
    """Equal scales (no heavy columns), zero scales, scales that are not finite, beside ordinary ones."""
    G, C = 128, 128 * 130
    W = synth.weights_llm(1024, C, seed=5, device=DEV)
    s = scales(C, 6)
    s[:20 * G] = 1.0
    s[30 * G:31 * G] = 0.0
    s[40 * G + 5] = float("nan")
    s[41 * G + 5] = float("inf")
    whole, parts, _ = both(windq, W, s, G, 20)
    same(whole, parts)


def test_weights_of_one_sign_and_degenerate_units(windq):
    G, C = 128, 128 * 130
    W = synth.weights_llm(1090, C, seed=7, device=DEV)
    W[:, 3 * G:9 * G] = W[:, 3 * G:9 * G].abs() + 0.001
    W[:, 12 * G:13 * G] = 0.0
    W[:, 14 * G:15 * G] = 0.25
    W[100:200, 16 * G:17 * G] = 0.0
    W[1024:, 18 * G:19 * G] *= 1000.0
    whole, parts, _ = both(windq, W, scales(C, 8), G, 20)
    same(whole, parts)


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_weights_that_are_not_finite(windq, value):
    G, C = 128, 128 * 130
    W = synth.weights_llm(1024, C, seed=9, device=DEV)
    s = scales(C, 10)
    for j in range(0, 20):          # in a heavy column of some units and a light one of others
        order = torch.argsort(s[j * G:(j + 1) * G].abs(), descending=True)
        W[(37 * j) % 1024, j * G + int(order[0 if j % 2 else G - 1])] = value
    whole, parts, _ = both(windq, W, s, G, 20)
    same(whole, parts)


def test_units_whose_light_columns_the_sampled_tiles_do_not_show(windq):
    """The plan looks at the light columns in the even tiles from the third on; here the others' light columns are 40 times
    larger, so that many candidates that were left out have to be scored after all."""
    G, C, R = 128, 128 * 130, 1024
    W = synth.weights_llm(R, C, seed=11, device=DEV).float()
    s = scales(C, 12)
    loud = torch.ones(R, device=DEV)
    for t in range(R // 64):
        if t % 2 == 1:
            loud[64 * t:64 * t + 64] = 40.0
    for j in range(0, C // G, 3):
        light = torch.argsort(s[j * G:(j + 1) * G].abs(), descending=True)[G // 2:]
        W[:, j * G + light] *= loud[:, None]
    whole, parts, listed = both(windq, W.bfloat16(), s, G, 20)
    assert listed >= 10
    same(whole, parts)
    again, _, _ = both(windq, W.bfloat16(), s, G, 20)
    assert all(torch.equal(x, y) for x, y in zip(whole, again))


def test_against_the_oracle_and_in_a_batch(windq):
    G, K, C = 128, 20, 128 * 130
    W = synth.weights_llm(1024, C, seed=13, device=DEV)
    s = scales(C, 14)
    small = synth.weights_llm(300, 1024, seed=15, device=DEV)
    err, clip, ref = windq.windq_fit_score_all_bits(W, s, G, 0, synth.clip_grid(K))
    batch = windq.windq_fit_score_all_bits_batch([small, W, small], [s[:1024].contiguous(), s, s[1024:2048].contiguous()], G, 0, synth.clip_grid(K))
    assert all(torch.equal(a, b) for a, b in zip(batch[1], (err, clip, ref)))
    units = [0, 7, 64, 129]
    cols = torch.cat([torch.arange(u * G, (u + 1) * G) for u in units]).to(DEV)
    o_err, o_clip, o_ref, table = O.fit_score_all_bits(W[:, cols].float().cpu().numpy(), s[cols].cpu().numpy(), G, 0, synth.clip_grid(K).numpy())
    g_err, g_clip = err[units].double().cpu().numpy(), clip[units].cpu().numpy()
    assert (np.abs(g_err - o_err) <= 1e-5 * o_err).all()
    for u, b in zip(*np.nonzero(g_clip != o_clip)):
        assert table[u, b, g_clip[u, b]] <= table[u, b].min() * (1 + 1e-9)
