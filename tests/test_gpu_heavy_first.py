"""fit+score of large matrices, heavy columns first: a unit's candidates are scored on the columns that carry most of its error, and
only those that may still win on the others.  Whatever the data, the results are those of scoring everything: here
of the same columns in matrices too small for that route.  Bar: 1e-5 as everywhere (both routes are good to about 1e-6); where two clip indices
differ, the oracle's errors at both have to be that close."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth, workload

pytestmark = pytest.mark.gpu
DEV = "cuda"
TILES = 2048        # fewer 64-row tiles: scored in one piece


def scales(C, seed):
    g = torch.Generator().manual_seed(seed)
    s = torch.exp(torch.randn(C, generator=g))
    s[torch.randperm(C, generator=g)[:C // 64]] *= 30.0
    return s.to(DEV)


def both(windq, W, s, G, K, unit_rows=0, cg=None, fused=False):
    """(outputs by the matrix's own route, outputs of its parts, the units scored a second time)."""
    R, C = W.shape
    cg = synth.clip_grid(K) if cg is None else cg
    call = windq.windq_features_fit_score if fused else windq.windq_fit_score_all_bits
    U, R_u = windq.n_units(R, C, G, unit_rows)
    per_chunk = R // R_u * ((R_u + 63) // 64)
    chunks = C // G
    assert per_chunk * chunks >= TILES and K * G >= 2560
    size = windq.workspace_bytes(windq.CALL_FEATURES_FIT_SCORE if fused else windq.CALL_FIT_SCORE, windq.WINDQ_BF16, R, C, G, unit_rows, K)
    at = windq.workspace_bytes(windq.CALL_UNIT_FEATURES, windq.WINDQ_BF16, R, C, G, unit_rows, 1) if fused else 0
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)
    whole = call(W, s, G, unit_rows, cg, ws=ws)
    torch.cuda.synchronize()
    lay = workload.FitWorkspace(R, C, G, unit_rows, K, at)
    n = int(ws[lay.redo_count:lay.redo_count + 4].view(torch.int32).item())
    listed = sorted(ws[lay.redo_list:lay.redo_list + 4 * n].view(torch.int32).tolist())
    assert len(set(listed)) == n and (fused or n == windq.windq_fit_score_rescored_units(ws, W, G, unit_rows, K))
    at = [0] + [chunks * (i + 1) // 2 for i in range(2)]
    parts = []
    for a, b in zip(at, at[1:]):
        assert per_chunk * (b - a) < TILES
        parts.append(call(W[:, a * G:b * G], s[a * G:b * G].contiguous(), G, unit_rows, cg))
    rb = R // R_u
    join = [torch.cat([p[i].reshape(rb, b - a, *p[i].shape[1:]) for p, (a, b) in zip(parts, zip(at, at[1:]))], 1).reshape(U, *whole[i].shape[1:])
            for i in range(len(whole))]
    return whole, join, listed


def oracle_of_unit(W, s, G, unit_rows, cg, u):
    """(least errors [6], clip indices [4], errors [4][K]) of one unit."""
    R_u, chunks = unit_rows or W.shape[0], W.shape[1] // G
    rb, j = u // chunks, u % chunks
    sub = W[rb * R_u:(rb + 1) * R_u, j * G:(j + 1) * G].float().cpu().numpy()
    err, clip, _, table = O.fit_score_all_bits(sub, s[j * G:(j + 1) * G].cpu().numpy(), G, 0, cg.numpy())
    return err[0], clip[0], table[0]


def same(whole, parts, W, s, G, cg, unit_rows=0):
    a, b = whole[-3].double().cpu().numpy(), parts[-3].double().cpu().numpy()
    assert np.array_equal(np.isnan(a), np.isnan(b))
    with np.errstate(invalid="ignore"):
        bad = ~(np.isnan(a) | (a == b) | (np.abs(a - b) <= 1e-5 * np.abs(b)))
    assert not bad.any(), (np.argwhere(bad)[:4], a[bad][:4], b[bad][:4])
    ci, cj = whole[-2].cpu().numpy(), parts[-2].cpu().numpy()
    assert (ci != cj).mean() <= 0.01
    for u in sorted(set(np.nonzero(ci != cj)[0])):          # (1e-6 of its error for the candidate of either route)
        table = oracle_of_unit(W, s, G, unit_rows, cg, u)[2]
        for bits in np.nonzero(ci[u] != cj[u])[0]:
            here, there = table[bits, ci[u, bits]], table[bits, cj[u, bits]]
            assert abs(here - there) <= 2e-6 * there
    assert torch.allclose(whole[-1], parts[-1], rtol=1e-6, equal_nan=True)
    if len(whole) == 4:
        assert torch.equal(whole[0], parts[0])                # the features are not touched


@pytest.mark.parametrize("R,C,G,K,unit_rows", [
    (1024, 128 * 129, 128, 20, 0), (1031, 64 * 124, 64, 40, 0), (1150, 192 * 118, 192, 17, 0), (1100, 256 * 116, 256, 64, 0),
    (2048, 128 * 66, 128, 41, 1024), (4200, 128 * 32, 128, 20, 0), (1024, 256 * 130, 256, 16, 0)])
def test_same_as_small_matrices(windq, R, C, G, K, unit_rows):
    W, s = synth.weights_llm(R, C, seed=R + K, device=DEV), scales(C, K)
    whole, parts, _ = both(windq, W, s, G, K, unit_rows, fused=K % 2 == 0)
    same(whole, parts, W, s, G, synth.clip_grid(K), unit_rows)


@pytest.mark.parametrize("fused", [False, True])
def test_window_of_a_wider_matrix(windq, fused):
    """Rows further apart than the columns, at an odd place of 16 bytes; what lies beside the window must not matter."""
    R, C, G, K = 1037, 128 * 126, 128, 20
    wide = torch.full((R, C + 136), float("nan"), dtype=torch.bfloat16, device=DEV)
    W = wide[:, 8:8 + C]
    W.copy_(synth.weights_llm(R, C, seed=21, device=DEV))
    s = scales(C, 22)
    whole, parts, _ = both(windq, W, s, G, K, fused=fused)
    same(whole, parts, W, s, G, synth.clip_grid(K))
    dense, _, _ = both(windq, W.contiguous(), s, G, K, fused=fused)
    assert all(torch.equal(x, y) for x, y in zip(whole, dense))


def test_grids_that_are_not_the_usual(windq):
    W = synth.weights_llm(1024, 128 * 130, seed=3, device=DEV)
    s = scales(W.shape[1], 4)
    for ratios in (np.linspace(0.05, 0.9, 24), np.linspace(0.9, 1.0, 20), np.linspace(0.97, 0.99, 33)):
        cg = torch.tensor(ratios, dtype=torch.float32)
        whole, parts, _ = both(windq, W, s, 128, len(cg), cg=cg)
        same(whole, parts, W, s, 128, cg)


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
    same(whole, parts, W, s, G, synth.clip_grid(20))


def test_weights_of_one_sign_and_degenerate_units(windq):
    G, C = 128, 128 * 130
    W = synth.weights_llm(1090, C, seed=7, device=DEV)
    W[:, 3 * G:9 * G] = W[:, 3 * G:9 * G].abs() + 0.001
    W[:, 12 * G:13 * G] = 0.0
    W[:, 14 * G:15 * G] = 0.25
    W[100:200, 16 * G:17 * G] = 0.0
    W[1024:, 18 * G:19 * G] *= 1000.0
    s = scales(C, 8)
    whole, parts, _ = both(windq, W, s, G, 20)
    same(whole, parts, W, s, G, synth.clip_grid(20))


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_weights_that_are_not_finite(windq, value):
    G, C = 128, 128 * 130
    W = synth.weights_llm(1024, C, seed=9, device=DEV)
    s = scales(C, 10)
    for j in range(0, 20):          # in a heavy column of some units and a light one of others
        order = torch.argsort(s[j * G:(j + 1) * G].abs(), descending=True)
        W[(37 * j) % 1024, j * G + int(order[0 if j % 2 else G - 1])] = value
    whole, parts, _ = both(windq, W, s, G, 20)
    same(whole, parts, W, s, G, synth.clip_grid(20))


def loud_light_columns(R, C, G, s, seed, every, first):
    """Weights whose light columns are 40 times larger in every third chunk, but not in the tiles first, first + every, ... by which the plan judges them."""
    W = synth.weights_llm(R, C, seed=seed, device=DEV).float()
    loud = torch.full(((R + 63) // 64,), 40.0, device=DEV)
    loud[:first] = 1.0
    loud[first::every] = 1.0
    loud = loud.repeat_interleave(64)[:R]
    for j in range(0, C // G, 3):
        light = torch.argsort(s[j * G:(j + 1) * G].abs(), descending=True)[G // 2:]
        W[:, j * G + light] *= loud[:, None]
    return W.bfloat16()


@pytest.mark.parametrize("fused", [False, True])
def test_units_whose_light_columns_the_sampled_tiles_do_not_show(windq, fused):
    """The plan looks at the light columns in the even tiles from the third on; here the others' light columns are 40 times
    larger, so that many candidates that were left out have to be scored after all."""
    G, C, R, cg = 128, 128 * 130, 1024, synth.clip_grid(20)
    s = scales(C, 12)
    W = loud_light_columns(R, C, G, s, 11, 2, 1)
    whole, parts, listed = both(windq, W, s, G, 20, fused=fused)
    assert len(listed) >= 10
    same(whole, parts, W, s, G, cg)
    again, _, _ = both(windq, W, s, G, 20, fused=fused)
    assert all(torch.equal(x, y) for x, y in zip(whole, again))
    g_err, g_clip = whole[-3].double().cpu().numpy(), whole[-2].cpu().numpy()
    for u in listed[:6]:
        o_err, o_clip, table = oracle_of_unit(W, s, G, 0, cg, u)
        assert (np.abs(g_err[u] - o_err) <= 1e-5 * o_err).all()
        for b in np.nonzero(g_clip[u] != o_clip)[0]:
            assert table[b, g_clip[u, b]] <= table[b].min() * (1 + 1e-9)


def test_listed_units_of_more_tiles_than_are_added_up_at_once(windq):
    """The second pass adds a unit's tiles up 1536 at a time; taller units take another way."""
    G, K, R, C = 64, 40, 64 * 1537 + 5, 128
    s = scales(C, 16)
    W = loud_light_columns(R, C, G, s, 17, 8, 2)
    whole, parts, listed = both(windq, W, s, G, K)
    assert 0 in listed
    same(whole, parts, W, s, G, synth.clip_grid(K))


def test_batch_of_steep_and_flat_matrices(windq):
    """Matrices that are scored heavy columns first, that could be but have flat scales, and that are too small, in one call: the bits of the single calls."""
    G, K = 128, 20
    cols = [128 * 129, 128 * 130, 128 * 4]
    Ws = [synth.weights_llm(1024, c, seed=c, device=DEV) for c in cols]
    ss = [scales(cols[0], 1), torch.ones(cols[1], device=DEV), scales(cols[2], 2)]
    cg = synth.clip_grid(K)
    batch = windq.windq_features_fit_score_batch(Ws, ss, G, 0, cg)
    for i in (0, 1, 2):
        assert all(torch.equal(a, b) for a, b in zip(batch[i], windq.windq_features_fit_score(Ws[i], ss[i], G, 0, cg)))


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
