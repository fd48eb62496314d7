"""fit+score where a tile's sweeps go to several workgroups, or all wavefronts share a sweep by columns: at the sizes where
the cut changes, against the oracle (errors 1e-5, clip indices but for ties of 1e-9), and a batch of both kinds against
the single calls, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def inputs(R, C, seed, dtype):
    W = synth.weights_llm(R, C, seed=seed, device=DEV, dtype=dtype)
    s = synth.activations_llm(64, C, seed=seed, device=DEV).float().abs().mean(0)
    return W, s


def compare(W, s, G, unit_rows, cg, out, mask=None):
    keep = None if mask is None else np.unpackbits(mask.cpu().numpy(), axis=1, bitorder="little")[:, :W.shape[1]] == 0
    o_err, o_clip, o_ref, table = O.fit_score_all_bits(W.float().cpu().numpy(), s.cpu().numpy(), G, unit_rows, cg.numpy(), keep=keep)
    g_err, g_clip = out[0].cpu().numpy().astype(np.float64), out[1].cpu().numpy()
    for u, b in zip(*np.nonzero(g_clip != o_clip)):
        assert table[u, b, g_clip[u, b]] <= table[u, b].min() * (1 + 1e-9), (u, b, g_clip[u, b], o_clip[u, b])
    assert (np.abs(g_err - o_err) <= 1e-5 * o_err).all(), np.max(np.abs(g_err - o_err) / (o_err + 1e-300))
    assert (np.abs(out[2].cpu().numpy() - o_ref) <= 1e-5 * o_ref).all()


@pytest.mark.parametrize("tiles", [1, 256, 257])
@pytest.mark.parametrize("G,K", [(8, 5), (40, 10), (64, 5), (64, 6), (120, 10), (128, 10), (184, 15), (192, 15), (64, 21)])
def test_at_the_edges_of_the_cut(windq, tiles, G, K):
    """Chunks on both sides of 64 columns per sweep, widths whose quarters are uneven or empty, 256 and 257 tiles; the last
    tile is not full."""
    rows = 64 * tiles - 5
    W, s = inputs(rows, G, tiles + G + K, torch.float32 if K % 2 else torch.bfloat16)
    cg = synth.clip_grid(K)
    compare(W, s, G, 0, cg, windq.windq_fit_score_all_bits(W, s, G, 0, cg))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("G,unit_rows,K", [(128, 0, 20), (64, 0, 40), (64, 64, 20), (256, 0, 64), (96, 0, 1)])
def test_small_matrices_of_every_route(windq, G, unit_rows, K, dtype):
    """With and without a mask, whole columns (the short route) and units of one tile (every column exact)."""
    W, s = inputs(448, 4 * G, G + K, dtype)
    cg = synth.clip_grid(K)
    compare(W, s, G, unit_rows, cg, windq.windq_fit_score_all_bits(W, s, G, unit_rows, cg))
    mask = windq.windq_salient_select(W, s, G, unit_rows, 30000)
    compare(W, s, G, unit_rows, cg, windq.windq_fit_score_all_bits(W, s, G, unit_rows, cg, mask=mask), mask=mask)


@pytest.mark.parametrize("K", [5, 10, 20, 40])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_a_batch_of_small_and_large_equals_the_single_calls(windq, dtype, K):
    shapes = [(130, 256), (64 * 140, 256), (64, 128), (3000, 768)]
    mats = [inputs(r, c, 10 + i, dtype) for i, (r, c) in enumerate(shapes)]
    cg = synth.clip_grid(K)
    batch = windq.windq_features_fit_score_batch([m[0] for m in mats], [m[1] for m in mats], 128, 0, cg)
    for (W, s), got in zip(mats, batch):
        feat = windq.windq_unit_features(W, s, 128, 0)
        want = (feat, *windq.windq_fit_score_all_bits(W, s, 128, 0, cg))
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want))


@pytest.mark.parametrize("G,K", [(64, 20), (64, 40), (64, 64), (96, 33), (128, 10), (64, 15), (32, 40), (40, 64), (256, 20)])
@pytest.mark.parametrize("tiles", [384, 385, 640, 641, 1024, 1025])
def test_the_size_of_the_launch_changes_no_bits(windq, tiles, G, K):
    """Launches on both sides of where a tile's sweeps go to fewer workgroups: matrices cut in quarters (of 256 tiles, or 64 where the
    chunk is narrow) and in one piece side by side, each as in its own call."""
    dtype = torch.float32 if K % 2 else torch.bfloat16
    per = 64 if G < 64 else 128
    rows = [64 * per - 5, 64 * per] + ([64 * (tiles - 2 * per)] if tiles <= 640 else [64 * 257, 64 * (tiles - 2 * per - 257)])
    mats = [inputs(r, G, 20 + i, dtype) for i, r in enumerate(rows)]
    cg = synth.clip_grid(K)
    batch = windq.windq_fit_score_all_bits_batch([m[0] for m in mats], [m[1] for m in mats], G, 0, cg)
    fused = windq.windq_features_fit_score_batch([m[0] for m in mats], [m[1] for m in mats], G, 0, cg)
    for i, ((W, s), got, both) in enumerate(zip(mats, batch, fused)):
        want = windq.windq_fit_score_all_bits(W, s, G, 0, cg)
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want))
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(both[1:], want))
        assert torch.equal(both[0], windq.windq_unit_features(W, s, G, 0))
        if i == 0 and tiles == 385:
            compare(W, s, G, 0, cg, got)


@pytest.mark.parametrize("G,K", [(64, 40), (128, 20), (32, 64)])
def test_the_size_of_a_masked_launch_changes_no_bits(windq, G, K):
    mats = [inputs(64 * 128 - 5, G, 30 + i, torch.bfloat16) for i in range(4)]
    masks = [windq.windq_salient_select(W, s, G, 0, 30000) for W, s in mats]
    cg = synth.clip_grid(K)
    batch = windq.windq_fit_score_all_bits_batch([m[0] for m in mats], [m[1] for m in mats], G, 0, cg, masks=masks)
    for (W, s), mask, got in zip(mats, masks, batch):
        want = windq.windq_fit_score_all_bits(W, s, G, 0, cg, mask=mask)
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want))
    compare(*mats[0], G, 0, cg, batch[0], mask=masks[0])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("tiles", [1, 15, 16, 17, 31, 33, 64, 80, 1001])
def test_a_units_tiles_are_added_in_one_order(windq, tiles, dtype):
    """Sixteen phases, side by side in four wavefronts (with the features) or one in each of sixteen (alone): the same bits, rounds
    that are full or not; the sums against the oracle."""
    W, s = inputs(64 * tiles - 1, 64, tiles, dtype)
    for K in (1, 13):
        cg = synth.clip_grid(K)
        alone = windq.windq_fit_score_all_bits(W, s, 64, 0, cg)
        fused = windq.windq_features_fit_score(W, s, 64, 0, cg)
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(fused[1:], alone))
        compare(W, s, 64, 0, cg, alone)


@pytest.mark.parametrize("G,K", [(64, 20), (64, 40), (128, 64), (32, 10), (48, 15), (32, 40), (64, 10)])
@pytest.mark.parametrize("small,large", [((3,), 700), ((60, 64, 64, 61), 300), ((256, 130), 700), ((250, 256), 200)])
def test_small_matrices_beside_large_ones(windq, small, large, G, K):
    """In quarters by two workgroups per tile or one per sweep, beside a matrix in one piece; the launch decides, no bit changes."""
    mats = [inputs(64 * t - 3, G, 40 + i, torch.bfloat16) for i, t in enumerate(small)] + [inputs(64 * 130, G * (large // 100), 50, torch.bfloat16)]
    cg = synth.clip_grid(K)
    batch = windq.windq_features_fit_score_batch([m[0] for m in mats], [m[1] for m in mats], G, 0, cg)
    for (W, s), got in zip(mats, batch):
        want = windq.windq_fit_score_all_bits(W, s, G, 0, cg)
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got[1:], want))
    compare(*mats[0], G, 0, cg, batch[0][1:])
