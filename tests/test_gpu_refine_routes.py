"""windq_refine_plan where its kernels can go wrong: trits whose bytes straddle blocks of eight weights, weights at the ends
of the ternary rule, scales that are not finite, and launches that come to their units in the order of their cost.
Against the oracle bit for bit, or against calls small enough to keep the matrix's own order."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def against_oracle(windq, W, s, G, action, n_iter, ppm=0, err=True):
    cg = synth.clip_grid(5)
    U, R_u = windq.n_units(W.shape[0], W.shape[1], G, 0)
    gen = torch.Generator().manual_seed(U)
    clip = torch.randint(0, 5, (U, 4), generator=gen, dtype=torch.uint8)
    off = windq.windq_plan_layout(action, R_u, G)
    mask = keep = None
    Wn, sn = W.float().cpu().numpy(), s.cpu().numpy()
    if ppm:
        mask = windq.windq_salient_select(W, s, G, 0, ppm)
        keep = O.salient_select(Wn, sn, G, 0, ppm)
    poison = torch.full((max(int(off[-1]), 16),), 0xAB, dtype=torch.uint8, device=DEV)
    codes, scale, offset, e = windq.windq_refine_plan(W, s, G, 0, action.to(DEV), clip.to(DEV), cg, off.to(DEV), n_iter, codes=poison, mask=mask)
    with np.errstate(all="ignore"):
        oc, osc, oof, oe = O.refine_plan(Wn, sn, G, 0, action.numpy(), clip.numpy(), cg.numpy(), off.numpy(), n_iter, keep=keep)
    assert np.array_equal(codes.cpu().numpy()[:int(off[-1])], oc)
    assert np.array_equal(scale.cpu().numpy().view(np.uint32), osc.view(np.uint32))
    assert np.array_equal(offset.cpu().numpy().view(np.uint32), oof.view(np.uint32))
    if err:
        assert np.all(np.abs(e.cpu().numpy() - oe) <= 1e-5 * oe)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("G", [8, 16, 24, 32, 40, 48, 64, 104])
def test_trits_at_every_place(windq, G, dtype):
    """Chunk widths that end at each of the five places of a byte, with and without a mask."""
    W = synth.weights_llm(9, 4 * G, seed=G, device=DEV, dtype=dtype)
    s = torch.rand(4 * G, generator=torch.Generator().manual_seed(G)).to(DEV) + 0.1
    action = torch.tensor([5, 6, 4, 5], dtype=torch.uint8)
    for n_iter in (0, 1, 3):
        against_oracle(windq, W, s, G, action, n_iter)
    against_oracle(windq, W, s, G, action, 2, ppm=200000)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_weights_at_the_ends_of_the_ternary_rule(windq, dtype):
    """|w| = gamma / 2 and 3 gamma / 2 (ties go to the even code), zeros of both signs, rows of one magnitude, one outlier."""
    G = 64
    W = torch.zeros(8, 3 * G)
    W[0, :] = torch.tensor([0.5, 1.5, -0.5, -1.5, 1.0, 1.0, -1.0, 1.0] * 24)       # mean 1
    W[1, :] = 0.25
    W[2, ::2] = -0.0
    W[2, 1::2] = 3.0
    W[3, 7::G] = -100.0
    W[4, :] = torch.tensor([1.0, -1.0, 0.0, -0.0] * 48)
    W[5, :] = torch.linspace(-2, 2, 3 * G)
    W[6, :] = torch.tensor([0.499, 0.501, 1.0, 2.0] * 48)
    s = torch.rand(3 * G, generator=torch.Generator().manual_seed(1)) + 0.5
    s[3::16] = 0.0
    for n_iter in (1, 2, 4):
        against_oracle(windq, W.to(dtype).to(DEV), s.to(DEV), G, torch.tensor([5, 6, 5], dtype=torch.uint8), n_iter)


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_scales_that_are_not_finite(windq, bad):
    """Such a column makes a round's sums infinite or NaN, and the round changes nothing."""
    G = 64
    W = synth.weights_llm(70, 3 * G, seed=3, device=DEV)
    s = torch.ones(3 * G)
    s[G + 5] = bad
    for n_iter in (1, 3):
        against_oracle(windq, W, s.to(DEV), G, torch.tensor([5, 5, 4], dtype=torch.uint8), n_iter, err=False)


@pytest.mark.parametrize("units", [512, 513, 5])
def test_order_by_cost_changes_nothing(windq, units):
    """More than 2048 tiles in a launch: units by cost where a matrix has at most 512, each tile as in a call of its own;
    entries that are no action, or lie outside the code stream, are skipped as ever."""
    G, n_iter = 8, 2
    rows = 64 * 3 if units > 5 else 64 * 300 - 7
    W = synth.weights_llm(rows, units * G, seed=units, device=DEV)
    s = torch.rand(units * G, generator=torch.Generator().manual_seed(2)).to(DEV) + 0.1
    U, R_u = windq.n_units(rows, units * G, G, 0)
    gen = torch.Generator().manual_seed(4)
    action = torch.randint(0, 7, (U,), generator=gen, dtype=torch.uint8)
    off = windq.windq_plan_layout(action, R_u, G)
    action[3], off[1] = 9, -16                                  # (off is read per unit)
    total = int(off[-1])
    clip = torch.randint(0, 5, (U, 4), generator=gen, dtype=torch.uint8).to(DEV)
    cg = synth.clip_grid(5)
    n = 2200 // (U * ((R_u + 63) // 64)) + 1
    assert n * U * ((R_u + 63) // 64) > 2048 >= U * ((R_u + 63) // 64)
    codes = [torch.full((max(total, 16),), 0xCD, dtype=torch.uint8, device=DEV) for _ in range(n + 1)]
    act_d, off_d = action.to(DEV), off.to(DEV)
    alone = windq.windq_refine_plan(W, s, G, 0, act_d, clip, cg, off_d, n_iter, codes=codes[n])
    batch = windq.windq_refine_plan_batch([W] * n, [s] * n, G, 0, [act_d] * n, [clip] * n, cg, [off_d] * n, n_iter, codes[:n])
    for got in batch:
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, alone))


@pytest.mark.parametrize("rows", [64 * 31, 64 * 16 + 1, 64 * 40 - 7])
def test_skipped_units_of_an_ordered_launch(windq, rows):
    """A workgroup takes several tiles of a skipped unit: every scale, offset and error of one is zero, whatever lay there, and the
    units between them are what they are in a call of their own."""
    G, units = 8, 150
    W = synth.weights_llm(rows, units * G, seed=rows, device=DEV)
    s = torch.ones(units * G, device=DEV)
    cg = synth.clip_grid(5)
    tiles = units * ((rows + 63) // 64)
    for every in (units + 1, 40, 2):                         # none, four and half of the units are not skipped
        action = torch.zeros(units, dtype=torch.uint8)
        action[every - 1::every] = 4
        off = windq.windq_plan_layout(action, rows, G)
        clip = torch.zeros(units, 4, dtype=torch.uint8, device=DEV)
        poison = lambda: tuple(torch.full((k,), 77.0, device=DEV) for k in (units * rows, units * rows, units))
        codes = [torch.full((max(int(off[-1]), 16),), 0xEE, dtype=torch.uint8, device=DEV) for _ in range(3)]
        n = 2048 // tiles + 1
        act_d, off_d = action.to(DEV), off.to(DEV)
        got = windq.windq_refine_plan_batch([W] * n, [s] * n, G, 0, [act_d] * n, [clip] * n, cg, [off_d] * n, 2, codes[:n], outs=[poison() for _ in range(n)])
        zero = action == 0
        for c, scale, offset, err in got:
            assert float(scale.view(units, rows)[zero.to(DEV)].abs().max()) == 0.0
            assert float(offset.view(units, rows)[zero.to(DEV)].abs().max()) == 0.0 and float(err[zero.to(DEV)].abs().max()) == 0.0
        if every <= units:
            u = every - 1                                     # its own call: a window of one chunk
            one = windq.windq_plan_layout(action[u:u + 1], rows, G)
            c1, sc1, of1, e1 = windq.windq_refine_plan(W[:, u * G:(u + 1) * G], s[:G], G, 0, act_d[u:u + 1], clip[:1], cg, one.to(DEV), 2)
            c, scale, offset, err = got[0]
            assert torch.equal(c[int(off[u]):int(off[u]) + int(one[-1])], c1[:int(one[-1])])
            assert torch.equal(scale.view(units, rows)[u], sc1) and torch.equal(offset.view(units, rows)[u], of1) and torch.equal(err[u], e1[0])
