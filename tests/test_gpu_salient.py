"""GPU parity of salient-weight protection (Sec. 3.5; App. "Salient Weight Protection")
against the oracle: the protected set bit for bit, INT8 codes and scales bit for bit,
errors to 1e-5."""
import numpy as np
import pytest
import torch

from oracle import windq_oracle as O
from paper_2605_26660_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
REL = 1e-5


def to_np(t):
    return t.float().cpu().numpy()


def check_select(windq, W, s, G, unit_rows, ppm):
    mask = windq.windq_salient_select(W, s, G, unit_rows, ppm)
    torch.cuda.synchronize()
    keep = O.salient_select(to_np(W), s.cpu().numpy(), G, unit_rows, ppm)
    want = O.pack_mask(keep)
    got = mask.cpu().numpy()
    assert got.shape == want.shape
    bad = np.argwhere(got != want)
    assert bad.size == 0, f"{len(bad)} mask bytes differ, first at {bad[0]}"
    U, R_u = windq.n_units(W.shape[0], W.shape[1], G, unit_rows)
    assert int(np.unpackbits(got).sum()) == U * windq.windq_n_protected(R_u * G, ppm)
    return mask, keep


def check_encode(windq, W, s, G, unit_rows, ppm, mask, keep):
    codes, scale, err = windq.windq_salient_encode(W, s, G, unit_rows, mask, ppm)
    torch.cuda.synchronize()
    o_codes, o_off, o_sigma, o_err = O.salient_encode(to_np(W), s.cpu().numpy(), G, unit_rows, keep)
    assert np.array_equal(codes.cpu().numpy().ravel(), o_codes)
    assert np.array_equal(scale.cpu().numpy().view(np.uint32), o_sigma.view(np.uint32))
    g = err.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(g - o_err) <= REL * np.abs(o_err) + 1e-300), np.max(np.abs(g - o_err) / (np.abs(o_err) + 1e-300))


@pytest.mark.parametrize("R,C,G,unit_rows,ppm,dtype", [
    (256, 512, 128, 0, 30000, torch.bfloat16), (256, 512, 128, 128, 30000, torch.bfloat16),
    (200, 256, 64, 100, 20000, torch.bfloat16), (512, 512, 64, 0, 30000, torch.float32),
    (8, 16, 8, 4, 250000, torch.float32), (70, 96, 32, 0, 500000, torch.bfloat16),
    (130, 256, 256, 0, 30000, torch.bfloat16), (64, 128, 128, 0, 1000000, torch.bfloat16),
    (64, 128, 128, 0, 0, torch.bfloat16), (64, 128, 128, 0, 100, torch.bfloat16)])
def test_select_and_encode(windq, R, C, G, unit_rows, ppm, dtype):
    W = synth.weights_llm(R, C, seed=71, device=DEV, dtype=dtype)
    X = synth.activations_llm(64, C, seed=72, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    mask, keep = check_select(windq, W, s, G, unit_rows, ppm)
    check_encode(windq, W, s, G, unit_rows, ppm, mask, keep)


def test_ties_are_taken_in_flat_index_order(windq):
    """bf16 weights under a constant scale: a few hundred distinct saliencies for tens of thousands of
    weights, so the threshold is shared by many and the tie rule decides most of the set."""
    W = synth.weights_llm(320, 256, seed=73, device=DEV)
    s = torch.ones(256, device=DEV)
    for unit_rows, ppm in ((0, 30000), (64, 30000), (0, 333333), (160, 900000)):
        mask, keep = check_select(windq, W, s, 128, unit_rows, ppm)
        check_encode(windq, W, s, 128, unit_rows, ppm, mask, keep)
    Wc = torch.full((192, 128), 0.25, dtype=torch.bfloat16, device=DEV)      # every saliency equal
    Wc[100:] = 0                                                             # and a second plateau at zero
    for ppm in (30000, 600000):
        mask, keep = check_select(windq, Wc, s[:128], 64, 96, ppm)
        check_encode(windq, Wc, s[:128], 64, 96, ppm, mask, keep)


@pytest.mark.parametrize("R,C,G,unit_rows,ppm,dtype", [
    (1, 64, 8, 0, 250000, torch.float32), (3, 1024, 512, 0, 50000, torch.bfloat16), (2048, 512, 512, 0, 30000, torch.bfloat16),
    (1030, 256, 128, 0, 1000, torch.bfloat16), (2304, 96, 96, 1152, 50000, torch.float32), (4100, 8, 8, 0, 30000, torch.bfloat16)])
def test_select_over_the_sizes_of_its_sample(windq, R, C, G, unit_rows, ppm, dtype):
    """Units smaller than the sample's least, read half, and sampled thinly; a mask of several rounds per tile."""
    W = synth.weights_llm(R, C, seed=78, device=DEV, dtype=dtype)
    s = torch.exp(torch.randn(C, generator=torch.Generator().manual_seed(5))).to(DEV)
    mask, keep = check_select(windq, W, s, G, unit_rows, ppm)
    check_encode(windq, W, s, G, unit_rows, ppm, mask, keep)


def flagged_units(windq, W, s, G, unit_rows, ppm):
    """The units that a selection took by digit passes over W: the list that it leaves in its workspace (after three histograms
    of 2048 counters per unit and the units' two ends, middle, counts and flags, each part on 256 bytes)."""
    code = windq.WINDQ_BF16 if W.dtype == torch.bfloat16 else windq.WINDQ_F32
    ws = torch.zeros(windq.workspace_bytes(windq.CALL_SALIENT, code, W.shape[0], W.shape[1], G, unit_rows), dtype=torch.uint8, device=DEV)
    windq.windq_salient_select(W, s, G, unit_rows, ppm, ws=ws)
    U, _ = windq.n_units(W.shape[0], W.shape[1], G, unit_rows)
    at = sum((n + 255) // 256 * 256 for n in (3 * U * 2048 * 4, 4 * U, 4 * U, 4 * U, 8 * U, 4 * U))
    n = int(ws[at:at + 4].view(torch.int32).item())
    return sorted(ws[at + 256:at + 256 + 4 * n].view(torch.int32).tolist())


def sampled_elements(R, G, dtype):
    """Which weights of a whole-column unit of more than 32768 the selection samples: 64-byte segments, a power of two of them,
    of evenly spread rows, one after the other along the columns."""
    seg = min(64 // (2 if dtype == torch.bfloat16 else 4), G & -G)
    n_seg = 32768 // seg
    hit = torch.zeros(R, G, dtype=torch.bool)
    for i in range(n_seg):
        at = i % (G // seg) * seg
        hit[(i * R + R // 2) // n_seg, at:at + seg] = True
    assert int(hit.sum()) == 32768
    return hit.to(DEV)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_select_and_encode_where_the_sample_misleads(windq, dtype):
    """Large weights only where the sample does not look, only where it does, and equal ones where it does not: the count of the
    pass over W refutes the bracket of those units, they are selected the long way (their ties too), the others
    from their lists; one tile then holds more protected weights than its part of the collection area."""
    R, C, G, ppm = 4096, 512, 128, 15000
    W = synth.weights_llm(R, C, seed=79, device=DEV, dtype=dtype)
    hit = sampled_elements(R, G, dtype)
    n_p = windq.windq_n_protected(R * G, ppm)
    unseen = (~hit[:2000].any(1)).nonzero().squeeze(1)[:70]
    W[unseen, :128] *= 64                                      # more above the bracket than are to be protected
    W[:400, 128:256] = torch.where(hit[:400], W[:400, 128:256] * 64, W[:400, 128:256])      # fewer in it
    assert n_p < 70 * 128 and int(hit[:400].sum()) < n_p
    W[unseen, 384:512] = 3.0                                   # more equal ones above it
    s = torch.ones(C, device=DEV)
    assert flagged_units(windq, W, s, G, 0, ppm) == [0, 1, 3]
    mask, keep = check_select(windq, W, s, G, 0, ppm)
    check_encode(windq, W, s, G, 0, ppm, mask, keep)


@pytest.mark.parametrize("R,C,G,unit_rows,dtype,spread", [
    (1024, 512, 64, 128, torch.bfloat16, 0.0), (1024, 512, 64, 128, torch.float32, 0.8),        # 8192 weights a unit: the smallest lists
    (1024, 512, 128, 256, torch.bfloat16, 0.8), (1028, 512, 128, 257, torch.bfloat16, 0.8),     # 32768, sampled whole, and one row more
    (4096, 512, 128, 0, torch.bfloat16, 0.0), (4096, 512, 128, 0, torch.float32, 0.5), (4096, 512, 128, 0, torch.bfloat16, 0.8),
    (1000, 960, 96, 0, torch.bfloat16, 0.8), (600, 512, 512, 0, torch.bfloat16, 0.3), (9000, 40, 40, 0, torch.float32, 0.3)])
def test_ordinary_weights_are_selected_from_the_list(windq, R, C, G, unit_rows, dtype, spread):
    """Weights of the usual kind, rows of one norm or of log-normal norms, at rates from 0.5 to 30 %: no unit needs the digit
    passes; small units hold the same set as the oracle finds."""
    W = synth.weights_llm(R, C, seed=80, device=DEV, dtype=torch.float32)
    W = (W * torch.exp(spread * torch.randn(R, 1, generator=torch.Generator().manual_seed(8))).to(DEV)).to(dtype)
    s = torch.exp(torch.randn(C, generator=torch.Generator().manual_seed(9))).to(DEV)
    for ppm in (5000, 30000, 50000, 100000) + ((300000,) if spread < 0.5 else ()):
        assert flagged_units(windq, W, s, G, unit_rows, ppm) == []
    check_select(windq, W, s, G, unit_rows, 50000)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("R,C,G,unit_rows", [(2048, 512, 128, 0), (1024, 256, 64, 128), (600, 1024, 512, 0), (130, 96, 32, 65), (640, 192, 96, 0)])
def test_weights_of_few_values(windq, R, C, G, unit_rows, dtype):
    """Equal weights, and weights rounded to a grid: lists that overflow before or during the pass over W, ties split in a list (more
    than are ranked one by one, and fewer) and by digit passes."""
    W = synth.weights_llm(R, C, seed=81, device=DEV, dtype=torch.float32)
    ones = torch.ones(C, device=DEV)
    for Wk in (torch.full_like(W, 0.25), torch.round(W / 0.01) * 0.01, torch.round(W / 0.001) * 0.001):
        Wk = Wk.to(dtype)
        for ppm in (5000, 30000, 200000):
            check_select(windq, Wk, ones, G, unit_rows, ppm)
    few = torch.full_like(W, 0.25).to(dtype)
    assert len(flagged_units(windq, few, ones, G, unit_rows, 30000)) == windq.n_units(R, C, G, unit_rows)[0]


def test_select_routes_agree(windq):
    """Selection from the units' candidate lists (the usual route) and by digit passes over W (taken when the
    mask cannot be addressed in whole dwords, or a unit's threshold bin outgrows its list) give the same mask."""
    W = synth.weights_llm(256, 512, seed=75, device=DEV)
    X = synth.activations_llm(64, 512, seed=76, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    for G, unit_rows, ppm in ((128, 0, 30000), (64, 64, 5000), (128, 128, 300000)):
        mask, keep = check_select(windq, W, s, G, unit_rows, ppm)
        buf = torch.zeros(256 * 64 + 8, dtype=torch.uint8, device=DEV)
        odd = buf[1:1 + 256 * 64].view(256, 64)                  # one byte off a dword boundary
        assert odd.data_ptr() % 4 != 0
        windq.windq_salient_select(W, s, G, unit_rows, ppm, out=odd)
        torch.cuda.synchronize()
        assert torch.equal(odd, mask)
    # a mask whose size is no multiple of four bytes
    W2 = synth.weights_llm(70, 24, seed=77, device=DEV)
    s2 = torch.rand(24, device=DEV) + 0.1
    check_select(windq, W2, s2, 8, 0, 100000)
    check_select(windq, W2, s2, 24, 35, 30000)


def test_all_zero_unit_has_zero_scale(windq):
    W = synth.weights_llm(128, 256, seed=74, device=DEV)
    W[:, :128] = 0
    s = torch.rand(256, device=DEV) + 0.1
    mask, keep = check_select(windq, W, s, 128, 0, 30000)
    codes, scale, err = windq.windq_salient_encode(W, s, 128, 0, mask, 30000)
    torch.cuda.synchronize()
    assert float(scale[0]) == 0.0 and float(err[0]) == 0.0 and int(codes[0].abs().max()) == 0
    check_encode(windq, W, s, 128, 0, 30000, mask, keep)


def test_full_size_7b_matrix_sampled(windq):
    """attn-shaped 4096 x 4096 bf16 at 3 %: whole mask on the device, sampled units against the oracle."""
    W = synth.weights_llm(4096, 4096, seed=75, device=DEV)
    X = synth.activations_llm(512, 4096, seed=76, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    G, ppm = 128, 30000
    mask = windq.windq_salient_select(W, s, G, 0, ppm)
    codes, scale, err = windq.windq_salient_encode(W, s, G, 0, mask, ppm)
    torch.cuda.synchronize()
    n_p = windq.windq_n_protected(4096 * G, ppm)
    bits_per_unit = np.unpackbits(mask.cpu().numpy(), axis=1, bitorder="little").reshape(4096, 32, G).sum(axis=(0, 2))
    assert np.all(bits_per_unit == n_p)
    for j in (0, 13, 31):
        cols = slice(j * G, (j + 1) * G)
        Wn, sn = to_np(W[:, cols]), s[cols].cpu().numpy()
        keep = O.salient_select(Wn, sn, G, 0, ppm)
        assert np.array_equal(mask[:, j * G // 8:(j + 1) * G // 8].cpu().numpy(), O.pack_mask(keep))
        o_codes, _, o_sigma, o_err = O.salient_encode(Wn, sn, G, 0, keep)
        assert np.array_equal(codes[j].cpu().numpy(), o_codes)
        assert float(scale[j]) == float(o_sigma[0])
        assert abs(float(err[j]) - o_err[0]) <= REL * o_err[0]
    # fit+score and apply-plan under the mask, in the benchmark's launch configuration
    cg = synth.clip_grid(20)
    e_m, idx_m, ref_m = windq.windq_fit_score_all_bits(W, s, G, 0, cg, mask=mask)
    action = torch.tensor([1 + (u % 6) for u in range(32)], dtype=torch.uint8)
    off = windq.windq_plan_layout(action, 4096, G)
    pcodes, pscale, poffset = windq.windq_apply_plan(W, G, 0, action.to(DEV), idx_m, cg, off.to(DEV), mask=mask)
    torch.cuda.synchronize()
    for j in (0, 13, 31):
        cols = slice(j * G, (j + 1) * G)
        Wn, sn = to_np(W[:, cols]), s[cols].cpu().numpy()
        keep = O.salient_select(Wn, sn, G, 0, ppm)
        o_err, o_idx, o_ref, table = O.fit_score_all_bits(Wn, sn, G, 0, cg.numpy(), keep=keep)
        gi = idx_m[j].cpu().numpy()
        for b in np.nonzero(gi != o_idx[0])[0]:
            assert table[0, b, gi[b]] <= table[0, b].min() * (1 + 1e-9)
        assert np.all(np.abs(e_m[j].cpu().numpy() - o_err[0]) <= REL * o_err[0])
        assert abs(float(ref_m[j]) - o_ref[0]) <= REL * o_ref[0]
        a1 = action[j:j + 1].numpy()
        off1 = O.plan_layout(a1, 4096, G)
        oc, osc, oof = O.apply_plan(Wn, G, 0, a1, gi[None, :], cg.numpy(), off1, keep=keep)
        assert np.array_equal(pcodes[int(off[j]):int(off[j]) + int(off1[1])].cpu().numpy(), oc)
        assert np.array_equal(pscale[j * 4096:(j + 1) * 4096].cpu().numpy().view(np.uint32), osc.view(np.uint32))
        assert np.array_equal(poffset[j * 4096:(j + 1) * 4096].cpu().numpy().view(np.uint32), oof.view(np.uint32))


# ---------------------------------------------- fit+score and apply-plan under the mask
def check_masked_fit_and_apply(windq, W, s, G, unit_rows, ppm, K):
    mask, keep = check_select(windq, W, s, G, unit_rows, ppm)
    cg = synth.clip_grid(K)
    err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, G, unit_rows, cg, mask=mask)
    torch.cuda.synchronize()
    Wn, sn = to_np(W), s.cpu().numpy()
    o_err, o_idx, o_ref, table = O.fit_score_all_bits(Wn, sn, G, unit_rows, cg.numpy(), keep=keep)
    g_err, g_idx, g_ref = err.cpu().numpy().astype(np.float64), clip_idx.cpu().numpy(), ref.cpu().numpy().astype(np.float64)
    for u, b in zip(*np.nonzero(g_idx != o_idx)):
        assert table[u, b, g_idx[u, b]] <= table[u, b].min() * (1 + 1e-9), (u, b)
    assert np.all(np.abs(g_err - o_err) <= REL * np.abs(o_err)), np.max(np.abs(g_err - o_err) / (np.abs(o_err) + 1e-300))
    assert np.all(np.abs(g_ref - o_ref) <= REL * np.abs(o_ref))
    U, R_u = windq.n_units(W.shape[0], W.shape[1], G, unit_rows)
    for trial in range(2):
        action = (torch.arange(U) + trial) % 7
        action = action.to(torch.uint8)
        off = windq.windq_plan_layout(action, R_u, G)
        codes = torch.full((max(int(off[-1]), 16),), 0xAB, dtype=torch.uint8, device=DEV)
        codes, scale, offset = windq.windq_apply_plan(W, G, unit_rows, action.to(DEV), clip_idx, cg, off.to(DEV),
                                                      codes=codes, mask=mask)
        torch.cuda.synchronize()
        o_codes, o_scale, o_offset = O.apply_plan(Wn, G, unit_rows, action.numpy(), g_idx, cg.numpy(), off.numpy(), keep=keep)
        assert np.array_equal(codes.cpu().numpy()[:int(off[-1])], o_codes)
        assert np.array_equal(scale.cpu().numpy().view(np.uint32), o_scale.view(np.uint32))
        assert np.array_equal(offset.cpu().numpy().view(np.uint32), o_offset.view(np.uint32))
    return g_err, o_err


@pytest.mark.parametrize("R,C,G,unit_rows,ppm,K,dtype", [
    (256, 512, 128, 0, 30000, 20, torch.bfloat16), (256, 512, 128, 128, 30000, 20, torch.bfloat16),
    (200, 256, 64, 100, 20000, 7, torch.bfloat16), (512, 512, 64, 0, 30000, 20, torch.float32),
    (8, 16, 8, 4, 250000, 3, torch.float32), (70, 96, 32, 0, 500000, 5, torch.bfloat16),
    (130, 256, 256, 0, 30000, 20, torch.bfloat16), (64, 128, 128, 0, 1000000, 4, torch.bfloat16),
    (64, 128, 128, 0, 0, 4, torch.bfloat16)])
def test_masked_fit_score_and_apply_plan(windq, R, C, G, unit_rows, ppm, K, dtype):
    W = synth.weights_llm(R, C, seed=81, device=DEV, dtype=dtype)
    X = synth.activations_llm(64, C, seed=82, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    check_masked_fit_and_apply(windq, W, s, G, unit_rows, ppm, K)


def test_protection_takes_the_outliers_out_of_the_fit(windq):
    """Heavy-tailed input columns stretch every group's range; with 3 % protected the 2-bit error of
    the rest falls well below the unprotected one (Sec. 3.5: why salient weights are kept apart)."""
    W = synth.weights_llm(512, 1024, seed=83, device=DEV)
    X = synth.activations_llm(64, 1024, seed=84, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    cg = synth.clip_grid(20)
    err0, _, _ = windq.windq_fit_score_all_bits(W, s, 128, 0, cg)
    g_err, _ = check_masked_fit_and_apply(windq, W, s, 128, 0, 30000, 20)
    assert float(np.sum(g_err[:, 3])) < 0.7 * float(err0[:, 3].double().sum())


def test_groups_with_nothing_kept(windq):
    """A mask that protects whole rows (not one the selector would write: it is an input like any other)."""
    W = synth.weights_llm(64, 256, seed=85, device=DEV)
    s = torch.rand(256, device=DEV) + 0.1
    keep = np.ones((64, 256), dtype=bool)
    keep[3] = False
    keep[10, :128] = False
    keep[11, 5:] = False
    mask = torch.from_numpy(O.pack_mask(keep)).to(DEV)
    cg = synth.clip_grid(6)
    err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, 128, 0, cg, mask=mask)
    torch.cuda.synchronize()
    o_err, o_idx, o_ref, _ = O.fit_score_all_bits(to_np(W), s.cpu().numpy(), 128, 0, cg.numpy(), keep=keep)
    assert np.all(np.abs(err.cpu().numpy() - o_err) <= REL * np.abs(o_err))
    for a in range(1, 7):
        action = torch.full((2,), a, dtype=torch.uint8)
        off = windq.windq_plan_layout(action, 64, 128)
        codes, scale, offset = windq.windq_apply_plan(W, 128, 0, action.to(DEV), None, None, off.to(DEV), mask=mask)
        torch.cuda.synchronize()
        o_codes, o_scale, o_offset = O.apply_plan(to_np(W), 128, 0, action.numpy(), None, np.ones(1, np.float32), off.numpy(), keep=keep)
        assert np.array_equal(codes.cpu().numpy()[:int(off[-1])], o_codes), a
        assert np.array_equal(scale.cpu().numpy().view(np.uint32), o_scale.view(np.uint32))
        assert np.array_equal(offset.cpu().numpy().view(np.uint32), o_offset.view(np.uint32))
        assert float(scale[3]) == 0.0 and float(offset[3]) == 0.0


@pytest.mark.parametrize("G", [32, 64, 128, 256])
def test_masked_apply_plan_wide_dynamic_range(windq, G):
    """Magnitudes spanning far more than an fp64 sum holds exactly, under a mask: the kept weights'
    sum of |w| is defined in column order."""
    gen = torch.Generator().manual_seed(91)
    R, C = 70, 2 * G
    expo = torch.randint(-120, 60, (R, C), generator=gen).double()
    mant = 1.0 + torch.rand(R, C, generator=gen, dtype=torch.float64)
    sign = torch.where(torch.rand(R, C, generator=gen) < 0.5, -1.0, 1.0).double()
    W = (sign * mant * torch.pow(torch.tensor(2.0, dtype=torch.float64), expo)).float().to(torch.bfloat16).to(DEV)
    s = torch.ones(C, device=DEV)
    mask, keep = check_select(windq, W, s, G, 0, 100000)
    for a in range(1, 7):
        action = torch.full((2,), a, dtype=torch.uint8)
        off = windq.windq_plan_layout(action, R, G)
        codes, scale, offset = windq.windq_apply_plan(W, G, 0, action.to(DEV), None, None, off.to(DEV), mask=mask)
        torch.cuda.synchronize()
        oc, osc, oof = O.apply_plan(to_np(W), G, 0, action.numpy(), None, np.ones(1, np.float32), off.numpy(), keep=keep)
        assert np.array_equal(codes.cpu().numpy()[:int(off[-1])], oc), a
        assert np.array_equal(scale.cpu().numpy().view(np.uint32), osc.view(np.uint32)), a
        assert np.array_equal(offset.cpu().numpy().view(np.uint32), oof.view(np.uint32)), a


# ------------------------------------------------- heuristic allocator, end to end
@pytest.mark.parametrize("R,C,G,unit_rows,dtype", [(256, 512, 128, 0, torch.bfloat16), (200, 256, 64, 100, torch.bfloat16),
                                                   (512, 512, 64, 0, torch.float32), (8, 16, 8, 4, torch.float32)])
def test_unit_saliency(windq, R, C, G, unit_rows, dtype):
    W = synth.weights_llm(R, C, seed=95, device=DEV, dtype=dtype)
    X = synth.activations_llm(64, C, seed=96, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    sal = windq.windq_unit_saliency(W, s, G, unit_rows)
    torch.cuda.synchronize()
    want = O.unit_saliency(to_np(W), s.cpu().numpy(), G, unit_rows)
    assert np.all(np.abs(sal.cpu().numpy() - want) <= REL * want)


def test_heuristic_plan_with_protection_and_fallback_end_to_end(windq):
    """Scores and errors from the device, plan and fallback on the host, plan applied under the mask:
    the allocator's plan meets Eq. 1 with Eq. 5's protection overhead, and equals the oracle's."""
    W = synth.weights_llm(512, 2048, seed=97, device=DEV)
    X = synth.activations_llm(64, 2048, seed=98, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    G, ppm = 128, 30000
    U, R_u = windq.n_units(512, 2048, G, 0)
    mask = windq.windq_salient_select(W, s, G, 0, ppm)
    cg = synth.clip_grid(20)
    err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, G, 0, cg, mask=mask)
    sal = windq.windq_unit_saliency(W, s, G, 0).cpu()
    n = torch.full((U,), R_u * G, dtype=torch.int64)
    n_p = torch.full((U,), windq.windq_n_protected(R_u * G, ppm), dtype=torch.int64)
    action, B, ok = windq.windq_heuristic_plan(sal, n, n_p, 200, 250000, 250000)
    o_action, o_B, o_ok = O.heuristic_plan(sal.numpy(), n.numpy(), n_p.numpy(), 200, 250000, 250000)
    assert ok and np.array_equal(action.numpy(), o_action) and B == o_B
    cb, tot = windq.windq_effective_bits(action, n, n_p)
    assert cb == B and cb <= 200 * tot
    a2 = action.clone()
    changed = windq.windq_fallback_promote(a2, err.cpu(), ref.cpu(), 0.2)
    want, n_want = O.fallback_promote(action.numpy(), err.cpu().numpy(), ref.cpu().numpy(), 0.2)
    assert np.array_equal(a2.numpy(), want) and changed == n_want
    off = windq.windq_plan_layout(a2, R_u, G)
    codes, scale, offset = windq.windq_apply_plan(W, G, 0, a2.to(DEV), clip_idx, cg, off.to(DEV), mask=mask)
    torch.cuda.synchronize()
    assert codes.numel() >= int(off[-1]) and torch.isfinite(scale).all()


@pytest.mark.parametrize("G", [8, 512])
def test_extreme_chunk_widths_under_protection(windq, G):
    R, C = 72, 2 * G
    W = synth.weights_llm(R, C, seed=121, device=DEV)
    s = torch.rand(C, device=DEV) + 0.1
    mask, keep = check_select(windq, W, s, G, 0, 60000)
    check_encode(windq, W, s, G, 0, 60000, mask, keep)
    check_masked_fit_and_apply(windq, W, s, G, 24, 60000, 6)
    # refinement and the way back, on the same shapes
    cg = synth.clip_grid(6)
    err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, G, 0, cg, mask=mask)
    action = torch.tensor([3, 5], dtype=torch.uint8)
    off = windq.windq_plan_layout(action, R, G)
    codes, scale, offset, e = windq.windq_refine_plan(W, s, G, 0, action.to(DEV), clip_idx, cg, off.to(DEV), 2, mask=mask)
    d_err, _ = windq.windq_dequant_plan(W, s, G, 0, action.to(DEV), off.to(DEV), codes, scale, offset, mask=mask)
    torch.cuda.synchronize()
    oc, osc, oof, oe = O.refine_plan(to_np(W), s.cpu().numpy(), G, 0, action.numpy(), clip_idx.cpu().numpy(), cg.numpy(),
                                     off.numpy(), 2, keep=keep)
    assert np.array_equal(codes.cpu().numpy()[:int(off[-1])], oc)
    assert np.array_equal(scale.cpu().numpy().view(np.uint32), osc.view(np.uint32))
    assert np.all(np.abs(e.cpu().numpy() - oe) <= REL * oe) and np.all(np.abs(d_err.cpu().numpy() - oe) <= 2 * REL * oe)
