"""GPU parity of windq_dequant_plan: the error recomputed from the packed artefact against the
oracle's and against what the fit reported; the reconstruction against the oracle's."""
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


def run_case(windq, W, s, G, unit_rows, K, ppm=0, oracle_units=True):
    cg = synth.clip_grid(K)
    mask = keep = None
    if ppm:
        mask = windq.windq_salient_select(W, s, G, unit_rows, ppm)
    err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, G, unit_rows, cg, mask=mask)
    U, R_u = windq.n_units(W.shape[0], W.shape[1], G, unit_rows)
    for shift in (0, 3):
        action = ((torch.arange(U) + shift) % 7).to(torch.uint8)
        off = windq.windq_plan_layout(action, R_u, G)
        codes, scale, offset = windq.windq_apply_plan(W, G, unit_rows, action.to(DEV), clip_idx, cg, off.to(DEV), mask=mask)
        d_err, w_hat = windq.windq_dequant_plan(W, s, G, unit_rows, action.to(DEV), off.to(DEV), codes, scale, offset, mask=mask)
        torch.cuda.synchronize()
        g = d_err.cpu().numpy().astype(np.float64)
        # the loop closes on the device's own numbers: error from the artefact = error the fit reported
        fit = err.cpu().numpy().astype(np.float64)
        want_fit = np.array([0.0 if a == 0 else fit[u, a - 1] for u, a in enumerate(action.tolist())])
        assert np.all(np.abs(g - want_fit) <= 2 * REL * want_fit), np.max(np.abs(g - want_fit) / (want_fit + 1e-300))
        if not oracle_units:
            continue
        Wn, sn = to_np(W), s.cpu().numpy()
        if ppm and keep is None:
            keep = O.salient_select(Wn, sn, G, unit_rows, ppm)
        args = (action.numpy(), off.numpy(), codes.cpu().numpy(), scale.cpu().numpy(), offset.cpu().numpy())
        o_err = O.dequant_error(Wn, sn, G, unit_rows, *args, keep=keep)
        assert np.all(np.abs(g - o_err) <= REL * o_err)
        o_hat = O.dequant_plan(Wn, G, unit_rows, *args, keep=keep)
        got = w_hat.cpu().numpy()
        # one fused multiply-add on the device, fp64-then-fp32 in the oracle: equal but for the last bit in rare cases
        assert np.all(np.abs(got - o_hat) <= np.spacing(np.abs(o_hat)))
        assert np.mean(got != o_hat) < 1e-3


@pytest.mark.parametrize("R,C,G,unit_rows,K,dtype", [
    (256, 512, 128, 0, 20, torch.bfloat16), (200, 256, 64, 100, 7, torch.bfloat16),
    (512, 512, 64, 0, 20, torch.float32), (24, 80, 40, 3, 5, torch.bfloat16), (70, 96, 32, 0, 4, torch.bfloat16),
    (64, 512, 256, 0, 6, torch.bfloat16)])
def test_dequant_closes_the_loop(windq, R, C, G, unit_rows, K, dtype):
    W = synth.weights_llm(R, C, seed=101, device=DEV, dtype=dtype)
    X = synth.activations_llm(64, C, seed=102, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    run_case(windq, W, s, G, unit_rows, K)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("R,C,G,unit_rows", [
    (65, 168, 24, 0),           # less than a pass of 256 pieces to a tile; trits that end within a byte
    (64, 280, 40, 0),           # a little more than one: some threads take two
    (63, 168, 56, 21),
    (130, 192, 96, 0),          # whole passes; the last tile has two rows
    (129, 672, 168, 43), (66, 1512, 504, 0),       # 504: the widest
])
def test_dequant_at_odd_widths(windq, R, C, G, unit_rows, dtype):
    W = synth.weights_llm(R, C, seed=R + C, device=DEV, dtype=dtype)
    X = synth.activations_llm(64, C, seed=107, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    run_case(windq, W, s, G, unit_rows, 5)
    run_case(windq, W, s, G, unit_rows, 5, ppm=50000)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("G", [8, 64, 96, 512])
@pytest.mark.parametrize("what_off,codes_off", [(1, 0), (0, 1), (3, 5)])
def test_dequant_with_buffers_off_the_wide_alignments(windq, G, dtype, what_off, codes_off):
    """w_hat on 4 bytes only, codes on any byte: the same numbers as from aligned buffers, also in one batch with them."""
    R, C = 70, 7 * G
    W = synth.weights_llm(R, C, seed=G, device=DEV, dtype=dtype)
    s = torch.rand(C, generator=torch.Generator().manual_seed(G)).add(0.1).to(DEV)
    cg = synth.clip_grid(4)
    _, clip_idx, _ = windq.windq_fit_score_all_bits(W, s, G, 0, cg)
    action = torch.arange(7, dtype=torch.uint8)
    off = windq.windq_plan_layout(action, R, G)
    a_dev, off_dev = action.to(DEV), off.to(DEV)
    codes, scale, offset = windq.windq_apply_plan(W, G, 0, a_dev, clip_idx, cg, off_dev)
    err, w_hat = windq.windq_dequant_plan(W, s, G, 0, a_dev, off_dev, codes, scale, offset)
    odd_codes = torch.empty(codes.numel() + 16, dtype=torch.uint8, device=DEV)[codes_off:codes_off + codes.numel()].copy_(codes)
    odd_what = torch.zeros(R * C + 4, dtype=torch.float32, device=DEV)[what_off:what_off + R * C].view(R, C)
    odd_err = torch.empty_like(err)
    for batch in (1, 2):
        odd_what.zero_()
        two = [W, W][:batch]
        outs = [(odd_err, odd_what), (torch.empty_like(err), torch.empty_like(w_hat))][:batch]
        windq.windq_dequant_plan_batch(two, [s] * batch, G, 0, [a_dev] * batch, [off_dev] * batch, [odd_codes, codes][:batch],
                                       [scale] * batch, [offset] * batch, outs=outs)
        torch.cuda.synchronize()
        assert torch.equal(odd_what, w_hat)
        # fp64 sums of the same terms, in another order
        assert torch.all((odd_err - err).abs() <= 2.4e-7 * err)
    assert torch.equal(outs[1][0], err) and torch.equal(outs[1][1], w_hat)


@pytest.mark.parametrize("R,C,G,unit_rows,ppm", [(256, 512, 128, 0, 30000), (200, 256, 64, 100, 50000), (70, 96, 32, 0, 300000)])
def test_dequant_under_a_protection_mask(windq, R, C, G, unit_rows, ppm):
    W = synth.weights_llm(R, C, seed=103, device=DEV)
    X = synth.activations_llm(64, C, seed=104, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    run_case(windq, W, s, G, unit_rows, 8, ppm=ppm)


def test_dequant_full_size_matrix_closes_the_loop_everywhere(windq):
    """mlp.down-shaped 4096 x 11008 bf16: every unit's error from the artefact equals the fit's."""
    W = synth.weights_llm(4096, 11008, seed=105, device=DEV)
    X = synth.activations_llm(512, 11008, seed=106, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    run_case(windq, W, s, 128, 0, 20, oracle_units=False)
    run_case(windq, W, s, 128, 0, 20, ppm=30000, oracle_units=False)


def test_malformed_entries_read_nothing(windq):
    W = synth.weights_llm(64, 256, seed=107, device=DEV)
    s = torch.ones(256, device=DEV)
    action = torch.tensor([1, 9], dtype=torch.uint8)
    off = torch.tensor([0, 64 * 128, 64 * 128], dtype=torch.int64)
    codes = torch.zeros(64 * 128, dtype=torch.uint8, device=DEV)
    scale = torch.zeros(128, device=DEV)
    offset = torch.zeros(128, device=DEV)
    err, w_hat = windq.windq_dequant_plan(W, s, 128, 0, action.to(DEV), off.to(DEV), codes, scale, offset)
    torch.cuda.synchronize()
    assert float(err[1]) == 0.0 and torch.equal(w_hat[:, 128:], W[:, 128:].float())
    short = codes[:1024]                                      # unit 0's payload no longer fits: treated as skip
    err, w_hat = windq.windq_dequant_plan(W, s, 128, 0, action.to(DEV), off.to(DEV), short, scale, offset)
    torch.cuda.synchronize()
    assert float(err[0]) == 0.0 and torch.equal(w_hat, W.float())
    odd = torch.tensor([8, 64 * 128, 64 * 128], dtype=torch.int64)     # not on a 16-byte boundary: skip as well
    big = torch.zeros(64 * 128 + 16, dtype=torch.uint8, device=DEV)
    err, w_hat = windq.windq_dequant_plan(W, s, 128, 0, action.to(DEV), odd.to(DEV), big, scale, offset)
    torch.cuda.synchronize()
    assert float(err[0]) == 0.0 and torch.equal(w_hat, W.float())


def test_offsets_near_the_end_of_int64_are_skipped_everywhere(windq):
    """An offset whose payload would end past 2^63 - 1 counts as skip in every call that takes a plan."""
    for R in (64, 3000):                                      # (either kernel of the product)
        W = synth.weights_llm(R, 1024, seed=108, device=DEV)
        s = torch.ones(1024, device=DEV)
        action = torch.tensor([1, 2, 3, 4, 5, 6, 4, 1], dtype=torch.uint8)
        off = windq.windq_plan_layout(action, R, 128)
        codes = torch.zeros(int(off[-1]), dtype=torch.uint8, device=DEV)
        far = torch.cat([torch.full((8,), 2 ** 63 - 16, dtype=torch.int64), off[-1:]]).to(DEV)
        a = action.to(DEV)
        _, scale, offset = windq.windq_apply_plan(W, 128, 0, a, None, None, far, codes=codes)
        assert int(codes.max()) == 0 and float(scale.abs().max()) == 0.0
        _, scale, offset, err = windq.windq_refine_plan(W, s, 128, 0, a, None, None, far, 2, codes=codes)
        assert int(codes.max()) == 0 and float(scale.abs().max()) == 0.0 and float(err.max()) == 0.0
        err, w_hat = windq.windq_dequant_plan(W, s, 128, 0, a, far, codes, scale, offset)
        assert float(err.max()) == 0.0 and torch.equal(w_hat, W.float())
        x = torch.ones(1024, device=DEV)
        mask = torch.zeros(R, 128, dtype=torch.uint8, device=DEV)
        want = W.double().sum(1)
        for m in (None, mask):
            y = windq.windq_dequant_gemv(W, 128, 0, a, far, codes, scale, offset, x, mask=m)
            assert bool(((y.double() - want).abs() <= 1e-6 * W.double().abs().sum(1)).all())


# ------------------------------------------------------- the product from the artefact
def gemv_case(windq, W, s, G, unit_rows, K, ppm=0):
    cg = synth.clip_grid(K)
    mask = keep = None
    if ppm:
        mask = windq.windq_salient_select(W, s, G, unit_rows, ppm)
        keep = O.salient_select(to_np(W), s.cpu().numpy(), G, unit_rows, ppm)
    err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, G, unit_rows, cg, mask=mask)
    U, R_u = windq.n_units(W.shape[0], W.shape[1], G, unit_rows)
    gen = torch.Generator().manual_seed(7)
    x = (torch.randn(W.shape[1], generator=gen) * torch.exp(torch.randn(W.shape[1], generator=gen))).to(DEV)
    for shift in (0, 4):
        action = ((torch.arange(U) + shift) % 7).to(torch.uint8)
        off = windq.windq_plan_layout(action, R_u, G)
        codes, scale, offset = windq.windq_apply_plan(W, G, unit_rows, action.to(DEV), clip_idx, cg, off.to(DEV), mask=mask)
        y = windq.windq_dequant_gemv(W, G, unit_rows, action.to(DEV), off.to(DEV), codes, scale, offset, x, mask=mask)
        torch.cuda.synchronize()
        args = (action.numpy(), off.numpy(), codes.cpu().numpy(), scale.cpu().numpy(), offset.cpu().numpy())
        want, mag = O.dequant_gemv(to_np(W), G, unit_rows, *args, x.cpu().numpy(), keep=keep)
        got = y.cpu().numpy().astype(np.float64)
        # y is a sum of signed terms: its natural scale is sum |w_hat x| (and y itself is rounded to fp32)
        assert np.all(np.abs(got - want) <= REL * mag + 1e-7 * np.abs(want)), np.max(np.abs(got - want) / (mag + 1e-300))


@pytest.mark.parametrize("R,C,G,unit_rows,K,dtype", [
    (256, 512, 128, 0, 20, torch.bfloat16), (200, 256, 64, 100, 7, torch.bfloat16),
    (512, 512, 64, 0, 20, torch.float32), (24, 80, 40, 3, 5, torch.bfloat16), (70, 96, 32, 0, 4, torch.bfloat16),
    (64, 512, 256, 0, 6, torch.bfloat16), (130, 1024, 512, 0, 3, torch.bfloat16), (16, 24, 8, 4, 3, torch.float32)])
def test_gemv_from_the_artefact(windq, R, C, G, unit_rows, K, dtype):
    W = synth.weights_llm(R, C, seed=111, device=DEV, dtype=dtype)
    X = synth.activations_llm(64, C, seed=112, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    gemv_case(windq, W, s, G, unit_rows, K)


@pytest.mark.parametrize("R,C,G,unit_rows,dtype", [
    (257, 128, 128, 0, torch.bfloat16),                 # one row more than a workgroup, one chunk
    (513, 7 * 8, 8, 0, torch.bfloat16), (300, 7 * 24, 24, 0, torch.float32),      # rows of 1 to 24 bytes, pieces cleared to whole dwords
    (260, 3 * 512, 512, 0, torch.bfloat16),             # the widest chunk: four to seven 16-byte steps per row
    (512, 7 * 96, 96, 256, torch.bfloat16)])
def test_gemv_at_the_edges_of_its_tables(windq, R, C, G, unit_rows, dtype):
    W = synth.weights_llm(R, C, seed=121, device=DEV, dtype=dtype)
    s = torch.ones(C, device=DEV)
    gemv_case(windq, W, s, G, unit_rows, 4)


def random_artefact(windq, R, C, G, unit_rows, dtype, masked, seed):
    """A packed plan of random bytes with all seven actions, and a random mask of 3 % of the weights."""
    g = torch.Generator().manual_seed(seed)
    W = synth.weights_llm(R, C, seed=seed, device=DEV, dtype=dtype)
    U, R_u = windq.n_units(R, C, G, unit_rows)
    action = ((torch.arange(U) + seed) % 7).to(torch.uint8)
    off = windq.windq_plan_layout(action, R_u, G)
    codes = torch.randint(0, 256, (max(int(off[-1]), 16),), generator=g, dtype=torch.uint8).to(DEV)
    scale = torch.rand(U * R_u, generator=g).mul(0.1).to(DEV)
    offset = torch.randn(U * R_u, generator=g).to(DEV)
    x = (torch.randn(C, generator=g) * torch.exp(torch.randn(C, generator=g))).to(DEV)
    mask = None
    if masked:
        bits = torch.rand(R, C, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV) < 0.03
        mask = (bits.view(R, C // 8, 8) * (2 ** torch.arange(8, device=DEV))).sum(2).to(torch.uint8)
    return dict(W=W, action=action.to(DEV), off=off.to(DEV), codes=codes, scale=scale, offset=offset, x=x, mask=mask)


def gemv_of(windq, A, G, unit_rows):
    return windq.windq_dequant_gemv(A["W"], G, unit_rows, A["action"], A["off"], A["codes"], A["scale"], A["offset"], A["x"], mask=A["mask"])


def check_against_reconstruction(windq, A, G, unit_rows, y):
    _, w_hat = windq.windq_dequant_plan(A["W"], torch.ones_like(A["x"]), G, unit_rows, A["action"], A["off"], A["codes"], A["scale"],
                                        A["offset"], mask=A["mask"])
    want = w_hat.double() @ A["x"].double()
    mag = w_hat.double().abs() @ A["x"].double().abs()
    bad = ((y.double() - want).abs() / (1e-6 * mag + 1e-7 * want.abs() + 1e-300)).max()
    assert float(bad) <= 1.0, float(bad)


# which kernel a matrix takes turns on its rows per unit (96; 256 under a mask), its weights (1.5 * 2^20; 4 * 2^20 under a mask)
# and, under a mask, the number of 256-row workgroups (256)
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("R,C,G,unit_rows,dtype", [
    (1760, 7 * 128, 128, 0, torch.bfloat16), (1750, 7 * 128, 128, 0, torch.bfloat16),           # just above 1.5 * 2^20, just below
    (28100, 7 * 8, 8, 0, torch.bfloat16), (9400, 7 * 24, 24, 0, torch.float32),                 # rows of 1 to 24 bytes
    (440, 7 * 512, 512, 0, torch.bfloat16), (1200, 7 * 512, 512, 0, torch.float32),             # few workgroups: skip units in parts
    (2304, 7 * 128, 128, 96, torch.bfloat16), (2280, 7 * 128, 128, 95, torch.float32),          # the shortest unit, and one row less
    (2352, 7 * 96, 96, 1176, torch.bfloat16), (4700, 7 * 128, 128, 0, torch.bfloat16),
    (5120, 7 * 128, 128, 256, torch.float32), (5100, 7 * 128, 128, 255, torch.bfloat16),
    (6300, 7 * 104, 104, 0, torch.bfloat16), (17000, 7 * 40, 40, 0, torch.bfloat16),            # masks of 13 and 5 bytes a row
    (77, 7 * 504, 504, 11, torch.bfloat16), (9, 7 * 16, 16, 3, torch.float32)])                 # lanes that share a row by LDS, by shuffles
def test_gemv_at_the_edges_of_its_routes(windq, R, C, G, unit_rows, dtype, masked):
    A = random_artefact(windq, R, C, G, unit_rows, dtype, masked, seed=R + masked)
    check_against_reconstruction(windq, A, G, unit_rows, gemv_of(windq, A, G, unit_rows))


def test_gemv_batch_of_all_routes(windq):
    """Small, large, masked and unmasked matrices in one batch: each as it would be alone."""
    G, shapes = 128, [(300, 512, False), (1800, 1024, False), (300, 512, True), (5000, 1024, True), (5000, 1024, False)]
    As = [random_artefact(windq, r, c, G, 0, torch.bfloat16, m, seed=50 + i) for i, (r, c, m) in enumerate(shapes)]
    alone = [gemv_of(windq, A, G, 0) for A in As]
    both = windq.windq_dequant_gemv_batch([A["W"] for A in As], G, 0, *([A[k] for A in As] for k in ("action", "off", "codes", "scale", "offset", "x")),
                                          masks=[A["mask"] for A in As])
    torch.cuda.synchronize()
    for A, one, b in zip(As, alone, both):
        assert torch.equal(one.view(torch.int32), b.view(torch.int32))
        check_against_reconstruction(windq, A, G, 0, b)


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("G,dtype,large", [(64, torch.bfloat16, (530, 32768)), (96, torch.bfloat16, (4400, 960)), (128, torch.float32, (520, 65536)),
                                           (72, torch.float32, (3000, 1440))])          # two rows a thread, one; lanes a power of two, or not
def test_gemv_batch_of_small_and_large(windq, G, dtype, large, masked):
    """Matrices whose lanes share rows, beside one whose lanes do not, in one launch: each as it would be alone."""
    shapes = [(200, 3 * G, not masked), (*large, masked), (65, 7 * G, masked), (1000, 2 * G, False)]
    As = [random_artefact(windq, r, c, G, 0, dtype, m, seed=70 + i) for i, (r, c, m) in enumerate(shapes)]
    alone = [gemv_of(windq, A, G, 0) for A in As]
    together = windq.windq_dequant_gemv_batch([A["W"] for A in As], G, 0, *([A[k] for A in As] for k in ("action", "off", "codes", "scale", "offset", "x")),
                                              masks=[A["mask"] for A in As])
    torch.cuda.synchronize()
    for A, one, b in zip(As, alone, together):
        assert torch.equal(one.view(torch.int32), b.view(torch.int32))
        check_against_reconstruction(windq, A, G, 0, b)


@pytest.mark.parametrize("R", [96, 4200])               # below and above the size from which tables are used
@pytest.mark.parametrize("bad", [float("inf"), 2.0 ** 120])
def test_gemv_with_values_no_table_may_hold(windq, R, bad):
    """A chunk of x with an infinity or a huge value is summed weight by weight: what the reconstruction times x gives in
    fp32, signs and NaN included, and the other chunks as ever."""
    W = synth.weights_llm(R, 6 * 64, seed=122, device=DEV)
    action = torch.tensor([6, 5, 4, 6, 5, 4], dtype=torch.uint8)
    off = windq.windq_plan_layout(action, R, 64)
    codes, scale, offset = windq.windq_apply_plan(W, 64, 0, action.to(DEV), None, None, off.to(DEV))
    x = torch.randn(6 * 64, generator=torch.Generator().manual_seed(3)).to(DEV)
    _, w_hat = windq.windq_dequant_plan(W, torch.ones(384, device=DEV), 64, 0, action.to(DEV), off.to(DEV), codes, scale, offset)
    for u in range(3):
        xb = x.clone()
        xb[64 * u + 5] = bad
        y = windq.windq_dequant_gemv(W, 64, 0, action.to(DEV), off.to(DEV), codes, scale, offset, xb).double()
        want = (w_hat.double() * xb.double()).sum(1)
        assert torch.equal(torch.isnan(y), torch.isnan(want)) and torch.equal(torch.isinf(y), torch.isinf(want))
        ok = torch.isfinite(want)
        assert bool(((y - want)[ok].abs() <= 1e-6 * (w_hat.double() * xb.double()).abs().sum(1)[ok]).all())
        assert torch.equal(torch.sign(y[torch.isinf(want)]), torch.sign(want[torch.isinf(want)]))


@pytest.mark.parametrize("R", [300, 6600])              # below and above the size from which tables are used
@pytest.mark.parametrize("G", [64, 40])
@pytest.mark.parametrize("positive", [True, False])
def test_gemv_with_scales_that_are_not_finite(windq, R, G, positive):
    """Rows whose stored scale or offset is infinite, NaN or huge: what the reconstruction times x gives, signs and NaN
    included, and the other rows as ever."""
    C = 6 * G
    W = synth.weights_llm(R, C, seed=123, device=DEV)
    W[:8, :G] = W[:8, :G].abs() + 0.01                 # signs all alike: a product of one sign
    action = torch.tensor([6, 5, 4, 6, 5, 4], dtype=torch.uint8)
    off = windq.windq_plan_layout(action, R, G)
    codes, scale, offset = windq.windq_apply_plan(W, G, 0, action.to(DEV), None, None, off.to(DEV))
    bad = [float("inf"), float("-inf"), float("nan"), 2.0 ** 120, -2.0 ** 120]
    sc, of = scale.view(6, R), offset.view(6, R)
    for i, v in enumerate(bad):
        for u in range(3):
            sc[u, 3 * i + u] = v
        of[2, 40 + i] = v
        sc[5, 280 + i] = v
    x = torch.randn(C, generator=torch.Generator().manual_seed(4)).to(DEV)
    x = x.abs() if positive else x
    _, w_hat = windq.windq_dequant_plan(W, torch.ones(C, device=DEV), G, 0, action.to(DEV), off.to(DEV), codes, scale, offset)
    y = windq.windq_dequant_gemv(W, G, 0, action.to(DEV), off.to(DEV), codes, scale, offset, x).double()
    want, mag = (w_hat.double() * x.double()).sum(1), (w_hat.double() * x.double()).abs().sum(1)
    assert bool(torch.isnan(want).any()) and (not positive or bool(torch.isinf(want).any()))
    assert torch.equal(torch.isnan(y), torch.isnan(want)) and torch.equal(torch.isinf(y), torch.isinf(want))
    inf, ok = torch.isinf(want), torch.isfinite(want)
    assert torch.equal(torch.sign(y[inf]), torch.sign(want[inf]))
    assert bool(((y - want)[ok].abs() <= 1e-6 * mag[ok]).all())


@pytest.mark.parametrize("R,C,G,unit_rows,ppm", [(256, 512, 128, 0, 30000), (70, 96, 32, 0, 300000), (24, 80, 40, 3, 100000)])
def test_gemv_under_a_protection_mask(windq, R, C, G, unit_rows, ppm):
    W = synth.weights_llm(R, C, seed=113, device=DEV)
    X = synth.activations_llm(64, C, seed=114, device=DEV)
    s, _ = windq.windq_calib_stats(X)
    gemv_case(windq, W, s, G, unit_rows, 8, ppm=ppm)


def test_gemv_full_size_against_the_reconstruction_and_in_a_batch(windq):
    """4096 x 11008 and 11008 x 4096 bf16: y against the fp64 product of the device's own reconstruction (which
    the oracle checks elsewhere), and sampled rows against the oracle; the batch call gives the same bits."""
    cg = synth.clip_grid(20)
    Ws, acts, offs, cods, scs, ofs, xs, ys = [], [], [], [], [], [], [], []
    for i, (R, C) in enumerate(((4096, 11008), (11008, 4096))):
        W = synth.weights_llm(R, C, seed=115 + i, device=DEV)
        X = synth.activations_llm(512, C, seed=117 + i, device=DEV)
        s, _ = windq.windq_calib_stats(X)
        err, clip_idx, ref = windq.windq_fit_score_all_bits(W, s, 128, 0, cg)
        U, R_u = windq.n_units(R, C, 128, 0)
        gen = torch.Generator().manual_seed(40 + i)
        action = torch.randint(0, 7, (U,), generator=gen, dtype=torch.uint8)
        off = windq.windq_plan_layout(action, R_u, 128)
        codes, scale, offset = windq.windq_apply_plan(W, 128, 0, action.to(DEV), clip_idx, cg, off.to(DEV))
        x = torch.randn(C, generator=gen).to(DEV)
        y = windq.windq_dequant_gemv(W, 128, 0, action.to(DEV), off.to(DEV), codes, scale, offset, x)
        _, w_hat = windq.windq_dequant_plan(W, s, 128, 0, action.to(DEV), off.to(DEV), codes, scale, offset)
        torch.cuda.synchronize()
        ref64 = w_hat.double() @ x.double()
        mag = w_hat.double().abs() @ x.double().abs()
        assert bool(torch.all((y.double() - ref64).abs() <= REL * mag + 1e-7 * ref64.abs()))
        rows = [0, 63, 64, R // 2 + 1, R - 1]
        want, omag = O.dequant_gemv(to_np(W), 128, 0, action.numpy(), off.numpy(), codes.cpu().numpy(), scale.cpu().numpy(),
                                    offset.cpu().numpy(), x.cpu().numpy(), rows=rows)
        got = y.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got[rows] - want[rows]) <= REL * omag[rows] + 1e-7 * np.abs(want[rows]))
        for lst, v in zip((Ws, acts, offs, cods, scs, ofs, xs, ys), (W, action.to(DEV), off.to(DEV), codes, scale, offset, x, y)):
            lst.append(v)
    both = windq.windq_dequant_gemv_batch(Ws, 128, 0, acts, offs, cods, scs, ofs, xs)
    torch.cuda.synchronize()
    for one, b in zip(ys, both):
        assert torch.equal(one.view(torch.int32), b.view(torch.int32))


def test_gemv_checks_its_arguments(windq):
    W = synth.weights_llm(64, 128, seed=119, device=DEV)
    a = torch.full((1,), 2, dtype=torch.uint8)
    off = windq.windq_plan_layout(a, 64, 128).to(DEV)
    codes = torch.zeros(int(off[-1]), dtype=torch.uint8, device=DEV)
    z = torch.zeros(64, device=DEV)
    x = torch.ones(128, device=DEV)
    with pytest.raises(windq.WindqError) as e:
        windq.windq_dequant_gemv(W, 96, 0, a.to(DEV), off, codes, z, z, x)
    assert e.value.status == windq.WINDQ_ESHAPE
    with pytest.raises(windq.WindqError) as e:
        windq.windq_dequant_gemv(W, 128, 0, a.to(DEV), off, codes, z, z, x, ws=torch.empty(64, dtype=torch.uint8, device=DEV))
    assert e.value.status == windq.WINDQ_EWORKSPACE
    with pytest.raises(windq.WindqError) as e:
        windq.windq_dequant_gemv_batch([W] * 9, 128, 0, [a.to(DEV)] * 9, [off] * 9, [codes] * 9, [z] * 9, [z] * 9, [x] * 9)
    assert e.value.status == windq.WINDQ_EINVAL
    y = windq.windq_dequant_gemv(W, 128, 0, a.to(DEV), off, codes, z, z, x)      # scale 0, offset 0: a zero matrix
    torch.cuda.synchronize()
    assert float(y.abs().max()) == 0.0
