"""windq_dequant_gemv in launches that come to their units in the order of their cost: against the product of the
reconstruction in fp64, to 1e-5 of sum |w_hat x| as everywhere; entries outside the plan's range count as skipped."""
import pytest
import torch

from paper_2605_26660_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("R,units,G,dtype,only", [
    (4096, 128, 32, torch.bfloat16, None),        # 1024 workgroups: the first size that is ordered
    (3585, 128, 32, torch.bfloat16, None),        # 1024, the last row range of a single row
    (3584, 128, 32, torch.float32, None),         # 896: in the matrix's own order
    (1024, 512, 8, torch.bfloat16, None), (1025, 513, 8, torch.bfloat16, None),       # as many units as are ordered, and one more
    (300, 511, 24, torch.float32, None),
    (4095, 130, 32, torch.bfloat16, (4,)), (4096, 128, 32, torch.bfloat16, (0, 6))])         # one class alone; the first and the last
def test_every_unit_is_multiplied_once(windq, R, units, G, dtype, only):
    C = units * G
    W = synth.weights_llm(R, C, seed=R + units, device=DEV, dtype=dtype)
    gen = torch.Generator().manual_seed(R)
    action = torch.randint(0, 7, (units,), generator=gen, dtype=torch.uint8)
    if only is not None:
        action = torch.tensor(only, dtype=torch.uint8)[action.long() % len(only)]
    off = windq.windq_plan_layout(action, R, G)
    clip = torch.zeros(units, 4, dtype=torch.uint8, device=DEV)
    codes = torch.zeros(int(off[-1]), dtype=torch.uint8, device=DEV)
    if only is None:
        action[7 % units], off[2] = 200, 1 << 62
    act_d, off_d = action.to(DEV), off.to(DEV)
    _, scale, offset = windq.windq_apply_plan(W, G, 0, act_d, clip, synth.clip_grid(3), off_d, codes=codes)
    s = torch.ones(C, device=DEV)
    x = torch.randn(C, generator=torch.Generator(device=DEV).manual_seed(R), device=DEV)
    _, w_hat = windq.windq_dequant_plan(W, s, G, 0, act_d, off_d, codes, scale, offset)
    y = torch.full((R,), float("nan"), device=DEV)
    windq.windq_dequant_gemv(W, G, 0, act_d, off_d, codes, scale, offset, x, out=y)
    want = w_hat.double() @ x.double()
    assert float(((y.double() - want).abs() / (w_hat.double().abs() @ x.double().abs())).max()) <= 1e-5
    both = windq.windq_dequant_gemv_batch([W, W], G, 0, [act_d] * 2, [off_d] * 2, [codes] * 2, [scale] * 2, [offset] * 2, [x] * 2)
    assert torch.equal(both[0], y) and torch.equal(both[1], y)
