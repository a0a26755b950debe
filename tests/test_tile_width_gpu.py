"""The line between 128- and 256-wide factor tiles: builds on both sides of it, alone (each by its own work) and as a call of many, at the
fewest rows a 256-wide workgroup gets, within the scratch that kfac_factor_workspace_bytes asks for."""
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from paper_1811_12019_amd import synth
from tests.test_parity_gpu import DEV, FACTOR_TOL

pytestmark = pytest.mark.gpu

GUARD, MARK = 4096, 0xA5


def reference(x, s):
    """Float64 on the device, from channels-last x."""
    x = x.double()
    if s.kh == 1:
        X = x.reshape(-1, s.C_in)
    else:
        X = torch.nn.functional.unfold(x.permute(0, 3, 1, 2), s.kh, padding=s.pad).transpose(1, 2).reshape(-1, s.C_in * s.kh * s.kw)
    X = torch.cat([X, torch.ones((X.shape[0], 1), dtype=torch.float64, device=DEV)], 1)
    return X.t() @ X / X.shape[0]


# 1,024 columns are ten 256-wide tiles; 30,400 rows make 16 ranges of 1,900 on average, the fewest that are taken, 30,336 ones of 1,896;
# ragged rows and columns: 36,792 rows are 23 ranges of 1,600, of which a multiple of 8 is kept, 16 of 2,300 (from 36,801 rows on it would be
# 24 of 1,534: narrow); one full tile of 256 columns, a third more work, in as many ranges as scratch allows, 256 of 1,911; shared tap
# sums: 272 workgroups
@pytest.mark.parametrize("shape,wide", [
    (synth.LayerShape("line", 30400, 1024, 1, 1, 8, 1, 1, 1, 0), True),
    (synth.LayerShape("under", 30336, 1024, 1, 1, 8, 1, 1, 1, 0), False),
    (synth.LayerShape("ragged", 4088, 1000, 1, 9, 8, 1, 1, 1, 0), True),
    (synth.LayerShape("full", 156, 256, 56, 56, 8, 1, 1, 1, 0), True),
    (synth.LayerShape("shared", 256, 256, 14, 14, 8, 3, 3, 1, 1), True)], ids=lambda v: getattr(v, "name", str(v)))
@pytest.mark.parametrize("dtype", [kb.KFAC_BF16, kb.KFAC_F16])
def test_width_of_one_build_and_of_many(shape, wide, dtype):
    s = shape
    g = torch.Generator(device=DEV).manual_seed(1)
    x = torch.randn((s.N, s.H, s.W, s.C_in), device=DEV, generator=g).clamp_(min=0).to(kb._TORCH_DTYPE[dtype])
    desc = kb.make_desc(s, kb.KFAC_NHWC, dtype, kb.KFAC_ORDER_C_KH_KW)
    need = kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc)
    want = reference(x, s)

    def run(n):
        outs = [torch.full((s.d_A, s.d_A), float("nan"), device=DEV) for _ in range(n)]
        ws = [torch.full((need + GUARD,), MARK, dtype=torch.uint8, device=DEV) for _ in range(n)]
        batch = kb.FactorBatch([(kb.KFAC_OP_FACTOR_A, desc, x, o, 0.0) for o in outs], device=DEV, ws=ws)
        kb.kfac_kernel_timing_enable(True)
        try:
            kb.kfac_factor_batched(batch)
            kernels = [k for k in kb.kfac_kernel_timing_report() if k.startswith("factor_tile_kernel<")]
        finally:
            kb.kfac_kernel_timing_enable(False)
        for o, w in zip(outs, ws):
            assert bool((w[need:] == MARK).all())
            assert torch.equal(o, o.t())
            assert float((o - want).norm() / want.norm()) < FACTOR_TOL and float((o - want).abs().max() / want.abs().max()) < FACTOR_TOL
        return outs, kernels

    (alone,), kernels = run(1)
    assert kernels == ["factor_tile_kernel<256, 16-bit>" if wide else "factor_tile_kernel<128, 16-bit>"], kernels
    few, kernels = run(3)                                    # few builds: cut as they would be alone
    assert len(kernels) == 1 and ("<256" in kernels[0]) == wide and all(torch.equal(o, alone) for o in few)
    _, kernels = run(16)                                     # by the work of all of them: enough for 256-wide tiles
    assert kernels == ["factor_tile_kernel<256, 16-bit>"], kernels
