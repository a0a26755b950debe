"""Ends and diagonals of factor tiles: block rows that the diagonal crosses or the matrix's end cuts, in every form of the result (square,
running average, packed triangle), with the matrix off the 16-byte grid and its surroundings guarded.  Against float64 on the host."""
import numpy as np
import pytest
import torch

from oracle import kfac_oracle as ko
from paper_1811_12019_amd import binding as kb
from paper_1811_12019_amd import synth
from tests.test_parity_gpu import DEV, FACTOR_TOL, rel_fro, rel_max

pytestmark = pytest.mark.gpu

GUARD = 1024
# columns: ends in the first, in a middle and in the last vector of a 32-row block, whole blocks and tiles, one to four tiles
COLS = [8, 24, 32, 36, 40, 60, 64, 68, 96, 100, 124, 128, 132, 160, 188, 192, 224, 252, 256, 292, 380, 420]
RUN, DECAY = 3.0, 0.95


def guarded(n):
    """n floats one off the 16-byte grid, in the middle of a marked buffer."""
    buf = torch.full((n + 2 * GUARD + 1,), 7.0, device=DEV)
    return buf, buf[GUARD + 1:GUARD + 1 + n]


@pytest.mark.parametrize("bias", [0, 1])
@pytest.mark.parametrize("dtype", [kb.KFAC_BF16, kb.KFAC_F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("cols", COLS + [1, 3, 37, 70, 101, 250, 399])          # (the others are no whole vectors)
def test_ends(cols, dtype, bias):
    shp = synth.LayerShape("ends", 3, cols, 5, 7, 24, 1, 1, 1, 0, has_bias=bool(bias))
    rng = np.random.default_rng([cols, bias])
    x = rng.standard_normal((3, cols, 5, 7)).astype(np.float32)
    if dtype == kb.KFAC_BF16:
        x = synth.round_to_bf16(x)
    ref = ko.factor_A(x, 1, 1, 1, 0, bool(bias), ko.ORDER_KH_KW_C)
    d = ref.shape[0]
    xt = torch.from_numpy(np.ascontiguousarray(x.transpose(0, 2, 3, 1))).to(DEV).to(kb._TORCH_DTYPE[dtype])
    desc = kb.make_desc(shp, kb.KFAC_NHWC, dtype, kb.KFAC_ORDER_KH_KW_C)
    ws = kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV)
    old = rng.standard_normal((d, d)).astype(np.float32)
    old = old + old.T
    # 16 builds of the same tensor, so that every width of columns goes to the tile kernel
    for form in ("square", "running", "packed"):
        bufs, outs = zip(*(guarded(d * (d + 1) // 2 if form == "packed" else d * d) for _ in range(16)))
        spare = [torch.empty((d, d), device=DEV) for _ in range(16)]
        if form == "running":
            for o in outs:
                o.copy_(torch.from_numpy(old).to(DEV).flatten())
            batch = kb.FactorBatch([(kb.KFAC_OP_FACTOR_A, desc, xt, s, 0.0) for s in spare], device=DEV,
                                   running=[o.view(d, d) for o in outs], decay=DECAY)
            want = DECAY * old.astype(np.float64) + (1 - DECAY) * ref
        elif form == "packed":
            batch = kb.FactorBatch([(kb.KFAC_OP_FACTOR_A, desc, xt, o, 0.0) for o in outs], device=DEV, packed=True)
            want = ko.pack_upper(ref)
        else:
            batch = kb.FactorBatch([(kb.KFAC_OP_FACTOR_A, desc, xt, o.view(d, d), 0.0) for o in outs], device=DEV)
            want = ref
        kb.kfac_factor_batched(batch)
        torch.cuda.synchronize()
        first = None
        for buf, o in zip(bufs, outs):
            assert bool((buf[:GUARD + 1] == 7).all()) and bool((buf[GUARD + 1 + o.numel():] == 7).all()), form
            got = o.cpu().numpy()
            if first is None:
                first = got
                full = got.astype(np.float64) if form == "packed" else got.reshape(d, d).astype(np.float64)
                assert rel_fro(full, want) < FACTOR_TOL and rel_max(full, want) < FACTOR_TOL, (form, d)
                if form != "packed":
                    np.testing.assert_array_equal(full, full.T)
            np.testing.assert_array_equal(got, first)
    # alone: the same bits for few builds as for one
    one = torch.empty((d, d), device=DEV)
    kb.kfac_factor_A(desc, xt, 0.0, one, ws)
    torch.cuda.synchronize()
    assert rel_fro(one.cpu().numpy(), ref) < FACTOR_TOL
