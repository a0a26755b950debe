"""The fp32-FMA factor kernel (small builds that would have to be repacked, and whatever the matrix cores cannot take): its row ranges at
their edges, the second pass's groups of eight and four partial sums, and the builds of a call in one launch."""
import numpy as np
import pytest
import torch

from oracle import kfac_oracle as ko
from paper_1811_12019_amd import binding as kb
from paper_1811_12019_amd import synth
from tests.test_parity_gpu import DEV, FACTOR_TOL, _NP_ROUND, rel_fro, rel_max

pytestmark = pytest.mark.gpu

NHWC, NCHW = kb.KFAC_NHWC, kb.KFAC_NCHW
CKK, KKC = kb.KFAC_ORDER_C_KH_KW, kb.KFAC_ORDER_KH_KW_C

# rows x columns of A: one slab and less; 64 | 65 rows (one range | three); 8 and 13 ranges of 32 rows; several tiles; the most ranges (160);
# the last row count of the kernel and the first that is repacked; none left of the bias column
SHAPES = [
    synth.LayerShape("r1", 1, 5, 1, 1, 3, 1, 1, 1, 0),
    synth.LayerShape("r64", 1, 63, 8, 8, 64, 1, 1, 1, 0),
    synth.LayerShape("r65", 5, 7, 13, 1, 65, 1, 1, 1, 0),
    synth.LayerShape("r250", 10, 3, 5, 5, 9, 3, 3, 1, 1),
    synth.LayerShape("r416", 4, 20, 13, 8, 5, 3, 3, 1, 1),
    synth.LayerShape("r512", 8, 16, 8, 8, 16, 3, 3, 1, 1),
    synth.LayerShape("r5225", 11, 30, 25, 19, 2, 1, 1, 1, 0),
    synth.LayerShape("r16383", 43, 3, 127, 3, 1, 1, 1, 1, 0),
    synth.LayerShape("r16384", 64, 3, 16, 16, 5, 1, 1, 1, 0),
    synth.LayerShape("nobias", 3, 33, 7, 5, 7, 3, 3, 2, 1, has_bias=False),
]


@pytest.mark.parametrize("layout,dtype,order", [(NCHW, kb.KFAC_BF16, CKK), (NHWC, kb.KFAC_F16, KKC), (NCHW, kb.KFAC_F32, KKC), (NHWC, kb.KFAC_F32, CKK)])
def test_small_builds_in_one_launch(layout, dtype, order):
    """As squares, packed triangles and running averages in one call of fifteen: the single calls' bits, and the oracle's values."""
    builds, refs = [], []
    for s in SHAPES:
        act, gout = _NP_ROUND[dtype](synth.make_act(s, 4)), _NP_ROUND[dtype](synth.make_gout(s, 4))
        desc = kb.make_desc(s, layout, dtype, order)
        builds.append((kb.KFAC_OP_FACTOR_A, desc, kb.to_device_tensor(act, layout, dtype, DEV), s.d_A))
        builds.append((kb.KFAC_OP_FACTOR_G, desc, kb.to_device_tensor(gout, layout, dtype, DEV), s.d_G))
        refs += [ko.factor_A(act, s.kh, s.kw, s.stride, s.pad, s.has_bias, order), ko.factor_G(gout)]
    for part in (slice(0, 15), slice(5, 20)):
        some = builds[part]
        full = [torch.full((d, d), float("nan"), device=DEV) for _, _, _, d in some]
        packed = [torch.full((kb.packed_elems(d),), float("nan"), device=DEV) for _, _, _, d in some]
        run = [torch.eye(d, device=DEV) * 2.0 + 0.25 for _, _, _, d in some]
        plain = [r.clone() for r in run]
        items = lambda outs: [(op, desc, x, o, 0.0) for (op, desc, x, _), o in zip(some, outs)]
        kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV))
        kb.kfac_factor_batched(kb.FactorBatch(items(packed), device=DEV, packed=True))
        kb.kfac_factor_batched(kb.FactorBatch(items(run), device=DEV, running=run, decay=0.9))
        kb.kfac_ema_batched(kb.EmaBatch(plain, full), 0.9)
        for ref, (op, desc, x, d), f, p, r, want in zip(refs[part], some, full, packed, run, plain):
            alone = torch.full((d, d), float("nan"), device=DEV)
            ws = kb.alloc_workspace(kb.kfac_factor_workspace_bytes(op, desc), DEV)
            (kb.kfac_factor_A if op == kb.KFAC_OP_FACTOR_A else kb.kfac_factor_G)(desc, x, 0.0, alone, ws)
            got = f.cpu().numpy()
            assert rel_fro(got, ref) < FACTOR_TOL and rel_max(got, ref) < FACTOR_TOL
            np.testing.assert_array_equal(got, alone.cpu().numpy())
            np.testing.assert_array_equal(p.cpu().numpy(), ko.pack_upper(got).astype(np.float32))
            np.testing.assert_array_equal(r.cpu().numpy(), want.cpu().numpy())


def test_more_small_builds_than_a_launch_holds():
    """130 builds of tensors that lie off every vector alignment (two launches: 120 and 10), each as its single call."""
    s = synth.LayerShape("r96", 3, 16, 8, 4, 4, 1, 1, 1, 0)
    desc = kb.make_desc(s, NHWC, kb.KFAC_BF16, KKC)
    n = s.N * s.C_in * s.H * s.W
    g = torch.Generator(device=DEV).manual_seed(2)
    xs = [torch.randn(n + 1, device=DEV, generator=g).bfloat16()[1:] for _ in range(130)]
    outs = [torch.full((s.d_A, s.d_A), float("nan"), device=DEV) for _ in xs]
    kb.kfac_factor_batched(kb.FactorBatch([(kb.KFAC_OP_FACTOR_A, desc, x, o, 0.0) for x, o in zip(xs, outs)], device=DEV))
    ws = kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV)
    for x, got in zip(xs, outs):
        alone = torch.full((s.d_A, s.d_A), float("nan"), device=DEV)
        kb.kfac_factor_A(desc, x, 0.0, alone, ws)
        np.testing.assert_array_equal(got.cpu().numpy(), alone.cpu().numpy())
        X = torch.cat([x.double().view(-1, s.C_in), torch.ones(s.R, 1, dtype=torch.float64, device=DEV)], 1)
        ref = (X.t() @ X / s.R).cpu().numpy()
        assert rel_fro(got.cpu().numpy(), ref) < FACTOR_TOL


def chained(X, rows):
    """X^T X of a few columns, in float32, as the kernel adds it: a chain of fused multiply-adds for every range of `rows` rows (a product of
    16-bit values is exact, and so is its sum with a partial sum in float64), then the ranges' sums eight at a time."""
    R, C = X.shape
    n = -(-R // rows)
    P = np.zeros((n * rows, C))
    P[:R] = X
    P = P.reshape(n, rows, C)
    acc = np.zeros((n, C, C), np.float32)
    for k in range(rows):
        acc = (acc + P[:, k, :, None] * P[:, k, None, :]).astype(np.float32)
    total, i = np.zeros((C, C), np.float32), 0
    while i + 8 <= n:
        a = acc[i:i + 8]
        total, i = total + (((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]))), i + 8
    for a in acc[i:]:
        total = total + a
    return total


@pytest.mark.parametrize("rows,longest", [(50176, 128), (401408, 400)])
def test_many_rows_off_the_vector_alignment(rows, longest):
    """Builds of many rows that the matrix cores cannot take: the error of chains of at most 128 rows, or of what 1,024 workgroups make, and no
    more (what the order of the ranges' last additions and the scale add stays below 2^-23)."""
    s = synth.LayerShape("rows", rows // 64, 64, 8, 8, 4, 1, 1, 1, 0, has_bias=False)
    desc = kb.make_desc(s, NHWC, kb.KFAC_BF16, KKC)
    x = torch.randn(rows * 64 + 1, device=DEV, generator=torch.Generator(device=DEV).manual_seed(5)).bfloat16()[1:]
    out = torch.full((s.d_A, s.d_A), float("nan"), device=DEV)
    kb.kfac_factor_A(desc, x, 0.0, out, kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV))
    X = x.float().cpu().numpy().reshape(rows, 64)[:, :8].astype(np.float64)
    ref = X.T @ X / rows
    bound = rel_fro(chained(X, longest) / np.float64(rows), ref) + 2.0 ** -23
    assert rel_fro(out[:8, :8].cpu().numpy(), ref) < bound
