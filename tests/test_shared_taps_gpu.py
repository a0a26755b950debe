"""3 x 3 layers of stride 1 and padding 1 built from the sums that tap pairs at the same offset share: channel counts one side and
the other of whole tiles, padded ones, the smallest images (4 pixels an axis), row ranges split and not, every kind of output."""
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
FORMS = [(NHWC, kb.KFAC_BF16, KKC), (NHWC, kb.KFAC_F16, CKK), (NCHW, kb.KFAC_BF16, CKK), (NCHW, kb.KFAC_F16, KKC),
         (NHWC, kb.KFAC_F32, CKK), (NHWC, kb.KFAC_F32, KKC), (NCHW, kb.KFAC_F32, CKK)]


def layer(N, C, H, W, bias=True):
    return synth.LayerShape(f"{N}x{C}x{H}x{W}", N, C, H, W, 8, 3, 3, 1, 1, has_bias=bias)


SHAPES = [
    layer(131, 64, 4, 4),                 # 64-wide tiles; two middle rows and columns
    layer(3, 61, 26, 27),                 # three padded channels
    layer(8, 64, 41, 40, bias=False),     # 13,120 rows: split
    layer(45, 125, 4, 6),                 # one 128-wide tile, three padded channels
    layer(33, 128, 11, 5),                # 1,815 rows
    layer(23, 192, 7, 9),                 # two tiles a dimension, the second half empty
    layer(16, 250, 13, 5, bias=False),    # two tiles, six padded channels
    layer(70, 256, 5, 4),
    layer(9, 384, 13, 9),                 # three tiles
    layer(400, 256, 3, 3),                # too small an image: dense tiles
]


def build_all(shapes, layout, dtype, order, seed):
    builds, refs = [], []
    for i, s in enumerate(shapes):
        act = _NP_ROUND[dtype](synth.make_act(s, seed + i))
        builds.append((kb.KFAC_OP_FACTOR_A, kb.make_desc(s, layout, dtype, order), kb.to_device_tensor(act, layout, dtype, DEV), s.d_A))
        refs.append(ko.factor_A(act, 3, 3, 1, 1, s.has_bias, order))
    return builds, refs


def check_outputs(builds, refs, ws=None):
    """Plain results against the oracle; running average and packed triangle against the plain ones, bit for bit.  Returns the plain
    results and the launches."""
    full = [torch.full((d, d), float("nan"), device=DEV) for _, _, _, d in builds]
    packed = [torch.full((kb.packed_elems(d),), float("nan"), device=DEV) for _, _, _, d in builds]
    run = [torch.eye(d, device=DEV) * 2.0 + 0.25 for _, _, _, d in builds]
    plain = [r.clone() for r in run]
    items = lambda outs: [(op, desc, x, o, 0.0) for (op, desc, x, _), o in zip(builds, outs)]
    kb.kfac_kernel_timing_enable(True)
    try:
        kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV, ws=ws))
        kb.kfac_factor_batched(kb.FactorBatch(items(packed), device=DEV, packed=True, ws=ws))
        kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV, running=run, decay=0.9, ws=ws))
        kernels = kb.kfac_kernel_timing_report()
    finally:
        kb.kfac_kernel_timing_enable(False)
    kb.kfac_ema_batched(kb.EmaBatch(plain, full), 0.9)
    for i, (ref, f, p, r, want_r) in enumerate(zip(refs, full, packed, run, plain)):
        got = f.cpu().numpy()
        if ref is not None:
            assert np.isfinite(got).all() and rel_fro(got, ref) < FACTOR_TOL and rel_max(got, ref) < FACTOR_TOL, (i, rel_fro(got, ref))
        np.testing.assert_array_equal(got, got.T)
        np.testing.assert_array_equal(p.cpu().numpy(), ko.pack_upper(got).astype(np.float32))
        np.testing.assert_array_equal(r.cpu().numpy(), want_r.cpu().numpy())
    return full, kernels


@pytest.mark.parametrize("layout,dtype,order", FORMS)
def test_shared_tap_sums(layout, dtype, order):
    """Ten builds in a call, each cut by its own work: against the oracle, the other kinds of output, the single call (bit for bit) and
    the end of the scratch."""
    builds, refs = build_all(SHAPES, layout, dtype, order, 90)
    guard, mark = 4096, 0xA5
    need = [kb.kfac_factor_workspace_bytes(op, desc) for op, desc, _, _ in builds]
    ws = [torch.full((n + guard,), mark, dtype=torch.uint8, device=DEV) for n in need]
    full, kernels = check_outputs(builds, refs, ws)
    assert kernels["factor_channels_kernel" if order == CKK else "factor_tile_reduce_kernel<1>"][1] == 3
    for n, w in zip(need, ws):
        assert bool((w[n:] == mark).all())
    for (_, desc, x, d), want, n in zip(builds, full, need):
        alone = torch.full((d, d), float("nan"), device=DEV)
        kb.kfac_factor_A(desc, x, 0.0, alone, kb.alloc_workspace(n, DEV))
        assert torch.equal(alone, want)


@pytest.mark.parametrize("layout,dtype,order", [(NHWC, kb.KFAC_BF16, KKC), (NHWC, kb.KFAC_F16, CKK)])
def test_shared_tap_sums_in_wide_tiles(layout, dtype, order):
    """A call of so much work (16 builds of 8,704 x 2,048) that 256-wide tiles are taken: one and two of them a dimension."""
    builds, refs = build_all([layer(70, 256, 5, 4), layer(30, 250, 21, 22), layer(9, 384, 13, 9), layer(8, 64, 41, 40)],
                             layout, dtype, order, 70)
    s = synth.LayerShape("anchor", 8704, 2048, 1, 1, 8, 1, 1, 1, 0)
    x = torch.randn((s.N, s.C_in), device=DEV).to(kb._TORCH_DTYPE[dtype])
    builds += [(kb.KFAC_OP_FACTOR_A, kb.make_desc(s, layout, dtype, order), x, s.d_A)] * 16
    _, kernels = check_outputs(builds, refs + [None] * 16)
    assert kernels["factor_tile_kernel<256, 16-bit>"][1] == 3 and kernels["factor_tile_kernel<64, 16-bit>"][1] == 3
    assert "factor_tile_kernel<128, 16-bit>" not in kernels


def test_non_finite_input():
    """An infinity at the image's edge reaches every entry whose tap pair meets its pixel inside the image, the bias row and the
    diagonal among them (products of it with the zero padding are not formed)."""
    s = layer(8, 64, 20, 20)
    act = _NP_ROUND[kb.KFAC_BF16](synth.make_act(s, 5))
    act[0, 3, 0, 0] = np.inf                                    # (N, C, H, W): the first pixel
    desc = kb.make_desc(s, NHWC, kb.KFAC_BF16, KKC)
    A = torch.zeros((s.d_A, s.d_A), device=DEV)
    kb.kfac_factor_A(desc, kb.to_device_tensor(act, NHWC, kb.KFAC_BF16, DEV), 0.0, A,
                     kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV))
    A = A.cpu()
    met = [t * 64 + 3 for t in (0, 1, 3, 4)]                    # the taps whose output pixel (0, 0) - t lies in the image
    assert not torch.isfinite(A[met, -1]).any() and not torch.isfinite(A[met, met]).any()
    rest = [t * 64 + 3 for t in (2, 5, 6, 7, 8)]
    assert torch.isfinite(A[rest][:, rest]).all()


@pytest.mark.parametrize("N", [2, 8], ids=["dense", "shared"])
@pytest.mark.parametrize("order", [KKC, CKK])
@pytest.mark.parametrize("pixel", [(0, 0), (19, 7), (9, 19), (11, 4)], ids=["corner", "last row", "last column", "inside"])
def test_where_a_non_finite_input_shows(N, order, pixel):
    """Every entry in which an infinity meets a value inside the image (any value: 0 times it is NaN) or the bias is not finite; entries of
    taps that never see it are."""
    s, c = layer(N, 64, 20, 20), 3
    act = _NP_ROUND[kb.KFAC_BF16](synth.make_act(s, 6))
    act[1, c, pixel[0], pixel[1]] = np.inf
    desc = kb.make_desc(s, NHWC, kb.KFAC_BF16, order)
    A = torch.zeros((s.d_A, s.d_A), device=DEV)
    kb.kfac_factor_A(desc, kb.to_device_tensor(act, NHWC, kb.KFAC_BF16, DEV), 0.0, A,
                     kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV))
    A = A.cpu()
    columns = lambda tap: torch.arange(64) + 64 * tap if order == KKC else torch.arange(64) * 9 + tap
    inside = lambda y, x: 0 <= y < 20 and 0 <= x < 20
    blind = []
    for t1 in range(9):
        y, x = pixel[0] - (t1 // 3 - 1), pixel[1] - (t1 % 3 - 1)          # the output pixel at which tap t1 sees the infinity
        row = int(columns(t1)[c])
        if not inside(y, x):
            blind.append(row)
            continue
        assert not torch.isfinite(A[row, -1]) and not torch.isfinite(A[row, row])
        for t2 in range(9):
            if inside(y + t2 // 3 - 1, x + t2 % 3 - 1):
                assert not torch.isfinite(A[row, columns(t2)]).any() and not torch.isfinite(A[columns(t2), row]).any(), (t1, t2)
    assert torch.isfinite(A[blind][:, blind]).all()
