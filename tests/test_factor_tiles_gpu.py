"""Matrix-core factor builder at the sizes where it can go wrong: tile widths 64 / 128 / 256 and one column either side,
padded channels, both column orders and layouts, every dtype, split and unsplit rows, every kind of output.  256-wide tiles are
taken by calls with workgroups and rows enough for them (takes_wide): test_wide_tiles makes such calls, the other tests' are too small."""
import numpy as np
import pytest
import torch

from oracle import kfac_oracle as ko
from paper_1811_12019_amd import binding as kb
from paper_1811_12019_amd import synth
from tests.test_parity_gpu import DEV, FACTOR_TOL, _NP_ROUND, check_factor_pair, rel_fro, rel_max

pytestmark = pytest.mark.gpu

NHWC, NCHW = kb.KFAC_NHWC, kb.KFAC_NCHW
CKK, KKC = kb.KFAC_ORDER_C_KH_KW, kb.KFAC_ORDER_KH_KW_C

EDGE_SHAPES = [
    synth.LayerShape("w64", 2, 64, 9, 9, 64, 1, 1, 1, 0),                  # exactly one narrow tile; odd pixel count
    synth.LayerShape("w65", 3, 65, 5, 7, 127, 1, 1, 1, 0),
    synth.LayerShape("w128", 1, 128, 6, 6, 128, 1, 1, 1, 0),
    synth.LayerShape("w129", 2, 129, 3, 5, 136, 1, 1, 1, 0),
    synth.LayerShape("w256long", 8, 256, 48, 47, 257, 1, 1, 1, 0),         # 18,048 rows: split
    synth.LayerShape("k3c16", 4, 16, 19, 18, 24, 3, 3, 1, 1),              # 144 columns
    synth.LayerShape("k3c57s2", 4, 57, 23, 21, 40, 3, 3, 2, 1),            # 64 padded channels, stride 2: 576 columns
    synth.LayerShape("k5c12", 2, 12, 14, 15, 9, 5, 5, 1, 2, has_bias=False),
    synth.LayerShape("fc1", 1, 520, 1, 1, 10, 1, 1, 1, 0),                 # one row
    synth.LayerShape("k3long", 8, 72, 41, 40, 33, 3, 3, 1, 1),             # 13,120 rows x 648 columns: split
]


@pytest.mark.parametrize("shape", EDGE_SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("layout,dtype,order", [
    (NHWC, kb.KFAC_BF16, KKC), (NHWC, kb.KFAC_F16, CKK), (NCHW, kb.KFAC_BF16, CKK), (NCHW, kb.KFAC_F16, KKC),
    (NHWC, kb.KFAC_F32, CKK), (NCHW, kb.KFAC_F32, CKK), (NCHW, kb.KFAC_F32, KKC)])
def test_factor_tile_edges(shape, layout, dtype, order):
    check_factor_pair(shape, layout, dtype, order, seed=7)


@pytest.mark.parametrize("layout,dtype,order", [(NCHW, kb.KFAC_BF16, CKK), (NHWC, kb.KFAC_BF16, KKC), (NCHW, kb.KFAC_F32, CKK)])
def test_narrow_layer_in_any_layout(layout, dtype, order):
    """conv1-like: 3 channels, 4,900 rows (16-bit: repacked to runs of pixels; fp32: to four channels)."""
    check_factor_pair(synth.LayerShape("g", 4, 3, 70, 70, 16, 7, 7, 2, 3, relu_input=False), layout, dtype, order, seed=3)


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("layout,dtype,order", [(NHWC, kb.KFAC_BF16, KKC), (NCHW, kb.KFAC_BF16, CKK), (NCHW, kb.KFAC_F32, CKK)])
def test_factor_outputs(many, layout, dtype, order):
    """Running average and packed triangle against the plain build, bit for bit, and the plain build against the oracle;
    ten builds, each cut as if alone, and 24, cut by their work together."""
    shapes = [EDGE_SHAPES[i] for i in (1, 3, 5, 6, 9)] + [synth.LayerShape("k1long", 6, 48, 50, 50, 304, 1, 1, 1, 0)]
    builds, refs = [], []
    for s in shapes:
        act, gout = _NP_ROUND[dtype](synth.make_act(s, 2)), _NP_ROUND[dtype](synth.make_gout(s, 2))
        desc = kb.make_desc(s, layout, dtype, order)
        builds.append((kb.KFAC_OP_FACTOR_A, desc, kb.to_device_tensor(act, layout, dtype, DEV), s.d_A))
        builds.append((kb.KFAC_OP_FACTOR_G, desc, kb.to_device_tensor(gout, layout, dtype, DEV), s.d_G))
        refs += [ko.factor_A(act, s.kh, s.kw, s.stride, s.pad, True, order), ko.factor_G(gout)]
    reps = 2 if many else 1                                                # 24 builds, or 12
    builds, refs = builds * reps, refs * reps
    if not many:
        builds, refs = builds[:10], refs[:10]
    full = [torch.full((d, d), float("nan"), device=DEV) for _, _, _, d in builds]
    packed = [torch.full((kb.packed_elems(d),), float("nan"), device=DEV) for _, _, _, d in builds]
    S0 = [torch.eye(d, device=DEV) * 2.0 + 0.25 for _, _, _, d in builds]
    run, plain = [s.clone() for s in S0], [s.clone() for s in S0]
    items = lambda outs: [(op, desc, x, o, 0.0) for (op, desc, x, _), o in zip(builds, outs)]
    kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV))
    kb.kfac_factor_batched(kb.FactorBatch(items(packed), device=DEV, packed=True))
    kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV, running=run, decay=0.9))
    kb.kfac_ema_batched(kb.EmaBatch(plain, full), 0.9)
    torch.cuda.synchronize()
    for ref, f, p, r, want_r in zip(refs, full, packed, run, plain):
        got = f.cpu().numpy()
        assert rel_fro(got, ref) < FACTOR_TOL and rel_max(got, ref) < FACTOR_TOL
        np.testing.assert_array_equal(got, got.T)
        np.testing.assert_array_equal(p.cpu().numpy(), ko.pack_upper(got).astype(np.float32))
        np.testing.assert_array_equal(r.cpu().numpy(), want_r.cpu().numpy())


@pytest.mark.parametrize("layout,dtype,order", [(NHWC, kb.KFAC_BF16, KKC), (NCHW, kb.KFAC_F16, CKK), (NHWC, kb.KFAC_F32, KKC)])
def test_few_builds_equal_single_calls(layout, dtype, order):
    """14 matrix-core builds in one call, each with enough rows to be split and together enough work that a cut by the whole
    call would split them differently (9,248 rows: 6 ranges instead of 8; fp32: 36 and more): each equals its single call bit
    for bit."""
    shapes = [synth.LayerShape("s3x3", 8, 48, 34, 34, 72, 3, 3, 1, 1), synth.LayerShape("s1x1", 8, 264, 34, 34, 136, 1, 1, 1, 0)]
    builds = []
    for i in range(7):
        s = shapes[i % 2]
        act, gout = _NP_ROUND[dtype](synth.make_act(s, 30 + i)), _NP_ROUND[dtype](synth.make_gout(s, 30 + i))
        desc = kb.make_desc(s, layout, dtype, order)
        builds.append((kb.KFAC_OP_FACTOR_A, desc, kb.to_device_tensor(act, layout, dtype, DEV), s.d_A))
        builds.append((kb.KFAC_OP_FACTOR_G, desc, kb.to_device_tensor(gout, layout, dtype, DEV), s.d_G))
    outs = [torch.full((d, d), float("nan"), device=DEV) for _, _, _, d in builds]
    kb.kfac_factor_batched(kb.FactorBatch([(op, desc, x, o, 0.0) for (op, desc, x, _), o in zip(builds, outs)], device=DEV))
    for (op, desc, x, d), got in zip(builds, outs):
        alone = torch.full((d, d), float("nan"), device=DEV)
        ws = kb.alloc_workspace(kb.kfac_factor_workspace_bytes(op, desc), DEV)
        (kb.kfac_factor_A if op == kb.KFAC_OP_FACTOR_A else kb.kfac_factor_G)(desc, x, 0.0, alone, ws)
        np.testing.assert_array_equal(got.cpu().numpy(), alone.cpu().numpy())


# 256-wide tiles: one column either side of one and two tiles, padded and mapped columns, one row, rows split into 2, 8 and 32
# ranges.
WIDE_SHAPES = [
    synth.LayerShape("w129", 2, 129, 9, 11, 255, 1, 1, 1, 0),              # 198 rows
    synth.LayerShape("w256", 1, 256, 5, 5, 257, 1, 1, 1, 0),               # 25 rows: less than a slab
    synth.LayerShape("w511", 3, 511, 7, 7, 512, 1, 1, 1, 0),
    synth.LayerShape("w513", 2, 513, 6, 5, 264, 1, 1, 1, 0),
    synth.LayerShape("onerow", 1, 768, 1, 1, 300, 1, 1, 1, 0),
    synth.LayerShape("k3c32s2", 4, 32, 23, 21, 136, 3, 3, 2, 1),           # 288 columns
    synth.LayerShape("k3c57", 4, 57, 19, 18, 200, 3, 3, 1, 1),             # 64 padded channels: 576 columns
    synth.LayerShape("k3nobias", 2, 40, 14, 15, 520, 3, 3, 1, 1, has_bias=False),
    synth.LayerShape("split2", 6401, 264, 1, 1, 136, 1, 1, 1, 0),          # 6,401 rows: ranges of 3,264 and 3,137
    synth.LayerShape("split8", 8, 72, 81, 80, 136, 3, 3, 1, 1),            # 51,840 rows x 648 columns
    synth.LayerShape("split32", 16, 8, 114, 113, 136, 1, 1, 1, 0),         # 206,112 rows
]


@pytest.mark.parametrize("layout,dtype,order", [
    (NHWC, kb.KFAC_BF16, KKC), (NHWC, kb.KFAC_F16, CKK), (NCHW, kb.KFAC_BF16, CKK), (NCHW, kb.KFAC_F16, KKC)])
def test_wide_tiles(layout, dtype, order):
    """256-wide tiles, which the library takes for calls with at least 150 workgroups of 1,900 rows on average and little padding: 16 builds of
    8,704 rows x 2,048 columns beside the shapes above make such a call.  Plain results against the oracle;
    running average and packed triangle against the plain ones, bit for bit; nothing is written beyond the scratch that
    kfac_factor_workspace_bytes asks for."""
    def anchor_build():
        s = synth.LayerShape("anchor", 8704, 2048, 1, 1, 8, 1, 1, 1, 0)
        act = _NP_ROUND[dtype](synth.make_act(s, 1))
        return s, act, (kb.KFAC_OP_FACTOR_A, kb.make_desc(s, layout, dtype, order), kb.to_device_tensor(act, layout, dtype, DEV), s.d_A)
    anchor, anchor_act, build = anchor_build()
    builds, refs = [build] * 16, [None] * 16                               # (one of them is checked: refs[0])
    refs[0] = ko.factor_A(anchor_act, 1, 1, 1, 0, True, order)
    for i, s in enumerate(WIDE_SHAPES):
        act, gout = _NP_ROUND[dtype](synth.make_act(s, 40 + i)), _NP_ROUND[dtype](synth.make_gout(s, 40 + i))
        desc = kb.make_desc(s, layout, dtype, order)
        if s.d_A > 129:                                                    # (more than 128 data columns)
            builds.append((kb.KFAC_OP_FACTOR_A, desc, kb.to_device_tensor(act, layout, dtype, DEV), s.d_A))
            refs.append(ko.factor_A(act, s.kh, s.kw, s.stride, s.pad, s.has_bias, order))
        builds.append((kb.KFAC_OP_FACTOR_G, desc, kb.to_device_tensor(gout, layout, dtype, DEV), s.d_G))
        refs.append(ko.factor_G(gout))
    guard, mark = 4096, 0xA5
    need = [kb.kfac_factor_workspace_bytes(op, desc) for op, desc, _, _ in builds]
    ws = [torch.full((n + guard,), mark, dtype=torch.uint8, device=DEV) for n in need]
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
    tiles = {k: n for k, (_, n) in kernels.items() if k.startswith("factor_tile_kernel<")}
    assert tiles == {"factor_tile_kernel<256, 16-bit>": 3}, kernels        # every build, in all three calls
    assert kernels["factor_tile_reduce_kernel<1>"][1] == kernels["factor_tile_reduce_kernel<4>"][1] == 3
    kb.kfac_ema_batched(kb.EmaBatch(plain, full), 0.9)
    torch.cuda.synchronize()
    for n, w in zip(need, ws):
        assert bool((w[n:] == mark).all())
    for i, (ref, f, p, r, want_r) in enumerate(zip(refs, full, packed, run, plain)):
        got = f.cpu().numpy()
        want = ref if ref is not None else full[0].cpu().numpy().astype(np.float64)
        assert np.isfinite(got).all(), i
        assert rel_fro(got, want) < FACTOR_TOL and rel_max(got, want) < FACTOR_TOL, (i, rel_fro(got, want), rel_max(got, want))
        np.testing.assert_array_equal(got, got.T)
        np.testing.assert_array_equal(p.cpu().numpy(), ko.pack_upper(got).astype(np.float32))
        np.testing.assert_array_equal(r.cpu().numpy(), want_r.cpu().numpy())


def test_wide_tiles_in_a_captured_graph():
    """A call of 256-wide tiles with split rows, captured and replayed: every replay equals the eager call."""
    s = synth.LayerShape("anchor", 8704, 2048, 1, 1, 8, 1, 1, 1, 0)
    desc = kb.make_desc(s, NHWC, kb.KFAC_BF16, KKC)
    x = torch.randn((s.N, s.C_in), device=DEV).to(torch.bfloat16)
    outs = [torch.full((s.d_A, s.d_A), float("nan"), device=DEV) for _ in range(16)]
    batch = kb.FactorBatch([(kb.KFAC_OP_FACTOR_A, desc, x, o, 0.0) for o in outs], device=DEV)
    kb.kfac_kernel_timing_enable(True)
    try:
        kb.kfac_factor_batched(batch)
        assert "factor_tile_kernel<256, 16-bit>" in kb.kfac_kernel_timing_report()
    finally:
        kb.kfac_kernel_timing_enable(False)
    want = [o.clone() for o in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kb.kfac_factor_batched(batch)
    for _ in range(3):
        for o in outs:
            o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.equal(o, w)


# up to four channels and an even stride (16-bit): a kernel row's pixels as one run of columns.  Even and odd kernel widths, one row,
# strides 2 and 4, pixels that no patch reaches, padding wider than the image's remainder.
RUN_SHAPES = [synth.LayerShape(f"c{C}k{kh}x{kw}s{stride}p{pad}", 3, C, 19 + C, 23 - C, 9 + C, kh, kw, stride, pad, has_bias=bias)
              for C, kh, kw, stride, pad, bias in [
                  (1, 1, 2, 2, 0, True), (1, 3, 3, 2, 1, False), (2, 5, 2, 4, 2, True), (2, 2, 4, 2, 0, True), (3, 7, 7, 2, 3, True),
                  (3, 3, 5, 4, 4, False), (4, 3, 3, 2, 1, True), (4, 1, 7, 2, 3, True), (4, 11, 11, 4, 5, True)]]


@pytest.mark.parametrize("layout,dtype,order", [
    (NHWC, kb.KFAC_BF16, KKC), (NHWC, kb.KFAC_F16, CKK), (NCHW, kb.KFAC_BF16, CKK), (NCHW, kb.KFAC_F16, KKC)])
def test_runs_of_pixels(layout, dtype, order):
    """Few-channel convolutions in a call of 18 builds (so that none is left to the generic kernel): against the oracle, and running
    average and packed triangle against the plain result, bit for bit."""
    builds, refs = [], []
    for i, s in enumerate(RUN_SHAPES):
        act, gout = _NP_ROUND[dtype](synth.make_act(s, 60 + i)), _NP_ROUND[dtype](synth.make_gout(s, 60 + i))
        desc = kb.make_desc(s, layout, dtype, order)
        builds.append((kb.KFAC_OP_FACTOR_A, desc, kb.to_device_tensor(act, layout, dtype, DEV), s.d_A))
        builds.append((kb.KFAC_OP_FACTOR_G, desc, kb.to_device_tensor(gout, layout, dtype, DEV), s.d_G))
        refs += [ko.factor_A(act, s.kh, s.kw, s.stride, s.pad, s.has_bias, order), ko.factor_G(gout)]
    full = [torch.full((d, d), float("nan"), device=DEV) for _, _, _, d in builds]
    packed = [torch.full((kb.packed_elems(d),), float("nan"), device=DEV) for _, _, _, d in builds]
    run = [torch.eye(d, device=DEV) * 2.0 + 0.25 for _, _, _, d in builds]
    plain = [r.clone() for r in run]
    items = lambda outs: [(op, desc, x, o, 0.0) for (op, desc, x, _), o in zip(builds, outs)]
    kb.kfac_kernel_timing_enable(True)
    try:
        kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV))
        kb.kfac_factor_batched(kb.FactorBatch(items(packed), device=DEV, packed=True))
        kb.kfac_factor_batched(kb.FactorBatch(items(full), device=DEV, running=run, decay=0.9))
        kernels = kb.kfac_kernel_timing_report()
    finally:
        kb.kfac_kernel_timing_enable(False)
    assert "factor_repack_kernel" in kernels and "factor_generic_kernel" not in kernels, kernels
    kb.kfac_ema_batched(kb.EmaBatch(plain, full), 0.9)
    for ref, f, p, r, want_r in zip(refs, full, packed, run, plain):
        got = f.cpu().numpy()
        assert np.isfinite(got).all() and rel_fro(got, ref) < FACTOR_TOL and rel_max(got, ref) < FACTOR_TOL
        np.testing.assert_array_equal(got, got.T)
        np.testing.assert_array_equal(p.cpu().numpy(), ko.pack_upper(got).astype(np.float32))
        np.testing.assert_array_equal(r.cpu().numpy(), want_r.cpu().numpy())


@pytest.mark.parametrize("layout,dtype", [(NHWC, kb.KFAC_BF16), (NCHW, kb.KFAC_F16), (NHWC, kb.KFAC_F32), (NCHW, kb.KFAC_F32)])
def test_tensor_off_the_vector_alignment(layout, dtype):
    """A tensor one element off the 16-byte grid (a slice of a larger buffer): repacked (NCHW) or read by the generic kernel (NHWC)."""
    s = synth.LayerShape("off", 3, 64, 17, 18, 72, 3, 3, 1, 1)
    act = _NP_ROUND[dtype](synth.make_act(s, 5))
    desc = kb.make_desc(s, layout, dtype, CKK)
    aligned = kb.to_device_tensor(act, layout, dtype, DEV)
    off = torch.empty(aligned.numel() + 8, dtype=aligned.dtype, device=DEV)[1:1 + aligned.numel()].view(aligned.shape)
    off.copy_(aligned)
    assert off.data_ptr() % 16 != 0
    A = torch.full((s.d_A, s.d_A), float("nan"), device=DEV)
    kb.kfac_factor_A(desc, off, 0.0, A, kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV))
    got, ref = A.cpu().numpy(), ko.factor_A(act, 3, 3, 1, 1, True, CKK)
    assert rel_fro(got, ref) < FACTOR_TOL and rel_max(got, ref) < FACTOR_TOL
    np.testing.assert_array_equal(got, got.T)
