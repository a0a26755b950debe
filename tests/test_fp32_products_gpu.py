"""Factors of fp32 tensors hold fp32 products, though the matrix cores take them in 16-bit pieces: errors against float64 are no larger than
those of fp32 products that are added up in fp32, in every feed and width of tile.  A missing product of pieces fails: without one of the
two smallest the error of one row is 1.13 times that of fp32 products, without one of the others more than 160 times (numpy, normal values)."""
import numpy as np
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from paper_1811_12019_amd import synth
from tests.test_parity_gpu import DEV

pytestmark = pytest.mark.gpu

NHWC, NCHW = kb.KFAC_NHWC, kb.KFAC_NCHW
CKK, KKC = kb.KFAC_ORDER_C_KH_KW, kb.KFAC_ORDER_KH_KW_C
EPS = 2.0 ** -24


def values(kind, shape, seed):
    """Channels last."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(shape, generator=g, device=DEV)
    if kind == "relu":
        x.clamp_(min=0)
    elif kind == "sparse":
        x *= torch.rand(shape, generator=g, device=DEV) < 0.05
        x[..., 0] = 1.0                                      # (no row and no matrix without a product)
    elif kind == "constant":                                 # (of one sign, the same bits lost in every row; the first loses the most)
        x = (1 + torch.rand(shape[-1], generator=g, device=DEV)).expand(shape).contiguous()
        x[..., 0] = 1.0077972
    elif kind == "scales":
        x *= torch.exp2(torch.randint(-20, 21, (shape[-1],), generator=g, device=DEV).float())
    return x


def unfolded(x, s):
    """Rows of [patch, 1] in (tap, channel) order."""
    if s.kh == 1:
        X = x.reshape(-1, s.C_in)
    else:
        X = torch.nn.functional.unfold(x.permute(0, 3, 1, 2).double(), s.kh, padding=s.pad, stride=s.stride)
        X = X.transpose(1, 2).reshape(-1, s.C_in, s.kh * s.kw).transpose(1, 2).reshape(-1, s.C_in * s.kh * s.kw).float()
    return torch.cat([X, torch.ones((X.shape[0], 1), device=DEV)], 1)


def build(x, s, layout):
    desc = kb.make_desc(s, layout, kb.KFAC_F32, KKC)
    t = x if layout == NHWC else x.permute(0, 3, 1, 2).contiguous()
    A = torch.full((s.d_A, s.d_A), float("nan"), device=DEV)
    kb.kfac_kernel_timing_enable(True)
    try:
        kb.kfac_factor_A(desc, t, 0.0, A, kb.alloc_workspace(kb.kfac_factor_workspace_bytes(kb.KFAC_OP_FACTOR_A, desc), DEV))
        kernels = kb.kfac_kernel_timing_report()
    finally:
        kb.kfac_kernel_timing_enable(False)
    assert any(k.startswith("factor_tile_kernel<") for k in kernels), kernels
    return A


def fp32_products(X):
    """X^T X / rows as fp32 multiply-adds, one after the other in ranges of 128 rows (the shortest a call cuts), whose sums are added."""
    total = None
    for r0 in range(0, X.shape[0], 128):
        acc = torch.zeros((X.shape[1], X.shape[1]), device=DEV)
        for row in X[r0:r0 + 128].double():
            acc = torch.addr(acc.double(), row, row).float()
        total = acc if total is None else total + acc
    return total / X.shape[0]


def error(A, want, unit):
    """2-norm, every column in its own size."""
    return float(((A.double() - want) / unit).norm() / (want / unit).norm())


ROWS = [(1, 1, 1), (2, 1, 1), (4, 1, 1), (1, 15, 7), (8, 7, 7), (12, 14, 14)]
FEEDS = [("pixels", synth.LayerShape("p", n, c, h, w, 8, 1, 1, 1, 0), NHWC) for n, h, w in ROWS for c in (60, 256)] + [
    ("planes", synth.LayerShape("p", 4, 192, 32, 32, 8, 1, 1, 1, 0), NCHW),
    ("repacked", synth.LayerShape("p", 9, 200, 23, 21, 8, 1, 1, 1, 0), NCHW),
    ("patches", synth.LayerShape("p", 3, 24, 9, 8, 8, 3, 3, 2, 1), NHWC),
    ("shared taps", synth.LayerShape("p", 4, 64, 24, 24, 8, 3, 3, 1, 1), NHWC),
    ("shared taps", synth.LayerShape("p", 3, 132, 20, 20, 8, 3, 3, 1, 1), NCHW)]


@pytest.mark.parametrize("kind", ["normal", "relu", "sparse", "constant", "scales"])
@pytest.mark.parametrize("feed,s,layout", FEEDS, ids=lambda v: v if isinstance(v, str) else getattr(v, "R", v) and f"{v.R}x{v.C_in}" if hasattr(v, "R") else None)
def test_errors_are_those_of_fp32_products(feed, s, layout, kind):
    x = values(kind, (s.N, s.H, s.W, s.C_in), 3)
    X = unfolded(x, s)
    want = X.double().t() @ X.double() / X.shape[0]
    size = want.diagonal().clamp(min=1e-30).sqrt()
    unit = size[:, None] * size[None]
    A = build(x, s, layout)
    assert torch.equal(A, A.t())
    got, bound = error(A, want, unit), error(fp32_products(X), want, unit)
    # a tenth for the rounding that the two do not share (the sums' order); 1 % where a single product is an entry
    assert got <= bound * (1.01 if s.R == 1 else 1.1)


def test_one_product():
    """One row: an entry is one product, rounded once, with at most 2^-31 of it missing and the small pieces' sum cut off seven times at
    2^-23 of 2^-5 of it."""
    s = synth.LayerShape("one", 1, 256, 1, 1, 8, 1, 1, 1, 0)
    for kind in ("normal", "constant", "scales"):
        x = values(kind, (1, 1, 1, 256), 4)
        X = unfolded(x, s).double()
        want = X.t() @ X
        assert float(((build(x, s, NHWC).double() - want).abs() / want.abs()).max()) <= 1.25 * EPS


@pytest.mark.parametrize("density", [1.0, 0.25])
def test_sums_of_squares_are_not_rounded_one_way(density):
    """Mean error of the diagonal in units of 2^-24 of an entry, which averaging over 32 ranges of rows does not take away: sums of squares of
    eight bits, rounded 46 times a range, were 0.8 too large and 1.2 too small.  fp32 products: 0.0 to 0.2 either way; 576 entries of 1.3 in the
    root mean square, of which the 9 of a channel are nearly the same sum: 0.16 of chance."""
    s = synth.LayerShape("squares", 32, 64, 28, 28, 8, 3, 3, 1, 1)
    for seed in range(2):
        x = values("normal", (32, 28, 28, 64), seed)
        x *= torch.rand(x.shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV) < density
        want = unfolded(x, s).double().square().sum(0) * float(np.float32(1.0 / s.R))      # (the scale's rounding is not the sums')
        got = build(x, s, NHWC).diagonal().double()
        assert abs(float(((got - want) / want).mean())) < 0.5 * EPS


def test_range_of_magnitudes():
    """The largest finite values stay finite, and from 2^-110 up an operand is whole; below, it is a multiple of 2^-133."""
    mantissa = 1.2345678
    small = torch.tensor([mantissa * 2.0 ** e for e in range(-149, -95)], dtype=torch.float64).float()
    other = torch.tensor([1.0, 2.0 ** 20, -2.0 ** 60, mantissa * 2.0 ** 126, 3.0, -3.4028235e38, 3.4028235e38, 3.3961775e38, 1e-3, -mantissa])
    x = torch.cat([small, other]).reshape(1, 1, 1, -1).to(DEV)
    s = synth.LayerShape("range", 1, x.shape[-1], 1, 1, 8, 1, 1, 1, 0)
    X = unfolded(x, s).double()
    want, A = X.t() @ X, build(x, s, NHWC).double()
    held = want.abs() < 3.4028235e38
    assert bool(torch.isfinite(A[held]).all())
    missing = torch.where(X[0].abs() < 2.0 ** -110, 2.0 ** -134, 0.0)
    bound = 1.25 * EPS * want.abs() + missing[:, None] * X.abs() + missing[None] * X.abs().t() + 2.0 ** -133      # (and where the result is tiny)
    assert bool(((A - want).abs() <= bound)[held].all())


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("feed,s,layout", [FEEDS[1], FEEDS[7], FEEDS[9]] + FEEDS[12:14], ids=["1x256", "105x256", "392x256", "planes", "repacked"])
def test_where_a_non_finite_value_shows(feed, s, layout, value):
    """In every entry of its column and row, the bias and the diagonal among them, and nowhere else."""
    x = values("relu", (s.N, s.H, s.W, s.C_in), 5)
    c = s.C_in - 3
    clean = build(x, s, layout)
    x[s.N - 1, s.H // 2, s.W - 1, c] = value
    A = build(x, s, layout)
    assert not torch.isfinite(A[c]).any() and not torch.isfinite(A[:, c]).any()
    rest = [i for i in range(s.d_A) if i != c]
    assert torch.equal(A[rest][:, rest], clean[rest][:, rest])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("pixel", [(0, 0), (9, 19), (11, 4)], ids=["corner", "edge", "inside"])
def test_where_a_non_finite_value_shows_with_shared_taps(pixel, value):
    s, c = synth.LayerShape("shared", 6, 64, 20, 20, 8, 3, 3, 1, 1), 3
    x = values("relu", (s.N, 20, 20, 64), 6)
    x[1, pixel[0], pixel[1], c] = value
    A = build(x, s, NHWC).cpu()
    inside = lambda y, xx: 0 <= y < 20 and 0 <= xx < 20
    for tap in range(9):
        y, xx = pixel[0] - (tap // 3 - 1), pixel[1] - (tap % 3 - 1)       # the output pixel at which this tap sees the value
        row = tap * 64 + c
        if not inside(y, xx):
            continue
        assert not torch.isfinite(A[row, -1]) and not torch.isfinite(A[row, row])
        for t2 in range(9):
            if inside(y + t2 // 3 - 1, xx + t2 % 3 - 1):
                assert not torch.isfinite(A[row, t2 * 64:t2 * 64 + 64]).any() and not torch.isfinite(A[t2 * 64:t2 * 64 + 64, row]).any()
    other = [i for i in range(s.d_A) if i % 64 != c or i == s.d_A - 1]
    assert torch.isfinite(A[other][:, other]).all()
