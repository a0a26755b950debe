"""Element-wise passes over more than 256 MB, which go past the caches, against the same items in calls that do not (the same bits), and
against plain torch.  And edges of preconditioning operands narrower than a vector."""
import numpy as np
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from tests.test_parity_gpu import DEV, PRE_TOL

pytestmark = pytest.mark.gpu

DIMS = [2600 + i for i in range(20)] + [1, 2, 3, 130]      # every start of a row against the 16-byte grid; packed together 273 MB


def squares(seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn((d, d), device=DEV, generator=g) for d in DIMS]


def form(call):
    """What `call` returns, and whether the kernel ran that goes past the caches (its name says so)."""
    kb.kfac_kernel_timing_enable(True)
    try:
        out = call()
        kernels = list(kb.kfac_kernel_timing_report())
    finally:
        kb.kfac_kernel_timing_enable(False)
    return out, any("stream>" in k for k in kernels)


def test_packing_beyond_the_caches():
    full = squares(1)
    some = [torch.full((kb.packed_elems(d),), float("nan"), device=DEV) for d in DIMS]
    alone = [torch.full_like(p, float("nan")) for p in some]
    assert form(lambda: kb.kfac_pack_upper_batched(kb.PackBatch(full, some)))[1]
    assert not any(form(lambda: kb.kfac_pack_upper_batched(kb.PackBatch([f], [p])))[1] for f, p in zip(full, alone))
    for d, f, p, q in zip(DIMS, full, some, alone):
        i, j = torch.triu_indices(d, d, device=DEV)
        assert torch.equal(p, q) and torch.equal(p, f[i, j]), d


def test_running_averages_beyond_the_caches():
    fresh, some = squares(2), squares(3)
    before, alone = [s.clone() for s in some], [s.clone() for s in some]
    assert form(lambda: kb.kfac_ema_batched(kb.EmaBatch(some, fresh), 0.9))[1]
    assert not any(form(lambda: kb.kfac_ema_batched(kb.EmaBatch([s], [f]), 0.9))[1] for s, f in zip(alone, fresh))
    decay = float(np.float32(0.9))
    rest = float(np.float32(1.0) - np.float32(0.9))
    for d, s, a, b, f in zip(DIMS, some, alone, before, fresh):
        assert torch.equal(s, a), d
        x, y = decay * b.double(), rest * f.double()              # a product and a sum, each rounded once to 24 bits
        assert bool(((s.double() - (x + y)).abs() <= 2.0 ** -24 * (y.abs() + (x + y).abs() * 1.0001)).all()), d


def test_change_rate_beyond_the_caches():
    x, prev = squares(4), squares(5)
    some, stream = form(lambda: kb.kfac_factor_diff_batched(kb.DiffBatch(x, prev)).cpu().tolist())
    assert stream
    for d, a, b, got in zip(DIMS, x, prev, some):
        one, stream = form(lambda: kb.kfac_factor_diff_batched(kb.DiffBatch([a], [b])).cpu().tolist())
        assert not stream and got == one[0], d
        want = float((a.double() - b.double()).norm() / b.double().norm())
        assert abs(got - want) <= 1e-6 * want, (d, got, want)      # differences and squares in 24 bits, of 32 elements a thread before it widens


@pytest.mark.parametrize("dtype", [kb.KFAC_BF16, kb.KFAC_F16, kb.KFAC_F32])
def test_bn_gradients_beyond_the_caches(dtype):
    g = torch.Generator(device=DEV).manual_seed(6)
    td = kb._TORCH_DTYPE[dtype]
    shapes = [(32, 56, 56, c) for c in (64, 72, 100, 128, 33, 8)] * 4 + [(2, 1, 1, 5), (3, 7, 7, 64)]
    tensors = [(torch.randn(s, device=DEV, generator=g).to(td), torch.randn(s, device=DEV, generator=g).to(td)) for s in shapes]
    some, stream = form(lambda: kb.kfac_bn_sample_grads_batched(kb.BnBatch([a for a, _ in tensors], [b for _, b in tensors], dtype)))
    assert stream
    for s, (a, b), got in zip(shapes, tensors, some):
        one, stream = form(lambda: kb.kfac_bn_sample_grads_batched(kb.BnBatch([a], [b], dtype))[0])
        assert not stream and torch.equal(got, one), s
        a, b = a.double().flatten(1, 2), b.double().flatten(1, 2)
        want = torch.cat([(a * b).sum(1), b.sum(1)], 1)
        size = torch.cat([(a * b).abs().sum(1), b.abs().sum(1)], 1)
        assert bool(((got.double() - want).abs() <= a.shape[1] * 2.0 ** -24 * size).all()), s       # (any order of fp32 sums)


@pytest.mark.parametrize("dims", [(1, 1), (2, 3), (3, 2), (1, 4), (5, 6), (129, 3), (3, 130), (131, 127)])
def test_precondition_narrow_operands(dims):
    dG, dA = dims
    rng = np.random.default_rng(dims)
    G, A, W = (rng.standard_normal(s).astype(np.float32) for s in ((dG, dG), (dA, dA), (dG, dA)))
    G, A = (G + G.T) / 2, (A + A.T) / 2
    P = torch.full((dG, dA), float("nan"), device=DEV)
    t = [torch.from_numpy(v).to(DEV) for v in (G, A, W)]
    kb.kfac_precondition(t[0], t[1], t[2], dG, dA, P, kb.alloc_workspace(kb.kfac_precondition_workspace_bytes(dG, dA)))
    # against the product of the magnitudes: sums of random signs may cancel
    bound = np.abs(G).astype(np.float64) @ np.abs(W) @ np.abs(A)
    want = G.astype(np.float64) @ W @ A
    assert float((np.abs(P.cpu().numpy() - want) / bound).max()) < PRE_TOL
