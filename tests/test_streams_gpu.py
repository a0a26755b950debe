"""Element-wise passes over more than 256 MB, which go past the caches, against the same items in calls that do not: the same bits.
And edges of preconditioning operands narrower than a vector."""
import numpy as np
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from tests.test_parity_gpu import DEV, PRE_TOL, rel_fro, rel_max

pytestmark = pytest.mark.gpu

DIMS = [2600 + i for i in range(20)] + [1, 2, 3, 130]      # every start of a row against the 16-byte grid; packed together 273 MB


def squares(seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn((d, d), device=DEV, generator=g) for d in DIMS]


def test_packing_beyond_the_caches():
    full = squares(1)
    some = [torch.full((kb.packed_elems(d),), float("nan"), device=DEV) for d in DIMS]
    alone = [torch.full_like(p, float("nan")) for p in some]
    kb.kfac_pack_upper_batched(kb.PackBatch(full, some))
    for f, p in zip(full, alone):
        kb.kfac_pack_upper_batched(kb.PackBatch([f], [p]))
    for d, f, p, q in zip(DIMS, full, some, alone):
        assert torch.equal(p, q), d
        if d <= 130:
            i, j = torch.triu_indices(d, d, device=DEV)
            assert torch.equal(p, f[i, j]), d


def test_running_averages_beyond_the_caches():
    fresh, some = squares(2), squares(3)
    alone = [s.clone() for s in some]
    kb.kfac_ema_batched(kb.EmaBatch(some, fresh), 0.9)
    for s, f in zip(alone, fresh):
        kb.kfac_ema_batched(kb.EmaBatch([s], [f]), 0.9)
    for d, s, a in zip(DIMS, some, alone):
        assert torch.equal(s, a), d


def test_change_rate_beyond_the_caches():
    x, prev = squares(4), squares(5)
    some = kb.kfac_factor_diff_batched(kb.DiffBatch(x, prev)).cpu().tolist()
    for d, a, b, got in zip(DIMS, x, prev, some):
        assert got == kb.kfac_factor_diff_batched(kb.DiffBatch([a], [b])).cpu().tolist()[0], d


@pytest.mark.parametrize("dtype", [kb.KFAC_BF16, kb.KFAC_F16, kb.KFAC_F32])
def test_bn_gradients_beyond_the_caches(dtype):
    g = torch.Generator(device=DEV).manual_seed(6)
    td = kb._TORCH_DTYPE[dtype]
    shapes = [(32, 56, 56, c) for c in (64, 72, 100, 128, 33, 8)] * 4 + [(2, 1, 1, 5), (3, 7, 7, 64)]
    tensors = [(torch.randn(s, device=DEV, generator=g).to(td), torch.randn(s, device=DEV, generator=g).to(td)) for s in shapes]
    some = kb.kfac_bn_sample_grads_batched(kb.BnBatch([a for a, _ in tensors], [b for _, b in tensors], dtype))
    for s, (a, b), got in zip(shapes, tensors, some):
        assert torch.equal(got, kb.kfac_bn_sample_grads_batched(kb.BnBatch([a], [b], dtype))[0]), s


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
