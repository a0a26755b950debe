"""The forms that inversions and preconditioning take by the size of a call: block counts around the groups of four elimination steps,
batches on both sides of 512 tiles (from which on the last group's updates come with the outputs), and products of up to 384 tiles, which
are made of half tiles.  Against float64 on the host, with the scratch's end guarded and the outputs off the 16-byte grid."""
import numpy as np
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from tests.test_parity_gpu import DEV, INV_TOL, PRE_TOL, rel_fro, rel_max

pytestmark = pytest.mark.gpu

LAM, GUARD, MARK = 0.05, 4096, 0xA5


def spd(d, seed):
    """A covariance of d / 2 + 1 samples: eigenvalues from 0 to about 4, so that the damped matrix's condition is below 100."""
    rng = np.random.default_rng([seed, d])
    X = rng.standard_normal((d // 2 + 1, d)).astype(np.float32)
    return (X.T @ X / np.float32(d)).astype(np.float32)


def off_grid(shape):
    """A matrix one float off the 16-byte grid."""
    n = int(np.prod(shape))
    return torch.full((n + 4,), float("nan"), device=DEV)[1:1 + n].view(shape)


# one block; the second block with one row; group boundaries (4, 5, 6, 8, 9, 10 blocks), whole and ragged; together 305 tiles
SMALL_BATCH = [1, 127, 128, 129, 256, 257, 500, 512, 513, 640, 700, 769, 1024, 1025, 1153, 1200]


@pytest.mark.parametrize("dims", [SMALL_BATCH, SMALL_BATCH + [1281, 1409, 1664], [2177, 2944]], ids=["305", "540", "447"])
def test_inverse_launch_forms(dims):
    S = [spd(d, 3) for d in dims]
    outs = [off_grid((d, d)) for d in dims]
    need = [kb.kfac_inverse_workspace_bytes(d) for d in dims]
    ws = [torch.full((n + GUARD,), MARK, dtype=torch.uint8, device=DEV) for n in need]
    planes = [torch.full((kb.kfac_inverse_planes_bytes(d) + GUARD,), MARK, dtype=torch.uint8, device=DEV) for d in dims]
    St = [torch.from_numpy(s).to(DEV) for s in S]
    batch = kb.InverseBatch(St, outs, [LAM] * len(dims), device=DEV, ws=ws, planes=planes)
    for _ in range(2):                                          # (the second finds the first one's scratch)
        kb.kfac_damped_inverse_batched(batch)
    assert not batch.info.any()
    for d, s, o, n, w, p in zip(dims, S, outs, need, ws, planes):
        got = o.cpu().numpy().astype(np.float64)
        np.testing.assert_array_equal(got, got.T)
        want = np.linalg.inv(s.astype(np.float64) + LAM * np.eye(d))
        assert rel_fro(got, want) < INV_TOL and rel_max(got, want) < INV_TOL, d
        assert bool((w[n:] == MARK).all()) and bool((p[-GUARD:] == MARK).all()), d


# (d_G, d_A): a few rows, ragged both ways, long contractions; all of them together 139 tiles, with more shapes 384 (the last call of
# half tiles), 385 and 411
SHAPES = [(1, 10), (5, 129), (64, 577), (129, 64), (255, 257), (512, 1153), (300, 2049), (1000, 500)]
MORE = SHAPES + [(1920, 2048), (128, 640)]


@pytest.mark.parametrize("shapes", [SHAPES[:4], SHAPES, MORE, MORE + [(100, 100)], SHAPES + [(2048, 2049)]],
                         ids=["few", "139", "384", "385", "411"])
@pytest.mark.parametrize("with_planes", [False, True])
def test_precondition_launch_forms(shapes, with_planes):
    rng = np.random.default_rng(9)
    G, A = [spd(g, 5) for g, _ in shapes], [spd(a, 6) for _, a in shapes]
    W = [(0.03 * rng.standard_normal(s)).astype(np.float32) for s in shapes]
    S = [torch.from_numpy(x).to(DEV) for x in G + A]
    inv = [torch.empty_like(x) for x in S]
    planes = [kb.alloc_workspace(kb.kfac_inverse_planes_bytes(x.shape[0]), DEV) for x in S] if with_planes else None
    kb.kfac_damped_inverse_batched(kb.InverseBatch(S, inv, [LAM] * len(S), device=DEV, planes=planes))
    n = len(shapes)
    out = [off_grid(s) for s in shapes]
    need = [kb.kfac_precondition_workspace_bytes(*s) for s in shapes]
    ws = [torch.full((k + GUARD,), MARK, dtype=torch.uint8, device=DEV) for k in need]
    kw = dict(Ginv_planes=planes[:n], Ainv_planes=planes[n:]) if with_planes else {}
    kb.kfac_precondition_batched(kb.PrecondBatch(inv[:n], inv[n:], [torch.from_numpy(w).to(DEV) for w in W], out, device=DEV, ws=ws, **kw))
    for s, gi, ai, w, o, k, b in zip(shapes, inv[:n], inv[n:], W, out, need, ws):
        want = gi.cpu().numpy().astype(np.float64) @ w.astype(np.float64) @ ai.cpu().numpy().astype(np.float64)
        got = o.cpu().numpy()
        assert rel_fro(got, want) < PRE_TOL and rel_max(got, want) < PRE_TOL, s
        assert bool((b[k:] == MARK).all()), s
