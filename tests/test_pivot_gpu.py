"""The sweep of one pivot block: every count of 16-wide sub-blocks, whole and ragged, alone and as a matrix's second block, and the first
pivot that is not positive at every place of a sub-block.  Against float64 on the host."""
import numpy as np
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from tests.test_launch_forms_gpu import spd
from tests.test_parity_gpu import INV_TOL, gpu_inverse, rel_fro, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [0, 128])
@pytest.mark.parametrize("blocks", range(1, 9))
def test_sub_blocks(first, blocks):
    for rows in (16 * blocks - 15, 16 * blocks - 9, 16 * blocks - 1, 16 * blocks):
        d = first + rows
        S = spd(d, blocks)
        got, info = gpu_inverse(S, 0.05)
        ref = np.linalg.inv(S.astype(np.float64) + np.float64(np.float32(0.05)) * np.eye(d))
        assert info == 0
        assert rel_fro(got, ref) < INV_TOL and rel_max(got, ref) < INV_TOL, d
        np.testing.assert_array_equal(got, got.T)


@pytest.mark.parametrize("d,bad", [(128, b) for b in list(range(17)) + [31, 64, 77, 112, 127]] + [(39, 38), (200, 128), (200, 143), (200, 199)])
def test_first_pivot_that_is_not_positive(d, bad):
    """Also where later ones are not positive either, and where it is zero and where it is not a number."""
    for value in (-2.0, -0.1, float("nan")):             # (-0.1 + the damping: exactly zero)
        S = np.eye(d, dtype=np.float32)
        S[bad, bad] = value
        S[d - 1, d - 1] = value
        assert gpu_inverse(S, 0.1)[1] == bad + 1


def eliminated_one_by_one(S):
    """Inverse by symmetric elimination in fp32, the columns one after the other, every update one multiply-add."""
    f32, f64 = np.float32, np.float64
    E = S.astype(f32)
    for k in range(len(E)):
        p = E[k, k]
        r = f32(1.0 / np.sqrt(f64(p)))
        u = (E[:, k] * r).astype(f32)
        new = (E.astype(f64) - np.outer(u.astype(f64), u.astype(f64))).astype(f32)
        new[:, k] = new[k] = (u * r).astype(f32)
        new[k, k] = -(r * r)
        E = new
    return -E.astype(f64)


@pytest.mark.parametrize("condition", [1e2, 1e4, 1e5])
@pytest.mark.parametrize("d", [5, 8, 13, 16])
def test_small_blocks_are_as_exact_as_single_eliminations(d, condition):
    rng = np.random.default_rng([d, int(condition)])
    ratio = []
    for _ in range(300):
        q, _ = np.linalg.qr(rng.standard_normal((d, d)))
        S = (q * np.logspace(0, -np.log10(condition), d)) @ q.T
        S = (0.5 * (S + S.T)).astype(np.float32)
        ref = np.linalg.inv(S.astype(np.float64))
        M, info = gpu_inverse(S, 0.0)
        assert info == 0
        ratio.append(np.log(rel_fro(M, ref) / rel_fro(eliminated_one_by_one(S), ref)))
    # (errors of a matrix spread over a decade: a mean of 300 logarithms is good to 4 %)
    assert np.exp(np.mean(ratio)) <= 1.1
