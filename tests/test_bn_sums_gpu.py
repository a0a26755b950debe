"""Sums of the Batch Normalization gradients: no less exact than chains of fp32 additions over 32,768 elements of a sample, whatever a
workgroup holds, and the same bits however many layers share a call."""
import pytest
import torch

from paper_1811_12019_amd import binding as kb
from tests.test_parity_gpu import DEV

pytestmark = pytest.mark.gpu

DTYPES = [kb.KFAC_F32, kb.KFAC_BF16, kb.KFAC_F16]
# one sum, two halves of one workgroup, 2, 4, 7 and 13 workgroups, several column blocks, positions that no lane count divides, halves
# that end beyond the last position
SHAPES = [(4, 49, 512), (4, 196, 256), (4, 784, 128), (2, 196, 1024), (4, 3136, 64), (2, 784, 512), (2, 12544, 64), (3, 1021, 72), (3, 4099, 64),
          (5, 197, 328), (3, 130, 1032), (1, 8195, 8)]


def tensors(shape, dtype, kind, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    rnd = torch.randn if kind == "normal" else torch.rand
    return [rnd(shape, generator=g, device=DEV).to(kb._TORCH_DTYPE[dtype]) for _ in range(2)]


def exact(x, g):
    x, g = x.double(), g.double()
    return torch.cat([(x * g).sum(1), g.sum(1)], 1)


def fp32_chains(x, g, dtype):
    """As exact(), in fp32: workgroups of at most 32,768 elements, each position lane a chain of multiply-adds, then the lanes and the
    workgroups one after the other."""
    N, HW, C = x.shape
    V = 4 if dtype == kb.KFAC_F32 else 8
    width = min(C // V, 64)
    lanes = 256 // width
    most = max(32768 // (width * V), 4 * lanes)
    chunks = -(-HW // most)
    sp = -(-HW // chunks)
    pad = lambda t: torch.nn.functional.pad(t.double(), (0, 0, 0, chunks * sp - HW)).reshape(N, chunks, sp, C)
    x, g = pad(x), pad(g)
    steps = -(-sp // lanes)
    cut = lambda t: torch.nn.functional.pad(t, (0, 0, 0, steps * lanes - sp)).reshape(N, chunks, steps, lanes, C)
    x, g = cut(x), cut(g)
    ds, db = (torch.zeros((N, chunks, lanes, C), device=DEV) for _ in range(2))
    for k in range(steps):
        ds = (ds.double() + x[:, :, k] * g[:, :, k]).float()
        db = (db.double() + g[:, :, k]).float()
    total = torch.cat([ds, db], 3)
    for axis in (2, 1):
        parts = total.unbind(axis if axis == 2 else 1)
        total = parts[0]
        for p in parts[1:]:
            total = total + p
    return total


@pytest.mark.parametrize("kind", ["normal", "positive"])
@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_errors_are_those_of_short_chains(shape, dtype, kind):
    got = chain = 0.0
    for seed in range(4):
        x, g = tensors(shape, dtype, kind, seed)
        want = exact(x, g)
        got += float((kb.kfac_bn_sample_grads(x, g, dtype).double() - want).norm() / want.norm())
        chain += float((fp32_chains(x, g, dtype).double() - want).norm() / want.norm())
    # (5 %: sums that are cut at other positions and added in another order are other samples of the same error, here of 2,000 to 16,000
    # values; chains of twice the length err 10 to 20 % more)
    assert got <= 1.05 * chain, (got / chain)


@pytest.mark.parametrize("dtype", DTYPES)
def test_same_bits_alone_and_together(dtype):
    """Alone, a layer of few workgroups is cut into twice as many as beside the others.  Within the scratch that is asked for."""
    ins = [tensors(s, dtype, "normal", i) for i, s in enumerate(SHAPES + [(40, 3136, 64)])]
    together = kb.kfac_bn_sample_grads_batched(kb.BnBatch([x for x, _ in ins], [g for _, g in ins], dtype))
    for (x, g), want in zip(ins, together):
        batch = kb.BnBatch([x], [g], dtype)
        need = 0 if batch.ws is None else batch.ws.numel()
        assert need <= kb.load_library().kfac_bn_sample_grads_workspace_bytes(x.shape[0], x.shape[2], x.shape[1])
        buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
        batch.ws = buf[:need] if need else None
        got = kb.kfac_bn_sample_grads_batched(batch)[0]
        assert torch.equal(got, want) and bool((buf[need:] == 0xA5).all()), x.shape
