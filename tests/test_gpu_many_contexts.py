"""More live contexts that have returned energies than the shared slab of pinned memory
has units (64), among them batches around a unit's and the slab's ends; then some closed
from the middle and others opened in their place. Every energy stays its context's own."""

import pytest
import torch

from paper_2103_04856_amd import fe, inputs

from gpu_helpers import HELFRICH_SC, log

pytestmark = pytest.mark.gpu


def _open(batch, seed):
    n = 8
    log(f"case many contexts batch={batch} seed={seed}")
    u = torch.from_numpy(inputs.uniform_noise(n, seed)).to("cuda").expand(batch, n, n, n).contiguous()
    ctx = fe.FeContext(u.shape, 1.0 / n, 2.0 / n, HELFRICH_SC, dtype=torch.float64)
    ref = ctx.energy_grad_async(u)[0].cpu()       # the same sweep and sums, into device memory
    assert torch.equal(ctx.energy_grad(u)[0], ref)   # takes pinned memory, kept until close
    return ctx, u, ref


def _check(held):
    for ctx, u, ref in held:
        assert torch.equal(ctx.energy_grad(u)[0], ref)
        assert torch.equal(ctx.energy(u), ctx.energy_grad_async(u, with_grad=False)[0].cpu())


def test_more_contexts_than_the_slab_holds():
    held = [_open(b, 100 + b) for b in (1, 64, 65, 129)]
    held += [_open(1 + k % 3, 200 + k) for k in range(70)]
    assert len(held) > 64
    _check(held)
    for i in (60, 41, 40, 39, 10, 2):
        held.pop(i)[0].close()
    held += [_open(b, 300 + b) for b in (129, 65, 1, 2, 4032, 4096, 4097)]
    _check(held)
    for ctx, _, _ in held:
        ctx.close()
    held = [_open(4032, 400), _open(1, 401)]      # a slab of their own
    _check(held)
    for ctx, _, _ in held:
        ctx.close()
