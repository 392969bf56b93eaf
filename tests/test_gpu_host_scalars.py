"""Energies that calls return to the host through pinned memory shared by the contexts
of a process: many live contexts (more than one slab holds), batches around a unit of
the slab and past all of it, contexts that come and go, and several threads."""

import threading

import pytest
import torch

from paper_2103_04856_amd import fe, inputs

from gpu_helpers import HELFRICH_SC, log

pytestmark = pytest.mark.gpu


def _call(batch, seed):
    n = 8
    u = torch.from_numpy(inputs.uniform_noise(n, seed)).to("cuda").expand(batch, n, n, n).contiguous()
    ctx = fe.FeContext(u.shape, 1.0 / n, 2.0 / n, HELFRICH_SC, dtype=torch.float64)
    ref, _ = ctx.energy_grad_async(u)         # the same sweep and sums, into device memory
    return ctx, u, ref.cpu()


def test_contexts_that_share_and_overflow_the_slab():
    held = []
    # 64, 65 and 4096 doubles lie at a unit's and the slab's ends; then 70 contexts of a unit each
    for k, batch in enumerate([1, 64, 65, 129, 4032, 4096, 4097] + [3] * 70):
        log(f"case host scalars {k} batch={batch}")
        held.append(_call(batch, 100 + k % 5))
        if k % 3 == 2:
            held.pop(0)[0].close()
    for ctx, u, ref in held:
        E, _ = ctx.energy_grad(u)
        assert torch.equal(E, ref)
    for ctx, u, ref in held:                  # nobody else's energies moved
        assert torch.equal(ctx.energy_grad(u)[0], ref)
        ctx.close()
    ctx, u, ref = _call(2, 7)                 # after the slab went back
    assert torch.equal(ctx.energy_grad(u)[0], ref)


def test_threads_with_contexts_of_their_own():
    bad = []

    def work(seed):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(5):
                ctx, u, ref = _call(1 + seed, 10 * seed + k)
                for _ in range(10):
                    if not torch.equal(ctx.energy_grad(u)[0], ref):
                        bad.append((seed, k))
                ctx.close()

    threads = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
