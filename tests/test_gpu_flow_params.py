"""Algorithm 1 across set_params: its captured iterations follow the parameters that the
context has now. A context that changes p between replayed loops against fresh contexts
that only ever had one p, from the same A and with cleared moments."""

import pytest
import torch

from paper_2103_04856_amd import fe

from gpu_helpers import ALL_TERMS, HELFRICH_SC, WILLMORE_QUARTER, log

pytestmark = pytest.mark.gpu


def _run(ctx, A, nsteps):
    B = A.shape[0]
    u = torch.empty((B,) + tuple(A.shape[2:]), dtype=A.dtype, device=A.device)
    ctx.hminus_reset()
    E = ctx.hminus_step(A, [0.1] * B, nsteps, sigma_k=1.0, u_out=u)
    torch.cuda.synchronize()
    return E, u, A.clone()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(1, 20, 40, 44), (3, 16, 24, 20)])
def test_flow_follows_set_params(shape, dtype):
    B, h = shape[0], 1.0 / shape[3]
    gen = torch.Generator().manual_seed(17)
    A0 = (0.4 * h * torch.randn((B, 3) + shape[1:], generator=gen, dtype=torch.float64)).to(dtype).cuda()
    A = A0.clone()
    ctx = fe.FeContext(shape, h, 2 * h, WILLMORE_QUARTER, dtype=dtype)
    # trace, no S terms, all terms, and batches that mix them where there is a batch; each
    # p is met twice, so that graphs are both captured and replayed
    mixed = ([WILLMORE_QUARTER, HELFRICH_SC, ALL_TERMS] * B)[:B]
    ps = [WILLMORE_QUARTER, HELFRICH_SC, ALL_TERMS, HELFRICH_SC, mixed, WILLMORE_QUARTER, ALL_TERMS]
    for k, p in enumerate(ps):
        log(f"case flow params {shape} {dtype} {k} p={p}")
        ctx.set_params(2 * h, p)
        A.copy_(A0)
        E, u, Ae = _run(ctx, A, 16)               # two replays of eight
        fresh = fe.FeContext(shape, h, 2 * h, p, dtype=dtype)
        Ef, uf, Af = _run(fresh, A0.clone(), 16)
        fresh.close()
        assert torch.equal(E, Ef), (k, E, Ef)
        assert torch.equal(u, uf) and torch.equal(Ae, Af), k
    ctx.close()
