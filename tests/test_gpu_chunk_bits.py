"""A gradient has the same bits in every z chunk length of one launch shape: each voxel
takes the same arithmetic wherever its chunk begins."""

import pytest
import torch

from paper_2103_04856_amd import fe, inputs

from gpu_helpers import ALL_TERMS, HELFRICH_SC, WILLMORE_QUARTER, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_gradient_bits_do_not_depend_on_the_z_chunk(dtype, field):
    n, B = 30, 2
    U = torch.stack([torch.from_numpy(inputs.uniform_noise(n, s)) for s in (61, 62)]).to(dtype).cuda()
    cf = torch.stack([torch.full((B, n, n, n), c) for c in ALL_TERMS], 1).to(dtype).cuda().contiguous()
    for p in ([WILLMORE_QUARTER] * B, [HELFRICH_SC] * B, [ALL_TERMS] * B, [HELFRICH_SC, ALL_TERMS]):
        ctx = fe.FeContext(U.shape, 1 / n, 2 / n, p, dtype=dtype)
        if field:
            ctx.set_coeff_field(cf)
        for v, (tx, ty, nt, mask) in enumerate(fe.variants()):
            if not mask & (1 if dtype == torch.float32 else 2):
                continue
            log(f"case chunk bits {dtype} field={field} p={p} {tx}x{ty}/{nt}")
            ctx.set_launch(v, n)
            ref = ctx.energy_grad(U)[1]
            for zc in (1, 2, 7, 15):
                ctx.set_launch(v, zc)
                assert torch.equal(ctx.energy_grad(U)[1], ref), (p, (tx, ty, nt), zc)
        ctx.close()
