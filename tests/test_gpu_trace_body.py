"""The sweeps of a p that depends on kappa1 + kappa2 alone (C1 = C3 = C5 = 0): energy
and gradient against the oracle where tiles, z chunks and precisions meet their edges,
steps, the box-masked form, and a batch that mixes such a p with others."""

import numpy as np
import pytest
import torch

from oracle import fe_oracle as fo, l2flow
from paper_2103_04856_amd import fe, inputs

from gpu_helpers import ALL_TERMS, HELFRICH_SC, TOL, check_energy_grad, log, oracle_input, rel_l2, to_dev

pytestmark = pytest.mark.gpu

# (k1 + k2 - 1.5)^2 + 0.7: every coefficient such a p can have
TRACE_P = (1.0, 2.0, 1.0, -3.0, -3.0, 2.95)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(1, 1, 5), (2, 3, 4), (7, 33, 31), (5, 20, 51), (23, 64, 65)])
def test_energy_and_gradient_match_the_oracle(shape, dtype):
    h = 1.0 / max(shape)
    u = np.random.default_rng(sum(shape)).uniform(-1, 1, size=shape)
    default = fe.FeContext((1,) + shape, h, 2 * h, TRACE_P, dtype=dtype).get_launch()[0]
    for zc in (0, 2):
        log(f"case trace {shape} {dtype} zc={zc}")
        check_energy_grad(u, h, 2 * h, TRACE_P, dtype, variant=default, z_chunk=zc)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_energy_only_steps_and_mixed_batches(dtype):
    n = 34
    h = 1.0 / n
    U = np.stack([inputs.uniform_noise(n, s) for s in (51, 52, 53)])
    tol_e, tol_g = TOL[dtype]["energy"], TOL[dtype]["grad"]
    # alone, with another p without S terms, and with one that has them
    for coeffs in ([TRACE_P] * 3, [TRACE_P, HELFRICH_SC, TRACE_P], [TRACE_P, HELFRICH_SC, ALL_TERMS]):
        log(f"case trace batch {dtype} {coeffs}")
        ud = to_dev(U, dtype)
        uo = oracle_input(ud)
        ctx = fe.FeContext(ud.shape, h, 2 * h, coeffs, dtype=dtype)
        E0 = ctx.energy(ud)
        E, g = ctx.energy_grad(ud)
        for b in range(3):
            Eo, go = fo.energy_grad(uo[b], h, 2 * h, coeffs[b])
            scale = fo.energy_abs(uo[b], h, 2 * h, coeffs[b])
            assert abs(E0[b].item() - Eo) <= tol_e * scale and abs(E[b].item() - Eo) <= tol_e * scale
            assert rel_l2(g[b].cpu().double().numpy(), go) <= tol_g
    ud = to_dev(U, dtype)
    uo = oracle_input(ud)
    ctx = fe.FeContext(ud.shape, h, 2 * h, TRACE_P, dtype=dtype)
    ctx.set_orientation(3.0, (0.6, 0.0, 0.8))
    ctx.step(ud, [0.1] * 3, 1e-3, 2)
    for b in range(3):
        v, _ = fo.descend(uo[b], h, 2 * h, TRACE_P, 0.1, 1e-3, 2, orient=(3.0, (0.6, 0.0, 0.8)))
        assert rel_l2(ud[b].cpu().double().numpy(), v) <= tol_g


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_replicate_boundaries(dtype):
    shape, h = (21, 34, 45), 1.0 / 45
    u = np.random.default_rng(5).uniform(-1, 1, size=shape)
    ud = to_dev(u, dtype)
    flow = fe.FeL2Flow(shape, h, 2 * h, TRACE_P, sigma_k=1.0, dtype=dtype)
    log(f"case trace replicate {dtype}")
    E, g = flow.energy_grad(ud)
    uo = ud.cpu().double().numpy()
    Eo, go = l2flow.energy_grad_replicate(uo, h, 2 * h, TRACE_P, 1.0)
    tol_e, tol_g = TOL[dtype]["energy"], TOL[dtype]["grad"]
    assert abs(E - Eo) <= tol_e * abs(Eo)
    assert rel_l2(g.cpu().double().numpy(), go) <= tol_g
