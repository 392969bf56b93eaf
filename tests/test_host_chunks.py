"""Automatic z chunks of gradient sweeps that run in small blocks (grids of fewer than 32
samples in x or y, and coefficient fields on them): enough chunks that a compute unit has
two waves per SIMD to issue from, where the grid has that many."""

import ctypes
import re

from host_stub import ASYM_P, F32, F64, HELFRICH_P, TRACE_P, run

CUS, SIMDS = 256, 4


def small_blocks(api):
    api.stub.stub_slots(12)                      # of 64 or 128 threads: at least what one holds
    for shape, batch, field in (((8, 8, 8), 1000, False), ((12, 12, 12), 256, False), ((10, 10, 10), 100, False),
                                ((20, 20, 20), 64, True), ((16, 16, 16), 128, True), ((200, 30, 16), 8, True),
                                ((4000, 12, 12), 1, False), ((20, 20, 20), 64, False)):
        for dtype in (F32, F64):
            for p in (TRACE_P, HELFRICH_P, ASYM_P):
                ctx = api.context(shape, p, dtype, batch)
                u = api.field((batch,) + shape[1:], shape[0] * (6 if field else 1))
                if field:
                    assert api.lib.fe_set_coeff_field(ctx, u) == 0
                api.log()
                assert api.lib.fe_energy_grad_async(ctx, u, ctypes.c_void_p(8), None) == 0, api.error()
                (name, blocks), = [x for x in api.log() if "grad_sweep" in x[0]]
                threads = int(re.search(r"grad_sweepI[fd]Li\d+ELi\d+ELi(\d+)E", name)[1])
                # about two: 1000 grids of 8^3 in two chunks each make 1.95
                assert threads <= 256 and blocks * threads / 64 >= 1.9 * SIMDS * CUS, (shape, batch, name, blocks)
                api.lib.fe_destroy(ctx)


def full_occupancy(api):
    """Where 24 blocks of 64 threads fit a compute unit, 20 are counted: 300 grids of 10^3
    in 8 x 8 tiles take two chunks, not five (16 and 18.7 us)."""
    api.stub.stub_slots(24)
    ctx = api.context((10, 10, 10), HELFRICH_P, F32, 300)
    api.log()
    assert api.lib.fe_energy_grad_async(ctx, api.field((300, 10, 10), 10), ctypes.c_void_p(8), None) == 0
    assert [b for n, b in api.log() if "grad_sweep" in n] == [2400]


def test_small_blocks_fill_the_chip():
    run(small_blocks)


def test_small_blocks_at_full_occupancy():
    run(full_occupancy)
