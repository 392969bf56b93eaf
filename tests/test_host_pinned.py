"""Pinned host memory for the energies that calls return, shared by the contexts of a
process in a slab of 64 units of 64 doubles: the slab full and past full, units given
back from the middle, requests around a unit's and the slab's ends, and none left."""

import ctypes

from host_stub import F64, HELFRICH_P, dbl, run

SHAPE = (4, 8, 8)


def _energy(api, ctx, batch, first):
    """fe_energy on ctx, whose energies the stub's kernel writes as first, first + 1, ..."""
    api.stub.stub_next(first)
    out = dbl([0.0] * batch)
    assert api.lib.fe_energy(ctx, api.field((batch,) + SHAPE[1:], SHAPE[0]), out) == 0, api.error()
    assert list(out) == [first + b for b in range(batch)]
    return api.stub.stub_energy()


def _disjoint(held):
    spans = sorted((at, at + 8 * batch) for _, batch, at in held)
    assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))


def full_slab(api):
    held = []

    def take(batch):
        ctx = api.context(SHAPE, batch=batch)
        held.append((ctx, batch, _energy(api, ctx, batch, 1000.0 * len(held))))

    def give(i):
        api.lib.fe_destroy(held.pop(i)[0])

    for _ in range(64):
        take(1)
    assert api.stub.stub_host_allocs() == 1          # one slab
    for batch in (1, 1, 64, 65):                     # past it: memory of their own
        take(batch)
    assert api.stub.stub_host_allocs() == 5
    _disjoint(held)
    for i in (40, 30, 29, 28, 10):                   # holes of one and three units
        give(i)
    take(129)                                        # three units, in the hole that holds them
    take(65)                                         # two: no such hole left
    take(64)
    take(2)
    assert api.stub.stub_host_allocs() == 6
    _disjoint(held)
    for k, (ctx, batch, at) in enumerate(held):      # everyone keeps their place
        assert _energy(api, ctx, batch, 7.0 * k) == at
    while held:
        give(len(held) // 2)
    assert api.stub.stub_host_live() == 0            # the slab went back with its last unit
    for batch in (4032, 4096, 4097, 1):              # 63 units, the whole slab, more, one
        take(batch)
    _disjoint(held)
    while held:
        give(0)
    assert api.stub.stub_host_live() == 0


def none_left(api):
    api.stub.stub_host_full(1)
    ctx = api.context(SHAPE, batch=3)
    at = _energy(api, ctx, 3, 5.0)                   # the device slot and a copy
    api.stub.stub_host_full(0)
    assert api.stub.stub_host_live() == 0
    assert _energy(api, ctx, 3, 6.0) != at           # pinned memory once there is some
    api.lib.fe_destroy(ctx)
    assert api.stub.stub_host_live() == 0


def flow_with_none_left(api):
    shape = (6, 8, 10)
    logs = []
    for full in (0, 1):
        api.stub.stub_host_full(full)
        L = ctypes.c_void_p()
        rc = api.lib.fe_l2_create(ctypes.byref(api.grid(shape, F64)), ctypes.c_double(0.2), dbl(HELFRICH_P),
                                  ctypes.c_double(1.0), None, ctypes.byref(L))
        assert rc == 0, api.error()
        u, E = api.field(shape), dbl([0.0])
        for first in (3.0, 4.0):
            api.stub.stub_next(first)
            assert api.lib.fe_l2_energy_grad(L, u, api.field(shape), E) == 0 and E[0] == first
        api.log()
        Es = dbl([0.0] * 2)
        assert api.lib.fe_l2_step(L, 2, Es) == 0 and list(Es) == [4.0, 4.0]
        logs.append(api.log())
        api.lib.fe_l2_destroy(L)
        assert api.stub.stub_host_live() == 0
    assert logs[0] == logs[1] and len(logs[0]) > 4    # the same iterations either way


def test_more_contexts_than_the_slab_holds():
    run(full_slab)


def test_no_pinned_memory():
    run(none_left)


def test_flow_without_pinned_memory():
    run(flow_with_none_left)
