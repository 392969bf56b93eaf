"""Pinned host memory for the energies that calls return, shared by the contexts of a
process in a slab of 64 units of 64 doubles: the slab full and past full, units given
back from the middle, requests around a unit's and the slab's ends, and none left."""

import ctypes

from host_stub import dbl, run

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


def test_more_contexts_than_the_slab_holds():
    run(full_slab)


def test_no_pinned_memory():
    run(none_left)
