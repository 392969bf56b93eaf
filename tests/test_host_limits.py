"""What the allocation-free entry point and saved tuning files accept, and what the
autotuner times."""

import ctypes
import os
import tempfile

from host_stub import ASYM_P, EINVAL, F32, F64, FULL, HELFRICH_P, NO_S, TRACE, TRACE_P, dbl, run


def _noalloc(api, shape, p, dtype):
    u, g = ctypes.c_void_p(4096), ctypes.c_void_p(8192)        # no kernel runs: the fields are never read
    return api.lib.fe_energy_grad_noalloc(ctypes.byref(api.grid(shape, dtype)), dbl([2.0 / shape[2]]), dbl(p), u, g,
                                          dbl([0.0]), None)


def thin_grids(api):
    """Grids with many tile columns and long in z, where the chunks that finish first need
    more partials than the static array holds: taken in longer chunks. 2 to 16 blocks per
    compute unit; 35667, 4462, 2319, 28906 and 31563 columns of 8 x 8 voxels."""
    for slots in (2, 3, 8, 16):
        api.stub.stub_slots(slots)
        for dtype in (F32, F64):
            for p in (TRACE_P, HELFRICH_P, ASYM_P):
                for shape in ((438, 285336, 8), (12256, 35696, 8), (21811, 18552, 8), (2300, 231248, 7),
                              (1485, 252504, 8)):
                    api.log()
                    assert _noalloc(api, shape, p, dtype) == 0, (slots, shape, api.error())
                    blocks = [b for n, b in api.log() if "grad_sweep" in n]
                    assert len(blocks) == 1 and blocks[0] <= 65280, (slots, shape, blocks)
    assert _noalloc(api, (1, 8192, 8192), HELFRICH_P, F32) == EINVAL      # 65536 columns of 32 x 32


def _autotune(api, ctx, shape, kind=1):
    us, cached = ctypes.c_double(), ctypes.c_int()
    u, work = api.field(shape), api.field(shape)
    assert api.lib.fe_autotune(ctx, u, work, kind, 1, ctypes.byref(us), ctypes.byref(cached)) == 0, api.error()
    return cached.value


def saved_choices(api):
    """A record saved before sweeps of a p in k1 + k2 alone had a body of their own serves
    such a context as it did; a record of its own goes first; choices timed in this process
    for another body are not taken."""
    shape = (8, 32, 32)
    path = os.path.join(tempfile.mkdtemp(), "tune.txt").encode()
    record = "32x32x8x1:f32:step:{}:-:stub {} {} 9.0\n"
    variant, z = ctypes.c_int(), ctypes.c_int()

    def launch(ctx):
        assert api.lib.fe_get_launch(ctx, ctypes.byref(variant), ctypes.byref(z)) == 0
        return variant.value, z.value

    for records, want in ((record.format("nos", 2, 4), (2, 4)),
                          (record.format("nos", 2, 4) + record.format("trace", 3, 2), (3, 2))):
        open(path, "w").write(records)
        api.lib.fe_tune_cache_clear()
        assert api.lib.fe_tune_cache_load(path) == 0
        ctx = api.context(shape, TRACE_P)
        assert _autotune(api, ctx, shape) == 1 and launch(ctx) == want
        assert _autotune(api, api.context(shape, HELFRICH_P), shape) == 1
        assert _autotune(api, api.context(shape, ASYM_P), shape) == 0
    api.lib.fe_tune_cache_clear()
    assert _autotune(api, api.context(shape, HELFRICH_P), shape) == 0
    assert _autotune(api, api.context(shape, TRACE_P), shape) == 0
    assert _autotune(api, api.context(shape, TRACE_P), shape) == 1


def tuned_sweeps(api):
    """The tuner times what a loop runs: steps without the energy where a launch shape has
    such a kernel (32 x 32 / 512 threads: the leading one), gradients with it."""
    for p, body in ((TRACE_P, TRACE), (HELFRICH_P, NO_S), (ASYM_P, FULL)):
        for kind in (0, 1, 2):
            ctx = api.context((8, 32, 32), p)
            api.lib.fe_tune_cache_clear()
            api.log()
            assert _autotune(api, ctx, (8, 32, 32), kind) == 0
            lead = [(m, b, e) for m, b, e in api.sweeps() if b == body]
            assert lead and all(s == (kind, body, kind == 0) for s in lead), (kind, body, set(lead))


def test_noalloc_takes_thin_grids():
    run(thin_grids)


def test_saved_choices_serve_the_bodies_they_did():
    run(saved_choices)


def test_the_tuner_times_the_sweeps_that_run():
    run(tuned_sweeps)
