"""Captured loops after the context's parameters, launch or fields change: a loop replays
the sweeps that its present parameters take, never those of an earlier call."""

import ctypes

from host_stub import ASYM_P, F32, F64, FULL, HELFRICH_P, NO_S, TRACE, TRACE_P, dbl, run

SHAPE = (20, 40, 44)


def _flow(api, ctx, A, nsteps):
    out = dbl([0.0])
    d = ctypes.c_double
    rc = api.lib.fe_hminus_step(ctx, A, dbl([0.1]), d(1.0), d(1e-3), d(0.9), d(0.999), d(1e-8), nsteps, None, out)
    assert rc == 0, api.error()


def _steps(api, ctx, u, nsteps):
    assert api.lib.fe_step(ctx, u, dbl([0.1]), ctypes.c_double(1e-3), nsteps, dbl([0.0])) == 0, api.error()


def _partials(log):
    """Blocks of the last sweep of a log, whose partials its finish adds."""
    return [blocks for name, blocks in log if "grad_sweep" in name][-1]


def flow(api):
    for dtype in (F32, F64):
        ctx = api.context(SHAPE, TRACE_P, dtype)
        A = api.field(SHAPE, 3)
        for nsteps in (8, 19, 3):
            for p, body in ((TRACE_P, TRACE), (HELFRICH_P, NO_S), (ASYM_P, FULL), (HELFRICH_P, NO_S), (TRACE_P, TRACE)):
                api.set_params(ctx, SHAPE, p)
                api.log()
                _flow(api, ctx, A, nsteps)
                sweeps = api.sweeps()
                assert [b for _, b, _ in sweeps] == [body] * nsteps, (nsteps, body, sweeps)
                assert sweeps[-1][2]                  # the energy that the call returns
                fresh = api.context(SHAPE, p, dtype)  # in the same z chunks as a context that never had another p
                _flow(api, fresh, A, nsteps)
                want = _partials(api.log())
                _flow(api, ctx, A, nsteps)
                assert _partials(api.log()) == want
                api.lib.fe_destroy(fresh)
        api.lib.fe_destroy(ctx)


def steps(api):
    ctx = api.context(SHAPE, TRACE_P)
    u = api.field(SHAPE)
    for nsteps in (17, 34, 5):
        for p, body in ((TRACE_P, TRACE), (HELFRICH_P, NO_S), (ASYM_P, FULL), (TRACE_P, TRACE)):
            api.set_params(ctx, SHAPE, p)
            api.log()
            _steps(api, ctx, u, nsteps)
            sweeps = api.sweeps()
            assert [b for _, b, _ in sweeps] == [body] * nsteps
            assert sweeps[-1][2]


def test_flow_replays_the_present_body():
    run(flow)


def test_steps_replay_the_present_body():
    run(steps)
