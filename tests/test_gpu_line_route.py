"""Which solver the steps run: line-per-lane solves on every mesh whose lines
have at least 4p + 1 dofs and whose operators decay within the compiled halo, the
direction's own schedule elsewhere and after a call that sets one; and the
steps of the shortest lines of either kind, against the oracle."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2604_19370_amd import iga, inputs
from test_gpu_ensemble import check_vs_oracle, fields, step_input
from test_gpu_line import SHAPES
from test_gpu_parity import TOL32, TOL64, dev, host, per_step_parity, plan_and_oracle, rel, upload

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def routes(pl):
    return pl.line_per_lane(0), pl.line_per_lane(1)


@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_shortest_lines(p, precision):
    """nel = 3p + 1 is the shortest that steps solve one line per lane."""
    short, first, long = 3 * p, 3 * p + 1, 97
    for ex, ey in [(2 * p + 1, 2 * p + 1), (short, long), (long, short), (first, first + 1),
                   (first + 1, long), (long, first)]:
        for scheme in ("strang", "pr"):
            print(f"{scheme} {ex}x{ey} p{p} {precision}", flush=True)
            sc = inputs.small_case(ex + 3 * ey + p, ex, ey, p, scheme)
            pl, od = plan_and_oracle(sc, precision)
            assert routes(pl) == (ex >= first, ey >= first)
            per_step_parity(pl, od, sc, 1, precision)
            pl.close()


@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_tile_edge_shapes_run_line_per_lane(p, precision):
    """The shapes of the tile-edge test, but its smallest mesh."""
    for nx, ny in SHAPES[1:]:
        sc = inputs.small_case(nx + ny + p, nx - p, ny - p, p, "strang")
        pl, _ = plan_and_oracle(sc, precision)
        assert routes(pl) == (True, True), (nx, ny)
        pl.close()


def test_slow_decay_and_set_schedules():
    sc = inputs.small_case(9, 200, 36, 2, "pr", dt=400.0)
    pl, _ = plan_and_oracle(sc, "fp64", coeffs=dict(c_nld=0.0, c_ign=0.0, c_rad=0.0, c_forcing=0.0))
    assert not pl.line_per_lane(0)
    pl.close()
    sc = inputs.small_case(10, 90, 70, 2, "strang")
    pl, _ = plan_and_oracle(sc, "fp32")
    for set_x in (lambda: pl.set_schedule(0, 2, 1), lambda: pl.set_window_schedule(0, 2, 17),
                  lambda: pl.set_column_schedule(16)):
        pl.factor()
        assert routes(pl) == (True, True)
        set_x()
        assert routes(pl) == (False, True)
    pl.close()


def test_autotune_after_a_column_schedule_keeps_line_per_lane():
    """A plan that was set to column waves before it is tuned: the steps run the
    line-per-lane x sweeps that the tuner found faster (84 us a step for 113 at
    this size), and match the oracle."""
    sc = inputs.regional_strang(seed=1, nel=1024, steps=1)
    pl, od = plan_and_oracle(sc, "fp32")
    pl.set_column_schedule(32)
    T, F = dev(sc.T0, True), dev(sc.fuel0, True)
    pl.autotune(T, F, reps=3)
    assert pl.line_per_lane(0)
    per_step_parity(pl, od, sc, 1, "fp32")
    per_step_parity(pl, od, sc, 1, "fp32", step=pl.step_noalloc)
    pl.close()


@pytest.mark.parametrize("nx,ny,precision", [(700, 620, "fp64"), (700, 620, "fp32"), (4096, 1200, "fp32")])
def test_autotune_chooses_the_schedule_beneath(nx, ny, precision):
    """iga_line_solve runs the schedule beneath the steps' line-per-lane solves:
    a poor one that was set (one line of eight wavefronts a workgroup: 24 us an
    x solve at 700^2 for 12) does not outlast the tuner, and whatever
    lies beneath, column waves too, every solve is served and correct (column
    waves that the steps run themselves do not serve which 2 along x)."""
    sc = inputs.small_case(nx + ny, nx, ny, 2, "strang")
    pl, od = plan_and_oracle(sc, precision)
    T, F = dev(sc.T0, pl.fp32), dev(sc.fuel0, pl.fp32)
    for dir in (0, 1):
        pl.set_schedule(dir, 1, 8)
    pl.autotune(T, F, reps=3)
    print(routes(pl), [dict(pl.schedule(d), **pl.solver(d)) for d in (0, 1)], flush=True)
    own_columns = pl.solver(0)["column"] and not pl.line_per_lane(0)
    X = np.random.default_rng(nx).standard_normal((nx + 2, ny + 2))
    for dir in (0, 1):
        s = pl.schedule(dir)
        assert (s["lines"], s["waves_per_line"]) != (1, 8)
        for which in (0, 1, 2):
            if own_columns and (dir, which) == (0, 2):
                continue
            x = dev(X, pl.fp32)
            pl.line_solve(dir, which, x)
            assert rel(host(x), oracle.line_solve(od, dir, which, X)) < (TOL32 if pl.fp32 else TOL64), (dir, which)
    per_step_parity(pl, od, sc, 1, precision)
    pl.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_ensemble_of_both_kinds_of_members(precision):
    """Members whose steps solve one line per lane in both directions, in one, and
    in none: as created and as tuned, every step matches the oracle, and the
    tuner leaves the fields as they are."""
    p = 2
    scs = [inputs.small_case(50 + i, ex, ey, p, scheme) for i, (ex, ey, scheme) in enumerate(
        [(150, 133, "strang"), (6, 90, "strang"), (90, 6, "strang"), (5, 5, "pr"), (130, 70, "explicit"),
         (6, 120, "explicit"), (70, 64, "pr")])]
    for sc in scs:
        pl, _ = plan_and_oracle(sc, precision)
        assert routes(pl) == (sc.nel_x > 3 * p, sc.nel_y > 3 * p)
        pl.close()
    ens = iga.Ensemble.from_scenarios(scs, precision=precision)
    Ts, Fs = fields(ens, scs)
    # two groups of line solves in each sweep, and the middle substep on its own
    assert ens.launches_per_step >= 2 + 8 + 1
    for tuned in (False, True):
        if tuned:
            ens.autotune(Ts, Fs, reps=2)
            for sc, T, F in zip(scs, Ts, Fs):
                assert torch.equal(T, dev(step_input(sc.T0, precision), ens.fp32))
                assert torch.equal(F, dev(step_input(sc.fuel0, precision), ens.fp32))
        for sc, T, F in zip(scs, Ts, Fs):
            upload(T, step_input(sc.T0, precision))
            upload(F, step_input(sc.fuel0, precision))
        ens.step(Ts, Fs)
        for m, sc in enumerate(scs):
            check_vs_oracle(sc, host(Ts[m]), host(Fs[m]), step_input(sc.T0, precision),
                            step_input(sc.fuel0, precision), precision)
            upload(Ts[m], step_input(sc.T0, precision))
            upload(Fs[m], step_input(sc.fuel0, precision))
    ens.close()


def test_ensemble_tuner_takes_no_fields():
    """The ensemble's tuner works on the members' scratch buffers: while it runs,
    the device's free memory does not fall by a member's field (33.6 MB).  The
    second of two calls is watched: the first loads the kernels."""
    scs = [inputs.small_case(60 + i, 2048, 2048, 2, scheme) for i, scheme in enumerate(("strang", "pr"))]
    ens = iga.Ensemble.from_scenarios(scs, precision="fp64")
    Ts, Fs = fields(ens, scs)
    ens.autotune(Ts, Fs, reps=1)
    torch.cuda.synchronize()
    free = [torch.cuda.mem_get_info()[0]]
    with ThreadPoolExecutor(1) as ex:
        call = ex.submit(ens.autotune, Ts, Fs, 1, torch.cuda.current_stream())
        while not call.done():
            free.append(torch.cuda.mem_get_info()[0])
        call.result()
    print(f"{len(free) - 1} readings, free memory fell by {(free[0] - min(free)) / 1e6:.1f} MB", flush=True)
    assert len(free) > 10 and free[0] - min(free) < 8 * Ts[0].numel()
    ens.close()
