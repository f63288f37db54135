"""Steps on their default line solves, one line per lane (64 lines and a tile of
rows per workgroup, twisted elimination): meshes whose lines end at and beside
tile edges, shorter than a tile, of the smallest size and with interior tiles,
more and fewer lines than a workgroup's 64; and beside the windowed solves in
the other direction, where Strang's fields change places.  Against the oracle."""
import pytest

from paper_2604_19370_amd import inputs
from test_gpu_parity import per_step_parity, plan_and_oracle

pytestmark = pytest.mark.gpu

# tiles hold 48 (double, p = 2), 64 or 96 (double, p = 3) rows; Nx = nel_x + p
SHAPES = [(0, 0), (64, 48), (96, 129), (193, 65), (520, 70), (70, 520)]


@pytest.mark.parametrize("p", [1, 2, 3])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_steps_at_tile_edges(p, precision, nx, ny):
    """Nx, Ny as given (the first: the smallest mesh)."""
    for scheme in ("strang", "pr"):
        ex, ey = (nx - p, ny - p) if nx else (2 * p + 1, 2 * p + 1)
        print(f"{scheme} {ex}x{ey} p{p} {precision}", flush=True)
        sc = inputs.small_case(nx + ny + p, ex, ey, p, scheme)
        pl, od = plan_and_oracle(sc, precision)
        per_step_parity(pl, od, sc, 1, precision)
        pl.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("dir", [0, 1])
def test_strang_with_windowed_solves_in_one_direction(precision, dir):
    sc = inputs.small_case(31, 150, 133, 2, "strang")
    pl, od = plan_and_oracle(sc, precision)
    pl.set_window_schedule(dir, 2, 17)
    per_step_parity(pl, od, sc, 2, precision, step=pl.step_noalloc)
    pl.close()
