"""Launch settings that are set back: the grid's own choice among the passes
is back with them."""
import pytest
import torch

pytestmark = pytest.mark.gpu

RUNS = ("steps", "series", "source", "source_series", "cotangents", "spin_tangent")


def _grid(gpu, nr, nth):
    return gpu.TeukGrid(0.5, -2, 2, nr, nth, -50.0, 150.0, 0.001, extract_rstar=[12.0], extract_theta=[1.0])


def _passes(g):
    return [g.get_pass(r) for r in RUNS]


def test_block_launch_off_again(gpu):
    """A grid whose default is no block pass, after one was set and turned off."""
    g = _grid(gpu, 6400, 64)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert g.block_launch() == (0, 0) and g.get_pass("steps")["kind"] == "tile"
    elif g.block_steps():
        pytest.skip("this device's default has a block pass")
    tile, before = g.tile(), _passes(g)
    g.set_block_launch(2, 16)
    assert g.get_pass("steps")["kind"] == "block"
    g.set_block_launch(0)
    assert g.get_pass("steps")["kind"] == "sweep"
    g.set_tile(*tile)
    assert _passes(g) == before
    g.close()


def test_block_launch_default_again(gpu):
    """A grid whose default is the block pass: off leaves the sweeps, also with
    the default tile; the default launch brings the choice back."""
    g = _grid(gpu, 400, 32)
    if not g.block_steps():
        pytest.skip("this device's default has no block pass")
    tile, block, before = g.tile(), g.block_launch(), _passes(g)
    g.set_block_launch(0)
    g.set_tile(*tile)
    assert g.get_pass("steps")["kind"] == "sweep"
    g.set_block_launch(*block)
    assert _passes(g) == before
    g.close()


@pytest.mark.parametrize("nr,nth", [(1600, 64), (6400, 256)])
def test_adjoint_tile_set_as_it_was(gpu, nr, nth):
    """The adjoint tile set to the values that the getter returned, and back to
    them after others: the kernels' own heights and the tile pass."""
    g = _grid(gpu, nr, nth)
    tile, before = g.adjoint_tile(), _passes(g)
    g.set_adjoint_tile(*tile)
    assert _passes(g) == before
    g.set_adjoint_tile(7, 2)
    p = g.get_pass("cotangents")
    assert (p["kind"], p["rows"], p["waves"]) == ("sweep", 7, 2)
    assert g.get_pass("spin_tangent")["rows"] == 7
    g.set_adjoint_tile(*tile)
    assert _passes(g) == before
    g.close()


def test_user_coefficients_with_a_source(gpu):
    """Both at once: single steps on small grids, where pairs wait for the
    coefficients on every row; pairs on large ones and without a source."""
    for nr, nth, steps in ((800, 48, 1), (6400, 256, 2)):
        g = gpu.TeukGrid(0.5, -2, 2, nr, nth, -50.0, 150.0, 0.001, coef_mode=gpu.TEUK_COEF_USER)
        assert g.get_pass("source")["steps"] == steps and g.get_pass("steps")["steps"] == 2
        g.close()
