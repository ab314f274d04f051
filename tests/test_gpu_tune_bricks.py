"""The stencil tuner on grids whose untuned passes run bricks: the brick kernel is
timed as the untuned configuration, also past a shape set by hand for every
family; where it stays the result says so, the family has no entry, and the
hand-set shape remains the other family's; what is reported is what runs."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

SHAPE, H = (24, 30, 26), (0.4, 0.45, 0.5)         # bricks win by far: the march has 2 tiles
HAND = (3, 0)                                     # 64x16/512


def _table(tmp_path):
    path = tmp_path / "table.txt"
    ofd.tune_save(path)
    rows = [tuple(int(v) for v in ln.split()) for ln in path.read_text().splitlines() if not ln.startswith("#")]
    nz, ny, nx = SHAPE
    return {r[0]: r[5:] for r in rows if r[1:5] == (nx, ny, nz, 8)}


def _iterate():
    """A CG iterate: its rounding follows the passes' reduction order."""
    g = np.random.default_rng(71).normal(size=SHAPE)
    s = ofd.PoissonSolver(SHAPE, H)
    x = to_dev(np.zeros(SHAPE))
    s.solve(to_dev(g), x, 1e-300, 12, allow_not_converged=True)
    s.close()
    return to_host(x)


@pytest.mark.parametrize("hand", [False, True])
@pytest.mark.parametrize("family", [ofd.TUNE_APPLY, ofd.TUNE_PASS])
def test_bricks_stay(family, hand, tmp_path):
    torch_cuda()
    announce("tune bricks", family, hand)
    try:
        ofd.set_stencil_config(SHAPE, 8, -1)
        bricks = _iterate()
        ofd.set_stencil_config(SHAPE, 8, *HAND)
        march = _iterate()
        assert not np.array_equal(bricks, march)
        if not hand:
            ofd.set_stencil_config(SHAPE, 8, -1)
        r = ofd.tune_stencil(SHAPE, H, ofd.F64, family, reps=20)
        assert r["group"] == 1 and r["shape_name"] == "bricks/1"
        assert 0 <= r["shape"] < 6 and r["best_ms"] == r["default_ms"]
        assert _table(tmp_path) == ({1 - family: HAND} if hand else {})
        runs_bricks = family == ofd.TUNE_PASS or not hand
        assert np.array_equal(_iterate(), bricks if runs_bricks else march)
        # both families tuned: nothing of the hand-set shape is left
        ofd.tune_stencil(SHAPE, H, ofd.F64, 1 - family, reps=20)
        assert _table(tmp_path) == {}
        assert np.array_equal(_iterate(), bricks)
    finally:
        ofd.set_stencil_config(SHAPE, 8, -1)


def test_march_is_named():
    torch_cuda()
    shape = (128, 160, 256)                       # over the limit of bricks
    announce("tune march", shape)
    try:
        r = ofd.tune_stencil(shape, H, ofd.F64, ofd.TUNE_APPLY, reps=3)
        assert r["group"] == 0 and r["shape_name"] == ofd.SHAPE_NAMES[r["shape"]]
    finally:
        ofd.set_stencil_config(shape, 8, -1)
