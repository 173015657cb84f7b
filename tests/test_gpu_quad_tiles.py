"""Four-cells-per-thread kernels on rows of at most 8, 16 and 32 lanes, where
a wave covers several rows: rows that end inside a tile's lanes, tiles that end
past the last row, solids, 3D and 2D, on grids too large for several sweeps to
a launch.  Three forced preconditioned iterations against the oracle (FP64,
1e-10: the sums differ in order only), and fewer tiles per launch than the
default (the tuner's choice) against the default within the same bound."""
import numpy as np
import pytest

from paper_2603_21869_amd import cases as C
from tests.parity import fluid
from tests.test_gpu_bottom import _case

pytestmark = pytest.mark.gpu

SHAPES = [((32, 64, 72), 4), ((24, 88, 64), 4), ((64, 40, 56), 4), ((56, 72, 40), 4),
          ((128, 40, 32), 4), ((96, 40, 40), 4), ((64, 2112, 1), 6), ((128, 1056, 1), 6)]


@pytest.mark.parametrize("solids", [False, True], ids=["open", "solids"])
@pytest.mark.parametrize("n,levels", SHAPES, ids=["x".join(map(str, s[0])) for s in SHAPES])
def test_short_rows(oracle, n, levels, solids):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm as nf
    case = _case(n, levels, (2, 2, 0), C.PREC_FP64, solids)
    m = fluid(case)
    b = np.random.default_rng(9).standard_normal((n[2], n[1], n[0])) * m
    ref = oracle.MG(case).solve(b, forced=3)[0]
    for tuned in (1.0, 0.0):
        g = nf.Grid(case)
        nf.nfvm_set_option(g.h, nf.NFVM_OPT_AUTOTUNE, tuned)
        x = g.mg_solve(b, tol=1e-30, max_cycles=3, forced_cycles=3, allow=(0, -5))[0]
        g.close()
        err = np.abs(x - ref)[m].max() / np.abs(ref[m]).max()
        print(f"[short rows] {n} tuned={tuned} err={err:.2e}", flush=True)
        assert err <= 1e-10
