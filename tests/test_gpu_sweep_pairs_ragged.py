"""Two level-0 sweeps per pass on grids large enough to take them whose last
tile of eight rows is partly past the box (260 rows, and fluid up to the last
one across a tile edge along x; all else solid, so that three levels suffice),
and in 2D: bitwise the solution of single sweeps."""
import numpy as np
import pytest

from paper_2603_21869_amd import cases as C

pytestmark = pytest.mark.gpu


def _rows260(prec):
    n = (512, 260, 128)
    c = C.channel3d(*n, Lx=10.24, Ly=5.2, Lz=2.56, n_levels=3, precision=prec)
    s = np.ones((n[2], n[1], n[0]), np.uint8)
    s[52:64, 240:260, 384:512] = 0  # (to the outlet; 480 cells of the coarsest level)
    c.solid = s
    return c


def _plane(prec):
    return C.channel2d(8448, 2048, L=264.0, H=64.0, n_levels=9, precision=prec)


@pytest.mark.parametrize("prec", [C.PREC_FP64, C.PREC_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("make", [_rows260, _plane], ids=["512x260x128", "8448x2048"])
def test_pairs_equal_single_sweeps(make, prec):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm as nf
    case = make(prec).copy(nu1=3, nu2=3)
    b = np.random.default_rng(6).standard_normal((case.n[2], case.n[1], case.n[0]))
    if case.solid is not None:
        b *= case.solid == 0
    out = []
    for pairs in (0.0, 1.0):
        g = nf.Grid(case)
        nf.nfvm_set_option(g.h, nf.NFVM_OPT_AUTOTUNE, 0.0)
        nf.nfvm_set_option(g.h, nf.NFVM_OPT_SWEEP_PAIRS, pairs)
        nf.nfvm_profile(g.h, 1 << nf.KERNELS.index("smooth0_pair"))
        out.append(g.mg_solve(b, tol=1e-30, max_cycles=3, forced_cycles=3, allow=(0, -5))[0])
        used = nf.nfvm_profile_read(g.h, nf.KERNELS.index("smooth0_pair"))["launches"]
        g.close()
        print(f"[pairs] {case.n} pairs={pairs} passes={used}", flush=True)
        assert (used > 0) == (pairs == 1.0)
    assert np.isfinite(out[0]).all() and np.abs(out[0]).max() > 0
    assert np.array_equal(out[0], out[1])
