"""Two level-0 sweeps per pass on grids large enough to take them: bitwise the
solution of single sweeps, with rows that end inside a tile of 62 four-cell
columns and tile rows and planes that end inside the box."""
import numpy as np
import pytest

from paper_2603_21869_amd import cases as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [C.PREC_FP64, C.PREC_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n,nu", [((576, 256, 128), (3, 3)), ((320, 448, 128), (3, 2))],
                         ids=["576x256x128", "320x448x128"])
def test_pairs_equal_single_sweeps(n, nu, prec):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm as nf
    case = C.serve_case(dict(n=n, geometry="room", seed=6, n_steps=1), prec, 1e-6)
    case = case.copy(nu1=nu[0], nu2=nu[1], nu_coarse=3)
    b = np.random.default_rng(5).standard_normal((n[2], n[1], n[0]))
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
        assert (used > 0) == (pairs == 1.0)
    assert np.array_equal(out[0], out[1])
