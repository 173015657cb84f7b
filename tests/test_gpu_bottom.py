"""The LDS bottom solver at the shapes where its parts begin and end: a top
level of at most 64 cells (one wave), of one to five cells per thread, swept
levels below it, a coarsest level inside one wave and a larger one, 2D and 3D,
solids, no pre- or no post-smoothing.  Three forced preconditioned iterations
against the oracle (FP64, 1e-10: the two sum the dense solve's terms in
different orders) and, in FP32, against the per-level kernels (1e-4 of the
largest value: a few hundred roundings of 6e-8 amplified by the coarse solve)."""
import numpy as np
import pytest

from paper_2603_21869_amd import cases as C
from tests.parity import fluid

pytestmark = pytest.mark.gpu

# cells, levels, pre / post / coarse sweeps
SHAPES = [((8, 8, 8), 3, (2, 2, 0)), ((32, 16, 8), 4, (2, 2, 0)), ((40, 24, 20), 3, (2, 2, 0)),
          ((32, 32, 32), 5, (3, 3, 6)), ((32, 32, 32), 4, (0, 2, 0)), ((52, 28, 20), 3, (1, 1, 3)),
          ((24, 24, 24), 4, (2, 0, 0)), ((64, 48, 1), 5, (2, 2, 0)), ((160, 112, 1), 4, (2, 2, 0)),
          ((44, 60, 1), 3, (1, 2, 4)), ((16, 256, 4), 3, (2, 1, 0)), ((64, 64, 64), 6, (2, 2, 2))]


def _case(n, levels, nu, prec, solids):
    nx, ny, nz = n
    if nz == 1:
        c = C.channel2d(nx, ny, L=nx / 32.0, H=ny / 32.0, n_levels=levels, precision=prec)
    else:
        c = C.channel3d(nx, ny, nz, Lx=0.02 * nx, Ly=0.02 * ny, Lz=0.02 * nz, n_levels=levels,
                        precision=prec)
    if solids:
        s = np.zeros((nz, ny, nx), np.uint8)
        s[nz // 4: nz // 2 + 1, ny // 3: ny // 2 + 1, nx // 2: nx // 2 + 5] = 1
        s[-2:, : ny // 3, 1:4] = 1
        c.solid = s
    return c.copy(nu1=nu[0], nu2=nu[1], nu_coarse=nu[2])


@pytest.mark.parametrize("solids", [False, True], ids=["open", "solids"])
@pytest.mark.parametrize("n,levels,nu", SHAPES,
                         ids=["x".join(map(str, s[0])) + f"-L{s[1]}-{s[2]}" for s in SHAPES])
def test_bottom_solver_shapes(oracle, n, levels, nu, solids):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm as nf
    case = _case(n, levels, nu, C.PREC_FP64, solids)
    m = fluid(case)
    b = np.random.default_rng(7).standard_normal((n[2], n[1], n[0])) * m
    g = nf.Grid(case)
    x, st, _ = g.mg_solve(b, tol=1e-30, max_cycles=3, forced_cycles=3, allow=(0, -5))
    g.close()
    ref = oracle.MG(case).solve(b, forced=3)[0]
    err = np.abs(x - ref)[m].max() / np.abs(ref[m]).max()
    print(f"[bottom] {n} L={levels} nu={nu} fp64 err={err:.2e}", flush=True)
    assert err <= 1e-10
    out = []
    for bottom in (1.0, 0.0):
        g = nf.Grid(case.copy(precision=C.PREC_FP32))
        nf.nfvm_set_option(g.h, nf.NFVM_OPT_BOTTOM, bottom)
        out.append(g.mg_solve(b, tol=1e-30, max_cycles=3, forced_cycles=3, allow=(0, -5))[0])
        g.close()
    err = np.abs(out[0] - out[1])[m].max() / np.abs(out[1][m]).max()
    print(f"[bottom] {n} fp32 on/off err={err:.2e}", flush=True)
    assert err <= 1e-4
