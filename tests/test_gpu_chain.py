"""Levels whose sweeps and transfers run several to a launch: boxes that end
inside the grid, every count of sweeps per launch, 2D and 3D, solids, one and
several coarse levels.  Three forced preconditioned iterations with the LDS
bottom solver off against the oracle (FP64, 1e-10 as for the single launches),
and batches in which a level is swept several to a launch in one grid and by
single launches in another or alone (bitwise equal, as every batch)."""
import numpy as np
import pytest

from paper_2603_21869_amd import cases as C
from tests.parity import fluid
from tests.test_gpu_bottom import _case

pytestmark = pytest.mark.gpu

# cells, levels, pre / post / coarse sweeps
SHAPES = [((8, 4, 4), 2, (2, 2, 0)), ((36, 28, 20), 3, (2, 2, 0)), ((64, 32, 32), 5, (3, 3, 6)),
          ((20, 44, 36), 3, (1, 1, 1)), ((100, 12, 8), 3, (4, 5, 0)), ((24, 40, 24), 4, (5, 7, 8)),
          ((128, 64, 16), 4, (1, 3, 2)), ((64, 64, 32), 4, (2, 1, 0)), ((52, 36, 1), 3, (2, 2, 0)),
          ((320, 192, 1), 5, (3, 3, 6)), ((6, 334, 1), 2, (6, 4, 0)), ((512, 256, 1), 5, (1, 2, 5))]


@pytest.mark.parametrize("solids", [False, True], ids=["open", "solids"])
@pytest.mark.parametrize("n,levels,nu", SHAPES,
                         ids=["x".join(map(str, s[0])) + f"-L{s[1]}-{s[2]}" for s in SHAPES])
def test_chain_shapes(oracle, n, levels, nu, solids):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm as nf
    case = _case(n, levels, nu, C.PREC_FP64, solids)
    m = fluid(case)
    b = np.random.default_rng(8).standard_normal((n[2], n[1], n[0])) * m
    g = nf.Grid(case)
    nf.nfvm_set_option(g.h, nf.NFVM_OPT_BOTTOM, 0.0)
    x, st, _ = g.mg_solve(b, tol=1e-30, max_cycles=3, forced_cycles=3, allow=(0, -5))
    g.close()
    ref = oracle.MG(case).solve(b, forced=3)[0]
    err = np.abs(x - ref)[m].max() / np.abs(ref[m]).max()
    print(f"[chain] {n} L={levels} nu={nu} err={err:.2e}", flush=True)
    assert err <= 1e-10


@pytest.mark.parametrize("prec", [C.PREC_FP64, C.PREC_MIXED], ids=["fp64", "mixed"])
def test_chain_in_batches(prec):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm as nf
    ns = [(128, 64, 64)] * 5 + [(64, 64, 32), (36, 20, 28)]  # (level 1: 5 x 65536 cells, ...)
    cases = [C.serve_case(dict(n=n, geometry=("channel", "room")[i % 2], seed=30 + i, n_steps=2),
                          prec, 1e-6).copy(n_steps=2) for i, n in enumerate(ns)]
    cases[1] = cases[1].copy(nu1=3, nu2=3, nu_coarse=5)
    ref = []
    for c in cases:
        g = nf.Grid(c)
        _, st = g.step(2)
        ref.append((st, g.fields()))
        g.close()
    grids = [nf.Grid(c) for c in cases]
    _, _, stats = nf.nfvm_step_batch([g.h for g in grids], 2)
    for i, (g, (st, f)) in enumerate(zip(grids, ref)):
        print(f"[chain] batch {ns[i]} cycles {[q['cycles'] for q in st]}", flush=True)
        assert [q["cycles"] for q in stats[i]] == [q["cycles"] for q in st], ns[i]
        h = g.fields()
        for k in f:
            assert np.array_equal(f[k], h[k]), (ns[i], k)
        g.close()
