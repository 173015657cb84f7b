"""The reverse modes of the explicit stage and of the destruction step at the
edges of their tiles: 60 columns by 6 (explicit) or 10 (destruction) rows, and
chunks of planes; grids one cell below, at and above them, single rows and
planes, 2D, and solids across tile edges, with NaN in the solid cells (their
values are never read).  Bar as for the whole-grid comparison: 1e-10 of the
largest value of the autodiff oracle (FP64 rounding of sums of a few dozen
terms, amplified by at most the cancellation between a cell's faces)."""
import numpy as np
import pytest

from paper_2603_21869_amd import cases as C

pytestmark = pytest.mark.gpu

# (cells, levels: the coarsest level holds at most 512 cells)
SHAPES = [((59, 8, 1), 1), ((61, 7, 1), 1), ((121, 4, 1), 1), ((180, 10, 1), 2), ((61, 4, 2), 1),
          ((121, 2, 2), 1), ((4, 11, 11), 1), ((7, 7, 10), 1), ((2, 2, 2), 1), ((58, 6, 6), 2),
          ((60, 10, 4), 2), ((62, 12, 4), 2), ((60, 8, 8), 2), ((120, 8, 4), 2),
          ((8, 22, 20), 2), ((122, 14, 2), 2), ((8, 4, 64), 2), ((128, 40, 24), 4)]


def _case(n, levels, solids):
    nx, ny, nz = n
    if nz == 1:
        return C.channel2d(nx, ny, L=4.0, H=1.0, n_levels=levels)
    c = C.channel3d(nx, ny, nz, Lx=0.02 * nx, Ly=0.02 * ny, Lz=0.02 * nz, n_levels=levels)
    if solids:
        s = np.zeros((nz, ny, nx), np.uint8)
        s[:, ny // 2, nx // 3: nx // 2 + 1] = 1  # a wall through the planes
        s[nz // 2, : ny // 2 + 1, max(0, nx - 4): nx - 2] = 1
        c.solid, c.T_solid = s, 300.0
    return c


@pytest.mark.parametrize("n,levels", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
@pytest.mark.parametrize("kind", ["explicit", "destroy"])
def test_reverse_mode_at_tile_edges(kind, n, levels):
    import torch
    from oracle import autodiff as AD
    from paper_2603_21869_amd import nfvm as nf
    solids = n[2] > 2
    case = _case(n, levels, solids)
    rng = np.random.default_rng(sum(n))
    sh = (n[2], n[1], n[0])
    f = {k: np.array(v, dtype=np.float64) for k, v in case.fields.items()}
    for a, nm in enumerate(("u", "v", "w")):
        f[nm] = f[nm] + 0.05 * rng.standard_normal(sh) * (a < case.dim)
    f["p"] = 0.05 * rng.standard_normal(sh)
    f["T"] = f["T"] + 2.0 * rng.standard_normal(sh)
    f["k"] = f["k"] * (1.0 + 0.5 * rng.random(sh)) + 1e-4
    f["omega"] = f["omega"] * (1.0 + 0.5 * rng.random(sh)) + 1.0
    bar = {nm: rng.standard_normal(sh) for nm in ("u", "v", "w", "T", "k", "omega")}
    tau = 10.0 * case.dt
    if kind == "explicit":
        ref = AD.explicit_vjp(case, f, bar)
    else:
        ref = AD.destroy_vjp(case, f, tau, bar["k"], bar["omega"])
    if solids:
        for nm in f:
            f[nm] = np.where(case.solid != 0, np.nan, f[nm])
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    st, yb = {k: dev(v) for k, v in f.items()}, {k: dev(v) for k, v in bar.items()}
    out = {nm: torch.full(sh, float("nan"), dtype=torch.float64, device="cuda") for nm in ref}
    ptr = lambda d: {k: v.data_ptr() for k, v in d.items()}
    g = nf.Grid(case)
    torch.cuda.synchronize()
    if kind == "explicit":
        nf.nfvm_explicit_adjoint_device(g.h, ptr(st), ptr(yb), ptr(out))
    else:
        nf.nfvm_destroy_adjoint_device(g.h, ptr(st), tau, yb["k"].data_ptr(),
                                       yb["omega"].data_ptr(), ptr(out))
    torch.cuda.synchronize()
    g.close()
    for nm in ref:
        got = out[nm].cpu().numpy()
        scale = max(np.abs(ref[nm]).max(), 1e-300)
        err = np.abs(got - ref[nm]).max() / scale
        print(f"[{kind}] {n} {nm} err={err:.2e}", flush=True)
        assert np.isfinite(got).all() and err <= 1e-10, (nm, err)

