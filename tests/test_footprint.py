"""nfvm_grid_footprint counts every buffer that a grid's set-up allocates (CPU:
the model is host code): the fields, the hierarchy, the solver's vectors and the
LDS bottom solver's constants, summed here from their own sizes for an MI355X
(160 KB of LDS per workgroup)."""
import os

import pytest

from paper_2603_21869_amd import cases as C

# bytes of a velocity, scalar, pressure, outer-solve value, of a level-0 and a
# coarse iterate, and of the V-cycle's arithmetic
SIZES = {C.PREC_FP64: (8, 8, 8, 8, 8, 8, 8), C.PREC_FP32: (4, 4, 4, 4, 4, 4, 4),
         C.PREC_MIXED: (8, 4, 8, 8, 4, 2, 4)}
COARSE_MAX, MAX_PATCHES = 512, 128


def _padded(n, dim):
    sx = (n[0] + 2 + 15) // 16 * 16
    return 32 + (n[2] + 2 * (dim == 3)) * sx * (n[1] + 2)


def _bottom_bytes(levels, dim, c):
    """The constants of the levels that fit one workgroup's LDS: per cell of the
    top one four words of indices, six coefficients and a factor; below it the
    coefficients, on swept levels also indices and factor; the coarsest cells'
    indices and, with at most 64 of them, their inverse."""
    used, top = 4 * COARSE_MAX, len(levels)
    for l in range(len(levels) - 1, 0, -1):
        nx, ny, nz = levels[l]
        cells = nx * ny * nz
        faces = (nx + 1) * ny * nz + nx * (ny + 1) * nz + (dim == 3) * nx * ny * (nz + 1)
        need = 4 * cells * c + 4 * faces + cells
        if used + need > 160 * 1024 - 4096:  # (less static LDS and rounding)
            break
        used, top = used + need, l
    if top > len(levels) - 2:
        return 0
    cells = [x * y * z for x, y, z in levels[top:]]
    total = cells[0] * (16 + 24 + c)
    total += sum(n * (24 + 16 + c) for n in cells[1:-1]) + cells[-1] * 24
    return total + 4 * cells[-1] + (cells[-1] ** 2 * c if cells[-1] <= 64 else 0)


def _buffers(case, prec):
    V, F, P, O, S0, SC, c = SIZES[prec]
    n, dim = case.n, case.dim
    levels = [(n[0] >> l, n[1] >> l, n[2] >> l if dim == 3 else 1) for l in range(case.n_levels)]
    T, N = _padded(n, dim), n[0] * n[1] * n[2]
    b = T * (6 * V + 7 * F + P + 1) + 8 * N
    b += T * (4 * O + 2 * S0)
    for l, m in enumerate(levels):
        wide = l == 0 or (prec == C.PREC_MIXED and m[0] * m[1] * m[2] >= 131072)
        b += _padded(m, dim) * (1 + 4 * dim + 3 * (S0 if wide else SC) + (2 if l == 0 else 1))
    b += 2 * COARSE_MAX ** 2 * 8 + 4 * COARSE_MAX + MAX_PATCHES * 80
    return b + _bottom_bytes(levels, dim, c)


@pytest.mark.parametrize("prec", sorted(SIZES), ids=["fp64", "fp32", "mixed"])
@pytest.mark.parametrize("n,levels", [((64, 64, 64), 6), ((64, 64, 64), 4), ((256, 128, 64), 7),
                                      ((48, 48, 40), 4), ((64, 16, 16), 3), ((192, 96, 1), 5),
                                      ((1024, 64, 1), 6), ((8, 8, 8), 2)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_footprint_counts_every_buffer(n, levels, prec):
    from paper_2603_21869_amd import nfvm
    if not os.path.exists(nfvm.LIB_PATH):
        pytest.skip("libnfvm.so not built")
    if n[2] == 1:
        case = C.channel2d(n[0], n[1], n_levels=levels, precision=prec)
    else:
        case = C.channel3d(*n, n_levels=levels, precision=prec)
    fp, own = nfvm.nfvm_grid_footprint(nfvm.Desc(case)), _buffers(case, prec)
    assert own <= fp <= own + (1 << 20) + own // 10, (fp, own)
