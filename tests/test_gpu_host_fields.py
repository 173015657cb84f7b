"""Fields loaded and read back through the chunked transfers: below their
threshold, with a last chunk of a few values, arrays shorter and longer than a
chunk and than the ring.  What a grid returns is bitwise what it returns into
pinned arrays (the runtime's own copy), and u, v, w, k, omega and p of an FP64
grid without fixed cells come back as loaded; one array given for several
results holds the last; two threads at once; a served request's fields."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2603_21869_amd import cases as C

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nf():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2603_21869_amd import nfvm
    nfvm.lib()
    return nfvm


def _grid(nf, n, prec=C.PREC_FP64):
    c = C.channel3d(*n, Lx=0.01 * n[0], Ly=0.01 * n[1], Lz=0.01 * n[2], precision=prec,
                    n_levels=C.max_levels(n, 3))
    g = nf.Grid(c)
    nf.nfvm_set_option(g.h, nf.NFVM_OPT_AUTOTUNE, 0.0)
    return g


def _fields(nf, shape, seed):
    r = np.random.default_rng(seed)
    f = {k: r.standard_normal(shape) for k in nf.FIELD_ORDER}
    for k in ("k", "omega"):
        f[k] = 1.0 + np.abs(f[k])
    f["T"] += 293.0
    return f


def _pinned(shape):
    import torch
    return torch.zeros(shape, dtype=torch.float64, pin_memory=True).numpy()


@pytest.mark.parametrize("prec", [C.PREC_FP64, C.PREC_MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n", [(32, 32, 16), (64, 64, 24), (128, 64, 32), (96, 96, 64),
                               (160, 128, 96)], ids=lambda n: "x".join(map(str, n)))
def test_round_trip(nf, n, prec):
    g = _grid(nf, n, prec)
    f = _fields(nf, g.shape, 11)
    g.set_fields(f)
    a = g.fields()
    b = {k: _pinned(g.shape) for k in nf.FIELD_ORDER}
    nf._check(nf.lib().nfvm_get_fields(g.h, ctypes.byref(nf._fields_struct(b))))
    for k in nf.FIELD_ORDER:
        assert np.array_equal(a[k], b[k]), (n, k)
    if prec == C.PREC_FP64:
        for k in ("u", "v", "w", "k", "p"):
            assert np.array_equal(a[k], f[k]), (n, k)
    pf = {k: _pinned(g.shape) for k in nf.FIELD_ORDER}
    for k in pf:
        pf[k][:] = f[k]
    g.set_fields(pf)
    c = g.fields()
    for k in nf.FIELD_ORDER:
        assert np.array_equal(a[k], c[k]), (n, k)
    one = np.zeros(g.shape)
    nf._check(nf.lib().nfvm_get_fields(
        g.h, ctypes.byref(nf._fields_struct({k: one for k in nf.FIELD_ORDER}))))
    assert np.array_equal(one, a["p"])
    lam = g.lambda2()
    plam = _pinned(g.shape)
    nf._check(nf.lib().nfvm_lambda2(g.h, plam.ctypes.data_as(ctypes.POINTER(ctypes.c_double))))
    assert np.array_equal(lam, plam)
    g.close()


def test_two_threads(nf):
    gs = [_grid(nf, (96, 96, 64), p) for p in (C.PREC_FP64, C.PREC_MIXED)]
    fs = [_fields(nf, g.shape, 20 + i) for i, g in enumerate(gs)]
    want = []
    for g, f in zip(gs, fs):
        g.set_fields(f)
        want.append(g.fields())
    bad = []

    def work(i):
        for _ in range(4):
            gs[i].set_fields(fs[i])
            got = gs[i].fields()
            bad.extend((i, k) for k in got if not np.array_equal(got[k], want[i][k]))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
    for g in gs:
        g.close()


def test_served_fields(nf):
    c = C.serve_case(dict(n=(96, 64, 64), geometry="channel", seed=4, n_steps=1), C.PREC_MIXED)
    d = nf.Desc(c)
    g = nf.Grid(c)
    f = g.fields()
    g.close()
    s = nf.nfvm_server_create(8e9, 2)
    t = nf.nfvm_submit(s, d, f, 0)
    nf.nfvm_server_drain(s)
    st, out, _ = nf.nfvm_poll(s, t, f["u"].shape)
    nf.nfvm_server_destroy(s)
    assert st == 0
    for k in f:
        assert np.array_equal(out[k], f[k]), k
