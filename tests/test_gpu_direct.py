"""Direct summation at the edges of its work splits against the CPU oracle:
FP32 (targets per workgroup 4, 16, 64 and 256 by the particle count; ragged
tiles) under the suite's force rule, FP64 for target counts that are no
multiple of a workgroup's four, with and without scratch (the same bits)."""
import ctypes as C

import numpy as np
import pytest

import nbody_inputs as I
from test_gpu_parity import TOL, _dev, _np, _say, nb, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 257, 1023, 1025, 16383, 16384 + 5, 65536 + 3, 262144 + 9])
def test_direct_fp32_edges(nb, torch, orc, n):
    p = I.plummer(n, 5)
    x, y, z, _, _, _, m = p.f32()
    ctx = nb.Context(nb.Params(), n_max=16)
    got = np.stack([_np(t) for t in ctx.direct(*(_dev(torch, a) for a in (x, y, z, m)))], 1)
    ctx.sync()
    sub = np.unique(np.concatenate([[0, n - 1], np.linspace(0, n - 1, min(n, 200)).astype(int)]))
    ref, A = orc.direct(np.stack([x, y, z], 1).astype(np.float64), m,
                        targets=sub.astype(np.int64), want_aabs=True)
    d = np.linalg.norm(got[sub] - ref, axis=1)
    _say("direct", n, "max |da| / A %.2g" % (d / np.maximum(A, 1e-300)).max())
    assert (d <= TOL * A).all()


@pytest.mark.parametrize("n,nt", [(1, 1), (300, 3), (5000, 5), (5000, 64), (70001, 17),
                                  (3000, 2501)])
def test_direct64_edges_and_scratch(nb, torch, orc, n, nt):
    g = I.plummer(n, 6)
    x, y, z, _, _, _, m = g.f32()
    rng = np.random.default_rng(n)
    tgt = rng.permutation(n)[:nt].astype(np.int64)
    T = _dev(torch, tgt)
    dev = [_dev(torch, a) for a in (x, y, z, m)]
    ctx = nb.Context(nb.Params(), n_max=16)
    acc, aabs, phi = ctx.direct64(*dev, T)
    ctx.sync()
    ra, rA, rphi = orc.direct(np.stack([x, y, z], 1).astype(np.float64), m, targets=tgt,
                              want_aabs=True, want_phi=True)
    for got, ref in ((_np(acc), ra), (_np(aabs), rA), (_np(phi), rphi)):
        assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
    # a context without a workspace sums the same slices in the workgroup
    cp, h = ctx.params.c(), C.c_void_p()
    assert nb.lib().nbody_create(C.byref(cp), nb._stream_handle(None), C.byref(h)) == 0
    out = torch.empty((5, nt), dtype=torch.float64, device="cuda")
    assert nb.lib().nbody_direct64(h, n, *[nb._ptr(t) for t in dev], nt, nb._ptr(T),
                                   *[nb._ptr(out[k]) for k in range(5)]) == 0
    torch.cuda.synchronize()
    nb.lib().nbody_destroy(h)
    for got, ref in zip((*acc.T, aabs, phi), out):
        np.testing.assert_array_equal(_np(got), _np(ref))
