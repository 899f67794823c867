"""The near field at the edges of its split over waves, passes and chunks: boxes of hundreds of points (several passes
of targets, several 64-source chunks per neighbour, the waves of a block sharing them) and of a few, one set and two,
all kernels, against FP64 dense sums.  The tree is cut at level 1, where every box neighbours every other, so the
near field is the whole product."""
import numpy as np
import pytest

import ffm_workloads as W
from gpu_common import FP32_RTOL, gpu_apply, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", range(8))
@pytest.mark.parametrize("n,m", [(3000, 0), (517, 0), (9, 0), (701, 1203), (1300, 5)])
def test_near_only(orc, kernel, n, m):
    import torch
    import paper_1909_05600_amd as ffm
    rng = np.random.default_rng(100 * kernel + n)
    Y = W.cube_points(n, rng, (0, 0, 0), 2.0)
    X = Y if m == 0 else W.cube_points(m, rng, (0, 0, 0), 2.0)
    # normals in random directions; weights of random sign
    NX, NY = W.sphere_points(len(X), rng), W.sphere_points(n, rng)
    if m == 0:
        NX = NY
    wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
    base, form, k = kernel % 2, kernel // 2, 5.0 if kernel % 2 else 0.0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    Yd = dev(Y)
    Xd = Yd if m == 0 else dev(X)
    kw = {1: {"normals": dev(NX)}, 2: {"source_normals": dev(NY)}}.get(form, {})
    gp = ffm.Plan(Xd, Yd, kernel, k, 1e-3, max_level=1, **kw)
    assert sum(gp.stats()["nfar"]) == 0
    v = gpu_apply(gp, wu)
    rows = np.arange(len(X))
    d = [lambda: orc.dense_rows(X, Y, wu, base, k, rows), lambda: orc.dense_rows_dn(X, Y, wu, base, k, NX, rows),
         lambda: orc.dense_rows_dl(X, Y, wu, base, k, NY, rows), lambda: orc.dense_rows_grad(X, Y, wu, base, k, rows)][form]()
    print("kernel %d n %d m %d: vs dense %.3e" % (kernel, n, m, rel(v, d)))
    assert rel(v, d) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))
