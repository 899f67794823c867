"""ACA of the Lagrange transfer matrices on the GPU (Sec. 2.2.2, eq. ffmACAmatvec: T ~ A B^T, applied as
A (B^T u~) in one kernel with both products on MFMA; reading R21: complete pivoting, tolerance eps / 4, FP64 on
the host at plan time).

Element-wise against the oracle FFM with identical parameters (its own ACA at the same levels): the rank of
every translation class equal to the oracle's, and v within FP32_RTOL; within eps of FP64 dense rows; close to
the GPU product with full transfer matrices; the planner's automatic choice and both forcing flags.
"""
import numpy as np
import pytest

import ffm_workloads as W
from gpu_common import FP32_RTOL, gpu_apply, gpu_plan, oracle_like, rel

pytestmark = pytest.mark.gpu


def _check_ranks(gp, op, levels):
    import paper_1909_05600_amd as ffm
    for l in levels:
        mine = {tuple(int(x) for x in row[:3]): int(row[3]) for row in gp.export(ffm.FFM_EXPORT_ACA_RANK, 0, l)}
        theirs = op.aca_ranks(l, op.eps / 4)
        assert mine == theirs, l


@pytest.mark.parametrize("kernel,k,eps,n", [(0, 0.0, 1e-4, 20000), (1, 9.0, 1e-3, 20000), (1, 20.0, 1e-4, 30000)])
def test_aca_matches_oracle(orc, kernel, k, eps, n):
    rng = np.random.default_rng(40 + n % 7)
    X = W.sphere_points(n, rng)
    wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
    gp = gpu_plan(X, X, kernel, k, eps)
    st = gp.stats()
    lev = [l for l in range(1, st["leaf"] + 1) if st["aca"][l]]
    assert lev, (st["method"], st["order"], st["aca_rank"])
    op = oracle_like(orc, gp, X, X, kernel, k, eps)
    _check_ranks(gp, op, lev)
    v = gpu_apply(gp, wu)
    vo = op.apply(wu)
    vf = gpu_apply(gpu_plan(X, X, kernel, k, eps, aca="off"), wu)
    rows = np.arange(0, n, 37)
    d = orc.dense_rows(X, X, wu, kernel, k, rows)
    print("kernel %d k=%g eps=%g: ACA levels %s (mean ranks %s of r = %s): vs oracle %.3e, vs dense %.3e, "
          "vs full-T GPU %.3e" % (kernel, k, eps, lev, [round(st["aca_rank"][l], 1) for l in lev],
                                  [st["order"][l] ** 3 for l in lev], rel(v, vo), rel(v[rows], d), rel(v, vf)))
    assert rel(v, vo) < FP32_RTOL
    assert rel(v[rows], d) <= eps
    assert rel(v, vf) <= eps / 2
    assert np.array_equal(v, gpu_apply(gp, wu))


def test_aca_flags(orc):
    """FFM_FLAG_ACA forces ACA at FP32 Lagrange levels with four nodes per axis (r = 64, where the planner keeps
    T); FFM_FLAG_NO_ACA keeps T everywhere; both flags together are refused; mixed precision keeps FP16 T."""
    import paper_1909_05600_amd as ffm
    w = W.laplace_sphere(8192, seed=7)
    auto = gpu_plan(w.X, w.X, 0, 0.0, w.eps)
    assert not any(auto.stats()["aca"])
    forced = gpu_plan(w.X, w.X, 0, 0.0, w.eps, aca="on")
    lev = [l for l in range(1, forced.stats()["leaf"] + 1) if forced.stats()["aca"][l]]
    assert lev
    op = oracle_like(orc, forced, w.X, w.X, 0, 0.0, w.eps)
    _check_ranks(forced, op, lev)
    v = gpu_apply(forced, w.wu)
    assert rel(v, op.apply(w.wu)) < FP32_RTOL
    assert rel(v, gpu_apply(auto, w.wu)) <= w.eps / 2
    off = gpu_plan(w.X, w.X, 0, 0.0, 1e-4, aca="off")
    assert not any(off.stats()["aca"])
    mixed = gpu_plan(w.X, w.X, 0, 0.0, w.eps, aca="on", precision=1)
    assert not any(mixed.stats()["aca"]) and any(mixed.stats()["prec"])
    import ctypes as C
    h = C.c_void_p()
    Xd = __import__("torch").from_numpy(w.X).cuda()
    bad = ffm.Options(0, 0, 0.0, 0, 0, ffm.FFM_FLAG_ACA | ffm.FFM_FLAG_NO_ACA)
    assert ffm.lib().ffm_plan(Xd.data_ptr(), w.n, Xd.data_ptr(), w.n, 0, 0.0, 1e-3, C.byref(bad), None,
                              C.byref(h)) == -1


def test_aca_in_a_batch():
    """A batch mixing ACA and full-T levels gives each instance bitwise its own apply."""
    import torch
    import paper_1909_05600_amd as ffm
    rng = np.random.default_rng(3)
    plans, wus, refs = [], [], []
    for n, kern, k, eps, aca in ((9000, 1, 15.0, 1e-3, "auto"), (7000, 0, 0.0, 1e-4, "auto"),
                                 (6000, 0, 0.0, 1e-3, "off"), (5000, 1, 6.0, 1e-3, "on")):
        X = W.sphere_points(n, rng)
        wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
        p = gpu_plan(X, X, kern, k, eps, aca=aca)
        plans.append(p)
        wus.append(torch.from_numpy(wu).cuda())
        refs.append(gpu_apply(p, wu))
    assert sum(any(p.stats()["aca"]) for p in plans) >= 2
    b = ffm.Batch(plans, graph=True)
    outs = b.apply(wus)
    torch.cuda.synchronize()
    for o, r in zip(outs, refs):
        assert np.array_equal(o.cpu().numpy().astype(np.complex128), r)
    b.destroy()


CHILD = r"""
import sys
import numpy as np, torch
sys.path.insert(0, %r)
import ffm_workloads as W
import paper_1909_05600_amd as ffm
rng = np.random.default_rng(11)
X = torch.from_numpy(W.sphere_points(5000, rng)).cuda()
wu = torch.from_numpy(((rng.standard_normal(5000) + 1j * rng.standard_normal(5000)) / 5000).astype(np.complex64)).cuda()
# the library is loaded, with the plan's kernels and the runtime's memory for them: sets of one class, one small set
for r1 in (5, 6):
    ffm.Plan(X[:100] * 0.05 + 2.0, X[-100:] * 0.05, 1, 5.0, 1e-3, n_leaf=8, r1_override=r1, aca="on").apply(wu[:100])
ffm.Plan(X[:300].contiguous(), X[:300].contiguous(), 1, 5.0, 1e-3, max_level=1).apply(wu[:300])
torch.cuda.synchronize()
free = torch.cuda.mem_get_info()[0]
p = ffm.Plan(X, X, 1, 5.0, 1e-3)
assert any(p.stats()["aca"])
np.save(sys.argv[1], p.apply(wu).cpu().numpy())
print("HELD", free - torch.cuda.mem_get_info()[0], int(p.plan_bytes()), flush=True)
"""


def test_aca_on_a_full_device(tmp_path):
    """The factorisation's scratch gives way: a plan of 5000 points (316 classes of r = 216 and 125) builds where no
    allocation may exceed 24 MB (the residuals by fewer blocks at a time, the factors with as many columns as the ranks
    found), with bitwise the same product.  With all memory at hand it takes the residuals of 316 blocks (236 MB) and 64
    columns of both factors (70 MB) for its two levels together, beside what the plan itself holds (20 MB for the lists'
    scratch and sizes rounded up to 2 MB)."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = []
    for limit in (None, 24 << 20):
        env = dict(os.environ)
        if limit:
            env["FFM_TEST_FAIL_ALLOC_ABOVE"] = str(limit)
        f = str(tmp_path / ("%s.npy" % limit))
        r = subprocess.run([sys.executable, "-c", CHILD % root, f], capture_output=True, text=True, env=env, timeout=300)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
        held, plan = [int(x) for x in [ln for ln in r.stdout.splitlines() if ln.startswith("HELD")][0].split()[1:]]
        print("limit %s: %.1f MB taken, plan %.1f MB" % (limit, held / 1e6, plan / 1e6))
        out.append((np.load(f), held - plan))
    assert np.array_equal(out[0][0], out[1][0])
    assert out[0][1] < (236 + 70 + 20) * 1e6
    assert out[1][1] < out[0][1]
