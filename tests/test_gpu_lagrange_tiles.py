"""Lagrange levels at the edges of their kernels' tiles: every node count per axis (16-row MFMA tiles of r1^2 rows,
2 r1 columns), boxes of a few points and of thousands (one to sixteen waves per box in the anterpolation, several
point ranges per box in the interpolation), against the oracle with identical parameters (FP32_RTOL) and bitwise
repeatable."""
import numpy as np
import pytest

import ffm_workloads as W
from gpu_common import FP32_RTOL, gpu_apply, gpu_plan, oracle_like, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel,r1", [(0, r1) for r1 in range(1, 9)] + [(1, 3), (1, 6)])
def test_node_counts(orc, kernel, r1):
    rng = np.random.default_rng(r1)
    X = W.sphere_points(3001, rng)
    wu = ((rng.standard_normal(3001) + 1j * rng.standard_normal(3001)) / 3001).astype(np.complex64)
    k = 2.0 if kernel else 0.0
    gp = gpu_plan(X, X, kernel, k, 1e-3, n_leaf=40, r1_override=r1, aca="off")
    st = gp.stats()
    assert any(o == r1 for o in st["order"][1:st["leaf"] + 1])
    v = gpu_apply(gp, wu)
    vo = oracle_like(orc, gp, X, X, kernel, k, 1e-3, n_leaf=40, r1=r1).apply(wu)
    print("kernel %d r1 %d: vs oracle %.3e" % (kernel, r1, rel(v, vo)))
    assert rel(v, vo) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))


@pytest.mark.parametrize("n", [11000, 57001, 90000])     # 196, 1018 and 1607 points per box of level 2
@pytest.mark.parametrize("dl", [False, True])
def test_points_per_box(orc, n, dl):
    import torch
    import paper_1909_05600_amd as ffm
    rng = np.random.default_rng(n)
    Y = W.sphere_points(n, rng)
    X = W.sphere_points(700, rng) * 0.98
    wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
    kernel = 4 if dl else 0
    kw = {"max_level": 3}
    nrm = {"source_normals": torch.from_numpy(Y).cuda()} if dl else {}
    gp = ffm.Plan(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), kernel, 0.0, 1e-3, **kw, **nrm)
    v = gpu_apply(gp, wu)
    vo = oracle_like(orc, gp, X, Y, kernel, 0.0, 1e-3, **kw, **({"source_normals": Y} if dl else {})).apply(wu)
    print("n %d dl %d: vs oracle %.3e" % (n, dl, rel(v, vo)))
    assert rel(v, vo) < FP32_RTOL
    # the roles exchanged: many targets per box
    if not dl:
        gt = gpu_plan(Y, X, 0, 0.0, 1e-3, **kw)
        w2 = wu[:700]
        assert rel(gpu_apply(gt, w2), oracle_like(orc, gt, Y, X, 0, 0.0, 1e-3, **kw).apply(w2)) < FP32_RTOL


@pytest.mark.parametrize("dl", [False, True])
def test_point_segments(orc, dl):
    """Level 2 with 16 boxes of 6250 points on average and boxes of a few hundred: segments (of whole rounds of a
    block, the last ones empty in small boxes) whose sums are added after."""
    import torch
    import paper_1909_05600_amd as ffm
    n = 100001
    rng = np.random.default_rng(n)
    Y = W.ellipsoid_points(n, rng)
    X = W.sphere_points(500, rng) * 0.9
    wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
    nrm = Y / np.linalg.norm(Y, axis=1, keepdims=True)
    kw = {"source_normals": torch.from_numpy(nrm).cuda()} if dl else {}
    kernel = 4 if dl else 0
    gp = ffm.Plan(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), kernel, 0.0, 1e-3, max_level=3, timing=True, **kw)
    v = gpu_apply(gp, wu)
    assert any(r["kernel"] == "k_sum_segments" for r in gp.launch_timing())
    vo = oracle_like(orc, gp, X, Y, kernel, 0.0, 1e-3, max_level=3, **({"source_normals": nrm} if dl else {})).apply(wu)
    print("dl %d: vs oracle %.3e" % (dl, rel(v, vo)))
    assert rel(v, vo) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))


@pytest.mark.parametrize("kernel,r1,eps,shift", [(0, 1, 1e-3, False), (0, 2, 1e-3, False), (0, 3, 1e-3, True),
                                                 (0, 4, 1e-3, False), (1, 3, 1e-3, False), (1, 5, 1e-3, True),
                                                 (0, 7, 1e-5, False), (1, 7, 1e-6, False)])
def test_aca_tiles(orc, kernel, r1, eps, shift):
    """The two ACA transfer kernels with ranks below and above one tile of 16, r1^3 below and above one tile of rows,
    groups of targets that do not fill, and two shifted sets (more classes, most targets without most of them)."""
    rng = np.random.default_rng(10 * r1 + kernel)
    X = W.sphere_points(2503, rng)
    Y = X if not shift else W.cube_points(1901, rng, (0.31, 0.17, -0.23), 1.7)
    wu = ((rng.standard_normal(len(Y)) + 1j * rng.standard_normal(len(Y))) / len(Y)).astype(np.complex64)
    k = 2.0 if kernel else 0.0
    gp = gpu_plan(X, Y, kernel, k, eps, n_leaf=40, r1_override=r1, aca="on")
    st = gp.stats()
    lev = [l for l in range(1, st["leaf"] + 1) if st["aca"][l]]
    assert lev
    op = oracle_like(orc, gp, X, Y, kernel, k, eps, n_leaf=40, r1=r1)
    v = gpu_apply(gp, wu)
    print("kernel %d r1 %d eps %g shift %d: mean ranks %s, vs oracle %.3e"
          % (kernel, r1, eps, shift, [round(st["aca_rank"][l], 1) for l in lev], rel(v, op.apply(wu))))
    assert rel(v, op.apply(wu)) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))


@pytest.mark.parametrize("kernel,r1", [(0, r1) for r1 in range(1, 9)] + [(1, 2), (1, 5), (1, 6)])
def test_mixed_node_counts(orc, kernel, r1):
    """FP16 levels: every count of 32-row slabs of r1^3 nodes, one and two row tiles per wave in the anterpolation, and
    point counts per box on both sides of 256 (row tiles in blocks of their own above).  u~ and T are each rounded to
    2^-11, twice for complex T: 2^-10 and 2^-9 of the output."""
    rng = np.random.default_rng(20 + r1)
    X = W.sphere_points(21001, rng)
    wu = ((rng.standard_normal(21001) + 1j * rng.standard_normal(21001)) / 21001).astype(np.complex64)
    k = 2.0 if kernel else 0.0
    gp = gpu_plan(X, X, kernel, k, 1e-3, n_leaf=80, r1_override=r1, aca="off", precision=1)
    g32 = gpu_plan(X, X, kernel, k, 1e-3, n_leaf=80, r1_override=r1, aca="off")
    v, v32 = gpu_apply(gp, wu), gpu_apply(g32, wu)
    print("kernel %d r1 %d: mixed vs fp32 %.3e" % (kernel, r1, rel(v, v32)))
    assert any(gp.stats()["prec"]) and rel(v, v32) < (2.0 ** -9 if kernel else 2.0 ** -10)
    assert np.array_equal(v, gpu_apply(gp, wu))


def test_aca_units_in_pieces():
    """Two cubes half a leaf box apart, Helmholtz with eight nodes per axis at k d = 18: 448 classes per octant with
    ranks up to 125, so a target group's unit list (68 bytes a unit) is longer than the LDS holds and is staged in
    pieces.  Against the same product with the full matrices: the factors meet a relative 2.5e-8, so the two differ by
    FP32 rounding."""
    import paper_1909_05600_amd as ffm
    rng = np.random.default_rng(8)
    n, box = 12000, 1.0 / 8
    X, Y = rng.random((n, 3)), rng.random((n, 3))
    X[0], X[1], Y[0], Y[1] = 0.0, 1.0, 0.0, 1.0
    Y += box / 2
    wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
    kw = dict(n_leaf=4, max_level=3, r1_override=8, kd_switch=25.0)
    gp = gpu_plan(X, Y, 1, 18.0 / box, 1e-7, **kw)
    assert gp.stats()["aca"][3]
    ranks = {tuple(int(x) for x in q[:3]): int(q[3]) for q in gp.export(ffm.FFM_EXPORT_ACA_RANK, 0, 3)}
    assert max(ranks.values()) <= 128
    # the target groups: 16 targets of one octant of their parents, in Morton order
    ijk = gp.export(ffm.FFM_EXPORT_BOX_IJK, 0, 3)
    far = gp.export(ffm.FFM_EXPORT_FAR, 0, 3)
    units = 0
    for octant in range(8):
        ts = [t for t in np.unique(far[:, 0]) if tuple(ijk[t] & 1) == (octant >> 2, octant >> 1 & 1, octant & 1)]
        for g in range(0, len(ts), 16):
            cls = {tuple(int(x) for x in q) for q in far[np.isin(far[:, 0], ts[g:g + 16])][:, 2:5]}
            units = max(units, sum((ranks[c] + 15) // 16 for c in cls))
    v, full = gpu_apply(gp, wu), gpu_apply(gpu_plan(X, Y, 1, 18.0 / box, 1e-7, aca="off", **kw), wu)
    print("ranks up to %d, %d units in the largest group: vs full matrices %.3e" % (max(ranks.values()), units, rel(v, full)))
    assert 68 * units > 160 * 1024
    assert rel(v, full) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))


@pytest.mark.parametrize("kernel", [0, 1, 3])
def test_aca_targets_without_far_pairs(orc, kernel):
    """Few sources within many targets: the rows of v~ that a level keeps go by the targets that have far pairs
    (every level's u~ of the source boxes and one product per far pair bound the workspace, as without ACA), and
    every target finds its own."""
    import torch
    import paper_1909_05600_amd as ffm
    n, k = 60000, 2.0 if kernel % 2 else 0.0
    rng = np.random.default_rng(5 + kernel)
    X = W.cube_points(n, rng, (0, 0, 0), 2.0)
    Y = W.cube_points(801, rng, (0.6, 0.5, 0.4), 0.15)
    N = W.sphere_points(n, rng)
    wu = ((rng.standard_normal(801) + 1j * rng.standard_normal(801)) / 801).astype(np.complex64)
    kw = dict(n_leaf=4, r1_override=6)
    nrm = {"normals": torch.from_numpy(N).cuda()} if kernel == 3 else {}
    gp = ffm.Plan(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(), kernel, k, 1e-3, aca="on", **kw, **nrm)
    st = gp.stats()
    lev = [l for l in range(1, st["leaf"] + 1) if st["aca"][l] and st["nfar"][l]]
    assert lev and any(st["nbox_x"][l] > 4 * st["nbox_y"][l] for l in lev)
    # without ACA: u~ of the source boxes and a product per far pair, 224 values of 8 bytes each, the points' u, v and
    # the parts' alignment to 256 bytes
    full = 8 * 224 * (max(st["nbox_y"][l] for l in lev) + max(st["nfar"][l] for l in lev)) + 8 * (n + 801) + 16 * 256
    assert gp.workspace_bytes() <= full
    v = gpu_apply(gp, wu)
    on = {"normals": N} if kernel == 3 else {}
    vo = oracle_like(orc, gp, X, Y, kernel, k, 1e-3, n_leaf=4, r1=6, **on).apply(wu)
    print("kernel %d: workspace %.1f of %.1f MB, vs oracle %.3e" % (kernel, gp.workspace_bytes() / 1e6, full / 1e6, rel(v, vo)))
    assert rel(v, vo) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))


@pytest.mark.parametrize("aca,r1,precision", [("on", 6, 0), ("off", 3, 0), ("off", 3, 1)])
def test_many_boxes(orc, aca, r1, precision):
    """A level of 16,000 boxes and 636,000 far pairs: class groups in eight regions (160 pairs per class and region), and
    at ACA levels expansion blocks of two waves (4096 blocks and more).  FP16 against FP32 as above (2^-10)."""
    n = 100000
    rng = np.random.default_rng(6)
    X = W.sphere_points(n, rng)
    wu = ((rng.standard_normal(n) + 1j * rng.standard_normal(n)) / n).astype(np.complex64)
    kw = dict(n_leaf=16, r1_override=r1, aca=aca)
    gp = gpu_plan(X, X, 0, 0.0, 1e-3, precision=precision, timing=True, **kw)
    st = gp.stats()
    leaf = st["leaf"]
    assert st["nfar"][leaf] >= 8 * 160 * st["nclass"][leaf]
    v = gpu_apply(gp, wu)
    if aca == "on":
        assert st["aca"][leaf]
        assert any(r["kernel"].startswith("k_lag_expand") and r["level"] == leaf and r["blocks"] >= 4096
                   for r in gp.launch_timing())
    if precision:
        assert rel(v, gpu_apply(gpu_plan(X, X, 0, 0.0, 1e-3, **kw), wu)) < 2.0 ** -10
    else:
        vo = oracle_like(orc, gp, X, X, 0, 0.0, 1e-3, n_leaf=16, r1=r1).apply(wu)
        print("aca %s r1 %d: vs oracle %.3e" % (aca, r1, rel(v, vo)))
        assert rel(v, vo) < FP32_RTOL
    assert np.array_equal(v, gpu_apply(gp, wu))


@pytest.mark.parametrize("r1", [2, 4, 6, 7, 8])
def test_ordered_sums_do_not_depend_on_the_split(r1):
    """FP16 levels sum u~ in point order, whatever the launch: boxes of a few points go to one block each, and, once the
    boxes hold 256 on average, their row tiles to blocks of their own with waves that only stage.  Four boxes of one
    point without weight take the same other boxes from one form to the other; the products are bitwise equal (all
    targets are far from all sources; the largest box, which sets the scale of u~ in FP16, is there in both)."""
    import torch
    import paper_1909_05600_amd as ffm
    rng = np.random.default_rng(r1)
    oct_ = lambda n, o: 3.0 + 0.5 * np.array([o >> 2, o >> 1 & 1, o & 1]) + 0.5 * rng.random((n, 3))  # noqa: E731
    Y = np.concatenate([[[3.0, 3.0, 3.0], [4.0, 4.0, 4.0]], oct_(100, 0), oct_(37, 3), oct_(201, 7), oct_(1500, 5)])
    Z = np.concatenate([Y] + [oct_(1, o) for o in (1, 2, 4, 6)])
    X = 0.1 * rng.random((300, 3))
    wu = np.zeros(len(Z), np.complex64)
    wu[:340] = (rng.standard_normal(340) + 1j * rng.standard_normal(340)) / 340
    out = []
    for S in (Z, Y):
        gp = ffm.Plan(torch.from_numpy(X).cuda(), torch.from_numpy(S).cuda(), 0, 0.0, 1e-3, n_leaf=8, max_level=1,
                      r1_override=r1, precision=1, timing=True)
        st = gp.stats()
        assert st["prec"][1] and st["nfar"][1] and not st["near_pairs"]
        v = gpu_apply(gp, wu[:len(S)])
        blocks = [r["blocks"] for r in gp.launch_timing() if r["kernel"] == "k_lag_anterp_ord"]
        tiles = (r1 ** 3 + 15) // 16
        boxes = st["fwd_boxes"][1]
        assert blocks == [boxes if S is Z else boxes * ((tiles + 7) // 8 if tiles > 16 else (tiles + 3) // 4)], blocks
        out.append(v)
    assert np.linalg.norm(out[0]) > 0 and np.array_equal(out[0], out[1])
