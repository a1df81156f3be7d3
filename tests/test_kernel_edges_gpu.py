"""The kernels at the sizes where their tiling, dispatch or rounding could go wrong, against the
oracle: lookups beside voxel faces, wave items around a row / chunk / tile, the sort's two forms,
full filter cells, neighbour lists at each list length, IMU segments around 16 samples and factors
around a block of 8, caller workspaces.

Bars: counts, keys, neighbours, filtered points and correspondences are bitwise equal; H, b, e and
gradients within the parity tests' bounds (tests/gpu_util.py); the same sums from another launch
shape are bitwise equal."""
import numpy as np
import pytest
import torch

import oracle
from oracle import imu as oimu
from oracle import preprocess as pp
from tests import se3, tiny
from tests.gpu_util import (TOL_FP64_ACC, cloud_dev, compare_factor, dev, point_gradient_error)
from tests.metrics import factor_errors
from tests.test_imu_gpu import G, SA, SBA, SBW, SG, make_factors
from tests.test_parity_gpu import check_map_equal
from tests.test_preprocess_gpu import host

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

COV = np.array([[.01], [0], [0], [.01], [0], [.001]], np.float32)


@pytest.fixture(scope="module")
def V():
    import paper_2202_00242_amd.vgicp as V
    return V


def covs(n):
    return np.ascontiguousarray(np.tile(COV, (1, n)))


def same(a, b, keys=("H", "b", "err", "inliers")):
    for k in keys:
        assert torch.equal(a[k], b[k]), k


# ------------------------------------------------------------------ lookups

@pytest.mark.parametrize("layout", [1, 2])
@pytest.mark.parametrize("res", [0.5, 0.3])
@pytest.mark.parametrize("shift", [0.0, 700.0, 3.0e5])
def test_batch_lookups_beside_voxel_faces(V, res, layout, shift):
    """Source points on voxel faces, an FP32 step to either side of them and a few FP32-transform
    error bounds away, near the origin, far from it, and so far that only the FP64 lookup may decide
    (5 km apart frames make its offset large): inlier counts are the oracle's exactly."""
    rng = np.random.default_rng(7)
    txyz = (rng.uniform(-4, 4, (3, 4000)) + shift).astype(np.float32)
    om = oracle.VoxelMap(txyz, covs(4000), res)
    m = V.vgicp_build_voxelmap(*cloud_dev(txyz, covs(4000)), res, layout=layout)
    k = np.round((rng.uniform(-5, 5, (3, 3001)) + shift) / res)
    face = (k * res).astype(np.float32)
    off = rng.choice([0.0, 1e-7, -1e-7, 3e-5, -3e-5, 1e-3, 0.1], (3, 3001))
    sxyz = np.nextafter(face, (face + rng.choice([-1, 0, 1], (3, 3001))).astype(np.float32))
    sxyz = (sxyz.astype(np.float64) + off * rng.integers(0, 2, (3, 3001))).astype(np.float32)
    poses = [np.eye(4), np.eye(4), se3.random_pose(rng, 0.3, 2.0)]
    far = np.eye(4)
    far[:3, 3] = [5000.0, -3000.0, 10.0]
    poses += [far, far @ poses[2]]
    factors = np.array([[0, 0, 0, 1, 1], [0, 0, 2, 2, 0], [0, 0, 3, 3, 1], [0, 0, 4, 4, 1]], np.int32)
    P = dev(np.array([se3.to12(T) for T in poses]))
    b = V.Batch([m], [cloud_dev(sxyz, covs(3001))], factors, len(poses))
    out = b.linearize(P)
    ev = b.evaluate(P)
    ov = b.overlap(P)
    rates, inliers = ov["rates"], ov["inliers"]
    torch.cuda.synchronize()
    for f, (_, _, ti, si, bi) in enumerate(factors):
        ref = oracle.linearize(om, sxyz, covs(3001), poses[ti], poses[si], bool(bi))
        assert ref["inliers"] > 0
        got = [int(x[f].item()) for x in (out["inliers"], ev["inliers"], inliers)]
        assert got == [ref["inliers"]] * 3, (f, got, ref["inliers"])
        d = 12 if bi else 6
        err = factor_errors(out["H"][f].cpu().numpy()[:d, :d], out["b"][f, :d].cpu().numpy(),
                            out["err"][f].item(), ref["H"], ref["b"], ref["e"])
        assert max(err["H"], err["b"], err["e"]) <= TOL_FP64_ACC, (f, err)


# ------------------------------------------------------------------ wave items

@pytest.mark.parametrize("sched", [(256, 2048, 1, 2), (256, 4096, 2, 4), (512, 4096, 4, 8),
                                   (512, 8192, 1, 4)])
def test_wave_items_around_rows_chunks_and_tiles(V, sched):
    """Clouds of one point to a few past a row (64), a wave's two rows, its chunk, a tile and two
    tiles; the same batch with other grids gives the same bits."""
    rng = np.random.default_rng(sum(sched))
    block, tile, per_cu, look = sched
    txyz, _ = tiny.cloud(rng, 3000, extent=2.0)
    sizes = sorted({max(1, n + d) for n in (1, 64, 128, 64 * look, block * look, tile, 2 * tile)
                    for d in (-1, 0, 1)})
    sources = [tiny.source_near(rng, txyz, n, noise=0.15) for n in sizes]
    m = V.vgicp_build_voxelmap(*cloud_dev(txyz, covs(3000)), 0.5)
    om = oracle.VoxelMap(txyz, covs(3000), 0.5)
    poses = [se3.random_pose(rng, 0.2, 1.0)]
    poses.append(poses[0] @ se3.random_pose(rng, 0.02, 0.03))
    factors = np.array([[0, i, 0, 1, i % 2] for i in range(len(sizes))], np.int32)
    P = dev(np.array([se3.to12(T) for T in poses]))
    b = V.Batch([m], [cloud_dev(x, covs(x.shape[1])) for x in sources], factors, 2)
    b.set_schedule(*sched)
    out, ev = b.linearize(P), b.evaluate(P)
    g = dev(np.ones(len(sizes)))
    gr = b.backward(P, g, 3, want_factors=True)
    ov = b.overlap(P)
    rates, inliers = ov["rates"], ov["inliers"]
    torch.cuda.synchronize()
    assert torch.equal(inliers, out["inliers"]) and torch.equal(ev["inliers"], inliers)
    for f, n in enumerate(sizes):
        bi = bool(f % 2)
        ref = oracle.linearize(om, sources[f], covs(n), *poses, bi)
        assert int(inliers[f].item()) == ref["inliers"], n
        if ref["inliers"] == 0:
            assert not out["H"][f].any() and not gr["grad_points"][f].any()
            continue
        assert rates[f].item() == ref["inliers"] / n
        d = 12 if bi else 6
        err = factor_errors(out["H"][f].cpu().numpy()[:d, :d], out["b"][f, :d].cpu().numpy(),
                            out["err"][f].item(), ref["H"], ref["b"], ref["e"])
        assert max(err["H"], err["b"], err["e"]) <= TOL_FP64_ACC, (n, err)
        assert abs(ev["err"][f].item() - ref["e"]) <= TOL_FP64_ACC * ref["e"]
        corr = oracle.evaluate(om, sources[f], covs(n), *poses)["corr"]
        rg = oracle.gradient(om, sources[f], covs(n), *poses, bi, corr)
        gf = gr["grad_factors"][f].cpu().numpy()[:d]
        assert np.max(np.abs(gf - rg["g_xi"])) <= 1e-9 * np.linalg.norm(rg["g_xi"])
        # FP32 outputs: their rounding, on the point's scale
        assert point_gradient_error(gr["grad_points"][f].cpu().numpy(), rg["g_points"], om,
                                    sources[f], covs(n), *poses, corr) <= 1e-6
    for other in (1, 2, 4):
        b.set_schedule(block, tile, other, look)
        same(b.linearize(P), out)
        again = b.backward(P, g, 3, want_factors=True)
        assert torch.equal(again["grad_factors"], gr["grad_factors"])
    torch.cuda.synchronize()


def test_one_shot_batch_is_the_prepared_one(V):
    rng = np.random.default_rng(5)
    txyz, _ = tiny.cloud(rng, 3000, extent=2.0)
    clouds = [cloud_dev(tiny.source_near(rng, txyz, n), covs(n)) for n in (1, 999, 9000)]
    m = V.vgicp_build_voxelmap(*cloud_dev(txyz, covs(3000)), 0.5)
    poses = [se3.random_pose(rng, 0.2, 1.0)]
    poses.append(poses[0] @ se3.random_pose(rng, 0.02, 0.03))
    P = dev(np.array([se3.to12(T) for T in poses]))
    factors = np.array([[0, c, 0, 1, 1] for c in (2, 0, 1, 2)], np.int32)
    want = V.Batch([m], clouds, factors, 2).linearize(P)
    for _ in range(3):  # the blocks of the call before come back
        same(V.vgicp_linearize_batched([m], clouds, P, factors), want)


# ------------------------------------------------------------------ sorts

@pytest.mark.parametrize("n", [1, 255, 1023, 1024, 1025, 1 << 18, (1 << 18) + 1])
def test_sort_sizes(V, n):
    """A tile of the sort is 1,024 pairs; above 2^18 pairs the other sort takes over."""
    rng = np.random.default_rng(n)
    xyz = rng.uniform(-15, 15, (3, n)).astype(np.float32)
    print(f"sorts of {n}", flush=True)
    check_map_equal(V, xyz, covs(n), 0.5)
    t = rng.uniform(0, 0.099, n).astype(np.float32)
    xo, to = V.vgicp_downsample(dev(xyz), 0.7, dev(t), 0.1)
    rx, rt, _, _ = pp.downsample(xyz, 0.7, t, 0.1)
    np.testing.assert_array_equal(host(xo), rx)
    np.testing.assert_array_equal(host(to), rt)
    rows = rng.choice(n, min(n, 300), replace=False)
    np.testing.assert_array_equal(host(V.vgicp_knn(dev(xyz), 10))[:, rows],
                                  pp.knn(xyz, 10, rows=rows))


@pytest.mark.parametrize("sizes", [[1] * 40, [(1 << 18) + 3], [5, 1 << 17, 0, (1 << 17) - 5, 70]])
def test_batch_point_order_of_many_and_large_clouds(V, sizes):
    """The batch's spatial copies: every point's gradient comes back at the caller's index (the
    single factor's gradient at that point; FP32 outputs of the same FP64 arithmetic)."""
    rng = np.random.default_rng(len(sizes))
    txyz = rng.uniform(-6, 6, (3, 40000)).astype(np.float32)
    m = V.vgicp_build_voxelmap(*cloud_dev(txyz, covs(40000)), 0.5)
    Tt = se3.random_pose(rng, 0.2, 1.0)
    Ts = Tt @ se3.random_pose(rng, 0.02, 0.03)
    clouds = [cloud_dev(rng.uniform(-7, 7, (3, n)).astype(np.float32), covs(n)) for n in sizes]
    factors = np.array([[0, c, 0, 1, 1] for c in range(len(sizes))], np.int32)
    b = V.Batch([m], clouds, factors, 2)
    g = b.backward(dev(np.array([se3.to12(Tt), se3.to12(Ts)])), dev(np.ones(len(sizes))), 3)
    for c, (x, cv) in enumerate(clouds):
        if x.shape[1] == 0:
            continue
        fw = V.vgicp_evaluate(m, x, cv, Tt, Ts, 3, want_corr=True)
        _, gp = V.vgicp_backward(m, x, cv, Tt, Ts, True, fw["corr"], dev(np.array([1.0])), 3)
        scale = gp.norm(dim=0)
        err = (g["grad_points"][c] - gp).abs().amax(0)
        assert bool((err[fw["corr"] < 0] == 0).all())
        assert bool((err <= 1e-6 * scale).all()), float((err / scale.clamp_min(1e-30)).max())


def test_batch_order_of_a_cloud_with_points_that_are_not_finite(V):
    """Such a cloud's cells reach the order's limits: the batch still reports it, its finite
    points count as before, and the other clouds' factors are not touched."""
    rng = np.random.default_rng(9)
    txyz, _ = tiny.cloud(rng, 2000, extent=2.0)
    good = tiny.source_near(rng, txyz, 1500)
    bad = good.copy()
    bad[0, 3], bad[1, 700], bad[2, 1499] = np.nan, np.inf, 3e37
    m = V.vgicp_build_voxelmap(*cloud_dev(txyz, covs(2000)), 0.5)
    om = oracle.VoxelMap(txyz, covs(2000), 0.5)
    P = dev(np.array([se3.to12(np.eye(4))] * 2))
    b = V.Batch([m], [cloud_dev(good, covs(1500)), cloud_dev(bad, covs(1500))],
                np.array([[0, 0, 0, 1, 1], [0, 1, 0, 1, 1]], np.int32), 2)
    out = b.linearize(P)
    with pytest.raises(V.VGICPError) as ei:
        V.vgicp_sync_status()
    assert ei.value.status == V.VGICP_E_NONFINITE
    ref = oracle.linearize(om, good, covs(1500), np.eye(4), np.eye(4), True)
    one = {k: out[k][0:1] if k in ("err", "inliers") else out[k][0]
           for k in ("H", "b", "err", "inliers")}
    compare_factor(one, ref, TOL_FP64_ACC)
    keep = np.ones(1500, bool)
    keep[[3, 700, 1499]] = False
    finite = oracle.linearize(om, np.ascontiguousarray(good[:, keep]), covs(1497), np.eye(4),
                              np.eye(4), True)
    assert int(out["inliers"][1].item()) == finite["inliers"]


@pytest.mark.parametrize("n", [63, 65, 4095, 4096, 4097, 9001])
def test_filter_cell_of_many_points(V, n):
    """One cell holding n timestamped points (4,096 is where the in-register ranks end), with equal
    timestamps among them, beside a few ordinary cells."""
    rng = np.random.default_rng(n)
    xyz = np.concatenate([rng.uniform(0.05, 0.95, (3, n)), rng.uniform(-9, 9, (3, 100))], 1)
    xyz = np.ascontiguousarray(xyz[:, rng.permutation(n + 100)], np.float32)
    t = np.round(rng.uniform(0, 0.099, n + 100), 4).astype(np.float32)
    xo, to = V.vgicp_downsample(dev(xyz), 1.0, dev(t), 0.1)
    rx, rt, _, _ = pp.downsample(xyz, 1.0, t, 0.1)
    np.testing.assert_array_equal(host(xo), rx)
    np.testing.assert_array_equal(host(to), rt)


# ------------------------------------------------------------------ neighbours

@pytest.mark.parametrize("k", [1, 6, 7, 10, 11, 16, 17, 32])
@pytest.mark.parametrize("n", [5, 63, 65, 1500])
def test_knn_list_lengths(V, k, n):
    rng = np.random.default_rng(100 * k + n)
    pts = (rng.normal(size=(3, n)) * np.array([[4.0], [4.0], [0.5]])).astype(np.float32)
    pts[:, n // 2:n // 2 + n // 8] = pts[:, :n // 8]
    np.testing.assert_array_equal(host(V.vgicp_knn(dev(pts), k)), pp.knn(pts, k))


# ------------------------------------------------------------------ IMU

def test_imu_segments_around_16_samples(V):
    rng = np.random.default_rng(21)
    lens = [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 1, 300]
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    rows, _, bias = make_factors(rng, len(lens), 301, 300)
    rows = np.ascontiguousarray(rows[:seg[-1]])
    pre, cov, jac = V.vgicp_imu_preintegrate_bias(dev(rows), dev(seg), dev(bias), SG, SA)
    pre, cov, jac = pre.cpu().numpy(), cov.cpu().numpy(), jac.cpu().numpy()
    for f in range(len(lens)):
        ref = oimu.preintegrate(rows[seg[f]:seg[f + 1]], bias[f], SG, SA)
        np.testing.assert_allclose(pre[f, :9].reshape(3, 3), ref["dR"], atol=1e-12)
        sc = max(1.0, np.abs(ref["dp"]).max(), np.abs(ref["dv"]).max())
        np.testing.assert_allclose(pre[f, 9:12], ref["dv"], atol=1e-12 * sc)
        np.testing.assert_allclose(pre[f, 12:15], ref["dp"], atol=1e-12 * sc)
        np.testing.assert_allclose(cov[f], ref["cov"], atol=1e-10 * np.abs(ref["cov"]).max())
        J = ref["J_bias"]
        assert np.abs(jac[f].reshape(9, 6) - J).max() <= 1e-12 * max(1.0, np.abs(J).max())


@pytest.mark.parametrize("F", [1, 3, 4, 5, 7, 8, 9, 17])
def test_imu_factor_counts(V, F):
    """A block holds 8 factors (16 lanes a preintegration): each factor's values do not depend on
    how many stand beside it, bit for bit, and are the oracle's."""
    rng = np.random.default_rng(22)
    N = 33
    rows, seg, bias = make_factors(rng, N, 40, min_len=2)
    poses = np.array([se3.to12(se3.random_pose(rng, 0.1, 0.5)) for _ in range(N + 1)])
    vel, bb = rng.normal(size=(N + 1, 3)), rng.normal(size=(N + 1, 6)) * 0.02
    st = np.stack([np.arange(N), np.arange(1, N + 1)], 1).astype(np.int32)

    def run(n):
        pre, cov, jac = V.vgicp_imu_preintegrate_bias(dev(rows[:seg[n]]), dev(seg[:n + 1]),
                                                      dev(bias[:n]), SG, SA)
        out = V.vgicp_imu_linearize_bias(pre, cov, jac, dev(bias[:n]), dev(st[:n]), dev(poses),
                                         dev(vel), dev(bb), G, SBA, SBW)
        return pre, cov, jac, out["H"], out["b"], out["err"]

    few, many = run(F), run(N)
    for a, b in zip(few, many):
        assert torch.equal(a, b[:F])
    f = F - 1
    ref = oimu.preintegrate(rows[seg[f]:seg[f + 1]], bias[f], SG, SA)
    lin = oimu.linearize_bias(ref, poses[f].reshape(3, 4), vel[f], bb[f],
                              poses[f + 1].reshape(3, 4), vel[f + 1], bb[f + 1], G, SBA, SBW)
    d = np.sqrt(np.maximum(np.diag(lin["H"]), 1e-300))
    H = few[3][f].cpu().numpy().reshape(30, 30)
    assert np.max(np.abs(H - lin["H"]) / np.outer(d, d)) <= 1e-8
    assert abs(few[5][f].item() - lin["e"]) <= 1e-8 * lin["e"]


# ------------------------------------------------------------------ single factors

@pytest.mark.parametrize("n", [0, 1, 256, 4097, 40000])
def test_caller_workspaces(V, n):
    """The forms with the caller's workspace give the bits of those without (an explicit stream takes
    the latter), refuse one that is absent or a byte short, and write nothing then. 40,000 points:
    more tiles than the backward's sum takes at a time."""
    rng = np.random.default_rng(n)
    txyz, _ = tiny.cloud(rng, 3000, extent=2.0)
    x, c = cloud_dev(tiny.source_near(rng, txyz, n) if n else np.zeros((3, 0)), covs(n))
    m = V.vgicp_build_voxelmap(*cloud_dev(txyz, covs(3000)), 0.5)
    Tt = se3.random_pose(rng, 0.2, 1.0)
    Ts = Tt @ se3.random_pose(rng, 0.02, 0.03)
    cs = torch.cuda.current_stream()
    g = dev(np.array([1.0]))
    for prec in (0, 3):
        a = V.vgicp_linearize(m, x, c, Tt, Ts, True, prec, want_corr=True)
        same(a, V.vgicp_linearize(m, x, c, Tt, Ts, True, prec, want_corr=True, stream=cs),
             ("H", "b", "err", "inliers", "corr"))
        e = V.vgicp_evaluate(m, x, c, Tt, Ts, prec, want_corr=True)
        same(e, V.vgicp_evaluate(m, x, c, Tt, Ts, prec, want_corr=True, stream=cs),
             ("err", "inliers", "corr"))
        for u, w in zip(V.vgicp_backward(m, x, c, Tt, Ts, True, e["corr"], g, prec),
                        V.vgicp_backward(m, x, c, Tt, Ts, True, e["corr"], g, prec, stream=cs)):
            assert torch.equal(u, w)
    if n >= 4097:
        gxi, _ = V.vgicp_backward(m, x, c, Tt, Ts, True, e["corr"], g, 3)
        om = oracle.VoxelMap(txyz, covs(3000), 0.5)
        sx = x.cpu().numpy()
        ref = oracle.gradient(om, sx, covs(n), Tt, Ts, True, e["corr"].cpu().numpy())["g_xi"]
        assert np.max(np.abs(gxi.cpu().numpy() - ref)) <= 1e-9 * np.linalg.norm(ref)
    need = V.vgicp_workspace_size(n)
    ws = torch.empty(max(need, 8), dtype=torch.uint8, device="cuda")
    err = torch.full((1,), -7.0, dtype=torch.float64, device="cuda")
    nin = torch.full((1,), -7, dtype=torch.int64, device="cuda")
    t12, s12 = (np.ascontiguousarray(se3.to12(T)) for T in (Tt, Ts))

    def call(ptr, size):
        return V._lib.vgicp_evaluate_workspace(
            m.handle, V._ptr(x), V._ptr(c), n, V._np_ptr(t12), V._np_ptr(s12), 0, V._ptr(err),
            V._ptr(nin), None, ptr, size, V._stream(None))

    assert call(None, need) == V.VGICP_E_INVALID_ARG
    assert call(V._ptr(ws), need - 1) == V.VGICP_E_CAPACITY
    torch.cuda.synchronize()
    assert err.item() == -7.0 and nin.item() == -7
    assert call(V._ptr(ws), need) == 0
    torch.cuda.synchronize()
    if n:
        assert nin.item() == int(e["inliers"].item())
    # the binding's forms
    same(V.vgicp_linearize_workspace(m, x, c, Tt, Ts, True, ws, 3, want_corr=True), a,
         ("H", "b", "err", "inliers", "corr"))
    same(V.vgicp_evaluate_workspace(m, x, c, Tt, Ts, ws, 3, want_corr=True), e,
         ("err", "inliers", "corr"))
    xi = np.full(6, 0.01)
    for u, w in zip(V.vgicp_backward_tangent_workspace(m, x, c, Tt, Ts, xi, xi, True, e["corr"], g,
                                                       ws, 3),
                    V.vgicp_backward_tangent(m, x, c, Tt, Ts, xi, xi, True, e["corr"], g, 3,
                                             stream=cs)):
        assert torch.equal(u, w)
    with pytest.raises(V.VGICPError):
        V.vgicp_evaluate_workspace(m, x, c, Tt, Ts, ws[:8], 3)
