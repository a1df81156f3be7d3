"""Calls from several host threads, each on a stream of its own, while the library hands the same kept
blocks around: every result is the one of a single thread, bit for bit."""
import threading

import numpy as np
import pytest
import torch

from tests import se3
from tests.gpu_util import cloud_dev, dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

ROUNDS, THREADS = 12, 3


def job(V, k):
    """One thread's program, with sizes of its own: a sweep, a map, a one-shot batch, a single factor."""
    rng = np.random.default_rng(k)
    n = 3000 + 2500 * k
    raw = rng.uniform(-8, 8, (3, 4 * n)).astype(np.float32)
    t = rng.uniform(0, 0.099, 4 * n).astype(np.float32)
    txyz = rng.uniform(-4, 4, (3, n)).astype(np.float32)
    cov = np.tile(np.array([[.01], [0], [0], [.01], [0], [.001]], np.float32), (1, n))
    Ts = [se3.random_pose(rng, 0.2, 1.0)]
    Ts.append(Ts[0] @ se3.random_pose(rng, 0.02, 0.03))
    P = dev(np.array([se3.to12(T) for T in Ts]))
    raw, t = dev(raw), dev(t)
    cloud = cloud_dev(txyz, cov)
    factors = np.array([[0, 0, 0, 1, 1], [0, 0, 1, 0, 0]], np.int32)
    torch.cuda.synchronize()

    def run():
        out = []
        pts, stamps = V.vgicp_downsample(raw, 0.5, t, 0.1)
        nbr = V.vgicp_knn(pts, 10)
        out += [pts, stamps, nbr, V.vgicp_point_covariances(pts, nbr)]
        m = V.vgicp_build_voxelmap(*cloud, 0.5)
        out += list(V.vgicp_voxelmap_export(m).values())
        one = V.vgicp_linearize_batched([m], [cloud], P, factors)
        single = V.vgicp_linearize(m, *cloud, Ts[0], Ts[1], True)
        out += [one[q] for q in ("H", "b", "err", "inliers")] + [single["H"]]
        torch.cuda.current_stream().synchronize()
        m.close()
        return out

    return run


def test_threads_and_streams_share_the_kept_blocks():
    import paper_2202_00242_amd.vgicp as V
    jobs = [job(V, k) for k in range(THREADS)]
    want = [j() for j in jobs]
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for r in range(ROUNDS):
                    for i, (a, b) in enumerate(zip(jobs[k](), want[k])):
                        if not torch.equal(a, b):
                            errors.append((k, r, i))
                    if k == 0 and r % 3 == 2:
                        V.vgicp_release_idle()
        except Exception as e:  # noqa: BLE001  (reported by the test)
            errors.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[:5]


def test_release_gives_the_kept_memory_back():
    import paper_2202_00242_amd.vgicp as V
    x, c = cloud_dev(np.random.default_rng(1).uniform(-9, 9, (3, 1 << 20)).astype(np.float32),
                     np.tile(np.array([[.01], [0], [0], [.01], [0], [.01]], np.float32), (1, 1 << 20)))
    V.vgicp_release_idle()
    V.vgicp_build_voxelmap(x, c, 0.5).close()
    held = torch.cuda.mem_get_info()[0]
    V.vgicp_release_idle()
    assert torch.cuda.mem_get_info()[0] >= held + (32 << 20)
    V.vgicp_build_voxelmap(x, c, 0.5).close()
