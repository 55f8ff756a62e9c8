"""What a refused scan leaves behind: the filter goes on as one that never saw it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2404_16370_amd import megapf as M
from paper_2404_16370_amd import synth as S


@pytest.fixture(scope="module")
def room():
    w = S.build_workload("room", map_points=100_000, scan_points=1100, frames=3)
    return dict(w=w, map=M.Map(w["map_xyz"], voxel=0.5))


def _filter(room, n=300):
    p = M.mp_filter_default_params(n_particles=n, k=8, lsh_bits=12, svgd_iters=2, window_c=16, d_max=1.0, seed=5)
    return M.Filter(room["map"], p, poses=S.gaussian_particles(n, S.pose8(*room["w"]["traj"][0]), 0.1, 0.3, 3))


@pytest.mark.parametrize("n", [60, 700])
@pytest.mark.parametrize("uploads", [1, 2])
def test_larger_refused_scan_leaves_the_last_ones(room, n, uploads):
    # a refused scan that needs more room than any before it: the walk records,
    # the odometry and the next step are those of a filter that never saw it
    scans = [np.ascontiguousarray(s[:n + 11 * q]) for q, s in enumerate(room["w"]["scans"][:uploads])]
    both = [_filter(room), _filter(room)]
    for f in both:
        for s in scans:
            f.scan_upload(s)
    for size in (4 * n, 60_000):
        bad = np.random.default_rng(size).uniform(-5, 5, (size, 3)).astype(np.float32)
        bad[size // 2, 1] = np.nan
        with pytest.raises(M.MegaPFError) as e:
            both[0].scan_upload(bad)
        assert e.value.status == M.MP_E_ARG
    x, y = both
    for name in ("scan", "scan_walk"):
        assert np.array_equal(x.debug_get(name), y.debug_get(name)), name
    if uploads == 2:
        for noalloc in (False, True):
            a, b = (f.odometry(iterations=5, noalloc=noalloc) for f in both)
            assert all(np.array_equal(a[q], b[q]) for q in b)
            assert a["inliers"] > n // 2
    for f in both:
        f.step()
    for name in ("poses", "psi", "prior"):
        assert np.array_equal(x.debug_get(name), y.debug_get(name)), name
    # and the next scan is taken as by the other filter
    nxt = np.ascontiguousarray(room["w"]["scans"][2])
    for f in both:
        f.scan_upload(nxt)
        f.step()
    a, b = (f.odometry(iterations=5) for f in both)
    assert all(np.array_equal(a[q], b[q]) for q in b)
    assert np.array_equal(x.debug_get("psi"), y.debug_get("psi"))
    for f in both:
        f.close()


@pytest.mark.parametrize("n", [300, 8193, 65_536])
def test_refused_upload_leaves_no_work_behind(room, n):
    # the upload that answers a refusal may come on another stream: nothing of
    # the refused one is still running on its own
    import torch
    f = _filter(room)
    good = np.random.default_rng(n).uniform(-5, 5, (n, 3)).astype(np.float32)
    bad = good.copy()
    bad[n - 1, 2] = np.inf
    one, other = torch.cuda.Stream(), torch.cuda.Stream()
    src = torch.from_numpy(bad).cuda()
    torch.cuda.synchronize()
    for _ in range(5):
        with pytest.raises(M.MegaPFError):
            f.scan_upload(src, stream=one.cuda_stream)
        assert one.query()
        f.scan_upload(good, stream=other.cuda_stream)
        other.synchronize()
    torch.cuda.synchronize()
    ref = _filter(room)
    ref.scan_upload(good)
    for name in ("scan", "scan_walk"):
        assert np.array_equal(f.debug_get(name), ref.debug_get(name)), name
    f.close()
    ref.close()
