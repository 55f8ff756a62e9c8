"""Filters on a map without Gaussians (no points, or none in a voxel of enough
points): every scan point is an outlier."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2404_16370_amd import megapf as M
from paper_2404_16370_amd import synth as S

FAR = np.array([5000.0, 0, 0], np.float32)


@pytest.fixture(scope="module")
def maps():
    rng = np.random.default_rng(0)
    cloud = rng.uniform(-2, 2, (4000, 3)).astype(np.float32) + FAR
    return dict(none=M.Map(np.zeros((0, 3), np.float32), voxel=0.5), sparse=M.Map(cloud[:2], voxel=0.5),
                hashed=M.Map(np.zeros((0, 3), np.float32), voxel=0.5, backend=M.MP_NNF_HASH),
                point=M.Map(cloud[:2], voxel=0.5, gauss_mode=M.MP_GAUSS_POINT),
                far=M.Map(cloud, voxel=0.5))


def _filter(m, n, **kw):
    p = M.mp_filter_default_params(n_particles=n, k=8, lsh_bits=12, svgd_iters=2, window_c=16, d_max=1.0, seed=5, **kw)
    f = M.Filter(m, p, poses=S.gaussian_particles(n, np.array([1, 0, 0, 0, 0, 0, 0, 0]), 0.1, 0.3, 3))
    f.scan_upload(np.random.default_rng(1).uniform(-5, 5, (700, 3)).astype(np.float32))
    return f


@pytest.mark.parametrize("kind", ["none", "sparse", "hashed", "point"])
@pytest.mark.parametrize("kw", [dict(), dict(lik_batch=2), dict(lik_layout=2), dict(lik_layout=2, lik_batch=4),
                                dict(scorer=M.MP_SCORER_SCOREFIELD)], ids=str)
def test_every_point_is_an_outlier(maps, kind, kw):
    assert M.MP_LIK_LAYOUT_GROUPED == 2
    f = _filter(maps[kind], 300, **kw)
    f.debug_stage(M.MP_STAGE_LIK)
    psi = f.debug_get("psi")
    assert np.all(psi[:, :6] == 0) and np.all(psi[:, 7] == 0)
    # the log-likelihood of a map that no point comes near
    ref = _filter(maps["far"], 300, **kw)
    ref.debug_stage(M.MP_STAGE_LIK)
    assert np.array_equal(psi, ref.debug_get("psi"))
    f.step()
    q = f.posterior_query(poses=True, weights=True)
    assert np.isfinite(q["poses"]).all() and abs(q["weights"].sum() - 1) < 1e-5
    assert np.all(f.debug_get("psi")[:, 7] == 0)
    f.close()
    ref.close()


def test_lookups_miss_and_a_batch_runs(maps):
    xyz = np.random.default_rng(2).uniform(-5, 5, (100, 3)).astype(np.float32)
    for kind in ("none", "sparse", "hashed", "point"):
        assert np.all(maps[kind].lookup(xyz) == -1) and maps[kind].info()["num_gauss"] == 0
    fs = [_filter(maps[k], 200 + 100 * q) for q, k in enumerate(("none", "far", "sparse"))]
    b = M.Batch(fs, autotune=False)
    for _ in range(3):
        b.step()
        for f in fs:
            assert np.all(f.debug_get("psi")[:, 7] == 0)
    b.close()
