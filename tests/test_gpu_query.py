"""A query's poses and weights in pieces, and the memory that it takes."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2404_16370_amd import megapf as M


@pytest.fixture(scope="module")
def world():
    return M.Map(np.random.default_rng(0).uniform(-5, 5, (20_000, 3)).astype(np.float32), voxel=0.5)


@pytest.mark.parametrize("n,stage", [(1, 0), (37, 0), (37, 36 * 37), (37, 36 * 37 - 1), (1000, 1000), (60_001, 1 << 20),
                                     (300_001, 2 << 20)])
def test_outputs_in_pieces(world, n, stage):
    # pieces of one particle (0), all in one, one short of it, ragged last ones;
    # host outputs, device outputs and one of each
    import torch
    f = M.Filter(world, M.mp_filter_default_params(n_particles=n, svgd_iters=1, seed=n))
    f.debug_set("query_stage", stage)
    f.debug_set("prior", np.random.default_rng(n).uniform(0, 1, n).astype(np.float32))
    P, W = f.debug_get("poses")[:, :7], f.debug_get("prior").astype(np.float64)
    q = f.posterior_query(poses=True, weights=True)
    assert np.array_equal(q["poses"], P) and np.array_equal(q["weights"], W)
    assert np.array_equal(f.posterior_query(poses=True)["poses"], P)
    assert np.array_equal(f.posterior_query(weights=True)["weights"], W)
    out = M.mp_posterior()
    for p_dev, w_dev in ((True, False), (False, True), (True, True)):
        p, w = torch.zeros((n, 7)), torch.zeros(n, dtype=torch.float64)
        p, w = (p.cuda() if p_dev else p), (w.cuda() if w_dev else w)
        M._check(M.lib().mp_posterior_query(f.handle, C.byref(out), M._ptr(p), M._ptr(w), M._stream(None)))
        assert np.array_equal(p.cpu().numpy(), P) and np.array_equal(w.cpu().numpy(), W)
        assert out.map_index == q["map_index"]
    # a value that is not finite, in the last piece
    bad = f.debug_get("poses")
    bad[n - 1, 5] = np.inf
    f.debug_set("poses", bad)
    got = np.zeros((n, 7), np.float32)
    assert M.lib().mp_posterior_query(f.handle, C.byref(out), M._ptr(got), None, M._stream(None)) == M.MP_E_NUMERIC
    assert np.array_equal(got, bad[:, :7])
    f.close()


def test_a_query_takes_no_device_memory(world):
    import torch
    n = 1 << 20
    f = M.Filter(world, M.mp_filter_default_params(n_particles=n, k=4, svgd_iters=1))
    f.posterior_query()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    q = f.posterior_query(poses=True, weights=True)
    assert torch.cuda.mem_get_info()[0] >= free
    assert np.array_equal(q["poses"], f.debug_get("poses")[:, :7])
    f.close()
