"""What mp_stage_times waits for."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2404_16370_amd import megapf as M


@pytest.fixture(scope="module")
def world():
    return M.Map(np.random.default_rng(0).uniform(-5, 5, (20_000, 3)).astype(np.float32), voxel=0.5)


def _filter(world, n=500):
    return M.Filter(world, M.mp_filter_default_params(n_particles=n, k=8, svgd_iters=2, d_max=1.0))


SCAN = np.random.default_rng(1).uniform(-5, 5, (300, 3)).astype(np.float32)


@pytest.mark.parametrize("upload_only", [False, True])
def test_other_streams_are_not_waited_for(world, upload_only):
    import torch
    f = _filter(world)
    own = torch.cuda.Stream()

    def work():
        f.scan_upload(SCAN, stream=own.cuda_stream)
        if not upload_only:
            f.step(stream=own.cuda_stream)

    work()
    f.stage_times()
    for _ in range(12):   # (streams share a few hardware queues: until one that `own` does not wait for)
        other = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            torch.cuda._sleep(600_000_000)   # some 0.25 s
        work()
        own.synchronize()
        if not other.query():
            break
    else:
        pytest.skip("every stream shares the filter's hardware queue")
    st = f.stage_times()
    assert not other.query()
    assert st["scan"][1] == 1 and 0.0 < st["scan"][0] < 100.0
    assert st["likelihood"][1] == (0 if upload_only else 2)
    torch.cuda.synchronize()
    f.close()


def test_the_filters_own_work_is_waited_for(world):
    # the step is behind other work of its stream, the upload on another one
    import torch
    f = _filter(world, 3000)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        f.scan_upload(SCAN, stream=a.cuda_stream)
        a.synchronize()
        with torch.cuda.stream(b):
            torch.cuda._sleep(100_000_000)
        f.step(stream=b.cuda_stream)
        st = f.stage_times()
        psi = f.debug_get("psi", stream=a.cuda_stream)   # not ordered behind the step but by the call above
        b.synchronize()
        assert np.array_equal(psi, f.debug_get("psi"))
        for name, count in (("lsh", 2), ("sort", 2), ("refresh", 2), ("likelihood", 2), ("svgd", 2), ("posterior", 1), ("scan", 1)):
            assert st[name][1] == count and 0.0 <= st[name][0] < 100.0, st
        assert st["posterior"][0] > 0.0 and st["likelihood_core"][0] > 0.0
    f.close()


def test_a_stream_that_is_gone(world):
    import torch
    hip = C.CDLL("libamdhip64.so")
    f = _filter(world)
    s = C.c_void_p()
    assert hip.hipStreamCreate(C.byref(s)) == 0
    f.scan_upload(SCAN, stream=s.value)
    f.step(stream=s.value)
    assert hip.hipStreamSynchronize(s) == 0 and hip.hipStreamDestroy(s) == 0
    st = f.stage_times()
    assert st["svgd"][1] == 2 and st["scan"][0] > 0.0
    f.scan_upload(SCAN)
    f.step()
    assert f.stage_times()["svgd"][1] == 2
    f.close()


def test_times_of_steps_and_uploads_in_any_turn(world):
    # asked for after each of a sequence, or only at its end: the same spans
    import torch
    a, b = _filter(world), _filter(world)
    dT = np.array([1, 0, 0, 0, 0, 0, 0], np.float32)
    for what in ("scan", "step", "step", "scan", "scan", "step", "pred", "empty", "pred", "scan", "step", "step"):
        for f in (a, b):
            if what == "scan":
                f.scan_upload(SCAN)
            elif what == "empty":
                f.scan_upload(np.zeros((0, 3), np.float32))
            else:
                f.step(dT if what == "pred" else None)
        st = a.stage_times()
        assert all(0.0 <= ms < 100.0 for ms, _ in st.values()), (what, st)
        if what == "step":
            assert st["svgd"][1] == 2 and st["svgd"][0] > 0.0 and st["scan"][0] > 0.0
    assert {k: v[1] for k, v in b.stage_times().items()} == {k: v[1] for k, v in a.stage_times().items()}
    torch.cuda.synchronize()
    assert a.stage_times() == a.stage_times()
    for f in (a, b):
        f.close()
