"""What pmace_simulate and pmace_simulate_static do beside their counts: a
position outside the object is refused with the output untouched, and a call
that returns no scale waits for the check of the positions only."""
import ctypes

import numpy as np
import pytest

from paper_2111_14240_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2111_14240_amd import pmace
    pmace.load_library()
    return pmace


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("np_", [32, 128, 160, 256])
@pytest.mark.parametrize("peak", [0.0, 1e5])
def test_refused_positions_leave_the_output(P, np_, static, peak):
    prob = synth.make_problem(np_ + 60, np_, 3, 25, None, seed=np_)
    n1, n2 = prob.x_true.shape
    call = P.simulate_static if static else P.simulate
    for bad in ([-1, 0], [0, -1], [n1 - np_ + 1, 0], [0, n2 - np_ + 1], [2**31 - 1, -2**31]):
        for at in (0, len(prob.pos) - 1):
            pos = np.array(prob.pos, np.int32)
            pos[at] = bad
            z = torch.full((len(pos), np_, np_), -7.0, device="cuda")
            print("[gpu-refused]", np_, static, peak, bad, at, flush=True)
            with pytest.raises(P.PMACEError) as e:
                call(prob.x_true, prob.probe, pos, peak, 3, out=z)
            assert e.value.status == P.PMACE_EINVAL
            torch.cuda.synchronize()
            assert bool((z == -7.0).all())


@pytest.mark.parametrize("static", [False, True])
def test_without_scale_the_call_does_not_wait(P, static):
    """20000 patterns of 128^2 keep the GPU busy for milliseconds after the
    positions are known to be good."""
    np_, n, J = 128, 400, 20000
    rng = np.random.default_rng(2)
    x = P.to_device_c64(synth.make_object(n, n, rng), "cuda")
    d = P.to_device_c64(synth.make_probe(np_), "cuda")
    pos = torch.as_tensor(rng.integers(0, n - np_ + 1, (J, 2)), dtype=torch.int32, device="cuda")
    z = torch.empty((J, np_, np_), device="cuda")
    lib = P.load_library()
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = torch.cuda.current_stream()
    sp = ctypes.c_void_p(int(stream.cuda_stream))
    ws = torch.empty(int(lib.pmace_simulate_footprint(np_, J)), dtype=torch.uint8, device="cuda")
    scale = ctypes.c_double()
    counts = []
    for want in (True, False):
        z.fill_(-7.0)
        torch.cuda.synchronize()
        sc = ctypes.byref(scale) if want else None
        if static:
            st = lib.pmace_simulate_static(n, n, np_, J, ptr(d), ptr(pos), ptr(x), 1e5, 9, ptr(z), sc, sp)
        else:
            st = lib.pmace_simulate(n, n, np_, J, ptr(d), ptr(pos), ptr(x), 1e5, 9, ptr(z), ptr(ws), ws.numel(),
                                    sc, sp)
        done = stream.query()
        assert st == P.PMACE_OK
        torch.cuda.synchronize()
        counts.append(z.clone())
        print("[gpu-refused] done at return", static, want, done, flush=True)
        assert done == want
    assert bool((counts[0] == counts[1]).all())
