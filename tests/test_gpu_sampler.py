"""The simulator's in-place Poisson counts against the sampler run one element
per thread on the same means and streams: equal count for count, at pattern
sizes around a workgroup's share of elements and over dark, mixed and bright
patterns."""
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


@pytest.mark.parametrize("np_,count", [(32, 1), (48, 7), (48, 57), (160, 3), (160, 331)])
@pytest.mark.parametrize("peak", [0.4, 12.0, 1e4, 1e8])
def test_counts_equal_the_plain_sampler(P, np_, count, peak):
    prob = synth.make_problem(np_ * 2, np_, 3, np_ // 3, None, seed=np_)
    pos = np.resize(prob.pos, (count, 2))
    z0, _ = P.simulate(prob.x_true, prob.probe, pos, None, seed=9)
    z, scale = P.simulate(prob.x_true, prob.probe, pos, peak, seed=9)
    lam = z0.cpu().numpy().astype(np.float64).ravel() * scale
    print(f"[gpu-sampler] np {np_} x {count}, peak {peak:g}: {np.mean(lam < 0.1):.3f} of the means under 0.1, "
          f"{np.mean(lam >= 10):.3f} of 10 and more", flush=True)
    assert np.array_equal(z.cpu().numpy().ravel(), P.poisson(lam, seed=9))
