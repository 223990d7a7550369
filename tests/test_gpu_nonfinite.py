"""NaN and Inf that take no part in a result must not reach it.

* a starting object whose unscanned pixels are NaN or Inf: only its covered
  pixels are read, so the run equals, bit for bit, the one with zeros there."""
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


def _inputs(n1, n2, np_, pos, seed):
    rng = np.random.default_rng(seed)
    x = synth.make_object(max(n1, n2), max(n1, n2), rng)[:n1, :n2]
    d = (synth.make_probe(np_) * 30).astype(np.complex64)
    z, _ = synth.simulate_intensities(x.astype(complex), d.astype(complex), pos, None, rng)
    x0 = synth.make_object(max(n1, n2), max(n1, n2), rng)[:n1, :n2].astype(np.complex64)
    return d, z, x0


@pytest.mark.parametrize("np_,agent,chunk", [(64, "whole patch", 0), (128, "split", 0), (160, "three-pass", 2),
                                             (192, "row-spectrum", 0), (256, "row-spectrum", 2)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_unscanned_start_pixels_are_not_read(P, np_, agent, chunk, bad):
    n1, n2 = np_ + 37, np_ + 75
    pos = np.array([[3, 5], [20, 9], [11, 40], [3, 5], [17, 33]], np.int32)
    d, z, x0 = _inputs(n1, n2, np_, pos, np_)
    covered = np.zeros((n1, n2), bool)
    for r, c in pos:
        covered[r:r + np_, c:c + np_] = True
    flags = {"split": P.PMACE_SPLIT_AGENT, "three-pass": P.PMACE_STAGED_AGENT,
             "row-spectrum": P.PMACE_ROWSPEC_AGENT}.get(agent, 0)
    got = []
    for outside in (0, bad):
        print("[gpu-nonfinite] start", np_, agent, outside, flush=True)
        start = np.where(covered, x0, np.complex64(complex(outside, outside)))
        R = P.Reconstruction(n1, n2, d, pos, z, 0.5, x0=start, flags=flags, chunk=chunk)
        assert R.agent == agent
        R.iterate(3)
        R.sync()
        got.append((R.get_state().cpu().numpy(), R.reconstruct().cpu().numpy()))
        R.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    assert np.isfinite(got[1][1]).all()
