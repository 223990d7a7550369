"""NaN and Inf that take no part in a result must not reach it.

* a starting object whose unscanned pixels are NaN or Inf: only its covered
  pixels are read, so the run equals, bit for bit, the one with zeros there;
* a state with a NaN in its first element: no other pixel reads that element
  (the gather's last group of list entries is filled up, and its lanes go over
  pixels that an entry's patch does not cover)."""
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


@pytest.mark.parametrize("np_,chunk,J", [(32, 0, 1), (32, 0, 5), (48, 0, 8), (64, 0, 9), (128, 0, 7), (160, 3, 7)])
def test_first_element_of_a_state_stays_its_own(P, np_, chunk, J):
    n1, n2 = np_ + 40, np_ + 90
    rng = np.random.default_rng(J)
    pos = np.stack([rng.integers(0, 41, J), rng.integers(0, 91, J)], 1).astype(np.int32)
    d, z, x0 = _inputs(n1, n2, np_, pos, 7 * np_)
    print("[gpu-nonfinite] first element", np_, chunk, J, flush=True)
    R = P.Reconstruction(n1, n2, d, pos, z, 0.5, flags=P.PMACE_STAGED_AGENT if np_ > 128 else 0, chunk=chunk)
    v = np.stack([x0[r:r + np_, c:c + np_] for r, c in pos])
    for j in range(J):
        R.set_state(v)
        ref = R.reconstruct().cpu().numpy()
        w = v.copy()
        w[j, 0, 0] = np.nan
        R.set_state(w)
        got = R.reconstruct().cpu().numpy()
        others = np.ones((n1, n2), bool)
        others[tuple(pos[j])] = False
        assert np.array_equal(got[others], ref[others]), j
    R.close()
