"""The set-up's device-built lists: one pass from a smooth start against the
oracle, where a list can go wrong: more positions than a workgroup's batch of
256, tile rows wider than a panel of 1024 tiles, several chunks with a ragged
last one, equal columns and repeated positions (ties), rows that no patch
covers, an object row in two segments; and the 256-point row pass where it
starts to take several positions per workgroup.  The bar is that of the parity
tests."""
import numpy as np
import pytest

from oracle import pmace_oracle as O
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


def _smooth(n1, n2, rng):
    x = synth.make_object(max(n1, 64), max(n2, 64), rng)
    return x[:n1, :n2].astype(np.complex64)


CASES = [
    # np, n1, n2, J, chunk, where the positions go
    (32, 70, 33000, 300, 0, "spread"),      # 1032 tile columns, two batches
    (48, 150, 97, 1, 0, "spread"),
    (64, 200, 131, 257, 0, "two columns"),
    (128, 400, 300, 40, 0, "corners"),      # rows in the middle uncovered
    (160, 300, 1300, 70, 33, "spread"),     # two segments, three chunks
    (192, 260, 300, 65, 0, "same"),
    (256, 300, 400, 17, 5, "two columns"),
    # row passes of several positions per workgroup: from 128 on, and a remainder
    (256, 300, 330, 127, 0, "spread"),
    (256, 300, 330, 128, 0, "spread"),
    (256, 300, 330, 201, 0, "spread"),
]


@pytest.mark.parametrize("np_,n1,n2,J,chunk,where", CASES)
def test_first_pass_matches_oracle(P, np_, n1, n2, J, chunk, where):
    rng = np.random.default_rng(np_ + J)
    pos = np.stack([rng.integers(0, n1 - np_ + 1, J), rng.integers(0, n2 - np_ + 1, J)], 1)
    if where == "two columns":
        pos[:, 1] = np.where(np.arange(J) % 3, 1, n2 - np_)
    elif where == "same":
        pos[:] = pos[0]
    elif where == "corners":
        pos = np.where(np.arange(J)[:, None] % 2, pos % 5, [n1 - np_, n2 - np_] - pos % 5)
    pos = pos.astype(np.int32)
    x, x0 = _smooth(n1, n2, rng), _smooth(n1, n2, rng)
    d = (synth.make_probe(np_) * 30).astype(np.complex64)
    z, _ = synth.simulate_intensities(x.astype(complex), d.astype(complex), pos, None, rng)
    print("[gpu-setup]", np_, n1, n2, J, chunk, where, flush=True)
    R = P.Reconstruction(n1, n2, d, pos, z, 0.5, 1.25, 0.5, x0=x0, chunk=chunk)
    shape = (n1, n2)
    covered = np.zeros(shape, bool)
    for r, c in pos:
        covered[r:r + np_, c:c + np_] = True
    assert np.array_equal(R.reconstruct().cpu().numpy(), np.where(covered, x0, 0))
    R.iterate(1)
    st = O.pmace_init(x0.astype(complex), pos, np_)
    st = O.pmace_iterate(st, d.astype(complex), O.amplitudes(z), pos, shape, 0.5, 1.25, 0.5, 1)
    for got, ref in ((R.get_state(), st.v), (R.reconstruct(), O.reconstruct(st, d.astype(complex), pos, shape, 1.25))):
        got = got.cpu().numpy()
        e = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"[gpu-setup]   rel {e:.2e} max {np.abs(got - ref).max() / np.abs(ref).max():.2e}", flush=True)
        assert e <= 1e-4 and np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    R.close()


SPARSE = [
    # np, n1, n2, J, chunk, agent: most gather tiles (row-spectrum: row items)
    # list nothing, and are left out
    (32, 600, 1100, 9, 0, ""),
    (64, 1024, 1024, 2, 0, ""),
    (96, 97, 4000, 3, 0, ""),               # rows of many tiles, few of them kept
    (128, 900, 700, 5, 0, ""),
    (160, 800, 1300, 9, 4, "staged"),       # chunks whose rows span the object
    (160, 2100, 4200, 6, 0, "rowspec"),     # segments without an item
    (256, 2000, 5200, 5, 3, "rowspec"),
]


@pytest.mark.parametrize("np_,n1,n2,J,chunk,agent", SPARSE)
def test_sparse_scans_match_oracle(P, np_, n1, n2, J, chunk, agent):
    """One pass and the states set again, on positions far apart."""
    rng = np.random.default_rng(np_ + J)
    pos = np.stack([rng.integers(0, n1 - np_ + 1, J), rng.integers(0, n2 - np_ + 1, J)], 1)
    pos[0], pos[-1] = 0, [n1 - np_, n2 - np_]
    pos = pos.astype(np.int32)
    x, x0 = _smooth(n1, n2, rng), _smooth(n1, n2, rng)
    d = (synth.make_probe(np_) * 30).astype(np.complex64)
    z, _ = synth.simulate_intensities(x.astype(complex), d.astype(complex), pos, None, rng)
    print("[gpu-setup] sparse", np_, n1, n2, J, chunk, agent, flush=True)
    flags = {"staged": P.PMACE_STAGED_AGENT, "rowspec": P.PMACE_ROWSPEC_AGENT}.get(agent, 0)
    R = P.Reconstruction(n1, n2, d, pos, z, 0.5, 1.25, 0.5, x0=x0, chunk=chunk, flags=flags)
    R.iterate(1)
    shape, dd = (n1, n2), d.astype(complex)
    st = O.pmace_init(x0.astype(complex), pos, np_)
    st = O.pmace_iterate(st, dd, O.amplitudes(z), pos, shape, 0.5, 1.25, 0.5, 1)
    ref = O.reconstruct(st, dd, pos, shape, 1.25)
    got = [R.get_state().cpu().numpy(), R.reconstruct().cpu().numpy()]
    R.set_state(st.v)
    got.append(R.reconstruct().cpu().numpy())
    R.sync()
    for g, r in zip(got, (st.v, ref, ref)):
        e = np.linalg.norm(g - r) / np.linalg.norm(r)
        print(f"[gpu-setup]   rel {e:.2e} max {np.abs(g - r).max() / np.abs(r).max():.2e}", flush=True)
        assert e <= 1e-4 and np.abs(g - r).max() <= 1e-4 * np.abs(r).max()
    R.close()


def test_captured_iterations_equal_launched_ones(P):
    """Np <= 64 replays a captured graph once 256 iterations have been asked
    for; the same number of iterations, launched in small calls, gives the
    same bits."""
    prob = synth.make_problem(96, 32, 3, 20, 1e5, 5)
    got = []
    for calls in ([130, 131, 40], [1] * 301):
        R = P.Reconstruction(prob.n1, prob.n2, prob.probe, prob.pos, prob.z, 0.5)
        for n in calls:
            R.iterate(n)
        got.append((R.get_state().cpu().numpy(), R.reconstruct().cpu().numpy()))
        R.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("np_,before", [(64, 0), (64, 300), (256, 0)])
def test_iterations_captured_by_the_caller(P, np_, before):
    """iterate() recorded into a caller's graph, on a reconstruction that has
    been in a batch and (before = 300) has a graph of its own: every replay,
    with other calls between them, equals the same iterations launched."""
    prob = synth.make_problem(2 * np_, np_, 3, np_ // 3, 1e5, 11)
    stream = torch.cuda.Stream()
    got = []
    for capture in (False, True):
        with torch.cuda.stream(stream):
            R = P.Reconstruction(prob.n1, prob.n2, prob.probe, prob.pos, prob.z, 0.5, stream=stream)
            B = P.Batch([R], tol=0.0, min_iter=0, max_iter=2)
            B.step(3)
            assert B.poll()[0].tolist() == [1]
            B.close()
            R.iterate(before)
            R.sync()
            graph = torch.cuda.CUDAGraph()
            if capture:
                print("[gpu-setup] caller's capture", np_, before, flush=True)
                with torch.cuda.graph(graph, stream=stream):
                    R.iterate(33)
            out = []
            for _ in range(3):
                graph.replay() if capture else R.iterate(33)
                R.sync()
                out.append(R.reconstruct().cpu().numpy())
                R.iterate(1)
            out.append(R.get_state().cpu().numpy())
            R.close()
        got.append(out)
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("np_", [48, 64])
def test_captured_iterations_of_other_sides(P, np_):
    """As test_captured_iterations_equal_launched_ones for the other sides that
    are captured, against the kernels launched because a call is too short."""
    prob = synth.make_problem(3 * np_, np_, 4, np_ // 2, 1e5, 5 + np_)
    got = []
    for calls in ([130, 131, 40], [31] * 9 + [22]):
        R = P.Reconstruction(prob.n1, prob.n2, prob.probe, prob.pos, prob.z, 0.5)
        for n in calls:
            R.iterate(n)
        R.sync()
        got.append((R.get_state().cpu().numpy(), R.reconstruct().cpu().numpy()))
        R.close()
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
