"""Several host threads driving their own handles at once (as the server's
worker threads do): fused SV circuits with gate products and fused DM
circuits with queued one- and two-qubit superoperators, each thread on its own
stream.  Every result must equal the same work done on one thread, bit for
bit (the kernels are deterministic), and nothing may fail."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nwq():
    from paper_2401_06861_amd import nwq as mod
    return mod


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


def _sv_job(nwq, torch, seed):
    n = 16
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = nwq.SVState(n, stream=stream, owned=True)
        try:
            st.set_fusion(12 + seed % 2)
            nwq.nwq_run_circuit(st.h, *nwq.circuit_arrays(W.brickwork_circuit(n, 12, seed=seed)))
            return np.array(st.expvals(W.single_site_terms(n, "Z")))
        finally:
            st.close()


def _dm_job(nwq, torch, seed):
    n = 8
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        st = nwq.DMState(n, stream=stream, owned=True)
        try:
            st.set_fusion(12)
            st.run(W.noisy_tfim_circuit(n, 3 + seed % 3))
            return np.array(st.expvals(W.single_site_terms(n, "Z"))), st.purity()
        finally:
            st.close()


def test_concurrent_handles_match_one_thread(nwq, torch):
    jobs = [(_sv_job, s) for s in range(4)] + [(_dm_job, s) for s in range(4)]
    want = [fn(nwq, torch, s) for fn, s in jobs]
    got = [None] * len(jobs)
    errors = []

    def work(i):
        try:
            torch.cuda.set_device(0)
            for _ in range(3):
                got[i] = jobs[i][0](nwq, torch, jobs[i][1])
        except Exception as e:   # reported below, not lost in the thread
            errors.append(repr(e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i, (w, g) in enumerate(zip(want, got)):
        if isinstance(w, tuple):
            assert np.array_equal(w[0], g[0]) and w[1] == g[1], i
        else:
            assert np.array_equal(w, g), i


def test_first_circuit_while_another_thread_captures(nwq, torch):
    """A handle's first circuit allocates its upload ring; a graph that another
    thread captures in global mode (torch's default) meanwhile stays valid, and
    the circuit gives the bits that it gives without a capture."""
    n = 8
    arrays = nwq.circuit_arrays(W.random_gate_list(n, 300, seed=3))

    def handle():
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            return nwq.SVState(n, stream=stream, owned=True)

    quiet = handle()
    nwq.nwq_run_circuit(quiet.h, *arrays)
    want = quiet.numpy()
    quiet.close()
    st, errors = handle(), []
    x = torch.zeros(1 << 10, device="cuda")
    torch.cuda.synchronize()

    def work():
        try:
            nwq.nwq_run_circuit(st.h, *arrays)
        except Exception as e:          # reported below, on the test's thread
            errors.append(e)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x += 1.0
        t = threading.Thread(target=work)
        t.start()
        t.join()
        x += 1.0
    assert not errors
    for i in range(3):
        g.replay()
        assert x[0].item() == 2.0 * (i + 1)
        assert np.array_equal(st.numpy(), want)
    st.close()


def test_upload_ring_grows_and_wraps(nwq, torch):
    """Circuits with no read in between whose programs pass the end of the
    first upload ring (256 KiB) and of the second (4 MiB): every program arrives
    whole (the same bits as with a read after each)."""
    n = 10
    circuits = [nwq.circuit_arrays(W.random_gate_list(n, 1500, seed=s)) for s in range(40)]
    states, grown = [], []
    for read in (False, True):
        st = nwq.SVState(n)
        empty = nwq.nwq_memory(st.h)
        for c in circuits:
            nwq.nwq_apply_circuit(st.h, *c)
            grown.append(nwq.nwq_memory(st.h) - empty)
            if read:
                st.numpy()
        states.append(st.numpy())
        st.close()
    assert np.array_equal(*states)
    assert grown[0] >= 256 << 10 and grown[39] == (4 << 20) + (256 << 10) and grown[:40] == grown[40:]
    assert abs(np.sum(np.abs(states[0]) ** 2) - 1.0) <= 1e-10
