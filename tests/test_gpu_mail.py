"""Results that come back through pinned boxes: forty threads with a handle and a stream each (more than there are boxes: some calls copy instead),
a running best that changes and one that stays between questions, a handle that has nothing to report, and one after a reset."""
import threading

import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import gpu  # noqa: F401

pytestmark = pytest.mark.gpu
PROBLEMS = [W.config3(), W.kshape_problem(4, 4), W.config4(), W.config1()]


def _answer(g):
    b = g.best()
    out = {k: b[k] for k in ("period", "index", "peak", "n_evaluated", "n_feasible", "n_reject", "feasible")}
    if b["feasible"]:
        c = g.best_candidate()
        out["candidate"] = (c["leads"], c["orders"], c["starts"].tolist())
    return out


def _walk(gpu, prob, salt, stream=None):
    """answers after each of six pieces of a range, asked twice, then of a new search"""
    g, out = gpu.Problem(prob), []
    space = min(g.candidate_count(), 1 << 30)
    for k in range(6):
        first = (salt * 7919 + k * 30011) % max(1, space - 600)
        g.eval_candidates(first, 500, stream=stream)
        out += [_answer(g), _answer(g)]
    g.reset()
    out.append(_answer(g))
    g.eval_candidates(0, 500, stream=stream)
    out.append(_answer(g))
    return out


def test_answers_of_many_threads(gpu):  # noqa: F811
    import torch
    want = {k: _walk(gpu, PROBLEMS[k % 4], k) for k in range(8)}
    got, failed = {}, []

    def work(k):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                got[k] = _walk(gpu, PROBLEMS[k % 4], k % 8, stream.cuda_stream)
            stream.synchronize()
        except Exception as e:          # noqa: BLE001 (reported below, with the thread's number)
            failed.append((k, repr(e)))
    threads = [threading.Thread(target=work, args=(k,)) for k in range(40)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    for k in range(40):
        assert got[k] == want[k % 8], k


@pytest.mark.parametrize("k", range(4))
def test_one_question_after_another(gpu, k):  # noqa: F811
    """asked after every piece, or once at the end: the same"""
    prob = PROBLEMS[k]
    g, once = gpu.Problem(prob), gpu.Problem(prob)
    space = min(g.candidate_count(), 4000)
    for at in range(0, space, 96):
        n = min(96, space - at)
        g.eval_candidates(at, n)
        once.eval_candidates(at, n)
        a = _answer(g)
        assert a == _answer(g)
    assert a == _answer(once)


def _hip_runtime():
    """the HIP runtime this process has loaded"""
    import ctypes as C
    return C.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))


def test_error_of_an_earlier_call(gpu):  # noqa: F811
    """A call that failed on this thread before (a device number there is not) is no failure of the launch that sends the mail: the box
    would go back while the kernel is on its way.  More questions than there are boxes, changing answers, a completion each."""
    hip = _hip_runtime()
    g, want = gpu.Problem(W.config3()), gpu.Problem(W.config3())

    def behind_an_error(ask):
        assert hip.hipSetDevice(1000) != 0
        try:
            return ask()
        finally:
            hip.hipGetLastError()

    for k in range(40):
        for p in (g, want):
            p.reset()
            p.eval_candidates(5003 * k, 400 + k)
        assert behind_an_error(lambda: _answer(g)) == _answer(want), k
        for p in (g, want):
            p.search_completions(16, 2, 70 * k, 64)
        assert behind_an_error(lambda: g.best_completion(16)["ordinal"]) == want.best_completion(16)["ordinal"], k


@pytest.mark.parametrize("k", range(4))
def test_copied_results(gpu, monkeypatch, k):  # noqa: F811
    """a call that finds no box copies: the same answers, to questions asked twice, after a reset, with and without anything to report, and
    the same completion"""
    want = _walk(gpu, PROBLEMS[k], 3 + k)
    monkeypatch.setenv("TESSEL_MAIL", "0")
    assert _walk(gpu, PROBLEMS[k], 3 + k) == want
    copied = gpu.Problem(W.config3())
    monkeypatch.delenv("TESSEL_MAIL")
    mailed = gpu.Problem(W.config3())
    got = []
    for g in (mailed, copied):
        with pytest.raises(gpu.TesselError) as e:
            g.best_completion(16)                                # nothing searched yet
        assert e.value.code == -7
        g.eval_candidates(100 * k, 400)
        for _ in range(2):
            g.search_completions(16, 2, 7 * k, 50 + k)
            b = g.best_completion(16)
            got.append((b["makespan"], b["ordinal"], b["start"].tolist()))
    assert got[:2] == got[2:]
