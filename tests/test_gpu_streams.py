"""Calls on different streams with different workspaces may overlap (the
library keeps no state between calls): two host threads, each on a stream of
its own, run the kNN and LOF entry points on different inputs at the same
time, and every result must equal the same call made alone."""
import sys
import threading

import numpy as np
import pytest

from paper_2110_14007_amd import workloads

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def test_two_threads_two_streams():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    from paper_2110_14007_amd import tod

    x1, _ = workloads.generate("C2", n=20000)
    x2, _ = workloads.generate("C1")
    a1 = torch.from_numpy(x1).cuda()
    a2 = torch.from_numpy(x2).cuda()
    torch.cuda.synchronize()
    say("serial reference runs")
    ref1 = [t.cpu().numpy() for t in tod.tod_knn(a1, a1, 20)]
    ref2 = [t.cpu().numpy() for t in tod.tod_lof(a2, 10)]
    torch.cuda.synchronize()

    results = {}
    errors = []

    def worker(name, fn):
        try:
            s = torch.cuda.Stream()  # default priority
            ws = tod.Workspace()
            out = []
            for _ in range(4):
                out.append([t.cpu().numpy() for t in fn(ws, s)])
            results[name] = out
        except Exception as e:  # reported below, after both threads end
            errors.append(repr(e))

    t1 = threading.Thread(target=worker, args=(
        "knn", lambda ws, s: tod.tod_knn(a1, a1, 20, workspace=ws, stream=s)))
    t2 = threading.Thread(target=worker, args=(
        "lof", lambda ws, s: tod.tod_lof(a2, 10, workspace=ws, stream=s)))
    say("two threads")
    t1.start()
    t2.start()
    t1.join()
    t2.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for got in results["knn"]:
        np.testing.assert_array_equal(got[0], ref1[0])
        np.testing.assert_array_equal(got[1], ref1[1])
    for got in results["lof"]:
        np.testing.assert_array_equal(got[0], ref2[0])
        np.testing.assert_array_equal(got[1], ref2[1])


def test_two_threads_different_lds():
    # The pruned scan's preparation takes LDS by the row length.  Two threads whose
    # calls need 43 KB and 147 KB of it for the same kernel, many times over.
    import torch
    from paper_2110_14007_amd import tod

    rng = np.random.default_rng(3)
    xs = [torch.from_numpy(rng.standard_normal((3000, d)).astype(np.float32)).cuda()
          for d in (20, 100)]
    opt = dict(reorder=1, ref_splits=1)
    refs = [tod.tod_knn_score(x, 5, tod.options(**opt), return_lists=True) for x in xs]
    torch.cuda.synchronize()
    errors = []

    def worker(x, ref):
        try:
            s, ws = torch.cuda.Stream(), tod.Workspace()
            for i in range(200):
                got = tod.tod_knn_score(x, 5, tod.options(**opt), ws, stream=s, return_lists=True)
                s.synchronize()
                if not all(torch.equal(a, b) for a, b in zip(got, ref)):
                    raise AssertionError("call %d differs" % i)
        except Exception as e:  # reported below, after both threads end
            errors.append(repr(e))

    threads = [threading.Thread(target=worker, args=a) for a in zip(xs, refs)]
    say("two threads, two row lengths")
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
