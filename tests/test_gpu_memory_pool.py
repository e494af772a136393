"""Reuse of the memory of freed graphs and finished builds: blocks pass between sizes, streams and
threads, and the results are those of first builds."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _check(mg, case, stream):
    src, dst, n, want = case
    with torch.cuda.stream(stream):
        g = mg.build_csr(src, dst, n, stream=stream)
        mg.normalize(g, stream=stream)
        stream.synchronize()
        a = g.arrays()
    assert np.array_equal(a["rowptr"].cpu().numpy(), want.rowptr)
    assert np.array_equal(a["col"].cpu().numpy().view(np.uint32), want.col)
    assert np.array_equal(a["deg"].cpu().numpy().view(np.uint32), np.diff(want.rowptr))
    g.free()


@pytest.mark.parametrize("n_threads", [1, 4])
def test_builds_in_reused_memory(n_threads):
    """Each thread builds and frees graphs of different sizes on a stream of its own; the cache is
    given back in the middle."""
    import paper_2501_01951_amd as mg

    mg.load_library()
    cases = []
    for scale in (6, 9, 12, 13):
        src, dst, n = gg.config_graph("c2", scale_override=scale)
        cases.append((torch.from_numpy(src.view(np.int32)).cuda(),
                      torch.from_numpy(dst.view(np.int32)).cuda(), n, oracle.build_csr(src, dst, n)))
    torch.cuda.synchronize()
    errors = []

    def work(t):
        try:
            stream = torch.cuda.Stream()
            for k in range(12):
                _check(mg, cases[(t + k) % len(cases)], stream)
                if k == 6 and t == 0:
                    mg.release_memory()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(t,)) for t in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
