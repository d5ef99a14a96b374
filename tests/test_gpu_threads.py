"""Synchronous calls from several host threads, each on its own stream, give
the results of the same calls made alone (each call borrows its own page of
pinned host memory for its small results), also when no page can be had."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gpz():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_10305_amd as g
    g.lib()
    return g


def one_user(gpz, k, rounds, out):
    """Round trips and reports of one thread's snapshots, as host values."""
    rng = np.random.default_rng(k)
    with torch.cuda.stream(torch.cuda.Stream()):
        for r in range(rounds):
            n, F = 500 + 997 * ((k * 7 + r) % 9), 1 + (k + r) % 4
            B = (1024, 512, 128)[(k + r) % 3]  # the usual parameters, and others
            host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
            dev = [torch.from_numpy(h).cuda() for h in host]
            ws = gpz.stats_workspace(F)
            eb = gpz.rel_ebs(dev, 1e-3, ws=ws)
            stream, perm = gpz.compress(dev, eb, block_size=B, want_perm=True)
            back = gpz.decompress(stream, n, F)
            st = gpz.error_stats(dev, back, eb, perm=perm, ws=ws)
            outliers, raw = gpz.stream_stats(stream, n, F, ws=ws)
            assert int(st["violations"].sum()) == 0
            out.append((stream.cpu().numpy().tobytes(), [b.cpu().numpy().tobytes() for b in back],
                        st["max_abs_err"].tolist(), st["range"].tolist(), outliers.tolist(), raw))
            with pytest.raises(gpz.GpzError):  # one word short: refused
                gpz.decompress(stream[:-4], n, F)


@pytest.mark.parametrize("fault", [False, True])
def test_threads_get_their_own_results(gpz, fault, monkeypatch):
    users, rounds = 8, 6
    alone = []
    for k in range(users):
        alone.append([])
        one_user(gpz, k, rounds, alone[-1])
    if fault:
        monkeypatch.setenv("GPZ_FAULT", "alloc")  # no new page: those at hand, then plain copies
    got = [[] for _ in range(users)]
    errors = []

    def body(k):
        try:
            one_user(gpz, k, rounds, got[k])
        except BaseException as e:  # noqa: BLE001 (reported by the main thread)
            errors.append(repr(e))
    threads = [threading.Thread(target=body, args=(k,)) for k in range(users)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not errors, errors
    assert got == alone
