"""GPU parity of the error report (bound check, sums of squares, range) at the
edges of its 1024-position chunks, against the CPU oracle.

Counts, maxima and ranges are exact.  A sum of squares adds at most n
non-negative terms, each rounded once, in another order than the oracle's:
n * 2^-52 relative bounds the difference."""
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


def permutation(kind, n, rng):
    """None, block-local (what compression returns), over the whole array, or
    one with duplicates and entries past the end."""
    if kind == "none":
        return None
    p = np.arange(n, dtype=np.uint32)
    if kind == "local":
        for b in range(0, n, 1024):
            p[b:b + 1024] = b + rng.permutation(min(1024, n - b))
    else:
        p = rng.permutation(n).astype(np.uint32)
    if kind == "broken":
        p[rng.integers(0, n, max(1, n // 50))] = n
        p[0] = 0xFFFFFFFF
        p[n // 2] = p[n - 1]
    return p


@pytest.mark.parametrize("kind", ["none", "local", "whole", "broken"])
@pytest.mark.parametrize("n,F,shift", [(1, 1, 0), (63, 2, 1), (1023, 3, 0), (1024, 1, 0),
                                       (1025, 2, 3), (4097, 64, 0), (300_001, 6, 1)])
@pytest.mark.parametrize("special", [False, True])
def test_report_at_chunk_edges(gpz, orc, n, F, shift, kind, special):
    print(f"[case] report n={n} F={F} shift={shift} perm={kind} special={special}", flush=True)
    rng = np.random.default_rng(n * 131 + F)
    perm = permutation(kind, n, rng)
    pad = shift  # fields start `shift` floats past an aligned address
    x = [(rng.standard_normal(n + pad) * 10.0 ** (f % 4)).astype(np.float32) for f in range(F)]
    eb = np.array([10.0 ** (f % 4 - 3) for f in range(F)], np.float32)
    if special:
        for f in range(F):
            for v in (np.nan, np.inf, -np.inf, -0.0):
                x[f][pad + rng.integers(0, n)] = v
        x[F - 1][:] = np.nan
    src = np.arange(n) if perm is None else np.minimum(perm, n - 1)
    # most pairs inside the bound, some outside, non-finite values kept or lost
    y = []
    for f in range(F):
        noise = (rng.uniform(-0.9, 0.9, n) * eb[f]).astype(np.float32)
        noise[rng.random(n) < 0.001] = 3 * eb[f]
        v = x[f][pad:][src] + noise
        keep = rng.random(n) < 0.5
        v = np.where(keep, x[f][pad:][src], v).astype(np.float32)
        if special:
            v[rng.integers(0, n)] = np.inf
        y.append(np.concatenate([np.zeros(pad, np.float32), v]))
    dx = [torch.from_numpy(a).cuda()[pad:] for a in x]
    dy = [torch.from_numpy(a).cuda()[pad:] for a in y]
    dp = None if perm is None else torch.from_numpy(perm.view(np.int32)).cuda()
    hx, hy = [a[pad:] for a in x], [a[pad:] for a in y]
    rv, rm = orc.bound_check(hx, hy, eb, perm=perm)
    ref = orc.error_stats(hx, hy, perm=perm)
    for _ in range(2):
        v, m = gpz.bound_check(dx, dy, eb, perm=dp)
        assert v.tolist() == rv.tolist() and m.tolist() == rm.tolist()
        st = gpz.error_stats(dx, dy, eb, perm=dp)
        assert st["violations"].tolist() == rv.tolist()
        assert st["max_abs_err"].tolist() == rm.tolist()
        assert (st["range"].view(np.uint32) == orc.field_range(hx).view(np.uint32)).all()
        assert np.allclose(st["sum_sq"], ref["sum_sq"], rtol=n * 2.0 ** -52, atol=0)


@pytest.mark.parametrize("n,F,shift", [(1, 1, 0), (7, 3, 1), (8191, 2, 0), (8192, 1, 0), (8193, 2, 3),
                                       (8192 * 3 + 5, 64, 2), (600_011, 5, 1), (8192 * 520, 1, 0)])
def test_range_at_chunk_edges(gpz, n, F, shift):
    """Every field's extremes are found wherever they lie: first, last and at
    the ends of the 8192-value chunks, each workgroup's range of which ends in
    the middle of a field."""
    rng = np.random.default_rng(n + F)
    for place in (0, n - 1, min(n - 1, 8191), n // 2):
        host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
        for f, h in enumerate(host):
            h[place] = 100.0 + f
            h[n - 1 - place] = -100.0 - f
            if n > 100:
                h[n // 3] = (np.nan, np.inf, -np.inf)[f % 3]
        dev = [torch.from_numpy(np.concatenate([np.full(shift, 1e9, np.float32), h])).cuda()[shift:]
               for h in host]
        got = gpz.field_range(dev, ws=gpz.stats_workspace(F))
        for f, h in enumerate(host):
            fin = h[np.isfinite(h)]
            assert got[f].tolist() == [fin.min(), fin.max()], (n, f, place)
