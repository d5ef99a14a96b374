"""Decoding of snapshots of few blocks (four waves a block, the record in LDS)
at the edges of that form: the block count where it ends, records longer than
its LDS (coded, raw, with 64-bit steps), outliers in every field, partial
blocks.  Decoded bits and error codes equal the oracle's."""
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


def check(gpz, orc, host, eb, B, K=3):
    n, F = host[0].size, len(host)
    print(f"[case] few n={n} F={F} B={B}", flush=True)
    ref, _ = orc.compress(host, eb, B=B, K=K)
    dev = torch.from_numpy(ref).cuda()
    out = [torch.full((n + 1,), 7.0, device="cuda") for _ in range(F)]
    gpz.decompress(dev, n, F, out=[o[:n] for o in out])
    for o, r in zip(out, orc.decompress(ref, n, F)):
        o = o.cpu().numpy()
        assert (o[:n].view(np.uint32) == r.view(np.uint32)).all() and o[n] == 7.0
    # an unaligned output takes the scalar stores
    gpz.decompress(dev, n, F, out=[o[1:] for o in out])
    for o, r in zip(out, orc.decompress(ref, n, F)):
        assert (o[1:].cpu().numpy().view(np.uint32) == r.view(np.uint32)).all()
    return ref


@pytest.mark.parametrize("blocks", [1, 2, 1023, 1024, 1025])
@pytest.mark.parametrize("B", [256, 512])
def test_block_counts(gpz, orc, B, blocks):
    """(four blocks per CU of a 256-CU device: up to 1024 blocks)"""
    rng = np.random.default_rng(blocks)
    for n in (blocks * B, blocks * B - B // 3):
        check(gpz, orc, [rng.standard_normal(n).astype(np.float32) for _ in range(2)], 1e-2, B)


@pytest.mark.parametrize("B", [256, 512, 1024, 2048])
@pytest.mark.parametrize("kind", ["short", "long", "raw", "wide", "outliers"])
def test_record_lengths(gpz, orc, B, kind):
    rng = np.random.default_rng(B)
    n = 3 * B + 77
    F = {"short": 1, "long": 24, "raw": 40, "wide": 30, "outliers": 7}[kind]
    host = [(rng.standard_normal(n) * 50).astype(np.float32) for _ in range(F)]
    eb = 1e-3
    if kind == "raw":  # every value an outlier
        host = [rng.integers(0, 2 ** 32, n, dtype=np.uint64).astype(np.uint32).view(np.float32).copy()
                for _ in range(F)]
        eb = 1e-30
    if kind == "wide":
        host[F // 2] = (rng.standard_normal(n) * 1e6).astype(np.float32)
    if kind == "outliers":
        for h in host:
            at = rng.integers(0, n, n // 9)
            h[at] = rng.choice(np.array([np.nan, np.inf, -np.inf], np.float32), at.size)
    check(gpz, orc, host, eb, B)


def test_damaged_records_are_refused_as_by_the_oracle(gpz, orc):
    rng = np.random.default_rng(3)
    n, F = 2500, 5
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    host[1][::7] = np.nan
    ref, _ = orc.compress(host, 1e-3)
    words = ref.view(np.uint32)
    at = list(range(8 + 2 + F + 3 + 4)) + sorted(rng.choice(words.size, 150, replace=False).tolist())
    for k in at:
        bad = words.copy()
        bad[k] ^= np.uint32(1) << np.uint32(rng.integers(0, 32))
        print(f"[case] damaged word {k}", flush=True)
        want = orc.decompress_status(bad.view(np.uint8), n, F)
        try:
            out = gpz.decompress(torch.from_numpy(bad.view(np.uint8)).cuda(), n, F)
            got = 0
        except gpz.GpzError as e:
            got = e.code
        assert (got == 0) == (want == 0), (k, got, want)
        if got == 0:
            for o, r in zip(out, orc.decompress(bad.view(np.uint8), n, F)):
                assert (o.cpu().numpy().view(np.uint32) == r.view(np.uint32)).all(), k
