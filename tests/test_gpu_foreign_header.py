"""A header or eb table of another stream than the one asked for is reported
whatever the number of blocks and the decoder (few blocks, one wave a block,
float64, batches), by block 0 alone, and nothing is decoded; synchronous calls
decode streams of every parameter."""
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


def damaged(words, F, nb):
    """(what, stream) with one header or eb word changed; the wide-record flag
    alone is free."""
    for k in range(8):
        bad = words.copy()
        bad[k] ^= np.uint32(1 << 16) if k == 1 else np.uint32(4)
        yield f"header word {k}", bad
    for f in (0, F - 1):
        bad = words.copy()
        bad[8 + 2 * (-(-nb // 64)) + f] = 0
        yield f"bound {f}", bad


@pytest.mark.parametrize("B", [256, 1024, 2048])
@pytest.mark.parametrize("blocks", [1, 3, 1100])
def test_queued(gpz, orc, B, blocks):
    rng = np.random.default_rng(blocks)
    n, F = blocks * B - 5, 2
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    words = orc.compress_parallel(host, 1e-2, B=B, threads=8)[0].view(np.uint32)
    p, err = gpz.params(F, block_size=B), torch.zeros(1, dtype=torch.int32, device="cuda")
    for what, bad in damaged(words, F, blocks):
        print(f"[case] B={B} blocks={blocks} {what}", flush=True)
        out = [torch.full((n,), 7.0, device="cuda") for _ in range(F)]
        gpz.decompress_async(torch.from_numpy(bad.view(np.uint8)).cuda(), n, F, out, err, p)
        assert int(err.item()) != 0, what
        assert all(bool((o == 7.0).all()) for o in out), what
    free = words.copy()
    free[1] ^= np.uint32(2 << 16)  # announces wide records: allowed without any
    out = [torch.empty(n, device="cuda") for _ in range(F)]
    gpz.decompress_async(torch.from_numpy(free.view(np.uint8)).cuda(), n, F, out, err, p)
    assert int(err.item()) == 0


def test_float64(gpz, orc):
    rng = np.random.default_rng(1)
    n, F = 1024 * 40 - 5, 2
    host = [rng.standard_normal(n) for _ in range(F)]
    words = orc.compress_parallel(host, 1e-2, threads=8)[0].view(np.uint32)
    for what, bad in damaged(words, F, 40):
        print(f"[case] float64 {what}", flush=True)
        out = [torch.full((n,), 7.0, device="cuda", dtype=torch.float64) for _ in range(F)]
        with pytest.raises(gpz.GpzError):
            gpz.decompress_f64(torch.from_numpy(bad.view(np.uint8)).cuda(), n, F, out=out)
        assert all(bool((o == 7.0).all()) for o in out), what


@pytest.mark.parametrize("blocks", [3, 1100])
@pytest.mark.parametrize("B,K,KF", [(64, 3, 3), (256, 3, 2), (512, 5, 3), (1024, 2, 3),
                                    (1024, 3, 1), (2048, 3, 3), (4096, 0, 3)])
def test_other_parameters(gpz, orc, B, K, KF, blocks):
    rng = np.random.default_rng(B + K)
    n, F = blocks * B - 7, 3
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    print(f"[case] B={B} K={K} KF={KF} n={n}", flush=True)
    ref = orc.compress_parallel(host, 1e-2, B=B, K=K, KF=KF, threads=8)[0]
    out = gpz.decompress(torch.from_numpy(ref).cuda(), n, F)
    for o, r in zip(out, orc.decompress(ref, n, F)):
        assert (o.cpu().numpy().view(np.uint32) == r.view(np.uint32)).all()
    dev = torch.from_numpy(ref).cuda()
    outliers, raw = gpz.stream_stats(dev, n, F)
    want, want_raw = orc.stream_stats(ref, n, F)
    assert raw == want_raw and [int(v) for v in outliers] == [int(v) for v in want]
