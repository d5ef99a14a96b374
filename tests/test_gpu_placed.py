"""Compression of many blocks, whose records are mostly copied inside the
encoder's launch: block counts about the point where that begins and at the
ends of its rows, raw and long records, blocks left for 64-bit steps anywhere
(then the copy kernel takes what the launch could not place), an output too
small, queued calls and graph replays.  Streams equal the oracle's byte for
byte; float64 at the default block size likewise."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

B = 256
ROW = 8 * 64  # blocks of a row: a superblock on each of 8 XCDs


@pytest.fixture(scope="module")
def gpz():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_10305_amd as g
    g.lib()
    return g


def snapshot(blocks, kind, seed, F=2):
    rng = np.random.default_rng(seed)
    n = blocks * B - 100
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    if kind == "raw":  # some blocks of random bits
        for b in rng.choice(blocks, 40, replace=False):
            h = host[rng.integers(0, F)][b * B:(b + 1) * B]
            h[:] = rng.integers(0, 2 ** 32, h.size, dtype=np.uint64).astype(np.uint32).view(np.float32)
    if kind == "first":
        host[0][:B] *= np.float32(1e6)
    if kind == "middle":
        host[1][blocks // 2 * B:(blocks // 2 + 1) * B] *= np.float32(1e6)
    if kind == "all":
        host[0][::B] = np.float32(1e6)
    if kind == "last":
        host[0][-B:] *= np.float32(1e6)
    return host


def check(gpz, orc, host, eb=1e-3):
    n, F = host[0].size, len(host)
    ref, ref_perm = orc.compress_parallel(host, eb, B=B, threads=8, want_perm=True)
    dev = [torch.from_numpy(h).cuda() for h in host]
    c = gpz.Compressor(n, F, gpz.params(F, block_size=B))
    for fill in (0xFF, 0x00):  # what an earlier call may have left
        c.ws.fill_(fill)
        s, perm = c.compress(dev, eb, want_perm=True)
        assert s.numel() == ref.size
        got = s.cpu().numpy()
        assert (got == ref).all(), int((got != ref).argmax())
        assert (perm.cpu().numpy().astype(np.uint32) == ref_perm).all()
    c.out.zero_()
    c.compress_async(dev, eb)
    assert int(c.nbytes_dev.item()) == ref.size
    assert (c.out[:ref.size].cpu().numpy() == ref).all()
    return ref, dev, c


@pytest.mark.parametrize("blocks", [12 * ROW, 13 * ROW - 1, 13 * ROW, 13 * ROW + 1, 14 * ROW + 65,
                                    15 * ROW, 15 * ROW + 1, 16 * ROW - 64, 16 * ROW, 17 * ROW + 7,
                                    40 * ROW + 333])
def test_block_counts(gpz, orc, blocks):
    print(f"[case] placed blocks={blocks}", flush=True)
    check(gpz, orc, snapshot(blocks, "plain", blocks))


@pytest.mark.parametrize("kind", ["raw", "first", "middle", "last", "all"])
def test_records_the_launch_cannot_place(gpz, orc, kind):
    print(f"[case] placed kind={kind}", flush=True)
    check(gpz, orc, snapshot(18 * ROW + 5, kind, 3))


def test_long_records(gpz, orc):
    """Records of more than 2048 words (40 fields of a 256-value block)."""
    check(gpz, orc, snapshot(17 * ROW, "plain", 9, F=40)[:40], eb=1e-5)


def test_output_too_small_and_replay(gpz, orc):
    host = snapshot(17 * ROW + 9, "plain", 4)
    ref, dev, c = check(gpz, orc, host)
    n, F, eb = host[0].size, len(host), np.full(2, 1e-3, np.float32)
    p = gpz.params(F, block_size=B)
    ptrs = (ctypes.c_void_p * F)(*[d.data_ptr() for d in dev])
    for short in (4, ref.size // 2, ref.size - 64):
        out = torch.full((ref.size,), 0xAB, dtype=torch.uint8, device="cuda")
        size = ctypes.c_uint64(0)
        rc = gpz.lib().gpz_compress(ptrs, n, F, eb.ctypes.data, ctypes.byref(p), out.data_ptr(),
                                    ref.size - short, ctypes.byref(size), None, c.ws.data_ptr(),
                                    c.ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert rc == gpz.GPZ_ENOSPC and size.value == ref.size
        assert (out == 0xAB).all()  # nothing is written
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        c.compress_async(dev, eb)
    other = snapshot(17 * ROW + 9, "middle", 5)
    ref2 = orc.compress_parallel(other, 1e-3, B=B, threads=8)[0]
    for k in (0, 1, 0, 1, 1, 0):
        for d, h in zip(dev, (host, other)[k]):
            d.copy_(torch.from_numpy(h))
        gpz.compress([dev[0][:5000]], 1e-3)  # eager work between replays
        g.replay()
        torch.cuda.synchronize()
        want = (ref, ref2)[k]
        assert int(c.nbytes_dev.item()) == want.size
        assert (c.out[:want.size].cpu().numpy() == want).all(), k


def test_float64(gpz, orc):
    rng = np.random.default_rng(8)
    n = 1024 * (16 * ROW + 3) - 17
    host = [rng.standard_normal(n), rng.standard_normal(n) + 1e9 * (np.arange(n) > n // 2)]
    ref, _ = orc.compress_parallel(host, 1e-3, threads=8)
    got, _ = gpz.compress_f64([torch.from_numpy(h).cuda() for h in host], 1e-3)
    assert got.numel() == ref.size and (got.cpu().numpy() == ref).all()
