"""Compression of few blocks (two launches, nothing cleared beforehand) at the
edges of that form: the block counts of a copy workgroup, a superblock and the
form itself, with none, some or all of the blocks left for 64-bit steps, the
workspace full of old words, synchronous, queued and replayed from a graph.
Streams and permutations equal the oracle's byte for byte."""
import ctypes

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


def snapshot(blocks, B, wide, seed):
    rng = np.random.default_rng(seed)
    n = blocks * B - (B // 3 if seed % 2 else 0)
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(3)]
    if wide == "all":
        host[1] *= np.float32(1e6)
    if wide == "some":
        for b in rng.choice(blocks, max(1, blocks // 5), replace=False):
            host[rng.integers(0, 3)][b * B:(b + 1) * B] *= np.float32(1e6)
    return host


@pytest.mark.parametrize("wide", ["none", "some", "all"])
@pytest.mark.parametrize("blocks", [1, 4, 5, 64, 65, 255, 256, 257])
@pytest.mark.parametrize("B", [256, 1024, 2048])
def test_block_counts(gpz, orc, blocks, B, wide):
    if B == 2048 and blocks > 65:
        pytest.skip("same kernels as 1024, more of the oracle's time")
    F, eb, p = 3, 1e-3, gpz.params(3, block_size=B)
    for seed in (blocks, blocks + 1):
        host = snapshot(blocks, B, wide, seed)
        n = host[0].size
        print(f"[case] few blocks={blocks} B={B} n={n} wide={wide}", flush=True)
        ref, ref_perm = orc.compress(host, eb, B=B, want_perm=True)
        dev = [torch.from_numpy(h).cuda() for h in host]
        c = gpz.Compressor(n, F, p)
        for fill in (0xFF, 0x01):  # what an earlier call may have left
            c.ws.fill_(fill)
            s, perm = c.compress(dev, eb, want_perm=True)
            assert s.numel() == ref.size and (s.cpu().numpy() == ref).all()
            assert (perm.cpu().numpy().astype(np.uint32) == ref_perm).all()
            c.ws.fill_(fill)
            c.out.zero_()
            c.compress_async(dev, eb)
            assert int(c.nbytes_dev.item()) == ref.size
            assert (c.out[:ref.size].cpu().numpy() == ref).all()


def test_replayed_from_a_graph(gpz, orc):
    B, F, eb = 256, 3, 1e-3
    hosts = [snapshot(40, B, w, 2) for w in ("none", "some", "all")]
    n = hosts[0][0].size
    refs = [orc.compress(h, eb, B=B)[0] for h in hosts]
    dev = [torch.from_numpy(h).cuda() for h in hosts[0]]
    c = gpz.Compressor(n, F, gpz.params(F, block_size=B))
    c.compress_async(dev, eb)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        c.compress_async(dev, eb)
    for k in (0, 1, 2, 0, 2, 1):
        for d, h in zip(dev, hosts[k]):
            d.copy_(torch.from_numpy(h))
        other, _ = gpz.compress(dev, eb)  # eager work between replays
        g.replay()
        torch.cuda.synchronize()
        assert int(c.nbytes_dev.item()) == refs[k].size, k
        assert (c.out[:refs[k].size].cpu().numpy() == refs[k]).all(), k
        assert other.numel() > 0


@pytest.mark.parametrize("wide", ["none", "some"])
def test_output_one_word_short(gpz, orc, wide):
    host = snapshot(30, 256, wide, 2)
    n, F, eb = host[0].size, 3, np.full(3, 1e-3, np.float32)
    ref, _ = orc.compress(host, eb, B=256)
    dev = [torch.from_numpy(h).cuda() for h in host]
    p = gpz.params(F, block_size=256)
    ws = torch.empty(gpz.compress_workspace_bytes(n, F, p), dtype=torch.uint8, device="cuda")
    ptrs = (ctypes.c_void_p * F)(*[d.data_ptr() for d in dev])
    for short, want in ((0, gpz.GPZ_OK), (4, gpz.GPZ_ENOSPC), (ref.size - 40, gpz.GPZ_ENOSPC)):
        out = torch.full((ref.size + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        size = ctypes.c_uint64(0)
        rc = gpz.lib().gpz_compress(ptrs, n, F, eb.ctypes.data, ctypes.byref(p), out.data_ptr(),
                                    ref.size - short, ctypes.byref(size), None, ws.data_ptr(),
                                    ws.numel(), torch.cuda.current_stream().cuda_stream)
        assert rc == want and size.value == ref.size
        got = out.cpu().numpy()
        assert (got[ref.size - short:] == 0xAB).all()
        if rc == gpz.GPZ_OK:
            assert (got[:ref.size] == ref).all()
