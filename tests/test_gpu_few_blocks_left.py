"""Compression of few blocks of 2048 (kernels of their own at that size) up to
the end of the form, and blocks left for 64-bit steps whose numbers fall into
each group of 64: every one has a workgroup of its own.  Streams and
permutations equal the oracle's byte for byte."""
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


def check(gpz, orc, host, B):
    n, F, eb = host[0].size, len(host), 1e-3
    ref, ref_perm = orc.compress_parallel(host, eb, B=B, threads=8, want_perm=True)
    dev = [torch.from_numpy(h).cuda() for h in host]
    c = gpz.Compressor(n, F, gpz.params(F, block_size=B))
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


@pytest.mark.parametrize("wide", ["none", "some", "all"])
@pytest.mark.parametrize("blocks", [66, 129, 255, 256, 257])
def test_block_counts_at_2048(gpz, orc, blocks, wide):
    rng = np.random.default_rng(blocks)
    n = blocks * 2048 - (600 if blocks % 2 else 0)
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(2)]
    if wide == "all":
        host[1] *= np.float32(1e6)
    if wide == "some":
        for b in rng.choice(blocks, blocks // 5, replace=False):
            host[b % 2][b * 2048:(b + 1) * 2048] *= np.float32(1e6)
    print(f"[case] blocks={blocks} B=2048 wide={wide}", flush=True)
    check(gpz, orc, host, 2048)


@pytest.mark.parametrize("at", [(0,), (255,), (63, 64), (127, 128, 191, 192), (5, 70, 140, 250),
                                tuple(range(1, 256, 2)), tuple(range(255))])
def test_each_left_block(gpz, orc, at):
    rng = np.random.default_rng(len(at))
    B, blocks = 256, 256
    host = [rng.standard_normal(blocks * B).astype(np.float32) for _ in range(2)]
    for b in at:
        host[b % 2][b * B + b] = np.float32(1e6)
    print(f"[case] left {at[:4]}... of {blocks}", flush=True)
    check(gpz, orc, host, B)
