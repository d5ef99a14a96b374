"""Batches at the job counts where the lookup of a block's job changes (a wave
compares 64 prefix entries at a time, up to 256 jobs; a search beyond), with
empty and one-block jobs among them: every stream and reconstruction equals
the plain call's."""
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


@pytest.mark.parametrize("njobs", [1, 63, 64, 65, 255, 256, 257])
@pytest.mark.parametrize("graph", [0, 1])
def test_every_job_is_found(gpz, njobs, graph):
    from paper_2508_10305_amd.batch import Batch, default_config
    print(f"[case] batch jobs={njobs} graph={graph}", flush=True)
    rng = np.random.default_rng(njobs)
    F, p = 3, gpz.params(3)
    sizes = [int(rng.choice([0, 1, 300, 1023, 1024, 1025, 2500])) for _ in range(njobs)]
    sizes[rng.integers(0, njobs)] = 3 * 64 * 1024 + 17  # one job of several superblocks
    host = [[rng.standard_normal(n).astype(np.float32) for _ in range(F)] for n in sizes]
    dev = [[torch.from_numpy(h).cuda() for h in hs] for hs in host]
    outs = [torch.zeros(gpz.max_compressed_bytes(n, F, p), dtype=torch.uint8, device="cuda")
            for n in sizes]
    decs = [[torch.zeros(max(n, 1), device="cuda")[:n] for _ in range(F)] for n in sizes]
    cfg = default_config()
    cfg.grid, cfg.use_graph = 0, graph
    b = Batch(dev, [1e-3] * njobs, outs, dec=decs, p=p, config=cfg)
    for _ in range(2):
        b.compress()
        b.decompress()
    nbytes = b.sizes()
    assert not b.errors().any()
    for j in range(njobs):
        s, _ = gpz.compress(dev[j], 1e-3)
        assert int(nbytes[j]) == s.numel() and torch.equal(outs[j][:s.numel()], s), j
        if sizes[j]:
            for a, r in zip(decs[j], gpz.decompress(s, sizes[j], F)):
                assert torch.equal(a, r), j
    b.close()
