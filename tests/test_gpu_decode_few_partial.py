"""Decoding of few blocks whose last, partial block has a record just under
the longest that is decoded from LDS (its arrays are extracted at all B
positions): decoded bits equal the oracle's, nothing is written past the end.
The reads' bounds are checked on the host (test_few_decode_layout.py)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("B,part,F,eb", [(2048, 1433, 6, 1e-4), (2048, 614, 8, 1e-6),
                                         (2048, 1743, 4, 1e-6), (1024, 512, 10, 1e-6),
                                         (1024, 901, 6, 1e-6), (256, 250, 20, 1e-6),
                                         (512, 500, 10, 1e-6)])
def test_long_record_of_a_partial_block(orc, B, part, F, eb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_10305_amd as gpz
    rng = np.random.default_rng(B + part)
    n = B + part
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    print(f"[case] partial n={n} F={F} B={B}", flush=True)
    ref, _ = orc.compress(host, eb, B=B)
    want = orc.decompress(ref, n, F)
    out = [torch.full((n + 1,), 7.0, device="cuda") for _ in range(F)]
    gpz.decompress(torch.from_numpy(ref).cuda(), n, F, out=[o[:n] for o in out])
    for o, r in zip(out, want):
        o = o.cpu().numpy()
        assert (o[:n].view(np.uint32) == r.view(np.uint32)).all() and o[n] == 7.0


@pytest.mark.parametrize("blocks", [511, 512, 513])
@pytest.mark.parametrize("F", [4, 5])
def test_end_of_the_form_at_2048(orc, blocks, F):
    """(two blocks per CU of a 256-CU device, up to four fields)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_10305_amd as gpz
    rng = np.random.default_rng(blocks)
    n = blocks * 2048 - 700
    host = [rng.standard_normal(n).astype(np.float32) for _ in range(F)]
    print(f"[case] B=2048 n={n} F={F}", flush=True)
    ref, _ = orc.compress_parallel(host, 1e-2, B=2048, threads=8)
    out = gpz.decompress(torch.from_numpy(ref).cuda(), n, F)
    for o, r in zip(out, orc.decompress(ref, n, F)):
        assert (o.cpu().numpy().view(np.uint32) == r.view(np.uint32)).all()
