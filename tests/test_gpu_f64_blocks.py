"""GPU parity of float64 snapshots at the default block size (one wave per
block) against the CPU oracle: streams, permutations and decoded bits, at the
edges of a block, at every stored width, and with mixed steps per field."""
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


def check(gpz, orc, host, eb, K=3, KF=None, shift=0, label=""):
    """`shift`: the device fields and outputs start that many doubles past a
    16-byte boundary."""
    n, F = host[0].size, len(host)
    print(f"[case] f64 {label} n={n} F={F} K={K} KF={KF} shift={shift}", flush=True)
    ref, ref_perm = orc.compress(host, eb, K=K, KF=KF, want_perm=True)
    dev = [torch.from_numpy(np.concatenate([np.zeros(shift), h])).cuda()[shift:] for h in host]
    got, perm = gpz.compress_f64(dev, eb, seg_bits=K, key_fields=KF, want_perm=True)
    g = got.cpu().numpy()
    assert g.size == ref.size and (g == ref).all(), label
    assert (perm.cpu().numpy().astype(np.uint32) == ref_perm).all(), label
    out = [torch.full((n + shift,), 7.0, dtype=torch.float64, device="cuda") for _ in range(F)]
    gpz.decompress_f64(got, n, F, out=[o[shift:] for o in out])
    for o, r in zip(out, orc.decompress(ref, n, F, f64=True)):
        o = o.cpu().numpy()
        assert (o[shift:].view(np.uint64) == r.view(np.uint64)).all(), label
        assert (o[:shift] == 7.0).all(), label


def mixed(n, F, rng):
    """Fields the float32 steps serve, fields they do not, blocks of both, and
    fields with non-finite values or values beyond float32."""
    out = []
    for f in range(F):
        x = rng.standard_normal(n) * 10.0 ** (f % 3)
        if f % 4 == 1:
            x += 1e9  # float32 cannot resolve the bound here
        if f % 4 == 2:
            x[n // 2:] += 1e9
        if f % 4 == 3 and n > 8:
            x[rng.integers(0, n, 6)] = [np.nan, np.inf, -np.inf, -0.0, 1e300, -np.nan]
        out.append(x)
    return out


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2049, 70_001])
@pytest.mark.parametrize("F,K,KF", [(1, 3, 1), (3, 3, 3), (6, 3, 3), (5, 5, 2), (4, 0, 3), (65 - 1, 1, 3)])
def test_block_edges(gpz, orc, n, F, K, KF):
    if n > 5000 and F > 6:
        n = 5001
    rng = np.random.default_rng(n * 7 + F)
    check(gpz, orc, mixed(n, F, rng), 1e-3, K=K, KF=KF, shift=n & 1, label="mixed")


@pytest.mark.parametrize("w", range(0, 54))
def test_every_width(gpz, orc, w):
    """Grid indices of up to w bits on an exact grid: near zero (32-bit steps
    up to 24 bits) and, where it stays exact, about 2^45 (64-bit steps at
    every width); key fields store the bits below their segment."""
    rng = np.random.default_rng(w)
    n = 1500  # a whole block and a partial one
    q = [rng.integers(0, 2 ** w, n).astype(np.float64) for _ in range(3)]
    q[1][:] = q[0][::-1]
    fields = [q[0], q[1], q[2]]
    if w <= 45:
        fields += [2.0 ** 45 + q[2], 2.0 ** 45 + q[0]]
        check(gpz, orc, fields[3:], 0.5, KF=1, label=f"wide w={w}")
    if w >= 2:
        fields[2][rng.integers(0, n, 5)] = np.nan
    check(gpz, orc, fields, 0.5, label=f"w={w}")


def test_raw_blocks_and_empty_range(gpz, orc):
    """Incompressible blocks (every value an outlier or full width), constant
    fields, and blocks with no finite value."""
    rng = np.random.default_rng(5)
    n = 3000
    huge = rng.standard_normal(n) * 1e200
    bits = rng.integers(0, 2 ** 64, n, dtype=np.uint64).view(np.float64).copy()
    check(gpz, orc, [huge, bits], 1e-3, label="raw")
    check(gpz, orc, [np.full(n, 2.5), np.full(n, np.nan), np.full(n, np.inf)], 1e-3, label="constant")
    check(gpz, orc, [np.full(n, 2.5), rng.standard_normal(n), huge], 1e-3, label="one raw field")


def test_damaged_streams_are_refused_as_by_the_oracle(gpz, orc):
    """One word of a stream changed at a time (headers, tables, lengths, record
    headers, field words, outlier lists, payloads): the GPU accepts it exactly
    when the oracle does, and then decodes the same bits."""
    rng = np.random.default_rng(11)
    n, F = 2500, 3
    host = mixed(n, F + 1, rng)[1:]  # wide, half wide, non-finite values
    ref, _ = orc.compress(host, 1e-3)
    words = ref.view(np.uint32)
    recs = 8 + 2 + F + 3  # header, one superblock, bounds, three lengths
    at = list(range(recs)) + [recs, recs + 1, recs + 2, recs + 3]
    at += sorted(rng.choice(np.arange(recs, words.size), 120, replace=False).tolist())
    for k in at:
        bad = words.copy()
        bad[k] ^= np.uint32(1) << np.uint32(rng.integers(0, 32))
        print(f"[case] damaged word {k}", flush=True)
        want = orc.decompress_status(bad.view(np.uint8), n, F, f64=True)
        dev = torch.from_numpy(bad.view(np.uint8)).cuda()
        try:
            out = gpz.decompress_f64(dev, n, F)
            got = 0
        except gpz.GpzError as e:
            got = e.code
        assert (got == 0) == (want == 0), (k, got, want)
        if got == 0:
            for o, r in zip(out, orc.decompress(bad.view(np.uint8), n, F, f64=True)):
                assert (o.cpu().numpy().view(np.uint64) == r.view(np.uint64)).all(), k
