"""Record copies inside the encoder's launch at every block size that has them
(B = 2048 has none, at the same sizes) and in float64: streams equal the oracle's, also from a workspace off the
alignment the copies ask for, and the copies do happen: the encoder's flags in
the workspace say which parts of a superblock it copied (all others are left to
the copy kernel, so the stream alone would not show a launch that copies
nothing)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SUPER, XCDS, PARTS = 64, 8, 4


def delay(B):
    return 8 if B >= 1024 else 12


@pytest.fixture(scope="module")
def gpz():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_10305_amd as g
    g.lib()
    return g


def compress(gpz, host, eb, B, shift=0):
    """(stream, flag word per superblock) through the C ABI, the workspace
    `shift` bytes off its alignment."""
    n, F = host[0].size, len(host)
    f64 = host[0].dtype == np.float64
    L, p = gpz.lib(), gpz.params(F, block_size=B)
    size = L.gpz_max_compressed_bytes_f64 if f64 else L.gpz_max_compressed_bytes
    need = L.gpz_compress_workspace_bytes_f64 if f64 else L.gpz_compress_workspace_bytes
    call = L.gpz_compress_f64 if f64 else L.gpz_compress
    dev = [torch.from_numpy(h).cuda() for h in host]
    out = torch.empty(size(n, F, ctypes.byref(p)), dtype=torch.uint8, device="cuda")
    ws = torch.full((need(n, F, ctypes.byref(p)) + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    ws = ws[shift:]
    assert ws.data_ptr() % 256 == shift
    ebs, got = np.full(F, eb, np.float32), ctypes.c_uint64(0)
    rc = call((ctypes.c_void_p * F)(*[d.data_ptr() for d in dev]), n, F, ebs.ctypes.data,
              ctypes.byref(p), out.data_ptr(), out.numel(), ctypes.byref(got), None,
              ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == gpz.GPZ_OK
    # the flags follow the slots, the 8 bytes a block and 28 bytes of counters
    nb = -(-n // B)
    ns = -(-nb // SUPER)
    slot = (1 + F * B * (2 if f64 else 1) + 3) // 4 * 4
    at = -(-nb * slot * 4 // 256) * 256 + nb * 8 + 28
    flags = ws[at:at + 4 * ns].cpu().numpy().view(np.uint32)
    return out[:got.value].cpu().numpy(), flags


def snapshot(B, rows, F, left=None, dtype=np.float32):
    rng = np.random.default_rng(B + rows)
    n = rows * XCDS * SUPER * B - B // 3
    host = [rng.standard_normal(n).astype(dtype) for _ in range(F)]
    if left is not None:
        host[0][left * B + 1] = 1e6 if dtype == np.float32 else np.nan
    return host


def parts(flags):
    return np.array([bin(int(v) & 15).count("1") for v in flags])


@pytest.mark.parametrize("B,rows", [(256, 16), (512, 16), (512, 19), (1024, 12), (1024, 15),
                                    (2048, 12), (2048, 13)])
def test_every_block_size(gpz, orc, B, rows):
    host = snapshot(B, rows, 2 if B < 1024 else 1)
    print(f"[case] placed B={B} rows={rows} n={host[0].size}", flush=True)
    ref = orc.compress_parallel(host, 1e-3, B=B, threads=8)[0]
    got, flags = compress(gpz, host, 1e-3, B)
    assert got.size == ref.size and (got == ref).all()
    placed = (rows - delay(B)) * XCDS
    if B <= 1024:
        # (waits are bounded, so not every part need be copied; a launch that
        # copies less than half has lost what it is for)
        assert parts(flags[:placed]).sum() > placed * PARTS // 2
        assert (flags[placed:] == 0).all()
    got, _ = compress(gpz, host, 1e-3, B, shift=16)
    assert got.size == ref.size and (got == ref).all()


@pytest.mark.parametrize("left", [0, 5 * SUPER + 3, 100 * SUPER])
def test_nothing_is_copied_past_a_left_block(gpz, orc, left):
    B, rows = 256, 30
    host = snapshot(B, rows, 2, left=left)
    print(f"[case] placed, block {left} left", flush=True)
    ref = orc.compress_parallel(host, 1e-3, B=B, threads=8)[0]
    got, flags = compress(gpz, host, 1e-3, B)
    assert got.size == ref.size and (got == ref).all()
    before = left // SUPER
    assert parts(flags[:before]).sum() >= before * PARTS // 2
    assert (flags[before:] == 0).all()


def test_float64(gpz, orc):
    rows = 13
    host = snapshot(1024, rows, 1, left=7, dtype=np.float64)
    print(f"[case] placed float64 n={host[0].size}", flush=True)
    ref = orc.compress_parallel(host, 1e-3, threads=8)[0]
    got, flags = compress(gpz, host, 1e-3, 1024)
    assert got.size == ref.size and (got == ref).all()
    placed = (rows - delay(1024)) * XCDS
    assert parts(flags[:placed]).sum() > placed * PARTS // 2
    assert (flags[placed:] == 0).all()
