"""Rows of 64 blocks inside a tile, against the oracle, bit for bit: first counters with every kind
of low byte (so that it wraps at different lanes of a row, or between rows), rows of whole AAD
blocks right before rows of whole data blocks, and sizes at the edges of a row, for GCM, counter
mode and GCM-SIV."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

from gpu_util import canaries_intact, guarded, host, to_dev  # noqa: E402

ROW = 1024
SHAPES = [(0, 0, 0), (7, 16, 0), (9, 8, 0)]


@pytest.fixture(scope="module")
def ctx():
    c = gcm.Context(device=0, key_slots=8)
    yield c
    c.close()


@pytest.mark.parametrize("key_len", [16, 24, 32])
@pytest.mark.parametrize("aad_len,n", [(0, 5 * ROW), (0, 5 * ROW - 16), (3 * ROW, 4 * ROW), (2 * ROW - 16, 9 * ROW + 16),
                                       (2 * ROW + 5, 9 * ROW - 1), (70 * ROW, 3 * ROW), (16, 40 * ROW + 1007)])
def test_gcm_rows_and_counters(ctx, key_len, aad_len, n):
    for seed in range(6):  # IVs of 16 bytes: J0, and with it the first counter's low byte, is arbitrary
        r = np.random.default_rng(100 * n + seed)
        key, iv = r.bytes(key_len), r.bytes(16 if seed else 12)
        aad, pt = (r.integers(0, 256, k, dtype=np.uint8) for k in (aad_len, n))
        ct_ref, tag_ref = oracle.gcm_encrypt(key, iv, aad, pt)
        print(f"key={key_len} aad={aad_len} n={n} seed={seed}", flush=True)
        aad_d, pt_d = to_dev(aad) if aad_len else None, to_dev(pt)
        ctx.set_launch(*SHAPES[seed % 3])
        try:
            full, ct_d = guarded(n)
            assert ctx.encrypt(key, iv, aad_d, pt_d, ct_d) == tag_ref
            assert np.array_equal(host(ct_d), ct_ref) and canaries_intact(full, n)
            back = torch.empty_like(pt_d)
            assert ctx.decrypt_verify(key, iv, aad_d, ct_d, tag_ref, back) and torch.equal(back, pt_d)
            assert not ctx.decrypt_verify(key, iv, aad_d, pt_d, tag_ref, back) and not back.any()
        finally:
            ctx.set_launch(0, 0, 0)


@pytest.mark.parametrize("n", [1, ROW - 16, ROW, ROW + 1, 4 * ROW, 17 * ROW - 15, 300 * ROW + 9])
def test_ctr_rows(ctx, n):
    for key_len in (16, 24, 32):
        r = np.random.default_rng(n + key_len)
        key, iv, data = r.bytes(key_len), r.bytes(12), r.integers(0, 256, n, dtype=np.uint8)
        full, dst = guarded(n)
        ctx.ctr_xcrypt(key, iv, to_dev(data), dst)
        assert np.array_equal(host(dst), oracle.gctr(key, iv + b"\x00\x00\x00\x02", data))
        assert canaries_intact(full, n)


@pytest.mark.parametrize("key_len", [16, 32])
@pytest.mark.parametrize("aad_len,n", [(0, ROW), (5 * ROW, 6 * ROW), (ROW + 3, 7 * ROW - 5), (66 * ROW, 33 * ROW + 1)])
def test_siv_rows(ctx, key_len, aad_len, n):
    for seed in range(4):  # the counter starts at the tag's low dword, whose low byte is arbitrary
        r = np.random.default_rng(7 * n + seed)
        key, nonce = r.bytes(key_len), r.bytes(12)
        aad, pt = (r.integers(0, 256, k, dtype=np.uint8) for k in (aad_len, n))
        ct_ref, tag_ref = oracle.gcm_siv_encrypt(key, nonce, aad, pt)
        aad_d, pt_d = to_dev(aad) if aad_len else None, to_dev(pt)
        ct_d, back, tag_d = torch.empty_like(pt_d), torch.empty_like(pt_d), to_dev(np.zeros(16, np.uint8))
        ok = torch.zeros(1, dtype=torch.int32, device="cuda")
        ctx.set_launch(*SHAPES[seed % 3])
        slot = ctx.key_register(key)
        try:
            ctx.siv_encrypt_async(slot, nonce, aad_d, pt_d, ct_d, tag_d)
            torch.cuda.synchronize()
            assert bytes(host(tag_d)) == tag_ref and np.array_equal(host(ct_d), ct_ref)
            ctx.siv_decrypt_verify_async(slot, nonce, aad_d, ct_d, tag_d, back, ok)
            torch.cuda.synchronize()
            assert int(ok) == 1 and torch.equal(back, pt_d)
        finally:
            ctx.key_release(slot)
            ctx.set_launch(0, 0, 0)


# Where the launch changes: one workgroup or more, rows of waves of their own up to the chip's last
# wave and tiles of more rows beyond it, and one tile more than there are waves.
@pytest.mark.parametrize("aad_len,n", [(0, 15 * ROW - 16), (0, 16 * ROW - 16), (16, 16 * ROW - 16), (5, 16 * ROW),
                                       (0, 255 * ROW - 16), (0, 4096 * ROW - 16), (16, 4096 * ROW - 16),
                                       (2880, 4097 * ROW), (16, 16384 * ROW - 16), (2880, 16384 * ROW)])
def test_launch_boundaries(ctx, aad_len, n):
    r = np.random.default_rng(n + aad_len)
    key, iv = r.bytes(32 if n % 3 else 16), r.bytes(12)
    aad, pt = (r.integers(0, 256, k, dtype=np.uint8) for k in (aad_len, n))
    ct_ref, tag_ref = oracle.gcm_encrypt(key, iv, aad, pt)
    plan = ctx.launch_plan(len(key), n, aad_len)
    print(f"aad={aad_len} n={n} {plan}", flush=True)
    aad_d, pt_d = to_dev(aad) if aad_len else None, to_dev(pt)
    full, ct_d = guarded(n)
    slot = ctx.key_register(key)
    try:
        ws = torch.full((ctx.workspace_size(n, aad_len),), 0xA5, dtype=torch.uint8, device="cuda")
        tag_d, ok = to_dev(np.zeros(16, np.uint8)), torch.full((1,), -1, dtype=torch.int32, device="cuda")
        ctx.encrypt_async(slot, iv, aad_d, pt_d, ct_d, tag_d, ws)
        torch.cuda.synchronize()
        assert bytes(host(tag_d)) == tag_ref and np.array_equal(host(ct_d), ct_ref) and canaries_intact(full, n)
        back = torch.empty_like(pt_d)
        ctx.decrypt_verify_async(slot, iv, aad_d, ct_d, tag_d, back, ok, ws)
        torch.cuda.synchronize()
        assert int(ok) == 1 and torch.equal(back, pt_d)
        tag_d[15] ^= 1
        ctx.decrypt_verify_async(slot, iv, aad_d, ct_d, tag_d, back, ok, ws)
        torch.cuda.synchronize()
        assert int(ok) == 0 and not back.any()
    finally:
        ctx.key_release(slot)
