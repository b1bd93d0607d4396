"""Serving where the context's memory holds a batch's plan with larger tiles, but not with the small
ones that are faster: the requests are served, one after another, and match the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

from gpu_util import to_dev  # noqa: E402


def test_serving_in_memory_for_larger_tiles_only():
    # one request of 3 MiB: 52 KiB of plan and partials with tiles of one row, 14 KiB with tiles of
    # four, beside the context's tables (see test_gpu_serve.py) and two key slots
    slot_bytes = 2048 + 65536 + 40 * 8192 + 16384
    c = gcm.Context(device=0, hbm_budget=5 * 256 * 4 + 47 * 4096 * 16 + 2 * slot_bytes + 256 + (24 << 10), key_slots=2)
    try:
        key, iv, n = bytes(range(32)), bytes(12), 3 << 20
        slot = c.key_register(key)
        pt = np.random.default_rng(59).integers(0, 256, n, dtype=np.uint8)
        ct, tag = oracle.gcm_encrypt(key, iv, b"", pt)
        x, y, t = to_dev(ct), torch.empty(n, dtype=torch.uint8, device="cuda"), to_dev(np.frombuffer(tag, np.uint8))
        srv = gcm.Server(c, n_streams=1, hbm_budget=64 << 20)
        try:
            for forged in (False, True, False):
                t[7] ^= forged
                y.fill_(0x5A)
                torch.cuda.synchronize()
                accepted, _ = srv.wait(srv.submit(1, slot, iv, None, x, y, t))
                t[7] ^= forged
                assert accepted == (not forged)
                assert np.array_equal(y.cpu().numpy(), np.zeros_like(pt) if forged else pt)
            assert srv.stats()["failed"] == 0
        finally:
            srv.stop()
    finally:
        c.close()
