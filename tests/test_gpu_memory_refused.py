"""A request for device memory that the runtime refuses leaves nothing behind: the call that made it
reports it, and the next call on another context runs and matches the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

from gpu_util import host, to_dev  # noqa: E402


def test_calls_after_a_refused_allocation():
    c = gcm.Context(device=0, key_slots=2)
    try:
        key, iv = bytes(range(16)), bytes(12)
        pt = np.random.default_rng(60).integers(0, 256, 70_000, dtype=np.uint8)
        ct, tag = oracle.gcm_encrypt(key, iv, b"", pt)
        src, dst, tag_d = to_dev(pt), torch.empty(70_000, dtype=torch.uint8, device="cuda"), to_dev(np.zeros(16, np.uint8))
        ws = torch.zeros(c.workspace_size(70_000, 0), dtype=torch.uint8, device="cuda")
        slot = c.key_register(key)
        torch.cuda.synchronize()
        with pytest.raises(gcm.GcmError) as e:
            gcm.Context(device=0, key_slots=1 << 20)  # 2^20 slots of 402 KiB: more than the card has
        assert e.value.code == gcm.GCM_E_NOMEM
        c.encrypt_async(slot, iv, None, src, dst, tag_d, ws)
        assert bytes(host(tag_d)) == tag and np.array_equal(host(dst), ct)
    finally:
        c.close()
