"""The accept flag may be written over the expected tag it answers for: the verdict is formed from
the tag as it was, in every workgroup that takes part."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

from gpu_util import to_dev  # noqa: E402


@pytest.fixture(scope="module")
def ctx():
    c = gcm.Context(device=0, key_slots=4)
    yield c
    c.close()


@pytest.mark.parametrize("siv", [False, True])
@pytest.mark.parametrize("at", [0, 12])  # the flag's place in the tag
@pytest.mark.parametrize("n", [1000, 300_001, 5 << 20])
def test_flag_over_the_expected_tag(ctx, n, at, siv):
    r = np.random.default_rng(n + at)
    key, iv, pt = r.bytes(32), r.bytes(12), r.integers(0, 256, n, dtype=np.uint8)
    ct, tag = (oracle.gcm_siv_encrypt if siv else oracle.gcm_encrypt)(key, iv, b"", pt)
    ct_d, back = to_dev(ct), torch.empty(n, dtype=torch.uint8, device="cuda")
    call = ctx.siv_decrypt_verify_async if siv else ctx.decrypt_verify_async
    ws = torch.zeros(ctx.siv_workspace_size(n, 0) if siv else ctx.workspace_size(n, 0), dtype=torch.uint8, device="cuda")
    slot = ctx.key_register(key)
    try:
        for forged in (False, True):
            for again in range(3):
                print(f"n={n} at={at} siv={siv} forged={forged} pass={again}", flush=True)
                tag_d = to_dev(np.frombuffer(tag, np.uint8))
                tag_d[5] ^= forged
                ok = tag_d[at:at + 4].view(torch.int32)
                back.fill_(0x5A)
                call(slot, iv, None, ct_d, tag_d, back, ok, ws)
                torch.cuda.synchronize()
                assert int(ok) == (0 if forged else 1)
                assert np.array_equal(back.cpu().numpy(), np.zeros_like(pt) if forged else pt)
    finally:
        ctx.key_release(slot)
