"""The reduction tree over single tile partials, which streamed messages and the host pipeline end
with, at every fan-in and at tile counts of one level and of several, of more than its 1024 leaves and
no power of the fan-in, against the oracle; and a search that does not time the fan-in where no tree
runs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

from gpu_util import host, to_dev  # noqa: E402

ROW = 1024  # bytes of a tile of 2^6 blocks


@pytest.fixture(scope="module")
def ctx():
    c = gcm.Context(device=0, key_slots=8)
    yield c
    c.close()


# bytes of the segments: 1, 2, 5, 37, 300, 1024, 1025 and 2100 tiles
SEGMENTS = [16, 2 * ROW, 5 * ROW - 16, 37 * ROW, 300 * ROW + 16, 1024 * ROW, 1025 * ROW, 2100 * ROW + 7]


@pytest.mark.parametrize("fanin", [2, 4, 8, 16])
def test_streams(ctx, fanin):
    r = np.random.default_rng(fanin)
    key, iv, aad = r.bytes(32), r.bytes(12), r.integers(0, 256, 70 * ROW + 3, dtype=np.uint8)
    pt = r.integers(0, 256, sum(SEGMENTS), dtype=np.uint8)
    ct, tag = oracle.gcm_encrypt(key, iv, aad, pt)
    slot = ctx.key_register(key)
    ctx.set_combine(fanin)
    ctx.set_launch(6, 16, 0)
    try:
        for op, src, want in ((0, pt, ct), (1, ct, pt)):
            print(f"fanin={fanin} op={op}", flush=True)
            s_d, d_d = to_dev(src), torch.zeros(pt.size, dtype=torch.uint8, device="cuda")
            tag_d, ok = to_dev(np.frombuffer(tag if op else bytes(16), np.uint8)), torch.zeros(1, dtype=torch.int32, device="cuda")
            st = ctx.stream_begin(op, slot, iv, to_dev(aad))
            at = 0
            for n in SEGMENTS:
                st.update(s_d[at:at + n], d_d[at:at + n])
                at += n
            st.final(tag_d, ok if op else None)
            st.close()
            assert np.array_equal(host(d_d), want)
            assert int(ok) == 1 if op else bytes(host(tag_d)) == tag
    finally:
        ctx.set_combine(0)
        ctx.set_launch(0, 0, 0)
        ctx.key_release(slot)


@pytest.mark.parametrize("fanin", [2, 4, 8, 16])
def test_host_pipeline(ctx, fanin):
    r = np.random.default_rng(100 + fanin)
    ctx.set_combine(fanin)
    ctx.set_launch(6, 16, 0)
    ctx.set_pipeline(256 << 10)
    try:
        for n in (5 * ROW + 7, 37 * ROW, 1023 * ROW + 16, 2100 * ROW + 1):
            print(f"fanin={fanin} n={n}", flush=True)
            key, iv, aad = r.bytes(16), r.bytes(12), r.integers(0, 256, 33, dtype=np.uint8)
            pt = r.integers(0, 256, n, dtype=np.uint8)
            ct, tag = oracle.gcm_encrypt(key, iv, aad, pt)
            out, back = np.empty_like(pt), np.empty_like(pt)
            assert ctx.encrypt_host(key, iv, aad, pt, out) == tag and np.array_equal(out, ct)
            assert ctx.decrypt_verify_host(key, iv, aad, out, tag, back) and np.array_equal(back, pt)
    finally:
        ctx.set_combine(0)
        ctx.set_launch(0, 0, 0)
        ctx.set_pipeline(0)


def test_search_times_a_shape_once():
    c = gcm.Context(device=0, key_slots=4)
    try:
        res = c.autotune(16, 1 << 20, reps=1)
        print(res, flush=True)
        # 2^8..2^16 blocks, three wave counts, and at most the planner's own shape
        assert res["candidates"] <= 9 * 3 + 1
        assert c.launch_plan(16, 1 << 20)["combine_fanin"] == res["combine_fanin"]
    finally:
        c.close()
