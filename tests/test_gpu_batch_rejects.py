"""Batches whose messages are all rejected: every output is cleared to its last byte and nothing else
is touched, for lengths at the edges of the zero-fill's chunks, more messages than one pass of it
takes, and messages of one workgroup and of many."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

CHUNK = 8192


@pytest.fixture(scope="module")
def ctx():
    c = gcm.Context(device=0, key_slots=4)
    yield c
    c.close()


def reject_all(ctx, lengths, aad_lens, shape):
    r = np.random.default_rng(len(lengths))
    n = len(lengths)
    lay = gcm.BatchLayout(lengths, aad_lens)
    buf = r.integers(0, 256, lay.total, dtype=np.uint8)  # no tag in it is right
    want = buf.copy()
    for i in range(n):
        want[lay.out_off[i]:lay.out_off[i] + lengths[i]] = 0
        want[lay.ok_base + 4 * i:lay.ok_base + 4 * i + 4] = 0
    slot = ctx.key_register(r.bytes(32))
    ctx.set_launch(*shape)
    try:
        dev = torch.from_numpy(buf).cuda()
        b = gcm.Batch(ctx, lay.jobs([1] * n, [slot] * n, [r.bytes(12) for _ in range(n)]), dev)
        for _ in range(2):
            b.launch()
        torch.cuda.synchronize()
        got = dev.cpu().numpy()
        b.close()
    finally:
        ctx.set_launch(0, 0, 0)
        ctx.key_release(slot)
    assert np.array_equal(got, want), f"first difference at byte {int(np.flatnonzero(got != want)[0])}"


# log2 tile, waves, workgroups a compute unit: the library's choice; rows in groups of four, so that
# every message of more than 4 KiB goes through the zero-fill; one workgroup for what fits 16 tiles of 1 MiB
SHAPES = [(0, 0, 0), (6, 12, 1), (16, 16, 1)]


@pytest.mark.parametrize("shape", SHAPES)
def test_edges_of_chunks(ctx, shape):
    edges = [0, 1, 15, 16, 17] + [k * CHUNK + d for k in (1, 2, 3, 8) for d in (-17, -16, -1, 0, 1, 15, 16, 17)]
    reject_all(ctx, edges * 6, [(7 * i) % 50 for i in range(len(edges) * 6)], shape)


def test_more_messages_than_one_pass_takes(ctx):
    # with and without one that is too long for a share of the grid alike
    r = np.random.default_rng(5)
    lengths = [int(x) for x in r.integers(4100, 20_000, 700)]
    reject_all(ctx, lengths, [0] * 700, SHAPES[1])
    lengths[600] = 1_000_003
    reject_all(ctx, lengths, [0] * 700, SHAPES[1])


@pytest.mark.parametrize("shape", SHAPES)
def test_uneven_messages(ctx, shape):
    r = np.random.default_rng(3)
    lengths = [int(x) for x in np.exp(r.uniform(np.log(4000), np.log(400_000), 300))]
    lengths[17], lengths[200], lengths[299] = 9_000_001, 3_000_000, 5_000_016
    reject_all(ctx, lengths, [0] * 300, shape)
