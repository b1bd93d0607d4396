"""Batches of small messages, run a row of 64 blocks per wave or in tiles: sizes at the edges of
rows and of the groups whose values are summed, every length of a last partial block in AAD and
payload, forged tags, few items and many, against the oracle; and the same batch under every
kernel that takes it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_23067_amd import gcm  # noqa: E402

pytestmark = pytest.mark.gpu

# log2 tile, waves, workgroups a compute unit: the library's choice, rows, tiles
SHAPES = [(0, 0, 0), (6, 8, 2), (6, 12, 1), (6, 16, 2), (7, 16, 1)]


@pytest.fixture(scope="module")
def ctx():
    c = gcm.Context(device=0, key_slots=8)
    yield c
    c.close()


def run(ctx, sizes, op, seed):
    """sizes: (aad bytes, payload bytes) of each message; every seventh decrypt is forged."""
    r = np.random.default_rng(seed)
    n = len(sizes)
    keys = [r.bytes(k) for k in (16, 24, 32)]
    slots = [ctx.key_register(k) for k in keys]
    which = [int(k) for k in r.integers(0, 3, n)]
    ivs = [r.bytes(12) for _ in range(n)]
    lens, aad_lens = [s[1] for s in sizes], [s[0] for s in sizes]
    lay = gcm.BatchLayout(lens, aad_lens)
    buf = r.integers(0, 256, lay.total, dtype=np.uint8)
    want = buf.copy()
    for i in range(n):
        aad = buf[lay.aad_off[i]:lay.aad_off[i] + aad_lens[i]]
        pt = want[lay.in_off[i]:lay.in_off[i] + lens[i]].copy()
        ct, tag = oracle.gcm_encrypt(keys[which[i]], ivs[i], aad, pt)
        t = slice(lay.tag_base + 16 * i, lay.tag_base + 16 * i + 16)
        o = slice(lay.out_off[i], lay.out_off[i] + lens[i])
        if op == 0:
            want[o], want[t] = ct, np.frombuffer(tag, np.uint8)
            continue
        forged = i % 7 == 3
        buf[lay.in_off[i]:lay.in_off[i] + lens[i]] = want[lay.in_off[i]:lay.in_off[i] + lens[i]] = ct
        buf[t] = np.frombuffer(tag, np.uint8)
        buf[t.start + i % 16] ^= np.uint8(forged)
        want[t] = buf[t]
        want[o] = 0 if forged else pt
        want[lay.ok_base + 4 * i:lay.ok_base + 4 * i + 4] = [not forged, 0, 0, 0]
    dev = torch.from_numpy(buf).cuda()
    b = gcm.Batch(ctx, lay.jobs([op] * n, [slots[w] for w in which], ivs), dev)
    b.launch()
    torch.cuda.synchronize()
    got = dev.cpu().numpy()
    b.close()
    for s in slots:
        ctx.key_release(s)
    assert np.array_equal(got, want), f"first difference at byte {int(np.flatnonzero(got != want)[0])}"  # also between the messages


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("op", [0, 1])
def test_edges_of_rows_and_groups(ctx, shape, op):
    # 16 blocks of AAD and payload in all, counted with the length block: 63, 64, 65 of a row, groups of
    # 4, 8 and 16 rows and one more, messages without payload, AAD or both
    sizes = [(0, 0), (5, 0), (0, 3), (16, 16), (1024, 0), (1008, 16), (0, 1008), (0, 1024), (0, 992), (8, 1000)]
    for rows in (4, 8, 12, 16, 33):
        sizes += [(0, 1024 * rows - 16), (2880, 1024 * rows - 2880 - 16), (7, 1024 * rows), (1024 * (rows - 1) + 1, 9)]
    ctx.set_launch(*shape)
    try:
        run(ctx, sizes, op, 1)
    finally:
        ctx.set_launch(0, 0, 0)


@pytest.mark.parametrize("shape", SHAPES[:1] + SHAPES[-1:])
def test_every_partial_block(ctx, shape):
    ctx.set_launch(*shape)
    try:
        run(ctx, [(a, 32 + p) for a in range(17) for p in range(16)], 0, 2)
        run(ctx, [(16 + a, p) for a in range(16) for p in range(17)], 1, 3)
    finally:
        ctx.set_launch(0, 0, 0)


@pytest.mark.parametrize("n,size", [(3000, 300), (700, 16 * 1024 + 5), (40, 70_000)])
def test_many_items_in_one_launch(ctx, n, size):
    r = np.random.default_rng(n)
    run(ctx, [(int(r.integers(0, 600)), int(r.integers(0, 2 * size))) for _ in range(n)], 1, 4)


def test_memory_for_larger_tiles_only():
    # four messages of 200 KiB: 15 KiB of plan and partials with one-row tiles, 5 KiB with the larger
    # tiles, beside the context's tables (see test_gpu_serve.py) and four key slots
    slot_bytes = 2048 + 65536 + 40 * 8192 + 16384
    c = gcm.Context(device=0, hbm_budget=5 * 256 * 4 + 47 * 4096 * 16 + 4 * slot_bytes + 256 + 8192, key_slots=4)
    try:
        run(c, [(0, 200 * 1024)] * 4, 0, 5)
    finally:
        c.close()
