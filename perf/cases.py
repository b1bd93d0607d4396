"""Performance cases: calls that users of this library make, over the sizes they make them at.

The sizes are those of the repository's own workloads (`paper_2602_23067_amd/workloads.py`,
`bench.py`): messages from 4 KiB (the floor of the mixed batches) through 1 MiB (the paper's
smallest file) and the 4096 x 4096 image (67,109,760 bytes) to the 16384 x 16384 image
(1,073,744,640 bytes), ragged sizes between, 128-, 192- and 256-bit keys, and the AAD of those
workloads (16 bytes, one 2880-byte FITS header, or 0..4 KiB at random).

A case's "kind" names the entry point:

  async    Context.encrypt_async / decrypt_verify_async, key resident, workspace kept
  oneshot  Context.encrypt / decrypt_verify: key bytes in, tag or verdict back on the host
  ctr      Context.ctr_async, counter mode without a tag
  siv      Context.siv_encrypt_async / siv_decrypt_verify_async, workspace kept
  batch    Batch.launch / graph_launch over a planned batch of messages with a key each
  stream   Context.stream_begin, GcmStream.update per segment, GcmStream.final
  fits     Context.fits_encrypt / fits_decrypt: the FITS container, host bytes to host bytes
"""
import math

import numpy as np
import torch

from paper_2602_23067_amd import gcm, workloads

KIB, MIB = 1 << 10, 1 << 20
IMAGE_4K = 67_109_760       # 4096 x 4096 float32, padded to whole FITS blocks
IMAGE_16K = 1_073_744_640   # 16384 x 16384 float32, padded to whole FITS blocks
HEADER = 2880
SMALLEST = 4 * KIB


def listed():
    return [
        # The smallest call of the mixed workloads, in a tight loop on a resident key: launches
        # and the latency of one tile are all there is.
        dict(name="enc_4k_aes128", kind="async", op=0, key=16, len=4 * KIB, aad=16),
        # A ragged small file checked on its own, verdict awaited: what a request handler does.
        dict(name="verify_65537_aes256", kind="oneshot", op=1, key=32, len=65_537, aad=HEADER),
        # The paper's smallest file with its cipher, tag awaited on the host.
        dict(name="enc_1m_aes128", kind="oneshot", op=0, key=16, len=MIB, aad=16),
        # One detector frame, decrypted and verified with a resident key.
        dict(name="verify_image4k_aes256", kind="async", op=1, key=32, len=IMAGE_4K, aad=HEADER),
        # The headline: one 16384 x 16384 image encrypted and tagged.
        dict(name="enc_image16k_aes256", kind="async", op=0, key=32, len=IMAGE_16K, aad=HEADER),
        # An archive job: messages of uneven length (median 1 MiB), a key each, one launch.
        dict(name="batch_enc_mixed", kind="batch", op=0, n=512, median=MIB, most=64 * MIB, tampered=0, graph=False),
        # Many small requests verified together by replaying a planned batch; one in twenty is
        # forged and zero-filled.
        dict(name="batch_verify_small", kind="batch", op=1, n=1024, median=16 * KIB, most=256 * KIB, tampered=51,
             graph=True),
        # A message that arrives in device segments, encrypted as they come.
        dict(name="stream_enc_256m", kind="stream", op=0, key=32, len=256 * MIB, aad=HEADER, segment=16 * MIB),
        # The misuse-resistant mode on one detector frame (two passes by construction).
        dict(name="siv_enc_image4k_aes256", kind="siv", op=0, key=32, len=IMAGE_4K, aad=HEADER),
        # The same mode verifying a small file: key derivation on every call counts here.
        dict(name="siv_verify_1m_aes128", kind="siv", op=1, key=16, len=MIB, aad=16),
        # Counter mode alone over a ragged buffer, the remaining key size.
        dict(name="ctr_16m_aes192", kind="ctr", op=0, key=24, len=16 * MIB + 1, aad=0),
        # The paper's container from a FITS file in host memory, copies and PCIe included.
        dict(name="fits_enc_2048", kind="fits", op=0, key=32, ny=2048, nx=2048),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["async", "async", "async", "oneshot", "oneshot", "batch", "batch", "stream", "siv", "siv", "ctr",
                       "fits"])
    op = rng.randrange(2)
    key = rng.choice([16, 32, 32, 24]) if kind != "siv" else rng.choice([16, 32])
    aad = rng.choice([0, 16, HEADER, rng.randrange(1, 4 * KIB)])
    if kind == "batch":
        median = _log(rng, 8 * KIB, MIB)
        n = min(_log(rng, 16, 1024), 512 * MIB // median)  # messages average about twice the median
        return dict(kind=kind, op=op, n=n, median=median, most=64 * median, tampered=rng.choice([0, n // 20]) * op,
                    graph=rng.random() < 0.5)
    if kind == "fits":
        return dict(kind=kind, op=op, key=key, ny=_log(rng, 64, 2048), nx=_log(rng, 64, 2048))
    if kind == "stream":
        segment = 16 * _log(rng, MIB // 16, 2 * MIB)
        return dict(kind=kind, op=op, key=key, len=_log(rng, 2 * segment, 256 * MIB), aad=aad, segment=segment)
    most = {"async": IMAGE_16K, "oneshot": IMAGE_4K, "siv": 256 * MIB, "ctr": 256 * MIB}[kind]
    size = _log(rng, SMALLEST, most)
    if rng.random() < 0.4:  # image-like: whole FITS blocks
        size = max(HEADER * 2, size // HEADER * HEADER)
    return dict(kind=kind, op=0 if kind == "ctr" else op, key=key, len=size, aad=0 if kind == "ctr" else aad)


# ---------------------------------------------------------------- inputs


def _host_bytes(seed, *path, n):
    return workloads.random_bytes(workloads.rng_for(seed, *path), n).tobytes()


def _header(seed, n):
    """n bytes of AAD on the GPU: FITS header cards, cut or repeated to size."""
    if n == 0:
        return None
    text = np.frombuffer(workloads.fits_header(workloads.rng_for(seed, 1)), dtype=np.uint8)
    return torch.from_numpy(np.resize(text, n).copy()).cuda()


def _pixels(gen, n):
    """n bytes of big-endian float32 sky (mean 1000, sigma 30), made on the GPU."""
    f = torch.empty((n + 3) // 4, dtype=torch.float32, device="cuda").normal_(1000.0, 30.0, generator=gen)
    b = f.view(torch.uint8).view(-1, 4)
    out = torch.empty_like(b)
    for k in range(4):
        out[:, k] = b[:, 3 - k]
    return out.view(-1)[:n]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _flip(t, at, bit):
    t[at] = t[at] ^ (1 << bit)


def prepare(case, seed):
    kind, op = case["kind"], case["op"]
    if kind == "fits":
        return _prepare_fits(case, seed)
    if kind == "batch":
        return _prepare_batch(case, seed)
    ctx = gcm.Context(device=0, key_slots=4)
    key, iv = _host_bytes(seed, 2, n=case["key"]), _host_bytes(seed, 3, n=12)
    slot = ctx.key_register(key)
    n, aad = case["len"], _header(seed, case["aad"])
    src = _pixels(_gen(seed), n)
    dst = torch.empty_like(src)
    tag = torch.zeros(16, dtype=torch.uint8, device="cuda")
    ok = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.zeros(ctx.siv_workspace_size(n, case["aad"]) if kind == "siv" else ctx.workspace_size(n, case["aad"]),
                     dtype=torch.uint8, device="cuda")
    s = dict(kind=kind, op=op, ctx=ctx, key=key, iv=iv, slot=slot, aad=aad, src=src, dst=dst, tag=tag, ok=ok, ws=ws)
    if op == 1:  # a valid ciphertext and its tag
        if kind == "siv":
            ctx.siv_encrypt_async(slot, iv, aad, src, dst, tag, ws)
        else:
            ctx.encrypt_async(slot, iv, aad, src, dst, tag, ws)
        s["src"], s["dst"] = dst, src
        torch.cuda.synchronize()
        s["tag_host"] = bytes(tag.cpu().numpy())
    if kind == "stream":
        step = case["segment"]
        s["parts"] = [(s["src"][at:at + step], s["dst"][at:at + step]) for at in range(0, n, step)]
    return s


def _prepare_batch(case, seed):
    n, op = case["n"], case["op"]
    shape = workloads.rng_for(n, case["median"])  # the lengths belong to the case, the bytes to the seed
    lengths = workloads.lognormal_lengths(shape, n, float(case["median"]), float(np.sqrt(2 * np.log(2))), SMALLEST,
                                          case["most"])
    aad_lens = shape.integers(0, 4 * KIB + 1, n)
    r = workloads.rng_for(seed, 4)
    keys = [workloads.random_bytes(r, 16 if r.integers(0, 2) == 0 else 32).tobytes() for _ in range(n)]
    ivs = [workloads.random_bytes(r, 12).tobytes() for _ in range(n)]
    ctx = gcm.Context(device=0, key_slots=n)
    slots = ctx.key_register_many(keys)
    lay = gcm.BatchLayout(lengths, aad_lens)
    base = torch.zeros(lay.total, dtype=torch.uint8, device="cuda")
    gen = _gen(seed)
    for i in range(n):
        base[lay.in_off[i]:lay.in_off[i] + lay.lengths[i]].random_(0, 256, generator=gen)
        if lay.aad_lens[i]:
            base[lay.aad_off[i]:lay.aad_off[i] + lay.aad_lens[i]].random_(0, 256, generator=gen)
    if op == 1:  # valid ciphertexts in place of the inputs, then the forged ones
        make = gcm.Batch(ctx, lay.jobs([0] * n, slots, ivs), base)
        make.launch()
        torch.cuda.synchronize()
        make.close()
        for i in range(n):
            base[lay.in_off[i]:lay.in_off[i] + lay.lengths[i]] = base[lay.out_off[i]:lay.out_off[i] + lay.lengths[i]]
        for i in r.choice(n, size=case["tampered"], replace=False):
            if r.random() < 0.5:
                _flip(base, lay.tag_base + 16 * int(i) + int(r.integers(0, 16)), int(r.integers(0, 8)))
            else:
                _flip(base, lay.in_off[i] + int(r.integers(0, lay.lengths[i])), int(r.integers(0, 8)))
    batch = gcm.Batch(ctx, lay.jobs([op] * n, slots, ivs), base)
    return dict(kind="batch", ctx=ctx, base=base, batch=batch, graph=case["graph"])


def _prepare_fits(case, seed):
    r = workloads.rng_for(seed, 5)
    ctx = gcm.Context(device=0, key_slots=4)
    key_h, key_d = (workloads.random_bytes(r, case["key"]).tobytes() for _ in range(2))
    nonce_h, nonce_d = (workloads.random_bytes(r, 12).tobytes() for _ in range(2))
    data = workloads.fits_file(r, case["ny"], case["nx"])
    s = dict(kind="fits", op=case["op"], ctx=ctx, data=data, key_h=key_h, key_d=key_d, nonce_h=nonce_h,
             nonce_d=nonce_d)
    if case["op"] == 1:
        s["data"] = ctx.fits_encrypt(data, key_h, key_d, nonce_h, nonce_d)
    return s


# ---------------------------------------------------------------- one pass


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "batch":
        if s["graph"]:
            s["batch"].graph_launch()
        else:
            s["batch"].launch()
        return s["base"]
    if kind == "fits":
        if s["op"] == 0:
            return np.frombuffer(ctx.fits_encrypt(s["data"], s["key_h"], s["key_d"], s["nonce_h"], s["nonce_d"]),
                                 dtype=np.uint8)
        data, code = ctx.fits_decrypt(s["data"], s["key_h"], s["key_d"])
        return np.frombuffer(data, dtype=np.uint8), code
    src, dst, aad, iv = s["src"], s["dst"], s["aad"], s["iv"]
    if kind == "ctr":
        ctx.ctr_async(s["slot"], iv, src, dst)
        return dst
    if kind == "oneshot":
        if s["op"] == 0:
            return dst, np.frombuffer(ctx.encrypt(s["key"], iv, aad, src, dst), dtype=np.uint8)
        return dst, ctx.decrypt_verify(s["key"], iv, aad, src, s["tag_host"], dst)
    if kind == "stream":
        st = ctx.stream_begin(s["op"], s["slot"], iv, aad)
        for a, b in s["parts"]:
            st.update(a, b)
        if s["op"] == 0:
            st.final(s["tag"])
        else:
            st.final(s["tag"], s["ok"])
        st.close()
    elif kind == "siv":
        if s["op"] == 0:
            ctx.siv_encrypt_async(s["slot"], iv, aad, src, dst, s["tag"], s["ws"])
        else:
            ctx.siv_decrypt_verify_async(s["slot"], iv, aad, src, s["tag"], dst, s["ok"], s["ws"])
    elif s["op"] == 0:
        ctx.encrypt_async(s["slot"], iv, aad, src, dst, s["tag"], s["ws"])
    else:
        ctx.decrypt_verify_async(s["slot"], iv, aad, src, s["tag"], dst, s["ok"], s["ws"])
    return (dst, s["tag"]) if s["op"] == 0 else (dst, s["ok"])


def work(case):
    """Payload read once and written once, AAD read once; the SIV encryption reads its payload
    twice, since the tag over all of it starts the counter.  No floating-point work."""
    if case["kind"] == "batch":  # expected sizes: lognormal with mean twice the median
        total = case["n"] * 2 * max(case["median"], SMALLEST)
        return {"bytes": 2 * total + case["n"] * (2 * KIB + 16), "flops": 0}
    if case["kind"] == "fits":
        return {"bytes": 2 * workloads.padded_len(4 * case["ny"] * case["nx"]), "flops": 0}
    passes = 3 if case["kind"] == "siv" and case["op"] == 0 else 2
    return {"bytes": passes * case["len"] + case["aad"] + 16, "flops": 0}


def exact(case, seed):
    """Ciphertexts, plaintexts, tags and verdicts are bytes and whole numbers: they are equal or
    wrong, and no value in 64-bit floating point stands behind them."""
    return None
