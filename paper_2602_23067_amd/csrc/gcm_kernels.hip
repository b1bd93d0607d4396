// gcm_kernels.hip -- AES-GCM kernels for CDNA4 (gfx950, wave64).
//
// Pipeline for one message (the paper's GPU pipeline: H-power generation,
// AES-CTR, GHASH map phase, combine_partial_ghash reduce phase, validation
// gate; here CTR and the GHASH map phase are fused into one pass):
//
//   k_key_setup / k_key_tables   once per key: round keys, H, H^(2^k), and
//                                the fixed-multiplier GHASH tables.
//   k_gcm_tiles                  per wave tile: AES-CTR + XOR + store, and a
//                                per-lane Horner over the ciphertext with the
//                                fixed multiplier H^64, then a per-lane
//                                fix-up product and an XOR across the wave
//                                -> one value, and one 16-byte partial for
//                                the tiles of a workgroup, lifted past what
//                                follows it; a message of one workgroup is
//                                finished here.
//   k_gcm_rows                   the same for messages of one-row tiles.
//   k_gcm_verdict                XOR of a message's partials, xor E_K(J0) ->
//                                tag / accept flag, and a rejected output
//                                cleared (a batch's by k_gcm_zerofill).
//   k_gcm_combine                streams and the host pipeline, whose tiles
//                                leave one partial each that nothing has
//                                lifted: a tree over them.
//
// AES-GCM-SIV (RFC 8452) reuses the same machinery: k_siv_derive builds a
// per-message key slot from the key-generating key and the nonce, the tile and
// row kernels run POLYVAL (as GHASH over byte-reversed blocks), counter
// mode with the little-endian counter, or both fused, and k_siv_verdict forms
// or checks the tag.
//
// No MFMA: the work is byte lookups and XORs, not a real-valued contraction.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "gcm_internal.h"
#include "gcm_plan.h"

namespace gcm {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- small helpers

__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ u32x4 xor3v(u32x4 a, u32x4 b, u32x4 c)
{
    return u32x4{xor3(a.x, b.x, c.x), xor3(a.y, b.y, c.y), xor3(a.z, b.z, c.z), xor3(a.w, b.w, c.w)};
}

__device__ __forceinline__ uint32_t rotl32(uint32_t x, int n) { return n ? (x << n) | (x >> (32 - n)) : x; }

__device__ __forceinline__ uint32_t byte_of(u32x4 a, int k)
{
    const uint32_t w = (k < 4) ? a.x : (k < 8) ? a.y : (k < 12) ? a.z : a.w;
    return (w >> (8 * (k & 3))) & 0xffu;
}

__device__ __forceinline__ uint32_t bswap32(uint32_t x) { return __builtin_bswap32(x); }

__device__ __forceinline__ uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// XOR of x over the 64 lanes of the wave, returned in every lane, without
// going through the LDS (where a shuffle would queue behind table lookups):
// DPP steps within each row of 16 lanes, then row swaps across the wave.
__device__ __forceinline__ uint32_t wave_xor_u32(uint32_t x)
{
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x141, 0xF, 0xF, false);  // row_half_mirror
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x140, 0xF, 0xF, false);  // row_mirror
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);  // rows 0<->1, 2<->3
    x = p[0] ^ p[1];
    const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);  // rows 0,1 <-> 2,3
    return q[0] ^ q[1];
}

// Workgroup barrier ordering LDS accesses only: a wave's outstanding global
// or spill stores do not hold the other waves at the barrier.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Read-only device data (key slots, descriptors, work lists) is read through
// the constant address space so uniform reads become scalar loads into SGPRs.
#define CONST_AS __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ const CONST_AS T *cptr(const void *p)
{
    return (const CONST_AS T *)(p);
}

// whole-struct read through the constant address space (word by word)
template <typename T>
__device__ __forceinline__ T load_const(const void *p)
{
    static_assert(sizeof(T) % 4 == 0, "word-sized struct expected");
    T v;
    uint32_t *dst = reinterpret_cast<uint32_t *>(&v);
    const CONST_AS uint32_t *src = cptr<uint32_t>(p);
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i)
        dst[i] = src[i];
    return v;
}

// Waits for every 64-byte line of a descriptor at once: the scalar cache starts
// cold, and a line read where its first field is needed is a wait of its own in
// the chain before the first row.
__device__ __forceinline__ void touch_lines(const CONST_AS MsgDesc *dp)
{
    const CONST_AS uint32_t *w = (const CONST_AS uint32_t *)dp;
    static_assert(sizeof(MsgDesc) > 128 && sizeof(MsgDesc) <= 192, "three lines, or four when not aligned");
    const uint32_t a = w[0], b = w[16], c = w[32], d = w[sizeof(MsgDesc) / 4 - 1];
    asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d));
}

// Payload buffers are addressed in the global address space so that their
// loads and stores use the vector-memory counter only and never make an LDS
// wait also wait for HBM.
#define GLOBAL_AS __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ GLOBAL_AS T *gptr(uint64_t addr)
{
    return (GLOBAL_AS T *)(addr);
}

// ---------------------------------------------------------------- AES tables
//
// S-box from GF(2^8) antilog/log tables with generator 0x03 (FIPS-197 sec.
// 5.1.1: multiplicative inverse followed by the affine map, written here in
// its rotate form b ^ rotl(b,1) ^ rotl(b,2) ^ rotl(b,3) ^ rotl(b,4) ^ 0x63).
// TE0[x] is the MixColumns column (2s, s, s, 3s) as a memory-order word;
// TE1..TE3 are its byte rotations.

__device__ __forceinline__ uint32_t gf8_xtime(uint32_t a) { return ((a << 1) ^ ((a & 0x80u) ? 0x1bu : 0u)) & 0xffu; }

__device__ __forceinline__ uint32_t rotl8(uint32_t x, int n) { return ((x << n) | (x >> (8 - n))) & 0xffu; }

__global__ void k_init_tables(uint32_t *te0, uint32_t *sbox)
{
    __shared__ uint8_t ex[256], lg[256];
    if (threadIdx.x == 0) {
        uint32_t x = 1;
        for (int i = 0; i < 255; ++i) {
            ex[i] = (uint8_t)x;
            lg[x] = (uint8_t)i;
            x = x ^ gf8_xtime(x);  // x * 0x03
        }
        lg[0] = 0;
    }
    __syncthreads();
    const uint32_t a = threadIdx.x;
    if (a < 256) {
        const uint32_t inv = a ? ex[(255 - lg[a]) % 255] : 0u;
        const uint32_t s = inv ^ rotl8(inv, 1) ^ rotl8(inv, 2) ^ rotl8(inv, 3) ^ rotl8(inv, 4) ^ 0x63u;
        const uint32_t s2 = gf8_xtime(s), s3 = s2 ^ s;
        const uint32_t t0 = s2 | (s << 8) | (s << 16) | (s3 << 24);
        te0[a] = t0;
        sbox[a] = s;
        // TE1..TE3 after the S-box (read by the scalar unit, which has no rotate)
        te0[kTe1Off + a] = rotl32(t0, 8);
        te0[kTe1Off + 256 + a] = rotl32(t0, 16);
        te0[kTe1Off + 512 + a] = rotl32(t0, 24);
    }
}

// One AES block with a fully unrolled round count (key setup only); te0/sb point at LDS copies, rk at registers or LDS.
template <int NR>
__device__ __forceinline__ void aes_block(const uint32_t *rk, const uint32_t *te0, const uint32_t *sb,
                                          const uint32_t in[4], uint32_t out[4])
{
    uint32_t s0 = in[0] ^ rk[0], s1 = in[1] ^ rk[1], s2 = in[2] ^ rk[2], s3 = in[3] ^ rk[3];
#pragma unroll
    for (int r = 1; r < NR; ++r) {
        const uint32_t t0 = te0[s0 & 0xff] ^ rotl32(te0[(s1 >> 8) & 0xff], 8) ^ rotl32(te0[(s2 >> 16) & 0xff], 16) ^
                            rotl32(te0[s3 >> 24], 24) ^ rk[4 * r + 0];
        const uint32_t t1 = te0[s1 & 0xff] ^ rotl32(te0[(s2 >> 8) & 0xff], 8) ^ rotl32(te0[(s3 >> 16) & 0xff], 16) ^
                            rotl32(te0[s0 >> 24], 24) ^ rk[4 * r + 1];
        const uint32_t t2 = te0[s2 & 0xff] ^ rotl32(te0[(s3 >> 8) & 0xff], 8) ^ rotl32(te0[(s0 >> 16) & 0xff], 16) ^
                            rotl32(te0[s1 >> 24], 24) ^ rk[4 * r + 2];
        const uint32_t t3 = te0[s3 & 0xff] ^ rotl32(te0[(s0 >> 8) & 0xff], 8) ^ rotl32(te0[(s1 >> 16) & 0xff], 16) ^
                            rotl32(te0[s2 >> 24], 24) ^ rk[4 * r + 3];
        s0 = t0;
        s1 = t1;
        s2 = t2;
        s3 = t3;
    }
    out[0] = (sb[s0 & 0xff] | (sb[(s1 >> 8) & 0xff] << 8) | (sb[(s2 >> 16) & 0xff] << 16) | (sb[s3 >> 24] << 24)) ^
             rk[4 * NR + 0];
    out[1] = (sb[s1 & 0xff] | (sb[(s2 >> 8) & 0xff] << 8) | (sb[(s3 >> 16) & 0xff] << 16) | (sb[s0 >> 24] << 24)) ^
             rk[4 * NR + 1];
    out[2] = (sb[s2 & 0xff] | (sb[(s3 >> 8) & 0xff] << 8) | (sb[(s0 >> 16) & 0xff] << 16) | (sb[s1 >> 24] << 24)) ^
             rk[4 * NR + 2];
    out[3] = (sb[s3 & 0xff] | (sb[(s0 >> 8) & 0xff] << 8) | (sb[(s1 >> 16) & 0xff] << 16) | (sb[s2 >> 24] << 24)) ^
             rk[4 * NR + 3];
}

// ---------------------------------------------------------------- key setup
//
// FIPS-197 sec. 5.2 key expansion on memory-order words: RotWord is a right
// rotation by 8 of the little-endian word, Rcon enters byte 0.

struct KeyArg {
    uint32_t w[8];
    uint32_t len;
};

// Keys travel to the device as by-value kernel arguments, in chunks that fit
// the 4 KiB argument segment: no staging buffer, stream-ordered, capturable.
struct KeyChunk {
    KeyArg keys[kKeyChunk];
    uint64_t slots[kKeyChunk];
};
struct SlotChunk {
    uint64_t slots[kKeyChunk];
};

__device__ __forceinline__ uint32_t sub_word(uint32_t t, const uint32_t *sb)
{
    return sb[t & 0xff] | (sb[(t >> 8) & 0xff] << 8) | (sb[(t >> 16) & 0xff] << 16) | (sb[t >> 24] << 24);
}

// GF(2^128) in "polynomial order": bit i of (lo, hi) is the coefficient of
// x^i.  Memory order is the same bytes with the bits of each byte reversed.
struct P128 {
    uint64_t lo, hi;
};

__device__ __forceinline__ uint32_t brev_bytes(uint32_t x) { return __builtin_bswap32(__builtin_bitreverse32(x)); }

__device__ __forceinline__ P128 mem_to_poly(const uint32_t m[4])
{
    P128 p;
    p.lo = (uint64_t)brev_bytes(m[0]) | ((uint64_t)brev_bytes(m[1]) << 32);
    p.hi = (uint64_t)brev_bytes(m[2]) | ((uint64_t)brev_bytes(m[3]) << 32);
    return p;
}

__device__ __forceinline__ u32x4 poly_to_mem(P128 p)
{
    return u32x4{brev_bytes((uint32_t)p.lo), brev_bytes((uint32_t)(p.lo >> 32)), brev_bytes((uint32_t)p.hi),
                 brev_bytes((uint32_t)(p.hi >> 32))};
}

// spread the 32 bits of x to the even bit positions of a 64-bit word
__device__ __forceinline__ uint64_t spread32(uint32_t x)
{
    uint64_t v = x;
    v = (v | (v << 16)) & 0x0000FFFF0000FFFFull;
    v = (v | (v << 8)) & 0x00FF00FF00FF00FFull;
    v = (v | (v << 4)) & 0x0F0F0F0F0F0F0F0Full;
    v = (v | (v << 2)) & 0x3333333333333333ull;
    v = (v | (v << 1)) & 0x5555555555555555ull;
    return v;
}

// squaring is GF(2)-linear: coefficient i moves to 2i, then the upper 128
// bits fold back through x^128 = x^7 + x^2 + x + 1 (twice at most).
__device__ P128 poly_square(P128 a)
{
    const uint64_t l0 = spread32((uint32_t)a.lo), l1 = spread32((uint32_t)(a.lo >> 32));
    const uint64_t h0 = spread32((uint32_t)a.hi), h1 = spread32((uint32_t)(a.hi >> 32));
    // value = (l0, l1) + (h0, h1) * x^128
    uint64_t tlo = h0 ^ (h0 << 1) ^ (h0 << 2) ^ (h0 << 7);
    uint64_t thi = h1 ^ ((h1 << 1) | (h0 >> 63)) ^ ((h1 << 2) | (h0 >> 62)) ^ ((h1 << 7) | (h0 >> 57));
    const uint64_t ov = (h1 >> 63) ^ (h1 >> 62) ^ (h1 >> 57);
    tlo ^= ov ^ (ov << 1) ^ (ov << 2) ^ (ov << 7);
    P128 r;
    r.lo = l0 ^ tlo;
    r.hi = l1 ^ thi;
    return r;
}

// fold (l0, l1) + (h0, h1) * x^128 back below x^128 (x^128 = x^7 + x^2 + x + 1)
__device__ __forceinline__ P128 poly_reduce(uint64_t l0, uint64_t l1, uint64_t h0, uint64_t h1)
{
    uint64_t tlo = h0 ^ (h0 << 1) ^ (h0 << 2) ^ (h0 << 7);
    uint64_t thi = h1 ^ ((h1 << 1) | (h0 >> 63)) ^ ((h1 << 2) | (h0 >> 62)) ^ ((h1 << 7) | (h0 >> 57));
    const uint64_t ov = (h1 >> 63) ^ (h1 >> 62) ^ (h1 >> 57);
    tlo ^= ov ^ (ov << 1) ^ (ov << 2) ^ (ov << 7);
    P128 r;
    r.lo = l0 ^ tlo;
    r.hi = l1 ^ thi;
    return r;
}

// v * x^i for 0 <= i < 128: a 256-bit shift, then one fold
__device__ __forceinline__ P128 poly_mul_xi(P128 v, int i)
{
    uint64_t w0 = 0, w1 = 0, w2 = 0, w3 = 0;
    if (i == 0) {
        w0 = v.lo;
        w1 = v.hi;
    } else if (i < 64) {
        w0 = v.lo << i;
        w1 = (v.hi << i) | (v.lo >> (64 - i));
        w2 = v.hi >> (64 - i);
    } else if (i == 64) {
        w1 = v.lo;
        w2 = v.hi;
    } else {
        const int j = i - 64;
        w1 = v.lo << j;
        w2 = (v.hi << j) | (v.lo >> (64 - j));
        w3 = v.hi >> (64 - j);
    }
    return poly_reduce(w0, w1, w2, w3);
}

// Frobenius tables: squaring is GF(2)-linear and does not depend on the key,
// so x -> x^(2^k) has a fixed byte-position table F_k (16 x 256 entries).
// Built once per context; key setup then forms all H^(2^k) in parallel, one
// lane per k, instead of a chain of 47 squarings.
__global__ __launch_bounds__(256) void k_frob_tables(u32x4 *frob)
{
    __shared__ u32x4 basis[128];  // (x^i)^(2^k), memory order
    const int k = blockIdx.x + 1;
    const int tid = threadIdx.x;
    if (tid < 128) {
        P128 v;
        v.lo = tid < 64 ? (1ull << tid) : 0ull;
        v.hi = tid < 64 ? 0ull : (1ull << (tid - 64));
        for (int q = 0; q < k; ++q)
            v = poly_square(v);
        basis[tid] = poly_to_mem(v);
    }
    __syncthreads();
    u32x4 *tab = frob + (uint64_t)blockIdx.x * 4096;
    for (int e = tid; e < 4096; e += 256) {
        const int j = e >> 8, b = e & 255;
        u32x4 acc = {0, 0, 0, 0};
        for (int t = 0; t < 8; ++t)
            if ((b >> t) & 1)
                acc ^= basis[8 * j + 7 - t];
        tab[e] = acc;
    }
}

// FIPS-197 key expansion with the key length fixed at compile time (fully
// unrolled, so the schedule stays in registers) into w and the slot header.
template <int NK>
__device__ __forceinline__ void expand_key(const uint32_t *kw, KeySlotHdr *hd, const uint32_t *sb, uint32_t *w)
{
    constexpr int NR = NK + 6, NW = 4 * (NR + 1);
#pragma unroll
    for (int i = 0; i < NK; ++i)
        w[i] = kw[i];
    uint32_t rcon = 1;
#pragma unroll
    for (int i = NK; i < NW; ++i) {
        uint32_t t = w[i - 1];
        if (i % NK == 0) {
            t = sub_word((t >> 8) | (t << 24), sb) ^ rcon;
            rcon = gf8_xtime(rcon);
        } else if (NK > 6 && i % NK == 4) {
            t = sub_word(t, sb);
        }
        w[i] = w[i - NK] ^ t;
    }
#pragma unroll
    for (int i = 0; i < 4 * (kMaxNr + 1); ++i)
        hd->rk[i] = i < NW ? w[i] : 0u;
    hd->nr = (uint32_t)NR;
    hd->key_len = (uint32_t)(4 * NK);
}

// key expansion, then H = E_K(0^128)
template <int NK>
__device__ __forceinline__ void expand_and_hash(const KeyArg &key, KeySlotHdr *hd, const uint32_t *te0,
                                                const uint32_t *sb, uint32_t h[4])
{
    constexpr int NR = NK + 6;
    uint32_t w[4 * (NR + 1)];
    expand_key<NK>(key.w, hd, sb, w);
    const uint32_t zero[4] = {0, 0, 0, 0};
    aes_block<NR>(w, te0, sb, zero, h);
}

// Lane k < kPowLevels of a wave writes H^(2^k) = F_k(H) to the
// slot header (F_0 is the identity).
__device__ __forceinline__ void write_hpow(KeySlotHdr *hd, const uint32_t *h, const u32x4 *__restrict__ frob, int k)
{
    if (k < kPowLevels) {
        const u32x4 H = u32x4{h[0], h[1], h[2], h[3]};
        u32x4 r = H;
        if (k > 0) {
            const u32x4 *F = frob + (uint64_t)(k - 1) * 4096;
            r = u32x4{0, 0, 0, 0};
            for (int j = 0; j < 16; ++j)
                r ^= F[j * 256 + byte_of(H, j)];
        }
        hd->hpow[k][0] = r.x;
        hd->hpow[k][1] = r.y;
        hd->hpow[k][2] = r.z;
        hd->hpow[k][3] = r.w;
    }
}

// AES tables (TE0 and the S-box as words) from global memory into LDS,
// by one 64-thread workgroup; the caller adds the barrier.
__device__ __forceinline__ void stage_aes_tables64(uint32_t *te0, uint32_t *sb, const uint32_t *te0g,
                                                   const uint32_t *sbg)
{
    uint32_t a[4], b[4];  // all eight loads in flight before the stores
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        a[r] = te0g[threadIdx.x + 64 * r];
        b[r] = sbg[threadIdx.x + 64 * r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        te0[threadIdx.x + 64 * r] = a[r];
        sb[threadIdx.x + 64 * r] = b[r];
    }
}

// One workgroup per key (blockIdx.x indexes `keys`/`slots`): the AES tables
// are staged in LDS, then one thread derives the round keys, H = E_K(0^128)
// and H^(2^k) by repeated squaring.
__global__ __launch_bounds__(64) void k_key_setup(KeyChunk chunk, const uint32_t *te0g, const uint32_t *sbg,
                                                  const u32x4 *__restrict__ frob)
{
    __shared__ uint32_t te0[256], sb[256];
    __shared__ uint32_t h_sh[4];
    stage_aes_tables64(te0, sb, te0g, sbg);
    lds_barrier();
    const KeyArg key = chunk.keys[blockIdx.x];
    KeySlotHdr *hd = reinterpret_cast<KeySlotHdr *>(chunk.slots[blockIdx.x]);
    if (threadIdx.x == 0) {
        uint32_t h[4];
        if (key.len == 16)
            expand_and_hash<4>(key, hd, te0, sb, h);
        else if (key.len == 24)
            expand_and_hash<6>(key, hd, te0, sb, h);
        else
            expand_and_hash<8>(key, hd, te0, sb, h);
        for (int i = 0; i < 4; ++i) {
            hd->h[i] = h[i];
            h_sh[i] = h[i];
        }
    }
    lds_barrier();
    write_hpow(hd, h_sh, frob, (int)threadIdx.x);
}

// a * b for one operand pair, all 64 lanes of the wave cooperating: lane i
// contributes the terms of bits i and i + 64 of a (b * x^i, b * x^(i + 64)),
// folded once, then an XOR across the wave sums them.  Every lane returns the
// product.
__device__ __forceinline__ u32x4 gf_mul_wave(u32x4 a, u32x4 b)
{
    const int lane = threadIdx.x & 63;
    const uint32_t am[4] = {a.x, a.y, a.z, a.w};
    const P128 pa = mem_to_poly(am);
    const uint32_t bm[4] = {b.x, b.y, b.z, b.w};
    const P128 pb = mem_to_poly(bm);
    const uint64_t m0 = 0ull - ((pa.lo >> lane) & 1u), m1 = 0ull - ((pa.hi >> lane) & 1u);
    const uint64_t w0 = pb.lo << lane, w1 = (pb.hi << lane) | ((pb.lo >> 1) >> (63 - lane));
    const uint64_t w2 = (pb.hi >> 1) >> (63 - lane);
    const P128 t = poly_reduce(w0 & m0, (w1 & m0) ^ (w0 & m1), (w2 & m0) ^ (w1 & m1), w2 & m1);
    const u32x4 r = poly_to_mem(t);
    return u32x4{wave_xor_u32(r.x), wave_xor_u32(r.y), wave_xor_u32(r.z), wave_xor_u32(r.w)};
}

// a * b + c * d, as above
__device__ __forceinline__ u32x4 gf_mul2_wave(u32x4 a, u32x4 b, u32x4 c, u32x4 d)
{
    const int lane = threadIdx.x & 63;
    uint64_t l0 = 0, l1 = 0, h0 = 0, h1 = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const u32x4 x = k ? c : a, y = k ? d : b;
        const uint32_t xm[4] = {x.x, x.y, x.z, x.w}, ym[4] = {y.x, y.y, y.z, y.w};
        const P128 px = mem_to_poly(xm), py = mem_to_poly(ym);
        const uint64_t m0 = 0ull - ((px.lo >> lane) & 1u), m1 = 0ull - ((px.hi >> lane) & 1u);
        const uint64_t w0 = py.lo << lane, w1 = (py.hi << lane) | ((py.lo >> 1) >> (63 - lane));
        const uint64_t w2 = (py.hi >> 1) >> (63 - lane);
        l0 ^= w0 & m0;
        l1 ^= (w1 & m0) ^ (w0 & m1);
        h0 ^= (w2 & m0) ^ (w1 & m1);
        h1 ^= w2 & m1;
    }
    const u32x4 r = poly_to_mem(poly_reduce(l0, l1, h0, h1));
    return u32x4{wave_xor_u32(r.x), wave_xor_u32(r.y), wave_xor_u32(r.z), wave_xor_u32(r.w)};
}

// Fixed-multiplier tables of one key (grid.y indexes the key).
//   blocks 0..39:   nibble-position table of H^(2^b)      (fix-ups, combine tree)
//   blocks 40..55:  byte-position table of H^64, position b - 40
//                   (per-lane Horner multiplier; one block per position, so
//                   that this table is not the launch's longest block)
//   blocks 56..71:  H^e, e = 0..63, and its 4-bit window table for the lane
//                   l = 63 - e that multiplies by it in the tile fix-up, one a wave
//   blocks 72..86:  the group lifts H^(2^s * j) and H^(64 e + 32), a wave those that
//                   share factors
// Bound by the vector units.  1024 keys: 459 us without lifts, 514 us with a wave
// and one to four products for each lift, 458 us this way (and without products
// by the field's one).
constexpr int kTab8Blocks = 16, kWinBlocks = kLanePows / 4;
constexpr int kLiftBlocks = (3 * kLiftLevels + 8 + 3) / 4;
constexpr int kKeyTableBlocks = kTab4Levels + kTab8Blocks + kWinBlocks + kLiftBlocks;
__global__ __launch_bounds__(256) void k_key_tables(SlotChunk chunk)
{
    __shared__ u32x4 basis[128];  // basis[i] = M * x^i, memory order
    __shared__ u32x4 m_sh;
    uint8_t *slot = reinterpret_cast<uint8_t *>(chunk.slots[blockIdx.y]);
    const KeySlotHdr *hd = reinterpret_cast<const KeySlotHdr *>(slot);
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    if (b < kTab4Levels + kTab8Blocks) {
        if (tid == 0) {
            const int lvl = b < kTab4Levels ? b : kStrideLevel;
            m_sh = u32x4{hd->hpow[lvl][0], hd->hpow[lvl][1], hd->hpow[lvl][2], hd->hpow[lvl][3]};
        }
    } else if (b >= kTab4Levels + kTab8Blocks + kWinBlocks) {
        // a wave forms powers that share factors, one product each
        const int q = 4 * (b - kTab4Levels - kTab8Blocks - kWinBlocks) + (int)uniform(tid >> 6);
        const auto pow2 = [&](int k) { return u32x4{hd->hpow[k][0], hd->hpow[k][1], hd->hpow[k][2], hd->hpow[k][3]}; };
        u32x4 *halves = reinterpret_cast<u32x4 *>(slot + kSlotTab8Off);
        u32x4 *high = reinterpret_cast<u32x4 *>(slot + kSlotLaneWinOff);
        const bool write = (tid & 63) == 0;
        if (q < 8) {  // H^(64 e + 32) for e = q, q + 8
            u32x4 m = pow2(5);
            for (int k = 0; k < 3; ++k)
                if ((q >> k) & 1)
                    m = gf_mul_wave(m, pow2(6 + k));
            const u32x4 m8 = gf_mul_wave(m, pow2(9));
            if (write)
                halves[q] = m, halves[q + 8] = m8;
            return;
        }
        const int chain = (q - 8) / kLiftLevels, lvl = kLiftLo + (q - 8) % kLiftLevels, at = lvl - kLiftLo;
        if (chain > 2)
            return;
        KeySlotHdr *out = reinterpret_cast<KeySlotHdr *>(slot);
        const auto lift = [&](int j, u32x4 m) {  // H^(2^lvl * j)
            u32x4 *dst = j < 9 ? reinterpret_cast<u32x4 *>(out->lift[(j - 3) >> 1][at]) : high + 8 * (j - 9) + at;
            if (write)
                *dst = m;
        };
        const bool upper = lvl <= kLiftHi - 2;  // j = 9, 11, 13, 15 too
        const u32x4 m1 = pow2(lvl);
        if (chain == 0) {
            const u32x4 m3 = gf_mul_wave(m1, pow2(lvl + 1)), m7 = gf_mul_wave(m3, pow2(lvl + 2));
            lift(3, m3);
            lift(7, m7);
            if (upper)
                lift(15, gf_mul_wave(m7, pow2(lvl + 3)));
        } else if (chain == 1) {
            const u32x4 m5 = gf_mul_wave(m1, pow2(lvl + 2));
            lift(5, m5);
            if (upper)
                lift(13, gf_mul_wave(m5, pow2(lvl + 3)));
        } else if (upper) {
            const u32x4 m9 = gf_mul_wave(m1, pow2(lvl + 3));
            lift(9, m9);
            lift(11, gf_mul_wave(m9, pow2(lvl + 1)));
        }
        return;
    } else {
        // H^e as the product of H^(2^k) over the set bits of e,
        // then lane v = 1..15 writes (v * H^e) mod P for lane 63 - e
        const int e = 4 * (b - kTab4Levels - kTab8Blocks) + (int)uniform(tid >> 6), lane = tid & 63;
        u32x4 m = {0x80u, 0u, 0u, 0u};  // the field's one
        bool one = true;
        for (int k = 0; k < 6; ++k)
            if ((e >> k) & 1) {
                const u32x4 h = {hd->hpow[k][0], hd->hpow[k][1], hd->hpow[k][2], hd->hpow[k][3]};
                m = one ? h : gf_mul_wave(m, h);
                one = false;
            }
        if (lane > 0 && lane < 16) {
            const uint32_t mm[4] = {m.x, m.y, m.z, m.w};
            const P128 pm = mem_to_poly(mm);
            P128 t;
            t.lo = 0;
            t.hi = 0;
            for (int i = 0; i < 4; ++i)
                if ((lane >> i) & 1) {
                    const P128 sh = poly_mul_xi(pm, i);
                    t.lo ^= sh.lo;
                    t.hi ^= sh.hi;
                }
            reinterpret_cast<u32x4 *>(slot + kSlotLaneWinOff)[kLanePows * lane + (63 - e)] =
                u32x4{(uint32_t)t.lo, (uint32_t)(t.lo >> 32), (uint32_t)t.hi, (uint32_t)(t.hi >> 32)};
        }
        return;
    }
    lds_barrier();
    if (tid < 128) {
        const uint32_t mm[4] = {m_sh.x, m_sh.y, m_sh.z, m_sh.w};
        basis[tid] = poly_to_mem(poly_mul_xi(mem_to_poly(mm), tid));
    }
    lds_barrier();
    if (b >= kTab4Levels) {
        // byte position k = b - kTab4Levels, value v = tid; entry-major:
        // (byte value v at position k) * M at index 16*v + k
        u32x4 *tab = reinterpret_cast<u32x4 *>(slot + kSlotTab8Off);
        const int k = b - kTab4Levels, v = tid;
        u32x4 acc = {0, 0, 0, 0};
        for (int t = 0; t < 8; ++t)
            if ((v >> t) & 1)
                acc ^= basis[8 * k + 7 - t];
        if (v)  // the entries of 0 hold lifts
            tab[16 * v + k] = acc;
        return;
    }
    u32x4 *tab = reinterpret_cast<u32x4 *>(slot + kSlotTab4Off + (uint64_t)b * kTab4Bytes);
    for (int e = tid; e < 512; e += 256) {
        const int j = e >> 4, nib = e & 15;
        const int byte = j >> 1, shift = (j & 1) ? 0 : 4;  // even j: high nibble
        u32x4 acc = {0, 0, 0, 0};
        for (int t = 0; t < 4; ++t)
            if ((nib >> t) & 1)
                acc ^= basis[8 * byte + 7 - (t + shift)];
        tab[e] = acc;
    }
}

// ---------------------------------------------------------------- GF(2^128) by table

// a * M with the nibble-position table of M (global memory, 32 gathers)
__device__ __forceinline__ u32x4 mul_tab4(u32x4 a, const u32x4 *__restrict__ tab)
{
    u32x4 r0 = {0, 0, 0, 0}, r1 = {0, 0, 0, 0};
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll 1
    for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t byte = (w[d] >> (8 * q)) & 0xffu;
            const int k = 4 * d + q;
            r0 ^= tab[(2 * k) * 16 + (byte >> 4)];
            r1 ^= tab[(2 * k + 1) * 16 + (byte & 15)];
        }
    }
    return r0 ^ r1;
}

// XOR over the 32 lanes of each half-wave (rows 0-1 and rows 2-3); every lane
// of the half-wave returns the sum.  All 64 lanes must execute it.
__device__ __forceinline__ uint32_t half_wave_xor_u32(uint32_t x)
{
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x141, 0xF, 0xF, false);  // row_half_mirror
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x140, 0xF, 0xF, false);  // row_mirror
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);  // rows 0<->1, 2<->3
    return p[0] ^ p[1];
}

// v * M for a v that all 32 lanes of a half-wave hold, with M's
// nibble-position table: lane q (0..31) reads the entry of nibble position q
// (one lookup instead of 32), then an XOR across the half-wave.  Every lane of
// the half-wave returns the product; all 64 lanes of the wave must execute
// it (active == false: the lane's half-wave contributes zero).
__device__ __forceinline__ u32x4 mul_tab4_half(u32x4 v, const u32x4 *__restrict__ tab, uint32_t q, bool active)
{
    u32x4 t = {0, 0, 0, 0};
    if (active) {
        const uint32_t k = q >> 1;  // byte position; even q: its high nibble
        const uint32_t wsel = k >> 2;
        const uint32_t word = wsel == 0 ? v.x : wsel == 1 ? v.y : wsel == 2 ? v.z : v.w;
        const uint32_t byte = (word >> (8 * (k & 3))) & 0xffu;
        t = tab[q * 16 + ((q & 1) ? (byte & 15u) : (byte >> 4))];
    }
    return u32x4{half_wave_xor_u32(t.x), half_wave_xor_u32(t.y), half_wave_xor_u32(t.z), half_wave_xor_u32(t.w)};
}

__device__ __forceinline__ u32x4 wave_xor_reduce(u32x4 a)
{
    return u32x4{wave_xor_u32(a.x), wave_xor_u32(a.y), wave_xor_u32(a.z), wave_xor_u32(a.w)};
}

// ---------------------------------------------------------------- fused tile kernel
//
// LDS layout of the passes with GHASH (148 KiB, one workgroup per CU):
//   [0, 64 KiB)        byte-position GHASH table of H^64 for the current key,
//                      entry-major: the product for byte value v at position
//                      k sits at byte 256*v + 16*k, so position k lives in
//                      bank group k (16 groups of four banks).
//   [64 KiB, 128 KiB)  AES T-tables: entry e of table t, copy c (c = 0..15)
//                      at 0x10000 + 256*e + 64*t + 4*c.
//   [128 KiB, 144 KiB) the key's lane fix-up window tables (slot layout).
//   [144 KiB, 148 KiB) the message's round-2 words (see CtrBlock): 16 bytes
//                      for each value of the low counter byte; then the tile
//                      values of a work item (two buffers of 16) and E_K(J0).
// and of counter mode alone (132 KiB):
//   [0, 128 KiB)       AES T-tables: entry e of table t, copy c (c = 0..31)
//                      at 0x10000 * (t >> 1) + 256 * e + 128 * (t & 1) + 4 * c.
//   [128 KiB, 132 KiB) the round-2 words.
//
// A wave64 ds_read_b32 takes two cycles, 32 lanes each, when no two lanes of a
// half-wave share a bank; random indices into one 1 KiB table cost about three
// times that.  With 32 copies lane l reads copy l & 31, a bank of its own
// whatever its index.  Beside the GHASH table there is room for 16 copies:
// lane l uses copy c = l & 15, and lane group g = (l >> 4) & 3 keeps its AES
// state rotated left by 8g bits.  Because T_t = rotl(T_0, 8t), a rotated state
// turns "table r, byte r" into "table (r+g)&3, byte (r+g)&3", so in every
// lookup instruction the four lane groups read four different tables and every
// lane again has a bank of its own; the price is a rotation of each round key
// word.  One v_perm_b32 per lookup builds the address from the state byte and
// the lane's table and copy.
// A ds_read_b128 serves 16 lanes per cycle, four banks each, so its 16 lanes
// must fall in 16 different bank groups.  The GHASH lookups get that from the
// schedule: in lookup j lane l reads position (j + l) & 15, with its
// accumulator held byte-rotated by l & 15 so that position is byte j of the
// rotated value; 16 consecutive lanes then read 16 different positions.

__device__ __forceinline__ uint32_t rotr_by(uint32_t x, uint32_t n) { return __builtin_amdgcn_alignbit(x, x, n); }

#define B0(x) ((x) & 0xffu)
#define B1(x) (((x) >> 8) & 0xffu)
#define B2(x) (((x) >> 16) & 0xffu)
#define B3(x) ((x) >> 24)

// The T-tables in LDS as a lane sees them; ROT: 16 copies, from LDS byte BASE,
// and a rotated state.
template <bool ROT, uint32_t BASE>
struct Tables;

template <>
struct Tables<false, 0> {
    const uint8_t *lds;
    uint32_t lo, hi;  // 4 * copy, 0x10000 | 4 * copy

    __device__ __forceinline__ Tables(const uint8_t *l, int lane) : lds(l)
    {
        lo = 4u * ((uint32_t)lane & 31u);
        hi = 0x10000u | lo;
    }
    __device__ __forceinline__ void pin() { asm volatile("" : "+v"(lo), "+v"(hi)); }
    // T_R[byte R of w]
    template <int R>
    __device__ __forceinline__ uint32_t look(uint32_t w) const
    {
        const uint32_t a = __builtin_amdgcn_perm(w, (R & 2) ? hi : lo, 0x0c020000u | ((4u + R) << 8));
        return *reinterpret_cast<const uint32_t *>(lds + 128 * (R & 1) + a);
    }
    // T_t[x] itself
    __device__ __forceinline__ uint32_t entry(int t, uint32_t x) const
    {
        return *reinterpret_cast<const uint32_t *>(lds + 0x10000 * (t >> 1) + 128 * (t & 1) + (x << 8 | lo));
    }
    __device__ __forceinline__ uint32_t rot(uint32_t x) const { return x; }
    // the S-box bytes of rows 0, 1 (2, 3), unrotated: S(x) sits in byte (t + 1) & 3 of table t's entry
    __device__ __forceinline__ uint32_t last01(uint32_t a, uint32_t b) const
    {
        return __builtin_amdgcn_perm(b, a, 0x0c0c0601u);
    }
    __device__ __forceinline__ uint32_t last23(uint32_t c, uint32_t d) const
    {
        return __builtin_amdgcn_perm(d, c, 0x04030c0cu);
    }
};

template <uint32_t BASE>
struct Tables<true, BASE> {
    const uint8_t *lds;
    uint32_t sel[4];          // v_perm selectors: byte u_r of the state word into bits 8..15
    uint32_t off[4];          // BASE | 64*u_r + 4*copy
    uint32_t sh;              // alignbit shift for rotl by 8g
    uint32_t fsel01, fsel23;  // last round: v_perm selectors of the S-box bytes

    __device__ __forceinline__ Tables(const uint8_t *l, int lane) : lds(l)
    {
        const uint32_t g = (uint32_t)(lane >> 4) & 3u, copy = (uint32_t)lane & 15u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t u = ((uint32_t)r + g) & 3u;
            sel[r] = 0x0c020000u | ((4u + u) << 8);
            off[r] = BASE | (u * 64u + copy * 4u);
        }
        const uint32_t u0 = g & 3u, u1 = (1u + g) & 3u, u2 = (2u + g) & 3u, u3 = (3u + g) & 3u;
        // S(x) sits in byte (u+1)&3 of table u
        fsel01 = ((u0 + 1u) & 3u) | ((4u + ((u1 + 1u) & 3u)) << 8) | 0x0c0c0000u;
        fsel23 = 0x00000c0cu | (((u2 + 1u) & 3u) << 16) | ((4u + ((u3 + 1u) & 3u)) << 24);
        sh = (32u - 8u * g) & 31u;
    }
    __device__ __forceinline__ void pin()
    {
        asm volatile("" : "+v"(sel[0]), "+v"(sel[1]), "+v"(sel[2]), "+v"(sel[3]), "+v"(off[0]), "+v"(off[1]), "+v"(off[2]), "+v"(off[3]));
        asm volatile("" : "+v"(sh), "+v"(fsel01), "+v"(fsel23));
    }
    template <int R>
    __device__ __forceinline__ uint32_t look(uint32_t w) const
    {
        return *reinterpret_cast<const uint32_t *>(lds + __builtin_amdgcn_perm(w, off[R], sel[R]));
    }
    __device__ __forceinline__ uint32_t entry(int t, uint32_t x) const
    {
        return *reinterpret_cast<const uint32_t *>(lds + BASE + 64 * t + (x << 8 | (off[0] & 63u)));
    }
    __device__ __forceinline__ uint32_t rot(uint32_t x) const { return rotr_by(x, sh); }
    __device__ __forceinline__ uint32_t last01(uint32_t a, uint32_t b) const { return __builtin_amdgcn_perm(b, a, fsel01); }
    __device__ __forceinline__ uint32_t last23(uint32_t c, uint32_t d) const { return __builtin_amdgcn_perm(d, c, fsel23); }
};

// Per-lane constants of the GHASH lookup schedule (q = lane & 15):
// pos[m] byte t = 16 * ((4m + t + q) & 15), the bank-group offset of lookup
// j = 4m + t; the accumulator is rotated by q bytes as a dword rotation by
// q >> 2 (two conditional swaps) and a byte shift of 8 * (q & 3) bits.
struct GhK {
    uint32_t pos[4];
    uint32_t sh;
    bool s2, s1;

    __device__ __forceinline__ void pin() { asm volatile("" : "+v"(pos[0]), "+v"(pos[1]), "+v"(pos[2]), "+v"(pos[3]), "+v"(sh)); }
};

__device__ __forceinline__ GhK gh_constants(int lane)
{
    GhK g;
    const uint32_t q = (uint32_t)lane & 15u;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        uint32_t w = 0;
        for (int t = 0; t < 4; ++t)
            w |= (((4u * m + t + q) & 15u) << 4) << (8 * t);
        g.pos[m] = w;
    }
    g.sh = 8u * (q & 3u);
    g.s2 = (q & 8u) != 0;
    g.s1 = (q & 4u) != 0;
    return g;
}

// byte i of the result is byte (i + q) & 15 of a
__device__ __forceinline__ u32x4 rot_bytes_lane(u32x4 a, const GhK &g)
{
    const u32x4 c = g.s2 ? u32x4{a.z, a.w, a.x, a.y} : a;
    const u32x4 b = g.s1 ? u32x4{c.y, c.z, c.w, c.x} : c;
    return u32x4{__builtin_amdgcn_alignbit(b.y, b.x, g.sh), __builtin_amdgcn_alignbit(b.z, b.y, g.sh),
                 __builtin_amdgcn_alignbit(b.w, b.z, g.sh), __builtin_amdgcn_alignbit(b.x, b.w, g.sh)};
}

// The Horner step a <- a * H^64 ^ x with the entry-major byte-position table at
// LDS offset 0: 16 lookups of 16 bytes, conflict-free across each 16-lane
// group, in four groups, so that they can be issued between the rounds of
// another row's AES.
struct GhashStep {
    uint32_t w[4];
    u32x4 acc, e[4];

    __device__ __forceinline__ void start(u32x4 a, u32x4 x, const GhK &g)
    {
        const u32x4 r = rot_bytes_lane(a, g);
        w[0] = r.x, w[1] = r.y, w[2] = r.z, w[3] = r.w;
        acc = x;
    }
    template <int G>
    __device__ __forceinline__ void issue(const uint8_t *__restrict__ lds, const GhK &g)
    {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            // address = 256 * (byte 4G + q of the rotated value) + 16 * position
            const uint32_t at = __builtin_amdgcn_perm(w[G], g.pos[G], 0x0c0c0000u | ((4u + q) << 8) | q);
            e[q] = *reinterpret_cast<const u32x4 *>(lds + at);
        }
    }
    __device__ __forceinline__ void absorb() { acc = xor3v(xor3v(e[0], e[1], e[2]), e[3], acc); }
};

__device__ __forceinline__ u32x4 ghash_mul8(u32x4 a, u32x4 x, const uint8_t *__restrict__ lds, const GhK &g)
{
    GhashStep s, t;  // two groups in flight
    s.start(a, x, g);
    t.start(a, u32x4{0, 0, 0, 0}, g);
    s.issue<0>(lds, g);
    t.issue<1>(lds, g);
    s.absorb();
    s.issue<2>(lds, g);
    t.absorb();
    t.issue<3>(lds, g);
    s.absorb();
    t.absorb();
    return s.acc ^ t.acc;
}

// Keeps the compiler's scheduler from moving anything across this point.
#define STAGE_END __builtin_amdgcn_sched_barrier(0)

// Rounds 3..NR of AES on the state columns after round 2.
//
// A round's sixteen lookups are issued by source column, and output column j
// is formed as soon as its last lookup (source column 3) is back, its own four
// lookups of the next round following at once, so that a wave always has
// lookups in flight.  Left to itself the compiler issues three to eight and
// waits for all of them, which left the LDS idle a third of the time in
// counter mode.
//
// With GH the GHASH step of the row before runs between the rounds: a group of
// its lookups after each of the first four rounds, absorbed a round later.
template <int NR, bool GH, typename TAB>
__device__ __forceinline__ u32x4 aes_rounds(u32x4 s, const CONST_AS uint32_t *rk, const TAB &tab, GhashStep &gs,
                                            const GhK &gk)
{
    uint32_t v[4][4];  // v[j][i]: the lookup of output column j in source column i, state row (i - j) & 3
#define ISSUE0(d, w) d[0][0] = tab.template look<0>(w), d[3][0] = tab.template look<1>(w), d[2][0] = tab.template look<2>(w), d[1][0] = tab.template look<3>(w)
#define ISSUE1(d, w) d[1][1] = tab.template look<0>(w), d[0][1] = tab.template look<1>(w), d[3][1] = tab.template look<2>(w), d[2][1] = tab.template look<3>(w)
#define ISSUE2(d, w) d[2][2] = tab.template look<0>(w), d[1][2] = tab.template look<1>(w), d[0][2] = tab.template look<2>(w), d[3][2] = tab.template look<3>(w)
#define ISSUE3(d, w) d[0][3] = tab.template look<3>(w), d[1][3] = tab.template look<2>(w), d[2][3] = tab.template look<1>(w), d[3][3] = tab.template look<0>(w)
    ISSUE0(v, s.x);
    ISSUE1(v, s.y);
    ISSUE2(v, s.z);
    ISSUE3(v, s.w);
    STAGE_END;
#pragma unroll
    for (int r = 3; r < NR; ++r) {
        uint32_t n[4][4];
        const uint32_t p0 = xor3(v[0][0], v[0][1], v[0][2]), p1 = xor3(v[1][0], v[1][1], v[1][2]);
        const uint32_t p2 = xor3(v[2][0], v[2][1], v[2][2]), p3 = xor3(v[3][0], v[3][1], v[3][2]);
        const uint32_t k0 = tab.rot(rk[4 * r + 0]), k1 = tab.rot(rk[4 * r + 1]);
        const uint32_t k2 = tab.rot(rk[4 * r + 2]), k3 = tab.rot(rk[4 * r + 3]);
        STAGE_END;
        const uint32_t t0 = xor3(p0, v[0][3], k0);
        ISSUE0(n, t0);
        STAGE_END;
        const uint32_t t1 = xor3(p1, v[1][3], k1);
        ISSUE1(n, t1);
        STAGE_END;
        const uint32_t t2 = xor3(p2, v[2][3], k2);
        ISSUE2(n, t2);
        STAGE_END;
        const uint32_t t3 = xor3(p3, v[3][3], k3);
        ISSUE3(n, t3);
        STAGE_END;
        if (GH && r >= 4 && r <= 7)
            gs.absorb();
        if (GH && r == 3)
            gs.template issue<0>(tab.lds, gk);
        if (GH && r == 4)
            gs.template issue<1>(tab.lds, gk);
        if (GH && r == 5)
            gs.template issue<2>(tab.lds, gk);
        if (GH && r == 6)
            gs.template issue<3>(tab.lds, gk);
        if (GH && r <= 7)
            STAGE_END;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[i][j] = n[i][j];
    }
    // last round: two v_perm pick a column's four S-box bytes into their
    // unrotated places, so the key is added as it is
    u32x4 o;
#define LAST(j, k)                                                                                                     \
    __builtin_amdgcn_bitop3_b32(tab.last01(v[j][j], v[j][((j) + 1) & 3]), tab.last23(v[j][((j) + 2) & 3], v[j][((j) + 3) & 3]), k, 0x56)
    o.x = LAST(0, rk[4 * NR + 0]);
    o.y = LAST(1, rk[4 * NR + 1]);
    o.z = LAST(2, rk[4 * NR + 2]);
    o.w = LAST(3, rk[4 * NR + 3]);
#undef LAST
    return o;
}

// T_t[x] read through the scalar cache (uniform x): TE0 at word 0, TE1..TE3
// from word kTe1Off of the table block
__device__ __forceinline__ uint32_t te_s(const CONST_AS uint32_t *te, int t, uint32_t x)
{
    return t == 0 ? te[x] : te[kTe1Off + 256 * (t - 1) + x];
}

// The counter block with its counter dword left out, after round 1: column i
// of round 1 is u[i] XOR one table entry of a counter byte.  GCM's big-endian
// counter is dword 3 (its low byte in state row 3), GCM-SIV's little-endian
// counter dword 0 (low byte in row 0); both low bytes reach column 0 of round 1.
template <bool SIV>
struct CtrBlock {
    uint32_t u0, u1, u2, u3;
    uint32_t k;  // the counter dword's word of round key 0

    // s: the counter block's dwords XOR round key 0 (the counter's own is not read)
    template <typename TAB>
    __device__ __forceinline__ void init(const uint32_t (&s)[4], const u32x4 &rk1, uint32_t key, const TAB &tab)
    {
        k = key;
        if (SIV) {
            u0 = uniform(tab.entry(1, B1(s[1])) ^ tab.entry(2, B2(s[2])) ^ tab.entry(3, B3(s[3])) ^ rk1.x);
            u1 = uniform(tab.entry(0, B0(s[1])) ^ tab.entry(1, B1(s[2])) ^ tab.entry(2, B2(s[3])) ^ rk1.y);
            u2 = uniform(tab.entry(0, B0(s[2])) ^ tab.entry(1, B1(s[3])) ^ tab.entry(3, B3(s[1])) ^ rk1.z);
            u3 = uniform(tab.entry(0, B0(s[3])) ^ tab.entry(2, B2(s[1])) ^ tab.entry(3, B3(s[2])) ^ rk1.w);
        } else {
            u0 = uniform(tab.entry(0, B0(s[0])) ^ tab.entry(1, B1(s[1])) ^ tab.entry(2, B2(s[2])) ^ rk1.x);
            u1 = uniform(tab.entry(0, B0(s[1])) ^ tab.entry(1, B1(s[2])) ^ tab.entry(3, B3(s[0])) ^ rk1.y);
            u2 = uniform(tab.entry(0, B0(s[2])) ^ tab.entry(2, B2(s[0])) ^ tab.entry(3, B3(s[1])) ^ rk1.z);
            u3 = uniform(tab.entry(1, B1(s[0])) ^ tab.entry(2, B2(s[1])) ^ tab.entry(3, B3(s[2])) ^ rk1.w);
        }
    }

    // Round-2 words of counters whose low byte is `low`: column 0 of round 1 is
    // the only one that byte reaches, and it does not depend on the upper bits,
    // so the four entries that round 2 reads of it are one 16-byte word a low
    // byte and message.
    template <typename TAB>
    __device__ __forceinline__ u32x4 low_words(uint32_t low, const TAB &tab) const
    {
        const uint32_t x0 = u0 ^ (SIV ? tab.entry(0, (low ^ k) & 0xffu) : tab.entry(3, low ^ B3(k)));
        return u32x4{tab.entry(0, B0(x0)), tab.entry(3, B3(x0)), tab.entry(2, B2(x0)), tab.entry(1, B1(x0))};
    }

    // the rest of the state after round 2, for upper counter bits `hi` (uniform)
    __device__ __forceinline__ u32x4 high_words(uint32_t hi, const CONST_AS uint32_t *rk,
                                                const CONST_AS uint32_t *te) const
    {
        const uint32_t v = SIV ? (hi << 8) ^ k : bswap32(hi << 8) ^ k;
        const uint32_t a1 = u1 ^ (SIV ? te_s(te, 3, B3(v)) : te_s(te, 2, B2(v)));
        const uint32_t a2 = u2 ^ (SIV ? te_s(te, 2, B2(v)) : te_s(te, 1, B1(v)));
        const uint32_t a3 = u3 ^ (SIV ? te_s(te, 1, B1(v)) : te_s(te, 0, B0(v)));
        return u32x4{te_s(te, 1, B1(a1)) ^ te_s(te, 2, B2(a2)) ^ te_s(te, 3, B3(a3)) ^ rk[8],
                     te_s(te, 0, B0(a1)) ^ te_s(te, 1, B1(a2)) ^ te_s(te, 2, B2(a3)) ^ rk[9],
                     te_s(te, 0, B0(a2)) ^ te_s(te, 1, B1(a3)) ^ te_s(te, 3, B3(a1)) ^ rk[10],
                     te_s(te, 0, B0(a3)) ^ te_s(te, 2, B2(a1)) ^ te_s(te, 3, B3(a2)) ^ rk[11]};
    }
    // the same through the LDS tables, `hi` being the lane's
    template <typename TAB>
    __device__ __forceinline__ u32x4 high_words_lds(uint32_t hi, const CONST_AS uint32_t *rk, const TAB &tab) const
    {
        const uint32_t v = SIV ? (hi << 8) ^ k : bswap32(hi << 8) ^ k;
        const uint32_t a1 = u1 ^ (SIV ? tab.entry(3, B3(v)) : tab.entry(2, B2(v)));
        const uint32_t a2 = u2 ^ (SIV ? tab.entry(2, B2(v)) : tab.entry(1, B1(v)));
        const uint32_t a3 = u3 ^ (SIV ? tab.entry(1, B1(v)) : tab.entry(0, B0(v)));
        return u32x4{tab.entry(1, B1(a1)) ^ tab.entry(2, B2(a2)) ^ tab.entry(3, B3(a3)) ^ rk[8],
                     tab.entry(0, B0(a1)) ^ tab.entry(1, B1(a2)) ^ tab.entry(2, B2(a3)) ^ rk[9],
                     tab.entry(0, B0(a2)) ^ tab.entry(1, B1(a3)) ^ tab.entry(3, B3(a1)) ^ rk[10],
                     tab.entry(0, B0(a3)) ^ tab.entry(2, B2(a1)) ^ tab.entry(3, B3(a2)) ^ rk[11]};
    }
};

// a * c_l for this lane's fixed multiplier c_l = H^(63 - lane), through its
// 4-bit window table in LDS (entry (v, l) = (v * c_l) mod P at
// win + 16 * (64 v + l)): a comb over the eight nibble positions of the
// four words of a, 256-bit accumulate with word-aligned XORs, one fold at the
// end.  32 conflict-free ds_read_b128 (16 consecutive lanes read 16
// different bank groups) and about 300 VALU instructions.
template <int LANES>
__device__ __forceinline__ u32x4 gf_mul_lanewin(u32x4 a, const uint8_t *__restrict__ wins, int lane)
{
    const uint32_t am[4] = {a.x, a.y, a.z, a.w};
    const P128 pa = mem_to_poly(am);
    const uint32_t aw[4] = {(uint32_t)pa.lo, (uint32_t)(pa.lo >> 32), (uint32_t)pa.hi, (uint32_t)(pa.hi >> 32)};
    const uint8_t *win = wins + 16u * (uint32_t)(lane & (LANES - 1));
    uint32_t acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 7; q >= 0; --q) {
#pragma unroll
        for (int k = 7; k > 0; --k)
            acc[k] = __builtin_amdgcn_alignbit(acc[k], acc[k - 1], 28);  // acc <<= 4
        acc[0] <<= 4;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const uint32_t v = (aw[w] >> (4 * q)) & 15u;
            const u32x4 t = *reinterpret_cast<const u32x4 *>(win + 16u * LANES * v);
            acc[w] ^= t.x;
            acc[w + 1] ^= t.y;
            acc[w + 2] ^= t.z;
            acc[w + 3] ^= t.w;
        }
    }
    const P128 r = poly_reduce((uint64_t)acc[0] | ((uint64_t)acc[1] << 32), (uint64_t)acc[2] | ((uint64_t)acc[3] << 32),
                               (uint64_t)acc[4] | ((uint64_t)acc[5] << 32), (uint64_t)acc[6] | ((uint64_t)acc[7] << 32));
    return poly_to_mem(r);
}

// Zero-padded load of block `blk` of a buffer of `total` bytes.  (All buffers
// are addressed in the global address space: a flat access anywhere in the row
// loop counts as an LDS access too, and the compiler then drains the LDS queue
// at every wait of the loop instead of waiting for the lookups it needs.)
__device__ __forceinline__ u32x4 load_block_partial(const GLOBAL_AS uint8_t *p, uint64_t blk, uint64_t total)
{
    const uint64_t off = blk * 16;
    if (off + 16 <= total)
        return *reinterpret_cast<const GLOBAL_AS u32x4 *>(p + off);
    // whole words, then the bytes after them: at most six loads that wait for
    // nothing but each other's issue (one byte after another, each on its way
    // before the next is asked for, took up to fifteen trips to memory)
    const uint32_t nb = off < total ? (uint32_t)(total - off) : 0u, q = nb & ~3u, k = nb & 3u;
    const GLOBAL_AS uint32_t *w = reinterpret_cast<const GLOBAL_AS uint32_t *>(p + off);
    const GLOBAL_AS uint8_t *e = p + off + q;
    uint32_t w0 = 0, w1 = 0, w2 = 0, b0 = 0, b1 = 0, b2 = 0;
    if (nb >= 4)
        w0 = w[0];
    if (nb >= 8)
        w1 = w[1];
    if (nb >= 12)
        w2 = w[2];
    if (k > 0)
        b0 = e[0];
    if (k > 1)
        b1 = e[1];
    if (k > 2)
        b2 = e[2];
    const uint32_t t = b0 | b1 << 8 | b2 << 16;
    return u32x4{q == 0 ? t : w0, q == 4 ? t : w1, q == 8 ? t : w2, q == 12 ? t : 0u};
}

__device__ __forceinline__ uint32_t keep_bytes(uint32_t w, int nb)  // keep the low nb bytes (nb may be <=0 or >=4)
{
    return nb <= 0 ? 0u : nb >= 4 ? w : (w & ((1u << (8 * nb)) - 1u));
}

__device__ __forceinline__ u32x4 mask_block(u32x4 v, uint64_t blk, uint64_t total)
{
    const uint64_t off = blk * 16;
    if (off + 16 <= total)
        return v;
    const int nb = (int)(total - off);  // 1..15 valid bytes
    return u32x4{keep_bytes(v.x, nb), keep_bytes(v.y, nb - 4), keep_bytes(v.z, nb - 8), keep_bytes(v.w, nb - 12)};
}

__device__ __forceinline__ void store_block_partial(GLOBAL_AS uint8_t *p, uint64_t blk, uint64_t total, u32x4 v)
{
    const uint64_t off = blk * 16;
    if (off + 16 <= total) {
        *reinterpret_cast<GLOBAL_AS u32x4 *>(p + off) = v;
        return;
    }
    const uint32_t nb = off < total ? (uint32_t)(total - off) : 0u, q = nb & ~3u, k = nb & 3u;
    GLOBAL_AS uint32_t *w = reinterpret_cast<GLOBAL_AS uint32_t *>(p + off);
    GLOBAL_AS uint8_t *e = p + off + q;
    const uint32_t t = q == 0 ? v.x : q == 4 ? v.y : q == 8 ? v.z : v.w;
    if (nb >= 4)
        w[0] = v.x;
    if (nb >= 8)
        w[1] = v.y;
    if (nb >= 12)
        w[2] = v.z;
    if (k > 0)
        e[0] = (uint8_t)t;
    if (k > 1)
        e[1] = (uint8_t)(t >> 8);
    if (k > 2)
        e[2] = (uint8_t)(t >> 16);
}

__device__ __forceinline__ u32x4 rev_block(u32x4 x) { return u32x4{bswap32(x.w), bswap32(x.z), bswap32(x.y), bswap32(x.x)}; }

// What a tile kernel does: GCM; counter mode only; GCM-SIV's POLYVAL alone
// (encrypt, first pass), its counter mode alone (second pass, once the tag is
// known), and its counter mode with the POLYVAL of the output (decrypt-verify).
constexpr int kGcm = 0, kCtr = 1, kSivHash = 2, kSivCtr = 3, kSivDec = 4;

template <int KIND>
struct Kind {
    static constexpr bool gh = KIND == kGcm || KIND == kSivHash || KIND == kSivDec;
    static constexpr bool aes = KIND != kSivHash;
    static constexpr bool siv = KIND == kSivHash || KIND == kSivCtr || KIND == kSivDec;
    using tables = Tables<gh, gh ? 0x10000u : 0u>;
    // LDS bytes: fix-up windows (GHASH passes), round-2 words, group sums, total
    static constexpr uint32_t windows = 0x20000u, round2 = gh ? 0x24000u : 0x20000u;
    static constexpr uint32_t sums = round2 + 0x1000u;
    static constexpr uint32_t firsts = sums + (gh ? 16u * (2 * 16 + 1) : 0u);  // a wave's first round-2 words
    static constexpr uint32_t lds = firsts + (aes ? 32u * 16 : 0u);
};

// A message's counter block; c1: the counter value of data block 0 (J0's own is
// one less, but for a streamed segment); cur: the round-2 words of upper
// counter bits hc.  load() asks for what it is made of while the tables are on
// their way, derive() looks the words up in the staged tables; the words of the
// waves' first rows are worked out by one wave, a lane each.  The sixteen waves
// issue what stands between the staging and the first row at four instructions
// a cycle between them, so that it counts (5000 cycles of 55000 at 16 MiB).
template <bool SIV>
struct Counters {
    CtrBlock<SIV> c;
    uint32_t c1, hc;
    u32x4 cur;
    uint32_t s[4];
    u32x4 rk1;
    uint32_t key;

    __device__ __forceinline__ void load(const CONST_AS MsgDesc *dp)
    {
        const CONST_AS uint32_t *rk = cptr<uint32_t>(reinterpret_cast<const void *>(dp->slot));
        const uint64_t jaddr = dp->j0;
        const CONST_AS uint32_t *jw = cptr<uint32_t>(reinterpret_cast<const void *>(jaddr));
        s[0] = dp->iv[0], s[1] = dp->iv[1], s[2] = dp->iv[2], s[3] = 0;  // J0 = IV || 0^31 || 1
        c1 = 2u + dp->ctr_off;
        if (SIV) {  // the counter block is the tag with its top bit set
            s[1] = jw[1], s[2] = jw[2], s[3] = jw[3];
            c1 = jw[0];
        } else if (jaddr) {  // J0 computed on the device from an IV that is not 96 bits
            s[0] = jw[0], s[1] = jw[1], s[2] = jw[2];
            c1 = bswap32(jw[3]) + 1u + dp->ctr_off;
        }
        key = rk[SIV ? 0 : 3];
        rk1 = u32x4{rk[4], rk[5], rk[6], rk[7]};
#pragma unroll
        for (int i = 0; i < 4; ++i)
            s[i] ^= rk[i];
    }
    template <typename TAB>
    __device__ __forceinline__ void derive(const TAB &tab)
    {
        c.init(s, rk1, key, tab);
    }
    // upper counter bits of the first row of tile t that has data
    __device__ __forceinline__ uint32_t first_row(const CONST_AS MsgDesc *dp, int64_t t, bool head) const
    {
        const int64_t jb = (t << dp->log2B) - (int64_t)dp->z - (int64_t)dp->na;  // data block index of the tile's start
        return ((uint32_t)(head || jb < 0 ? -((-jb) & 63) : jb) + c1) >> 8;
    }
};

// One wave processes wave tile t of a message: rows of 64 consecutive blocks,
// lane l on block 64 r + l, so every load and store moves one contiguous KiB.
// Rows [fa, fb) hold 64 whole data blocks and rows [aa, ab) 64 whole AAD
// blocks; the others (zero padding, partial blocks, the length block) load and
// store lane by lane.  E_K(J0) is the keystream block of the lane before the
// first data block, whose counter is J0's own; only where no such lane exists
// (no AAD and no padding) does the first wave run a row ahead of its tile for it.  A streamed segment's
// counters start ctr_off blocks after J0 + 1.
// a_l = sum_r X_(64r+l) * (H^64)^(R-1-r) by Horner on lane l, then the tile's
// value is sum_l a_l * H^(63-l).  GCM-SIV hashes byte-reversed blocks.
template <int NR, int KIND>
__device__ __forceinline__ u32x4 wave_tile(const CONST_AS MsgDesc *dp, uint64_t t, bool head,
                                           const Counters<Kind<KIND>::siv> &cs, uint8_t *__restrict__ lds,
                                           const typename Kind<KIND>::tables &tab, const GhK &gk,
                                           const CONST_AS uint32_t *te, u32x4 *__restrict__ ekg)
{
    constexpr bool GH = Kind<KIND>::gh, SIV = Kind<KIND>::siv, AES = Kind<KIND>::aes;
    const int lane = threadIdx.x & 63;
    const CONST_AS uint32_t *rk = cptr<uint32_t>(reinterpret_cast<const void *>(dp->slot));
    const CtrBlock<SIV> &c = cs.c;
    const uint32_t c1 = cs.c1;

    const uint32_t log2B = dp->log2B;
    const int32_t R = (int32_t)(1u << (log2B - 6));
    const int64_t vbase = (int64_t)(t << log2B) - (int64_t)dp->z;  // GHASH index of lane 0, row 0
    // the first row: the head of the message starts at index 0 (which may lie
    // in the tile before this one), any other tile at its own row 0
    const int32_t r0 = head ? (int32_t)((-vbase) >> 6) : 0;
    const int64_t na = (int64_t)dp->na, nfull = (int64_t)(dp->len >> 4);
    // rows whose 64 blocks all lie in blocks [first, end) of the sequence
    auto whole_rows = [&](int64_t first, int64_t end, int32_t &lo, int32_t &hi) {
        const int64_t l = first - vbase, h = end - vbase - 64;  // 64 r >= l, 64 r <= h
        const int64_t f0 = (l + 63) >> 6, f1 = (h >> 6) + 1;
        lo = f0 > (int64_t)r0 ? (f0 < (int64_t)R ? (int32_t)f0 : R) : r0;
        hi = f1 > (int64_t)lo ? (f1 < (int64_t)R ? (int32_t)f1 : R) : lo;
    };
    int32_t fa, fb, aa = 0, ab = 0;
    const int64_t jb = vbase - na;  // data block index of lane 0, row 0
    if (!head && jb >= 0 && jb + 64 * (int64_t)R <= nfull) {
        fa = 0, fb = R;  // whole data blocks throughout, as in nearly every tile
    } else {
        whole_rows(na, na + nfull, fa, fb);
        if (GH) {
            const int64_t end = (int64_t)(dp->aad_len >> 4);
            whole_rows(0, KIND == kGcm && end == na ? end - 1 : end, aa, ab);
        }
    }

    uint32_t hc = cs.hc;  // upper counter bits `cur` belongs to
    u32x4 cur = cs.cur;
    // The state after round 2 of the row whose first counter is `base`: its
    // counters are base + lane (mod 2^32), whose upper 24 bits change at most
    // once inside the row, and then by one.
    auto round2 = [&](uint32_t base) {
        const uint32_t low = (base + (uint32_t)lane) & 255u;
        u32x4 s = *reinterpret_cast<const u32x4 *>(lds + Kind<KIND>::round2 + 16u * low);
        const uint32_t h = base >> 8;
        if (h != hc) {
            cur = c.high_words(h, rk, te);
            hc = h;
        }
        if ((base & 255u) > 192u) {
            const uint32_t h1 = (h + 1u) & 0xffffffu;
            const u32x4 nxt = c.high_words(h1, rk, te);
            const bool up = low < (base & 255u);  // this lane's low counter byte wrapped inside the row
            s ^= u32x4{up ? nxt.x : cur.x, up ? nxt.y : cur.y, up ? nxt.z : cur.z, up ? nxt.w : cur.w};
            cur = nxt;
            hc = h1;
        } else {
            s ^= cur;
        }
        return u32x4{tab.rot(s.x), tab.rot(s.y), tab.rot(s.z), tab.rot(s.w)};
    };

    // GHASH runs one row behind: a is the Horner value without the pending row xp
    u32x4 a = {0, 0, 0, 0}, xp = {0, 0, 0, 0};
    const bool first = KIND == kGcm && dp->ctr_off == 0;  // E_K(J0) is wanted
    const bool ek = first && head && (dp->z & 63) == 0 && na == 0;
    __builtin_amdgcn_s_setprio(3);
    for (int32_t r = ek ? r0 - 1 : r0; r < R;) {
        if (GH && r >= aa && r < ab) {
            // rows of 64 whole AAD blocks: GHASH alone
            const GLOBAL_AS u32x4 *src = gptr<const u32x4>(dp->aad) + (vbase + 64 * (int64_t)r) + lane;
            for (; r < ab; ++r, src += 64) {
                const u32x4 x = *src;
                a = ghash_mul8(a, xp, lds, gk);
                xp = SIV ? rev_block(x) : x;
            }
            continue;
        }
        if (r < fa || r >= fb) {
            // a row with zero padding, AAD, a partial block or the length
            // block, or the extra row for E_K(J0)
            const CONST_AS MsgDesc *bp = dp;
            asm volatile("" : "+s"(bp));
            const bool ekrow = ek && r < r0;
            const int64_t v0 = vbase + 64 * (int64_t)r, v = v0 + lane;
            const int64_t ndat = (int64_t)bp->n;
            const bool data = v >= na && v < na + ndat;
            const uint64_t j = (uint64_t)(v - na);
            // some lane needs a keystream block (the one before the first data block for E_K(J0))
            const bool hot = AES && (ekrow || (v0 + 64 > (first ? na - 1 : na) && v0 < na + ndat));
            u32x4 ks = {0, 0, 0, 0}, x = {0, 0, 0, 0};
            if (!ekrow && v >= 0 && v < na + ndat && (GH || data))  // on its way during the rounds
                x = load_block_partial(data ? gptr<const uint8_t>(bp->in) : gptr<const uint8_t>(bp->aad),
                                       data ? j : (uint64_t)v, data ? bp->len : bp->aad_len);
            if (hot) {
                GhashStep none;
                ks = aes_rounds<NR, false>(round2(ekrow ? c1 - 1u : (uint32_t)jb + 64u * (uint32_t)r + c1), rk, tab, none, gk);
            }
            ++r;
            if (first && hot && (ekrow ? lane == 0 : v == na - 1)) {
                *reinterpret_cast<u32x4 *>(lds + Kind<KIND>::sums + 16 * 32) = ks;
                *ekg = ks;  // after the message's partials
            }
            if (ekrow)
                continue;
            if (AES && data) {
                const u32x4 o = x ^ ks;
                store_block_partial(gptr<uint8_t>(bp->out), j, bp->len, o);
                x = (SIV || bp->op == 0) ? mask_block(o, j, bp->len) : x;
            } else if (GH && v == na + ndat) {
                const uint64_t abits = bp->aad_len * 8, cbits = bp->len * 8;
                x = SIV ? u32x4{(uint32_t)abits, (uint32_t)(abits >> 32), (uint32_t)cbits, (uint32_t)(cbits >> 32)}
                        : u32x4{bswap32((uint32_t)(abits >> 32)), bswap32((uint32_t)abits),
                                bswap32((uint32_t)(cbits >> 32)), bswap32((uint32_t)cbits)};
            }
            if (GH) {
                if (r > r0 + 1)  // nothing precedes the tile's first row
                    a = ghash_mul8(a, xp, lds, gk);
                xp = SIV ? rev_block(x) : x;
            }
            continue;
        }
        // Rows of 64 whole data blocks.  Issue priority falls as the wave gets
        // through them (at 5/8, 3/4 and 7/8), so that waves the arbiter has
        // left behind catch up and the compute unit stays full until its last
        // tile ends.  Rounded so that a wave with two rows or more passes
        // through all levels: 16 MiB (four rows) 16.2 -> 14.8 us in counter
        // mode with AES-128, a 256 MiB stream in 16 MiB segments 446 -> 418 us.
        const int32_t span = fb - fa;
        const int32_t q1 = fa + (5 * span >> 3), q2 = fa + (3 * span >> 2), q3 = fa + (7 * span >> 3);
        const GLOBAL_AS uint8_t *src = gptr<const uint8_t>(dp->in) + 16 * (jb + 64 * (int64_t)r);
        GLOBAL_AS uint8_t *dst = gptr<uint8_t>(dp->out) + 16 * (jb + 64 * (int64_t)r);
        uint32_t base = (uint32_t)jb + 64u * (uint32_t)r + c1;
        const uint32_t loff = 16u * (uint32_t)lane;
        const bool enc = SIV || dp->op == 0;
        for (; r < fb; ++r, src += 1024, dst += 1024, base += 64) {
            if (r == q1)
                __builtin_amdgcn_s_setprio(2);
            if (r == q2)
                __builtin_amdgcn_s_setprio(1);
            if (r == q3)
                __builtin_amdgcn_s_setprio(0);
            const u32x4 x = *reinterpret_cast<const GLOBAL_AS u32x4 *>(src + loff);
            if (!AES) {
                a = ghash_mul8(a, xp, lds, gk);
                xp = SIV ? rev_block(x) : x;
                continue;
            }
            const CONST_AS uint32_t *rkr = rk;
            asm volatile("" : "+s"(rkr));  // round keys are read again each row instead of held across all of them
            GhashStep gs;
            if (GH)
                gs.start(a, xp, gk);
            const u32x4 s = round2(base);
            const u32x4 o = x ^ aes_rounds<NR, GH>(s, rkr, tab, gs, gk);
            __builtin_nontemporal_store(o, reinterpret_cast<GLOBAL_AS u32x4 *>(dst + loff));
            if (GH) {
                a = gs.acc;
                xp = enc ? o : x;
                if (SIV)
                    xp = rev_block(xp);
            }
        }
    }
    if (!GH)
        return a;
    if (R > r0 + 1)
        a = ghash_mul8(a, xp, lds, gk);
    else
        a = xp;
    // fix-up: a * H^(63 - lane) through the lane's window table in LDS
    return wave_xor_reduce(gf_mul_lanewin<64>(a, lds + Kind<KIND>::windows, lane));
}

// T-tables into LDS, every copy of every entry: a thread's loads, then its
// stores (the caller does other things between them and adds the barrier).
//
// 32 copies: 16-byte unit i of each 64 KiB half holds four copies of entry
// i >> 4 of table ((i >> 3) & 1), in the upper half of the table after next.
// 16 copies: unit i of the 64 KiB holds four copies of entry i >> 4 of table
// (i >> 2) & 3.
template <int NT>
struct StageTables {
    static constexpr int kPer = (4096 + NT - 1) / NT;
    uint32_t v[kPer];

    __device__ __forceinline__ void load(const uint32_t *__restrict__ te0g)
    {
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int i = (int)threadIdx.x + r * NT;
            v[r] = i < 4096 ? te0g[i >> 4] : 0u;
        }
    }
    template <bool ROT, uint32_t BASE>
    __device__ __forceinline__ void store(u32x4 *lds_v, const Tables<ROT, BASE> &) const
    {
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int i = (int)threadIdx.x + r * NT;
            if (i >= 4096)
                break;
            if (ROT) {
                const uint32_t x = rotr_by(v[r], (32u - 8u * ((uint32_t)(i >> 2) & 3u)) & 31u);
                lds_v[BASE / 16 + i] = u32x4{x, x, x, x};
            } else {
                const uint32_t lo = (i & 8) ? rotl32(v[r], 8) : v[r];  // tables 0, 1
                const uint32_t hi = rotr_by(lo, 16);                   // tables 2, 3
                lds_v[i] = u32x4{lo, lo, lo, lo};
                lds_v[4096 + i] = u32x4{hi, hi, hi, hi};
            }
        }
    }
};

// The key's GHASH table of H^64 (64 KiB, LDS bytes [0, 64 KiB)) and its lane
// fix-up windows (16 KiB, LDS bytes [128 KiB, 144 KiB)) from the key slot: a
// thread's loads, then its stores (the caller does other things between them
// and adds the barriers).
template <int NT>
struct StageKeys {
    static constexpr uint32_t kTab = 4096, kWin = 1024;
    static constexpr int kPerT = (int)((kTab + NT - 1) / NT), kPerW = (int)((kWin + NT - 1) / NT);
    u32x4 a[kPerT], b[kPerW];

    __device__ __forceinline__ void load(uint64_t slot)
    {
        const GLOBAL_AS u32x4 *tab = gptr<const u32x4>(slot + kSlotTab8Off);
        const GLOBAL_AS u32x4 *win = gptr<const u32x4>(slot + kSlotLaneWinOff);
        // entries of 0: the slot keeps lifts there
#pragma unroll
        for (int r = 0; r < kPerT; ++r) {
            const uint32_t q = threadIdx.x + (uint32_t)(r * NT);
            if (kTab % NT == 0 || q < kTab)
                a[r] = q < 16 ? u32x4{0, 0, 0, 0} : tab[q];
        }
#pragma unroll
        for (int r = 0; r < kPerW; ++r) {
            const uint32_t q = threadIdx.x + (uint32_t)(r * NT);
            if (kWin % NT == 0 || q < kWin)
                b[r] = q < (uint32_t)kLanePows ? u32x4{0, 0, 0, 0} : win[q];
        }
    }
    __device__ __forceinline__ void store(u32x4 *lds_v) const
    {
#pragma unroll
        for (int r = 0; r < kPerT; ++r) {
            const uint32_t q = threadIdx.x + (uint32_t)(r * NT);
            if (kTab % NT == 0 || q < kTab)
                lds_v[q] = a[r];
        }
#pragma unroll
        for (int r = 0; r < kPerW; ++r) {
            const uint32_t q = threadIdx.x + (uint32_t)(r * NT);
            if (kWin % NT == 0 || q < kWin)
                lds_v[8192 + q] = b[r];
        }
    }
};

// A workgroup covers WAVES consecutive tiles of a message per work item; one
// message (single) or a batch with a list of items.
//
// What bounds it is the LDS.  Per row of 64 blocks and CU, AES-256: 192 b32
// lookups of two cycles, one b128 of four for round 2 and 16 b128 of GHASH, 453
// cycles (by the counter of its active cycles) of 528 over the whole launch, with
// 427 vector instructions.  (16 waves that do nothing else get a b32 lookup every
// 2.05 cycles, every 2.27 where each address depends on the lookup before, as it
// does in AES.)  1 GiB with AES-256 / AES-128:
//   GCM           1058 -> 1039 us, 823 -> 805 us
//   counter mode  1006 ->  824 us, 746 -> 627 us (32 table copies: no key
//                 rotations, 449 cycles a row where it took 566)
//   SIV encrypt   1150 -> 1059 us, 917 -> 854 us
// against a loop with 197 lookups, whose waits drained the LDS queue every few
// lookups in counter mode, and with 16 copies in every pass.
//
// Groups: wave tile t of T stands for position t - T of the sequence of tiles
// counted from its end, and a work item covers the tiles of WAVES consecutive
// places of the sequence padded at its start to a multiple of 2^log2G, so its
// groups are whole.  Each wave multiplies its tile's value by H^(B * j) for the
// j tiles of the group after it, and one wave XORs a group's values and lifts
// the sum past the groups after it: about 2 us at the end of an item, for which
// the tree over 4097 partials that followed 1 GiB (18 us) becomes an XOR of 256
// (2.4 us).  A message of one group needs nothing at all after the tiles:
// the same wave multiplies by H once more, adds E_K(J0) and writes the tag or
// compares it, and clears a rejected output.
__device__ __forceinline__ void finish_message(const CONST_AS MsgDesc *dp, u32x4 v, u32x4 ek, bool times_h)
{
    const int lane = threadIdx.x & 63;
    u32x4 s = v;
    if (times_h) {
        const CONST_AS KeySlotHdr *hd = cptr<KeySlotHdr>(reinterpret_cast<const void *>(dp->slot));
        s = gf_mul_wave(v, u32x4{hd->hpow[0][0], hd->hpow[0][1], hd->hpow[0][2], hd->hpow[0][3]});
    }
    if (dp->yout) {
        if (lane == 0)
            *gptr<u32x4>(dp->yout) = s;
        return;
    }
    const u32x4 tag = s ^ ek;
    const int tl = (int)dp->tag_len;  // T = MSB_t of the full tag
    const uint32_t mine = byte_of(tag, lane & 15);
    GLOBAL_AS uint8_t *dst = gptr<uint8_t>(dp->tag);
    if (dp->op == 0) {
        if (lane < tl)
            dst[lane] = (uint8_t)mine;
        return;
    }
    // every byte is compared, whatever the others gave
    const uint32_t diff = lane < tl ? mine ^ dst[lane] : 0u;
    const bool ok = __builtin_amdgcn_ballot_w64(diff != 0) == 0;
    if (lane == 0)
        *gptr<int32_t>(dp->ok) = ok ? 1 : 0;
    if (ok)
        return;
    GLOBAL_AS uint8_t *out = gptr<uint8_t>(dp->out);
    const uint64_t len = dp->len, nfull = len >> 4;
    for (uint64_t j = (uint64_t)lane; j < nfull; j += 64)
        reinterpret_cast<GLOBAL_AS u32x4 *>(out)[j] = u32x4{0, 0, 0, 0};
    if (lane < (int)(len & 15))
        out[nfull * 16 + (uint64_t)lane] = 0;
}

// XOR over aligned sets of n = 4, 8 or 16 lanes; every lane of a set returns it
__device__ __forceinline__ uint32_t set_xor_u32(uint32_t x, int n)
{
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    x ^= __builtin_amdgcn_update_dpp(0u, x, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
    const uint32_t y = x ^ __builtin_amdgcn_update_dpp(0u, x, 0x141, 0xF, 0xF, false);  // row_half_mirror
    x = n > 4 ? y : x;
    const uint32_t z = x ^ __builtin_amdgcn_update_dpp(0u, x, 0x140, 0xF, 0xF, false);  // row_mirror
    return n > 8 ? z : x;
}

// H^(B * e) for B = 2^log2B, 1 <= e <= 15 (uniform), from the slot
__device__ __forceinline__ u32x4 group_lift(uint64_t slot, uint32_t log2B, uint32_t e)
{
    const CONST_AS KeySlotHdr *hd = cptr<KeySlotHdr>(reinterpret_cast<const void *>(slot));
    const uint32_t z = (uint32_t)__builtin_ctz(e), j = e >> z, at = log2B - kLiftLo + z;
    const CONST_AS uint32_t *w = j == 1  ? hd->hpow[kLiftLo + at]
                                 : j < 9 ? hd->lift[(j - 3) >> 1][at]
                                         : cptr<uint32_t>(reinterpret_cast<const void *>(slot + kSlotLaneWinOff)) +
                                               4 * (8 * (j - 9) + at);
    return u32x4{w[0], w[1], w[2], w[3]};
}

// v * H^(2^s * e) (e uniform), by digits of four bits while the slot has their
// powers, then by bits
__device__ __forceinline__ u32x4 lift_by(u32x4 v, uint64_t slot, uint32_t s, uint64_t e)
{
    const CONST_AS KeySlotHdr *hd = cptr<KeySlotHdr>(reinterpret_cast<const void *>(slot));
#pragma unroll 1
    for (; e; ) {
        const bool digit = s <= (uint32_t)kLiftHi - 2;
        const uint32_t d = (uint32_t)e & (digit ? 15u : 1u);
        if (d)
            v = gf_mul_wave(v, digit ? group_lift(slot, s, d)
                                     : u32x4{hd->hpow[s][0], hd->hpow[s][1], hd->hpow[s][2], hd->hpow[s][3]});
        e >>= digit ? 4 : 1;
        s += digit ? 4 : 1;
    }
    return v;
}

// One wave: the values of group `part` of the WAVES tile values in `sums`, groups
// of G, to the message's partial, multiplied by H^(blocks of the groups after it)
// so that the verdict is their XOR; or, for a message of one group, to its tag.
// The three groups of twelve waves are three waves' work: 64 MiB in tiles of one
// row 255 -> 193 us, 1 MiB of GCM-SIV verified 21.2 -> 20.2.
template <int WAVES>
constexpr uint32_t kParts = WAVES == 12 ? 3 : 1;  // groups of an item (group_log2)

template <int WAVES>
__device__ __forceinline__ void sum_group(const CONST_AS MsgDesc *dp, const u32x4 *sums, const u32x4 *ekw, uint32_t G,
                                          uint32_t log2G, bool finish, bool times_h, uint32_t first, uint32_t part,
                                          uint64_t nparts, u32x4 *__restrict__ partials)
{
    const int lane = threadIdx.x & 63, n = (int)G;
    const uint64_t at = ((uint64_t)first >> log2G) + part;
    if (at >= nparts)
        return;
    const u32x4 v = lane < n ? sums[part * G + (uint32_t)lane] : u32x4{0, 0, 0, 0};
    const u32x4 g = {set_xor_u32(v.x, n), set_xor_u32(v.y, n), set_xor_u32(v.z, n), set_xor_u32(v.w, n)};
    const u32x4 y = {uniform(g.x), uniform(g.y), uniform(g.z), uniform(g.w)};
    if (finish) {
        finish_message(dp, y, *ekw, times_h);
        return;
    }
    const u32x4 p = lift_by(y, dp->slot, dp->log2B + log2G, nparts - 1 - at);
    if (lane == 0)
        partials[dp->tile_base + at] = p;
}

template <int WAVES, bool BATCH, int KIND>
__global__ __launch_bounds__(WAVES * 64) void k_gcm_tiles(MsgDesc single, const MsgDesc *__restrict__ descs,
                                                          const WorkItem *__restrict__ items, uint32_t n_items,
                                                          const uint32_t *__restrict__ te0g,
                                                          u32x4 *__restrict__ partials, uint32_t *counters)
{
    using K = Kind<KIND>;
    __shared__ u32x4 lds_v[K::lds / 16];
    uint8_t *lds = reinterpret_cast<uint8_t *>(lds_v);
    const CONST_AS uint32_t *te = cptr<uint32_t>(te0g);
    const int lane = threadIdx.x & 63;
    const int wave = (int)uniform(threadIdx.x >> 6);  // wave-uniform: row bookkeeping stays scalar
    typename K::tables tab(lds, lane);
    GhK gk = gh_constants(lane);

    if (KIND == kGcm && blockIdx.x == 0 && threadIdx.x == 0)
        counters[0] = 0;  // reject count for this launch (read by the zero-fill)

    // The T-tables, and a single message's key tables and counter block, are
    // staged here: the chain of scalar loads behind the counter block runs
    // while the tables are on their way.
    uint64_t cur_slot = 0;
    uint32_t cur_msg = 0xffffffffu;
    uint32_t turn = 0;  // items done: its low bit picks the buffer of tile values, the wave that sums rotates
    Counters<K::siv> cs = {};
    {
        const CONST_AS MsgDesc *dp = (const CONST_AS MsgDesc *)__builtin_amdgcn_kernarg_segment_ptr();  // `single`
        StageTables<WAVES * 64> st;
        StageKeys<WAVES * 64> sk;
        if (K::aes)
            st.load(te0g);
        if (!BATCH)
            touch_lines(dp);
        if (K::gh && !BATCH) {
            cur_slot = dp->slot;
            sk.load(cur_slot);
        }
        tab.pin();  // worked out while the tables are on their way
        gk.pin();
        if (K::aes && !BATCH)
            cs.load(dp);
        if (K::aes)
            st.store(lds_v, tab);
        if (K::gh && !BATCH)
            sk.store(lds_v);
        if (!BATCH) {
            lds_barrier();
            if (K::aes)
                cs.derive(tab);
        }
    }
    for (uint32_t it = blockIdx.x; it < n_items; it += gridDim.x) {
        const CONST_AS MsgDesc *dp = (const CONST_AS MsgDesc *)__builtin_amdgcn_kernarg_segment_ptr();  // `single`
        const CONST_AS MsgDesc *next = dp;
        uint32_t first, msg = 0;
        if (BATCH) {
            const WorkItem w = load_const<WorkItem>(items + it);
            const uint32_t nit = it + gridDim.x;
            next = cptr<MsgDesc>(descs + (nit < n_items ? cptr<WorkItem>(items + nit)->msg : w.msg));
            dp = cptr<MsgDesc>(descs + w.msg);
            touch_lines(dp);
            first = w.first_tile;
            msg = w.msg;
        } else {
            asm volatile("" : "+s"(dp));  // fields are read where they are used, not before the first item
            first = (uint32_t)dp->tile_lo + it * WAVES;
        }
        // log2G and flags, one scalar load
        const uint32_t gf = K::gh ? *(const CONST_AS uint32_t *)&dp->log2G : 0u;
        const uint32_t log2G = gf & 0xffffu, G = 1u << log2G, merge = (gf >> 17) & 1u;
        const bool finish = (gf >> 16) & 1u;
        static_assert(kFinish == 1 && kMerge == 2, "bits of flags");
        const uint64_t run = dp->n_tiles - merge;
        int64_t t = (int64_t)first + wave - (int64_t)((0u - (uint32_t)run) & (G - 1u));
        const bool head = t == 0;
        u32x4 p = {0, 0, 0, 0};
        const bool mine = t >= 0 && t < (int64_t)dp->tile_hi - (int64_t)merge;
        t += merge;
        const bool fresh = BATCH ? msg != cur_msg : turn == 0;
        uint64_t next_slot = 0;
        uint32_t ahead = 0;
        if (BATCH && fresh) {
            // a new message: its key's GHASH tables (unless staged already) and
            // its round-2 words
            const uint64_t slot = dp->slot;
            const bool stage = K::gh && slot != cur_slot;
            StageKeys<WAVES * 64> sk;
            if (stage)
                sk.load(slot);
            next_slot = next->slot;
            cs.load(dp);
            lds_barrier();  // the last item's reads, and the T-tables before the first
            if (stage) {
                sk.store(lds_v);
                cur_slot = slot;
            }
            cs.derive(tab);
            cur_msg = msg;
        }
        if (fresh) {
            if (K::aes && threadIdx.x < 256)
                lds_v[K::round2 / 16 + threadIdx.x] = cs.c.low_words(threadIdx.x, tab);
            if (K::aes && wave == 4) {  // lane w for wave w
                const int64_t tw = t - wave + (lane & 15);
                const uint32_t h = cs.first_row(dp, tw, tw == (int64_t)merge);
                const u32x4 hw = cs.c.high_words_lds(h, cptr<uint32_t>(reinterpret_cast<const void *>(dp->slot)), tab);
                if (lane < 16)
                    lds_v[K::firsts / 16 + 2 * lane] = hw, lds_v[K::firsts / 16 + 2 * lane + 1].x = h;
            }
            lds_barrier();
            if (K::aes) {
                const u32x4 *f = lds_v + K::firsts / 16 + 2 * wave;
                cs.cur = u32x4{uniform(f->x), uniform(f->y), uniform(f->z), uniform(f->w)};
                cs.hc = uniform(f[1].x);
            }
        }
        if (BATCH && K::gh && fresh && next_slot != cur_slot && threadIdx.x < 640) {
            // the next item's tables into this XCD's L2, a word of each 128-byte
            // line: 1024 messages, median 16 KiB, a key each, 93.9 -> 90.4 us
            const uint32_t q = threadIdx.x;
            ahead = *gptr<const uint32_t>(next_slot + (q < 512 ? kSlotTab8Off + 128 * q : kSlotLaneWinOff + 128 * (q - 512)));
        }
        const uint64_t nparts = (run + G - 1) >> log2G;
        u32x4 *ekg = partials + (K::gh ? dp->tile_base + nparts : 0);
        if (mine) {
            const uint32_t nr = K::aes ? dp->nr : 14;
            if (nr == 10)
                p = wave_tile<10, KIND>(dp, (uint64_t)t, head, cs, lds, tab, gk, te, ekg);
            else if (nr == 12 && !K::siv)
                p = wave_tile<12, KIND>(dp, (uint64_t)t, head, cs, lds, tab, gk, te, ekg);
            else
                p = wave_tile<14, KIND>(dp, (uint64_t)t, head, cs, lds, tab, gk, te, ekg);
        }
        if (BATCH)
            asm volatile("" ::"v"(ahead));
        const uint32_t my_turn = turn++;
        if (!K::gh)
            continue;
        const u32x4 *ekw = lds_v + K::sums / 16 + 32;
        if (log2G == 0) {
            if (mine && lane == 0)
                partials[dp->tile_base + (uint64_t)t] = p;
            continue;
        }
        const uint32_t after = G - 1u - ((uint32_t)wave & (G - 1u));  // tiles of the group after this one
        if (mine && after)
            p = gf_mul_wave(p, group_lift(dp->slot, dp->log2B, after));
        u32x4 *sums = lds_v + K::sums / 16 + 16 * (my_turn & 1u);
        if (lane == 0)
            sums[wave] = p;
        if (finish && dp->op == 1)
            __builtin_amdgcn_s_waitcnt(0);  // this wave's output is out before a rejected one is cleared
        lds_barrier();
        const uint32_t part = ((uint32_t)wave + WAVES - my_turn % WAVES) % WAVES;
        if (part < kParts<WAVES>)
            sum_group<WAVES>(dp, sums, ekw, G, log2G, finish, true, first, kParts<WAVES> > 1 ? part : 0, nparts, partials);
    }
}

// ---------------------------------------------------------------- one row per wave
//
// Messages whose tiles are single rows (up to 4 MiB: every row of the message
// has a wave of its own).  What counts is the length of the chain from the
// launch to the tag, and a good part of that is fetching instructions that run
// once: a launch starts with a cold instruction cache, and the unrolled rounds
// of the tile kernel took 3 us for one row where the same row takes 1 us in a
// loop.  So the rounds and the fix-up are loops here, the round count is a
// variable, and no counter mode caching is done (the chain of scalar loads
// behind it took longer than the 27 lookups it saves).  The payload, the
// T-tables and the fix-up windows are all requested before anything is waited
// for.  No wave has a Horner step to do, so the 64 KiB GHASH table is not staged.
// E_K(J0) is worked out by the lane of the length block, which has no keystream
// block of its own and is always the last lane of the last row.
//
// The fix-up takes windows of H^(32 - n), n = lane & 31 (8 KiB), which includes
// GHASH's last factor H: the lower half-wave's sum has 32 more places to go,
// which its product with the group lift takes along.
//   [0, 64 KiB) T-tables, 16 copies; [64 KiB, 72 KiB) windows, entry (v, n) at
//   byte 16 * (32 v + n); then the row values and E_K(J0)
// 1 MiB, AES-128, one-shot: 39.3 us with the tile kernel (10.8 us) and a tree
// over 1027 partials (11.8 us), 29.0 us with this one (9.4 us, half of it the
// staging) and the verdict (2.4 us).
// A batch of small messages goes the same way, an item of WAVES rows after
// another, so that a message costs 8 KiB of windows and not 80 KiB of tables; two
// workgroups of eight waves share a compute unit and hide each other's waits
// (72.3 KiB of LDS each; the launch bound asks for no more registers than that).
// A wave issues some 990 vector instructions for an item, with a row or without,
// which keep the vector units busy 69% of the time, the LDS 30%; the rest is the
// start of an item.  1024 messages with a median of 4 KiB and 2 KiB of AAD, 12022
// rows: 79 us by tiles, 39 us.
constexpr uint32_t kRowWin = 0x10000u, kRowSums = 0x12000u;

template <int WAVES, bool BATCH, int KIND>
__global__ __launch_bounds__(WAVES * 64, BATCH ? WAVES / 2 : 1) void k_gcm_rows(MsgDesc single, const MsgDesc *__restrict__ descs,
                                                         const WorkItem *__restrict__ items, uint32_t n_items,
                                                         const uint32_t *__restrict__ te0g,
                                                         u32x4 *__restrict__ partials, uint32_t *counters)
{
    constexpr bool SIV = Kind<KIND>::siv, AES = Kind<KIND>::aes;
    constexpr int NT = WAVES * 64, kWinPer = (512 + NT - 1) / NT;
    __shared__ u32x4 lds_v[kRowSums / 16 + 17];
    uint8_t *lds = reinterpret_cast<uint8_t *>(lds_v);
    u32x4 *ekw = lds_v + kRowSums / 16 + 16;
    StageTables<NT> st;
    if (AES)
        st.load(te0g);
    if (AES && BATCH)
        st.store(lds_v, Tables<true, 0>(lds, threadIdx.x & 63));
    if (KIND == kGcm && blockIdx.x == 0 && threadIdx.x == 0)
        counters[0] = 0;  // reject count for this launch

    for (uint32_t it = blockIdx.x, turn = 0; it < n_items; it += gridDim.x, ++turn) {
        uint32_t tid = threadIdx.x;
        if (BATCH)  // what depends on the lane alone is worked out again for each item rather than held in registers
            asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const int wave = (int)uniform(tid >> 6);
        const Tables<true, 0> tab(lds, lane);
        const CONST_AS MsgDesc *dp = (const CONST_AS MsgDesc *)__builtin_amdgcn_kernarg_segment_ptr();  // `single`
        uint32_t first = it * WAVES;
        if (BATCH) {
            const WorkItem w = load_const<WorkItem>(items + it);
            dp = cptr<MsgDesc>(descs + w.msg);
            first = w.first_tile;
        }
        touch_lines(dp);
        const uint64_t slot = dp->slot, T = dp->n_tiles;
        u32x4 win[kWinPer];
        {
            const GLOBAL_AS u32x4 *src = gptr<const u32x4>(slot + kSlotLaneWinOff);
#pragma unroll
            for (int r = 0; r < kWinPer; ++r) {
                const uint32_t q = tid + (uint32_t)(r * NT);
                win[r] = q >= 32 && q < 512 ? src[64 * (q >> 5) + 31 + (q & 31)] : u32x4{0, 0, 0, 0};
            }
        }
        const uint32_t gf = *(const CONST_AS uint32_t *)&dp->log2G;
        const uint32_t log2G = gf & 0xffffu, G = 1u << log2G;
        const bool finish = (gf >> 16) & 1u;
        const int64_t t = (int64_t)first + wave - (int64_t)((0u - (uint32_t)T) & (G - 1u));
        const bool mine = t >= 0 && t < (int64_t)T;

        // this lane's block of the sequence and its bytes
        const int64_t na = (int64_t)dp->na, ndat = (int64_t)dp->n;
        const int64_t v0 = 64 * t - (int64_t)dp->z, v = v0 + lane;
        const bool data = mine && v >= na && v < na + ndat;
        const uint64_t j = (uint64_t)(v - na);
        u32x4 x = {0, 0, 0, 0};
        if (mine && v == na + ndat) {
            const uint64_t abits = dp->aad_len * 8, cbits = dp->len * 8;
            x = SIV ? u32x4{(uint32_t)abits, (uint32_t)(abits >> 32), (uint32_t)cbits, (uint32_t)(cbits >> 32)}
                    : u32x4{bswap32((uint32_t)(abits >> 32)), bswap32((uint32_t)abits), bswap32((uint32_t)(cbits >> 32)),
                            bswap32((uint32_t)cbits)};
        } else if (mine && v >= 0 && v < na + ndat) {  // data or AAD
            x = load_block_partial(data ? gptr<const uint8_t>(dp->in) : gptr<const uint8_t>(dp->aad),
                                   data ? j : (uint64_t)v, data ? dp->len : dp->aad_len);
        }

        // the lifts of this row's value, and of its lower half (32 places more)
        const uint32_t after = G - 1u - ((uint32_t)wave & (G - 1u));
        u32x4 lift = {0x80u, 0, 0, 0};
        if (after)
            lift = group_lift(slot, 6, after);
        const CONST_AS uint32_t *l32 = cptr<uint32_t>(reinterpret_cast<const void *>(slot + kSlotTab8Off)) + 4 * after;
        const u32x4 lift32 = {l32[0], l32[1], l32[2], l32[3]};

        // the counter block, whitened; the counter dword is the lane's
        const CONST_AS uint32_t *rk = cptr<uint32_t>(reinterpret_cast<const void *>(slot));
        const uint32_t nr = dp->nr;
        uint32_t w0 = dp->iv[0], w1 = dp->iv[1], w2 = dp->iv[2], cj0 = 1u;
        const uint64_t jaddr = dp->j0;
        if (SIV || jaddr) {
            const CONST_AS uint32_t *jw = cptr<uint32_t>(reinterpret_cast<const void *>(jaddr));
            w0 = jw[SIV ? 1 : 0], w1 = jw[SIV ? 2 : 1], w2 = jw[SIV ? 3 : 2];
            cj0 = SIV ? jw[0] : bswap32(jw[3]);
        }
        const uint32_t c1 = SIV ? cj0 : cj0 + 1u;
        if (AES) {  // the round keys' four lines at once, not one after another in the rounds
            const uint32_t l0 = rk[0], l1 = rk[16], l2 = rk[32], l3 = rk[48];
            asm volatile("" ::"s"(l0), "s"(l1), "s"(l2), "s"(l3));
        }
        // some lane needs a keystream block; the length block's needs E_K(J0)
        const bool ekl = KIND == kGcm && mine && v == na + ndat;
        const bool hot = AES && mine && ((v0 + 64 > na && v0 < na + ndat) || (KIND == kGcm && t + 1 == (int64_t)T));

        if (AES && !BATCH)
            st.store(lds_v, tab);
#pragma unroll
        for (int r = 0; r < kWinPer; ++r) {
            const uint32_t q = tid + (uint32_t)(r * NT);
            if (512 % NT == 0 || q < 512)
                lds_v[kRowWin / 16 + q] = win[r];
        }
        lds_barrier();

        if (hot) {
            const uint32_t ctr = ekl ? cj0 : (uint32_t)(v0 - na) + c1 + (uint32_t)lane;
            uint32_t s0 = (SIV ? ctr : w0) ^ rk[0], s1 = (SIV ? w0 : w1) ^ rk[1], s2 = (SIV ? w1 : w2) ^ rk[2];
            uint32_t s3 = (SIV ? w2 : bswap32(ctr)) ^ rk[3];
            s0 = tab.rot(s0), s1 = tab.rot(s1), s2 = tab.rot(s2), s3 = tab.rot(s3);
            const CONST_AS uint32_t *k = rk + 4;
            uint32_t k0 = k[0], k1 = k[1], k2 = k[2], k3 = k[3];
            uint32_t a[4][4];
#pragma unroll 1
            for (uint32_t r = 1;; ++r) {
                ISSUE0(a, s0);
                ISSUE1(a, s1);
                ISSUE2(a, s2);
                ISSUE3(a, s3);
                if (r == nr)
                    break;
                k += 4;  // the next round's key (the one after the last round key is never used)
                const uint32_t n0 = k[0], n1 = k[1], n2 = k[2], n3 = k[3];
                s0 = xor3(xor3(a[0][0], a[0][1], a[0][2]), a[0][3], tab.rot(k0));
                s1 = xor3(xor3(a[1][0], a[1][1], a[1][2]), a[1][3], tab.rot(k1));
                s2 = xor3(xor3(a[2][0], a[2][1], a[2][2]), a[2][3], tab.rot(k2));
                s3 = xor3(xor3(a[3][0], a[3][1], a[3][2]), a[3][3], tab.rot(k3));
                k0 = n0, k1 = n1, k2 = n2, k3 = n3;
            }
#define LAST(q, key)                                                                                                   \
        (uint32_t)__builtin_amdgcn_bitop3_b32(tab.last01(a[q][q], a[q][((q) + 1) & 3]), tab.last23(a[q][((q) + 2) & 3], a[q][((q) + 3) & 3]), key, 0x56)
            const u32x4 ks = {LAST(0, k0), LAST(1, k1), LAST(2, k2), LAST(3, k3)};
#undef LAST
            if (ekl) {
                *ekw = ks;
                partials[dp->tile_base + ((T + G - 1) >> log2G)] = ks;
            }
            if (data) {
                const u32x4 o = x ^ ks;
                store_block_partial(gptr<uint8_t>(dp->out), j, dp->len, o);
                x = (SIV || dp->op == 0) ? mask_block(o, j, dp->len) : x;
            }
        }
        if (SIV)
            x = rev_block(x);

        // x * H^(32 - n): the comb of gf_mul_lanewin in a loop, entries one step ahead
        u32x4 y;
        {
            const uint32_t xm[4] = {x.x, x.y, x.z, x.w};
            const P128 px = mem_to_poly(xm);
            uint32_t aw[4] = {(uint32_t)px.lo, (uint32_t)(px.lo >> 32), (uint32_t)px.hi, (uint32_t)(px.hi >> 32)};
            const uint8_t *base = lds + kRowWin + 16u * ((uint32_t)lane & 31u);
            uint32_t acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            u32x4 e[4];
#pragma unroll
            for (int w = 0; w < 4; ++w)
                e[w] = *reinterpret_cast<const u32x4 *>(base + 512u * (aw[w] >> 28));
#pragma unroll 1
            for (int q = 0; q < 8; ++q) {
                u32x4 f[4];
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    f[w] = e[w];
                    aw[w] <<= 4;
                    e[w] = *reinterpret_cast<const u32x4 *>(base + 512u * (aw[w] >> 28));
                }
#pragma unroll
                for (int i = 7; i > 0; --i)
                    acc[i] = __builtin_amdgcn_alignbit(acc[i], acc[i - 1], 28);  // acc <<= 4
                acc[0] <<= 4;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    acc[w] ^= f[w].x;
                    acc[w + 1] ^= f[w].y;
                    acc[w + 2] ^= f[w].z;
                    acc[w + 3] ^= f[w].w;
                }
            }
            y = poly_to_mem(poly_reduce((uint64_t)acc[0] | ((uint64_t)acc[1] << 32), (uint64_t)acc[2] | ((uint64_t)acc[3] << 32),
                                        (uint64_t)acc[4] | ((uint64_t)acc[5] << 32), (uint64_t)acc[6] | ((uint64_t)acc[7] << 32)));
        }
        u32x4 lo, hi;  // sums of the lower and the upper half-wave
        {
            const uint32_t w[4] = {half_wave_xor_u32(y.x), half_wave_xor_u32(y.y), half_wave_xor_u32(y.z),
                                   half_wave_xor_u32(y.w)};
            const auto q0 = __builtin_amdgcn_permlane32_swap(w[0], w[0], false, false);
            const auto q1 = __builtin_amdgcn_permlane32_swap(w[1], w[1], false, false);
            const auto q2 = __builtin_amdgcn_permlane32_swap(w[2], w[2], false, false);
            const auto q3 = __builtin_amdgcn_permlane32_swap(w[3], w[3], false, false);
            lo = u32x4{q0[0], q1[0], q2[0], q3[0]};
            hi = u32x4{q0[1], q1[1], q2[1], q3[1]};
        }
        const u32x4 p = gf_mul2_wave(lo, lift32, hi, lift);
        u32x4 *sums = lds_v + kRowSums / 16;
        if (lane == 0)
            sums[wave] = p;
        if (finish && dp->op == 1)
            __builtin_amdgcn_s_waitcnt(0);  // this wave's output is out before a rejected one is cleared
        lds_barrier();
        const uint32_t part = ((uint32_t)wave + WAVES - turn % WAVES) % WAVES;
        if (part < kParts<WAVES>)
            sum_group<WAVES>(dp, sums, ekw, G, log2G, finish, false, first, kParts<WAVES> > 1 ? part : 0,
                             (T + G - 1) >> log2G, partials);
        if (!BATCH)
            break;  // every workgroup has one item
    }
}

// ---------------------------------------------------------------- verdict

// clears a rejected message's output, a share in each workgroup of 256
template <typename D>
__device__ __forceinline__ void clear_output(const D *d)
{
    GLOBAL_AS uint8_t *out = gptr<uint8_t>(d->out);
    const uint64_t len = d->len, nfull = len >> 4, stride = (uint64_t)gridDim.x * 256;
    for (uint64_t q = (uint64_t)blockIdx.x * 256 + threadIdx.x; q < nfull; q += stride)
        __builtin_nontemporal_store(u32x4{0, 0, 0, 0}, reinterpret_cast<GLOBAL_AS u32x4 *>(out) + q);
    if (blockIdx.x == 0 && threadIdx.x < (len & 15))
        out[nfull * 16 + threadIdx.x] = 0;
}

// A grouped message's tag: the XOR of its partials (already lifted), times H
// where they do not hold that factor, XOR E_K(J0).  Encrypt writes the tag;
// decrypt compares it without early exit and writes the accept flag.  A batch
// has one workgroup per message and leaves rejected messages in the list that
// k_gcm_zerofill reads; a single message has as many workgroups as clearing
// its output takes, each of which forms the verdict by itself.
template <bool BATCH>
__global__ __launch_bounds__(256) void k_gcm_verdict(MsgDesc single, const MsgDesc *__restrict__ descs,
                                                     const u32x4 *__restrict__ partials, uint32_t *counters)
{
    __shared__ u32x4 sh[4];
    const CONST_AS MsgDesc *dp = BATCH ? cptr<MsgDesc>(descs + blockIdx.x)
                                       : (const CONST_AS MsgDesc *)__builtin_amdgcn_kernarg_segment_ptr();
    const uint32_t gf = *(const CONST_AS uint32_t *)&dp->log2G, log2G = gf & 0xffffu, flags = gf >> 16;
    if (flags & kFinish)
        return;  // the tile kernel has
    const int lane = threadIdx.x & 63, wave = (int)uniform(threadIdx.x >> 6);
    const uint64_t run = dp->n_tiles - ((flags & kMerge) ? 1 : 0), P = (run + (1ull << log2G) - 1) >> log2G;
    const u32x4 *part = partials + dp->tile_base;
    const u32x4 ek = part[P];
    const int tl = (int)dp->tag_len;  // T = MSB_t of the full tag
    GLOBAL_AS uint8_t *dst = gptr<uint8_t>(dp->tag);
    const uint32_t want = dp->op == 1 && lane < tl ? dst[lane] : 0u;  // asked for with the partials
    u32x4 s = {0, 0, 0, 0};
    for (uint64_t i = threadIdx.x; i < P; i += 256)
        s ^= part[i];
    s = wave_xor_reduce(s);
    if (lane == 0)
        sh[wave] = s;
    asm volatile("" ::"v"(want));  // every wave has the expected tag before the flag, which may lie in it, is written
    lds_barrier();
    s = sh[0] ^ sh[1] ^ sh[2] ^ sh[3];
    if (!(flags & kRows)) {
        const CONST_AS KeySlotHdr *hd = cptr<KeySlotHdr>(reinterpret_cast<const void *>(dp->slot));
        s = gf_mul_wave(s, u32x4{hd->hpow[0][0], hd->hpow[0][1], hd->hpow[0][2], hd->hpow[0][3]});
    }
    const bool lead = (BATCH || blockIdx.x == 0) && threadIdx.x == 0;
    const u32x4 tag = s ^ ek;
    const uint32_t mine = byte_of(tag, lane & 15);
    if (dp->op == 0) {
        if (wave == 0 && lane < tl)
            dst[lane] = (uint8_t)mine;
        return;
    }
    const uint32_t diff = lane < tl ? mine ^ want : 0u;
    const bool ok = __builtin_amdgcn_ballot_w64(diff != 0) == 0;
    if (lead)
        *gptr<int32_t>(dp->ok) = ok ? 1 : 0;
    if (ok)
        return;
    if (BATCH) {
        if (lead) {
            const uint32_t pos = atomicAdd(&counters[0], 1u);
            counters[1 + pos] = blockIdx.x;
        }
        return;
    }
    clear_output(dp);
}

// ---------------------------------------------------------------- combine + tag

constexpr int kCombineThreads = 1024;
constexpr int kCombineLog2 = 10;

// S = sum_t p_t * H^((T-1-t)*B + 1); tag = S xor E_K(J0).  Thread i runs a
// Horner over partials i, i+1024, ... with the fixed multiplier H^(1024*B);
// its value then needs the weight H^((T-1-t_last)*B), and with N = 2^k >=
// min(T, 1024) leaves and r = T mod N that weight is H^((N-1-j)*B) for leaf
// j = (i - r) mod N.  A tree of fan-in F = 2^LOGF over the leaves closes the
// sum: a node whose F children each span w leaves is the Horner
// (((c_0*H^(B*w) ^ c_1)*H^(B*w) ^ c_2) ...) ^ c_(F-1), so the levels use the
// tables of H^(B*2^(LOGF*lev)) and the tree has ceil(k / LOGF) levels and
// N - 1 products in all (F = 2 is the binary tree L*H^(B*2^lev) ^ R); one
// more *H accounts for GHASH's final multiplication.  The nibble tables this needs
// (at most 12 of 8 KiB) are staged in LDS first, so every multiply is 32 LDS
// reads.  E_K(J0) was left by the tile kernel right after the message's T
// partials.
template <bool BATCH, int LOGF>
__global__ __launch_bounds__(kCombineThreads) void k_gcm_combine(const MsgDesc *__restrict__ descs, MsgDesc single,
                                                                 const u32x4 *__restrict__ partials)
{
    __shared__ u32x4 tabs[kCombineLog2 + 2][512];  // [0]: H; [1+k]: H^(B*2^k), k = 0..10
    __shared__ u32x4 leaf[kCombineThreads];
    const MsgDesc d = BATCH ? load_const<MsgDesc>(descs + blockIdx.x) : single;
    const uint32_t i = threadIdx.x;
    const uint64_t T = d.n_tiles;

    // the first eight partials of this thread, loaded ahead of the table staging
    u32x4 pv[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint64_t t = (uint64_t)i + (uint64_t)q * kCombineThreads;
        pv[q] = t < T ? partials[d.tile_base + t] : u32x4{0, 0, 0, 0};
    }

    // exponent bits needed for T-1-t_last < min(T, 1024), and whether any
    // thread owns more than one partial
    const uint64_t span = T < (uint64_t)kCombineThreads ? T : (uint64_t)kCombineThreads;
    int nbits = 0;
    while (nbits < kCombineLog2 && (1ull << nbits) < span)
        ++nbits;
    const bool horner = T > (uint64_t)kCombineThreads;
    {
        // all of a thread's table loads are issued before any is stored
        const GLOBAL_AS u32x4 *g = gptr<const u32x4>(d.slot + kSlotTab4Off);
        const int ntab = 1 + (horner ? kCombineLog2 + 1 : nbits);
        constexpr int kPer = ((kCombineLog2 + 2) * 512 + kCombineThreads - 1) / kCombineThreads;
        u32x4 st[kPer];
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int e = (int)i + r * kCombineThreads;
            const int tix = e >> 9;
            const int lvl = tix == 0 ? 0 : (int)d.log2B + tix - 1;
            if (e < ntab * 512)
                st[r] = g[(uint64_t)lvl * 512 + (e & 511)];
        }
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int e = (int)i + r * kCombineThreads;
            if (e < ntab * 512)
                tabs[e >> 9][e & 511] = st[r];
        }
    }
    lds_barrier();

    u32x4 acc = {0, 0, 0, 0};
    if (i < T) {
        for (uint64_t t0 = i; t0 < T; t0 += 8 * (uint64_t)kCombineThreads) {
            if (t0 != i) {
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const uint64_t t = t0 + (uint64_t)q * kCombineThreads;
                    pv[q] = t < T ? partials[d.tile_base + t] : u32x4{0, 0, 0, 0};
                }
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint64_t t = t0 + (uint64_t)q * kCombineThreads;
                if (t < T)
                    acc = (horner ? mul_tab4(acc, tabs[1 + kCombineLog2]) : acc) ^ pv[q];
            }
        }
    }
    // leaves: thread i (< N) at (i - r) mod N; threads without partials hold 0
    const uint32_t N = 1u << nbits;
    const uint32_t r = (uint32_t)(T & (uint64_t)(N - 1));
    if (i < N)
        leaf[(i - r) & (N - 1)] = acc;
    lds_barrier();
    for (int lev = 0; lev < nbits; lev += LOGF) {
        const int span = nbits - lev < LOGF ? nbits - lev : LOGF;  // log2 of this level's children per node
        const uint32_t kids = 1u << span, w = 1u << lev;           // children, leaves per child
        const uint32_t nodes = N >> (lev + span);
        const u32x4 *tab = tabs[1 + lev];                            // H^(B*w)
        if (nodes > kCombineThreads / 32) {
            // wide levels: one thread per node (bound by LDS bandwidth)
            if (i < nodes) {
                const uint32_t a = i << (lev + span);
                u32x4 v = leaf[a];
                for (uint32_t c = 1; c < kids; ++c)
                    v = mul_tab4(v, tab) ^ leaf[a + c * w];
                leaf[a] = v;
            }
        } else {
            // narrow levels (bound by latency): 32 lanes per node, one lookup
            // each per product; node i / 32 is uniform across each half-wave,
            // whose reads of its leaves precede its write, and other nodes
            // touch other leaves
            const uint32_t pp = i >> 5;
            const bool act = pp < nodes;
            const uint32_t a = act ? pp << (lev + span) : 0u;
            u32x4 v = act ? leaf[a] : u32x4{0, 0, 0, 0};
            for (uint32_t c = 1; c < kids; ++c) {
                v = mul_tab4_half(v, tab, i & 31u, act);
                if (act)
                    v ^= leaf[a + c * w];
            }
            if (act && (i & 31u) == 0)
                leaf[a] = v;
        }
        lds_barrier();
    }
    // * H, by the first half-wave
    const u32x4 s = mul_tab4_half(i < 32 ? leaf[0] : u32x4{0, 0, 0, 0}, tabs[0], i & 31u, i < 32);
    if (BATCH) {
        // streamed segments: hand on each one's GHASH value, first multiplied by
        // H^lift (the blocks of the message that follow the segment) with the key
        // slot's nibble tables of H^(2^k), one half-wave product per set bit
        if (i >= 64)
            return;
        u32x4 y = s;
        const u32x4 *g4 = reinterpret_cast<const u32x4 *>(d.slot + kSlotTab4Off);
        for (uint64_t e = d.lift, k = 0; e && k < (uint64_t)kTab4Levels; e >>= 1, ++k)
            if (e & 1u)
                y = mul_tab4_half(y, g4 + k * 512, i & 31u, i < 32);
        if (i == 0)
            *reinterpret_cast<u32x4 *>(d.yout) = y;
        return;
    }
    if (i == 0) {
        const u32x4 tag = s ^ partials[d.tile_base + T];
        const uint32_t tw[4] = {tag.x, tag.y, tag.z, tag.w};
        const int tl = (int)d.tag_len;  // T = MSB_t of the full tag
        if (d.op == 0) {
            uint8_t *dst = reinterpret_cast<uint8_t *>(d.tag);
            for (int k = 0; k < tl; ++k)
                dst[k] = (uint8_t)(tw[k >> 2] >> (8 * (k & 3)));
        } else {
            const uint8_t *exp = reinterpret_cast<const uint8_t *>(d.tag);
            uint32_t diff = 0;
            for (int k = 0; k < tl; ++k)
                diff |= ((tw[k >> 2] >> (8 * (k & 3))) & 0xffu) ^ exp[k];
            *reinterpret_cast<int32_t *>(d.ok) = diff == 0 ? 1 : 0;
        }
    }
}

// ---------------------------------------------------------------- streamed message tag

// GHASH of a message fed in segments is the XOR of the segments' own GHASH
// values, each multiplied by H^(blocks after it) (the combine's lift); the
// tag adds E_K(J0).  One wave: lane l XORs values l, l + 64, ..., then an
// XOR across the wave.  Encrypt writes tag_len bytes of the tag; decrypt
// compares them without early exit and writes the accept flag.
__global__ __launch_bounds__(64) void k_gcm_fold(const u32x4 *__restrict__ vals, uint32_t k,
                                                 const u32x4 *__restrict__ ekj0, uint8_t *tag, int32_t *ok,
                                                 uint32_t op, uint32_t tag_len, uint64_t slot, u32x4 lenblk)
{
    const uint32_t lane = threadIdx.x;
    u32x4 acc = {0, 0, 0, 0};
    for (uint32_t j = lane; j < k; j += 64)
        acc ^= vals[j];
    acc = wave_xor_reduce(acc);
    if (slot) {
        // GHASH's last block, the length block L, enters as L * H (the
        // slot's nibble table of H^(2^0)); the values above were lifted past it
        const u32x4 *g4 = reinterpret_cast<const u32x4 *>(slot + kSlotTab4Off);
        acc ^= mul_tab4_half(lenblk, g4, lane & 31u, lane < 32);
    }
    if (lane != 0)
        return;
    const u32x4 t = acc ^ *ekj0;
    const uint32_t tw[4] = {t.x, t.y, t.z, t.w};
    if (op == 0) {
        for (uint32_t b = 0; b < tag_len; ++b)
            tag[b] = (uint8_t)(tw[b >> 2] >> (8 * (b & 3)));
    } else {
        uint32_t diff = 0;
        for (uint32_t b = 0; b < tag_len; ++b)
            diff |= ((tw[b >> 2] >> (8 * (b & 3))) & 0xffu) ^ tag[b];
        *ok = diff == 0 ? 1 : 0;
    }
}

// ---------------------------------------------------------------- J0 for other IV lengths

// J0 = GHASH_H(IV || 0^s || 0^64 || [8*len(IV)]_64) (SP 800-38D sec. 7.1,
// step 2), by Horner over the IV blocks with the nibble table of H staged in
// LDS; one workgroup, written to j0_out (16 bytes).
__global__ __launch_bounds__(64) void k_gcm_j0(IvArg iv, uint64_t slot, u32x4 *j0_out, u32x4 *y_zero)
{
    if (y_zero && threadIdx.x == 0)
        *y_zero = u32x4{0, 0, 0, 0};  // a new stream's GHASH value
    if (iv.len == 12) {  // J0 = IV || 0^31 || 1
        if (threadIdx.x == 0) {
            uint32_t w[3] = {0, 0, 0};
            for (int k = 0; k < 12; ++k)
                w[k >> 2] |= (uint32_t)iv.b[k] << (8 * (k & 3));
            *j0_out = u32x4{w[0], w[1], w[2], 0x01000000u};
        }
        return;
    }
    __shared__ u32x4 tab[512];
    const GLOBAL_AS u32x4 *src = gptr<const u32x4>(slot + kSlotTab4Off);  // level 0: H
    u32x4 st[8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
        st[r] = src[threadIdx.x + 64 * r];
#pragma unroll
    for (int r = 0; r < 8; ++r)
        tab[threadIdx.x + 64 * r] = st[r];
    lds_barrier();
    if (threadIdx.x != 0)
        return;
    u32x4 y = {0, 0, 0, 0};
    const uint32_t n = iv.len;
    for (uint32_t off = 0; off < n; off += 16) {
        uint32_t w[4] = {0, 0, 0, 0};
        for (uint32_t k = 0; k < 16 && off + k < n; ++k)
            w[k >> 2] |= (uint32_t)iv.b[off + k] << (8 * (k & 3));
        y = mul_tab4(y ^ u32x4{w[0], w[1], w[2], w[3]}, tab);
    }
    const uint64_t bits = (uint64_t)n * 8;
    y = mul_tab4(y ^ u32x4{0u, 0u, bswap32((uint32_t)(bits >> 32)), bswap32((uint32_t)bits)}, tab);
    *j0_out = y;
}

// ---------------------------------------------------------------- zero-fill on reject

// The rejected messages of a batch share the grid.  Short ones (`longest`: the
// batch's longest that may come here) take as many workgroups each: workgroup b
// clears a part of message b mod n_rej, so that their descriptors are read side
// by side (51 messages of 34 KiB on average: 4.1 us; 12.6 when the whole grid
// cleared one after another).  Where such a share may be more than 256 KiB, some
// 2 us of one workgroup, the messages are taken 256 at a time, their lengths
// summed in chunks of 8 KiB, and a workgroup clears its share of the chunks
// whatever messages those are in: about 1 us more, but 512 rejected messages of
// up to 27 MiB, 1.2 GiB in all, 1485 -> 1401 us.
constexpr uint32_t kZeroChunk = 8192;  // 256 messages have fewer than 2^32 chunks
constexpr uint64_t kZeroShare = 256ull << 10;

// blocks [from, to) of a buffer, a workgroup's every stride-th 256
__device__ __forceinline__ void zero_blocks(uint64_t out, uint64_t from, uint64_t to, uint64_t stride)
{
    GLOBAL_AS u32x4 *dst = gptr<u32x4>(out);
    for (uint64_t j = from + threadIdx.x; j < to; j += stride)
        __builtin_nontemporal_store(u32x4{0, 0, 0, 0}, dst + j);
}

__global__ __launch_bounds__(256) void k_gcm_zerofill(const MsgDesc *__restrict__ descs,
                                                      const uint32_t *__restrict__ counters, uint64_t longest)
{
    const uint32_t n_rej = *cptr<uint32_t>(counters);
    if (n_rej == 0)
        return;
    const uint32_t parts = gridDim.x > n_rej ? gridDim.x / n_rej : 1u;  // workgroups a message
    if (longest <= parts * kZeroShare) {
        for (uint32_t w = blockIdx.x; w < n_rej * parts; w += gridDim.x) {
            const uint32_t part = w / n_rej;
            const CONST_AS MsgDesc *dp = cptr<MsgDesc>(descs + cptr<uint32_t>(counters)[1 + w % n_rej]);
            const uint64_t len = dp->len;
            zero_blocks(dp->out, (uint64_t)part * 256, len >> 4, (uint64_t)parts * 256);
            if (part == 0 && threadIdx.x < (len & 15))
                gptr<uint8_t>(dp->out)[(len & ~15ull) + threadIdx.x] = 0;
        }
        return;
    }
    __shared__ uint32_t upto[256];  // chunks of this message and those before it
    __shared__ uint64_t out[256], len[256];
    __shared__ uint32_t waves[4], first;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = uniform(tid >> 6);
    for (uint32_t base = 0; base < n_rej; base += 256) {
        uint32_t mine = 0;
        if (base + tid < n_rej) {
            const GLOBAL_AS MsgDesc *d = gptr<const MsgDesc>((uint64_t)(descs + counters[1 + base + tid]));
            const uint64_t o = d->out, l = d->len;
            out[tid] = o;
            len[tid] = l;
            mine = (uint32_t)((l + kZeroChunk - 1) / kZeroChunk);
        }
        uint32_t sum = mine;
#pragma unroll
        for (uint32_t k = 1; k < 64; k <<= 1) {
            const uint32_t below = __shfl_up(sum, k);
            sum += lane >= k ? below : 0u;
        }
        if (lane == 63)
            waves[wave] = sum;
        lds_barrier();
        uint32_t total = 0;
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            const uint32_t here = waves[w];
            total += here;
            sum += w < wave ? here : 0u;
        }
        upto[tid] = sum;
        total = uniform(total);
        const uint32_t each = total / gridDim.x, rest = total % gridDim.x;
        const uint32_t lo = blockIdx.x * each + (blockIdx.x < rest ? blockIdx.x : rest);
        const uint32_t hi = lo + each + (blockIdx.x < rest ? 1u : 0u);
        if (lo < sum && lo >= sum - mine)
            first = tid;  // the message of chunk lo
        lds_barrier();
        for (uint32_t c = lo, m = uniform(first); c < hi; ++m) {
            const uint32_t start = m ? upto[m - 1] : 0u, end = upto[m] < hi ? upto[m] : hi;
            if (end <= c)
                continue;  // a message without payload
            const uint64_t L = len[m], to = (uint64_t)(end - start) * kZeroChunk;
            zero_blocks(out[m], (uint64_t)(c - start) * (kZeroChunk / 16), (to < L ? to : L) >> 4, 256);
            if (to >= L && tid < (L & 15))
                gptr<uint8_t>(out[m])[(L & ~15ull) + tid] = 0;
            c = end;
        }
        lds_barrier();  // before the next 256
    }
}

// ---------------------------------------------------------------- AES-GCM-SIV (RFC 8452)
//
// POLYVAL through GHASH: with BR the reversal of a block's 16 bytes,
// POLYVAL(H, X_1..X_s) = BR(GHASH_H'(BR(X_1), ..., BR(X_s))) where H' is
// BR(H) times x in GHASH's field (RFC 8452 appendix A).  A per-message slot
// holds the derived encryption key's round keys and H' with every GHASH table
// of an ordinary key slot, so the tiles, the lane fix-ups and the group
// lifts run unchanged on byte-reversed blocks.  The counter block is the tag
// with the top bit of byte 15 set; its bytes 0..3 (memory-order dword 0) are
// a little-endian 32-bit counter, so dword 0 is the column that varies, where
// GCM's counter varies column 3.

struct SivArg {
    uint32_t nonce[3];
    uint32_t pad;
};

// Both kernels below are a chain of a few thousand cycles, and what they add to
// it is instructions fetched once: the rounds are a loop, and a block's four
// columns take a lane each.

// One column of an AES block in each lane: lanes 4 i .. 4 i + 3 encrypt block i.
// in: the lane's column; rk: all round keys, in LDS; te0, sb: tables in LDS.
__device__ __forceinline__ uint32_t aes_columns(uint32_t in, const uint32_t *rk, uint32_t nr, const uint32_t *te0,
                                                const uint32_t *sb)
{
    const uint32_t c = threadIdx.x & 3u;
    uint32_t s = in ^ rk[c], key = rk[4 + c];
    const auto columns = [](uint32_t x, uint32_t &s1, uint32_t &s2, uint32_t &s3) {  // the next three columns
        s1 = __builtin_amdgcn_update_dpp(0u, x, 0x39, 0xF, 0xF, false);  // quad_perm [1,2,3,0]
        s2 = __builtin_amdgcn_update_dpp(0u, x, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
        s3 = __builtin_amdgcn_update_dpp(0u, x, 0x93, 0xF, 0xF, false);  // quad_perm [3,0,1,2]
    };
    uint32_t s1, s2, s3;
#pragma unroll 1
    for (uint32_t r = 1; r < nr; ++r) {
        columns(s, s1, s2, s3);
        const uint32_t next = rk[4 * (r + 1) + c];
        s = te0[B0(s)] ^ rotl32(te0[B1(s1)], 8) ^ rotl32(te0[B2(s2)], 16) ^ rotl32(te0[B3(s3)], 24) ^ key;
        key = next;
    }
    columns(s, s1, s2, s3);
    return (sb[B0(s)] | sb[B1(s1)] << 8 | sb[B2(s2)] << 16 | sb[B3(s3)] << 24) ^ key;
}

// Two waves: the message keys from the key-generating key in slot `kgk`
// (first halves of AES_KGK(LE32(i) || nonce): i = 0, 1 the authentication
// key, i = 2, 3 (and 4, 5 for a 256-bit key) the encryption key), expanded
// into slot `out` with H' and its powers H'^(2^k), which the second wave forms
// meanwhile.  With `tag_in` (decrypt) the counter block is also formed from the
// received tag at `ctr_out`.
__global__ __launch_bounds__(128) void k_siv_derive(uint64_t kgk, SivArg na, uint64_t out, const uint8_t *tag_in,
                                                    u32x4 *ctr_out, const uint32_t *te0g, const uint32_t *sbg,
                                                    const u32x4 *__restrict__ frob)
{
    __shared__ uint32_t te0[256], sb[256], rk[4 * (kMaxNr + 2)], half[12];
    const CONST_AS KeySlotHdr *kh = cptr<KeySlotHdr>(reinterpret_cast<const void *>(kgk));
    KeySlotHdr *hd = reinterpret_cast<KeySlotHdr *>(out);
    const uint32_t tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63u;
    {
        const uint32_t t0 = te0g[tid], t1 = te0g[tid + 128], b0 = sbg[tid], b1 = sbg[tid + 128];
        const uint32_t k = tid < 4 * (kMaxNr + 1) ? reinterpret_cast<const KeySlotHdr *>(kgk)->rk[tid] : 0u;
        te0[tid] = t0, te0[tid + 128] = t1, sb[tid] = b0, sb[tid + 128] = b1;
        if (tid < 4 * (kMaxNr + 2))
            rk[tid] = k;
    }
    const uint32_t nr = kh->nr;
    uint32_t tagb = 0;
    if (tag_in && wave == 1 && lane < 16)
        tagb = tag_in[lane];
    lds_barrier();
    const bool k128 = nr == 10;
    if (wave == 0) {
        // the key-generating blocks are independent: block lane / 4
        const uint32_t c = lane & 3u;
        const uint32_t o = aes_columns(c == 0 ? lane >> 2 : c == 1 ? na.nonce[0] : c == 2 ? na.nonce[1] : na.nonce[2],
                                       rk, nr, te0, sb);
        if (c < 2 && lane < (k128 ? 16u : 24u))
            half[2 * (lane >> 2) + c] = o;
    }
    lds_barrier();
    if (wave == 0) {
        // FIPS-197 key expansion in a loop, every lane alike
        const uint32_t nk = k128 ? 4u : 8u, nw = 4 * (nr + 1);
        uint32_t w0 = half[4], w1 = half[5], w2 = half[6], w3 = half[7];
        uint32_t w4 = 0, w5 = 0, w6 = 0, w7 = w3;
        rk[0] = w0, rk[1] = w1, rk[2] = w2, rk[3] = w3;
        if (!k128) {
            w4 = half[8], w5 = half[9], w6 = half[10], w7 = half[11];
            rk[4] = w4, rk[5] = w5, rk[6] = w6, rk[7] = w7;
        }
        uint32_t rcon = 1;
#pragma unroll 1
        for (uint32_t i = nk; i < nw;) {
            w0 ^= sub_word((w7 >> 8) | (w7 << 24), sb) ^ rcon;
            rcon = gf8_xtime(rcon);
            w1 ^= w0, w2 ^= w1, w3 ^= w2;
            rk[i] = w0, rk[i + 1] = w1, rk[i + 2] = w2, rk[i + 3] = w3;
            i += 4;
            w7 = k128 ? w3 : w7;
            if (!k128 && i < nw) {
                w4 ^= sub_word(w3, sb);
                w5 ^= w4, w6 ^= w5, w7 ^= w6;
                rk[i] = w4, rk[i + 1] = w5, rk[i + 2] = w6, rk[i + 3] = w7;
                i += 4;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        if (lane < 4 * (kMaxNr + 1))
            hd->rk[lane] = lane < nw ? rk[lane] : 0u;
        if (lane == 0) {
            hd->nr = nr;
            hd->key_len = 4 * nk;
        }
        return;
    }
    const uint32_t br[4] = {bswap32(half[3]), bswap32(half[2]), bswap32(half[1]), bswap32(half[0])};
    const u32x4 hp = poly_to_mem(poly_mul_xi(mem_to_poly(br), 1));
    if (lane == 0)
        hd->h[0] = hp.x, hd->h[1] = hp.y, hd->h[2] = hp.z, hd->h[3] = hp.w;
    if (tag_in && lane < 16)
        reinterpret_cast<uint8_t *>(ctr_out)[lane] = (uint8_t)(lane == 15 ? tagb | 0x80u : tagb);
    const uint32_t hw[4] = {hp.x, hp.y, hp.z, hp.w};
    write_hpow(hd, hw, frob, (int)lane);
}

// The end of a GCM-SIV message: S = BR(POLYVAL value) with the nonce XORed into
// bytes 0..11 and the top bit of byte 15 cleared; tag = AES(S) under the slot's
// encryption key.  The POLYVAL value is the XOR of the partials (times H' where
// they do not hold that factor), or in d.yout where the tile kernel has formed
// it.  Encrypt (d.op 0): one workgroup writes the tag and the counter block.
// Decrypt: all 16 bytes are compared with the received tag without early exit;
// every workgroup forms the verdict by itself, and clears its share of a
// rejected output.  As three kernels (verdict, tag, zero-fill) the end of 1 MiB
// verified took 2.1 + 3.8 + 1.7 us and the gaps between them.
__global__ __launch_bounds__(256) void k_siv_verdict(MsgDesc d, SivArg na, u32x4 *ctr_out,
                                                     const u32x4 *__restrict__ partials,
                                                     const uint32_t *te0g, const uint32_t *sbg)
{
    __shared__ uint32_t te0[256], sb[256], rk[4 * (kMaxNr + 2)];
    __shared__ u32x4 sh[4];
    const uint32_t tid = threadIdx.x;
    const int lane = (int)(tid & 63u), wave = (int)uniform(tid >> 6);
    const CONST_AS KeySlotHdr *hd = cptr<KeySlotHdr>(reinterpret_cast<const void *>(d.slot));
    const uint32_t t0 = te0g[tid], b0 = sbg[tid];
    const uint32_t key = tid < 4 * (kMaxNr + 1) ? gptr<const KeySlotHdr>(d.slot)->rk[tid] : 0u;
    const uint32_t want = d.op == 1 && lane < 16 ? gptr<const uint8_t>(d.tag)[lane] : 0u;
    const uint64_t run = d.n_tiles - ((d.flags & kMerge) ? 1 : 0), P = (run + (1ull << d.log2G) - 1) >> d.log2G;
    const bool formed = d.flags & kFinish;
    u32x4 s = {0, 0, 0, 0};
    if (formed)
        s = *gptr<const u32x4>(d.yout);
    else
        for (uint64_t i = tid; i < P; i += 256)
            s ^= partials[d.tile_base + i];
    te0[tid] = t0, sb[tid] = b0;
    if (tid < 4 * (kMaxNr + 2))
        rk[tid] = key;
    if (!formed) {
        s = wave_xor_reduce(s);
        if (lane == 0)
            sh[wave] = s;
    }
    asm volatile("" ::"v"(want));  // before the flag, which may lie in the expected tag, is written
    lds_barrier();
    if (!formed) {
        s = sh[0] ^ sh[1] ^ sh[2] ^ sh[3];
        if (!(d.flags & kRows))
            s = gf_mul_wave(s, u32x4{hd->hpow[0][0], hd->hpow[0][1], hd->hpow[0][2], hd->hpow[0][3]});
    }
    const u32x4 sv = rev_block(s);
    const uint32_t c = tid & 3u;
    const uint32_t t = aes_columns(c == 0   ? sv.x ^ na.nonce[0]
                                   : c == 1 ? sv.y ^ na.nonce[1]
                                   : c == 2 ? sv.z ^ na.nonce[2]
                                            : sv.w & 0x7fffffffu,
                                   rk, hd->nr, te0, sb);
    const u32x4 tag = {(uint32_t)__builtin_amdgcn_readlane(t, 0), (uint32_t)__builtin_amdgcn_readlane(t, 1),
                       (uint32_t)__builtin_amdgcn_readlane(t, 2), (uint32_t)__builtin_amdgcn_readlane(t, 3)};
    const uint32_t mine = byte_of(tag, lane & 15);
    if (d.op == 0) {
        if (wave == 0 && lane < 16)
            gptr<uint8_t>(d.tag)[lane] = (uint8_t)mine;
        if (tid == 0)
            *ctr_out = u32x4{tag.x, tag.y, tag.z, tag.w | 0x80000000u};
        return;
    }
    const uint32_t diff = lane < 16 ? mine ^ want : 0u;
    const bool ok = __builtin_amdgcn_ballot_w64(diff != 0) == 0;
    if (blockIdx.x == 0 && tid == 0)
        *gptr<int32_t>(d.ok) = ok ? 1 : 0;
    if (!ok)
        clear_output(&d);
}

// ---------------------------------------------------------------- host-side launchers

hipError_t launch_init_tables(uint32_t *te0, uint32_t *sbox, void *frob, hipStream_t s)
{
    hipLaunchKernelGGL(k_init_tables, dim3(1), dim3(256), 0, s, te0, sbox);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_frob_tables, dim3(kPowLevels - 1), dim3(256), 0, s, reinterpret_cast<u32x4 *>(frob));
    return hipGetLastError();
}

size_t frob_table_bytes() { return (size_t)(kPowLevels - 1) * 4096 * 16; }

// Expand n keys (key i: key_lens[i] bytes at keys + key_off[i]) into the
// slots at slot_addrs[i], in launches of kKeyChunk keys.
hipError_t launch_key_setup(const uint8_t *const *keys, const uint32_t *key_lens, const uint64_t *slot_addrs,
                            uint32_t n, const uint32_t *te0, const uint32_t *sbox, const void *frob, hipStream_t s)
{
    for (uint32_t base = 0; base < n; base += kKeyChunk) {
        const uint32_t m = n - base < (uint32_t)kKeyChunk ? n - base : (uint32_t)kKeyChunk;
        KeyChunk kc{};
        SlotChunk sc{};
        for (uint32_t j = 0; j < m; ++j) {
            const uint8_t *key = keys[base + j];
            const uint32_t len = key_lens[base + j];
            for (uint32_t i = 0; i < len / 4; ++i)
                kc.keys[j].w[i] = (uint32_t)key[4 * i] | ((uint32_t)key[4 * i + 1] << 8) |
                                  ((uint32_t)key[4 * i + 2] << 16) | ((uint32_t)key[4 * i + 3] << 24);
            kc.keys[j].len = len;
            kc.slots[j] = slot_addrs[base + j];
            sc.slots[j] = slot_addrs[base + j];
        }
        hipLaunchKernelGGL(k_key_setup, dim3(m), dim3(64), 0, s, kc, te0, sbox, reinterpret_cast<const u32x4 *>(frob));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_key_tables, dim3(kKeyTableBlocks, m), dim3(256), 0, s, sc);
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <int WAVES>
static hipError_t launch_tiles_w(const MsgDesc *descs, const WorkItem *items, uint32_t n_items, const MsgDesc *single,
                                 const uint32_t *te0, u32x4 *partials, uint32_t *counters, uint32_t grid,
                                 bool rows, hipStream_t s)
{
    if (descs && rows)
        hipLaunchKernelGGL((k_gcm_rows<WAVES, true, kGcm>), dim3(grid), dim3(WAVES * 64), 0, s, MsgDesc{}, descs, items,
                           n_items, te0, partials, counters);
    else if (descs)
        hipLaunchKernelGGL((k_gcm_tiles<WAVES, true, kGcm>), dim3(grid), dim3(WAVES * 64), 0, s, MsgDesc{}, descs,
                           items, n_items, te0, partials, counters);
    else if (single->op == 2)
        hipLaunchKernelGGL((k_gcm_tiles<WAVES, false, kCtr>), dim3(grid), dim3(WAVES * 64), 0, s, *single, nullptr,
                           nullptr, n_items, te0, partials, counters);
    else if (single->flags & kRows)
        hipLaunchKernelGGL((k_gcm_rows<WAVES, false, kGcm>), dim3(n_items), dim3(WAVES * 64), 0, s, *single, nullptr,
                           nullptr, n_items, te0, partials, counters);
    else
        hipLaunchKernelGGL((k_gcm_tiles<WAVES, false, kGcm>), dim3(grid), dim3(WAVES * 64), 0, s, *single, nullptr,
                           nullptr, n_items, te0, partials, counters);
    return hipGetLastError();
}

hipError_t launch_tiles(int waves, const MsgDesc *descs, const WorkItem *items, uint32_t n_items,
                        const MsgDesc *single, const uint32_t *te0, void *partials, uint32_t *counters, uint32_t grid,
                        bool rows, hipStream_t s)
{
    u32x4 *p = reinterpret_cast<u32x4 *>(partials);
    switch (waves) {
    case 8:
        return launch_tiles_w<8>(descs, items, n_items, single, te0, p, counters, grid, rows, s);
    case 12:
        return launch_tiles_w<12>(descs, items, n_items, single, te0, p, counters, grid, rows, s);
    case 16:
        return launch_tiles_w<16>(descs, items, n_items, single, te0, p, counters, grid, rows, s);
    default:
        return hipErrorInvalidValue;
    }
}

int max_groups_per_cu(int waves)
{
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (waves) {
    case 8:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_gcm_tiles<8, false, kGcm>, 8 * 64, 0);
        break;
    case 12:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_gcm_tiles<12, false, kGcm>, 12 * 64, 0);
        break;
    case 16:
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_gcm_tiles<16, false, kGcm>, 16 * 64, 0);
        break;
    }
    return (e == hipSuccess && n > 0) ? n : 1;
}

template <int LOGF>
static void launch_combine_f(const MsgDesc *descs, uint32_t n_msgs, const MsgDesc *single, const u32x4 *p, hipStream_t s)
{
    if (descs)
        hipLaunchKernelGGL((k_gcm_combine<true, LOGF>), dim3(n_msgs), dim3(kCombineThreads), 0, s, descs, MsgDesc{}, p);
    else
        hipLaunchKernelGGL((k_gcm_combine<false, LOGF>), dim3(1), dim3(kCombineThreads), 0, s, nullptr, *single, p);
}

hipError_t launch_combine(const MsgDesc *descs, uint32_t n_msgs, const MsgDesc *single, const void *partials,
                          uint32_t fanin, hipStream_t s)
{
    const u32x4 *p = reinterpret_cast<const u32x4 *>(partials);
    switch (fanin) {
    case 2:
        launch_combine_f<1>(descs, n_msgs, single, p, s);
        break;
    case 4:
        launch_combine_f<2>(descs, n_msgs, single, p, s);
        break;
    case 8:
        launch_combine_f<3>(descs, n_msgs, single, p, s);
        break;
    case 16:
        launch_combine_f<4>(descs, n_msgs, single, p, s);
        break;
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_verdict(const MsgDesc *descs, uint32_t n_msgs, const MsgDesc *single, const void *partials,
                          uint32_t *counters, hipStream_t s)
{
    const u32x4 *p = reinterpret_cast<const u32x4 *>(partials);
    if (descs) {
        hipLaunchKernelGGL(k_gcm_verdict<true>, dim3(n_msgs), dim3(256), 0, s, MsgDesc{}, descs, p, counters);
    } else {
        hipLaunchKernelGGL(k_gcm_verdict<false>, dim3(verdict_groups(*single)), dim3(256), 0, s, *single, nullptr, p, counters);
    }
    return hipGetLastError();
}

hipError_t launch_fold(const void *vals, uint32_t k, const void *ekj0, uint8_t *tag, int32_t *ok, uint32_t op,
                       uint32_t tag_len, uint64_t slot, const uint32_t lenblk[4], hipStream_t s)
{
    const u32x4 l = lenblk ? u32x4{lenblk[0], lenblk[1], lenblk[2], lenblk[3]} : u32x4{0, 0, 0, 0};
    hipLaunchKernelGGL(k_gcm_fold, dim3(1), dim3(64), 0, s, reinterpret_cast<const u32x4 *>(vals), k,
                       reinterpret_cast<const u32x4 *>(ekj0), tag, ok, op, tag_len, lenblk ? slot : 0, l);
    return hipGetLastError();
}

hipError_t launch_j0(const IvArg &iv, uint64_t slot, void *j0_out, void *y_zero, hipStream_t s)
{
    hipLaunchKernelGGL(k_gcm_j0, dim3(1), dim3(64), 0, s, iv, slot, reinterpret_cast<u32x4 *>(j0_out),
                       reinterpret_cast<u32x4 *>(y_zero));
    return hipGetLastError();
}

hipError_t launch_zerofill(const MsgDesc *descs, const uint32_t *counters, uint32_t grid, uint64_t longest, hipStream_t s)
{
    hipLaunchKernelGGL(k_gcm_zerofill, dim3(grid), dim3(256), 0, s, descs, counters, longest);
    return hipGetLastError();
}

hipError_t launch_siv_derive(uint64_t kgk_slot, const uint8_t nonce[12], uint64_t out_slot, const uint8_t *tag_in,
                             void *ctr_out, const uint32_t *te0, const uint32_t *sbox, const void *frob, hipStream_t s)
{
    SivArg a{};
    for (int i = 0; i < 3; ++i)
        a.nonce[i] = (uint32_t)nonce[4 * i] | ((uint32_t)nonce[4 * i + 1] << 8) | ((uint32_t)nonce[4 * i + 2] << 16) |
                     ((uint32_t)nonce[4 * i + 3] << 24);
    hipLaunchKernelGGL(k_siv_derive, dim3(1), dim3(128), 0, s, kgk_slot, a, out_slot, tag_in,
                       reinterpret_cast<u32x4 *>(ctr_out), te0, sbox, reinterpret_cast<const u32x4 *>(frob));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    SlotChunk sc{};
    sc.slots[0] = out_slot;
    hipLaunchKernelGGL(k_key_tables, dim3(kKeyTableBlocks, 1), dim3(256), 0, s, sc);
    return hipGetLastError();
}

hipError_t launch_siv_verdict(const MsgDesc &d, const uint8_t nonce[12], void *ctr_out, const void *partials,
                              const uint32_t *te0, const uint32_t *sbox, hipStream_t s)
{
    SivArg a{};
    for (int i = 0; i < 3; ++i)
        a.nonce[i] = (uint32_t)nonce[4 * i] | ((uint32_t)nonce[4 * i + 1] << 8) | ((uint32_t)nonce[4 * i + 2] << 16) |
                     ((uint32_t)nonce[4 * i + 3] << 24);
    hipLaunchKernelGGL(k_siv_verdict, dim3(verdict_groups(d)), dim3(256), 0, s, d, a, reinterpret_cast<u32x4 *>(ctr_out),
                       reinterpret_cast<const u32x4 *>(partials), te0, sbox);
    return hipGetLastError();
}

// pass 0: POLYVAL (encrypt), 1: counter mode (encrypt), 2: both (decrypt-verify)
template <int WAVES>
static hipError_t launch_siv_tiles_w(int pass, const MsgDesc &d, uint32_t n_items, const uint32_t *te0, u32x4 *p,
                                     uint32_t grid, hipStream_t s)
{
    if (pass == 0 && (d.flags & kRows))
        hipLaunchKernelGGL((k_gcm_rows<WAVES, false, kSivHash>), dim3(n_items), dim3(WAVES * 64), 0, s, d, nullptr,
                           nullptr, n_items, te0, p, nullptr);
    else if (pass == 2 && (d.flags & kRows))
        hipLaunchKernelGGL((k_gcm_rows<WAVES, false, kSivDec>), dim3(n_items), dim3(WAVES * 64), 0, s, d, nullptr,
                           nullptr, n_items, te0, p, nullptr);
    else if (pass == 0)
        hipLaunchKernelGGL((k_gcm_tiles<WAVES, false, kSivHash>), dim3(grid), dim3(WAVES * 64), 0, s, d, nullptr,
                           nullptr, n_items, te0, p, nullptr);
    else if (pass == 1)
        hipLaunchKernelGGL((k_gcm_tiles<WAVES, false, kSivCtr>), dim3(grid), dim3(WAVES * 64), 0, s, d, nullptr,
                           nullptr, n_items, te0, p, nullptr);
    else
        hipLaunchKernelGGL((k_gcm_tiles<WAVES, false, kSivDec>), dim3(grid), dim3(WAVES * 64), 0, s, d, nullptr,
                           nullptr, n_items, te0, p, nullptr);
    return hipGetLastError();
}

hipError_t launch_siv_tiles(int waves, int pass, const MsgDesc &d, uint32_t n_items, const uint32_t *te0,
                            void *partials, uint32_t grid, hipStream_t s)
{
    u32x4 *p = reinterpret_cast<u32x4 *>(partials);
    if (pass < 0 || pass > 2)
        return hipErrorInvalidValue;
    switch (waves) {
    case 8:
        return launch_siv_tiles_w<8>(pass, d, n_items, te0, p, grid, s);
    case 12:
        return launch_siv_tiles_w<12>(pass, d, n_items, te0, p, grid, s);
    case 16:
        return launch_siv_tiles_w<16>(pass, d, n_items, te0, p, grid, s);
    default:
        return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------- fixed device scratch

// Workspace of the allocation-free entry point: a module-scope array that
// every device the library runs on holds until the process ends.  Host code
// never passes its name to a kernel (on the host it is only a stand-in
// symbol); it passes the device address looked up below.
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];

// Device address of `scratch` on `device`, looked up once per device with
// that device current and kept for every later context on it.
hipError_t scratch_address(int device, void **out)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices)
        return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess)
            return e;
        if (cur != device) {
            e = hipSetDevice(device);
            if (e != hipSuccess)
                return e;
        }
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device)
            (void)hipSetDevice(cur);
        if (e != hipSuccess)
            return e;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

}  // namespace gcm
