// gcm_plan.h -- launch planning shared by every entry point: argument and
// aliasing checks, tile geometry, per-message descriptors, batch work lists
// and workspace sizes.  It holds no HIP state (plain C++ over the layouts of
// gcm_internal.h), so the same code runs inside the library and in a
// CPU-only harness built with the address and undefined-behaviour
// sanitizers.
//
// Geometry (the paper's map phase over wave tiles): a message's GHASH input
// X = A || 0-pad || C || 0-pad || L has m = n_A + n + 1 blocks (SP 800-38D
// GCM-AE step 5), left-padded with z zero blocks so that m + z = T * 2^log2B
// (GHASH(0^z || X) = GHASH(X)); wave tile t covers padded positions
// [t * 2^log2B, (t + 1) * 2^log2B).  The tiles of a workgroup leave one 16-byte
// partial together (set_groups), but for streams and the host pipeline, whose
// tiles leave one each.
#pragma once
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <numeric>
#include <vector>

#include "../../include/gcm_mi355.h"
#include "gcm_internal.h"

namespace gcm {

constexpr uint64_t kMaxLen = (1ull << 36) - 32;  // 2^39 - 256 bits (SP 800-38D sec. 5.2.1.1)
constexpr uint64_t kMaxAad = (1ull << 61) - 1;   // < 2^64 bits

// A launch shape: wave tile size (log2 blocks; for a batch, the cap on its
// messages' tile sizes), waves per workgroup, resident workgroups per compute
// unit, and the fan-in of the tree over tile partials (streams, pipeline).  Results
// never depend on it, only speed does.
struct Shape {
    uint32_t log2B = 16, waves = 16, gpc = 1, fanin = 2;
};
// An autotune cache entry: the fastest shape of its search, and whether calls use
// it, or were at least as fast with the shape they have without an entry.
struct TuneEntry : Shape {
    bool faster = true;
};

// size bucket of the autotune caches: floor(log2 x) (0 for x <= 1)
inline uint32_t size_bucket(uint64_t x)
{
    uint32_t b = 0;
    while (b < 63 && (2ull << b) <= x)
        ++b;
    return b;
}

inline bool valid_fanin(uint32_t f) { return f == 2 || f == 4 || f == 8 || f == 16; }

// An error found while planning: a GCM_E_* code and its message.
struct PlanError {
    int code = GCM_OK;
    char msg[256] = {0};
};

inline int plan_fail(PlanError *e, int code, const char *fmt, ...)
{
    if (e) {
        e->code = code;
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(e->msg, sizeof e->msg, fmt, ap);
        va_end(ap);
    }
    return code;
}

// GHASH blocks of a message: AAD blocks, data blocks and the length block.
inline uint64_t ghash_blocks(uint64_t aad_len, uint64_t len) { return (aad_len + 15) / 16 + (len + 15) / 16 + 1; }

inline uint32_t ceil_log2_u64(uint64_t x)
{
    uint32_t l = 0;
    while (l < 63 && (1ull << l) < x)
        ++l;
    return l;
}

// [a, a + alen) and [b, b + blen) share a byte (empty ranges share none);
// written without forming a + alen, so no address can overflow it.
inline bool ranges_overlap(uint64_t a, uint64_t alen, uint64_t b, uint64_t blen)
{
    if (!alen || !blen)
        return false;
    return a >= b ? a - b < blen : b - a < alen;
}

// Tile size of one message launched alone, by makespan: `resident` waves
// run tiles k, k + R, ...; tile 0 holds the zero prefix, whose whole rows are
// skipped; each tile adds a fixed cost (fix-up, partial) of about kTileCost
// blocks.  Tiles of one or two rows only while every tile gets a wave of its
// own.  Ties go to the larger tile (fewer partials).
inline uint32_t heuristic_log2B(uint64_t m, uint64_t resident)
{
    constexpr uint64_t kTileCost = 64;
    if (resident == 0)
        resident = 1;
    uint64_t best_cost = ~0ull;
    uint32_t best_l = 16;
    for (uint32_t l = 16; l >= 6; --l) {
        const uint64_t B = 1ull << l;
        const uint64_t T = (m + B - 1) / B;
        if (l < 8 && T > resident)
            continue;
        const uint64_t z = T * B - m;
        const uint64_t n0 = (T + resident - 1) / resident, n1 = T > 1 ? (T - 1 + resident - 1) / resident : 0;
        const uint64_t c0 = (n0 - 1) * B + (B - z / 64 * 64) + kTileCost * n0;
        const uint64_t c1 = n1 * (B + kTileCost);
        const uint64_t cost = std::max(c0, c1);
        if (cost < best_cost) {
            best_cost = cost;
            best_l = l;
        }
    }
    return best_l;
}

// Rows of 64 blocks that the busiest compute unit runs for one message
// launched with tiles of 2^l blocks in workgroups of `waves` waves: item k
// (tiles [k*waves, (k+1)*waves)) goes to workgroup k mod grid, grid =
// min(items, cus * gpc), and each tile costs its rows plus about one row of
// fix-up.  Used to compare shapes, not to predict times.
inline uint64_t busiest_cu_rows(uint64_t m, uint32_t l, uint32_t waves, uint64_t cus, uint32_t gpc)
{
    const uint64_t B = 1ull << l, T = (m + B - 1) / B;
    const uint64_t items = (T + waves - 1) / waves;
    const uint64_t slots = cus * (gpc ? gpc : 1);
    const uint64_t grid = items < slots ? items : slots;
    uint64_t tiles = 0;  // workgroup 0's, its items k*grid
    for (uint64_t k = 0; k * grid < items; ++k) {
        const uint64_t first = k * grid * waves;
        tiles += T - first < waves ? T - first : waves;
    }
    return tiles * (B / 64 + 1) * (gpc ? gpc : 1);
}

// Waves per workgroup for one message (tile size from heuristic_log2B for
// that many waves).  Sixteen unless the message has fewer tiles than the
// chip has wave slots: then 16-wave workgroups would crowd its tiles onto a
// fraction of the compute units, and 12 or 8 waves a workgroup spread them
// over more.  Among 16, 12 and 8 the one whose busiest compute unit has the
// fewest rows (busiest_cu_rows) wins, ties to more waves.  gpc(w): groups a
// compute unit holds with w waves.
template <typename Gpc>
inline uint32_t heuristic_waves(uint64_t m, uint64_t cus, Gpc gpc)
{
    const uint32_t g16 = gpc(16);
    const uint32_t l16 = heuristic_log2B(m, cus * g16 * 16);
    const uint64_t t16 = (m + (1ull << l16) - 1) >> l16;
    if ((t16 + 15) / 16 >= cus * g16)
        return 16;
    uint32_t best_w = 16;
    uint64_t best = busiest_cu_rows(m, l16, 16, cus, g16);
    for (uint32_t w : {12u, 8u}) {
        const uint32_t g = gpc(w);
        const uint32_t l = heuristic_log2B(m, cus * g * w);
        const uint64_t load = busiest_cu_rows(m, l, w, cus, g);
        if (load < best) {
            best = load;
            best_w = w;
        }
    }
    return best_w;
}

// Tiles that suffice for every message of at most m GHASH blocks planned by
// the heuristics above (t_own: the m-block message's own tile count): a
// tile size below 2^8 blocks is only chosen while the tiles fit the
// resident waves (at most `resident_max` over the wave counts), larger ones
// give at most ceil(m / 256) tiles.  The tile count is not monotonic in the
// length (a longer message may take larger tiles), so a workspace sized for
// the longest message of a set needs this bound, not its own count.
inline uint64_t tiles_bound_upto(uint64_t m, uint64_t t_own, uint64_t resident_max)
{
    const uint64_t small = std::min<uint64_t>((m + 63) / 64, resident_max);
    return std::max<uint64_t>(t_own, std::max<uint64_t>(small, (m + 255) / 256));
}

// Tile size of one message inside a batch: about one workgroup item (waves
// tiles) for small messages, at most 2^cap blocks per tile for large ones,
// so the persistent workgroups see items of similar cost.  cap: 6..20.
inline uint32_t batch_msg_log2B(uint64_t m, uint32_t waves, uint32_t cap)
{
    const uint32_t l = std::max<uint32_t>(6, ceil_log2_u64((m + waves - 1) / waves));
    return std::min(l, std::max<uint32_t>(6, cap));
}

// Whether a batch of n messages, m GHASH blocks in all, goes to the row kernel
// (one-row tiles, two workgroups of eight waves a compute unit).  A row takes it
// 1100 cycles with AES-128, 1230 with AES-256, where the tile kernel takes 388 and
// 523; but an item of the tile kernel costs some 12000 cycles besides, most of them
// for the 80 KiB of key tables, so that messages of up to some 17 rows are better
// off with rows (1024 messages, median 8 KiB with 1 KiB of AAD: 55 us, 63 with tiles;
// median 16 KiB: 89 and 78), and so is what gives every wave slot of the chip at
// most a row (64 messages, median 16 KiB: 15 us, 27 with tiles).
inline bool batch_rows(uint64_t n, uint64_t m, uint64_t cus) { return m <= 1024 * n || m <= 64 * 16 * cus; }

// Workspace: a counter and reject list (4 + 4 * n_msgs bytes, rounded up to
// 256), then per message its T tile partials followed by two 16-byte slots:
// E_K(J0) (left by the tile or row kernel, after the partials) and J0 (IVs other than
// 96 bits).
inline uint64_t workspace_counter_bytes(uint64_t n_msgs) { return ((4 + 4 * n_msgs) + 255) / 256 * 256; }
inline uint64_t workspace_bytes_for(uint64_t total_tiles, uint64_t n_msgs)
{
    return workspace_counter_bytes(n_msgs) + 16 * (total_tiles + 2 * n_msgs);
}

inline void fill_desc(MsgDesc *d, uint32_t op, const uint8_t *iv, uint64_t aad, uint64_t aad_len, uint64_t in,
                      uint64_t out, uint64_t len, uint64_t tag, uint64_t ok, uint64_t slot_addr, uint32_t nr,
                      uint32_t log2B, uint32_t waves, uint64_t tile_base)
{
    memset(d, 0, sizeof *d);
    d->in = in;
    d->out = out;
    d->aad = aad;
    d->tag = tag;
    d->ok = ok;
    d->len = len;
    d->aad_len = aad_len;
    d->slot = slot_addr;
    d->n = (len + 15) / 16;
    d->na = (aad_len + 15) / 16;
    d->m = d->na + d->n + 1;
    const uint64_t B = 1ull << log2B;
    d->n_tiles = (d->m + B - 1) / B;
    d->z = d->n_tiles * B - d->m;
    d->tile_lo = 0;
    d->tile_hi = d->n_tiles;
    d->tile_base = tile_base;
    for (int i = 0; i < 3; ++i)
        d->iv[i] = (uint32_t)iv[4 * i] | ((uint32_t)iv[4 * i + 1] << 8) | ((uint32_t)iv[4 * i + 2] << 16) |
                   ((uint32_t)iv[4 * i + 3] << 24);
    d->op = op;
    d->log2B = log2B;
    d->nr = nr;
    d->groups = (uint32_t)((d->n_tiles + waves - 1) / waves);
    d->tag_len = 16;
}

// Tiles whose partials a workgroup of `waves` waves sums into one: the largest
// power of two that divides the wave count (its groups then never straddle a
// work item).  The sum is a product and an XOR in the tile kernel, where a tree
// would spend a level on it: with 16 waves a 1 GiB message leaves 257 partials
// instead of 4097.
inline uint16_t group_log2(uint32_t waves) { return waves == 16 ? 4 : waves == 8 ? 3 : waves == 12 ? 2 : 0; }

// tiles that a launch of the whole message runs, and partials it leaves
inline uint64_t tiles_run(const MsgDesc &d) { return d.n_tiles - ((d.flags & kMerge) ? 1 : 0); }
inline uint64_t n_partials(const MsgDesc &d) { return (tiles_run(d) + (1ull << d.log2G) - 1) >> d.log2G; }

// Group the descriptor's tiles for workgroups of `waves` waves; a message of
// one group is finished by the tile kernel if its result is wanted right then.
// There one wave clears a rejected output, 17 us a MiB, which a batch hides up to
// the 1 MiB of its largest items (600 rejected messages of 200 KiB: 168 us, 187
// with a verdict and the zero-fill after the tiles; 2000 of 250 KiB: 577, 608),
// but not 10 MiB launched alone (2694 us, 2870 where one wave clears them).
constexpr uint64_t kFinishClear = 1ull << 20;
inline void set_groups(MsgDesc *d, uint32_t waves, bool whole)
{
    d->log2G = group_log2(waves);
    d->flags = 0;
    if (whole && d->log2G && n_partials(*d) == 1 && (d->op != 1 || d->len <= kFinishClear))
        d->flags = kFinish;
}

// One message launched alone on `slots` resident workgroups.  The planner lets
// a message have one tile more than there are waves, because tile 0 holds the
// zero prefix and is short; as a work item of its own it would hold up the
// sixteen tiles of the next item of its workgroup (6 us of a 67 MB message's
// 85), so that tile 1's wave takes it along.
// Tiles of one row go to the row kernel, as long as every workgroup is resident
// at once (it stages the AES tables in each).
inline void set_groups_single(MsgDesc *d, uint32_t waves, uint64_t slots)
{
    set_groups(d, waves, true);
    if (d->log2G && d->n_tiles > slots * waves && d->n_tiles % waves == 1)
        d->flags |= kMerge;
    else if (d->log2G && d->log2B == 6 && d->n_tiles <= slots * waves)
        d->flags |= kRows;
}

// Workgroups of a single message's verdict: on decrypt enough to clear a
// rejected output at the memory's rate.  Each of them reads the expected tag and
// the first writes the accept flag, so that a flag that lies in the tag leaves
// room for one only.
inline uint32_t verdict_groups(const MsgDesc &d)
{
    const uint64_t chunks = (d.len / 16 + 255) / 256;
    if (d.op != 1 || chunks < 1 || ranges_overlap(d.ok, 4, d.tag, d.tag_len))
        return 1;
    return (uint32_t)std::min<uint64_t>(chunks, 1024);
}

// Device buffers of one message: NULL with a non-zero length, 16-byte
// alignment of AAD and payload, and aliasing.  The output may equal the
// input exactly (in place) but may not overlap it otherwise, nor overlap the
// AAD (still being hashed while other waves write output), the tag (written
// or compared after the output is written) or the accept flag.  tag / ok of
// 0 are not checked.
inline int check_buffers(uint64_t aad, uint64_t aad_len, uint64_t in, uint64_t out, uint64_t len, uint64_t tag,
                         uint64_t tag_len, uint64_t ok, PlanError *err)
{
    if ((len && (!in || !out)) || (aad_len && !aad))
        return plan_fail(err, GCM_E_ARG, "NULL device buffer with non-zero length");
    if ((aad_len && (aad & 15)) || (len && ((in & 15) || (out & 15))))
        return plan_fail(err, GCM_E_ARG, "device buffers must be 16-byte aligned");
    if (len && in != out && ranges_overlap(in, len, out, len))
        return plan_fail(err, GCM_E_ALIAS, "input and output overlap without being identical");
    if (ranges_overlap(out, len, aad, aad_len))
        return plan_fail(err, GCM_E_ALIAS, "output overlaps the AAD");
    if (tag && ranges_overlap(out, len, tag, tag_len))
        return plan_fail(err, GCM_E_ALIAS, "output overlaps the tag");
    if (ok && ranges_overlap(out, len, ok, 4))
        return plan_fail(err, GCM_E_ALIAS, "output overlaps the accept flag");
    return GCM_OK;
}

inline int check_lengths(uint64_t aad_len, uint64_t len, PlanError *err)
{
    if (len > kMaxLen || aad_len > kMaxAad)
        return plan_fail(err, GCM_E_TOOLONG, "len %llu / aad_len %llu beyond the SP 800-38D limits",
                         (unsigned long long)len, (unsigned long long)aad_len);
    return GCM_OK;
}

// The key table as the planner sees it.
struct SlotView {
    uint64_t base = 0;              // device address of slot 0
    uint32_t n_slots = 0;
    const uint8_t *used = nullptr;  // [n_slots] 1 = registered
    const uint32_t *nr = nullptr;   // [n_slots] AES rounds
    uint64_t addr(uint32_t s) const { return base + kSlotBytes * (uint64_t)s; }
    bool valid(uint32_t s) const { return s < n_slots && used[s]; }
};

// One job of a batch against a base allocation of base_bytes bytes.
inline int check_job(const gcm_job &j, uint32_t idx, uint64_t base_bytes, const SlotView &slots, PlanError *err)
{
    if (j.op > 1)
        return plan_fail(err, GCM_E_ARG, "job %u: op %u is neither 0 (encrypt) nor 1 (decrypt-verify)", idx, j.op);
    if (j.reserved != 0)
        return plan_fail(err, GCM_E_ARG, "job %u: reserved field must be 0", idx);
    if (!slots.valid(j.key_slot))
        return plan_fail(err, GCM_E_SLOT, "job %u: key slot %u is not registered", idx, j.key_slot);
    if (j.len > kMaxLen || j.aad_len > kMaxAad)
        return plan_fail(err, GCM_E_TOOLONG, "job %u: len %llu / aad_len %llu beyond the SP 800-38D limits", idx,
                         (unsigned long long)j.len, (unsigned long long)j.aad_len);
    auto inside = [&](uint64_t off, uint64_t len) { return off <= base_bytes && len <= base_bytes - off; };
    if (!inside(j.in_off, j.len) || !inside(j.out_off, j.len) || !inside(j.aad_off, j.aad_len) ||
        !inside(j.tag_off, 16) || (j.op == 1 && !inside(j.ok_off, 4)))
        return plan_fail(err, GCM_E_ARG, "job %u: a buffer lies outside the %llu-byte base allocation", idx,
                         (unsigned long long)base_bytes);
    if ((j.len && ((j.in_off | j.out_off) & 15)) || (j.aad_len && (j.aad_off & 15)) || (j.op == 1 && (j.ok_off & 3)))
        return plan_fail(err, GCM_E_ARG, "job %u: payload offsets must be 16-byte aligned and ok_off 4-byte aligned",
                         idx);
    if (j.len && j.in_off != j.out_off && ranges_overlap(j.in_off, j.len, j.out_off, j.len))
        return plan_fail(err, GCM_E_ALIAS, "job %u: input and output overlap without being identical", idx);
    if (ranges_overlap(j.out_off, j.len, j.aad_off, j.aad_len) || ranges_overlap(j.out_off, j.len, j.tag_off, 16) ||
        (j.op == 1 && ranges_overlap(j.out_off, j.len, j.ok_off, 4)))
        return plan_fail(err, GCM_E_ALIAS, "job %u: output overlaps its AAD, tag or accept flag", idx);
    return GCM_OK;
}

// One message of a batch, with absolute device addresses.
struct PlanMsg {
    uint32_t op = 0;
    uint32_t key_slot = 0;
    uint8_t iv[12] = {0};
    uint64_t aad = 0, aad_len = 0, in = 0, out = 0, len = 0, tag = 0, ok = 0;
};

inline PlanMsg plan_msg_from_job(const gcm_job &j, uint64_t base)
{
    PlanMsg p;
    p.op = j.op;
    p.key_slot = j.key_slot;
    memcpy(p.iv, j.iv, 12);
    p.aad = base + j.aad_off;
    p.aad_len = j.aad_len;
    p.in = base + j.in_off;
    p.out = base + j.out_off;
    p.len = j.len;
    p.tag = base + j.tag_off;
    p.ok = base + j.ok_off;
    return p;
}

// The persistent launch of a batch: descriptors (message i's partials start
// at tile_base, after the n_tiles + 2 slots of the messages before it), and
// the work list -- items of `waves` consecutive wave tiles of one message -- by
// key slot, which spread_items shares out among the workgroups.
struct BatchPlan {
    std::vector<MsgDesc> descs;
    std::vector<WorkItem> items;
    uint64_t total_tiles = 0;   // sum of n_tiles
    uint64_t partial_slots = 0; // sum of n_tiles + 2 (the workspace's per-message part)
    uint64_t payload = 0;
    bool any_decrypt = false;
    // messages that the tile kernel does not finish by itself, and decrypts among them
    bool any_combine = false, any_zerofill = false;
    uint64_t longest_zerofill = 0;  // payload bytes of the longest of the latter
    bool rows = false;  // all tiles are single rows, run by the row kernel
    uint64_t workspace_bytes() const { return workspace_counter_bytes(descs.size()) + 16 * partial_slots; }
};

inline void plan_batch(const PlanMsg *msgs, uint32_t n, const SlotView &slots, uint32_t waves, uint32_t cap_log2B,
                       BatchPlan *p)
{
    p->descs.assign(n, MsgDesc{});
    p->items.clear();
    p->total_tiles = p->partial_slots = p->payload = 0;
    p->any_decrypt = p->any_combine = p->any_zerofill = false;
    p->longest_zerofill = 0;
    p->rows = cap_log2B <= 6 && group_log2(waves) != 0;
    uint64_t tile_base = 0, n_items = 0;
    for (uint32_t i = 0; i < n; ++i) {
        const PlanMsg &j = msgs[i];
        const uint32_t log2B = batch_msg_log2B(ghash_blocks(j.aad_len, j.len), waves, cap_log2B);
        fill_desc(&p->descs[i], j.op, j.iv, j.aad, j.aad_len, j.in, j.out, j.len, j.tag, j.ok, slots.addr(j.key_slot),
                  slots.nr[j.key_slot], log2B, waves, tile_base);
        set_groups(&p->descs[i], waves, true);
        if (p->rows)
            p->descs[i].flags |= kRows;
        p->any_combine |= !(p->descs[i].flags & kFinish);
        if (!(p->descs[i].flags & kFinish) && j.op == 1) {
            p->any_zerofill = true;
            p->longest_zerofill = std::max(p->longest_zerofill, j.len);
        }
        tile_base += p->descs[i].n_tiles + 2;  // partials, then the E_K(J0) and J0 slots
        p->total_tiles += p->descs[i].n_tiles;
        p->any_decrypt |= j.op == 1;
        p->payload += j.len;
        n_items += p->descs[i].groups;
    }
    p->partial_slots = tile_base;
    // by key slot, a slot's messages as they come: a counting sort, unless the
    // table has many more slots than the batch has messages
    std::vector<uint32_t> order(n);
    if (slots.n_slots / 4 <= n) {
        std::vector<uint32_t> at(slots.n_slots + 1, 0);
        for (uint32_t i = 0; i < n; ++i)
            ++at[msgs[i].key_slot + 1];
        for (uint32_t k = 0; k < slots.n_slots; ++k)
            at[k + 1] += at[k];
        for (uint32_t i = 0; i < n; ++i)
            order[at[msgs[i].key_slot]++] = i;
    } else {
        std::iota(order.begin(), order.end(), 0u);
        std::stable_sort(order.begin(), order.end(),
                         [&](uint32_t a, uint32_t c) { return msgs[a].key_slot < msgs[c].key_slot; });
    }
    p->items.reserve(n_items);
    for (uint32_t i : order)
        for (uint64_t t = 0; t < p->descs[i].n_tiles; t += waves)
            p->items.push_back(WorkItem{i, (uint32_t)t});
}

// LDS cycles of a work item of `tiles` tiles of 2^log2B blocks, as far as they
// matter for tile sizes and for spreading items over workgroups: 523 a row of 64
// blocks with AES-256 and proportionally fewer with smaller keys (the compute
// unit is busy), but not less than its longest wave takes alone, and some 12000
// for getting started and summing up.  In the row kernel every wave goes through
// nearly all of it, with a row or without: 6.9 us an item of one row, 8.4 of
// eight with AES-128, 7.7 and 9.4 with AES-256.
constexpr uint64_t kItemStart = 12000, kRowCost = 38;  // kRowCost: a row and AES round
inline uint64_t item_cost(uint32_t log2B, uint32_t nr, uint64_t tiles, bool rows)
{
    if (rows)
        return 9700 + 425 * nr + 460 * tiles;
    return kItemStart + (1ull << (log2B - 6)) * nr * std::max<uint64_t>(tiles * kRowCost, 320);
}

// tiles of the item that begins at place first_tile
inline uint32_t item_tiles(const MsgDesc &d, uint32_t first_tile, uint32_t waves)
{
    const uint64_t G = 1ull << d.log2G, pad = (0 - d.n_tiles) & (G - 1);  // empty places before tile 0
    const uint64_t lo = std::max<uint64_t>(first_tile, pad), hi = std::min<uint64_t>(first_tile + waves, pad + d.n_tiles);
    return hi > lo ? (uint32_t)(hi - lo) : 0;
}

inline uint64_t item_cost(const MsgDesc &d, uint32_t first_tile, uint32_t waves)
{
    return item_cost(d.log2B, d.nr, item_tiles(d, first_tile, waves), d.flags & kRows);
}

// Cap on the tile sizes of a batch run by the tile kernel on `groups` resident
// workgroups of `waves` waves, 2^8..2^12 blocks: small tiles start more items,
// with large ones the longest item decides.  The cap whose estimate is least: the
// workgroups' mean cost and an eighth of the largest item (about what
// spread_items leaves between the mean and the longest workgroup), or the largest
// item alone where that is more; a workgroup that goes on with a message it has
// begun stages no tables and starts the item in a quarter of the time.  Over 32 batches of 4 to 4096 messages of 16 KiB
// to 8 MiB on average, every cap measured, it is within 1.5% of the best one; one
// cap for all of them, or a cap from the number of blocks alone, was up to 1.5
// times it (64 messages, median 64 KiB: 27.8 us with 2^8, 41.2 with 2^9; 512 of
// 1 MiB: 1506, 1291, 1190, 1146 and 1140 us with 2^8 to 2^12).
inline uint32_t batch_cap_log2B(const PlanMsg *msgs, uint32_t n, const SlotView &slots, uint32_t waves, uint64_t groups)
{
    uint64_t items[5] = {}, more[5] = {}, work = 0;  // more: those beyond the first round of a message
    uint64_t most[3] = {};                           // blocks of the largest message by key size
    for (uint32_t i = 0; i < n; ++i) {
        const uint64_t m = ghash_blocks(msgs[i].aad_len, msgs[i].len);
        const uint32_t nr = slots.nr[msgs[i].key_slot];
        const uint64_t k = (m - 1) / ((uint64_t)waves << 8);
        for (uint32_t c = 0; c < 5; ++c) {
            items[c] += (k >> c) + 1;
            more[c] += (k >> c) + 1 > groups ? (k >> c) + 1 - groups : 0;
        }
        work += (m + 63) / 64 * nr * kRowCost;
        uint64_t &mm = most[(nr - 10) / 2];
        mm = std::max(mm, m);
    }
    uint32_t best_cap = 12;
    uint64_t best = ~0ull;
    for (uint32_t cap = 12; cap >= 8; --cap) {
        uint64_t big = 0;
        for (uint32_t q = 0; q < 3; ++q)
            if (most[q]) {
                const uint32_t l = batch_msg_log2B(most[q], waves, cap);
                const uint64_t T = (most[q] + (1ull << l) - 1) >> l;
                big = std::max(big, item_cost(l, 10 + 2 * q, std::min<uint64_t>(T, waves), false));
            }
        const uint64_t it = items[cap - 8], g = std::max<uint64_t>(1, std::min(it, groups));
        const uint64_t starts = kItemStart * it - kItemStart * 3 / 4 * more[cap - 8];
        const uint64_t cost = std::max(big, (starts + work) / g + big / 8);
        if (cost < best) {
            best = cost;
            best_cap = cap;
        }
    }
    return best_cap;
}

// The order in which `grid` workgroups take the work list, workgroup g items g,
// g + grid, ...: handed out the largest first, in every round the largest left
// to the workgroup with the least so far.  In message order the longest sum of a
// workgroup was a fifth above the mean with 512 messages of 1 MiB (median,
// lognormal; 1204 us), and half as much again as the mean with 1024 of 16 KiB
// (124 us).  What a workgroup has been given it runs in the list's order, by key
// slot and message, so that it stages each key's tables once, however few keys
// the messages share; items of up to six on average the largest first, but
// together by message and key (1024 messages, median 16 KiB: 86.8 us, 87.3 in the
// list's order; 2000 of 1 MiB: 3298 us, 3191 in the list's, where workgroups run
// parts of a message at the same time).
inline void spread_items(const std::vector<MsgDesc> &descs, uint32_t waves, uint32_t grid, std::vector<WorkItem> *items)
{
    const size_t n = items->size(), g = grid;
    if (n <= g || g < 2)
        return;
    const bool rows = descs[(*items)[0].msg].flags & kRows;  // as all of them
    // the items by cost: a counting sort over (tile size, key size, tiles)
    constexpr uint32_t kTiles = 16 + 1, kClasses = (20 - 6 + 1) * 3 * kTiles;
    std::vector<uint32_t> cls(n), count(kClasses, 0), by_cost(n);
    for (size_t i = 0; i < n; ++i) {
        const MsgDesc &d = descs[(*items)[i].msg];
        cls[i] = ((d.log2B - 6) * 3 + (d.nr - 10) / 2) * kTiles + item_tiles(d, (*items)[i].first_tile, waves);
        ++count[cls[i]];
    }
    std::vector<std::pair<uint64_t, uint32_t>> used;  // cost, class
    std::vector<uint64_t> cost(kClasses, 0);
    for (uint32_t c = 0; c < kClasses; ++c)
        if (count[c]) {
            cost[c] = item_cost(6 + c / (3 * kTiles), 10 + 2 * (c / kTiles % 3), c % kTiles, rows);
            used.push_back({cost[c], c});
        }
    std::sort(used.begin(), used.end(), std::greater<std::pair<uint64_t, uint32_t>>());
    uint32_t sum = 0;
    for (const auto &u : used) {
        const uint32_t here = count[u.second];
        count[u.second] = sum;
        sum += here;
    }
    for (size_t i = 0; i < n; ++i)
        by_cost[count[cls[i]]++] = (uint32_t)i;
    std::vector<std::pair<uint64_t, uint32_t>> load(g);  // cost so far, workgroup
    for (size_t k = 0; k < g; ++k)
        load[k] = {0, (uint32_t)k};
    std::vector<uint32_t> taker(n);
    bool moved = false;  // a round of items of equal cost leaves the order of the loads as it is
    for (size_t at = 0; at < n; at += g) {
        if (moved)
            std::sort(load.begin(), load.end());
        const size_t m = std::min(g, n - at);
        for (size_t k = 0; k < m; ++k) {
            taker[by_cost[at + k]] = load[k].second;
            load[k].first += cost[cls[by_cost[at + k]]];
        }
        moved = cost[cls[by_cost[at]]] != cost[cls[by_cost[at + m - 1]]];
    }
    // the workgroups with an item in the last round, the first of `load`, come first
    std::vector<uint32_t> next(g), run(n);
    for (size_t k = 0; k < g; ++k)
        next[load[k].second] = (uint32_t)k;
    const bool few = n <= 6 * g;
    for (size_t k = 0; k < n; ++k) {
        const uint32_t i = few ? by_cost[k] : (uint32_t)k;
        uint32_t &to = next[taker[i]];
        run[to] = i;
        to += (uint32_t)g;
    }
    if (few) {
        std::vector<uint32_t> msg(n, 0), slot(n, 0);  // numbered in the list's order
        for (size_t i = 1; i < n; ++i) {
            const uint32_t m = (*items)[i].msg, before = (*items)[i - 1].msg;
            msg[i] = msg[i - 1] + (m != before);
            slot[i] = slot[i - 1] + (descs[m].slot != descs[before].slot);
        }
        // an item goes behind the last one of its message, or else of its key
        for (size_t p = g; p < n && slot[n - 1] + 1 < n; ++p) {
            const uint32_t i = run[p];
            size_t to = 0;  // none yet
            for (size_t q = p; q >= g; q -= g) {
                const uint32_t j = run[q - g];
                if (msg[j] == msg[i]) {
                    to = q;
                    break;
                }
                if (slot[j] == slot[i] && !to)
                    to = q;
            }
            to = to ? to : p;
            for (size_t q = p; q > to; q -= g)
                run[q] = run[q - g];
            run[to] = i;
        }
    }
    std::vector<WorkItem> out(n);
    for (size_t k = 0; k < n; ++k)
        out[k] = (*items)[run[k]];
    items->swap(out);
}

// Device bytes a message adds to the batch that carries it, for any launch
// shape the library may pick (tiles of at least 64 blocks, items of at least
// 8 waves): its descriptor, work items, accept flag, reject-list entry, tile
// partials with their two extra slots, and room for the four 256-byte
// roundings of a batch's sections.
inline uint64_t batch_overhead_bound(uint64_t aad_len, uint64_t len)
{
    const uint64_t T = (ghash_blocks(aad_len, len) + 63) / 64;
    return sizeof(MsgDesc) + sizeof(WorkItem) * ((T + 7) / 8) + 4 + 4 + 16 * (T + 2) + 4 * 256;
}

}  // namespace gcm
