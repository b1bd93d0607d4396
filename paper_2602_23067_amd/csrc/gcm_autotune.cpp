// gcm_autotune.cpp -- exhaustive launch-shape search (the paper tunes its
// kernel parameters per GPU the same way: an exhaustive sweep, keeping the
// fastest), with a bit-equality check across every candidate.
//
// Single messages: for one (key size, message size) point the search times
// every shape of the tile kernel in {log2 tile blocks} x {waves per workgroup} x
// {groups per CU} on a scratch message with HIP events, and the planner's own
// shape, which may be the row kernel's, requires all of them to produce the same
// tag (the counter map and GHASH exponents derive from block indices only), and
// records the fastest in the context's cache, keyed by (key bytes,
// floor(log2 len)), with the fan-in at which the reduction tree that streams and
// the host pipeline end with was fastest for the shape that is used.
//
// Batches: the same search over {waves} x {groups per CU} x {cap on the
// messages' tile sizes} and the planner's own shape on the caller's own batch,
// every point's tags and accept flags compared with the first point's, recorded
// under (floor(log2 messages), floor(log2 payload bytes)).
//
// Calls use a recorded shape if it was faster than the planner's own
// (TuneEntry::faster): 1 MiB with AES-128 takes 12 us in rows, 19 in the best
// tiles of the search.
//
// Every planner (one-shot, asynchronous, batches, the serving loop, host
// pipeline, streamed segments) consults these caches when no explicit shape
// is set with gcm_set_launch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/gcm_mi355.h"
#include "gcm_host.h"

using namespace gcm;

namespace {

const uint32_t kWaveOpts[3] = {8, 12, 16};
const uint32_t kFaninOpts[4] = {2, 4, 8, 16};

// Candidate groups per CU for a workgroup size: 1 .. what the occupancy
// calculator allows (the tile kernel's 149 KiB of LDS hold it to one on
// gfx950, so this dimension has a single point there).
std::vector<uint32_t> gpc_options(uint32_t waves)
{
    std::vector<uint32_t> v;
    const uint32_t mx = (uint32_t)max_groups_per_cu((int)waves);
    for (uint32_t g = 1; g <= mx && g <= 4; ++g)
        v.push_back(g);
    return v;
}

// A shape replaces the planner's own if it takes less than 99% of its time; the
// two are timed in turn this often.
constexpr uint32_t kTurns = 4;
bool is_faster(float shape_ms, float own_ms) { return shape_ms < 0.99f * own_ms; }

bool same(const Shape &x, const Shape &y) { return x.log2B == y.log2B && x.waves == y.waves && x.gpc == y.gpc; }

struct Timer {
    hipEvent_t a = nullptr, b = nullptr;
    hipError_t init()
    {
        hipError_t e = hipEventCreate(&a);
        return e == hipSuccess ? hipEventCreate(&b) : e;
    }
    // f's work on `s`, the mean of `reps` passes in ms, added to *ms
    template <typename F>
    hipError_t add(hipStream_t s, uint32_t reps, float *ms, F f)
    {
        hipError_t e = hipSuccess;
        float total = 0.f;
        for (uint32_t r = 0; r < reps && e == hipSuccess; ++r) {
            e = hipEventRecord(a, s);
            if (e == hipSuccess)
                e = f();
            if (e == hipSuccess)
                e = hipEventRecord(b, s);
            if (e == hipSuccess)
                e = hipEventSynchronize(b);
            float one = 0.f;
            if (e == hipSuccess)
                e = hipEventElapsedTime(&one, a, b);
            total += one;
        }
        *ms += total / (float)reps;
        return e;
    }
    ~Timer()
    {
        if (a)
            (void)hipEventDestroy(a);
        if (b)
            (void)hipEventDestroy(b);
    }
};

}  // namespace

extern "C" int gcm_autotune(gcm_ctx *ctx, uint32_t key_len, uint64_t len, uint32_t reps, gcm_tune_result *out,
                            void *stream)
{
    GCM_ABI_TRY
        if (!ctx)
            return fail(GCM_E_ARG, "gcm_autotune: NULL context");
        if (key_len != 16 && key_len != 24 && key_len != 32)
            return fail(GCM_E_KEYLEN, "gcm_autotune: key length %u", key_len);
        if (len == 0 || len > kMaxLen)
            return fail(GCM_E_ARG, "gcm_autotune: len must be in 1..2^36-32");
        if (reps == 0)
            reps = 3;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        std::lock_guard<std::mutex> g(ctx->mu);
        hipError_t e = hipSetDevice(ctx->device);
        if (e != hipSuccess)
            return fail_hip(e, "hipSetDevice");

        // scratch: payload in/out + workspace sized for the smallest tile
        const uint64_t m = ghash_blocks(0, len);
        const uint64_t ws_bytes = workspace_bytes_for((m + 63) / 64, 1);
        const uint64_t pay = (len + 255) / 256 * 256;
        const uint64_t bytes = 2 * pay + ws_bytes + 256;
        uint8_t *buf = nullptr;
        int rc = ctx_alloc(ctx, reinterpret_cast<void **>(&buf), bytes);
        if (rc)
            return rc;
        uint8_t *in = buf, *outp = buf + pay, *ws = outp + pay;
        uint8_t *tag = ws + ws_bytes;
        e = hipMemsetAsync(in, 0x5c, len, s);
        uint8_t key[32];
        for (uint32_t i = 0; i < 32; ++i)
            key[i] = (uint8_t)(0x3d * i + 7);
        const uint8_t iv[12] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12};
        uint32_t slot = 0;
        if (e == hipSuccess) {
            rc = register_key_locked(ctx, key, key_len, &slot, s);
            if (rc) {
                ctx_free(ctx, buf, bytes);
                return rc;
            }
        }
        Timer tm;
        if (e == hipSuccess)
            e = tm.init();

        float best_ms = 1e30f;
        TuneEntry best;
        uint32_t tried = 0;
        bool all_equal = true;
        uint8_t ref_tag[16], cur_tag[16];
        bool have_ref = false;
        const bool save_prof = ctx->prof;
        ctx->prof = false;
        auto desc = [&](const Shape &sh) {
            MsgDesc d;
            fill_desc(&d, 0, iv, 0, 0, (uint64_t)in, (uint64_t)outp, len, (uint64_t)tag, 0,
                      (uint64_t)(ctx->d_slots + kSlotBytes * slot), key_len / 4 + 6, sh.log2B, sh.waves, 0);
            return d;
        };
        auto check = [&]() {  // the tag of the last pass
            const hipError_t r = hipMemcpy(cur_tag, tag, 16, hipMemcpyDeviceToHost);
            if (r == hipSuccess && !have_ref) {
                std::memcpy(ref_tag, cur_tag, 16);
                have_ref = true;
            } else if (r == hipSuccess && std::memcmp(ref_tag, cur_tag, 16) != 0) {
                all_equal = false;
            }
            return r;
        };
        auto pass = [&](const Shape &sh) {
            const int r = launch_single(ctx, desc(sh), sh, ws, s);
            rc = rc ? rc : r;
            return r ? hipErrorUnknown : hipSuccess;
        };
        auto time_shape = [&](const Shape &sh, float *ms) {
            hipError_t r = pass(sh);  // warm-up
            if (r == hipSuccess)
                r = tm.add(s, reps, ms, [&] { return pass(sh); });
            return r == hipSuccess ? check() : r;
        };
        for (uint32_t l = 8; l <= 16 && e == hipSuccess; ++l) {
            if ((1ull << l) > 4 * m && l > 8)
                break;  // tiles larger than the whole message add nothing
            for (uint32_t w : kWaveOpts)
                for (uint32_t gpc : gpc_options(w)) {
                    if (e != hipSuccess)
                        break;
                    Shape sh;
                    sh.log2B = l;
                    sh.waves = w;
                    sh.gpc = gpc;
                    float ms = 0.f;
                    e = time_shape(sh, &ms);
                    ++tried;
                    if (e == hipSuccess && ms < best_ms) {
                        best_ms = ms;
                        static_cast<Shape &>(best) = sh;
                    }
                }
        }
        const Shape own = heuristic_shape(ctx, m);
        if (!same(best, own)) {
            ++tried;
            float best_sum = 0.f, own_sum = 0.f;
            for (uint32_t k = 0; k < kTurns && e == hipSuccess; ++k) {
                e = time_shape(own, &own_sum);
                if (e == hipSuccess)
                    e = time_shape(best, &best_sum);
            }
            best.faster = is_faster(best_sum, own_sum);
        }
        // The tree over single partials, which whole-message launches do without
        // but streams and the host pipeline end with, at every fan-in.
        if (e == hipSuccess) {
            const Shape &used = best.faster ? static_cast<const Shape &>(best) : own;
            const MsgDesc d = desc(used);
            rc = launch_tile_range(ctx, d, used, ws, s);
            e = rc ? hipErrorUnknown : hipSuccess;
            float least = 1e30f, sum[4] = {0.f, 0.f, 0.f, 0.f};
            for (uint32_t k = 0; k <= kTurns && e == hipSuccess; ++k)
                for (uint32_t f = 0; f < 4 && e == hipSuccess; ++f) {
                    float ms = 0.f;
                    e = tm.add(s, reps, &ms, [&] {
                        return launch_combine(nullptr, 1, &d, ws + workspace_counter_bytes(1), kFaninOpts[f], s);
                    });
                    if (k)
                        sum[f] += ms;  // the first round is the warm-up
                    else if (e == hipSuccess)
                        e = check();
                }
            for (uint32_t f = 0; f < 4; ++f)
                if (sum[f] < least) {
                    least = sum[f];
                    best.fanin = kFaninOpts[f];
                }
        }
        ctx->prof = save_prof;
        (void)hipStreamSynchronize(s);
        ctx->slot_used[slot] = 0;
        ctx_free(ctx, buf, bytes);
        if (rc)
            return rc;
        if (e != hipSuccess)
            return fail_hip(e, "autotune");
        if (!all_equal)
            return fail(GCM_E_INTERNAL, "autotune: launch shapes disagree on the tag (geometry dependence)");
        ctx->tuned[(uint64_t)key_len << 32 | size_bucket(len)] = best;
        if (out) {
            std::memset(out, 0, sizeof *out);
            out->log2_tile_blocks = best.log2B;
            out->waves_per_group = best.waves;
            out->candidates = tried;
            out->best_ms = best_ms;
            out->gbs = (double)len / (best_ms * 1e-3) / 1e9;
            out->groups_per_cu = best.gpc;
            out->combine_fanin = best.fanin;
        }
        return GCM_OK;
    GCM_ABI_CATCH
}

extern "C" int gcm_batch_autotune(gcm_ctx *ctx, const gcm_job *jobs, uint32_t n, uint8_t *base_d, uint64_t base_bytes,
                                  uint32_t reps, gcm_tune_result *out, void *stream)
{
    GCM_ABI_TRY
        if (!ctx || (n && (!jobs || !base_d)))
            return fail(GCM_E_ARG, "gcm_batch_autotune: NULL argument");
        if (n == 0)
            return fail(GCM_E_ARG, "gcm_batch_autotune: empty batch");
        if ((uintptr_t)base_d & 255)
            return fail(GCM_E_ARG, "gcm_batch_autotune: base_d must be 256-byte aligned");
        // every point reruns the batch, so it must leave its inputs intact
        for (uint32_t i = 0; i < n; ++i)
            if (jobs[i].len && jobs[i].in_off == jobs[i].out_off)
                return fail(GCM_E_ARG, "gcm_batch_autotune: job %u runs in place (a rerun would read its output)",
                            i);
        if (reps == 0)
            reps = 3;
        hipStream_t s = reinterpret_cast<hipStream_t>(stream);
        std::lock_guard<std::mutex> g(ctx->mu);
        hipError_t e = hipSetDevice(ctx->device);
        if (e != hipSuccess)
            return fail_hip(e, "hipSetDevice");
        uint64_t payload = 0;
        for (uint32_t i = 0; i < n; ++i)
            payload += jobs[i].len;

        // results of every point: tags (16 B) and, for decrypts, flags (4 B)
        std::vector<uint8_t> ref(20ull * n), cur(20ull * n);
        auto fetch = [&](std::vector<uint8_t> &dst) -> hipError_t {
            hipError_t r = hipStreamSynchronize(s);
            for (uint32_t i = 0; i < n && r == hipSuccess; ++i) {
                r = hipMemcpy(dst.data() + 20ull * i, base_d + jobs[i].tag_off, 16, hipMemcpyDeviceToHost);
                if (r == hipSuccess && jobs[i].op == 1)
                    r = hipMemcpy(dst.data() + 20ull * i + 16, base_d + jobs[i].ok_off, 4, hipMemcpyDeviceToHost);
            }
            return r;
        };
        Timer tm;
        e = tm.init();
        if (e != hipSuccess)
            return fail_hip(e, "hipEventCreate");
        std::vector<PlanMsg> msgs(n);
        {
            const SlotView sv = slot_view(ctx);
            PlanError err;
            for (uint32_t i = 0; i < n; ++i) {
                if (check_job(jobs[i], i, base_bytes, sv, &err))
                    return plan_error(err);
                msgs[i] = plan_msg_from_job(jobs[i], (uint64_t)base_d);
            }
        }
        uint32_t tried = 0;
        bool have_ref = false, all_equal = true;
        int rc = GCM_OK;
        const bool save_prof = ctx->prof;
        ctx->prof = false;
        auto time_shape = [&](const Shape &sh, float *ms) {
            gcm_batch *b = nullptr;
            rc = batch_create_locked(ctx, jobs, n, base_d, base_bytes, &sh, &b);
            if (rc)
                return hipErrorUnknown;
            hipError_t r = batch_enqueue(b, s);  // warm-up
            if (r == hipSuccess)
                r = tm.add(s, reps, ms, [&] { return batch_enqueue(b, s); });
            if (r == hipSuccess)
                r = fetch(have_ref ? cur : ref);
            batch_free_locked(b);
            if (r != hipSuccess)
                return r;
            if (!have_ref)
                have_ref = true;
            else if (cur != ref)
                all_equal = false;
            ++tried;
            return r;
        };
        // every shape and the planner's own in every turn, so that a shape is not
        // chosen for a moment in which the clock was high
        std::vector<TuneEntry> shapes;
        for (uint32_t w : kWaveOpts)
            for (uint32_t gpc : gpc_options(w))
                for (uint32_t cap = 8; cap <= 12; ++cap) {
                    TuneEntry t;
                    t.log2B = cap;
                    t.waves = w;
                    t.gpc = gpc;
                    shapes.push_back(t);
                }
        Shape own = batch_rule(ctx, msgs.data(), n, true);
        std::vector<float> sum(shapes.size(), 0.f);
        float own_sum = 0.f;
        for (uint32_t k = 0; k < kTurns && e == hipSuccess; ++k) {
            e = time_shape(own, &own_sum);
            if (rc == GCM_E_NOMEM && k == 0) {  // as gcm_batch_create does
                rc = GCM_OK;
                own = batch_rule(ctx, msgs.data(), n, false);
                e = time_shape(own, &own_sum);
            }
            for (size_t q = 0; q < shapes.size() && e == hipSuccess; ++q)
                e = time_shape(shapes[q], &sum[q]);
        }
        const size_t at = std::min_element(sum.begin(), sum.end()) - sum.begin();
        TuneEntry best = shapes[at];
        const float best_ms = sum[at] / (float)kTurns;
        best.faster = is_faster(sum[at], own_sum);
        ctx->prof = save_prof;
        if (rc)
            return rc;
        if (e != hipSuccess)
            return fail_hip(e, "batch autotune");
        if (!all_equal)
            return fail(GCM_E_INTERNAL, "batch autotune: launch shapes disagree on a tag or flag (geometry dependence)");
        ctx->tuned_batch[(uint64_t)size_bucket(n) << 32 | size_bucket(payload)] = best;
        if (out) {
            std::memset(out, 0, sizeof *out);
            out->log2_tile_blocks = best.log2B;
            out->waves_per_group = best.waves;
            out->candidates = tried;
            out->best_ms = best_ms;
            out->gbs = (double)payload / (best_ms * 1e-3) / 1e9;
            out->groups_per_cu = best.gpc;
            out->combine_fanin = best.fanin;
        }
        return GCM_OK;
    GCM_ABI_CATCH
}

// Cache file: {"arch": ..., "entries": [...], "batch_entries": [...]}, each
// entry four size/shape integers, the groups per CU, the fan-in, and whether the
// shape was faster than the planner's own (which a file may lack: it was).
extern "C" int gcm_autotune_save(gcm_ctx *ctx, const char *path)
{
    GCM_ABI_TRY
        if (!ctx || !path)
            return fail(GCM_E_ARG, "gcm_autotune_save: NULL argument");
        std::lock_guard<std::mutex> g(ctx->mu);
        hipDeviceProp_t p;
        if (hipGetDeviceProperties(&p, ctx->device) != hipSuccess)
            std::strcpy(p.gcnArchName, "unknown");
        FILE *f = std::fopen(path, "w");
        if (!f)
            return fail(GCM_E_ARG, "gcm_autotune_save: cannot open %s", path);
        std::fprintf(f, "{\"arch\": \"%s\", \"entries\": [", p.gcnArchName);
        bool first = true;
        for (auto &kv : ctx->tuned) {
            std::fprintf(f,
                         "%s{\"key_bytes\": %u, \"len_log2\": %u, \"log2_tile_blocks\": %u, \"waves\": %u, "
                         "\"groups_per_cu\": %u, \"fanin\": %u, \"faster\": %u}",
                         first ? "" : ", ", (uint32_t)(kv.first >> 32), (uint32_t)(kv.first & 0xffffffffu),
                         kv.second.log2B, kv.second.waves, kv.second.gpc, kv.second.fanin, kv.second.faster ? 1u : 0u);
            first = false;
        }
        std::fprintf(f, "], \"batch_entries\": [");
        first = true;
        for (auto &kv : ctx->tuned_batch) {
            std::fprintf(f,
                         "%s{\"msgs_log2\": %u, \"payload_log2\": %u, \"tile_cap_log2\": %u, \"waves\": %u, "
                         "\"groups_per_cu\": %u, \"fanin\": %u, \"faster\": %u}",
                         first ? "" : ", ", (uint32_t)(kv.first >> 32), (uint32_t)(kv.first & 0xffffffffu),
                         kv.second.log2B, kv.second.waves, kv.second.gpc, kv.second.fanin, kv.second.faster ? 1u : 0u);
            first = false;
        }
        std::fprintf(f, "]}\n");
        std::fclose(f);
        return GCM_OK;
    GCM_ABI_CATCH
}

static bool valid_entry(unsigned lt, unsigned wv, unsigned gp, unsigned fi)
{
    return lt >= 6 && lt <= 20 && (wv == 8 || wv == 12 || wv == 16) && gp >= 1 && gp <= 64 && valid_fanin(fi);
}

static TuneEntry tune_entry(uint32_t log2B, uint32_t waves, uint32_t gpc, uint32_t fanin, uint32_t faster)
{
    TuneEntry t;
    t.log2B = log2B, t.waves = waves, t.gpc = gpc, t.fanin = fanin, t.faster = faster != 0;
    return t;
}

// Minimal reader for the format gcm_autotune_save writes; a cache for another
// architecture is rejected as a whole.
extern "C" int gcm_autotune_load(gcm_ctx *ctx, const char *path)
{
    GCM_ABI_TRY
        if (!ctx || !path)
            return fail(GCM_E_ARG, "gcm_autotune_load: NULL argument");
        FILE *f = std::fopen(path, "r");
        if (!f)
            return fail(GCM_E_ARG, "gcm_autotune_load: cannot open %s", path);
        std::string text;
        char buf[4096];
        size_t n;
        while ((n = std::fread(buf, 1, sizeof buf, f)) > 0)
            text.append(buf, n);
        std::fclose(f);
        hipDeviceProp_t p;
        if (hipGetDeviceProperties(&p, ctx->device) != hipSuccess)
            return fail(GCM_E_HIP, "gcm_autotune_load: device query failed");
        if (text.find(std::string("\"arch\": \"") + p.gcnArchName + "\"") == std::string::npos)
            return fail(GCM_E_ARG, "gcm_autotune_load: cache is for another architecture");
        std::lock_guard<std::mutex> g(ctx->mu);
        size_t pos = 0;
        uint32_t loaded = 0;
        while ((pos = text.find("{\"key_bytes\":", pos)) != std::string::npos) {
            unsigned kb, ll, lt, wv, gp, fi, fa = 1;
            if (std::sscanf(text.c_str() + pos,
                            "{\"key_bytes\": %u, \"len_log2\": %u, \"log2_tile_blocks\": %u, \"waves\": %u, "
                            "\"groups_per_cu\": %u, \"fanin\": %u, \"faster\": %u}",
                            &kb, &ll, &lt, &wv, &gp, &fi, &fa) >= 6 &&
                (kb == 16 || kb == 24 || kb == 32) && ll < 64 && valid_entry(lt, wv, gp, fi)) {
                ctx->tuned[(uint64_t)kb << 32 | ll] = tune_entry(lt, wv, gp, fi, fa);
                ++loaded;
            }
            ++pos;
        }
        pos = 0;
        while ((pos = text.find("{\"msgs_log2\":", pos)) != std::string::npos) {
            unsigned nl, pl, lt, wv, gp, fi, fa = 1;
            if (std::sscanf(text.c_str() + pos,
                            "{\"msgs_log2\": %u, \"payload_log2\": %u, \"tile_cap_log2\": %u, \"waves\": %u, "
                            "\"groups_per_cu\": %u, \"fanin\": %u, \"faster\": %u}",
                            &nl, &pl, &lt, &wv, &gp, &fi, &fa) >= 6 &&
                nl < 64 && pl < 64 && valid_entry(lt, wv, gp, fi)) {
                ctx->tuned_batch[(uint64_t)nl << 32 | pl] = tune_entry(lt, wv, gp, fi, fa);
                ++loaded;
            }
            ++pos;
        }
        return loaded ? GCM_OK : fail(GCM_E_ARG, "gcm_autotune_load: no entries in %s", path);
    GCM_ABI_CATCH
}
