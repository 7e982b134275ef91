// Host side of libkvq: configuration checks, byte-budget accounting, shrink policies (Sec. 3.1), the page
// allocator over the caller's arena, device table maintenance and the C ABI declared in include/kvq.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <cstdlib>
#include <limits>
#include <memory>
#include <new>
#include <vector>

#include "../../include/kvq.h"
#include "kvq_internal.h"
#include "kvq_ring.h"

namespace {

constexpr int kMaxOrder = 4;  // allocation blocks of 1, 2, 4, 8, 16 units; a unit is one metadata block
constexpr int kRingSegments = 4;
constexpr uint64_t kRingSegmentBytes = 1u << 20;  // the pinned staging ring: 4 segments of 1 MiB
constexpr uint64_t kNoSum = 0x7ff0dead0000beefull;  // a signalling NaN

// Markers of the staging ring: one HIP event per segment, recorded on the cache's stream.
struct RingEvents {
    hipEvent_t ev[kRingSegments] = {};
    hipStream_t stream = nullptr;
    bool record(int i) { return hipEventRecord(ev[i], stream) == hipSuccess; }
    bool wait(int i) { return hipEventSynchronize(ev[i]) == hipSuccess; }
};

int order_of_bits(int bits) { return bits == 16 ? 4 : bits == 8 ? 3 : bits == 4 ? 2 : 1; }
// Kernel time of one 2/4/8/16-bit tile, measured, in units of which a workgroup does 1,000 in 0.9 us.
constexpr int kTileTime[4] = {100, 145, 250, 300};
bool valid_bits(int b) { return b == 16 || b == 8 || b == 4 || b == 2; }

// A set of numbers below n that finds its smallest: a bit for each, and a bit per word of the level below on the levels above.
class NumberSet {
public:
    bool init(uint64_t n, bool full) {
        levels_.clear();
        for (uint64_t bits = n;;) {
            const uint64_t words = std::max<uint64_t>(1, (bits + 63) / 64);
            levels_.emplace_back(static_cast<uint64_t*>(std::calloc(words, sizeof(uint64_t))));  // (pages of zeros cost nothing until written)
            if (!levels_.back()) return false;
            if (full) {
                std::memset(levels_.back().get(), 0xff, (size_t)(bits / 64) * sizeof(uint64_t));
                if (bits % 64) levels_.back()[(size_t)(bits / 64)] = (1ull << (bits % 64)) - 1;
            }
            if (words == 1) return true;
            bits = words;
        }
    }
    bool empty() const { return levels_.back()[0] == 0; }
    uint32_t smallest() const {
        uint64_t i = 0;
        for (size_t l = levels_.size(); l-- > 0;) i = i * 64 + (uint64_t)__builtin_ctzll(levels_[l][i]);
        return (uint32_t)i;
    }
    bool has(uint32_t i) const { return levels_[0][i / 64] >> (i % 64) & 1; }
    void add(uint32_t i) {
        for (auto& words : levels_) {
            const uint64_t old = words[i / 64];
            words[i / 64] = old | 1ull << (i % 64);
            if (old) return;
            i /= 64;
        }
    }
    void remove(uint32_t i) {
        for (auto& words : levels_) {
            if (words[i / 64] &= ~(1ull << (i % 64))) return;
            i /= 64;
        }
    }

private:
    struct Free { void operator()(uint64_t* p) const { std::free(p); } };
    std::vector<std::unique_ptr<uint64_t[], Free>> levels_;
};

// Buddy allocator in units.  Code blocks need 2^order units (2-bit: 2, 4-bit: 4, 8-bit: 8, 16-bit: 16),
// metadata blocks one unit, so every size is a power of two and freed space coalesces without compaction.
// (With the free blocks in std::set a prompt of 16,000 tokens that is shrunk twice spent 55 of the host's 137 us here, and more than a
// launch takes on most calls.)
class Buddy {
public:
    bool init(uint32_t n_super) {
        for (int o = 0; o <= kMaxOrder; ++o)
            if (!free_[o].init((uint64_t)n_super << (kMaxOrder - o), o == kMaxOrder)) return false;
        free_units_ = (uint64_t)n_super << kMaxOrder;
        return true;
    }
    bool alloc(int order, uint32_t* off) {
        int o = order;
        while (o <= kMaxOrder && free_[o].empty()) ++o;
        if (o > kMaxOrder) return false;
        uint32_t blk = free_[o].smallest();
        free_[o].remove(blk);
        blk <<= o;
        while (o > order) {
            --o;
            free_[o].add((blk >> o) + 1);
        }
        free_units_ -= 1u << order;
        *off = blk;
        return true;
    }
    void release(uint32_t off, int order) {
        free_units_ += 1u << order;
        uint32_t blk = off >> order;
        while (order < kMaxOrder && free_[order].has(blk ^ 1)) {
            free_[order].remove(blk ^ 1);
            blk >>= 1;
            ++order;
        }
        free_[order].add(blk);
    }
    uint64_t free_units() const { return free_units_; }

private:
    NumberSet free_[kMaxOrder + 1];
    uint64_t free_units_ = 0;
};

struct Page {
    int bits = 16;
    int n = 0;              // tokens stored
    uint32_t code_unit = 0; // allocation offsets in units
    uint32_t meta_unit = 0; // valid when the page has metadata (bits < 16, or the integer 16-bit tier)
};

struct Run {  // neighbouring pages of one width
    int page_end, bits;
};

struct Layer {
    uint64_t budget = 0;
    int fbit = 2;
    int T = 0;
    bool reparam = false;  // keys stored as K / lambda, queries multiplied by lambda (Sec. 3.3)
    bool poisoned = false; // an enqueue failed after the host tables had been updated: unusable until kvq_cache_reset
    std::vector<Page> pages;
    // the pages as runs of one width, of the state runs_version; see runs_of
    mutable std::vector<Run> runs;
    mutable uint64_t runs_version = ~0ull;
    // what the split count was worked out from and the count itself; split plan cache of kvq_decode_attention
    uint64_t count_key[3] = {};
    int count_splits = 1;
    int plan_tiles = -1, plan_splits = 0;
    bool plan_side_by_side = false;
    uint64_t version = 0, plan_version = ~0ull;
    int32_t split_begin[KVQ_MAX_SPLITS + 1];
};

}  // namespace

struct kvq_cache {
    kvq_config_t cfg;
    int units = 0, tpp = 0, gqa = 0, max_pages = 0;
    bool dry = false;
    uint8_t* arena = nullptr;
    uint64_t arena_bytes = 0;
    uint64_t unit_bytes = 0;
    uint64_t table_off = 0, jobs_off = 0, part_o_off = 0, part_ml_off = 0, counters_off = 0, flags_off = 0, pages_off = 0;
    uint64_t reparam_off = 0;  // per block: lambda [n_kv_heads][128] fp32, then 1 / lambda
    uint32_t v_epoch = 4;      // see KvqVMark; 0 is what a cleared word holds
    uint32_t v_turn = 1;       // tag of the next launch that appends below 16 bits, above the epoch; see kvq_v_marked
    KvqVMark v_mark() const { return KvqVMark{reinterpret_cast<uint32_t*>(arena + flags_off), v_epoch}; }
    Buddy buddy;
    std::vector<Layer> layers;
    uint8_t* ring = nullptr;
    uint8_t* ring_dev = nullptr;  // the same pinned memory as the device addresses it
    KvqStagingRing<RingEvents, kRingSegments> ring_ctl;
    RingEvents ring_events;
    uint64_t* sums = nullptr;   // behind the ring: 2 sums for each workgroup of the error kernel, kNoSum between calls
    bool sums_at_rest = false;
    bool device_ready = false;
    bool enqueue_failed = false;  // a block was left unusable since the device's counters were last cleared
    int splits_override = 0;
    int fused_merge = 1;
    int deterministic = 0;
    int shift_strategy = KVQ_SHIFT_EQUIVALENT;  // how 2b -> b steps treat codes, S and Z (Sec. 4.3.1)
    int tier16 = KVQ_TIER16_FP16;               // what a 16-bit token is: raw fp16, or 16-bit codes with (S, Z)
    bool int16() const { return tier16 == KVQ_TIER16_INT16; }
    bool has_meta(int bits) const { return bits < 16 || int16(); }
    int tile_cost[4] = {kTileTime[0], kTileTime[1], kTileTime[2], kTileTime[3]};  // KVQ_OPT_TILE_COST_*
    int target_workgroups = 256;

    uint64_t bpth(int bits) const {
        return kvq_bytes_per_token_head(bits, cfg.head_dim, cfg.group, cfg.count_metadata_in_budget, int16() ? 1 : 0);
    }
    uint64_t unit_off_bytes(uint32_t unit) const { return pages_off + (uint64_t)unit * unit_bytes; }
    KvqPageDesc desc(const Page& p) const {
        KvqPageDesc d;
        d.code_off256 = (uint32_t)(unit_off_bytes(p.code_unit) / 256);
        d.meta_off256 = has_meta(p.bits) ? (uint32_t)(unit_off_bytes(p.meta_unit) / 256) : 0u;
        d.bits = (uint32_t)p.bits;
        d.int16 = (p.bits == 16 && int16()) ? 1u : 0u;
        return d;
    }
    float* lambda_dev(int layer) const {  // lambda of the block; its reciprocals follow
        return reinterpret_cast<float*>(arena + reparam_off) + (size_t)layer * 2 * cfg.n_kv_heads * KVQ_D;
    }
    KvqPageDesc* table_dev(int layer) const {
        return reinterpret_cast<KvqPageDesc*>(arena + table_off) + (size_t)layer * max_pages;
    }
};

namespace {

struct Regions {
    uint64_t table_off, jobs_off, part_o_off, part_ml_off, counters_off, flags_off, reparam_off, pages_off;
};
uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }

bool check_config(const kvq_config_t* c) {
    if (!c) return false;
    if (c->n_layers < 1 || c->batch < 1 || c->n_kv_heads < 1 || c->n_q_heads < 1) return false;
    if (c->head_dim != KVQ_D || (c->group != 32 && c->group != 64 && c->group != 128)) return false;
    if (c->n_q_heads % c->n_kv_heads != 0 || c->n_q_heads / c->n_kv_heads > KVQ_MAX_GQA) return false;
    if (c->page_tokens < 32 || c->page_tokens % 32 != 0 || c->page_tokens > 32768) return false;
    if (c->max_tokens < 1 || c->max_tokens > (1 << 26)) return false;  // tile indices stay below 2^21 (exact magic division)
    if (c->window < 0 || c->window % c->page_tokens != 0) return false;
    if (c->n_sink < 0 || c->n_sink % c->page_tokens != 0) return false;
    if (c->policy != KVQ_POLICY_PAPER && c->policy != KVQ_POLICY_OLDEST_FIRST) return false;
    if ((int64_t)c->batch * c->n_kv_heads > 65535) return false;
    return true;
}

Regions layout_regions(const kvq_config_t* c) {
    Regions r;
    uint64_t units = (uint64_t)c->batch * c->n_kv_heads;
    uint64_t max_pages = ((uint64_t)c->max_tokens + c->page_tokens - 1) / c->page_tokens;
    uint64_t off = 0;
    r.table_off = off;     off = align_up(off + (uint64_t)c->n_layers * max_pages * sizeof(KvqPageDesc), 256);
    r.jobs_off = off;      off = align_up(off + max_pages * sizeof(KvqRequantJob), 256);
    r.part_o_off = off;    off = align_up(off + units * KVQ_MAX_SPLITS * 16 * KVQ_D * sizeof(float), 256);
    r.part_ml_off = off;   off = align_up(off + units * KVQ_MAX_SPLITS * 32 * sizeof(float), 256);
    r.counters_off = off;  off = align_up(off + units * KVQ_COUNTER_STRIDE * sizeof(uint32_t), 256);
    r.flags_off = off;     off = align_up(off + 64, 256);
    r.reparam_off = off;   off = align_up(off + (uint64_t)c->n_layers * 2 * c->n_kv_heads * KVQ_D * sizeof(float), 256);
    r.pages_off = align_up(off, 4096);
    return r;
}

hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }

// Copy `bytes` of host data to device memory in stream order through the pinned staging ring (in pieces of at most
// one ring segment).  The host waits only if it is a whole ring ahead of the device.
kvq_status_t upload(kvq_cache* c, void* dst_dev, const void* src, uint64_t bytes, hipStream_t s) {
    c->ring_events.stream = s;
    const uint8_t* from = static_cast<const uint8_t*>(src);
    uint8_t* to = static_cast<uint8_t*>(dst_dev);
    while (bytes) {
        const uint64_t n = std::min<uint64_t>(bytes, c->ring_ctl.segment_bytes());
        const int64_t at = c->ring_ctl.reserve(c->ring_events, n, 64);
        if (at < 0) return KVQ_E_HIP;
        std::memcpy(c->ring + at, from, n);
        if (hipMemcpyAsync(to, c->ring + at, n, hipMemcpyHostToDevice, s) != hipSuccess) return KVQ_E_HIP;
        from += n; to += n; bytes -= n;
    }
    return KVQ_OK;
}

// Place `bytes` of host data (at most one ring segment) in the pinned staging ring and return where (a host address
// the device can read as well); the space is not reused before the work enqueued on s after this call has completed.
kvq_status_t stage(kvq_cache* c, const void* src, uint64_t bytes, hipStream_t s, const void** where) {
    if (bytes == 0 || bytes > c->ring_ctl.segment_bytes()) return KVQ_E_INVALID;
    c->ring_events.stream = s;
    const int64_t at = c->ring_ctl.reserve(c->ring_events, bytes, 256);
    if (at < 0) return KVQ_E_HIP;
    std::memcpy(c->ring + at, src, bytes);
    *where = c->ring_dev + at;
    return KVQ_OK;
}

kvq_status_t ensure_device(kvq_cache* c, hipStream_t s) {
    if (c->dry || c->device_ready) return KVQ_OK;
    // counters and flags are adjacent regions: one fill clears both
    if (kvq_launch_fill_u32(reinterpret_cast<uint32_t*>(c->arena + c->counters_off), 0u,
                            (size_t)((c->flags_off + 64 - c->counters_off) / sizeof(uint32_t)), s) != hipSuccess)
        return KVQ_E_HIP;
    c->device_ready = true;
    return KVQ_OK;
}

kvq_status_t upload_table(kvq_cache* c, int layer, int first, int last, hipStream_t s) {
    if (c->dry || last <= first) return KVQ_OK;
    std::vector<KvqPageDesc> d((size_t)(last - first));
    for (int i = first; i < last; ++i) d[(size_t)(i - first)] = c->desc(c->layers[(size_t)layer].pages[(size_t)i]);
    return upload(c, c->table_dev(layer) + first, d.data(), d.size() * sizeof(KvqPageDesc), s);
}

// Accounting and launch plans look at widths only, of which a block of thousands of pages has a few runs.  An append extends them, a page that goes
// down makes them stale.  (131,000 tokens in pages of 32, a step a launch: looking at every page cost the host 7 of 31 us.)
const std::vector<Run>& runs_of(const Layer& L) {
    if (L.runs_version != L.version) {
        L.runs.clear();
        for (size_t i = 0; i < L.pages.size(); ++i) {
            if (L.runs.empty() || L.runs.back().bits != L.pages[i].bits) L.runs.push_back(Run{(int)i + 1, L.pages[i].bits});
            else L.runs.back().page_end = (int)i + 1;
        }
        L.runs_version = L.version;
    }
    return L.runs;
}

// (every page but the last is full)
uint64_t bytes_used(const kvq_cache* c, const Layer& L) {
    uint64_t u = 0;
    int64_t t = 0;
    for (const Run& r : runs_of(L)) {
        const int64_t end = std::min<int64_t>((int64_t)r.page_end * c->cfg.page_tokens, L.T);
        u += (uint64_t)(end - t) * c->units * c->bpth(r.bits);
        t = end;
    }
    return u;
}

// Width of the block's bulk: smallest width among pages after the sink (16 if there is none).
int current_bits(const kvq_cache* c, const Layer& L) {
    const int first = c->cfg.n_sink / c->cfg.page_tokens;
    int b = 16;
    for (const Run& r : runs_of(L))
        if (r.page_end > first) b = std::min(b, r.bits);
    return b;
}

// Sink pages and pages overlapping the most recent `window` tokens are never lowered.
bool is_protected(const kvq_cache* c, int T, int page) {
    const int P = c->cfg.page_tokens;
    if (page < c->cfg.n_sink / P) return true;
    return c->cfg.window > 0 && (int64_t)(page + 1) * P > (int64_t)T - c->cfg.window;
}

struct Lowering {  // one page to lower and the blocks allocated for it
    int page, from, to;
    uint32_t new_code = 0, new_meta = 0;
};

// Allocate destination blocks for a set of lowerings (a metadata block too when the source page has none); on
// failure release what was taken.
bool alloc_lowerings(kvq_cache* c, std::vector<Lowering>& low) {
    for (size_t i = 0; i < low.size(); ++i) {
        bool ok = c->buddy.alloc(order_of_bits(low[i].to), &low[i].new_code);
        bool ok2 = true;
        if (ok && !c->has_meta(low[i].from)) ok2 = c->buddy.alloc(0, &low[i].new_meta);
        if (!ok || !ok2) {
            if (ok) c->buddy.release(low[i].new_code, order_of_bits(low[i].to));
            for (size_t k = 0; k < i; ++k) {
                c->buddy.release(low[k].new_code, order_of_bits(low[k].to));
                if (!c->has_meta(low[k].from)) c->buddy.release(low[k].new_meta, 0);
            }
            return false;
        }
    }
    return true;
}

// Pages of the integer 16-bit tier go down one halving at a time; raw fp16 pages reach any width in one step.
bool lowers_in_steps(const kvq_cache* c, const std::vector<Lowering>& low) {
    return !low.empty() && c->int16() && low[0].from == 16 && low[0].to < 8;
}

// Destination blocks of the first step of run_lowerings, taken ahead of it (so that a caller can find out that the
// arena is full before it changes anything), and their release when that caller gives up.  A later step of a chain
// cannot run out of blocks: each step has just freed a larger block per page than the next one takes.
bool alloc_first_step(kvq_cache* c, std::vector<Lowering>& low) {
    if (low.empty()) return true;
    const int to = low[0].to;
    const bool steps = lowers_in_steps(c, low);
    if (steps) for (auto& w : low) w.to = 8;
    const bool ok = alloc_lowerings(c, low);
    if (steps) for (auto& w : low) w.to = to;
    return ok;
}
void release_first_step(kvq_cache* c, std::vector<Lowering>& low) {
    const bool steps = lowers_in_steps(c, low);
    for (auto& w : low) {
        c->buddy.release(w.new_code, order_of_bits(steps ? 8 : w.to));
        if (!c->has_meta(w.from)) c->buddy.release(w.new_meta, 0);
    }
}

// Enqueue the kernel for lowerings that all share (from, to) -- one halving, or fp16 values to any width -- then
// commit the host tables.  allocated: the destination blocks are in `low` already.
kvq_status_t run_lowering_step(kvq_cache* c, int layer, std::vector<Lowering>& low, hipStream_t s, bool allocated = false) {
    if (low.empty()) return KVQ_OK;
    Layer& L = c->layers[(size_t)layer];
    const int from = low[0].from, to = low[0].to;
    const bool fresh_meta = !c->has_meta(from);  // raw fp16 pages carry no metadata yet
    if (!allocated && !alloc_lowerings(c, low)) return KVQ_E_OOM;
    if (!c->dry) {
        std::vector<KvqRequantJob> jobs(low.size());
        for (size_t i = 0; i < low.size(); ++i) {
            const Page& p = L.pages[(size_t)low[i].page];
            jobs[i].src_code_off256 = (uint32_t)(c->unit_off_bytes(p.code_unit) / 256);
            jobs[i].dst_code_off256 = (uint32_t)(c->unit_off_bytes(low[i].new_code) / 256);
            jobs[i].meta_off256 = (uint32_t)(c->unit_off_bytes(fresh_meta ? low[i].new_meta : p.meta_unit) / 256);
            jobs[i].tiles_page = kvq_job_tiles_page((p.n + KVQ_TILE_TOKENS - 1) / KVQ_TILE_TOKENS, low[i].page);
        }
        KvqRequantJob* jd = reinterpret_cast<KvqRequantJob*>(c->arena + c->jobs_off);
        const bool by_arg = jobs.size() <= (size_t)KVQ_JOBS_BY_ARG;  // short lists ride in the kernel arguments
        kvq_status_t st = by_arg ? KVQ_OK : upload(c, jd, jobs.data(), jobs.size() * sizeof(KvqRequantJob), s);
        hipError_t e = hipSuccess;
        if (st == KVQ_OK) {
            const KvqRequantJob* jh = by_arg ? jobs.data() : nullptr;
            e = fresh_meta ? kvq_launch_quant16(to, c->arena, c->table_dev(layer), jd, jh, (int)jobs.size(), c->tpp, c->units, c->v_mark(), c->cfg.group, s)
                             : kvq_launch_shrink(to, c->shift_strategy, c->arena, c->table_dev(layer), jd, jh, (int)jobs.size(), c->tpp, c->units, c->v_mark(), s);
        }
        if (st != KVQ_OK || e != hipSuccess) {
            for (auto& w : low) {
                c->buddy.release(w.new_code, order_of_bits(w.to));
                if (fresh_meta) c->buddy.release(w.new_meta, 0);
            }
            return st != KVQ_OK ? st : KVQ_E_HIP;
        }
    }
    for (auto& w : low) {
        Page& p = L.pages[(size_t)w.page];
        c->buddy.release(p.code_unit, order_of_bits(p.bits));  // reused only by work enqueued later
        p.code_unit = w.new_code;
        if (fresh_meta) p.meta_unit = w.new_meta;
        p.bits = to;
    }
    L.version++;
    return KVQ_OK;
}

// Lower a set of pages that share (from, to).  Pages of the integer 16-bit tier go down one halving at a time
// (16 -> 8 -> 4 -> 2 by the configured shift strategy); raw fp16 pages are quantized to the target width directly.
// first_allocated: alloc_first_step has been called on `low`.
kvq_status_t run_lowerings(kvq_cache* c, int layer, std::vector<Lowering>& low, hipStream_t s, bool first_allocated = false) {
    if (low.empty()) return KVQ_OK;
    const int to = low[0].to;
    if (!lowers_in_steps(c, low)) return run_lowering_step(c, layer, low, s, first_allocated);
    for (int b = 8; b >= to; b /= 2) {
        const bool have = first_allocated && b == 8;
        for (auto& w : low) {
            w.from = 2 * b;
            w.to = b;
            if (!have) w.new_code = w.new_meta = 0;
        }
        kvq_status_t st = run_lowering_step(c, layer, low, s, have);
        if (st != KVQ_OK) return st;  // the pages stay at the width they reached
    }
    return KVQ_OK;
}

void build_segments(const kvq_cache* c, const Layer& L, std::vector<kvq_segment_info_t>& out) {
    const int P = c->cfg.page_tokens;
    out.clear();
    for (size_t i = 0; i < L.pages.size(); ++i) {
        int t0 = (int)i * P, t1 = t0 + L.pages[i].n;
        if (!out.empty() && out.back().bits == L.pages[i].bits) out.back().token_end = t1;
        else out.push_back(kvq_segment_info_t{t0, t1, L.pages[i].bits});
    }
}

// Index of a width in kTileTime and tile_cost (the narrow widths are bound by de-quantization work, the wide ones by their
// bytes).
int cost_index(int bits) { return bits == 16 ? 3 : bits == 8 ? 2 : bits == 4 ? 1 : 0; }

// Tiles of the longest of n ranges of the same number of tiles, as plan_splits cuts them for the kernels for short ranges.
int longest_even(int n_tiles, int n, int tpp) {
    const int k = (n_tiles + n - 1) / n;
    return n > 1 && tpp % 2 == 0 ? (k + 1) & ~1 : k;
}
// Ranges of about the same sum of cost[cost_index(width)], none of more than `most` tiles, written to split_begin.
void cut_by_cost(const kvq_cache* c, Layer& L, int n_tiles, int n_splits, const uint64_t (&costs)[4], int most) {
    const int tpp = c->tpp;
    const std::vector<Run>& runs = runs_of(L);
    const auto tiles_to = [&](const Run& r) { return (int)std::min<int64_t>((int64_t)r.page_end * tpp, n_tiles); };
    uint64_t total = 0;
    int done = 0;
    for (const Run& r : runs) {
        total += (uint64_t)(tiles_to(r) - done) * costs[cost_index(r.bits)];
        done = tiles_to(r);
    }
    int sp = 1;
    L.split_begin[0] = 0;
    uint64_t cum = 0;
    done = 0;
    for (size_t i = 0; i < runs.size() && sp < n_splits; ++i) {
        const int nt = tiles_to(runs[i]) - done;
        if (nt <= 0) break;
        const uint64_t cost = costs[cost_index(runs[i].bits)], run_end = cum + cost * (uint64_t)nt;
        while (sp < n_splits) {
            uint64_t target = (total * sp + n_splits - 1) / n_splits;
            if (target > run_end) break;
            uint64_t k = target <= cum ? 0 : (target - cum + cost - 1) / cost;
            if ((tpp & 1) == 0) k = std::min<uint64_t>((k + 1) & ~1ull, (uint64_t)nt);  // chunks are tile pairs
            int64_t at = std::min<int64_t>((int64_t)done + (int64_t)k, (int64_t)L.split_begin[sp - 1] + most);
            int64_t least = n_tiles - (int64_t)(n_splits - sp) * most;  // (what the later ranges can take)
            if ((tpp & 1) == 0) least = (least + 1) & ~1ll;
            at = std::max(at, least);
            // at least one tile is left for every later range: what this cuts off an even boundary is a range of one tile
            L.split_begin[sp] = (int)std::min<int64_t>(at, n_tiles - (n_splits - sp));
            ++sp;
        }
        cum = run_end;
        done += nt;
    }
    while (sp <= n_splits) L.split_begin[sp++] = n_tiles;
}
int longest_of(const Layer& L, int n_splits) {
    int longest = 0;
    for (int i = 0; i < n_splits; ++i) longest = std::max(longest, L.split_begin[i + 1] - L.split_begin[i]);
    return longest;
}

// Split of the tile range (n_splits <= n_tiles, or one split of nothing), balanced by tile costs.  The last range is never empty: the
// workgroup that holds the last tile is the one that stores the token a launch appends, behind its own reads of that tile.
// side_by_side: a light launch for the kernels for short ranges, which take a range's tiles side by side, so that how many there are counts
// beside how wide they are: every tile costs as much as a 16-bit one more, and no range gets a tile more for a SIMD than equal ones
// would have (4 x 1,024 tokens of 2, 4, 8 and 16 bits x 2 units in 32 splits 7.2 us without this and 6.7).  Forty drawn blocks of
// several widths, best of all split counts, with 0, 60, 120, 200, 300, 500 and infinitely many of the default units more: 3.9, 2.0, 1.6, 1.1, 0.9,
// 0.9 and 0.9 % slower on average than the best of these.
void plan_splits(kvq_cache* c, Layer& L, int n_tiles, int n_splits, bool side_by_side) {
    if (L.plan_tiles == n_tiles && L.plan_splits == n_splits && L.plan_side_by_side == side_by_side && L.plan_version == L.version) return;
    L.plan_tiles = n_tiles;
    L.plan_splits = n_splits;
    L.plan_side_by_side = side_by_side;
    L.plan_version = L.version;
    uint64_t costs[4];
    const uint64_t more = side_by_side ? (uint64_t)c->tile_cost[3] : 0u;
    for (int i = 0; i < 4; ++i) costs[i] = (uint64_t)c->tile_cost[i] + more;
    cut_by_cost(c, L, n_tiles, n_splits, costs, side_by_side ? (longest_even(n_tiles, n_splits, c->tpp) + 3) & ~3 : n_tiles);
}

}  // namespace

extern "C" {

uint64_t kvq_bytes_per_token_head(int32_t bits, int32_t head_dim, int32_t group, int32_t count_metadata,
                                  int32_t int16_tier) {
    if (!valid_bits(bits) || head_dim <= 0 || group <= 0) return 0;
    uint64_t n = 2ull * head_dim * bits / 8;
    if (count_metadata && (bits < 16 || int16_tier)) n += 2ull * (head_dim / group) * 4;
    return n;
}

uint64_t kvq_arena_bytes(const kvq_config_t* cfg, uint64_t payload_bytes) {
    if (!check_config(cfg)) return 0;
    Regions r = layout_regions(cfg);
    uint64_t super = (32ull * cfg->page_tokens * cfg->batch * cfg->n_kv_heads) << kMaxOrder;
    return r.pages_off + align_up(payload_bytes, super);
}

kvq_status_t kvq_cache_create(const kvq_config_t* cfg, const uint64_t* block_budget_bytes_host,
                              const uint8_t* block_fbit_host, void* arena_dev, uint64_t arena_bytes,
                              kvq_cache_t** out) {
    if (!out) return KVQ_E_INVALID;
    *out = nullptr;
    if (!check_config(cfg) || !block_budget_bytes_host || !block_fbit_host) return KVQ_E_INVALID;
    for (int i = 0; i < cfg->n_layers; ++i)
        if (!valid_bits(block_fbit_host[i])) return KVQ_E_INVALID;
    if (arena_dev && (reinterpret_cast<uintptr_t>(arena_dev) & 255u)) return KVQ_E_INVALID;
    kvq_cache* c = new (std::nothrow) kvq_cache();
    if (!c) return KVQ_E_OOM;
    c->cfg = *cfg;
    c->units = cfg->batch * cfg->n_kv_heads;
    c->tpp = cfg->page_tokens / KVQ_TILE_TOKENS;
    c->gqa = cfg->n_q_heads / cfg->n_kv_heads;
    c->max_pages = (cfg->max_tokens + cfg->page_tokens - 1) / cfg->page_tokens;
    c->dry = (arena_dev == nullptr);
    c->arena = static_cast<uint8_t*>(arena_dev);
    c->arena_bytes = arena_bytes;
    c->unit_bytes = 32ull * cfg->page_tokens * c->units;
    Regions r = layout_regions(cfg);
    c->table_off = r.table_off; c->jobs_off = r.jobs_off; c->part_o_off = r.part_o_off;
    c->part_ml_off = r.part_ml_off; c->counters_off = r.counters_off; c->flags_off = r.flags_off; c->pages_off = r.pages_off;
    c->reparam_off = r.reparam_off;
    uint64_t super = c->unit_bytes << kMaxOrder;
    if (arena_bytes < c->pages_off + super) { delete c; return KVQ_E_OOM; }
    uint64_t n_super = (arena_bytes - c->pages_off) / super;
    if ((c->pages_off + n_super * super) / 256 > 0xffffffffull) { delete c; return KVQ_E_INVALID; }
    if (!c->buddy.init((uint32_t)n_super)) { delete c; return KVQ_E_OOM; }
    c->layers.resize((size_t)cfg->n_layers);
    for (int i = 0; i < cfg->n_layers; ++i) {
        c->layers[(size_t)i].budget = block_budget_bytes_host[i];
        c->layers[(size_t)i].fbit = block_fbit_host[i];
    }
    if (!c->dry) {
        c->ring_ctl.init(kRingSegmentBytes);
        // (coherent: the host reads sums while the kernel that stores them runs)
        if (hipHostMalloc(reinterpret_cast<void**>(&c->ring), c->ring_ctl.total_bytes() + 2 * KVQ_ERR_MAX_WGS * sizeof(uint64_t),
                          hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
            delete c;
            return KVQ_E_HIP;
        }
        for (int i = 0; i < kRingSegments; ++i) {
            if (hipEventCreateWithFlags(&c->ring_events.ev[i], hipEventDisableTiming) != hipSuccess) {
                for (int k = 0; k < i; ++k) (void)hipEventDestroy(c->ring_events.ev[k]);
                (void)hipHostFree(c->ring);
                delete c;
                return KVQ_E_HIP;
            }
        }
        if (hipHostGetDevicePointer(reinterpret_cast<void**>(&c->ring_dev), c->ring, 0) != hipSuccess) {
            for (int i = 0; i < kRingSegments; ++i) (void)hipEventDestroy(c->ring_events.ev[i]);
            (void)hipHostFree(c->ring);
            delete c;
            return KVQ_E_HIP;
        }
        c->sums = reinterpret_cast<uint64_t*>(c->ring + c->ring_ctl.total_bytes());
        std::fill_n(c->sums, 2 * KVQ_ERR_MAX_WGS, kNoSum);
        c->sums_at_rest = true;
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess &&
            prop.multiProcessorCount > 0)
            c->target_workgroups = prop.multiProcessorCount;  // one 8-wavefront workgroup per compute unit
    }
    *out = c;
    return KVQ_OK;
}

void kvq_cache_destroy(kvq_cache_t* c) {
    if (!c) return;
    if (c->ring) {
        (void)hipHostFree(c->ring);
        for (int i = 0; i < kRingSegments; ++i) (void)hipEventDestroy(c->ring_events.ev[i]);
    }
    delete c;
}

}  // extern "C"

namespace {

// What a deferred single-token append leaves for the attention launch to do.
struct DeferredAppend {
    bool active = false;
    int t_old = 0;
    int fresh_page = -1;  // the page the token starts, whose table entry the launch writes; -1: the page exists
    KvqPageDesc desc{};
};

// Bookkeeping of an append, worked out without touching the cache: entry width, tokens and pages afterwards, the window pages
// the append evicts and the width they go to.
struct AppendPlan {
    int e = 16, T = 0, n_pages = 0, bcur = 16;
    std::vector<int> evicted;
};

kvq_status_t plan_append(const kvq_cache_t* c, int32_t layer, int32_t n_new, int32_t entry_bits, AppendPlan& pl) {
    const Layer& L = c->layers[(size_t)layer];
    const kvq_config_t& cfg = c->cfg;
    const int P = cfg.page_tokens;
    if (L.poisoned) return KVQ_E_STATE;
    if ((int64_t)L.T + n_new > cfg.max_tokens) return KVQ_E_STATE;
    int e = entry_bits;
    if (e == 0) e = (cfg.policy == KVQ_POLICY_OLDEST_FIRST || cfg.window > 0) ? 16 : current_bits(c, L);
    if (L.T % P != 0 && L.pages.back().bits != e) return KVQ_E_STATE;
    const bool evict = entry_bits == 0 && cfg.policy == KVQ_POLICY_PAPER && cfg.window > 0;
    pl.e = e;
    const int T = pl.T = L.T + n_new;
    pl.n_pages = (int)(((int64_t)T + P - 1) / P);
    pl.evicted.clear();
    pl.bcur = 16;
    uint64_t used = bytes_used(c, L) + (uint64_t)n_new * c->units * c->bpth(e);
    if (evict) pl.bcur = current_bits(c, L);  // (the new pages have 16 bits)
    if (pl.bcur < 16) {
        const int first = cfg.n_sink / P;
        int i = std::max((int)L.pages.size(), first);
        while (i > first && L.pages[(size_t)i - 1].bits == 16) --i;  // start of the trailing 16-bit run
        for (; i < pl.n_pages && (int64_t)T - (int64_t)i * P >= (int64_t)cfg.window + P; ++i) {
            pl.evicted.push_back(i);
            used -= (uint64_t)P * c->units * (c->bpth(16) - c->bpth(pl.bcur));
        }
    }
    if (used > L.budget) return KVQ_E_BUDGET;
    return KVQ_OK;
}

bool append_args_ok(const kvq_cache_t* c, int32_t layer, const void* k_dev, const void* v_dev, int32_t n_new,
                    int32_t entry_bits) {
    if (!c || layer < 0 || layer >= c->cfg.n_layers || n_new < 0 || n_new >= KVQ_MAX_APPEND_TOKENS) return false;
    if (entry_bits != 0 && !valid_bits(entry_bits)) return false;
    if (n_new > 0 && !c->dry && (!k_dev || !v_dev)) return false;
    return true;
}

// What a planned append takes from the arena: its new pages, and the pages that leave the window in this call with the
// blocks they are lowered into behind the append.  All of it is taken before anything changes, so that a full arena can
// still be reported with nothing changed.
struct AppendBlocks {
    std::vector<Page> fresh;
    std::vector<Lowering> low;
};

void release_fresh(kvq_cache_t* c, AppendBlocks& bl) {
    for (Page& p : bl.fresh) {
        c->buddy.release(p.code_unit, order_of_bits(p.bits));
        if (c->has_meta(p.bits)) c->buddy.release(p.meta_unit, 0);
    }
    bl.fresh.clear();
}
void release_append(kvq_cache_t* c, AppendBlocks& bl) {
    release_first_step(c, bl.low);
    release_fresh(c, bl);
}

// Takes the blocks of a planned append; on an error none is held.
kvq_status_t reserve_append(kvq_cache_t* c, int32_t layer, const AppendPlan& pl, AppendBlocks& bl, hipStream_t s) {
    for (int i = (int)c->layers[(size_t)layer].pages.size(); i < pl.n_pages; ++i) {
        Page p;
        p.bits = pl.e;
        const bool ok = c->buddy.alloc(order_of_bits(p.bits), &p.code_unit);
        if (!ok || (c->has_meta(p.bits) && !c->buddy.alloc(0, &p.meta_unit))) {
            if (ok) c->buddy.release(p.code_unit, order_of_bits(p.bits));
            release_fresh(c, bl);
            return KVQ_E_OOM;
        }
        bl.fresh.push_back(p);
    }
    for (int i : pl.evicted) bl.low.push_back(Lowering{i, 16, pl.bcur});
    if (!alloc_first_step(c, bl.low)) {
        release_fresh(c, bl);
        return KVQ_E_OOM;
    }
    const kvq_status_t st = ensure_device(c, s);
    if (st != KVQ_OK) release_append(c, bl);
    return st;
}

// Carries a planned append out whose blocks have been taken.  defer != nullptr: a one-token append into the 16-bit tier, with
// defer_narrow into any width, is not launched but described in *defer.  The caller must then launch the attention with it, or mark the block unusable: the
// token, and the table entry of a page that it starts, are written by that launch and by nothing else.
kvq_status_t commit_append(kvq_cache_t* c, int32_t layer, const AppendPlan& pl, AppendBlocks& bl, const void* k_dev,
                           const void* v_dev, int32_t n_new, const float* cos_sin_dev, hipStream_t s, DeferredAppend* defer,
                           bool defer_narrow) {
    Layer& L = c->layers[(size_t)layer];
    const int P = c->cfg.page_tokens, e = pl.e;
    const size_t old_pages = L.pages.size();
    std::vector<Lowering>& low = bl.low;
    kvq_status_t st = KVQ_OK;
    const int t_old = L.T, T = pl.T;
    for (const Page& p : bl.fresh) L.pages.push_back(p);
    for (size_t i = (size_t)(t_old / P); i < L.pages.size(); ++i) L.pages[i].n = std::min(P, T - (int)i * P);
    L.T = T;
    if (L.runs_version == L.version && !L.runs.empty() && L.runs.back().bits == e) {  // new pages have the width e
        L.runs.back().page_end = (int)L.pages.size();
        L.runs_version = L.version + 1;
    }
    L.version++;
    // From here on the host tables count the new tokens: a failing enqueue leaves the block unusable (poisoned).
    if (!c->dry && defer && n_new == 1 && (e == 16 || defer_narrow)) {
        defer->active = true;
        defer->t_old = t_old;
        defer->desc = c->desc(L.pages[(size_t)(t_old / P)]);
        defer->fresh_page = t_old % P == 0 ? t_old / P : -1;
    } else if (!c->dry) {
        const int pg0 = t_old / P, pg1 = (T - 1) / P;
        KvqAppendPages pages;
        pages.n = pg1 - pg0 + 1 <= KVQ_APPEND_ARG_PAGES ? pg1 - pg0 + 1 : 0;
        pages.first_page = pg0;
        pages.fresh = (int)old_pages - pg0;
        pages.bits = (uint32_t)e;
        pages.int16 = (e == 16 && c->int16()) ? 1u : 0u;
        for (int i = 0; i < pages.n; ++i) {
            const KvqPageDesc d = c->desc(L.pages[(size_t)(pg0 + i)]);
            pages.code_off256[i] = d.code_off256;
            pages.meta_off256[i] = d.meta_off256;
        }
        if (pages.n == 0) {  // too many for the kernel arguments: the table is uploaded and read
            st = upload_table(c, layer, (int)old_pages, (int)L.pages.size(), s);
            if (st != KVQ_OK) {
                release_first_step(c, low);
                L.poisoned = true;
                return st;
            }
        }
        if (kvq_launch_append(e, c->arena, c->table_dev(layer), k_dev, v_dev, t_old, n_new, c->tpp, c->units,
                              pages, c->v_mark(), c->cfg.group,
                              L.reparam ? c->lambda_dev(layer) + c->cfg.n_kv_heads * KVQ_D : nullptr, c->cfg.n_kv_heads,
                              cos_sin_dev, c->int16(), s) != hipSuccess) {
            release_first_step(c, low);
            L.poisoned = true;
            return KVQ_E_HIP;
        }
    }
    if (!low.empty()) {
        st = run_lowerings(c, layer, low, s, true);
        if (st != KVQ_OK) { L.poisoned = true; return st; }  // the plan counted these pages at their new width
    }
    return KVQ_OK;
}

kvq_status_t append_impl(kvq_cache_t* c, int32_t layer, const void* k_dev, const void* v_dev, int32_t n_new,
                         int32_t entry_bits, const float* cos_sin_dev, void* hip_stream, DeferredAppend* defer) {
    if (!append_args_ok(c, layer, k_dev, v_dev, n_new, entry_bits)) return KVQ_E_INVALID;
    if (n_new == 0) return KVQ_OK;
    AppendPlan pl;
    AppendBlocks bl;
    kvq_status_t st = plan_append(c, layer, n_new, entry_bits, pl);
    if (st == KVQ_OK) st = reserve_append(c, layer, pl, bl, as_stream(hip_stream));
    if (st != KVQ_OK) return st;
    return commit_append(c, layer, pl, bl, k_dev, v_dev, n_new, cos_sin_dev, as_stream(hip_stream), defer, true);
}

}  // namespace

extern "C" {

kvq_status_t kvq_quantize_append(kvq_cache_t* c, int32_t layer, const void* k_dev, const void* v_dev,
                                 int32_t n_new, int32_t entry_bits, void* hip_stream) {
    return append_impl(c, layer, k_dev, v_dev, n_new, entry_bits, nullptr, hip_stream, nullptr);
}

kvq_status_t kvq_quantize_append_rope(kvq_cache_t* c, int32_t layer, const void* k_dev, const void* v_dev,
                                      int32_t n_new, int32_t entry_bits, const float* cos_sin_dev, void* hip_stream) {
    return append_impl(c, layer, k_dev, v_dev, n_new, entry_bits, cos_sin_dev, hip_stream, nullptr);
}

kvq_status_t kvq_progressive_requant(kvq_cache_t* c, int32_t layer, int32_t segment, int32_t reserve_tokens,
                                     void* hip_stream, int32_t* n_pages_done) {
    if (n_pages_done) *n_pages_done = 0;
    if (!c || layer < 0 || layer >= c->cfg.n_layers || segment < -1 || reserve_tokens < 0) return KVQ_E_INVALID;
    Layer& L = c->layers[(size_t)layer];
    const kvq_config_t& cfg = c->cfg;
    const int P = cfg.page_tokens;
    if (L.poisoned) return KVQ_E_STATE;
    hipStream_t s = as_stream(hip_stream);
    kvq_status_t st = ensure_device(c, s);
    if (st != KVQ_OK) return st;

    if (segment >= 0) {
        std::vector<kvq_segment_info_t> segs;
        build_segments(c, L, segs);
        if (segment >= (int)segs.size()) return KVQ_E_STATE;
        const kvq_segment_info_t sg = segs[(size_t)segment];
        if (sg.bits == 2) return KVQ_E_STATE;
        // A run that ends in the partly filled last page: lowering it would leave that page at a width other than the
        // one the policy appends at (16 bits under OLDEST_FIRST or with a window), and no token could follow.
        if (sg.token_end == L.T && L.T % P != 0 && (cfg.policy == KVQ_POLICY_OLDEST_FIRST || cfg.window > 0))
            return KVQ_E_STATE;
        std::vector<Lowering> low;
        for (int i = sg.token_begin / P; i < (sg.token_end + P - 1) / P; ++i) low.push_back(Lowering{i, sg.bits, sg.bits / 2});
        st = run_lowerings(c, layer, low, s);
        if (st == KVQ_OK && n_pages_done) *n_pages_done = (int32_t)low.size();
        return st;
    }
    if (cfg.policy == KVQ_POLICY_PAPER) {
        const int bcur = current_bits(c, L);
        if (bcur <= L.fbit) return KVQ_E_BUDGET;
        std::vector<Lowering> low;
        for (int i = 0; i < (int)L.pages.size(); ++i)
            if (L.pages[(size_t)i].bits == bcur && !is_protected(c, L.T, i)) low.push_back(Lowering{i, bcur, bcur / 2});
        if (low.empty()) return KVQ_E_BUDGET;
        st = run_lowerings(c, layer, low, s);
        if (st == KVQ_OK && n_pages_done) *n_pages_done = (int32_t)low.size();
        return st;
    }
    // OLDEST_FIRST
    const uint64_t need = (uint64_t)reserve_tokens * c->units * c->bpth(16);
    int done = 0;
    while (bytes_used(c, L) + need > L.budget) {
        int pick = -1;
        for (int i = cfg.n_sink / P; i < (int)L.pages.size(); ++i) {
            const Page& p = L.pages[(size_t)i];
            if (p.bits > L.fbit && p.n == P && (int64_t)(i + 1) * P <= (int64_t)L.T - cfg.window) { pick = i; break; }
        }
        if (pick < 0) { if (n_pages_done) *n_pages_done = done; return KVQ_E_BUDGET; }
        std::vector<Lowering> low{Lowering{pick, L.pages[(size_t)pick].bits, L.pages[(size_t)pick].bits / 2}};
        st = run_lowerings(c, layer, low, s);
        if (st != KVQ_OK) { if (n_pages_done) *n_pages_done = done; return st; }
        ++done;
    }
    if (n_pages_done) *n_pages_done = done;
    return KVQ_OK;
}

}  // extern "C"

namespace {

// What the block's tiles cost by the weights of KVQ_OPT_TILE_COST_* (relative, in a scale the caller chooses) and what they take
// the attention kernel (in units of kTileTime), how many of them are 2 and 16 bits wide, and the bytes of one (sequence, KV head).
struct TileCensus {
    int n2 = 0, n16 = 0, n_all = 0;
    int narrowest = 0, widest = 0;  // the least and the most time of a tile
    uint64_t cost = 0, time = 0, bytes = 0;
};
TileCensus tile_census(const kvq_cache_t* c, Layer& L, int n_tiles) {
    TileCensus t;
    for (const Run& r : runs_of(L)) {
        const int nt = (int)std::min<int64_t>((int64_t)r.page_end * c->tpp, n_tiles) - t.n_all, b = r.bits;
        if (nt <= 0) break;
        t.n_all += nt;
        t.narrowest = t.narrowest ? std::min(t.narrowest, kTileTime[cost_index(b)]) : kTileTime[cost_index(b)];
        t.widest = std::max(t.widest, kTileTime[cost_index(b)]);
        if (b == 2) t.n2 += nt;
        if (b == 16) t.n16 += nt;
        t.cost += (uint64_t)nt * (uint64_t)c->tile_cost[cost_index(b)];
        t.time += (uint64_t)nt * (uint64_t)kTileTime[cost_index(b)];
        t.bytes += (uint64_t)nt * (2u * kvq_tile_code_bytes(b) + (c->has_meta(b) ? KVQ_META_TILE_BYTES : 0u));
    }
    return t;
}

// Tiles of the longest of n ranges of the same time.
uint64_t longest_range(const TileCensus& t, int n) {
    const uint64_t per = (uint64_t)n * (uint64_t)std::max(t.narrowest, 1);
    return std::min<uint64_t>((t.time + per - 1) / per, (uint64_t)t.n_all);
}
// Loads of partial outputs a thread of the split merge issues for n splits, in the steps that merge_splits has.
int merge_loads(int gqa, int n) {
    const int groups = std::max(1, std::min(16 / gqa, n)), rounds = (n + groups - 1) / groups;
    for (int k : {2, 4, 8, 12, 16})
        if (rounds <= k) return k;
    return 16 + (rounds - 16 + 7) / 8 * 8;
}
// Splits of one (sequence, KV head) that take least, at most max_splits: as many as make ranges of some 1, 2, 4, ... tiles, or
// max_splits.  A launch whose splits are short is a chain of latencies; what the split count changes of it, in us, tile times in units
// of 1,000:
//   the range    of up to 16 tiles: 0.25 x its time, for every further tile of a SIMD (beyond 4, 8, 12) 0.05 + 2.8 x a tile's time -- the
//                first time the widest tile's, then the mean one's -- and 0.2 beyond 12; of more tiles, which are streamed: 2.6,
//                0.57 per eight tiles and 0.26 x its time
//   the merge    2.0 (behind streamed ranges 1.8) for publishing, ticket and the last workgroup's trip to memory, 0.007 (0.004) per
//                split (tickets on one counter come in turn), twice that beyond 64, 0.16 (0.14) per load a thread issues, 0.7 (0.77) for
//                every further round of eight beyond 16, and 0.35 behind short ranges that take more than half of the compute
//                units (more than eight query heads per KV head leave one slot group, which loads 16 splits a round: beyond 16
//                splits a range of such a unit keeps 16 tiles, 512 tiles of 16 bits x 1 unit 12.6 in 32 and 13.2 in 48)
// Up to eight tiles, and up to 12 unless they are wide, one workgroup takes all.
// Fitted to launches of 1, 2, 4, ... 128 units of 3 to 4,000 tiles (2, 4 or 8 bits with four tiles of 16, all of 16, 2 / 4 / 16) in 1 to
// 128 splits, 1 to 8 query heads per KV head, over blocks in turn from memory: 600 shapes.  How much slower the choice is than the best
// count tried, on average, with the model for byte planes below, ranges cut by cost, and with this one, cut as plan_splits does: up to
// 12 tiles 1.6 and 0.5 %, 13 to 16 4.9 and 1.1, 17 to 64 3.4 and 1.2, 65 to 256 3.5 and 0.8, beyond 3.8 and 1.4.  64 units x 12 tiles of 4 bits 7.8 us in four splits and 5.9 in one,
// 16 x 32 of 2, 4 and 16 bits 7.7 in 12 and 6.9 in eight, 1 x 320 of 4 bits 9.6 in 52 and 8.5 in 32.
int planned_splits(const kvq_cache* c, const TileCensus& t, int n_tiles, int max_splits) {
    max_splits = std::max(1, std::min(max_splits, std::min(n_tiles, KVQ_MAX_SPLITS)));
    if (n_tiles <= 8 || max_splits == 1) return 1;
    if (16 / c->gqa == 1) max_splits = std::min(max_splits, std::max(16, (n_tiles + 15) / 16));
    const double total = 1e-3 * (double)t.time, mean = total / n_tiles;
    if (n_tiles <= 12 && mean <= 0.25) return 1;
    const double first = 0.05 + 2.8e-3 * t.widest, next = 0.05 + 2.8 * mean;
    int best = 1;
    double least = 0.0;
    for (int range : {0, 256, 192, 128, 96, 64, 48, 40, 32, 24, 20, 16, 14, 12, 10, 8, 7, 6, 5, 4, 3, 2, 1}) {
        int n = range ? (n_tiles + range - 1) / range : 1;
        const bool most = range == 1 || n >= max_splits;
        if (most) n = max_splits;
        const int tiles = longest_even(n_tiles, n, c->tpp);
        const bool few = tiles <= KVQ_SHORT_TILES;
        double us = few ? first * (tiles > 4) + next * ((tiles > 8) + (tiles > 12)) + 0.2 * (tiles > 12) + 0.25 * total / n
                        : 2.6 + 0.57 / 8 * tiles + 0.26 * total / n;
        if (n > 1) {
            const int loads = merge_loads(c->gqa, n), more = std::max(0, loads - 16) / 8, per = n + std::max(0, n - 64);
            us += few ? 2.0 + 0.007 * per + 0.16 * std::min(loads, 16) + 0.7 * more + (2 * n * c->units > c->target_workgroups ? 0.35 : 0.0)
                      : 1.8 + 0.004 * per + 0.14 * std::min(loads, 16) + 0.77 * more;
        }
        if (range == 0 || us < least) { least = us; best = n; }
        if (most && range) break;
    }
    return best;
}

// The same for a block of byte planes, whose tiles hold a wavefront up so long that ranges are better cut by time: as many splits as
// make ranges of some 4, 8, 16, ... tiles, or max_splits.  A launch whose splits are short is a chain of latencies; what the split count changes of it, in us:
//   the range    0.7 per 1,000 units of its tile time (what a compute unit needs to fetch and expand its tiles), and 0.8 for
//                every eight tiles beyond the first (the wavefronts take another one)
//   the merge    1.8 for publishing, ticket and the last workgroup's trip to memory, 0.02 per split (tickets on one counter come
//                in turn), 0.06 per load a thread issues, 0.7 for every further round of eight beyond 16
// Fitted to launches of 1, 2, 4, ... 128 units of 8 to 1,024 tiles at each width in 1 to 64 splits (5 query heads per KV head;
// 320 launches, when a further round took a little longer than now): the choice is 1.1 % slower than the best count tried, 14 % at
// worst.
int planned_splits_planes(const kvq_cache* c, const TileCensus& t, int n_tiles, int max_splits) {
    max_splits = std::max(1, std::min(max_splits, std::min(n_tiles, KVQ_MAX_SPLITS)));
    int best = 1;
    double least = 0.0;
    for (int range : {0, 256, 128, 64, 32, 24, 16, 8, 4, 1}) {
        int n = range ? std::max(1, (int)longest_range(t, range)) : 1;  // (the two are each other's quotient)
        const bool most = range == 1 || n >= max_splits;
        if (most) n = max_splits;
        double us = 0.7e-3 * (double)t.time / n + 0.8 * ((int)(longest_range(t, n) + 7) / 8 - 1);
        if (n > 1) {
            const int loads = merge_loads(c->gqa, n);
            us += 1.8 + 0.02 * n + 0.06 * loads + (loads > 16 ? 0.7 * ((loads - 16) / 8) : 0.0);
        }
        if (range == 0 || us < least) { least = us; best = n; }
        if (most && range) break;
    }
    return best;
}

// Most splits of one (sequence, KV head) that pay in a batch, most of whose launches stream their ranges: none up to 20
// tiles, beyond that sqrt(time / 80), or one per 16 tiles for a unit or two by themselves (max_wgs / 2) as long as the
// merge issues all its loads in one round.  More than eight query heads per KV head leave the merge one slot group, which loads
// 16 splits a round: beyond 16 splits a range of such a unit keeps 16 tiles.  A count a little above the 16 of every slot group,
// which cost one round of the merge's loads, is brought down to it.
// Measured in launches of one cache on the streaming kernels with the merge they had then (us): 10 tiles 6.9 in one split and 8.7 at best
// in several, 20 of 16 bits 9.1 and 9.0, 32 10.3 and 9.5, 24 of mixed widths 9.3 in eight and 11.0 in two, 79 of 16 bits 10.6 in 16 and 11.9
// in five, 128 of 2 bits 10.8 in 12 and 11.5 in eight; 1,000 of 2 bits, 4 heads, one unit 13.2 in 63 and 14.8 in 35, four units 15.2 and 14.9;
// 16 heads, 256 of 16 bits x 8 units 14.3 in 16 and 15.7 in 31; 1,500 of 8 bits x 3 units 15.7 in 64 and 16.3 in 68.  (Ranges of 17 to 20 tiles,
// which this leaves whole, keep a batch from the kernels for short ranges.)
int useful_batch_splits(const kvq_cache* c, uint64_t time, int n_tiles, int max_wgs) {
    if (n_tiles <= 20) return 1;
    const int groups = std::max(1, 16 / c->gqa), per16 = (n_tiles + 15) / 16;
    const int alone = std::min(std::min(per16, 16 * groups), max_wgs / 2 / c->units);
    int n = std::max(alone, (int)std::sqrt((double)time / 80.0));
    if (groups == 1) n = std::min(n, std::max(16, per16));
    if (n > 16 * groups && n <= 20 * groups) n = 16 * groups;
    return std::max(1, std::min(n, std::min(n_tiles, KVQ_MAX_SPLITS)));
}

int tiles_of(int n_tokens) { return (n_tokens + KVQ_TILE_TOKENS - 1) / KVQ_TILE_TOKENS; }
// A token that the launch itself appends is not read from the cache: the tiles of the older ones are split.
int tiles_read(const Layer& L, const DeferredAppend& app) { return tiles_of(app.active ? app.t_old : L.T); }

// Fills the parameter block of one attention launch over block `layer`.  batch_splits > 0: the splits per (sequence, KV
// head) this cache gets in a ragged batch; 0: the whole device serves it.
kvq_status_t fill_attn_params(kvq_cache_t* c, int32_t layer, const void* q_dev, void* out_dev, int32_t out_is_fp32,
                              float softmax_scale, const DeferredAppend* app, const void* k_new, const void* v_new,
                              const float* cos_sin_dev, int batch_splits, KvqAttnParams& p) {
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !q_dev || !out_dev) return KVQ_E_INVALID;
    if (c->dry) return KVQ_E_STATE;
    Layer& L = c->layers[(size_t)layer];
    if (L.T == 0 || L.poisoned) return KVQ_E_STATE;
    const int n_tokens = app && app->active ? app->t_old : L.T;
    const int n_tiles = app ? tiles_read(L, *app) : tiles_of(L.T);
    int n_splits = c->splits_override > 0 ? c->splits_override : batch_splits;
    bool side_by_side = false;
    if (n_splits <= 0) {
        // One workgroup per compute unit when a good part of the tiles is 2 bits wide (those are bound by vector
        // issue and want every unit) or the launch is short (what counts is the length of one range: 8K tokens x 32 units
        // of 4 bits, 43 MB, 15.1 us on all units and 16.5 on three quarters; of 8 bits, 75 MB, 18.5 and 19.1).  A longer
        // launch over wider tiles is bound by HBM, and there three quarters of the units stream measurably faster than all of them
        // (16-bit blocks of 87 to 160 MB 3 to 4 %, 4-, 8- and 16-bit blocks of 350 MB and more 4 to 7 %).  Not every block
        // gains: 32,256 tokens of 8 bits x 16 units (153 MB) take 30.7 us with the 12 splits this gives, 29.6 with 10 or 16
        // and 28.6 with 14, and 8,192 of 16 bits x 16 units (67 MB) 16.1 with 12 or 16: how the ranges divide into rounds of
        // eight tiles weighs as much there.
        const TileCensus t = tile_census(c, L, n_tiles);
        int wgs = c->target_workgroups;
        // Where the splits that three quarters give a unit leave three eighths of the compute units idle or more (39, 49 to 53, 65 to 79
        // and 97 to 128 units), all of them take part.  With three quarters and with all, 4 heads: 39 units x 900 tiles of 4 bits 36.8 and 34.3
        // us, 51 x 700 37.1 and 34.9, 65 x 600 44.1 and 36.5, 76 x 500 38.9 and 36.6, 97 x 400 52.5 and 37.4, 112 x 400 52.7 and 42.9, 128 x 300
        // 41.9 and 37.2; 39 x 200 of 16 bits 24.8 and 24.0, 51 x 150 24.4 and 23.8, 65 x 120 26.4 and 24.4, 76 x 100 24.1 and 23.5, 97 x 80 29.6
        // and 23.6, 112 x 64 25.0 and 22.4, 128 x 64 25.9 and 25.3.
        if (4 * t.n2 < t.n_all && t.bytes * (uint64_t)c->units > 320000ull * (uint64_t)wgs && wgs * 3 / 4 / c->units * c->units * 8 >= wgs * 5)
            wgs = wgs * 3 / 4;
        // (as long as the tiles of each width are as many as last time, and the tier's the same, so are the splits)
        const bool planes = c->int16() && t.n16 > 0;
        const uint64_t key[3] = {t.time, (uint64_t)n_tiles << 32 | (uint32_t)t.n16,
                                 (uint64_t)t.widest << 32 | (uint64_t)planes << 31 | (uint32_t)(wgs / c->units)};
        if (std::memcmp(L.count_key, key, sizeof key) != 0) {
            L.count_splits = (planes ? planned_splits_planes : planned_splits)(c, t, n_tiles, wgs / c->units);
            std::memcpy(L.count_key, key, sizeof key);
        }
        n_splits = L.count_splits;
        // two halves of a range of wide tiles that one workgroup takes in a few rounds stay one, unless they are long reads: 128 units x 20
        // or 24 tiles of 8 bits take the same in one and in two and 32 of them 12.2 and 12.6 us, 24 of 16 bits (393 KB) 11.3 and 10.2, 24 of 2 bits 10.3 and 8.5
        if (n_splits == 2 && n_tiles <= 32 && (planes || t.narrowest >= kTileTime[2]) && t.bytes <= 375000) n_splits = 1;
        // (heavy launches in few splits are better cut by time: 32 units x 2,146 tokens of 8 and 16 bits, 28 MB, in eight splits 10.0 us with
        // ranges of the same cost and 10.8 side by side, 2,042 of 2 and 16 bits, 19 MB, 9.8 and 10.4; in more than 16 splits a unit drawn
        // blocks of 300 and more tiles are 3 % faster side by side on average)
        side_by_side = !planes && (t.bytes * (uint64_t)c->units <= 16000000u || n_splits > 16) && longest_even(n_tiles, n_splits, c->tpp) <= KVQ_SHORT_TILES;
    }
    n_splits = std::max(1, std::min(n_splits, std::min(KVQ_MAX_SPLITS, n_tiles)));
    plan_splits(c, L, n_tiles, n_splits, side_by_side);
    p.short_ranges = longest_of(L, n_splits) <= KVQ_SHORT_TILES ? 1 : 0;

    p.arena = c->arena;
    p.table = c->table_dev(layer);
    p.q = q_dev;
    p.lambda = L.reparam ? c->lambda_dev(layer) : nullptr;
    p.out = out_dev;
    p.part_o = reinterpret_cast<float*>(c->arena + c->part_o_off);
    p.part_ml = reinterpret_cast<float*>(c->arena + c->part_ml_off);
    p.counters = reinterpret_cast<uint32_t*>(c->arena + c->counters_off);
    p.v_mark = c->v_mark().word;
    p.v_tag = c->v_epoch | (app && app->active && app->desc.bits < 16 ? c->v_turn : 0u);
    p.n_tokens = n_tokens;
    p.tiles_per_page = c->tpp;
    p.tpp_magic = c->tpp > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)c->tpp - 1) / (uint64_t)c->tpp) : 0u;
    p.gqa = c->gqa;
    p.n_q_heads = c->cfg.n_q_heads;
    p.n_kv_heads = c->cfg.n_kv_heads;
    p.kv_magic = p.n_kv_heads > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)p.n_kv_heads - 1) / (uint64_t)p.n_kv_heads) : 0u;
    p.n_splits = n_splits;
    p.merge_groups = std::max(1, std::min(16 / c->gqa, n_splits));
    p.merge_rounds = (n_splits + p.merge_groups - 1) / p.merge_groups;
    p.gqa_magic = 65536u / (uint32_t)c->gqa + 1u;
    p.out_fp32 = out_is_fp32 ? 1 : 0;
    p.fused_merge = c->fused_merge;
    p.deterministic = c->deterministic;
    p.int16_tier = c->int16() ? 1 : 0;
    const float scale = softmax_scale != 0.f ? softmax_scale : 1.0f / std::sqrt((float)c->cfg.head_dim);
    p.scale_log2 = scale * 1.44269504088896340736f;
    std::memcpy(p.split_begin, L.split_begin, sizeof(int32_t) * (size_t)(n_splits + 1));
    for (int i = n_splits + 1; i <= KVQ_MAX_SPLITS; ++i) p.split_begin[i] = n_tiles;
    p.app_t_old = -1;
    p.app_page = -1;
    p.app_desc = KvqPageDesc{0, 0, 0, 0};
    p.app_k = p.app_v = nullptr;
    p.app_rope = p.app_rinv = nullptr;
    if (app && app->active) {
        p.app_t_old = app->t_old;
        p.app_desc = app->desc;
        p.app_page = app->fresh_page;
        p.app_k = k_new;
        p.app_v = v_new;
        p.app_rope = cos_sin_dev;
        p.app_rinv = L.reparam ? c->lambda_dev(layer) + c->cfg.n_kv_heads * KVQ_D : nullptr;
    }
    p.app_gspan = c->cfg.group / 32;
    return KVQ_OK;
}

kvq_status_t attention_impl(kvq_cache_t* c, int32_t layer, const void* q_dev, void* out_dev, int32_t out_is_fp32,
                            float softmax_scale, void* hip_stream, const DeferredAppend* app, const void* k_new,
                            const void* v_new, const float* cos_sin_dev) {
    KvqAttnParams p;
    kvq_status_t st = fill_attn_params(c, layer, q_dev, out_dev, out_is_fp32, softmax_scale, app, k_new, v_new,
                                       cos_sin_dev, 0, p);
    if (st != KVQ_OK) return st;
    if (kvq_launch_attention(p, c->units, as_stream(hip_stream)) != hipSuccess) return KVQ_E_HIP;
    if (p.v_tag != c->v_epoch) c->v_turn ^= 3u;
    return KVQ_OK;
}

// One cache's part in dealing a batch's workgroups: the tile time of one of its (sequence, KV head) units, how many units it
// has, the most splits per unit that pay, the splits per unit it gets.
struct BatchShare {
    uint64_t cost;
    int units, max_splits, splits;
};

// The device's workgroups are dealt to the caches so that the most loaded workgroup is as light as possible: every cache
// starts with one split per unit; the cache whose workgroups carry the most tile time gets one more split, as long as the
// workgroups last (and the cache's splits pay).  Every compute unit is used: with ranges of unequal length the heaviest
// workgroup decides the launch time, which outweighs the few percent a block of equal ranges gains from leaving a quarter of
// the units idle.
// The steps of this that make a workgroup lighter which carries more than some load are made in one go for a load at which
// they fit: they all come before the others, and none of them is refused.  (One by one, each step a look at all caches, they
// took longer than the launch: 64 caches of 1,000 tokens 18 of the call's 84 us on the host, 16 of 5,000 tokens 4 of 26.)
void deal_workgroups(std::vector<BatchShare>& share, int wgs) {
    uint64_t load = 0;
    for (BatchShare& c : share) { c.splits = 1; load = std::max(load, c.cost); }
    const auto splits_at = [](const BatchShare& c, uint64_t l) {  // the fewest splits that leave a workgroup no more than l
        return (int)std::min<uint64_t>((uint64_t)c.max_splits, c.cost / (l + 1) + 1);
    };
    const auto used_at = [&](uint64_t l) {
        int64_t used = 0;
        for (const BatchShare& c : share) used += (int64_t)splits_at(c, l) * c.units;
        return used;
    };
    int64_t used = used_at(load);
    if (used > wgs) return;
    if (const int64_t u = used_at(0); u <= wgs) {  // enough for all that pays
        load = 0;
        used = u;
    }
    while (load > 0) {
        const uint64_t less = load - load / 4 - 1;
        const int64_t u = used_at(less);
        if (u > wgs) break;
        load = less;
        used = u;
    }
    std::vector<uint64_t> per_wg(share.size());
    for (size_t i = 0; i < share.size(); ++i) {
        share[i].splits = splits_at(share[i], load);
        per_wg[i] = share[i].cost / (uint64_t)share[i].splits;
    }
    for (;;) {
        size_t pick = share.size();
        uint64_t worst = 0, refused = 0;
        for (size_t i = 0; i < share.size(); ++i) {
            const BatchShare& c = share[i];
            if (c.splits >= c.max_splits) continue;
            if (used + c.units > wgs) refused = std::max(refused, per_wg[i]);
            else if (per_wg[i] > worst) { worst = per_wg[i]; pick = i; }
        }
        // stop once a heavier cache could still be split but no longer fits into the workgroups that are left:
        // more splits elsewhere would not lighten the heaviest workgroup, only add merge work
        if (pick == share.size() || refused > worst) return;
        share[pick].splits++;
        per_wg[pick] = share[pick].cost / (uint64_t)share[pick].splits;
        used += share[pick].units;
    }
}

// The attention launch of a ragged batch over block `layer` of n caches, with the appends deferred to it (k_dev, v_dev and
// cos_sin_dev are looked at for those only).
kvq_status_t batch_attention(kvq_cache_t* const* caches, int32_t n, int32_t layer, const std::vector<DeferredAppend>& app,
                             const void* const* k_dev, const void* const* v_dev, const float* const* cos_sin_dev,
                             const void* const* q_dev, void* const* out_dev, int32_t out_is_fp32, float softmax_scale,
                             hipStream_t s) {
    std::vector<BatchShare> share((size_t)n);
    for (int i = 0; i < n; ++i) {
        kvq_cache_t* c = caches[i];
        Layer& L = c->layers[(size_t)layer];
        if (L.T == 0) return KVQ_E_STATE;
        const int n_tiles = tiles_read(L, app[(size_t)i]);
        const TileCensus t = tile_census(c, L, n_tiles);
        share[(size_t)i] = BatchShare{t.cost, c->units, useful_batch_splits(c, t.time, n_tiles, c->target_workgroups), 1};
    }
    deal_workgroups(share, caches[0]->target_workgroups);
    std::vector<KvqAttnParams> params((size_t)n);
    for (int i = 0; i < n; ++i) {
        kvq_status_t st = fill_attn_params(caches[i], layer, q_dev[i], out_dev[i], out_is_fp32, softmax_scale,
                                           &app[(size_t)i], k_dev ? k_dev[i] : nullptr, v_dev ? v_dev[i] : nullptr,
                                           cos_sin_dev ? cos_sin_dev[i] : nullptr, share[(size_t)i].splits, params[(size_t)i]);
        if (st != KVQ_OK) return st;
    }
    // Parameter blocks of up to 16 caches travel in the kernel arguments.  Those of more the kernel reads straight from the pinned
    // staging ring of the first cache (host memory the device can address): a copy into the arena would be a separate transfer
    // between two kernels on the stream, which costs more than the workgroups' first reads travelling over the host link.
    kvq_cache_t* lead = caches[0];
    const KvqAttnParams* params_dev = nullptr;
    kvq_status_t st = KVQ_OK;
    if (!kvq_batch_fits_args(params.data(), n))
        st = stage(lead, params.data(), params.size() * sizeof(KvqAttnParams), s, reinterpret_cast<const void**>(&params_dev));
    std::vector<int> units((size_t)n);
    for (int i = 0; i < n; ++i) units[(size_t)i] = caches[i]->units;
    if (st == KVQ_OK && kvq_launch_attention_batch(params_dev, params.data(), units.data(), n, s) != hipSuccess) st = KVQ_E_HIP;
    return st;
}

// One attention launch over block `layer` of n caches, optionally with each cache's one-token append in front.
kvq_status_t batch_impl(kvq_cache_t* const* caches, int32_t n, int32_t layer, const void* const* k_dev,
                        const void* const* v_dev, const float* const* cos_sin_dev, const void* const* q_dev,
                        void* const* out_dev, int32_t out_is_fp32, float softmax_scale, void* hip_stream, bool append) {
    if (!caches || n < 1 || n > KVQ_MAX_BATCH_CACHES || !q_dev || !out_dev) return KVQ_E_INVALID;
    if (append && (!k_dev || !v_dev)) return KVQ_E_INVALID;
    for (int i = 0; i < n; ++i) {
        kvq_cache_t* c = caches[i];
        if (!c || layer < 0 || layer >= c->cfg.n_layers || !q_dev[i] || !out_dev[i]) return KVQ_E_INVALID;
        if (append && (!k_dev[i] || !v_dev[i])) return KVQ_E_INVALID;
        if (c->dry) return KVQ_E_STATE;
        if (c->int16() != caches[0]->int16()) return KVQ_E_INVALID;  // one kernel serves one kind of 16-bit tier
        for (int k = 0; k < i; ++k)
            if (caches[k] == c) return KVQ_E_INVALID;
    }
    hipStream_t s = as_stream(hip_stream);
    std::vector<DeferredAppend> app((size_t)n);
    kvq_status_t st = KVQ_OK;
    if (append) {
        // all or nothing: every append is planned and its blocks are taken before the first one is carried out, so that
        // what the host can find out, a full arena too, leaves every cache as it was
        std::vector<AppendPlan> plans((size_t)n);
        std::vector<AppendBlocks> blocks((size_t)n);
        for (int i = 0; i < n; ++i) {
            st = plan_append(caches[i], layer, 1, 0, plans[(size_t)i]);
            if (st != KVQ_OK) return st;
        }
        int held = 0, done = 0;  // caches whose blocks are taken, whose append has been begun
        while (held < n && (st = reserve_append(caches[held], layer, plans[(size_t)held], blocks[(size_t)held], s)) == KVQ_OK) ++held;
        while (st == KVQ_OK && done < n) {
            const int i = done++;
            st = commit_append(caches[i], layer, plans[(size_t)i], blocks[(size_t)i], k_dev[i], v_dev[i], 1,
                               cos_sin_dev ? cos_sin_dev[i] : nullptr, s, &app[(size_t)i], false);
        }
        if (st != KVQ_OK)
            for (int i = done; i < held; ++i) release_append(caches[i], blocks[(size_t)i]);
    }
    if (st == KVQ_OK) st = batch_attention(caches, n, layer, app, k_dev, v_dev, cos_sin_dev, q_dev, out_dev, out_is_fp32, softmax_scale, s);
    if (st != KVQ_OK)  // the host tables count tokens nobody wrote
        for (int i = 0; i < n; ++i)
            if (app[(size_t)i].active) caches[i]->layers[(size_t)layer].poisoned = true;
    return st;
}

}  // namespace

extern "C" {

kvq_status_t kvq_decode_attention(kvq_cache_t* c, int32_t layer, const void* q_dev, void* out_dev,
                                  int32_t out_is_fp32, float softmax_scale, void* hip_stream) {
    return attention_impl(c, layer, q_dev, out_dev, out_is_fp32, softmax_scale, hip_stream, nullptr, nullptr, nullptr,
                          nullptr);
}

kvq_status_t kvq_decode_attention_static(kvq_cache_t* c, int32_t layer, const void* q_dev, void* out_dev,
                                         int32_t out_is_fp32, float softmax_scale, void* hip_stream) {
    KvqAttnParams p;
    kvq_status_t st = fill_attn_params(c, layer, q_dev, out_dev, out_is_fp32, softmax_scale, nullptr, nullptr, nullptr,
                                       nullptr, 0, p);
    if (st != KVQ_OK) return st;
    if (c->units > KVQ_STATIC_MAX_UNITS || (int64_t)c->units * p.n_splits > KVQ_STATIC_MAX_WGS) return KVQ_E_LIMIT;
    unsigned char* scr = nullptr;
    if (kvq_static_scratch(&scr) != hipSuccess) return KVQ_E_HIP;
    hipStream_t s = as_stream(hip_stream);
    p.part_o = reinterpret_cast<float*>(scr);
    p.part_ml = reinterpret_cast<float*>(scr + KVQ_STATIC_PART_O_BYTES);
    p.counters = reinterpret_cast<uint32_t*>(scr + KVQ_STATIC_PART_O_BYTES + KVQ_STATIC_PART_ML_BYTES);
    // The array keeps what the last call left.  Partials are written before they are read; the arrival counters must
    // start at zero (a kernel leaves them there, but a launch that failed half-way would not): a fill kernel, which a
    // caller may also capture into a graph.
    if (p.n_splits > 1 && p.fused_merge &&
        kvq_launch_fill_u32(p.counters, 0u, (size_t)c->units * KVQ_COUNTER_STRIDE, s) != hipSuccess)
        return KVQ_E_HIP;
    return kvq_launch_attention(p, c->units, s) == hipSuccess ? KVQ_OK : KVQ_E_HIP;
}

kvq_status_t kvq_append_decode_attention(kvq_cache_t* c, int32_t layer, const void* k_dev, const void* v_dev,
                                         const float* cos_sin_dev, const void* q_dev, void* out_dev,
                                         int32_t out_is_fp32, float softmax_scale, void* hip_stream) {
    if (!q_dev || !out_dev) return KVQ_E_INVALID;  // nothing may be appended when the attention cannot follow
    if (c && c->dry) return KVQ_E_STATE;
    DeferredAppend app;
    kvq_status_t st = append_impl(c, layer, k_dev, v_dev, 1, 0, cos_sin_dev, hip_stream, &app);
    if (st != KVQ_OK) return st;
    st = attention_impl(c, layer, q_dev, out_dev, out_is_fp32, softmax_scale, hip_stream, &app, k_dev, v_dev, cos_sin_dev);
    if (st != KVQ_OK && app.active) c->layers[(size_t)layer].poisoned = true;  // the host tables count a token nobody wrote
    return st;
}

kvq_status_t kvq_decode_attention_batch(kvq_cache_t* const* caches, int32_t n_caches, int32_t layer,
                                        const void* const* q_dev, void* const* out_dev, int32_t out_is_fp32,
                                        float softmax_scale, void* hip_stream) {
    return batch_impl(caches, n_caches, layer, nullptr, nullptr, nullptr, q_dev, out_dev, out_is_fp32, softmax_scale,
                      hip_stream, false);
}

kvq_status_t kvq_append_decode_attention_batch(kvq_cache_t* const* caches, int32_t n_caches, int32_t layer,
                                               const void* const* k_dev, const void* const* v_dev,
                                               const float* const* cos_sin_dev, const void* const* q_dev,
                                               void* const* out_dev, int32_t out_is_fp32, float softmax_scale,
                                               void* hip_stream) {
    return batch_impl(caches, n_caches, layer, k_dev, v_dev, cos_sin_dev, q_dev, out_dev, out_is_fp32, softmax_scale,
                      hip_stream, true);
}

kvq_status_t kvq_cache_describe(const kvq_cache_t* c, int32_t layer, kvq_segment_info_t* segs_host, int32_t cap,
                                int32_t* n, uint64_t* bytes_used_out, int32_t* n_tokens, int32_t* current_bits_out) {
    if (!c || layer < 0 || layer >= c->cfg.n_layers || cap < 0 || (cap > 0 && !segs_host)) return KVQ_E_INVALID;
    const Layer& L = c->layers[(size_t)layer];
    std::vector<kvq_segment_info_t> segs;
    build_segments(c, L, segs);
    for (int i = 0; i < std::min<int>(cap, (int)segs.size()); ++i) segs_host[i] = segs[(size_t)i];
    if (n) *n = (int32_t)segs.size();
    if (bytes_used_out) *bytes_used_out = bytes_used(c, L);
    if (n_tokens) *n_tokens = L.T;
    if (current_bits_out) *current_bits_out = current_bits(c, L);
    return KVQ_OK;
}

kvq_status_t kvq_cache_export_segment(kvq_cache_t* c, int32_t layer, int32_t segment, int32_t which,
                                      void* codes_host, void* scales_host, void* zeros_host, void* hip_stream) {
    if (!c || layer < 0 || layer >= c->cfg.n_layers || segment < 0 || !codes_host) return KVQ_E_INVALID;
    if (which != KVQ_WHICH_K && which != KVQ_WHICH_V) return KVQ_E_INVALID;
    if (c->dry) return KVQ_E_STATE;
    const Layer& L = c->layers[(size_t)layer];
    if (L.poisoned) return KVQ_E_STATE;
    std::vector<kvq_segment_info_t> segs;
    build_segments(c, L, segs);
    if (segment >= (int)segs.size()) return KVQ_E_STATE;
    const kvq_segment_info_t sg = segs[(size_t)segment];
    const int b = sg.bits, P = c->cfg.page_tokens, tpp = c->tpp;
    const bool meta_out = c->has_meta(b), planes = b == 16 && c->int16();
    if (meta_out && (!scales_host || !zeros_host)) return KVQ_E_INVALID;
    hipStream_t s = as_stream(hip_stream);
    const int n_seg = sg.token_end - sg.token_begin;
    const size_t row_bytes = (size_t)KVQ_D * b / 8;
    const size_t code_block = (size_t)c->unit_bytes * b;
    std::vector<uint8_t> code(code_block), meta(meta_out ? (size_t)c->unit_bytes : 0);
    uint8_t* oc = static_cast<uint8_t*>(codes_host);
    uint16_t* os = static_cast<uint16_t*>(scales_host);
    uint16_t* oz = static_cast<uint16_t*>(zeros_host);
    for (int pg = sg.token_begin / P; pg < (sg.token_end + P - 1) / P; ++pg) {
        const Page& p = L.pages[(size_t)pg];
        if (hipMemcpyAsync(code.data(), c->arena + c->unit_off_bytes(p.code_unit), code_block, hipMemcpyDeviceToHost, s) != hipSuccess)
            return KVQ_E_HIP;
        if (meta_out && hipMemcpyAsync(meta.data(), c->arena + c->unit_off_bytes(p.meta_unit), meta.size(), hipMemcpyDeviceToHost, s) != hipSuccess)
            return KVQ_E_HIP;
        if (hipStreamSynchronize(s) != hipSuccess) return KVQ_E_HIP;
        for (int u = 0; u < c->units; ++u) {
            for (int tl = 0; tl < p.n; ++tl) {
                const int tip = tl / KVQ_TILE_TOKENS, t = tl % KVQ_TILE_TOKENS;
                const size_t tslot = (size_t)u * tpp + tip;
                const uint8_t* tile = code.data() + (tslot * 2 + (size_t)which) * kvq_tile_code_bytes(b);
                const size_t tok_seg = (size_t)pg * P + tl - sg.token_begin;
                uint8_t* row = oc + ((size_t)u * n_seg + tok_seg) * row_bytes;
                std::memset(row, 0, row_bytes);
                for (int d = 0; d < KVQ_D; ++d) {
                    int lane, slot;
                    if (which == KVQ_WHICH_K) kvq_k_slot(t, d, &lane, &slot);
                    else kvq_v_slot(t, d, &lane, &slot);
                    const uint32_t bit = (uint32_t)slot * b;
                    if (planes) {  // high-byte plane, then low-byte plane, each laid out like an 8-bit tile
                        row[2 * d] = tile[512u * 8 + kvq_tile_byte(lane, (uint32_t)slot)];
                        row[2 * d + 1] = tile[kvq_tile_byte(lane, (uint32_t)slot)];
                    } else if (b == 16) {
                        const uint8_t* src = tile + kvq_tile_byte(lane, bit / 8);
                        row[2 * d] = src[0];
                        row[2 * d + 1] = src[1];
                    } else {
                        uint32_t v = (tile[kvq_tile_byte(lane, bit / 8)] >> (bit % 8)) & ((1u << b) - 1u);
                        row[(size_t)d * b / 8] |= (uint8_t)(v << ((d * b) % 8));
                    }
                }
                if (meta_out) {
                    const uint16_t* m = reinterpret_cast<const uint16_t*>(meta.data() + tslot * KVQ_META_TILE_BYTES);
                    // the device keeps one (S, Z) per run of 32 channels (a group of 64 or 128 channels repeats
                    // its pair); the canonical format has one per group
                    const int gspan = c->cfg.group / KVQ_G, ngrp = KVQ_D / c->cfg.group;
                    for (int gg = 0; gg < ngrp; ++gg) {
                        const int g = gg * gspan;
                        size_t oi = ((size_t)u * n_seg + tok_seg) * ngrp + gg;
                        if (which == KVQ_WHICH_K) { os[oi] = m[t * 4 + g]; oz[oi] = m[128 + t * 4 + g]; }
                        else { os[oi] = m[256 + kvq_vmeta_index(t, g)]; oz[oi] = m[384 + kvq_vmeta_index(t, g)]; }
                    }
                }
            }
        }
    }
    return KVQ_OK;
}

kvq_status_t kvq_cache_set_option(kvq_cache_t* c, int32_t option, int32_t value) {
    if (!c) return KVQ_E_INVALID;
    switch (option) {
        case KVQ_OPT_SPLITS:
            if (value < 0 || value > KVQ_MAX_SPLITS) return KVQ_E_INVALID;
            c->splits_override = value;
            return KVQ_OK;
        case KVQ_OPT_FUSED_MERGE:
            c->fused_merge = value ? 1 : 0;
            return KVQ_OK;
        case KVQ_OPT_DETERMINISTIC:
            c->deterministic = value ? 1 : 0;
            return KVQ_OK;
        case KVQ_OPT_SHIFT_STRATEGY:
            if (value != KVQ_SHIFT_EQUIVALENT && value != KVQ_SHIFT_DIRECT && value != KVQ_SHIFT_MODIFIED) return KVQ_E_INVALID;
            c->shift_strategy = value;
            return KVQ_OK;
        case KVQ_OPT_TIER16:
            if (value != KVQ_TIER16_FP16 && value != KVQ_TIER16_INT16) return KVQ_E_INVALID;
            for (const auto& L : c->layers)
                if (L.T != 0) return KVQ_E_STATE;  // the tier decides what every 16-bit page holds
            c->tier16 = value;
            return KVQ_OK;
        case KVQ_OPT_TILE_COST_2BIT:
        case KVQ_OPT_TILE_COST_4BIT:
        case KVQ_OPT_TILE_COST_8BIT:
        case KVQ_OPT_TILE_COST_16BIT:
            if (value < 1 || value > 1000000) return KVQ_E_INVALID;
            c->tile_cost[option - KVQ_OPT_TILE_COST_2BIT] = value;
            for (auto& L : c->layers) L.plan_tiles = -1;
            return KVQ_OK;
        default: return KVQ_E_INVALID;
    }
}

kvq_status_t kvq_cache_set_reparam(kvq_cache_t* c, int32_t layer, const float* lambda_dev, void* hip_stream) {
    if (!c || layer < 0 || layer >= c->cfg.n_layers) return KVQ_E_INVALID;
    Layer& L = c->layers[(size_t)layer];
    if (L.T != 0) return KVQ_E_STATE;
    if (!lambda_dev) { L.reparam = false; return KVQ_OK; }
    if (!c->dry) {
        kvq_status_t st = ensure_device(c, as_stream(hip_stream));
        if (st != KVQ_OK) return st;
        if (kvq_launch_reparam_store(lambda_dev, c->lambda_dev(layer), c->cfg.n_kv_heads * KVQ_D, as_stream(hip_stream)) != hipSuccess)
            return KVQ_E_HIP;
    }
    L.reparam = true;
    return KVQ_OK;
}

kvq_status_t kvq_calibrate_lambda(const void* k_calib_dev, int32_t batch, int32_t n_kv_heads, int32_t n_tokens,
                                  float alpha, float* lambda_dev, void* hip_stream) {
    if (!k_calib_dev || !lambda_dev || batch < 1 || n_kv_heads < 1 || n_tokens < 1 || !(alpha >= 0.0f && alpha <= 4.0f))
        return KVQ_E_INVALID;
    return kvq_launch_calibrate(k_calib_dev, batch, n_kv_heads, n_tokens, alpha, 1.0e-5f, lambda_dev,
                                as_stream(hip_stream)) == hipSuccess ? KVQ_OK : KVQ_E_HIP;
}

namespace {
kvq_status_t cache_error(kvq_cache_t* c, int32_t layer, bool l1, const void* k_ref_dev, const void* v_ref_dev,
                         const float* gk_dev, const float* gv_dev, double* out_host, void* hip_stream) {
    if (!c || layer < 0 || layer >= c->cfg.n_layers || !k_ref_dev || !v_ref_dev || !out_host) return KVQ_E_INVALID;
    if (c->dry) return KVQ_E_STATE;
    const Layer& L = c->layers[(size_t)layer];
    if (L.T == 0 || L.poisoned) return KVQ_E_STATE;
    hipStream_t s = as_stream(hip_stream);
    // The workgroups store their sums straight into pinned memory, where the host adds them up as they come: no accumulators to
    // clear, no copy back, and no wait for the end of the kernel, whose completion signal reaches the host some 5 us behind the last
    // sum.  A sum that is not there yet reads as a NaN no sum can be (its quiet bit is clear: arithmetic gives quiet ones).  All that a
    // workgroup reads it has read before it stores, so that with the last sum the inputs are the caller's again.  What keeps the host
    // waiting longer than a millisecond, work in front of the kernel as a rule, or an error, is left to the stream's synchronization.
    // Whole calls with gradients, with the synchronization and now, the first over a cache and repeated ones: 16 units x 137 tokens 24.3 and
    // 13.1 us, 17.0 and 11.8; 64 x 2,048 56 and 46, 52 and 43; 4 x 4,000 25 and 15, 20.1 and 13.9.
    const int n = 2 * kvq_error_workgroups(L.T, c->units);
    if (!c->sums_at_rest) {  // an earlier call failed: its kernel may still have sums to store
        if (hipStreamSynchronize(s) != hipSuccess) return KVQ_E_HIP;
        std::fill_n(c->sums, 2 * KVQ_ERR_MAX_WGS, kNoSum);
    }
    c->sums_at_rest = false;
    if (kvq_launch_error(l1, c->arena, c->table_dev(layer), k_ref_dev, v_ref_dev, gk_dev, gv_dev, L.T, c->tpp, c->units,
                         reinterpret_cast<double*>(c->ring_dev + c->ring_ctl.total_bytes()), s) != hipSuccess)
        return KVQ_E_HIP;
    bool waited = false;
    const auto start = std::chrono::steady_clock::now();
    const auto sum_at = [&](int i, uint64_t* bits) {
        for (int spins = 0; (*bits = __atomic_load_n(&c->sums[i], __ATOMIC_ACQUIRE)) == kNoSum; ++spins) {
            if (waited) return false;  // the stream is done and the sum is not there
            if (spins % 64 != 63 || std::chrono::steady_clock::now() - start < std::chrono::milliseconds(1)) continue;
            if (hipStreamSynchronize(s) != hipSuccess) return false;
            waited = true;
        }
        return true;
    };
    uint64_t bits;
    for (int i = n - 1; i >= 0; i -= 64)  // (a look here and there first: what is added up then is there as a rule, line behind line)
        if (!sum_at(i, &bits)) return KVQ_E_HIP;
    double sum[2] = {0.0, 0.0};
    for (int i = 0; i < n; ++i) {
        if (!sum_at(i, &bits)) return KVQ_E_HIP;
        double x;
        std::memcpy(&x, &bits, sizeof x);
        sum[i & 1] += x;
    }
    std::fill_n(c->sums, n, kNoSum);
    c->sums_at_rest = true;
    out_host[0] = sum[0];
    out_host[1] = sum[1];
    return KVQ_OK;
}
}  // namespace

kvq_status_t kvq_cache_sq_error(kvq_cache_t* c, int32_t layer, const void* k_ref_dev, const void* v_ref_dev,
                                double* sq_err_host, void* hip_stream) {
    return cache_error(c, layer, false, k_ref_dev, v_ref_dev, nullptr, nullptr, sq_err_host, hip_stream);
}

kvq_status_t kvq_cache_sensitivity(kvq_cache_t* c, int32_t layer, const void* k_ref_dev, const void* v_ref_dev,
                                   const float* gk_dev, const float* gv_dev, double* s_host, void* hip_stream) {
    return cache_error(c, layer, true, k_ref_dev, v_ref_dev, gk_dev, gv_dev, s_host, hip_stream);
}

// Eq. 6 of Sec. 3.2, exactly: multiple-choice knapsack by the list of non-dominated (memory, cost) states
// (Nemhauser-Ullmann).  After block i the list holds, by increasing memory and strictly decreasing cost, every
// total that no other choice of widths for blocks 0..i beats in both; a state remembers its predecessor and choice.
kvq_status_t kvq_allocate_bits(int32_t n_blocks, int32_t n_choices, const double* s, const uint64_t* mem,
                               uint64_t budget, int32_t* choice_out, double* total_s_out, uint64_t* total_mem_out) {
    if (n_blocks < 1 || n_blocks > 4096 || n_choices < 1 || n_choices > 16 || !s || !mem || !choice_out) return KVQ_E_INVALID;
    for (int64_t i = 0; i < (int64_t)n_blocks * n_choices; ++i)
        if (!(s[i] >= 0.0) || !std::isfinite(s[i])) return KVQ_E_INVALID;
    struct State { uint64_t m; double cost; int32_t prev; int32_t choice; };
    const size_t kMaxStates = 1u << 22;
    std::vector<std::vector<State>> layers((size_t)n_blocks);
    std::vector<State> cur{State{0, 0.0, -1, -1}}, cand;
    for (int i = 0; i < n_blocks; ++i) {
        cand.clear();
        for (int32_t p = 0; p < (int32_t)cur.size(); ++p)
            for (int32_t ch = 0; ch < n_choices; ++ch) {
                const uint64_t m = cur[(size_t)p].m + mem[(size_t)i * n_choices + ch];
                if (m < cur[(size_t)p].m || m > budget) continue;  // overflow or over budget
                cand.push_back(State{m, cur[(size_t)p].cost + s[(size_t)i * n_choices + ch], p, ch});
            }
        if (cand.empty()) return KVQ_E_BUDGET;
        // by memory, then cost, then (for reproducible ties) predecessor and choice
        std::sort(cand.begin(), cand.end(), [](const State& a, const State& b) {
            if (a.m != b.m) return a.m < b.m;
            if (a.cost != b.cost) return a.cost < b.cost;
            if (a.prev != b.prev) return a.prev < b.prev;
            return a.choice < b.choice;
        });
        std::vector<State>& keep = layers[(size_t)i];
        double best = std::numeric_limits<double>::infinity();
        for (const State& st : cand)
            if (st.cost < best) { keep.push_back(st); best = st.cost; }
        if (keep.size() > kMaxStates) return KVQ_E_OOM;
        cur = keep;
    }
    // the cheapest state is the last one (largest memory within the budget)
    int32_t at = (int32_t)layers[(size_t)n_blocks - 1].size() - 1;
    const State fin = layers[(size_t)n_blocks - 1][(size_t)at];
    for (int i = n_blocks - 1; i >= 0; --i) {
        const State& st = layers[(size_t)i][(size_t)at];
        choice_out[i] = st.choice;
        at = st.prev;
    }
    if (total_s_out) *total_s_out = fin.cost;
    if (total_mem_out) *total_mem_out = fin.m;
    return KVQ_OK;
}

kvq_status_t kvq_stream_read_probe(kvq_cache_t* c, const void* buf_dev, uint64_t bytes, int32_t n_workgroups,
                                   void* hip_stream) {
    if (!c || c->dry || !buf_dev || bytes < 16 || n_workgroups < 1 || n_workgroups > (1 << 20)) return KVQ_E_INVALID;
    if (reinterpret_cast<uintptr_t>(buf_dev) & 15u) return KVQ_E_INVALID;
    uint32_t* sink = reinterpret_cast<uint32_t*>(c->arena + c->jobs_off);  // never written in practice
    return kvq_launch_stream_read(buf_dev, bytes, n_workgroups, sink, as_stream(hip_stream)) == hipSuccess ? KVQ_OK : KVQ_E_HIP;
}

kvq_status_t kvq_cache_reset(kvq_cache_t* c, int32_t layer) {
    if (!c || layer < -1 || layer >= c->cfg.n_layers) return KVQ_E_INVALID;
    const int first = layer < 0 ? 0 : layer, last = layer < 0 ? c->cfg.n_layers : layer + 1;
    for (int l = first; l < last; ++l) {
        Layer& L = c->layers[(size_t)l];
        c->enqueue_failed = c->enqueue_failed || L.poisoned;
        for (const Page& p : L.pages) {
            c->buddy.release(p.code_unit, order_of_bits(p.bits));
            if (c->has_meta(p.bits)) c->buddy.release(p.meta_unit, 0);
        }
        L.pages.clear();
        L.T = 0;
        L.version++;
        L.plan_tiles = -1;
        L.poisoned = false;
    }
    // An empty cache starts over: the mark that some V scale was large must not outlive the data that set it, and if an
    // enqueue had failed the next call that enqueues work clears the device's counters and mark again, in stream order.
    bool all_empty = true;
    for (const Layer& L : c->layers) all_empty = all_empty && L.T == 0;
    if (all_empty) {
        if ((c->v_epoch += 4) == 0) c->v_epoch = 4;
        if (c->enqueue_failed) c->device_ready = c->enqueue_failed = false;
    }
    return KVQ_OK;
}

uint64_t kvq_cache_arena_free_bytes(const kvq_cache_t* c) { return c ? c->buddy.free_units() * c->unit_bytes : 0; }

const char* kvq_status_string(kvq_status_t s) {
    switch (s) {
        case KVQ_OK: return "ok";
        case KVQ_E_INVALID: return "invalid argument or unsupported configuration";
        case KVQ_E_BUDGET: return "block byte budget exceeded or nothing left to shrink";
        case KVQ_E_OOM: return "arena out of memory";
        case KVQ_E_STATE: return "call does not fit the cache state";
        case KVQ_E_HIP: return "HIP runtime error";
        case KVQ_E_LIMIT: return "launch exceeds the static scratch of kvq_decode_attention_static";
    }
    return "unknown status";
}

}  // extern "C"
