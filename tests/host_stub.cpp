// The library's host code over a fake device: arena and pinned memory are plain host memory, the launchers of
// paper_2505_18610_amd/csrc/kvq_internal.h are replaced by stubs that do to the page tables what the kernels do and check
// what the kernels would read.  tests/test_host_stub.py builds it with kvq_host.cpp and a HIP runtime that is stubbed below;
// argument: the scenario.  Exit code 0 = pass.  No GPU and no HIP library is involved.
#include <hip/hip_runtime.h>
#include <sys/mman.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <memory>
#include <random>
#include <string>
#include <vector>

#include "kvq.h"
#include "../paper_2505_18610_amd/csrc/kvq_internal.h"

// ---- the HIP runtime, as far as the host code uses it
extern "C" {
unsigned host_memory_flags = 0;
hipError_t hipHostMalloc(void** p, size_t n, unsigned int flags) { host_memory_flags = flags; *p = aligned_alloc(256, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned int) { *d = h; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t);  // (below, with the launches)
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) { memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
}

namespace {

int failures = 0;
#define CHECK(cond, ...)                                                          \
    do {                                                                          \
        if (!(cond)) { ++failures; printf("line %d: %s: ", __LINE__, #cond); printf(__VA_ARGS__); printf("\n"); } \
    } while (0)

int launches = 0, fail_launch = -1;  // the launch with this number fails
hipError_t launched() { return launches++ == fail_launch ? hipErrorLaunchFailure : hipSuccess; }

std::vector<std::function<void()>> in_flight;  // what the device has still to do, in stream order (sums of the error kernel)
bool sums_late = false;                        // a kernel's sums arrive when the next kernel starts or the stream is waited for
bool fail_sync = false;
void finish_in_flight() {
    for (const auto& f : in_flight) f();
    in_flight.clear();
}

std::map<const uint8_t*, uint64_t> arena_size;  // every arena by its address
KvqAttnParams last;                             // parameters of the last attention launch
std::vector<KvqAttnParams> last_batch;          // of the last batched one

void check_table(const uint8_t* arena, const KvqPageDesc* table, int n_tokens, int tpp) {
    const int pages = (n_tokens + 32 * tpp - 1) / (32 * tpp);
    for (int i = 0; i < pages; ++i) {
        const KvqPageDesc& d = table[i];
        CHECK(d.bits == 16 || d.bits == 8 || d.bits == 4 || d.bits == 2, "page %d of %d has %u bits", i, pages, d.bits);
        CHECK((uint64_t)d.code_off256 * 256 < arena_size[arena], "page %d of %d lies at %u", i, pages, d.code_off256);
    }
}
// The launch's workgroups, one a unit, start and end in an order of chance; each reads the mark of large V scales at its start and,
// where the launch quantizes a token, leaves its own at its end.
std::mt19937 chance(3);
bool token_is_large = false;  // the V scale of the token that a step appends, in one unit
int acted = 0;                // how many workgroups of the last launch took the path for large scales
void mark_of_large_scales(const KvqAttnParams& p, int units) {
    uint32_t* const word = const_cast<uint32_t*>(p.v_mark);
    const bool sets = p.app_t_old >= 0 && p.app_desc.bits < 16;
    const int large_unit = token_is_large ? (int)(chance() % (unsigned)units) : -1;
    std::vector<int> waiting, running;
    for (int i = 0; i < units; ++i) waiting.push_back(i);
    acted = 0;
    while (!waiting.empty() || !running.empty()) {
        const bool start = running.empty() || (!waiting.empty() && chance() % 2);
        std::vector<int>& from = start ? waiting : running;
        const size_t k = chance() % from.size();
        const int unit = from[k];
        from.erase(from.begin() + (long)k);
        if (start) {
            acted += kvq_v_marked(*word, p.v_tag, sets) ? 1 : 0;
            running.push_back(unit);
        } else if (sets) {
            *word = kvq_v_mark_left(*word, p.v_tag, unit == large_unit);
        }
    }
    CHECK(acted == 0 || acted == units, "%d of %d workgroups saw the mark", acted, units);
}
void attention(const KvqAttnParams& p) {
    last = p;
    check_table(p.arena, p.table, p.n_tokens, p.tiles_per_page);
    if (p.app_page >= 0) const_cast<KvqPageDesc*>(p.table)[p.app_page] = p.app_desc;
    // the plan: the ranges follow one another, and in pages of an even number of tiles they start at even ones unless
    // they hold a single tile (chunks of two tiles must not straddle pages)
    const int n_tiles = (p.n_tokens + 31) / 32;
    CHECK(p.split_begin[0] == 0 && p.split_begin[p.n_splits] == n_tiles, "plan of %d tiles ends at %d", n_tiles, p.split_begin[p.n_splits]);
    for (int i = 0; i < p.n_splits; ++i) {
        const int a = p.split_begin[i], b = p.split_begin[i + 1];
        CHECK(a <= b, "range %d of %d: %d .. %d", i, p.n_splits, a, b);
        // the workgroup of the last range stores the token the launch appends: nobody else may be reading that tile
        CHECK(i + 1 < p.n_splits || n_tiles == 0 || b > a, "the last of %d ranges of %d tiles is empty", p.n_splits, n_tiles);
        CHECK(b - a <= 1 || p.tiles_per_page % 2 == 1 || a % 2 == 0, "range %d of %d: %d .. %d", i, p.n_splits, a, b);
    }
}

}  // namespace

extern "C" hipError_t hipStreamSynchronize(hipStream_t) {
    if (fail_sync) return hipErrorUnknown;
    finish_in_flight();
    return hipSuccess;
}
hipError_t kvq_launch_append(int bits, uint8_t* arena, KvqPageDesc* table, const void*, const void*, int t_old, int n_new, int tpp,
                             int, const KvqAppendPages& ap, KvqVMark, int, const float*, int, const float*, bool int16, hipStream_t) {
    const hipError_t e = launched();
    if (e != hipSuccess) return e;
    for (int i = ap.fresh; i < ap.n; ++i) table[ap.first_page + i] = KvqPageDesc{ap.code_off256[i], ap.meta_off256[i], ap.bits, ap.int16};
    check_table(arena, table, t_old + n_new, tpp);
    (void)bits; (void)int16;
    return hipSuccess;
}
static hipError_t requant(int to, KvqPageDesc* table, const KvqRequantJob* dev, const KvqRequantJob* host, int n) {
    const hipError_t e = launched();
    if (e != hipSuccess) return e;
    for (int i = 0; i < n; ++i) {
        const KvqRequantJob& j = host ? host[i] : dev[i];
        table[j.tiles_page >> 11] = KvqPageDesc{j.dst_code_off256, j.meta_off256, (uint32_t)to, 0u};
    }
    return hipSuccess;
}
hipError_t kvq_launch_shrink(int to, int, uint8_t*, KvqPageDesc* table, const KvqRequantJob* dev, const KvqRequantJob* host, int n, int, int,
                             KvqVMark, hipStream_t) { return requant(to, table, dev, host, n); }
hipError_t kvq_launch_quant16(int to, uint8_t*, KvqPageDesc* table, const KvqRequantJob* dev, const KvqRequantJob* host, int n, int, int,
                              KvqVMark, int, hipStream_t) { return requant(to, table, dev, host, n); }
hipError_t kvq_launch_reparam_store(const float*, float*, int, hipStream_t) { return launched(); }
hipError_t kvq_launch_calibrate(const void*, int, int, int, float, float, float*, hipStream_t) { return launched(); }
int kvq_error_workgroups(int, int) { return 1; }
hipError_t kvq_launch_error(bool, const uint8_t* arena, const KvqPageDesc* table, const void*, const void*, const float*, const float*,
                            int n_tokens, int tpp, int, double* partial, hipStream_t) {
    const hipError_t e = launched();
    if (e != hipSuccess) return e;
    check_table(arena, table, n_tokens, tpp);
    finish_in_flight();
    in_flight.push_back([=] { partial[0] = n_tokens; partial[1] = -n_tokens; });
    if (!sums_late) finish_in_flight();
    return hipSuccess;
}
hipError_t kvq_launch_stream_read(const void*, size_t, int, uint32_t*, hipStream_t) { return launched(); }
hipError_t kvq_launch_fill_u32(uint32_t* dst, uint32_t value, size_t n, hipStream_t) {
    const hipError_t e = launched();
    if (e == hipSuccess) for (size_t i = 0; i < n; ++i) dst[i] = value;
    return e;
}
hipError_t kvq_static_scratch(unsigned char** ptr) { static unsigned char scratch[KVQ_STATIC_SCRATCH_BYTES]; *ptr = scratch; return hipSuccess; }
hipError_t kvq_launch_attention(const KvqAttnParams& p, int units, hipStream_t) {
    const hipError_t e = launched();
    if (e == hipSuccess) { attention(p); mark_of_large_scales(p, units); }
    return e;
}
hipError_t kvq_launch_merge(const KvqAttnParams&, int, hipStream_t) { return launched(); }
bool batch_by_args = false;  // the last batched launch had no parameter blocks in device-visible memory
hipError_t kvq_launch_attention_batch(const KvqAttnParams* dev, const KvqAttnParams* p, const int*, int n, hipStream_t) {
    batch_by_args = !dev;
    CHECK(dev || kvq_batch_fits_args(p, n), "%d caches do not fit the arguments", n);
    const hipError_t e = launched();
    for (int i = 0; i < n && e == hipSuccess; ++i) attention(p[i]);
    last_batch.assign(p, p + n);
    return e;
}

namespace {

uint16_t input[1 << 10];  // never read by a stub
float factors[128];
double sums[2];

struct Cache {
    kvq_cache_t* c = nullptr;
    kvq_config_t cfg{};
    uint8_t* arena = nullptr;
    // supers: allocation blocks of 16 units (a page of raw 16-bit tokens takes 16 units, metadata one)
    Cache(int page_tokens, int supers, int tier16, int policy = KVQ_POLICY_PAPER, int window = 0, int batch = 1, int kv = 1, int heads = 1) {
        cfg.n_layers = 1; cfg.batch = batch; cfg.n_kv_heads = kv; cfg.n_q_heads = kv * heads; cfg.head_dim = 128; cfg.group = 32;
        cfg.max_tokens = 1 << 18; cfg.page_tokens = page_tokens; cfg.policy = policy; cfg.window = window;
        const uint64_t budget = 1ull << 50;
        const uint8_t fbit = 2;
        const uint64_t bytes = kvq_arena_bytes(&cfg, (uint64_t)supers * 16 * 32 * page_tokens * batch * kv);
        arena = static_cast<uint8_t*>(aligned_alloc(256, (bytes + 255) / 256 * 256));
        memset(arena, 0xEE, bytes);
        arena_size[arena] = bytes;
        CHECK(kvq_cache_create(&cfg, &budget, &fbit, arena, bytes, &c) == KVQ_OK, "create");
        CHECK(kvq_cache_set_option(c, KVQ_OPT_TIER16, tier16) == KVQ_OK, "tier");
    }
    ~Cache() { kvq_cache_destroy(c); free(arena); }
    Cache(const Cache&) = delete;
    kvq_status_t append(int n, int bits = 0) { return kvq_quantize_append(c, 0, input, input, n, bits, nullptr); }
    kvq_status_t attend() { return kvq_decode_attention(c, 0, input, input, 0, 0.f, nullptr); }
    kvq_status_t step() { return kvq_append_decode_attention(c, 0, input, input, nullptr, input, input, 0, 0.f, nullptr); }
    int tokens() const { int T = -1; kvq_cache_describe(c, 0, nullptr, 0, nullptr, nullptr, &T, nullptr); return T; }
    uint64_t free_bytes() const { return kvq_cache_arena_free_bytes(c); }
};

kvq_status_t batch_step(const std::vector<Cache*>& caches) {
    std::vector<kvq_cache_t*> cs;
    for (Cache* c : caches) cs.push_back(c->c);
    std::vector<const void*> in(cs.size(), input);
    std::vector<void*> out(cs.size(), input);
    return kvq_append_decode_attention_batch(cs.data(), (int)cs.size(), 0, in.data(), in.data(), nullptr, in.data(), out.data(), 0, 0.f, nullptr);
}

// A ragged step in which one cache's arena is full: no cache may change, whatever their order and where in its page the
// others' token falls, and every cache goes on working.
void batch_full_arena() {
    for (int tier16 : {0, 1})
        for (int full_at : {0, 1, 2})
            for (int have : {64, 65, 95}) {
                Cache a(32, 8, tier16), b(32, 8, tier16), full(32, tier16 ? 2 : 1, tier16);
                std::vector<Cache*> all{&a, &b};
                all.insert(all.begin() + full_at, &full);
                CHECK(a.append(have) == KVQ_OK && b.append(33) == KVQ_OK && full.append(32) == KVQ_OK, "prompts");
                const uint64_t fa = a.free_bytes(), fb = b.free_bytes(), ff = full.free_bytes();
                const kvq_status_t st = batch_step(all);
                CHECK(st == KVQ_E_OOM, "%s", kvq_status_string(st));
                CHECK(a.tokens() == have && b.tokens() == 33 && full.tokens() == 32, "%d %d %d tokens, tier %d, full cache %d", a.tokens(), b.tokens(), full.tokens(), tier16, full_at);
                CHECK(a.free_bytes() == fa && b.free_bytes() == fb && full.free_bytes() == ff, "blocks not given back");
                CHECK(a.attend() == KVQ_OK && b.attend() == KVQ_OK && full.attend() == KVQ_OK, "attention");
                CHECK(batch_step({&a, &b}) == KVQ_OK && a.tokens() == have + 1 && b.tokens() == 34, "the step without the full cache");
                CHECK(a.step() == KVQ_OK && a.attend() == KVQ_OK && b.attend() == KVQ_OK, "steps");
            }
}

// A ragged step in which a launch fails: a cache whose token was not written may not be read any more, one whose append had
// not begun is unchanged.
void batch_failing_launch() {
    for (int which = 0; which < 3; ++which) {
        Cache a(32, 8, 0), q(32, 8, 0), z(32, 8, 0);
        // `a` and `z` append inside the attention launch, `q` (8 bits, no window) by a launch of its own in front of it
        CHECK(a.append(64) == KVQ_OK && q.append(64, 8) == KVQ_OK && z.append(64) == KVQ_OK, "prompts");
        const uint64_t fz = z.free_bytes();
        fail_launch = which < 2 ? launches + which : -1;  // 0: q's append; 1: the attention launch
        const kvq_status_t st = batch_step({&a, &q, &z});
        fail_launch = -1;
        if (which == 2) {
            CHECK(st == KVQ_OK && a.attend() == KVQ_OK && q.attend() == KVQ_OK && z.attend() == KVQ_OK, "%s", kvq_status_string(st));
            continue;
        }
        CHECK(st == KVQ_E_HIP, "%s", kvq_status_string(st));
        CHECK(a.attend() == KVQ_E_STATE && a.step() == KVQ_E_STATE, "a cache whose token nobody wrote is read, case %d", which);
        if (which == 0) {
            CHECK(q.attend() == KVQ_E_STATE, "q");
            CHECK(z.tokens() == 64 && z.free_bytes() == fz && z.attend() == KVQ_OK && z.step() == KVQ_OK, "z: %d tokens", z.tokens());
        } else {
            CHECK(q.attend() == KVQ_OK && q.tokens() == 65, "q holds its token");
            CHECK(z.attend() == KVQ_E_STATE, "z");
        }
        CHECK(kvq_cache_reset(a.c, -1) == KVQ_OK && a.append(64) == KVQ_OK && a.attend() == KVQ_OK, "reset");
    }
}

// Steps below 16 bits set the mark of large V scales in the launch that reads it.  A launch's workgroups agree on it whatever their
// order (checked above), the launch that sets it does not act on it, every later one does, also behind a step whose launch
// failed, until the cache is emptied.
void mark_set_by_a_step() {
    for (int round = 0; round < 300; ++round) {
        Cache a(32, 40, round % 2, KVQ_POLICY_PAPER, 0, 2, 8, 2);
        for (int life = 0; life < 3; ++life) {
            CHECK(a.append(64, 4) == KVQ_OK, "prompt");
            bool marked = false;
            for (int step = 0; step < 24; ++step) {
                switch (chance() % 6) {
                    case 0: CHECK(a.attend() == KVQ_OK && acted == (marked ? 16 : 0), "attention: %d", acted); break;
                    case 1: {
                        std::vector<kvq_cache_t*> one{a.c};
                        std::vector<const void*> in{input};
                        std::vector<void*> out{input};
                        CHECK(kvq_decode_attention_batch(one.data(), 1, 0, in.data(), out.data(), 0, 0.f, nullptr) == KVQ_OK, "batch");
                        CHECK(kvq_v_marked(*last.v_mark, last.v_tag, false) == marked, "batch");
                        break;
                    }
                    default:
                        token_is_large = chance() % 8 == 0;
                        CHECK(a.step() == KVQ_OK && acted == (marked ? 16 : 0), "step %d, large %d: %d", step, token_is_large, acted);
                        marked = marked || token_is_large;
                        token_is_large = false;
                }
            }
            if (life == 1) {
                fail_launch = launches;
                CHECK(a.step() == KVQ_E_HIP, "a failing step");
                fail_launch = -1;
            }
            CHECK(kvq_cache_reset(a.c, -1) == KVQ_OK, "reset");
        }
    }
}

// A step that fails in one block does not lose the mark that another block's step has set.
void mark_outlives_a_failing_step() {
    kvq_config_t cfg{};
    cfg.n_layers = 2; cfg.batch = 1; cfg.n_kv_heads = 4; cfg.n_q_heads = 4; cfg.head_dim = 128; cfg.group = 32;
    cfg.max_tokens = 1 << 12; cfg.page_tokens = 32; cfg.policy = KVQ_POLICY_PAPER;
    const uint64_t budget[2] = {1ull << 50, 1ull << 50};
    const uint8_t fbit[2] = {2, 2};
    const uint64_t bytes = kvq_arena_bytes(&cfg, 1 << 22);
    uint8_t* const arena = static_cast<uint8_t*>(aligned_alloc(256, (bytes + 255) / 256 * 256));
    arena_size[arena] = bytes;
    kvq_cache_t* c = nullptr;
    CHECK(kvq_cache_create(&cfg, budget, fbit, arena, bytes, &c) == KVQ_OK, "create");
    const auto step = [&](int layer) { return kvq_append_decode_attention(c, layer, input, input, nullptr, input, input, 0, 0.f, nullptr); };
    for (int l = 0; l < 2; ++l) CHECK(kvq_quantize_append(c, l, input, input, 40, 8, nullptr) == KVQ_OK, "prompt");
    for (int before = 0; before < 2; ++before) {
        CHECK(step(0) == KVQ_OK && acted == 0, "step");
        if (before) CHECK(step(0) == KVQ_OK && acted == 0, "step");
        token_is_large = true;
        CHECK(step(0) == KVQ_OK && acted == 0, "the step that sets it");
        token_is_large = false;
        fail_launch = launches;
        CHECK(step(1) == KVQ_E_HIP, "a failing step");
        fail_launch = -1;
        for (int k = 0; k < 4; ++k) CHECK(step(0) == KVQ_OK && acted == 4, "step %d behind it: %d", k, acted);
        CHECK(kvq_cache_reset(c, -1) == KVQ_OK, "reset");
        for (int l = 0; l < 2; ++l) CHECK(kvq_quantize_append(c, l, input, input, 40, 8, nullptr) == KVQ_OK, "prompt");
    }
    kvq_cache_destroy(c);
    free(arena);
}

// Arenas whose tables reach beyond what the offsets in the kernel arguments hold (the partials of 65,528 units are 64 GiB) go by the
// parameter blocks in memory.
void batch_of_large_arenas() {
    for (int batch : {1, 8000, 8191}) {
        kvq_config_t cfg{};
        cfg.n_layers = 1; cfg.batch = batch; cfg.n_kv_heads = 8; cfg.n_q_heads = 8; cfg.head_dim = 128; cfg.group = 32;
        cfg.max_tokens = 1 << 10; cfg.page_tokens = 32; cfg.policy = KVQ_POLICY_PAPER;
        const uint64_t budget = 1ull << 50, bytes = kvq_arena_bytes(&cfg, 1);
        const uint8_t fbit = 2;
        void* const mem = mmap(nullptr, bytes, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);  // (little of it is touched)
        if (mem == MAP_FAILED) { printf("no address space for %llu bytes\n", (unsigned long long)bytes); continue; }
        arena_size[static_cast<uint8_t*>(mem)] = bytes;
        kvq_cache_t* c = nullptr;
        CHECK(kvq_cache_create(&cfg, &budget, &fbit, mem, bytes, &c) == KVQ_OK, "create");
        const void* in = input;
        void* out = input;
        CHECK(kvq_quantize_append(c, 0, input, input, 8, 16, nullptr) == KVQ_OK, "prompt");
        for (int step = 0; step < 2; ++step) {
            CHECK(kvq_append_decode_attention_batch(&c, 1, 0, &in, &in, nullptr, &in, &out, 0, 0.f, nullptr) == KVQ_OK, "batch %d", batch);
            CHECK(batch_by_args == (batch < 8191), "batch %d", batch);
        }
        kvq_cache_destroy(c);
        munmap(mem, bytes);
    }
}

// A block whose launch failed after the bookkeeping is refused by every call that reads it, until it is emptied.
void failed_block_is_refused() {
    for (int tier16 : {0, 1})
        for (int fused : {0, 1}) {
            Cache a(32, 8, tier16);
            CHECK(a.append(64) == KVQ_OK, "prompt");
            fail_launch = launches;
            const kvq_status_t st = fused ? a.step() : a.append(1);
            fail_launch = -1;
            CHECK(st == KVQ_E_HIP, "%s", kvq_status_string(st));
            CHECK(kvq_cache_sq_error(a.c, 0, input, input, sums, nullptr) == KVQ_E_STATE, "squared error");
            CHECK(kvq_cache_sensitivity(a.c, 0, input, input, factors, factors, sums, nullptr) == KVQ_E_STATE, "sensitivity");
            CHECK(a.attend() == KVQ_E_STATE && a.step() == KVQ_E_STATE && a.append(1) == KVQ_E_STATE, "attention, appends");
            CHECK(kvq_decode_attention_static(a.c, 0, input, input, 0, 0.f, nullptr) == KVQ_E_STATE, "static attention");
            CHECK(batch_step({&a}) == KVQ_E_STATE, "batch");
            CHECK(kvq_progressive_requant(a.c, 0, 0, 0, nullptr, nullptr) == KVQ_E_STATE, "shrink");
            CHECK(kvq_cache_export_segment(a.c, 0, 0, KVQ_WHICH_K, input, input, input, nullptr) == KVQ_E_STATE, "export");
            CHECK(kvq_cache_reset(a.c, 0) == KVQ_OK && a.append(65) == KVQ_OK && a.attend() == KVQ_OK, "reset");
            CHECK(kvq_cache_sq_error(a.c, 0, input, input, sums, nullptr) == KVQ_OK, "squared error behind the reset");
        }
}

// The sums of a call that failed while its kernel was on its way are not taken for the next call's.
void sums_behind_a_failing_call() {
    Cache a(32, 8, 0);
    CHECK(host_memory_flags & hipHostMallocCoherent, "the host reads them while the kernel runs");
    CHECK(a.append(40) == KVQ_OK, "prompt");
    sums_late = true;
    for (int round = 0; round < 3; ++round) {
        fail_sync = true;
        CHECK(kvq_cache_sq_error(a.c, 0, input, input, sums, nullptr) == KVQ_E_HIP, "a wait that fails");
        CHECK(kvq_cache_sq_error(a.c, 0, input, input, sums, nullptr) == KVQ_E_HIP, "and fails again");
        fail_sync = false;
        CHECK(a.append(1) == KVQ_OK, "a token more");
        for (int again = 0; again < 2; ++again) {
            CHECK(kvq_cache_sq_error(a.c, 0, input, input, sums, nullptr) == KVQ_OK, "the next call");
            CHECK(sums[0] == a.tokens() && sums[1] == -a.tokens(), "%g and %g of %d tokens", sums[0], sums[1], a.tokens());
        }
    }
    fail_launch = launches;
    CHECK(kvq_cache_sq_error(a.c, 0, input, input, sums, nullptr) == KVQ_E_HIP, "a launch that fails");
    fail_launch = -1;
    CHECK(kvq_cache_sensitivity(a.c, 0, input, input, factors, factors, sums, nullptr) == KVQ_OK && sums[0] == a.tokens(), "the next call");
    sums_late = false;
}

// The split plan over lengths, widths, page sizes and split counts: what check and attention() above ask of every launch.
void split_plans() {
    for (int page : {32, 64, 96, 256})
        for (int narrow : {0, 1, 5, 10, 40})
            for (int bits : {8, 2})
                for (int rest = 1; rest <= 3 * page; rest += page / 4 + 1) {
                    Cache a(page, 64, 0);
                    CHECK((narrow == 0 || a.append(narrow * page, bits) == KVQ_OK) && a.append(rest, 16) == KVQ_OK, "prompt");
                    const int n_tiles = (a.tokens() + 31) / 32;
                    for (int splits : {0, 2, 3, 5, n_tiles / 2, n_tiles - 1, n_tiles, 128}) {
                        if (splits < 0 || splits > 128) continue;
                        CHECK(kvq_cache_set_option(a.c, KVQ_OPT_SPLITS, splits) == KVQ_OK, "option");
                        CHECK(a.attend() == KVQ_OK, "attention");
                        CHECK(last.n_splits <= n_tiles && (splits == 0 || last.n_splits == (splits < n_tiles ? splits : n_tiles)), "%d splits", last.n_splits);
                    }
                }
    // 128 units leave two workgroups to a range, which it takes beyond 32 tiles; one unit by itself takes a split per 16 tiles
    for (int tiles : {20, 21, 32, 33}) {
        Cache a(64, 40, 0, KVQ_POLICY_PAPER, 0, 16, 8);
        CHECK(a.append(32 * tiles - 1, 8) == KVQ_OK && a.attend() == KVQ_OK && last.n_splits == (tiles > 32 ? 2 : 1), "%d tiles, %d splits", tiles, last.n_splits);
    }
    Cache wide(64, 100, 0, KVQ_POLICY_PAPER, 0, 16, 8);
    CHECK(wide.append(24 * 32, 16) == KVQ_OK && wide.attend() == KVQ_OK && wide.attend() == KVQ_OK && last.n_splits == 2, "%d splits", last.n_splits);
    Cache one(256, 40, 0);
    CHECK(one.append(32000, 2) == KVQ_OK && one.attend() == KVQ_OK && last.n_splits == 63, "%d splits", last.n_splits);
    for (int tokens : {256 * 32, 500 * 32}) {  // 16 query heads per KV head
        Cache heads(256, 70, 0, KVQ_POLICY_PAPER, 0, 1, 1, 16);
        CHECK(heads.append(tokens, 16) == KVQ_OK && heads.attend() == KVQ_OK && last.n_splits == (tokens + 511) / 512, "%d splits", last.n_splits);
    }
    // a step on top of 640 tokens of 2 bits and 33 of 16 bits, as the library splits it by itself
    Cache a(64, 64, 0, KVQ_POLICY_PAPER, 64);
    CHECK(a.append(640, 2) == KVQ_OK && a.append(33, 16) == KVQ_OK && a.step() == KVQ_OK && last.app_t_old == 673, "step");
}

// A plan knows the pages as they are, however they came about: after random appends, shrinks and emptyings it is that of a
// block built at once with the same widths.  And ranges that are cut for the kernels for short ranges give no SIMD a tile more
// than equal ones would.
void plans_follow_the_pages() {
    std::mt19937 rng(11);
    const auto R = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    for (int round = 0; round < 40; ++round) {
        const int page = 32 * R(1, 4), units = 1 << R(0, 2), tier16 = R(0, 3) == 0;
        Cache a(page, 60, tier16, KVQ_POLICY_PAPER, 0, 1, units, R(1, 8));
        for (int step = 0; step < 20; ++step) {
            const int bits[4] = {2, 4, 8, 16};
            switch (R(0, 5)) {
                case 0: kvq_progressive_requant(a.c, 0, R(0, 2), 0, nullptr, nullptr); break;
                case 1: if (R(0, 9) == 0) kvq_cache_reset(a.c, -1); break;
                case 2: a.step(); break;
                default: if (a.tokens() < 25 * page) a.append(R(1, 3) * page - a.tokens() % page, a.tokens() % page ? 0 : bits[R(0, 3)]);
            }
            if (a.tokens() == 0 || a.attend() != KVQ_OK) continue;
            const std::vector<int32_t> got(last.split_begin, last.split_begin + last.n_splits + 1);
            kvq_segment_info_t segs[64];
            int m = 0;
            kvq_cache_describe(a.c, 0, segs, 64, &m, nullptr, nullptr, nullptr);
            Cache b(page, 60, tier16, KVQ_POLICY_PAPER, 0, 1, units, a.cfg.n_q_heads / units);
            for (int k = 0; k < m; ++k) CHECK(b.append(segs[k].token_end - segs[k].token_begin, segs[k].bits) == KVQ_OK, "segment %d of %d", k, m);
            CHECK(b.attend() == KVQ_OK, "attention");
            const std::vector<int32_t> fresh(last.split_begin, last.split_begin + last.n_splits + 1);
            CHECK(got == fresh, "round %d, step %d: %zu ranges, %zu in a fresh block", round, step, got.size() - 1, fresh.size() - 1);
            const int n = last.n_splits, n_tiles = (a.tokens() + 31) / 32, even = (n_tiles + n - 1) / n + 1;
            if (!tier16 && n > 16 && even <= 16)
                for (int i = 0; i < n; ++i) CHECK(got[(size_t)i + 1] - got[(size_t)i] <= (even + 3) / 4 * 4, "range %d of %d tiles in %d: %d", i, n_tiles, n, got[(size_t)i + 1] - got[(size_t)i]);
        }
    }
}

// A block that is emptied, changes to the other 16-bit tier and is filled alike is split as a fresh one of that tier: the tiers have
// different rules, though the tiles are as many and as wide.
void plans_follow_the_tier() {
    for (int units : {1, 2, 8, 16})
        for (int tiles : {12, 24, 40, 64, 120, 250})
            for (int tier16 : {0, 1}) {
                Cache a(64, 200, tier16, KVQ_POLICY_PAPER, 0, 1, units, 4), b(64, 200, 1 - tier16, KVQ_POLICY_PAPER, 0, 1, units, 4);
                CHECK(a.append(32 * tiles, 16) == KVQ_OK && a.attend() == KVQ_OK, "the first tier");
                CHECK(kvq_cache_reset(a.c, -1) == KVQ_OK && kvq_cache_set_option(a.c, KVQ_OPT_TIER16, 1 - tier16) == KVQ_OK, "the other tier");
                std::vector<int32_t> plan[2];
                for (Cache* c : {&a, &b}) {
                    CHECK(c->append(32 * tiles, 16) == KVQ_OK && c->attend() == KVQ_OK, "attention");
                    plan[c == &b].assign(last.split_begin, last.split_begin + last.n_splits + 1);
                }
                CHECK(plan[0] == plan[1], "%d units x %d tiles: %zu ranges, %zu in a fresh block", units, tiles, plan[0].size() - 1, plan[1].size() - 1);
            }
}

// The tile costs are relative: their scale changes neither how many splits a launch takes nor where they lie.
void tile_costs_are_relative() {
    for (int narrow : {8, 30, 200}) {
        std::vector<int32_t> plan, batch_plan;
        for (int scale : {0, 1, 5, 25, 3000}) {  // 0: the costs the library comes with, 20 : 29 : 50 : 60
            Cache a(64, 200, 0), b(64, 200, 0);
            for (Cache* c : {&a, &b}) {
                const int costs[4] = {20, 29, 50, 60};
                for (int i = 0; i < 4 && scale; ++i)
                    CHECK(kvq_cache_set_option(c->c, KVQ_OPT_TILE_COST_2BIT + i, costs[i] * scale) == KVQ_OK, "option");
                CHECK(c->append(narrow * 64, 2) == KVQ_OK && c->append(64 * narrow, 4) == KVQ_OK && c->append(100, 16) == KVQ_OK, "prompt");
            }
            for (bool batched : {false, true}) {
                kvq_cache_t* cs[2] = {a.c, b.c};
                const void* q[2] = {input, input};
                void* out[2] = {input, input};
                CHECK((batched ? kvq_decode_attention_batch(cs, 2, 0, q, out, 0, 0.f, nullptr) : a.attend()) == KVQ_OK, "attention");
                const std::vector<int32_t> now(last.split_begin, last.split_begin + last.n_splits + 1);
                std::vector<int32_t>& first = batched ? batch_plan : plan;
                if (scale == 0) first = now;
                CHECK(now == first, "%zu instead of %zu splits with costs x %d, %d pages, batched %d", now.size() - 1, first.size() - 1, scale, narrow, batched);
            }
        }
    }
}

// How a ragged batch shares the workgroups: the same as by giving one split at a time to the cache with the heaviest
// workgroups.  And dealing them does not dominate the call (step by step: 7 times as long).
void batch_shares() {
    std::mt19937 rng(5);
    const auto R = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    for (int round = 0; round < 60; ++round) {
        const int n = round < 3 ? 64 : R(1, 20);
        std::vector<std::unique_ptr<Cache>> caches;
        std::vector<kvq_cache_t*> cs;
        for (int i = 0; i < n; ++i) {
            caches.emplace_back(new Cache(64, 60, 0, KVQ_POLICY_PAPER, 0, 1, round < 3 ? 1 : 1 << R(0, R(0, 4))));
            Cache& c = *caches.back();
            const int bits[3] = {2, 4, 8};
            const int pages = R(0, R(0, 1) ? 40 : 4);
            if (round % 4 == 1) for (int k = 0; k < 4; ++k) kvq_cache_set_option(c.c, KVQ_OPT_TILE_COST_2BIT + k, R(1, R(1, 9)));
            CHECK((pages == 0 || c.append(pages * 64, bits[R(0, 2)]) == KVQ_OK) && c.append(R(1, 300), 16) == KVQ_OK, "prompt");
            cs.push_back(c.c);
        }
        std::vector<const void*> q((size_t)n, input);
        std::vector<void*> out((size_t)n, input);
        CHECK(kvq_decode_attention_batch(cs.data(), n, 0, q.data(), out.data(), 0, 0.f, nullptr) == KVQ_OK, "batch");
        const std::vector<KvqAttnParams> got = last_batch;
        // the most splits that pay and the tile time of a unit, as the library works them out
        std::vector<uint64_t> cost;
        std::vector<int> most, splits((size_t)n, 1);
        int used = 0;
        for (int i = 0; i < n; ++i) {
            kvq_segment_info_t segs[8];
            int m = 0, weight[4] = {100, 145, 250, 300};
            if (round % 4 == 1) { cost.clear(); break; }  // (random costs: only the plan checks of attention())
            kvq_cache_describe(cs[(size_t)i], 0, segs, 8, &m, nullptr, nullptr, nullptr);
            uint64_t time = 0;
            int tiles = 0;
            for (int k = 0; k < m; ++k) {
                const int nt = (segs[k].token_end + 31) / 32 - segs[k].token_begin / 32;
                tiles += nt;
                time += (uint64_t)nt * (uint64_t)weight[segs[k].bits == 16 ? 3 : segs[k].bits == 8 ? 2 : segs[k].bits == 4 ? 1 : 0];
            }
            cost.push_back(time);
            const int alone = std::min((tiles + 15) / 16, 128 / caches[(size_t)i]->cfg.n_kv_heads);  // (one query head per KV head)
            most.push_back(tiles <= 20 ? 1 : std::min(std::min(tiles, 128), std::max(alone, (int)std::sqrt((double)time / 80.0))));
            used += caches[(size_t)i]->cfg.n_kv_heads;
        }
        if (cost.empty()) continue;
        for (;;) {
            int pick = -1;
            uint64_t worst = 0;
            for (int i = 0; i < n; ++i) {
                if (splits[(size_t)i] >= most[(size_t)i] || used + caches[(size_t)i]->cfg.n_kv_heads > 256) continue;
                if (cost[(size_t)i] / (uint64_t)splits[(size_t)i] > worst) { worst = cost[(size_t)i] / (uint64_t)splits[(size_t)i]; pick = i; }
            }
            bool blocked = pick < 0;
            for (int i = 0; i < n; ++i)
                blocked |= splits[(size_t)i] < most[(size_t)i] && cost[(size_t)i] / (uint64_t)splits[(size_t)i] > worst;
            if (blocked) break;
            splits[(size_t)pick]++;
            used += caches[(size_t)pick]->cfg.n_kv_heads;
        }
        for (int i = 0; i < n; ++i)
            CHECK(got[(size_t)i].n_splits == splits[(size_t)i], "round %d, cache %d of %d: %d splits, %d expected", round, i, n, got[(size_t)i].n_splits, splits[(size_t)i]);
    }
    double us[2];
    for (int longer : {0, 1}) {
        std::vector<std::unique_ptr<Cache>> caches;
        std::vector<kvq_cache_t*> cs;
        for (int i = 0; i < 64; ++i) {
            caches.emplace_back(new Cache(256, 20, 0));
            CHECK(caches.back()->append(longer ? 500 + 16 * i : 8 * i + 8, 16) == KVQ_OK, "prompt");  // up to 6 pages
            cs.push_back(caches.back()->c);
        }
        std::vector<const void*> q(64, input);
        std::vector<void*> out(64, input);
        us[longer] = 1e9;
        for (int rep = 0; rep < 20; ++rep) {
            const auto t0 = std::chrono::steady_clock::now();
            for (int k = 0; k < 20; ++k) kvq_decode_attention_batch(cs.data(), 64, 0, q.data(), out.data(), 0, 0.f, nullptr);
            us[longer] = std::min(us[longer], std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count() / 20);
        }
    }
    printf("host time of a batch of 64: one split each %.1f us, several %.1f us\n", us[0], us[1]);
    CHECK(us[1] < 3 * us[0], "%.1f and %.1f us", us[0], us[1]);
}

const std::map<std::string, std::function<void()>> scenarios = {
    {"batch_full_arena", batch_full_arena},
    {"batch_failing_launch", batch_failing_launch},
    {"failed_block_is_refused", failed_block_is_refused},
    {"sums_behind_a_failing_call", sums_behind_a_failing_call},
    {"batch_of_large_arenas", batch_of_large_arenas},
    {"mark_set_by_a_step", mark_set_by_a_step},
    {"mark_outlives_a_failing_step", mark_outlives_a_failing_step},
    {"split_plans", split_plans},
    {"plans_follow_the_pages", plans_follow_the_pages},
    {"plans_follow_the_tier", plans_follow_the_tier},
    {"tile_costs_are_relative", tile_costs_are_relative},
    {"batch_shares", batch_shares},
};

}  // namespace

int main(int argc, char** argv) {
    const auto it = scenarios.find(argc > 1 ? argv[1] : "");
    if (it == scenarios.end()) { printf("no such scenario\n"); return 2; }
    it->second();
    (void)last;
    printf("%s: %d failures\n", argv[1], failures);
    return failures ? 1 : 0;
}
