// Internal interface between the host bookkeeping (kvq_host.cpp) and the kernel translation units.
#ifndef KVQ_INTERNAL_H
#define KVQ_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>
#include "kvq_layout.h"

// Mark of a cache that holds a V scale >= 256 (it selects the attention kernels' overflow-proof V path): the quantizing kernels
// store the cache's current epoch into the word, the mark is set while the word holds a value of that epoch, and emptying the cache
// moves the epoch on, so that nothing has to be cleared on the device.  Epochs are multiples of four.
struct KvqVMark {
    uint32_t* word;
    uint32_t epoch;
};
// An attention launch that appends a token below 16 bits reads the mark and may set it, and which of its workgroups reads behind
// which other's store is chance.  No decision may hang on that: the V path changes the rounding, also where the caller asked for
// reproducible results, and the wavefronts of a workgroup have to take the same one.  The launch does not need its own token's mark
// (it attends to it in fp32).  So its tag is the epoch plus 1 or 2, in turn from one such launch to the next; it sets the mark by
// storing the tag, which it does not act on itself and every other launch does, and where it found another launch's tag it stores
// the epoch in its place before the turn comes back to that one.  The tag of every other launch is the epoch.
__host__ __device__ inline bool kvq_v_marked(uint32_t word, uint32_t tag, bool sets) {
    const uint32_t of = sets && word == tag ? 0u : word & ~3u;  // (no epoch is 0)
    return of == (sets ? tag & ~3u : tag);
}
// What such a launch leaves in the word.  large: the scale of its token's V is.
__host__ __device__ inline uint32_t kvq_v_mark_left(uint32_t word, uint32_t tag, bool large) {
    return kvq_v_marked(word, tag, true) ? tag & ~3u : large ? tag : word;
}

// The device page tables are written by the kernels that make the pages: an append, a re-quantization or the attention
// launch that appends a token gets the new entries in its arguments and stores them beside its other output.  (A copy
// from pinned memory in front of or behind each of them cost 4 us of copy kernel and 2 to 6 us of gaps.)
struct KvqRequantJob {        // one page to re-quantize
    uint32_t src_code_off256; // source code block
    uint32_t dst_code_off256; // destination code block
    uint32_t meta_off256;     // metadata block (updated in place for 2b -> b, written for fp16 -> b)
    uint32_t tiles_page;      // low 11 bits: tiles of the page that hold tokens (the kernels leave the others alone); above
                              // them the page's index in the block's table, whose entry the kernel rewrites
};
// a page holds at most 1,024 tiles and a block at most 2^21 pages (2^26 tokens in pages of 32)
inline uint32_t kvq_job_tiles_page(int n_tiles, int page) { return (uint32_t)n_tiles | ((uint32_t)page << 11); }

// Up to KVQ_JOBS_BY_ARG jobs ride in the kernel arguments (no table upload in front of the launch);
// longer lists are read from the uploaded table.
#define KVQ_JOBS_BY_ARG 192
struct KvqJobArgs {
    int32_t n;  // 0: read the table
    int32_t pad[3];
    KvqRequantJob jobs[KVQ_JOBS_BY_ARG];
};

// Every unit's arrival counter has 64 bytes of its own.  Tickets of workgroups that end at about the same time are atomics at
// the device's point of coherence, which takes those on one line in turn, some 12 ns each: with the counters of all units
// packed into one line 256 workgroups waited up to 3 us for theirs (2,560 tiles of 2 bits x 8 units in 32 splits 21.6 -> 19.5
// us, 64 tiles of 4 bits x 8 units in 32 splits 9.7 -> 7.7; 128 and 256 bytes apart are no better than 64).
#define KVQ_COUNTER_STRIDE 16  // in counters
struct KvqAttnHead {
    const uint8_t* arena;
    const KvqPageDesc* table;  // this block's page table
    const void* q;             // fp16 [batch, n_q_heads, 128]
    const float* lambda;       // [n_kv_heads][128] reparameterization factors applied to q at load, or null
    void* out;                 // [batch, n_q_heads, 128] fp16 or fp32
    float* part_o;             // [unit][split][16][128] un-normalised partial outputs
    float* part_ml;            // [unit][split][16] pairs (running max in log2 units, sum)
    uint32_t* counters;        // [unit * KVQ_COUNTER_STRIDE] arrival counters of the fused merge (kept at zero between launches)
    const uint32_t* v_mark;    // the word of KvqVMark: some V scale of the cache is >= 256 (set by the kernels that quantize)
    uint32_t v_tag;            // see kvq_v_marked
    int32_t n_tokens;          // tokens read from the cache (without the one this launch appends)
    int32_t tiles_per_page;
    uint32_t tpp_magic;        // ceil(2^32 / tiles_per_page) (unused when tiles_per_page == 1)
    int32_t gqa;               // query heads per KV head
    int32_t n_q_heads;
    int32_t n_kv_heads;
    uint32_t kv_magic;         // ceil(2^32 / n_kv_heads) (unused when n_kv_heads == 1)
    int32_t n_splits;
    int32_t out_fp32;
    int32_t fused_merge;
    int32_t deterministic;     // 1: static chunk-to-wavefront assignment (bit-reproducible summation order)
    int32_t short_ranges;      // 1: no range is longer than KVQ_SHORT_TILES (selects the kernel)
    int32_t int16_tier;        // 1: 16-bit pages hold integer codes in byte planes (selects the kernel)
    float scale_log2;          // softmax scale * log2(e)
    int32_t merge_groups;      // split merge: slot groups that share the splits of a head, splits of a group,
    int32_t merge_rounds;
    uint32_t gqa_magic;        // 65536 / gqa + 1
    // a one-token append done by the workgroup of a unit's last split (app_t_old < 0: none)
    int32_t app_t_old;         // tokens before the append
    KvqPageDesc app_desc;      // page of the new token
    int32_t app_page;          // the table entry the launch has to write (the token starts the page), or -1
    const void* app_k;         // fp16 [batch, n_kv_heads, 1, 128]
    const void* app_v;
    const float* app_rope;     // [1][128] cos | sin of the new position, or null
    const float* app_rinv;     // [n_kv_heads][128] reciprocal reparameterization factors, or null
    int32_t app_gspan;         // quantization group / 32 (integer tier and below 16 bits: the new token is quantized, Eq. 1-2)
};
// A launch none of whose ranges is longer takes the kernels for short ranges (kvq_attention_short.hip), two tiles to a
// wavefront; beyond that the streaming kernels, which overlap the loads of later tiles with the arithmetic of earlier ones,
// catch up: blocks in turn, 600 MB of them, ranges of 24 tiles of 4 bits x 64 units 13.5 us and 12.4 streaming, of 17 tiles of
// 4 and 16 bits x 4 units 11.6 and 10.6, of 24 tiles of 16 bits x 64 units 20.3 and 21.1, of 32 tiles of 2 bits x 32 units 13.2 and
// 12.6; ranges of 16 tiles: 4 bits x 8 units 8.6 and 9.6.
#define KVQ_SHORT_TILES 16
struct KvqAttnParams : KvqAttnHead {
    int32_t split_begin[KVQ_MAX_SPLITS + 1];  // tile index where each split starts
};

// kvq_quant.hip
// One append call takes fewer than 2^23 tokens per sequence: the kernels address the rows of a unit's input through a
// buffer descriptor with 32-bit byte offsets (256 bytes per row; offsets up to a few tiles beyond the last row occur).
#define KVQ_MAX_APPEND_TOKENS (1 << 23)
// Pages of one append call.  Up to KVQ_APPEND_ARG_PAGES of them ride in the kernel arguments (n > 0), which also saves
// the dependent read of the device table; an append that touches more reads the table, which then holds them already.
#define KVQ_APPEND_ARG_PAGES 128
struct KvqAppendPages {
    int32_t n;           // pages the append touches, 0: read the table
    int32_t first_page;  // index of the first of them
    int32_t fresh;       // entries fresh .. n - 1 are new: the kernel writes them into the table
    uint32_t bits;
    uint32_t int16;
    uint32_t code_off256[KVQ_APPEND_ARG_PAGES], meta_off256[KVQ_APPEND_ARG_PAGES];
};
// table: the block's device page table, read (n == 0) or written (fresh entries)
hipError_t kvq_launch_append(int bits, uint8_t* arena, KvqPageDesc* table, const void* k_in,
                             const void* v_in, int t_old, int n_new, int tiles_per_page, int units,
                             const KvqAppendPages& pages, KvqVMark mark, int group,
                             const float* rinv, int n_kv_heads, const float* rope, bool int16, hipStream_t s);
// table: the block's device page table; the kernels write the entries of the pages they re-quantize
hipError_t kvq_launch_shrink(int dst_bits, int strategy, uint8_t* arena, KvqPageDesc* table, const KvqRequantJob* jobs_dev,
                             const KvqRequantJob* jobs_host, int n_jobs, int tiles_per_page, int units,
                             KvqVMark mark, hipStream_t s);
hipError_t kvq_launch_quant16(int dst_bits, uint8_t* arena, KvqPageDesc* table, const KvqRequantJob* jobs_dev,
                              const KvqRequantJob* jobs_host, int n_jobs, int tiles_per_page, int units,
                              KvqVMark mark, int group, hipStream_t s);
hipError_t kvq_launch_reparam_store(const float* lambda, float* dst, int n, hipStream_t s);
hipError_t kvq_launch_calibrate(const void* k, int batch, int n_kv_heads, int n_tokens, float alpha, float floor_,
                                float* lambda, hipStream_t s);
// partial: 2 doubles (K, V) for each of kvq_error_workgroups() workgroups, at most KVQ_ERR_MAX_WGS (four per compute
// unit: 16 wavefronts, what hides the latency of the row loads); device-visible memory
#define KVQ_ERR_MAX_WGS 1024
int kvq_error_workgroups(int n_tokens, int units);
hipError_t kvq_launch_error(bool l1, const uint8_t* arena, const KvqPageDesc* table, const void* k_ref,
                            const void* v_ref, const float* gk, const float* gv, int n_tokens, int tiles_per_page,
                            int units, double* partial, hipStream_t s);
hipError_t kvq_launch_stream_read(const void* buf, size_t bytes, int n_workgroups, uint32_t* sink, hipStream_t s);
hipError_t kvq_launch_fill_u32(uint32_t* dst, uint32_t value, size_t n, hipStream_t s);

// A ragged batch: several caches (each with its own length, widths and tables) served by one attention launch.  The
// parameter blocks sit in device memory; the map tells a workgroup which cache it works for.
#define KVQ_MAX_BATCH_CACHES 64
struct KvqBatchMap {
    int32_t n;
    int32_t wg_begin[KVQ_MAX_BATCH_CACHES + 1];  // first workgroup of every cache; [n] = grid size
};

// A batch of few caches has its parameters in the kernel arguments instead: what differs from cache to cache, pointers into the arena as
// offsets in units of 16 bytes (0: none; the table alone may lie at the arena's start), and the ranges of all caches one after the other.
#define KVQ_BATCH_ARG_CACHES 16
#define KVQ_BATCH_ARG_SPLITS 320
struct KvqBatchCache {
    const uint8_t* arena;
    const void *q, *app_k, *app_v;
    void* out;
    const float* app_rope;
    uint32_t table16, lambda16, part_o16, part_ml16, counters16, v_mark16;
    uint32_t v_tag;
    int32_t n_tokens, tiles_per_page;
    uint32_t tpp_magic;
    int32_t gqa, n_q_heads, n_kv_heads;
    uint32_t kv_magic;
    int32_t n_splits, merge_groups, merge_rounds;
    uint32_t gqa_magic;
    float scale_log2;
    uint32_t flags;       // bit 0: out_fp32, 1: fused_merge, 2: deterministic, 3: reciprocal factors for the new token, 4: its page's int16; from bit 8 on its gspan
    int32_t split_at;     // where the cache's ranges begin in split_begin
    int32_t app_t_old, app_page;
    uint32_t app_code_off256, app_meta_off256;
};
struct KvqBatchArgs {
    int32_t n;
    int32_t wg_begin[KVQ_BATCH_ARG_CACHES + 1];  // first workgroup of every cache; entries from n on hold the grid size
    KvqBatchCache cache[KVQ_BATCH_ARG_CACHES];
    int32_t split_begin[KVQ_BATCH_ARG_SPLITS];
};
static_assert(sizeof(KvqBatchArgs) <= 3840, "kernel arguments end at 4 KiB");
// Whether the parameters of these caches fit (their parameter blocks need not be in device-visible memory then).  An offset reaches
// 64 GiB, which an arena's tables exceed where the cache has tens of thousands of units (1 MiB of partials each) or thousands of blocks.
inline bool kvq_batch_fits_args(const KvqAttnParams* p, int n) {
    if (n > KVQ_BATCH_ARG_CACHES) return false;
    int ranges = 0;
    for (int i = 0; i < n; ++i) {
        ranges += p[i].n_splits + 1;
        for (const void* x : {(const void*)p[i].table, (const void*)p[i].lambda, (const void*)p[i].part_o, (const void*)p[i].part_ml,
                              (const void*)p[i].counters, (const void*)p[i].v_mark})
            if (x && (uint64_t)(static_cast<const uint8_t*>(x) - p[i].arena) >> 36) return false;
    }
    return ranges <= KVQ_BATCH_ARG_SPLITS;
}

// Static scratch of kvq_decode_attention_static (kvq_attention.hip): room for the partials of KVQ_STATIC_MAX_WGS
// workgroups (units * splits of one launch) and their arrival counters (a launch of more than one split per unit has at most
// half as many units as workgroups).
#define KVQ_STATIC_MAX_WGS 512
#define KVQ_STATIC_MAX_UNITS 4096
#define KVQ_STATIC_PART_O_BYTES ((size_t)KVQ_STATIC_MAX_WGS * 16 * KVQ_D * sizeof(float))
#define KVQ_STATIC_PART_ML_BYTES ((size_t)KVQ_STATIC_MAX_WGS * 32 * sizeof(float))
#define KVQ_STATIC_COUNTER_BYTES ((size_t)(KVQ_STATIC_MAX_WGS / 2) * KVQ_COUNTER_STRIDE * sizeof(uint32_t))
#define KVQ_STATIC_SCRATCH_BYTES (KVQ_STATIC_PART_O_BYTES + KVQ_STATIC_PART_ML_BYTES + KVQ_STATIC_COUNTER_BYTES)
// Device address of the scratch array on the current device (looked up once per device, no allocation).
hipError_t kvq_static_scratch(unsigned char** ptr);

// kvq_attention.hip
hipError_t kvq_launch_attention(const KvqAttnParams& p, int units, hipStream_t s);
hipError_t kvq_launch_attention_short(const KvqAttnParams& p, int units, hipStream_t s);  // kernel only, no merge
hipError_t kvq_launch_merge(const KvqAttnParams& p, int units, hipStream_t s);
hipError_t kvq_launch_attention_i16_append(const KvqAttnParams& p, int units, hipStream_t s);  // kernel only, no merge
hipError_t kvq_launch_attention_append_narrow(const KvqAttnParams& p, int units, hipStream_t s);  // kernel only, no merge
// kvq_attention_batch.hip, kvq_attention_short.hip: the bare kernel launches kvq_launch_attention_batch wraps
hipError_t kvq_launch_attention_short_batch(const KvqAttnParams* params_dev, const KvqBatchMap& map, bool int16, hipStream_t s);
hipError_t kvq_launch_attention_short_batch(const KvqBatchArgs& args, bool int16, hipStream_t s);
hipError_t kvq_launch_attention_batch_kernel(const KvqAttnParams* params_dev, const KvqBatchMap& map, bool int16,
                                             hipStream_t s);
hipError_t kvq_launch_attention_batch_kernel(const KvqBatchArgs& args, bool int16, hipStream_t s);
// params_dev: the n parameter blocks in device memory (in stream order), or null where they fit the kernel arguments
// (kvq_batch_fits_args); params_host: the same blocks on the host;
// units[i]: (sequence, KV head) units of cache i
hipError_t kvq_launch_attention_batch(const KvqAttnParams* params_dev, const KvqAttnParams* params_host,
                                      const int* units, int n, hipStream_t s);

#endif
