// Decode attention over one cache -- one kernel for a raw fp16 16-bit tier (the default), one for an integer 16-bit
// tier (a cache has one kind, so neither carries the other's path) -- the split-merge kernel and the launchers.  The
// device code is in kvq_attention_body.h; the ragged-batch kernels that share it are compiled on their own, so that
// they do not change the inlining and register allocation of these.
#include "kvq_attention_body.h"

#include <mutex>

namespace {

// Scratch of kvq_decode_attention_static: split partials, (max, sum) pairs and arrival counters in the device image
// of this library instead of the caller's arena, for callers that cannot allocate.  Every GPU the library runs on
// holds its own copy until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels are given the address that call returns.
static __device__ __align__(256) unsigned char scratch[KVQ_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices];  // device address of `scratch` per device, looked up once

// grid = (splits, units); 512 threads = 8 wavefronts, one workgroup per compute unit.
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    attention_body<false, false, 0>(P, P.split_begin[blockIdx.x], P.split_begin[blockIdx.x + 1], sh);
}

// The same with a one-token append into the raw fp16 tier in front (kvq_append_decode_attention).
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_append_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    attention_body<false, false, KVQ_APPEND_16>(P, P.split_begin[blockIdx.x], P.split_begin[blockIdx.x + 1], sh);
}

// The same for a cache whose 16-bit tier holds integer codes in byte planes (KVQ_TIER16_INT16).
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_i16_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    attention_body<true, false, 0>(P, P.split_begin[blockIdx.x], P.split_begin[blockIdx.x + 1], sh);
}

// Same thread count as the attention kernel, so both merge variants add in the same order.
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_merge_kernel(const KvqAttnParams P) {
    __shared__ float lds[KVQ_MERGE_LDS_FLOATS];
    merge_splits<false>(P, blockIdx.x, threadIdx.x, merge_lane(P, blockIdx.x, threadIdx.x), lds);
}

}  // namespace

#ifdef KVQ_PHASE_STAMPS
// Measurement build only: copies the stamps of the last launch of the single-cache kernels to the host.
extern "C" int kvq_phase_stamps_read(unsigned long long* host) {
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(kvq_phase_stamps), sizeof(unsigned long long) * KVQ_STAMP_WGS * KVQ_STAMP_SLOTS);
}
#endif

hipError_t kvq_static_scratch(unsigned char** ptr) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = static_cast<unsigned char*>(p);
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

hipError_t kvq_launch_merge(const KvqAttnParams& p, int units, hipStream_t s) {
    hipLaunchKernelGGL(kvq_merge_kernel, dim3(units), dim3(KVQ_ATTN_THREADS), 0, s, p);
    return hipGetLastError();
}

hipError_t kvq_launch_attention(const KvqAttnParams& p, int units, hipStream_t s) {
    if (p.short_ranges) { hipError_t e0 = kvq_launch_attention_short(p, units, s); if (e0 != hipSuccess) return e0; }
    else if (p.app_t_old >= 0 && p.app_desc.bits < 16) { hipError_t e0 = kvq_launch_attention_append_narrow(p, units, s); if (e0 != hipSuccess) return e0; }
    else if (p.int16_tier && p.app_t_old >= 0) { hipError_t e0 = kvq_launch_attention_i16_append(p, units, s); if (e0 != hipSuccess) return e0; }
    else if (p.int16_tier) hipLaunchKernelGGL(kvq_attention_i16_kernel, dim3(p.n_splits, units), dim3(KVQ_ATTN_THREADS), 0, s, p);
    else if (p.app_t_old >= 0) hipLaunchKernelGGL(kvq_attention_append_kernel, dim3(p.n_splits, units), dim3(KVQ_ATTN_THREADS), 0, s, p);
    else hipLaunchKernelGGL(kvq_attention_kernel, dim3(p.n_splits, units), dim3(KVQ_ATTN_THREADS), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (p.n_splits > 1 && !p.fused_merge) e = kvq_launch_merge(p, units, s);
    return e;
}

// The parameter blocks as kernel arguments.  (Whatever they point to in the arena is aligned to 16 bytes, and the reciprocal factors follow the
// factors.)
static bool pack_batch_args(const KvqAttnParams* params, const KvqBatchMap& map, int n, KvqBatchArgs& a) {
    if (!kvq_batch_fits_args(params, n)) return false;
    a.n = n;
    for (int i = 0; i <= KVQ_BATCH_ARG_CACHES; ++i) a.wg_begin[i] = map.wg_begin[i < n ? i : n];
    int at = 0;
    for (int i = 0; i < n; ++i) {
        const KvqAttnParams& p = params[i];
        KvqBatchCache& c = a.cache[i];
        const auto offset = [&](const void* x) { return x ? (uint32_t)((uint64_t)(static_cast<const uint8_t*>(x) - p.arena) / 16) : 0u; };
        c.arena = p.arena; c.q = p.q; c.out = p.out; c.app_k = p.app_k; c.app_v = p.app_v; c.app_rope = p.app_rope;
        c.table16 = offset(p.table); c.lambda16 = offset(p.lambda); c.part_o16 = offset(p.part_o); c.part_ml16 = offset(p.part_ml);
        c.counters16 = offset(p.counters); c.v_mark16 = offset(p.v_mark);
        c.v_tag = p.v_tag; c.n_tokens = p.n_tokens; c.tiles_per_page = p.tiles_per_page; c.tpp_magic = p.tpp_magic;
        c.gqa = p.gqa; c.n_q_heads = p.n_q_heads; c.n_kv_heads = p.n_kv_heads; c.kv_magic = p.kv_magic;
        c.n_splits = p.n_splits; c.merge_groups = p.merge_groups; c.merge_rounds = p.merge_rounds; c.gqa_magic = p.gqa_magic;
        c.scale_log2 = p.scale_log2;
        c.flags = (p.out_fp32 ? 1u : 0u) | (p.fused_merge ? 2u : 0u) | (p.deterministic ? 4u : 0u) | (p.app_rinv ? 8u : 0u) |
                  (p.app_desc.int16 ? 16u : 0u) | (uint32_t)p.app_gspan << 8;
        c.split_at = at;
        c.app_t_old = p.app_t_old; c.app_page = p.app_page;
        c.app_code_off256 = p.app_desc.code_off256; c.app_meta_off256 = p.app_desc.meta_off256;
        for (int k = 0; k <= p.n_splits; ++k) a.split_begin[at++] = p.split_begin[k];
    }
    return true;
}

hipError_t kvq_launch_attention_batch(const KvqAttnParams* params_dev, const KvqAttnParams* params_host,
                                      const int* units, int n, hipStream_t s) {
    if (n < 1 || n > KVQ_MAX_BATCH_CACHES) return hipErrorInvalidValue;
    KvqBatchMap map;
    map.n = n;
    int wgs = 0;
    for (int i = 0; i < n; ++i) {
        map.wg_begin[i] = wgs;
        wgs += params_host[i].n_splits * units[i];
    }
    for (int i = n; i <= KVQ_MAX_BATCH_CACHES; ++i) map.wg_begin[i] = wgs;
    const bool int16 = params_host[0].int16_tier != 0;
    // One launch, one kernel: that for short ranges where every cache's are.  Calls in a train, streaming kernel and this one, four
    // sequences of 300 tokens x 8 units 9.1 -> 7.2 us, 100 to 2,000 x 8 11.9 -> 9.4, 3,500 x 8 of 4 / 16 bits (14 tiles a range) 13.2 -> 11.9
    // and 17.7 -> 15.6, 32 of 500 x 8 (16 tiles) 15.5 -> 14.3 and 19.4 -> 18.0; with ranges of 20 tiles in it, 32 of 640 x 8 of 8 bits, it
    // took 17.2 and streaming 16.9.
    bool short_ranges = true;
    for (int i = 0; i < n; ++i) short_ranges = short_ranges && params_host[i].short_ranges;
    hipError_t e;
    if (!params_dev) {
        KvqBatchArgs args;
        if (!pack_batch_args(params_host, map, n, args)) return hipErrorInvalidValue;
        e = short_ranges ? kvq_launch_attention_short_batch(args, int16, s) : kvq_launch_attention_batch_kernel(args, int16, s);
    } else {
        e = short_ranges ? kvq_launch_attention_short_batch(params_dev, map, int16, s) : kvq_launch_attention_batch_kernel(params_dev, map, int16, s);
    }
    for (int i = 0; i < n && e == hipSuccess; ++i)
        if (params_host[i].n_splits > 1 && !params_host[i].fused_merge) e = kvq_launch_merge(params_host[i], units[i], s);
    return e;
}
