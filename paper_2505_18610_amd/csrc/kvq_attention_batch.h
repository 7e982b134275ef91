// What a workgroup of a ragged batch works on: its cache's parameters, its unit and split, its tiles.
#ifndef KVQ_ATTENTION_BATCH_H
#define KVQ_ATTENTION_BATCH_H
#include "kvq_attention_body.h"

namespace {

// The parameter block of the workgroup's cache lies in host memory where the arguments do not hold it.  It is fetched over the link once, a dword per thread, and
// handed out from LDS: the head as scalars (read lane by lane from one register), the range of the split by index.  (Read
// field by field as the kernel comes to them, the blocks cost two to three dependent trips over the link.)
constexpr int kHeadDwords = sizeof(KvqAttnHead) / 4, kBlockDwords = sizeof(KvqAttnParams) / 4;
static_assert(kBlockDwords - kHeadDwords == KVQ_MAX_SPLITS + 1 + (KVQ_MAX_SPLITS + 1) % 2, "split_begin follows the head (padded to 8 bytes)");
static_assert(kHeadDwords <= 64 && kBlockDwords <= KVQ_ATTN_THREADS && sizeof(KvqAttnHead) % 8 == 0, "one dword per lane, one per thread");
struct HeadWords { uint32_t w[kHeadDwords]; };

struct BatchWork { int split, unit, t_begin, t_end; };

__device__ __forceinline__ KvqAttnHead batch_work(const KvqAttnParams* __restrict__ params, const KvqBatchMap& map,
                                                  uint32_t (&block)[kBlockDwords], BatchWork& work) {
    const int wg = blockIdx.x, tid = threadIdx.x;
    int ci = 0;
    for (int i = 1; i < map.n; ++i) ci = (wg >= map.wg_begin[i]) ? i : ci;
    if (tid < kBlockDwords) block[tid] = reinterpret_cast<const uint32_t*>(params + ci)[tid];
    __syncthreads();
    const uint32_t mine = block[min(tid & 63, kHeadDwords - 1)];
    HeadWords h;
#pragma unroll
    for (int i = 0; i < kHeadDwords; ++i) h.w[i] = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
    KvqAttnHead P = __builtin_bit_cast(KvqAttnHead, h);
    P.arena = as_global(P.arena); P.table = as_global(P.table); P.lambda = as_global(P.lambda);
    P.q = as_global(static_cast<const _Float16*>(P.q)); P.out = as_global(static_cast<float*>(P.out));
    P.part_o = as_global(P.part_o); P.part_ml = as_global(P.part_ml);
    P.counters = as_global(P.counters); P.v_mark = as_global(P.v_mark);
    P.app_k = as_global(static_cast<const _Float16*>(P.app_k)); P.app_v = as_global(static_cast<const _Float16*>(P.app_v));
    P.app_rope = as_global(P.app_rope); P.app_rinv = as_global(P.app_rinv);
    const int local = wg - map.wg_begin[ci];
    work.unit = local / P.n_splits;  // splits of a unit are neighbours
    work.split = local - work.unit * P.n_splits;
    const int* split_begin = reinterpret_cast<const int*>(block + kHeadDwords);
    work.t_begin = __builtin_amdgcn_readfirstlane(split_begin[work.split]);
    work.t_end = __builtin_amdgcn_readfirstlane(split_begin[work.split + 1]);
    return P;
}

// The same from the kernel arguments.  (A trip over the host link and the hand-out through LDS took 1.3 us of every workgroup's start:
// calls in a train, link and arguments, sixteen sequences of 2K to 32K tokens x 4 units 39.8 and 37.7 us, drawn batches of 2 to 16
// sequences 10 % less on average, 130 and 400 tokens x 4 6.9 and 6.3.)
// AT_ONCE: all of the cache's parameters are read before anything is done with them, as the kernels for short ranges want them; the
// streaming kernels read them where they are needed, which leaves them 30 scalar registers.
template <bool AT_ONCE>
__device__ __forceinline__ KvqAttnHead batch_work(const KvqBatchArgs& args, BatchWork& work) {
    const int wg = blockIdx.x;
    int ci = 0;
#pragma unroll
    for (int i = 1; i < KVQ_BATCH_ARG_CACHES; ++i) ci += wg >= args.wg_begin[i] ? 1 : 0;
    ci = min(ci, args.n - 1);
    KvqBatchCache b = args.cache[ci];
    const int first = args.wg_begin[ci];
    const uint8_t *arena = b.arena, *q = static_cast<const uint8_t*>(b.q), *k = static_cast<const uint8_t*>(b.app_k), *v = static_cast<const uint8_t*>(b.app_v);
    uint8_t* out = static_cast<uint8_t*>(b.out);
    if constexpr (AT_ONCE) asm volatile("" : "+s"(arena), "+s"(q), "+s"(k), "+s"(v), "+s"(out), "+s"(b.app_rope), "+s"(b.table16), "+s"(b.lambda16), "+s"(b.part_o16),
                      "+s"(b.part_ml16), "+s"(b.counters16), "+s"(b.v_mark16), "+s"(b.v_tag), "+s"(b.n_tokens), "+s"(b.tiles_per_page),
                      "+s"(b.tpp_magic), "+s"(b.gqa), "+s"(b.n_q_heads), "+s"(b.n_kv_heads), "+s"(b.kv_magic), "+s"(b.n_splits),
                      "+s"(b.merge_groups), "+s"(b.merge_rounds));
    if constexpr (AT_ONCE) asm volatile("" : "+s"(b.gqa_magic), "+s"(b.scale_log2), "+s"(b.flags), "+s"(b.split_at), "+s"(b.app_t_old), "+s"(b.app_page),
                      "+s"(b.app_code_off256), "+s"(b.app_meta_off256));
    const int local = wg - first;
    work.unit = local / b.n_splits;  // splits of a unit are neighbours
    work.split = local - work.unit * b.n_splits;
    work.t_begin = args.split_begin[b.split_at + work.split];
    work.t_end = args.split_begin[b.split_at + work.split + 1];
    uint8_t* const base = const_cast<uint8_t*>(as_global(arena));
    KvqAttnHead P = {};
    P.arena = base;
    P.table = reinterpret_cast<const KvqPageDesc*>(base + (uint64_t)b.table16 * 16u);
    P.q = as_global(q);
    P.lambda = b.lambda16 ? reinterpret_cast<const float*>(base + (uint64_t)b.lambda16 * 16u) : nullptr;
    P.out = as_global(out);
    P.part_o = reinterpret_cast<float*>(base + (uint64_t)b.part_o16 * 16u);
    P.part_ml = reinterpret_cast<float*>(base + (uint64_t)b.part_ml16 * 16u);
    P.counters = reinterpret_cast<uint32_t*>(base + (uint64_t)b.counters16 * 16u);
    P.v_mark = reinterpret_cast<const uint32_t*>(base + (uint64_t)b.v_mark16 * 16u);
    P.v_tag = b.v_tag; P.n_tokens = b.n_tokens; P.tiles_per_page = b.tiles_per_page; P.tpp_magic = b.tpp_magic;
    P.gqa = b.gqa; P.n_q_heads = b.n_q_heads; P.n_kv_heads = b.n_kv_heads; P.kv_magic = b.kv_magic;
    P.n_splits = b.n_splits; P.merge_groups = b.merge_groups; P.merge_rounds = b.merge_rounds; P.gqa_magic = b.gqa_magic;
    P.out_fp32 = (int)(b.flags & 1u); P.fused_merge = (int)(b.flags >> 1 & 1u); P.deterministic = (int)(b.flags >> 2 & 1u);
    P.scale_log2 = b.scale_log2;
    P.app_t_old = b.app_t_old; P.app_page = b.app_page;
    P.app_desc = KvqPageDesc{b.app_code_off256, b.app_meta_off256, 16u, b.flags >> 4 & 1u};
    P.app_k = as_global(k); P.app_v = as_global(v); P.app_rope = as_global(b.app_rope);
    P.app_rinv = (b.flags & 8u) ? reinterpret_cast<const float*>(base + (uint64_t)b.lambda16 * 16u) + (size_t)b.n_kv_heads * KVQ_D : nullptr;
    P.app_gspan = (int)(b.flags >> 8);
    return P;
}

}  // namespace
#endif
