// What a workgroup of a ragged batch works on: its cache's parameters, its unit and split, its tiles.
#ifndef KVQ_ATTENTION_BATCH_H
#define KVQ_ATTENTION_BATCH_H
#include "kvq_attention_body.h"

namespace {

// The parameter block of the workgroup's cache lies in host memory.  It is fetched over the link once, a dword per thread, and
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

}  // namespace
#endif
