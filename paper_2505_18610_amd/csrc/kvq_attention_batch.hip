// Decode attention over a ragged batch: grid.x = sum over the caches of splits * units.  A workgroup looks its cache
// up in the map, takes that cache's parameter block (read-only for the whole launch) and runs the
// same body as the single-cache kernels.
#include "kvq_attention_body.h"

namespace {

// The parameter block of the workgroup's cache lies in host memory.  It is fetched over the link once, a dword per thread, and
// handed out from LDS: the head as scalars (read lane by lane from one register), the range of the split by index.  (Read
// field by field as the kernel comes to them, the blocks cost two to three dependent trips over the link.)
constexpr int kHeadDwords = sizeof(KvqAttnHead) / 4, kBlockDwords = sizeof(KvqAttnParams) / 4;
static_assert(kBlockDwords - kHeadDwords == KVQ_MAX_SPLITS + 1 + (KVQ_MAX_SPLITS + 1) % 2, "split_begin follows the head (padded to 8 bytes)");
static_assert(kHeadDwords <= 64 && kBlockDwords <= KVQ_ATTN_THREADS && sizeof(KvqAttnHead) % 8 == 0, "one dword per lane, one per thread");
struct HeadWords { uint32_t w[kHeadDwords]; };

template <bool I16>
__device__ __forceinline__ void batch_body(const KvqAttnParams* __restrict__ params, const KvqBatchMap& map, AttnShared& sh,
                                           uint32_t (&block)[kBlockDwords]) {
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
    const int unit = local / P.n_splits, split = local - unit * P.n_splits;  // splits of a unit are neighbours
    const int* split_begin = reinterpret_cast<const int*>(block + kHeadDwords);
    attention_body<I16, true, true>(P, __builtin_amdgcn_readfirstlane(split_begin[split]),
                                    __builtin_amdgcn_readfirstlane(split_begin[split + 1]), sh, split, unit);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_batch_kernel(const KvqAttnParams* __restrict__ params,
                                                                               const KvqBatchMap map) {
    __shared__ AttnShared sh;
    __shared__ uint32_t block[kBlockDwords];
    batch_body<false>(params, map, sh, block);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_batch_i16_kernel(const KvqAttnParams* __restrict__ params,
                                                                                   const KvqBatchMap map) {
    __shared__ AttnShared sh;
    __shared__ uint32_t block[kBlockDwords];
    batch_body<true>(params, map, sh, block);
}

}  // namespace

hipError_t kvq_launch_attention_batch_kernel(const KvqAttnParams* params_dev, const KvqBatchMap& map, bool int16,
                                             hipStream_t s) {
    const int wgs = map.wg_begin[map.n];
    if (int16) hipLaunchKernelGGL(kvq_attention_batch_i16_kernel, dim3(wgs), dim3(KVQ_ATTN_THREADS), 0, s, params_dev, map);
    else hipLaunchKernelGGL(kvq_attention_batch_kernel, dim3(wgs), dim3(KVQ_ATTN_THREADS), 0, s, params_dev, map);
    return hipGetLastError();
}
