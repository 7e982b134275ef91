// Decode attention over a ragged batch: grid.x = sum over the caches of splits * units.  A workgroup looks its cache
// up in the map, takes that cache's parameter block (read-only for the whole launch) and runs the
// same body as the single-cache kernels.
#include "kvq_attention_batch.h"

namespace {

template <bool I16>
__device__ __forceinline__ void batch_body(const KvqAttnParams* __restrict__ params, const KvqBatchMap& map, AttnShared& sh,
                                           uint32_t (&block)[kBlockDwords]) {
    BatchWork work;
    const KvqAttnHead P = batch_work(params, map, block, work);
    attention_body<I16, true, KVQ_APPEND_16>(P, work.t_begin, work.t_end, sh, work.split, work.unit);
}
template <bool I16>
__device__ __forceinline__ void batch_body(const KvqBatchArgs& args, AttnShared& sh) {
    BatchWork work;
    const KvqAttnHead P = batch_work<false>(args, work);
    attention_body<I16, true, KVQ_APPEND_16>(P, work.t_begin, work.t_end, sh, work.split, work.unit);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_batch_args_kernel(const KvqBatchArgs args) {
    __shared__ AttnShared sh;
    batch_body<false>(args, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_batch_args_i16_kernel(const KvqBatchArgs args) {
    __shared__ AttnShared sh;
    batch_body<true>(args, sh);
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

hipError_t kvq_launch_attention_batch_kernel(const KvqBatchArgs& args, bool int16, hipStream_t s) {
    const dim3 grid(args.wg_begin[args.n]), block(KVQ_ATTN_THREADS);
    if (int16) hipLaunchKernelGGL(kvq_attention_batch_args_i16_kernel, grid, block, 0, s, args);
    else hipLaunchKernelGGL(kvq_attention_batch_args_kernel, grid, block, 0, s, args);
    return hipGetLastError();
}
hipError_t kvq_launch_attention_batch_kernel(const KvqAttnParams* params_dev, const KvqBatchMap& map, bool int16,
                                             hipStream_t s) {
    const int wgs = map.wg_begin[map.n];
    if (int16) hipLaunchKernelGGL(kvq_attention_batch_i16_kernel, dim3(wgs), dim3(KVQ_ATTN_THREADS), 0, s, params_dev, map);
    else hipLaunchKernelGGL(kvq_attention_batch_kernel, dim3(wgs), dim3(KVQ_ATTN_THREADS), 0, s, params_dev, map);
    return hipGetLastError();
}
