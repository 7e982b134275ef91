// The streaming attention kernels with a one-token append into a page of 8, 4 or 2 bits in front (a decode step of a block without a
// window that has been shrunk).  A translation unit of their own: kernels added to a unit change the inlining of the others.
// What bounds it is what bounds the step's other kernels; the token costs two wavefronts some 0.5 us before the join and its elements go
// out behind it.  Appended by a launch of its own it cost 3.4 to 4.3 us a step (steps in a train, two launches and now): 764 tokens of 4 bits
// x 8 units 10.3 and 6.9 us, 1,000 of 2 bits x 2 10.1 and 6.7, 16,000 of 4 bits x 16 17.9 and 14.1, 8,192 of 8 bits x 32 22.6 and 18.4;
// prompts of 16,000 x 16 and 8,192 x 32 with their first step 150.9 and 146.7, 117.9 and 114.8.
#include "kvq_attention_body.h"

namespace {

__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_append_narrow_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    attention_body<false, false, KVQ_APPEND_NARROW>(P, P.split_begin[blockIdx.x], P.split_begin[blockIdx.x + 1], sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_i16_append_narrow_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    attention_body<true, false, KVQ_APPEND_NARROW>(P, P.split_begin[blockIdx.x], P.split_begin[blockIdx.x + 1], sh);
}

}  // namespace

hipError_t kvq_launch_attention_append_narrow(const KvqAttnParams& p, int units, hipStream_t s) {
    const dim3 grid(p.n_splits, units), block(KVQ_ATTN_THREADS);
    if (p.int16_tier) hipLaunchKernelGGL(kvq_attention_i16_append_narrow_kernel, grid, block, 0, s, p);
    else hipLaunchKernelGGL(kvq_attention_append_narrow_kernel, grid, block, 0, s, p);
    return hipGetLastError();
}
