// Decode attention over short ranges: no workgroup of the launch has more than KVQ_SHORT_TILES tiles, two per wavefront.
//
// What bounds such a launch is latency, a chain of trips to memory with little work in between, so this path is built
// to keep the chain short.  The parameters come in one go and stay in scalar registers; a wavefront knows its tiles from its
// index, reads their page entries itself, and issues the loads of its tiles before anything else, with no barrier, no
// staging and no claim in front; the queries go straight from memory into operand registers beside them; the two wavefronts
// with the fewest tiles take an appended token.  The end of a range is that of the streaming kernels (kvq_attention_body.h).
// Stamps, 3 tiles of 4 and 16 bits in each of 8 ranges x 8 units: page entries there at 0.6 us, loads out at 0.9, first
// tile there at 1.5, range done at 2.5, joined at 2.9 (streaming kernels: inputs staged at 0.9, range done at 4.0, joined at
// 4.9).  Launches in a train, streaming kernels and these: 764 tokens of 4 and 16 bits x 8 units 8.6 -> 6.7 us, with an appended
// token 8.5 -> 6.7, 2,500 tokens of 16 bits x 8 units 9.3 -> 6.5, one tile x one unit 5.1 -> 3.9; with 16-bit codes 764 tokens
// 9.5 -> 7.6.  The loads are streaming ones here too: plain ones are 0.4 us faster on blocks that lie in the L2 caches, but
// 0.2 us slower on blocks that come from memory.  A batch has kernels of its own, which find their parameters as the streaming ones do.
#include "kvq_attention_batch.h"

namespace {

// The parameters, all read at once: left alone the compiler reads them one by one where they are used first, each a trip of
// its own to the constant cache.  (A pointer that has gone through the registers of an asm is generic to the compiler, every
// access a flat one, behind which every wait is a wait for all loads: hence as_global.)
__device__ __forceinline__ KvqAttnHead read_head(const KvqAttnParams& params) {
    KvqAttnHead h = params;
    const _Float16* q = static_cast<const _Float16*>(h.q);
    float* out = static_cast<float*>(h.out);
    asm volatile("" : "+s"(h.arena), "+s"(h.table), "+s"(q), "+s"(h.lambda), "+s"(out), "+s"(h.part_o), "+s"(h.part_ml),
                      "+s"(h.counters), "+s"(h.v_mark), "+s"(h.v_tag), "+s"(h.n_tokens), "+s"(h.tiles_per_page),
                      "+s"(h.tpp_magic), "+s"(h.gqa), "+s"(h.n_q_heads), "+s"(h.n_kv_heads), "+s"(h.kv_magic),
                      "+s"(h.n_splits), "+s"(h.out_fp32), "+s"(h.fused_merge), "+s"(h.scale_log2),
                      "+s"(h.merge_groups), "+s"(h.merge_rounds), "+s"(h.gqa_magic));
    h.arena = as_global(h.arena); h.table = as_global(h.table); h.lambda = as_global(h.lambda);
    h.q = as_global(q); h.out = as_global(out);
    h.part_o = as_global(h.part_o); h.part_ml = as_global(h.part_ml);
    h.counters = as_global(h.counters); h.v_mark = as_global(h.v_mark);
    return h;
}

template <class T>
__device__ inline T scalar_load(const T* p) {  // through the constant cache; p uniform, not written by this launch (but for the mark, see kvq_v_marked)
    return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// Query operands arranged for tiles of width class CLS (load_q_ops) from a lane's own 8 channels of every group.
template <int CLS>
__device__ inline void arrange_q(QOps& Q, const u32x4 (&raw)[4]) {
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (CLS == 16) {
                Q.q[grp][v] = raw[grp][v];
            } else {
                const uint32_t w = __builtin_amdgcn_perm(raw[grp][2 + (v >> 1)], raw[grp][v >> 1], (v & 1) ? 0x07060302u : 0x05040100u);
                float f = 1.0f;
                if (CLS == 4) f = (v & 1) ? 0.0625f : 1.0f;
                if (CLS == 2) f = (v == 0) ? 1.0f : (v == 1) ? 0.25f : (v == 2) ? 0.0625f : 0.015625f;
                const half2v fs = {(_Float16)f, (_Float16)f};
                Q.q[grp][v] = f == 1.0f ? w : __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, w) * fs);
            }
        }
}
__device__ inline void sum_q(QOps& Q, const u32x4 (&raw)[4], int lane, float scale_log2) {
    const int j = lane >> 4;
    float sum[4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
        sum[grp] = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) sum[grp] += mixf(raw[grp][v], 0) + mixf(raw[grp][v], 1);
    }
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
        const float s = across_halves<Sum>(across_rows<Sum>(sum[grp])) * scale_log2;
        const _Float16 h = (_Float16)s, l = (_Float16)(s - (float)h);
        const uint32_t mine = (j == 0) ? __builtin_bit_cast(uint16_t, h) : (j == 1) ? __builtin_bit_cast(uint16_t, l) : 0u;
        if (grp & 1) Q.qsum[grp >> 1] |= mine << 16;
        else Q.qsum[grp >> 1] = mine;
    }
}

// A tile and, if n is 2, the one behind it, of the same width: all loads first, then the arithmetic.
struct TilePair { const uint8_t *code[2], *meta[2]; };
template <int B>
__device__ __forceinline__ void short_tiles(WaveState& st, QOps& Q, u32x4 (&qraw)[4], const TilePair& at, int n, int tile,
                                            uint8_t* meta_lds, int n_tokens, float scale_log2, int lane, bool fresh) {
    constexpr int W = code_bits<B>();
    asm volatile("" : "+v"(lane));  // what the widths derive from the lane index is not to be kept for all of them at once
    const uint32_t lane_off = 16u * lane;
    uint32_t kw[2][2 * W], vw[2][2 * W];
    u32x4 m[2];
    const auto load_k = [&](int k) {
        load_string<2 * W>(at.code[k], lane_off, kw[k]);
        if constexpr (has_meta<B>()) m[k] = load_stream16(at.meta[k] + lane_off);
    };
    const auto load_v = [&](int k) { load_string<2 * W>(at.code[k] + 512u * W, lane_off, vw[k]); };
    // Four strings of 16 bits at once are more registers than there are: of raw values the last one, of byte planes (whose
    // expansion takes more of them) the second tile's two follow where strings have been used up.
    load_k(0);
    load_v(0);
    if (n > 1) {
        if (B != KVQ_I16) load_k(1);
        if (W < 16) load_v(1);
    }
    asm volatile("" : "+s"(n));
    // (opaque: the operands of all widths would be arranged in front of the loads)
    asm volatile("" : "+v"(qraw[0]), "+v"(qraw[1]), "+v"(qraw[2]), "+v"(qraw[3]));
#ifdef KVQ_NO_ARITHMETIC  // every load issued and waited for in the same order, no tile computed on (kvq_attention_body.h)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k == 1 && n < 2) break;
        keep_loaded(kw[k]);
        if constexpr (has_meta<B>()) keep_loaded(m[k]);
        if (W == 16 && k == 0 && n > 1) {
            if (B == KVQ_I16) load_k(1);
            else load_v(1);
        }
        keep_loaded(vw[k]);
        if (B == KVQ_I16 && k == 0 && n > 1) load_v(1);
    }
#else
    arrange_q<q_class<B>()>(Q, qraw);
    if constexpr (has_meta<B>()) sum_q(Q, qraw, lane, scale_log2);
    if (fresh) st.oexp = v_exponent<B>(st.safe_v);
    else set_accumulator_exponent(st, v_exponent<B>(st.safe_v));
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        if (k == 1 && n < 2) break;
        __builtin_amdgcn_sched_barrier(0);  // (keeps the next tile's arithmetic out of this one's registers)
        if constexpr (has_meta<B>()) {
            *reinterpret_cast<u32x4*>(meta_lds + k * KVQ_META_TILE_BYTES + lane * 16) = m[k];
            wave_lds_sync();
        }
        float s[1][2][4];
        uint32_t pop[1][4];
        const int tok0[1] = {(tile + k) * KVQ_TILE_TOKENS};
        scores_tile<B>(Q, kw[k], meta_lds + k * KVQ_META_TILE_BYTES, scale_log2, lane, s[0]);
        if constexpr (W == 16) {
            if (k == 0 && n > 1) {
                asm volatile("" : "+v"(s[0][0][0]) :: "memory");
                if (B == KVQ_I16) load_k(1);
                else load_v(1);
            }
        }
        softmax_stage<B, 1>(st, s, tok0, n_tokens, lane, pop, k == 0 && fresh);
        if (B < 16 && st.safe_v) accumulate_tile<B, true>(st, vw[k], meta_lds + k * KVQ_META_TILE_BYTES, meta_lds + KVQ_WAVE_LDS_CONST, pop[0], lane);
        else accumulate_tile<B, false>(st, vw[k], meta_lds + k * KVQ_META_TILE_BYTES, meta_lds + KVQ_WAVE_LDS_CONST, pop[0], lane);
        if constexpr (B == KVQ_I16) {
            if (k == 0 && n > 1) {
                asm volatile("" : "+v"(st.o[7]) :: "memory");
                load_v(1);
            }
        }
    }
    if constexpr (has_meta<B>()) wave_lds_sync();
#endif
}

template <bool I16, int APPEND>
__device__ __forceinline__ void short_range(const KvqAttnHead& P, const int t_begin, const int t_end, const int split, const int unit,
                                            AttnShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane >> 4, n = lane & 15;
    const int b = div_magic(unit, P.n_kv_heads, P.kv_magic), hk = unit - b * P.n_kv_heads;
    KVQ_STAMP(0);
    KVQ_STAMP_ID();
    uint32_t mark = scalar_load(P.v_mark);
    // ---- the tiles of this wavefront: two where there are more than eight, but of 10 to 12 the first wavefronts take two and the
    // others one: wavefronts w and w + 4 share a SIMD, and six wavefronts of two tiles would give the first SIMDs four tiles where
    // three do (12 tiles of 4 bits x 256 units 8.0 -> 7.0 us, of 8 bits 9.1 -> 8.3, of 2 bits x 8 units 6.4 -> 5.6; streaming 7.6, 8.9 and
    // 7.1).  Of 9 or of 13 and more the fullest SIMD has three or four tiles either way, and byte planes, whose second tile follows the
    // first, take longer spread (9 tiles x 256 units 9.8 and 10.9 us).
    const int n_tiles = t_end - t_begin;
    // (wavefronts that take two, a digit for each number of tiles from 1 to 16; as compares and selects they cost steps 1 %)
    const int twos = (int)(0x8888432800000000ull >> (4 * ((n_tiles - 1) & 15))) & 15;
    int t = t_begin + wave + min(wave, twos);
    const int t_hi = min(t + 1 + (wave < twos ? 1 : 0), t_end);
    const int tpp = P.tiles_per_page;
    const u32x4* const table = reinterpret_cast<const u32x4*>(P.table);
    // page entries of the tile t and the one behind it, which may lie in the next page
    int tip = 0;
    u32x4 pd[2] = {};
    const auto look_up = [&]() {
        const int page = div_magic(t, tpp, P.tpp_magic);
        tip = t - page * tpp;
        pd[0] = pd[1] = scalar_load(table + page);
        if (t + 1 < t_hi && tip + 1 == tpp) pd[1] = scalar_load(table + page + 1);
    };
    if (t < t_hi) look_up();
    // ---- its queries: lane (j, n) takes channels 32 grp + 8 j .. + 7 of head n
    u32x4 qraw[4] = {};
    if (n < P.gqa) {
        const _Float16* row = static_cast<const _Float16*>(P.q) + ((size_t)b * P.n_q_heads + hk * P.gqa + n) * KVQ_D + 8 * j;
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) qraw[grp] = *reinterpret_cast<const u32x4*>(row + 32 * grp);
        if (P.lambda) {  // Q Lambda of the channel-wise reparameterization (Sec. 3.3, Eq. 7): fp32 product, RNE to fp16
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) qraw[grp] = __builtin_bit_cast(u32x4, kvq_dev::scale_keys8(qraw[grp], P.lambda + hk * KVQ_D + 32 * grp + 8 * j));
        }
    }
    // The last two wavefronts, which have the fewest tiles, take the appended token: its rows to LDS and, from the queries they
    // hold anyway, its scores.
    if (APPEND && P.app_t_old >= 0 && split == P.n_splits - 1 && wave >= KVQ_ATTN_WAVES - 2) {
        const int which = wave & 1;
        stage_new_token<I16, APPEND>(P, sh, unit, hk, which, lane);
        if (!which) {
            wave_lds_sync();
            float s = 0.f;
#pragma unroll
            for (int grp = 0; grp < 4; ++grp)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4v k = *reinterpret_cast<const float4v*>(&sh.new_x[0][32 * grp + 8 * j + 4 * h]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) s = fmaf(mixf(qraw[grp][2 * h + (i >> 1)], i & 1), k[i], s);
                }
            s = across_halves<Sum>(across_rows<Sum>(s));
            if (j == 0) sh.new_score[n] = s * P.scale_log2;
        }
    }
    uint8_t* const my_meta = sh.meta + wave * KVQ_WAVE_LDS_BYTES;
    if (lane < 8) reinterpret_cast<uint32_t*>(my_meta + KVQ_WAVE_LDS_CONST)[lane] = lane < 4 ? 0x3c003c00u : 0u;
    WaveState st;
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) st.o[nt] = float4v{0.f, 0.f, 0.f, 0.f};
    st.zl = float4v{0.f, 0.f, 0.f, 0.f};
    st.m = -INFINITY;
    st.oexp = 0;
    asm volatile("" : "+v"(st.o[0]), "+v"(st.o[1]), "+v"(st.o[2]), "+v"(st.o[3]), "+v"(st.o[4]), "+v"(st.o[5]), "+v"(st.o[6]),
                      "+v"(st.o[7]), "+v"(st.zl), "+v"(st.m));  // while the page entry is on its way
    asm volatile("" : "+s"(mark), "+s"(pd[0]), "+s"(pd[1]));
    st.safe_v = kvq_v_marked(mark, P.v_tag, APPEND == KVQ_APPEND_NARROW) ? 1 : 0;
    QOps Q;
    KVQ_STAMP(1);
    bool fresh = true;
    while (t < t_hi) {
        const uint32_t bits = pd[0].z;
        const int n = t + 1 < t_hi && pd[1].z == bits ? 2 : 1;
        TilePair at;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint64_t tslot = (uint64_t)unit * tpp + (k && tip + 1 < tpp ? tip + 1 : k ? 0 : tip);
            at.code[k] = P.arena + (uint64_t)pd[k].x * 256u + tslot * (1024u * bits);
            at.meta[k] = P.arena + (uint64_t)pd[k].y * 256u + tslot * KVQ_META_TILE_BYTES;
        }
        switch (bits) {
            case 16: short_tiles<I16 ? KVQ_I16 : 16>(st, Q, qraw, at, n, t, my_meta, P.n_tokens, P.scale_log2, lane, fresh); break;
            case 8: short_tiles<8>(st, Q, qraw, at, n, t, my_meta, P.n_tokens, P.scale_log2, lane, fresh); break;
            case 4: short_tiles<4>(st, Q, qraw, at, n, t, my_meta, P.n_tokens, P.scale_log2, lane, fresh); break;
            default: short_tiles<2>(st, Q, qraw, at, n, t, my_meta, P.n_tokens, P.scale_log2, lane, fresh); break;
        }
        t += n;
        fresh = false;
        if (t < t_hi) look_up();
    }
    KVQ_STAMP(2);
    // (the thread index is put together again: kept across the tiles it would be a register too many)
    int zero = 0;
    asm volatile("" : "+v"(zero));
    finish_workgroup<I16, APPEND, true>(P, sh, st, split, unit, 64 * wave + (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (uint32_t)zero)));
}

template <bool I16, int APPEND>
__device__ __forceinline__ void short_body(const KvqAttnParams& params, AttnShared& sh) {
    const int split = blockIdx.x, unit = blockIdx.y;
    const int t_begin = params.split_begin[split], t_end = params.split_begin[split + 1];
    const KvqAttnHead P = read_head(params);
    short_range<I16, APPEND>(P, t_begin, t_end, split, unit, sh);
}
// A ragged batch all of whose ranges are short.
template <bool I16>
__device__ __forceinline__ void short_batch_body(const KvqAttnParams* __restrict__ params, const KvqBatchMap& map, AttnShared& sh,
                                                 uint32_t (&block)[kBlockDwords]) {
    BatchWork work;
    const KvqAttnHead P = batch_work(params, map, block, work);
    short_range<I16, KVQ_APPEND_16>(P, work.t_begin, work.t_end, work.split, work.unit, sh);
}

__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    short_body<false, 0>(P, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_append_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    short_body<false, KVQ_APPEND_16>(P, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_i16_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    short_body<true, 0>(P, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_i16_append_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    short_body<true, KVQ_APPEND_16>(P, sh);
}

__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_append_narrow_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    short_body<false, KVQ_APPEND_NARROW>(P, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_i16_append_narrow_kernel(const KvqAttnParams P) {
    __shared__ AttnShared sh;
    short_body<true, KVQ_APPEND_NARROW>(P, sh);
}

template <bool I16>
__device__ __forceinline__ void short_batch_body(const KvqBatchArgs& args, AttnShared& sh) {
    BatchWork work;
    const KvqAttnHead P = batch_work<true>(args, work);
    short_range<I16, KVQ_APPEND_16>(P, work.t_begin, work.t_end, work.split, work.unit, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_batch_args_kernel(const KvqBatchArgs args) {
    __shared__ AttnShared sh;
    short_batch_body<false>(args, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_batch_args_i16_kernel(const KvqBatchArgs args) {
    __shared__ AttnShared sh;
    short_batch_body<true>(args, sh);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_batch_kernel(const KvqAttnParams* __restrict__ params,
                                                                                     const KvqBatchMap map) {
    __shared__ AttnShared sh;
    __shared__ uint32_t block[kBlockDwords];
    short_batch_body<false>(params, map, sh, block);
}
__global__ __launch_bounds__(KVQ_ATTN_THREADS) void kvq_attention_short_batch_i16_kernel(const KvqAttnParams* __restrict__ params,
                                                                                         const KvqBatchMap map) {
    __shared__ AttnShared sh;
    __shared__ uint32_t block[kBlockDwords];
    short_batch_body<true>(params, map, sh, block);
}

}  // namespace

hipError_t kvq_launch_attention_short_batch(const KvqBatchArgs& args, bool int16, hipStream_t s) {
    const dim3 grid(args.wg_begin[args.n]), block(KVQ_ATTN_THREADS);
    if (int16) hipLaunchKernelGGL(kvq_attention_short_batch_args_i16_kernel, grid, block, 0, s, args);
    else hipLaunchKernelGGL(kvq_attention_short_batch_args_kernel, grid, block, 0, s, args);
    return hipGetLastError();
}
hipError_t kvq_launch_attention_short_batch(const KvqAttnParams* params_dev, const KvqBatchMap& map, bool int16, hipStream_t s) {
    const dim3 grid(map.wg_begin[map.n]), block(KVQ_ATTN_THREADS);
    if (int16) hipLaunchKernelGGL(kvq_attention_short_batch_i16_kernel, grid, block, 0, s, params_dev, map);
    else hipLaunchKernelGGL(kvq_attention_short_batch_kernel, grid, block, 0, s, params_dev, map);
    return hipGetLastError();
}
hipError_t kvq_launch_attention_short(const KvqAttnParams& p, int units, hipStream_t s) {
    const dim3 grid(p.n_splits, units), block(KVQ_ATTN_THREADS);
    const bool append = p.app_t_old >= 0;
    if (append && p.app_desc.bits < 16) {
        if (p.int16_tier) hipLaunchKernelGGL(kvq_attention_short_i16_append_narrow_kernel, grid, block, 0, s, p);
        else hipLaunchKernelGGL(kvq_attention_short_append_narrow_kernel, grid, block, 0, s, p);
    } else if (p.int16_tier && append) hipLaunchKernelGGL(kvq_attention_short_i16_append_kernel, grid, block, 0, s, p);
    else if (p.int16_tier) hipLaunchKernelGGL(kvq_attention_short_i16_kernel, grid, block, 0, s, p);
    else if (append) hipLaunchKernelGGL(kvq_attention_short_append_kernel, grid, block, 0, s, p);
    else hipLaunchKernelGGL(kvq_attention_short_kernel, grid, block, 0, s, p);
    return hipGetLastError();
}
#ifdef KVQ_PHASE_STAMPS
// Measurement build only: the stamps of the last launch of these kernels.
extern "C" int kvq_phase_stamps_read_short(unsigned long long* host) {
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(kvq_phase_stamps), sizeof(unsigned long long) * KVQ_STAMP_WGS * KVQ_STAMP_SLOTS);
}
#endif
