// Quantize-on-append, fp16 -> b-bit page quantization and the Equivalent Right Shift kernels (gfx950).
//
// Quantizer: Sec. 2.2 Eq. 1-2 (asymmetric min-max per group of 32 channels of one token of one KV head).
// Shrinking: Sec. 3.1 Eq. 3 with S_b = (2^b + 1) S_2b and Z kept.
// All kernels work directly in the tile layout described in kvq_layout.h: one wavefront owns one tile and
// every lane quantizes the 64 slots it will later feed to the matrix cores.
#include "kvq_quant_dev.h"

#include <type_traits>

#include <algorithm>

namespace {

using namespace kvq_q;
using kvq_dev::div_magic;
using kvq_dev::as_global;

// Work of the append kernels: one wavefront per string, a (tile, K | V) of one (sequence, KV head) unit; the WAVES
// wavefronts of a workgroup take neighbouring strings of a unit and share nothing.  PLAIN instantiations serve keys that
// arrive rotated in a block without reparameterization (rope and rinv are null): they carry none of that code, which is
// the bulk of the general kernels' registers.
// by_unit: the units of a string follow one another in the grid instead of the strings of a unit.  The table rows of the
// string's tokens, 512 bytes a token and as much as its keys and values in one unit, are then read by all units at about
// the same time and come from the caches.  For the raw 16-bit tier, 32 units and more and at least 98,304 rows of all units together.
// Rotated keys, with and without, over the same input / from memory: 2,048 x 64 25.6 and 27.7 / 27.5 and 30.4 us, 4,096 x 128 84
// and 90 / 99 and 103; of 32 units what memory gains outweighs what the caches lose, 4,096 x 32 25.6 and 25.0 / 28.6 and 30.1, scaled too
// 26.3 and 26.7 / 28.8 and 31.9, 8,192 x 32 46.3 and 44.4 / 51.7 and 54.0, scaled too 46.4 and 45.7 / 53.0 and 55.7; of fewer it loses, 16,384
// x 16 50.5 and 43.3 / 54.4 and 52.0, x 8 30.8 and 24.2 / 32.0 and 27.8; 1,024 x 64 (65,536 rows) 14.4 and 14.5 / 15.9 and 17.6.  Into the
// integer tier it loses: 4,096 x 128 113 and 108 / 112 and 109, 2,048 x 64 25.0 and 24.3 / 32.7 and 31.0, 8,192 x 8 17.9 and 15.1.  Into 8,
// 4 and 2 bits, where the arithmetic weighs more, it loses 3 to 7 % at every size.
// What a launch's kernels need, read at once at their start: left alone the compiler reads the arguments one by one where they
// are used first, each a trip to the constant cache or beyond, and three quotients and the lookup of the page entry stood in
// front of the rows as well.  Now rows and angles are asked for first and the page entry behind them, needed only for the stores.
// Kernel times before and after: 1,024 tokens x 16 units, rotated, into 8 / 4 bits 6.76 / 6.84 and 6.32 / 6.48 us; 2,500 x 8 at
// 16 bits 6.88 and 6.64; 2,048 x 32, rotated and scaled, into 8 / 4 / 2 bits 15.4 / 15.0 / 14.9 and 13.3 / 13.3 / 13.1 and into the
// integer tier 24.5 and 20.9; keys that need no preparation 1 to 3 % (64 units x 2,048 at 16 bits 21.8 and 22.1).
struct AppendArgs {
    uint8_t* arena;
    KvqPageDesc* table;
    const uint16_t *k, *v;
    const float *rinv, *rope;
    uint32_t* v_word;
    int32_t t_old, n_new, tpp;
    uint32_t tpp_magic;
    int32_t tile0, n_strings, by_unit, n_kv_heads;
    uint32_t kv_magic, v_epoch;
    int32_t gspan;
    int32_t stream_v;  // see append16_v_tile
    KvqAppendPages pages;
};
struct AppendString {  // one wavefront's string
    int which, unit, tile, page;
    uint64_t tslot;
    const float* rinv_head;
};
template <bool PLAIN>
__device__ __forceinline__ void read_append_args(const AppendArgs& args, AppendArgs& A) {
    uint8_t* arena = args.arena;
    KvqPageDesc* table = args.table;
    const uint16_t *k = args.k, *v = args.v;
    const float *rinv = args.rinv, *rope = args.rope;
    uint32_t* word = args.v_word;
    A.t_old = args.t_old; A.n_new = args.n_new; A.tpp = args.tpp; A.tpp_magic = args.tpp_magic; A.tile0 = args.tile0;
    A.n_strings = args.n_strings; A.by_unit = args.by_unit; A.n_kv_heads = args.n_kv_heads; A.kv_magic = args.kv_magic;
    A.v_epoch = args.v_epoch; A.gspan = args.gspan; A.stream_v = args.stream_v;
    asm volatile("" : "+s"(arena), "+s"(table), "+s"(k), "+s"(v), "+s"(word), "+s"(A.t_old), "+s"(A.n_new), "+s"(A.tpp), "+s"(A.tpp_magic),
                      "+s"(A.tile0), "+s"(A.n_strings), "+s"(A.v_epoch), "+s"(A.gspan), "+s"(A.stream_v));
    if constexpr (!PLAIN) asm volatile("" : "+s"(rinv), "+s"(rope), "+s"(A.by_unit), "+s"(A.n_kv_heads), "+s"(A.kv_magic));
    A.arena = as_global(arena); A.table = as_global(table); A.k = as_global(k); A.v = as_global(v);
    A.rinv = as_global(rinv); A.rope = as_global(rope); A.v_word = as_global(word);
}
template <bool PLAIN, int WAVES>
__device__ __forceinline__ bool append_string(const AppendArgs& A, int wave, AppendString& t) {
    int s = blockIdx.x;
    t.unit = blockIdx.y;
    if (!PLAIN && A.by_unit) { const int q = s / A.by_unit; t.unit = s - q * A.by_unit; s = q; }
    const int string = s * WAVES + wave;
    t.which = string & 1;
    t.tile = A.tile0 + (string >> 1);
    t.page = div_magic(t.tile, A.tpp, A.tpp_magic);
    t.tslot = (uint64_t)t.unit * A.tpp + (t.tile - t.page * A.tpp);
    t.rinv_head = nullptr;
    if (!PLAIN && A.rinv) t.rinv_head = A.rinv + (t.unit - div_magic(t.unit, A.n_kv_heads, A.kv_magic) * A.n_kv_heads) * KVQ_D;
    return string < A.n_strings;
}

// Append into the 16-bit tier: the new rows are copied into the tile layout.  A workgroup is a tile, its first wavefront the keys and
// its second the values.  Workgroups go to the eight XCDs in turn: with one string each, keys and values in turn, all keys, which
// are rotated and scaled, were on every other XCD and the others had little to do.  One wavefront a workgroup and now: 1,024 tokens x
// 16 units rotated 6.1 and 5.1 us, 2,500 x 8 7.0 and 6.0, 1,024 x 32 9.3 and 7.5, 2,048 x 32 15.4 and 14.3, neither rotated nor scaled
// 2,500 x 8 4.4 and 4.1, 1,024 x 32 5.5 and 5.0; 3,840 to 4,224 strings of such keys take 0.3 us longer over a repeated input, 2,048 x 32 10.0 and
// 10.3, and the same from memory, 16.1 and 16.2.
// FIVE: with 92 registers five wavefronts fit on a SIMD, otherwise, with 104, four.  Scaled keys of 4,097 to 4,608 and 5,121 to 5,632
// strings, the odd steps of half a wavefront a SIMD beyond four, end earlier with five (16 units x 144 tiles 16.4 us and 17.8, from memory
// 18.1 and 19.4; x 164 19.1 and 19.2, 19.2 and 20.1); 4,992 strings are alike, and keys that are only rotated lose 1 to 4 % of it.
template <bool PLAIN, bool FIVE>
__global__ __launch_bounds__(128) void kvq_append16_kernel(const AppendArgs args) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[32 * 256];  // of the wavefront with the values
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    AppendArgs A;
    read_append_args<PLAIN>(args, A);
    AppendString t;
    append_string<PLAIN, 2>(A, wave, t);  // (the number of strings is even)
    const kvq_dev::NewRows rows((t.which ? A.v : A.k) + (uint64_t)t.unit * A.n_new * KVQ_D, A.t_old, A.n_new);
    const int tok0 = t.tile * KVQ_TILE_TOKENS;
    // the page entry is looked up behind the loads of the rows
    const auto code = [&]() {
        const KvqPageDesc pd = append_desc<false>(A.table, args.pages, t.page);
        return A.arena + (uint64_t)pd.code_off256 * 256u + (t.tslot * 2 + t.which) * (512u * 16);
    };
    if (t.which) kvq_dev::append16_v_tile<8>(code, rows, tok0, lane, lds, A.stream_v, 0);  // (wavefront-uniform)
    else kvq_dev::append16_k_tile<FIVE, 2>(code, rows, tok0, lane, PLAIN ? nullptr : A.rope, PLAIN ? nullptr : t.rinv_head, 0);
    if (wave == 1) write_fresh_pages(A.table, args.pages, lane);
}
// The same for keys that need no preparation and more than 16,384 strings.  Two tiles a workgroup, half as many workgroups to
// dispatch: one tile a workgroup and two, over the same input / from memory, 4,096 tokens x 96 units (24,576 strings) 62.6 and 60.7 us / 76.7
// and 76.4, 8,192 x 64 88.8 and 81.0 / 104 and 101, 4,096 x 128 92 and 88 / 113 and 107; 4,096 x 64 (16,384) 40.0 and 40.0 / 55.1 and 55.8.  One string a
// workgroup beyond that: with two tiles and one string, 8,192 x 64 (32,768) 81.2 and 88.4 / 101 and 101, 10,240 x 64 (40,960) 104 and
// 108 / 126 and 126, 12,288 x 64 (49,152) 129.0 and 127.4 / 149 and 146, 14,336 x 64 151.5 and 147.9 / 173 and 170.6, 8,192 x 128 216 and 205 /
// 221 and 218, 16,384 x 64 183.6 and 180.6 / 196 and 193, 16,384 x 128 450 and 435 / 433 and 424.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void kvq_append16_bulk_kernel(const AppendArgs args) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[(WAVES + 1) / 2][32 * 256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    AppendArgs A;
    read_append_args<true>(args, A);
    AppendString t;
    const bool mine = append_string<true, WAVES>(A, wave, t);
    if (wave == (WAVES > 1 ? 1 : 0)) write_fresh_pages(A.table, args.pages, lane);
    if (!mine) return;
    const kvq_dev::NewRows rows((t.which ? A.v : A.k) + (uint64_t)t.unit * A.n_new * KVQ_D, A.t_old, A.n_new);
    const int tok0 = t.tile * KVQ_TILE_TOKENS;
    const auto code = [&]() {
        const KvqPageDesc pd = append_desc<false>(A.table, args.pages, t.page);
        return A.arena + (uint64_t)pd.code_off256 * 256u + (t.tslot * 2 + t.which) * (512u * 16);
    };
    if (t.which) kvq_dev::append16_v_tile<8>(code, rows, tok0, lane, lds[wave >> 1], A.stream_v, 0);
    else kvq_dev::append16_k_tile<false, 2>(code, rows, tok0, lane, nullptr, nullptr, 0);
}
// The same with two wavefronts per string, which share nothing: of keys each takes 16 tokens, of values 64 channels.  For less
// than 1,024 strings, launches that leave SIMDs without a wavefront otherwise, where the chain of one is what counts.  One wavefront per
// string and two, over the same input / from memory: rotated and scaled, 64 tokens x 8 units 3.8 and 3.5 us / 3.8 and 3.6, 700 x 8 4.2 and
// 3.9 / 4.3 and 4.1, 1,500 x 8 5.1 and 4.9 / 5.5 and 5.4, 1,024 x 16 (1,024 strings) 5.6 and 5.4 / 5.6 and 5.9, 1,536 x 16 6.4 and 6.3 / 6.9 and
// 7.6; neither, 64 x 8 2.9 and 2.7 / 2.9 and 2.8, 1,500 x 8 alike, 1,280 x 8 3.6 and 3.6 / 4.5
// and 4.2, 1,536 x 16 4.2 and 4.6 / 5.3 and 5.6.
template <bool PLAIN>
__global__ __launch_bounds__(256) void kvq_append16_pair_kernel(const AppendArgs args) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][32 * 128];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave & 1;
    AppendArgs A;
    read_append_args<PLAIN>(args, A);
    AppendString t;
    append_string<PLAIN, 2>(A, wave >> 1, t);
    const kvq_dev::NewRows rows((t.which ? A.v : A.k) + (uint64_t)t.unit * A.n_new * KVQ_D, A.t_old, A.n_new);
    const int tok0 = t.tile * KVQ_TILE_TOKENS;
    const auto code = [&]() {
        const KvqPageDesc pd = append_desc<false>(A.table, args.pages, t.page);
        return A.arena + (uint64_t)pd.code_off256 * 256u + (t.tslot * 2 + t.which) * (512u * 16);
    };
    if (t.which) kvq_dev::append16_v_tile<4>(code, rows, tok0, lane, lds[half], A.stream_v, 4 * half);
    else kvq_dev::append16_k_tile<false, 1>(code, rows, tok0, lane, PLAIN ? nullptr : A.rope, PLAIN ? nullptr : t.rinv_head, half);
    if (wave == 3) write_fresh_pages(A.table, args.pages, lane);
}

// Quantizing append (B = 8, 4, 2), built on the row-owner core.
// Four wavefronts per workgroup, each with a string and LDS of its own: 1 to 2 % faster on bulk appends than one-wavefront
// workgroups (a quarter of the workgroups to dispatch).
#define KVQ_APPEND_WG_WAVES 4
// PAIR: two wavefronts per string, one for each 16 tokens, two strings per workgroup.  A launch of one or two strings per
// SIMD (1,024 of them) leaves each alone with some 1,000 to 1,700 vector instructions; shared by two it ends earlier, and with half
// the registers for its rows (88 instead of 112 with angles) more of it fits on a SIMD.  What a pair costs: factors are read twice,
// and each wavefront gathers the whole string's codes to store half of them (into 2 bits, one chunk a lane, one stores all).
// kvq_pair_strings draws the line: by how the 1,024 SIMDs fill, in steps of 1,024 strings with one wavefront each and of 512 with two.
// Time of two wavefronts per string over that of one, launches in a train, 16 units x 32 to 110 tiles, over the same input, which the
// caches hold / over inputs in turn from memory:
//   into 8 / 4 / 2 bits            2,080 to 2,560 strings                       2,624 to 3,008                               3,136 to 3,520
//   neither rotated nor scaled     0.90, 0.98, 0.87 / 0.88 to 1.01, 0.95, 0.86  0.96, 1.06, 0.95 / 1.07, 1.00, 0.92  0.91, 1.03, 0.89 / 0.96, 0.93, 0.87
//   rotated                        0.85, 0.90, 0.83 / 0.83 to 0.93, 0.89, 0.82  0.91, 0.98, 0.87 / 1.02, 0.94, 0.88  0.90, 0.94, 0.85 / 0.90, 0.91, 0.86
//   scaled                         0.96, 0.99, 0.93 / 0.94, 0.98, 0.90          1.19, 1.21, 1.09 / 1.21, 1.14, 1.05  1.13, 1.17, 1.06 / 1.03, 1.09, 1.03
//   both                           0.95, 0.98, 0.92 / 0.92, 0.95, 0.89          1.02, 1.05, 0.99 / 1.04, 1.00, 0.97  1.00, 1.03, 0.95 / 0.98, 0.97, 0.93
// 2,048 and 3,072 fill the SIMDs without a rest either way: 1.03 to 1.30 / 0.98 to 1.25 of 4 bits or scaled.  Below 1,600 all but one of
// these gain, up to 26 %.  3,500 to 40,000 strings: 8 bits 0.90 to 1.05 / 0.92 to 0.98, 4 bits 0.92 to 1.07 / 0.92 to 0.99, scaled ones from
// memory 1.00 to 1.07, rotated ones by how often the table is read.
static bool kvq_pair_strings(int bits, int64_t strings, bool rotated, bool scaled) {
    if (bits == 4 || scaled) return strings != 2048 && strings < (scaled && !rotated ? 2561 : 3072);
    return bits == 2 || rotated || strings < 4608;
}
template <int B, bool PLAIN, bool PAIR>
__global__ __launch_bounds__(64 * KVQ_APPEND_WG_WAVES) void kvq_append_q_kernel(const AppendArgs args) {
    __shared__ __attribute__((aligned(16))) uint8_t lds_all[KVQ_APPEND_WG_WAVES][KVQ_LDS_CODES];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const lds = lds_all[PAIR ? wave >> 1 : wave];
    const int lane = threadIdx.x & 63, j = lane >> 4, n = lane & 15;
    AppendArgs A;
    read_append_args<PLAIN>(args, A);
    AppendString t;
    // (the number of strings is even: with pairs every workgroup has two, K and V of one tile)
    const bool mine = append_string<PLAIN, PAIR ? 2 : KVQ_APPEND_WG_WAVES>(A, PAIR ? wave >> 1 : wave, t);
    if (wave == 0) write_fresh_pages(A.table, args.pages, lane);
    if (!mine) return;
    const int which = t.which, t_old = A.t_old, gspan = A.gspan;
    const KvqVMark mark{A.v_word, A.v_epoch};
    const int tok0 = t.tile * KVQ_TILE_TOKENS;
    const kvq_dev::NewRows rows((which ? A.v : A.k) + (uint64_t)t.unit * A.n_new * KVQ_D, t_old, A.n_new);
    const int grp = lane & 3;
    constexpr int PASSES = PAIR ? 1 : 2;
    const int pass0 = PAIR ? wave & 1 : 0;
    uint32_t w[PASSES][16];
    load_owner_rows(w, rows, tok0 + 16 * pass0, lane);
    const bool rotates = !PLAIN && !which && A.rope;
    OwnerAngles angles;
    if (rotates) load_owner_angles(angles, rows, tok0 + 16 * pass0 + (lane >> 2), lane, A.rope);
    __builtin_amdgcn_sched_barrier(0);  // all of these loads first
    const KvqPageDesc pd = append_desc<PLAIN>(A.table, args.pages, t.page);
    uint8_t* code = A.arena + (uint64_t)pd.code_off256 * 256u + (t.tslot * 2 + which) * (512u * B);
    uint8_t* meta = A.arena + (uint64_t)pd.meta_off256 * 256u + t.tslot * KVQ_META_TILE_BYTES;
    if (rotates) {
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const int tok = tok0 + 16 * (pass0 + pass) + (lane >> 2);
            if (pass) load_owner_angles(angles, rows, tok, lane, A.rope);
            rotate_owner_keys(w[pass], angles, rows.has(tok), rows.all(tok0), lane);
        }
    }
    if (!PLAIN && !which && t.rinv_head) {
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) scale_owner_keys(w[pass], lane, t.rinv_head);
    }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        const int tl = 16 * (pass0 + pass) + (lane >> 2);
        const int tok = tok0 + tl;
        uint32_t codes[32];
        uint16_t S, Z;
        quantize_owner<B>(w[pass], codes, &S, &Z, gspan);  // tokens that are not new quantize zeros: codes 0, S = Z = 0
        note_large_v_scale(mark, which, S);
        scatter_codes(lds, which, tl, grp, codes);
        if (tok >= t_old) store_meta_owner(meta, which, tl, grp, S, Z);
    }
    if (PAIR) __syncthreads();
    else wave_sync_lds();
    if (PAIR && (B == 2 || tok0 < t_old) && pass0 != 0) return;  // one chunk, or one merged with stored tokens: no halves
    uint32_t str[2 * B];
    gather_string<B>(lds, which, lane, str);
    // stored tokens keep their bits
    uint32_t keep = 0;
    if (!which) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
            if (tok0 + 8 * (n >> 2) + 4 * sub + (n & 3) < t_old) keep |= 1u << sub;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (tok0 + 8 * j + i < t_old) keep |= 1u << i;
    }
    if (tok0 < t_old) {  // (wavefront-uniform) the tile already holds tokens: it is rewritten step by step, plain stores
        if (keep) {
            uint32_t old[2 * B];
            load_chunks<B>(code, lane, old);
#pragma unroll
            for (int d = 0; d < 2 * B; ++d) {
                uint32_t m = which ? v_token_mask<B>(keep, d) : (((keep >> (d / B)) & 1u) ? 0xffffffffu : 0u);
                str[d] = (old[d] & m) | (str[d] & ~m);
            }
        }
        store_chunks<B>(code, lane, str);
        asm volatile("" ::: "memory");  // keeps the two kinds of store apart (merged, they would both be plain ones)
        return;
    }
    // a tile made of new tokens only is written once and read much later: streaming stores (with plain stores the
    // bulk appends run a quarter slower)
    if constexpr (PAIR && B > 2) {  // each wavefront of the pair stores half of the string's chunks
        constexpr int HALF = B / 4;
        const uint32_t second = pass0 ? 0xffffffffu : 0u;
#pragma unroll
        for (int c = 0; c < HALF; ++c) {
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (str[4 * c + e] & ~second) | (str[4 * (c + HALF) + e] & second);
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(code + ((c + HALF * pass0) * 64 + lane) * 16));
        }
    } else {
        store_chunks_stream<B>(code, lane, str);
    }
}

// Append into the integer 16-bit tier: Eq. 1-2 with 2^16 - 1 levels by the same owner lanes; the high and the low
// bytes of the codes then travel through LDS and into the tile's two byte planes like two 8-bit tiles.
// A workgroup is a tile (see kvq_append16_kernel).  Two wavefronts share a string: each quantizes 16 tokens and then writes one
// plane; with 90 registers instead of 111 one more of them fits on a SIMD, and the chain of a small launch is half as long.  A
// workgroup of one string and one wavefront, and now, over the same input / from memory: rotated 64 tokens x 8 units 5.2 and 4.5 us,
// 1,024 x 16 7.8 and 7.0 / 8.7 and 7.4, 1,280 x 32 13.2 and 10.7 / 14.5 and 11.4, 2,048 x 32 18.0 and 14.8 / 21.1 and 18.3, 2,048 x 64
// 27.4 and 24.3 / 35.8 and 31.0, 4,096 x 128 116 and 108; rotated and scaled 2,048 x 32 20.2 and 18.0 / 23.0 and 20.0; neither 1,024 x 16
// 6.6 and 6.2 / 7.0 and 6.7, 2,048 x 32 14.3 and 13.8 / 17.4 and 17.3, 2,048 x 64 23.0 and 22.4 / 29.6 and 28.4.  (A wavefront a string and a
// tile a workgroup: 3 to 14 % behind that, but for 4,096 strings of scaled keys, 16.5 / 18.3.)
// SHARE: how many wavefronts share a string.  Ready keys of more than 32,768 strings take one, a workgroup each: with two and one,
// 8,192 x 64 (32,768) 106.8 and 107.1 / 106 and 107, 6,144 x 96 117.7 and 116.9 / 117.6 and 118.3, 5,120 x 128 (40,960) 139.5 and 132.8 / 136 and 135, 12,288 x
// 64 160.6 and 157.7 / 166 and 158.5, 16,384 x 64 215.5 and 209.9 / 220 and 209, 4,096 x 256 216 and 200 / 215 and 203.5, 16,384 x 128 451 and 417 / 456 and
// 421; rotated ones gain by two at every size (16,384 x 64 230 and 219), scaled ones are alike from 65,536 strings on.
template <bool PLAIN, int SHARE>
__device__ __forceinline__ void append_i16(const AppendArgs& args, uint8_t (*lds_all)[2][KVQ_LDS_CODES]) {
    static_assert(SHARE == 2 || PLAIN, "keys to rotate and scale are always shared");
    const int wave = SHARE == 2 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0, half = wave & 1;
    auto& lds = lds_all[wave >> 1];
    const int lane = threadIdx.x & 63, j = lane >> 4, n = lane & 15;
    AppendArgs A;
    read_append_args<PLAIN>(args, A);
    AppendString t;
    append_string<PLAIN, SHARE>(A, wave >> 1, t);  // (the number of strings is even)
    if (SHARE == 1 || wave == 3) write_fresh_pages(A.table, args.pages, lane);
    const int which = t.which, t_old = A.t_old, gspan = A.gspan;
    const int tok0 = t.tile * KVQ_TILE_TOKENS;
    const kvq_dev::NewRows rows((which ? A.v : A.k) + (uint64_t)t.unit * A.n_new * KVQ_D, t_old, A.n_new);
    const int grp = lane & 3;
    uint32_t w[2 / SHARE][16];
    load_owner_rows(w, rows, tok0 + 16 * half, lane);
    const bool rotates = !PLAIN && !which && A.rope;
    OwnerAngles angles;
    if (rotates) load_owner_angles(angles, rows, tok0 + 16 * half + (lane >> 2), lane, A.rope);
    __builtin_amdgcn_sched_barrier(0);  // all of these loads first
    const KvqPageDesc pd = append_desc<PLAIN>(A.table, args.pages, t.page);
    uint8_t* code = A.arena + (uint64_t)pd.code_off256 * 256u + (t.tslot * 2 + which) * (512u * 16);
    uint8_t* meta = A.arena + (uint64_t)pd.meta_off256 * 256u + t.tslot * KVQ_META_TILE_BYTES;
    if (rotates) rotate_owner_keys(w[0], angles, rows.has(tok0 + 16 * half + (lane >> 2)), rows.all(tok0), lane);
    if (!PLAIN && !which && t.rinv_head) scale_owner_keys(w[0], lane, t.rinv_head);
#pragma unroll
    for (int pass = 0; pass < 2 / SHARE; ++pass) {
        const int tl = 16 * (half + pass) + (lane >> 2), tok = tok0 + tl;
        uint32_t codes[32];
        uint16_t S, Z;
        quantize_owner<16>(w[pass], codes, &S, &Z, gspan);
        scatter_codes<1>(lds[0], which, tl, grp, codes);
        scatter_codes<0>(lds[1], which, tl, grp, codes);
        if (tok >= t_old) store_meta_owner(meta, which, tl, grp, S, Z);
    }
    if (SHARE == 2) __syncthreads();
    else wave_sync_lds();
    uint32_t keep = 0;  // stored tokens keep their bits
    if (!which) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
            if (tok0 + 8 * (n >> 2) + 4 * sub + (n & 3) < t_old) keep |= 1u << sub;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (tok0 + 8 * j + i < t_old) keep |= 1u << i;
    }
#pragma unroll
    for (int plane = half; plane < half + 2 / SHARE; ++plane) {
        uint32_t str[16];
        gather_string<8>(lds[plane], which, lane, str);
        uint8_t* dst = code + plane * (512u * 8);
        if (tok0 < t_old && keep) {
            uint32_t old[16];
            load_chunks<8>(dst, lane, old);
#pragma unroll
            for (int d = 0; d < 16; ++d) {
                uint32_t m = which ? v_token_mask<8>(keep, d) : (((keep >> (d / 8)) & 1u) ? 0xffffffffu : 0u);
                str[d] = (old[d] & m) | (str[d] & ~m);
            }
        }
        if (tok0 >= t_old) {
            store_chunks_stream<8>(dst, lane, str);
        } else {
            store_chunks<8>(dst, lane, str);
            asm volatile("" ::: "memory");  // keeps the two kinds of store apart
        }
    }
}
template <bool PLAIN>
__global__ __launch_bounds__(256) void kvq_append_i16_kernel(const AppendArgs args) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][2][KVQ_LDS_CODES];
    append_i16<PLAIN, 2>(args, lds);
}
__global__ __launch_bounds__(64) void kvq_append_i16_bulk_kernel(const AppendArgs args) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[1][2][KVQ_LDS_CODES];
    append_i16<true, 1>(args, lds);
}

// ------------------------------------------------------------------------------------- fp16 page -> b bits
// grid.x = 2 * n_jobs * tiles_per_page, grid.y = unit, 64 threads.  Direct quantization (Eq. 1-2) of a page
// that still holds raw fp16 values: the tile is first laid out [token][channel] in LDS, then quantized by
// owner lanes exactly like an append.
template <int B>
__global__ __launch_bounds__(64) void kvq_quant16_kernel(uint8_t* __restrict__ arena, KvqPageDesc* __restrict__ table,
                                                         const KvqRequantJob* __restrict__ jobs, int tpp,
                                                         const KvqVMark mark, int gspan,
                                                         const KvqJobArgs ja) {
    // One LDS block: [pad | raw rows 0..15 | raw rows 16..31].  The codes of both passes go to the first KVQ_LDS_CODES bytes,
    // i.e. the pad and the rows of the first pass, which every lane has read by the time the first codes are written (the
    // LDS carries out a wavefront's instructions in order); the rows of the second pass are not touched.  8.1 KiB per
    // wavefront instead of 12.1: the LDS then admits 19 wavefronts per compute unit instead of 13 (16 -> 8: +7 %).
    __shared__ __attribute__((aligned(16))) uint8_t lds_block[(KVQ_LDS_CODES - 16 * 256) + 32 * 256];
    uint8_t* const lds = lds_block;
    uint8_t* const raw_lds = lds_block + (KVQ_LDS_CODES - 16 * 256);
    const int lane = threadIdx.x, j = lane >> 4, n = lane & 15;
    const int which = blockIdx.x & 1;
    const int idx = blockIdx.x >> 1;
    const int job = idx / tpp, tip = idx - job * tpp;
    const int unit = blockIdx.y;
    const KvqRequantJob jb = ja.n ? ja.jobs[job] : jobs[job];
    if (tip >= (int)(jb.tiles_page & 2047u)) return;  // tiles of a partly filled page that hold no token yet (wavefront-uniform)
    if (blockIdx.y == 0 && tip == 0 && lane == 0) table[jb.tiles_page >> 11] = KvqPageDesc{jb.dst_code_off256, jb.meta_off256, B, 0u};
    const uint64_t tslot = (uint64_t)unit * tpp + tip;
    const uint8_t* src = arena + (uint64_t)jb.src_code_off256 * 256u + (tslot * 2 + which) * (512u * 16);
    uint8_t* dst = arena + (uint64_t)jb.dst_code_off256 * 256u + (tslot * 2 + which) * (512u * B);
    uint8_t* meta = arena + (uint64_t)jb.meta_off256 * 256u + tslot * KVQ_META_TILE_BYTES;
    {
        uint32_t in[32];
        load_chunks_stream<16>(src, lane, in);
        // LDS rows are tokens (256 bytes); the bytes of row r are rotated by 32 * (r / 8), so that the four lane
        // quarters, which write rows 8 apart, land in different banks
        if (!which) {
#pragma unroll
            for (int p = 0; p < 8; ++p) {  // piece (sub, grp): 8 consecutive channels of one token
                const int sub = p >> 2, g = p & 3;
                const int t = 8 * (n >> 2) + 4 * sub + (n & 3);
                *reinterpret_cast<u32x4*>(raw_lds + t * 256 + (((32 * g + 8 * j) * 2 + 32 * (t >> 3)) & 255)) =
                    u32x4{in[4 * p], in[4 * p + 1], in[4 * p + 2], in[4 * p + 3]};
            }
        } else {
#pragma unroll
            for (int d = 0; d < 32; ++d) {  // dword d = slots 2d, 2d+1 = tokens 8j + (2d%8), +1 of channel 16*(d/4)+n
                const int nt = d >> 2, i = (2 * d) & 7;
                const int col = ((16 * nt + n) * 2 + 32 * j) & 255;  // rows 8j + i and 8j + i + 1 share the rotation
                *reinterpret_cast<uint16_t*>(raw_lds + (8 * j + i) * 256 + col) = (uint16_t)(in[d] & 0xffff);
                *reinterpret_cast<uint16_t*>(raw_lds + (8 * j + i + 1) * 256 + col) = (uint16_t)(in[d] >> 16);
            }
        }
    }
    wave_sync_lds();
    const int grp = lane & 3;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int tl = 16 * pass + (lane >> 2);
        uint32_t w[16];
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // the two 32-byte halves of the group's 64 bytes (the rotation may wrap between them)
            const u32x4* rp = reinterpret_cast<const u32x4*>(raw_lds + tl * 256 + ((grp * 64 + 32 * h + 32 * (tl >> 3)) & 255));
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                u32x4 v = rp[c];
                w[8 * h + 4 * c] = v.x; w[8 * h + 4 * c + 1] = v.y; w[8 * h + 4 * c + 2] = v.z; w[8 * h + 4 * c + 3] = v.w;
            }
        }
        uint32_t codes[32];
        uint16_t S, Z;
        quantize_owner<B>(w, codes, &S, &Z, gspan);
        note_large_v_scale(mark, which, S);
        scatter_codes(lds, which, tl, grp, codes);
        store_meta_owner(meta, which, tl, grp, S, Z);
    }
    wave_sync_lds();
    uint32_t str[2 * B];
    gather_string<B>(lds, which, lane, str);
    store_chunks_stream<B>(dst, lane, str);
}

// ------------------------------------------------------------------------------- Equivalent Right Shift
// Eq. 3 on packed codes, slot order preserved, several codes per 32-bit multiply (no carry can cross a field:
// 13*(15+2) < 2^8 and 241*(255+8) < 2^16).  From the integer 16-bit tier the product 65281 * (X + 128) needs all 32
// bits of an unsigned multiply (largest value 4,286,546,303), so that step takes one multiply per code.
__device__ inline uint32_t shrink_4_to_2(uint32_t w) {  // 8 nibbles -> 8 two-bit codes (16 bits)
    uint32_t e = w & 0x0f0f0f0fu, o = (w >> 4) & 0x0f0f0f0fu;
    e = (((e + 0x02020202u) * 13u) >> 6) & 0x03030303u;
    o = (((o + 0x02020202u) * 13u) >> 6) & 0x03030303u;
    uint32_t c = e | (o << 2);
    c = (c | (c >> 4)) & 0x00ff00ffu;
    return (c | (c >> 8)) & 0xffffu;
}
__device__ inline uint32_t shrink_16_to_8(uint32_t hi, uint32_t lo) {  // 4 high bytes, 4 low bytes -> 4 bytes
    uint32_t out = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t x = (((hi >> (8 * k)) & 0xffu) << 8) | ((lo >> (8 * k)) & 0xffu);
        out |= ((65281u * (x + 128u)) >> 24) << (8 * k);
    }
    return out;
}
__device__ inline uint32_t shrink_8_to_4(uint32_t w) {  // 4 bytes -> 4 nibbles (16 bits)
    uint32_t e = w & 0x00ff00ffu, o = (w >> 8) & 0x00ff00ffu;
    e = (((e + 0x00080008u) * 241u) >> 12) & 0x000f000fu;
    o = (((o + 0x00080008u) * 241u) >> 12) & 0x000f000fu;
    uint32_t c = e | (o << 4);
    return (c | (c >> 8)) & 0xffffu;
}

// The two other strategies of the ablation (Sec. 4.3.1) keep the upper B bits of every 2B-bit code.
__device__ inline uint32_t trunc_4_to_2(uint32_t w) {  // 8 nibbles -> their upper two bits, packed (16 bits)
    uint32_t e = (w >> 2) & 0x03030303u, o = (w >> 6) & 0x03030303u;
    uint32_t c = e | (o << 2);
    c = (c | (c >> 4)) & 0x00ff00ffu;
    return (c | (c >> 8)) & 0xffffu;
}
__device__ inline uint32_t trunc_8_to_4(uint32_t w) {  // 4 bytes -> their upper nibbles, packed (16 bits)
    uint32_t e = (w >> 4) & 0x000f000fu, o = (w >> 12) & 0x000f000fu;
    uint32_t c = e | (o << 4);
    return (c | (c >> 8)) & 0xffffu;
}

#define KVQ_SHIFT_EQUIVALENT_ 0
#define KVQ_SHIFT_DIRECT_ 1
#define KVQ_SHIFT_MODIFIED_ 2

// grid.x = n_jobs * tiles_per_page, grid.y = unit, 64 threads; one wavefront shrinks the K and the V tile of
// one (page, unit, tile) from 2B to B bits and rewrites its 256 scales (and, for the Modified strategy, zero
// points) in place.  B = 8 is the step out of the integer 16-bit tier.
//   STRAT 0, Equivalent Right Shift (Eq. 3):  codes by Eq. 3, S <- (2^B + 1) S, Z kept
//   STRAT 1, Direct Right Shift:              codes >> B,     S <- (2^B + 1) S, Z kept
//   STRAT 2, Modified Right Shift:            codes >> B,     S <- 2^B S,       Z <- Z + (2^B S - S) / 2
// Products and the sum are formed in fp32 (the products are exact) and rounded to nearest-even into fp16.
template <int B, int STRAT>
__global__ __launch_bounds__(64) void kvq_shrink_kernel(uint8_t* __restrict__ arena, KvqPageDesc* __restrict__ table,
                                                        const KvqRequantJob* __restrict__ jobs, int tpp,
                                                        const KvqVMark mark, const KvqJobArgs ja) {
    const int lane = threadIdx.x;
    const int job = blockIdx.x / tpp, tip = blockIdx.x - job * tpp;
    const int unit = blockIdx.y;
    const KvqRequantJob jb = ja.n ? ja.jobs[job] : jobs[job];
    if (tip >= (int)(jb.tiles_page & 2047u)) return;  // tiles of a partly filled page that hold no token yet (wavefront-uniform)
    if (blockIdx.y == 0 && tip == 0 && lane == 0) table[jb.tiles_page >> 11] = KvqPageDesc{jb.dst_code_off256, jb.meta_off256, B, 0u};
    const uint64_t tslot = (uint64_t)unit * tpp + tip;
    const uint8_t* src = arena + (uint64_t)jb.src_code_off256 * 256u + tslot * 2 * (512u * 2 * B);
    uint8_t* dst = arena + (uint64_t)jb.dst_code_off256 * 256u + tslot * 2 * (512u * B);
    uint8_t* meta = arena + (uint64_t)jb.meta_off256 * 256u + tslot * KVQ_META_TILE_BYTES;
    // K scales at +0, K zero points at +256, V scales at +512, V zero points at +768: 64 dwords each, one
    // dword (two fp16) per lane, a zero point at the same index as its scale
    uint32_t sk = reinterpret_cast<const uint32_t*>(meta)[lane];
    uint32_t sv = reinterpret_cast<const uint32_t*>(meta + 512)[lane];
    uint32_t zk = 0u, zv = 0u;
    if constexpr (STRAT == KVQ_SHIFT_MODIFIED_) {
        zk = reinterpret_cast<const uint32_t*>(meta + 256)[lane];
        zv = reinterpret_cast<const uint32_t*>(meta + 768)[lane];
    }
#pragma unroll
    for (int kv = 0; kv < 2; ++kv) {
        uint32_t in[4 * B];
        load_chunks_stream<2 * B>(src + kv * (512u * 2 * B), lane, in);
        uint32_t out[2 * B];
#pragma unroll
        for (int d = 0; d < 2 * B; ++d) {
            if constexpr (B == 8) {  // source: high-byte plane in[0..15], low-byte plane in[16..31]
                if constexpr (STRAT == KVQ_SHIFT_EQUIVALENT_) out[d] = shrink_16_to_8(in[d], in[16 + d]);
                else out[d] = in[d];
            } else if constexpr (STRAT == KVQ_SHIFT_EQUIVALENT_) {
                if constexpr (B == 2) out[d] = shrink_4_to_2(in[2 * d]) | (shrink_4_to_2(in[2 * d + 1]) << 16);
                else out[d] = shrink_8_to_4(in[2 * d]) | (shrink_8_to_4(in[2 * d + 1]) << 16);
            } else {
                if constexpr (B == 2) out[d] = trunc_4_to_2(in[2 * d]) | (trunc_4_to_2(in[2 * d + 1]) << 16);
                else out[d] = trunc_8_to_4(in[2 * d]) | (trunc_8_to_4(in[2 * d + 1]) << 16);
            }
        }
        store_chunks_stream<B>(dst + kv * (512u * B), lane, out);
    }
    const float f = STRAT == KVQ_SHIFT_MODIFIED_ ? (float)(1 << B) : (float)((1 << B) + 1);
    uint32_t nk = 0u, nv = 0u, nzk = 0u, nzv = 0u;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float s_k = h2f((uint16_t)(sk >> (16 * h))), s_v = h2f((uint16_t)(sv >> (16 * h)));
        const float nk32 = s_k * f, nv32 = s_v * f;
        nk |= (uint32_t)f2h_rn(nk32) << (16 * h);
        nv |= (uint32_t)f2h_rn(nv32) << (16 * h);
        if constexpr (STRAT == KVQ_SHIFT_MODIFIED_) {
            const float hk = 0.5f * (nk32 - s_k), hv = 0.5f * (nv32 - s_v);  // exact
            nzk |= (uint32_t)f2h_rn(h2f((uint16_t)(zk >> (16 * h))) + hk) << (16 * h);
            nzv |= (uint32_t)f2h_rn(h2f((uint16_t)(zv >> (16 * h))) + hv) << (16 * h);
        }
    }
    reinterpret_cast<uint32_t*>(meta)[lane] = nk;
    reinterpret_cast<uint32_t*>(meta + 512)[lane] = nv;
    if constexpr (STRAT == KVQ_SHIFT_MODIFIED_) {
        reinterpret_cast<uint32_t*>(meta + 256)[lane] = nzk;
        reinterpret_cast<uint32_t*>(meta + 768)[lane] = nzv;
    }
    note_large_v_scale(mark, 1, (uint16_t)(nv & 0xffff));
    note_large_v_scale(mark, 1, (uint16_t)(nv >> 16));
}

// --------------------------------------------------------------------------------- reconstruction error
// 16 bytes from the address of any element (a reference may be a view that starts at an odd one): one 16-byte load,
// through the caches where several lanes or loads share a line, streaming where a load instruction covers whole lines.
typedef u32x4 u32x4_any __attribute__((aligned(2)));
__device__ inline u32x4 load16_any(const void* p) { return *static_cast<const u32x4_any*>(p); }
__device__ inline u32x4 load16_any_stream(const void* p) {
    return __builtin_nontemporal_load(static_cast<const u32x4_any*>(p));
}
// 8 codes of B bits (piece p of a lane's string) -> 8 bytes, the inverse of pack8.
template <int B>
__device__ inline void unpack8(const uint32_t* str, int p, uint32_t* w0, uint32_t* w1) {
    if constexpr (B == 8) {
        *w0 = str[2 * p]; *w1 = str[2 * p + 1];
    } else if constexpr (B == 4) {
        const uint32_t lo = str[p] & 0x0f0f0f0fu, hi = (str[p] >> 4) & 0x0f0f0f0fu;
        *w0 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);
        *w1 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);
    } else {
        const uint32_t h = str[p >> 1] >> (16 * (p & 1));
        uint32_t a = h & 0xffu, b = (h >> 8) & 0xffu;
        a = (a | (a << 12)) & 0x000f000fu; b = (b | (b << 12)) & 0x000f000fu;
        *w0 = (a | (a << 6)) & 0x03030303u;
        *w1 = (b | (b << 6)) & 0x03030303u;
    }
}
// Byte codes of one tile string -> LDS [32 tokens][128 channels]; the columns of row t are rotated by 32 (t / 8), which
// puts the four lane quarters of a V string, whose rows are 8 apart, into different banks.
// behind: called once the loads of the codes are issued.
template <int B, class Behind>
__device__ inline void rows_of_string(uint8_t* lds, const uint8_t* code, int which, int lane, Behind behind) {
    const int j = lane >> 4, n = lane & 15;
    uint32_t str[2 * B];
    load_chunks_stream<B>(code, lane, str);
    __builtin_amdgcn_sched_barrier(0);
    behind();
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        uint32_t w[2];
        unpack8<B>(str, p, &w[0], &w[1]);
        if (!which) {
            const int t = 8 * (n >> 2) + 4 * (p >> 2) + (n & 3);
            uint32_t* dst = reinterpret_cast<uint32_t*>(lds + t * 128 + ((32 * (p & 3) + 32 * (t >> 3) + 8 * j) & 127));
            dst[0] = w[0]; dst[1] = w[1];
        } else {
            const int col = (16 * p + n + 32 * j) & 127;
#pragma unroll
            for (int i = 0; i < 8; ++i) lds[(8 * j + i) * 128 + col] = (uint8_t)(w[i >> 2] >> (8 * (i & 3)));
        }
    }
}
// The same for raw fp16 values: [32 tokens][128 channels] halves, rows rotated by 64 bytes per 8 tokens.
template <class Behind>
__device__ inline void rows_of_raw(uint8_t* lds, const uint8_t* code, int which, int lane, Behind behind) {
    const int j = lane >> 4, n = lane & 15;
    uint32_t in[32];
    load_chunks_stream<16>(code, lane, in);
    __builtin_amdgcn_sched_barrier(0);
    behind();
    if (!which) {
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int t = 8 * (n >> 2) + 4 * (p >> 2) + (n & 3);
            *reinterpret_cast<u32x4*>(lds + t * 256 + ((64 * (p & 3) + 64 * (t >> 3) + 16 * j) & 255)) =
                u32x4{in[4 * p], in[4 * p + 1], in[4 * p + 2], in[4 * p + 3]};
        }
    } else {
#pragma unroll
        for (int d = 0; d < 32; ++d) {
            const int i = (2 * d) & 7, col = (2 * (16 * (d >> 2) + n) + 64 * j) & 255;
            *reinterpret_cast<uint16_t*>(lds + (8 * j + i) * 256 + col) = (uint16_t)(in[d] & 0xffff);
            *reinterpret_cast<uint16_t*>(lds + (8 * j + i + 1) * 256 + col) = (uint16_t)(in[d] >> 16);
        }
    }
}

// Over a block's stored tokens, with x_hat = code * S + Z (or the raw value of a 16-bit tile) and x the reference fp16
// tensor [unit][token][128]: partial[2 * workgroup + which] = sum over the workgroup's share of K (which = 0), V (1) of
//   KVQ_ERR_SQ: (x_hat - x)^2
//   KVQ_ERR_L1, _L1_GRAD, _L1_ONE_GRAD: |g * (x_hat - x)|, the terms of the sensitivity of Sec. 3.2, Eq. 5, with gradient tensors
//               [unit][token][128] fp32 for none, both or one of K and V (g = 1 where there is none)
// fp32 over 32 elements of a lane (eight tokens x 4 channels), fp64 beyond; the host adds the workgroups up in order.
//
// Bound by the references and gradients (4 + 8 bytes per cached token and channel against at most 2 of codes), which are
// rows while the codes are tiles: every wavefront turns one tile string to rows in LDS and then reads both row by row, 32
// lanes to a token and 4 channels a lane, so that a load instruction covers whole lines (512 bytes of references, 1 KiB of
// gradients) and can stream.  Six tokens of every lane are on their way at any time, the first six from behind the loads of
// the codes on: with eight the kernel would spill at four wavefronts per SIMD, which is also what the LDS holds.  (With a
// lane taking 32 channels of a token a load instruction touched 64 lines, four instructions one after the other the same
// ones, and nothing was asked for before the codes were in LDS.)  A fixed number of workgroups strides over the strings and
// leaves two numbers each, without atomics.  Whole calls, of which launch and synchronization are some 11 us, with a lane's 32
// channels and now: 64 units x 2,048 tokens at 4 bits with gradients (219 MB) 53.2 and 47.9 us, without 31.0 and 27.3, 128 x 4,096 (880 MB)
// 157 and 142 and 69 and 65; the integer tier with gradients 57 and 55; streaming loads against plain ones 142 and 155.
#define KVQ_ERR_WAVES 4
#define KVQ_ERR_AHEAD 6
enum { KVQ_ERR_SQ, KVQ_ERR_L1, KVQ_ERR_L1_GRAD, KVQ_ERR_L1_ONE_GRAD };  // (one: K or V comes without gradients)
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
struct ErrorStep { uint32_t units, tiles; };  // from a wavefront's string to its next
template <int MODE>
__global__ __launch_bounds__(64 * KVQ_ERR_WAVES) __attribute__((amdgpu_waves_per_eu(4))) void kvq_error_kernel(const uint8_t* __restrict__ arena,
                                                       const KvqPageDesc* __restrict__ table,
                                                       const uint16_t* __restrict__ k_ref,
                                                       const uint16_t* __restrict__ v_ref,
                                                       const float* __restrict__ gk, const float* __restrict__ gv,
                                                       int n_tokens, int tpp, uint32_t tpp_magic, int n_tiles, int units,
                                                       ErrorStep step, double* __restrict__ partial) {
    __shared__ __attribute__((aligned(16))) uint8_t rows[KVQ_ERR_WAVES][32 * 256];
    __shared__ f32x2 metas[KVQ_ERR_WAVES][128];  // [token][group]: scale, zero point
    __shared__ double sums[KVQ_ERR_WAVES];
    constexpr int AHEAD = KVQ_ERR_AHEAD, ROWS = KVQ_TILE_TOKENS / 2;
    const int thread_lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int which = wave & 1;  // a wavefront's strings are all of K or all of V: the stride is even
    uint8_t* const lds = rows[wave];
    f32x2* const meta = metas[wave];
    const uint16_t* const ref = which ? v_ref : k_ref;
    const float* const grad = which ? gv : gk;
    const uint32_t first = (uint32_t)(blockIdx.x * (KVQ_ERR_WAVES / 2) + (wave >> 1));
    int unit = (int)(first / (uint32_t)n_tiles), tile = (int)(first - (uint32_t)unit * (uint32_t)n_tiles);
    double total = 0.0;
    while (unit < units) {
        int lane = thread_lane;
        asm("" : "+v"(lane));  // addresses in LDS are made anew for each string: kept across strings they would take half the registers
        const int half = lane >> 5, c4 = 4 * (lane & 31);
        const int page = div_magic(tile, tpp, tpp_magic), tip = tile - page * tpp;
        const KvqPageDesc pd = table[page];
        const uint64_t tslot = (uint64_t)unit * tpp + tip;
        const uint8_t* code = arena + (uint64_t)pd.code_off256 * 256u + (tslot * 2 + which) * (512u * pd.bits);
        const uint32_t* meta_in = reinterpret_cast<const uint32_t*>(arena + (uint64_t)pd.meta_off256 * 256u +
                                                                    tslot * KVQ_META_TILE_BYTES) + (which ? 128 : 0);
        const uint64_t tile_row = (uint64_t)unit * n_tokens + (uint64_t)tile * KVQ_TILE_TOKENS;
        const int left = n_tokens - tile * KVQ_TILE_TOKENS;
        // (buffers that end with the last token: what lies beyond reads as zeros)
        const auto ref_tile = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(ref + tile_row * KVQ_D), 0,
                                                                min(left, KVQ_TILE_TOKENS) * (KVQ_D * 2), 0x00020000);
        const bool weighs = MODE == KVQ_ERR_L1_GRAD || (MODE == KVQ_ERR_L1_ONE_GRAD && grad);
        const auto grad_tile = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(weighs ? grad + tile_row * KVQ_D : nullptr), 0,
                                                                 weighs ? min(left, KVQ_TILE_TOKENS) * (KVQ_D * 4) : 0, 0x00020000);
        const float no_weight = weighs ? 0.0f : 1.0f;  // (gradients that are not there read as zeros)
        u32x2 x[AHEAD];
        u32x4 g[AHEAD];
        const auto load = [&](int i) {
            x[i % AHEAD] = __builtin_amdgcn_raw_buffer_load_b64(ref_tile, 8 * lane + 512 * i, 0, 2);
            if (MODE >= KVQ_ERR_L1_GRAD) g[i % AHEAD] = __builtin_amdgcn_raw_buffer_load_b128(grad_tile, 16 * lane + 1024 * i, 0, 2);
        };
        const bool raw = pd.bits == 16 && !pd.int16;
        const auto behind_codes = [&]() {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) load(i);
            __builtin_amdgcn_sched_barrier(0);
        };
        const uint32_t ms = raw ? 0u : meta_in[lane], mz = raw ? 0u : meta_in[64 + lane];
        switch (pd.bits) {
            case 2: rows_of_string<2>(lds, code, which, lane, behind_codes); break;
            case 4: rows_of_string<4>(lds, code, which, lane, behind_codes); break;
            case 8: rows_of_string<8>(lds, code, which, lane, behind_codes); break;
            default:
                if (raw) {
                    rows_of_raw(lds, code, which, lane, behind_codes);
                } else {  // byte planes: high bytes, then low bytes
                    rows_of_string<8>(lds, code, which, lane, [] {});
                    rows_of_string<8>(lds + 4096, code + 512u * 8, which, lane, behind_codes);
                }
        }
        if (!raw) {
            int put[2];  // where the lane's two entries of the tile's metadata go
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int at = 2 * lane + e, v = at & 31;  // (kvq_vmeta_index the other way)
                put[e] = which ? ((v >> 3) * 8 + ((v & 7) >> 1) + 4 * (v & 1)) * 4 + (at >> 5) : at;
            }
            meta[put[0]] = f32x2{h2f((uint16_t)ms), h2f((uint16_t)mz)};
            meta[put[1]] = f32x2{h2f((uint16_t)(ms >> 16)), h2f((uint16_t)(mz >> 16))};
        }
        wave_sync_lds();
        // x_hat - x = code * S + (Z - x): the difference of two fp16 numbers is exact in fp32 and the fused
        // multiply-add rounds once, so large codes times large scales lose nothing before the subtraction
        const auto sum_up = [&](auto kind) {  // 0: bytes, 1: byte planes, 2: raw
            constexpr int KIND = decltype(kind)::value;
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                const int t = 2 * i + half;
                f32x2 sz = {0.f, 0.f};
                u32x2 b;
                if (KIND == 2) {
                    b = *reinterpret_cast<const u32x2*>(lds + half * 256 + ((2 * c4 + 64 * (i >> 2)) & 255) + 512 * i);
                } else {
                    sz = meta[4 * half + (c4 >> 5) + 8 * i];
                    const uint8_t* const at = lds + half * 128 + ((c4 + 32 * (i >> 2)) & 127) + 256 * i;
                    b.x = *reinterpret_cast<const uint32_t*>(at);
                    b.y = KIND == 1 ? *reinterpret_cast<const uint32_t*>(at + 4096) : 0u;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float xe = h2f((uint16_t)(x[i % AHEAD][e >> 1] >> (16 * (e & 1))));
                    float dx;
                    if (KIND == 2) {
                        dx = h2f((uint16_t)(b[e >> 1] >> (16 * (e & 1)))) - xe;
                    } else {
                        float cd = (float)((b.x >> (8 * e)) & 0xffu);
                        if (KIND == 1) cd = fmaf(cd, 256.0f, (float)((b.y >> (8 * e)) & 0xffu));  // exact
                        dx = fmaf(cd, sz.x, sz.y - xe);
                    }
                    if (t >= left) dx = 0.0f;
                    if (MODE == KVQ_ERR_SQ) acc[e] = fmaf(dx, dx, acc[e]);
                    else if (MODE == KVQ_ERR_L1) acc[e] += fabsf(dx);
                    else acc[e] = fmaf(fabsf(__uint_as_float(g[i % AHEAD][e])) + (MODE == KVQ_ERR_L1_ONE_GRAD ? no_weight : 0.0f), fabsf(dx), acc[e]);
                }
                if (i + AHEAD < ROWS) load(i + AHEAD);
                if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (left alone, all rows are read from LDS first)
                if (i % 8 == 7) {  // 32 elements
                    total += (double)((acc[0] + acc[1]) + (acc[2] + acc[3]));
                    acc[0] = acc[1] = acc[2] = acc[3] = 0.f;
                }
            }
        };
        if (raw) sum_up(std::integral_constant<int, 2>());
        else if (pd.int16) sum_up(std::integral_constant<int, 1>());
        else sum_up(std::integral_constant<int, 0>());
        wave_sync_lds();
        unit += (int)step.units;
        tile += (int)step.tiles;
        if (tile >= n_tiles) { tile -= n_tiles; ++unit; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o);
    if (thread_lane == 0) sums[wave] = total;
    __syncthreads();
    // The host is waiting for it: one store that is not held back, into coherent memory, which the L2 caches do not keep.  (Device scope is past
    // what could hold it.  System scope costs launches of some 250 workgroups 1 us: 4 units x 4,000 tokens with gradients 14.0 us and 15.2, a
    // plain store 14.2; 64 x 2,048 43.0, 43.0 and 44.0.  At the latest the end of the kernel shows it, for which the host waits after a while.)
    if (threadIdx.x < 2)
        __hip_atomic_store(&partial[2 * blockIdx.x + threadIdx.x], sums[threadIdx.x] + sums[threadIdx.x + 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------------ channel-wise reparameterization
// dst[0 .. n) = lambda, dst[n .. 2n) = 1 / lambda (one correctly rounded fp32 division per channel).
__global__ void kvq_reparam_store_kernel(const float* __restrict__ lambda, float* __restrict__ dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) { const float l = lambda[i]; dst[i] = l; dst[n + i] = 1.0f / l; }
}
// Eq. 8: lambda[h][i] = max(max over sequences and tokens of |K|, floor)^alpha, pow in fp64, rounded to fp32.  Every workgroup raises
// its own maxima and an atomic maximum joins them: lambda holds float bit patterns of non-negative values, whose unsigned order is
// their order, and the rounded power keeps the order of its arguments (alpha >= 0; of two different fp16 magnitudes the powers are
// further apart than fp64 errs, or so near to 1 that both round to it), so the joined result is the power of the joint maximum.  A
// third launch that raised the maxima in place took 2.4 us and more.  256 threads: 16 lanes x 16 bytes read one row of 128 channels,
// a workgroup 16 rows at a time, eight loads in flight per lane; the 16 row groups meet in LDS and 128 atomics go out whose result
// nobody waits for (looking first whether a channel exceeds what is there costs 20 us: the look is a trip to memory at the end of
// every workgroup, the atomics are not).
//   FLAT = false: grid.x = (sequence, KV head) units, grid.y = slices of a unit's tokens
//   FLAT = true:  grid.x = KV heads, grid.y = slices of a head's rows, the tokens of all its sequences in turn; a row's place
//                 is stepped along, 16 rows being step_seqs sequences and step_tokens tokens
// Bound by the one read of the keys.  32 sequences x 8 heads x 2,048 tokens (134 MB): 24 us over keys read for the first
// time, 5.6 TB/s, and 21 over the same ones again, which the last-level cache partly holds (82 with 2-byte loads, a 64-bit
// division per row and 1,024 slices per head).  The stepping costs the long sequences 2 to 3 %; on short ones a workgroup per unit
// pays its atomics and powers for few rows.  Whole calls, three launches before and two now: 134 MB of 8 heads 24.6 and 23.2 us over
// the same keys, 26.3 and 24.5 from memory, 33 MB 11.4 and 7.9, 16 MB of one head 24.6 and 13.7, small ones 9 to 11 and 7.5 to 8.  Whole
// calls over 134 MB of 8 heads, FLAT = false and true: 2,048 tokens a sequence 22.0 and 22.3 us, 512 23.2 and 23.1, 256 23.5 and 23.8,
// 128 24.0 and 24.2, 64 31.8 and 23.7, 16 81.6 and 24.5; from memory 256 tokens 25.0 and 26.2; 64 heads, 268 MB: 512 42.3 and 41.5,
// 256 42.7 and 41.4, 128 43.5 and 41.7, 64 48.0 and 42.2: the line is at 256 tokens.
template <bool FLAT>
__global__ __launch_bounds__(256) void kvq_absmax_kernel(const uint16_t* __restrict__ k, int n_kv_heads, int n_tokens,
                                                         int n_rows, int slice_rows, int step_seqs, int step_tokens,
                                                         float alpha, float floor_, uint32_t* __restrict__ acc) {
    __shared__ __attribute__((aligned(16))) uint32_t part[16][KVQ_D / 2];
    const int c8 = threadIdx.x & 15, rg = threadIdx.x >> 4, head = FLAT ? blockIdx.x : blockIdx.x % n_kv_heads;
    const int r0 = blockIdx.y * slice_rows, r1 = r0 + min(slice_rows, n_rows - r0);
    int r = r0 + rg;
    const uint16_t* p;
    int t = r;
    int64_t step = 16 * KVQ_D, wrap = 0;
    if (FLAT) {
        t = r % n_tokens;
        const int64_t seq_rows = (int64_t)n_kv_heads * n_tokens;
        p = k + ((r / n_tokens) * seq_rows + (int64_t)head * n_tokens + t) * KVQ_D + 8 * c8;
        step = (step_seqs * seq_rows + step_tokens) * KVQ_D;
        wrap = (seq_rows - n_tokens) * KVQ_D;  // on to the next sequence
    } else {
        p = k + ((int64_t)blockIdx.x * n_tokens + t) * KVQ_D + 8 * c8;
    }
    const auto next = [&]() {
        const uint16_t* const at = p;
        p += step;
        if (FLAT) {
            t += step_tokens;
            if (t >= n_tokens) { t -= n_tokens; p += wrap; }
        }
        return at;
    };
    uint32_t m[4] = {0u, 0u, 0u, 0u};
    for (; r + 7 * 16 < r1; r += 8 * 16) {
        u32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = load16_any_stream(next());
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) m[e] = pk_max_u(m[e], v[u][e] & 0x7fff7fffu);
    }
    for (; r < r1; r += 16) {
        const u32x4 v = load16_any_stream(next());
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = pk_max_u(m[e], v[e] & 0x7fff7fffu);
    }
    *reinterpret_cast<u32x4*>(&part[rg][4 * c8]) = u32x4{m[0], m[1], m[2], m[3]};
    __syncthreads();
    if (threadIdx.x < KVQ_D) {
        const _Float16* const col = reinterpret_cast<const _Float16*>(&part[0][0]) + threadIdx.x;
        _Float16 w = col[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) w = __builtin_elementwise_max(w, col[r * KVQ_D]);
        const float lam = (float)pow((double)fmaxf((float)w, floor_), (double)alpha);
        atomicMax(acc + head * KVQ_D + threadIdx.x, __float_as_uint(lam));
    }
}

// Plain streaming read (16 bytes per lane, 4 non-temporal loads in flight): the practical HBM read ceiling of the device,
// against which the attention kernel's bandwidth is put next to the published peak.
__global__ __launch_bounds__(256) void kvq_stream_read_kernel(const u32x4* __restrict__ p, size_t n,
                                                              uint32_t* __restrict__ sink) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i + 3 * stride < n; i += 4 * stride) {
        u32x4 a = __builtin_nontemporal_load(p + i), b = __builtin_nontemporal_load(p + i + stride);
        u32x4 c = __builtin_nontemporal_load(p + i + 2 * stride), d = __builtin_nontemporal_load(p + i + 3 * stride);
        acc ^= a ^ b ^ c ^ d;
    }
    for (; i < n; i += stride) acc ^= __builtin_nontemporal_load(p + i);
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) sink[0] = 1u;  // practically never: keeps the loads alive
}

__global__ void kvq_fill_u32_kernel(uint32_t* dst, uint32_t value, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = value;
}

}  // namespace

hipError_t kvq_launch_append(int bits, uint8_t* arena, KvqPageDesc* table, const void* k_in,
                             const void* v_in, int t_old, int n_new, int tiles_per_page, int units,
                             const KvqAppendPages& ap, KvqVMark mark, int group,
                             const float* rinv, int n_kv_heads, const float* rope, bool int16, hipStream_t s) {
    const int gspan = group / KVQ_G;
    int tile0 = t_old / KVQ_TILE_TOKENS;
    int tile1 = (t_old + n_new + KVQ_TILE_TOKENS - 1) / KVQ_TILE_TOKENS;
    const int n_strings = 2 * (tile1 - tile0);
    const bool plain = !rinv && !rope;
    const uint16_t* k = static_cast<const uint16_t*>(k_in);
    const uint16_t* v = static_cast<const uint16_t*>(v_in);
    const int64_t strings = (int64_t)n_strings * units;
    const bool pair = kvq_pair_strings(bits, strings, rope != nullptr, rinv != nullptr);
    // How the 16-bit tier's V rows are read: new values have usually just been written and lie in the caches, which streaming
    // loads make less of.  128 units x 2,000 tokens (131 MB of keys and values) 43 us with plain loads of V and 51 with streaming
    // ones, 64 x 2,000 21 and 25, 32 x 2,000 10.9 and 12.6 (from 230 MB of buffers in turn 13.4 and 13.0), 600 x 50 12.1 and 13.0,
    // up to 16 x 1,024 alike.  An input that the 256 MB last-level cache does not hold gains by streaming past it: 64 x 8,192 (268
    // MB) 86 and 85, from buffers in turn 102 and 94.  Beside keys that are prepared, streaming is the better or the same: 32 x
    // 2,000 16.0 and 16.0, from buffers in turn 18.9 and 15.8.
    const int stream_v = !plain || (int64_t)units * n_new * (2 * 256) > (192 << 20);
    const bool bulk = strings > 16384;  // see kvq_append16_bulk_kernel
    const bool few = strings < 1024;  // see kvq_append16_pair_kernel
    const bool five = rinv && strings > 4096 && strings <= 5632 && (strings + 511) / 512 % 2 == 1;  // see kvq_append16_kernel
    const int by_unit = !plain && bits == 16 && !int16 && units >= 32 && (int64_t)units * n_new >= 98304 ? units : 0;
    AppendArgs A;
    A.arena = arena; A.table = table; A.k = k; A.v = v; A.rinv = rinv; A.rope = rope; A.v_word = mark.word; A.v_epoch = mark.epoch;
    A.t_old = t_old; A.n_new = n_new; A.tpp = tiles_per_page; A.tile0 = tile0; A.n_strings = n_strings; A.by_unit = by_unit;
    A.n_kv_heads = n_kv_heads; A.gspan = gspan; A.stream_v = stream_v;
    const auto magic = [](int d) { return d > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)d - 1) / (uint64_t)d) : 0u; };
    A.tpp_magic = magic(tiles_per_page);
    A.kv_magic = magic(n_kv_heads);
    A.pages = ap;
    // A row of the table is read by the L2 of every XCD that a string with its tokens runs on.  Workgroups go to the eight XCDs in
    // turn, so these are 8 / gcd(8, workgroups of a unit) of them, for an odd number all eight: with two wavefronts per string, a
    // workgroup a tile, 4 n + 3 tiles then took longer than with one, half as many workgroups.  Up to three idle workgroups a unit make
    // it a multiple of four.  One wavefront each / two / now, over the same input and from memory: into 8 bits 52 units x 191 tiles 43.0,
    // 55.6, 39.6 and 56.2, 58.1, 52.4 us, 47 x 127 29.2, 30.3, 26.2 and 37.2, 35.0, 34.0; into 2 bits 39 x 255 41.2, 50.1, 37.1 and 48.6, 49.2, 43.1.
    // Up to 120 workgroups, some two MB of rows, the caches hold them all the same, and three idle ones are too large a part.
    const auto workgroups = [&](int n) { return rope && bits < 16 && n > 120 ? (n + 3) / 4 * 4 : n; };
#define KVQ_APPEND_LAUNCH(kernel_, waves_, per_)                                                                           \
    do {                                                                                                                 \
        const int n_wg = workgroups((n_strings + waves_ - 1) / waves_);                                                  \
        const dim3 grid = by_unit ? dim3((unsigned)n_wg * (unsigned)units) : dim3(n_wg, units);                          \
        hipLaunchKernelGGL((kernel_), grid, dim3(64 * waves_ * per_), 0, s, A);                                          \
    } while (0)
    switch (bits + (int16 && bits == 16 ? 1 : 0)) {
        case 17:
            if (plain && strings > 32768) KVQ_APPEND_LAUNCH(kvq_append_i16_bulk_kernel, 1, 1);
            else if (plain) KVQ_APPEND_LAUNCH(kvq_append_i16_kernel<true>, 2, 2);
            else KVQ_APPEND_LAUNCH(kvq_append_i16_kernel<false>, 2, 2);
            break;
        case 16:
            if (plain && few) KVQ_APPEND_LAUNCH(kvq_append16_pair_kernel<true>, 2, 2);
            else if (plain && strings >= 49152) KVQ_APPEND_LAUNCH(kvq_append16_bulk_kernel<1>, 1, 1);
            else if (plain && bulk) KVQ_APPEND_LAUNCH(kvq_append16_bulk_kernel<4>, 4, 1);
            else if (plain) KVQ_APPEND_LAUNCH((kvq_append16_kernel<true, false>), 2, 1);
            else if (few) KVQ_APPEND_LAUNCH(kvq_append16_pair_kernel<false>, 2, 2);
            else if (five) KVQ_APPEND_LAUNCH((kvq_append16_kernel<false, true>), 2, 1);
            else KVQ_APPEND_LAUNCH((kvq_append16_kernel<false, false>), 2, 1);
            break;
#define KVQ_APPEND_CASE(b_, plain_alone_)                                                                                \
        case b_:                                                                                                         \
            if (plain && pair) KVQ_APPEND_LAUNCH((kvq_append_q_kernel<b_, true, true>), 2, 2);                           \
            else if (plain) plain_alone_;                                                                                \
            else if (pair) KVQ_APPEND_LAUNCH((kvq_append_q_kernel<b_, false, true>), 2, 2);                              \
            else KVQ_APPEND_LAUNCH((kvq_append_q_kernel<b_, false, false>), KVQ_APPEND_WG_WAVES, 1);                     \
            break;
        KVQ_APPEND_CASE(8, KVQ_APPEND_LAUNCH((kvq_append_q_kernel<8, true, false>), KVQ_APPEND_WG_WAVES, 1))
        KVQ_APPEND_CASE(4, KVQ_APPEND_LAUNCH((kvq_append_q_kernel<4, true, false>), KVQ_APPEND_WG_WAVES, 1))
        KVQ_APPEND_CASE(2, return hipErrorInvalidValue)  // (kvq_pair_strings: such strings are always shared)
        default: return hipErrorInvalidValue;
    }
#undef KVQ_APPEND_CASE
#undef KVQ_APPEND_LAUNCH
    return hipGetLastError();
}

static void fill_job_args(KvqJobArgs& ja, const KvqRequantJob* jobs_host, int n_jobs) {
    ja.n = (jobs_host && n_jobs <= KVQ_JOBS_BY_ARG) ? n_jobs : 0;
    ja.pad[0] = ja.pad[1] = ja.pad[2] = 0;
    for (int i = 0; i < ja.n; ++i) ja.jobs[i] = jobs_host[i];
}

// jobs_host != nullptr and n_jobs <= KVQ_JOBS_BY_ARG: the list travels in the kernel arguments and jobs_dev is
// not read; otherwise jobs_dev must already hold the list (in stream order).
hipError_t kvq_launch_shrink(int dst_bits, int strategy, uint8_t* arena, KvqPageDesc* table, const KvqRequantJob* jobs_dev,
                             const KvqRequantJob* jobs_host, int n_jobs, int tiles_per_page, int units,
                             KvqVMark mark, hipStream_t s) {
    dim3 grid(n_jobs * tiles_per_page, units), block(64);
    KvqJobArgs ja;
    fill_job_args(ja, jobs_host, n_jobs);
#define KVQ_SHRINK_CASE(B_, S_) \
    hipLaunchKernelGGL((kvq_shrink_kernel<B_, S_>), grid, block, 0, s, arena, table, jobs_dev, tiles_per_page, mark, ja)
    switch (dst_bits * 4 + strategy) {
        case 8 * 4 + 0: KVQ_SHRINK_CASE(8, 0); break;
        case 8 * 4 + 1: KVQ_SHRINK_CASE(8, 1); break;
        case 8 * 4 + 2: KVQ_SHRINK_CASE(8, 2); break;
        case 4 * 4 + 0: KVQ_SHRINK_CASE(4, 0); break;
        case 4 * 4 + 1: KVQ_SHRINK_CASE(4, 1); break;
        case 4 * 4 + 2: KVQ_SHRINK_CASE(4, 2); break;
        case 2 * 4 + 0: KVQ_SHRINK_CASE(2, 0); break;
        case 2 * 4 + 1: KVQ_SHRINK_CASE(2, 1); break;
        case 2 * 4 + 2: KVQ_SHRINK_CASE(2, 2); break;
        default: return hipErrorInvalidValue;
    }
#undef KVQ_SHRINK_CASE
    return hipGetLastError();
}

int kvq_error_workgroups(int n_tokens, int units) {
    const int64_t strings = 2ll * ((n_tokens + KVQ_TILE_TOKENS - 1) / KVQ_TILE_TOKENS) * units;
    return (int)std::min<int64_t>((strings + KVQ_ERR_WAVES - 1) / KVQ_ERR_WAVES, KVQ_ERR_MAX_WGS);
}

hipError_t kvq_launch_error(bool l1, const uint8_t* arena, const KvqPageDesc* table, const void* k_ref,
                            const void* v_ref, const float* gk, const float* gv, int n_tokens, int tiles_per_page,
                            int units, double* partial, hipStream_t s) {
    const int n_tiles = (n_tokens + KVQ_TILE_TOKENS - 1) / KVQ_TILE_TOKENS;
    const int wgs = kvq_error_workgroups(n_tokens, units);
    const dim3 grid(wgs), block(64 * KVQ_ERR_WAVES);
    const uint16_t* k = static_cast<const uint16_t*>(k_ref);
    const uint16_t* v = static_cast<const uint16_t*>(v_ref);
    const uint32_t stride = (uint32_t)wgs * (KVQ_ERR_WAVES / 2);  // in tiles (a tile takes two wavefronts; 2^31 of them hold 4 TB)
    const ErrorStep step{stride / (uint32_t)n_tiles, stride % (uint32_t)n_tiles};
    const uint32_t magic = tiles_per_page > 1 ? (uint32_t)(((1ull << 32) + (uint64_t)tiles_per_page - 1) / (uint64_t)tiles_per_page) : 0u;
#define KVQ_ERR_LAUNCH(mode_) \
    hipLaunchKernelGGL(kvq_error_kernel<mode_>, grid, block, 0, s, arena, table, k, v, gk, gv, n_tokens, tiles_per_page, magic, n_tiles, units, step, partial)
    if (!l1) KVQ_ERR_LAUNCH(KVQ_ERR_SQ);
    else if (!gk && !gv) KVQ_ERR_LAUNCH(KVQ_ERR_L1);
    else if (!gk || !gv) KVQ_ERR_LAUNCH(KVQ_ERR_L1_ONE_GRAD);
    else KVQ_ERR_LAUNCH(KVQ_ERR_L1_GRAD);
#undef KVQ_ERR_LAUNCH
    return hipGetLastError();
}

hipError_t kvq_launch_quant16(int dst_bits, uint8_t* arena, KvqPageDesc* table, const KvqRequantJob* jobs_dev,
                              const KvqRequantJob* jobs_host, int n_jobs, int tiles_per_page, int units,
                              KvqVMark mark, int group, hipStream_t s) {
    dim3 grid(2 * n_jobs * tiles_per_page, units), block(64);
    KvqJobArgs ja;
    fill_job_args(ja, jobs_host, n_jobs);
    switch (dst_bits) {
        case 8: hipLaunchKernelGGL(kvq_quant16_kernel<8>, grid, block, 0, s, arena, table, jobs_dev, tiles_per_page, mark, group / KVQ_G, ja); break;
        case 4: hipLaunchKernelGGL(kvq_quant16_kernel<4>, grid, block, 0, s, arena, table, jobs_dev, tiles_per_page, mark, group / KVQ_G, ja); break;
        case 2: hipLaunchKernelGGL(kvq_quant16_kernel<2>, grid, block, 0, s, arena, table, jobs_dev, tiles_per_page, mark, group / KVQ_G, ja); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t kvq_launch_reparam_store(const float* lambda, float* dst, int n, hipStream_t s) {
    hipLaunchKernelGGL(kvq_reparam_store_kernel, dim3((n + 255) / 256), dim3(256), 0, s, lambda, dst, n);
    return hipGetLastError();
}

hipError_t kvq_launch_calibrate(const void* k, int batch, int n_kv_heads, int n_tokens, float alpha, float floor_,
                                float* lambda, hipStream_t s) {
    const int n = n_kv_heads * KVQ_D;
    const int64_t rows = (int64_t)batch * n_tokens;  // of one head; 256 bytes each
    if (rows >= (1ll << 31) - 256) return hipErrorInvalidValue;  // more than the device holds
    hipLaunchKernelGGL(kvq_fill_u32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, reinterpret_cast<uint32_t*>(lambda), 0u, (size_t)n);
    // About 1,024 workgroups (four per compute unit), each of at least 128 rows: the eight loads of a lane.
    const uint16_t* keys = static_cast<const uint16_t*>(k);
    uint32_t* acc = reinterpret_cast<uint32_t*>(lambda);
    if (n_tokens >= 256) {
        const int units = batch * n_kv_heads;
        const int want = std::max(1, (1024 + units - 1) / units);
        const int slice = std::max(128, ((n_tokens + want - 1) / want + 15) / 16 * 16);
        hipLaunchKernelGGL(kvq_absmax_kernel<false>, dim3(units, (n_tokens + slice - 1) / slice), dim3(256), 0, s, keys, n_kv_heads,
                           n_tokens, n_tokens, slice, 0, 16, alpha, floor_, acc);
    } else {
        // (with more heads than workgroups are wanted, slices of about 2,048 rows, so that the last ones idle little)
        const int64_t want = std::max<int64_t>((1024 + n_kv_heads - 1) / n_kv_heads, std::min<int64_t>(1024, (rows + 2047) / 2048));
        const int slice = (int)std::max<int64_t>(128, ((rows + want - 1) / want + 15) / 16 * 16);
        hipLaunchKernelGGL(kvq_absmax_kernel<true>, dim3(n_kv_heads, (unsigned)((rows + slice - 1) / slice)), dim3(256), 0, s, keys,
                           n_kv_heads, n_tokens, (int)rows, slice, 16 / n_tokens, 16 % n_tokens, alpha, floor_, acc);
    }
    return hipGetLastError();
}

hipError_t kvq_launch_stream_read(const void* buf, size_t bytes, int n_workgroups, uint32_t* sink, hipStream_t s) {
    hipLaunchKernelGGL(kvq_stream_read_kernel, dim3((unsigned)n_workgroups), dim3(256), 0, s,
                       static_cast<const u32x4*>(buf), bytes / 16, sink);
    return hipGetLastError();
}

hipError_t kvq_launch_fill_u32(uint32_t* dst, uint32_t value, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(kvq_fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, value, n);
    return hipGetLastError();
}
