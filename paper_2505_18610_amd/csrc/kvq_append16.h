// Device code shared by the append kernels and the attention kernels: the optional rotary embedding (Sec. 3.3, Eq. 9) and
// channel-wise reparameterization (Sec. 3.3, Eq. 7) of new keys, and the writing of new fp16 tokens into a tile of the
// 16-bit tier (raw values in the tile layout of kvq_layout.h).
#ifndef KVQ_APPEND16_H
#define KVQ_APPEND16_H

#include <hip/hip_runtime.h>
#include "kvq_layout.h"

namespace kvq_dev {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Quotients by launch constants: n / d = mulhi(n, magic), magic = ceil(2^32 / d), exact for n < 2^22, d <= 2^10 and for
// n, d < 2^16.  (A division of scalars is some thirty dependent instructions, several of which stood in front of the first load.)
__device__ inline int div_magic(int n, int d, uint32_t magic) { return d == 1 ? n : (int)__umulhi((uint32_t)n, magic); }
// Tells the compiler that a pointer which comes out of registers points to global memory: unlike a kernel argument's it
// would be generic, every access a flat one, and behind flat loads every wait is a wait for all loads in flight.
template <class T>
__device__ inline T* as_global(T* p) { return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p; }

__device__ inline float h2f(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
__device__ inline uint16_t f2h_rn(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }  // RNE

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_any __attribute__((aligned(4)));  // tables of fp32 need not start at a multiple of 16 bytes

// The fp16 value in the low (hi = 0) or high (hi = 1) half of w times x, rounded once to fp32: a fused multiply-add of
// mixed precision with -0 as the addend, which leaves every product as it is, instead of a conversion and a product.
__device__ inline float half_times(uint32_t w, int hi, float x) {
    float r;
    if (hi) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(x), "s"(-0.0f));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(x), "s"(-0.0f));
    return r;
}
__device__ inline uint32_t pack_rn2(float lo, float hi) {  // two floats -> fp16, nearest even
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, h2{(_Float16)lo, (_Float16)hi});
}

// K Lambda^{-1} of Eq. 7 on one pair of channels: fp32 product with the channel's reciprocal factor, rounded to
// nearest-even into fp16: two separate IEEE roundings (the products come out of asm, so the compiler cannot fuse them with the
// conversion into an instruction that rounds once, 1 fp16 ulp apart in about one element of 10^4).
__device__ inline uint32_t scale_pair(uint32_t w, float r_lo, float r_hi) {
    return pack_rn2(half_times(w, 0, r_lo), half_times(w, 1, r_hi));
}
// 8 consecutive channels; rinv: their reciprocal factors.
__device__ inline u32x4 scale_keys8(u32x4 v, const float* rinv) {
    const f32x4 r0 = *reinterpret_cast<const f32x4_any*>(rinv), r1 = *reinterpret_cast<const f32x4_any*>(rinv + 4);
    return u32x4{scale_pair(v.x, r0.x, r0.y), scale_pair(v.y, r0.z, r0.w), scale_pair(v.z, r1.x, r1.y),
                 scale_pair(v.w, r1.z, r1.w)};
}

// Rotary embedding (Sec. 3.3, Eq. 9) of one pair of channels: own * cos - partner * sin in the lower half of the head, own *
// cos + partner * sin in the upper.  Every product and the sum are separate fp32 operations, the result is rounded to fp16
// (the empty asm keeps the sum from being fused with the conversion).  sign: 0x80008000 in the lower half, where it turns
// the partner's signs over, 0 in the upper; the difference is the sum with the negated product.
__device__ inline uint32_t rope2(uint32_t own, uint32_t partner, uint32_t sign, float c0, float c1, float s0, float s1) {
    partner ^= sign;
    float lo = half_times(own, 0, c0) + half_times(partner, 0, s0);
    float hi = half_times(own, 1, c1) + half_times(partner, 1, s1);
    asm("" : "+v"(lo), "+v"(hi));
    return pack_rn2(lo, hi);
}
// Eight consecutive angles of a token's table row [cos 64 | sin 64].
struct Angles8 { f32x4 c[2], s[2]; };
__device__ inline Angles8 load_angles8(const float* row, int i0) {
    Angles8 a;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        a.c[h] = *reinterpret_cast<const f32x4_any*>(row + i0 + 4 * h);
        a.s[h] = *reinterpret_cast<const f32x4_any*>(row + 64 + i0 + 4 * h);
    }
    return a;
}
// 8 consecutive channels of one token; partner: the channels +- 64 of the same token.
__device__ inline u32x4 rope8(u32x4 own, u32x4 partner, const Angles8& a, uint32_t sign) {
    u32x4 r;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        r[e] = rope2(own[e], partner[e], sign, a.c[e >> 1][(2 * e) & 3], a.c[e >> 1][(2 * e + 1) & 3], a.s[e >> 1][(2 * e) & 3],
                     a.s[e >> 1][(2 * e + 1) & 3]);
    return r;
}

// The new rows of one unit as a buffer: a lane whose token is not new (before t_old or at or after t_new) gets an offset
// beyond it (n_new < 2^23 rows of 256 bytes end below 2^31) and reads zeros -- no branch around the loads.
struct NewRows {
    __amdgpu_buffer_rsrc_t rsrc;
    int t_old, n_new;
    __device__ NewRows(const uint16_t* in, int t_old_, int n_new_)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(in), 0, n_new_ * (KVQ_D * 2), 0x00020000)),
          t_old(t_old_), n_new(n_new_) {}
    __device__ uint32_t offset(int tok) const {
        const uint32_t rel = (uint32_t)(tok - t_old);
        return rel < (uint32_t)n_new ? rel * (uint32_t)(KVQ_D * 2) : 0x80000000u;
    }
    __device__ bool has(int tok) const { return (uint32_t)(tok - t_old) < (uint32_t)n_new; }
    __device__ bool all(int tok0) const { return tok0 >= t_old && tok0 + KVQ_TILE_TOKENS <= t_old + n_new; }  // of a tile
    __device__ u32x4 load(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0); }
    __device__ uint16_t load_half(uint32_t off) const { return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)off, 0, 0); }
    __device__ u32x4 load_stream(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 2); }
    // index of the token's table row; tokens that are not new get a row that exists
    __device__ uint64_t row(int tok) const { return (uint64_t)max(0, min(tok - t_old, n_new - 1)); }
};

// One wavefront writes the new tokens that fall into one K tile of a 16-bit page.  code_at: called behind the loads of the
// rows, gives the tile's address; tok0: its first token.
// A tile that holds no older token is written in full with streaming stores (it is read much later; slots of tokens that
// are not there yet are zero, so partially filled tiles stay well defined); otherwise only the new tokens' 16-byte chunks
// are stored.  rope: table of the new tokens, fp32 [n_new][128], or null; rinv_head: the 128 reciprocal reparameterization
// factors of this KV head, or null.
// A lane holds all four channel groups of its two tokens, so the rotation's partner channels are its own registers and
// eight angles serve two groups; all loads are issued before the arithmetic.  (With the angles read one by one and the
// partner read again, 8,192 new tokens x 32 units took 271 us with rotation against 56 without.)
// LATE: the last eight angles are asked for behind the lookup of the page, which saves the registers for one more wavefront on every
// SIMD and costs 2 to 4 % where that does not matter.
// SUBS: the lane's tokens that are taken, both of them or, with first_sub, one.
template <bool LATE, int SUBS, class Code>
__device__ inline void append16_k_tile(Code code_at, const NewRows& rows, int tok0, int lane, const float* rope,
                                       const float* rinv_head, int first_sub) {
    const int j = lane >> 4, n = lane & 15;
    const int tok1 = tok0 + 8 * (n >> 2) + (n & 3) + 4 * first_sub;
    u32x4 v[SUBS][4];
    bool isnew[SUBS];
#pragma unroll
    for (int sub = 0; sub < SUBS; ++sub) {
        const int tok = tok1 + 4 * sub;
        isnew[sub] = rows.has(tok);
        const uint32_t off = rows.offset(tok) + 16u * j;
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) v[sub][grp] = rows.load(off + 64u * grp);
    }
    Angles8 a[SUBS][2];
    if (rope) {
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            const float* row = rope + rows.row(tok1 + 4 * sub) * KVQ_D;
#pragma unroll
            for (int p = 0; p < 2; ++p)
                if (!LATE || !sub || !p) a[sub][p] = load_angles8(row, 32 * p + 8 * j);
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // all of these loads first
    uint8_t* const code = code_at();
    if (rope) {
        if (LATE) a[SUBS - 1][1] = load_angles8(rope + rows.row(tok1 + 4 * (SUBS - 1)) * KVQ_D, 32 + 8 * j);
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const u32x4 lo = rope8(v[sub][p], v[sub][p + 2], a[sub][p], 0x80008000u);
                v[sub][p + 2] = rope8(v[sub][p + 2], v[sub][p], a[sub][p], 0u);
                v[sub][p] = lo;
            }
        if (!rows.all(tok0)) {  // (uniform) the zeros of tokens that are not new: a rotated one may be negative
            asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
            for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) v[sub][grp] = isnew[sub] ? v[sub][grp] : u32x4{0u, 0u, 0u, 0u};
        }
    }
    if (rinv_head) {
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) v[sub][grp] = scale_keys8(v[sub][grp], rinv_head + 32 * grp + 8 * j);
    }
    uint8_t* const to = code + first_sub * 4096 + lane * 16;
    if (tok0 < rows.t_old) {
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub)
            if (isnew[sub]) {
#pragma unroll
                for (int grp = 0; grp < 4; ++grp) *reinterpret_cast<u32x4*>(to + (sub * 4 + grp) * 1024) = v[sub][grp];
            }
        return;
    }
#pragma unroll
    for (int c = 0; c < 4 * SUBS; ++c) __builtin_nontemporal_store(v[c >> 2][c & 3], reinterpret_cast<u32x4*>(to + c * 1024));
}

// The same for a V tile.  A tile of new tokens only goes through LDS: the rows are read with 16-byte loads (a wavefront
// instruction covers one contiguous KiB of the input), parked as [token][channel] and picked up in the tile layout (lane (j,
// n): tokens 8j .. 8j+7 of channels 16 nt + n).  Rows are rotated by 32 bytes per 8 tokens so that the four lane quarters,
// which read rows 8 apart, use different banks.  lds: 8 KiB of this wavefront alone, 16-byte aligned.  stream
// (wavefront-uniform): read the rows with streaming loads, which pass the caches by.
// A tile that holds older tokens gets the new ones' values one by one, straight from the input: there are few as a rule, one
// in a decode step, and the trip through LDS only makes the chain longer (kernel of 1 / 8 / 24 tokens x 8 units 2.6 / 3.3 / 3.6
// us, through LDS 4.7 / 4.8 / 4.6; 1 / 8 / 24 x 600 units 3.0 / 4.6 / 7.2 and 5.1 / 5.2 / 8.0).
// CHUNKS: eight, the whole tile, or four: the 64 channels from 16 first_chunk on (a wavefront instruction covers 128 bytes of each
// of eight rows; lds: 4 KiB).
template <int CHUNKS, class Code>
__device__ inline void append16_v_tile(Code code_at, const NewRows& rows, int tok0, int lane, uint8_t* lds, bool stream, int first_chunk) {
    const int j = lane >> 4, n = lane & 15;
    if (tok0 < rows.t_old) {
        uint8_t* const code = code_at();
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (rows.has(tok0 + 8 * j + i)) {
                const uint32_t off = rows.offset(tok0 + 8 * j + i) + 2u * n + 32u * first_chunk;
                uint16_t x[CHUNKS];
#pragma unroll
                for (int c = 0; c < CHUNKS; ++c) x[c] = rows.load_half(off + 32u * c);
#pragma unroll
                for (int c = 0; c < CHUNKS; ++c)
                    *reinterpret_cast<uint16_t*>(code + ((first_chunk + c) * 64 + lane) * 16 + 2 * i) = x[c];
            }
        return;
    }
    constexpr int PITCH = 32 * CHUNKS, LANES = 2 * CHUNKS, ROWS = 64 / LANES;  // bytes and lanes of a row, rows of an instruction
    const int row = lane / LANES, piece = 16 * (lane % LANES);
    u32x4 v[CHUNKS];
    if (stream) {
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) v[c] = rows.load_stream(rows.offset(tok0 + ROWS * c + row) + piece + 32 * first_chunk);
    } else {
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) v[c] = rows.load(rows.offset(tok0 + ROWS * c + row) + piece + 32 * first_chunk);
    }
    __builtin_amdgcn_sched_barrier(0);
    uint8_t* const code = code_at();
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const int tl = ROWS * c + row;
        *reinterpret_cast<u32x4*>(lds + tl * PITCH + ((piece + 32 * (tl >> 3)) & (PITCH - 1))) = v[c];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {  // a chunk of the lane's string = a channel block, tokens 8j + 0..7
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r0 = 8 * j + 2 * e, r1 = r0 + 1;      // same group of 8 rows: same rotation
            const int col = ((16 * c + n) * 2 + 32 * j) & (PITCH - 1);
            const uint32_t lo = *reinterpret_cast<const uint16_t*>(lds + r0 * PITCH + col);
            const uint32_t hi = *reinterpret_cast<const uint16_t*>(lds + r1 * PITCH + col);
            w[e] = lo | (hi << 16);
        }
        __builtin_nontemporal_store(u32x4{w[0], w[1], w[2], w[3]}, reinterpret_cast<u32x4*>(code + ((first_chunk + c) * 64 + lane) * 16));
    }
}

}  // namespace kvq_dev

#endif
