// Device code of the quantizers shared by the append, requantization and attention kernels (gfx950): Eq. 1-2 by
// "owner" lanes and the way codes travel through LDS into the tile layout of kvq_layout.h.
#ifndef KVQ_QUANT_DEV_H
#define KVQ_QUANT_DEV_H

#include "kvq_internal.h"
#include "kvq_append16.h"

namespace kvq_q {

using kvq_dev::u32x4;
using kvq_dev::h2f;
using kvq_dev::f2h_rn;

// (S, Z) of one group from its min and max (both exact fp16 values held as float), Eq. 2.
__device__ inline void group_params(float mn, float mx, int levels, uint16_t* S, uint16_t* Z, float* Sf) {
    float s32 = (mx - mn) / (float)levels;  // one fp32 subtract, one correctly rounded fp32 divide
    *S = f2h_rn(s32);
    *Z = f2h_rn(mn);
    *Sf = h2f(*S);
}
// Eq. 1 with the stored scale; a zero scale maps the whole group to code 0.
__device__ inline uint32_t code_of(float x, float mn, float Sf, int levels) {
    if (Sf == 0.0f) return 0u;
    float r = rintf((x - mn) / Sf);
    r = fminf(fmaxf(r, 0.0f), (float)levels);
    return (uint32_t)r;
}

template <int B>
__device__ inline uint32_t v_token_mask(uint32_t kb, int dw) {
    constexpr int per = 32 / B;  // slots per dword
    constexpr uint32_t field = (B == 32) ? 0xffffffffu : ((1u << B) - 1u);
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < per; ++e) {
        int slot = dw * per + e;
        int tok = slot & 7;
        if ((kb >> tok) & 1u) m |= field << (e * B);
    }
    return m;
}

template <int B>
__device__ inline void store_chunks(uint8_t* tile, int lane, const uint32_t (&str)[2 * B]) {
#pragma unroll
    for (int c = 0; c < B / 2; ++c) {
        u32x4 v = {str[4 * c], str[4 * c + 1], str[4 * c + 2], str[4 * c + 3]};
        *reinterpret_cast<u32x4*>(tile + (c * 64 + lane) * 16) = v;
    }
}
template <int B>
__device__ inline void load_chunks(const uint8_t* tile, int lane, uint32_t (&str)[2 * B]) {
#pragma unroll
    for (int c = 0; c < B / 2; ++c) {
        u32x4 v = *reinterpret_cast<const u32x4*>(tile + (c * 64 + lane) * 16);
        str[4 * c] = v.x; str[4 * c + 1] = v.y; str[4 * c + 2] = v.z; str[4 * c + 3] = v.w;
    }
}
// Streaming variants for the page-at-a-time kernels, which read and write every byte exactly once.
template <int B>
__device__ inline void load_chunks_stream(const uint8_t* tile, int lane, uint32_t (&str)[2 * B]) {
#pragma unroll
    for (int c = 0; c < B / 2; ++c) {
        u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(tile + (c * 64 + lane) * 16));
        str[4 * c] = v.x; str[4 * c + 1] = v.y; str[4 * c + 2] = v.z; str[4 * c + 3] = v.w;
    }
}
template <int B>
__device__ inline void store_chunks_stream(uint8_t* tile, int lane, const uint32_t (&str)[2 * B]) {
#pragma unroll
    for (int c = 0; c < B / 2; ++c) {
        u32x4 v = {str[4 * c], str[4 * c + 1], str[4 * c + 2], str[4 * c + 3]};
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(tile + (c * 64 + lane) * 16));
    }
}

// ------------------------------------------------------------------------------ row-owner quantizer core
// Quantized widths are produced by "owner" lanes: in each of two passes over a 32-token tile, lane l owns the
// group (token 16*pass + l/4, channels 32*(l%4) .. +31): 64 contiguous bytes, so the minimum and maximum need
// no cross-lane traffic.  The owner writes its 32 codes as bytes to LDS -- [token][channel] for a K tile,
// [channel][token] for a V tile -- from where every lane gathers the slots of the tile layout with 8-byte reads.
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

__device__ inline uint32_t pk_min_u(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(half2v, a), __builtin_bit_cast(half2v, b)));
}
__device__ inline uint32_t pk_max_u(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(half2v, a), __builtin_bit_cast(half2v, b)));
}

// x - mn for the fp16 value in the low (hi = 0) or high (hi = 1) half of w, in one instruction: x * 1.0 - mn with
// the single rounding of a fused multiply-add, which is the rounding of the fp32 subtraction (the conversion of
// x to fp32 is exact), instead of a conversion followed by a subtraction.
__device__ inline float half_minus(uint32_t w, int hi, float mn) {
    float r;
    if (hi) asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(mn));
    else asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(w), "v"(mn));
    return r;
}

// The owners' rows of 16 tokens per pass from tok0 on: all 16-byte loads in flight together; tokens that are not new
// read as zeros, which is what they quantize.
template <int PASSES>
__device__ inline void load_owner_rows(uint32_t (&w)[PASSES][16], const kvq_dev::NewRows& rows, int tok0, int lane) {
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        const uint32_t off = rows.offset(tok0 + 16 * pass + (lane >> 2)) + 64u * (lane & 3);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const u32x4 v = rows.load(off + 16u * c);
            w[pass][4 * c] = v.x; w[pass][4 * c + 1] = v.y; w[pass][4 * c + 2] = v.z; w[pass][4 * c + 3] = v.w;
        }
    }
}
// Rotation and reparameterization of the owners' keys of one pass, as configured.  The owner of the channels +- 64 of the same
// token is the lane two further in the quad, so the partner channels are a data-parallel move away; a lane reads the 32 angles of
// its channels with 16-byte loads, which the callers issue together with the rows.  (With the partner read again from memory and
// the angles one by one, 8,192 new tokens x 32 units into 8, 4 or 2 bits took 166 to 172 us with rotation, 45 to 52 without.)
struct OwnerAngles { kvq_dev::Angles8 a[4]; };
__device__ inline void load_owner_angles(OwnerAngles& a, const kvq_dev::NewRows& rows, int tok, int lane, const float* rope) {
    const float* row = rope + rows.row(tok) * KVQ_D;
#pragma unroll
    for (int c = 0; c < 4; ++c) a.a[c] = kvq_dev::load_angles8(row, 32 * (lane & 1) + 8 * c);
}
__device__ inline void rotate_owner_keys(uint32_t (&w)[16], const OwnerAngles& a, bool isnew, bool all_new, int lane) {
    const int grp = lane & 3;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        u32x4 own = {w[4 * c], w[4 * c + 1], w[4 * c + 2], w[4 * c + 3]}, partner;
#pragma unroll
        for (int e = 0; e < 4; ++e)  // quad_perm 2 3 0 1
            partner[e] = (uint32_t)__builtin_amdgcn_mov_dpp((int)own[e], 0x4E, 0xf, 0xf, true);
        own = kvq_dev::rope8(own, partner, a.a[c], grp >= 2 ? 0u : 0x80008000u);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[4 * c + e] = own[e];
    }
    if (!all_new) {  // (uniform) the zeros of tokens that are not new: a rotated one may be negative
        asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
        for (int e = 0; e < 16; ++e) w[e] = isnew ? w[e] : 0u;
    }
}
__device__ inline void scale_owner_keys(uint32_t (&w)[16], int lane, const float* rinv_head) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const u32x4 v = kvq_dev::scale_keys8(u32x4{w[4 * c], w[4 * c + 1], w[4 * c + 2], w[4 * c + 3]}, rinv_head + 32 * (lane & 3) + 8 * c);
        w[4 * c] = v.x; w[4 * c + 1] = v.y; w[4 * c + 2] = v.z; w[4 * c + 3] = v.w;
    }
}

#define KVQ_LDS_CODES_K 4096                       // K: [32 tokens][128 channels] code bytes
#define KVQ_LDS_VGRP (32 * 32 + 16)                // V: per group [32 channels][32 tokens] code bytes, skewed
#define KVQ_LDS_CODES (4 * KVQ_LDS_VGRP)           // room for either arrangement

// Eq. 1-2 for the 32 fp16 values in w[16] (two per dword).  The low 8 bits (B = 16: 16 bits) of codes[e] receive the code of
// element e; the bits above them are not the code's.
// gspan = G / 32: a quantization group of G = 64 or 128 channels spans 2 or 4 neighbouring owner lanes (the
// owners of one token's four 32-channel runs are lanes 4k .. 4k+3), which then share min, max and so (S, Z).
//
// The definition rounds the correctly rounded fp32 quotient (x - Z) / S to the nearest integer.  The quotient comes from a
// reciprocal multiply and one correction by the exact remainder: with y = rcp(S) (1 ulp), t = d y and r = d - t S, which a
// fused multiply-add forms exactly (S has 11 significant bits and t is off by a few ulp, so r has at most 14), q = t + r y
// differs from d / S by less than 2^-20 ulp before its rounding.  d / S itself is never nearer than 2^-12 ulp to a point
// where that rounding changes: d - m S, m a midpoint of two fp32 numbers, is a non-zero multiple of half an ulp of m times
// the last place of S.  So q is the IEEE quotient for every d and S that occur (nothing here is subnormal in fp32), at
// every width, without a division.  Five operations per element (six at 16 bits); the division that used to be carried
// out near half-integers cost a quarter of the 8-bit passes a slow path of twice the code, and the 16-bit codes all of
// theirs.
template <int B>
__device__ inline void quantize_owner(const uint32_t (&w)[16], uint32_t (&codes)[32], uint16_t* S, uint16_t* Z,
                                      int gspan) {
    constexpr int levels = (1 << B) - 1;
    uint32_t mn2 = pk_min_u(w[0], w[1]), mx2 = pk_max_u(w[0], w[1]);  // (no plain copy of a loaded register: the copy
#pragma unroll                                                        //  would be placed, with a full wait, beside the load)
    for (int k = 2; k < 16; ++k) { mn2 = pk_min_u(mn2, w[k]); mx2 = pk_max_u(mx2, w[k]); }
    float mn = fminf(h2f((uint16_t)(mn2 & 0xffff)), h2f((uint16_t)(mn2 >> 16)));
    float mx = fmaxf(h2f((uint16_t)(mx2 & 0xffff)), h2f((uint16_t)(mx2 >> 16)));
    if (gspan >= 2) { mn = fminf(mn, __shfl_xor(mn, 1)); mx = fmaxf(mx, __shfl_xor(mx, 1)); }
    if (gspan >= 4) { mn = fminf(mn, __shfl_xor(mn, 2)); mx = fmaxf(mx, __shfl_xor(mx, 2)); }
    float Sf;
    group_params(mn, mx, levels, S, Z, &Sf);
    const float y = Sf != 0.0f ? __builtin_amdgcn_rcpf(Sf) : 0.0f;  // a zero scale maps the whole group to code 0
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const float d = half_minus(w[e >> 1], e & 1, mn);
        const float t = d * y;
        const float q = fmaf(fmaf(-t, Sf, d), y, t);
        // rounded to the nearest even integer by adding 1.5 * 2^23, which leaves it in the low bits (those of a NaN are 0);
        // 16-bit codes are clamped one by one: a scale rounded down lifts every other group's maximum above the top level
        codes[e] = __float_as_uint((B == 16 ? __builtin_amdgcn_fmed3f(q, 0.0f, (float)levels) : q) + 12582912.0f);
    }
    if constexpr (B < 16) {
        // In the narrow widths only a scale rounded down to a subnormal lifts a code above the top level, and no element's
        // quotient exceeds that of the group maximum (x <= mx, every step is monotone): decided once per group.
        const float dm = mx - mn, tm = dm * y;
        const bool over = fmaf(fmaf(-tm, Sf, dm), y, tm) > (float)levels + 0.25f;
        if (__any(over)) {
            asm volatile("" ::: "memory");  // keeps this a branch
            const float top = over ? (float)levels + 12582912.0f : INFINITY;
#pragma unroll
            for (int e = 0; e < 32; ++e)  // (a NaN, whose code is 0, is not above the top)
                codes[e] = __uint_as_float(codes[e]) > top ? __float_as_uint(top) : codes[e];
        }
    }
}

// Owner -> LDS: byte BYTE of every code.  tl = token in tile, grp = channel group, which = 0 K / 1 V.
template <int BYTE = 0>
__device__ inline void scatter_codes(uint8_t* lds, int which, int tl, int grp, const uint32_t (&codes)[32]) {
    if (!which) {
        uint32_t d[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            d[k] = __builtin_amdgcn_perm(codes[4 * k + 1], codes[4 * k], 0x0c0c0400u + 0x0101u * BYTE) |
                   __builtin_amdgcn_perm(codes[4 * k + 3], codes[4 * k + 2], 0x04000c0cu + 0x01010000u * BYTE);
        u32x4* dst = reinterpret_cast<u32x4*>(lds + tl * 128 + grp * 32);
        dst[0] = u32x4{d[0], d[1], d[2], d[3]};
        dst[1] = u32x4{d[4], d[5], d[6], d[7]};
    } else {
        uint8_t* dst = lds + grp * KVQ_LDS_VGRP + tl;
#pragma unroll
        for (int c = 0; c < 32; ++c) dst[c * 32] = (uint8_t)(codes[c] >> (8 * BYTE));
    }
}

// 8 code bytes (b0 in the low byte of w0) -> 8 codes of B bits, packed little-endian into the low 8*B bits.
template <int B>
__device__ inline void pack8(uint32_t w0, uint32_t w1, uint32_t* lo, uint32_t* hi) {
    if constexpr (B == 8) {
        *lo = w0; *hi = w1;
    } else if constexpr (B == 4) {
        uint32_t x = w0 | (w0 >> 4), y = w1 | (w1 >> 4);
        *lo = __builtin_amdgcn_perm(y, x, 0x06040200u);
        *hi = 0u;
    } else {
        uint32_t x = w0 | (w0 >> 6), y = w1 | (w1 >> 6);
        x |= x >> 12; y |= y >> 12;
        *lo = __builtin_amdgcn_perm(y, x, 0x0c0c0400u);
        *hi = 0u;
    }
}

// LDS -> the lane's packed string of the tile layout.
template <int B>
__device__ inline void gather_string(const uint8_t* lds, int which, int lane, uint32_t (&str)[2 * B]) {
    const int j = lane >> 4, n = lane & 15;
#pragma unroll
    for (int d = 0; d < 2 * B; ++d) str[d] = 0u;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const uint8_t* src;
        if (!which) {
            const int sub = p >> 2, grp = p & 3;
            const int t = 8 * (n >> 2) + 4 * sub + (n & 3);
            src = lds + t * 128 + grp * 32 + 8 * j;
        } else {
            const int ch = 16 * p + n;  // piece p = channel block nt
            src = lds + (ch >> 5) * KVQ_LDS_VGRP + (ch & 31) * 32 + 8 * j;
        }
        const uint32_t w0 = reinterpret_cast<const uint32_t*>(src)[0], w1 = reinterpret_cast<const uint32_t*>(src)[1];
        uint32_t lo, hi;
        pack8<B>(w0, w1, &lo, &hi);
        if constexpr (B == 8) { str[2 * p] = lo; str[2 * p + 1] = hi; }
        else if constexpr (B == 4) { str[p] = lo; }
        else { str[p >> 1] |= lo << (16 * (p & 1)); }
    }
}

__device__ inline void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The attention kernel multiplies probabilities (<= 1) by up to 64 and by the V scale in fp16; a cache that ever
// holds a V scale of 256 or more (a value range no attention layer produces) is marked and takes the kernel's
// overflow-proof path instead.
__device__ inline void note_large_v_scale(const KvqVMark& mark, int which, uint16_t S) {
    if (which && h2f(S) >= 256.0f) __hip_atomic_store(mark.word, mark.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Owner lanes write the (S, Z) of their group straight to the tile's metadata.
__device__ inline void store_meta_owner(uint8_t* meta, int which, int tl, int grp, uint16_t S, uint16_t Z) {
    uint16_t* ms = reinterpret_cast<uint16_t*>(meta + (which ? 512 : 0));
    uint16_t* mz = reinterpret_cast<uint16_t*>(meta + (which ? 768 : 256));
    const int idx = which ? kvq_vmeta_index(tl, grp) : tl * 4 + grp;
    ms[idx] = S;
    mz[idx] = Z;
}

// ------------------------------------------------------------------------------------------------ append
// Descriptor of the page a string lies in, and the table entries of the call's new pages, which the first workgroup writes.
// (The offsets become scalar inside each branch: left alone, the two branches are merged into one load through a selected
//  pointer, which can only be a flat load, and while a flat load is pending every wait for a global load becomes a wait
//  for all of them.)
// SCALAR: a call of more pages than the arguments hold reads the table, which it does not write, through the constant cache: a vector
// load is waited for behind all the rows asked for before it, which the quantizers of keys that are ready feel (2 units x 40,031
// tokens, 626 pages, into 8 / 4 bits 14.2 / 14.3 us with vector loads and 13.4 / 13.4; the integer tier 19.1 and 18.3), the others do not.
template <bool SCALAR>
__device__ inline KvqPageDesc append_desc(const KvqPageDesc* table, const KvqAppendPages& ap, int page) {
    KvqPageDesc r;
    r.bits = 0u;
    r.int16 = 0u;
    page = __builtin_amdgcn_readfirstlane(page);
    if (ap.n == 0 && SCALAR) {
        const auto* const entry = (const __attribute__((address_space(4))) KvqPageDesc*)(uintptr_t)(table + page);
        r.code_off256 = entry->code_off256;
        r.meta_off256 = entry->meta_off256;
    } else if (ap.n == 0) {
        r.code_off256 = __builtin_amdgcn_readfirstlane(table[page].code_off256);
        r.meta_off256 = __builtin_amdgcn_readfirstlane(table[page].meta_off256);
    } else {
        r.code_off256 = ap.code_off256[page - ap.first_page];
        r.meta_off256 = ap.meta_off256[page - ap.first_page];
        asm volatile("" : "+s"(r.code_off256), "+s"(r.meta_off256));
    }
    return r;
}
__device__ inline void write_fresh_pages(KvqPageDesc* table, const KvqAppendPages& ap, int lane) {
    if (blockIdx.x != 0 || blockIdx.y != 0) return;
    for (int i = ap.fresh + lane; i < ap.n; i += 64)
        table[ap.first_page + i] = KvqPageDesc{ap.code_off256[i], ap.meta_off256[i], ap.bits, ap.int16};
}

}  // namespace kvq_q

#endif
