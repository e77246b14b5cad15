// Quantisation of one 32-token tile with G = 32 by one wavefront, everything in registers (KIVI Section 3.1 formula, Section
// 3.3 grouping): the bulk forms of a prompt, and the flush that rides in a decoding launch.  The lanes load the elements
// whose codes they will pack, group minimum and maximum come from packed fp16 min / max in registers plus at most two
// cross-lane steps, the partial words of the lanes that share a word are combined with DPP moves, and nothing goes
// through LDS.  (Instruction counts and rates: at the kernels, kivi_quantize.hip.)
//
// The value of a code is a bit contract: fp32 subtract, IEEE fp32 division, round-half-even, clamp (encode()).  The fast
// path reaches the same code with one explicit fused multiply-add per element and falls back to encode() where a quotient
// lies close enough to a rounding tie for the two to differ.  The only fused operations are the ones written as fmaf();
// no other product is added to anything, but for the tolerance in group_const and sums of codes, which are exact.
#pragma once

#include "kivi_internal.h"

#include <hip/hip_fp16.h>

#include <type_traits>

namespace kivi {
namespace tile {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
// packed fp16 minimum / maximum (v_pk_min_f16 / v_pk_max_f16): exact, no arithmetic.  Written as
// instructions: the builtins make the compiler quiet signalling NaNs first (one more instruction per
// operand), which finite inputs -- the precondition of the quantiser -- do not need.
__device__ __forceinline__ half2v pk_min(half2v a, half2v b) {
    half2v r;
    asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ half2v pk_max(half2v a, half2v b) {
    half2v r;
    asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ uint32_t encode(float x, float z, float s, float levels) {
    float r = (x - z) / s;                 // IEEE fp32 division (correctly rounded)
    r = __builtin_rintf(r);                // round half to even
    r = fminf(fmaxf(r, 0.0f), levels);     // NaN (0/0) -> 0
    return s == 0.0f ? 0u : (uint32_t)r;
}

// Group constants: zero-point and scale (for the exact path), and for the fast path y ~ 1/s,
// c0 = fl(-z * y) and the tolerance below (y = c0 = 0 when the scale is 0, which makes every code
// of the group 0).  The key kernel keeps them in LDS as one array per constant, so that the
// constants of the consecutive channels a word covers are read as vectors (3 % on that kernel; the
// same for the consecutive tokens of a value word gained 3 % at 4 bits and lost 4 % at 2 bits).
struct GroupConst { float z, s, y, c0, tol; };

__device__ __forceinline__ GroupConst group_const(float lo, float s) {
#pragma clang fp contract(off)
    // y: the hardware reciprocal (1 ulp: relative error <= 2^-23), one instruction instead of a division
    const float y = s == 0.0f ? 0.0f : __builtin_amdgcn_rcpf(s);
    const float c0 = -lo * y;
    // q' = fl(x * y + c0) against the contract's q = fl(fl(x - z) / s), with Q the exact quotient:
    // |q - Q| <= Q * 2^-23 and |q' - Q| <= Q * 2^-22 + |z / s| * 2^-22 * 1.001 (error of y in both
    // products, roundings of c0 and of the sum), so for Q <= 16.1:  |q' - q| < 5.8e-6 + |c0| * 2.4e-7.
    // Twice that as tolerance.
    // (scale below the smallest normal fp16 number: its rounding error is not relative, the quotient
    // can pass `levels`: tolerance 1 = always the exact path)
    return GroupConst{lo, s, y, c0, (s != 0.0f && s < 6.103515625e-05f) ? 1.0f : 1.2e-5f + fabsf(c0) * 4.8e-7f};
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;      // quad_perm [1,0,3,2], [2,3,0,1]
__device__ __forceinline__ uint32_t as_bits(half2v x) {
    union { half2v h; uint32_t u; } a;
    a.h = x;
    return a.u;
}
__device__ __forceinline__ half2v as_half2(uint32_t x) {
    union { half2v h; uint32_t u; } a;
    a.u = x;
    return a.h;
}
__device__ __forceinline__ float half_bits_to_float(uint32_t low16) { return (float)as_half2(low16).x; }
// {a.x, b.x} and {a.y, b.y} (one byte-permute instruction each)
__device__ __forceinline__ half2v low_halves(half2v a, half2v b) {
    return as_half2(__builtin_amdgcn_perm(as_bits(b), as_bits(a), 0x05040100u));
}
__device__ __forceinline__ half2v high_halves(half2v a, half2v b) {
    return as_half2(__builtin_amdgcn_perm(as_bits(b), as_bits(a), 0x07060302u));
}
template <int CTRL>
__device__ __forceinline__ half2v dpp_h2(half2v x) {
    union { half2v h; int i; } a, r;
    a.h = x;
    r.i = __builtin_amdgcn_mov_dpp(a.i, CTRL, 0xF, 0xF, true);
    return r.h;
}
// A wavefront-uniform pointer pinned to scalar registers: keeps the compiler from folding a lane offset
// into it early and then carrying every row address in vector registers (64-bit vector multiply-adds).
typedef const half2v __attribute__((address_space(1)))* GlobalHalf2Ptr;       // keeps the loads global (not flat)
__device__ __forceinline__ GlobalHalf2Ptr uniform_pointer(const void* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<GlobalHalf2Ptr>(((uint64_t)hi << 32) | lo);
}
// mask ? a : b per bit (one bitfield-insert instruction)
__device__ __forceinline__ uint32_t select_bits(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

__device__ __forceinline__ float encode_fast16(_Float16 x, float y, float c0, float& dev) {
    const float q = fmaf((float)x, y, c0);
    const float r = __builtin_rintf(q);
    dev = fmaxf(dev, fabsf(q - r));
    return r;
}

// Keys: lane l holds channels 2l, 2l + 1 of all 32 tokens (each row load of the wavefront is one
// contiguous 256-byte row).  A channel's group is the lane's own column: no cross-lane step for
// minimum and maximum.  A word of the packed tile (tokens t0 and t0 + 16, 8 or 4 consecutive
// channels) is shared by 4 (B = 2) or 2 (B = 4) neighbouring lanes.
// x: the lane's two channels of the 32 tokens; put_group(scales, zero-points) of the two channels; put_word(index, word)
template <int BITS, class PutGroup, class PutWord>
__device__ __forceinline__ void quantize_key_tile(const half2v (&x)[kTileTokens], int lane, PutGroup&& put_group, PutWord&& put_word) {
    constexpr float levels = (float)((1 << BITS) - 1);
    half2v mn[16], mx[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) { mn[i] = pk_min(x[i], x[i + 16]); mx[i] = pk_max(x[i], x[i + 16]); }
#pragma unroll
    for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
        for (int i = 0; i < w; ++i) { mn[i] = pk_min(mn[i], mn[i + w]); mx[i] = pk_max(mx[i], mx[i + w]); }

    float y[2], c0[2], zf[2], sf[2], tol = 0.f;
    half2v s2, z2;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float lo = (float)mn[0][i], hi = (float)mx[0][i];
        const _Float16 s16 = (_Float16)((hi - lo) / levels);          // fp32 division, rounded to nearest even
        const GroupConst gc = group_const(lo, (float)s16);
        y[i] = gc.y; c0[i] = gc.c0; zf[i] = gc.z; sf[i] = gc.s;
        tol = fmaxf(tol, gc.tol);
        s2[i] = s16;
        z2[i] = mn[0][i];
    }
    put_group(s2, z2);

    const int ks = lane >> 4, q = (lane >> 2) & 3, k = lane & 3;     // channel 2l = ks*32 + q*8 + 2k
    const int shift = BITS == 2 ? 2 * k : 4 * (k & 1);
    const uint32_t m0 = 0u - (uint32_t)(k & 1), m1 = 0u - (uint32_t)(k >> 1);
    const float thr = 0.5f - tol;
    // four tokens t0 (and their partners t0 + 16) at a time: byte i*2 + uo of the lane's partial word
    // holds the code of (channel 2l + i, token t0 + 16 uo) -- bits (e&1)*16 + 8*uo of the layout --
    // and the shift moves it to the lane's channel pair
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
        uint32_t pw[4];
        float dev = 0.f;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            const int t0 = blk * 4 + tt;
            uint32_t w = 0;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int uo = 0; uo < 2; ++uo)
                    w = __builtin_amdgcn_cvt_pk_u8_f32(encode_fast16(x[t0 + 16 * uo][i], y[i], c0[i], dev), i * 2 + uo, w);
            pw[tt] = w;
        }
        if (dev > thr) {      // rare: a quotient next to a rounding tie; redo the lane's 16 codes with true divisions
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                const int t0 = blk * 4 + tt;
                uint32_t w = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int uo = 0; uo < 2; ++uo)
                        w |= encode((float)x[t0 + 16 * uo][i], zf[i], sf[i], levels) << (8 * (i * 2 + uo));
                pw[tt] = w;
            }
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) pw[tt] <<= shift;
        // The lanes that share a word combine their partial words so that each ends up with a different
        // token's complete word (a transpose over the lane group, 3 instructions per exchange): with the
        // odd neighbour, the odd lane keeps the odd tokens and hands over the even ones, and vice versa;
        // at 2 bits the same once more two lanes apart.
        const uint32_t a = select_bits(m0, pw[1], pw[0]) | dpp_u32<kQuadXor1>(select_bits(m0, pw[0], pw[1]));   // token (k & 1)
        const uint32_t c = select_bits(m0, pw[3], pw[2]) | dpp_u32<kQuadXor1>(select_bits(m0, pw[2], pw[3]));   // token 2 + (k & 1)
        if (BITS == 2) {
            const uint32_t w = select_bits(m1, c, a) | dpp_u32<kQuadXor2>(select_bits(m1, a, c));               // token k
            put_word((q * 16 + blk * 4 + k) * 4 + ks, w);
        } else {
            const int i = ks * 2 + (k >> 1);
            put_word((i >> 2) * 256 + (q * 16 + blk * 4 + (k & 1)) * 4 + (i & 3), a);
            put_word((i >> 2) * 256 + (q * 16 + blk * 4 + 2 + (k & 1)) * 4 + (i & 3), c);
        }
    }
}

// Values: lane (tl = l / 16, seg = l % 16) holds channels seg*8 .. seg*8 + 7 of tokens 8 tl .. 8 tl + 7
// (a 16-byte load per token).  A group is 32 channels of a token = the 4 lanes of a quad; lane jj of
// the quad derives the constants of tokens jj and jj + 4 and the others get them by quad broadcasts.
// A word (8 tokens, channels c and c + 16) is shared by the lanes seg and seg ^ 2.
// put_entry(index, scale, zero-point): index = token * 4 + group inside the tile; put_word as above
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
union ValueRow {
    uint4v v4;
    half2v h2[4];
    _Float16 h[8];
};
template <int BITS, class PutEntry, class PutWord>
__device__ __forceinline__ void quantize_value_tile(const ValueRow (&x)[8], int lane, PutEntry&& put_entry, PutWord&& put_word) {
    constexpr float levels = (float)((1 << BITS) - 1);
    const int tl = lane >> 4, seg = lane & 15, g = seg >> 2, jj = seg & 3, odd = (seg >> 1) & 1;
    // Group minimum / maximum of every token.  In the lane: packed fp16 min / max over its 8 channels
    // (exact, no arithmetic); the halves of two tokens are then combined into one register
    // (token i in the low half, token i + 1 in the high half), so that the two exchanges inside the quad
    // serve two tokens at once.  Lane jj adopts the tokens jj and jj + 4.
    half2v pmn[4], pmx[4];
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        half2v lo2[2], hi2[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            lo2[d] = pk_min(pk_min(x[i + d].h2[0], x[i + d].h2[1]), pk_min(x[i + d].h2[2], x[i + d].h2[3]));
            hi2[d] = pk_max(pk_max(x[i + d].h2[0], x[i + d].h2[1]), pk_max(x[i + d].h2[2], x[i + d].h2[3]));
        }
        half2v mn = pk_min(low_halves(lo2[0], lo2[1]), high_halves(lo2[0], lo2[1]));
        half2v mx = pk_max(low_halves(hi2[0], hi2[1]), high_halves(hi2[0], hi2[1]));
        mn = pk_min(mn, dpp_h2<kQuadXor1>(mn)); mx = pk_max(mx, dpp_h2<kQuadXor1>(mx));
        mn = pk_min(mn, dpp_h2<kQuadXor2>(mn)); mx = pk_max(mx, dpp_h2<kQuadXor2>(mx));
        pmn[i >> 1] = mn;
        pmx[i >> 1] = mx;
    }
    float my_lo[2], my_hi[2];
    {
        const uint32_t upper = 0u - (uint32_t)(jj >> 1);     // tokens 2, 3 (6, 7) are in the second register of a slot
        const int sh = 16 * (jj & 1);
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            my_lo[sl] = half_bits_to_float(select_bits(upper, as_bits(pmn[2 * sl + 1]), as_bits(pmn[2 * sl])) >> sh);
            my_hi[sl] = half_bits_to_float(select_bits(upper, as_bits(pmx[2 * sl + 1]), as_bits(pmx[2 * sl])) >> sh);
        }
    }
    float gy[2], gc0[2], gz[2], gs[2], tol = 0.f;
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
        const _Float16 s16 = (_Float16)((my_hi[sl] - my_lo[sl]) / levels);
        const GroupConst gc = group_const(my_lo[sl], (float)s16);
        gy[sl] = gc.y; gc0[sl] = gc.c0; gz[sl] = gc.z; gs[sl] = gc.s;
        tol = fmaxf(tol, gc.tol);
        put_entry((tl * 8 + jj + 4 * sl) * 4 + g, s16, (_Float16)my_lo[sl]);
    }
    tol = fmaxf(tol, dpp_f32<kQuadXor1>(tol));
    tol = fmaxf(tol, dpp_f32<kQuadXor2>(tol));
    const float thr = 0.5f - tol;
    // constants of token i for every lane of the quad: from lane i & 3, slot i >> 2
    auto quad_bcast = [](float v, auto sel) {
        constexpr int S = decltype(sel)::value;
        return dpp_f32<S | (S << 2) | (S << 4) | (S << 6)>(v);
    };
    float yi[8], ci[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        auto pick = [&](const float (&a)[2]) {
            const float v = a[i >> 2];
            switch (i & 3) {
                case 0: return quad_bcast(v, std::integral_constant<int, 0>{});
                case 1: return quad_bcast(v, std::integral_constant<int, 1>{});
                case 2: return quad_bcast(v, std::integral_constant<int, 2>{});
                default: return quad_bcast(v, std::integral_constant<int, 3>{});
            }
        };
        yi[i] = pick(gy);
        ci[i] = pick(gc0);
    }

    constexpr int WPC = BITS / 2;                    // words per channel: tokens 0-7 (B = 2) or 0-3, 4-7 (B = 4)
    uint32_t wq[8][WPC];
    // two channels at a time; bit of token e inside its word: (e&1)*16 + B*((e>>1) & (8/B - 1)), plus 8 for
    // the lanes whose channels are the upper 16 of their 32-channel group (odd)
#pragma unroll
    for (int jb = 0; jb < 4; ++jb) {
        float dev = 0.f;
#pragma unroll
        for (int j = 2 * jb; j < 2 * jb + 2; ++j) {
            // the codes of a word lie in bits 0-7 and 16-23: their sum is exact in one fp32 number
            float acc[WPC];
#pragma unroll
            for (int a = 0; a < WPC; ++a) acc[a] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int bit = (e & 1) * 16 + BITS * ((e >> 1) & (8 / BITS - 1));
                float& dstf = acc[BITS == 2 ? 0 : (e >> 2)];
                dstf = fmaf(encode_fast16(x[e].h[j], yi[e], ci[e], dev), (float)(1u << bit), dstf);
            }
#pragma unroll
            for (int a = 0; a < WPC; ++a) wq[j][a] = (uint32_t)acc[a];
        }
        // a quotient next to a rounding tie anywhere in the wavefront (rare): all lanes redo these two
        // channels with true divisions (uniform branch: the quad broadcasts inside need every lane)
        if (__builtin_amdgcn_ballot_w64(dev > thr) != 0) {
            float zi[8], si[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                auto pick = [&](const float (&a)[2]) {
                    const float v = a[i >> 2];
                    switch (i & 3) {
                        case 0: return quad_bcast(v, std::integral_constant<int, 0>{});
                        case 1: return quad_bcast(v, std::integral_constant<int, 1>{});
                        case 2: return quad_bcast(v, std::integral_constant<int, 2>{});
                        default: return quad_bcast(v, std::integral_constant<int, 3>{});
                    }
                };
                zi[i] = pick(gz);
                si[i] = pick(gs);
            }
#pragma unroll
            for (int j = 2 * jb; j < 2 * jb + 2; ++j) {
                uint32_t w[WPC];
#pragma unroll
                for (int a = 0; a < WPC; ++a) w[a] = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int bit = (e & 1) * 16 + BITS * ((e >> 1) & (8 / BITS - 1));
                    w[BITS == 2 ? 0 : (e >> 2)] |= encode((float)x[e].h[j], zi[e], si[e], levels) << bit;
                }
#pragma unroll
                for (int a = 0; a < WPC; ++a) wq[j][a] = w[a];
            }
        }
    }
    // combine with the lane that holds the other 16 channels of the group, then each of the two stores
    // four of the eight channels' words
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int a = 0; a < WPC; ++a) {
            uint32_t w = wq[j][a] << (8 * odd);
            w |= dpp_u32<kQuadXor2>(w);
            wq[j][a] = w;
        }
    const uint32_t omask = 0u - (uint32_t)odd;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int a = 0; a < WPC; ++a) {
            const uint32_t mine = (wq[m + 4][a] & omask) | (wq[m][a] & ~omask);     // a bitfield insert, not an indexed array
            const int r = (seg & 1) * 8 + m + 4 * odd;             // channel % 16
            if (BITS == 2) {
                put_word((tl * 16 + r) * 4 + g, mine);
            } else {
                const int i = g * 2 + a;
                put_word((i >> 2) * 256 + (tl * 16 + r) * 4 + (i & 3), mine);
            }
        }
}

// The 32 rows before ring slot `start` (the first one after them), channels 2 lane, 2 lane + 1
template <class Params>
__device__ __forceinline__ void load_key_rows_before(const Params& p, int64_t unit, int start, int lane, half2v (&x)[kTileTokens]) {
    const int first = start - kTileTokens, k0 = first < 0 ? first + p.cap_r : first;
    const char* kr = reinterpret_cast<const char*>(p.k_resid + unit * p.cap_r * kHeadDim);
#pragma unroll
    for (int t = 0; t < kTileTokens; ++t) {
        const int i = k0 + t;
        x[t] = *reinterpret_cast<const half2v*>(kr + (uint32_t)((i >= p.cap_r ? i - p.cap_r : i) * (kHeadDim * 2) + lane * 4));
    }
}
// ... rows 8 (lane / 16) + i, channels 8 (lane % 16) ..
template <class Params>
__device__ __forceinline__ void load_value_rows_before(const Params& p, int64_t unit, int start, int lane, ValueRow (&y)[8]) {
    const int first = start - kTileTokens, v0 = first < 0 ? first + p.cap_r : first;
    const __half* vr = p.v_resid + unit * p.cap_r * kHeadDim + (lane & 15) * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int at = v0 + (lane >> 4) * 8 + i;
        y[i].v4 = *reinterpret_cast<const uint4v*>(vr + (at >= p.cap_r ? at - p.cap_r : at) * kHeadDim);
    }
}

// The tile that leaves the window in a decoding step (K and V split alike, G = 32): the 32 tokens before the window, out of the rings
// of `unit` into a slot in LDS (key codes, value codes, key scales, key zero-points, value scales, value zero-points) and, with
// `store`, into tile `at` of the packed arrays.  One wavefront; wave_lds_sync() or the like has to follow.
template <int BITS>
__device__ __forceinline__ void flush_tile(const DecodeParams& p, int64_t unit, int64_t at, int lane, unsigned char* slot, bool store) {
    constexpr int kCodeBytes = kTileTokens * kHeadDim * BITS / 8;
    half2v x[kTileTokens];
    ValueRow y[8];
    load_key_rows_before(p, unit, p.k_r_start, lane, x);
    load_value_rows_before(p, unit, p.v_r_start, lane, y);
    uint32_t* kcodes = const_cast<uint32_t*>(p.k_codes) + at * (kCodeBytes / 4);
    uint32_t* vcodes = const_cast<uint32_t*>(p.v_codes) + at * (kCodeBytes / 4);
    uint32_t* lds = reinterpret_cast<uint32_t*>(slot);
    _Float16* lds_scales = reinterpret_cast<_Float16*>(slot + 2 * kCodeBytes);
    auto put_pair = [&](const __half* array, int which, half2v v) {
        if (store) *reinterpret_cast<half2v*>(const_cast<__half*>(array) + at * kHeadDim + 2 * lane) = v;
        *reinterpret_cast<half2v*>(lds_scales + which * 128 + 2 * lane) = v;
    };
    quantize_key_tile<BITS>(x, lane,
        [&](half2v s2, half2v z2) {
            put_pair(p.k_scale, 0, s2);
            put_pair(p.k_zero, 1, z2);
        },
        [&](int i, uint32_t w) {
            if (store) kcodes[i] = w;
            lds[i] = w;
        });
    quantize_value_tile<BITS>(y, lane,
        [&](int i, _Float16 s, _Float16 z) {
            if (store) {
                reinterpret_cast<_Float16*>(const_cast<__half*>(p.v_scale))[at * 128 + i] = s;
                reinterpret_cast<_Float16*>(const_cast<__half*>(p.v_zero))[at * 128 + i] = z;
            }
            lds_scales[256 + i] = s;
            lds_scales[384 + i] = z;
        },
        [&](int i, uint32_t w) {
            if (store) vcodes[i] = w;
            lds[kCodeBytes / 4 + i] = w;
        });
}

// Keys and values of such a tile into the packed arrays alone, one wavefront each; start: the rings' first slots after the flush
template <int BITS, class Params>
__device__ __forceinline__ void flush_keys(const Params& p, int64_t unit, int64_t at, int start, int lane) {
    half2v x[kTileTokens];
    load_key_rows_before(p, unit, start, lane, x);
    uint32_t* codes = const_cast<uint32_t*>(p.k_codes) + at * (kTileTokens * kHeadDim * BITS / 32);
    quantize_key_tile<BITS>(x, lane,
        [&](half2v s2, half2v z2) {
            *reinterpret_cast<half2v*>(const_cast<__half*>(p.k_scale) + at * kHeadDim + 2 * lane) = s2;
            *reinterpret_cast<half2v*>(const_cast<__half*>(p.k_zero) + at * kHeadDim + 2 * lane) = z2;
        },
        [&](int i, uint32_t w) { codes[i] = w; });
}
template <int BITS, class Params>
__device__ __forceinline__ void flush_values(const Params& p, int64_t unit, int64_t at, int start, int lane) {
    ValueRow y[8];
    load_value_rows_before(p, unit, start, lane, y);
    uint32_t* codes = const_cast<uint32_t*>(p.v_codes) + at * (kTileTokens * kHeadDim * BITS / 32);
    quantize_value_tile<BITS>(y, lane,
        [&](int i, _Float16 s, _Float16 z) {
            reinterpret_cast<_Float16*>(const_cast<__half*>(p.v_scale))[at * 128 + i] = s;
            reinterpret_cast<_Float16*>(const_cast<__half*>(p.v_zero))[at * 128 + i] = z;
        },
        [&](int i, uint32_t w) { codes[i] = w; });
}

}  // namespace tile
}  // namespace kivi
