// Format conversion kernels: min-max round-to-nearest group quantization + bit packing
// (paper Sec. 3.1 for the three stored components; Sec. 6.1 / App. C for the quantizer),
// packing of externally chosen codes, and the inverse.  Integer results are bit-exact by
// construction: every float operation is a single correctly rounded IEEE fp32 operation.
// The __f*_rn functions of this toolchain are the plain operators, which the compiler would fuse
// (1 - i * step and p * hi - p * lo became fused multiply-adds and moved a scale across an fp16
// rounding tie in one group of three thousand), so this file is compiled with -ffp-contract=off
// (the build script passes it; a pragma here would not reach the header's inline functions).
#include <type_traits>

#include "qeft_internal.h"

namespace qeft {
namespace {

// ---- step 1: (scale, zero) of every (row, group); one wavefront per pair ------------------
__global__ __launch_bounds__(256) void rtn_params_kernel(Layer L, const __half* __restrict__ W, int64_t ldw,
                                                         __half* __restrict__ scales, __half* __restrict__ zeros) {
    const int64_t pair = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // over [OC][group_stride]
    const int lane = threadIdx.x & 63;
    if (pair >= (int64_t)L.oc * L.gs) return;
    const int o = (int)(pair / L.gs), gi = (int)(pair % L.gs);
    if (gi >= L.ng) {   // padding entry
        if (lane == 0) {
            scales[pair] = __float2half_rn(0.f);
            zeros[pair] = __float2half_rn(0.f);
        }
        return;
    }
    const int j0 = gi * L.g;
    const int len = min(L.g, L.kq - j0);
    float lo = 0.f, hi = 0.f;  // the range always contains 0
    for (int j = lane; j < len; j += 64) {
        const float v = __half2float(W[(size_t)o * ldw + j0 + j]);
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off, 64));
        hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    }
    if (lane == 0) {
        const float qmax = (float)((1 << L.bits) - 1);
        const float s32 = __fdiv_rn(hi - lo, qmax);
        __half s16, z16;
        if (s32 == 0.f) {
            s16 = __float2half_rn(1.f);
            z16 = __float2half_rn(0.f);
        } else {
            s16 = __float2half_rn(s32);
            if (__half2float(s16) == 0.f) s16 = __ushort_as_half((unsigned short)1);  // smallest subnormal
            const float s = __half2float(s16);
            float z = rintf(__fdiv_rn(0.f - lo, s));
            z = fminf(fmaxf(z, 0.f), qmax);
            z16 = __float2half_rn(z);
        }
        scales[pair] = s16;
        zeros[pair] = z16;
    }
}

// Word wd of a row from the codes of its columns (code(j) is asked for j < Kq only).  Whole codes per word:
// columns per * wd .. + per - 1 at bits b i.  Dense 3-bit: every code whose bits 3j .. 3j+2 meet bits
// 32 wd .. 32 wd + 31 of the row, shifted to its place (the two codes at the ends may lie partly outside).
template <class F>
__device__ __forceinline__ uint32_t build_word(const Layer& L, int wd, F code) {
    uint32_t word = 0;
    if (L.dense) {
        const int j0 = (32 * wd) / 3, j1 = (32 * wd + 31) / 3;
        for (int j = j0; j <= j1; ++j) {
            if (j >= L.kq) break;
            const int sh = 3 * j - 32 * wd;   // -2 .. 31
            const uint32_t c = code(j);
            word |= sh >= 0 ? c << sh : c >> -sh;
        }
        return word;
    }
    const int per = (L.bits == 4) ? 8 : 10;
    for (int i = 0; i < per; ++i) {
        const int j = wd * per + i;
        if (j < L.kq) word |= code(j) << (L.bits * i);
    }
    return word;
}

// ---- step 2: one thread per 32-bit word: quantize its 8 / 10 columns and pack ------------
__global__ __launch_bounds__(256) void rtn_words_kernel(Layer L, const __half* __restrict__ W, int64_t ldw,
                                                        const __half* __restrict__ scales,
                                                        const __half* __restrict__ zeros, uint32_t* __restrict__ qweight) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)L.oc * L.stride) return;
    const int o = (int)(idx / L.stride), wd = (int)(idx % L.stride);
    const float qmax = (float)((1 << L.bits) - 1);
    qweight[idx] = build_word(L, wd, [&](int j) {
        const size_t gi = (size_t)o * L.gs + j / L.g;
        const float s = __half2float(scales[gi]);
        const float z = __half2float(zeros[gi]);
        const float v = __half2float(W[(size_t)o * ldw + j]);
        const float q = rintf(__fdiv_rn(v, s)) + z;
        return (uint32_t)fminf(fmaxf(q, 0.f), qmax);
    });
}

// ---- both steps in one pass for 4-bit codes and groups of 128 -----------------------------------
// One wavefront per (row, 512 columns = 4 groups = 64 words): lane l reads the 16 bytes of columns
// 8 l .. 8 l + 7 - its word - and belongs to group l / 16.  Minimum and maximum go through the 16
// lanes of the group with four data-parallel-primitive moves; every lane then derives the group's
// (scale, zero-point) with the same correctly rounded fp32 operations as the two-step kernels
// (bit-identical results), quantizes its 8 columns and stores its word: W is read once, with
// 16-byte loads, and the codes leave as 256 contiguous bytes per wavefront.  Columns past Kq count
// as zeros (neutral: a group's range always contains 0) and give zero codes; the wave of a row's
// last chunk also zeroes the row's padding parameters.
__device__ __forceinline__ float dpp16_min(float v) {
    auto mv = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, false));
    };
    v = fminf(v, mv(v, std::integral_constant<int, 0xB1>{}));    // lane ^ 1
    v = fminf(v, mv(v, std::integral_constant<int, 0x4E>{}));    // lane ^ 2
    v = fminf(v, mv(v, std::integral_constant<int, 0x141>{}));   // mirrored halves of the row of 16
    v = fminf(v, mv(v, std::integral_constant<int, 0x140>{}));   // mirrored row
    return v;
}

__global__ __launch_bounds__(256) void rtn_fused_w4g128_kernel(Layer L, const __half* __restrict__ W, int64_t ldw,
                                                               uint32_t* __restrict__ qweight, __half* __restrict__ scales,
                                                               __half* __restrict__ zeros, int chunks) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    const int64_t wv = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (wv >= (int64_t)L.oc * chunks) return;
    const int o = (int)(wv / chunks), ch = (int)(wv % chunks);
    const int word = 64 * ch + lane, col = 8 * word;
    // Kq is a multiple of 8 here, so a word is entirely inside or entirely outside the row
    const bool live = col < L.kq;
    const u4 raw = live ? *reinterpret_cast<const u4*>(W + (size_t)o * ldw + col) : u4{0u, 0u, 0u, 0u};
    const h8 h = __builtin_bit_cast(h8, raw);
    float v[8], lo = 0.f, hi = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[e] = (float)h[e];
        lo = fminf(lo, v[e]);
        hi = fmaxf(hi, v[e]);
    }
    lo = dpp16_min(lo);
    hi = -dpp16_min(-hi);
    const float qmax = 15.f;
    const float s32 = __fdiv_rn(hi - lo, qmax);
    __half s16, z16;
    if (s32 == 0.f) {
        s16 = __float2half_rn(1.f);
        z16 = __float2half_rn(0.f);
    } else {
        s16 = __float2half_rn(s32);
        if (__half2float(s16) == 0.f) s16 = __ushort_as_half((unsigned short)1);  // smallest subnormal
        float z = rintf(__fdiv_rn(0.f - lo, __half2float(s16)));
        z = fminf(fmaxf(z, 0.f), qmax);
        z16 = __float2half_rn(z);
    }
    const float s = __half2float(s16), z = __half2float(z16);
    uint32_t out = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float q = rintf(__fdiv_rn(v[e], s)) + z;
        q = fminf(fmaxf(q, 0.f), qmax);
        out |= (uint32_t)q << (4 * e);
    }
    if (word < L.stride) qweight[(size_t)o * L.stride + word] = live ? out : 0u;
    const int gi = 4 * ch + (lane >> 4);
    if ((lane & 15) == 0 && gi < L.gs) {
        const bool real = gi < L.ng;
        scales[(size_t)o * L.gs + gi] = real ? s16 : __float2half_rn(0.f);
        zeros[(size_t)o * L.gs + gi] = real ? z16 : __float2half_rn(0.f);
    }
    // parameter padding past the groups this row's chunks cover
    if (ch == chunks - 1) {
        const int gi2 = 4 * chunks + lane;
        if (gi2 < L.gs) {
            scales[(size_t)o * L.gs + gi2] = __float2half_rn(0.f);
            zeros[(size_t)o * L.gs + gi2] = __float2half_rn(0.f);
        }
    }
}

// ---- group-wise grid search with truncation (paper Sec. 3.1) -------------------------------------
// For every (row, group): candidate i shrinks the min-max range (0 included) by p_i = 1 - i * step,
// derives (scale, zero-point) with the rules above, quantizes and scores the squared weight error;
// the first candidate with the smallest error is kept (candidate 0 = plain min-max).  One group per
// 16 lanes (a lane holds 8 consecutive columns; lanes past the group width hold zeros, which cost
// nothing), four groups per wavefront.  The error is summed in a fixed order - a lane's 8 columns
// left to right, one rounding each, then a balanced tree over the 16 lanes - so that the decisions
// can be reproduced exactly elsewhere.
//
// The kernel is bound by vector instructions (4096 x 4096, 80 candidates: 1.3 G scores).  What keeps them few:
//  * Scale, zero-point and reciprocal of 16 candidates are derived at once, one per lane of the group's 16, and handed
//    round by row broadcasts.
//  * A column's score needs no division.  r = rint(v * (1 / s)) differs from rint(v / s) only where v / s is exactly half
//    way between two integers: v and s are fp16, so any other quotient of magnitude 1/4 ... 256 is at least 2^-13 from a tie
//    (|2 a 2^k - (2 n + 1) b| / 2 b with a, b < 2^11), while the product is off by 2^-15 at most, and larger ones clamp.
//    On a tie both neighbours leave the same |v - s r| = s / 2, so the score is the same number either way; the codes
//    themselves are taken at the end by the rules above, with the division.
//  * v - s r in one fused operation is exact where the product and the difference are rounded separately, because s r is
//    exact (11 bits times an integer below 16).
//  * A candidate whose two least and two greatest columns alone already err by more than the best score so far cannot win and is
//    not scored (the sum of non-negative terms is at least any of them; 2^-10 covers its rounding).  Narrow ranges clip the extremes
//    hard: of an 80-candidate grid 27 are scored on normally distributed weights at 4 bits, 49 at 3 (31 and 60 by the two extremes
//    alone), and the rounds of 16 whose widest candidate is beyond hope are not entered.
//  * Candidates are scored in twos, whose sums over the 16 lanes share their moves; even lanes keep the best of the first ones,
//    odd lanes of the second ones.
//  * The weak block is copied by waves of the same launch.
//  * Where a quotient itself is needed its divisor is short, and three instructions give the bits of a division's ten (short_div); the
//    row and chunk of a wave are scalar; the row broadcasts start from nothing that has to be cleared; a candidate past the grid's end scores as no number.
// 4096 x 4096, 80 candidates, whole call (us): 919 with two divisions per weight and candidate and every candidate scored, 123 with the
// bound by two columns, single candidates and the copy in a launch of its own (117 in the harness of the figures that follow), 110 with general
// divisions, 91 now; 3 bits, ten codes a word 211 -> 188 -> 165, dense (the words in this pass too) 215 -> 174 -> 147.
// Of a pair's hundred vector instructions eighty are the five per value and candidate; a packed or 16-bit form would not give the same sums.
// sum over the 16 lanes of a row whose neighbours (lane ^ 1) are added already, separately for even and odd lanes.  Each step is an
// exchange between two halves, so that both add the same two numbers and all lanes of a class end with the same bits: they decide
// by them one by one, and a rotation by four would leave every other quad with another order (two candidates in one group's codes).
__device__ __forceinline__ float dpp16_sum_rest(float v) {
    auto mv = [](float x, auto ctrl) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true)); };
    v = __fadd_rn(v, mv(v, std::integral_constant<int, 0x4E>{}));    // lane ^ 2
    const int b = __builtin_bit_cast(int, v), on = __builtin_amdgcn_mov_dpp(b, 0x104, 0xf, 0x5, true);   // lane ^ 4: quads 0 and 2 read four lanes on,
    v = __fadd_rn(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(on, b, 0x114, 0xf, 0xA, false)));   // quads 1 and 3 four lanes back
    return __fadd_rn(v, mv(v, std::integral_constant<int, 0x128>{}));   // lane ^ 8
}

// Reciprocal and quotient rounded correctly, where the divisor b is a normal number of at most 11 bits (Newton's step, and Markstein's correction of
// a quotient by its remainder; a general division takes about ten instructions).  1 / b: the instruction's error of 1 ulp leaves 2^-46 after the step, and no 1 / b
// of such a b lies within 2^-36 of half way between two floats.  a / b: a * rb errs by 1.5 ulp at most, so the remainder is exact, and the
// corrected quotient is off by 2^-23 ulp before its rounding, a / b never within 2^-12 ulp of half way.  No infinities.
__device__ __forceinline__ float short_rcp(float b) {
    const float r = __builtin_amdgcn_rcpf(b);
    return __builtin_fmaf(__builtin_fmaf(-b, r, 1.f), r, r);
}
__device__ __forceinline__ float short_div(float a, float b, float rb, float q) { return __builtin_fmaf(__builtin_fmaf(-q, b, a), rb, q); }   // q = a * rb

// WORDS: 4: 4-bit codes in groups of 128, 3: dense 3-bit codes in groups of 128, whose words the same lanes then store (0:
// rtn_words_kernel does).
template <int WORDS>
__global__ __launch_bounds__(256) void search_params_kernel(Layer L, const __half* __restrict__ W, int64_t ldw,
                                                            __half* __restrict__ scales, __half* __restrict__ zeros,
                                                            uint32_t* __restrict__ qweight, __half* __restrict__ weak, int chunks,
                                                            int copy_waves, int n_grid, float step) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    const int64_t wv = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - copy_waves;
    const int lane = threadIdx.x & 63;
    if (wv < 0) {   // the launch's first waves copy the weak block, 8 columns per lane (a launch of its own took 5 us)
        const int64_t idx = 64 * (wv + copy_waves) + lane;
        const int per = L.k >> 3;
        if (idx < (int64_t)L.oc * per) {
            const int64_t r = idx / per;
            const int c = 8 * (int)(idx - r * per);
            *reinterpret_cast<u4*>(weak + r * L.k + c) = *reinterpret_cast<const u4*>(W + r * ldw + L.kq + c);
        }
        return;
    }
    if (wv >= (int64_t)L.oc * chunks) return;
    const int o = (int)((uint32_t)wv / (uint32_t)chunks), ch = (int)((uint32_t)wv - (uint32_t)o * (uint32_t)chunks);   // (2^31 waves would take 2 TB of W)
    const int grp = 4 * ch + (lane >> 4), t = lane & 15;   // grp < gs: chunks = gs / 4
    const int col = grp * L.g + 8 * t;
    const bool live = grp < L.ng && 8 * t < L.g && col < L.kq;   // Kq % 8 == 0: whole octets
    const u4 raw = live ? *reinterpret_cast<const u4*>(W + (size_t)o * ldw + col) : u4{0u, 0u, 0u, 0u};
    const h8 h = __builtin_bit_cast(h8, raw);
    float v[8], lo0 = 0.f, hi0 = 0.f, lo1 = 0.f, hi1 = 0.f;   // the group's two least and two greatest values, 0 among them
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[e] = (float)h[e];
        lo1 = __builtin_amdgcn_fmed3f(lo0, lo1, v[e]);
        lo0 = fminf(lo0, v[e]);
        hi1 = __builtin_amdgcn_fmed3f(hi0, hi1, v[e]);
        hi0 = fmaxf(hi0, v[e]);
    }
    auto two_least = [](float& a, float& b) {   // of the 16 lanes of a row, in every lane
        auto merge = [&](auto ctrl) {
            auto mv = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true)); };
            const float c = mv(a), d = mv(b);
            b = fminf(fmaxf(a, c), fminf(b, d));
            a = fminf(a, c);
        };
        merge(std::integral_constant<int, 0xB1>{});
        merge(std::integral_constant<int, 0x4E>{});
        merge(std::integral_constant<int, 0x141>{});
        merge(std::integral_constant<int, 0x140>{});
    };
    two_least(lo0, lo1);
    hi0 = -hi0, hi1 = -hi1;
    two_least(hi0, hi1);
    hi0 = -hi0, hi1 = -hi1;
    const float qmax = (float)((1 << L.bits) - 1), rqmax = short_rcp(qmax);
    // scale, its reciprocal and zero-point of candidate i of this lane's group
    struct Params {
        float s, rs, z;
    };
    auto params = [&](int i) {
        const float p = __fsub_rn(1.f, __fmul_rn((float)i, step));
        const float lo = __fmul_rn(p, lo0), hi = __fmul_rn(p, hi0);
        const float range = __fsub_rn(hi, lo), s32 = short_div(range, qmax, rqmax, range * rqmax);
        Params r{1.f, 1.f, 0.f};
        if (s32 != 0.f) {
            __half s16 = __float2half_rn(s32);
            if (__half2float(s16) == 0.f) s16 = __ushort_as_half((unsigned short)1);
            r.s = __half2float(s16);
            r.rs = short_rcp(r.s);
            const float below = __fsub_rn(0.f, lo);
            r.z = rintf(short_div(below, r.s, r.rs, below * r.rs));
            r.z = fminf(fmaxf(r.z, 0.f), qmax);
        }
        return r;
    };
    // error of one value under (s, 1 / s, z): nz = -z, uz = qmax - z
    auto miss = [](float x, float s, float rs, float nz, float uz) {
        return __builtin_fmaf(-__builtin_amdgcn_fmed3f(rintf(x * rs), nz, uz), s, x);
    };
    auto xor1 = [](float x) { return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, true)); };
    const bool odd = (t & 1) != 0;
    // the best of the even candidates in the even lanes, of the odd ones in the odd lanes
    float best_e = __builtin_inff();
    int best_i = -1;
    // the better of the neighbours' two classes: scores are no less than 0, and as whole numbers need no instruction to quiet a NaN
    auto least_of_both = [&]() {
        const uint32_t mine = __builtin_bit_cast(uint32_t, best_e), its = __builtin_bit_cast(uint32_t, xor1(best_e));
        return __builtin_bit_cast(float, mine < its ? mine : its);
    };
    float to_beat = best_e;
    for (int i0 = 0; i0 < n_grid; i0 += 16) {
        if (i0 > 0) {
            // A candidate's codes end within s / 2 of p hi0 and p lo0, and s rounded up moves the upper end by qmax times as much: by 2^-11 of s
            // (0.52 s covers that and the roundings of z and p), among subnormal scales by up to 2^-24.  So a value x beyond misses by
            // x - p hi0 - half at least, and by more under every narrower candidate: done once that is too much for all groups
            const float p = 1.f - (float)i0 * step, half = 0.52f * (p * (hi0 - lo0) * rqmax) + (qmax + 1.f) * 0x1p-24f;
            auto beyond = [&](float x) {
                const float e = fmaxf(fmaxf(x - p * hi0, p * lo0 - x) - half, 0.f);
                return e * e;
            };
            const float least = (beyond(lo0) + beyond(hi0)) + (beyond(lo1) + beyond(hi1));
            // (equal is too much as well, the earlier candidate stays: groups of zeros, the padding of a row among them)
            if (__ballot(!(least * (1.f - 0x1p-7f) >= to_beat)) == 0) break;
        }
        const Params mine = params(i0 + t);   // candidate i0 + t
        // (past the grid's end: no number, whose score is never the better one)
        const float s_l = i0 + t < n_grid ? mine.s : __builtin_nanf(""), z_l = mine.z, rs_l = mine.rs;
        auto missed = [&](float x) {
            const float e = miss(x, s_l, rs_l, -z_l, qmax - z_l);
            return e * e;
        };
        const float bound_l = ((missed(lo0) + missed(hi0)) + (missed(lo1) + missed(hi1))) * (1.f - 0x1p-10f);
        auto pair = [&](auto j_c) {
            constexpr int J = decltype(j_c)::value;
            // any of the four groups' candidates J, J + 1 that could still win
            if ((__ballot(bound_l < to_beat) & (0x0003000300030003ull << J)) == 0) return;
            float acc[2];
            auto score = [&](auto k_c) {
                constexpr int K = decltype(k_c)::value;
                auto from = [](float x) {   // lane J + K of the row of 16
                    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x150 + J + K, 0xf, 0xf, false));
                };
                const float s = from(s_l), rs = from(rs_l), z = from(z_l), uz = qmax - z;
                float a = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = miss(v[e], s, rs, -z, uz);
                    a = e == 0 ? __fmul_rn(d, d) : __builtin_fmaf(d, d, a);
                }
                acc[K] = a;
            };
            score(std::integral_constant<int, 0>{});
            score(std::integral_constant<int, 1>{});
            // both sums over the 16 lanes at once: the first ends in the even lanes, the second in the odd ones
            const float err = dpp16_sum_rest(__fadd_rn(odd ? acc[1] : acc[0], xor1(odd ? acc[0] : acc[1])));
            const bool better = err < best_e;
            best_e = better ? err : best_e;
            best_i = better ? i0 + J + (t & 1) : best_i;
            to_beat = least_of_both();
        };
        pair(std::integral_constant<int, 0>{});
        pair(std::integral_constant<int, 2>{});
        pair(std::integral_constant<int, 4>{});
        pair(std::integral_constant<int, 6>{});
        pair(std::integral_constant<int, 8>{});
        pair(std::integral_constant<int, 10>{});
        pair(std::integral_constant<int, 12>{});
        pair(std::integral_constant<int, 14>{});
    }
    // the better of the two classes, the first candidate where they are equal; none (a score that is no number): scale 1
    const float other_e = xor1(best_e);
    const int other_i = __builtin_amdgcn_update_dpp(0, best_i, 0xB1, 0xf, 0xf, false);
    if (other_e < best_e || (other_e == best_e && (uint32_t)other_i < (uint32_t)best_i)) best_i = other_i;
    Params best = params(best_i);
    if (best_i < 0) best = Params{1.f, 1.f, 0.f};
    if (t == 0) {
        const bool real = grp < L.ng;
        scales[(size_t)o * L.gs + grp] = __float2half_rn(real ? best.s : 0.f);
        zeros[(size_t)o * L.gs + grp] = __float2half_rn(real ? best.z : 0.f);
    }
    if constexpr (WORDS != 0) {
        uint32_t out = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            // (beyond 1024 of scale an infinity may be, and any code clamps: the correction leads from there past it)
            const float q0 = __builtin_amdgcn_fmed3f(v[e] * best.rs, -1024.f, 1024.f);
            const float q = __fadd_rn(rintf(short_div(v[e], best.s, best.rs, q0)), best.z);
            out |= (uint32_t)__builtin_amdgcn_fmed3f(q, 0.f, qmax) << (WORDS * e);   // (no number: 0)
        }
        if (!live) out = 0u;
        if constexpr (WORDS == 4) {
            const int word = 16 * grp + t;   // (gs groups of 16 words reach past the row's padded end)
            if (word < L.stride) qweight[(size_t)o * L.stride + word] = out;
        } else {   // four lanes' 24 bits are three words, of which lane q < 3 has the head in its own bits and the rest in the next lane's
            const int q = t & 3, word = 12 * grp + 3 * (t >> 2) + q;
            const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)out, 0xF9, 0xf, 0xf, false);   // quad_perm [1,2,3,3]
            if (q < 3 && word < L.stride) qweight[(size_t)o * L.stride + word] = (out >> (8 * q)) | (next << (24 - 8 * q));
        }
    }
}

__global__ __launch_bounds__(256) void pack_words_kernel(Layer L, const uint8_t* __restrict__ codes,
                                                         uint32_t* __restrict__ qweight) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)L.oc * L.stride) return;
    const int o = (int)(idx / L.stride), wd = (int)(idx % L.stride);
    const uint32_t mask = (1u << L.bits) - 1u;
    qweight[idx] = build_word(L, wd, [&](int j) { return (uint32_t)codes[(size_t)o * L.kq + j] & mask; });
}

__global__ __launch_bounds__(256) void unpack_codes_kernel(Layer L, uint8_t* __restrict__ codes) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)L.oc * L.kq) return;
    const int o = (int)(idx / L.kq), j = (int)(idx % L.kq);
    codes[idx] = (uint8_t)code_at(L, L.qweight + (size_t)o * L.stride, j);
}

// One thread per 8 columns of a row of the mixed weight: 16 bytes out.
__global__ __launch_bounds__(256) void dequantize_kernel(Layer L, __half* __restrict__ out) {
    const int chunks = L.ic >> 3;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)L.oc * chunks) return;
    const int o = (int)(idx / chunks), j0 = 8 * (int)(idx % chunks);
    const uint32_t* row = L.qweight + (size_t)o * L.stride;
    __half v[8];
    if (j0 + 8 <= L.kq && (L.g & 7) == 0) {   // the usual case: eight quantized columns of one group
        const size_t gi = (size_t)o * L.gs + j0 / L.g;
        const float sc = __half2float(L.scales[gi]), zp = __half2float(L.zeros[gi]);
        if (L.dense) {                        // 24 bits starting at bit 3 j0 = 24 (j0 / 8) of the row
            const int bit = 3 * j0, w0 = bit >> 5, sh = bit & 31;
            uint32_t c = row[w0] >> sh;
            if (sh > 8) c |= row[w0 + 1] << (32 - sh);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __float2half_rn(sc * ((float)((c >> (3 * e)) & 7u) - zp));
        } else if (L.bits == 4) {
            const uint32_t c = row[j0 >> 3];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __float2half_rn(sc * ((float)((c >> (4 * e)) & 15u) - zp));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __float2half_rn(sc * ((float)code_at(L, row, j0 + e) - zp));
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int j = j0 + e;
            if (j < L.kq) {
                const size_t gi = (size_t)o * L.gs + j / L.g;
                v[e] = __float2half_rn(__half2float(L.scales[gi]) * ((float)code_at(L, row, j) - __half2float(L.zeros[gi])));
            } else {
                v[e] = L.weak[(size_t)o * L.k + (j - L.kq)];
            }
        }
    }
    *reinterpret_cast<uint4*>(out + (size_t)o * L.ic + j0) = *reinterpret_cast<const uint4*>(v);
}

// The codes of a 3-bit layer, either layout, as the 4-bit layout's words (8 codes each): a wave per row, four words per lane
// and turn.  Eight codes are 24 bits; three rounds of "upper half up" open a gap above every code.  Memory-bound: 5120 x 5120
// reads 9.7 MB and writes 12.8 in 6.6 us from the dense layout, 8.3 from ten codes per word (two words per thread over a grid
// of rows: 11; the fp16 copy: 17).
template <bool DENSE>
__global__ __launch_bounds__(256) void expand3_kernel(Layer L, uint32_t* __restrict__ out, int words4, int stride4) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const int64_t o = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (o >= L.oc) return;
    const uint32_t* row = L.qweight + (size_t)o * L.stride;
    for (int q = threadIdx.x & 63; 4 * q < stride4; q += 64) {
        uint32_t c[4];
        if constexpr (DENSE) {   // 32 codes are 96 bits: words 3 q .. 3 q + 2
            const uint32_t a = row[min(3 * q, L.stride - 1)], b = row[min(3 * q + 1, L.stride - 1)], d = row[min(3 * q + 2, L.stride - 1)];
            c[0] = a;
            c[1] = __builtin_amdgcn_alignbit(b, a, 24);
            c[2] = __builtin_amdgcn_alignbit(d, b, 16);
            c[3] = d >> 8;
        } else {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const int j0 = 8 * (4 * q + h), at = j0 / 10;
                const uint64_t lo = row[min(at, L.stride - 1)], hi = row[min(at + 1, L.stride - 1)];
                c[h] = (uint32_t)((lo | hi << 30) >> (3 * (j0 - 10 * at)));
            }
        }
        u4 v;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            uint32_t x = c[h];
            x = (x & 0xfffu) | (x & 0xfff000u) << 4;
            x = (x & 0x003f003fu) | (x & 0x0fc00fc0u) << 2;
            x = (x & 0x07070707u) | (x & 0x38383838u) << 1;
            v[h] = 4 * q + h < words4 ? x : 0u;   // (Kq is a multiple of 8: whole words)
        }
        *reinterpret_cast<u4*>(out + (size_t)o * stride4 + 4 * q) = v;
    }
}

// compact [OC][G] parameters into the padded [OC][group_stride] arrays (padding zero)
__global__ __launch_bounds__(256) void pad_groups_kernel(Layer L, const __half* __restrict__ s_in,
                                                         const __half* __restrict__ z_in, __half* __restrict__ s_out,
                                                         __half* __restrict__ z_out) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)L.oc * L.gs) return;
    const int o = (int)(idx / L.gs), gi = (int)(idx % L.gs);
    const bool real = gi < L.ng;
    s_out[idx] = real ? s_in[(size_t)o * L.ng + gi] : __float2half_rn(0.f);
    z_out[idx] = real ? z_in[(size_t)o * L.ng + gi] : __float2half_rn(0.f);
}

// rows x cols fp16 copy between two leading dimensions
__global__ __launch_bounds__(256) void copy2d_kernel(const __half* __restrict__ src, int64_t lds, __half* __restrict__ dst,
                                                     int64_t ldd, int64_t rows, int cols) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= rows * cols) return;
    const int64_t r = idx / cols;
    const int c = (int)(idx % cols);
    dst[r * ldd + c] = src[r * lds + c];
}

void copy2d(const __half* src, int64_t lds, __half* dst, int64_t ldd, int64_t rows, int cols, hipStream_t s) {
    if (rows * cols == 0 || src == dst) return;
    copy2d_kernel<<<ceil_div(rows * cols, 256), 256, 0, s>>>(src, lds, dst, ldd, rows, cols);
}

}  // namespace

hipError_t pack_rtn(const Layer& L, const __half* W, int64_t ldw, uint32_t* qweight, __half* scales, __half* zeros,
                    __half* weak, hipStream_t s) {
    if (L.kq > 0 && L.bits == 4 && L.g == 128 && (L.kq & 7) == 0 && (ldw & 7) == 0 && ((uintptr_t)W & 15) == 0) {
        const int chunks = ceil_div(L.stride, 64);
        rtn_fused_w4g128_kernel<<<ceil_div((int64_t)L.oc * chunks, 4), 256, 0, s>>>(L, W, ldw, qweight, scales, zeros, chunks);
    } else if (L.kq > 0) {
        const int64_t pairs = (int64_t)L.oc * L.gs;
        rtn_params_kernel<<<ceil_div(pairs, 4), 256, 0, s>>>(L, W, ldw, scales, zeros);
        rtn_words_kernel<<<ceil_div((int64_t)L.oc * L.stride, 256), 256, 0, s>>>(L, W, ldw, scales, zeros, qweight);
    }
    copy2d(W + L.kq, ldw, weak, L.k, L.oc, L.k, s);
    return hipGetLastError();
}

bool pack_search_supported(const Layer& L, int64_t ldw, const void* W) {
    return (L.g & 7) == 0 && L.g <= 128 && (L.kq & 7) == 0 && (ldw & 7) == 0 && ((uintptr_t)W & 15) == 0;
}

hipError_t pack_search(const Layer& L, const __half* W, int64_t ldw, int n_grid, float step, uint32_t* qweight,
                       __half* scales, __half* zeros, __half* weak, hipStream_t s) {
    if (L.kq > 0) {
        const int chunks = L.gs / 4;
        const bool copies = L.k > 0 && (L.k & 7) == 0;   // (the columns then lie 16-byte aligned on both sides)
        const int copy_waves = copies ? ceil_div((int64_t)L.oc * (L.k >> 3), 64) : 0;
        const int grid = ceil_div((int64_t)L.oc * chunks + copy_waves, 4);
        if (L.bits == 4 && L.g == 128) {
            search_params_kernel<4><<<grid, 256, 0, s>>>(L, W, ldw, scales, zeros, qweight, weak, chunks, copy_waves, n_grid, step);
        } else if (L.dense && L.g == 128) {
            search_params_kernel<3><<<grid, 256, 0, s>>>(L, W, ldw, scales, zeros, qweight, weak, chunks, copy_waves, n_grid, step);
        } else {
            search_params_kernel<0><<<grid, 256, 0, s>>>(L, W, ldw, scales, zeros, qweight, weak, chunks, copy_waves, n_grid, step);
            rtn_words_kernel<<<ceil_div((int64_t)L.oc * L.stride, 256), 256, 0, s>>>(L, W, ldw, scales, zeros, qweight);
        }
        if (copies) return hipGetLastError();
    }
    copy2d(W + L.kq, ldw, weak, L.k, L.oc, L.k, s);
    return hipGetLastError();
}

hipError_t pack_codes(const Layer& L, const uint8_t* codes, const __half* scales_in, const __half* zeros_in,
                      const __half* weak_in, uint32_t* qweight, __half* scales, __half* zeros, __half* weak, hipStream_t s) {
    if (L.kq > 0) {
        pack_words_kernel<<<ceil_div((int64_t)L.oc * L.stride, 256), 256, 0, s>>>(L, codes, qweight);
        pad_groups_kernel<<<ceil_div((int64_t)L.oc * L.gs, 256), 256, 0, s>>>(L, scales_in, zeros_in, scales, zeros);
    }
    copy2d(weak_in, L.k, weak, L.k, L.oc, L.k, s);
    return hipGetLastError();
}

hipError_t dequantize_fp16(const Layer& L, __half* out, hipStream_t s) {
    const int64_t n = (int64_t)L.oc * (L.ic >> 3);
    dequantize_kernel<<<ceil_div(n, 256), 256, 0, s>>>(L, out);
    return hipGetLastError();
}

hipError_t expand3(const Layer& L, uint32_t* out, int words4, int stride4, hipStream_t s) {
    if (L.dense) expand3_kernel<true><<<ceil_div(L.oc, 4), 256, 0, s>>>(L, out, words4, stride4);
    else expand3_kernel<false><<<ceil_div(L.oc, 4), 256, 0, s>>>(L, out, words4, stride4);
    return hipGetLastError();
}

hipError_t unpack(const Layer& L, uint8_t* codes, __half* scales, __half* zeros, __half* weak, hipStream_t s) {
    if (L.kq > 0) {
        if (codes) unpack_codes_kernel<<<ceil_div((int64_t)L.oc * L.kq, 256), 256, 0, s>>>(L, codes);
        if (scales) copy2d(L.scales, L.gs, scales, L.ng, L.oc, L.ng, s);
        if (zeros) copy2d(L.zeros, L.gs, zeros, L.ng, L.oc, L.ng, s);
    }
    if (weak) copy2d(L.weak, L.k, weak, L.k, L.oc, L.k, s);
    return hipGetLastError();
}

}  // namespace qeft
