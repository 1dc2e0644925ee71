// The weak block's gradient in strips of output channels, and how its tokens are split: the workgroup body that gemm.hip launches on its
// own and that both input-gradient files append to launches of theirs.
#pragma once

#include "gemm_common.h"
#include "qeft_internal.h"

namespace qeft {
namespace gemm {

// ======================================================================================= weak gradient
// A[i = c][k = m] = Xw[m][c], B[j = oc][k = m] = dY[m][oc]: both operands are read transposed.
// The tokens are split over `splits` workgroups per strip of output channels; each writes an fp32 partial
// [OC][k] slab, summed in slab order by a second kernel (no atomics: deterministic).
// The kernel is sized for what bounds it - reading dY once from
// HBM: a workgroup owns 64 output channels x up to 128 or 64 weak columns over a range of tokens, so the
// MFMA tiles hold no padding and a dY row contributes 128 contiguous bytes.  Both operands have
// the contraction index (the token) as their row index; instead of transposing 8 x 8 blocks in
// registers, the tiles go to LDS as they are ([token][column], rows padded by 64 bytes) and the
// fragments are read with the transposing LDS load of gfx950 (ds_read_b64_tr_b16: the 16 lanes
// of a group each name 4 consecutive halfs; output lane l receives element l % 4 of source
// lanes l / 4, l / 4 + 4, l / 4 + 8, l / 4 + 12).  With source lane s pointing at row k0 + s / 4,
// columns c0 + 4 (s % 4) .., a group receives columns c0 .. c0 + 15 of rows k0 .. k0 + 3 - four
// consecutive contraction steps for 16 MFMA rows; two such loads make one fragment.
// Wave w multiplies weak columns 32 w .. 32 w + 31 against the 64 channels; in pieces of 64 columns 32 (w % 2) .. against 32 channels.  With one split
// the result goes straight to dW, otherwise into fp32 slabs as above.
constexpr int WG_OC = 64;                             // output channels per workgroup
// Row pitches: a transposing fragment read takes, per half wave, 4 rows x 64 bytes (two 16-lane groups side by
// side), so consecutive rows must sit 16 (or 48) banks apart: 256 + 64 and 128 + 64 bytes.  (With + 32 bytes a
// third of the LDS cycles of this kernel were bank conflicts.)
constexpr int wg_a_pitch(int kw) { return kw * 2 + 64; }   // bytes per token row of the Xw tile
constexpr int WG_B_PITCH = WG_OC * 2 + 64;            // ... of the dY tile
constexpr int wg_lds(int kw) { return 2 * BK * (wg_a_pitch(kw) + WG_B_PITCH); }   // A0 A1 B0 B1
constexpr int WG_LDS = wg_lds(128);

// A weak block wider than KW = 128 or 64 columns is taken in pieces of KW (workgroup index = ((strip, piece), split)): the pieces
// of a strip read the same dY rows and sit next to each other in the grid.
// (bid: the workgroup's index among the strip workgroups; lds: its dynamic shared memory, wg_lds(KW) bytes)
template <int KW>
__device__ __forceinline__ void weak_grad_strip_body(unsigned char* lds, int bid, int oc_total, int k_total, const __half* __restrict__ dY, int M,
                                                     int64_t lddy, const __half* __restrict__ Xw, int64_t ldxw,
                                                     float* __restrict__ part, int splits, int chunk, void* dW,
                                                     int out_f32, int accumulate) {
    typedef short s4 __attribute__((ext_vector_type(4)));
    typedef short s8 __attribute__((ext_vector_type(8)));
    using lds_s4 = __attribute__((address_space(3))) s4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int WG_A_PITCH = wg_a_pitch(KW), WG_A_BYTES = BK * WG_A_PITCH, WG_B_BYTES = BK * WG_B_PITCH;
    constexpr int CH = KW / 8, AU = CH / 4, AR = 256 / CH;   // Xw: chunks of a token, requests of a thread, tokens apart
    constexpr int T = KW / 64;                               // 32 x 32 tiles of a wave: all of the strip's channels, or half
    const int halves = (k_total + KW - 1) / KW;
    const int split = bid % splits, rest = bid / splits;
    const int kh = rest % halves, t_oc = rest / halves;
    const int k = min(KW, k_total - KW * kh);   // this workgroup's weak columns: KW kh .. KW kh + k - 1
    Xw += KW * kh;
    const int oc0 = t_oc * WG_OC;
    const int mb = split * chunk, me = min(mb + chunk, M);
    const int nst = (me - mb + BK - 1) / BK;
    const int fr = lane & 31, fk = lane >> 5;

    // producers: 16-byte chunks, copied as they are.  Xw tile: 64 tokens x CH chunks, AU per
    // thread (token ar + AR u, chunk ac); dY tile: 64 tokens x 8 chunks, two per thread (token
    // br + 32 u, chunk bc).  Chunks past k or past the last channel read column 0 and are zeroed.
    const int ar = tid / CH, ac = tid % CH, br = tid >> 3, bc = tid & 7;
    const bool a_ok = 8 * ac < k, b_ok = oc0 + 8 * bc < oc_total;
    const u4 zero4 = u4{0u, 0u, 0u, 0u};
    // Addresses: a scalar base per stage plus a per-thread byte offset computed once (this kernel is bound by
    // its single wave's instruction stream, and per-load address arithmetic was a third of it).  A stage whose
    // 64 tokens would pass the end of the matrices is fetched 64 tokens back from the end instead (M >= 64) and
    // put() keeps only the rows that belong to it; stages past the range re-read the last one and store zeros.
    using gptr = const __attribute__((address_space(1))) char*;
    using g_u4 = const __attribute__((address_space(1))) u4;
    uint32_t aoff[AU], boff[2];
#pragma unroll
    for (int u = 0; u < AU; ++u) aoff[u] = (uint32_t)(((int64_t)(ar + AR * u) * ldxw + (a_ok ? 8 * ac : 0)) * 2);
#pragma unroll
    for (int u = 0; u < 2; ++u) boff[u] = (uint32_t)(((int64_t)(br + 32 * u) * lddy + (b_ok ? oc0 + 8 * bc : 0)) * 2);
    const bool cols_full = __builtin_amdgcn_readfirstlane((int)(k >= KW && oc0 + WG_OC <= oc_total)) != 0;   // no thread's chunk is zeroed
    auto first_token = [&](int st) { return min(mb + BK * min(st, nst - 1), M - BK); };   // of the 64 tokens fetched for stage st
    // three stages of fetches in flight per thread (registers), a fourth in LDS being multiplied
    u4 va[3][AU], vb[3][2];
    auto fetch = [&](auto set_c, int st) {
        constexpr int SET = decltype(set_c)::value;
        const int t0 = first_token(st);
        const char* ab = reinterpret_cast<const char*>(Xw) + (int64_t)t0 * ldxw * 2;
        const char* bb = reinterpret_cast<const char*>(dY) + (int64_t)t0 * lddy * 2;
        asm volatile("" : "+s"(ab), "+s"(bb));
#pragma unroll
        for (int u = 0; u < AU; ++u) va[SET][u] = *reinterpret_cast<g_u4*>((gptr)ab + aoff[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u) vb[SET][u] = *reinterpret_cast<g_u4*>((gptr)bb + boff[u]);
    };
    auto put = [&](auto set_c, int st, int buf) {   // stage st, held by register set SET, into LDS buffer buf
        constexpr int SET = decltype(set_c)::value;
        const int m0 = mb + BK * st, t0 = first_token(st);
        unsigned char* sA = lds + buf * WG_A_BYTES;
        unsigned char* sB = lds + 2 * WG_A_BYTES + buf * WG_B_BYTES;
        if (cols_full && st < nst && m0 + BK <= me) {   // a whole stage, whole columns (wave-uniform): the registers as they are
#pragma unroll
            for (int u = 0; u < AU; ++u) *reinterpret_cast<u4*>(sA + (ar + AR * u) * WG_A_PITCH + 16 * ac) = va[SET][u];
#pragma unroll
            for (int u = 0; u < 2; ++u) *reinterpret_cast<u4*>(sB + (br + 32 * u) * WG_B_PITCH + 16 * bc) = vb[SET][u];
        } else if (st >= nst) {   // past the range: a tile of zeros
#pragma unroll
            for (int u = 0; u < AU; ++u) *reinterpret_cast<u4*>(sA + (ar + AR * u) * WG_A_PITCH + 16 * ac) = zero4;
#pragma unroll
            for (int u = 0; u < 2; ++u) *reinterpret_cast<u4*>(sB + (br + 32 * u) * WG_B_PITCH + 16 * bc) = zero4;
        } else {
            // fetched row r holds token t0 + r; it belongs to the stage when that lies in [m0, me), and its tile row
            // is token - m0.  shift = m0 - t0 > 0 only for the last stage of the matrices: fetched rows [shift, 64)
            // fill tile rows [0, 64 - shift), the rest of the tile is zero.
            const int shift = m0 - t0;
#pragma unroll
            for (int u = 0; u < AU; ++u) {
                const int r = ar + AR * u, tok = t0 + r;
                if (r >= shift) *reinterpret_cast<u4*>(sA + (r - shift) * WG_A_PITCH + 16 * ac) = (a_ok && tok < me) ? va[SET][u] : zero4;
                if (r >= BK - shift) *reinterpret_cast<u4*>(sA + r * WG_A_PITCH + 16 * ac) = zero4;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int r = br + 32 * u, tok = t0 + r;
                if (r >= shift) *reinterpret_cast<u4*>(sB + (r - shift) * WG_B_PITCH + 16 * bc) = (b_ok && tok < me) ? vb[SET][u] : zero4;
                if (r >= BK - shift) *reinterpret_cast<u4*>(sB + r * WG_B_PITCH + 16 * bc) = zero4;
            }
        }
    };

    f16v acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;

    // fragment addressing: lane = 16 g + s; rows (tokens) 8 (g / 2) + s / 4 (+ 4 for the second
    // load, + 16 per k-block), columns 16 (g % 2) + 4 (s % 4) of the wave's 32
    const int g = lane >> 4, s = lane & 15;
    const int wa = T == 2 ? wave : wave & 1, wb = T == 2 ? 0 : wave >> 1;   // the wave's weak columns 32 wa .., channels 32 wb ..
    const int frow = 8 * (g >> 1) + (s >> 2), fcol = 16 * (g & 1) + 4 * (s & 3);
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
    const uint32_t fa = lds0 + frow * WG_A_PITCH + 2 * (32 * wa + fcol);
    const uint32_t fb = lds0 + 2 * WG_A_BYTES + frow * WG_B_PITCH + 2 * (32 * wb + fcol);
    auto frag = [&](uint32_t addr, int pitch) {   // 8 contraction steps: rows +0..3 and +4..7
        const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(size_t)(addr));
        const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(size_t)(addr + 4 * pitch));
        return __builtin_bit_cast(h8, s8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w});
    };

    // stage st (already in LDS buffer st & 1, fetched through register set SET): refill the set
    // with stage st + 3, multiply, move stage st + 1 from the next set into the other buffer
    auto stage = [&](auto set_c, int st) {
        constexpr int SET = decltype(set_c)::value;
        const int cur = st & 1;
        fetch(set_c, st + 3);
        __builtin_amdgcn_sched_barrier(0);   // issue the fetches first: they are what the stage waits for
        const uint32_t a0 = fa + cur * WG_A_BYTES, b0 = fb + cur * WG_B_BYTES;
        // fragments are read one k-block ahead of the MFMAs that use them (one wave per SIMD: nothing else hides the LDS latency)
        h8 a[2], b[T][2];
        auto frags = [&](int ks) {
            a[ks & 1] = frag(a0 + 16 * ks * WG_A_PITCH, WG_A_PITCH);
#pragma unroll
            for (int t = 0; t < T; ++t) b[t][ks & 1] = frag(b0 + 16 * ks * WG_B_PITCH + 64 * t, WG_B_PITCH);
        };
        frags(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) frags(ks + 1);
#pragma unroll
            for (int t = 0; t < T; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks & 1], b[t][ks & 1], acc[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        put(std::integral_constant<int, (SET + 1) % 3>{}, st + 1, cur ^ 1);
        __syncthreads();
    };
    fetch(std::integral_constant<int, 0>{}, 0);
    fetch(std::integral_constant<int, 1>{}, 1);
    fetch(std::integral_constant<int, 2>{}, 2);
    put(std::integral_constant<int, 0>{}, 0, 0);
    __syncthreads();
    // always three stages per turn, with no branch between them (the compiler's wait counting then
    // lets two stages of fetches stay in flight); stages past the range multiply zeros
    for (int st = 0; st < nst; st += 3) {
        stage(std::integral_constant<int, 0>{}, st);
        stage(std::integral_constant<int, 1>{}, st + 1);
        stage(std::integral_constant<int, 2>{}, st + 2);
    }
    if (32 * wa >= k) return;   // this wave's weak columns do not exist
    // lane (fr, fk) holds, for channel oc0 + 32 (wb + t) + fr, weak columns 32 wa + 8 g + 4 fk .. + 3
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int j = oc0 + 32 * (wb + t) + fr;
        if (j >= oc_total) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 32 * wa + 8 * q + 4 * fk;
            if (i >= k) continue;
            f4 r = f4{acc[t][4 * q + 0], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]};
            const size_t at = (size_t)j * k_total + KW * kh + i;
            if (splits > 1) {
                *reinterpret_cast<f4*>(part + (size_t)split * oc_total * k_total + at) = r;
            } else if (out_f32) {
                f4* o = reinterpret_cast<f4*>((float*)dW + at);
                *o = accumulate ? *o + r : r;
            } else {
                __half* o = (__half*)dW + at;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = __float2half_rn(accumulate ? __half2float(o[e]) + r[e] : r[e]);
            }
        }
    }
}

// A stage's 64 tokens are addressed by 32-bit byte offsets from its first: pitches of up to 2^25 elements, past them the general kernel.
inline bool strip_offsets_fit(int64_t ld) { return ld <= 2 * (int64_t)QEFT_MAX_DIM; }

// The strips as a launch carries them; n workgroups (0: none).
struct Strips {
    int n, oc, k, M;
    int64_t lddy, ldxw;
    const __half *dY, *Xw;
    float* part;
    int splits, chunk, kw;
    void* dW;
    int out_f32, accumulate;
};
__device__ __forceinline__ void weak_grad_strip(unsigned char* lds, int bid, const Strips& S) {
    if (S.kw == 128) weak_grad_strip_body<128>(lds, bid, S.oc, S.k, S.dY, S.M, S.lddy, S.Xw, S.ldxw, S.part, S.splits, S.chunk, S.dW, S.out_f32, S.accumulate);
    else weak_grad_strip_body<64>(lds, bid, S.oc, S.k, S.dY, S.M, S.lddy, S.Xw, S.ldxw, S.part, S.splits, S.chunk, S.dW, S.out_f32, S.accumulate);
}

// The most ways the tokens are split for the strip kernel: about one workgroup per CU, every split a whole number of
// stages.  The workspace is sized for it.
inline int weak_grad_strip_most(int oc, int k, int64_t M) {
    const int tiles = ceil_div(oc, WG_OC) * ceil_div(k, 128);
    const int stages = ceil_div(M, BK);
    int want = ceil_div(256, tiles);
    if (want > stages) want = stages;
    if (want < 1) want = 1;
    return ceil_div(M, ceil_div(stages, want) * BK);
}
// The split and the pieces taken: a stage of 64 tokens costs a workgroup about 0.62 us where the piece's 128 weak columns all exist, 1.06 where
// some do not, 0.42 and 0.7 in pieces of 64 (half the multiplications, two thirds of the loads and LDS accesses, in a stream that nothing else hides);
// workgroups past one per CU count in full there, by 0.3 where columns are missing (a stage that waits leaves room for another's).  Twice as many pieces
// read dY twice as often: they count in full where strips begin between cache lines (OC no multiple of 64), by 0.6 elsewhere where unsplit ones are more than two per CU (by 0.3 too, us against pieces
// of 128: 27160 / 12216 channels, k = 96 / 72, M = 1441 / 1990 51.7 / 37.1 against 33.8 / 29.5; 13824, k = 224, 4096: 100 against 78.6; but 14336, k = 96, 1331 20.8 against 24.4, 11008, k = 72, 2183
// in two splits 26.7 against 28.7).
// Three pieces in place of two gain at any number of them (26200, k = 136, 77: 12.3 against 15.6).  A
// split costs the second launch and its partial slab's way through memory (2 us once, 0.65 us per MB
// and, where columns are missing, 0.13 us each).  Pieces of 64 read dY once for each: in whole blocks of 128 only where all have a CU
// of their own (8192 channels, k = 256, M = 512 / 4096: 10.9 / 50.5 us against 10.0 / 40.2 by 128), and unsplit: behind tiles that fill the GPU twice as many
// workgroups cost more than their shorter time saves (1024 x 8192 at 2000, forward and backward: 90.9 us against 88.9).  Measured, pieces of 128 -> this rule, us:
// 4096 channels, k = 128, M = 200 / 512 / 777 / 1000: 7.5 / 8.8 / 12.3 / 12.9 -> 5.9 / 6.9 / 9.4 / 10.8; 5120 channels at
// 1000 / 2000 14.0 / 19.3 -> 10.8 / 17.0; 13824 channels, k = 64, M = 200 / 777 / 1500 / 3000: 8.8 / 18.0 / 23.4 / 36.9 -> 6.0 / 9.7 /
// 13.6 / 22.7; 4096 channels, k = 16, M = 777 / 2000 11.0 / 14.2 -> 9.0 / 11.3.  As many splits as above against the rule's, pieces of 128: 11008 channels,
// M = 512 / 2048: 19.0 / 26.0 against 9.5 / 22.6 (one; two at M = 3000).
struct StripPlan {
    int splits, chunk, kw;
    int workgroups(int oc, int k) const { return ceil_div(oc, WG_OC) * ceil_div(k, kw) * splits; }
};
inline StripPlan weak_grad_strip_split(int oc, int k, int64_t M) {
    const int stages = ceil_div(M, BK), most = weak_grad_strip_most(oc, k, M);
    const double slab_mb = (double)oc * k * 4e-6;
    double best = 1e30;
    StripPlan p = {1, stages * BK, 128};
    for (int kw = 64; kw <= 128; kw += 64) {
        const int tiles = ceil_div(oc, WG_OC) * ceil_div(k, kw);
        const bool full = k % kw == 0, twice = kw == 64 && ceil_div(k, 64) == 2 * ceil_div(k, 128);   // (k = 65 to 128: two pieces, not one)
        if (kw == 128 && k <= 64) break;
        const double stage_us = kw == 128 ? (full ? 0.62 : 1.06) : (full ? 0.42 : 0.7);
        for (int s = 1; s <= most; ++s) {
            const double w = (double)tiles * s / 256.0;
            if (kw == 64 && k % 128 == 0 && (w > 1 || s > 1)) break;
            const double t = (w <= 1 ? 1 : ((full && kw == 128) || (twice && oc % WG_OC != 0) ? w : (twice && tiles > 2 * 256 ? 0.1 + 0.6 * w : 0.7 + 0.3 * w))) * stage_us * ceil_div(stages, s) + (s > 1 ? 2.0 + ((full ? 0.0 : 0.13) + 0.65 * slab_mb) * s : 0.0);
            if (t < best) {
                best = t;
                p.chunk = ceil_div(stages, s) * BK;
                p.kw = kw;
            }
        }
    }
    p.splits = ceil_div(M, p.chunk);
    return p;
}

// The strips of g for a launch of an input gradient, cut as they would be alone (same bits): S.n = 0 where there are none to take or the
// workspace has no room for their slabs behind what the input gradient uses of it.
inline Strips make_strips(const WeakGrad* g, const __half* dY, int64_t M, int64_t lddy, size_t used) {
    Strips S = {};
    if (!g || !weak_grad_mfma_supported(g->oc, g->k, M) || !strip_offsets_fit(lddy) || !strip_offsets_fit(g->ldxw)) return S;
    const StripPlan p = weak_grad_strip_split(g->oc, g->k, M);
    S.splits = p.splits;
    S.chunk = p.chunk;
    S.kw = p.kw;
    if (S.splits > 1) {
        const size_t need = (size_t)S.splits * g->oc * g->k * sizeof(float);
        if (!g->ws || g->ws_bytes < need || ((g->ws_bytes - need) & ~(size_t)15) < used) return S;
        S.part = reinterpret_cast<float*>(g->ws + ((g->ws_bytes - need) & ~(size_t)15));
    }
    S.n = p.workgroups(g->oc, g->k);
    S.oc = g->oc;
    S.k = g->k;
    S.M = (int)M;
    S.lddy = lddy;
    S.ldxw = g->ldxw;
    S.dY = dY;
    S.Xw = g->Xw;
    S.dW = g->dW;
    S.out_f32 = g->out_f32;
    S.accumulate = g->accumulate;
    return S;
}
// behind the launch that carried S
inline hipError_t finish_strips(WeakGrad* g, const Strips& S, hipStream_t s) {
    if (S.n == 0) return hipSuccess;
    g->done = true;
    return S.splits > 1 ? weak_grad_reduce(S.part, S.splits, (int64_t)S.oc * S.k, S.dW, S.out_f32, S.accumulate, s) : hipSuccess;
}

}  // namespace gemm
}  // namespace qeft
