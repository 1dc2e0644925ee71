// Forward and input gradient of 4-bit layers where the 256 x 256 tiles of gemm.hip are too few to occupy the GPU and no
// workspace was given to split them (or the split's fp16 partial tiles and second launch cost more): tiles of 128 channels x
// 64 or 128 rows.  (Paper Sec. 3.2.1 and Sec. 3.3: short prompts, fine-tuning at a few hundred tokens.)
//
// A workgroup is 2 x KW waves: wave (ow, kw) multiplies 64 channels x all rows over the kw-th share of the contraction, so a
// tile keeps up to eight waves busy without a wave tile so narrow that LDS reads or conversions outweigh the products; the
// shares' partial tiles meet in LDS in fp32 and a fixed order.  As in gemm.hip the weights are converted into MFMA operand
// registers and only activations (and, for the input gradient, raw codes) pass through LDS: 64-step pipeline, fragments two
// k-blocks ahead, one barrier per 64 columns.
//
// What bounds it: vector issue.  An MFMA 32x32x16 holds a SIMD's issue for 12 of its 32 cycles and every vector instruction
// for 4, also with two waves per SIMD (measured: 33 cycles per MFMA with up to 5 of them, 44 with 8, 60 with 12).  A wave of
// 64 rows converts 17 instructions per word for 2 products each and runs 11.8 per MFMA (counted); of 128 rows 7.2 to 7.5.  A launch costs 8 to
// 10 us beyond its stages (first fetches from HBM, the exchange of partial tiles, stores).
// Measured, without a workspace, before -> now (us): forward 4096 x 4096 at M = 333 / 512 / 777: 77 -> 26 / 29 / 40,
// 4096 x 11008 at 512: 206 -> 72; input gradient 4096 x 4096 at 333 / 512 / 777: 90 -> 31 / 35 / 50, 11008 x 4096 at 512:
// 228 -> 86.  Forward with a K-split workspace, 4096 x 4096 at 333 / 512: 32 / 34 -> 26 / 29; 5120 x 5120 at 333: 38 -> 33.
// Tried and not kept: four stages of activations on the way instead of two (no change: not latency), the activations requested half
// a stage later (10 % slower), codes requested four stages (a cache line) at a time (4 to 15 % slower), four shares of the contraction
// in the forward (no change at two waves per SIMD, uneven shares), conversions of one operation less (no change: timing variants
// without conversions or without any memory access still take 80 to 95 % of the time), weak columns after
// the quantized ones (exposes their fetch), conversions as the compiler orders them (chains of dependent packed operations).
#include <type_traits>
#include <utility>

#include "gemm_common.h"
#include "qeft_internal.h"
#include "weak_strip.h"

namespace qeft {
using namespace gemm;
namespace {

typedef __attribute__((address_space(3))) u4 lds_u4;
typedef __attribute__((address_space(3))) h8 lds_h8;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) f4 lds_f4;
typedef int v2i __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(3))) s4 lds_s4;
using gptr = const __attribute__((address_space(1))) unsigned char*;
using g_u4 = const __attribute__((address_space(1))) u4;
using g_u2 = const __attribute__((address_space(1))) u2;
using g_u16 = const __attribute__((address_space(1))) uint16_t;

// a wave-uniform base the compiler keeps in scalar registers
__device__ __forceinline__ gptr sbase(const void* p) {
    asm volatile("" : "+s"(p));
    return (gptr)p;
}
__device__ __forceinline__ uint32_t lds_at(const void* p) { return (uint32_t)(size_t)(__attribute__((address_space(3))) const unsigned char*)p; }
__device__ __forceinline__ uint32_t pack2(float a, float b) { return h2_bits(h2{(_Float16)a, (_Float16)b}); }
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

template <int... Ts, class F>
__device__ __forceinline__ void each_slot(std::integer_sequence<int, Ts...>, F&& f) {
    (f(std::integral_constant<int, Ts>{}), ...);
}

// The K groups' partial tiles (64 x 32 J of a wave: MFMA tile q = 2 j + i) meet in LDS: tiles q of owner q / QT, which adds
// the others' in the order of the K groups and stores rows of 32 channels.  chan(i) = first channel of row block i; out[m][channel].
template <int J, int KW>
__device__ __forceinline__ void finish(f16v (&acc)[2][J], unsigned char* lds, int ow, int kw, int wave, int lane, __half* Y, int64_t ldy, int c0,
                                       int nc, int m0, int M) {
    constexpr int QT = 2 * J / KW;
    const int fr = lane & 31, fk = lane >> 5;
    float* part = reinterpret_cast<float*>(lds);   // [ow][owner][sender][QT][4][64][4]
#pragma unroll
    for (int q = 0; q < 2 * J; ++q) {
        const int owner = q / QT;
        if (owner != kw) {
            float* p = part + ((((ow * KW + owner) * (KW - 1) + (kw < owner ? kw : kw - 1)) * QT + q % QT) << 10) + 4 * lane;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<f4*>(p + 256 * e) = f4{acc[q & 1][q >> 1][4 * e], acc[q & 1][q >> 1][4 * e + 1], acc[q & 1][q >> 1][4 * e + 2], acc[q & 1][q >> 1][4 * e + 3]};
        }
    }
    __syncthreads();
    f16v own[QT];
#pragma unroll
    for (int o = 0; o < KW; ++o)
        if (o == kw) {
#pragma unroll
            for (int q = 0; q < QT; ++q) own[q] = acc[(o * QT + q) & 1][(o * QT + q) >> 1];
        }
    for (int s = 0; s < KW - 1; ++s) {
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            const float* p = part + ((((ow * KW + kw) * (KW - 1) + s) * QT + q) << 10) + 4 * lane;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f4 t = *reinterpret_cast<const f4*>(p + 256 * e);
#pragma unroll
                for (int x = 0; x < 4; ++x) own[q][4 * e + x] += t[x];
            }
        }
    }
    __syncthreads();
    unsigned char* stg = lds + wave * 2048;   // 32 rows of 64 bytes
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        const int tq = kw * QT + q, i = tq & 1, j = tq >> 1;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<u2*>(stg + fr * 64 + (((g ^ (fr >> 1)) & 3) << 4) + 8 * fk) =
                u2{pack2(own[q][4 * g], own[q][4 * g + 1]), pack2(own[q][4 * g + 2], own[q][4 * g + 3])};
        wave_lds_fence();
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int r = 16 * it + (lane >> 2), c = lane & 3;
            const u4 v = *reinterpret_cast<const u4*>(stg + r * 64 + (((c ^ (r >> 1)) & 3) << 4));
            const int m = m0 + 32 * j + r, o = c0 + 32 * i + 8 * c;
            if (m < M && o < nc) *reinterpret_cast<u4*>(Y + (size_t)m * ldy + o) = v;
        }
        wave_lds_fence();
    }
}

struct Conv {
    uint32_t m0 = 0x000f000fu, m1 = 0x00f000f0u, g0 = 0x64006400u, g1 = 0x54005400u;
    uint32_t cq[8], w8[2];
    __device__ __forceinline__ Conv() { asm volatile("" : "+v"(m0), "+v"(m1), "+v"(g0), "+v"(g1)); }
    // pair p = 4 i + a of word w: nibbles at bits 0..3 of a half become 1024 + q, at bits 4..7 64 + q
    __device__ __forceinline__ void mask(int p, uint32_t w) {
        const int a = p & 3, i = p >> 2;
        if (a == 2) w8[i] = w >> 8;
        const uint32_t src = a < 2 ? w : w8[i];
        cq[p] = (a & 1) ? ((src & m1) | g1) : ((src & m0) | g0);
    }
    __device__ __forceinline__ void base(int p) {
        const h2 k1024 = h2{(_Float16)1024.f, (_Float16)1024.f}, k64 = h2{(_Float16)64.f, (_Float16)64.f};
        cq[p] = h2_bits(bits_h2(cq[p]) - ((p & 1) ? k64 : k1024));
    }
    __device__ __forceinline__ void zero(int p, h2 z) { cq[p] = h2_bits(bits_h2(cq[p]) - z); }
    __device__ __forceinline__ uint32_t scale(int p, h2 s) const { return h2_bits(bits_h2(cq[p]) * s); }
    // the same pair with one rounding (see dequant_once), half by half
    _Float16 lo[8];
    __device__ __forceinline__ void first(int p, h2 s, float nzs) { lo[p] = dequant_once_first(bits_h2(cq[p]).x, s.x, nzs); }
    __device__ __forceinline__ uint32_t second(int p, h2 s, float nzs) const { return h2_bits(h2{lo[p], dequant_once(bits_h2(cq[p]).y, s.y, nzs)}); }
};

// The rows of the activation operand ([m][contraction], fp16): the 128 threads of a K group fetch its tile of 32 J rows x
// 64 columns, thread tk rows tk / 8 + 16 u, chunk tk % 8.
template <int J, int SETS>
struct RowTile {
    static constexpr int NX = 2 * J, XT = 32 * J * 128;
    const unsigned char* xb;
    uint32_t xrow[NX], xw[4], fb[8];
    int xc;
    u4 v[SETS][NX];
    __device__ __forceinline__ RowTile(const __half* X, int64_t ldx, int m0, int M, int tk, uint32_t lds0, int fr, int fkbase) {
        const int xr = tk >> 3;
        xc = tk & 7;
        xb = reinterpret_cast<const unsigned char*>(X + (size_t)m0 * ldx);
        const uint32_t pitch = (uint32_t)ldx * 2u, last = (uint32_t)min(M - 1 - m0, 32 * J) * pitch;
#pragma unroll
        for (int u = 0; u < NX; ++u) xrow[u] = min((uint32_t)(xr + 16 * u) * pitch, last);
        // rows 16 apart differ in bit 1 of the swizzle: write bases for four; fragment reads: one base per XOR constant
#pragma unroll
        for (int u = 0; u < 4; ++u) xw[u] = lds0 + (uint32_t)tile_off(xr + 16 * u, xc);
#pragma unroll
        for (int x = 0; x < 8; ++x) fb[x] = lds0 + (uint32_t)fr * 128u + ((((uint32_t)(fkbase ^ (fr & 7) ^ (fr >> 3))) ^ (uint32_t)x) << 4);
    }
    // 64 columns from col on; past ncols (a multiple of 8): the row's last 8
    __device__ __forceinline__ void load(int set, int u, int col, int ncols) {
        v[set][u] = *reinterpret_cast<g_u4*>(sbase(xb) + (xrow[u] + 2u * (uint32_t)min(col + 8 * xc, ncols - 8)));
    }
    // 64 columns from col on, all of them within the row; after chunk_in_row()
    __device__ __forceinline__ void load_whole(int set, int u, int col) { v[set][u] = *reinterpret_cast<g_u4*>(sbase(xb + 2 * col) + xrow[u]); }
    __device__ __forceinline__ void chunk_in_row() {
#pragma unroll
        for (int u = 0; u < NX; ++u) xrow[u] += 16u * (uint32_t)xc;
    }
    __device__ __forceinline__ void put(int u, int buf, u4 x) { *reinterpret_cast<lds_u4*>(xw[u & 3] + (uint32_t)((u >> 2) * 8192 + buf * XT)) = x; }
    __device__ __forceinline__ h8 frag(int j, int buf, int chunk) const {   // chunk: XOR part of the chunk index
        return *reinterpret_cast<const lds_h8*>(fb[chunk ^ (4 * (j & 1))] + (uint32_t)(j * 4096 + buf * XT));
    }
    __device__ __forceinline__ void opaque() {   // keeps base + constant from being hoisted into a register per constant
        asm volatile("" : "+v"(fb[0]), "+v"(fb[1]), "+v"(fb[2]), "+v"(fb[3]), "+v"(fb[4]), "+v"(fb[5]), "+v"(fb[6]), "+v"(fb[7]));
        asm volatile("" : "+v"(xw[0]), "+v"(xw[1]), "+v"(xw[2]), "+v"(xw[3]));
    }
};

// ---- forward -----------------------------------------------------------------------------------------------------
template <int J, int KW, int MINW, bool ONCE>
__global__ __launch_bounds__(128 * KW, MINW) void fwd_tile_kernel(Layer L, const __half* __restrict__ X, int M, int64_t ldx, __half* __restrict__ Y,
                                                                 int64_t ldy, int tiles_n, int tiles_m) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    constexpr int DX = 2, DA = 4;               // stages of activations / codes on the way
    using Rows = RowTile<J, DX>;
    constexpr int NX = Rows::NX, XT = Rows::XT, S = 2 * J;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ow = wave & 1, kw = wave >> 1;
    const int fr = lane & 31, fk = lane >> 5;
    const int tile = xcd_tile(tiles_n * tiles_m);
    if (tile < 0) return;
    int t_n, t_m;
    tile_coords(tile, tiles_n, tiles_m, t_n, t_m);
    const int ob = t_n * 128, m0 = t_m * (32 * J);
    const int nchunks = (L.ng + 3) >> 2, turns = (nchunks + KW - 1) / KW;
    const u4 zero4 = u4{0u, 0u, 0u, 0u};

    const unsigned char* wt = reinterpret_cast<const unsigned char*>(L.qweight + (size_t)ob * L.stride);
    const unsigned char* st_ = reinterpret_cast<const unsigned char*>(L.scales + (size_t)ob * L.gs);
    const unsigned char* zt = reinterpret_cast<const unsigned char*>(L.zeros + (size_t)ob * L.gs);
    uint32_t aoff[2], poff[2];
    int arow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        arow[i] = min(64 * ow + 32 * i + fr, L.oc - 1 - ob);
        aoff[i] = (uint32_t)arow[i] * (uint32_t)(L.stride * 4) + 16u * fk;
        poff[i] = (uint32_t)arow[i] * (uint32_t)(L.gs * 2);
    }
    // k-block ks of a stage, half fk: columns 32 fk + 8 ks .. + 7 (a lane's 16 bytes of codes are its words of all four)
    Rows x(X, ldx, m0, M, tid & 127, lds_at(lds) + (uint32_t)(kw * 2 * XT), fr, 4 * fk);

    u4 araw[DA][2];
    u2 szs[2], szz[2], nzs[2], nzz[2];
    const int nst = (L.kq + 63) / 64;
    auto load_a = [&](int set, int st) {
#pragma unroll
        for (int i = 0; i < 2; ++i) araw[set][i] = *reinterpret_cast<g_u4*>(sbase(wt + 32 * min(st, nst - 1)) + aoff[i]);
    };
    auto load_par = [&](int g) {
        const int g4 = min(g, L.ng - 1) & ~3;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            nzs[i] = *reinterpret_cast<g_u2*>(sbase(st_ + 2 * g4) + poff[i]);
            nzz[i] = *reinterpret_cast<g_u2*>(sbase(zt + 2 * g4) + poff[i]);
        }
    };

    f16v acc[2][J];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // weak block: stage w (64 columns) belongs to K group w % KW; fp16 fragments straight from the stored block
    const int nweak = (L.k + 63) >> 6, kpos = max(L.k, 8);
    u4 wf[2][4], xwk[NX];
    auto load_weak = [&](int w) {
#pragma unroll
        for (int u = 0; u < NX; ++u)
            xwk[u] = *reinterpret_cast<g_u4*>(sbase(x.xb) + (x.xrow[u] + 2u * (uint32_t)min(L.kq + 64 * w + 8 * x.xc, L.ic - 8)));
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                wf[i][ks] = ld16(L.weak + (size_t)(ob + arow[i]) * L.k + min(64 * w + 32 * fk + 8 * ks, kpos - 8));
    };
    auto put_weak = [&](int w, int buf) {
        const bool live = 64 * w + 8 * x.xc < L.k;
#pragma unroll
        for (int u = 0; u < NX; ++u) x.put(u, buf, live ? xwk[u] : zero4);
    };
    auto mul_weak = [&](int w, int buf) {
        if (64 * w >= L.k) return;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const bool live = 64 * w + 32 * fk + 8 * ks < L.k;   // both operands: nothing past the block may meet the zeros of the other
            h8 b[J];
#pragma unroll
            for (int j = 0; j < J; ++j) b[j] = x.frag(j, buf, ks);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const h8 a = __builtin_bit_cast(h8, live ? wf[i][ks] : zero4);
#pragma unroll
                for (int j = 0; j < J; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b[j], acc[i][j], 0, 0, 0);
            }
        }
    };

    // quantized stages: turn t of K group kw is chunk t KW + kw (four groups = eight stages of 64 columns)
    auto stage_of = [&](int chunk, int e) { return 8 * (chunk + (e >> 3) * KW) + (e & 7); };   // stage e of the turn, running on into the next
    load_weak(kw);
    load_par(4 * kw);
#pragma unroll
    for (int d = 0; d < DX; ++d)
#pragma unroll
        for (int u = 0; u < NX; ++u) x.load(d, u, 64 * stage_of(kw, d), L.kq);
#pragma unroll
    for (int d = 0; d < DA; ++d) load_a(d, stage_of(kw, d));
    __builtin_amdgcn_sched_barrier(0);
    put_weak(kw, 1);
    {
        const bool live = 64 * stage_of(kw, 0) + 8 * x.xc < L.kq;
#pragma unroll
        for (int u = 0; u < NX; ++u) x.put(u, 0, live ? permute_x(x.v[0][u]) : zero4);
#pragma unroll
        for (int u = 0; u < NX; ++u) x.load(0, u, 64 * stage_of(kw, DX), L.kq);
    }
    __syncthreads();
    mul_weak(kw, 1);
    __syncthreads();

    Conv cv;
    h8 bfr[4][J];   // fragments are read two k-blocks ahead
    u4 afr[2][2];
    h2 z2[2], s2[2];
    float mzs[2];   // - zero-point * scale (ONCE)
    auto latch = [&](int q) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const h2 sv = bits_h2(q < 2 ? szs[i].x : szs[i].y), zv = bits_h2(q < 2 ? szz[i].x : szz[i].y);
            z2[i] = (q & 1) ? h2{zv.y, zv.y} : h2{zv.x, zv.x};
            s2[i] = (q & 1) ? h2{sv.y, sv.y} : h2{sv.x, sv.x};
            if constexpr (ONCE) mzs[i] = neg_zs(z2[i].x, s2[i].x);
        }
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) szs[i] = nzs[i], szz[i] = nzz[i];
    latch(0);
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        cv.mask(p, araw[0][p >> 2].x);
        cv.base(p);
        if constexpr (ONCE) cv.first(p, s2[p >> 2], mzs[p >> 2]);
        else cv.zero(p, z2[p >> 2]);
        afr[0][p >> 2][p & 3] = ONCE ? cv.second(p, s2[p >> 2], mzs[p >> 2]) : cv.scale(p, s2[p >> 2]);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) bfr[0][j] = x.frag(j, 0, 0), bfr[1][j] = x.frag(j, 0, 1);
    for (int t = 0; t < turns; ++t) {
        const int chunk = t * KW + kw, next = chunk + KW;
        load_par(4 * next);
        auto stage = [&](auto e_c) {
            constexpr int E = decltype(e_c)::value, CUR = E & 1, NXT = CUR ^ 1, SETX = (E + 1) % DX;
            const int s_put = stage_of(chunk, E + 1), s_ld = stage_of(chunk, E + 1 + DX);
            if (64 * s_put + 64 > L.kq) {   // columns past Kq become zeros
                const bool live = 64 * s_put + 8 * x.xc < L.kq;
#pragma unroll
                for (int u = 0; u < NX; ++u) x.v[SETX][u] = live ? x.v[SETX][u] : zero4;
            }
            x.opaque();
            u4 px[2];
            auto slot = [&](auto t_c) {
                constexpr int T = decltype(t_c)::value, ks = T / S, m = T % S, i = m / J, j = m % J, kn = (ks + 1) & 3;
                constexpr int EN = ks < 3 ? E : E + 1;   // stage of the next k-block
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, afr[ks & 1][i]), bfr[ks][j], acc[i][j], 0, 0, 0);
                if (ks == 3 && m == 0) {
                    if (E == 7) {
#pragma unroll
                        for (int ii = 0; ii < 2; ++ii) szs[ii] = nzs[ii], szz[ii] = nzz[ii];
                    }
                    if (E & 1) latch(((E + 1) >> 1) & 3);
                }
                // conversion of the next k-block in four phases of independent operations
                constexpr int PP = 32 / S;
#pragma unroll
                for (int o = m * PP; o < (m + 1) * PP; ++o) {
                    const int ph = o >> 3, p = o & 7;
                    if (ph == 0) cv.mask(p, araw[EN % DA][p >> 2][kn]);
                    else if (ph == 1) cv.base(p);
                    else if (ph == 2) {
                        if constexpr (ONCE) cv.first(p, s2[p >> 2], mzs[p >> 2]);
                        else cv.zero(p, z2[p >> 2]);
                    } else
                        afr[kn & 1][p >> 2][p & 3] = ONCE ? cv.second(p, s2[p >> 2], mzs[p >> 2]) : cv.scale(p, s2[p >> 2]);
                }
                if (m % 2 == 0) bfr[(ks + 2) & 3][m / 2] = x.frag(m / 2, ks < 2 ? CUR : NXT, (ks + 2) & 3);
                // next stage's activations, chunk by chunk: permuted in one slot, stored and refilled in the next.  128 rows: without
                // gaps, so that the last stores are long done when the barrier waits for them (4096 x 11008, M = 777: 97.5 us with gaps, 94.3
                // without); 64 rows: a slot has twice the conversions and no room for both (M = 512: 66.2, without gaps 69.1)
                constexpr int GAP = J == 2 ? 2 : 1;
                if constexpr (T % GAP == 0 && T / GAP < NX) px[(T / GAP) & 1] = permute_x(x.v[SETX][T / GAP]);
                if constexpr (T > 0 && (T - 1) % GAP == 0 && (T - 1) / GAP < NX) {
                    constexpr int u = (T - 1) / GAP;
                    x.put(u, NXT, px[u & 1]);
                    x.load(SETX, u, 64 * s_ld, L.kq);
                }
                if (ks == 3 && m == S - 1) {
                    load_a(E % DA, stage_of(chunk, E + DA));
                    // the next stage's first conversions stay here, behind this k-block's products: the compiler moves them below the
                    // branch at the head of that stage otherwise, 34 vector instructions beside no product (4096 x 11008, M = 256: 59 us,
                    // 55 so)
                    asm volatile("" : "+v"(afr[0][0]), "+v"(afr[0][1]));
                }
                if (ks == 1 && m == S - 1) __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            };
            each_slot(std::make_integer_sequence<int, 4 * S>{}, slot);
        };
        each_slot(std::make_integer_sequence<int, 8>{}, stage);
    }
    __syncthreads();
    for (int w0 = KW; w0 < nweak; w0 += KW) {
        load_weak(w0 + kw);
        put_weak(w0 + kw, 0);
        __syncthreads();
        mul_weak(w0 + kw, 0);
        __syncthreads();
    }
    finish<J, KW>(acc, lds, ow, kw, wave, lane, Y, ldy, ob + 64 * ow, L.oc, m0, M);
}

// ---- input gradient --------------------------------------------------------------------------------------------------
// The contraction runs along the rows of the stored matrices, which the MFMA wants as 8 consecutive rows of one channel per
// lane.  Raw codes pass through LDS as they are stored and are read with gfx950's transposing 4-bit load (16 lanes name 16
// rows of 16 codes; lane s receives the 16 rows of column s, lowest row in the lowest nibble - checked with a probe): what a
// lane gets is a packed word as in the forward, and the same conversion follows with the rows' zero-points and scales as
// vectors.  A tile is either quantized or weak, whatever Kq (the GEMM of gemm.hip
// puts a partial group and weak columns into one tile and then takes its LDS-staged form); weak ones read fp16 with the 16-bit form.
// RAGGED: OC is no multiple of 64.
// D: strips of the weak gradient behind the tiles (the one-call backward), on CUs that have no tile or are done with theirs.  The whole backward, two
// launches -> one, us: 1024 x 8192 at M = 128 17 -> 12; 2048 x 3000 with 16 weak columns at 128 / 1000 23 / 37 -> 17 / 32; 5120 x 5120 with 64 at 333 / 777
// 49 / 104 -> 41 / 94.
template <int J, int KW, int MINW, bool ONCE, bool RAGGED>
__global__ __launch_bounds__(128 * KW, MINW) void dx_tile_kernel(Layer L, const __half* __restrict__ dY, int M, int64_t lddy,
                                                                __half* __restrict__ dX, int64_t lddx, int tiles_n, int tiles_m, Strips D) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    if ((int)blockIdx.x >= (int)gridDim.x - D.n) {   // behind the tiles: a strip of the weak gradient, by four waves
        if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < 4) weak_grad_strip(lds, (int)blockIdx.x - ((int)gridDim.x - D.n), D);
        return;
    }
    constexpr int DX = 2;
    using Rows = RowTile<J, DX>;
    constexpr int NX = Rows::NX, XT = Rows::XT, S = 2 * J;
    // a stage of codes (64 rows of 128 channels) and of parameters (per 8 rows: zero-points, scales; ONCE: fp32 - zero-point * scale, scales)
    constexpr int CT = 64 * 64, VS = ONCE ? 32 : 16, VT = 8 * (VS + 16);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ow = wave & 1, kw = wave >> 1;
    const int fr = lane & 31, fk = lane >> 5, tk = tid & 127;
    const int tile = xcd_tile(tiles_n * tiles_m);
    if (tile < 0) return;
    int t_n, t_m;
    tile_coords(tile, tiles_n, tiles_m, t_n, t_m);
    // quantized tiles first (the last may be part of a group), then those of the weak block
    const int nq = (L.kq + 127) >> 7;
    const int c0 = t_n < nq ? t_n * 128 : L.kq + (t_n - nq) * 128, m0 = t_m * (32 * J);
    const int nst = (L.oc + 63) >> 6, turns = (nst + 2 * KW - 1) / (2 * KW);   // a turn: two stages of each K group
    const u4 zero4 = u4{0u, 0u, 0u, 0u};

    const uint32_t lx = lds_at(lds) + (uint32_t)(kw * 2 * XT);
    // k-block ks of a stage, half fk: rows 32 (ks / 2) + 16 fk + 8 (ks % 2) .. + 7
    Rows x(dY, lddy, m0, M, tk, lx, fr, 2 * fk);
    auto chunk_of = [](int ks) { return 4 * (ks >> 1) + (ks & 1); };
    auto stage_of = [&](int t, int e) { return 2 * ((t + (e >> 1)) * KW + kw) + (e & 1); };
    // Rows of a stage: 64 from 64 st on; the last stage of an OC that is no multiple of 64 begins at OC - 64, and what it shares with
    // the one before counts as zeros in dY, as do stages past the last.  (No clamp per row, and no read past the stored matrices.
    // RAGGED has to be known here: with the selects below in every call, 4096 x 4096 at M = 777 took 52.8 us against 51.3.)
    auto first_row = [&](int st) { return RAGGED ? min(64 * st, L.oc - 64) : 64 * st; };
    auto stage_live = [&](int st) { return RAGGED ? st < nst && first_row(st) + 8 * x.xc >= 64 * st : st < nst; };
    auto load_y = [&](int set, int u, int st) {
        if constexpr (RAGGED) x.load_whole(set, u, first_row(st));
        else x.load(set, u, 64 * st, L.oc);
    };

    f16v acc[2][J];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    if (t_n < nq) {
        const uint32_t lc = lds_at(lds) + (uint32_t)(KW * 2 * XT + kw * 2 * CT);
        const uint32_t lv = lds_at(lds) + (uint32_t)(KW * (2 * XT + 2 * CT) + kw * 2 * VT);
        // codes: thread tk fetches half a row of the stage (row tk / 2, 32 bytes); parameters: threads 0 .. 63 the scales,
        // 64 .. 127 the zero-points, one row each (ONCE: a row's two lie 32 lanes apart in one wave, which swaps its halves and stores both
        // values from both lanes; a branch here would make the compiler wait for every request on the way, and these requests, 64
        // cache lines each, are as dear as the codes')
        const unsigned char* wt = reinterpret_cast<const unsigned char*>(L.qweight) + c0 / 2;
        const int crow = tk >> 1, cpart = tk & 1, prow = ONCE ? 32 * ow + (lane & 31) : tk & 63;
        const uint32_t wpitch = (uint32_t)L.stride * 4u;
        const unsigned char* pt = reinterpret_cast<const unsigned char*>((ow == 0 ? L.scales : L.zeros) + c0 / 128);   // (threads 0 .. 63: wave 0 of the K group)
        const uint32_t coff = (uint32_t)crow * wpitch + 32u * cpart, poff = (uint32_t)prow * (uint32_t)(L.gs * 2);
        const unsigned char* pl = reinterpret_cast<const unsigned char*>((lane < 32 ? L.scales : L.zeros) + c0 / 128) + poff;   // (ONCE)
        u4 cw[DX][2];
        uint32_t pv[DX];
        if constexpr (RAGGED) x.chunk_in_row();
        auto load_c = [&](int set, int st) {   // (stages past the last repeat it; their rows of dY are zeroed)
            const int sc = min(st, nst - 1);
            gptr p = sbase(wt + (size_t)first_row(sc) * wpitch) + coff;
            cw[set][0] = *reinterpret_cast<g_u4*>(p);
            cw[set][1] = *reinterpret_cast<g_u4*>(p + 16);
            const size_t at = (size_t)first_row(sc) * (uint32_t)(L.gs * 2);
            if constexpr (ONCE) pv[set] = *(g_u16*)(pl + at);
            else pv[set] = *reinterpret_cast<g_u16*>(sbase(pt + at) + poff);
        };
        // chunk c (32 channels) of row r sits in slot c ^ (r / 4 % 4): the 16 rows of a transposing read then spread over the banks
        const uint32_t cst = lc + (uint32_t)(crow * 64);
        const uint32_t csw = (uint32_t)((crow >> 2) & 3);
        const int pat = (prow & 3) * 2 + ((prow >> 2) & 1);   // rows r and r + 4 of 8 side by side, as a word's pairs
        const uint32_t pst = lv + (uint32_t)((prow >> 3) * (VS + 16) + (ow == 0 && !ONCE ? VS + 2 * pat : (VS / 8) * pat));
        const uint32_t pss = lv + (uint32_t)((prow >> 3) * (VS + 16) + VS + 2 * pat);   // (ONCE)
        auto put_c = [&](int set, int buf) {
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<lds_u4*>(cst + (((2 * cpart + h) ^ csw) << 4) + (uint32_t)(buf * CT)) = cw[set][h];
            if constexpr (ONCE) {
                const auto sz = __builtin_amdgcn_permlane32_swap(pv[set], pv[set], false, false);   // the scale, the zero-point
                *reinterpret_cast<lds_f32*>(pst + (uint32_t)(buf * VT)) = neg_zs(bits_h2(sz[1]).x, bits_h2(sz[0]).x);
                *reinterpret_cast<lds_u16*>(pss + (uint32_t)(buf * VT)) = (uint16_t)sz[0];
            } else
                *reinterpret_cast<lds_u16*>(pst + (uint32_t)(buf * VT)) = (uint16_t)pv[set];
        };
        // a transposing read hands lane s of each 16 the 16 rows of column s of a 16 x 16 block of codes; block row 32 p + 16 fk,
        // column block 32 i + 16 (lane / 16 % 2) of the wave's 64 channels
        const int tr = 16 * fk + (lane & 15);
        uint32_t trb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) trb[i] = lc + (uint32_t)(tr * 64) + (uint32_t)(((2 * ow + i) ^ ((tr >> 2) & 3)) << 4) + 8u * ((lane >> 4) & 1);
        v2i raw[2][2];   // [p][i]: rows 32 p + 16 fk + 0 .. 7, 8 .. 15 of the lane's channel
        auto read_raw = [&](int p, int i, int buf) {
            raw[p][i] = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(size_t)(trb[i] + (uint32_t)(p * 2048 + buf * CT)));
        };
        u4 zv[2], sv[2];
        f4 nzs[2][2];
        const uint32_t vb = lv + (uint32_t)(2 * (VS + 16)) * fk;
        auto read_par = [&](int set, int ks, int buf) {
            const uint32_t at = vb + (uint32_t)(chunk_of(ks) * (VS + 16) + buf * VT);
            if constexpr (ONCE) {
#pragma unroll
                for (int h = 0; h < 2; ++h) nzs[set][h] = *reinterpret_cast<const lds_f4*>(at + (uint32_t)(16 * h));
            } else
                zv[set] = *reinterpret_cast<const lds_u4*>(at);
            sv[set] = *reinterpret_cast<const lds_u4*>(at + VS);
        };
        auto convert_zero = [&](Conv& c, int set, int p) {
            if constexpr (ONCE) c.first(p, bits_h2(sv[set][p & 3]), nzs[set][(p & 3) >> 1][2 * (p & 1)]);
            else c.zero(p, bits_h2(zv[set][p & 3]));
        };
        auto convert_scale = [&](const Conv& c, int set, int p) {
            if constexpr (ONCE) return c.second(p, bits_h2(sv[set][p & 3]), nzs[set][(p & 3) >> 1][2 * (p & 1) + 1]);
            else return c.scale(p, bits_h2(sv[set][p & 3]));
        };

#pragma unroll
        for (int d = 0; d < DX; ++d) {
            load_c(d, stage_of(0, d));
#pragma unroll
            for (int u = 0; u < NX; ++u) load_y(d, u, stage_of(0, d));
        }
        __builtin_amdgcn_sched_barrier(0);
        {
            const bool live = stage_live(stage_of(0, 0));
            put_c(0, 0);
#pragma unroll
            for (int u = 0; u < NX; ++u) x.put(u, 0, live ? permute_x(x.v[0][u]) : zero4);
            load_c(0, stage_of(0, DX));
#pragma unroll
            for (int u = 0; u < NX; ++u) load_y(0, u, stage_of(0, DX));
        }
        __syncthreads();
        Conv cv;
        h8 bfr[4][J];
        u4 afr[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i) read_raw(0, i, 0);
        read_par(0, 0, 0);
        read_par(1, 1, 0);
#pragma unroll
        for (int j = 0; j < J; ++j) bfr[0][j] = x.frag(j, 0, chunk_of(0)), bfr[1][j] = x.frag(j, 0, chunk_of(1));
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            cv.mask(p, (uint32_t)raw[0][p >> 2].x);
            cv.base(p);
            convert_zero(cv, 0, p);
            afr[0][p >> 2][p & 3] = convert_scale(cv, 0, p);
        }
        read_par(0, 2, 0);
        for (int t = 0; t < turns; ++t) {
            auto stage = [&](auto e_c) {
                constexpr int E = decltype(e_c)::value, CUR = E & 1, NXT = CUR ^ 1, SETX = (E + 1) % DX;
                const int s_put = stage_of(t, E + 1), s_ld = stage_of(t, E + 1 + DX);
                if (64 * s_put + 64 > L.oc) {   // rows past OC, or before the stage's own
                    const bool live = stage_live(s_put);
#pragma unroll
                    for (int u = 0; u < NX; ++u) x.v[SETX][u] = live ? x.v[SETX][u] : zero4;
                }
                x.opaque();
                u4 px[2];
                auto slot = [&](auto t_c) {
                    constexpr int T = decltype(t_c)::value, ks = T / S, m = T % S, i = m / J, j = m % J, kn = (ks + 1) & 3;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, afr[ks & 1][i]), bfr[ks][j], acc[i][j], 0, 0, 0);
                    constexpr int PP = 32 / S;
#pragma unroll
                    for (int o = m * PP; o < (m + 1) * PP; ++o) {
                        const int ph = o >> 3, p = o & 7;
                        if (ph == 0) cv.mask(p, (uint32_t)raw[kn >> 1][p >> 2][kn & 1]);
                        else if (ph == 1) cv.base(p);
                        else if (ph == 2) convert_zero(cv, kn & 1, p);
                        else afr[kn & 1][p >> 2][p & 3] = convert_scale(cv, kn & 1, p);
                    }
                    if (m % 2 == 0) bfr[(ks + 2) & 3][m / 2] = x.frag(m / 2, ks < 2 ? CUR : NXT, chunk_of((ks + 2) & 3));
                    // the second half's codes early in k-block 0, the next stage's first half behind the barrier
                    if (ks == 0 && m < 2) read_raw(1, m, CUR);
                    if (ks == 2 && m < 2) read_raw(0, m, NXT);
                    if constexpr (T < 2 * NX) {
                        constexpr int u = T / 2;
                        if (T % 2 == 0) px[u & 1] = permute_x(x.v[SETX][u]);
                        else {
                            x.put(u, NXT, px[u & 1]);
                            load_y(SETX, u, s_ld);
                        }
                    }
                    if (T == 2) {
                        put_c(SETX, NXT);
                        load_c(SETX, s_ld);
                    }
                    if (ks == 1 && m == S - 1) __syncthreads();
                    // parameters of the k-block after the next: their set is free once this conversion's scales are used
                    if (m == S - 1) read_par(kn & 1, (ks + 3) & 3, ks < 1 ? CUR : NXT);
                    __builtin_amdgcn_sched_barrier(0);
                };
                each_slot(std::make_integer_sequence<int, 4 * S>{}, slot);
            };
            each_slot(std::make_integer_sequence<int, 2>{}, stage);
        }
        __syncthreads();
    } else {
        // weak channels: the fp16 block's rows through LDS, fragments read with the transposing 16-bit load.  Stages of 32
        // rows in two buffers (64 rows would leave room for one: writes and products would wait for each other, and the one
        // weak tile of a panel would end 9 us after the quantized ones), four stages on the way.
        constexpr int WP = 272;                  // bytes per row of 128 weak columns (256 + 16: rows spread over the banks)
        constexpr int WT = 32 * WP, YT = 32 * J * 64, NY = J;
        const int nst32 = (L.oc + 31) >> 5, turns32 = (nst32 + KW - 1) / KW;
        const uint32_t ly = lds_at(lds) + (uint32_t)(kw * 2 * YT), lw = lds_at(lds) + (uint32_t)(KW * 2 * YT + kw * 2 * WT);
        const int yr = tk >> 2, yc = tk & 3;     // dY: rows yr + 32 u, chunk yc of the stage's four
        const int wr = tk >> 4, wc = tk & 15;    // weak block: rows wr + 8 u, chunk wc
        const uint32_t pitch = (uint32_t)lddy * 2u, ylast = (uint32_t)min(M - 1 - m0, 32 * J) * pitch;
        uint32_t yoff[NY];
#pragma unroll
        for (int u = 0; u < NY; ++u) yoff[u] = min((uint32_t)(yr + 32 * u) * pitch, ylast) + 16u * yc;
        const uint32_t woff = (uint32_t)wr * (uint32_t)(L.k * 2) + 2u * (uint32_t)min(c0 - L.kq + 8 * wc, L.k - 8);
        const uint32_t yput = ly + (uint32_t)(yr * 64 + ((yc ^ ((yr >> 2) & 3)) << 4)), wput = lw + (uint32_t)(wr * WP + 16 * wc);
        u4 yv[4][NY], wv[4][4];
        auto first32 = [&](int st) { return RAGGED ? min(32 * st, L.oc - 32) : 32 * st; };   // (as first_row)
        auto fetch = [&](int set, int e) {   // (stages past the last repeat it; both operands are zeroed)
            const int r0 = first32(min(e * KW + kw, nst32 - 1));
#pragma unroll
            for (int u = 0; u < NY; ++u) yv[set][u] = *reinterpret_cast<g_u4*>(sbase(x.xb + 2 * r0) + yoff[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) wv[set][u] = *reinterpret_cast<g_u4*>(sbase(L.weak + (size_t)(r0 + 8 * u) * L.k) + woff);
        };
        auto put = [&](int set, int e, int buf) {
            const int st = e * KW + kw, skip = st < nst32 ? 32 * st - first32(st) : 32;   // rows of the stage before its own
            const bool live = RAGGED ? 8 * yc >= skip : st < nst32;
#pragma unroll
            for (int u = 0; u < NY; ++u) *reinterpret_cast<lds_u4*>(yput + (uint32_t)(u * 2048 + buf * YT)) = live ? yv[set][u] : zero4;
#pragma unroll
            for (int u = 0; u < 4; ++u) *reinterpret_cast<lds_u4*>(wput + (uint32_t)(u * 8 * WP + buf * WT)) = (RAGGED ? wr + 8 * u >= skip : live) ? wv[set][u] : zero4;
        };
#pragma unroll
        for (int e = 0; e < 4; ++e) fetch(e, e);
        put(0, 0, 0);
        fetch(0, 4);
        const int g = lane >> 4, s = lane & 15;
        const uint32_t fa = lw + (uint32_t)((8 * (g >> 1) + (s >> 2)) * WP + 2 * (64 * ow + 16 * (g & 1) + 4 * (s & 3)));
        const uint32_t fb = ly + (uint32_t)(fr * 64), fsw = (uint32_t)((fr >> 2) & 3);
        __syncthreads();
        auto stage = [&](int e, auto set_c) {
            constexpr int SET = decltype(set_c)::value, CUR = SET & 1, NXT = CUR ^ 1, SN = (SET + 1) & 3;
            h8 a[2][2], b[2][J];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {   // rows 16 ks + 8 fk .. + 7 of the stage: chunk 2 ks + fk
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint32_t at = fa + (uint32_t)(16 * ks * WP + 64 * i + CUR * WT);
                    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(size_t)at);
                    const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(size_t)(at + 4 * WP));
                    a[ks][i] = __builtin_bit_cast(h8, s8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w});
                }
#pragma unroll
                for (int j = 0; j < J; ++j) b[ks][j] = *reinterpret_cast<const lds_h8*>(fb + (uint32_t)(j * 2048 + CUR * YT) + (((uint32_t)(2 * ks + fk) ^ fsw) << 4));
            }
            put(SN, e + 1, NXT);
            fetch(SN, e + 5);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks][i], b[ks][j], acc[i][j], 0, 0, 0);
            __syncthreads();
        };
        for (int e = 0; e < turns32; e += 4) {   // (stages past the last multiply zeros)
            stage(e, std::integral_constant<int, 0>{});
            stage(e + 1, std::integral_constant<int, 1>{});
            stage(e + 2, std::integral_constant<int, 2>{});
            stage(e + 3, std::integral_constant<int, 3>{});
        }
    }
    finish<J, KW>(acc, lds, ow, kw, wave, lane, dX, lddx, c0 + 64 * ow, t_n < nq ? L.kq : L.ic, m0, M);
}

inline int dx_tiles(const Layer& L) { return ceil_div(L.kq, 128) + ceil_div(L.k, 128); }

template <int J, int KW>
constexpr int finish_lds() { return 2 * (KW - 1) * 2 * J * 4096; }

template <int J, int KW, int MINW, bool ONCE>
hipError_t launch_fwd(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, hipStream_t s) {
    static bool attr = false;
    constexpr int XL = KW * 2 * 32 * J * 128, LDS_BYTES = XL > finish_lds<J, KW>() ? XL : finish_lds<J, KW>();
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void*)fwd_tile_kernel<J, KW, MINW, ONCE>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int tn = ceil_div(L.oc, 128), tm = ceil_div(M, 32 * J);
    Layer A = L;
    if (A.k == 0) A.weak = reinterpret_cast<const __half*>(A.qweight);   // requests whose result is not used
    fwd_tile_kernel<J, KW, MINW, ONCE><<<xcd_grid(tn * tm), 128 * KW, LDS_BYTES, s>>>(A, X, (int)M, ldx, Y, ldy, tn, tm);
    return hipGetLastError();
}

template <int J, int KW, int MINW, bool ONCE, bool RAGGED>
hipError_t launch_dx(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s, WeakGrad* g) {
    static bool attr = false;
    constexpr int XT = 32 * J * 128, QL = KW * (2 * XT + 2 * 4096 + 2 * (ONCE ? 384 : 256)), WL = KW * 2 * (XT / 2 + 32 * 272);
    constexpr int A = QL > WL ? QL : WL, LDS_BYTES = A > finish_lds<J, KW>() ? A : finish_lds<J, KW>();
    static_assert(LDS_BYTES <= 160 * 1024 && LDS_BYTES >= WG_LDS, "");
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void*)dx_tile_kernel<J, KW, MINW, ONCE, RAGGED>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int tn = dx_tiles(L), tm = ceil_div(M, 32 * J);
    const Strips D = make_strips(g, dY, M, lddy, g ? g->used : 0);
    dx_tile_kernel<J, KW, MINW, ONCE, RAGGED><<<xcd_grid(tn * tm) + D.n, 128 * KW, LDS_BYTES, s>>>(L, dY, (int)M, lddy, dX, lddx, tn, tm, D);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? finish_strips(g, D, s) : e;
}

}  // namespace

// Estimated times (us), fitted to the 7B, 13B and 70B shapes at 97 to 1500 rows; w: workgroups per CU.
namespace {
struct Est {
    double t;
    int j;   // rows per tile / 32
};
Est best_of(double t2, int tiles, int64_t M, double second, double t4) {
    const double w2 = (double)tiles * ceil_div(M, 64) / 256.0, w4 = (double)tiles * ceil_div(M, 128) / 256.0;
    const double f2 = w2 <= 1 ? 1 : (w2 <= 2 ? second + 0.2 * (w2 - 1) : (w2 > 2.2 ? w2 : 2.2)), f4 = w4 <= 1 ? 1 : (double)(int)(w4 + 0.999);
    return t2 * f2 <= t4 * f4 ? Est{t2 * f2, 2} : Est{t4 * f4, 4};
}
Est est_fwd(const Layer& L, int64_t M) {
    const int n = 8 * ceil_div((L.ng + 3) / 4, 2);   // stages of a K group
    return best_of(n * 0.68 + 6, ceil_div(L.oc, 128), M, 1.5, n * 1.05 + 8);
}
Est est_dx(const Layer& L, int64_t M) {
    const int nst = ceil_div(L.oc, 64);
    return best_of(2 * ceil_div(nst, 8) * 1.6 + 7, dx_tiles(L), M, 1.65, 2 * ceil_div(nst, 4) * 1.3 + 8);
}
// share of a 256-row tile's time that a GEMM panel of M rows takes (the forward's panels are cut to the rows)
double panel(int64_t M) {
    const int rows = ceil_div(M, ceil_div(M, 256)), j = rows <= 128 ? 4 : ceil_div(rows, 32);
    return 0.15 + 0.85 * j / 8;
}
// the tiled GEMM without a split: rounds of 256 tiles x stages of 64
double est_gemm(int channels, int64_t M, int stages, double per_stage) {
    const int64_t tiles = (int64_t)ceil_div(channels, 256) * ceil_div(M, 256);
    return (double)((tiles + 255) / 256) * stages * per_stage + 8;
}
// the unsplit forward; a last stage of quantized columns that ends early is converted ahead of its products, and so are the weak columns behind it
double est_gemm_fwd(const Layer& L, int64_t M) {
    const int whole = ceil_div(L.kq, 64) + ceil_div(L.k, 64);
    if (L.kq % 64 == 0) return est_gemm(L.oc, M, whole, 1.15 * panel(M));
    if (!fwd_in_registers(L)) return 2.4 * est_gemm(L.oc, M, whole, 1.15);
    return est_gemm(L.oc, M, L.kq / 64 + 3 * ceil_div(L.ic - L.kq / 64 * 64, 64), 1.3 * panel(M));
}
// the tiled GEMM with every tile split: a share's stages, the partial tiles' traffic (us per slot), the second launch
double est_split(const GemmSplit& p, double fixed, double per_stage) { return fixed + p.stages * per_stage + 0.035 * p.tiles * p.splits; }
// the unsplit input gradient
double est_gemm_dx(const Layer& L, int64_t M) {
    const int stages = ceil_div(L.oc, 64);
    if (!dx_in_registers(L)) return 3.3 * est_gemm(L.ic, M, stages, 1.3);
    return est_gemm(dx_columns(L), M, stages, L.kq % 128 == 0 ? 1.3 : 1.4);
}
}  // namespace

// (32-bit offsets from a panel's first row: 128 rows of up to 2^23 elements.)  The estimate has to be 5 % ahead.  Measured
// with a split workspace, GEMM against this kernel: forward 4096 x 4096, M = 333: 32 us against 26, M = 512: 34 against 29,
// 5120 x 5120, M = 333: 38 against 33, 6144 x 6144, M = 320: 48 against 44; M = 777 on 4096 x 4096: 43 against 40 (GEMM
// kept: too close), 4096 x 11008, M = 333: 56 against 62; input gradient 2560 x 7168, M = 320: 36 against 32.
// Rows whose quantized part is not whole stages are the register GEMM's too, without a split and with a last stage at three times the others' time (with 8 or 16
// weak columns, it against this kernel: 4096 x 4096 at 1500 / 2048 / 4096 86 / 91 / 119 us against 71 / 82 / 161, 5120 x 5120 at 1500 / 2048 106 / 107 against 95 / 139, 11008 x
// 4096 at 333 / 777 68 / 80 against 62 / 105).  Rows of less than a stage leave the LDS-staged GEMM, at 2.4 times the time.
bool fwd_tile_preferred(const Layer& L, int64_t M, int64_t ldx, bool split_ws) {
    if (L.ng <= 0 || M <= 16 || ldx > (QEFT_MAX_DIM >> 1)) return false;
    const GemmSplit p = split_ws ? gemm_fwd_split(L, M) : GemmSplit{1, 0, 0, false};
    if (p.splits > 1) return !p.tail && est_fwd(L, M).t < 0.95 * est_split(p, 11, 1.45 * panel(M));
    return est_fwd(L, M).t < 0.95 * est_gemm_fwd(L, M);
}
// The input gradient.  Against the split the estimate has to be 15 % ahead (its weak tiles run longer than
// estimated), 25 % where the split takes less than 28 us.  Measured, split GEMM against this kernel: 2560 x 7168 at M = 256 / 320 /
// 512 (estimates 0.80 apart) 28.6 / 36.7 / 38.9 us against 24.9 / 33.6 / 34.9, 6144 x 6144 at 320 (0.83) 49.0 against 48.4; the other way
// 4096 x 11008 at 320 (0.88) 57.6 against 59.5, 5120 x 5120 at 333 (0.91) 40.0 against 42.2, 4096 x 4096 at 333 / 512 (0.99) 33.0 / 35.7
// against 34.1 / 35.8.  The short launches would gain 1 to 2 us (2048 x 1152 at 333 / 512 rows, 0.78: 20.3 / 21.1 against 19.0 / 18.9) and
// keep the split's arithmetic, which callers that give the room for it rely on (the one-call backward's test there).  A partial last
// group costs the register GEMM part of a half and its split; estimated at 1.4 us a stage it is taken where it is ahead (forward and backward, us,
// it against this kernel: 4096 x 4096 with 64 weak columns at 777 / 1500 / 2048 121 / 146 / 169 against 91 / 150 / 212, 13824 x 5120 with 64 at 777 / 1500
// 361 / 486 against 339 / 510).  An OC that is no multiple of 64 leaves the GEMM its LDS-staged form, at 3.3 to 4.5 times the time (us, that form against this kernel: 4104 x 4096 at M = 64 / 777 /
// 2048: 292 / 292 / 292 against 35 / 60 / 111; 7184 x 5712 at 64 / 512 / 2048: 572 / 569 / 559 against 53 / 93 / 260).
bool dx_tile_preferred(const Layer& L, int64_t M, int64_t lddy, bool split_ws) {
    if (L.ng <= 0 || M <= 16 || lddy > (QEFT_MAX_DIM >> 1)) return false;
    const GemmSplit p = split_ws ? gemm_dx_split(L, M) : GemmSplit{1, 0, 0, false};
    if (p.splits > 1) {
        const double split = est_split(p, 12, 1.5);
        return !p.tail && est_dx(L, M).t < (split < 28 ? 0.75 : 0.85) * split;
    }
    return est_dx(L, M).t < 0.95 * est_gemm_dx(L, M);
}

// The panel kernel for few rows, where its estimate is 10 % ahead of what would run otherwise (32-bit offsets as above; the small tiles of up to 512 weight rows are
// estimated 1.6 us too long: 488 x 5064 at M = 277 9.1 us there against 10.3).  Of more than 256 rows, splits
// of longer parts than one chunk of 8 stages are as fast (5120 x 5120 with 64 weak columns at 384, forward before it: 72.8 us against 75.7; 4096 x 4096
// at 384, single chunks: 57.8 and 50.5), and short ones keep their arithmetic, as above (2048 x 1152 at 512 rows: 21 us, 12 by panels).
bool dx_panel_preferred(const Layer& L, int64_t M, int64_t lddy, bool split_ws) {
    if (L.ng <= 0 || M <= 16 || lddy > (QEFT_MAX_DIM >> 1)) return false;
    const GemmSplit p = split_ws ? gemm_dx_split(L, M) : GemmSplit{1, 0, 0, false};
    if (p.splits > 1 && M > 256 && (p.tail || p.stages > 8 || est_split(p, 12, 1.5) < 28)) return false;
    const bool tiles = dx_tile_preferred(L, M, lddy, split_ws), split = !tiles && p.splits > 1 && !p.tail;
    const double other = tiles ? est_dx(L, M).t - (L.oc <= 512 ? 1.6 : 0.0) : (split ? est_split(p, 12, 1.5) : est_gemm_dx(L, M));
    return dx_panel_estimate(L, M, split) < 0.9 * other;
}

// A 3-bit layer whose quantized columns are not whole stages (forward: 64 columns) or whole groups (input gradient): its 4-bit copy
// N has the kernels above but not the register GEMM, which its fp16 copy D always has, with a split where there is room.  Either
// way's time is the kernel's estimate and the copy's pass (and, for D, four times the weights to read), fitted to both ways of 190
// random calls of 65 layers at 17 to 4000 rows (7 to 11 % spread).  The estimate has to be 6 % (forward) or 10 % ahead: the choice
// is then slower than the fp16 copy by more than 3 % in 2 of 828 other calls (5 % at most) and within 1 % of the faster way on
// average.  us, 4-bit copy against fp16 copy: input gradient of 8192 x 8192 with 64 weak columns at M = 48 / 200 / 333 / 2048: 73 / 109 /
// 109 / 434 against 91 / 99 / 119 / 277; forward of 13824 x 5120 with 16 at M = 210 / 571 / 1066: 64 / 150 / 234 against 116 / 180 / 243, of
// 5120 x 13824 with 72 at M = 803: 256 against 189.
bool fwd_copy4_preferred(const Layer& N, const Layer& D, int64_t M, int64_t ldx, bool split_n, bool split_d) {
    const bool in_registers = fwd_in_registers(N, M, ldx);
    if ((N.kq % 64 == 0 && in_registers) || (fwd_mid_supported(N, M, ldx) && fwd_mid_preferred(N, M, split_n))) return true;
    const bool tiles = fwd_tile_preferred(N, M, ldx, split_n);
    if (!tiles && !in_registers) return false;
    const GemmSplit p = split_d ? gemm_fwd_split(D, M) : GemmSplit{1, 0, 0, false};
    const double n = (double)N.oc * N.ic / (1 << 20);
    double t16;
    if (D.ic % 64 != 0) t16 = 1.1 * est_gemm(D.oc, M, ceil_div(D.ic, 64), 1.15 * 2.4) + 1.2 * n;
    else if (p.splits > 1 && !p.tail) t16 = 8 + 1.31 * p.stages + 0.09 * p.tiles * p.splits + n;
    else t16 = est_gemm(D.oc, M, D.ic / 64, 1.45 * panel(M)) + 2 + 1.1 * n - (p.tail ? 1.45 * (D.ic / 64 * panel(M) - p.stages) - 10 : 0);
    return (tiles ? est_fwd(N, M).t : est_gemm_fwd(N, M)) + 0.2 * n + 3.5 < 0.94 * t16;
}
bool dx_copy4_preferred(const Layer& N, const Layer& D, int64_t M, int64_t lddy, bool split_n, bool split_d) {
    const bool in_registers = dx_in_registers(N, M, lddy);
    if ((N.kq % 128 == 0 && in_registers) || dx_panel_preferred(N, M, lddy, split_n)) return true;
    const bool tiles = dx_tile_preferred(N, M, lddy, split_n);
    if (!tiles && !in_registers) return false;
    const GemmSplit p = split_d ? gemm_dx_split(D, M) : GemmSplit{1, 0, 0, false};
    const double rounds = (int64_t)dx_tiles(N) * ceil_div(M, 64) > 512 ? 1.25 : 1.0, n = (double)N.oc * N.ic / (1 << 20);   // (a third round of tiles is underestimated)
    // (rows that are not whole stages leave the fp16 copy the LDS-staged form; us, 4-bit copy against it: 4104 x 4096 with 64 weak columns,
    // M = 64 / 777 / 2048: 41 / 67 / 174 against 160 / 166 / 168; 4456 x 14848 at 64 / 184 / 777: 51 / 75 / 229 against 206 / 208 / 218)
    double gemm = D.oc % 64 == 0 ? est_gemm(D.ic, M, D.oc / 64, 1.3) : est_gemm(D.ic, M, ceil_div(D.oc, 64), 2.0);
    if (p.splits > 1) gemm = p.tail ? gemm - D.oc / 64 * 1.3 + p.stages * 1.5 + 12 : est_split(p, 12, 1.5);   // (tail: the last round's tiles only)
    return (tiles ? rounds * est_dx(N, M).t : est_gemm_dx(N, M)) + 0.28 * n + 1.5 < 0.9 * (1.05 * gemm + 0.85 * n);
}

hipError_t fwd_tile(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, hipStream_t s) {
    const bool two = est_fwd(L, M).j == 2;
    if (L.once) return two ? launch_fwd<2, 2, 2, true>(L, X, M, ldx, Y, ldy, s) : launch_fwd<4, 2, 1, true>(L, X, M, ldx, Y, ldy, s);
    return two ? launch_fwd<2, 2, 2, false>(L, X, M, ldx, Y, ldy, s) : launch_fwd<4, 2, 1, false>(L, X, M, ldx, Y, ldy, s);
}
hipError_t dx_tile(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s, WeakGrad* g) {
    using Launch = hipError_t (*)(const Layer&, const __half*, int64_t, int64_t, __half*, int64_t, hipStream_t, WeakGrad*);
#define QEFT_DX(O, R) {launch_dx<2, 4, 2, O, R>, launch_dx<4, 2, 1, O, R>}
    static const Launch table[2][2][2] = {{QEFT_DX(false, false), QEFT_DX(false, true)}, {QEFT_DX(true, false), QEFT_DX(true, true)}};
#undef QEFT_DX
    return table[L.once ? 1 : 0][L.oc % 64 != 0 ? 1 : 0][est_dx(L, M).j == 2 ? 0 : 1](L, dY, M, lddy, dX, lddx, s, g);
}

}  // namespace qeft
