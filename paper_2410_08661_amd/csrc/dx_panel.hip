// Input gradient of 4-bit layers (and 4-bit copies of 3-bit ones) for few rows: fine-tuning steps of some ten to some hundred tokens
// (paper Sec. 3.3).  Tiles of 32 or 64 channels x 32, 64 or 128 rows, so that a layer's few thousand channels occupy the CUs without a workspace: tiles of 128
// channels leave 33 workgroups for 64 rows of a 4096-wide layer, and a split of 256 x 256 tiles multiplies three quarters of padding and sums
// partial tiles in a second launch.
//
// A workgroup's waves take every KS-th stage of 64 weight rows each and share nothing until their partial tiles meet in LDS (fp32, fixed order), so
// the loop has no barrier.  A stage of dY (its rows' 128 bytes, chunks XOR-placed by the row on the way) and of codes (16 or 32 bytes of each of the
// 64 weight rows) goes from memory to a piece of the wave's LDS by itself (buffer loads that write LDS) while the stage before is multiplied.  Codes
// are read with the transposing 4-bit load (see gemm_tile.hip), which leaves a lane the 16 rows of its channel; scales and zero-points vary along the
// contraction and pass through LDS as vectors.  Conversion as there: one rounding of q - z (exact for whole zero-points up to 2048), one of
// the product, or (ONCE) one alone.  A tile is either quantized or weak.
// What bounds it: the requests' way through the L1.  A stage asks for 64 lines of codes, as many of scales and of zero-points, and for its rows' lines of
// dY, whatever the tile's width; hence 64 channels as soon as they leave no CU without work.  (Two stages on their way, with
// parameters by direct loads and the transposing reads in assembly, were no faster: 4096 x 4096 at M = 64 / 128 14.7 / 17.8 us against 13.0 / 16.7.)
// Measured, input and weak gradient in one call, small tiles or split -> here, us: 4096 x 4096 at M = 64 / 128 / 192 26 / 27 / 28.5 -> 14 / 16.5 / 18;
// 4096 x 11008 at 64 30 -> 23; 5120 x 5120 with 64 weak columns at 64 / 128 35.5 -> 19 / 22.5; 2048 x 3000 with 16 at 64 /
// 192 17 -> 8.5 / 10.5; 13824 x 5120 with 16 at 64 to 192 88 -> 60; 3-bit 5120 x 5120 at 64 36 -> 29; 8192 x 1024 at 64 25 -> 16; 520 x 1160 at 128 11 -> 5.5.
// 64 x 128 tiles, with the forward before it: 4096 x 4096 at 300 / 384 / 512 54.8 / 57.8 / 63 -> 47.3 / 50.5 / 60.6; 5120 x 5120 with 64 at 256 62.6 -> 58;
// 13824 x 5120 with 16 at 256 132 -> 124.  There products, conversions and LDS take about a microsecond each of a stage's three; conversions spread between the
// products by scheduling groups gave nothing more.
#include <type_traits>

#include "gemm_common.h"
#include "qeft_internal.h"
#include "weak_strip.h"

namespace qeft {
using namespace gemm;
namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef short s8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) v2i lds_v2i;
typedef __attribute__((address_space(3))) s4 lds_s4;
typedef __attribute__((address_space(3))) u4 lds_u4;
typedef __attribute__((address_space(3))) h8 lds_h8;
typedef __attribute__((address_space(3))) f4 lds_f4;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;

__device__ __forceinline__ uint32_t pack2(float a, float b) { return h2_bits(h2{(_Float16)a, (_Float16)b}); }
template <int N>
__device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

constexpr int DXP_PAR = 384;                                       // - zero * scale or zero, scale of 64 rows
constexpr int dxp_piece(int NI, int J) { return J * 4096 + NI * 1024 + DXP_PAR; }   // a wave's LDS: dY, codes, parameters of a stage; 32 channels of its partial tile

// Tiles of 32 NI channels (of one group: 128 is a multiple of them) x 32 J rows.
template <int NI, int J, bool ONCE>
__global__ __launch_bounds__(512) void dx_panel_kernel(Layer L, const __half* __restrict__ dY, int M, int64_t lddy, __half* __restrict__ dX,
                                                       int64_t lddx, int tiles_n, int tiles_m, Strips D) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    if ((int)blockIdx.x >= (int)gridDim.x - D.n) {   // behind the tiles: a strip of the weak gradient, by four waves
        if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) < 4) weak_grad_strip(lds, (int)blockIdx.x - ((int)gridDim.x - D.n), D);
        return;
    }
    const int lane = threadIdx.x & 63, fr = lane & 31, fk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), KS = blockDim.x >> 6;
    const int per_xcd = (tiles_n * tiles_m + 7) >> 3;
    const int v = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (v >= tiles_n * tiles_m) return;
    const int t_n = v / tiles_m, t_m = v - t_n * tiles_m;   // neighbours on an XCD share their codes
    constexpr int C = 32 * NI;
    const int nq = (L.kq + C - 1) / C;
    const bool weak = t_n >= nq;
    const int c0 = weak ? L.kq + C * (t_n - nq) : C * t_n, m0 = t_m * 32 * J;
    unsigned char* mine = lds + (size_t)wave * dxp_piece(NI, J);
    const uint32_t at = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)mine;
    const auto ybuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half*>(dY + (size_t)m0 * lddy), 0, (int)0xffffffff, 0x00020000);
    const uint32_t ypitch = (uint32_t)lddy * 2u, ylast = (uint32_t)min(M - 1 - m0, 32 * J) * ypitch;
    const h8 zero8 = __builtin_bit_cast(h8, u4{0u, 0u, 0u, 0u});

    f16v acc[NI][J];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    if (!weak) {
        // 64 weight rows of stage st: from 64 st on, the last 64 where OC is no multiple of 64 (what is shared with the stage before counts as zeros,
        // in both operands: an infinite weight counted already may not meet the zeros of dY)
        auto first_row = [&](int st) { return min(64 * st, L.oc - 64); };
        const int nst = (L.oc + 63) >> 6;
        unsigned char* wl = mine + J * 4096;
        const uint32_t at_w = at + J * 4096, at_p = at_w + NI * 1024;
        const uint32_t ycol = 16u * (uint32_t)((lane & 7) ^ (lane >> 3));   // slot lane % 8 of row 8 u + lane / 8 holds chunk slot ^ row % 8
        auto load_y = [&](int r0) {
#pragma unroll
            for (int u = 0; u < 4 * J; ++u)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ybuf, (__attribute__((address_space(3))) void*)(mine + 1024 * u), 16,
                                                         (int)(min((uint32_t)(8 * u + (lane >> 3)) * ypitch, ylast) + ycol), 2 * r0, 0, 0);
        };
        h8 b[4][J];
        auto read_y = [&](int ks, int chunk) {
#pragma unroll
            for (int j = 0; j < J; ++j) b[ks][j] = *reinterpret_cast<const lds_h8*>((size_t)(at + (uint32_t)((32 * j + fr) * 128 + ((chunk ^ (fr & 7)) << 4))));
        };
        const size_t wpitch = (size_t)L.stride * 4, ppitch = (size_t)L.gs * 2;
        const unsigned char* wt = reinterpret_cast<const unsigned char*>(L.qweight) + c0 / 2;
        const unsigned char* st_ = reinterpret_cast<const unsigned char*>(L.scales + c0 / 128) + (size_t)lane * ppitch;
        const unsigned char* zt = reinterpret_cast<const unsigned char*>(L.zeros + c0 / 128) + (size_t)lane * ppitch;
        uint32_t mask = 0x000f000fu, magic = 0x64006400u;
        asm volatile("" : "+v"(mask), "+v"(magic));
        uint32_t sv, zv;
        auto issue = [&](int st) {
            const int r0 = first_row(min(st, nst - 1));
            sv = *reinterpret_cast<const unsigned short*>(st_ + (size_t)r0 * ppitch);
            zv = *reinterpret_cast<const unsigned short*>(zt + (size_t)r0 * ppitch);
            const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(wt + (size_t)r0 * wpitch), 0, (int)0xffffffff, 0x00020000);
#pragma unroll
            for (int u = 0; u < NI; ++u)   // 64 / NI rows of 16 NI bytes
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void*)(wl + 1024 * u), 16,
                                                         (int)((uint32_t)((64 * u + lane) / NI) * (uint32_t)wpitch + 16u * (uint32_t)(lane % NI)), 0, 0, 0);
            load_y(r0);
        };
        issue(wave);
#pragma clang loop unroll(disable)
        for (int st = wave; st < nst; st += KS) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<0>();
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" : "+v"(sv), "+v"(zv));   // (used behind the wait)
            if (first_row(st) + lane < 64 * st) sv = zv = 0u;   // (a weight of zero, whatever its code)
            if constexpr (ONCE) *reinterpret_cast<lds_f32*>((size_t)(at_p + 4u * lane)) = neg_zs(bits_h2(zv).x, bits_h2(sv).x);
            else *reinterpret_cast<lds_u16*>((size_t)(at_p + 2u * lane)) = (uint16_t)zv;
            *reinterpret_cast<lds_u16*>((size_t)(at_p + 256u + 2u * lane)) = (uint16_t)sv;
            wave_lds_fence();
            // k-block ks = (p, h), half fk: rows 32 p + 16 fk + 8 h .. + 7, chunk 4 p + 2 fk + h
            v2i raw[NI][2];
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    raw[i][p] = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lds_v2i*)(size_t)(at_w + (uint32_t)((32 * p + 16 * fk + (lane & 15)) * (16 * NI) + 16 * i + 8 * ((lane >> 4) & 1))));
            u4 sc[4], zp[4];
            f4 nz[4][2];
            constexpr int PH = J == 4 ? 2 : 1;   // (128 rows: fragments of two k-blocks at a time, or registers go to scratch memory)
#pragma unroll
            for (int ph = 0; ph < PH; ++ph) {
#pragma unroll
                for (int ks = 4 * ph / PH; ks < 4 * (ph + 1) / PH; ++ks) {
                    const int chunk = 4 * (ks >> 1) + 2 * fk + (ks & 1);
                    sc[ks] = *reinterpret_cast<const lds_u4*>((size_t)(at_p + 256u + 16u * chunk));
                    if constexpr (ONCE) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) nz[ks][h] = *reinterpret_cast<const lds_f4*>((size_t)(at_p + 32u * chunk + 16u * h));
                    } else
                        zp[ks] = *reinterpret_cast<const lds_u4*>((size_t)(at_p + 16u * chunk));
                    read_y(ks, chunk);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (ph == PH - 1) {
                    wave_lds_fence();
                    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): all is in registers before its place is filled again
                    __builtin_amdgcn_sched_barrier(0);
                    issue(st + KS);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (64 * st + 64 > L.oc) {
#pragma unroll
                    for (int ks = 4 * ph / PH; ks < 4 * (ph + 1) / PH; ++ks) {
                        const bool live = first_row(st) + 8 * (4 * (ks >> 1) + 2 * fk + (ks & 1)) >= 64 * st;
#pragma unroll
                        for (int j = 0; j < J; ++j) b[ks][j] = live ? b[ks][j] : zero8;
                    }
                }
#pragma unroll
                for (int ks = 4 * ph / PH; ks < 4 * (ph + 1) / PH; ++ks)
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const uint32_t w = (uint32_t)raw[i][ks >> 1][ks & 1], w4 = w >> 4;
                        const h2 k1024 = h2{(_Float16)1024.f, (_Float16)1024.f};
                        u4 a;
#pragma unroll
                        for (int p = 0; p < 4; ++p) {   // rows 2 p and 2 p + 1: a byte of the word beside the same byte moved down by a code
                            const h2 q = bits_h2((__builtin_amdgcn_perm(w4, w, 0x0c040c00u + 0x00010001u * (uint32_t)p) & mask) | magic) - k1024;
                            const h2 s = bits_h2(sc[ks][p]);
                            if constexpr (ONCE) {
                                const _Float16 lo = dequant_once_first(q.x, s.x, nz[ks][p >> 1][2 * (p & 1)]);
                                a[p] = h2_bits(h2{lo, dequant_once(q.y, s.y, nz[ks][p >> 1][2 * (p & 1) + 1])});
                            } else
                                a[p] = h2_bits((q - bits_h2(zp[ks][p])) * s);
                        }
#pragma unroll
                        for (int j = 0; j < J; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, a), b[ks][j], acc[i][j], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
        const size_t kpitch = (size_t)L.k * 2;
        // stages of 32 weight rows
        constexpr int CH = 4 * NI, WP = 64 * NI;   // chunks and bytes of a row of the tile's weak columns
        static_assert(J * 2048 + 32 * WP <= dxp_piece(NI, J), "");
        auto first_row = [&](int st) { return min(32 * st, L.oc - 32); };
        const int nst = (L.oc + 31) >> 5;
        unsigned char* wl = mine + J * 2048;
        const uint32_t wcol = 2u * (uint32_t)min(c0 - L.kq + 8 * (lane % CH), L.k - 8);
        const uint32_t ycol = 16u * (uint32_t)((lane & 3) ^ ((lane >> 3) & 3));   // slot lane % 4 of row 16 u + lane / 4 holds chunk slot ^ row / 2 % 4
        auto issue = [&](int st) {
            const int r0 = first_row(min(st, nst - 1));
            const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half*>(L.weak + (size_t)r0 * L.k), 0, (int)0xffffffff, 0x00020000);
#pragma unroll
            for (int u = 0; u < 2 * NI; ++u)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void*)(wl + 1024 * u), 16,
                                                         (int)((uint32_t)((64 * u + lane) / CH) * (uint32_t)kpitch + wcol), 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 2 * J; ++u)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(ybuf, (__attribute__((address_space(3))) void*)(mine + 1024 * u), 16,
                                                         (int)(min((uint32_t)(16 * u + (lane >> 2)) * ypitch, ylast) + ycol), 2 * r0, 0, 0);
        };
        const int g = lane >> 4, s = lane & 15;
        const uint32_t fa = at + J * 2048 + (uint32_t)((8 * (g >> 1) + (s >> 2)) * WP + 2 * (16 * (g & 1) + 4 * (s & 3)));
        issue(wave);
#pragma clang loop unroll(disable)
        for (int st = wave; st < nst; st += KS) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vm<0>();
            __builtin_amdgcn_sched_barrier(0);
            wave_lds_fence();
            h8 a[2][NI], b[2][J];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {   // rows 16 ks + 8 fk .. + 7: chunk 2 ks + fk
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const s4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(size_t)(fa + (uint32_t)(16 * WP * ks + 64 * i)));
                    const s4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(size_t)(fa + (uint32_t)(16 * WP * ks + 64 * i + 4 * WP)));
                    a[ks][i] = __builtin_bit_cast(h8, s8{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w});
                }
#pragma unroll
                for (int j = 0; j < J; ++j) b[ks][j] = *reinterpret_cast<const lds_h8*>((size_t)(at + (uint32_t)((32 * j + fr) * 64 + (((2 * ks + fk) ^ ((fr >> 1) & 3)) << 4))));
            }
            wave_lds_fence();
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_sched_barrier(0);
            issue(st + KS);
            __builtin_amdgcn_sched_barrier(0);
            if (32 * st + 32 > L.oc) {   // both operands: nothing counted already may meet the zeros of the other
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    const bool live = first_row(st) + 8 * (2 * ks + fk) >= 32 * st;
#pragma unroll
                    for (int i = 0; i < NI; ++i) a[ks][i] = live ? a[ks][i] : zero8;
#pragma unroll
                    for (int j = 0; j < J; ++j) b[ks][j] = live ? b[ks][j] : zero8;
                }
            }
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks][i], b[ks][j], acc[i][j], 0, 0, 0);
        }
    }

    // the waves' partial tiles meet in LDS (each in its wave's piece), 32 channels at a time; wave w sums quarters w, w + KS, ...: quarter 4 j + g of
    // lane (fr, fk) is channels 8 g + 4 fk .. + 3 of row 32 j + fr
    wait_vm<0>();   // (requests of a stage past the wave's last)
    const int limit = weak ? L.ic : L.kq;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f4*>(mine + ((4 * j + g) << 10) + 16 * lane) = f4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        __syncthreads();
        for (int q = wave; q < 4 * J; q += KS) {
            f4 y = *reinterpret_cast<const f4*>(lds + (q << 10) + 16 * lane);
            for (int w = 1; w < KS; ++w) {
                const f4 p = *reinterpret_cast<const f4*>(lds + (size_t)w * dxp_piece(NI, J) + (q << 10) + 16 * lane);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] += p[e];
            }
            const int m = m0 + 32 * (q >> 2) + fr, c = c0 + 32 * i + 8 * (q & 3) + 4 * fk;
            if (m < M && c < limit) *reinterpret_cast<u2*>(dX + (size_t)m * lddx + c) = u2{pack2(y[0], y[1]), pack2(y[2], y[3])};
        }
    }
}

inline int dxp_tiles(const Layer& L, int c) { return ceil_div(L.kq, c) + ceil_div(L.k, c); }

template <int NI, int J, bool ONCE>
hipError_t launch(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s, WeakGrad* g) {
    static bool attr = false;
    constexpr int KS = 8, LDS_BYTES = KS * dxp_piece(NI, J) > WG_LDS ? KS * dxp_piece(NI, J) : WG_LDS;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void*)dx_panel_kernel<NI, J, ONCE>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr = true;
    }
    const int tn = dxp_tiles(L, 32 * NI), tm = ceil_div(M, 32 * J);
    const Strips D = make_strips(g, dY, M, lddy, g ? g->used : 0);
    dx_panel_kernel<NI, J, ONCE><<<8 * ceil_div((int64_t)tn * tm, 8) + D.n, 64 * KS, LDS_BYTES, s>>>(L, dY, (int)M, lddy, dX, lddx, tn, tm, D);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? finish_strips(g, D, s) : e;
}

}  // namespace

// Estimated time (us) of the best tile for a call, all of whose workgroups have a CU of their own (more than that and a few of them take a second
// turn: none then).  n: stages of a wave; fitted to the shapes above at 17 to 512 rows, within 15 %.  No less than a stage takes however few tiles share the
// caches, and than many rows bring with them (tall narrow layers and thousands of rows, over 1000 layers looked at, were estimated at half of their time: us, here against
// the small tiles, 6960 x 896 at M = 1182 51 / 38, 10752 x 360 with 72 weak columns at 4087 104 / 81) - except against a split (split), whose partial tiles are rounded to fp16:
// it is the quicker one for some of these layers (24064 x 576 with 64 at 57: 51 / 38), and the tile of a call stays the one that leaves most CUs to the weak gradient's strips.
// Rows of codes about a multiple of 4 KB apart put a
// request's 64 lines on few channels of the L2 (8192 x 8192 with 256 weak columns at M = 64 / 128, forward before it: 40.5 / 42.5 us here, 37.5 / 40 by a split).
namespace {
struct Pick {
    double us, least;
    int tile;   // 0: 32 channels x 32 rows, 1: 32 x 64, 2: 64 x 64, 3: 64 x 128
};
Pick pick(const Layer& L, int64_t M) {
    const double n = ceil_div(ceil_div(L.oc, 64), 8), wide = L.ic / 1024.0;
    const int apart = 4 * L.stride % 4096;
    const bool few = 4 * L.stride > 2048 && (apart < 192 || apart > 4096 - 192);
    const double c0[4] = {0.4, 0.75, 1.2, 2.1}, c1[4] = {0.7, 0.6, 0.55, 0.7}, c2[4] = {0.05, 0.06, 0.065, 0.065};
    const double fixed[4] = {3.0, 3.0, 4.0, 5.3}, stage[4] = {0.9, 1.28, 1.43, 2.17}, rows = 0.6e-6 * (double)M * (L.oc + L.ic);
    Pick best = {1e30, 1e30, 0};
    for (int t = 0; t < 4; ++t) {
        const int64_t wgs = (int64_t)dxp_tiles(L, t >= 2 ? 64 : 32) * ceil_div(M, t == 0 ? 32 : (t == 3 ? 128 : 64));
        const double us = (few ? 8.5 : 3.5) + (few ? 1.1 : 1.0) * n * (c0[t] + c1[t] * (double)wgs / 256 + c2[t] * wide);
        if (wgs <= 256 && us < best.us) best = {us, fixed[t] + n * stage[t] + rows, t};
    }
    return best;
}
}  // namespace
double dx_panel_estimate(const Layer& L, int64_t M, bool split) {
    const Pick p = pick(L, M);
    return split || p.us > p.least ? p.us : p.least;
}
hipError_t dx_panel(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s, WeakGrad* g) {
    using Launch = hipError_t (*)(const Layer&, const __half*, int64_t, int64_t, __half*, int64_t, hipStream_t, WeakGrad*);
    static const Launch table[4][2] = {{launch<1, 1, false>, launch<1, 1, true>}, {launch<1, 2, false>, launch<1, 2, true>}, {launch<2, 2, false>, launch<2, 2, true>}, {launch<2, 4, false>, launch<2, 4, true>}};
    return table[pick(L, M).tile][L.once ? 1 : 0](L, dY, M, lddy, dX, lddx, s, g);
}

}  // namespace qeft
