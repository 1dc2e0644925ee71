// Prefill / fine-tune path (paper Sec. 3.3): the large-M products of the fused layer as tiled
// fp16 MFMA GEMMs with fp32 accumulation (tiling and LDS layout: gemm_common.h).
//
//   forward    Y [M][OC]  = X  . W^T            contraction over IC (quantized part, then weak block)
//   backward   dX[M][IC]  = dY . W              contraction over OC, through the full mixed weight
//   weak grad  dW[OC][k]  = dY^T . X[:, weak]   contraction over the M tokens (Eq. 5, weak block only)
//
// Two families of kernels live here.
//   * gemm_fwd_rega_kernel / gemm_dx_rega_kernel: the 4-bit codes are dequantized straight into the
//     MFMA operand registers of the wave that multiplies them; LDS carries only the fp16 activation
//     tile (and, for dX, the raw codes transposed at 16-bit granularity).  Waves are stacked
//     along the weight rows (64 rows x 256 tokens each) so that every code is converted once;
//     software-pipelined in steps of one MFMA with static LDS / global addressing.  The forward
//     kernel can also split the K range over workgroups (few output tiles: fp16 partial tiles in a
//     workspace, summed by splitk_reduce_kernel).  Described at each kernel.
//   * gemm_fwd_kernel / gemm_dx_kernel: producer threads dequantize into an fp16 weight tile in
//     LDS.  Simpler, LDS-bound, kept for the shapes the register kernels do not take.
//
// Dequantization: codes become exact fp16 numbers by or-ing exponent bits onto masked nibbles
// (two codes per instruction): 1024 + q for a nibble at bits 0..3 of a half, 64 + q for one at
// bits 4..7 (mantissa bit 4 then weighs 1); then ((h - base) - z) * s in packed fp16: the first
// subtraction is exact, the second rounds once (exact for integer zero-points), the product once.
// The nibbles of a word come out in the order (0,4)(1,5)(2,6)(3,7); in the forward kernels the
// activations of quantized stages are permuted to match.
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "gemm_common.h"
#include "weak_strip.h"

namespace qeft {
namespace {

using namespace gemm;

// ======================================================================================= forward
struct FwdStage {
    u4 qa[2];        // quantized stage: 4 code words of rows r and r+128
    uint32_t sz[2];  // their (scale, zero-point)
    RowLoader wk;    // weak stage: fp16 weights
    RowLoader x;     // activations
};

__global__ __launch_bounds__(256) void gemm_fwd_kernel(Layer L, const __half* __restrict__ X, int M, int64_t ldx,
                                                       __half* __restrict__ Y, int64_t ldy, int tiles_oc) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int tile = xcd_tile(tiles_oc * ((M + BT - 1) / BT));
    if (tile < 0) return;
    int t_oc, t_m;
    tile_coords(tile, tiles_oc, (M + BT - 1) / BT, t_oc, t_m);
    const int oc0 = t_oc * BT, m0 = t_m * BT;
    const int nq_st = (L.kq + BK - 1) / BK, nw_st = (L.k + BK - 1) / BK, nst = nq_st + nw_st;
    const Consts cst = make_consts();

    const int ar = tid >> 1, ah = tid & 1;  // quantized A: rows ar and ar+128, half ah of the stage's 8 words
    const int arow0 = min(oc0 + ar, L.oc - 1), arow1 = min(oc0 + ar + 128, L.oc - 1);

    auto load_stage = [&](FwdStage& s, int st) {
        if (st < nq_st) {
            s.qa[0] = ld16(L.qweight + (size_t)arow0 * L.stride + 8 * st + 4 * ah);
            s.qa[1] = ld16(L.qweight + (size_t)arow1 * L.stride + 8 * st + 4 * ah);
            const int g = st >> 1;
            s.sz[0] = (uint32_t)__half_as_ushort(L.scales[(size_t)arow0 * L.gs + g]) |
                      ((uint32_t)__half_as_ushort(L.zeros[(size_t)arow0 * L.gs + g]) << 16);
            s.sz[1] = (uint32_t)__half_as_ushort(L.scales[(size_t)arow1 * L.gs + g]) |
                      ((uint32_t)__half_as_ushort(L.zeros[(size_t)arow1 * L.gs + g]) << 16);
            s.x.load(X, ldx, m0, M, BK * st, L.kq, tid, false);   // columns past Kq belong to the weak block
        } else {
            const int c0 = BK * (st - nq_st);
            s.wk.load(L.weak, L.k, oc0, L.oc, c0, L.k, tid, true);
            s.x.load(X + L.kq, ldx, m0, M, c0, L.k, tid, false);
        }
    };
    auto store_stage = [&](const FwdStage& s, int st, unsigned char* sA, unsigned char* sB) {
        if (st < nq_st) {
#pragma unroll
            for (int rr = 0; rr < 2; ++rr) {
                const _Float16 sc = bits_h2(s.sz[rr])[0], zp = bits_h2(s.sz[rr])[1];
                const h2 s2 = h2{sc, sc}, z2 = h2{zp, zp};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = s.qa[rr][i];
                    u4 r;
#pragma unroll
                    for (int p = 0; p < 4; ++p) r[p] = dequant_pair(((w >> (4 * p)) & cst.mask) | cst.magic, z2, s2);
                    *reinterpret_cast<u4*>(sA + tile_off(ar + 128 * rr, 4 * ah + i)) = r;
                }
            }
            s.x.store(sB, tid, true);
        } else {
            s.wk.store(sA, tid, false);
            s.x.store(sB, tid, false);
        }
    };

    f16v acc[4][4];
    zero_acc(acc);
    FwdStage stg;
    load_stage(stg, 0);
    store_stage(stg, 0, lds, lds + 2 * TILE_BYTES);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        const int cur = st & 1;
        if (st + 1 < nst) load_stage(stg, st + 1);
        compute_stage(lds + cur * TILE_BYTES, lds + (2 + cur) * TILE_BYTES, acc, wm, wn, lane);
        if (st + 1 < nst) store_stage(stg, st + 1, lds + (cur ^ 1) * TILE_BYTES, lds + (2 + (cur ^ 1)) * TILE_BYTES);
        __syncthreads();
    }
    store_f16(acc, Y, ldy, oc0, L.oc, m0, M, wm, wn, lane);
}

// ------------------------------------------------------------------------- forward, weights in registers
// One packed word is 8 consecutive columns of one output channel - exactly the 8 k-values one
// lane feeds into a 32x32x16 MFMA as its A operand.  So the quantized weights never touch LDS:
// lane (fr, fk) of a wave fetches, for each of its 32-row blocks, the 16 bytes holding words
// 4 fk .. 4 fk + 3 of its row for the stage, and dequantizes word ks straight into the A fragment
// of k-block ks (the k-blocks of a stage are numbered so that this works: block ks covers the
// columns of words ks and 4 + ks; the X fragments are read from LDS chunk 4 fk + ks to match).
// LDS holds only the activations (two 32 KB buffers).
//  * 4 waves stacked along the output channels, each 64 channels x 256 tokens (2 x 8 MFMA tiles):
//    every word is converted by exactly one wave, and each wave reads all eight X fragments of a
//    k-block - per MFMA the same LDS traffic as a kernel that reads both operands from LDS.
//    Conversion is what limits the kernel: measured on gfx950, a wave hides about four vector
//    instructions behind each 32x32x16 MFMA and pays in full for any more.
//  * a stage is 64 steps of one MFMA; a scheduling barrier after every step pins its share of
//    the other work: even steps read one X fragment of the next k-block and (first half of the
//    stage) permute and store half an X chunk of the next stage; odd steps convert one pair of
//    codes of the next k-block.
//  * one workgroup barrier per stage, after step 47; the last k-block reads the next stage's
//    first X fragments behind it.
//  * scales / zero-points: 8 bytes (four groups) per row and array every 8 stages, latched into a
//    packed register per row when the group changes.
struct RegConsts {
    uint32_t m0, m1, g0, g1;
};
__device__ __forceinline__ RegConsts make_reg_consts() {
    RegConsts c{0x000f000fu, 0x00f000f0u, 0x64006400u, 0x54005400u};
    asm volatile("" : "+v"(c.m0), "+v"(c.m1), "+v"(c.g0), "+v"(c.g1));
    return c;
}
// Pair P of a word (P = 0..3 -> codes (c0,c4) (c1,c5) (c2,c6) (c3,c7)); w8 = w >> 8.  Codes at bits
// 0..3 of a half become 1024 + q, codes at bits 4..7 become 64 + q (exponent chosen so that
// mantissa bit 4 weighs 1); (h - base) is exact, then - z and * s as everywhere else.
template <int P>
__device__ __forceinline__ uint32_t dequant_pair_of(uint32_t w, uint32_t w8, h2 z2, h2 s2, const RegConsts& c) {
    const h2 b0 = h2{(_Float16)1024.f, (_Float16)1024.f}, b1 = h2{(_Float16)64.f, (_Float16)64.f};
    const uint32_t src = P < 2 ? w : w8;
    const uint32_t h = (P & 1) ? ((src & c.m1) | c.g1) : ((src & c.m0) | c.g0);
    return h2_bits(((bits_h2(h) - ((P & 1) ? b1 : b0)) - z2) * s2);
}
__device__ __forceinline__ h8 dequant_word(uint32_t w, uint32_t zs, const RegConsts& c) {
    const h2 v = bits_h2(zs);
    const h2 z2 = h2{v.x, v.x}, s2 = h2{v.y, v.y};
    const uint32_t w8 = w >> 8;
    const u4 r = u4{dequant_pair_of<0>(w, w8, z2, s2, c), dequant_pair_of<1>(w, w8, z2, s2, c),
                    dequant_pair_of<2>(w, w8, z2, s2, c), dequant_pair_of<3>(w, w8, z2, s2, c)};
    return __builtin_bit_cast(h8, r);
}

constexpr int REGA_LDS = 4 * TILE_BYTES;   // X0 X1 and one tile for the weak block's weights; 32 KB per wave in the epilogue

// fp16 epilogue of a 64 (i) x 256 (j) wave tile through 32 KB of LDS of the wave's own: rows j of
// 128 bytes, 16-byte chunks XOR-swizzled with j, then 16-byte global stores (128 contiguous bytes
// per row).  QUADS = false: accumulator tile t_i row 8 g + 4 fk + e is i = 32 t_i + row; QUADS =
// true (the input-gradient kernel's quantized halves): it is i = 4 (row % 16) + t_i + 2 (row / 16).
// i0 and ni multiples of 8, out rows 16-byte aligned.  No barrier: one wave, in-order LDS.
template <bool QUADS, int JT>
__device__ __forceinline__ void store_f16_lds(const f16v (&acc)[2][JT], unsigned char* stage, __half* out, int64_t ld,
                                                     int i0, int ni, int j0, int nj, int lane) {
    const int fr = lane & 31, fk = lane >> 5;
    auto pack = [](float a, float b) { return h2_bits(h2{(_Float16)a, (_Float16)b}); };
#pragma unroll
    for (int tj = 0; tj < JT; ++tj) {
        unsigned char* row = stage + (tj * 32 + fr) * 128;
        const int sw = fr & 7;
        if (!QUADS) {
#pragma unroll
            for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<u2*>(row + (((4 * ti + g) ^ sw) << 4) + 8 * fk) =
                        u2{pack(acc[ti][tj][4 * g + 0], acc[ti][tj][4 * g + 1]), pack(acc[ti][tj][4 * g + 2], acc[ti][tj][4 * g + 3])};
        } else {
            // channels 4 c .. 4 c + 3, c = 8 g0 + 4 fk + e: (t_i, g) = (0, g0) (1, g0) (0, g0 + 2) (1, g0 + 2)
#pragma unroll
            for (int g0 = 0; g0 < 2; ++g0)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<u2*>(row + (((4 * g0 + 2 * fk + (e >> 1)) ^ sw) << 4) + 8 * (e & 1)) =
                        u2{pack(acc[0][tj][4 * g0 + e], acc[1][tj][4 * g0 + e]), pack(acc[0][tj][4 * (g0 + 2) + e], acc[1][tj][4 * (g0 + 2) + e])};
        }
    }
    const int c = lane & 7, r8 = lane >> 3;
    const int i = i0 + 8 * c;
#pragma unroll 8
    for (int it = 0; it < 4 * JT; ++it) {
        const int r = 8 * it + r8;
        const u4 v = *reinterpret_cast<const u4*>(stage + r * 128 + ((c ^ (r & 7)) << 4));
        if (j0 + r < nj && i < ni) *reinterpret_cast<u4*>(out + (size_t)(j0 + r) * ld + i) = v;
    }
}

// K split (splits > 1): a workgroup (tile, sp) of a split tile multiplies the quantized stages [sp * sps, (sp + 1) * sps)
// only - the last split also the weak block - and stores its partial tile as fp16 into its slot of `part` (BT rows of
// BT halves); splitk_reduce_kernel adds the partials.  Either every tile is split (launches with too few tiles to occupy
// the CUs) or only those of the last, partly filled round (split_tile).  sps is a multiple of 8 stages, so every split
// starts on a boundary of the four-group parameter fetches.
// J: panels of 32 J rows.  The last panel of 256 rows may be mostly empty (333 rows: two panels, 65 % of them rows); the
// launch then keeps its panels and tiles and takes the smallest J that covers the rows in as many equal panels.
template <int... Ts, class F>
__device__ __forceinline__ void each_step(std::integer_sequence<int, Ts...>, F&& f) {
    (f(std::integral_constant<int, Ts>{}), ...);
}

template <int J, bool ONCE>
__global__ __launch_bounds__(256) void gemm_fwd_rega_kernel(Layer L, const __half* __restrict__ X, int M, int64_t ldx,
                                                            __half* __restrict__ Y, int64_t ldy, int tiles_oc, int wide_stores,
                                                            int splits, int sps, int tail_first, __half* __restrict__ part) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int PM = 32 * J;
    const int tiles_m = (M + PM - 1) / PM, tiles_all = tiles_oc * tiles_m;
    int tile, sp, slot;
    if (!split_tile(tiles_all, tail_first, splits, tile, sp, slot)) return;
    int t_oc, t_m;
    tile_coords(tile, tiles_oc, tiles_m, t_oc, t_m);
    const int oc0 = t_oc * BT, m0 = t_m * PM;
    const bool is_split = slot >= 0;
    const bool last_split = !is_split || sp == splits - 1;
    const int s_first = sp * sps;                                      // first stage of this workgroup
    // a layer without quantized columns (the fp16 copy of a 3-bit layer) is split along its weak stages instead:
    // a split is then the layer whose weak block starts 64 s_first columns further on
    const bool weak_split = is_split && L.kq == 0;
    const int nq = weak_split ? 0 : (is_split ? min(sps, L.kq / BK - s_first) : L.kq / BK);
    // weak stages: whole 64-column stages take the direct path below (A fragments straight from the fp16
    // block), a ragged block the LDS-staged stages at the end
    const int nwf = weak_split ? min(sps, L.k / BK - s_first) : ((L.kq % BK == 0 && L.k % BK == 0 && last_split) ? L.k / BK : 0);
    const int ns = nq + nwf;
    if (is_split) {
        // the epilogue addresses Y[m][oc] with absolute indices: point it at the slot's (m0, oc0)
        Y = part + (size_t)slot * (BT * BT) - ((size_t)m0 * BT + oc0);
        ldy = BT;
        wide_stores = 1;
    }
    const RegConsts cst = make_reg_consts();
    using lds_u4 = __attribute__((address_space(3))) u4;
    using lds_h8 = __attribute__((address_space(3))) h8;
    using gptr = const __attribute__((address_space(1))) char*;
    using g_u4 = const __attribute__((address_space(1))) u4;
    using g_u2 = const __attribute__((address_space(1))) u2;
    const int fr = lane & 31, fk = lane >> 5;

    // global addresses: wave-uniform 64-bit base (scalar registers) + 32-bit lane offset
    // (a stage is 32 bytes of codes per row, half a group = one byte of each parameter array per row, 128 bytes of X per token)
    const char* wt = reinterpret_cast<const char*>(L.qweight + (size_t)oc0 * L.stride) + 32 * s_first;
    const char* st_ = reinterpret_cast<const char*>(L.scales + (size_t)oc0 * L.gs) + s_first;
    const char* zt = reinterpret_cast<const char*>(L.zeros + (size_t)oc0 * L.gs) + s_first;
    const char* xt = reinterpret_cast<const char*>(X + (size_t)m0 * ldx) + 2 * BK * s_first;
    const char* wk = reinterpret_cast<const char*>(L.weak + (size_t)oc0 * L.k) + (weak_split ? 2 * BK * s_first : 0);
    uint32_t aoff[2], szoff[2], xoff[J];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t row = (uint32_t)min(wave * 64 + 32 * i + fr, L.oc - 1 - oc0);
        aoff[i] = (row * (uint32_t)L.stride + 4u * fk) * 4u;
        szoff[i] = row * (uint32_t)L.gs * 2u;
    }
    const int xr = tid >> 3, xc = tid & 7;   // X chunk u of this thread: tile row xr + 32 u, chunk column xc
#pragma unroll
    for (int u = 0; u < J; ++u) xoff[u] = ((uint32_t)min(xr + 32 * u, M - 1 - m0) * (uint32_t)ldx + 8u * xc) * 2u;
    auto sbase = [](const char* p) {
        asm volatile("" : "+s"(p));
        return (gptr)p;
    };

    // LDS addresses: base register + compile-time offset.  Rows 64 apart share the swizzle, rows
    // 32 apart differ in bit 2 of it, so chunk writes use two bases and fragment reads one base
    // per XOR constant.
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
    uint32_t xw[2] = {lds0 + (uint32_t)tile_off(xr, xc), lds0 + (uint32_t)tile_off(xr + 32, xc)};
    uint32_t fb[8];
    {
        const uint32_t base = (uint32_t)((4 * fk) ^ (fr & 7) ^ (fr >> 3));
#pragma unroll
        for (int x = 0; x < 8; ++x) fb[x] = lds0 + (uint32_t)fr * 128u + ((base ^ (uint32_t)x) << 4);
    }

    u4 araw[2][2];      // codes: set = stage parity, row block i; word ks of the stage in component ks
    u4 xv[J];           // X of the stage after the current one
    u2 szs[2], szz[2];  // scales / zero-points of four consecutive groups, per row block
    uint32_t lsz[2];    // latched group: zero-point in the low half, scale in the high half
    float nzs[2];       // ... and - zero-point * scale (ONCE)
    _Float16 lo[8];     // first halves of the pairs (ONCE)
    u4 afr[2][2];       // A fragments as packed halfs, written one pair at a time
    h8 bfr[2][J];
    uint32_t cq[8];     // the conversion pipeline: one register per pair of the k-block being converted
    uint32_t w8[2];     // word >> 8 per row block
    u4 px;              // the X chunk being permuted
    auto load_a = [&](int set, int i, int st) { araw[set][i] = *reinterpret_cast<g_u4*>(sbase(wt + 32 * st) + aoff[i]); };
    auto load_x = [&](int u, int st) { xv[u] = *reinterpret_cast<g_u4*>(sbase(xt + 2 * BK * st) + xoff[u]); };
    auto load_sz = [&](int g4) {   // groups g4 .. g4 + 3 (g4 a multiple of 4; the arrays are padded to a multiple of 8 groups)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            szs[i] = *reinterpret_cast<g_u2*>(sbase(st_ + 2 * g4) + szoff[i]);
            szz[i] = *reinterpret_cast<g_u2*>(sbase(zt + 2 * g4) + szoff[i]);
        }
    };
    auto latch = [&](int g) {
        const int sh = 16 * (g & 3);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint64_t s64 = ((uint64_t)szs[i].y << 32) | szs[i].x, z64 = ((uint64_t)szz[i].y << 32) | szz[i].x;
            lsz[i] = ((uint32_t)(z64 >> sh) & 0xffffu) | ((uint32_t)(s64 >> sh) << 16);
            if constexpr (ONCE) nzs[i] = neg_zs(bits_h2(lsz[i]).x, bits_h2(lsz[i]).y);
        }
    };
    auto put_x = [&](int u, int buf) {
        *reinterpret_cast<lds_u4*>(xw[u & 1] + (uint32_t)((u >> 1) * 8192 + buf * TILE_BYTES)) = permute_x(xv[u]);
    };
    auto read_b = [&](int set, int j, int buf, int kn) {
        bfr[set][j] = *reinterpret_cast<const lds_h8*>(fb[kn ^ (4 * (j & 1))] + (uint32_t)(j * 4096 + buf * TILE_BYTES));
    };

    f16v acc[2][J];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // the columns behind the whole stages, as fp16 through LDS: the weak block where it is ragged, and ahead of it the rest of the quantized
    // columns where those are (n_rest, whole words).  Chunk u of this thread is tile row xr + 32 u, 16-byte column xc of the stage
    // (columns past the end read the row's last 8 and are zeroed when stored).  Such a stage costs about three of the others, once; before, these layers had
    // the small tiles at any size: 4096 x 11008 with 16 weak columns at 4096 rows 396 -> 304 us, 8192 x 8192 at 1500 225 -> 189, 13824 x 5120 at 777 141 -> 114
    const int c_tail = L.kq / BK * BK, n_rest = L.kq - c_tail, n_tail = L.ic - c_tail;
    const int nw = (nwf || !last_split) ? 0 : (n_tail + BK - 1) / BK;
    const u4 zero4 = u4{0u, 0u, 0u, 0u};
    u4 wa[8], wb[J];
    auto load_weak = [&](int w) {
        const int col = min(BK * w + 8 * xc, n_tail - 8);
#pragma unroll
        for (int u = 0; u < J; ++u) wb[u] = ld16(X + (size_t)min(m0 + xr + 32 * u, M - 1) * ldx + c_tail + col);
        if (col < n_rest) {
            uint32_t word[8];
            _Float16 sc[8], zp[8];
            const _Float16 *ps = reinterpret_cast<const _Float16*>(L.scales) + (c_tail >> 7), *pz = reinterpret_cast<const _Float16*>(L.zeros) + (c_tail >> 7);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const size_t row = (size_t)min(oc0 + xr + 32 * u, L.oc - 1);
                word[u] = L.qweight[row * L.stride + ((c_tail + col) >> 3)];
                sc[u] = ps[row * L.gs];
                zp[u] = pz[row * L.gs];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float nz = ONCE ? neg_zs(zp[u], sc[u]) : 0.f;
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const h2 q = h2{(_Float16)(float)((word[u] >> (8 * p)) & 15u), (_Float16)(float)((word[u] >> (8 * p + 4)) & 15u)};
                    wa[u][p] = h2_bits(ONCE ? h2{dequant_once(q.x, sc[u], nz), dequant_once(q.y, sc[u], nz)} : (q - h2{zp[u], zp[u]}) * h2{sc[u], sc[u]});
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) wa[u] = ld16(L.weak + (size_t)min(oc0 + xr + 32 * u, L.oc - 1) * L.k + (col - n_rest));
        }
    };

    if (nq > 0) {
        const int s1 = min(1, nq - 1), s1x = min(1, ns - 1);
#pragma unroll
        for (int u = 0; u < J; ++u) load_x(u, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) load_a(0, i, 0);
        load_sz(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) load_a(1, i, s1);
#pragma unroll
        for (int u = 0; u < J; ++u) {
            put_x(u, 0);
            load_x(u, s1x);
        }
        latch(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const h8 raw = __builtin_bit_cast(h8, dequant_word(araw[0][i].x, ONCE ? 0x3c000000u : lsz[i], cst));   // (z = 0, s = 1: the codes)
            h8 w = raw;
            if constexpr (ONCE) {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = dequant_once(raw[e], bits_h2(lsz[i]).y, nzs[i]);
            }
            afr[0][i] = __builtin_bit_cast(u4, w);
        }
        // the pipeline finishes "the previous k-block's last pair" in its first two steps: hand it
        // that pair of the first k-block in the state it expects (masked and rebased)
        cq[7] = h2_bits(bits_h2(((araw[0][1].x >> 8) & cst.m1) | cst.g1) - h2{(_Float16)64.f, (_Float16)64.f});
#pragma unroll
        for (int e = 0; e < 7; ++e) cq[e] = 0u;
        w8[0] = w8[1] = 0u;
        px = u4{0u, 0u, 0u, 0u};
        __syncthreads();
#pragma unroll
        for (int j = 0; j < J; ++j) read_b(0, j, 0, 0);

        // stage st: X in buffer CUR, codes in set CUR
        auto stage = [&](int st, auto cur_c) {
            constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1, S = 2 * J;   // S: steps per k-block
            const int sl = min(st + 2, nq - 1), slx = min(st + 2, ns - 1);   // the activations run on into the weak stages
            // keep "base + constant" from being hoisted out of the loop into a register per constant:
            // inside the stage it folds into the instruction's offset field
            asm volatile("" : "+v"(fb[0]), "+v"(fb[1]), "+v"(fb[2]), "+v"(fb[3]), "+v"(fb[4]), "+v"(fb[5]), "+v"(fb[6]), "+v"(fb[7]));
            asm volatile("" : "+v"(xw[0]), "+v"(xw[1]), "+v"(aoff[0]), "+v"(aoff[1]));
#pragma unroll
            for (int u = 0; u < J; ++u) asm volatile("" : "+v"(xoff[u]));
            auto step = [&](auto t_c) {
                constexpr int T = decltype(t_c)::value, ks = T / S, t = T % S, i = t / J, j = t % J, kn = (ks + 1) & 3;
                constexpr int SRC = ks < 3 ? CUR : NXT;   // where the next k-block comes from
                if (T == 3 * S + (J == 8 ? 2 : 0) && CUR == 1) {
                    // the pairs converted from here on belong to the next stage, which opens a new group:
                    // latch it, and when it was the last of the four held in registers fetch the
                    // following four (needed two stages from now)
                    const int g = min(st + 1, nq - 1) >> 1;
                    latch(g);
                    if ((g & 3) == 3 && 2 * (g + 1) < nq) load_sz(g + 1);
                }
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, afr[ks & 1][i]), bfr[ks & 1][j], acc[i][j], 0, 0, 0);
                // Conversion of the next k-block's two words, software-pipelined so that no step holds
                // two dependent instructions: pair a = t / 2 is masked at step 2a, rebased at 2a + 1,
                // has its zero-point subtracted at 2a + 2 and is scaled at 2a + 3 (ONCE: its first half, its second half;
                // the last pair finishes in the first two steps of the following k-block, before its row block is used).
                const h2 b0 = h2{(_Float16)1024.f, (_Float16)1024.f}, b1 = h2{(_Float16)64.f, (_Float16)64.f};
                if constexpr (J == 8) {
                    constexpr int a = t >> 1, ap = (a + 7) & 7;   // this step's young pair, and the one two steps older
                    constexpr int aci = a >> 2, apci = ap >> 2;
                    const h2 zs_old = bits_h2(lsz[apci]);
                    if ((t & 1) == 0) {
                        const uint32_t w = araw[SRC][aci][kn];
                        if ((a & 3) == 1) w8[aci] = w >> 8;
                        const uint32_t src = (a & 3) < 2 ? w : w8[aci];
                        cq[a] = (a & 1) ? ((src & cst.m1) | cst.g1) : ((src & cst.m0) | cst.g0);
                        if constexpr (ONCE) lo[ap] = dequant_once_first(bits_h2(cq[ap]).x, zs_old.y, nzs[apci]);
                        else cq[ap] = h2_bits(bits_h2(cq[ap]) - h2{zs_old.x, zs_old.x});
                    } else {
                        cq[a] = h2_bits(bits_h2(cq[a]) - ((a & 1) ? b1 : b0));
                        // pair 7 of the previous conversion belongs to the k-block now being multiplied
                        afr[a == 0 ? (ks & 1) : (kn & 1)][apci][ap & 3] =
                            h2_bits(ONCE ? h2{lo[ap], dequant_once(bits_h2(cq[ap]).y, zs_old.y, nzs[apci])} : bits_h2(cq[ap]) * h2{zs_old.y, zs_old.y});
                    }
                } else {   // fewer steps: the four operations of the eight pairs one after the other, evenly over the k-block
#pragma unroll
                    for (int o = 32 * t / S; o < 32 * (t + 1) / S; ++o) {
                        const int pr = o & 7, ci = pr >> 2;
                        const h2 zs = bits_h2(lsz[ci]);
                        if (o < 8) {
                            const uint32_t w = araw[SRC][ci][kn];
                            if ((pr & 3) == 2) w8[ci] = w >> 8;
                            const uint32_t src = (pr & 3) < 2 ? w : w8[ci];
                            cq[pr] = (pr & 1) ? ((src & cst.m1) | cst.g1) : ((src & cst.m0) | cst.g0);
                        } else if (o < 16) cq[pr] = h2_bits(bits_h2(cq[pr]) - ((pr & 1) ? b1 : b0));
                        else if (o < 24) {
                            if constexpr (ONCE) lo[pr] = dequant_once_first(bits_h2(cq[pr]).x, zs.y, nzs[ci]);
                            else cq[pr] = h2_bits(bits_h2(cq[pr]) - h2{zs.x, zs.x});
                        } else
                            afr[kn & 1][ci][pr & 3] =
                                h2_bits(ONCE ? h2{lo[pr], dequant_once(bits_h2(cq[pr]).y, zs.y, nzs[ci])} : bits_h2(cq[pr]) * h2{zs.y, zs.y});
                    }
                }
                if ((t & 1) == 0) {
                    read_b(kn & 1, t >> 1, SRC, kn);
                    if constexpr (T >= 4 && T <= 4 * J && (T & 3) == 0) {   // the chunk permuted in the two odd steps before
                        constexpr int u = (T >> 2) - 1;
                        *reinterpret_cast<lds_u4*>(xw[u & 1] + (uint32_t)((u >> 1) * 8192 + NXT * TILE_BYTES)) = px;
                    }
                } else {
                    if constexpr (T < 4 * J) {   // X chunk u of the next stage: half of the permutation per odd step
                        constexpr int u = T >> 2;
                        if ((T & 2) == 0) {
                            px.x = __builtin_amdgcn_perm(xv[u].z, xv[u].x, 0x05040100u);
                            px.y = __builtin_amdgcn_perm(xv[u].z, xv[u].x, 0x07060302u);
                        } else {
                            px.z = __builtin_amdgcn_perm(xv[u].w, xv[u].y, 0x05040100u);
                            px.w = __builtin_amdgcn_perm(xv[u].w, xv[u].y, 0x07060302u);
                            load_x(u, slx);
                        }
                    }
                    if (ks == 3 && j == J - 1 && J % 2 == 0) load_a(CUR, i, sl);
                }
                if (ks == 3 && j == J - 1 && J % 2 == 1) load_a(CUR, i, sl);   // (an odd J puts these steps on either parity)
                if (T == 3 * S - 1) __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            };
            each_step(std::make_integer_sequence<int, 4 * S>{}, step);
        };
        int st = 0;
        for (; st + 1 < nq; st += 2) {
            stage(st, std::integral_constant<int, 0>{});
            stage(st + 1, std::integral_constant<int, 1>{});
        }
        if (nq & 1) stage(st, std::integral_constant<int, 0>{});
        if (nwf == 0) __syncthreads();
    }

    // ---- weak block, whole stages: the same 64-step stage without a conversion ------------------------
    // The activation pipeline above simply runs on (the weak columns follow the quantized ones in X), so the
    // tiles keep the chunk order of the 4-bit conversion.  A lane's A fragment of k-block kn is 16 contiguous
    // bytes of its row of the fp16 block: it is fetched one stage ahead into the register of the k-block just
    // consumed and brought into the tiles' chunk order by four byte permutes while the previous k-block is
    // multiplied.  No weight passes through LDS.
    if (nwf > 0) {
        u4 wfr[2][4];      // [row block][k-block]
        uint32_t woff[2];  // (computed here: the stage loop above has no register to carry them)
#pragma unroll
        for (int i = 0; i < 2; ++i)
            woff[i] = ((uint32_t)min(wave * 64 + 32 * i + fr, L.oc - 1 - oc0) * (uint32_t)L.k + 32u * fk) * 2u;
        auto load_w = [&](int i, int kn, uint32_t off) {   // scalar base + lane offset + immediate
            wfr[i][kn] = *reinterpret_cast<g_u4*>(((gptr)wk + off) + 16 * kn);
        };
        auto order_w = [&](int i, int kn, int dst) {   // A fragment in the tiles' chunk order
            const u4 v = wfr[i][kn];
            afr[dst][i].x = __builtin_amdgcn_perm(v.z, v.x, 0x05040100u);
            afr[dst][i].y = __builtin_amdgcn_perm(v.z, v.x, 0x07060302u);
            afr[dst][i].z = __builtin_amdgcn_perm(v.w, v.y, 0x05040100u);
            afr[dst][i].w = __builtin_amdgcn_perm(v.w, v.y, 0x07060302u);
        };
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int kn = 0; kn < 4; ++kn) load_w(i, kn, woff[i]);
        if (nq == 0) {   // no stage has run yet: start the activation pipeline here
            const int s1x = min(1, ns - 1);
#pragma unroll
            for (int u = 0; u < J; ++u) load_x(u, 0);
#pragma unroll
            for (int u = 0; u < J; ++u) {
                put_x(u, 0);
                load_x(u, s1x);
            }
            px = u4{0u, 0u, 0u, 0u};
            __syncthreads();
#pragma unroll
            for (int j = 0; j < J; ++j) read_b(0, j, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            order_w(i, 0, 0);
            load_w(i, 0, woff[i] + (uint32_t)(2 * BK * min(1, nwf - 1)));
        }

        // weak stage w: X in buffer CUR
        auto wstage = [&](int w, auto cur_c) {
            constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1, S = 2 * J;   // S: steps per k-block
            const int slx = min(nq + w + 2, ns - 1);
            uint32_t wo1[2], wo2[2];   // this thread's rows in the next stage and in the one after
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                wo1[i] = woff[i] + (uint32_t)(2 * BK * min(w + 1, nwf - 1));
                wo2[i] = woff[i] + (uint32_t)(2 * BK * min(w + 2, nwf - 1));
            }
            asm volatile("" : "+v"(fb[0]), "+v"(fb[1]), "+v"(fb[2]), "+v"(fb[3]), "+v"(fb[4]), "+v"(fb[5]), "+v"(fb[6]), "+v"(fb[7]));
            asm volatile("" : "+v"(xw[0]), "+v"(xw[1]), "+v"(wo1[0]), "+v"(wo1[1]), "+v"(wo2[0]), "+v"(wo2[1]));
#pragma unroll
            for (int u = 0; u < J; ++u) asm volatile("" : "+v"(xoff[u]));
            auto step = [&](auto t_c) {
                constexpr int T = decltype(t_c)::value, ks = T / S, t = T % S, i = t / J, j = t % J, kn = (ks + 1) & 3;
                constexpr int SRC = ks < 3 ? CUR : NXT;          // tile of the next k-block
                constexpr int O0 = J == 8 ? 4 : 2, L0 = J == 8 ? 10 : (J > 4 ? 8 : 6), L1 = J == 8 ? 12 : (J > 5 ? 10 : (J > 4 ? 9 : 7));
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, afr[ks & 1][i]), bfr[ks & 1][j], acc[i][j], 0, 0, 0);
                if ((t & 1) == 0) {
                    read_b(kn & 1, t >> 1, SRC, kn);
                    if constexpr (T >= 4 && T <= 4 * J && (T & 3) == 0) {   // the chunk permuted in the two odd steps before
                        constexpr int u = (T >> 2) - 1;
                        *reinterpret_cast<lds_u4*>(xw[u & 1] + (uint32_t)((u >> 1) * 8192 + NXT * TILE_BYTES)) = px;
                    }
                    // the next k-block's fragments (k-block 0 of the next stage behind the last one), one row block
                    // per step; each register is then refilled with the same k-block one stage on
                    if (t == O0) order_w(0, kn, kn & 1);
                    if (t == O0 + 2) order_w(1, kn, kn & 1);
                    if (t == L0) load_w(0, kn, ks < 3 ? wo1[0] : wo2[0]);
                    if (t == L1) load_w(1, kn, ks < 3 ? wo1[1] : wo2[1]);
                } else {
                    if (t == L1) load_w(1, kn, ks < 3 ? wo1[1] : wo2[1]);
                    if constexpr (T < 4 * J) {   // X chunk u of the next stage: half of the permutation per odd step
                        constexpr int u = T >> 2;
                        if ((T & 2) == 0) {
                            px.x = __builtin_amdgcn_perm(xv[u].z, xv[u].x, 0x05040100u);
                            px.y = __builtin_amdgcn_perm(xv[u].z, xv[u].x, 0x07060302u);
                        } else {
                            px.z = __builtin_amdgcn_perm(xv[u].w, xv[u].y, 0x05040100u);
                            px.w = __builtin_amdgcn_perm(xv[u].w, xv[u].y, 0x07060302u);
                            load_x(u, slx);
                        }
                    }
                }
                if (T == 3 * S - 1) __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            };
            each_step(std::make_integer_sequence<int, 4 * S>{}, step);
        };
        int w = 0;
        if (nq & 1) {   // the first weak stage sits in tile 1
            wstage(0, std::integral_constant<int, 1>{});
            w = 1;
        }
        for (; w + 1 < nwf; w += 2) {
            wstage(w, std::integral_constant<int, 0>{});
            wstage(w + 1, std::integral_constant<int, 1>{});
        }
        if (w < nwf) wstage(w, std::integral_constant<int, 0>{});
        __syncthreads();
    }
    if (nw > 0) load_weak(0);

    // ---- weak block: plain fp16 stages with both operands through LDS -------------------------------
    // Stage w sits in tiles (w & 1) [X] and 2 + (w & 1) [weights].  While its four k-blocks are
    // multiplied (fragments read one block ahead), stage w + 1 moves from the registers into the
    // other pair of tiles, a quarter per k-block, and stage w + 2 is fetched.
    auto store_weak = [&](int w, int q) {   // chunks 2 q, 2 q + 1 of this thread, of stage w
        unsigned char* sB = lds + (w & 1) * TILE_BYTES;
        unsigned char* sA = lds + (2 + (w & 1)) * TILE_BYTES;
        const bool ok = BK * w + 8 * xc < n_tail;
#pragma unroll
        for (int u = 2 * q; u < 2 * q + 2; ++u) {
            *reinterpret_cast<u4*>(sA + tile_off(xr + 32 * u, xc)) = ok ? wa[u] : zero4;
            if (u < J) *reinterpret_cast<u4*>(sB + tile_off(xr + 32 * u, xc)) = ok ? wb[u < J ? u : 0] : zero4;
        }
    };
    if (nw > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) store_weak(0, q);
        if (nw > 1) load_weak(1);
        __syncthreads();
    }
    for (int w = 0; w < nw; ++w) {
        const unsigned char* sB = lds + (w & 1) * TILE_BYTES;
        const unsigned char* sA = lds + (2 + (w & 1)) * TILE_BYTES;
        FragsT<2, J> f[2];
        load_frags_t<2, J>(f[0], sA, sB, wave * 64, 0, lane, 0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) load_frags_t<2, J>(f[(ks + 1) & 1], sA, sB, wave * 64, 0, lane, ks + 1);
            mfma_block_t<2, J>(f[ks & 1], acc);
            if (w + 1 < nw) store_weak(w + 1, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (w + 2 < nw) load_weak(w + 2);
        if (w + 1 < nw) __syncthreads();
    }
    if (wide_stores) __syncthreads();   // the epilogue reuses the tiles
    if (wide_stores)
        store_f16_lds<false, J>(acc, lds + wave * TILE_BYTES, Y, ldy, oc0 + wave * 64, L.oc, m0, M, lane);
    else
        store_f16_t<2, J>(acc, Y, ldy, oc0 + wave * 64, L.oc, m0, M, lane);
}

// ======================================================================================= backward dX
// A[i = ic][k = oc] = W[oc][ic], B[j = m][k = oc] = dY[m][oc].  Thread (ko = t / 32, io = t % 32)
// produces the 8 x 8 block of 8 weight rows x one word column (8 input channels).
struct DxStage {
    uint32_t qw[8];   // quantized columns: the word of each of the 8 rows
    uint32_t sz[8];   // (scale, zero-point) of each row for this column's group
    ColLoader wk;     // weak columns: 8 rows x 8 fp16
    RowLoader dy;
};

__global__ __launch_bounds__(256) void gemm_dx_kernel(Layer L, const __half* __restrict__ dY, int M, int64_t lddy,
                                                      __half* __restrict__ dX, int64_t lddx, int tiles_ic, int ic_start) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int tile = xcd_tile(tiles_ic * ((M + BT - 1) / BT));
    if (tile < 0) return;
    int t_ic, t_m;
    tile_coords(tile, tiles_ic, (M + BT - 1) / BT, t_ic, t_m);
    const int ic0 = ic_start + t_ic * BT, m0 = t_m * BT;
    const int nst = (L.oc + BK - 1) / BK;
    const Consts cst = make_consts();

    const int ko = tid >> 5, io = tid & 31;
    const int ic = ic0 + 8 * io;          // first of this thread's 8 input channels
    const bool quant = ic < L.kq;         // Kq is a multiple of 8: a block is all quantized or all weak
    const int wcol = ic >> 3, grp = ic >> 7;

    auto load_stage = [&](DxStage& s, int st) {
        const int k0 = BK * st;
        if (quant) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int row = min(k0 + 8 * ko + e, L.oc - 1);   // rows past OC meet zero columns of dY
                s.qw[e] = L.qweight[(size_t)row * L.stride + wcol];
                s.sz[e] = (uint32_t)__half_as_ushort(L.scales[(size_t)row * L.gs + grp]) |
                          ((uint32_t)__half_as_ushort(L.zeros[(size_t)row * L.gs + grp]) << 16);
            }
        } else {
            s.wk.load(L.weak, L.k, k0, L.oc, ic0 - L.kq, L.k, tid);
        }
        s.dy.load(dY, lddy, m0, M, k0, L.oc, tid, false);
    };
    auto store_stage = [&](const DxStage& s, unsigned char* sA, unsigned char* sB) {
        if (quant) {
            u4 out[8];
#pragma unroll
            for (int p = 0; p < 4; ++p) {   // rows 2p and 2p+1 side by side
                const h2 s2 = h2{bits_h2(s.sz[2 * p])[0], bits_h2(s.sz[2 * p + 1])[0]};
                const h2 z2 = h2{bits_h2(s.sz[2 * p])[1], bits_h2(s.sz[2 * p + 1])[1]};
#pragma unroll
                for (int b = 0; b < 4; ++b) {   // byte b of both words: codes 2b and 2b+1
                    const uint32_t sel = 0x0c000c00u | ((4u + b) << 16) | (uint32_t)b;
                    const uint32_t t = __builtin_amdgcn_perm(s.qw[2 * p + 1], s.qw[2 * p], sel);
                    out[2 * b][p] = dequant_pair((t & cst.mask) | cst.magic, z2, s2);
                    out[2 * b + 1][p] = dequant_pair(((t >> 4) & cst.mask) | cst.magic, z2, s2);
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) *reinterpret_cast<u4*>(sA + tile_off(8 * io + j, ko)) = out[j];
        } else {
            s.wk.store(sA, tid);
        }
        s.dy.store(sB, tid, false);
    };

    f16v acc[4][4];
    zero_acc(acc);
    DxStage stg;
    load_stage(stg, 0);
    store_stage(stg, lds, lds + 2 * TILE_BYTES);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        const int cur = st & 1;
        if (st + 1 < nst) load_stage(stg, st + 1);
        compute_stage(lds + cur * TILE_BYTES, lds + (2 + cur) * TILE_BYTES, acc, wm, wn, lane);
        if (st + 1 < nst) store_stage(stg, lds + (cur ^ 1) * TILE_BYTES, lds + (2 + (cur ^ 1)) * TILE_BYTES);
        __syncthreads();
    }
    store_f16(acc, dX, lddx, ic0, L.ic, m0, M, wm, wn, lane);
}

// ------------------------------------------------------------------------- backward dX, weights in registers
// C[i = ic][j = m] = sum_oc W[oc][ic] dY[m][oc].  The A operand of a 32x32x16 MFMA wants, per
// lane, 8 consecutive k = 8 consecutive weight ROWS of one input channel, while the stored
// matrices run along the channels.  Both kinds of weight therefore pass through LDS as "lines":
// one line holds, for the stage's 64 rows, one 16-bit column of the stored matrix, two rows to a
// 32-bit word - so 16 bytes of a line are 8 consecutive rows, paired along k.
//  * Quantized half (128 channels = 16 word columns, one group): line (W, h) is the 16-bit half h
//    of word column W, i.e. raw 4-bit codes, an eighth of the fp16 tile.  Lane (fr, fk) reads rows
//    16 ks + 8 fk .. + 7 of line (fr / 2, fr % 2): four registers whose nibble i (of both halves)
//    is channel 4 fr + i.  A fragment i is then one mask-and-or per register (no permute), and a
//    lane's four accumulators for fixed (row, column) are four consecutive channels of dX.
//    Scales and zero-points vary along k here: they are staged as fp16 vectors per row.
//  * Weak half (128 fp16 channels): a line is simply one channel; 16 bytes of it are an A fragment
//    as it stands.  Fragment i of lane fr is channel fr + 32 i.
// Everything else is the forward kernel's pipeline: 4 waves of 128 x 128, 16 slots of four MFMAs
// per stage, quantized fragments converted three slots ahead, dY staged through LDS unchanged,
// one barrier per stage after slot 11.  A tile is 256 channels = two halves, each quantized or
// weak; the two waves that own a half follow its kind.  Where Kq is no multiple of 128 the last quantized half ends early - its
// words past the row's are clamped, its channels past Kq not stored - and the weak halves begin behind it: the tiles cover
// dx_columns(L) columns, the weak channels moved up by as many as are missing there.  (That share of a half is multiplied for nothing; a half of both kinds
// would give its two waves different code.  Forward and backward,
// us, small tiles -> here: 8192 x 8192 with 64 weak columns at M = 1500 540 -> 387; 5120 x 5120 with 64 at 2048 271 -> 228; 4096 x 11008 with 16 at 777 235 -> 187.)
// Requires dx_in_registers(L).
constexpr int DX_LINE = 144;                      // 64 rows x 2 bytes + 16: consecutive lines 4 banks apart
constexpr int DX_HALF = 128 * DX_LINE;            // lines of one half (a quantized half uses the first 32)
constexpr int DX_LINES = 2 * DX_HALF;
constexpr int DX_SZ = 2 * 2 * 64 * 2;             // [half][zero, scale][row] fp16
constexpr int DX_SZ_ONCE = 2 * (64 * 4 + 64 * 2); // [half][- zero * scale fp32, scale fp16][row]
constexpr int DX_LINE_BASE = 2 * TILE_BYTES;      // dY0 dY1 | lines0 lines1 | sz0 sz1
constexpr int DX_SZ_BASE = DX_LINE_BASE + 2 * DX_LINES;
constexpr int DX_LDS = DX_SZ_BASE + 2 * DX_SZ_ONCE;

// H0, H1: kinds of the tile's two halves: 0 quantized, 1 weak.  ONCE: see dequant_once; the rows' - zero * scale in fp32 then take the
// zero-points' place (four registers, and a third LDS read per k-block).
template <int H0, int H1, bool ONCE>
__device__ __forceinline__ void dx_tile(const Layer& L, const __half* __restrict__ dY, int M, int64_t lddy,
                                        __half* __restrict__ dX, int64_t lddx, int ic0, int m0, unsigned char* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave >> 1, lb = wave & 1;   // the tile half this wave works in, and which 64 channels of it
    const int nst = L.oc / BK;
    const RegConsts cst = make_reg_consts();
    using lds_u4 = __attribute__((address_space(3))) u4;
    using lds_u32 = __attribute__((address_space(3))) uint32_t;
    using lds_u16 = __attribute__((address_space(3))) unsigned short;
    using lds_f32 = __attribute__((address_space(3))) float;
    using lds_f4 = __attribute__((address_space(3))) f4;
    using lds_h8 = __attribute__((address_space(3))) h8;
    using gptr = const __attribute__((address_space(1))) char*;
    using g_u4 = const __attribute__((address_space(1))) u4;
    using g_u16 = const __attribute__((address_space(1))) unsigned short;
    constexpr bool ANYQ = H0 == 0 || H1 == 0;
    constexpr int NW = 2 * (H0 + H1);   // weak items per thread: (row pair, 8 channels) blocks
    const int fr = lane & 31, fk = lane >> 5;
    auto sbase = [](const char* p) {
        asm volatile("" : "+s"(p));
        return (gptr)p;
    };

    // ---- producers: global addresses (wave-uniform 64-bit base + 32-bit lane offset) ---------------
    // dY: chunk u of this thread is tile row xr + 32 u, chunk column xc
    const int xr = tid >> 3, xc = tid & 7;
    const char* dyt = reinterpret_cast<const char*>(dY + (size_t)m0 * lddy);
    uint32_t dyoff[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) dyoff[u] = ((uint32_t)min(xr + 32 * u, M - 1 - m0) * (uint32_t)lddy + 8u * xc) * 2u;
    // codes: rows 2 rp, 2 rp + 1 of the stage, word columns 4 xc .. 4 xc + 3 of the tile, i.e. of half
    // xc / 4 (columns past the stored row are clamped; such channels are never stored)
    const int rp = tid >> 3;
    const bool code_thread = H0 == 0 && (H1 == 0 || xc < 4);
    uint32_t coff = ((uint32_t)(2 * rp) * (uint32_t)L.stride + (uint32_t)min((ic0 >> 3) + 4 * xc, L.stride - 4)) * 4u;
    const char* wt = reinterpret_cast<const char*>(L.qweight);
    const size_t wstage = (size_t)BK * L.stride * 4, wrow = (size_t)L.stride * 4;
    // scales / zero-points: thread (row = tid % 64, half = tid / 64 % 2) of waves 0 and 1
    const bool sz_wave = H0 == 0 && (H1 == 0 ? wave < 2 : wave < 1);
    uint32_t szoff = ((uint32_t)(tid & 63) * (uint32_t)L.gs + (uint32_t)min((ic0 >> 7) + ((tid >> 6) & 1), L.gs - 1)) * 2u;
    const char* st_ = reinterpret_cast<const char*>(L.scales);
    const char* zt = reinterpret_cast<const char*>(L.zeros);
    const size_t szstage = (size_t)BK * L.gs * 2;
    // weak: item n of this thread is rows 2 rp, 2 rp + 1 x channels 8 c .. 8 c + 7 of a weak half,
    // c = xc + 8 (n % 2); the halves in the order they are weak (channel blocks past k are clamped)
    uint32_t woff[NW > 0 ? NW : 1];
    const char* wkt = reinterpret_cast<const char*>(L.weak);
    const size_t wkstage = (size_t)BK * L.k * 2, wkrow = (size_t)L.k * 2;
#pragma unroll
    for (int n = 0; n < NW; ++n) {
        const int half = (H0 == 1) ? n / 2 : 1;
        const int kc = ic0 + 128 * half - ((L.kq + 127) & ~127) + 8 * (xc + 8 * (n & 1));   // (the weak halves begin at a multiple of 128)
        woff[n] = ((uint32_t)(2 * rp) * (uint32_t)L.k + (uint32_t)max(min(kc, L.k - 8), 0)) * 2u;
    }

    // ---- LDS addresses: base register + compile-time offset ---------------------------------------
    const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
    uint32_t xw[2] = {lds0 + (uint32_t)tile_off(xr, xc), lds0 + (uint32_t)tile_off(xr + 32, xc)};
    uint32_t fb[4];   // dY fragments, indexed by (XOR constant) / 2
#pragma unroll
    for (int x = 0; x < 4; ++x)
        fb[x] = lds0 + (uint32_t)fr * 128u + ((((uint32_t)(fk ^ (fr & 7) ^ (fr >> 3))) ^ (2u * x)) << 4);
    // lines: the 16-byte chunk t of a line (rows 8 t .. 8 t + 7) sits at slot t ^ (line / 8 % 8), so that
    // the eight threads that write one row pair into eight different line groups spread over the banks
    const uint32_t lw = (((uint32_t)((rp >> 2) ^ xc)) << 4) + (uint32_t)(rp & 3) * 4u;   // position of row pair rp, line group xc (mod 8)
    uint32_t cwr = lds0 + DX_LINE_BASE + (uint32_t)(xc >> 2) * DX_HALF + (uint32_t)(8 * (xc & 3)) * DX_LINE + lw;
    uint32_t wwr[NW > 0 ? NW : 1];
#pragma unroll
    for (int n = 0; n < NW; ++n) {
        const int half = (H0 == 1) ? n / 2 : 1;
        wwr[n] = lds0 + DX_LINE_BASE + (uint32_t)half * DX_HALF + (uint32_t)(8 * (xc + 8 * (n & 1))) * DX_LINE + lw;
    }
    constexpr uint32_t SZ = ONCE ? DX_SZ_ONCE : DX_SZ, SC = ONCE ? 256 : 128;   // bytes of a buffer; where a half's scales start
    uint32_t szw = lds0 + DX_SZ_BASE + (uint32_t)((tid >> 6) & 1) * (SZ / 2) + (uint32_t)(tid & 63) * 2u;
    const uint32_t szw4 = szw + (uint32_t)((tid & 63) * 2);

    u4 dyv[8];            // dY of the stage after the current one
    u4 cw0, cw1;          // its code words (two rows)
    unsigned short sv, zv;
    u4 ww[NW > 0 ? NW : 1][2];   // its weak blocks (two rows each)
    auto load_dy = [&](int u, int st) { dyv[u] = *reinterpret_cast<g_u4*>(sbase(dyt + 2 * BK * st) + dyoff[u]); };
    auto load_codes = [&](int st) {
        if (code_thread) {
            cw0 = *reinterpret_cast<g_u4*>(sbase(wt + st * wstage) + coff);
            cw1 = *reinterpret_cast<g_u4*>(sbase(wt + st * wstage + wrow) + coff);
        }
    };
    auto load_sz = [&](int st) {
        if (sz_wave) {
            sv = *reinterpret_cast<g_u16*>(sbase(st_ + st * szstage) + szoff);
            zv = *reinterpret_cast<g_u16*>(sbase(zt + st * szstage) + szoff);
        }
    };
    auto load_weak = [&](int n, int st) {
        ww[n][0] = *reinterpret_cast<g_u4*>(sbase(wkt + st * wkstage) + woff[n]);
        ww[n][1] = *reinterpret_cast<g_u4*>(sbase(wkt + st * wkstage + wkrow) + woff[n]);
    };
    auto put_dy = [&](int u, int buf) {
        *reinterpret_cast<lds_u4*>(xw[u & 1] + (uint32_t)((u >> 1) * 8192 + buf * TILE_BYTES)) = dyv[u];
    };
    auto put_codes = [&](int q, int buf) {   // word column 4 xc + q: low halves of both rows, high halves
        if (code_thread) {
            *reinterpret_cast<lds_u32*>(cwr + (uint32_t)((2 * q) * DX_LINE + buf * DX_LINES)) =
                __builtin_amdgcn_perm(cw1[q], cw0[q], 0x05040100u);
            *reinterpret_cast<lds_u32*>(cwr + (uint32_t)((2 * q + 1) * DX_LINE + buf * DX_LINES)) =
                __builtin_amdgcn_perm(cw1[q], cw0[q], 0x07060302u);
        }
    };
    auto put_sz = [&](int buf) {
        if (sz_wave) {
            if constexpr (ONCE)
                *reinterpret_cast<lds_f32*>(szw4 + (uint32_t)(buf * SZ)) =
                    neg_zs(__builtin_bit_cast(_Float16, zv), __builtin_bit_cast(_Float16, sv));
            else
                *reinterpret_cast<lds_u16*>(szw + (uint32_t)(buf * SZ)) = zv;
            *reinterpret_cast<lds_u16*>(szw + (uint32_t)(SC + buf * SZ)) = sv;
        }
    };
    auto put_weak = [&](int n, int buf) {    // channel e of the block: rows 2 rp | 2 rp + 1
#pragma unroll
        for (int e = 0; e < 8; ++e)
            *reinterpret_cast<lds_u32*>(wwr[n] + (uint32_t)(e * DX_LINE + buf * DX_LINES)) =
                __builtin_amdgcn_perm(ww[n][1][e >> 1], ww[n][0][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
    };

    f16v acc[2][8];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // ---- stage 0 into buffer 0, stage 1 into the registers ------------------------------------------
    {
        const int s1 = min(1, nst - 1);
#pragma unroll
        for (int u = 0; u < 8; ++u) load_dy(u, 0);
        if (ANYQ) {
            load_codes(0);
            load_sz(0);
        }
#pragma unroll
        for (int n = 0; n < NW; ++n) load_weak(n, 0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            put_dy(u, 0);
            load_dy(u, s1);
        }
        if (ANYQ) {
#pragma unroll
            for (int q = 0; q < 4; ++q) put_codes(q, 0);
            load_codes(s1);
            put_sz(0);
            load_sz(s1);
        }
#pragma unroll
        for (int n = 0; n < NW; ++n) {
            put_weak(n, 0);
            load_weak(n, s1);
        }
        __syncthreads();
    }

    // this slot's share of staging stage st+1 into buffer NXT and fetching stage sl
    auto produce = [&](auto s_c, auto nxt_c, int sl) {
        constexpr int S = decltype(s_c)::value, NXT = decltype(nxt_c)::value;
        if (S < 8) {
            put_dy(S, NXT);
            load_dy(S, sl);
        }
        if (ANYQ) {
            if (S == 8) {
                put_codes(0, NXT);
                put_codes(1, NXT);
            } else if (S == 9) {
                put_codes(2, NXT);
                put_codes(3, NXT);
                load_codes(sl);
            } else if (S == 10) {
                put_sz(NXT);
                load_sz(sl);
            }
        }
        constexpr int n = S - (12 - NW);   // weak items in the last slots before the barrier
        if (NW > 0 && n >= 0 && n < NW) {
            put_weak(n, NXT);
            load_weak(n, sl);
        }
    };
    auto protect = [&]() {   // keep "base + constant" out of loop-invariant registers: it folds into the offset field
        asm volatile("" : "+v"(fb[0]), "+v"(fb[1]), "+v"(fb[2]), "+v"(fb[3]), "+v"(xw[0]), "+v"(xw[1]), "+v"(cwr), "+v"(szw), "+v"(coff), "+v"(szoff));
        asm volatile("" : "+v"(dyoff[0]), "+v"(dyoff[1]), "+v"(dyoff[2]), "+v"(dyoff[3]), "+v"(dyoff[4]), "+v"(dyoff[5]), "+v"(dyoff[6]), "+v"(dyoff[7]));
#pragma unroll
        for (int n = 0; n < NW; ++n) asm volatile("" : "+v"(woff[n]), "+v"(wwr[n]));
    };
    // ---- consumers: wave w owns 64 channels (block lb = w % 2 of half w / 2) x all 256 tokens --------
    // A stage is 64 steps of one MFMA (k-block T / 16, channel fragment T / 8 % 2, token fragment
    // T % 8) with a scheduling barrier after each: even steps read one dY fragment of the next
    // k-block, odd steps 4 S + 1 carry the producers' slot S, and the conversion of the next
    // k-block's codes is spread so that no step holds two dependent instructions.
    h8 bfr[2][8];
    u4 afr[2][2];   // A fragments of a k-block (set = block parity), as packed halfs
    auto read_b = [&](int set, int j, int buf, int kn) {
        bfr[set][j] = *reinterpret_cast<const lds_h8*>(fb[kn ^ (2 * (j & 1))] + (uint32_t)(j * 4096 + buf * TILE_BYTES));
    };
    const int icw = ic0 + 128 * half + 64 * lb;
    auto mfma_step = [&](auto t_c) {
        constexpr int T = decltype(t_c)::value, ks = T >> 4, i = (T >> 3) & 1, j = T & 7;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8, afr[ks & 1][i]), bfr[ks & 1][j], acc[i][j], 0, 0, 0);
    };
    auto produce_step = [&](auto t_c, auto nxt_c, int sl) {
        constexpr int T = decltype(t_c)::value;
        if ((T & 3) == 1 && T < 48) produce(std::integral_constant<int, (T >> 2)>{}, nxt_c, sl);
    };
    auto run_stages = [&](auto&& stage) {
        int st = 0;
        for (; st + 1 < nst; st += 2) {
            stage(st, std::integral_constant<int, 0>{});
            stage(st + 1, std::integral_constant<int, 1>{});
        }
        if (nst & 1) stage(st, std::integral_constant<int, 0>{});
        __syncthreads();   // every wave is done with the staging buffers
    };
#define QEFT_STEPS8(F, B)                                                                                        \
    F(std::integral_constant<int, (B) + 0>{}); F(std::integral_constant<int, (B) + 1>{});                       \
    F(std::integral_constant<int, (B) + 2>{}); F(std::integral_constant<int, (B) + 3>{});                       \
    F(std::integral_constant<int, (B) + 4>{}); F(std::integral_constant<int, (B) + 5>{});                       \
    F(std::integral_constant<int, (B) + 6>{}); F(std::integral_constant<int, (B) + 7>{});
#define QEFT_STEPS64(F)                                                                                          \
    QEFT_STEPS8(F, 0) QEFT_STEPS8(F, 8) QEFT_STEPS8(F, 16) QEFT_STEPS8(F, 24) QEFT_STEPS8(F, 32) QEFT_STEPS8(F, 40) \
    QEFT_STEPS8(F, 48) QEFT_STEPS8(F, 56)

    // ---- a wave in a quantized half ---------------------------------------------------------------------
    // Lane fr reads line 16 lb + fr % 16 (both lanes fr and fr + 16 the same one) and takes nibble
    // t + 2 (fr / 16) of its 16-bit words for fragment t: after a per-lane shift by 0 or 8 bits,
    // fragment 0 is the nibble at bits 0..3 (as 1024 + q) and fragment 1 the one at bits 4..7 (as
    // 64 + q), the two positions that lie inside the fp16 mantissa.  Row fr of fragment t is channel
    // 4 (fr % 16) + t + 2 (fr / 16) of the wave's 64, so a lane's accumulators (0, g, e) (1, g, e)
    // (0, g + 2, e) (1, g + 2, e) are four consecutive channels.
    auto run_quant = [&]() {
        uint32_t crd[4];  // code lines, indexed by k-block
        {
            const int ln = 16 * lb + (fr & 15);
            const int cl = (ln >> 3) + 4 * half;   // the line's group in the chunk swizzle: its writer's xc
#pragma unroll
            for (int kn = 0; kn < 4; ++kn)
                crd[kn] = lds0 + DX_LINE_BASE + (uint32_t)half * DX_HALF + (uint32_t)ln * DX_LINE + ((uint32_t)((fk ^ cl) ^ (2 * kn)) << 4);
        }
        uint32_t szr = lds0 + DX_SZ_BASE + (uint32_t)half * (SZ / 2) + 16u * fk;
        uint32_t nsh = 8u * (uint32_t)(fr >> 4);
        u4 cf;            // code words of the k-block being converted: register p = rows 2p | 2p+1
        u4 cfs;           // ... shifted to this lane's nibbles
        h8 zf, sf;        // zero-points and scales of its 8 rows
        f4 nzs[2];        // - zero-point * scale (ONCE)
        _Float16 lo[8];   // first halves of the pairs (ONCE)
        uint32_t cq[8];   // the conversion pipeline, one register per pair
        auto read_codes = [&](int buf, int kn) {
            cf = *reinterpret_cast<const lds_u4*>(crd[kn] + (uint32_t)(buf * DX_LINES));
            if constexpr (ONCE) {
#pragma unroll
                for (int h = 0; h < 2; ++h) nzs[h] = *reinterpret_cast<const lds_f4*>(szr + 16u * fk + (uint32_t)(64 * kn + 16 * h + buf * SZ));
            } else
                zf = *reinterpret_cast<const lds_h8*>(szr + (uint32_t)(32 * kn + buf * SZ));
            sf = *reinterpret_cast<const lds_h8*>(szr + (uint32_t)(SC + 32 * kn + buf * SZ));
        };
        const h2 b0 = h2{(_Float16)1024.f, (_Float16)1024.f}, b1 = h2{(_Float16)64.f, (_Float16)64.f};
        // pair a = 4 t + p (fragment t, register p) goes through: mask, rebase, zero-point, scale
        auto cv_mask = [&](auto a_c) {
            constexpr int a = decltype(a_c)::value;
            cq[a] = (a < 4) ? ((cfs[a & 3] & cst.m0) | cst.g0) : ((cfs[a & 3] & cst.m1) | cst.g1);
        };
        auto cv_base = [&](auto a_c) {
            constexpr int a = decltype(a_c)::value;
            cq[a] = h2_bits(bits_h2(cq[a]) - (a < 4 ? b0 : b1));
        };
        auto cv_zero = [&](auto a_c) {
            constexpr int a = decltype(a_c)::value, p = a & 3;
            if constexpr (ONCE) lo[a] = dequant_once_first(bits_h2(cq[a]).x, sf[2 * p], nzs[p >> 1][2 * (p & 1)]);
            else cq[a] = h2_bits(bits_h2(cq[a]) - h2{zf[2 * p], zf[2 * p + 1]});
        };
        auto cv_scale = [&](auto a_c, int set) {
            constexpr int a = decltype(a_c)::value, p = a & 3;
            afr[set][a >> 2][p] = h2_bits(ONCE ? h2{lo[a], dequant_once(bits_h2(cq[a]).y, sf[2 * p + 1], nzs[p >> 1][2 * (p & 1) + 1])}
                                               : bits_h2(cq[a]) * h2{sf[2 * p], sf[2 * p + 1]});
        };
        // pair a enters the pipeline at step 4 + a of the k-block (the lines are read at step 0, shifted
        // at step 3) and leaves it at step 7 + a <= 14
        auto convert_step = [&](auto t_c, int buf_src) {
            constexpr int T = decltype(t_c)::value, ks = T >> 4, t = T & 15, kn = (ks + 1) & 3;
            if (t == 0) read_codes(buf_src, kn);
            if (t == 3) {
#pragma unroll
                for (int p = 0; p < 4; ++p) cfs[p] = cf[p] >> nsh;
            }
            if (t >= 4 && t <= 11) cv_mask(std::integral_constant<int, (t - 4) & 7>{});
            if (t >= 5 && t <= 12) cv_base(std::integral_constant<int, (t - 5) & 7>{});
            if (t >= 6 && t <= 13) cv_zero(std::integral_constant<int, (t - 6) & 7>{});
            if (t >= 7 && t <= 14) cv_scale(std::integral_constant<int, (t - 7) & 7>{}, kn & 1);
        };
        // k-block 0 of stage 0, unpipelined
        read_codes(0, 0);
#pragma unroll
        for (int j = 0; j < 8; ++j) read_b(0, j, 0, 0);
#pragma unroll
        for (int p = 0; p < 4; ++p) cfs[p] = cf[p] >> nsh;
        QEFT_STEPS8(cv_mask, 0)
        QEFT_STEPS8(cv_base, 0)
        QEFT_STEPS8(cv_zero, 0)
        {
            auto sc0 = [&](auto a_c) { cv_scale(a_c, 0); };
            QEFT_STEPS8(sc0, 0)
        }

        auto stage = [&](int st, auto cur_c) {
            constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1;
            const int sl = min(st + 2, nst - 1);
            protect();
            asm volatile("" : "+v"(crd[0]), "+v"(crd[1]), "+v"(crd[2]), "+v"(crd[3]), "+v"(szr));
            auto step = [&](auto t_c) {
                constexpr int T = decltype(t_c)::value, ks = T >> 4, t = T & 15, kn = (ks + 1) & 3;
                constexpr int SRC = ks < 3 ? CUR : NXT;   // where the next k-block comes from
                mfma_step(t_c);
                if ((t & 1) == 0) read_b(kn & 1, t >> 1, SRC, kn);
                convert_step(t_c, SRC);
                produce_step(t_c, std::integral_constant<int, NXT>{}, sl);
                if (T == 47) __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            };
            QEFT_STEPS64(step)
        };
        run_stages(stage);
        store_f16_lds<true, 8>(acc, lds + wave * TILE_BYTES, dX, lddx, icw, L.kq, m0, M, lane);
    };

    // ---- a wave in a weak half --------------------------------------------------------------------------
    // Fragment t of lane fr is line (channel) 64 lb + 32 t + fr of the half, 16 bytes of it as they are.
    auto run_weak = [&]() {
        uint32_t wrd[4];  // weak lines of fragment 0, indexed by (XOR constant) / 2
#pragma unroll
        for (int x = 0; x < 4; ++x)
            wrd[x] = lds0 + DX_LINE_BASE + (uint32_t)half * DX_HALF + (uint32_t)(64 * lb + fr) * DX_LINE +
                     ((uint32_t)((fk ^ (fr >> 3)) ^ (2 * x)) << 4);
        auto read_a = [&](int set, int i, int buf, int kn) {
            afr[set][i] = *reinterpret_cast<const lds_u4*>(wrd[kn ^ (2 * (i & 1))] + (uint32_t)(i * 32 * DX_LINE + buf * DX_LINES));
        };
#pragma unroll
        for (int j = 0; j < 8; ++j) read_b(0, j, 0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) read_a(0, i, 0, 0);

        auto stage = [&](int st, auto cur_c) {
            constexpr int CUR = decltype(cur_c)::value, NXT = CUR ^ 1;
            const int sl = min(st + 2, nst - 1);
            protect();
            asm volatile("" : "+v"(wrd[0]), "+v"(wrd[1]), "+v"(wrd[2]), "+v"(wrd[3]));
            auto step = [&](auto t_c) {
                constexpr int T = decltype(t_c)::value, ks = T >> 4, t = T & 15, kn = (ks + 1) & 3;
                constexpr int SRC = ks < 3 ? CUR : NXT;
                mfma_step(t_c);
                if ((t & 1) == 0) read_b(kn & 1, t >> 1, SRC, kn);
                if (t == 3 || t == 7) read_a(kn & 1, t >> 2, SRC, kn);
                produce_step(t_c, std::integral_constant<int, NXT>{}, sl);
                if (T == 47) __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            };
            QEFT_STEPS64(step)
        };
        run_stages(stage);
        store_f16_lds<false, 8>(acc, lds + wave * TILE_BYTES, dX, lddx, icw - (-L.kq & 127), L.ic, m0, M, lane);
    };
#undef QEFT_STEPS64
#undef QEFT_STEPS8

    if (H0 == H1) {
        if (H0 == 0) run_quant(); else run_weak();
    } else {
        if (half == 0) run_quant(); else run_weak();
    }
}

// splits > 1: a workgroup (tile, sp) of a split tile contracts over the weight rows [sp * rps, (sp + 1) * rps) only (rps
// a multiple of 64: whole stages) and stores its partial tile as fp16 into its slot of `part`; splitk_reduce_kernel
// adds them.  Which tiles are split: split_tile.  The rows of a stored layer are independent, so a split is simply the
// layer made of those rows.
template <bool ONCE>
__device__ __forceinline__ void dx_rega_body(unsigned char* lds, Layer L, const __half* __restrict__ dY, int M, int64_t lddy,
                                             __half* __restrict__ dX, int64_t lddx, int tiles_ic, int splits,
                                             int rps, int tail_first, __half* __restrict__ part) {
    const int tiles_all = tiles_ic * ((M + BT - 1) / BT);
    int tile, sp, slot;
    if (!split_tile(tiles_all, tail_first, splits, tile, sp, slot)) return;
    int t_ic, t_m;
    tile_coords(tile, tiles_ic, (M + BT - 1) / BT, t_ic, t_m);
    const int ic0 = t_ic * BT, m0 = t_m * BT;
    if (slot >= 0) {
        const int r0 = sp * rps;
        L.qweight += (size_t)r0 * L.stride;
        L.scales += (size_t)r0 * L.gs;
        L.zeros += (size_t)r0 * L.gs;
        L.weak += (size_t)r0 * L.k;
        L.oc = min(rps, L.oc - r0);
        dY += r0;
        // the tile stores dX[m][ic] with absolute indices: point it at the slot's (m0, ic0)
        dX = part + (size_t)slot * (BT * BT) - ((size_t)m0 * BT + ic0);
        lddx = BT;
    }
    // a half is weak when it starts at or past Kq; without a weak block the surplus
    // half of the last tile runs as a quantized one on clamped addresses and stores nothing
    const bool w0 = L.k > 0 && ic0 >= L.kq, w1 = L.k > 0 && ic0 + 128 >= L.kq;
    if (w0) dx_tile<1, 1, ONCE>(L, dY, M, lddy, dX, lddx, ic0, m0, lds);
    else if (w1) dx_tile<0, 1, ONCE>(L, dY, M, lddy, dX, lddx, ic0, m0, lds);
    else dx_tile<0, 0, ONCE>(L, dY, M, lddy, dX, lddx, ic0, m0, lds);
}
template <bool ONCE>
__global__ __launch_bounds__(256) void gemm_dx_rega_kernel(Layer L, const __half* __restrict__ dY, int M, int64_t lddy,
                                                           __half* __restrict__ dX, int64_t lddx, int tiles_ic, int splits,
                                                           int rps, int tail_first, __half* __restrict__ part) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    dx_rega_body<ONCE>(lds, L, dY, M, lddy, dX, lddx, tiles_ic, splits, rps, tail_first, part);
}

template <int KW>
__global__ __launch_bounds__(256) void weak_grad_strip_kernel(int oc_total, int k_total, const __half* __restrict__ dY, int M,
                                                              int64_t lddy, const __half* __restrict__ Xw, int64_t ldxw,
                                                              float* __restrict__ part, int splits, int chunk, void* dW,
                                                              int out_f32, int accumulate) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    weak_grad_strip_body<KW>(lds, (int)blockIdx.x, oc_total, k_total, dY, M, lddy, Xw, ldxw, part, splits, chunk, dW, out_f32, accumulate);
}

// The input gradient and the weak block's gradient of one layer in ONE launch: the first n_dx workgroups are the
// tiles of gemm_dx_rega_kernel (no split), the rest the strips of weak_grad_strip_kernel.  Both read dY; the
// strips are dispatched as compute units fall free, i.e. into the partly empty last round of tiles (688 tiles on
// 256 units leave 80 of them idle for a third of the launch), where they cost nothing.
template <bool ONCE>
__global__ __launch_bounds__(256) void gemm_dx_dw_kernel(Layer L, const __half* __restrict__ dY, int M, int64_t lddy,
                                                         __half* __restrict__ dX, int64_t lddx, int tiles_ic, int n_dx, Strips S) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    if ((int)blockIdx.x >= n_dx) {
        weak_grad_strip(lds, (int)blockIdx.x - n_dx, S);
        return;
    }
    dx_rega_body<ONCE>(lds, L, dY, M, lddy, dX, lddx, tiles_ic, 1, 0, 0, nullptr);
}

__global__ __launch_bounds__(256) void weak_grad_reduce_kernel(const float* __restrict__ part, int splits, int64_t n,
                                                               void* dW, int out_f32, int accumulate) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float s = 0.f;
    for (int p = 0; p < splits; ++p) s += part[(size_t)p * n + i];
    if (out_f32) {
        float* o = (float*)dW + i;
        *o = accumulate ? *o + s : s;
    } else {
        __half* o = (__half*)dW + i;
        *o = __float2half_rn(accumulate ? __half2float(*o) + s : s);
    }
}

hipError_t raise_lds_limit(const void* fn, bool& done) {
    if (done) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, GEMM_LDS);
    if (e == hipSuccess) done = true;
    return e;
}

}  // namespace

// The tiled kernels round every dequantized weight once to fp16 (relative 2^-11).  Over a long contraction these
// roundings average out far below the parity bar; a sum of a handful of terms has no such averaging and single
// outputs can leave the per-element bar, so contractions shorter than 64 terms (IC here, OC for the input
// gradient) take the general kernels, which keep s (q - z) in fp32.
constexpr int MIN_CONTRACTION = 64;

bool gemm_fwd_supported(const Layer& L, int64_t M) {
    return M >= 1 && L.bits == 4 && L.g == 128 && (L.kq % 8) == 0 && (L.k % 8) == 0 && (L.oc % 8) == 0 && L.ic >= MIN_CONTRACTION;
}

namespace {
// Sum of the partial tiles of the split tiles: workgroup (tail index, r) adds the `splits` slots of rows 8 r .. 8 r + 7
// of one tile, 8 outputs (16 bytes) per thread, fp32 sum in split order, one rounding.  n: columns of the output
// (tiles_n tiles of them); pm: rows of a panel (a slot has room for 256).
__device__ __forceinline__ void splitk_reduce_body(int bid, const __half* __restrict__ part, int splits, int tiles_all, int tiles_n,
                                                   int tail_first, int M, int pm, int n, __half* __restrict__ Y, int64_t ldy) {
    const int tt = bid >> 5, part32 = bid & 31;
    const int tile = split_tail_tile(tiles_all, tail_first, tt);
    if (tile < 0) return;
    int t_n, t_m;
    tile_coords(tile, tiles_n, (M + pm - 1) / pm, t_n, t_m);
    const int n0 = t_n * BT, m0 = t_m * pm;
    const bool wide = (ldy & 7) == 0 && (reinterpret_cast<uintptr_t>(Y) & 15) == 0;
    const __half* p0 = part + (size_t)tt * splits * (BT * BT);
    {
        const int row = part32 * 8 + (threadIdx.x >> 5), c = threadIdx.x & 31;
        const int m = m0 + row, col = n0 + 8 * c;
        if (row >= pm || m >= M || col >= n) return;
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll 4
        for (int p = 0; p < splits; ++p) {
            const u4 v = ld16(p0 + (size_t)p * (BT * BT) + row * BT + 8 * c);
            const h8 h = __builtin_bit_cast(h8, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += (float)h[e];
        }
        __half* y = Y + (size_t)m * ldy + col;
        if (col + 8 <= n && wide) {
            h8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (_Float16)acc[e];
            *reinterpret_cast<u4*>(y) = __builtin_bit_cast(u4, o);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (col + e < n) y[e] = __float2half_rn(acc[e]);
        }
    }
}

__global__ __launch_bounds__(256) void splitk_reduce_kernel(const __half* __restrict__ part, int splits, int tiles_all, int tiles_n,
                                                            int tail_first, int M, int pm, int n, __half* __restrict__ Y, int64_t ldy) {
    splitk_reduce_body((int)blockIdx.x, part, splits, tiles_all, tiles_n, tail_first, M, pm, n, Y, ldy);
}
// The same behind an input gradient that was split, with the strips of the weak gradient ahead of it in the grid: either alone is short and
// leaves most of the GPU waiting for it.  One launch instead of two, the whole backward, us: 4096 x 4096 at M = 200 / 512 / 777 34 / 42.5 / 56 ->
// 29 / 37 / 51; 11008 x 4096 at 512 / 2048 72 / 206 -> 66 / 200; 3-bit 5120 x 5120 at 1000 91 -> 85.  65 KB of LDS for every workgroup (49 in pieces of 64 weak columns) leaves a CU two or three at
// a time; with its partial tiles four requests at a time the sum takes no longer for it.
__global__ __launch_bounds__(256) void splitk_reduce_dw_kernel(const __half* __restrict__ part, int splits, int tiles_all, int tiles_n,
                                                               int tail_first, int M, int n, __half* __restrict__ dX, int64_t lddx, Strips S) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    if ((int)blockIdx.x < S.n) weak_grad_strip(lds, (int)blockIdx.x, S);
    else splitk_reduce_body((int)blockIdx.x - S.n, part, splits, tiles_all, tiles_n, tail_first, M, BT, n, dX, lddx);
}

// Which tiles to split and how, for a launch of `tiles` tiles whose contraction has `chunks` units of 8 stages.
//   fewer than 160 tiles: all of them, as many ways as bring the workgroups to about the number of CUs (at most 16);
//   otherwise the tiles of each XCD's last round when that round fills at most half of the XCD's 32 CUs, as many ways as
//   fill it (at most 8) - provided the time saved on that round (stage_us per stage) is well above the cost of the
//   partial tiles' traffic and the second launch.
struct SplitPlan {
    int splits = 1, chunks_per_split = 0, tail_first = 0;
};
SplitPlan plan_split(int tiles, int stages) {
    SplitPlan p;
    const int chunks = stages / 8;
    if (chunks < 2) return p;
    int want;
    if (tiles < 160) {
        want = 256 / tiles;
        want = want > 16 ? 16 : want;
    } else {
        const int per = ceil_div(tiles, N_XCD), full = per / 32 * 32, rem = per - full;
        if (rem == 0 || rem > 16 || full == 0) return p;
        want = 32 / rem;
        want = want > 8 ? 8 : want;
        p.tail_first = full;
    }
    const int chunks_all = ceil_div(stages, 8);   // a ragged last chunk included
    want = want > chunks_all ? chunks_all : want;
    if (want < 2) return SplitPlan();
    p.chunks_per_split = ceil_div(chunks_all, want);   // at most `want` splits
    p.splits = ceil_div(stages, p.chunks_per_split * 8);
    if (p.splits < 2) return SplitPlan();
    if (p.tail_first > 0) {
        // measured: a stage takes 1.6 - 1.8 us with every CU busy; the second launch 7 - 9 us for 256 slots
        const double saved = (stages - p.chunks_per_split * 8) * 1.6;                                // us
        const double cost = 8.0 + split_tail_tiles(tiles, p.tail_first) * p.splits * 0.05;           // us: 128 KB written and read per slot
        if (saved < 1.5 * cost) return SplitPlan();
    }
    return p;
}
size_t split_workspace(int tiles, const SplitPlan& p) {
    return p.splits > 1 ? (size_t)split_tail_tiles(tiles, p.tail_first) * p.splits * BT * BT * sizeof(__half) : 0;
}
}  // namespace

// K split of the forward: units of 8 stages (512 columns)
static SplitPlan gemm_fwd_plan(const Layer& L, int64_t M) {
    const int tiles = ceil_div(L.oc, BT) * ceil_div(M, BT);
    if (L.kq == 0 && L.k > 0 && L.k % BK == 0) return plan_split(tiles, L.k / BK);   // all fp16: the weak stages are split
    if (L.kq <= 0 || L.kq % BK != 0) return SplitPlan();
    return plan_split(tiles, L.kq / BK);
}

size_t gemm_fwd_split_workspace(const Layer& L, int64_t M) {
    return split_workspace(ceil_div(L.oc, BT) * ceil_div(M, BT), gemm_fwd_plan(L, M));
}

GemmSplit gemm_fwd_split(const Layer& L, int64_t M) {
    const SplitPlan p = gemm_fwd_plan(L, M);
    return GemmSplit{p.splits, 8 * p.chunks_per_split, ceil_div(L.oc, BT) * ceil_div(M, BT), p.tail_first > 0};
}

hipError_t gemm_fwd(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, void* ws, hipStream_t s) {
    const int tiles_oc = ceil_div(L.oc, BT), tiles_m = ceil_div(M, BT);
    hipError_t e;
    if (fwd_in_registers(L, M, ldx)) {   // weights straight into MFMA operand registers
        // as many panels as of 256 rows, each of the fewest rows: the tiles, the splits and the workspace stay what they are,
        // and a tile multiplies less padding (us, panels of 256 rows before -> now: 13824 x 5120 with its split, M = 300 / 333 /
        // 400 / 1300: 74 / 75 / 77 / 204 -> 58 / 65 / 72 / 185; 4096 x 11008, M = 777: 96 -> 89; multiples of 256 unchanged)
        using Kern = void (*)(Layer, const __half*, int, int64_t, __half*, int64_t, int, int, int, int, int, __half*);
#define QEFT_REGA(ONCE) {gemm_fwd_rega_kernel<4, ONCE>, gemm_fwd_rega_kernel<5, ONCE>, gemm_fwd_rega_kernel<6, ONCE>, \
                         gemm_fwd_rega_kernel<7, ONCE>, gemm_fwd_rega_kernel<8, ONCE>}
        static const Kern table[2][5] = {QEFT_REGA(false), QEFT_REGA(true)};
#undef QEFT_REGA
        static bool attr[2][5] = {};
        const int rows = ceil_div(M, tiles_m), j = rows <= 128 ? 4 : ceil_div(rows, 32);
        const Kern kern = table[L.once][j - 4];
        if (!attr[L.once][j - 4]) {
            e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, REGA_LDS);
            if (e != hipSuccess) return e;
            attr[L.once][j - 4] = true;
        }
        const int tiles = tiles_oc * tiles_m;
        const int wide = (ldy % 8 == 0) && (reinterpret_cast<uintptr_t>(Y) % 16 == 0);
        const SplitPlan p = ws ? gemm_fwd_plan(L, M) : SplitPlan();
        if (p.splits > 1) {
            __half* part = (__half*)ws;
            kern<<<split_grid(tiles, p.tail_first, p.splits), 256, REGA_LDS, s>>>(L, X, (int)M, ldx, Y, ldy, tiles_oc, wide, p.splits,
                                                                                 p.chunks_per_split * 8, p.tail_first, part);
            splitk_reduce_kernel<<<32 * split_tail_tiles(tiles, p.tail_first), 256, 0, s>>>(part, p.splits, tiles, tiles_oc, p.tail_first, (int)M,
                                                                                           32 * j, L.oc, Y, ldy);
            return hipGetLastError();
        }
        kern<<<xcd_grid(tiles), 256, REGA_LDS, s>>>(L, X, (int)M, ldx, Y, ldy, tiles_oc, wide, 1, 0, 0, nullptr);
    } else {
        static bool attr = false;
        e = raise_lds_limit((const void*)gemm_fwd_kernel, attr);
        if (e != hipSuccess) return e;
        gemm_fwd_kernel<<<xcd_grid(tiles_oc * tiles_m), 256, GEMM_LDS, s>>>(L, X, (int)M, ldx, Y, ldy, tiles_oc);
    }
    return hipGetLastError();
}

bool gemm_dx_supported(const Layer& L, int64_t M) {
    return M > 16 && L.bits == 4 && L.g == 128 && (L.kq % 8) == 0 && (L.k % 8) == 0 && (L.oc % 8) == 0 &&
           (L.ic % 8) == 0 && L.oc >= MIN_CONTRACTION;
}

// Row split of the input gradient, as for the forward: units of 8 stages (512 rows).
static SplitPlan gemm_dx_plan(const Layer& L, int64_t M) {
    if (!dx_in_registers(L) || L.kq % 128 != 0) return SplitPlan();   // (a slot has no room for the weak channels' other place)
    return plan_split(ceil_div(L.ic, BT) * ceil_div(M, BT), L.oc / BK);
}

size_t gemm_dx_split_workspace(const Layer& L, int64_t M) {
    return split_workspace(ceil_div(L.ic, BT) * ceil_div(M, BT), gemm_dx_plan(L, M));
}

GemmSplit gemm_dx_split(const Layer& L, int64_t M) {
    const SplitPlan p = gemm_dx_plan(L, M);
    return GemmSplit{p.splits, 8 * p.chunks_per_split, ceil_div(L.ic, BT) * ceil_div(M, BT), p.tail_first > 0};
}

// (defined below: tiles and strips in one launch)
static hipError_t gemm_dx_dw(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, const Strips& S, hipStream_t s);
static bool gemm_dx_dw_preferred(const Strips& S);

hipError_t gemm_dx(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, void* ws, hipStream_t s, WeakGrad* g) {
    const bool in_registers = dx_in_registers(L, M, lddy);
    const int tiles_m = ceil_div(M, BT), tiles_ic = ceil_div(in_registers ? dx_columns(L) : L.ic, BT);
    hipError_t e;
    if (in_registers) {
        static bool attr[2] = {};
        const auto kern = L.once ? gemm_dx_rega_kernel<true> : gemm_dx_rega_kernel<false>;
        if (!attr[L.once]) {
            e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, DX_LDS);
            if (e != hipSuccess) return e;
            attr[L.once] = true;
        }
        const int tiles = tiles_ic * tiles_m;
        const SplitPlan p = ws ? gemm_dx_plan(L, M) : SplitPlan();
        if (p.splits > 1) {
            __half* part = (__half*)ws;
            kern<<<split_grid(tiles, p.tail_first, p.splits), 256, DX_LDS, s>>>(L, dY, (int)M, lddy, dX, lddx, tiles_ic, p.splits,
                                                                                              p.chunks_per_split * 8 * BK, p.tail_first, part);
            const int n_sum = 32 * split_tail_tiles(tiles, p.tail_first);
            const Strips S = make_strips(g, dY, M, lddy, g ? (size_t)((unsigned char*)ws - g->ws) + split_workspace(tiles, p) : 0);
            if (S.n > 0) {
                static bool dw_attr = false;
                if (!dw_attr) {
                    e = hipFuncSetAttribute((const void*)splitk_reduce_dw_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, WG_LDS);
                    if (e != hipSuccess) return e;
                    dw_attr = true;
                }
                splitk_reduce_dw_kernel<<<S.n + n_sum, 256, wg_lds(S.kw), s>>>(part, p.splits, tiles, tiles_ic, p.tail_first, (int)M, L.ic, dX, lddx, S);
                e = hipGetLastError();
                return e == hipSuccess ? finish_strips(g, S, s) : e;
            }
            splitk_reduce_kernel<<<n_sum, 256, 0, s>>>(part, p.splits, tiles, tiles_ic, p.tail_first, (int)M, BT, L.ic, dX, lddx);
            return hipGetLastError();
        }
        const Strips S = make_strips(g, dY, M, lddy, g ? g->used : 0);
        if (S.n > 0 && gemm_dx_dw_preferred(S)) {
            e = gemm_dx_dw(L, dY, M, lddy, dX, lddx, S, s);
            return e == hipSuccess ? finish_strips(g, S, s) : e;
        }
        kern<<<xcd_grid(tiles), 256, DX_LDS, s>>>(L, dY, (int)M, lddy, dX, lddx, tiles_ic, 1, 0, 0, nullptr);
    } else {
        static bool attr = false;
        e = raise_lds_limit((const void*)gemm_dx_kernel, attr);
        if (e != hipSuccess) return e;
        gemm_dx_kernel<<<xcd_grid(tiles_ic * tiles_m), 256, GEMM_LDS, s>>>(L, dY, (int)M, lddy, dX, lddx, tiles_ic, 0);
    }
    return hipGetLastError();
}

bool weak_grad_mfma_supported(int oc, int k, int64_t M) {
    return M >= 64 && k >= 8 && k <= BT && (k % 8) == 0 && (oc % 8) == 0;
}

size_t weak_grad_mfma_workspace(int oc, int k, int64_t M) {
    const int splits = weak_grad_strip_most(oc, k, M);
    return splits > 1 ? (size_t)splits * oc * k * sizeof(float) : 0;
}

hipError_t weak_grad_mfma(int oc, int k, const __half* dY, int64_t M, int64_t lddy, const __half* Xw, int64_t ldxw,
                          void* dW, int out_f32, int accumulate, void* ws, hipStream_t s) {
    if (!strip_offsets_fit(lddy) || !strip_offsets_fit(ldxw)) return weak_grad_generic(oc, k, dY, M, lddy, Xw, ldxw, dW, out_f32, accumulate, s);
    const StripPlan p = weak_grad_strip_split(oc, k, M);
    const auto kern = p.kw == 128 ? weak_grad_strip_kernel<128> : weak_grad_strip_kernel<64>;
    static bool strip_attr[2] = {};
    if (!strip_attr[p.kw == 128]) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, wg_lds(p.kw));
        if (e != hipSuccess) return e;
        strip_attr[p.kw == 128] = true;
    }
    kern<<<p.workgroups(oc, k), 256, wg_lds(p.kw), s>>>(oc, k, dY, (int)M, lddy, Xw, ldxw, (float*)ws, p.splits, p.chunk, dW, out_f32, accumulate);
    hipError_t e = hipGetLastError();
    return e == hipSuccess && p.splits > 1 ? weak_grad_reduce((const float*)ws, p.splits, (int64_t)oc * k, dW, out_f32, accumulate, s) : e;
}
hipError_t weak_grad_reduce(const float* part, int splits, int64_t n, void* dW, int out_f32, int accumulate, hipStream_t s) {
    weak_grad_reduce_kernel<<<ceil_div(n, 256), 256, 0, s>>>(part, splits, n, dW, out_f32, accumulate);
    return hipGetLastError();
}

// dX and dW_weak of one layer in one launch (see gemm_dx_dw_kernel), for layers the register kernel takes.
// Taken for weak blocks of up to 128 columns (one piece of 128, or two of 64).  The strips follow the tiles in the grid, so they start on
// whichever compute units finish their last tile first: in the idle part of a partly empty last round, or, when the
// tiles fill their rounds, in the few microseconds by which the tiles' ends differ.  Inside the combined launch a strip
// workgroup has a compute unit to itself (the launch reserves the tile kernel's LDS and registers for every workgroup;
// on its own the strip kernel runs two per unit), so a weak gradient that is heavy next to that idle time loses more
// than it gains.  Measured at M = 4096, the two calls against the one: 11008 x 4096 (256 tiles) 388 -> 382 us,
// 4096 x 4096 (256 tiles) 165 -> 163, 4096 x 11008 (688 tiles) 363 -> 350, 5120 x 5120 281 -> 262, 13824 x 5120
// 699 -> 670; with a 256-wide weak block (two pieces of 128 per strip of channels) 8192 x 8192 at M = 2048 257 -> 252
// but 28672 x 8192 862 -> 877.
static bool gemm_dx_dw_preferred(const Strips& S) { return S.k <= 128; }

static hipError_t gemm_dx_dw(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, const Strips& S, hipStream_t s) {
    const int tiles_ic = ceil_div(dx_columns(L), BT), n_dx = xcd_grid(tiles_ic * ceil_div(M, BT));
    static bool attr[2] = {};
    constexpr int LDS_BYTES = DX_LDS > WG_LDS ? DX_LDS : WG_LDS;
    const auto kern = L.once ? gemm_dx_dw_kernel<true> : gemm_dx_dw_kernel<false>;
    if (!attr[L.once]) {
        hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr[L.once] = true;
    }
    kern<<<n_dx + S.n, 256, LDS_BYTES, s>>>(L, dY, (int)M, lddy, dX, lddx, tiles_ic, n_dx, S);
    return hipGetLastError();
}

}  // namespace qeft
