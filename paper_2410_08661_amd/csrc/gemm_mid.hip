// Forward of 4-bit layers for 2 to 672 rows (up to 16: long rows and small layers; from 97: few tiles) and of 3-bit layers from 2 rows on: several sequences
// decoded together, short prompts, draft tokens.  (Paper Sec. 3.2.1; the rows between the matrix-vector kernels' 16 and the sizes at which 256 x 256 tiles occupy the GPU.)
//
// A layer's codes are read once per panel of up to 48 rows, where passes of the 16-row kernel read them once per 16 rows
// and the tiled GEMM leaves OC / 256 of 256 compute units working on the whole contraction.  What bounds the kernel: every
// workgroup reads its panel of X in full (48 rows x 2 IC bytes against 8 IC bytes of codes per tile of 16 channels), and each
// kilobyte of it costs a CU about 13 ns on its way through the L1, whatever the order of groups or the pitch of the rows
// (4096 x 11008 at 8 / 24 / 40 rows: 11.6 / 16.7 / 20.8 us).  Hence as few, as wide workgroups as still occupy every CU (rule at fwd_mid).
//
// Mapping: 16x16x32 MFMA, rows of X as the A operand, 16 channels as the B operand (a packed word is a lane's 8 contraction
// elements), a group of 128 columns at a time.  The workgroup's waves take every KS-th pair of neighbouring groups each and share
// nothing until the end, so the main loop has no barrier.  A group's rows and a pair's codes go from memory to a piece of the wave's LDS
// by themselves (buffer loads that write LDS: no registers, so the next group's rows and the next pair's codes are on the way while a
// group is multiplied), chunks XOR-placed by the row on the way; the wave reads them back as fragments once, the rows into nibble
// order, and multiplies all its channel tiles.  The codes' way through LDS is for the L1: a lane that fetches its own fragment shares no
// line with its neighbours, and each of the 64 takes one of the L1's tag cycles, which were 70 % of the CUs' time (counters at
// M = 40, 22016 x 4096: 34.6k of 50k cycles; matrix pipe 11k, vector issue 19k; 22.3k of 48k now); 8 rows x 128 bytes per request are 16 cycles.  In pairs,
// because a half line fetched alone holds a whole one.  Dequantization as in the 16-row kernels, on the accumulator and without
// rounding the weights: s (sum x (1024 + q) - (1024 + z) Sx), two FMAs per accumulator and group.  Partial tiles meet in LDS in a fixed
// order (fp32).
// Measured (rows through registers, lanes fetching their own fragments, single groups -> now, us): 22016 x 4096 (gate/up) at M = 24 / 40 / 64:
// 24.4 / 29.0 / 41.4 -> 21.2 / 25.3 / 32.1; 4096 x 11008: 18.0 / 23.3 / 24.1 -> 16.7 / 20.8 / 20.1; 5120 x 13824: 30.4 / 37.7 / 37.7 -> 26.3 / 31.3 / 30.2;
// 8192 x 8192: 20.2 / 24.6 / 29.0 -> 17.7 / 21.0 / 23.6; 4096 x 4096 at M = 40 / 96: 10.6 / 11.9 -> 9.8 / 11.3.
// 3-bit codes are multiplied as they are stored (Codes3), fetched by the lanes that use them (us, ten codes a word): 5120 x 5120,
// M = 2 / 16 / 40: 8.0 / 9.2 / 13.4; 15360 x 5120 (q/k/v) M = 8 / 40: 14.9 / 22.9; 27648 x 5120 (gate/up) M = 8: 25.2; 1024 x 2048, M = 8: 4.3.
// Tried and no faster: X requests that bypass the caches (nt: 10 to 30 % slower), other orders of the groups per workgroup, 80 and 96
// channels per workgroup (48 rows spill; 64 channels have 249 of 256 registers, see LEAN).
// Tried and not kept: 64 rows per panel (registers spill, 2 to 5 times slower).
#include <type_traits>

#include <climits>
#include "qeft_internal.h"

namespace qeft {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u3w __attribute__((ext_vector_type(3), aligned(4)));   // three / four words at any word of a row
typedef uint32_t u4w __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ h8 as_h8(u4 v) { return __builtin_bit_cast(h8, v); }
__device__ __forceinline__ uint32_t pack2(float a, float b) { return __builtin_bit_cast(uint32_t, h2{(_Float16)a, (_Float16)b}); }
// waits until at most N of the wave's requests to memory are under way
template <int N>
__device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// The pairs of codes of a word lie four apart, (0,4)(1,5)(2,6)(3,7), where each takes a shift and a mask (7 instructions per word).  Either the
// activations are brought into that order - 4 instructions per 8 of a row -, or the codes into theirs, two instructions more per word: a byte of
// the word beside the same byte of the word moved down by a code.
__device__ __forceinline__ uint32_t neighbours(uint32_t w, uint32_t w4, int p) { return __builtin_amdgcn_perm(w4, w, 0x0c040c00u + 0x00010001u * (uint32_t)p); }
__device__ __forceinline__ u4 permute_x(u4 v) {
    u4 r;
    r.x = __builtin_amdgcn_perm(v.z, v.x, 0x05040100u);
    r.y = __builtin_amdgcn_perm(v.z, v.x, 0x07060302u);
    r.z = __builtin_amdgcn_perm(v.w, v.y, 0x05040100u);
    r.w = __builtin_amdgcn_perm(v.w, v.y, 0x07060302u);
    return r;
}

// How a layer's codes are stored.
enum Fmt { W4 = 0, W3_DENSE = 1, W3_TEN = 2 };

// Three-bit codes.  A lane's 32 columns of a group are 96 consecutive bits of a dense row: three words.  Ten codes to a word
// (W3_TEN): columns 32 c .. + 31 start at code p = 32 c % 10 of word 32 c / 10, and p <= 8, so they lie in four words whose 30-bit
// payloads are first joined to the same three (nine instructions, the shift 3 p the lane's own).  Pairs are neighbours, as the activations lie:
// in each ten of the 32 codes the odd ones move up by 13 bits to the upper half, and every pair is a shift and a mask away; codes 30 and
// 31 are a pair of their own.  (Pairs of codes five apart take two instructions less per 32 codes, but 15 for every 16 rows to bring the
// activations into their order.)
struct Codes3 {
    uint32_t ya[3], yb[3], r;
    template <Fmt F>
    __device__ __forceinline__ void take(u4 w, uint32_t shift) {
        uint32_t a = w.x, b = w.y, c = w.z;
        if (F == W3_TEN) {
            const uint32_t c0 = w.x | (w.y << 30), c1 = (w.y >> 2) | (w.z << 28), c2 = (w.z >> 4) | (w.w << 26), c3 = w.w >> 6;
            a = __builtin_amdgcn_alignbit(c1, c0, shift);
            b = __builtin_amdgcn_alignbit(c2, c1, shift);
            c = __builtin_amdgcn_alignbit(c3, c2, shift);
        }
        const uint32_t t[3] = {a, __builtin_amdgcn_alignbit(b, a, 30), __builtin_amdgcn_alignbit(c, b, 28)}, t3 = c >> 26;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            ya[i] = (t[i] & 0xffffu) | ((t[i] << 13) & 0xffff0000u);   // codes 0 .. 5 of the ten
            yb[i] = (t[i] >> 18) | ((t[i] >> 18) << 13);               // 6 .. 9
        }
        r = t3 | (t3 << 13);
    }
    // codes 2 P and 2 P + 1 at bits 0 .. 2 of each half
    __device__ __forceinline__ uint32_t bits(int P) const {
        const int i = P / 5 < 3 ? P / 5 : 0, q = P % 5;
        return P == 15 ? r : (q < 3 ? ya[i] >> (6 * q) : yb[i] >> (6 * (q - 3)));
    }
};

// bytes of LDS of a wave, without the parameters
constexpr int mid_piece(int MT, int NT, bool codes) {
    const int main = MT * 4096 + (codes ? NT * 2048 : 0), sum = MT * NT * 1024;
    return main > sum ? main : sum;
}

struct MidArgs {
    const uint32_t* qweight[MAX_GROUP];
    const __half* scales[MAX_GROUP];
    const __half* zeros[MAX_GROUP];
    const __half* weak[MAX_GROUP];
    __half* Y[MAX_GROUP];
    int64_t ldy[MAX_GROUP];
    int oc[MAX_GROUP];
    int tile_begin[MAX_GROUP];   // first tile of 16 NT channels of layer i; INT_MAX when absent
    int n_tiles, tiles_m;        // tiles of channels over all layers, panels of 16 MT rows
    const __half* X;
    int64_t ldx;
    int M, kq, k, ng, stride, gs;
};

// One workgroup: 16 NT channels x 16 MT rows of Y over the whole contraction, which its KS waves divide; the partial tiles
// meet in LDS at the end (fp32, fixed order).
// XR: requests of activations per group, 4 rows each (MT = 1: as many as there are rows; else all of the tile's).
constexpr int mid_waves(int MT, int NT) { return MT == 1 && NT == 1 ? 12 : 8; }   // the most waves of a workgroup
template <int MT, int NT, Fmt F, int XR>
__global__ __launch_bounds__(64 * mid_waves(MT, NT)) void fwd_mid_kernel(MidArgs A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int XB = MT * 4096;                        // a wave's piece of LDS: a group of activations, (4-bit) the codes of two groups,
    constexpr int WB = mid_piece(MT, NT, F == W4);       // (at the end a partial tile),
    constexpr int PB = NT * 128;                         // and (zero-point, scale) of two groups of up to 64 channels
    static_assert(MT == 1 || XR == 4 * MT, "");
    // the widest tile has no registers for an offset per request: taken from the first row's each time (kept, they went to scratch memory
    // and came back behind waits for the rows just requested)
    constexpr bool LEAN = MT * NT == 12;
    constexpr bool AS_THEY_LIE = F != W4 || 2 * MT > NT;   // the activations stay in column order
    const int lane = threadIdx.x & 63;
    const int KS = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kb = lane >> 4;

    const int per_xcd = (A.n_tiles * A.tiles_m + 7) >> 3;
    const int v = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (v >= A.n_tiles * A.tiles_m) return;
    const int t_n = v / A.tiles_m, t_m = v - t_n * A.tiles_m;
    const int li = (t_n >= A.tile_begin[1]) + (t_n >= A.tile_begin[2]) + (t_n >= A.tile_begin[3]);
    const int oc = A.oc[li];
    const int o0 = (t_n - A.tile_begin[li]) * (16 * NT), m0 = t_m * (16 * MT);

    unsigned char* mine = lds + (size_t)wave * WB;
    unsigned char* par = lds + (size_t)KS * WB + (size_t)wave * PB;
    const int last_g = A.ng - 1;

    const unsigned char* wbase = reinterpret_cast<const unsigned char*>(A.qweight[li] + (size_t)o0 * A.stride);
    const __half* sbase = A.scales[li] + (size_t)o0 * A.gs;
    const __half* zbase = A.zeros[li] + (size_t)o0 * A.gs;
    uint32_t woff[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) woff[t] = (uint32_t)min(16 * t + n, oc - 1 - o0) * (uint32_t)(A.stride * 4) + (F == W3_DENSE ? 12u * kb : 0u);
    static_assert(NT <= 4, "");
    const uint32_t poff = (uint32_t)min(min(lane, 16 * NT - 1), oc - 1 - o0) * (uint32_t)A.gs;
    const int xr = lane >> 4, xc = lane & 15;    // request u of a group of activations: row 4 u + xr, to slot xc: chunk xc ^ (row % 16)
    const unsigned char* xbase = reinterpret_cast<const unsigned char*>(A.X + (size_t)m0 * A.ldx);
    const uint32_t xpitch = (uint32_t)A.ldx * 2u;
    const auto xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(xbase), 0, (int)0xffffffff, 0x00020000);
    const int mlast = A.M - 1 - m0;
    const uint32_t xoff0 = (uint32_t)xr * xpitch, xlast = (uint32_t)min(mlast, 16 * MT) * xpitch;

    u4 wq[2][NT];         // codes and (zero-point, scale) of two groups
    uint32_t zs[2][NT];
    uint32_t ps, pz;
    // ten codes per word: the lane's first word of a group and its shift (four words are there: 32 c / 10 + 4 is at most the row's
    // padded length for every c with a column before Kq; the min is for lanes past it)
    const uint32_t last_w = 4u * (uint32_t)(A.stride - 4);
    auto first_word = [&](int g) { return min(4u * ((uint32_t)(128 * g + 32 * kb) / 10u), last_w); };
    auto shift_of = [&](int g) { return 3u * ((uint32_t)(128 * g + 32 * kb) % 10u); };
    auto load_w = [&](int set, int t, int g) {
        const int gc = min(g, last_g);
        if constexpr (F == W3_DENSE) {
            const u3w v = *reinterpret_cast<const u3w*>(wbase + (size_t)(48 * gc) + woff[t]);
            wq[set][t] = u4{v.x, v.y, v.z, 0u};
        } else
            wq[set][t] = *reinterpret_cast<const u4w*>(wbase + first_word(gc) + woff[t]);
    };
    // the rows' 256-byte pieces of group g go to LDS by themselves; columns past Kq repeat the last 8
    auto load_x = [&](int g) {
        uint32_t col[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) col[c] = (uint32_t)(2 * min(128 * g + 8 * (xc ^ (4 * c + xr)), A.kq - 8));
        uint32_t first = xoff0;
        if constexpr (LEAN) asm volatile("" : "+v"(first));
#pragma unroll
        for (int u = 0; u < XR; ++u) {
            const uint32_t off = min(first + (uint32_t)(4 * u) * xpitch, xlast) + col[u & 3];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xbuf, (__attribute__((address_space(3))) void*)(mine + 1024 * u), 16, (int)off, 0, 0, 0);
        }
    };
    // codes of groups 2 p and 2 p + 1: 8 rows x 128 bytes per request, so that neighbouring lanes read neighbouring bytes (a lane
    // fetching its own fragment shares no bytes with its neighbours, and each of its 16 bytes is an access to the L1's tags)
    const auto wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(wbase), 0, (int)0xffffffff, 0x00020000);
    unsigned char* codes = mine + XB;
    const uint32_t cpitch = (uint32_t)(A.stride * 4), coff0 = (uint32_t)(lane >> 3) * cpitch, clast = (uint32_t)min(oc - 1 - o0, 16 * NT) * cpitch;
    auto load_codes = [&](int p) {
        uint32_t col[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) col[c] = (uint32_t)min(128 * p + 16 * ((lane & 7) ^ (4 * c + (lane >> 4))), 4 * A.stride - 16);
        uint32_t first = coff0;
        if constexpr (LEAN) asm volatile("" : "+v"(first));
#pragma unroll
        for (int u = 0; u < 2 * NT; ++u) {
            const uint32_t off = min(first + (uint32_t)(8 * u) * cpitch, clast) + col[u & 1];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wbuf, (__attribute__((address_space(3))) void*)(codes + 1024 * u), 16, (int)off, 0, 0, 0);
        }
    };
    // parameters of groups 2 p and 2 p + 1: a lane fetches those of one channel and hands them out through LDS (rows of scales and
    // zero-points are padded to eights)
    auto load_par = [&](int p) {
        ps = *reinterpret_cast<const uint32_t*>(sbase + poff + 2 * min(p, last_g >> 1));
        pz = *reinterpret_cast<const uint32_t*>(zbase + poff + 2 * min(p, last_g >> 1));
    };
    auto put_par = [&]() {
        if (lane < 16 * NT)
            *reinterpret_cast<u2*>(par + 8 * lane) = u2{__builtin_amdgcn_perm(ps, pz, 0x05040100u), __builtin_amdgcn_perm(ps, pz, 0x07060302u)};
    };

    f4 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[a][t] = f4{0.f, 0.f, 0.f, 0.f};

    uint32_t mask = F == W4 ? 0x000f000fu : 0x00070007u, magic = 0x64006400u;
    u4 ones = u4{0x3c003c00u, 0x3c003c00u, 0x3c003c00u, 0x3c003c00u};
    asm volatile("" : "+v"(mask), "+v"(magic), "+v"(ones.x), "+v"(ones.y), "+v"(ones.z), "+v"(ones.w));

    // weak block: 32 columns at a time, dealt to the waves; the first of a wave is requested ahead of everything else
    u4 xw[MT], ww[NT];
    const int kpos = max(A.k, 8), nweak = (A.k + 31) >> 5;
    auto load_weak = [&](int b) {
        const int cc = min(32 * b + 8 * kb, kpos - 8);
#pragma unroll
        for (int a = 0; a < MT; ++a)
            xw[a] = *reinterpret_cast<const u4*>(xbase + (size_t)min(16 * a + n, mlast) * xpitch + 2 * min(A.kq + cc, A.kq + A.k - 8));
#pragma unroll
        for (int t = 0; t < NT; ++t) ww[t] = *reinterpret_cast<const u4*>(A.weak[li] + (size_t)min(o0 + 16 * t + n, oc - 1) * A.k + cc);
    };
    auto mul_weak = [&](int b) {
        const bool live = 32 * b + 8 * kb < A.k;   // both operands: nothing past the block may meet the zeros of the other
        const u4 z = u4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const u4 wl = live ? ww[t] : z;
#pragma unroll
            for (int a = 0; a < MT; ++a) acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(live ? xw[a] : z), as_h8(wl), acc[a][t], 0, 0, 0);
        }
    };

    load_weak(wave);
    if (2 * wave >= A.ng) mul_weak(wave);
    else {
        const int npair = (A.ng + 1) >> 1, npw = (npair - wave + KS - 1) / KS;
        const int ngw = 2 * npw - ((A.ng & 1) && wave + (npw - 1) * KS == npair - 1 ? 1 : 0);
        auto group = [&](int i) { return 2 * ((i >> 1) * KS + wave) + (i & 1); };
        {
            load_par(wave);
            if constexpr (F == W4) load_codes(wave);
            load_x(group(0));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (F != W4) {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    load_w(0, t, group(0));
                    load_w(1, t, group(1));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            mul_weak(wave);
        }
        // group i: its codes are in set i % 2, its activations reach LDS while group i - 1 is multiplied, its codes a step earlier
        auto step = [&](int i, auto set_c) {
            constexpr int SET = decltype(set_c)::value;
            const int g = group(i);
            u4 xa[MT][4];
            __builtin_amdgcn_sched_barrier(0);
            // even groups wait for all that was requested (3-bit: but the codes), odd ones leave what was requested behind their
            // activations: the next pair's codes
            wait_vm<F == W4 ? (SET == 0 ? 0 : 2 * NT) : (SET == 0 ? 2 * NT : 0)>();
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (SET == 0) {
                asm volatile("" : "+v"(ps), "+v"(pz));   // (used behind the wait, not ahead of it)
                put_par();
            }
            wave_lds_fence();
#pragma unroll
            for (int a = 0; a < MT; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int xn = min(n, 4 * XR - 1);   // (rows that were not fetched stand for rows past M)
                    xa[a][q] = *reinterpret_cast<const u4*>(mine + (16 * a + xn) * 256 + (((4 * kb + q) ^ xn) << 4));
                }
            if constexpr (SET == 0) {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const u2 v = *reinterpret_cast<const u2*>(par + 8 * (16 * t + n));
                    zs[0][t] = v.x;
                    zs[1][t] = v.y;
                    if constexpr (F == W4) {
#pragma unroll
                        for (int e = 0; e < 2; ++e) wq[e][t] = *reinterpret_cast<const u4*>(codes + (16 * t + n) * 128 + (((4 * e + kb) ^ (n >> 1)) << 4));
                    }
                }
            }
            wave_lds_fence();
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): all is in registers before its place is filled again
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (SET == 0) load_par((i >> 1) * KS + KS + wave);
            load_x(group(i + 1));
            __builtin_amdgcn_sched_barrier(0);   // (the odd group's wait counts the requests behind these)
            if constexpr (SET == 0 && F == W4) load_codes((i >> 1) * KS + KS + wave);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t wshift = F == W3_TEN ? shift_of(g) : 0u;
            if (128 * g + 128 > A.kq) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool live = 128 * g + 32 * kb + 8 * q < A.kq;
#pragma unroll
                    for (int a = 0; a < MT; ++a) xa[a][q] = live ? xa[a][q] : u4{0u, 0u, 0u, 0u};
                }
            }
            if constexpr (!AS_THEY_LIE) {
#pragma unroll
                for (int a = 0; a < MT; ++a)
#pragma unroll
                    for (int q = 0; q < 4; ++q) xa[a][q] = permute_x(xa[a][q]);
            }
            f4 sx[MT];
#pragma unroll
            for (int a = 0; a < MT; ++a) sx[a] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int a = 0; a < MT; ++a) sx[a] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(xa[a][q]), as_h8(ones), sx[a], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const u4 w = wq[SET][t];
                f4 tmp[MT];
#pragma unroll
                for (int a = 0; a < MT; ++a) tmp[a] = f4{0.f, 0.f, 0.f, 0.f};
                Codes3 c3;
                if constexpr (F != W4) c3.take<F>(w, wshift);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t wi = w[q], w4 = wi >> 4;
                    u4 c;
#pragma unroll
                    for (int p = 0; p < 4; ++p) c[p] = ((F != W4 ? c3.bits(4 * q + p) : (AS_THEY_LIE ? neighbours(wi, w4, p) : wi >> (4 * p))) & mask) | magic;
#pragma unroll
                    for (int a = 0; a < MT; ++a) tmp[a] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(xa[a][q]), as_h8(c), tmp[a], 0, 0, 0);
                }
                if constexpr (SET == 1 && F != W4) {
                    load_w(0, t, group(i + 1));
                    load_w(1, t, group(i + 2));
                }
                const h2 p = __builtin_bit_cast(h2, zs[SET][t]);
                const float sf = (float)p.y, cz = -(1024.f + (float)p.x);
#pragma unroll
                for (int a = 0; a < MT; ++a)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[a][t][e] = fmaf(sf, fmaf(cz, sx[a][e], tmp[a][e]), acc[a][t][e]);
            }
        };
        int i = 0;
#pragma clang loop unroll(disable)
        for (; i + 1 < ngw; i += 2) {
            step(i, std::integral_constant<int, 0>{});
            step(i + 1, std::integral_constant<int, 1>{});
        }
        if (i < ngw) step(i, std::integral_constant<int, 0>{});
    }

    for (int b = wave + KS; b < nweak; b += KS) {
        load_weak(b);
        mul_weak(b);
    }

    // An infinite activation makes a group's sum x (1024 + q) and its Sx infinite alike, and their difference no number where
    // x s (q - z) is an infinity.  Outputs that come out as no number are therefore taken again from the products x w that are not
    // finite, which alone decide.  A wave does it, a row of its tile at a time: it looks through the row's quantized columns, 1024
    // per turn, and forms the products of the groups in which something is not finite, lane (n, kb) for channel n and the group's
    // columns 32 kb .. + 31.  (4096 x 11008, one infinity late in one of 40 rows: 22 us -> 32; the whole sum in plain order by a lane
    // per output: 2180.)  want: the channels asked for.
    auto repair_row = [&](int m, int col, uint32_t want) {
        const unsigned char* x = reinterpret_cast<const unsigned char*>(A.X + (size_t)m * A.ldx);
        const int o = min(o0 + col, oc - 1);
        const unsigned char* words = reinterpret_cast<const unsigned char*>(A.qweight[li] + (size_t)o * A.stride);
        const __half *sc = A.scales[li] + (size_t)o * A.gs, *zp = A.zeros[li] + (size_t)o * A.gs, *wk = A.weak[li] + (size_t)o * A.k;
        float r = 0.f;
        auto add = [&](float p) { r += p - p == 0.f ? 0.f : p; };
        auto settled = [&]() {   // every channel asked for is no number already
            uint64_t b = __ballot(r != r);
            b |= b >> 32;
            b |= b >> 16;
            return ((uint32_t)b & want) == want;
        };
        for (int j = 8 * kb; j < A.k; j += 32) {
            const h8 xv = as_h8(*reinterpret_cast<const u4*>(x + 2 * (size_t)(A.kq + j))), wv = as_h8(*reinterpret_cast<const u4*>(wk + j));
#pragma unroll
            for (int e = 0; e < 8; ++e) add((float)xv[e] * (float)wv[e]);
        }
        auto code3 = [](const unsigned char* row, int j) -> uint32_t {   // the code of column j, one at a time
            const uint32_t* p = reinterpret_cast<const uint32_t*>(row);
            if (F == W3_TEN) return (p[j / 10] >> (3 * (j % 10))) & 7u;
            const int w0 = (3 * j) >> 5, sh = (3 * j) & 31;
            return ((sh > 29 ? (p[w0] >> sh) | (p[w0 + 1] << (32 - sh)) : p[w0] >> sh)) & 7u;
        };
        auto not_finite = [](u4 v) {
            bool f = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) f = f || (v[e] & 0x7c00u) == 0x7c00u || (v[e] & 0x7c000000u) == 0x7c000000u;
            return f;
        };
#pragma clang loop unroll(disable)
        for (int c0 = 0; c0 < A.kq && !settled(); c0 += 1024) {
            u4 v[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) v[t] = *reinterpret_cast<const u4*>(x + 2 * (size_t)min(c0 + 512 * t + 8 * lane, A.kq - 8));
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const uint64_t found = __ballot(not_finite(v[t]));   // (columns past Kq repeat the row's last 8)
#pragma clang loop unroll(disable)
                for (int s = 0; s < 4; ++s) {
                    const int g = (c0 >> 7) + 4 * t + s;
                    if (g >= A.ng || ((found >> (16 * s)) & 0xffffu) == 0) continue;
                    const float a = __half2float(sc[g]), b = __half2float(zp[g]);
                    u4 w = u4{0u, 0u, 0u, 0u};
                    if constexpr (F == W4) w = *reinterpret_cast<const u4*>(words + 64 * (size_t)g + 16 * kb);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int c = 128 * g + 32 * kb + 8 * q;
                        const h8 xv = as_h8(*reinterpret_cast<const u4*>(x + 2 * (size_t)min(c, A.kq - 8)));
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (c < A.kq) add((float)xv[e] * (a * ((float)(F == W4 ? (w[q] >> (4 * e)) & 15u : code3(words, c + e)) - b)));
                    }
                }
            }
        }
        r += __shfl_xor(r, 16);
        return r + __shfl_xor(r, 32);
    };

    // the waves' partial tiles meet in LDS (each in its wave's piece); wave w sums tiles w, w + KS, ...
    wait_vm<0>();   // (the last step's requests, of a group past the wave's last, go there too)
    __half* Y = A.Y[li] + (size_t)m0 * A.ldy[li] + o0;
    const int64_t ldy = A.ldy[li];
    __syncthreads();
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            *reinterpret_cast<f4*>(mine + ((a * NT + t) << 10) + 16 * lane) = acc[a][t];
    __syncthreads();
    for (int q = wave; q < MT * NT; q += KS) {
        f4 y = f4{0.f, 0.f, 0.f, 0.f};
        for (int w = 0; w < KS; ++w) {
            const f4 p = *reinterpret_cast<const f4*>(lds + (size_t)w * WB + (q << 10) + 16 * lane);
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] += p[e];
        }
        const int row = 16 * (q / NT) + 4 * kb, col = 16 * (q % NT) + n;
        const float any = (y[0] + y[1]) + (y[2] + y[3]);   // (no number as well where two infinities cancel: looked at one by one below)
        if (__builtin_expect(A.ng > 0 && __ballot(any != any) != 0, 0)) {
#pragma clang loop unroll(disable)
            for (int i = 0; i < 16; ++i) {   // row 4 b + e of the tile
                const int b = i >> 2, e = i & 3;
                const float mine_y = e == 0 ? y[0] : (e == 1 ? y[1] : (e == 2 ? y[2] : y[3]));
                const uint32_t want = (uint32_t)(__ballot(mine_y != mine_y && row + e <= mlast && o0 + col < oc) >> (16 * b)) & 0xffffu;
                if (want == 0) continue;
                const float r = repair_row(m0 + row - 4 * kb + i, col, want);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (t == e && kb == b && y[t] != y[t] && r - r != 0.f) y[t] = r;
            }
        }
        // lane (n, kb) holds rows 4 kb .. 4 kb + 3 of channel n; a 4 x 4 transpose inside each quad of lanes gives it
        // channels 4 (n / 4) .. + 3 of row 4 kb + n % 4: one 8-byte store
        const uint32_t p0 = pack2(y[0], y[1]), p1 = pack2(y[2], y[3]);
        const bool hi = (lane & 2) != 0, odd = (lane & 1) != 0;
        auto swap2 = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, false); };   // lane ^ 2
        auto swap1 = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, false); };   // lane ^ 1
        const uint32_t other = swap2(hi ? p0 : p1);
        const uint32_t lo2 = hi ? other : p0, hi2 = hi ? p1 : other;   // channels (n % 4) & 1 and + 2 of the quad, this lane's two rows
        const uint32_t lo1 = swap1(lo2), hi1 = swap1(hi2);
        const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
        // even lane: (own row-0, neighbour's row-0); odd lane: (neighbour's row-1, own row-1)
        const uint32_t q0 = __builtin_amdgcn_perm(lo1, lo2, sel), q1 = __builtin_amdgcn_perm(hi1, hi2, sel);
        const int a = q / NT, t = q % NT;
        const int m = 16 * a + 4 * kb + (n & 3), o = 16 * t + 4 * (n >> 2);
        if (m <= mlast && o0 + o + 4 <= oc) *reinterpret_cast<u2*>(Y + (size_t)m * ldy + o) = u2{q0, q1};
        else if (F != W4 && m <= mlast) {   // (4-bit layers come with whole eights of channels)
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (o0 + o + e < oc) reinterpret_cast<uint16_t*>(Y + (size_t)m * ldy + o)[e] = (uint16_t)((e < 2 ? q0 : q1) >> (16 * (e & 1)));
        }
    }
}

template <int MT, int NT, Fmt F, int XR>
hipError_t launch_mid(const MidArgs& A, int KS, hipStream_t s) {
    static bool attr = false;
    const size_t lds_bytes = (size_t)KS * (mid_piece(MT, NT, F == W4) + NT * 128);
    if (lds_bytes > 160 * 1024) return hipErrorInvalidValue;
    if (!attr) {
        hipError_t e = hipFuncSetAttribute((const void*)fwd_mid_kernel<MT, NT, F, XR>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr = true;
    }
    fwd_mid_kernel<MT, NT, F, XR><<<8 * ceil_div((int64_t)A.n_tiles * A.tiles_m, 8), 64 * KS, lds_bytes, s>>>(A);
    return hipGetLastError();
}

}  // namespace

// (Rows are addressed with 32-bit offsets from the panel's first: 48 rows of up to 2^24 elements.)
bool fwd_mid_supported(const Layer& L, int64_t M, int64_t ldx) {
    if (L.g != 128 || (L.kq % 8) != 0 || (L.k % 8) != 0 || ldx > QEFT_MAX_DIM) return false;
    if (L.bits == 3) return M > 0 && L.kq >= 8 && (!L.dense || 12 * L.ng <= L.stride);   // (dense: a lane reads 12 bytes of a group, so whole groups fit the padded row)
    return M > 1 && (L.oc % 8) == 0 && (M > 16 || L.kq >= 8);
}

// Up to 96 rows (two panels) always.  Above, by what this kernel's time goes with - tiles of 16 channels x panels for each CU - against the
// tiled kernels', whose few tiles each walk the whole contraction and whose time hardly depends on the rows: up to 5 per CU (672 rows
// were looked at), for up to 192 rows up to 6 and for rows that are short for the tiled kernels' stages more.  With a workspace for a K split the other side is quicker on long rows:
// up to 5120 columns as before, up to 8192 for few channels, and small layers of up to 192 rows, where the split's fixed cost
// (partial tiles, second launch) is more than half of its time.
// us, here against the tiled kernels (in brackets: with the split): 2048 x 2048 at M = 240 / 480 / 640: 10.0 / 13.9 / 18.5 against 14.7 / 15.0 /
// 15.2; 512 x 512 at 240 / 640: 4.8 / 5.7 against 10.0 / 10.1; 1024 x 8192 at 240 / 640: 17.2 / 28.8 against 40 / 41 (27 / 29); 2048 x 8192 at 336 /
// 480: 26.3 / 37.1 against 41 / 42 (29.7 / 33.8); 4096 x 4096 at 97 / 192 / 240 / 288: 17 / 18.5 / 21.6 / 28 against 23 / 24 / 23.8 / 24 (19 / 23 /
// 27.5 / 27.5); 5120 x 5120 at 192 / 240: 25 / 33 against 28 / 28 (26 / 30); 4096 x 11008 at 97 / 192 / 240 / 288: 34 / 38 / 49 / 62 against 62 / 61 / 61 / 61
// (27 / 34 / 40 / 44); 5120 x 13824 at 192: 60 against 77 (44); 6144 x 6144 at 192 / 240: 32 / 41 against 36 / 36.5; but 8192 x 2048 at 97 / 192:
// 18 / 20 against 15 / 16, 11008 x 4096: 40 / 43 against 27 / 39, 13824 x 5120: 50 / 65 against 34 / 49.
// Without a workspace at M = 97 / 144 / 192: 7680 x 8192 36 / 39 / 51 against 48 / 47 / 47, 7680 x 4096 20 / 21 / 28 against 24 / 24 / 25, 7680 x 2048 13.5 / 13.7 / 17.1 against 15.1 /
// 15.3 / 15.3; but 8192 x 8192 49 / 50 / 52 against 48 / 47 / 48.  Short rows: 12288 x 640 10.2 / 10.8 / 12.2 against 11.2 / 15.8 / 17.2, 12288 x 1536 15.7 / 16.2 / 18.1 against
// 15.7 / 21.4 / 21.6, 8192 x 1536 13.0 / 13.3 / 14.6 against 15.6 / 15.7 / 15.7; but 12288 x 1024 12.9 / 13.0 / 14.3 against 11.0 / 14.7 / 14.7, 12288 x 2048 18.5 / 19.0 / 21.5 against
// 15.5 / 20.7 / 21.0.  Wider short rows, M = 120 / 144 / 192: 16384 x 640 - / - / 14.8 against - / - / 17.3, 14336 x 384 - / - / 11.0 against - / - / 13.3, but 20480 x 256 10.5 / 10.9 / 12.9 against 9.9 / 10.8 /
// 11.9; nine to twelve groups where 128-row tiles begin a second: 16384 x 1408 18.1 / 18.5 / 26.2 against 16.8 / 25.4 / 23.9, 14336 x 1408 16.5 / 17.1 / 25.9 against 16.0 / 24.9 / 22.7.
bool fwd_mid_preferred(const Layer& L, int64_t M, bool split_ws) {
    if (M <= 96 || M > 672) return M <= 96;
    const int64_t panels = ceil_div(M, 48), tiles = panels * ceil_div(L.oc, 16);
    if (!split_ws) {
        if (tiles <= 5 * 256 || M > 192) return tiles <= 5 * 256;
        return (L.oc <= 6144 && tiles <= 6 * 256) || (M <= 144 && L.oc <= 7680) || (L.ng <= 5 && L.oc <= 16384) ||
               (L.ng > 8 && L.ng <= 12 && L.oc <= 12288 && (M <= 144 || L.oc <= 9216 || 3 * ceil_div(L.oc, 128) > 256)) ||   // (above 144 rows: 10240 x 1536 17.3 against 16.0, one round of 128 x 64 tiles)
               (L.ng > 8 && L.ng <= 12 && L.oc <= 16384 && M > 128 && M <= 144);
    }
    if (L.oc > 5120) return false;
    if (M <= 192 && panels * L.oc * L.ic <= (int64_t)3 * 5120 * 5120) return true;
    return tiles <= 5 * 256 && (L.ic <= 5120 || (L.ic <= 8192 && L.oc <= 2048 && 2 * tiles <= 7 * 256));
}

// Layers that share their input, without a workspace; alone: each of them takes this kernel by itself.  Otherwise the one launch still gains where no layer is wide
// (each alone would leave the tiled kernels few workgroups), above 144 rows on long rows and while the launch stays short, and where a third panel holds all rows
// and the tiled kernels begin a second tile of 128.  us, one launch against the layers one by one, M = 97 / 144 / 192: 8192 + 2 x 1024 x 8192 50 / 52 / 74 against 78 / 78 / 80;
// 2 x 8192 x 8192 76 / 78 / 99 against 96 / 94 / 96; 2 x 7168 x 7168 64 / 67 / 83.5 against 86 / 84 / 84; 2 x 8192 x 2048 26 / 24 / 34 against 32 / 32 / 33; 8192 + 1024 x 2048
// 18 / 18 / 26 against 22 / 22 / 22; 2 x 11008 x 4096 60 / 63 / 75 against 54 / 75 / 76; 2 x 13824 x 5120 86 / 91 / - against 66 / 94 / -; 12288 + 1024 x 4096 40 / 41.5 / 51 against 37 / 47 / 47;
// 9216 + 1024 x 4096 28 / 30 / 42 against 36 / 39 / 37.
bool fwd_mid_group_preferred(const Layer* Ls, int n, int64_t M) {
    bool alone = true;
    int64_t widest = 0, sum = 0;
    for (int i = 0; i < n; ++i) {
        alone = alone && fwd_mid_preferred(Ls[i], M, false);
        widest = Ls[i].oc > widest ? Ls[i].oc : widest;
        sum += Ls[i].oc;
    }
    if (alone || M > 192) return alone;
    if (M > 144) return widest <= 8192 && sum <= 14336 && Ls[0].ng > 32;
    return widest <= (M > 128 ? 13824 : 8192) || sum <= 10240;
}

// 3-bit layers with room for a copy: up to 96 rows, and while the codes over all panels are few - the copy's pass alone is 4 to 10 us
// and the kernels behind it take as long as for a 4-bit layer.  us, through a copy against here (ten codes a word): 14848 x 4456 at
// M = 48 / 96: 42 / 52 against 25 / 37; 5120 x 5120 at M = 40 / 96 / 192 / 240 / 333: 24 / 27 / 34 / 37 / 45 against 14 / 17 / 28 /
// 34 / 53; 4096 x 4096 at 333 / 500: 32 / 39 against 30 / 44; 2048 x 2048 at 500 / 700 / 1000: 21 / 22 / 22 against 16 / 19 / 29; wide layers
// sooner: 12288 x 640 at 240 / 500: 23 / 29 against 18 / 36.  Layers under 2^20 weights have the fp16
// copy alone: 512 x 512 at 48 / 1000: 17 / 21 against 5 / 7, 1000 x 1000: 49 / 53 against 6 / 12.
// Up to 192 rows wide and long layers too: 11008 x 4096 at M = 97 / 192: 44 / 48 against 35 / 40 (dense 39 / 41 against 35 / 39), 4096 x 11008: 43 / 49
// against 34 / 38, 8192 x 2048: 24 / 24.5 against 17 / 18, 8192 x 8192: 53 / 61 against 46 / 52 (dense 45 / 52 against 46 / 50: left), 13824 x 5120:
// 57 / 66 against 46 / 60.
bool fwd_mid3_preferred(const Layer& L, int64_t M, int64_t ldx) {
    if (!fwd_mid_supported(L, M, ldx)) return false;
    if (M <= 96) return true;
    const int64_t panels = ceil_div(M, 48), weights = (int64_t)L.oc * L.ic;
    if (weights < ((int64_t)1 << 20)) return panels <= 30;
    if (M <= 192 && panels * weights <= (L.dense ? 7 : 11) * (int64_t)(5120 * 5120)) return true;
    return panels <= 15 && panels * weights <= (L.oc <= 5120 ? 5 : 1) * (int64_t)(5120 * 5120);
}

// 4-bit layers at 2 to 16 rows, `tiles` tiles of 16 channels in the launch: here where a row's contraction does not fit the registers of
// one workgroup of the 16-row kernel in one pass (more than 32 groups of 128), except wide launches of long rows, and one tile per CU of shorter
// rows.  us, the 16-row kernel (M = 2: the small-M kernel) against here: 5120 x 5120 at M = 2 / 4 / 8 / 16: 9.3 / 10.3 / 10.9 / 11.5 against 7.5 /
// 7.4 / 7.7 / 8.5; 5120 x 13824: 17.7 / 23.9 / 20.8 / 23.7 against 17.2 / 17.0 / 18.7 / 21.8; 4096 x 11008 at 4 / 8 / 16: 11.6 / 12.9 / 15.4 against
// 10.6 / 11.6 / 13.2; 27648 x 5120 (gate/up) at 2 / 4 / 8: 22.7 / 26.6 / 28.7 against 24.6 / 25.6 / 25.4; 1024 x 8192 at 8: 9.4 against 7.3; 57344 x 8192
// at 4 / 8 / 16: 67 / 77 / 75 against 79 / 76 / 80; at 2, 8192 x 8192: 12.0 against 12.7, 8192 x 28672: 42 against 34; 4096 x 4096 at 2 / 4 / 16: 5.6 / 6.3 / 7.0 against 5.8 / 5.9 / 6.8; but 12288 x 4096 at 8: 10.1
// against 12.6, 22016 x 4096: 14.5 against 16.6.
// Wide launches, 640 to 2048 tiles x 33 to 111 groups looked at (time there over time here): up to 768 tiles 1.0 to 1.5 at every M; 40 groups 0.96 to 1.2;
// M = 3 / 4, 47 to 79 groups 0.81 to 1.07 / 0.85 to 1.02, but M = 4 at 1152 to 1536 tiles 0.97 to 1.32; 95 and 111 groups M = 4 1.0 to 1.4, M = 3 0.83 to 1.1 up to
// 1024 tiles, 0.95 to 1.15 above, 127 groups 1.15; M = 6 to 16, 55 groups and more, 0.95 to 1.05 up to 1024 tiles, above 0.87 to 1.06 (28672 x 8192 at M = 4 / 16: 34 / 38.5 us against 39 / 42.5).
bool fwd_mid_few_preferred(const Layer& L, int64_t M, int64_t ldx, int tiles) {
    if (L.bits != 4 || M < 2 || M > 16 || !fwd_mid_supported(L, M, ldx)) return false;
    if (L.ng <= 32) return M > 2 && tiles <= 256;
    if (M == 2) return tiles <= 320 || (tiles <= 512 && L.ng > 128);
    if (tiles > 2048) return false;
    if (M > 4) return tiles <= 1024 || L.ng <= 48;
    if (tiles <= 768 || L.ng <= 44) return true;
    return M == 4 ? L.ng > 90 || (tiles > 1024 && tiles <= 1536) : L.ng > (tiles > 1024 ? 90 : 120);
}

// Tiles of 16 NT channels and KS waves.  A CU holds one workgroup of eight waves or two of four (registers and LDS), and a workgroup
// reads its whole panel of X whatever its width, so: the narrowest tile whose workgroups are all resident at eight waves,
// else at four, else the widest.  (us at M = 40, KS = 8: 4096 x 4096 NT = 1 / 2: 9.9 / 11.3; 8192 x 8192 NT = 2 / 3 / 4: 21.7 / 24.4 / 30.7;
// 22016 x 4096: KS = 4 and NT = 2 / 3 / 4: 29.4 / 25.4 / 33.2, KS = 8 and NT = 3: 30.2; 27648 x 5120: KS = 4 48 / 43 / 41.)
hipError_t fwd_mid(const Layer* Ls, int n, const __half* X, int64_t M, int64_t ldx, __half* const* Y, const int64_t* ldy, hipStream_t s) {
    const Layer& L = Ls[0];
    const int panels = ceil_div(M, 48), MT = ceil_div(M, (int64_t)panels * 16);
    const int tiles_m = ceil_div(M, 16 * MT);
    auto tiles_at = [&](int nt) {
        int64_t t = 0;
        for (int i = 0; i < n; ++i) t += ceil_div(Ls[i].oc, 16 * nt);
        return t;
    };
    // A grid is counted in threads, in 32 bits, and a larger one runs in part only, without an error: more rows than fit with the narrowest
    // tiles and most waves go in several launches (3-bit layers without a workspace, results of 13 GB and more)
    const int64_t most = 48 * (((int64_t)0xffffffff / 768 - 8) / tiles_at(1));
    if (M > most) {
        for (int64_t m0 = 0; m0 < M; m0 += most) {
            __half* ys[MAX_GROUP];
            for (int i = 0; i < n; ++i) ys[i] = Y[i] + m0 * ldy[i];
            const hipError_t e = fwd_mid(Ls, n, X + m0 * ldx, M - m0 < most ? M - m0 : most, ldx, ys, ldy, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    int NT = 1, KS = 8;
    while (NT < 4 && tiles_at(NT) * tiles_m > 256) ++NT;
    if (tiles_at(NT) * tiles_m > 256) {
        KS = 4;
        NT = tiles_at(3) * tiles_m <= 512 ? 3 : 4;
    }
    // (up to 8 rows, one narrow tile per CU and many groups: a third wave on each SIMD.  us, the 7B block in 4 / 3 bits, the down projection with eight waves / twelve: M = 2 41.6 /
    // 41.1 and 44.4 / 44.1, M = 8 43.7 / 42.9 and 46.8 / 46.5; 3000 x 12000 at 8 8.1 / 7.8; from 16 rows on no better: M = 16 48.6 / 48.7, 2048 x 16384 in 3 bits at 30
    // 16.4 / 17.4; sixteen waves no better than twelve, 4096 x 4096 at 8 6.6 / 6.7)
    if (NT == 1 && KS == 8 && M <= 8 && L.ng >= 64) KS = 12;
    const bool w4 = L.bits == 4;
    const int pairs = (L.ng + 1) / 2, weak = ceil_div(L.k, 32);   // (a wave's least share is two groups, or 32 weak columns)
    // Few pairs leave waves without one, or LDS three waves of four: two waves instead, of which a CU holds four workgroups - three of the widest tile - and the
    // narrowest tile with which all are resident; where none is, one wave, of which 32 channels leave room for eight.  Not for launches that are resident
    // at eight waves, nor where the weak block is most of the work and is better divided by four.  us, before / in twos: 12288 x 640, four groups, at M = 48 / 96 8.4 / 7.5 and
    // 9.6 / 8.8; 16384 x 384 at 17 8.7 / 6.5; 2 x 5504 x 2048 at 97 25.2 / 18.4, 3 x 2048 x 2048 at 192 18.5 / 15.5, 16384 x 1024 at 96 13.8 / 11.7; 32768 x 2048 at 96, not
    // resident, 35.7 / 39.1.  256 weak columns, in twos / fours: 8192 x 768 at 96 9.0 / 7.7, 4096 x 768 at 192 8.7 / 7.4.  Two waves / one: 28672 x 640 at 96 17.9 / 13.9.
    if (w4 && pairs > 0 && ((pairs <= 2 && weak <= 4 && tiles_at(1) * tiles_m > 256) || (pairs <= 8 && MT == 3 && NT == 4 && KS == 4))) {
        int nt = 1;
        while (nt < 4 && tiles_at(nt) * tiles_m > 1024) ++nt;
        if (nt < 4 || tiles_at(4) * tiles_m <= 768) NT = nt, KS = 2;
        else if (pairs <= 2 && tiles_at(2) * tiles_m <= 2048) NT = 2, KS = 1;
    }
    // (up to 4 rows, many tiles: the panel is little and narrow tiles start sooner; 3-bit codes, 12288 x 4096 at M = 2: 9.8 us against 11.4,
    // 15360 x 5120: 14.1 against 15.0, 27648 x 5120: 24.6 against 26.8)
    if (!w4 && M <= 4 && NT >= 3) NT = 1, KS = 4;
    const int fit = 160 * 1024 / (KS == 4 ? 2 : 1) / (mid_piece(MT, NT, w4) + NT * 128);
    KS = KS > fit ? fit : KS;
    // (48 rows and four tiles of 4-bit codes leave LDS for seven waves, two to three on a SIMD; four, one on each, are as quick or quicker.  us, seven against four:
    // 12288 x 4096 at M = 40 19.1 / 17.6, 4096 x 4096 at M = 97 / 192 15.7 / 15.5 and 16.5 / 15.7, 8192 x 2048 at M = 96 12.4 / 11.2, 16384 x 16384 at
    // M = 48 61 / 58, 4096 x 11008 at M = 97 31.4 / 32.6, 8192 x 28672 at M = 96 85.5 / 85.1)
    if (KS == 7) KS = pairs == 5 || pairs == 6 ? pairs : 4;
    // Waves without a pair take weak columns where these are twice as many steps as pairs (eight steps beside six pairs: 3 to 7 % slower), while all workgroups
    // stay resident (eight waves a CU, and LDS).  us, as many waves as pairs / so: 512 x 448, 256 weak
    // columns, at M = 48 5.7 / 4.5, 8192 x 384 at 119 8.1 / 6.8; 3-bit 512 x 384, 128 of them, at 17 4.3 / 3.8; but not resident, 128 weak columns, 28672 x 384 at 96 12.9 / 16.6, 3-bit 12288 x 512 at 119 10.2 / 14.2.
    const auto resident = [&](int waves) {
        const int64_t per_cu = (tiles_at(NT) * tiles_m + 255) / 256;
        return per_cu * waves <= 8 && per_cu * waves * (mid_piece(MT, NT, w4) + NT * 128) <= 160 * 1024;
    };
    if (pairs > 0 && KS > pairs) {
        const int shares = weak >= 2 * pairs ? weak : pairs;
        KS = KS < shares ? KS : shares;
        while (KS > pairs && !resident(KS)) --KS;
    }
    MidArgs A = {};
    int tiles = 0;
    for (int i = 0; i < MAX_GROUP; ++i) {
        const Layer& Li = Ls[i < n ? i : 0];
        A.qweight[i] = Li.qweight;
        A.scales[i] = Li.scales;
        A.zeros[i] = Li.zeros;
        A.weak[i] = Li.k > 0 ? Li.weak : reinterpret_cast<const __half*>(Li.qweight);   // (k = 0: a request whose result is not used)
        A.Y[i] = Y[i < n ? i : 0];
        A.ldy[i] = ldy[i < n ? i : 0];
        A.oc[i] = Li.oc;
        A.tile_begin[i] = i < n ? tiles : INT_MAX;
        if (i < n) tiles += ceil_div(Li.oc, 16 * NT);
    }
    A.n_tiles = tiles;
    A.tiles_m = tiles_m;
    A.X = X;
    A.ldx = ldx;
    A.M = (int)M;
    A.kq = L.kq;
    A.k = L.k;
    A.ng = L.ng;
    A.stride = L.stride;
    A.gs = L.gs;
    using Launch = hipError_t (*)(const MidArgs&, int, hipStream_t);
#define QEFT_MID(MT, F, XR) {launch_mid<MT, 1, F, XR>, launch_mid<MT, 2, F, XR>, launch_mid<MT, 3, F, XR>, launch_mid<MT, 4, F, XR>}
#define QEFT_MID3(F) {QEFT_MID(1, F, 1), QEFT_MID(1, F, 2), QEFT_MID(1, F, 4), QEFT_MID(2, F, 8), QEFT_MID(3, F, 12)}
    static const Launch f4b[5][4] = QEFT_MID3(W4);
    static const Launch f3b[2][5][4] = {QEFT_MID3(W3_TEN), QEFT_MID3(W3_DENSE)};
#undef QEFT_MID3
#undef QEFT_MID
    const int xi = MT > 1 ? MT + 1 : (M <= 4 ? 0 : (M <= 8 ? 1 : 2));
    return (w4 ? f4b[xi] : f3b[L.dense ? 1 : 0][xi])[NT - 1](A, KS, s);
}

}  // namespace qeft
