// Internal declarations shared by the translation units of libqeft (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "qeft.h"

namespace qeft {

// Everything a kernel needs to know about one stored layer (see qeft.h for the format).
struct Layer {
    int oc, ic, k, bits, g;
    int dense;     // 1: dense 3-bit layout (a row's codes as one bit string), 0: whole codes per word
    int kq;        // ic - k
    int ng;        // groups per row
    int gs;        // row pitch of scales / zeros in elements (ng rounded up to a multiple of 8)
    int words;     // used words per row
    int stride;    // words per row incl. padding (multiple of 4)
    int once;      // 1 (the 4-bit copy of a 3-bit layer): the tiled kernels round s (q - z) once also where z is fractional
    const uint32_t* qweight;
    const __half* scales;
    const __half* zeros;
    const __half* weak;
};

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Code of column j of a row of packed words, either layout (the plain definition: conversion and fallback kernels).
__device__ __forceinline__ uint32_t code_at(const Layer& L, const uint32_t* __restrict__ row, int j) {
    if (L.dense) {
        const int bit = 3 * j, w0 = bit >> 5, sh = bit & 31;
        uint32_t v = row[w0] >> sh;
        if (sh > 29) v |= row[w0 + 1] << (32 - sh);   // the code straddles two words (never the row's last one)
        return v & 7u;
    }
    const int per = (L.bits == 4) ? 8 : 10;
    return (row[j / per] >> (L.bits * (j % per))) & ((1u << L.bits) - 1u);
}

// ---- generic kernels: any shape, bits and alignment; plain loops (generic.hip) ------
hipError_t fwd_generic(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, hipStream_t s);
hipError_t bwd_dx_generic(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s);
hipError_t weak_grad_generic(int oc, int k, const __half* dY, int64_t M, int64_t lddy, const __half* Xw, int64_t ldxw,
                             void* dW, int out_f32, int accumulate, hipStream_t s);

// ---- weak columns at arbitrary channels: gather / scatter through a workspace (irregular.hip) ----
size_t irregular_workspace(int ic, int64_t M);   // [M][IC rounded up to 8] fp16
hipError_t gather_cols(const __half* X, int64_t M, int64_t ldx, const int* perm, int ic, __half* Xs, int64_t ldo, hipStream_t s);
hipError_t scatter_cols(const __half* Ds, int64_t M, const int* perm, int ic, __half* dX, int64_t lddx, hipStream_t s);

// ---- global weak-column selection and offline reordering (reorder.hip) --------------------------
size_t sens_workspace(int d, int64_t tokens);
hipError_t sensitivity(const __half* X, int64_t tokens, int64_t ldx, int d, int n_batch, float* out, float* ws, hipStream_t s);
hipError_t topk_vote(const float* v, int d, int k, int* idx_out, float* s_global, hipStream_t s);
hipError_t weak_order(const int* idx, int k, int d, int* perm, hipStream_t s);
hipError_t gather_rows16(const __half* W, int64_t ldw, const int* perm, int rows, int src_rows, int cols, __half* out, int64_t ldo,
                         hipStream_t s);

hipError_t merge_weak(const __half* tuned, const __half* base, int64_t oc, int k, const int* idx, int target_cols,
                      __half* target, int64_t ldt, hipStream_t s);

// ---- format conversion (pack.hip) ----------------------------------------------------
hipError_t pack_rtn(const Layer& L, const __half* W, int64_t ldw, uint32_t* qweight, __half* scales, __half* zeros,
                    __half* weak, hipStream_t s);
bool pack_search_supported(const Layer& L, int64_t ldw, const void* W);
hipError_t pack_search(const Layer& L, const __half* W, int64_t ldw, int n_grid, float step, uint32_t* qweight,
                       __half* scales, __half* zeros, __half* weak, hipStream_t s);
hipError_t pack_codes(const Layer& L, const uint8_t* codes, const __half* scales_in, const __half* zeros_in,
                      const __half* weak_in, uint32_t* qweight, __half* scales, __half* zeros, __half* weak, hipStream_t s);
hipError_t unpack(const Layer& L, uint8_t* codes, __half* scales, __half* zeros, __half* weak, hipStream_t s);
// The whole mixed weight as fp16 [OC][IC] (IC a multiple of 8): s (q - z) rounded once, then the weak block.
hipError_t dequantize_fp16(const Layer& L, __half* out, hipStream_t s);
// The codes of a 3-bit layer in the 4-bit layout, [OC][stride4] words of which words4 hold codes (Kq a multiple of 8).
hipError_t expand3(const Layer& L, uint32_t* out, int words4, int stride4, hipStream_t s);

// ---- decode path: fused dequant matrix-vector product for M <= 16 (gemv.hip) -------------
bool gemv_supported(const Layer& L, int64_t M, int64_t ldx);
hipError_t gemv_fwd(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, hipStream_t s);
// Several layers that share the input (same IC, k, bits and group size; any OC each) in one
// launch of the small-M kernel: its row tiles are those of layer 0, then layer 1, ...
constexpr int MAX_GROUP = 4;
struct GroupTail {            // layers 1 .. 3 of a group (layer 0 travels as the kernel's Layer)
    const uint32_t* qweight[MAX_GROUP - 1];
    const __half* scales[MAX_GROUP - 1];
    const __half* zeros[MAX_GROUP - 1];
    const __half* weak[MAX_GROUP - 1];
    __half* Y[MAX_GROUP - 1];
    int64_t ldy[MAX_GROUP - 1];
    int oc[MAX_GROUP - 1];
    int tile_begin[MAX_GROUP - 1];   // first 16-row tile of the layer; INT_MAX when absent
};
// Decode with the activations in original channel order, gathered through perm inside the kernel
// (weak columns at arbitrary channels); *handled = false when the shape does not fit that kernel.
hipError_t gemv_fwd_perm(const Layer& L, const int* perm, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy,
                         hipStream_t s, bool* handled);
// *handled = false (and nothing launched) when the shapes do not fit the one-launch kernel
hipError_t gemv_fwd_group(const Layer* Ls, int n, const __half* X, int64_t M, int64_t ldx, __half* const* Y,
                          const int64_t* ldy, hipStream_t s, bool* handled);

// Decode at M = 1: rows per wavefront, activations in registers (gemv_dot.hip).  Ls[0 .. n) share the input;
// perm (or nullptr) gathers the activations from original channel order.  *handled = false: not this kernel's shape.
hipError_t gemv_dot_fwd(const Layer* Ls, int n, const int* perm, const __half* X, __half* const* Y, hipStream_t s, bool* handled);

// ---- forward between the decode sizes and the large GEMM (gemm_mid.hip); Ls[0 .. n) share the input ----
bool fwd_mid_supported(const Layer& L, int64_t M, int64_t ldx);
bool fwd_mid_preferred(const Layer& L, int64_t M, bool split_ws);   // split_ws: the caller's workspace holds the partial tiles of the GEMM's K split
bool fwd_mid_group_preferred(const Layer* Ls, int n, int64_t M);   // one launch for all of them, without a workspace
bool fwd_mid_few_preferred(const Layer& L, int64_t M, int64_t ldx, int tiles);
bool fwd_mid3_preferred(const Layer& L, int64_t M, int64_t ldx);     // a 3-bit layer's codes as they are, rather than a copy in the caller's workspace
hipError_t fwd_mid(const Layer* Ls, int n, const __half* X, int64_t M, int64_t ldx, __half* const* Y, const int64_t* ldy, hipStream_t s);

// A weak-block gradient to take along with an input gradient, where the kernels chosen for that have room for it beside their own work (done is
// set then).  ws: the caller's workspace, its first `used` bytes taken.
struct WeakGrad {
    int oc, k;
    const __half* Xw;
    int64_t ldxw;
    void* dW;
    int out_f32, accumulate;
    unsigned char* ws;
    size_t ws_bytes, used;
    bool done;
};

// ---- forward and input gradient in tiles of 128 channels x 64 / 128 rows (gemm_tile.hip) for layers the GEMMs below support.
// split_ws: the caller's workspace holds the partial tiles of the GEMM's split ----
bool fwd_tile_preferred(const Layer& L, int64_t M, int64_t ldx, bool split_ws);
bool dx_tile_preferred(const Layer& L, int64_t M, int64_t lddy, bool split_ws);
// Of the two copies of a 3-bit layer, N (4-bit codes) and D (fp16), whether N is the one to multiply (never where its kernel would
// round s (q - z) twice); split_n, split_d: room for the split behind either
bool fwd_copy4_preferred(const Layer& N, const Layer& D, int64_t M, int64_t ldx, bool split_n, bool split_d);
bool dx_copy4_preferred(const Layer& N, const Layer& D, int64_t M, int64_t lddy, bool split_n, bool split_d);
hipError_t fwd_tile(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, hipStream_t s);
hipError_t dx_tile(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s, WeakGrad* g = nullptr);

// ---- input gradient of few rows in tiles of 32 or 64 channels x 32 to 128 rows (dx_panel.hip), for layers the GEMMs below support ----
double dx_panel_estimate(const Layer& L, int64_t M, bool split);   // us, beside a split's or another; more than any call takes where the tiles do not all find a CU
bool dx_panel_preferred(const Layer& L, int64_t M, int64_t lddy, bool split_ws);
hipError_t dx_panel(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, hipStream_t s, WeakGrad* g = nullptr);

// ---- prefill / fine-tune path: MFMA GEMMs (gemm.hip) ---------------------------------------
bool gemm_fwd_supported(const Layer& L, int64_t M);
// The register kernels address a panel's rows (256 at most) by 32-bit byte offsets from its first.  What they do not reach - a pitch of more than 8.4
// million elements under 256 rows - is the LDS-staged kernels', whose row addresses are of 64 bits.
inline bool panel_offsets_fit(int64_t rows, int64_t ld) { return ld <= (int64_t)1 << 32 && ((rows < 256 ? rows : 256) - 1) * 2 * ld + 128 <= (int64_t)1 << 32; }
// The forward's GEMM with weights in registers: at least a stage of quantized columns (what is left of them, whole words, goes with the weak block), or whole stages of fp16 ones.
inline bool fwd_in_registers(const Layer& L) { return L.kq >= 64 ? L.kq % 8 == 0 : (L.kq == 0 && L.k > 0 && L.k % 64 == 0); }
inline bool fwd_in_registers(const Layer& L, int64_t M, int64_t ldx) { return fwd_in_registers(L) && panel_offsets_fit(M, ldx) && panel_offsets_fit(L.oc, L.k); }
// ws: optional device workspace of gemm_fwd_split_workspace() bytes (16-byte aligned); with it, launches of few tiles, or with a
// sparsely filled last round of tiles, split K (for dX: the weight rows) of those tiles
hipError_t gemm_fwd(const Layer& L, const __half* X, int64_t M, int64_t ldx, __half* Y, int64_t ldy, void* ws, hipStream_t s);
size_t gemm_fwd_split_workspace(const Layer& L, int64_t M);
// what a GEMM with a workspace would do: ways a tile is split, 64-wide stages per way, tiles, and whether only the last round's are
struct GemmSplit {
    int splits, stages, tiles;
    bool tail;
};
GemmSplit gemm_fwd_split(const Layer& L, int64_t M);
GemmSplit gemm_dx_split(const Layer& L, int64_t M);
bool gemm_dx_supported(const Layer& L, int64_t M);
// The input gradient's GEMM with weights in registers: whole stages of 64 rows, blocks of 8 weak channels; its tiles cover dx_columns columns.
inline bool dx_in_registers(const Layer& L) { return L.oc % 64 == 0 && L.k % 8 == 0 && (L.kq % 128 == 0 || (L.kq >= 128 && L.kq % 8 == 0)); }
inline bool dx_in_registers(const Layer& L, int64_t M, int64_t lddy) { return dx_in_registers(L) && panel_offsets_fit(M, lddy); }
inline int dx_columns(const Layer& L) { return L.k > 0 ? (L.kq + 127) / 128 * 128 + L.k : L.ic; }
hipError_t gemm_dx(const Layer& L, const __half* dY, int64_t M, int64_t lddy, __half* dX, int64_t lddx, void* ws, hipStream_t s, WeakGrad* g = nullptr);
size_t gemm_dx_split_workspace(const Layer& L, int64_t M);
bool weak_grad_mfma_supported(int oc, int k, int64_t M);
size_t weak_grad_mfma_workspace(int oc, int k, int64_t M);
hipError_t weak_grad_mfma(int oc, int k, const __half* dY, int64_t M, int64_t lddy, const __half* Xw, int64_t ldxw,
                          void* dW, int out_f32, int accumulate, void* ws, hipStream_t s);

// dW = the sum of the strips' partial slabs, in their order
hipError_t weak_grad_reduce(const float* part, int splits, int64_t n, void* dW, int out_f32, int accumulate, hipStream_t s);

}  // namespace qeft
