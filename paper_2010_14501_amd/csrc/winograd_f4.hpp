// What the two one-kernel Winograd F(4x4, 3x3) forms share: the one-dimensional maps, the division of a launch into work items and
// the addresses of a tile's input patch and outputs.
//
//   Y = A^T [ (G g G^T) .* (B^T d B) ] A     per 6x6 input tile d, 3x3 filter g, 4x4 output tile Y
#pragma once
#include "bn_affine.hpp"
#include "buffer_addr.hpp"
#include "kernels.hpp"

namespace monet {

// B^T in twelve multiply-adds
//   B^T = [4 0 -5 0 1 0; 0 -4 -4 1 1 0; 0 4 -4 -1 1 0; 0 -2 -1 2 1 0; 0 2 -1 -2 1 0; 0 4 0 -5 0 1]
__device__ inline void f4_bt(float v0, float v1, float v2, float v3, float v4, float v5, float (&o)[6]) {
    const float p = __builtin_fmaf(-4.0f, v2, v4), q = __builtin_fmaf(-4.0f, v1, v3);
    const float r = v4 - v2, t = v3 - v1;
    o[0] = __builtin_fmaf(4.0f, v0, __builtin_fmaf(-5.0f, v2, v4));
    o[1] = p + q;
    o[2] = p - q;
    o[3] = __builtin_fmaf(2.0f, t, r);
    o[4] = __builtin_fmaf(-2.0f, t, r);
    o[5] = __builtin_fmaf(4.0f, v1, __builtin_fmaf(-5.0f, v3, v5));
}
__device__ inline void f4_g(float g0, float g1, float g2, float (&o)[6]) {
    o[0] = 0.25f * g0;
    o[1] = (-1.0f / 6.0f) * (g0 + g1 + g2);
    o[2] = (-1.0f / 6.0f) * (g0 - g1 + g2);
    o[3] = (1.0f / 24.0f) * g0 + (1.0f / 12.0f) * g1 + (1.0f / 6.0f) * g2;
    o[4] = (1.0f / 24.0f) * g0 - (1.0f / 12.0f) * g1 + (1.0f / 6.0f) * g2;
    o[5] = g2;
}
//   A^T = [1 1 1 1 1 0; 0 1 -1 2 -2 0; 0 1 1 4 4 0; 0 1 -1 8 -8 1]
__device__ inline void f4_at(float m0, float m1, float m2, float m3, float m4, float m5, float (&o)[4]) {
    const float p = m1 + m2, q = m1 - m2, r = m3 + m4, t = m3 - m4;
    o[0] = m0 + p + r;
    o[1] = __builtin_fmaf(2.0f, t, q);
    o[2] = __builtin_fmaf(4.0f, r, p);
    o[3] = __builtin_fmaf(8.0f, t, q) + m5;
}

constexpr int FUSED_TILES = 32;     // tiles per workgroup
constexpr int FUSED_OUT = 64;       // output channels per workgroup
constexpr int FUSED_CUS = 256;      // one workgroup per CU (LDS)

struct FusedGeom {
    int N, H, W, th, tw;
    int64_t T;          // tiles
    int red, outc;      // reduction / output channels
    int nch;            // chunks of the reduction
    int kblocks;        // ceil(outc / 64)
    int64_t items;      // ceil(T / 32) * kblocks
    // Items [main_items, items) are worked as two half items of 32 output channels each (the ragged last round of a launch
    // with few items: a half item takes about 0.6 of a whole one, and twice as many CUs take part).  main_items is a
    // multiple of 8; main_items == items: no item is halved.
    int64_t main_items;
};

// Hardware deals workgroups to the 8 XCDs in turn; item = (id mod 8) * (grid / 8) + id / 8 gives each XCD a
// contiguous share, so that neighbouring tile rows (shared halo) and the channel blocks of one tile range (same input)
// meet in one L2.  The grid is a multiple of 8; items beyond the last one do nothing.
// Every XCD takes its share of the whole items first, then its share of the half items, so that the short ones come
// last everywhere.
struct FusedItem {
    int64_t tb;      // block of 32 tiles
    int ob, nh;      // first block of 32 output channels and how many of them
};
__device__ __forceinline__ bool fused_item(const FusedGeom &gm, FusedItem &it) {
    const int64_t id = blockIdx.x, xcd = id & 7, idx = id >> 3;
    const int64_t pm = gm.main_items >> 3;
    int64_t item;
    int hsel = 0;
    it.nh = 2;
    if (gm.main_items == gm.items) {      // no item is halved: a contiguous share of the items per XCD
        item = xcd * ((int64_t)gridDim.x >> 3) + idx;
        if (item >= gm.items) return false;
    } else if (idx < pm) {
        item = xcd * pm + idx;
    } else {
        const int64_t nhalf = (gm.items - gm.main_items) * 2, pt = (nhalf + 7) >> 3;
        const int64_t j = xcd * pt + (idx - pm);
        if (idx - pm >= pt || j >= nhalf) return false;
        item = gm.main_items + (j >> 1);
        it.nh = 1;
        hsel = (int)(j & 1);
    }
    it.tb = item / gm.kblocks;
    it.ob = 2 * (int)(item - it.tb * gm.kblocks) + hsel;
    return it.ob * 32 < gm.outc;      // else: the second half of a last, half-empty channel block
}

// Geometry and grid of a launch; throws for shapes beyond the kernels' 32-bit offsets.
inline int64_t fused_geometry(FusedGeom &gm, const ConvShape &cs, bool adjoint, int chunk) {
    gm.N = cs.N; gm.H = cs.H; gm.W = cs.W;
    gm.th = (cs.H + 3) / 4; gm.tw = (cs.W + 3) / 4;
    gm.T = (int64_t)cs.N * gm.th * gm.tw;
    gm.red = adjoint ? cs.K : cs.C;
    gm.outc = adjoint ? cs.C : cs.K;
    gm.nch = gm.red / chunk;
    gm.kblocks = (gm.outc + FUSED_OUT - 1) / FUSED_OUT;
    gm.items = (gm.T + FUSED_TILES - 1) / FUSED_TILES * gm.kblocks;
    // the ragged last round: at most half a round of whole items beyond a multiple of the CU count becomes at most one
    // round of half items
    gm.main_items = gm.items;
    if (gm.items % FUSED_CUS && gm.items % FUSED_CUS <= FUSED_CUS / 2) gm.main_items = gm.items - gm.items % FUSED_CUS;      // also a launch of at most half a round
    const int64_t grid = gm.main_items == gm.items ? (gm.items + 7) / 8 * 8 : gm.main_items + ((gm.items - gm.main_items) * 2 + 7) / 8 * 8;
    if (gm.T < 1 || gm.T >= 0x7fffffffll || grid >= 0x7fffffffll || (int64_t)(cs.N * (int64_t)cs.H + 8) * cs.W * std::max(gm.red, gm.outc) * 4 >= ((int64_t)1 << 32) - 65536)
        throw KernelError("conv_winograd_fused: shape out of range (input and output must have fewer than 2^32 bytes each)");
    return grid;
}

// winograd_pieces.hip: whether a layer's products take two fp16 pieces per operand, and its launches
bool winograd_pieces_applies(const ConvShape &cs, bool adjoint);
void conv_winograd_pieces(hipStream_t st, const float *in, const float *w, float *out, const ConvShape &cs, bool adjoint, bool accumulate, float *ws,
                          const BnAffine &bn);

// winograd_wgrad.hip: whether a filter gradient's horizontal maps are made on the way into its GEMMs; floats of one image's vertical maps; estimated microseconds of a chunk
// of images with room for `most` ranges; dU (+)= the transformed filter gradient of the images of `cs`.  `parts`: room for `most` (>= 1) partial results of 36 * K * C floats.
bool winograd_wgrad_applies(const ConvShape &cs);
size_t winograd_wgrad_image_floats(const ConvShape &cs);
int winograd_wgrad_most_images(const ConvShape &cs);      // of one chunk
double winograd_wgrad_estimate(const ConvShape &cs, int images, int most);
void conv_winograd_wgrad_maps(hipStream_t st, const float *x, const float *dy, float *maps, float *dU, float *parts, const ConvShape &cs, int most, bool accumulate);

}  // namespace monet
