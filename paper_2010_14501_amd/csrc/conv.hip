// Convolution forward, input-gradient and weight-gradient as implicit GEMMs on the matrix cores of gfx950, NHWC fp32
// activations, KRSC fp32 filters; fp32 products from bf16 instructions (v_mfma_f32_32x32x16_bf16), see below.
//
//   forward : Y[m, k]   = sum_{r,s,c} X[n, p*st+r-pad, q*st+s-pad, c] * W[k, r, s, c]     m = (n,p,q)
//   dgrad   : dX[m, c]  = sum_{r,s,k} dY[n, (h+pad-r)/st, (w+pad-s)/st, k] * W[k, r, s, c] m = (n,h,w)
//   wgrad   : dW[k, j]  = sum_{m}     dY[m, k] * X[n, p*st+r-pad, q*st+s-pad, c]           j = (r,s,c)
//
// These are the convolution operator and the two backward operators it is split into in the
// paper's Appendix D (parameter-gradient, then input-gradient).  wgrad with splits > 1 writes
// one partial result per split into a workspace and sums them in split order: the workspace /
// time trade-off the schedule chooses between (Section 4, "Forward/Backward Operator
// Optimization").
//
// One workgroup computes a (64*WM) x (32*WN) tile with WM*WN waves, each wave a 64x32 sub-tile as two 32x32 MFMA blocks.  The
// reduction runs in steps of 16, double-buffered through LDS: while step t is multiplied, step t+1 is split and written
// to the other LDS buffer, and the loads of step t+2 (t+3) are issued into the registers it leaves.  LDS holds each operand as three
// planes of bf16 pieces, two neighbouring reduction indices per 32-bit word; an operand contiguous along its row / column index
// in memory is paired on the way in.
//
// What bounds it: on large layers the power limit (3x3, 256 -> 256, 56x56, batch 176: 205 TFLOP/s = 1.23 PFLOP/s of bf16
// instructions at 1.4 - 1.7 GHz; torch's own bf16 matmul of 8192 reaches 1.14, of 16384 1.36), against 134 TFLOP/s with the fp32
// instruction; on small ones the length of one step (0.7 - 0.8 us from load to barrier), so that half of the peak needs two
// workgroups per CU; on layers with few channels memory.
//
// The position of a reduction step -- (r, s, c0) forward, (tap, k0) dgrad, (n, p, q) of each
// staged row for wgrad -- is carried from step to step by increments; no integer division is
// executed inside the main loop of the aligned ("fast") variants.
//
// dgrad with stride st > 1 runs one GEMM per residue class (h mod st, w mod st) of the input
// position: within a class only the filter taps r = r0 + st*i, s = s0 + st*j contribute, so no
// multiply-by-zero work is issued (a 3x3 stride-2 layer does 9 taps in total, not 36).
//
// Workgroup ids are remapped so that consecutive work items (same activation rows, neighbouring
// filter columns) run on the same XCD and share its L2: hardware deals workgroups to the 8 XCDs
// round-robin, so logical item = (id mod 8) * (grid/8) + id / 8.  A work item is (tile, reduction
// split) with the tile index fastest, so a launch with few tiles and many splits (weight
// gradients) still spreads over all XCDs and the tiles of one split share their operand rows.
#include <type_traits>
#include <utility>

#include "bf16_pieces.hpp"
#include "bn_affine.hpp"
#include "buffer_addr.hpp"
#include "kernels.hpp"
#include "tile_stats.hpp"

namespace monet {

typedef float floatx16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int BK = 16;        // reduction step
constexpr int KTAB = 256;     // reduction indices in the element-wise forward loader's table
constexpr int NUM_XCD = 8;

// LDS tile of one operand: three planes (h, m, l) of 32-bit words that hold two neighbouring reduction indices.
//   reduction contiguous in memory: [k / 8][row][(k % 8) / 2], one 16-byte read per lane; the second half 64 bytes further on, so that the
//     four lanes that write one row's 16 indices do not meet in a bank
//   row / column contiguous: [k / 2][column], four 4-byte reads per lane
constexpr int kc_half(int rows) { return rows * 4 + 16; }
constexpr int rc_row(int cols) { return cols + 4; }
constexpr int plane_words(bool kc, int n) { return kc ? 2 * kc_half(n) : 8 * rc_row(n); }

enum ConvMode { FWD = 0, DGRAD = 1, WGRAD = 2 };

struct TileArgs {
    const float *a;   // FWD: x, DGRAD: dy, WGRAD: dy
    const float *b;   // FWD: w, DGRAD: w,  WGRAD: x
    float *out;       // FWD: y, DGRAD: dx, WGRAD: dw or workspace
    ConvShape cs;
    int64_t Mg;       // GEMM rows (DGRAD: of residue class 0, the largest)
    int Ng;           // GEMM columns
    int64_t Kg;       // reduction length (DGRAD: recomputed per class)
    int tiles_n;
    int64_t total_tiles;
    int splits;                // reduction splits (>= 1); split z writes partial result z
    int64_t out_elems;         // elements of one (partial) result
    int accumulate;            // FWD/DGRAD, whole result only: add into the output
    // whole result only: its stores pass the caches by.  For results of at least 256 MiB, what the last-level cache holds: whoever
    // reads such a result next starts with a part that has left the cache, and the stores then only push out the operands
    // (1x1, 64 -> 256, 56x56, batch 184: 237 -> 202 us; its input gradient's mirror 226 -> 191).  Smaller results are found in the
    // cache by the next kernel: streaming them too cost MobileNetV2's step 1 %.
    int stream;
    float *stats_part;         // FWD, whole results only: BatchNorm partial statistics of the output (tile_stats.hpp), or null
    BnAffine affine;           // FWD, whole results only: BatchNorm apply step of the output in the epilogue (gamma == null: off)
    unsigned a_bytes, b_bytes;             // operand sizes for the aligned loaders' descriptors: an element that does not exist is a load beyond them and reads zero
    int64_t batch_a, batch_b, batch_out;   // FWD / WGRAD with gridDim.z > 1: z-th GEMM of a batch, operands and result this many floats apart
    // decoding a row index into (image, row, column) without a division: floor(n / Q) = umulhi(n, q_mul) >> q_shift for
    // n < 2^31 (Q >= 2), likewise P (forward rows, the filter gradient's reduction rows) and W, H (input-gradient rows at
    // stride 1); set by launch_tile
    unsigned q_mul, q_shift, p_mul, p_shift, w_mul, w_shift, h_mul, h_shift;
};

template <class F, int... I>
__device__ __forceinline__ void for_each_int(F &f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}

// Where a wave's 64 x 32 results go: first row and column, the launch's (or residue class's) rows, the class's map and place (input gradient), the
// whole result or a slab.
struct TilePlace {
    int64_t row, rows;
    int col, Hc, Wc, ph, pw;
    bool inside;      // the workgroup's tile lies inside the result whole
    bool whole;       // the whole reduction: what is accumulated on is there
    float *out;
};

// Results of a wave: the lane holds column l32 of rows 8*(v/4) + 4*g + v%4 of each 32x32 block.  `stage`: 16 x 32 floats of LDS that are the wave's own.
// ALIGNED: the statistics or the BatchNorm step behind a forward pass may ride along, a filter gradient may take 16-byte stores.
template <int MODE, bool ALIGNED>
__device__ __forceinline__ void write_results(const TileArgs &ta, const floatx16 (&acc)[2], float *stage, const TilePlace &at, int lane) {
    const ConvShape &cs = ta.cs;
    const int l32 = lane & 31, g = lane >> 5;
    const int64_t row0 = at.row, Mg = at.rows;
    const int col0 = at.col, Hc = at.Hc, Wc = at.Wc, ph = at.ph, pw = at.pw;
    float *out = at.out;
    const bool do_acc = MODE != WGRAD && ta.accumulate && at.whole;
    // (Element-wise loaders too, except for the filter gradient: results of few terms are bound by their stores.  1x1, 2 -> 64 input gradient,
    // 416x608, batch 11: 224 us with 4-byte stores, 143 so; accumulating 686 and 346.)
    if ((ALIGNED || MODE != WGRAD) && (ta.Ng & 3) == 0) {
        // Vector path: each wave transposes its 64x32 result through a private 16x32 LDS patch, four
        // passes of 16 rows, and writes whole 16-byte pieces, 128 contiguous bytes per row.
        const bool want_stats = ALIGNED && MODE == FWD && ta.stats_part != nullptr;
        LaneStats ls;
        ls.init();
        // a lane writes the same four columns in every pass: one pair of BatchNorm coefficients each
        const bool want_affine = ALIGNED && MODE == FWD && ta.affine.gamma != nullptr;
        float bn_a[4] = {1, 1, 1, 1}, bn_b[4] = {0, 0, 0, 0};
        if (MODE == FWD && want_affine) {
            const int c0 = col0 + 4 * (lane & 7);
            if (c0 < ta.Ng) {
#pragma unroll
                for (int j = 0; j < 4; ++j) bn_affine_coeffs(ta.affine.gamma, ta.affine.beta, ta.affine.stats, ta.Ng, c0 + j, bn_a[j], bn_b[j]);
            }
        }
        // the sign code of a ReLU applied here: per row one half word (32 columns) per wave; the values are read once more
        // from the LDS patch with lane = column, two rows at a time, so that one ballot is two half words
        const bool want_mask = MODE == FWD && want_affine && ta.affine.relu && ta.affine.mask != nullptr && col0 < ta.Ng;
        float bn_ac = 1.0f, bn_bc = 0.0f;
        if (MODE == FWD && want_mask) bn_affine_coeffs(ta.affine.gamma, ta.affine.beta, ta.affine.stats, ta.Ng, col0 + l32, bn_ac, bn_bc);
        // A tile that lies inside the result whole (all but the last row of tiles and, for widths that are no multiple
        // of the tile, the last column) writes through buffer addressing: the descriptor starts at the tile, a lane's
        // byte offset inside the tile never changes and the row of a pass is a scalar offset, so a store costs no vector
        // instruction for its address and none for a bounds test.
        const bool inside = at.inside && ta.Ng < (1 << 24) && !(MODE == DGRAD && cs.stride > 1);
        const unsigned row_bytes = (unsigned)ta.Ng * 4u;
        const int64_t tile_at = (row0) * ta.Ng + col0;
        const __amdgpu_buffer_rsrc_t r_out = buffer_of(out + tile_at);
        const __amdgpu_buffer_rsrc_t r_relu = buffer_of(MODE == FWD && ta.affine.relu_out ? ta.affine.relu_out + tile_at : out + tile_at);
        const unsigned t_voff = (unsigned)(lane >> 3) * row_bytes + 16u * (unsigned)(lane & 7);
        const bool past_caches = MODE != WGRAD && ta.stream;
        auto put4 = [&](__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, bf4 v) {
            if (past_caches) buffer_store4_stream(r, voff, soff, v);      // uniform over the launch
            else buffer_store4(r, voff, soff, v);
        };
        auto emit = [&](auto whole_tile) {
            constexpr bool IN = decltype(whole_tile)::value;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int mi = q >> 1, vbase = 8 * (q & 1);
#pragma unroll
                for (int vv = 0; vv < 8; ++vv) stage[(8 * (vv >> 2) + 4 * g + (vv & 3)) * 32 + l32] = acc[mi][vbase + vv];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int idx = lane + 64 * i, rl = idx >> 3, c4 = idx & 7;
                    float4 val = *(const float4 *)&stage[rl * 32 + 4 * c4];
                    const int64_t row = row0 + 16 * q + rl;
                    const int col = col0 + 4 * c4;
                    if (IN || (row < Mg && col < ta.Ng)) {
                        const unsigned t_soff = (unsigned)(16 * q + 8 * i) * row_bytes;
                        int64_t orow = row;
                        if (!IN && MODE == DGRAD && cs.stride > 1) {
                            // rows are bounded below 2^31 by the host: 32-bit divisions
                            const unsigned r32 = (unsigned)row, t = r32 / (unsigned)Wc, n = t / (unsigned)Hc;
                            const int wc = (int)(r32 - t * (unsigned)Wc), hc = (int)(t - n * (unsigned)Hc);
                            orow = ((int64_t)n * cs.H + (hc * cs.stride + ph)) * cs.W + (wc * cs.stride + pw);
                        }
                        float4 *dst = (float4 *)(out + orow * ta.Ng + col);
                        if (do_acc) {
                            float4 o;
                            if (IN) { const bf4 t = buffer_load4(r_out, t_voff, t_soff); o = make_float4(t.x, t.y, t.z, t.w); }
                            else o = *dst;
                            val.x += o.x; val.y += o.y; val.z += o.z; val.w += o.w;
                        }
                        if (MODE == FWD && want_affine)
                            val = float4{bn_affine(val.x, bn_a[0], bn_b[0]), bn_affine(val.y, bn_a[1], bn_b[1]), bn_affine(val.z, bn_a[2], bn_b[2]),
                                         bn_affine(val.w, bn_a[3], bn_b[3])};
                        if (MODE == FWD && want_affine && ta.affine.relu) {
                            const float4 rv = float4{relu_clamp(val.x, ta.affine.relu), relu_clamp(val.y, ta.affine.relu),
                                                     relu_clamp(val.z, ta.affine.relu), relu_clamp(val.w, ta.affine.relu)};
                            if (ta.affine.relu_out) {
                                if (IN) put4(r_relu, t_voff, t_soff, bf4{rv.x, rv.y, rv.z, rv.w});
                                else *(float4 *)(ta.affine.relu_out + orow * ta.Ng + col) = rv;
                            } else val = rv;
                        }
                        if (IN) put4(r_out, t_voff, t_soff, bf4{val.x, val.y, val.z, val.w});
                        else *dst = val;
                    }
                }
                if (MODE == FWD && want_stats) {
                    // the statistics' own assignment: lanes of a column group take rows (lane / 8) % 4 + 4 i of the pass, in order (the upper
                    // 32 lanes repeat the lower ones)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int rl = ((lane >> 3) & 3) + 4 * i;
                        const float4 val = *(const float4 *)&stage[rl * 32 + 4 * (lane & 7)];
                        if (!IN) {
                            if (row0 + 16 * q + rl < Mg && col0 + 4 * (lane & 7) < ta.Ng) ls.add(val.x, val.y, val.z, val.w);
                        } else if (q == 0 && i == 0) ls.add_first(val.x, val.y, val.z, val.w);
                        else ls.add_next(val.x, val.y, val.z, val.w);
                    }
                }
                if (MODE == FWD && want_mask) {      // uniform over the wave
                    unsigned half = 0;
#pragma unroll
                    for (int rr = 0; rr < 8; ++rr) {
                        const float e = bn_affine(stage[(2 * rr + g) * 32 + l32], bn_ac, bn_bc);
                        const bool pass = ta.affine.relu == 2 ? (e > 0.0f && e < 6.0f) : e > 0.0f;
                        const unsigned long long word = __ballot(pass);
                        if (lane == 2 * rr) half = (unsigned)word;
                        if (lane == 2 * rr + 1) half = (unsigned)(word >> 32);
                    }
                    const int64_t mrow = row0 + 16 * q + lane;       // lanes 0 .. 15 hold the half words of the pass's rows
                    if (lane < 16 && mrow < Mg) ((unsigned *)ta.affine.mask)[(mrow * ta.Ng + col0) >> 5] = half;
                }
            }
        };
        if (inside) emit(std::true_type{});
        else emit(std::false_type{});
        if (MODE == FWD && want_stats) {
            // this wave's 64 rows are one row group of the statistics; lanes l, l^8, l^16, l^24 share their columns
            float n, mean[4], m2[4];
            merge_lane_stats<8>(ls, lane, n, mean, m2);
            const int64_t first = row0;
            if (first < Mg) store_group_stats<8>(ta.stats_part, first / STAT_ROWS, ta.Ng, col0 + 4 * (lane & 7), lane, mean, m2);
        }
        return;
    }
    const int col = col0 + l32;
    if (col >= ta.Ng) return;
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            // four consecutive rows: with strided residue classes, the first one's place is decoded and the others' follow from it
            const int64_t first = row0 + mi * 32 + 8 * v4 + 4 * g;
            int wc = 0, hc = 0, n = 0;
            if (MODE == DGRAD && cs.stride > 1) {   // class row (n,hc,wc) -> position (n, hc*st+ph, wc*st+pw)
                const unsigned r32 = (unsigned)first, t = r32 / (unsigned)Wc;      // rows are bounded below 2^31 by the host
                n = (int)(t / (unsigned)Hc);
                wc = (int)(r32 - t * (unsigned)Wc), hc = (int)(t - (unsigned)n * (unsigned)Hc);
            }
            float *dst[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                int64_t orow = first + j;
                if (MODE == DGRAD && cs.stride > 1) {
                    orow = ((int64_t)n * cs.H + (hc * cs.stride + ph)) * cs.W + (wc * cs.stride + pw);
                    if (++wc == Wc) {
                        wc = 0;
                        if (++hc == Hc) { hc = 0; ++n; }
                    }
                }
                dst[j] = out + orow * ta.Ng + col;
            }
            float r[4] = {acc[mi][4 * v4], acc[mi][4 * v4 + 1], acc[mi][4 * v4 + 2], acc[mi][4 * v4 + 3]};
            if (do_acc) {      // the four loads together
                float o[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = first + j < Mg ? *dst[j] : 0.0f;
#pragma unroll
                for (int j = 0; j < 4; ++j) r[j] += o[j];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (first + j < Mg) *dst[j] = r[j];
        }
}

// TAG names the use, in profiles and for the order of a batch's work items: 0 a convolution, 1 / 2 / 3 the batched GEMMs of a Winograd forward / input gradient /
// filter gradient
// FAST: 0 element-wise loaders, 1 aligned loaders, 2 aligned loaders of a 1x1 layer whose last reduction step is partly
// empty (a kernel of its own: the two tests per step would cost the other layers 2 %, measured on ResNet-50), 3 aligned
// loaders of a larger filter over channels that are a multiple of 4 but not of 16: a step straddles filter taps, every
// lane carries the tap and channel of its four reduction indices (5x5 filter, 24 -> 64 channels, 14x14 maps, batch 320:
// 160 -> 38 us forward, 134 -> 82 us input gradient against the element-wise loaders), 4 as 1 with a single register stage, for reductions of at
// most six steps (1x1, C -> 256, 56x56, batch 184, one stage against two: C = 32: 123 and 138 us, 64: 173 and 197, 96: 225 and 242; beyond the
// line the gain shrinks: 112: 256 and 268, 128: 316 and 328, 192: 421 and 430, 256 level; level at every C on 14x14)
// Registers: 128 in the eight-wave tiles and for FAST 2 and 4 (four waves per SIMD), where the narrow tile's FAST 2 spills 2 forward and 5 in the
// input gradient; up to 168 in the others, where the 64x64 filter gradient spills 1.
// KS: groups of waves that share a tile and take the reduction's steps in turn, each with operand tiles of its own in LDS; their sums are added at the end.
template <int MODE, int WM, int WN, int FAST, int TAG = 0, int KS = 1>
__global__ __launch_bounds__(64 * WM * WN * KS, KS == 1 && (WM * WN < 4 || (WM * WN == 4 && FAST != 2 && FAST != 4)) ? 3 : 4) void conv_tile_kernel(TileArgs ta) {
    static_assert(KS == 1 || (MODE != WGRAD && FAST == 1), "aligned forward passes and input gradients only");
    // Register stages of the aligned variants: loads run this many steps ahead of the split.  The tiles of at most four waves take
    // two at three waves per SIMD (1x1, 1024 -> 256, 14x14, batch 184: 123 against 142 us with one), the larger ones, and short
    // reductions, which live from many workgroups at once (64 -> 256, 56x56: 214 against 245 us), one at four (128 registers).
    constexpr int STAGES = (FAST == 1 || FAST == 3) && WM * WN <= 4 && KS == 1 && !(FAST == 3 && WN == 1) ? 2 : 1;
    constexpr int BM = 64 * WM, BN = 32 * WN, NT = 64 * WM * WN;
    constexpr bool A_KC = (MODE != WGRAD);          // A operand reduction-contiguous?
    constexpr bool B_KC = (MODE == FWD);
    constexpr int A_PL = plane_words(A_KC, BM), B_PL = plane_words(B_KC, BN);
    constexpr int A_SZ = 3 * A_PL, B_SZ = 3 * B_PL;
    // float4 slots of an operand's tile per thread; a tile with fewer slots than threads is loaded twice (same value, same place)
    constexpr int SA = BM * 4, SB = BN * 4, LA = SA >= NT ? SA / NT : 1, LB = SB >= NT ? SB / NT : 1;
    __shared__ __attribute__((aligned(16))) unsigned As_all[KS][2][A_SZ];
    __shared__ __attribute__((aligned(16))) unsigned Bs_all[KS][2][B_SZ];
    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    unsigned (&As)[2][A_SZ] = As_all[group];
    unsigned (&Bs)[2][B_SZ] = Bs_all[group];
    __shared__ int redo;     // the pieces do not hold this tile's numbers: once more with the fp32 matrix instruction
    // First layers (3 input channels): the element-wise forward loader looks the (r, s, c) of a reduction index up
    // instead of dividing (measured 925 -> 815 us on the ResNet-50 stem).  Only the 64 columns wide tiles have
    // the LDS to spare (2 KiB), and those are the ones results up to 64 channels wide, i.e. every first layer, use.
    constexpr bool HAS_KTAB = !FAST && MODE == FWD && BN == 64;
    __shared__ int2 ktab[HAS_KTAB ? KTAB : 1];   // x = ((r*W + s)*C + c), y = r | s << 8, or y < 0 beyond the reduction
    // Aligned filter gradient: the output positions of four reduction steps, decoded once for the whole workgroup by the 64 lanes of one
    // wave: x = byte offset of the position's window in the (shifted) input tensor, y = bit per filter tap that falls inside the
    // image.  Two such tables: one is written while the other is read.
    constexpr bool ROWTAB = FAST && MODE == WGRAD;
    constexpr int TABLE = 4 * BK;
    __shared__ uint2 rowtab[ROWTAB ? 2 * TABLE : 1];

    if (MODE != DGRAD) {   // batched GEMMs (the 16 products of a Winograd convolution) share one launch
        ta.a += (int64_t)blockIdx.z * ta.batch_a;
        ta.b += (int64_t)blockIdx.z * ta.batch_b;
        ta.out += (int64_t)blockIdx.z * ta.batch_out;
    }
    const ConvShape &cs = ta.cs;
    const int tid = threadIdx.x - group * NT, lane = tid & 63, wave = tid >> 6;      // within the group
    const int wm = wave / WN, wn = wave % WN;
    const int l32 = lane & 31, g = lane >> 5;
    const int tid_a = SA < NT ? tid % SA : tid, tid_b = SB < NT ? tid % SB : tid;

    // XCD-aware order of the (tile, split) work items
    const int nsplit = ta.splits;
    // all indices of work items and reduction steps are 32 bits wide (bounded by the host): a 64-bit division is 150 scalar
    // instructions, and four of them per wave were a microsecond of every tile
    const unsigned tiles = (unsigned)ta.total_tiles;
    // Each GEMM of a batch deals its shares from another XCD on: the shares without an item (12 items in shares of two: the last two) would fall to the same
    // XCDs 36 times.  Winograd filter gradient, batch 184 of 14x14, 256 -> 256: 230 and 185 us; batch 176 of 56x56, 256 -> 256: 2082 and 2014; where memory bounds
    // it (112x112, 128 -> 128) level.  Shares that are even already stay where they are (8, 16, 32 items: 0.6 - 1.0 % slower turned, single ones 10 %;
    // 9 - 11 items 0.91 of the time, others 0.94 - 1.0).
    const unsigned first = MODE == DGRAD || TAG == 0 || tiles * (unsigned)nsplit % NUM_XCD == 0 ? 0u : blockIdx.z;      // (an input gradient's classes read the same rows: each stays with its XCD; a launch
    // that is no batch has nothing to turn, and without the sum its code is faster: 3x3 stride 2, 128 -> 128, 56x56, batch 184, filter gradient 273 and 269 us)
    const unsigned item = (blockIdx.x + first) % NUM_XCD * (gridDim.x / NUM_XCD) + blockIdx.x / NUM_XCD;
    if (item >= tiles * (unsigned)nsplit) return;
    const int split = nsplit > 1 ? (int)(item / tiles) : 0;
    const unsigned logical = item - (unsigned)split * tiles;
    const int64_t tile_m = logical / (unsigned)ta.tiles_n;
    const int tile_n = (int)(logical - (unsigned)tile_m * (unsigned)ta.tiles_n);
    const int64_t row0 = tile_m * BM;
    const int col0 = tile_n * BN;
    const int RSC = (int)cs.RSC();

    // ---------------- DGRAD: residue class of this launch slice
    int64_t Mg = ta.Mg, Kg = ta.Kg;
    int ph = 0, pw = 0, r0 = 0, s0 = 0, nr = cs.R, ns = cs.S, bh = cs.pad, bw = cs.pad, Hc = cs.H, Wc = cs.W;
    // blockIdx.z = residue class (DGRAD only)
    if (MODE == DGRAD) {
        const int st = cs.stride;
        const int cls = blockIdx.z;
        ph = cls / st;
        pw = cls % st;
        Hc = (cs.H - ph + st - 1) / st;
        Wc = (cs.W - pw + st - 1) / st;
        r0 = (ph + cs.pad) % st;
        s0 = (pw + cs.pad) % st;
        nr = r0 < cs.R ? (cs.R - r0 + st - 1) / st : 0;
        ns = s0 < cs.S ? (cs.S - s0 + st - 1) / st : 0;
        bh = (ph + cs.pad - r0) / st;
        bw = (pw + cs.pad - s0) / st;
        Mg = (int64_t)cs.N * Hc * Wc;
        Kg = (int64_t)nr * ns * cs.K;
        if (row0 >= Mg) return;
        if (Kg == 0 && ta.accumulate && nsplit == 1) return;       // this class receives no contribution
    }

    // reduction range of this workgroup: split z takes steps [z*sps, (z+1)*sps) (possibly none: it
    // then contributes zeros to its partial result)
    int kt0 = 0, kt1 = (int)(((unsigned)Kg + BK - 1) / BK);
    if (nsplit > 1) {
        const int sps = (int)(((unsigned)kt1 + (unsigned)nsplit - 1) / (unsigned)nsplit);
        kt0 = min(split * sps, kt1);       // split * sps < steps + splits * splits / 16: far below 2^31
        kt1 = min(kt0 + sps, kt1);
    }

    // ---------------- per-slot constants of the A loader
    // reduction-contiguous A (FWD / DGRAD): slot = (row, float4 j): idx = tid + s*NT, row = idx/4, j = idx%4
    // row-contiguous operand (L slots per thread, n rows or columns): slots 2u, 2u + 1 are the float4 at the same column of two
    // neighbouring reduction indices, which share a word in LDS; with one slot per thread the neighbour sits n / 4 lanes away
    auto rc_red = [&](int t, int s, int L, int n) { return L == 1 ? t / (n / 4) : 2 * ((t + (s >> 1) * NT) / (n / 4)) + (s & 1); };
    auto rc_col4 = [&](int t, int s, int L, int n) { return L == 1 ? t % (n / 4) : (t + (s >> 1) * NT) % (n / 4); };
    int64_t a_base[LA];   // FWD/DGRAD: image base + j4; WGRAD: unused
    int a_h0[LA], a_w0[LA];
    bool a_ok[LA];
#pragma unroll
    for (int s = 0; s < LA; ++s) {
        int idx = tid_a + s * NT;
        if (A_KC) {
            int64_t m = row0 + idx / 4;
            a_ok[s] = m < Mg;
            int64_t mm = a_ok[s] ? m : 0;
            if (MODE == FWD) {
                const unsigned m32 = (unsigned)mm;                                 // rows are bounded below 2^31 by the host
                const unsigned t = cs.Q == 1 ? m32 : __umulhi(m32, ta.q_mul) >> ta.q_shift;
                const unsigned nn = cs.P == 1 ? t : __umulhi(t, ta.p_mul) >> ta.p_shift;
                int q = (int)(m32 - t * (unsigned)cs.Q);
                int p = (int)(t - nn * (unsigned)cs.P);
                int n = (int)nn;
                a_h0[s] = p * cs.stride - cs.pad;
                a_w0[s] = q * cs.stride - cs.pad;
                a_base[s] = (int64_t)n * cs.H * cs.W * cs.C + (idx % 4) * 4;
            } else {   // DGRAD: m = (n, hc, wc) within the residue class
                const unsigned m32 = (unsigned)mm;
                unsigned t, nn;
                if (cs.stride == 1) {      // the one class is the tensor itself: Wc = W, Hc = H
                    t = cs.W == 1 ? m32 : __umulhi(m32, ta.w_mul) >> ta.w_shift;
                    nn = cs.H == 1 ? t : __umulhi(t, ta.h_mul) >> ta.h_shift;
                } else {
                    t = m32 / (unsigned)Wc;
                    nn = t / (unsigned)Hc;
                }
                int wc = (int)(m32 - t * (unsigned)Wc);
                int hc = (int)(t - nn * (unsigned)Hc);
                int n = (int)nn;
                a_h0[s] = hc + bh;      // p = a_h0 - tap row
                a_w0[s] = wc + bw;
                a_base[s] = (int64_t)n * cs.P * cs.Q * cs.K + (idx % 4) * 4;
            }
        } else {
            int k4 = rc_col4(tid_a, s, LA, BM);
            a_h0[s] = rc_red(tid_a, s, LA, BM);                    // red row within the step
            a_w0[s] = (int)(row0 + k4 * 4);                 // first out-channel of the float4
            a_ok[s] = a_w0[s] < cs.K;
            a_base[s] = 0;
        }
    }
    // ---------------- per-slot constants of the B loader
    int b_i0[LB], b_i1[LB], b_i2[LB];
    bool b_ok[LB];
    // WGRAD: (n, p, q) of the row each slot stages in the next step
    int w_n[LB], w_p[LB], w_q[LB];
#pragma unroll
    for (int s = 0; s < LB; ++s) {
        int idx = tid_b + s * NT;
        w_n[s] = w_p[s] = w_q[s] = 0;
        if (B_KC) {          // FWD: slot = (filter k, float4 j)
            b_i0[s] = col0 + idx / 4;
            b_ok[s] = b_i0[s] < cs.K;
            b_i1[s] = (idx % 4) * 4;
            b_i2[s] = 0;
        } else {             // slot = (red row, float4 along the column index)
            int c4 = rc_col4(tid_b, s, LB, BN);
            int col = col0 + c4 * 4;
            b_i0[s] = rc_red(tid_b, s, LB, BN);                    // red row within the step
            if (MODE == DGRAD) {
                b_i1[s] = col;                              // input channel c
                b_ok[s] = col < cs.C;
                b_i2[s] = 0;
            } else {         // WGRAD: column = (r,s,c)
                b_ok[s] = col < RSC;
                int cc = b_ok[s] ? col : 0;
                int rs = cc / cs.C;
                b_i1[s] = (rs / cs.S) * cs.W + (rs % cs.S);   // r*W + s: pixel offset of the tap
                b_i2[s] = cc % cs.C;                          // c
                // tap (r, s) packed for the bounds test
                b_i1[s] |= (rs / cs.S) << 24;
                b_i2[s] |= (rs % cs.S) << 24;
            }
        }
    }

    // ---------------- aligned forward / input-gradient loaders: buffer addressing
    // A matrix instruction leaves room for about six vector instructions, which the splits use up, so an address is split into what
    // differs between lanes and never changes (a 32-bit byte offset per slot, computed once) and what changes from step
    // to step and is the same for every lane (the filter tap and the channel block: a scalar offset).  The descriptor of
    // the activation operand starts `a_shift` floats before the tensor, enough for the most negative tap offset, and ends with the
    // tensor: an absent element (padding, rows beyond the tensor) is a load at BUFFER_ABSENT, which reads zero.
    // Bit t of a_taps says whether tap t of the slot exists.  The host takes this path only for tensors the 32-bit
    // offsets can span and for filters of at most 32 taps.
    unsigned a_voff[LA], a_taps[LA], b_voff[LB];
    int64_t a_shift = 0;
    if (FAST && MODE != WGRAD) {
        const int row = MODE == FWD ? cs.W : cs.Q, inner = MODE == FWD ? cs.C : cs.K;
        const int tr = MODE == FWD ? cs.R : nr, ts = MODE == FWD ? cs.S : ns;
        const int64_t back = MODE == FWD ? ((int64_t)cs.pad * row + cs.pad) * inner : 0;                    // most negative slot offset
        const int64_t reach = ((int64_t)(tr > 0 ? tr - 1 : 0) * row + (ts > 0 ? ts - 1 : 0)) * inner;       // largest tap offset
        a_shift = MODE == FWD ? (back > reach ? back : reach) : reach;
#pragma unroll
        for (int s = 0; s < LA; ++s) {
            a_voff[s] = (unsigned)((a_base[s] + ((int64_t)a_h0[s] * row + a_w0[s]) * inner + (MODE == FWD ? a_shift : 0)) * 4);
            unsigned rows = 0, cols = 0, taps = 0;
            for (int r = 0; r < tr; ++r)
                if (MODE == FWD ? (unsigned)(a_h0[s] + r) < (unsigned)cs.H : (unsigned)(a_h0[s] - r) < (unsigned)cs.P) rows |= 1u << r;
            for (int c = 0; c < ts; ++c)
                if (MODE == FWD ? (unsigned)(a_w0[s] + c) < (unsigned)cs.W : (unsigned)(a_w0[s] - c) < (unsigned)cs.Q) cols |= 1u << c;
            for (int r = 0; r < tr; ++r)
                if ((rows >> r) & 1) taps |= cols << (r * ts);
            a_taps[s] = a_ok[s] ? taps : 0u;      // a row beyond the tensor has no tap
        }
#pragma unroll
        for (int s = 0; s < LB; ++s)
            b_voff[s] = b_ok[s] ? (unsigned)(((int64_t)b_i0[s] * RSC + b_i1[s]) * 4) : BUFFER_ABSENT;
    }
    // Aligned filter gradient: dy rows advance by a scalar offset; the window of an output position comes from the
    // row table, the slot adds its tap and channel and tests its tap's bit.  The input descriptor starts b_shift floats
    // early (a window begins up to `pad` rows and columns before the image).
    unsigned w_tapbit[LB];
    int64_t b_shift = 0;
    if (FAST && MODE == WGRAD) {
        b_shift = ((int64_t)cs.pad * cs.W + cs.pad) * cs.C;
#pragma unroll
        for (int s = 0; s < LA; ++s) a_voff[s] = a_ok[s] ? (unsigned)(((int64_t)a_h0[s] * cs.K + a_w0[s]) * 4) : BUFFER_ABSENT;
#pragma unroll
        for (int s = 0; s < LB; ++s) {
            const int r = b_i1[s] >> 24, ss = b_i2[s] >> 24;
            b_voff[s] = (unsigned)(((int64_t)(b_i1[s] & 0xffffff) * cs.C + (b_i2[s] & 0xffffff)) * 4);
            w_tapbit[s] = b_ok[s] ? 1u << (r * cs.S + ss) : 0u;
        }
    }
    // FAST == 3: reduction index of this lane's float4 (A; FWD's B has the same) or filter row (DGRAD's B) in the step to load, as
    // (tap, channel), and the tap's offset
    struct LaneTap { int c, row, col; unsigned bit, off; };
    constexpr int UB3 = LB == 1 ? 1 : LB / 2;
    LaneTap la3, lb3[UB3];
    __amdgpu_buffer_rsrc_t ra = buffer_of(ta.a - a_shift, ta.a_bytes + (unsigned)a_shift * 4u),
                           rb = buffer_of(ta.b - b_shift, ta.b_bytes + (unsigned)b_shift * 4u);
    int w_t = 0;      // step, counted from the start of the range, that the next load reads
    // Decodes the output positions of reduction steps `step` .. `step` + 3: the last wave alone, no lane switched off on the way
    // (the branch is uniform over the wave, the rest are selects).  Measured: a version in which only 16 lanes ran this code, under
    // a narrowed execution mask while the step's loads were still in flight, now and then lost one row of a step on the two-wave
    // tile shapes when several workgroups shared a compute unit; whole waves do not (kernel test with many short ranges).  With a table
    // per step every step waited for the wave that wrote it (3x3, 256 -> 256, 56x56, batch 176: 4.06 against 3.81 ms).
    auto fill_rows = [&](int step, int table) {
        if (ROWTAB && __builtin_amdgcn_readfirstlane(tid >> 6) == NT / 64 - 1) {
            const int e = lane;
            const int m = step * BK + e;
            const bool in = m < (int)Kg;
            const unsigned m32 = in ? (unsigned)m : 0u;
            const unsigned t = cs.Q == 1 ? m32 : __umulhi(m32, ta.q_mul) >> ta.q_shift;
            const unsigned q = m32 - t * (unsigned)cs.Q;
            const unsigned n = cs.P == 1 ? t : __umulhi(t, ta.p_mul) >> ta.p_shift;
            const unsigned pp = t - n * (unsigned)cs.P;
            const int h0 = (int)pp * cs.stride - cs.pad, w0 = (int)q * cs.stride - cs.pad;
            const int rlo = max(0, -h0), rhi = min(cs.R, cs.H - h0), clo = max(0, -w0), chi = min(cs.S, cs.W - w0);
            const unsigned rows = rhi > rlo ? (unsigned)((1ull << rhi) - (1ull << rlo)) : 0u;
            const unsigned cols = chi > clo ? (unsigned)((1ull << chi) - (1ull << clo)) : 0u;
            unsigned taps = 0;
            for (int r = 0; r < cs.R; ++r) taps |= ((rows >> r) & 1u) ? cols << (r * cs.S) : 0u;
            const unsigned pix = (unsigned)((((int64_t)n * cs.H + h0) * cs.W + w0) * cs.C + b_shift) * 4u;
            rowtab[table * TABLE + e] = make_uint2(in ? pix : 0u, in ? taps : 0u);
        }
    };

    // ---------------- position of the next step to load (uniform over the workgroup)
    int kk0;
    int u_r, u_s, u_c;   // FWD: (r, s, c0); DGRAD: (tap row, tap column, k0)
    auto to_start = [&] {
        kk0 = (kt0 + group) * BK;
        u_r = u_s = u_c = 0;
        if (MODE != WGRAD && kt0 + group > 0) {  // a later reduction split (or group) starts in the middle: locate it once
            const int inner = MODE == FWD ? cs.C : cs.K, cols = MODE == FWD ? cs.S : max(ns, 1);      // (a class without a tap has no step, but a second group)
            const int tap = (int)((unsigned)kk0 / (unsigned)inner);
            u_c = kk0 - tap * inner;
            u_r = tap / cols;
            u_s = tap % cols;
        }
        if constexpr (FAST == 3) {
            auto place = [&](LaneTap &t, int at) {
                const int inner = MODE == FWD ? cs.C : cs.K, cols = MODE == FWD ? cs.S : max(ns, 1), taps = MODE == FWD ? cs.R * cs.S : nr * ns;
                const int tap = at / inner;
                t.c = at - tap * inner;
                t.row = tap / cols;
                t.col = tap - t.row * cols;
                t.bit = tap < taps ? 1u << tap : 0u;
            };
            place(la3, kk0 + (tid % 4) * 4);
            if (MODE == DGRAD) {
#pragma unroll
                for (int u = 0; u < UB3; ++u) place(lb3[u], kk0 + b_i0[LB == 1 ? 0 : 2 * u]);
            }
        }
        if (MODE == WGRAD && !FAST) {
#pragma unroll
            for (int s = 0; s < LB; ++s) {
                const int64_t m = kk0 + b_i0[s];
                const unsigned m32 = m < Kg ? (unsigned)m : 0u, t = m32 / (unsigned)cs.Q;
                w_q[s] = (int)(m32 % (unsigned)cs.Q);
                w_p[s] = (int)(t % (unsigned)cs.P);
                w_n[s] = (int)(t / (unsigned)cs.P);
            }
        }
    };
    to_start();

    const bool use_ktab = HAS_KTAB && (ta.Kg + BK - 1) / BK * BK <= KTAB;
    if (HAS_KTAB && use_ktab) {
        for (int kk = tid; kk < KTAB; kk += NT) {
            int2 e = make_int2(0, -1);
            if (kk < Kg) {
                const int rs = kk / cs.C, c = kk % cs.C;
                const int r = rs / cs.S, ss = rs % cs.S;
                e = make_int2((r * cs.W + ss) * cs.C + c, r | (ss << 8));
            }
            ktab[kk] = e;
        }
        __syncthreads();
    }

    float4 a_regs[STAGES][LA], b_regs[STAGES][LB];
    unsigned long long w_row[LB];       // aligned filter gradient: the table entries of this lane's B slots

    // In the aligned variants every load is issued unconditionally: one of an absent element (padding, rows beyond the tensor) goes
    // to an offset beyond the descriptor and reads zero, so neither a branch around it nor a select behind it is needed.
    int left;                           // reduction indices of the step being loaded (BK but for the last one of some layers)
    bool part_step;
    auto begin_load = [&] {
        if constexpr (FAST == 3) {
            // the tap's offset from the slot's: FWD forwards in the image, DGRAD backwards (the descriptor starts a_shift floats early)
            la3.off = MODE == FWD ? (unsigned)(((la3.row * cs.W + la3.col) * cs.C + la3.c) * 4)
                                  : (unsigned)(((int)a_shift - (la3.row * cs.Q + la3.col) * cs.K + la3.c) * 4);
            if (MODE == DGRAD) {
#pragma unroll
                for (int u = 0; u < UB3; ++u)
                    lb3[u].off = ((unsigned)lb3[u].c * (unsigned)RSC + (unsigned)(((r0 + cs.stride * lb3[u].row) * cs.S + s0 + cs.stride * lb3[u].col) * cs.C)) * 4u;
            }
        }
        // 1x1 layers whose reduction length is a multiple of 4 only: the last step holds `left` < 16 reduction indices
        // (uniform over the workgroup; every other step, and every step of the other layers, is whole)
        left = min((int)Kg - kk0, BK);
        part_step = FAST == 2 && MODE != WGRAD && left < BK;
        if (ROWTAB) {
#pragma unroll
            for (int s = 0; s < LB; ++s) w_row[s] = *(const unsigned long long *)&rowtab[(w_t & 7) * BK + b_i0[s]];
        }
    };
    auto load_a = [&](float4 (&a_reg)[LA], const int s) {
            int idx = tid_a + s * NT;
            float4 v = make_float4(0, 0, 0, 0);
            bool ok;
            if (MODE == FWD) {
                if constexpr (FAST == 3) {
                    const bf4 q = buffer_load4(ra, (a_taps[s] & la3.bit) ? a_voff[s] - (unsigned)(tid % 4) * 16u + la3.off : BUFFER_ABSENT, 0u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (FAST) {
                    // scalar: tap number and offset
                    const unsigned tapoff = (unsigned)(((int64_t)u_r * cs.W + u_s) * cs.C);
                    ok = (a_taps[s] >> (u_r * cs.S + u_s)) & 1u;
                    if (part_step) ok = ok && (idx % 4) * 4 < left;
                    const bf4 q = buffer_load4(ra, ok ? a_voff[s] : BUFFER_ABSENT, (tapoff + (unsigned)u_c) * 4u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (HAS_KTAB && use_ktab) {
                    // branch-free: an element outside the image or the reduction reads the tensor's first word and is zeroed
                    float e[4];
                    const float *pix = ta.a + (a_base[s] - (idx % 4) * 4 + ((int64_t)a_h0[s] * cs.W + a_w0[s]) * cs.C);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int2 t = ktab[(int)kk0 + (idx % 4) * 4 + u];
                        const int h = a_h0[s] + (t.y & 0xff), w = a_w0[s] + ((t.y >> 8) & 0xff);
                        const bool in = a_ok[s] && t.y >= 0 && (unsigned)h < (unsigned)cs.H && (unsigned)w < (unsigned)cs.W;
                        const float got = *(in ? pix + t.x : ta.a);
                        e[u] = in ? got : 0.0f;
                    }
                    v = make_float4(e[0], e[1], e[2], e[3]);
                } else {
                    float e[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        int kk = (int)kk0 + (idx % 4) * 4 + u;
                        if (a_ok[s] && kk < Kg) {
                            int rs = kk / cs.C, c = kk % cs.C;
                            int r = rs / cs.S, ss = rs % cs.S;
                            int h = a_h0[s] + r, w = a_w0[s] + ss;
                            if ((unsigned)h < (unsigned)cs.H && (unsigned)w < (unsigned)cs.W)
                                e[u] = ta.a[a_base[s] - (idx % 4) * 4 + ((int64_t)h * cs.W + w) * cs.C + c];
                        }
                    }
                    v = make_float4(e[0], e[1], e[2], e[3]);
                }
            } else if (MODE == DGRAD) {
                // reduction index = (tap row, tap column, k); FAST: K % 16 == 0 so a step stays inside one tap
                if constexpr (FAST == 3) {
                    const bf4 q = buffer_load4(ra, (a_taps[s] & la3.bit) ? a_voff[s] - (unsigned)(tid % 4) * 16u + la3.off : BUFFER_ABSENT, 0u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (FAST) {
                    // the descriptor starts a_shift floats early: tap (u_r, u_s) lies tapoff floats before the slot's offset
                    const unsigned tapoff = (unsigned)(((int64_t)u_r * cs.Q + u_s) * cs.K);
                    ok = (a_taps[s] >> (u_r * ns + u_s)) & 1u;
                    if (part_step) ok = ok && (idx % 4) * 4 < left;
                    const bf4 q = buffer_load4(ra, ok ? a_voff[s] : BUFFER_ABSENT, ((unsigned)a_shift - tapoff + (unsigned)u_c) * 4u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else {
                    float e[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        int kk = (int)kk0 + (idx % 4) * 4 + u;
                        if (a_ok[s] && kk < Kg) {
                            int tap = kk / cs.K, k = kk % cs.K;
                            int p = a_h0[s] - tap / ns, q = a_w0[s] - tap % ns;
                            if ((unsigned)p < (unsigned)cs.P && (unsigned)q < (unsigned)cs.Q)
                                e[u] = ta.a[a_base[s] - (idx % 4) * 4 + ((int64_t)p * cs.Q + q) * cs.K + k];
                        }
                    }
                    v = make_float4(e[0], e[1], e[2], e[3]);
                }
            } else {   // WGRAD: A[red = m][row = k] = dy[m][k]
                int64_t m = kk0 + a_h0[s];
                if (FAST) {
                    const bf4 q = buffer_load4(ra, a_h0[s] < left ? a_voff[s] : BUFFER_ABSENT, (unsigned)kk0 * (unsigned)cs.K * 4u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (m < Kg) {
                    float e[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (a_w0[s] + u < cs.K) e[u] = ta.a[m * cs.K + a_w0[s] + u];
                    v = make_float4(e[0], e[1], e[2], e[3]);
                }
            }
            a_reg[s] = v;
    };
    auto load_b = [&](float4 (&b_reg)[LB], const int s) {
            float4 v = make_float4(0, 0, 0, 0);
            if (MODE == FWD) {
                if (FAST) {
                    unsigned vo = b_voff[s];
                    if (FAST == 3 && b_i1[s] >= left) vo = BUFFER_ABSENT;
                    if (part_step && b_i1[s] >= left) vo = BUFFER_ABSENT;      // beyond the filter row's end
                    const bf4 q = buffer_load4(rb, vo, (unsigned)kk0 * 4u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else {
                    float e[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (b_ok[s] && kk0 + b_i1[s] + u < Kg) e[u] = ta.b[(int64_t)b_i0[s] * RSC + kk0 + b_i1[s] + u];
                    v = make_float4(e[0], e[1], e[2], e[3]);
                }
            } else if (MODE == DGRAD) {
                // B[red = (tap, k)][col = c] = W[k][r0 + st*tr][s0 + st*ts][c]
                int64_t kk = kk0 + b_i0[s];
                if constexpr (FAST == 3) {
                    // the two slots of a word are filters k, k + 1 of the same tap (K is a multiple of 4)
                    const LaneTap &t = lb3[LB == 1 ? 0 : s >> 1];
                    const bf4 q = buffer_load4(rb, t.bit && b_ok[s] ? t.off + (LB == 1 ? 0u : (unsigned)(s & 1) * (unsigned)RSC * 4u) + (unsigned)b_i1[s] * 4u : BUFFER_ABSENT, 0u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (FAST) {
                    // a step reaches beyond the reduction only in the last step of a 1x1 layer with K % 16 != 0 (part_step)
                    const int r = r0 + cs.stride * u_r, ss = s0 + cs.stride * u_s;
                    unsigned vo = b_voff[s];
                    if (part_step && b_i0[s] >= left) vo = BUFFER_ABSENT;      // a filter beyond the last one
                    const bf4 q = buffer_load4(rb, vo, (unsigned)(((int64_t)u_c * RSC + (r * cs.S + ss) * cs.C) * 4));
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (kk < Kg) {
                    int tap = (int)kk / cs.K, k = (int)kk % cs.K;
                    int r = r0 + cs.stride * (tap / ns), ss = s0 + cs.stride * (tap % ns);
                    const float *src = ta.b + (int64_t)k * RSC + (r * cs.S + ss) * cs.C + b_i1[s];
                    float e[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (b_i1[s] + u < cs.C) e[u] = src[u];
                    v = make_float4(e[0], e[1], e[2], e[3]);
                }
            } else {   // WGRAD: B[red = m][col = (r,s,c)] = x[n, p*st+r-pad, q*st+s-pad, c]
                int64_t m = kk0 + b_i0[s];
                if (FAST) {
                    const unsigned pix = (unsigned)w_row[s], taps = (unsigned)(w_row[s] >> 32);
                    const bf4 q = buffer_load4(rb, (taps & w_tapbit[s]) ? pix + b_voff[s] : BUFFER_ABSENT, 0u);
                    v = make_float4(q.x, q.y, q.z, q.w);
                } else if (m < Kg) {
                    int h0 = w_p[s] * cs.stride - cs.pad, w0 = w_q[s] * cs.stride - cs.pad;
                    const float *img = ta.b + (int64_t)w_n[s] * cs.H * cs.W * cs.C;
                    {
                        float e[4] = {0, 0, 0, 0};
                        int col = col0 + rc_col4(tid_b, s, LB, BN) * 4;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            int cc = col + u;
                            if (cc < RSC) {
                                int rs = cc / cs.C, c = cc % cs.C;
                                int r = rs / cs.S, ss = rs % cs.S;
                                int h = h0 + r, w = w0 + ss;
                                if ((unsigned)h < (unsigned)cs.H && (unsigned)w < (unsigned)cs.W)
                                    e[u] = img[((int64_t)h * cs.W + w) * cs.C + c];
                            }
                        }
                        v = make_float4(e[0], e[1], e[2], e[3]);
                    }
                }
            }
            b_reg[s] = v;
    };
    auto advance = [&] {     // to the next step
        kk0 += BK * KS;
        if constexpr (FAST == 3) {
            auto next = [&](LaneTap &t) {
                const int inner = MODE == FWD ? cs.C : cs.K, cols = MODE == FWD ? cs.S : ns, rows = MODE == FWD ? cs.R : nr;
                t.c += BK;
                while (t.c >= inner) {       // once, or up to four times for 4 .. 12 channels
                    t.c -= inner;
                    if (++t.col == cols) { t.col = 0; ++t.row; }
                }
                t.bit = t.row < rows ? 1u << (t.row * cols + t.col) : 0u;
            };
            next(la3);
            if (MODE == DGRAD) {
#pragma unroll
                for (int u = 0; u < UB3; ++u) next(lb3[u]);
            }
        } else if (MODE != WGRAD && KS > 1) {
            u_c += BK * KS;
            const int inner = MODE == FWD ? cs.C : cs.K, cols = MODE == FWD ? cs.S : ns;
            while (u_c >= inner) { u_c -= inner; if (++u_s == cols) { u_s = 0; ++u_r; } }
        } else if (MODE == FWD) {
            u_c += BK;
            if (u_c >= cs.C) { u_c = 0; if (++u_s == cs.S) { u_s = 0; ++u_r; } }
        } else if (MODE == DGRAD) {
            u_c += BK;
            if (u_c >= cs.K) { u_c = 0; if (++u_s == ns) { u_s = 0; ++u_r; } }
        } else if (FAST) {
            // kk0 now names the step after the one just loaded: if it is the first of a table, the table is written now; every wave
            // finished reading that table four steps ago, and a barrier follows before the next load
            ++w_t;
            if ((w_t & 3) == 0) fill_rows(kk0 / BK, (w_t >> 2) & 1);
        } else {
#pragma unroll
            for (int s = 0; s < LB; ++s) {
                w_q[s] += BK;
                while (w_q[s] >= cs.Q) {
                    w_q[s] -= cs.Q;
                    if (++w_p[s] == cs.P) { w_p[s] = 0; ++w_n[s]; }
                }
            }
        }
    };

    auto load_tiles = [&](auto set) {
        begin_load();
#pragma unroll
        for (int s = 0; s < LA; ++s) load_a(a_regs[decltype(set)::value], s);
#pragma unroll
        for (int s = 0; s < LB; ++s) load_b(b_regs[decltype(set)::value], s);
        advance();
    };

    unsigned lost = 0;      // bits of operands too small to be three pieces

    // One operand's slot (two slots where they share words), split into pieces and written as words of two neighbouring
    // reduction indices.
    auto put_unit = [&](auto kc, auto count, auto width, auto unit, int t, unsigned *dst, const auto &reg) {
        constexpr bool KC = decltype(kc)::value;
        constexpr int L = decltype(count)::value, n = decltype(width)::value, PL = plane_words(KC, n), u = decltype(unit)::value;
        auto pieces = [&](float x, float y) { return split_pair(x, y, lost); };
        if constexpr (KC) {
            const int idx = t + u * NT;
            const float4 v = reg[u];
            const Pieces p = pieces(v.x, v.y), q = pieces(v.z, v.w);
            unsigned *at = dst + ((idx % 4) >> 1) * kc_half(n) + (idx / 4) * 4 + (idx & 1) * 2;
            *(uint2 *)at = make_uint2(p.h, q.h);
            *(uint2 *)(at + PL) = make_uint2(p.m, q.m);
            *(uint2 *)(at + 2 * PL) = make_uint2(p.l, q.l);
        } else if constexpr (L > 1) {
            const float4 v = reg[2 * u], w = reg[2 * u + 1];
            const Pieces p0 = pieces(v.x, w.x), p1 = pieces(v.y, w.y), p2 = pieces(v.z, w.z), p3 = pieces(v.w, w.w);
            unsigned *at = dst + (rc_red(t, 2 * u, L, n) >> 1) * rc_row(n) + rc_col4(t, 2 * u, L, n) * 4;
            *(uint4 *)at = make_uint4(p0.h, p1.h, p2.h, p3.h);
            *(uint4 *)(at + PL) = make_uint4(p0.m, p1.m, p2.m, p3.m);
            *(uint4 *)(at + 2 * PL) = make_uint4(p0.l, p1.l, p2.l, p3.l);
        } else {
            // n / 4 lanes hold one reduction index, the next n / 4 its neighbour: after exchanging the second half of the one with
            // the first half of the other a lane holds both indices of two columns
            static_assert(n == 32 || n == 64 || n == 128, "one slot per thread: 8, 16 or 32 lanes per reduction index");
            const float4 v = reg[0];
            const int red = rc_red(t, 0, L, n);
            unsigned *at = dst + (red >> 1) * rc_row(n) + rc_col4(t, 0, L, n) * 4 + (red & 1) * 2;
            if constexpr (n == 32) {
                // 8 lanes apart: the halves of a row of 16 lanes change places
                auto other = [](float f) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(f), 0x128, 0xf, 0xf, false)); };      // row_ror:8
                const bool odd = red & 1;
                const float g0 = other(odd ? v.x : v.z), g1 = other(odd ? v.y : v.w);
                const Pieces p = pieces(odd ? g0 : v.x, odd ? v.z : g0), q = pieces(odd ? g1 : v.y, odd ? v.w : g1);
                *(uint2 *)at = make_uint2(p.h, q.h);
                *(uint2 *)(at + PL) = make_uint2(p.m, q.m);
                *(uint2 *)(at + 2 * PL) = make_uint2(p.l, q.l);
                return;
            }
            auto swap = [&](float a, float b) {
                if constexpr (n <= 64) return __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
                else return __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            };
            const auto e0 = swap(v.x, v.z), e1 = swap(v.y, v.w);
            const Pieces p = pieces(__uint_as_float(e0[0]), __uint_as_float(e0[1])), q = pieces(__uint_as_float(e1[0]), __uint_as_float(e1[1]));
            *(uint2 *)at = make_uint2(p.h, q.h);
            *(uint2 *)(at + PL) = make_uint2(p.m, q.m);
            *(uint2 *)(at + 2 * PL) = make_uint2(p.l, q.l);
        }
    };
    constexpr int UA = A_KC || LA == 1 ? LA : LA / 2, UB = B_KC || LB == 1 ? LB : LB / 2, UNITS = UA + UB;
    // unit i of the step held in register stage `set` goes to LDS buffer `buf`; `again`: and its registers take the next loads
    auto unit = [&](auto i, int buf, auto set, auto again) {
        constexpr int u = decltype(i)::value;
        float4 (&a_reg)[LA] = a_regs[decltype(set)::value];
        float4 (&b_reg)[LB] = b_regs[decltype(set)::value];
        if constexpr (u < UA) {
            put_unit(std::bool_constant<A_KC>{}, std::integral_constant<int, LA>{}, std::integral_constant<int, BM>{}, std::integral_constant<int, u>{}, tid_a, As[buf], a_reg);
            if constexpr (decltype(again)::value) {
                if constexpr (A_KC || LA == 1) load_a(a_reg, u);
                else { load_a(a_reg, 2 * u); load_a(a_reg, 2 * u + 1); }
            }
        } else {
            put_unit(std::bool_constant<B_KC>{}, std::integral_constant<int, LB>{}, std::integral_constant<int, BN>{}, std::integral_constant<int, u - UA>{}, tid_b, Bs[buf], b_reg);
            if constexpr (decltype(again)::value) {
                if constexpr (B_KC || LB == 1) load_b(b_reg, u - UA);
                else { load_b(b_reg, 2 * (u - UA)); load_b(b_reg, 2 * (u - UA) + 1); }
            }
        }
    };
    auto each_unit = [&](auto f) {
        for_each_int(f, std::make_integer_sequence<int, UNITS>{});
    };
    auto store_tiles = [&](int buf, auto set) {
        each_unit([&](auto i) { unit(i, buf, set, std::false_type{}); });
    };

    // Two sums per result: the h * h terms and the five smaller ones.  A matrix instruction rounds its sum to fp32; the smaller terms'
    // sum is 2^-8 of the result, so that one rounding per 16 products counts.  All six into one sum would be faster by 5 % (half
    // the accumulators, three workgroups per CU), but 1.2 - 1.3 times further from 64 bits than the fp32 matrix instruction, and 3 times for
    // filter gradients over many ranges (the unit's rounding leans towards minus infinity by 0.004 ulp, which the ranges add up).
    floatx16 acc[2], low[2];
    // Fragments of one plane: reduction indices 8g .. 8g+7 of this lane's rows / columns.
    auto fragment = [&](auto kc, auto width, const unsigned *plane, int r) {
        constexpr int n = decltype(width)::value;
        if constexpr (decltype(kc)::value) return __builtin_bit_cast(bf16x8, *(const uintx4 *)(plane + g * kc_half(n) + r * 4));
        else {
            const unsigned *at = plane + 4 * g * rc_row(n) + r;
            return __builtin_bit_cast(bf16x8, uintx4{at[0], at[rc_row(n)], at[2 * rc_row(n)], at[3 * rc_row(n)]});
        }
    };
    struct Rows { bf16x8 b[2]; };      // the wave's 64 rows as two blocks of 32
    auto frag_a = [&](int buf, int p) {
        Rows f;
#pragma unroll
        for (int i = 0; i < 2; ++i) f.b[i] = fragment(std::bool_constant<A_KC>{}, std::integral_constant<int, BM>{}, As[buf] + p * A_PL, wm * 64 + i * 32 + l32);
        return f;
    };
    auto frag_b = [&](int buf, int p) { return fragment(std::bool_constant<B_KC>{}, std::integral_constant<int, BN>{}, Bs[buf] + p * B_PL, wn * 32 + l32); };
    auto term = [&](floatx16 (&sum)[2], const Rows &x, const bf16x8 &y) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) sum[mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.b[mi], y, sum[mi], 0, 0, 0);
    };
    auto compute = [&](int buf) {
        const Rows ah = frag_a(buf, 0), am = frag_a(buf, 1), al = frag_a(buf, 2);
        const bf16x8 bh = frag_b(buf, 0), bm = frag_b(buf, 1), bl = frag_b(buf, 2);
        term(acc, ah, bh); term(low, ah, bm); term(low, am, bh); term(low, am, bm); term(low, ah, bl); term(low, al, bh);
    };
    // One step of the aligned variants: the matrix instructions of the step in LDS buffer `buf`, and between them, unit by unit,
    // the split and LDS write of the next step (register stage `set`) and the loads of a later one into the registers just freed.  A bf16 matrix
    // instruction leaves room for about six vector instructions of the same SIMD (measured: 2.2 PFLOP/s with 0 .. 6 of them,
    // 1.7 with 10); the fences keep the compiler from gathering the splits, which costs 70 registers.
    auto step = [&](int buf, auto set) {
        begin_load();
        const Rows ah = frag_a(buf, 0);
        const bf16x8 bh = frag_b(buf, 0), bm = frag_b(buf, 1);
        const Rows am = frag_a(buf, 1);
        Rows al;
        bf16x8 bl;
        __builtin_amdgcn_sched_barrier(0);
        auto chunk = [&](auto j) {
            constexpr int J = decltype(j)::value;
            if constexpr (J == 0) { term(acc, ah, bh); term(low, ah, bm); }
            else if constexpr (J == 1) { term(low, am, bh); term(low, am, bm); al = frag_a(buf, 2); bl = frag_b(buf, 2); }
            else { term(low, ah, bl); term(low, al, bh); }
            each_unit([&](auto i) {
                if constexpr (decltype(i)::value * 3 / UNITS == J) unit(i, buf ^ 1, set, std::true_type{});
            });
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        chunk(std::integral_constant<int, 0>{}); chunk(std::integral_constant<int, 1>{}); chunk(std::integral_constant<int, 2>{});
        advance();
        __syncthreads();
    };

    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = low[i][v] = 0.0f;
    };
    clear();
    // One product per result (one input channel forward, one output channel in the input gradient, 1x1): the three terms the pieces
    // leave out, up to 2^-24 of it, are more than the fp32 product's rounding, and no sum hides them (normwise 2.63e-8 against 2.55e-8;
    // from two products on the pieces are the closer ones: 2.56e-8 against 3.08e-8).
    const bool single = !FAST && Kg == 1;
    if (tid == 0) redo = single;      // read behind the barriers below
    if (kt0 < kt1 && !single) {
        // a group's turns, as many for each: turns beyond the range multiply zeros
        const int steps = (kt1 - kt0 + KS - 1) / KS;
        if (ROWTAB) {
            fill_rows(kt0, 0);
            __syncthreads();
        }
        const std::integral_constant<int, 0> s0{};
        const std::integral_constant<int, STAGES - 1> s1{};
        auto loading = [&](int t) {      // step t is about to be loaded: beyond the range the loads touch no memory
            if (KS == 1 ? t >= steps : kt0 + group + t * KS >= kt1) {
                ra = buffer_of(ta.a, 0);
                rb = buffer_of(ta.b, 0);
            }
        };
        if (KS > 1) loading(0);
        load_tiles(s0);
        if constexpr (FAST) {
            if constexpr (STAGES == 2) {
                if (steps > 1) load_tiles(s1);
            }
            store_tiles(0, s0);
            if (KS > 1) loading(STAGES);
            if (steps > STAGES) load_tiles(s0);
            __syncthreads();
            int t = 0;
            if constexpr (STAGES == 2) {
                for (; t + 2 < steps; t += 2) {
                    loading(t + 3);
                    step(0, s1);
                    loading(t + 4);
                    step(1, s0);
                }
                if (t + 1 < steps) {
                    loading(t + 3);
                    step(0, s1);
                }
            } else {
                for (; t + 1 < steps; ++t) {
                    loading(t + 2);
                    step(t & 1, s0);
                }
            }
        } else {
            store_tiles(0, s0);
            __syncthreads();
            for (int t = 0; t + 1 < steps; ++t) {
                load_tiles(s0);
                __builtin_amdgcn_sched_barrier(0);
                compute(t & 1);
                __builtin_amdgcn_sched_barrier(0);
                store_tiles((t + 1) & 1, s0);
                __syncthreads();
            }
        }
        compute((steps - 1) & 1);
    }
    auto join = [&] {
#pragma unroll
        for (int i = 0; i < 2; ++i) acc[i] += low[i];
    };
    join();
    // An infinity or a NaN in the result says that an operand held one, that a value near the type's largest rounded to infinity in
    // bf16, or that a product or a sum overflowed: pieces of such numbers do not add up to what fp32 arithmetic gives.  Bits lost in the
    // split say that an operand lies below 2^-110.  Such a tile is worked once more with the fp32 matrix instruction.
    // What that costs (3x3, 256 -> 256, 56x56, batch 32, every tile affected): forward 735 -> 1700 us, the fp32 kernel took 1020;
    // 1x1, 1024 -> 256, 14x14, batch 184: 130 -> 310.  Otherwise: one barrier and 32 additions per tile, one vector instruction per pair of
    // operands (0 - 3 % of a layer).
    {
        float probe[4] = {0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            probe[0] += acc[0][v];
            probe[1] += acc[0][v + 8];
            probe[2] += acc[1][v];
            probe[3] += acc[1][v + 8];
        }
        const float sum = (probe[0] + probe[1]) + (probe[2] + probe[3]);
        if (!(__builtin_fabsf(sum) < __builtin_inff()) || pieces_lost(lost)) redo = 1;
    }
    __syncthreads();       // also: every wave is done with the operand tiles in LDS
    if (redo) {
        ra = buffer_of(ta.a - a_shift, ta.a_bytes + (unsigned)a_shift * 4u);
        rb = buffer_of(ta.b - b_shift, ta.b_bytes + (unsigned)b_shift * 4u);
        clear();
        to_start();
        w_t = 0;
        if (ROWTAB) {
            fill_rows(kt0, 0);
            __syncthreads();
        }
        // One step at a time, nothing overlapped: these tiles are rare.  The operands lie in the first buffer's place as floats,
        // [row][17] where the reduction is contiguous, else [reduction index][column + 4].
        auto whole = [](auto kc, auto width, int red, int r) {
            if constexpr (decltype(kc)::value) return r * (BK + 1) + red;
            else return red * (decltype(width)::value + 4) + r;
        };
        auto put_whole = [&](auto kc, auto count, auto width, int t, float *dst, const auto &reg) {
            constexpr bool KC = decltype(kc)::value;
            constexpr int L = decltype(count)::value, n = decltype(width)::value;
            static_assert((KC ? n * (BK + 1) : BK * (n + 4)) <= 2 * 3 * plane_words(KC, n), "a step's floats fit the two buffers");
#pragma unroll
            for (int s = 0; s < L; ++s) {
                const float e[4] = {reg[s].x, reg[s].y, reg[s].z, reg[s].w};
                const int idx = t + s * NT;
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    dst[KC ? whole(kc, width, (idx % 4) * 4 + u, idx / 4) : whole(kc, width, rc_red(t, s, L, n), rc_col4(t, s, L, n) * 4 + u)] = e[u];
            }
        };
        const std::bool_constant<A_KC> kc_a{};
        const std::bool_constant<B_KC> kc_b{};
        const std::integral_constant<int, BM> rows{};
        const std::integral_constant<int, BN> cols{};
        float *fa = (float *)&As[0][0], *fb = (float *)&Bs[0][0];
        for (int t = kt0 + group; t < kt1 + group; t += KS) {      // as many turns for every group
            if (KS > 1 && t >= kt1) {
                ra = buffer_of(ta.a, 0);
                rb = buffer_of(ta.b, 0);
            }
            load_tiles(std::integral_constant<int, 0>{});
            put_whole(kc_a, std::integral_constant<int, LA>{}, rows, tid_a, fa, a_regs[0]);
            put_whole(kc_b, std::integral_constant<int, LB>{}, cols, tid_b, fb, b_regs[0]);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < BK; k += 2) {
                if (k >= (int)Kg - t * BK) break;      // beyond the reduction
                const float y = fb[whole(kc_b, cols, k + g, wn * 32 + l32)];
#pragma unroll
                for (int mi = 0; mi < 2; ++mi)
                    acc[mi] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[whole(kc_a, rows, k + g, wm * 64 + mi * 32 + l32)], y, acc[mi], 0, 0, 0);
            }
            __syncthreads();
        }
    }

    // ---------------- epilogue
    constexpr int NW = WM * WN;
    static_assert(2 * A_SZ >= NW * 512 || 2 * B_SZ >= NW * 512, "the epilogue's patches fit one operand's tiles");
    __syncthreads();   // every wave has finished reading the operand tiles
    if constexpr (KS > 1) {
        // the other groups' sums come through LDS, one of the two blocks at a time
        float *pass = (float *)&As_all[0][0][0];
        static_assert(sizeof(As_all) >= (KS - 1) * NW * 1024 * 4, "a block of every other group's waves fits the operand tiles");
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (i) __syncthreads();
            if (group > 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) pass[(((group - 1) * NW + wave) * 16 + v) * 64 + lane] = acc[i][v];
            }
            __syncthreads();
            if (group == 0) {
#pragma unroll
                for (int o = 0; o < KS - 1; ++o)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][v] += pass[((o * NW + wave) * 16 + v) * 64 + lane];
            }
        }
        __syncthreads();
        if (group > 0) return;
    }
    float *stage = (float *)(2 * A_SZ >= NW * 512 ? &As[0][0] : &Bs[0][0]) + wave * 512;
    const TilePlace at{row0 + wm * 64, Mg, col0 + wn * 32, Hc, Wc, ph, pw, row0 + BM <= Mg && col0 + BN <= ta.Ng, nsplit == 1, ta.out + (int64_t)split * ta.out_elems};
    write_results<MODE, FAST != 0>(ta, acc, stage, at, lane);
}

// Launches of few results: a workgroup of eight waves per 64 x 32 or 32 x 32 of them, the reduction steps dealt to the waves in turn.  Each wave loads its operands straight
// into the matrix instruction's lanes (eight reduction indices of a row or column), splits them there and adds up a block of its own; the
// eight blocks are added in wave order through LDS, and the first wave writes the result.  No operand passes through LDS, no wave waits for
// another before the end, and all loads of a wave's first two steps are on their way at once: such launches are bound by latency.  The tile kernel
// takes 0.7 us for each of the steps it works one after another, and needs a second kernel where its reduction is cut.
// Measured against it (us; the tile kernel with the ranges a graph declares, cut where it says so): 3x3, 16 -> 16, 16x16, batch 2: forward 8.9 and 6.2, input gradient 9.7
// and 6.9; 1x1, 1024 -> 256, 14x14, batch 1: input gradient (cut) 12.9 and 7.7, filter gradient 14.9 and 7.7; 3x3, 60 -> 92, 13x17, batch 3: forward (cut)
// 12.5 and 9.3, uncut 23.2 and 9.3; 3x3, 512 -> 512, 7x7, batch 1, uncut: 140 and 44.  (All with 64 rows.)
// Per step of a wave 1.2 us forward and in the input gradient, 1.7 in the filter gradient with 64 rows (vector instructions of two waves per SIMD, loads that touch a cache
// line per row), 0.6 to 0.8 and 1.1 with 32, so that long reductions over few tiles are better spread over the GPU.
constexpr int SHORT_WAVES = 8;

// BLOCKS: blocks of 32 rows
template <int MODE, int BLOCKS>
__device__ __forceinline__ void short_tile(const TileArgs &ta) {
    __shared__ float part[SHORT_WAVES][16 * BLOCKS][64];
    __shared__ int redo[BLOCKS];      // blocks of 32 rows one by one: both forms of the kernel then give a row the same bits
    const ConvShape &cs = ta.cs;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned tile_m = blockIdx.x / (unsigned)ta.tiles_n;
    const int64_t row0 = (int64_t)tile_m * (32 * BLOCKS);
    const int col0 = (int)(blockIdx.x - tile_m * (unsigned)ta.tiles_n) * 32, col = col0 + l32;
    const int RSC = (int)cs.RSC();
    if (tid < BLOCKS) redo[tid] = 0;

    // residue class of an input gradient, as in the tile kernel
    int64_t Mg = ta.Mg, Kg = ta.Kg;
    int ph = 0, pw = 0, r0 = 0, s0 = 0, nr = cs.R, ns = cs.S, bh = 0, bw = 0, Hc = cs.H, Wc = cs.W;
    if (MODE == DGRAD) {
        const int st = cs.stride, cls = blockIdx.z;
        ph = cls / st;
        pw = cls % st;
        Hc = (cs.H - ph + st - 1) / st;
        Wc = (cs.W - pw + st - 1) / st;
        r0 = (ph + cs.pad) % st;
        s0 = (pw + cs.pad) % st;
        nr = r0 < cs.R ? (cs.R - r0 + st - 1) / st : 0;
        ns = s0 < cs.S ? (cs.S - s0 + st - 1) / st : 0;
        bh = (ph + cs.pad - r0) / st;
        bw = (pw + cs.pad - s0) / st;
        Mg = (int64_t)cs.N * Hc * Wc;
        Kg = (int64_t)nr * ns * cs.K;
        if (row0 >= Mg) return;
        if (Kg == 0 && ta.accumulate) return;       // this class receives no contribution
    }
    const int steps = (int)(((unsigned)Kg + BK - 1) / BK);

    // What a lane keeps of its two rows and its column: byte offsets, and one bit per filter tap that exists (see the tile kernel's loaders).
    const int row = MODE == FWD ? cs.W : cs.Q, inner = MODE == FWD ? cs.C : cs.K, taps_n = MODE == FWD ? cs.S : ns;
    const int64_t reach = MODE == WGRAD ? 0 : ((int64_t)(nr > 0 ? nr - 1 : 0) * row + (ns > 0 ? ns - 1 : 0)) * inner;
    const int64_t back = ((int64_t)cs.pad * cs.W + cs.pad) * cs.C;      // how far before its image a window begins
    const int64_t a_shift = MODE == FWD ? (back > reach ? back : reach) : reach, b_shift = MODE == WGRAD ? back : 0;
    unsigned a_voff[BLOCKS], a_taps[BLOCKS], b_voff = 0, b_tapbit = 0;
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) {
        const int64_t m = row0 + 32 * i + l32;
        const bool ok = m < Mg;
        if (MODE == WGRAD) {
            a_voff[i] = (unsigned)m * 4u;
            a_taps[i] = ok;
            continue;
        }
        const unsigned m32 = ok ? (unsigned)m : 0u, rw = (unsigned)(MODE == FWD ? cs.Q : Wc), rh = (unsigned)(MODE == FWD ? cs.P : Hc);
        const unsigned t = m32 / rw, n = t / rh;
        const int w = (int)(m32 - t * rw), h = (int)(t - n * rh);
        const int h0 = MODE == FWD ? h * cs.stride - cs.pad : h + bh, w0 = MODE == FWD ? w * cs.stride - cs.pad : w + bw;
        const int64_t image = MODE == FWD ? (int64_t)n * cs.H * cs.W * cs.C : (int64_t)n * cs.P * cs.Q * cs.K;
        a_voff[i] = (unsigned)((image + ((int64_t)h0 * row + w0) * inner + a_shift) * 4);
        unsigned rows = 0, cols = 0, taps = 0;
        for (int r = 0; r < nr; ++r)
            if (MODE == FWD ? (unsigned)(h0 + r) < (unsigned)cs.H : (unsigned)(h0 - r) < (unsigned)cs.P) rows |= 1u << r;
        for (int c = 0; c < ns; ++c)
            if (MODE == FWD ? (unsigned)(w0 + c) < (unsigned)cs.W : (unsigned)(w0 - c) < (unsigned)cs.Q) cols |= 1u << c;
        for (int r = 0; r < nr; ++r)
            if ((rows >> r) & 1) taps |= cols << (r * ns);
        a_taps[i] = ok ? taps : 0u;
    }
    int b_r = 0, b_s = 0;
    if (MODE == WGRAD) {
        const int cc = col < RSC ? col : 0, rs = cc / cs.C;
        b_r = rs / cs.S;
        b_s = rs - b_r * cs.S;
        b_voff = (unsigned)((((int64_t)b_r * cs.W + b_s) * cs.C + (cc - rs * cs.C)) * 4);
        b_tapbit = col < RSC;
    } else {
        b_tapbit = col < ta.Ng;
        b_voff = MODE == FWD ? (unsigned)((int64_t)col * RSC * 4) : (unsigned)col * 4u;
    }
    const __amdgpu_buffer_rsrc_t ra = buffer_of(ta.a - a_shift, ta.a_bytes + (unsigned)a_shift * 4u), rb = buffer_of(ta.b - b_shift, ta.b_bytes + (unsigned)b_shift * 4u);
    const unsigned by_cols = taps_n > 0 ? (1024u + taps_n - 1) / taps_n : 0u;      // tap / taps_n for tap < 32

    struct Step { float a[BLOCKS][8], b[8]; };      // reduction indices 16 t + 8 g .. + 7
    auto load = [&](Step &s, int t) {
        if constexpr (MODE == WGRAD) {
            const unsigned m0 = (unsigned)t * BK + 8u * g, q0 = m0 < (unsigned)Kg ? m0 : 0u;
            const unsigned tt = cs.Q == 1 ? q0 : __umulhi(q0, ta.q_mul) >> ta.q_shift;
            unsigned n = cs.P == 1 ? tt : __umulhi(tt, ta.p_mul) >> ta.p_shift, q = q0 - tt * (unsigned)cs.Q, p = tt - n * (unsigned)cs.P;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool in = m0 + e < (unsigned)Kg;
                const int h0 = (int)p * cs.stride - cs.pad, w0 = (int)q * cs.stride - cs.pad;
                const bool here = in && b_tapbit && (unsigned)(h0 + b_r) < (unsigned)cs.H && (unsigned)(w0 + b_s) < (unsigned)cs.W;
                // windows begin up to b_shift floats before the tensor, where its descriptor starts: the sum is not negative, and below 2^32 bytes
                const unsigned pix = (((n * (unsigned)cs.H + (unsigned)h0) * (unsigned)cs.W + (unsigned)w0) * (unsigned)cs.C + (unsigned)b_shift) * 4u;
                s.b[e] = buffer_load(rb, here ? pix + b_voff : BUFFER_ABSENT, 0u);
#pragma unroll
                for (int i = 0; i < BLOCKS; ++i) s.a[i][e] = buffer_load(ra, in && a_taps[i] ? (m0 + e) * (unsigned)cs.K * 4u + a_voff[i] : BUFFER_ABSENT, 0u);
                if (++q == (unsigned)cs.Q) {
                    q = 0;
                    if (++p == (unsigned)cs.P) { p = 0; ++n; }
                }
            }
        } else {
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const unsigned kk = (unsigned)t * BK + 8u * g + 4u * f;      // four indices of one filter tap: inner channels are a multiple of 4
                const bool in = kk < (unsigned)Kg;
                const unsigned tap = in ? __umulhi(kk, ta.q_mul) >> ta.q_shift : 0u, c = kk - tap * (unsigned)inner;
                const unsigned r = (tap * by_cols) >> 10, ss = tap - r * (unsigned)taps_n;
                const unsigned step = MODE == FWD ? ((r * cs.W + ss) * cs.C + c) * 4u : (unsigned)((int)c - (int)((r * cs.Q + ss) * cs.K)) * 4u;
#pragma unroll
                for (int i = 0; i < BLOCKS; ++i) {
                    const bf4 v = buffer_load4(ra, in && ((a_taps[i] >> tap) & 1u) ? a_voff[i] + step : BUFFER_ABSENT, 0u);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s.a[i][4 * f + e] = v[e];
                }
                if constexpr (MODE == FWD) {
                    const bf4 v = buffer_load4(rb, in && b_tapbit ? b_voff + kk * 4u : BUFFER_ABSENT, 0u);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s.b[4 * f + e] = v[e];
                } else {
                    // W[k][r0 + st * r][s0 + st * ss][col], k = c .. c + 3
                    const unsigned at = (c * (unsigned)RSC + (unsigned)(((r0 + cs.stride * (int)r) * cs.S + s0 + cs.stride * (int)ss) * cs.C)) * 4u + b_voff;
#pragma unroll
                    for (int e = 0; e < 4; ++e) s.b[4 * f + e] = buffer_load(rb, in && b_tapbit ? at + (unsigned)(e * RSC) * 4u : BUFFER_ABSENT, 0u);
                }
            }
        }
    };

    floatx16 acc[2], low[2];      // the h * h terms and the rest, as in the tile kernel
    constexpr int COLUMN = BLOCKS == 1 ? 0 : BLOCKS;      // both blocks share the column operand
    unsigned lost[COLUMN + 1] = {};
    bool again[BLOCKS] = {};
    auto multiply = [&](const Step &s, auto pieces) {
        if constexpr (decltype(pieces)::value) {
            const PieceRow b = split_row(s.b, lost[COLUMN]);
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i) {
                const PieceRow a = split_row(s.a[i], lost[i]);
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, acc[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, low[i], 0, 0, 0);
                low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, low[i], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < BLOCKS; ++i)
                if (BLOCKS == 1 || again[i]) {      // uniform over the workgroup
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(s.a[i][e], s.b[e], acc[i], 0, 0, 0);
                }
        }
    };
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = low[i][v] = 0.0f;
    {
        Step s0, s1;
        int t = wave;
        if (t < steps) load(s0, t);
        if (t + SHORT_WAVES < steps) load(s1, t + SHORT_WAVES);
        for (; t < steps; t += 2 * SHORT_WAVES) {
            multiply(s0, std::true_type{});
            if (t + 2 * SHORT_WAVES < steps) load(s0, t + 2 * SHORT_WAVES);
            if (t + SHORT_WAVES < steps) {
                multiply(s1, std::true_type{});
                if (t + 3 * SHORT_WAVES < steps) load(s1, t + 3 * SHORT_WAVES);
            }
        }
    }
    // once more on the fp32 instruction where the pieces do not hold an operand, as in the tile kernel
    float probe[BLOCKS] = {};
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[i][v] += low[i][v];
            probe[i] += acc[i][v];
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i)
        if (!(__builtin_fabsf(probe[i]) < __builtin_inff()) || pieces_lost(lost[i] | lost[COLUMN])) redo[i] = 1;
    __syncthreads();
    bool any = false;
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i) {
        again[i] = __builtin_amdgcn_readfirstlane(redo[i]) != 0;
        any |= again[i];
    }
    if (any) {
#pragma unroll
        for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = BLOCKS == 1 || again[i] ? 0.0f : acc[i][v];
        for (int t = wave; t < steps; t += SHORT_WAVES) {
            Step s;
            load(s, t);
            multiply(s, std::false_type{});
        }
    }
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[wave][16 * i + v][lane] = acc[i][v];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16 * BLOCKS / SHORT_WAVES; ++k) {
        const int v = wave * (16 * BLOCKS / SHORT_WAVES) + k;
        double sum = 0;      // rounded once: fp32 sums in turn would be further from 64 bits than the tile kernel's one chain
#pragma unroll
        for (int w = 0; w < SHORT_WAVES; ++w) sum += (double)part[w][v][lane];
        part[0][v][lane] = (float)sum;
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int i = 0; i < BLOCKS; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = part[0][16 * i + v][lane];
    const TilePlace at{row0, BLOCKS == 2 ? Mg : std::min(Mg, row0 + 32), col0, Hc, Wc, ph, pw, BLOCKS == 2 && row0 + 64 <= Mg && col0 + 32 <= ta.Ng, true, ta.out};
    write_results<MODE, true>(ta, acc, &part[1][0][0], at, lane);
}

// 64 rows of results a workgroup, or 32: half the vector and matrix instructions per step, and twice the workgroups, where the launch leaves at least half of the CUs idle (see
// short_halves).  The same bits, also beside a row that is worked once more in fp32.  us with 64 and with 32 rows: 3x3, 32 -> 64, 12x12, batch 2: 8.3 and 6.3, input gradient 8.1 and 6.2; 1x1, 384 -> 64, 9x9, batch 4 9.0 and 6.9; filter
// gradient of 3x3, 24 -> 64, 14x14 7.6 and 5.9.  (Both in one kernel cost the one of 64 rows 0.3 us; 32 rows with up to 256 workgroups of 64, two on a CU: forward 1.15 of the time.)
namespace rows64 {
template <int MODE>
__global__ __launch_bounds__(64 * SHORT_WAVES) void conv_short_kernel(TileArgs ta) {
    short_tile<MODE, 2>(ta);
}
}  // namespace rows64
namespace rows32 {
template <int MODE>
__global__ __launch_bounds__(64 * SHORT_WAVES) void conv_short_kernel(TileArgs ta) {
    short_tile<MODE, 1>(ta);
}
}  // namespace rows32

// Sums `splits` partial results in a fixed order.  Block = SL waves; wave sl adds splits sl, sl+SL, ...
// of 64 consecutive elements (four independent partial sums per lane to keep loads in flight),
// then the SL per-wave sums are added in wave order.
template <int SL>
__global__ __launch_bounds__(64 * SL) void split_reduce_kernel(const float *__restrict__ ws, float *dw, int64_t n, int splits, int accumulate) {
    __shared__ float sh[SL][64];
    const int lane = threadIdx.x & 63, sl = threadIdx.x >> 6;
    for (int64_t base = (int64_t)blockIdx.x * 64; base < n; base += (int64_t)gridDim.x * 64) {
        const int64_t i = base + lane;
        float s0 = 0, s1 = 0, s2 = 0, s3 = 0;
        if (i < n) {
            int z = sl;
            for (; z + 3 * SL < splits; z += 4 * SL) {
                s0 += ws[(int64_t)z * n + i];
                s1 += ws[(int64_t)(z + SL) * n + i];
                s2 += ws[(int64_t)(z + 2 * SL) * n + i];
                s3 += ws[(int64_t)(z + 3 * SL) * n + i];
            }
            for (; z < splits; z += SL) s0 += ws[(int64_t)z * n + i];
        }
        sh[sl][lane] = (s0 + s1) + (s2 + s3);
        __syncthreads();
        if (sl == 0 && i < n) {
            float s = sh[0][lane];
#pragma unroll
            for (int j = 1; j < SL; ++j) s += sh[j][lane];
            dw[i] = accumulate ? dw[i] + s : s;
        }
        __syncthreads();
    }
}

void launch_split_reduce(hipStream_t st, const float *ws, float *dw, int64_t n, int splits, bool accumulate) {
    const int acc = accumulate ? 1 : 0;
    int grid = (int)std::min<int64_t>((n + 63) / 64, 8192);
    if (splits >= 64) hipLaunchKernelGGL((split_reduce_kernel<16>), dim3(grid), dim3(1024), 0, st, ws, dw, n, splits, acc);
    else if (splits >= 16) hipLaunchKernelGGL((split_reduce_kernel<4>), dim3(grid), dim3(256), 0, st, ws, dw, n, splits, acc);
    else hipLaunchKernelGGL((split_reduce_kernel<1>), dim3(grid), dim3(64), 0, st, ws, dw, n, splits, acc);
    hip_check(hipGetLastError(), "split reduce launch");
}

void set_row_magic(TileArgs &ta) {
    magic_of((unsigned)ta.cs.Q, ta.q_mul, ta.q_shift);
    magic_of((unsigned)ta.cs.P, ta.p_mul, ta.p_shift);
    magic_of((unsigned)ta.cs.W, ta.w_mul, ta.w_shift);
    magic_of((unsigned)ta.cs.H, ta.h_mul, ta.h_shift);
}

void check_shape(const ConvShape &cs) {
    if (cs.N <= 0 || cs.H <= 0 || cs.W <= 0 || cs.C <= 0 || cs.K <= 0 || cs.R <= 0 || cs.S <= 0 || cs.stride <= 0 || cs.pad < 0)
        throw KernelError("conv: bad shape");
    if (cs.P != (cs.H + 2 * cs.pad - cs.R) / cs.stride + 1 || cs.Q != (cs.W + 2 * cs.pad - cs.S) / cs.stride + 1 || cs.P <= 0 || cs.Q <= 0)
        throw KernelError("conv: output size does not match input, filter, stride and padding");
    if ((int64_t)cs.R * cs.S * cs.C > (1ll << 24) || (int64_t)cs.R * cs.S * cs.K > (1ll << 24) || cs.M() > (1ll << 31) - 64 ||
        (int64_t)cs.N * cs.H * cs.W > (1ll << 31) - 64 || (int64_t)cs.H * cs.W >= (1 << 24) || cs.R > 127 || cs.S > 127)
        throw KernelError("conv: shape too large");
    if (cs.stride > 8) throw KernelError("conv: stride too large");
}

// How a launch divides its reduction.  `splits` > 1 asks for that many ranges on every tile: partial results go
// to as many full-size slabs, which a second kernel adds in range order.  (Cutting only the ragged last round of tiles and adding the
// parts inside the kernel paid with the fp32 matrix instruction; with tiles worked three times faster the device-wide release it
// needs costs more than the idle CUs: 1x1, 1024 -> 256, 14x14, batch 184: 144 us with it, 130 without.)
constexpr int NUM_CU = 256;

// Workgroups of a tile shape that are on a CU together: LDS (160 KiB) and three or four waves per SIMD.
constexpr int resident_workgroups(int mode, int wm, int wn) {
    const int bytes = 2 * 3 * 4 * (plane_words(mode != WGRAD, 64 * wm) + plane_words(mode == FWD, 32 * wn)) + 512;
    return std::min(160 * 1024 / bytes, wm * wn <= 4 ? 12 / (wm * wn) : 16 / (wm * wn));
}
// The caller's `splits` is the most ranges a launch may cut its reduction into; it takes fewer where more only cost partial
// results.  `slots`: workgroups of the tile shape that are on the GPU together.
//   Filter gradients (few tiles, many ranges): the fullest of one to four rounds of workgroups, by an estimate of the matrix
//   instructions (180 TFLOP/s, 7 % lost to the uneven end of a single round) and of writing and reading the slabs (4 TB/s).
//   Over 13 layers of the networks at half a round to six rounds (forced): what it takes is within 5 % of the best of them and 4 - 10 % ahead
//   of what was asked for on small results (1x1, 64 -> 64, 56x56: 768 ranges 80 us, 1536 78, 4096 100; 1x1, 1024 -> 256, 14x14: 16 ranges
//   152, 32 128, 64 135; 3x3 stride 2, 128 -> 128, 56x56: 28 ranges 326, 56 271, 85 - taken - 286, 113 287).
//   Forward / input gradient: at most five workgroups per CU; beyond that the slabs cost more than the better balance gives.
int useful_splits(int mode, int splits, int64_t tiles, int64_t slots, double flops, double slab_bytes) {
    if (mode != WGRAD) return (int)std::max<int64_t>(1, std::min<int64_t>(splits, (5 * NUM_CU + tiles - 1) / tiles));
    int best = 1;
    double best_us = 0;
    for (int64_t r = 1; r <= 4; ++r) {
        const int s = (int)std::max<int64_t>(1, std::min<int64_t>(splits, slots * r / tiles));
        const double work = (double)(tiles * s), rounds = (double)((tiles * s + slots - 1) / slots);
        const double us = flops / 180e6 * (rounds * slots / work) * (1 + 0.07 / rounds) + (s > 1 ? s * slab_bytes * 2 / 4e6 : 0);
        if (r == 1 || us < best_us) { best = s; best_us = us; }
    }
    return best;
}

// Tile shapes that the choice below takes: 0: 128x128, 3: 128x64 for every mode, 6: 128x32 and 7: 64x128 forward and for input gradients, 4: 64x128 and 5: 64x64 for filter gradients.  1 (256x64)
// and 2 (64x256) stand for the nearest of these.
int g_cfg_override = -1;   // tuning and test aid: force one tile shape, and exactly the ranges asked for, on every launch

// the ranges a caller asked for, no more than there are steps; its workspace has to hold them whatever kernel runs
int check_splits(int splits, int64_t steps, int64_t out_elems, const float *ws, size_t ws_bytes, const char *who) {
    if (splits < 1) throw KernelError(std::string(who) + ": splits must be >= 1");
    if (splits > steps) splits = (int)std::max<int64_t>(steps, 1);
    if (splits > 1 && (!ws || ws_bytes < (size_t)splits * out_elems * 4)) throw KernelError(std::string(who) + ": workspace too small for the requested splits");
    return splits;
}

// Two groups of waves per workgroup (KS of the tile kernel): launches that leave a CU at most eight waves, two per SIMD.  One wave's vector instructions follow each other
// at 5 - 7 cycles, two waves' at 2.7 each, and loads, splits and barriers of one group pass under the other's matrix instructions.  Uncut: 3x3, 256 -> 256, 14x14,
// batch 16: 73 and 53 us; 3x3, 512 -> 512, 7x7, batch 64: 142 and 105; 1x1, 512 -> 128, 28x28, batch 20: 20.7 and 18.2; cut: 1x1, 25088 -> 4096, batch 176: 293 and
// 259.  With twice the workgroups the groups only get in each other's way: 3x3, 128 -> 128, 28x28, batch 16, in five ranges 36 and 44 us; 1x1, 128 -> 512,
// 28x28, batch 20: 19 and 25.  Adding the groups' sums takes a microsecond: with few steps a launch is level or loses (3x3, 32 -> 64, 100x100, batch 6, 18 steps: 19.8
// and 20.6; 1x1, 2048 -> 1000, batch 184, 16 ranges of eight: 18.6 and 19.3; 3x3, 256 -> 256, 14x14, batch 16, ranges of 29: 31.9 and 32.1).
template <int WM, int WN>
bool two_wave_groups(int64_t workgroups, int64_t steps) {
    return steps >= 32 && workgroups <= (WM * WN == 8 ? 1 : 2) * NUM_CU;
}

template <int MODE, int WM, int WN, int TAG = 0>
void launch_tile(hipStream_t st, TileArgs ta, bool fast, int zdim, float *out, int splits, float *ws, size_t ws_bytes, int64_t steps,
                 bool accumulate, const char *who) {
    constexpr int BM = 64 * WM, BN = 32 * WN, NT = 64 * WM * WN;
    set_row_magic(ta);
    splits = check_splits(splits, steps, ta.out_elems, ws, ws_bytes, who);
    if (splits > 1 && g_cfg_override < 0)
        splits = useful_splits(MODE, splits, (ta.Mg + BM - 1) / BM * ((ta.Ng + BN - 1) / BN) * zdim, (int64_t)NUM_CU * resident_workgroups(MODE, WM, WN),
                               2.0 * ta.Mg * ta.Ng * ta.Kg * zdim, 4.0 * ta.out_elems);
    int64_t tiles_m = (ta.Mg + BM - 1) / BM;
    ta.tiles_n = (ta.Ng + BN - 1) / BN;
    ta.total_tiles = tiles_m * ta.tiles_n;
    ta.out = out;
    ta.splits = 1;
    ta.accumulate = accumulate ? 1 : 0;
    ta.stream = MODE != WGRAD && TAG == 0 && splits == 1 && ta.out_elems * 4 >= (256ll << 20);
    bool slabs = false;
    if (splits > 1 || (MODE == WGRAD && accumulate)) {      // a filter gradient is accumulated by the kernel that adds its ranges
        slabs = true;
        ta.out = ws;
        ta.splits = splits;
    }
    const int64_t blocks = (ta.total_tiles * ta.splits + NUM_XCD - 1) / NUM_XCD * NUM_XCD;
    if (blocks > 0x7fffffffll) throw KernelError("conv: too many tiles");
    dim3 grid((unsigned)blocks, 1, (unsigned)zdim);
    if constexpr (TAG != 0) {
        if (!fast) throw KernelError("conv: batched GEMMs need aligned shapes");
        hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 1, TAG>), grid, dim3(NT), 0, st, ta);
    } else {
        // forward or input-gradient channels that are no multiple of 16
        const bool part = MODE == FWD ? ta.cs.C % BK != 0 : MODE == DGRAD ? ta.cs.K % BK != 0 : false;
        if constexpr (MODE != WGRAD && WM == 1) {      // 1x1 layers of few rows
            if (!fast || ta.cs.R * ta.cs.S > 1) throw KernelError("conv: this tile shape is for aligned 1x1 layers");
            if (part) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 2>), grid, dim3(NT), 0, st, ta); }
            else { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 1>), grid, dim3(NT), 0, st, ta); }
        } else if constexpr (MODE != WGRAD) {
            if constexpr (WM == 2 && WN >= 2) {
                if (fast && !part && g_cfg_override < 0 && two_wave_groups<WM, WN>(blocks * zdim, steps / ta.splits)) {
                    hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 1, 0, 2>), grid, dim3(2 * NT), 0, st, ta);
                    hip_check(hipGetLastError(), "conv launch");
                    if (slabs) launch_split_reduce(st, ws, out, ta.out_elems, splits, accumulate);
                    return;
                }
            }
            if (fast && part && ta.cs.R * ta.cs.S > 1) {
                if constexpr (WM == 2 && WN <= 2) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 3>), grid, dim3(NT), 0, st, ta); }
                else throw KernelError("conv: straddling reduction steps need the 128x64 tile");
            }
            else if (fast && part) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 2>), grid, dim3(NT), 0, st, ta); }
            else if (fast && WM * WN <= 4 && steps <= 6) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, WM * WN <= 4 ? 4 : 1>), grid, dim3(NT), 0, st, ta); }
            else if (fast) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 1>), grid, dim3(NT), 0, st, ta); }
            else { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 0>), grid, dim3(NT), 0, st, ta); }
        } else {
            if (fast) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 1>), grid, dim3(NT), 0, st, ta); }
            else if constexpr (WM * WN <= 4) { hipLaunchKernelGGL((conv_tile_kernel<MODE, WM, WN, 0>), grid, dim3(NT), 0, st, ta); }
            else throw KernelError("conv: element-wise filter gradients have no 128x128 tile");
        }
    }
    hip_check(hipGetLastError(), "conv launch");
    if (slabs) launch_split_reduce(st, ws, out, ta.out_elems, splits, accumulate);
}

// Choice measured on the ResNet-50, VGG-16, MobileNetV2 and inception layer sets.  The square tile moves the least through LDS and
// L2 per product (3x3, 256 -> 256, 56x56, batch 176: 3.25 ms against 3.67 with 128x64), the 128x64 tile has twice as many workgroups,
// four of them on a CU: it is the faster one where a reduction is short and the time goes into loads and stores (1x1, 64 -> 256, 56x56,
// batch 184: 214 against 250 us) and where square tiles are too few to fill the GPU evenly (1x1, 160 -> 960, 7x7, batch 272: 47 against
// 76 us; 1x1, 512 -> 128, 28x28: 126 against 132; at 2256 tiles, 1x1, 256 -> 1024, 14x14: 126 against 118).  Around the lines, 1x1, C -> 256, square
// against narrow: 9016 tiles (56x56), 5 steps 187 and 205 us, 8 steps 282 and 328; 2254 (28x28), 6 steps 57 and 60, 8 steps 66 and 76; 564
// (14x14), level from 2 to 16 steps.  A reduction cut into
// ranges fills it anyway.  `straddle`: reduction steps that cross filter taps.
// Results of up to 32 columns leave half of the 128x64 tile's matrix instructions to columns that do not exist.  6: 128x32, two waves per workgroup (narrow_tile below).
// 7: 64x128 for cut 1x1 layers of at most 64 rows (a small batch's fully connected layer: half of 128 rows would not exist): 25088 -> 4096, batch 64: forward 153 and
// 115 us, input gradient 149 and 107; 2048 -> 1000, batch 64: 14.2 and 12.7.  Uncut it has no more workgroups than the 128x128 tile's groups (700 and 734).
// Element-wise loaders (`fast` false) are bound by loading: a wider tile reads each activation for fewer column tiles.  Forward, 128x64
// against 128x128: 5x5, 141 -> 464, 106x106, batch 2: 1459 and 897 us; 3x3, 258 -> 514, 14x14, batch 64: 709 and 389; 1x1, 18 -> 239,
// 90x90, batch 23: 67 and 56.  Input gradient of the first: 2643 and 2001; of a 3x3 layer, 416 -> 1, in one step: 60 and 52; of a 2x2 stride-3 layer,
// 145 -> 17, in two steps: 55 and 65, where square tiles cover a third more columns: short reductions take them up to a fifth.
// Forward the narrow tile has a table of reduction indices for up to 256 of them: 5x5, 10 -> 192, 28x28, batch 64: 68 and 88 (a third more
// columns); 5x5, 3 -> 96, 112x112, batch 32: 124 and 117 (as many).
// Element-wise filter gradients take 128x64 in place of 128x128, whose 128 registers they exceed: 5x5 stride 3, 438 -> 392, 32x32, batch 38: 501
// and 756 us; 3x3, 258 -> 514, 14x14, batch 64, ten ranges: 434 and 501; 1x1, 438 -> 391, 32x32, batch 38, 64 ranges: 251 and 287.
// (It loses where its twice as many tiles just begin a second round: 7x7, 402 -> 304, 16x16, batch 10: 221 and 196.)
//
// 128x32: the same workgroups as the 128x64 tile, with half the waves each and four on a CU (1024 in a round) where that has three (768).  Times against the 128x64
// tile, 5900 launches of up to 32 columns in all: 640 - 768 workgroups 0.92, - 1024 (one round for two) 0.80; 1024 - 1536 (two rounds both) 1.03 - 1.09 forward, 0.97 - 1.01
// in the input gradient, up to 1.38; from there 0.88 - 0.95 in the input gradient, 0.95 - 1.04 forward, 0.92 - 0.96 from 2560 on.  3x3, 64 -> 32, 90x90, batch 16 (1013, 36 steps): 61
// and 48 us; 3x3, 8 <- 180, 75x78, batch 26, input gradient (1252): 195 and 236.  Beyond one round 1x1 layers are level or lose (1.01 - 1.03: they move memory), and so do
// straddling reductions that are long or, forward, strided (0.95 - 0.98, single ones to 1.20: that variant has one register stage of loads here); aligned reductions of less than eight steps are
// level (0.98 - 1.02).  `workgroups`: of the residue classes that have a filter tap; the others only write zeros.  Cut launches keep the wider tile: their ranges are further
// workgroups.  Half as many waves per workgroup lose where there are few (5x5, 24 -> 64, 14x14, batch 320, input gradient, 490 of them: 91 and 95).
bool narrow_tile(int mode, int64_t workgroups, int64_t steps, int taps, int stride, bool straddle) {
    if (workgroups < 640 || (!straddle && steps < (taps > 1 ? 8 : 16))) return false;
    if (workgroups <= 4 * NUM_CU) return true;
    return taps > 1 && workgroups >= (mode == DGRAD ? 6 : 10) * NUM_CU && !(straddle && (steps >= 100 || (mode == FWD && stride > 1)));
}
// `busy`: residue classes that have a filter tap
int pick_cfg(int mode, int64_t Mg, int64_t Ng, int64_t steps, int64_t classes, int64_t busy, int taps, int stride, int splits, bool fast, bool straddle) {
    if (mode == WGRAD) {
        static const int nearest[6] = {0, 3, 4, 3, 4, 5};
        if (g_cfg_override >= 0) return nearest[g_cfg_override] == 0 && !fast ? 3 : nearest[g_cfg_override];
        if (Ng <= 64) return Mg <= 64 ? 5 : 3;
        if (Mg <= 64) return (Ng + 127) / 128 * 128 <= (Ng + 63) / 64 * 64 * 9 / 8 ? 4 : 5;
        return fast ? 0 : 3;
    }
    if (g_cfg_override < 0 && fast && Ng <= 32 && splits == 1 && narrow_tile(mode, (Mg + 127) / 128 * busy, steps, taps, stride, straddle)) return 6;
    if (g_cfg_override < 0 && fast && taps == 1 && splits > 1 && Mg <= 64 && Ng > 64) return 7;      // at most 64 rows
    if (straddle) return 3;      // straddling lanes carry their tap: registers the larger tile does not have
    if (g_cfg_override >= 0) return g_cfg_override == 0 ? 0 : 3;
    if (Ng <= 64) return 3;
    if (splits > 1) return 0;
    if (!fast) return steps > (mode == FWD ? KTAB / BK : 6) || (Ng + 127) / 128 * 128 * 5 <= (Ng + 63) / 64 * 64 * 6 ? 0 : 3;
    return steps > 6 && (Mg + 127) / 128 * ((Ng + 127) / 128) * classes >= 6 * NUM_CU ? 0 : 3;
}

template <int MODE, class... Rest>
void launch_cfg(int cfg, Rest... rest) {
    if (cfg == 0) launch_tile<MODE, 2, 4>(rest...);
    else if (MODE == WGRAD && cfg == 4) launch_tile<WGRAD, 1, 4>(rest...);
    else if (MODE == WGRAD && cfg == 5) launch_tile<WGRAD, 1, 2>(rest...);
    else if (MODE != WGRAD && cfg == 7) launch_tile<MODE == WGRAD ? FWD : MODE, 1, 4>(rest...);
    else if (MODE != WGRAD && cfg == 6) launch_tile<MODE == WGRAD ? FWD : MODE, 2, 1>(rest...);
    else launch_tile<MODE, 2, 2>(rest...);
}

// Launches of few results (see conv_short_kernel): at most one workgroup per CU, and from four steps on: up to three, the tile kernel's chain has fewer roundings.
// A launch that the tile kernel would work uncut takes it up to 512 steps (0.45 us each there; 288 steps: 140 us against 44).  One that it would cut
// into ranges costs 11 - 15 us there with the second kernel, however long.  Time here over time there, 8000 launches with the ranges that a graph declares, mean and
// 90th percentile by steps: forward 32 - 39 0.75 / 0.87, 44 - 47 0.84 / 0.97, 52 - 55 0.96 / 1.12; input gradient 40 - 43 0.85 / 0.93, 48 - 51 0.90 / 0.97, 56 - 63 0.99 / 1.10;
// accumulating, which costs the second kernel nothing there and a read of the result here, 36 - 39 0.88 / 0.99, 44 - 47 0.97 / 1.08, 48 - 51 1.01 / 1.10, with 128 workgroups and
// more 48 - 51 0.84 / 0.99; filter gradient of more than 64 rows and 32 workgroups and more 36 - 39 0.85 / 0.88, 40 - 43 0.91 / 0.97, 44 - 47 0.99 / 1.03; of at most 64 rows, for which
// the tile kernel has tiles of 64, 28 - 31 0.85 / 0.90, 32 - 35 0.94 / 1.02, 40 - 43 1.10 / 1.15.
// With a workgroup per 32 rows (short_halves) it is faster: 3000 launches of either kind, uncut 0.81 / 0.87 of the time of the 64-row form.  Cut, time here over time there: forward
// 66 - 71 steps 0.73 / 0.76, 72 - 77 0.83 / 0.97, 90 - 95 0.91 / 1.04; input gradient 60 - 65 0.80 / 0.85, 78 - 83 0.94 / 0.98, 90 - 95 1.02 / 1.07; accumulating 60 - 65 0.86 / 0.91,
// 66 - 71 0.93 / 1.00, 72 - 77 1.00 / 1.04; filter gradient of more than 64 rows 54 - 59 0.88 / 0.92, 60 - 65 0.95 / 1.02; of at most 64 36 - 41 0.84 / 0.95, 42 - 47 0.96 / 1.01.
// Below eight workgroups of 64 rows a cut forward or input-gradient launch is the tile kernel's: it is given its ranges there.
// `steps` of the longest residue class.
bool short_halves(int mode, const TileArgs &ta, int64_t classes) {
    return (ta.Mg + 63) / 64 * ((ta.Ng + 31) / 32) * classes <= NUM_CU / 2 && !(mode == FWD && ta.stats_part);      // BatchNorm's partial statistics are of 64 rows
}
bool short_applies(int mode, const TileArgs &ta, int64_t steps, int64_t classes, bool fast, bool cut, bool accumulate = false) {
    const int64_t tiles = (ta.Mg + 63) / 64 * ((ta.Ng + 31) / 32) * classes;
    int64_t longest = 512;
    if (cut && short_halves(mode, ta, classes)) longest = mode == WGRAD ? (ta.Mg > 64 ? 58 : 40) : accumulate ? 68 : 80;
    else if (cut) longest = mode == DGRAD ? (accumulate && tiles < 128 ? 40 : 52) : mode == WGRAD ? (tiles >= 32 && ta.Mg > 64 ? 44 : 32) : 40;
    return fast && g_cfg_override < 0 && steps >= 4 && steps <= longest && tiles >= (cut && mode != WGRAD ? 8 : 1) && tiles <= NUM_CU;
}
template <int MODE>
void launch_short(hipStream_t st, TileArgs ta, int classes, float *out, bool accumulate) {
    set_row_magic(ta);
    if (MODE != WGRAD) magic_of((unsigned)(MODE == FWD ? ta.cs.C : ta.cs.K), ta.q_mul, ta.q_shift);      // a reduction index' filter tap
    ta.tiles_n = (ta.Ng + 31) / 32;
    ta.out = out;
    ta.splits = 1;
    ta.accumulate = accumulate ? 1 : 0;
    ta.stream = 0;
    const bool halves = short_halves(MODE, ta, classes);
    const dim3 grid((unsigned)((halves ? (ta.Mg + 31) / 32 : (ta.Mg + 63) / 64) * ta.tiles_n), 1, (unsigned)classes);
    if (halves) hipLaunchKernelGGL((rows32::conv_short_kernel<MODE>), grid, dim3(64 * SHORT_WAVES), 0, st, ta);
    else hipLaunchKernelGGL((rows64::conv_short_kernel<MODE>), grid, dim3(64 * SHORT_WAVES), 0, st, ta);
    hip_check(hipGetLastError(), "conv launch");
}

// the batched GEMMs only ever see the two tile shapes the forward heuristic picks
template <int TAG, class... Rest>
void launch_batched(int cfg, Rest... rest) {
    if (cfg == 3) launch_tile<FWD, 2, 2, TAG>(rest...);
    else launch_tile<FWD, 2, 4, TAG>(rest...);
}

}  // namespace

void conv_force_tile(int cfg) { g_cfg_override = cfg; }

// layers whose epilogue takes the statistics or the BatchNorm behind them: reduction steps of 16 do not straddle filter taps,
// C % 16 == 0, or a 1x1 layer (one tap) with C % 4 == 0, whose last step is partly empty
bool conv_fwd_aligned(const ConvShape &cs) { return cs.C % BK == 0 || (cs.R == 1 && cs.S == 1 && cs.C % 4 == 0); }

bool conv_epilogue_writes_mask(const ConvShape &cs, bool winograd_fused) {
    (void)winograd_fused;      // both forms: a word of the code is 64 consecutive channels of one position
    return cs.K % 64 == 0;
}

// floor(n / d) = umulhi(n, mul) >> shift for every n < 2^31 (d >= 2): mul = ceil(2^(31 + l) / d) with l = ceil(log2 d)
// fits 32 bits, and its excess over 2^(31 + l) / d, below d / 2^(31 + l) <= 2^-31, times n stays below one unit
void magic_of(unsigned d, unsigned &mul, unsigned &shift) {
    mul = 0; shift = 0;
    if (d < 2) return;
    unsigned l = 0;
    while (((uint64_t)1 << l) < d) ++l;
    mul = (unsigned)((((uint64_t)1 << (31 + l)) + d - 1) / d);
    shift = l - 1;
}
void split_reduce(hipStream_t st, const float *ws, float *out, int64_t n, int splits, bool accumulate) {
    launch_split_reduce(st, ws, out, n, splits, accumulate);
}

namespace {
struct SplitGemm { int64_t rows, cols, steps; int classes; };
SplitGemm split_gemm_of(int which, const ConvShape &cs) {
    if (which == 0) return {cs.M(), cs.K, (cs.RSC() + BK - 1) / BK, 1};
    const int st = cs.stride;
    return {(int64_t)cs.N * ((cs.H + st - 1) / st) * ((cs.W + st - 1) / st), cs.C,
            ((int64_t)std::max(1, cs.R / st) * std::max(1, cs.S / st) * cs.K + BK - 1) / BK, st * st};
}
}  // namespace

// Ranges for a launch that was given a workspace but not told to cut its reduction (splits == 1): with at most half as many square tiles as
// CUs, as many ranges as fill the GPU once and the workspace holds, of at least eight steps each.  3x3, 512 -> 512, 7x7, batch 1: 141 us
// uncut, 18 so; 1x1, 2048 -> 512, 7x7, batch 2: 66 and 14.
static int ranges_by_workspace(const SplitGemm &sg, int64_t out_elems, const float *ws, size_t ws_bytes) {
    if (!ws || sg.classes != 1 || g_cfg_override >= 0) return 1;
    const int64_t tiles = (sg.rows + 127) / 128 * (sg.cols <= 64 ? 1 : (sg.cols + 127) / 128);
    return (int)std::max<int64_t>(1, std::min<int64_t>({NUM_CU / tiles, sg.steps / 8, 16, (int64_t)(ws_bytes / 4) / out_elems}));
}

size_t conv_workspace_bytes(int which, const ConvShape &cs, int splits) {
    check_shape(cs);
    const SplitGemm sg = split_gemm_of(which, cs);
    if (splits > sg.steps) splits = (int)std::max<int64_t>(sg.steps, 1);
    if (splits > 1) return (size_t)splits * 4 * (which == 0 ? cs.M() * cs.K : (int64_t)cs.N * cs.H * cs.W * cs.C);
    static const int shape[6][2] = {{128, 128}, {256, 64}, {64, 256}, {128, 64}, {64, 128}, {64, 64}};
    const int cfg = g_cfg_override >= 0 ? g_cfg_override : sg.cols <= 64 ? 1 : 0;
    const int64_t bm = shape[cfg][0], bn = shape[cfg][1];
    const int64_t tiles = ((sg.rows + bm - 1) / bm) * ((sg.cols + bn - 1) / bn);
    const int64_t tail = tiles % NUM_CU;
    if (sg.classes != 1 || tail == 0) return 0;
    const int64_t s = std::min<int64_t>({NUM_CU / tail, sg.steps / 4, 16});
    return s >= 2 ? (size_t)(s * tail * bm * bn * 4) : 0;
}

void gemm_batched(hipStream_t st, const float *a, const float *b, float *out, int batch, int64_t rows, int cols, int red, bool adjoint_use) {
    if (batch < 1 || rows < 1 || cols < 1 || red < 1 || red % BK || cols % 4) throw KernelError("gemm_batched: bad shape");
    // the aligned loader addresses each operand plane with 32-bit byte offsets
    if (rows * red * 4 >= ((int64_t)1 << 32) - (1 << 20) || (int64_t)cols * red * 4 >= ((int64_t)1 << 32) - (1 << 20))
        throw KernelError("gemm_batched: an operand plane of 4 GiB or more");
    ConvShape cs{1, 1, (int)rows, red, cols, 1, 1, 1, 0, 1, (int)rows};
    check_shape(cs);
    TileArgs ta{};
    ta.a = a; ta.b = b; ta.cs = cs;
    ta.Mg = rows; ta.Ng = cols; ta.Kg = red;
    ta.out_elems = rows * cols;
    ta.a_bytes = (unsigned)(rows * red * 4); ta.b_bytes = (unsigned)((int64_t)cols * red * 4);
    ta.batch_a = rows * red; ta.batch_b = (int64_t)cols * red; ta.batch_out = rows * cols;
    const int cfg = cols <= 64 ? 3 : 0;
    if (adjoint_use) launch_batched<2>(cfg, st, ta, true, batch, out, 1, (float *)nullptr, (size_t)0, (int64_t)red / BK, false, "gemm_batched");
    else launch_batched<1>(cfg, st, ta, true, batch, out, 1, (float *)nullptr, (size_t)0, (int64_t)red / BK, false, "gemm_batched");
}

// out[z][m][n] = sum_t a[z][t][m] b[z][t][n]: the reduction runs over the rows of both operands (weight-gradient form);
// `splits` partial results per GEMM go to ws (splits * batch * m * n floats) and are added in range order; accumulate: and to what out
// holds (the workspace has room for one result at least)
void gemm_tn_batched(hipStream_t st, const float *a, const float *b, float *out, int batch, int64_t red, int m, int n, int splits,
                     float *ws, size_t ws_bytes, bool accumulate) {
    if (batch < 1 || red < 1 || m < 1 || n < 1 || m % 4 || n % 4) throw KernelError("gemm_tn_batched: bad shape");
    ConvShape cs{1, 1, (int)red, n, m, 1, 1, 1, 0, 1, (int)red};
    check_shape(cs);
    TileArgs ta{};
    ta.a = a; ta.b = b; ta.cs = cs;
    ta.Mg = m; ta.Ng = n; ta.Kg = red;
    ta.out_elems = (int64_t)batch * m * n;
    ta.a_bytes = (unsigned)(red * m * 4); ta.b_bytes = (unsigned)(red * n * 4);
    ta.batch_a = red * m; ta.batch_b = red * n; ta.batch_out = (int64_t)m * n;
    // the aligned loader addresses each operand plane with 32-bit byte offsets
    if (red * m * 4 >= ((int64_t)1 << 32) - (1 << 20) || red * n * 4 >= ((int64_t)1 << 32) - (1 << 20))
        throw KernelError("gemm_tn_batched: an operand plane of 4 GiB or more");
    if (accumulate && (!ws || ws_bytes < (size_t)ta.out_elems * 4)) throw KernelError("gemm_tn_batched: an accumulated result needs a workspace of its size");
    launch_tile<WGRAD, 2, 4, 3>(st, ta, true, batch, out, splits, ws, ws_bytes, (red + BK - 1) / BK, accumulate, "gemm_tn_batched");
}

void conv_fwd(hipStream_t st, const float *x, const float *w, float *y, const ConvShape &cs, int splits, float *ws, size_t ws_bytes,
              bool accumulate, float *stats_part, const BnAffine *affine) {
    check_shape(cs);
    // first layers (three input channels): input rows staged in LDS as they lie in memory (stem.hip)
    if (g_cfg_override < 0 && splits == 1 && !accumulate && !stats_part && !affine && stem_applies(cs)) {
        stem_fwd(st, x, w, y, cs);
        return;
    }
    TileArgs ta{};
    ta.a = x; ta.b = w; ta.cs = cs;
    ta.a_bytes = (unsigned)((int64_t)cs.N * cs.H * cs.W * cs.C * 4); ta.b_bytes = (unsigned)(cs.K * cs.RSC() * 4);
    ta.Mg = cs.M(); ta.Ng = cs.K; ta.Kg = cs.RSC();
    ta.out_elems = ta.Mg * ta.Ng;
    // the aligned loader addresses both operands with 32-bit byte offsets (plus one tap's reach) and keeps one bit per filter tap
    const int64_t span32 = ((int64_t)1 << 32) - (1 << 20);
    const int64_t reach = ((int64_t)(cs.R + cs.pad) * cs.W + cs.S + cs.pad) * cs.C * 4;
    bool fast = cs.C % 4 == 0 && cs.R * cs.S <= 32 && (int64_t)cs.N * cs.H * cs.W * cs.C * 4 + reach < span32 && cs.K * cs.RSC() * 4 < span32;
    if ((stats_part || affine) && (!fast || !conv_fwd_aligned(cs) || cs.K % 4 || splits != 1 || accumulate))
        throw KernelError("conv_fwd: statistics or BatchNorm in the epilogue need C % 16 == 0 (1x1: C % 4 == 0), K % 4 == 0, splits == 1 and no accumulation");
    if (stats_part && affine) throw KernelError("conv_fwd: either the statistics of the output or its BatchNorm apply step, not both");
    if (affine && (!affine->gamma || !affine->beta || !affine->stats)) throw KernelError("conv_fwd: incomplete BatchNorm coefficients");
    if (affine && affine->mask && (!affine->relu || cs.K % 64)) throw KernelError("conv_fwd: a sign code in the epilogue needs the ReLU and K % 64 == 0");
    const int64_t steps = (ta.Kg + BK - 1) / BK;
    ta.stats_part = stats_part;
    if (affine) ta.affine = *affine;
    if (short_applies(FWD, ta, steps, 1, fast, splits > 1 || ranges_by_workspace(split_gemm_of(0, cs), ta.out_elems, ws, ws_bytes) > 1)) {
        check_splits(splits, steps, ta.out_elems, ws, ws_bytes, "conv_fwd");
        launch_short<FWD>(st, ta, 1, y, accumulate);
        return;
    }
    if (splits == 1) {
        splits = ranges_by_workspace(split_gemm_of(0, cs), ta.out_elems, ws, ws_bytes);
        if (splits > 1 && (stats_part || affine)) {      // the sums are complete only behind the second kernel: what rode in the epilogue follows it
            conv_fwd(st, x, w, y, cs, splits, ws, ws_bytes);
            if (stats_part) bn_stats_row_groups(st, y, stats_part, cs.M(), cs.K);
            else if (affine->relu)
                fwd_chain(st, y, nullptr, affine->gamma, affine->beta, affine->stats, cs.K, affine->relu_out ? y : nullptr, nullptr,
                          affine->relu_out ? affine->relu_out : y, (uint64_t *)affine->mask, ta.out_elems, affine->relu == 2);
            else bn_apply(st, y, y, affine->gamma, affine->beta, affine->stats, cs.M(), cs.K);
            return;
        }
    }
    launch_cfg<FWD>(pick_cfg(FWD, ta.Mg, ta.Ng, steps, 1, 1, cs.R * cs.S, cs.stride, splits, fast, fast && !conv_fwd_aligned(cs)), st, ta, fast, 1, y, splits, ws, ws_bytes, steps, accumulate, "conv_fwd");
}

void conv_dgrad(hipStream_t st, const float *dy, const float *w, float *dx, const ConvShape &cs, bool accumulate, int splits, float *ws,
                size_t ws_bytes) {
    check_shape(cs);
    TileArgs ta{};
    ta.a = dy; ta.b = w; ta.cs = cs;
    ta.a_bytes = (unsigned)(cs.M() * cs.K * 4); ta.b_bytes = (unsigned)(cs.K * cs.RSC() * 4);
    const SplitGemm sg = split_gemm_of(1, cs);   // rows of residue class (0,0), the largest; the shortest class reduction bounds the splits
    ta.Mg = sg.rows;
    ta.Ng = cs.C;
    ta.Kg = 0;   // per class, computed in the kernel
    ta.out_elems = (int64_t)cs.N * cs.H * cs.W * cs.C;
    const int64_t span32 = ((int64_t)1 << 32) - (1 << 20);
    const int64_t reach = ((int64_t)cs.R * cs.Q + cs.S) * cs.K * 4;
    bool fast = cs.K % 4 == 0 && cs.C % 4 == 0 && cs.R * cs.S <= 32 && cs.M() * cs.K * 4 + reach < span32 && cs.K * cs.RSC() * 4 < span32;
    const int64_t longest = ((int64_t)((cs.R + cs.stride - 1) / cs.stride) * ((cs.S + cs.stride - 1) / cs.stride) * cs.K + BK - 1) / BK;
    if (short_applies(DGRAD, ta, longest, sg.classes, fast, splits > 1 || ranges_by_workspace(sg, ta.out_elems, ws, ws_bytes) > 1, accumulate)) {
        check_splits(splits, sg.steps, ta.out_elems, ws, ws_bytes, "conv_dgrad");
        launch_short<DGRAD>(st, ta, sg.classes, dx, accumulate);
        return;
    }
    if (splits == 1) splits = ranges_by_workspace(sg, ta.out_elems, ws, ws_bytes);
    launch_cfg<DGRAD>(pick_cfg(DGRAD, ta.Mg, ta.Ng, sg.steps, sg.classes, (int64_t)std::min(cs.R, cs.stride) * std::min(cs.S, cs.stride), cs.R * cs.S, cs.stride, splits, fast, fast && cs.K % BK != 0 && cs.R * cs.S > 1), st, ta, fast, sg.classes, dx, splits, ws, ws_bytes, sg.steps, accumulate, "conv_dgrad");
}

void conv_wgrad(hipStream_t st, const float *x, const float *dy, float *dw, const ConvShape &cs, int splits, float *ws, size_t ws_bytes) {
    check_shape(cs);
    // first layers (three input channels): input rows staged in LDS as they lie in memory (stem.hip)
    if (g_cfg_override < 0 && ws && stem_wgrad_applies(cs, splits, ws_bytes)) {
        stem_wgrad(st, x, dy, dw, cs, splits, ws, ws_bytes);
        return;
    }
    // 1x1 layers with at most 32 channels on one side: streamed straight into the matrix instruction (pointwise.hip)
    if (g_cfg_override < 0 && ws && pointwise_wgrad_applies(cs, splits, ws_bytes)) {
        pointwise_wgrad(st, x, dy, dw, cs, splits, ws, ws_bytes);
        return;
    }
    TileArgs ta{};
    ta.a = dy; ta.b = x; ta.cs = cs;
    ta.a_bytes = (unsigned)(cs.M() * cs.K * 4); ta.b_bytes = (unsigned)((int64_t)cs.N * cs.H * cs.W * cs.C * 4);
    ta.Mg = cs.K; ta.Ng = (int)cs.RSC(); ta.Kg = cs.M();
    ta.out_elems = (int64_t)cs.K * cs.RSC();
    // the aligned loader addresses both operands with 32-bit byte offsets and keeps one bit per filter tap
    const int64_t span32 = ((int64_t)1 << 32) - (1 << 20);
    const int64_t lead = ((int64_t)cs.pad * cs.W + cs.pad) * cs.C * 4;
    bool fast = cs.K % 4 == 0 && cs.C % 4 == 0 && cs.R * cs.S <= 32 && cs.M() * cs.K * 4 < span32 &&
                (int64_t)cs.N * cs.H * cs.W * cs.C * 4 + lead < span32;
    const int64_t steps = (ta.Kg + BK - 1) / BK;
    if (short_applies(WGRAD, ta, steps, 1, fast, splits > 1)) {
        check_splits(splits, steps, ta.out_elems, ws, ws_bytes, "conv_wgrad");
        launch_short<WGRAD>(st, ta, 1, dw, false);
        return;
    }
    launch_cfg<WGRAD>(pick_cfg(WGRAD, ta.Mg, ta.Ng, 0, 1, 1, cs.R * cs.S, cs.stride, splits, fast, false), st, ta, fast, 1, dw, splits, ws, ws_bytes, steps, false, "conv_wgrad");
}

}  // namespace monet
