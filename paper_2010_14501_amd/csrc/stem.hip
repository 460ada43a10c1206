// First layers: convolutions of a three-channel image (7x7 / stride 2, 3x3 / stride 1 or 2).  With C = 3 a reduction
// step of the tile kernel in conv.hip straddles filter taps, so its loader goes element by element (46-56 TFLOP/s on the
// ResNet-50 stem).  Here the input rows a tile of output positions needs are copied to LDS once, as they lie in memory
// (N,H,W,3: the S taps of a filter row are S*3 consecutive floats), and the matrix instruction's operand is read from
// there directly:
//
//   y[m][k] = sum_r sum_j  x_row(m, r)[j] * w[k][r][j],   j = 3 s + c in [0, 3 S),
//   x_row(m, r) = LDS row (pr * ST + r), starting at column (qq * ST) * 3        (m = (pr, qq) inside the tile)
//
// so consecutive output positions are ST*3 floats apart in LDS and no patch matrix is ever formed.  The reduction of a
// filter row is padded from 3 S to the next even number (the matrix instruction takes two reduction indices; the filter
// value of the padding is zero, its input value a float of the position's own window read a second time).
//
// Forward, 3x3 filters and 7x7 ones whose rows in pieces exceed LDS (stem7_fwd_kernel below takes the others): mfma_f32_32x32x2f32 with A = positions x reduction
// (lane (m, h) reads LDS[off(m) + r * rowlen + 2 t + h]),
// B = the filters of 32 output channels, resident in registers for the whole launch (R * ceil(3 S / 2) values per lane).
// A wave takes four blocks of 32 consecutive positions and 32 output channels; a workgroup (K / 32 waves per group of
// four blocks, at most four waves) one tile of up to 224 positions: whole output rows if they fit, else a segment of
// one row.  Workgroups loop over tiles.
//
// Filter gradient, 7x7: dw[k][r][j] = sum_m dy[m][k] * x_row(m, r)[j]: A = dy (positions are the reduction index now, read
// from memory in the layout of v_mfma_f32_32x32x16_bf16: lane (k, h) loads dy[m + 8 h + i][k], i < 8), B = lane (col, h) reads
// LDS[off(m + 8 h + i) + r(col) * rowlen + j(col)] with col = (r, j) flattened; both are split into bf16 pieces in registers
// (bf16_pieces.hpp), 48 vector instructions per operand beside six matrix instructions per 32 columns.  7x7, 64 channels, 224x224,
// batch 184: 568 us on the fp32 instruction, 473 so (76 and 92 TFLOP/s), error against 64 bits 8.5e-7 and 3.1e-7; bound by the chain of LDS reads,
// splits and matrix instructions of two waves per SIMD (256 registers; the compiler spills 32 of them around the second pass in fp32, none
// inside the loop over tiles).  The 3x3 filters keep the fp32 instruction in both directions.  Wave kb of a workgroup owns the 32 output
// channels 32 kb .. 32 kb + 31 and all R * 3 S columns; the workgroups' partial results are added in a fixed order by
// split_reduce.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "bf16_pieces.hpp"
#include "buffer_addr.hpp"
#include "kernels.hpp"

namespace monet {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

struct StemGeom {
    int N, H, W, P, Q, K, pad;
    int nrow, qn;            // tile: nrow output rows x qn output columns (qn == Q, or nrow == 1)
    int row_tiles, col_tiles;
    int64_t tiles;           // N * row_tiles * col_tiles
    int rows_in;             // input rows under a tile: (nrow - 1) * ST + R
    int rowlen;              // floats per LDS row (multiple of 4)
    int xlead;               // LDS column of the tile's first input float (the float (q0 * ST - pad) * 3 of an image row)
};

// Copies the input rows under tile (n, p0, q0) to LDS, zero where the image ends, in two steps: the loads into registers
// (piece tid + k * nthreads of the tile's rows_in x rowlen / 4 pieces of 16 bytes, k < FILL: the host checks that this
// covers the tile) and the LDS writes, so that other work can be issued between the two.  LDS column e of row ri holds
// float fbase + e of image row h0 + ri, fbase = (q0 * ST - pad) * 3 - xlead (a multiple of 4 whenever W is one, so that
// the 16-byte pieces stay aligned).
constexpr int FILL = 8;
template <int ST>
__device__ __forceinline__ void stem_fill_load(float4 (&v)[FILL], const float *__restrict__ x, const StemGeom &gm, int n, int p0, int q0, int tid,
                                               int nthreads, int k0 = 0) {
    const int row4 = gm.rowlen / 4, rowf = gm.W * 3;
    const int h0 = p0 * ST - gm.pad, fbase = (q0 * ST - gm.pad) * 3 - gm.xlead;
    const bool aligned = (gm.W & 3) == 0 && (fbase & 3) == 0 && ((uintptr_t)x & 15) == 0;
    const float *img = x + (int64_t)n * gm.H * rowf;
    const int first = tid + k0 * nthreads;      // pieces first + k * nthreads, k < FILL
    int ri = first / row4, e4 = first - ri * row4;
    const int dr = nthreads / row4, de = nthreads - dr * row4;
#pragma unroll
    for (int k = 0; k < FILL; ++k) {
        v[k] = make_float4(0, 0, 0, 0);
        const int h = h0 + ri, f = fbase + 4 * e4;
        if (ri < gm.rows_in && (unsigned)h < (unsigned)gm.H) {
            const float *src = img + (int64_t)h * rowf;
            if (aligned && f >= 0 && f + 3 < rowf) v[k] = *(const float4 *)(src + f);
            else {
                if ((unsigned)f < (unsigned)rowf) v[k].x = src[f];
                if ((unsigned)(f + 1) < (unsigned)rowf) v[k].y = src[f + 1];
                if ((unsigned)(f + 2) < (unsigned)rowf) v[k].z = src[f + 2];
                if ((unsigned)(f + 3) < (unsigned)rowf) v[k].w = src[f + 3];
            }
        }
        ri += dr; e4 += de;
        if (e4 >= row4) { e4 -= row4; ++ri; }
    }
}
__device__ __forceinline__ void stem_fill_write(float *lds, const float4 (&v)[FILL], const StemGeom &gm, int tid, int nthreads, int k0 = 0) {
    const int total = gm.rows_in * (gm.rowlen / 4);
#pragma unroll
    for (int k = 0; k < FILL; ++k) {
        const int idx = tid + (k0 + k) * nthreads;
        if (idx < total) *(float4 *)&lds[4 * idx] = v[k];
    }
}

__device__ __forceinline__ void tile_origin(const StemGeom &gm, int64_t tile, int &n, int &p0, int &q0) {
    const int per_img = gm.row_tiles * gm.col_tiles;
    n = (int)(tile / per_img);
    const int t = (int)(tile - (int64_t)n * per_img);
    p0 = (t / gm.col_tiles) * gm.nrow;
    q0 = (t % gm.col_tiles) * gm.qn;
}

template <int R, int S, int ST>
__global__ __launch_bounds__(256, 2) void stem_fwd_kernel(const float *__restrict__ x, const float *__restrict__ w, float *__restrict__ y, StemGeom gm) {
    extern __shared__ float lds[];
    constexpr int RUN = 3 * S, KP = (RUN + 1) / 2, MBW = 4;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = wave % (gm.K / 32);      // this wave's block of 32 output channels ...
    const int mg = wave / (gm.K / 32);      // ... and group of MBW position blocks
    const int nthreads = blockDim.x;
    // filters of channel 32 nb + l32: w[k][r][2 t + h], zero beyond the row's 3 S values
    float wr[R][KP];
    {
        const float *wk = w + (int64_t)(nb * 32 + l32) * (R * RUN);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < KP; ++t) wr[r][t] = 2 * t + h < RUN ? wk[r * RUN + 2 * t + h] : 0.0f;
    }
    // LDS offset of this lane's position in every block (position 32 b + l32 of the tile; positions beyond the tile read
    // position 0), plus h: the lane's share of a reduction pair
    int aoff[MBW];
#pragma unroll
    for (int b = 0; b < MBW; ++b) {
        int m = 32 * (MBW * mg + b) + l32;
        if (m >= gm.nrow * gm.qn) m = 0;
        const int pr = gm.nrow == 1 ? 0 : m / gm.qn, qq = m - pr * gm.qn;
        aoff[b] = pr * ST * gm.rowlen + qq * ST * 3 + gm.xlead + h;
    }
    float4 staged[FILL];
    if ((int64_t)blockIdx.x < gm.tiles) {
        int n, p0, q0;
        tile_origin(gm, blockIdx.x, n, p0, q0);
        stem_fill_load<ST>(staged, x, gm, n, p0, q0, tid, nthreads);
        stem_fill_write(lds, staged, gm, tid, nthreads);
    }
    __syncthreads();
    for (int64_t tile = blockIdx.x; tile < gm.tiles; tile += gridDim.x) {
        int n, p0, q0;
        tile_origin(gm, tile, n, p0, q0);
        // the compiler must not carry the addresses derived from these offsets (one per filter row and block) from tile to
        // tile in registers: they cost one addition each and there are more of them than registers to spare
#pragma unroll
        for (int b = 0; b < MBW; ++b) asm volatile("" : "+v"(aoff[b]));
        floatx16 acc[MBW];
#pragma unroll
        for (int b = 0; b < MBW; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][i] = 0.0f;
        // position blocks of the nominal tile this wave works on (the last group may hold fewer than MBW)
        const int nblk = min(MBW, (gm.nrow * gm.qn + 31) / 32 - MBW * mg);
        // one reduction pair ahead: the LDS reads of pair s + 1 are issued before the matrix instructions of pair s
        float a_cur[MBW], a_nxt[MBW];
        auto read_pair = [&](int r, int t, float (&a)[MBW]) {
            const float *row = lds + r * gm.rowlen + 2 * t;
#pragma unroll
            for (int b = 0; b < MBW; ++b) {
                // the padding slot of an odd row length (h = 1 of the last pair, filter value zero) reads the value of
                // h = 0 again: a float of this position's own window, so that nothing foreign can turn 0 * x into NaN
                a[b] = row[(RUN & 1) && t == KP - 1 ? aoff[b] - h : aoff[b]];
            }
        };
        read_pair(0, 0, a_cur);
#pragma unroll
        for (int s = 0; s < R * KP; ++s) {
            if (s + 1 < R * KP) read_pair((s + 1) / KP, (s + 1) % KP, a_nxt);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < MBW; ++b)
                if (b < nblk) acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(a_cur[b], wr[s / KP][s % KP], acc[b], 0, 0, 0);      // uniform over the wave
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < MBW; ++b) a_cur[b] = a_nxt[b];
        }
        // The next tile's input is requested before this tile's results are stored and goes to LDS after them: its latency
        // passes while the stores are issued, and the stores drain while the next tile is computed (memory operations
        // complete in the order of issue, so waiting for these loads does not wait for the stores behind them).
        const int64_t next = tile + gridDim.x;
        if (next < gm.tiles) {      // uniform over the workgroup
            int n2, p2, q2;
            tile_origin(gm, next, n2, p2, q2);
            stem_fill_load<ST>(staged, x, gm, n2, p2, q2, tid, nthreads);
        }
        __builtin_amdgcn_sched_barrier(0);
        // positions of the tile are consecutive in y when the tile is whole rows or part of one row: position m lies m * K
        // floats behind the tile's first.  Buffer addressing: the lane's part of the offset (4 h rows, its channel) never
        // changes, the rest is the same for every lane.
        const int rows_here = min(gm.nrow, gm.P - p0), cols_here = min(gm.qn, gm.Q - q0);
        const int npos = gm.nrow == 1 ? cols_here : rows_here * gm.qn;
        const __amdgpu_buffer_rsrc_t ry = buffer_of(y + (((int64_t)n * gm.P + p0) * gm.Q + q0) * gm.K);
        const unsigned kbytes = (unsigned)gm.K * 4u;
        const unsigned voff = (unsigned)(32 * MBW * mg + 4 * h) * kbytes + (unsigned)(nb * 32 + l32) * 4u;
        if (npos >= 32 * (MBW * mg + nblk)) {      // uniform over the wave: every position of its blocks exists
#pragma unroll
            for (int b = 0; b < MBW; ++b)
                if (b < nblk) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) buffer_store(ry, voff, (unsigned)(32 * b + 8 * (i / 4) + (i % 4)) * kbytes, acc[b][i]);
                }
        } else {
#pragma unroll
            for (int b = 0; b < MBW; ++b)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int m = 32 * (MBW * mg + b) + 8 * (i / 4) + 4 * h + (i % 4);
                    if (b < nblk && m < npos) buffer_store(ry, voff, (unsigned)(32 * b + 8 * (i / 4) + (i % 4)) * kbytes, acc[b][i]);
                }
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();      // every wave has read this tile from LDS
        if (next < gm.tiles) stem_fill_write(lds, staged, gm, tid, nthreads);
        __syncthreads();
    }
}

// Forward pass of the 7x7 / stride 2 filter on bf16 pieces.  The input rows under a tile are split once, on their way to LDS, where the three planes of pieces lie as the
// rows do in memory; a filter row's 21 values are three groups of eight (the last three with a filter value of zero), and a reduction step of 16 is two groups, one per half wave: eleven
// steps.  A window begins 6 elements after its neighbour's, on a word boundary, so that a lane's group is four words in a row.  The first two pieces of the filters of a wave's 32 channels stay
// in registers for all its tiles (88 of them), the third in LDS.
// 224x224, 64 channels: batch 184 517 us on the fp32 instruction, 412 so; batch 8 36.4 and 25.4; batch 1 19.8 and 15.0; error against 64 bits 2.2e-7 and 7.0e-8.  What bounds it: 3.1e11 flop of matrix
// instructions (147 products padded to 176), 250 us at the power limit, and 203 us for everything else, which overlap in part: two waves per SIMD.  Stores between the next block's matrix instructions in place of
// behind the own block's: 455 -> 410; the next tile's loads before this tile's products: 485 -> 451, waited for before the first store, since the number of stores behind them is not known to the
// compiler; two blocks at a time 473.  Splitting each window on its way into the instruction had been slower than fp32 (842).
constexpr int STEM7_STEPS = 11;
constexpr int64_t STEM7_WORKGROUPS = 512;      // two on a CU: 416 us; 768 450, 1024 460, 256 489 (batch 184; each loads its filters once)

struct Stem7Geom {
    StemGeom g;              // xlead = 0, whole rows (col_tiles == 1)
    unsigned img_mul, img_shift, qn_mul, qn_shift, row4_mul, row4_shift;      // floor(n / d) = umulhi(n, mul) >> shift; d == 1: mul == 0
    unsigned bytes;          // of an image
};
__device__ __forceinline__ unsigned divide(unsigned n, unsigned mul, unsigned shift) { return mul ? __umulhi(n, mul) >> shift : n; }
struct Stem7Tile { int n, p0; };
__device__ __forceinline__ Stem7Tile stem7_tile(const Stem7Geom &a, unsigned tile) {
    const unsigned n = divide(tile, a.img_mul, a.img_shift);
    return {(int)n, (int)(tile - n * (unsigned)a.g.row_tiles) * a.g.nrow};
}

// The rows under a tile in pieces of 16 bytes, piece tid + k * nthreads; four floats of a row at any offset, zero where the image ends.
__device__ __forceinline__ void stem7_fill_load(bf4 (&v)[FILL], const float *__restrict__ x, const Stem7Geom &a, Stem7Tile at, int tid, int nthreads) {
    const StemGeom &gm = a.g;
    const int row4 = gm.rowlen / 4, rowf = gm.W * 3;
    const __amdgpu_buffer_rsrc_t r = buffer_of((const char *)x + (int64_t)at.n * a.bytes, a.bytes);
    int f0 = -gm.pad * 3;
    asm volatile("" : "+s"(f0));      // anew for every tile: kept from tile to tile, the places in a row would spill (0.4 us a launch)
    const int h0 = at.p0 * 2 - gm.pad;
#pragma unroll
    for (int k = 0; k < FILL; ++k) {
        const int idx = tid + k * nthreads, ri = (int)divide((unsigned)idx, a.row4_mul, a.row4_shift), f = f0 + 4 * (idx - ri * row4), h = h0 + ri;
        const bool row = ri < gm.rows_in && (unsigned)h < (unsigned)gm.H;
        if (f >= 0 && f + 3 < rowf) v[k] = buffer_load4(r, row ? (unsigned)(h * rowf + f) * 4u : BUFFER_ABSENT, 0u);
        else {
#pragma unroll
            for (int u = 0; u < 4; ++u) v[k][u] = buffer_load(r, row && (unsigned)(f + u) < (unsigned)rowf ? (unsigned)(h * rowf + f + u) * 4u : BUFFER_ABSENT, 0u);
        }
    }
}
// ... and their three planes of bf16 pieces, `plane` words apart
__device__ __forceinline__ void stem7_fill_write(unsigned *lds, const bf4 (&v)[FILL], const StemGeom &gm, int plane, int tid, int nthreads, unsigned &lost) {
    const int total = gm.rows_in * (gm.rowlen / 4);
#pragma unroll
    for (int k = 0; k < FILL; ++k) {
        const int idx = tid + k * nthreads;
        if (idx < total) {
            const Pieces a = split_pair(v[k].x, v[k].y, lost), b = split_pair(v[k].z, v[k].w, lost);
            uint2 *at = (uint2 *)(lds + 2 * idx);
            at[0] = make_uint2(a.h, b.h);
            at[plane / 2] = make_uint2(a.m, b.m);
            at[plane] = make_uint2(a.l, b.l);
        }
    }
}

__global__ __launch_bounds__(256, 2) void stem7_fwd_kernel(const float *__restrict__ x, const float *__restrict__ w, float *__restrict__ y, Stem7Geom a) {
    const StemGeom &gm = a.g;
    extern __shared__ float lds[];
    constexpr int R = 7, ST = 2, RUN = 21, KP = 11, MBW = 4;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nthreads = blockDim.x;
    const int nb = wave % (gm.K / 32), mgs = nthreads / 64 / (gm.K / 32);      // as in stem_fwd_kernel
    const int plane = gm.rows_in * gm.rowlen / 2;                    // words
    const float *wk = w + (int64_t)(nb * 32 + l32) * (R * RUN);
    float *rows = lds + gm.K / 32 * (STEM7_STEPS * 64 * 4);
    unsigned lost_w = 0;
    struct { bf16x8 h, m; } wr[STEM7_STEPS];
    bf16x8 *wl = (bf16x8 *)lds + nb * (STEM7_STEPS * 64) + lane;      // the third pieces: every wave of these channels writes and reads the same
#pragma unroll
    for (int t = 0; t < STEM7_STEPS; ++t) {
        const int group = 2 * t + h, r = group / 3, j = 8 * (group - 3 * r);
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = r < R && j + i < RUN ? wk[r * RUN + j + i] : 0.0f;
        const PieceRow p = split_row(v, lost_w);
        wr[t] = {p.h, p.m};
        wl[64 * t] = p.l;
        __builtin_amdgcn_sched_barrier(0);
    }
    const unsigned *pieces = (const unsigned *)rows;
    bf4 staged[FILL];
    unsigned lost = 0;      // of the tile in LDS
    const unsigned tiles = (unsigned)gm.tiles;
    if (blockIdx.x < tiles) {
        stem7_fill_load(staged, x, a, stem7_tile(a, blockIdx.x), tid, nthreads);
        stem7_fill_write((unsigned *)rows, staged, gm, plane, tid, nthreads, lost);
    }
    __syncthreads();
    int mg = wave / (gm.K / 32);
    for (unsigned tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        // The wave's group of position blocks: another one for every tile, as the last group has fewer blocks (seven in all on maps of 112 columns).
        if (++mg >= mgs) mg = 0;
        // LDS word of this lane's position in every block (positions beyond the tile read position 0)
        auto word_of = [&](int b) {
            int m = 32 * (MBW * mg + b) + l32;
            if (m >= gm.nrow * gm.qn) m = 0;
            const int pr = gm.nrow == 1 ? 0 : (int)divide((unsigned)m, a.qn_mul, a.qn_shift);
            return (pr * ST * gm.rowlen + (m - pr * gm.qn) * ST * 3) / 2;
        };
        const auto [n, p0] = stem7_tile(a, tile);
        const int nblk = min(MBW, (gm.nrow * gm.qn + 31) / 32 - MBW * mg);      // position blocks of the nominal tile this wave works on
        // the descriptor ends with the tile: a position beyond it is not stored
        const unsigned kbytes = (unsigned)gm.K * 4u;
        const __amdgpu_buffer_rsrc_t ry = buffer_of(y + ((int64_t)n * gm.P + p0) * gm.Q * gm.K, (unsigned)(min(gm.nrow, gm.P - p0) * gm.Q) * kbytes);
        const unsigned voff = (unsigned)(32 * MBW * mg + 4 * h) * kbytes + (unsigned)(nb * 32 + l32) * 4u;
        auto store_one = [&](int b, int i, const floatx16 &v) { buffer_store(ry, voff, (unsigned)(32 * b + 8 * (i / 4) + (i % 4)) * kbytes, v[i]); };
        auto store = [&](int b, const floatx16 &v) {
#pragma unroll
            for (int i = 0; i < 16; ++i) store_one(b, i, v);
        };
        const unsigned next = tile + gridDim.x;      // fewer than 2^31 tiles
        if (next < tiles) stem7_fill_load(staged, x, a, stem7_tile(a, next), tid, nthreads);      // uniform over the workgroup
        float probe = 0.0f;
        floatx16 prev;      // the block before: its stores go out between the matrix instructions
        auto block = [&](int b, int words, auto first) {
            floatx16 acc, low[2];      // the smaller terms in two sums: a product waits for the one before it on the same sum
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[i] = low[0][i] = low[1][i] = 0.0f;
            bf16x8 ah, am, al, bl;
            unsigned word;
            auto place = [&](int t) {
                // groups 2 t and 2 t + 1: the second eight elements on or, from the third of a row, at the next row's start; the last step has one (its other half's filter
                // values are zero: that half reads the same group)
                const int at = (2 * t / 3 * gm.rowlen + 8 * (2 * t % 3)) / 2, step = t == STEM7_STEPS - 1 ? 0 : 2 * t % 3 == 2 ? (gm.rowlen - 16) / 2 : 4;
                word = (unsigned)(words + h * step + at);
                asm volatile("" : "+v"(word));      // an address of its own each time: eleven of them would take the registers
            };
            auto read = [&](int p) {
                const unsigned *from = pieces + p * plane + word;
                return __builtin_bit_cast(bf16x8, uintx4{from[0], from[1], from[2], from[3]});
            };
            place(0);
            ah = read(0);
            bl = wl[0];
            am = read(1);
            al = read(2);
#pragma unroll
            for (int t = 0; t < STEM7_STEPS; ++t) {      // a plane of the next step is read as soon as the products of this step's are issued
                const bool more = t + 1 < STEM7_STEPS;
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, wr[t].h, acc, 0, 0, 0);
                low[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, wr[t].m, low[0], 0, 0, 0);
                low[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, low[1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (more) {
                    place(t + 1);
                    ah = read(0);
                    bl = wl[64 * (t + 1)];
                }
                __builtin_amdgcn_sched_barrier(0);
                low[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, wr[t].h, low[0], 0, 0, 0);
                low[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, wr[t].m, low[1], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (more) am = read(1);
                __builtin_amdgcn_sched_barrier(0);
                low[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, wr[t].h, low[0], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (more) al = read(2);
                if constexpr (!decltype(first)::value) {
#pragma unroll
                    for (int i = 16 * t / STEM7_STEPS; i < 16 * (t + 1) / STEM7_STEPS; ++i) store_one(b - 1, i, prev);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // The next tile's loads end here, ahead of the stores: waiting for them behind a number of stores that is not known would wait for those as well.
            if constexpr (decltype(first)::value) {
#pragma unroll
                for (int k = 0; k < FILL; ++k) asm volatile("" : "+v"(staged[k].x), "+v"(staged[k].y), "+v"(staged[k].z), "+v"(staged[k].w));
            }
            acc += low[0] + low[1];
#pragma unroll
            for (int i = 0; i < 16; ++i) probe += acc[i];
            prev = acc;
        };
        block(0, word_of(0), std::true_type{});
#pragma unroll 1
        for (int b = 1; b < nblk; ++b) block(b, word_of(b), std::false_type{});      // uniform over the wave
        store(nblk - 1, prev);
        // An infinity or a NaN in a result, or an operand below 2^-110: the tile once more on the fp32 instruction.
        if (__syncthreads_or(!(__builtin_fabsf(probe) < __builtin_inff()) || pieces_lost(lost | lost_w))) {
            const int total = gm.rows_in * (gm.rowlen / 4);
            for (int idx = tid; idx < total; idx += nthreads) {      // the rows as they are
                const int ri = idx / (gm.rowlen / 4), e = 4 * (idx - ri * (gm.rowlen / 4));
                const int hh = p0 * ST - gm.pad + ri, f = e - gm.pad * 3;
                for (int u = 0; u < 4; ++u)
                    rows[4 * idx + u] = (unsigned)hh < (unsigned)gm.H && (unsigned)(f + u) < (unsigned)(gm.W * 3) ? x[((int64_t)n * gm.H + hh) * gm.W * 3 + f + u] : 0.0f;
            }
            __syncthreads();
            for (int b = 0; b < nblk; ++b) {
                int m = 32 * (MBW * mg + b) + l32;
                if (m >= gm.nrow * gm.qn) m = 0;
                const int pr = gm.nrow == 1 ? 0 : m / gm.qn, at = pr * ST * gm.rowlen + (m - pr * gm.qn) * ST * 3;
                floatx16 acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0.0f;
                for (int r = 0; r < R; ++r)
                    for (int t = 0; t < KP; ++t) {      // the padding of the last pair: filter value zero, the window's own value again
                        const int j = 2 * t + h < RUN ? 2 * t + h : 2 * t;
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(rows[at + r * gm.rowlen + j], 2 * t + h < RUN ? wk[r * RUN + j] : 0.0f, acc, 0, 0, 0);
                    }
                store(b, acc);
            }
            __syncthreads();
        }
        lost = 0;
        if (next < tiles) stem7_fill_write((unsigned *)rows, staged, gm, plane, tid, nthreads, lost);
        __syncthreads();
    }
}

// Filter gradient: a workgroup of K / 32 waves walks tiles like the forward kernel; wave kb keeps the 32 x (R * 3 S)
// block of dw of its output channels in registers (NBC column blocks of 32) over all its tiles and leaves it in
// part[workgroup] at the end.

// LDS offset of this lane's column (r, j) in every column block relative to a position's window; a column beyond
// R * 3 S reads the window's first float into a result column that is never written
template <int R, int S, int NBC>
__device__ __forceinline__ void wgrad_columns(int (&coloff)[NBC], const StemGeom &gm) {
    constexpr int RUN = 3 * S, COLS = R * RUN;
    const int l32 = threadIdx.x & 31;
#pragma unroll
    for (int c = 0; c < NBC; ++c) {
        int col = 32 * c + l32;
        if (col >= COLS) col = 0;
        coloff[c] = (col / RUN) * gm.rowlen + col % RUN;
    }
}
// this workgroup's partial result, laid out as dw[k][r][s][c]: lane holds column l32 of rows 8 (i / 4) + 4 h + i % 4
template <int R, int S, int NBC>
__device__ __forceinline__ void wgrad_store(const floatx16 (&acc)[NBC], float *part, const StemGeom &gm) {
    constexpr int COLS = R * 3 * S;
    const int l32 = threadIdx.x & 31, h = (threadIdx.x & 63) >> 5, kb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *mine = part + (int64_t)blockIdx.x * gm.K * COLS;
#pragma unroll
    for (int c = 0; c < NBC; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = kb * 32 + 8 * (i / 4) + 4 * h + (i % 4), col = 32 * c + l32;
            if (col < COLS) mine[row * COLS + col] = acc[c][i];
        }
}
// acc = this workgroup's sums over all its tiles with the fp32 matrix instruction
template <int R, int S, int ST, int NBC>
__device__ __forceinline__ void wgrad_tiles_fp32(floatx16 (&acc)[NBC], const int (&coloff)[NBC], float *lds, const float *__restrict__ x,
                                                 const float *__restrict__ dy, const StemGeom &gm) {
    constexpr int U = NBC >= 4 ? 8 : 16;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int kb = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nthreads = blockDim.x;
#pragma unroll
    for (int c = 0; c < NBC; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][i] = 0.0f;
    const int total4 = gm.rows_in * (gm.rowlen / 4);
    for (int64_t tile = blockIdx.x; tile < gm.tiles; tile += gridDim.x) {
        int n, p0, q0;
        tile_origin(gm, tile, n, p0, q0);
        __syncthreads();      // the previous tile has been read
        for (int k0 = 0; k0 * nthreads < total4; k0 += FILL) {
            float4 staged[FILL];
            stem_fill_load<ST>(staged, x, gm, n, p0, q0, tid, nthreads, k0);
            stem_fill_write(lds, staged, gm, tid, nthreads, k0);
        }
        __syncthreads();
        const int rows_here = min(gm.nrow, gm.P - p0), cols_here = min(gm.qn, gm.Q - q0);
        const int npos = gm.nrow == 1 ? cols_here : rows_here * gm.qn;      // positions of the tile that exist: m * K floats apart in dy
        const __amdgpu_buffer_rsrc_t rdy = buffer_of(dy + (((int64_t)n * gm.P + p0) * gm.Q + q0) * gm.K);
        const unsigned kbytes = (unsigned)gm.K * 4u, lbytes = (unsigned)(kb * 32 + l32) * 4u;
        // groups of U position pairs, two register sets: the dy loads of the next group are issued before the matrix
        // instructions of the current one
        struct Set { float a[U]; int po[U]; };
        auto load = [&](Set &t, int m0) {      // pairs (m0 + 2 u, m0 + 2 u + 1), this lane takes position m0 + 2 u + h
            int m = m0 + h;
            int pr = gm.nrow == 1 ? 0 : m / gm.qn, qq = m - pr * gm.qn;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float got = buffer_load(rdy, (m < npos ? (unsigned)m * kbytes : 0u) + lbytes, 0u);      // in bounds either way
                t.a[u] = m < npos ? got : 0.0f;
                const bool in = pr < gm.nrow;      // a nominal position: its window lies in the staged rows
                t.po[u] = in ? pr * ST * gm.rowlen + qq * ST * 3 + gm.xlead : gm.xlead;
                m += 2; qq += 2;
                if (qq >= gm.qn) { qq -= gm.qn; ++pr; }
            }
        };
        // A position beyond the tile is no term of the sum: neither operand may stand there as it is (its window in LDS is real
        // image data, and zero times an infinity would be a NaN).  Only a tile's last group has such positions.
        auto compute = [&](const Set &t, int m0) {
            if (m0 + 2 * U <= npos) {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int c = 0; c < NBC; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(t.a[u], lds[t.po[u] + coloff[c]], acc[c], 0, 0, 0);
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int c = 0; c < NBC; ++c) {
                        const float w = lds[t.po[u] + coloff[c]];
                        acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(t.a[u], m0 + 2 * u + h < npos ? w : 0.0f, acc[c], 0, 0, 0);
                    }
            }
        };
        const int groups = (npos + 2 * U - 1) / (2 * U);
        Set s0, s1;
        if (groups > 0) load(s0, 0);
        for (int g = 0; g < groups; g += 2) {
            if (g + 1 < groups) load(s1, (g + 1) * 2 * U);
            __builtin_amdgcn_sched_barrier(0);
            compute(s0, g * 2 * U);
            __builtin_amdgcn_sched_barrier(0);
            if (g + 2 < groups) load(s0, (g + 2) * 2 * U);
            __builtin_amdgcn_sched_barrier(0);
            if (g + 1 < groups) compute(s1, (g + 1) * 2 * U);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Filter gradient of the 7x7 / stride 2 filter on bf16 pieces.
template <int R, int S, int ST>
__global__ __launch_bounds__(256, 2) void stem7_wgrad_kernel(const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part, StemGeom gm) {
    extern __shared__ float lds[];
    constexpr int NBC = (R * 3 * S + 31) / 32;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int kb = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nthreads = blockDim.x;
    int coloff[NBC];
    wgrad_columns<R, S>(coloff, gm);
    floatx16 acc[NBC], low[NBC];      // the h * h terms and the smaller ones
    const int total4 = gm.rows_in * (gm.rowlen / 4);
    __shared__ int redo;              // an infinity or a NaN in the result, or an operand too small to split: all tiles once more on the fp32 instruction
#pragma unroll
    for (int c = 0; c < NBC; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][i] = low[c][i] = 0.0f;
    if (tid == 0) redo = 0;           // read behind the barriers below
    unsigned lost = 0;      // bits of operands too small to be three pieces
    for (int64_t tile = blockIdx.x; tile < gm.tiles; tile += gridDim.x) {
        int n, p0, q0;
        tile_origin(gm, tile, n, p0, q0);
        __syncthreads();      // the previous tile has been read
        for (int k0 = 0; k0 * nthreads < total4; k0 += FILL) {
            float4 staged[FILL];
            stem_fill_load<ST>(staged, x, gm, n, p0, q0, tid, nthreads, k0);
            stem_fill_write(lds, staged, gm, tid, nthreads, k0);
        }
        __syncthreads();
        const int rows_here = min(gm.nrow, gm.P - p0), cols_here = min(gm.qn, gm.Q - q0);
        const int npos = gm.nrow == 1 ? cols_here : rows_here * gm.qn;      // positions of the tile that exist: m * K floats apart in dy
        // the descriptor ends with the tile: a position beyond it reads zero
        const __amdgpu_buffer_rsrc_t rdy = buffer_of(dy + (((int64_t)n * gm.P + p0) * gm.Q + q0) * gm.K, (unsigned)(npos * gm.K) * 4u);
        const unsigned kbytes = (unsigned)gm.K * 4u, lbytes = (unsigned)(kb * 32 + l32) * 4u;
        // groups of 16 positions, two register sets: the dy loads of the next group are issued before the matrix
        // instructions of the current one.  A position beyond the tile contributes zero times its window
        // in LDS; where that holds an infinity the NaN sends the workgroup to the fp32 pass.
        struct Set { float a[8]; };
        auto load = [&](Set &t, int m0) {      // this lane takes positions m0 + 8 h .. m0 + 8 h + 7
            const unsigned first = (unsigned)(m0 + 8 * h) * kbytes + lbytes;
#pragma unroll
            for (int i = 0; i < 8; ++i) t.a[i] = buffer_load(rdy, first, (unsigned)i * kbytes);
        };
        auto compute = [&](const Set &t, int m0) {
            int po[8];
            {
                const int m = m0 + 8 * h;
                int pr = gm.nrow == 1 ? 0 : m / gm.qn, qq = m - pr * gm.qn;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const bool in = pr < gm.nrow && qq < gm.qn;      // a nominal position: its window lies in the staged rows
                    po[i] = in ? pr * ST * gm.rowlen + qq * ST * 3 + gm.xlead : gm.xlead;
                    ++qq;
                    if (gm.nrow > 1 && qq >= gm.qn) { qq -= gm.qn; ++pr; }
                }
            }
            const PieceRow a = split_row(t.a, lost);
            float v[8], next[8];
            auto read = [&](int c, float (&o)[8]) {
#pragma unroll
                for (int i = 0; i < 8; ++i) o[i] = lds[po[i] + coloff[c]];
            };
            read(0, v);
#pragma unroll
            for (int c = 0; c < NBC; ++c) {
                if (c + 1 < NBC) read(c + 1, next);
                __builtin_amdgcn_sched_barrier(0);
                const PieceRow b = split_row(v, lost);
                acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.h, acc[c], 0, 0, 0);
                low[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.m, low[c], 0, 0, 0);
                low[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.h, low[c], 0, 0, 0);
                low[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.m, b.m, low[c], 0, 0, 0);
                low[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.h, b.l, low[c], 0, 0, 0);
                low[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.l, b.h, low[c], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);      // the splits of several columns gathered ahead would not fit the registers
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = next[i];
            }
        };
        const int groups = (npos + 15) / 16;
        Set s0, s1;
        if (groups > 0) load(s0, 0);
        for (int g = 0; g < groups; g += 2) {
            if (g + 1 < groups) load(s1, (g + 1) * 16);
            __builtin_amdgcn_sched_barrier(0);
            compute(s0, g * 16);
            if (g + 2 < groups) load(s0, (g + 2) * 16);
            __builtin_amdgcn_sched_barrier(0);
            if (g + 1 < groups) compute(s1, (g + 1) * 16);
        }
    }
#pragma unroll
    for (int c = 0; c < NBC; ++c) acc[c] += low[c];
    __syncthreads();      // redo is zero, also where there was no tile
    {
        float sum = 0.0f;
#pragma unroll
        for (int c = 0; c < NBC; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += acc[c][i];
        if (!(__builtin_fabsf(sum) < __builtin_inff()) || pieces_lost(lost)) redo = 1;
    }
    __syncthreads();
    if (redo) wgrad_tiles_fp32<R, S, ST>(acc, coloff, lds, x, dy, gm);      // uniform over the workgroup
    wgrad_store<R, S>(acc, part, gm);
}

// Filter gradient of the 3x3 filters, on the fp32 matrix instruction: 27 columns, bound by reading dy, which groups of 16 positions
// in place of 32 slowed down (stride 1, 64 channels, 224x224, batch 176: 755 against 866 us).
template <int R, int S, int ST>
__global__ __launch_bounds__(256, 2) void stem_wgrad_kernel(const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part, StemGeom gm) {
    extern __shared__ float lds[];
    constexpr int NBC = (R * 3 * S + 31) / 32;
    int coloff[NBC];
    wgrad_columns<R, S>(coloff, gm);
    floatx16 acc[NBC];
    wgrad_tiles_fp32<R, S, ST>(acc, coloff, lds, x, dy, gm);
    wgrad_store<R, S>(acc, part, gm);
}

struct StemPlan { bool ok; int R, S, ST, mbw; StemGeom gm; size_t lds_bytes; };

StemPlan stem_plan(const ConvShape &cs) {
    StemPlan sp{};
    if (cs.C != 3 || cs.R != cs.S || cs.K % 32 || cs.K < 32 || cs.K > 128) return sp;
    if (!((cs.R == 7 && cs.stride == 2) || (cs.R == 3 && (cs.stride == 1 || cs.stride == 2)))) return sp;
    if (cs.pad < 0 || cs.pad > cs.R || (int64_t)cs.N * cs.H * cs.W * 3 >= ((int64_t)1 << 31) || cs.M() * cs.K >= ((int64_t)1 << 40)) return sp;
    sp.R = cs.R; sp.S = cs.S; sp.ST = cs.stride;
    StemGeom &gm = sp.gm;
    gm.N = cs.N; gm.H = cs.H; gm.W = cs.W; gm.P = cs.P; gm.Q = cs.Q; gm.K = cs.K; gm.pad = cs.pad;
    // a tile: as many whole output rows as 224 positions hold (seven blocks of 32: two waves' worth), else segments of one
    // row; with 96 or 128 output channels one wave's worth, so that a workgroup stays within four waves
    const int cap = cs.K > 64 ? 128 : 224;
    if (cs.Q <= cap) { gm.nrow = std::max(1, std::min(cap / cs.Q, cs.P)); gm.qn = cs.Q; }
    else { gm.nrow = 1; gm.qn = cap; }
    const int blocks = (gm.nrow * gm.qn + 31) / 32;
    sp.mbw = (blocks + 3) / 4;      // groups of four position blocks, one wave each per 32 output channels
    if (sp.mbw * (cs.K / 32) > 4) return sp;
    gm.row_tiles = (cs.P + gm.nrow - 1) / gm.nrow;
    gm.col_tiles = (cs.Q + gm.qn - 1) / gm.qn;
    gm.tiles = (int64_t)cs.N * gm.row_tiles * gm.col_tiles;
    gm.rows_in = (gm.nrow - 1) * cs.stride + cs.R;
    gm.xlead = (4 - (cs.pad * 3) % 4) % 4;
    // floats of an LDS row: up to the last tap of the tile's last position, plus the reduction padding, rounded up
    const int need = gm.xlead + ((gm.qn - 1) * cs.stride + cs.S) * 3 + 2;
    gm.rowlen = (need + 3) / 4 * 4;
    sp.lds_bytes = (size_t)gm.rows_in * gm.rowlen * sizeof(float);
    if (sp.lds_bytes > 64 * 1024 || gm.rows_in * (gm.rowlen / 4) > FILL * 64 * (cs.K / 32) * sp.mbw) return sp;
    sp.ok = true;
    return sp;
}

template <int R, int S, int ST>
void launch_stem_fwd(hipStream_t st, const float *x, const float *w, float *y, const StemPlan &sp) {
    const unsigned block = 64u * (unsigned)(sp.gm.K / 32) * (unsigned)sp.mbw;
    // workgroups of a launch: each keeps its filters for all its tiles (measured on the ResNet-50, MobileNetV2 and VGG-16
    // first layers: 1024 workgroups at or near the best time, 256 and one per tile 10-25 % slower)
    const unsigned grid = (unsigned)std::min<int64_t>(sp.gm.tiles, 1024);
    if constexpr (R == 7) {
        Stem7Geom a{};
        StemGeom &gm = a.g = sp.gm;
        gm.xlead = 0;
        gm.rowlen = ((gm.qn - 1) * 6 + 24 + 3) / 4 * 4;      // the last window's third group of eight ends inside
        magic_of((unsigned)gm.row_tiles, a.img_mul, a.img_shift);
        magic_of((unsigned)gm.qn, a.qn_mul, a.qn_shift);
        magic_of((unsigned)gm.rowlen / 4, a.row4_mul, a.row4_shift);
        const int64_t image = (int64_t)gm.H * gm.W * 12;
        a.bytes = (unsigned)image;
        const size_t bytes = (size_t)gm.rows_in * gm.rowlen * 6 + (size_t)gm.K / 32 * STEM7_STEPS * 1024;
        // Beyond 64 KiB (64 channels and 168 positions in a row or more, 96 and 123, 128 and 78, or two rows of 60 to 64, rows cut into segments among them) the fp32 instruction stays.
        if (gm.col_tiles == 1 && bytes <= 64 * 1024 && image < 12ll << 28 && gm.tiles < ((int64_t)1 << 30)) {
            hipLaunchKernelGGL(stem7_fwd_kernel, dim3((unsigned)std::min(sp.gm.tiles, STEM7_WORKGROUPS)), dim3(block), bytes, st, x, w, y, a);
            hip_check(hipGetLastError(), "stem_fwd launch");
            return;
        }
    }
    hipLaunchKernelGGL((stem_fwd_kernel<R, S, ST>), dim3(grid), dim3(block), sp.lds_bytes, st, x, w, y, sp.gm);
    hip_check(hipGetLastError(), "stem_fwd launch");
}

// workgroups of the filter gradient: one partial result each, as many as the caller's split count allows
int stem_wgrad_groups(const StemPlan &sp, int splits) { return (int)std::min<int64_t>({(int64_t)splits, (int64_t)1024, sp.gm.tiles}); }

template <int R, int S, int ST>
void launch_stem_wgrad(hipStream_t st, const float *x, const float *dy, float *ws, const StemPlan &sp, int groups) {
    if constexpr (R == 7) hipLaunchKernelGGL((stem7_wgrad_kernel<R, S, ST>), dim3((unsigned)groups), dim3(64u * (unsigned)(sp.gm.K / 32)), sp.lds_bytes, st, x, dy, ws, sp.gm);
    else hipLaunchKernelGGL((stem_wgrad_kernel<R, S, ST>), dim3((unsigned)groups), dim3(64u * (unsigned)(sp.gm.K / 32)), sp.lds_bytes, st, x, dy, ws, sp.gm);
    hip_check(hipGetLastError(), "stem_wgrad launch");
}

}  // namespace

bool stem_applies(const ConvShape &cs) { return stem_plan(cs).ok; }

bool stem_wgrad_applies(const ConvShape &cs, int splits, size_t ws_bytes) {
    const StemPlan sp = stem_plan(cs);
    if (!sp.ok || splits < 2) return false;
    // the filter gradient fills LDS in rounds of FILL pieces per thread: any tile the forward plan accepts will do
    return ws_bytes >= (size_t)stem_wgrad_groups(sp, splits) * cs.K * cs.RSC() * sizeof(float);
}

void stem_wgrad(hipStream_t st, const float *x, const float *dy, float *dw, const ConvShape &cs, int splits, float *ws, size_t ws_bytes) {
    if (!stem_wgrad_applies(cs, splits, ws_bytes)) throw KernelError("stem_wgrad: shape, split count or workspace not supported");
    const StemPlan sp = stem_plan(cs);
    const int groups = stem_wgrad_groups(sp, splits);
    if (sp.R == 7) launch_stem_wgrad<7, 7, 2>(st, x, dy, ws, sp, groups);
    else if (sp.ST == 2) launch_stem_wgrad<3, 3, 2>(st, x, dy, ws, sp, groups);
    else launch_stem_wgrad<3, 3, 1>(st, x, dy, ws, sp, groups);
    split_reduce(st, ws, dw, (int64_t)cs.K * cs.RSC(), groups, false);
}

void stem_fwd(hipStream_t st, const float *x, const float *w, float *y, const ConvShape &cs) {
    const StemPlan sp = stem_plan(cs);
    if (!sp.ok) throw KernelError("stem_fwd: needs three input channels, a 7x7 / stride 2 or 3x3 / stride 1 or 2 filter and 32, 64, 96 or 128 output channels");
    if (sp.R == 7) launch_stem_fwd<7, 7, 2>(st, x, w, y, sp);
    else if (sp.ST == 2) launch_stem_fwd<3, 3, 2>(st, x, w, y, sp);
    else launch_stem_fwd<3, 3, 1>(st, x, w, y, sp);
}

}  // namespace monet
