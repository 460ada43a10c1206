// Filter gradient of a 3x3 / stride 1 / pad 1 layer by Winograd F(4x4, 3x3): dW = G^T [ sum over tiles (A dy A^T) .* (B^T d B) ] G
//
// Each two-dimensional map is a vertical one and a horizontal one.  The vertical maps go through memory, six rows for every four of the map (1.5 times the tensors
// instead of the 2.25 of the tiles mapped both ways):
//   X[a][n, ti][j][c] = (B^T d)[a][j], columns j = 0 .. 4 tw + 1 of the input from column -1 on      D[a][n, ti][j][k] = (A dy)[a][j], columns 0 .. 4 tw - 1
// with zeros where the map ends, so that nobody behind them tests for its border.  The horizontal ones are made on the way into the 36 GEMMs: a workgroup owns one row a
// of the transform positions (z = 6a .. 6a + 5), 64 filters and 64 input channels, and walks a range of tiles in chunks of 16, double-buffered through LDS:
//   * eight waves map: a lane reads the six (four) columns of one tile for two channels, exchanges one of them with the lane that has the neighbouring tile, maps, splits into
//     three bf16 pieces per float (bf16_pieces.hpp) and leaves words of two tiles in LDS;
//   * eight waves multiply the chunk before, three blocks of 32 x 32 each of the 24 (six positions, 2 x 2 blocks), on v_mfma_f32_32x32x16_bf16 as in conv.hip: six per
//     fp32 product, the h * h terms and the rest in sums of their own.
// What bounds it (176x112x112, 128 -> 128: in eight chunks of images 1.09 ms of vertical maps at 5.2 TB/s, 1.72 ms of GEMMs, 0.05 ms of range sums): the waves that map, 200 vector instructions a chunk each, of which 144 split; 1.5 us a chunk,
// 1.0 without their loads, 0.9 for the matrix instructions alone.  Words of two tiles keep their LDS reads and writes free of conflicts (a quarter of the LDS cycles with the channels in
// order).  Measured and not taken: both maps of either operand in this kernel, which reads every patch once for each of its six rows (3390 us against 3105 of the workspace form, 2807 this way);
// loads four chunks ahead (3 % slower); every partial sum in a place of its own for the range sum to add (1 - 10 % slower than adding to the range's).
#include "bf16_pieces.hpp"
#include "winograd_f4.hpp"

namespace monet {

namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int CT = 16;                     // tiles per chunk
constexpr int WAVES = 8, BLOCK = 64;       // waves of each kind; filters, input channels of a workgroup
constexpr int ROW = BLOCK;                 // words of one pair of tiles: channels 0, 2, .. 62, 1, 3, .. 63 of the block
constexpr int PLANE = CT / 2 * ROW;        // words of one position's piece
constexpr int OPERAND = 6 * 3 * PLANE;     // one operand of a chunk

struct VerticalArgs {
    const float *x, *dy;
    float *X, *D;
    int H, W, C, K;
    unsigned rows, th, px, pd;      // rows of tiles (images * th); columns of X and D
    unsigned blocks_x;              // workgroups of X, the others make D
};

// One thread per (row of tiles, column, four channels).
__global__ __launch_bounds__(256) void wino4_vertical_kernel(VerticalArgs a) {
    const bool is_x = blockIdx.x < a.blocks_x;      // uniform
    const unsigned chan4 = (unsigned)(is_x ? a.C : a.K) / 4, cols = is_x ? a.px : a.pd;
    const unsigned idx = (is_x ? blockIdx.x : blockIdx.x - a.blocks_x) * 256u + threadIdx.x;      // a plane has fewer than 2^28 of them
    if (idx >= a.rows * cols * chan4) return;
    const unsigned pos = idx / chan4, c4 = idx - pos * chan4, r = pos / cols, j = pos - r * cols;
    const unsigned n = r / a.th;
    const int h0 = 4 * (int)(r - n * a.th);
    const int64_t plane = a.rows * cols * chan4;
    f4 *out = (f4 *)(is_x ? a.X : a.D) + idx;
    f4 v[6], o[6];
    const int w = is_x ? (int)j - 1 : (int)j, first = is_x ? h0 - 1 : h0;
    const f4 *in = (const f4 *)(is_x ? a.x : a.dy) + (((int64_t)n * a.H + first) * a.W + w) * chan4 + c4;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int h = first + i;
        v[i] = f4{0, 0, 0, 0};
        if ((is_x || i < 4) && (unsigned)w < (unsigned)a.W && (unsigned)h < (unsigned)a.H) v[i] = in[(int64_t)i * a.W * chan4];
    }
    if (is_x) {
        const f4 p = v[4] - 4.0f * v[2], q = v[3] - 4.0f * v[1], s = v[4] - v[2], t = v[3] - v[1];
        o[0] = 4.0f * v[0] - 5.0f * v[2] + v[4];
        o[1] = p + q;
        o[2] = p - q;
        o[3] = s + 2.0f * t;
        o[4] = s - 2.0f * t;
        o[5] = 4.0f * v[1] - 5.0f * v[3] + v[5];
    } else {
        const f4 p = v[0] + v[2], q = v[1] + v[3], s = v[0] + 4.0f * v[2], t = 2.0f * v[1] + 8.0f * v[3];
        o[0] = v[0];
        o[1] = p + q;
        o[2] = p - q;
        o[3] = s + t;
        o[4] = s - t;
        o[5] = v[3];
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) out[i * plane] = o[i];
}

struct WgradArgs {
    const float *X, *D;
    float *out;               // [range][36][K][C]
    int C, K;
    unsigned T, tw, tw_mul, tw_shift;      // tiles; floor(n / tw) = umulhi(n, mul) >> shift
    unsigned px, pd;                       // columns of X and D
    unsigned chunks, per_range, items;
    unsigned per_part;        // chunks whose products are added up in the matrix instruction, before their sum goes to memory
    int kb, cb;               // blocks of 64 filters, input channels
    unsigned x_plane, d_plane;      // bytes
};

struct Range { unsigned first, last; };      // chunks

// The waves that map, each the same two tiles of every chunk.
__device__ __forceinline__ void map_tiles(const WgradArgs &a, unsigned *lds, int *redo, int wave, int lane, int row, int kblock, int cblock, Range at) {
    const int l32 = lane & 31, g = lane >> 5;
    const unsigned first = at.first, last = at.last;
    const __amdgpu_buffer_rsrc_t rx = buffer_of((const char *)a.X + (int64_t)row * a.x_plane, a.x_plane), rd = buffer_of((const char *)a.D + (int64_t)row * a.d_plane, a.d_plane);
    const int cx = cblock * BLOCK + 2 * l32, cd = kblock * BLOCK + 2 * l32;      // two channels per lane (their number is a multiple of 4)
    struct Raw { f2 x[6], d[4]; };
    auto load2 = [](__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff) { return __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0)); };
    // tile 2 * wave + g of the chunk; a tile beyond the last one, or beyond the range, reads zeros
    auto load = [&](Raw &raw, unsigned chunk) {
        const unsigned t = chunk * CT + 2u * wave + g;
        const bool in = chunk < last && t < a.T;
        const unsigned r = a.tw == 1 ? t : __umulhi(t, a.tw_mul) >> a.tw_shift, j = 4u * (t - r * a.tw);
        const unsigned vx = in && cx < a.C ? ((r * a.px + j) * (unsigned)a.C + (unsigned)cx) * 4u : BUFFER_ABSENT;
        const unsigned vd = in && cd < a.K ? ((r * a.pd + j) * (unsigned)a.K + (unsigned)cd) * 4u : BUFFER_ABSENT;
#pragma unroll
        for (int b = 0; b < 6; ++b) raw.x[b] = load2(rx, vx, (unsigned)(b * a.C) * 4u);
#pragma unroll
        for (int b = 0; b < 4; ++b) raw.d[b] = load2(rd, vd, (unsigned)(b * a.K) * 4u);
    };
    // put(operand, position, values of both tiles), operand 0: dy, 1: x; one channel per lane
    auto map = [&](const Raw &raw, auto loaded, auto put) {
        // (channel 2 l32 + g of both tiles) from (channels 2 l32, 2 l32 + 1 of tile g)
        auto pair_up = [](f2 v, float (&s)[2]) {
            const auto e = __builtin_amdgcn_permlane32_swap(__float_as_uint(v.x), __float_as_uint(v.y), false, false);
            s[0] = __uint_as_float(e[0]);
            s[1] = __uint_as_float(e[1]);
        };
        float sx[6][2], sd[4][2], o[2][6];
#pragma unroll
        for (int b = 0; b < 6; ++b) pair_up(raw.x[b], sx[b]);
#pragma unroll
        for (int b = 0; b < 4; ++b) pair_up(raw.d[b], sd[b]);
        __builtin_amdgcn_sched_barrier(0);
        loaded();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 2; ++u) f4_bt(sx[0][u], sx[1][u], sx[2][u], sx[3][u], sx[4][u], sx[5][u], o[u]);
#pragma unroll
        for (int b = 0; b < 6; ++b) put(1, b, o[0][b], o[1][b]);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float p = sd[0][u] + sd[2][u], q = sd[1][u] + sd[3][u];
            const float r = __builtin_fmaf(4.0f, sd[2][u], sd[0][u]), t = __builtin_fmaf(8.0f, sd[3][u], 2.0f * sd[1][u]);
            o[u][0] = sd[0][u];
            o[u][1] = p + q;
            o[u][2] = p - q;
            o[u][3] = r + t;
            o[u][4] = r - t;
            o[u][5] = sd[3][u];
        }
#pragma unroll
        for (int b = 0; b < 6; ++b) put(0, b, o[0][b], o[1][b]);
    };
    unsigned lost = 0;
    const int put_at = wave * ROW + lane;
    auto put_pieces = [&](unsigned buf) {
        unsigned *base = lds + buf * (2 * OPERAND) + put_at;
        return [&lost, base](int operand, int b, float v0, float v1) {
            unsigned *to = base + operand * OPERAND + 3 * b * PLANE;
            const Pieces p = split_pair(v0, v1, lost);
            to[0] = p.h;
            to[PLANE] = p.m;
            to[2 * PLANE] = p.l;
        };
    };
    // chunk c + 1 is mapped while c is multiplied; its loads were issued two chunks earlier
    Raw even, odd;      // chunks first, first + 2, ..; first + 1, ..
    load(even, first);
    load(odd, first + 1);
    map(even, [&] { load(even, first + 2); }, put_pieces(0));
    __syncthreads();
    for (unsigned c = first; c < last; c += 2) {
        map(odd, [&] { load(odd, c + 3); }, put_pieces(1));
        __syncthreads();
        if (c + 1 >= last) break;
        map(even, [&] { load(even, c + 4); }, put_pieces(0));
        __syncthreads();
    }
    if (pieces_lost(lost)) *redo = 1;
    __syncthreads();
    if (!*redo) return;
    float *f = (float *)lds;      // [operand][position][tile][channel]
    for (unsigned c = first; c < last; ++c) {
        load(even, c);
        map(even, [] {}, [&](int operand, int b, float v0, float v1) {
            float *to = f + operand * OPERAND + (b * CT + 2 * wave) * ROW + lane;
            to[0] = v0;
            to[ROW] = v1;
        });
        __syncthreads();
        __syncthreads();
    }
}

// The waves that multiply, and write the results.
__device__ __forceinline__ void multiply_tiles(const WgradArgs &a, const unsigned *lds, int *redo, int wave, int lane, int row, int kblock, int cblock, unsigned range, Range at) {
    const int l32 = lane & 31, g = lane >> 5;
    const unsigned first = at.first, last = at.last;
    // this wave's blocks: 32 filters (half), both halves of the channels at position z2, one of them at position z1
    const int half = wave & 1, quad = wave >> 1;
    const int z2 = quad + (quad + 1) / 2, z1 = quad < 2 ? 1 : 4, j1 = quad & 1;      // z2 = 0, 2, 3, 5
    floatx16 acc[3], low[3];
    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = low[i][v] = 0.0f;
    };
    const unsigned lane_at = 4 * g * ROW + l32;
    auto multiply = [&](unsigned buf_at) {
        auto from = [&](unsigned at, int block) {      // an address of its own each time: kept from chunk to chunk they would take the registers
            at += buf_at + lane_at + 32u * block;
            asm volatile("" : "+v"(at));
            return lds + at;
        };
        auto fragment = [&](const unsigned *at) { return __builtin_bit_cast(bf16x8, uintx4{at[0], at[ROW], at[2 * ROW], at[3 * ROW]}); };
        bf16x8 ah, am, al;
        auto filters = [&](int z) {
            const unsigned *at = from(3 * z * PLANE, half);
            ah = fragment(at);
            am = fragment(at + PLANE);
            al = fragment(at + 2 * PLANE);
        };
        auto block = [&](int i, int z, int j) {
            const unsigned *at = from(OPERAND + 3 * z * PLANE, j);
            const bf16x8 bh = fragment(at), bm = fragment(at + PLANE), bl = fragment(at + 2 * PLANE);
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, acc[i], 0, 0, 0);
            low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bm, low[i], 0, 0, 0);
            low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bh, low[i], 0, 0, 0);
            low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(am, bm, low[i], 0, 0, 0);
            low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, low[i], 0, 0, 0);
            low[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, low[i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        filters(z2);
        block(0, z2, 0);
        block(1, z2, 1);
        filters(z1);
        block(2, z1, j1);
    };
    // Lane (l32, g) holds column l32 of rows 8 * (v / 4) + 4 * g + v % 4 of a block: channel 2 * l32 + j and filters 2 * row + half of the workgroup's 64.  A row beyond the last filter
    // lies beyond the plane.
    auto store = [&](bool add) {
        const int k0 = kblock * BLOCK + half + 8 * g;
        const unsigned plane = (unsigned)a.K * (unsigned)a.C;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int z = 6 * row + (i < 2 ? z2 : z1), col = cblock * BLOCK + 2 * l32 + (i < 2 ? i : j1);
            const __amdgpu_buffer_rsrc_t ro = buffer_of(a.out + ((int64_t)range * 36 + z) * plane, plane * 4u);
            const unsigned voff = col < a.C ? ((unsigned)k0 * (unsigned)a.C + (unsigned)col) * 4u : BUFFER_ABSENT;
            if (add) {
                float old[16];
#pragma unroll
                for (int v = 0; v < 16; ++v) old[v] = buffer_load(ro, voff, (unsigned)(2 * (8 * (v >> 2) + (v & 3)) * a.C) * 4u);
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][v] += old[v];
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) buffer_store(ro, voff, (unsigned)(2 * (8 * (v >> 2) + (v & 3)) * a.C) * 4u, acc[i][v]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    float probe = 0.0f;
    __syncthreads();
    for (unsigned c = first; c < last;) {
        const bool later = c > first;
        clear();
        const unsigned end = min(c + a.per_part, last);
        for (; c < end; ++c) {
            multiply((c - first) % 2 * (2 * OPERAND));
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            acc[i] += low[i];
#pragma unroll
            for (int v = 0; v < 16; ++v) probe += acc[i][v];
        }
        store(later);
    }
    // An infinity, a NaN or a mapped value below 2^-110: once more on the fp32 instruction, as in conv.hip.
    if (!(__builtin_fabsf(probe) < __builtin_inff())) *redo = 1;
    __syncthreads();
    if (!*redo) return;
    const float *f = (const float *)lds;
    for (unsigned c = first; c < last;) {
        const bool later = c > first;
        clear();
        const unsigned end = min(c + a.per_part, last);
        for (; c < end; ++c) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int z = i < 2 ? z2 : z1, j = i < 2 ? i : j1;
#pragma unroll
                for (int k = 0; k < CT; k += 2)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(f[(z * CT + k + g) * ROW + half * 32 + l32], f[OPERAND + (z * CT + k + g) * ROW + j * 32 + l32], acc[i], 0, 0, 0);
            }
            __syncthreads();
        }
        store(later);
    }
}

__global__ __launch_bounds__(64 * 2 * WAVES) void wino4_wgrad_kernel(WgradArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned lds[4 * OPERAND];
    __shared__ int redo;
    // A contiguous share of the items per XCD (winograd_f4.hpp), ranges slowest and rows next: the blocks that read the same columns meet in one L2.
    const unsigned item = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (item >= a.items) return;
    const unsigned blocks = (unsigned)(a.kb * a.cb), per = 6 * blocks;
    const unsigned range = item / per, rest = item - range * per, row = rest / blocks, b = rest - row * blocks;
    const int kblock = (int)(b / (unsigned)a.cb), cblock = (int)(b - (unsigned)kblock * (unsigned)a.cb);
    const Range at{range * a.per_range, min((range + 1) * a.per_range, a.chunks)};
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (threadIdx.x == 0) redo = 0;      // set behind barriers
    if (wave < WAVES) multiply_tiles(a, lds, &redo, wave, lane, (int)row, kblock, cblock, range, at);
    else map_tiles(a, lds, &redo, wave - WAVES, lane, (int)row, kblock, cblock, at);
}

// workgroups of one range
int64_t blocks_of(const ConvShape &cs) { return 6ll * ((cs.K + BLOCK - 1) / BLOCK) * ((cs.C + BLOCK - 1) / BLOCK); }
int64_t tiles_of(const ConvShape &cs) { return (int64_t)cs.N * ((cs.H + 3) / 4) * ((cs.W + 3) / 4); }
size_t columns_of(const ConvShape &cs) { return (size_t)((cs.W + 3) / 4) * 4 + 2; }
constexpr int64_t PLANE_FLOATS = ((int64_t)1 << 30) - 16384;      // a plane is addressed with 32-bit byte offsets

struct Split { unsigned per_range; double us; };
// How a launch divides the `chunks` of its reduction, into at most `most` ranges: the quickest of one to four rounds of workgroups, at 1.5 us a chunk, 8 us a workgroup and 4 TB/s for
// the partial results.
Split split_of(unsigned chunks, int most, const ConvShape &cs) {
    const int64_t per = blocks_of(cs);
    Split best{0, 0};
    for (int round = 1; round <= 4; ++round) {
        unsigned r = (unsigned)std::max<int64_t>(1, std::min<int64_t>({(int64_t)most, (int64_t)chunks, FUSED_CUS * round / per}));
        const unsigned len = (chunks + r - 1) / r;
        r = (chunks + len - 1) / len;
        const double us = (double)((per * r + FUSED_CUS - 1) / FUSED_CUS) * (1.5 * len + 8) + (r > 1 ? r * 36.0 * cs.K * cs.C * 4 * 2 / 4e6 : 0);
        if (best.per_range == 0 || us < best.us) best = {len, us};
    }
    return best;
}

}  // namespace

size_t winograd_wgrad_image_floats(const ConvShape &cs) { return 6 * (size_t)((cs.H + 3) / 4) * (columns_of(cs) * cs.C + (columns_of(cs) - 2) * cs.K); }

int winograd_wgrad_most_images(const ConvShape &cs) {
    const int64_t th = (cs.H + 3) / 4, tw = (cs.W + 3) / 4;
    return (int)std::min<int64_t>({(int64_t)cs.N, PLANE_FLOATS / (th * (int64_t)columns_of(cs) * std::max(cs.C, cs.K)), ((1 << 24) - 1) / (th * tw)});
}

// Measured against the workspace form (us in a launched graph, that form and this).  Its tiles of 128 x 128 leave half of themselves empty where one side has no more than 64 channels: up to five
// pairs of blocks 0.42 - 0.97 of its time at any number of tiles (176x112x112 64 -> 128 2417 and 1665, 8x28x28 320 -> 64 41 and 31).  With two blocks and more on both sides, four or six pairs,
// 0.76 - 0.99 from 256 to 900 tiles and from 3000 on (176x112x112 128 -> 128 3099 and 2750); in between the ranges that fill the CUs cost more to add up than they save (1568 tiles
// 128 -> 128 47.4 and 53.4, 2048 192 -> 128 73.4 and 78.2), from 129 to 255 that form works uncut (196 tiles 36.3 and 39.6).  Every further pair reads and splits the vertical maps
// once more, while those tiles do with fewer of both: from eight on 1.0 - 1.7 (184x14x14 256 -> 256 189 and 230, 176x28x28 512 -> 512 1667 and 1800), except for few tiles, where
// two launches less count, as long as one round of workgroups does it: up to 128 tiles and 42 pairs 0.83 - 1.0 (1x14x14 320 -> 256 23.8 and 21.2), with 49 pairs and more 1.0 - 1.48
// (32x7x7 1024 -> 1024 118 and 160).
bool winograd_wgrad_applies(const ConvShape &cs) {
    const int64_t pairs = blocks_of(cs) / 6, tiles = tiles_of(cs);
    const bool wide = cs.K > BLOCK && cs.C > BLOCK;
    if (winograd_wgrad_most_images(cs) < 1) return false;
    if (tiles <= 128) return blocks_of(cs) <= FUSED_CUS;
    return pairs <= (wide ? 0 : 5) || (pairs <= 6 && ((tiles >= 256 && tiles <= 900) || tiles >= 3000));
}

double winograd_wgrad_estimate(const ConvShape &cs, int images, int most) {
    ConvShape part = cs;
    part.N = images;
    const double map_bytes = (double)images * cs.H * cs.W * (cs.C + cs.K) * 4 * 2.5;
    return split_of((unsigned)((tiles_of(part) + CT - 1) / CT), most, cs).us + map_bytes / 5.5e6 + 12;
}

void conv_winograd_wgrad_maps(hipStream_t st, const float *x, const float *dy, float *maps, float *dU, float *parts, const ConvShape &cs, int most, bool accumulate) {
    if (cs.N > winograd_wgrad_most_images(cs)) throw KernelError("conv_winograd_wgrad: a plane of 4 GiB or more");
    const unsigned th = (unsigned)(cs.H + 3) / 4, tw = (unsigned)(cs.W + 3) / 4, rows = (unsigned)cs.N * th;
    VerticalArgs v{};
    v.x = x; v.dy = dy;
    v.H = cs.H; v.W = cs.W; v.C = cs.C; v.K = cs.K;
    v.rows = rows; v.th = th; v.px = 4 * tw + 2; v.pd = 4 * tw;
    v.X = maps; v.D = maps + (size_t)6 * rows * v.px * cs.C;
    v.blocks_x = (rows * v.px * (cs.C / 4) + 255) / 256;
    const unsigned blocks_d = (rows * v.pd * (cs.K / 4) + 255) / 256;
    WgradArgs a{};
    a.X = v.X; a.D = v.D;
    a.C = cs.C; a.K = cs.K;
    a.tw = tw; a.T = rows * tw;
    magic_of(tw, a.tw_mul, a.tw_shift);
    a.px = v.px; a.pd = v.pd;
    a.x_plane = rows * v.px * cs.C * 4; a.d_plane = rows * v.pd * cs.K * 4;
    a.chunks = (a.T + CT - 1) / CT;
    a.kb = (cs.K + BLOCK - 1) / BLOCK; a.cb = (cs.C + BLOCK - 1) / BLOCK;
    a.per_range = split_of(a.chunks, most, cs).per_range;
    // One rounding per chunk: beyond these lengths the error grows past the workspace form's (184x28x28 128 -> 128, 35 chunks 1.40e-6, 64 1.79e-6, that form 1.57e-6; 32x30x30 112 -> 96, 8 chunks
    // 0.94, 12 0.99 and 0.96).
    a.per_part = std::max(a.chunks < 64 ? 12u : 8u, std::min(40u, a.chunks / 16));
    const unsigned ranges = (a.chunks + a.per_range - 1) / a.per_range;
    a.items = (unsigned)blocks_of(cs) * ranges;
    const bool whole = ranges == 1 && !accumulate;
    a.out = whole ? dU : parts;
    hipLaunchKernelGGL(wino4_vertical_kernel, dim3(v.blocks_x + blocks_d), dim3(256), 0, st, v);
    hipLaunchKernelGGL(wino4_wgrad_kernel, dim3((a.items + 7) / 8 * 8), dim3(64 * 2 * WAVES), 0, st, a);
    hip_check(hipGetLastError(), "winograd filter gradient launch");
    if (!whole) split_reduce(st, parts, dU, 36ll * cs.K * cs.C, (int)ranges, accumulate);
}

}  // namespace monet
