// Winograd F(4x4, 3x3) in one kernel, its products on the fp16 matrix cores in two pieces per operand (winograd_fused.hip is the same form on
// the fp32 instruction, for reductions that are too short or ragged for this one).
//
// A workgroup (sixteen waves, four per SIMD) owns 32 tiles x 64 output channels for all 36 positions z of the transformed tile.  The
// reduction runs in chunks of 16 channels, double-buffered through LDS:
//   * waves 12-15 load the 6x6 patch of one tile for two neighbouring channels per lane, transform it, split it into pieces and
//     leave them in LDS in the order in which the matrix instruction's lanes read them;
//   * waves 0-11 multiply three positions each (96 accumulators per lane);
//   * the transformed filters come from the workspace, already in pieces and in lane order.
//
// Pieces.  v = h + m with h and m in fp16, each rounded to nearest: 22 bits and the sign of m, one bit less than fp32's 24.  Of a product the terms m*h, h*m and
// h*h are kept; every term is exact in the matrix unit, whose sums are fp32: three roundings per 16 products instead of one per two.  Against 64
// bits that is closer than the fp32 instruction on dense operands of at least 64 reduction channels (normwise, 28x28, ReLU'd input, 64 / 128 / 256 / 512 channels:
// 1.13 / 1.40 / 1.85 / 2.40e-6, the fp32 instruction 1.42 / 1.94 / 2.74 / 3.71e-6; 10 % of the values present 1.29 / 1.59 / 2.09 / 2.78 and 1.44 / 1.94 / 2.69 / 3.74); below, the pieces'
// 2^-23 shows and the fp32 form stays.  It is the coarser one where most products are of zeros, for which the fp32 instruction rounds nothing: 30 % of the (image, channel)
// planes present 1.11 / 1.36 / 1.75 / 2.31 and 0.92 / 1.15 / 1.53 / 2.07, 3 % 0.94 / 0.96 / 1.06 / 1.32 and 0.62 / 0.64 / 0.70 / 0.84.  Measured and not taken: the m*m term and filters transformed
// in 64 bits, 0.86 - 0.99 of the error for 4 - 5 % of the time and 10 us of a call; all four terms in two 16x16x32 instructions, 6 % slower and no closer (it rounds more than once); sums of the small terms apart, which would halve the roundings, need 16 registers of the 8 there are.
//
// Range.  fp16 reaches from 2^-24 to 2^16, so both operands carry powers of two: a filter one per output channel (its largest weight comes
// to lie in [2^13, 2^14)), a tile one that its first chunk with a value other than zero sets (that patch's largest value in [2^5, 2^6); transformed
// values are up to a hundred times as large).  A later chunk with a value above 2^9 sets it anew, and the waves that multiply take their sums along (a maximum and a flag
// per chunk: 1247 and 1261 us on the first layer below, 104.1 and 106.2 on the second).  What is left of an operand below 2^-25 in that scale
// is lost.  Two tests say whether that can show in a result: the 36 sums of a (tile, channel) are all finite (else an operand was an infinity or a
// NaN), and the largest of them is at least 2^20 times what the lost parts can add up to, unless all weights of the channel are zero.  That is, for n channels
// of which the tile has a value other than zero and a largest value a (scaled): n * 2^-25 * (2^14 + 100 a), all signs alike; dense random data lie near 2^21 * sqrt(n), a
// hundred times above the bound at 512 channels.  (One bound for all tiles, 2^11 * sqrt(all channels), was one that signs alike could break by sqrt(channels), and sent most
// launches with less than 0.5 % of the values present to the second pass: a tile with two such values has small sums that nothing is lost from.)  A half item that fails is worked once more on the fp32
// instruction, patches and filters transformed into LDS a chunk at a time.  What that costs with every half item affected: first layer below 1308 -> 3833 us, second
// 109 -> 333 (the fp32 form, which takes both halves from one transform and its filters from the workspace: 2080 and 200).  Ordinary operands stay clear of it: 0.3 % of the
// values present, filters of zeros, channels of very different size.  Those that do not: large inputs that meet weights of almost nothing, or of nothing at all (a
// network with most of its filter planes pruned: sums of zero, which cannot be told from lost ones).
//
// What it measured (us, batch 176 of 112x112, 128 -> 128 channels / 184 of 14x14, 256 -> 256 / 184 of 28x28, 128 -> 128 / 176 of 28x28, 512 -> 512, on one card): fp32
// form 2081 / 196 / 171 / 1924, this one 1282 / 109 / 103 / 1047.  A chunk takes 3.2 us where its matrix instructions alone take 1.3 (measured with the
// other parts left out, at the power limit's clock), and an item another 14 us for its first patch and its outputs.  What the chunk waits for is the vector
// memory path: 147 KB of filters and 74 KB of patches per chunk (at 64 bytes per clock 1.7 us) and the latency of the patches, whose registers
// are free again only when the patch before is split.  Eight waves of which four make the patches and multiply less took the same time to 2 %;
// higher wave priority for the patches nothing.
#include "winograd_f4.hpp"

namespace monet {

namespace {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));

constexpr int FT = FUSED_TILES, FK = FUSED_OUT;
constexpr int CH = 16;                          // reduction channels per chunk
constexpr int NZ = 3, MUL_WAVES = 12;           // positions of a wave that multiplies; four more waves make the patches
constexpr int THREADS = 64 * (MUL_WAVES + 4);
constexpr int V_WORDS = 36 * 2 * FT * CH / 2;   // one V buffer: [z][piece][channels 8g .. 8g+7][tile][4 words of two channels]
constexpr int MROW = 33;                        // row of M[z][tile][.] in LDS
constexpr int LDS_WORDS = 36 * FT * MROW;       // 152 064 bytes; the two V buffers take the first 147 456
constexpr int WROW = 33, WZ = 2 * CH * WROW;    // second pass: row of V[z][channel][tile] and U[z][channel][output channel], one behind the other for each z
static_assert(2 * V_WORDS <= LDS_WORDS && 36 * WZ <= LDS_WORDS, "V buffers must fit");
constexpr int EMPTY = -1000;                    // scale of a tile without a value other than zero
constexpr int TARGET = 6, LIMIT = 9;            // a tile's largest value so far lies in [2^5, 2^6) when its scale is set, and is at most 2^9
constexpr int ZERO_FILTER = -128;               // scale of an output channel without a weight other than zero: its code is 0
constexpr int FILTER_WORKGROUPS = 2 * FUSED_CUS;
constexpr unsigned CHUNK_BYTES = 2048;          // one (position, 32 output channels, chunk) of the filters: two planes of 64 lanes x 16 bytes

// exponent e of |v| < 2^e for the bits of a float that is not negative (subnormals count as 2^-126)
__device__ __forceinline__ int exponent_of(float v) { return (int)(__float_as_uint(v) >> 23) - 126; }
__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }      // -126 <= e <= 127
__device__ __forceinline__ unsigned word_of(f16x2 v) { return __builtin_bit_cast(unsigned, v); }

// (a, b) as pieces
struct Pieces16 { f16x2 h, m; };
__device__ __forceinline__ Pieces16 split16(float a, float b) {
    Pieces16 p;
    p.h = __builtin_convertvector(f2{a, b}, f16x2);
    // the rests, exact in fp32: one instruction each that takes h as it is
    float ra, rb;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(ra) : "v"(word_of(p.h)), "v"(a));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rb) : "v"(word_of(p.h)), "v"(b));
    p.m = __builtin_convertvector(f2{ra, rb}, f16x2);
    return p;
}
// the larger of m, |a| and |b|
__device__ __forceinline__ float max_abs(float m, float a, float b) {
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
    return m;
}

// Transformed filters in pieces:
//   Up[z][out / 32][red / 16][piece][lane][j],  lane = 32 * (red % 16 / 8) + out % 32,  j = red % 8
// `out` runs over the output channels padded to a multiple of 64 (zeros).  The power of two of output channel k, plus 128, lies in the lowest
// bits of the eight m pieces of (z = 0, chunk 0, channels 0 .. 7): a unit of m's last place there, 2^-23 of the value or, of values too small for two pieces, 2^-24
// in the filter's scale.  Code 0 says that the channel has no weight other than zero: its pieces and sums are zeros, and exact.
// One workgroup: 32 output channels x 16 reduction channels; each finds the largest weight of its channels by itself (a few
// microseconds; a launch of its own would cost as much, and the workspace has no room for its result).  LONG: `chunks` times as many reduction channels, for layers
// that give the CUs two workgroups each all the same: the largest weights are read once per workgroup, 19 GB at 2048 -> 2048 channels, 7x7, batch 1, with one chunk each
// (1371 us; 781 so, the fp32 form 1000; 1024 -> 1024, 26x38, batch 11: 544 and 490).
// ADJ: forward pass (out = K, red = C) or input gradient (out = C, red = K, filter turned by 180 degrees).
template <bool ADJ, bool LONG>
__global__ __launch_bounds__(512) void wino4_filter_pieces_kernel(const float *__restrict__ w, unsigned short *__restrict__ Up, int K, int C, int o32, int chunks) {
    __shared__ float part[16][32];
    __shared__ int scale[32];
    const int outc = ADJ ? C : K, red = ADJ ? K : C, nch = red / CH, groups = LONG ? (nch + chunks - 1) / chunks : nch;
    const int ob = blockIdx.x / groups, first = (blockIdx.x - ob * groups) * (LONG ? chunks : 1), tid = threadIdx.x;
    const int len = 9 * red;      // weights of one output channel
    {
        // forward: a row of w; 16 lanes share it.  Input gradient: a column of w seen as [9 * red][C]; 32 lanes read neighbouring columns.
        const int o = ob * 32 + (ADJ ? tid & 31 : tid >> 4), sub = ADJ ? tid >> 5 : tid & 15;
        float mx = 0.0f;
        if (o < outc) {
            const float *p = ADJ ? w + o : w + (int64_t)o * len;
            const int64_t step = ADJ ? C : 1;
#pragma unroll 12
            for (int i = sub; i < len; i += 16) mx = fmaxf(mx, fabsf(p[i * step]));
        }
        part[sub][ADJ ? tid & 31 : tid >> 4] = mx;
    }
    __syncthreads();
    if (tid < 32) {
        float mx = 0.0f;
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, part[i][tid]);
        scale[tid] = mx > 0.0f ? min(14 - exponent_of(mx), 126) : ZERO_FILTER;
    }
    __syncthreads();
    const int ol = tid >> 4, o = ob * 32 + ol, last = LONG ? min(first + chunks, nch) : first + 1;
    for (int ch = first; ch < last; ++ch) {
        const int c = ch * CH + (tid & 15);
        float g[3][3];
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int s = 0; s < 3; ++s)
                g[r][s] = o >= outc ? 0.0f : (ADJ ? w[((int64_t)c * 9 + (2 - r) * 3 + (2 - s)) * C + o] : w[((int64_t)o * 9 + r * 3 + s) * C + c]);
        float t[3][6];      // t[s][a] = (G g)[a][s]
#pragma unroll
        for (int s = 0; s < 3; ++s) f4_g(g[0][s], g[1][s], g[2][s], t[s]);
        const float sc = scale[ol] == ZERO_FILTER ? 1.0f : power_of_two(scale[ol]);
        const unsigned code = (unsigned)(scale[ol] + 128) >> (c & 7);
        const int lane = 32 * ((c & 15) >> 3) + ol;
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            float u[6];
            f4_g(t[0][a], t[1][a], t[2][a], u);
#pragma unroll
            for (int b = 0; b < 6; ++b) {
                const int z = 6 * a + b;
                const Pieces16 p = split16(u[b] * sc, 0.0f);
                unsigned short m = (unsigned short)word_of(p.m);
                if (z == 0 && c < 8) m = (unsigned short)((m & ~1u) | (code & 1u));
                unsigned short *at = Up + ((((int64_t)z * o32 + ob) * nch + ch) * 2 * 64 + lane) * 8 + (c & 7);
                at[0] = (unsigned short)word_of(p.h);
                at[64 * 8] = m;
            }
        }
    }
}

// Byte offsets of the six patch columns and rows of one (tile, channel): element (a, b) of chunk ch sits at x + col[b] + row[a] + 64 * ch.  A
// column or row outside the map, and every one of a tile that does not exist, is ABSENT: added without wrapping, that is
// beyond the descriptor of any tensor, and the load reads zero.
constexpr unsigned ABSENT = BUFFER_ABSENT;
struct Patch { unsigned col[6], row[6]; };
__device__ __forceinline__ unsigned patch_at(const Patch &p, int a, int b) { return __builtin_elementwise_add_sat(p.col[b], p.row[a]); }

// tinfo[tile] = {byte offset of output element (image, 4 * ti, 4 * tj, channel 0), rows | columns << 8 of the 4x4 output tile
// that lie inside the map (0 for a tile beyond the last one), scale, what a channel's largest sum has to reach}
struct TileInfo { unsigned off, extent; int scale; float enough; };

__device__ __forceinline__ Patch patch_of(const FusedGeom &gm, int64_t tb, int pt, int channel, TileInfo *info) {
    Patch p;
#pragma unroll
    for (int a = 0; a < 6; ++a) p.col[a] = p.row[a] = ABSENT;
    const unsigned t = (unsigned)(tb * FT) + pt;      // the host checks that there are fewer than 2^31 tiles
    unsigned off = 0, extent = 0;
    if (t < (unsigned)gm.T) {
        const unsigned tj = t % (unsigned)gm.tw, r = t / (unsigned)gm.tw;
        const unsigned ti = r % (unsigned)gm.th, n = r / (unsigned)gm.th;
        const int h0 = 4 * (int)ti - 1, w0 = 4 * (int)tj - 1;
        const int64_t e = ((int64_t)n * gm.H * gm.W) * gm.red + channel;
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            if ((unsigned)(h0 + a) < (unsigned)gm.H) p.row[a] = (unsigned)((int64_t)(h0 + a) * gm.W * gm.red * 4);
            if ((unsigned)(w0 + a) < (unsigned)gm.W) p.col[a] = (unsigned)((e + (int64_t)(w0 + a) * gm.red) * 4);
        }
        off = (unsigned)((((int64_t)n * gm.H + 4 * ti) * gm.W + 4 * tj) * gm.outc * 4);
        extent = (unsigned)min(4, gm.H - 4 * (int)ti) | ((unsigned)min(4, gm.W - 4 * (int)tj) << 8);
    }
    if (info) {
        info->off = off;
        info->extent = extent;
    }
    return p;
}

// Word of a V buffer, within a position and piece, that starts the eight channels 8 * half .. of a tile.  The tiles of the second half are exchanged in
// fours, so that the eight lanes that write a tile's 16 channels meet in no bank.
__device__ __forceinline__ int v_word(int tile, int half) { return half * (4 * FT) + (tile ^ (half << 2)) * 4; }

// Tiles whose scale a chunk changed, for the waves that multiply it: whether any of the eight tiles of a wave that makes patches, and the power of two by which
// each one's sums so far are smaller in the new scale.  As many as there are V buffers.
struct Growth {
    unsigned any[2][4];
    float by[2][FT];
};

struct Ops {      // what a workgroup reads
    __amdgpu_buffer_rsrc_t x, u;
    int nch, o32, ob;
};

// The reduction loop of a wave that makes the patches of eight tiles: a chunk's patch is transformed, split and left in LDS while the other waves
// multiply the chunk before.  Leaves the scale of the lane's tile and what its sums have to reach.
__device__ __forceinline__ void make_patches(const Ops &op, unsigned *lds, Growth &grown, int lane, int pt, const Patch &patch, TileInfo &info) {
    f2 d[36];
    int scale = EMPTY, present = 0;      // `present`: the lane's chunks with a value other than zero
    float largest = 0.0f;
    float factor = 1.0f, limit = 0.0f;      // a patch with a value beyond `limit` changes the scale
    auto load_row = [&](const Patch &p, int a, int ch) {
#pragma unroll
        for (int b = 0; b < 6; ++b)
            d[a * 6 + b] = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(op.x, (int)patch_at(p, a, b), ch * (CH * 4), 0));
    };
    // Transforms the patch of both channels in place, columns first, and leaves its pieces in V.  A row's registers take the patch of chunk `ch` as
    // soon as its pieces are out: what a load waits for memory passes under the other rows.
    auto transform_store = [&](int buf, int ch) {
        unsigned *V = lds + buf * V_WORDS;
        auto map_row = [&](int i) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float o[6];
                f4_bt(d[i][e], d[i + 1][e], d[i + 2][e], d[i + 3][e], d[i + 4][e], d[i + 5][e], o);
#pragma unroll
                for (int k = 0; k < 6; ++k) d[i + k][e] = o[k];
            }
        };
        float mx = 0.0f;              // the two maps make it a hundred times as large at most
#pragma unroll
        for (int i = 0; i < 36; ++i) mx = max_abs(mx, d[i].x, d[i].y);
        present += mx > 0.0f;
        largest = fmaxf(largest, mx);
        unsigned any_grown = 0;
        if (__any(mx > limit)) {      // uniform over the wave: a tile's first value other than zero, or one that its scale does not hold
            mx = fmaxf(mx, __shfl_xor(mx, 1));      // the eight lanes of a tile
            mx = fmaxf(mx, __shfl_xor(mx, 2));
            mx = fmaxf(mx, __shfl_xor(mx, 4));
            float less = 1.0f;      // what the tile's sums so far are multiplied by
            if (mx > limit) {
                const int now = min(TARGET - exponent_of(mx), 124);
                // (sums that shrink by more than 2^126 are far below the new ones' last place in any case)
                if (scale != EMPTY) less = power_of_two(max(now - scale, -126));
                scale = now;
                factor = power_of_two(scale);
                limit = power_of_two(min(LIMIT - scale, 127));
            }
            any_grown = __any(less != 1.0f);
            if ((lane & 7) == 0) grown.by[buf][pt] = less;
        }
        if (lane == 0) grown.any[buf][pt >> 3] = any_grown;
        // columns, and the power of two with them: f4_bt with its coefficients times `factor` and three products more
        const float s4 = 4.0f * factor, s5 = -5.0f * factor;
#pragma unroll
        for (int b = 0; b < 6; ++b)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float v0 = d[b][e], v1 = d[6 + b][e], v2 = d[12 + b][e], v3 = d[18 + b][e];
                const float f3 = factor * v3, f4 = factor * d[24 + b][e], f5 = factor * d[30 + b][e];
                const float p = __builtin_fmaf(-s4, v2, f4), q = __builtin_fmaf(-s4, v1, f3), r = __builtin_fmaf(-factor, v2, f4), t = __builtin_fmaf(-factor, v1, f3);
                d[b][e] = __builtin_fmaf(s4, v0, __builtin_fmaf(s5, v2, f4));
                d[6 + b][e] = p + q;
                d[12 + b][e] = p - q;
                d[18 + b][e] = __builtin_fmaf(2.0f, t, r);
                d[24 + b][e] = __builtin_fmaf(-2.0f, t, r);
                d[30 + b][e] = __builtin_fmaf(s4, v1, __builtin_fmaf(s5, v3, f5));
            }
        unsigned *at = V + v_word(pt, (lane & 7) >> 2) + (lane & 3);
        Patch p = patch;
#pragma unroll
        for (int a = 0; a < 6; ++a) asm volatile("" : "+v"(p.row[a]));      // the 36 sums are made here: kept from chunk to chunk they would be spilled
        map_row(0);
#pragma unroll
        for (int a = 0; a < 6; ++a) {
            if (a < 5) map_row(6 * a + 6);
#pragma unroll
            for (int z = 6 * a; z < 6 * a + 6; ++z) {
                const Pieces16 q = split16(d[z].x, d[z].y);
                at[z * (16 * FT)] = word_of(q.h);
                at[z * (16 * FT) + 8 * FT] = word_of(q.m);
            }
            __builtin_amdgcn_sched_barrier(0);
            load_row(p, a, ch);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

#pragma unroll
    for (int a = 0; a < 6; ++a) load_row(patch, a, 0);
    transform_store(0, op.nch > 1 ? 1 : 0);
    __syncthreads();
    for (int ch = 0; ch < op.nch; ++ch) {
        // V[next] was last read before the barrier that ended chunk ch - 1
        if (ch + 1 < op.nch) transform_store((ch + 1) & 1, ch + 2 < op.nch ? ch + 2 : ch + 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 1; i < 8; i *= 2) {
        present += __shfl_xor(present, i);
        largest = fmaxf(largest, __shfl_xor(largest, i));
    }
    if ((lane & 7) == 0) {      // read behind the caller's next barrier
        info.scale = scale;
        info.enough = (float)(2 * present) * 0x1p-5f * (0x1p14f + 100.0f * (largest * factor));      // (an infinity fails the other test)
    }
}

// The reduction loop of a wave that multiplies: NZ positions from z0 on.  HALF: only the block of 32 output channels ob (acc[.][0]), else
// ob and ob + 1.
template <bool HALF>
__device__ __forceinline__ void multiply(const Ops &op, const unsigned *lds, const Growth &grown, int z0, int lane, floatx16 (&acc)[NZ][2]) {
    const int nch = op.nch;
#pragma unroll
    for (int zi = 0; zi < NZ; ++zi)
#pragma unroll
        for (int h = 0; h < (HALF ? 1 : 2); ++h)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[zi][h][i] = 0.0f;
    // Filters of one position and one block of 32 output channels at a time, RING of them ahead, each into the registers its predecessor has just left.
    constexpr int BLOCKS = HALF ? 1 : 2, UNITS = NZ * BLOCKS, RING = HALF ? 3 : 2;
    static_assert(UNITS % RING == 0, "a unit keeps its registers from chunk to chunk");
    struct Piece { f16x8 h, m; };
    Piece bq[RING];
    const unsigned lane16 = (unsigned)lane * 16u;
    const unsigned hbytes = (unsigned)nch * CHUNK_BYTES, zbytes = (unsigned)op.o32 * hbytes;      // the host checks the workspace's size
    const unsigned ubase = (unsigned)z0 * zbytes + (unsigned)op.ob * hbytes;
    auto load_b = [&](int u, int ch) {
        const unsigned so = ubase + (u / BLOCKS) * zbytes + (u % BLOCKS) * hbytes + (unsigned)ch * CHUNK_BYTES;
        bq[u % RING].h = __builtin_bit_cast(f16x8, buffer_load4(op.u, lane16, so));
        bq[u % RING].m = __builtin_bit_cast(f16x8, buffer_load4(op.u, lane16 + 1024u, so));
    };
    auto load_a = [&](const unsigned *V, int zi) {
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const unsigned *at = V + (z0 + zi) * (16 * FT) + v_word(lane & 31, lane >> 5);
        return Piece{__builtin_bit_cast(f16x8, *(const u4 *)at), __builtin_bit_cast(f16x8, *(const u4 *)(at + 8 * FT))};
    };
#pragma unroll
    for (int u = 0; u < RING; ++u) load_b(u, 0);
    __syncthreads();
    for (int ch = 0; ch < nch; ++ch) {
        const unsigned *V = lds + (ch & 1) * V_WORDS;
        const unsigned any = grown.any[ch & 1][lane & 3];
        // tiles whose scale this chunk changed: rows 8 * wave + 4 * (lane / 32) .. + 3 of the products are registers 4 * wave .. + 3
        if (const unsigned long long changed = __ballot(any != 0)) {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if ((changed >> v) & 1u) {
                    const float4 by = *(const float4 *)&grown.by[ch & 1][8 * v + 4 * (lane >> 5)];
#pragma unroll
                    for (int zi = 0; zi < NZ; ++zi)
#pragma unroll
                        for (int h = 0; h < BLOCKS; ++h) {
                            acc[zi][h][4 * v] *= by.x;
                            acc[zi][h][4 * v + 1] *= by.y;
                            acc[zi][h][4 * v + 2] *= by.z;
                            acc[zi][h][4 * v + 3] *= by.w;
                        }
                }
        }
        const int nx = ch + 1 < nch ? ch + 1 : ch;      // the last chunk requests filters that exist (its own) instead of branching; nothing reads them
#pragma unroll
        for (int zi = 0; zi < NZ; ++zi) {
            const Piece a = load_a(V, zi);
#pragma unroll
            for (int h = 0; h < BLOCKS; ++h) {
                const int u = zi * BLOCKS + h;
                const Piece &f = bq[u % RING];
                acc[zi][h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.m, f.h, acc[zi][h], 0, 0, 0);
                acc[zi][h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h, f.m, acc[zi][h], 0, 0, 0);
                acc[zi][h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h, f.h, acc[zi][h], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (u + RING < UNITS) load_b(u + RING, ch);
                else load_b(u + RING - UNITS, nx);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();      // V[next] complete; every wave is done reading V[cur]
    }
}

// ADJ: input gradient.  EPI: 0 plain store, 1 added to what is there, 2 followed by the BatchNorm multiply-add.
template <bool ADJ, int EPI>
__global__ __launch_bounds__(THREADS) void wino4_pieces_kernel(const float *__restrict__ x, const float *__restrict__ Up, const float *__restrict__ w, float *y,
                                                           FusedGeom gm, BnAffine bn) {
    __shared__ __attribute__((aligned(16))) unsigned lds[LDS_WORDS];
    __shared__ TileInfo tinfo[FT];
    __shared__ __attribute__((aligned(16))) Growth grown;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // the same for the whole wave: kept in a scalar register
    FusedItem it;
    if (!fused_item(gm, it)) return;
    const unsigned in_bytes = (unsigned)((int64_t)gm.N * gm.H * gm.W * gm.red * 4), out_bytes = (unsigned)((int64_t)gm.N * gm.H * gm.W * gm.outc * 4);
    const Ops op{buffer_of(x, in_bytes), buffer_of(Up), gm.nch, gm.kblocks * 2, it.ob};

    floatx16 acc[NZ][2];
    const bool makes = wave >= MUL_WAVES;
    const int z0 = NZ * wave;
    if (!makes) {
        if (it.nh == 2) multiply<false>(op, lds, grown, z0, lane, acc);
        else multiply<true>(op, lds, grown, z0, lane, acc);
    } else {
        // lane = 8 * (tile % 8) + channel / 2: eight neighbouring lanes read 64 bytes
        const int pt = (wave - MUL_WAVES) * 8 + (lane >> 3);
        const bool first = (lane & 7) == 0;
        const Patch patch = patch_of(gm, it.tb, pt, 2 * (lane & 7), first ? &tinfo[pt] : nullptr);
        make_patches(op, lds, grown, lane, pt, patch, tinfo[pt]);
    }

    // ---- output transform, 32 channels at a time: thread = (channel ok_ of the half, tile tl).  Output element
    // (a, b) of a tile sits at byte y + [(a * W + b) * outc * 4] + the thread's own 32-bit offset (tile + channel).
    const int ok_ = tid & 31, tl = tid >> 5;
    const unsigned obytes = (unsigned)gm.outc * 4, orow = (unsigned)gm.W * obytes;
    const __amdgpu_buffer_rsrc_t ry = buffer_of(y, out_bytes);
    const bool two = EPI == 2 && bn.relu && bn.relu_out != nullptr;           // ReLU output beside the BatchNorm's
    const __amdgpu_buffer_rsrc_t ry2 = buffer_of(two ? bn.relu_out : y, out_bytes);
    float *M = (float *)lds;

    auto stage = [&](auto half) {
#pragma unroll
        for (int zi = 0; zi < NZ; ++zi)
            if (!makes) {
#pragma unroll
                for (int i = 0; i < 16; ++i) M[((z0 + zi) * FT + 8 * (i >> 2) + 4 * g + (i & 3)) * MROW + l32] = acc[zi][decltype(half)::value][i];
            }
    };
    // the 16 outputs of (tile tl, channel ok_) before their scale, and the largest of the 36 sums
    auto outputs = [&](float (&o)[4][4]) {
        const float *mp = M + tl * MROW + ok_;
        float s[6][4], mx = 0.0f;      // s[b][a] = (A^T m)[a][b]
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            float m[6];
#pragma unroll
            for (int a = 0; a < 6; ++a) m[a] = mp[(6 * a + b) * (FT * MROW)];
#pragma unroll
            for (int a = 0; a < 6; a += 2) mx = max_abs(mx, m[a], m[a + 1]);
            f4_at(m[0], m[1], m[2], m[3], m[4], m[5], s[b]);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a) f4_at(s[0][a], s[1][a], s[2][a], s[3][a], s[4][a], s[5][a], o[a]);
        return mx;
    };
    auto emit = [&](int kout, const float (&o)[4][4], int scale, float bn_a, float bn_b) {
        const unsigned extent = kout < gm.outc ? tinfo[tl].extent : 0u, voff = tinfo[tl].off + (unsigned)kout * 4u;
        const int nr = (int)(extent & 0xff), nc = (int)(extent >> 8);
        unsigned *mask32 = EPI == 2 && bn.relu ? (unsigned *)bn.mask : nullptr;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const unsigned so = a * orow + b * obytes;
                const bool here = a < nr && b < nc;
                const unsigned at = here ? voff : ABSENT;      // beyond the descriptor: loads zero, stores nothing
                float v = __builtin_ldexpf(o[a][b], -scale);
                if (EPI == 1) v += buffer_load(ry, at, so);
                if (EPI == 2) v = bn_affine(v, bn_a, bn_b);
                if (EPI == 2 && mask32) {      // uniform over the wave
                    // the sign code of the ReLU: the 32 lanes of a half wave hold 32 consecutive channels of one position, half
                    // a word of the code; its first lane writes it
                    const bool pass = here && (bn.relu == 2 ? (v > 0.0f && v < 6.0f) : v > 0.0f);
                    const unsigned long long word = __ballot(pass);
                    const unsigned half = lane < 32 ? (unsigned)word : (unsigned)(word >> 32);
                    if ((lane & 31) == 0 && here) mask32[(voff + so) >> 7] = half;
                }
                if (EPI == 2 && bn.relu) {
                    const float rv = relu_clamp(v, bn.relu);
                    if (two) buffer_store(ry2, at, so, rv);
                    else v = rv;
                }
                buffer_store(ry, at, so, v);
            }
        }
    };
    auto coefficients = [&](int kout, float &a, float &b) {
        a = 1.0f;
        b = 0.0f;
        if (EPI == 2 && kout < gm.outc) bn_affine_coeffs(bn.gamma, bn.beta, bn.stats, gm.outc, kout, a, b);
    };

    unsigned again = 0;      // halves whose pieces do not hold their numbers
    auto finish = [&](auto half) {
        constexpr int h = decltype(half)::value;
        if (h >= it.nh || (it.ob + h) * 32 >= gm.outc) return;      // uniform over the workgroup
        stage(half);
        // the power of two of this thread's filter
        const int kout = (it.ob + h) * 32 + ok_;
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        const u4 low = __builtin_bit_cast(u4, buffer_load4(op.u, (unsigned)ok_ * 16u + 1024u, (unsigned)(it.ob + h) * gm.nch * CHUNK_BYTES));
        int fscale = -128;
#pragma unroll
        for (int i = 0; i < 4; ++i) fscale += (int)(((low[i] & 1u) << (2 * i)) | (((low[i] >> 16) & 1u) << (2 * i + 1)));
        float bn_a, bn_b;
        coefficients(kout, bn_a, bn_b);
        __syncthreads();
        float o[4][4], sum = 0.0f;
        const float mx = outputs(o);
#pragma unroll
        for (int a = 0; a < 4; ++a) sum += (o[a][0] + o[a][1]) + (o[a][2] + o[a][3]);
        const int scale = tinfo[tl].scale;
        const bool exists = kout < gm.outc && tinfo[tl].extent;
        const bool bad = exists && (!(fabsf(sum) < __builtin_inff()) || (scale != EMPTY && fscale != ZERO_FILTER && mx < tinfo[tl].enough));
        if (__syncthreads_or(bad)) again |= 1u << h;      // the barrier also: everyone has read this half
        else emit(kout, o, (scale == EMPTY ? 0 : scale) + fscale, bn_a, bn_b);
    };
    finish(std::integral_constant<int, 0>{});
    finish(std::integral_constant<int, 1>{});
    if (!again) return;

    // ---- on the fp32 instruction, one half at a time.  Threads 0 .. 511 transform the patch of one (tile, channel) of a chunk each, the others one filter; both
    // load the next chunk's while twelve waves multiply.
    const int t512 = tid & (FT * CH - 1);
    const int pt = t512 >> 4, pc = t512 & 15;                                          // patches: 16 lanes read 64 bytes of a pixel
    const int uo = ADJ ? t512 & 31 : t512 >> 4, uc = ADJ ? t512 >> 5 : t512 & 15;      // filters: neighbouring lanes read neighbouring weights
    const unsigned w_ch = ADJ ? 9u * gm.outc * 4u : 4u, w_tap = (ADJ ? gm.outc : gm.red) * 4u;      // bytes from channel to channel and from tap to tap
    const __amdgpu_buffer_rsrc_t rw = buffer_of(w, 9u * gm.outc * gm.red * 4u);
    const int put = wave >= FT * CH / 64 ? (CH + uc) * WROW + uo : pc * WROW + pt;
    auto reduce = [&](auto role, int ob) {      // the chunks of block ob of 32 output channels; every wave passes the same barriers
        constexpr bool FILTERS = decltype(role)::value;
        Patch patch;
        unsigned w_at = 0;
        if constexpr (!FILTERS) patch = patch_of(gm, it.tb, pt, pc, nullptr);
        else if (ob * 32 + uo < gm.outc) w_at = (unsigned)(ob * 32 + uo) * (ADJ ? 4u : 9u * gm.red * 4u) + uc * w_ch;
        else w_at = ABSENT;
        float d[FILTERS ? 9 : 36];
        auto load = [&](int ch) {
            if constexpr (!FILTERS) {
#pragma unroll
                for (int a = 0; a < 6; ++a) asm volatile("" : "+v"(patch.row[a]));      // the 36 sums are made here, as above
#pragma unroll
                for (int a = 0; a < 6; ++a)
#pragma unroll
                    for (int b = 0; b < 6; ++b) d[a * 6 + b] = buffer_load(op.x, patch_at(patch, a, b), ch * (CH * 4));
            } else {
#pragma unroll
                for (int i = 0; i < 9; ++i) d[i] = buffer_load(rw, w_at, ch * CH * w_ch + (ADJ ? 8 - i : i) * w_tap);
            }
        };
#pragma unroll
        for (int zi = 0; zi < NZ; ++zi)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[zi][0][i] = 0.0f;
        load(0);
        for (int ch = 0; ch < gm.nch; ++ch) {
            int at = put;
            asm volatile("" : "+v"(at));      // not an address per position kept over the loop
            __syncthreads();      // the products of the chunk before, or the outputs of the half before, have been read
            if constexpr (!FILTERS) {
                float o[6];
#pragma unroll
                for (int b = 0; b < 6; ++b) {
                    f4_bt(d[b], d[6 + b], d[12 + b], d[18 + b], d[24 + b], d[30 + b], o);
#pragma unroll
                    for (int a = 0; a < 6; ++a) d[6 * a + b] = o[a];
                }
#pragma unroll
                for (int a = 0; a < 6; ++a) {
                    f4_bt(d[6 * a], d[6 * a + 1], d[6 * a + 2], d[6 * a + 3], d[6 * a + 4], d[6 * a + 5], o);
#pragma unroll
                    for (int b = 0; b < 6; ++b) M[at + (6 * a + b) * WZ] = o[b];
                }
            } else {
                float t[3][6];      // t[s][a] = (G g)[a][s]
#pragma unroll
                for (int s = 0; s < 3; ++s) f4_g(d[s], d[3 + s], d[6 + s], t[s]);
#pragma unroll
                for (int a = 0; a < 6; ++a) {
                    float u[6];
                    f4_g(t[0][a], t[1][a], t[2][a], u);
#pragma unroll
                    for (int b = 0; b < 6; ++b) M[at + (6 * a + b) * WZ] = u[b];
                }
            }
            load(ch + 1 < gm.nch ? ch + 1 : ch);      // the last chunk loads its own again instead of branching
            __syncthreads();
            if (makes) continue;
#pragma unroll
            for (int zi = 0; zi < NZ; ++zi) {
#pragma unroll
                for (int j = 0; j < CH / 2; ++j) {
                    const float *from = M + (z0 + zi) * WZ + (2 * j + g) * WROW + l32;
                    acc[zi][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(from[0], from[CH * WROW], acc[zi][0], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    for (int h = 0; h < 2; ++h) {
        if (!((again >> h) & 1u)) continue;
        const int ob = it.ob + h;
        if (wave < FT * CH / 64) reduce(std::false_type{}, ob);
        else reduce(std::true_type{}, ob);
        __syncthreads();
        stage(std::integral_constant<int, 0>{});
        __syncthreads();
        const int kout = ob * 32 + ok_;
        float bn_a, bn_b;
        coefficients(kout, bn_a, bn_b);
        float o[4][4];
        outputs(o);
        emit(kout, o, 0, bn_a, bn_b);
    }
}

}  // namespace

bool winograd_pieces_applies(const ConvShape &cs, bool adjoint) {
    const int red = adjoint ? cs.K : cs.C, out = adjoint ? cs.C : cs.K;
    return red % CH == 0 && red >= 64 && (int64_t)36 * ((out + FK - 1) / FK * FK) * red * 4 < ((int64_t)1 << 32);
}

void conv_winograd_pieces(hipStream_t st, const float *in, const float *w, float *out, const ConvShape &cs, bool adjoint, bool accumulate, float *ws,
                          const BnAffine &bn) {
    FusedGeom gm;
    const int64_t grid = fused_geometry(gm, cs, adjoint, CH);
    const int o32 = gm.kblocks * 2;
    const int chunks = std::max(1, (int)((int64_t)o32 * gm.nch / FILTER_WORKGROUPS));
    const dim3 fg((unsigned)(o32 * ((gm.nch + chunks - 1) / chunks))), fwg(512), wg(THREADS), gd((unsigned)grid);
    if (adjoint) {
        hipLaunchKernelGGL((chunks > 1 ? wino4_filter_pieces_kernel<true, true> : wino4_filter_pieces_kernel<true, false>), fg, fwg, 0, st, w, (unsigned short *)ws, cs.K, cs.C, o32, chunks);
        if (accumulate) hipLaunchKernelGGL((wino4_pieces_kernel<true, 1>), gd, wg, 0, st, in, (const float *)ws, w, out, gm, bn);
        else hipLaunchKernelGGL((wino4_pieces_kernel<true, 0>), gd, wg, 0, st, in, (const float *)ws, w, out, gm, bn);
    } else {
        hipLaunchKernelGGL((chunks > 1 ? wino4_filter_pieces_kernel<false, true> : wino4_filter_pieces_kernel<false, false>), fg, fwg, 0, st, w, (unsigned short *)ws, cs.K, cs.C, o32, chunks);
        if (bn.gamma) hipLaunchKernelGGL((wino4_pieces_kernel<false, 2>), gd, wg, 0, st, in, (const float *)ws, w, out, gm, bn);
        else if (accumulate) hipLaunchKernelGGL((wino4_pieces_kernel<false, 1>), gd, wg, 0, st, in, (const float *)ws, w, out, gm, bn);
        else hipLaunchKernelGGL((wino4_pieces_kernel<false, 0>), gd, wg, 0, st, in, (const float *)ws, w, out, gm, bn);
    }
    hip_check(hipGetLastError(), "winograd pieces launch");
}

}  // namespace monet
