// Internal declarations shared by the HIP sources of libhgf (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/hgf.h"
#include "hgf_once.h"

namespace hgf {

constexpr int kTileRows = 32;        // a packed tile covers 32 rows ...
constexpr int kTileCols = 128;       // ... by 128 columns of 2-bit codes
constexpr int kTileBytes = 1024;
constexpr int kMaxGroup = 4;         // layers reading the same activations launched together

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));

// ---- branch-free guarded loads ---------------------------------------------------------
// A load inside a conditional makes the compiler wait for every outstanding load at the
// join, which serialises the memory pipeline.  These helpers go through a buffer
// descriptor instead: an offset at or beyond the descriptor's size reads as zero, so a
// guard becomes a select on the offset and the loads stay back to back.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr unsigned kOob = 0xFFFFFF00u;         // beyond any descriptor in this library
__device__ inline rsrc_t make_rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
__device__ inline v4u buf_load16(rsrc_t r, unsigned off, bool ok = true)
{
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(ok ? off : kOob), 0, 0));
}
__device__ inline v4u buf_load16_stream(rsrc_t r, unsigned off)   // read-once data: non-temporal
{
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 2));
}
__device__ inline unsigned buf_load4(rsrc_t r, unsigned off, bool ok = true)
{
    return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)(ok ? off : kOob), 0, 0);
}
__device__ inline unsigned short buf_load2(rsrc_t r, unsigned off, bool ok = true)
{
    return (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)(ok ? off : kOob), 0, 0);
}
__device__ inline _Float16 half_bits(unsigned short u) { return __builtin_bit_cast(_Float16, u); }
// Eight consecutive fp16 of a row-major matrix behind `r`, starting at element `elem`;
// elements at column >= cols_left read as zero.  VEC: the eight are 16-byte aligned and
// all in range or all out.
template <bool VEC>
__device__ inline v8h buf_load8h(rsrc_t r, unsigned elem, int cols_left, bool ok)
{
    if (VEC) return __builtin_bit_cast(v8h, buf_load16(r, elem * 2u, ok && cols_left > 0));
    v8h v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = half_bits(buf_load2(r, (elem + e) * 2u, ok && e < cols_left));
    return v;
}

// Same, visible to every compute unit of the device: partial results that one workgroup
// writes and another reads within a single launch bypass the per-XCD L2 (sc1).
__device__ inline unsigned buf_load4_agent(rsrc_t r, unsigned off, bool ok = true)
{
    return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, (int)(ok ? off : kOob), 0, 16);
}
__device__ inline void buf_store16_agent(rsrc_t r, unsigned off, v4f v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, (int)off, 0, 16);
}

// ---- arithmetic shared by the kernels ---------------------------------------------------
// Four bytes of 2-bit codes (T+1) -> the four int8 operand registers of one MFMA.
__device__ inline v4i widen_codes(uint32_t w)
{
    v4i a;
    a[0] = (int)(w & 0x03030303u);
    a[1] = (int)((w >> 2) & 0x03030303u);
    a[2] = (int)((w >> 4) & 0x03030303u);
    a[3] = (int)((w >> 6) & 0x03030303u);
    return a;
}
__device__ inline float silu(float h) { return h / (1.0f + expf(-h)); }
// The int8 operands of five MFMAs from 16 bytes of base-3 codes, one digit of every byte each.  Bytes
// are taken apart in pairs of 16 bits, whose products with these multipliers floor to the quotients by
// 3, 9, 27 and 81 for every byte up to 242; digit i is quotient i - 3 quotient i+1, four at a time
// (nothing is borrowed between bytes).  1.4 vector instructions per weight.
typedef unsigned short v2us __attribute__((ext_vector_type(2)));
__device__ inline void base3_digits(v4u bytes, v4i (&digit)[5])
{
    auto halves = [](unsigned v) { return __builtin_bit_cast(v2us, v); };
    auto word = [](v2us v) { return __builtin_bit_cast(unsigned, v); };
    auto triple = [](unsigned v) {                  // (as a multiplication it would run at a quarter of the rate)
        unsigned t;
        asm("v_lshl_add_u32 %0, %1, 1, %1" : "=v"(t) : "v"(v));
        return t;
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned b = bytes[i];
        const v2us e = halves(b & 0x00ff00ffu), o = halves((b >> 8) & 0x00ff00ffu);
        auto quotient = [&](unsigned short mul, int shift) {
            return word((e * mul) >> (unsigned short)shift) | ((word(o * mul) >> (shift - 8)) & 0x7f007f00u);
        };
        const unsigned short m3 = 85;
        const unsigned q1 = __builtin_amdgcn_perm(word(o * m3 + m3), word(e * m3 + m3), 0x07030501u);
        const unsigned q2 = quotient(57, 9), q3 = quotient(19, 9), q4 = word((e * (unsigned short)203) >> (unsigned short)14) |
                                                                        word((o * (unsigned short)203) >> (unsigned short)14) << 8;
        digit[0][i] = (int)(b - triple(q1));
        digit[1][i] = (int)(q1 - triple(q2));
        digit[2][i] = (int)(q2 - triple(q3));
        digit[3][i] = (int)(q3 - triple(q4));
        digit[4][i] = (int)q4;
    }
}

// fp16 of the exact product, rounded once.  (The compiler joins a product and its conversion into this instruction
// in some places and not in others; kernels that have to give the same bits say it.)
__device__ inline _Float16 product_half(float a, float b)
{
    uint32_t r;
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(r) : "v"(a), "v"(b));
    return half_bits((unsigned short)r);
}
// fp32 product of fp16 half H (0: low, 1: high) of `packed` and the fp32 `scale`, rounded once
// (an FMA whose addend is zero), without a conversion instruction of its own
template <int H>
__device__ inline float scaled_half(uint32_t packed, float scale)
{
    float r;
    if (H == 0) asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(packed), "v"(scale));
    else asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(packed), "v"(scale));
    return r;
}
// Eight int8 codes round(x * inv), half to even, of the fp16 in x, by adding 1.5 * 2^23 to the products: a code is
// its sum's low byte.  |x| is at most the token's maximum, so there is nothing to clip, unless the token is `odd`
// (it holds an infinity or what is not a number): the median makes -127 of what is not a number, as clipping by
// minimum and maximum does.  The codes are added to `sum`.
__device__ inline uint2 eight_codes(v4u x, float inv, bool odd, int &sum)
{
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = e & 1 ? scaled_half<1>(x[e >> 1], inv) : scaled_half<0>(x[e >> 1], inv);
    if (odd) {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = __builtin_amdgcn_fmed3f(f[e], -127.0f, 127.0f);
    }
    uint32_t q[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = __builtin_bit_cast(uint32_t, f[4 * h + e] + 12582912.0f);
        q[h] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u), __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), 0x05040100u);
        sum = __builtin_amdgcn_sdot4((int)q[h], 0x01010101, sum, false);
    }
    return make_uint2(q[0], q[1]);
}
// Running maximum of fp16 magnitudes, two at a time (they order like their bits); kOddBits and above: an infinity or
// what is not a number.
constexpr uint32_t kOddBits = 0x7c00u;
__device__ inline uint32_t max_magnitudes(v4u x, uint32_t mx)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) asm("v_pk_max_u16 %0, %1, %2" : "=v"(mx) : "v"(mx), "v"(x[d] & 0x7fff7fffu));
    return mx;
}
__device__ inline bool odd_magnitudes(uint32_t mx) { return (mx & 0xffffu) >= kOddBits || mx >= kOddBits << 16; }
__device__ inline float larger_magnitude(uint32_t mx)
{
    return fmaxf((float)half_bits((unsigned short)mx), (float)half_bits((unsigned short)(mx >> 16)));
}
// The same where some are odd: what is not a number counts for nothing.
__device__ inline float max_odd(v4u x, float amax)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf((float)half_bits((unsigned short)(x[e >> 1] >> (16 * (e & 1))))));
    return amax;
}
// Wave-wide reductions with the result in every lane.  The lanes of a row of 16 exchange
// through the data-parallel-primitive modifiers of the vector ALU (xor 1, xor 2, mirror within
// 8, mirror within 16: four dependent instructions); the four rows are then combined from
// scalar reads of one lane each.  (A shuffle through LDS per butterfly step costs an LDS
// round trip each: six in a row were half a microsecond of the decode chain.)
template <int CTRL>
__device__ inline int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
__device__ inline float wave_max(float v)
{
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0xB1>(__builtin_bit_cast(int, v))));    // quad_perm [1,0,3,2]
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0x4E>(__builtin_bit_cast(int, v))));    // quad_perm [2,3,0,1]
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0x141>(__builtin_bit_cast(int, v))));   // row_half_mirror
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0x140>(__builtin_bit_cast(int, v))));   // row_mirror
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}
__device__ inline int wave_sum(int v)
{
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
           __builtin_amdgcn_readlane(v, 48);
}
// Sec. 2.2.1 activation quantiser: round half to even, clip to [-127, 127].
__device__ inline int quant1(float x, float inv)
{
    float q = rintf(x * inv);
    q = fminf(fmaxf(q, -127.0f), 127.0f);
    return (int)q;
}

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// ---- workspace layout -------------------------------------------------------------
// [ flags | exchange buffers of the single-launch path | x_q | s_x | rowsum | h16 |
//   weight-quantiser sums | spare ]   (hgf_workspace_init zeroes the flags and fills the exchange
//   buffers with the sentinel pattern)
constexpr int kNumFlags = 64;                              // int32 words: launch counter, arrival count, sticky error
constexpr size_t kZeroBytes = size_t(kNumFlags) * 4;
constexpr int kWsumBlocks = 1024;                          // fp64 partial sums of |W|

struct Workspace {
    int32_t *flags;      // zero region: [0] correction workgroups done, [1] decode workgroups done,
                         // [2] sticky: a bounded wait ran out
    unsigned char *mail; // two exchange buffers of kMailBytes, sentinel-filled between launches
    unsigned char *xchg; // two sets of kStackSetBytes for the whole-stack launch and the task queue, likewise
    int8_t *xq;
    float *s_x;
    int32_t *rowsum;
    _Float16 *h16;       // kMaxGroup x [M, h_stride] SiLU(A x), zero padded (one per layer of a group)
    size_t h16_each;     // bytes per layer
    double *wsum;        // [kWsumBlocks]
    unsigned char *spare; // direct path: slices of A x; further quantisations where layers have LayerNorms of their own
    size_t spare_bytes;
    size_t bytes;        // total bytes needed
};

// Carves `base` for a call of the given sizes (base may be null: sizes only).  `groups`: layers
// that may share one launch (kMaxGroup for layer lists, 1 for a single layer); `with_stack`:
// include the exchange regions of the whole-stack launch (else `xchg` is null).
Workspace carve_workspace(void *base, int M, int d_in, int d_out, int rank, int groups = kMaxGroup,
                          bool with_stack = true);

__host__ __device__ inline int h_rank_tiles(int rank)   // rank tiles of 16, rounded to a power of two (1, 2, 4, 8)
{
    int t = (rank + 15) / 16, p = 1;
    while (p < t) p *= 2;
    return p;
}
__host__ __device__ inline int h_stride(int rank)       // row stride of h16 in elements (multiple of 32)
{
    int s = 16 * h_rank_tiles(rank);
    return s < 32 ? 32 : s;
}

// ---- grouped launches: up to kMaxGroup layers that read the same activations ----------

struct ProLayer {
    const _Float16 *A;   // [rank, K]
    _Float16 *h16;       // [M, hstride] SiLU(A x): whole tiles of 16 ranks are written
    float *hpart;        // S > 1 instead: [S, M, hstride] partial sums of A x
    int rank, hstride;
};
// One quantisation of the tokens.  xq: groups of 32 tokens (the last one smaller), 32 Kp bytes apart,
// each [Kp / 16][tokens of the group][16]; one set per layer where LayerNorms differ.  base3: Kp / 80
// units, each [digit 0 .. 4][tokens][16 bytes]: byte g of digit i is column 80 unit + 5 g + i.
struct ProTokens {
    int8_t *xq;
    float *s_x;
    int32_t *rowsum;
    const float *gamma, *beta;   // LayerNorm in front (gamma null: none; beta null: zero)
    float eps;
};
struct ProParams {
    const _Float16 *x;
    float *amax_zero;    // nullable: [M] floats the quantising workgroups set to zero (a later kernel's atomic max)
    int M, K, Kp, G, NQ; // layers; quantisations
    int S;               // slices of d_in
    int base3;           // x_q as the base-3 kernel reads it (M <= 32)
    int by_rows;         // as the prefill kernel reads them: x_q [M][Kp], SiLU(A x) padded with zeros to hstride
    int token_tiles;
    ProLayer L[kMaxGroup];
    ProTokens Q[kMaxGroup];
    int job_start[kMaxGroup + 1];
};

struct DecLayer {
    const v4u *packed;
    const float *s_w;
    const _Float16 *B;
    const _Float16 *alpha;
    const _Float16 *h16;     // [M, hstride] fp16 SiLU(A x)
    const float *hpart;      // or its slices, as in ProLayer
    const int8_t *xq;        // as in ProTokens
    const float *s_x;
    const int32_t *rowsum;
    _Float16 *y;
    int32_t *acc_debug;
    int N, RBn, rank, hstride;
    int b_aligned;           // B starts at a multiple of 16 bytes
};
struct DecodeParams {
    int M, Kp, KT, G;
    int hsteps;              // 16-rank steps of the widest layer
    int S;                   // slices of A x
    int base3;               // packed: base-3 rows
    DecLayer L[kMaxGroup];
    int wg_start[kMaxGroup + 1];   // running sum of the layers' row units
    // SwiGLU pair (G == 2, both layers of one shape): layer 0 (gate) and layer 1 (up); z = SiLU(y_gate) *
    // y_up goes to L[1].y; L[0].y is unused.
    int pair;
    float *amax_out;         // pair, nullable: per-token max |z| (zeroed before the launch; combined with atomic max)
};

// Short rows: one launch per group, every workgroup prepares its tokens itself.
struct ShortLayer {
    const v4u *packed;
    const float *s_w;
    const _Float16 *A, *B, *alpha;
    const float *gamma, *beta;   // as in ProTokens
    _Float16 *y;
    int32_t *acc_debug;
    float eps;
    int N, RBn, rank;
    int b_aligned;               // rows of B are whole aligned pieces of 8 ranks
};
struct ShortParams {
    const _Float16 *x;
    int M, K, Kp, KT, G, pair;   // pair: as in DecodeParams
    int plog, token_groups;      // log2 of a workgroup's tokens
    int KS;                      // wavefronts that share a row-block's k-tiles
    int vec;                     // rows of x and of every A are whole aligned pieces of 16 bytes
    int ustride, part_off, h_off, red_off;   // LDS: bytes between units of 16 columns; A x in parts; SiLU(A x); partial tiles
    float *amax_out;
    int wg_start[kMaxGroup + 1]; // running sum of the layers' row units
    ShortLayer L[kMaxGroup];
};
constexpr size_t kShortLdsMax = 150 * 1024;

// Single persistent launch for a handful of tokens: every workgroup quantises the tokens
// itself, streams its share of the row-blocks ("units") and exchanges the partial sums of
// A x with the others through a sentinel-filled buffer in the workspace.
constexpr int kMaxFusedM = 4, kMaxFusedB3M = 2;
constexpr int kMaxFusedK = 12288;
constexpr int kFusedSplit = 24;                               // slices of d_in at most (512 columns each)
constexpr size_t kMailLayerBytes = size_t(64) * HGF_MAX_RANK * 4;   // 64 (slice, token) rows of fp32 per layer
constexpr size_t kMailBytes = kMailLayerBytes * kMaxGroup;    // one exchange buffer; the workspace holds two
struct FusedParams {
    const _Float16 *x;            // [M, K] fp16
    int M, K, Kp, KT, TPW, G;     // TPW: tiles of a unit per streaming wavefront; Kp: whole k-tiles
    int base3;                    // packed: base-3 rows; a k-tile is 32 bytes of every row = 160 columns (G == 1)
    unsigned row_bytes;           // of them
    int own_polls;                // reads of the exchange before a workgroup of the base-3 launch helps itself
    DecLayer L[kMaxGroup];        // h16 unused
    const _Float16 *A[kMaxGroup];
    int ustart[kMaxGroup + 1];    // running sum of the layers' row-blocks
    int job_start[kMaxGroup + 1]; // running sum of the layers' (rank tile, slice) jobs
    int nwg;                      // workgroups of the launch
    int S, pairs, pairs_per_slice;
    int xstride, tile_off, h_off; // LDS: bytes per quantised token row; offsets of the units' int32 sums and of SiLU(A x)
    int unit_off, unit_stride, unit_alpha;   // LDS: staged epilogue operands (B rows, alpha) per unit
    unsigned char *mail;          // two exchange buffers of kMailBytes
    int32_t *flags;               // [0] launch counter, [1] workgroups done, [2] sticky: a wait ran out
};

// One persistent launch over a list of phases (groups of layers) for a handful of tokens.
// Sized so that the whole description fits the 4 KiB of kernel arguments.
constexpr int kStackMaxLayers = 48;
constexpr int kStackMaxPhases = 36;
constexpr size_t kStackActBytes = size_t(6) << 20;     // per set: exchange copies of the layers' outputs ...
constexpr size_t kStackSetBytes = size_t(8) << 20;     // ... followed by the partial sums of A x
struct StackLayer {                                    // 64 bytes
    const v4u *packed;
    const float *s_w;
    const _Float16 *A, *B, *alpha;
    _Float16 *y;
    int N, rank;
    unsigned act_off;             // byte offset of the output's exchange copy ([M][N] fp16, N % 8 == 0)
    int reserved;
};
struct StackPhase {                                    // 24 bytes
    const _Float16 *x_ext;        // the tokens, when they were written before the launch; else null
    int K;
    short first_layer, G;
    unsigned src_off;             // else: byte offset of their exchange copy
    unsigned mail_off;            // byte offset of the phase's partial sums of A x
};
// Time stamps of the whole-stack launch (a measurement aid, off unless a buffer is set): each
// role's first lane notes the device-wide 100 MHz clock at fixed points of kTracePhases
// consecutive phases; the words leave through LDS at the end of the launch.
constexpr int kTraceRoles = 11;       // contracting wavefronts 0..7, slice wavefront, unit wavefront, loader 0
constexpr int kTracePhases = 4;
constexpr int kTraceIds = 8;
struct StackParams {
    int M, nphases, nwg, trace_ph0;   // trace_ph0: first traced phase
    unsigned long long *trace;        // null, or [nwg][kTraceRoles][kTracePhases][kTraceIds] time stamps
    int32_t *flags;               // [2] sticky error, [4] launch counter, [5] workgroups done, [6], [7] extents used
    unsigned char *xchg;          // two sets of kStackSetBytes
    unsigned act_used, mail_used;
    int xstride, h_par, tile_off, tile_par, h_off, unit_off, unit_stride, unit_alpha, jx_off, ring_off, ring_slots;   // LDS layout
    int mem_polls, lds_polls;     // tries after which a wait for another workgroup / another wavefront gives up
    StackPhase ph[kStackMaxPhases];
    StackLayer L[kStackMaxLayers];
};
static_assert(sizeof(StackParams) <= 4096, "kernel arguments");

// A list of phases for 5 to 16 tokens as a queue of tasks, see hgf_batch.hip.
constexpr int kBatchTokens = 16;
constexpr int kBatchMinPhases = 5;
constexpr size_t kLastLevelCache = size_t(256) << 20;  // the Infinity Cache: a list of more weights finds none of them there
constexpr int kBatchMaxLayers = 40, kBatchMaxPhases = 16;
constexpr int kBatchSlices = 6;                        // slices of A x at most: d_in <= 12288
constexpr int kBatchWords = 512;                       // unit tasks of a phase at most
// A launch takes the whole-stack launch's set whose turn it is: copies of the layers' outputs in the place of its
// copies, from the first address that is a multiple of kBatchActAlign (no line holds two row-blocks' outputs); in the
// place of its sums of A x the tasks' words, [phase][kBatchWords], and this launch's sums.
constexpr size_t kBatchActAlign = 256;
constexpr size_t kBatchActBytes = kStackActBytes - kBatchActAlign;
constexpr size_t kBatchMailBytes = kStackSetBytes - kStackActBytes;
constexpr size_t kBatchPhaseWords = size_t(kBatchWords) * 4;   // bytes
struct BatchLayer {                                    // 64 bytes
    const v4u *packed;
    const float *s_w;
    const _Float16 *A, *B, *alpha;
    _Float16 *y;
    int N, rank;
    unsigned act_off, mail_off;                        // bytes: its copy; its sums of A x ([slice][token][h_stride] fp32) behind
                                                       // the set's copies
};
struct BatchPhase {                                    // 80 bytes
    const _Float16 *x_ext;                             // the tokens, when they were written before the launch (src_phase < 0)
    unsigned src_off;                                  // else: their copy
    int K, task0;                                      // its first task; job tasks come first
    int unit_end[3], job_end[3];                       // ends of its first layers' units and jobs (2^30 past the last)
    int units, jobs;                                   // row-blocks; tiles of A x
    int h_off, h_layer, red_off;                       // LDS: SiLU(A x), bytes of it per layer; partial tiles (0: in the tokens' place)
    unsigned char first_layer, G, upt, S;              // upt: units of a task at most
    short src_phase, src_layer;
    int unit_tasks;
};
struct BatchParams {
    int32_t *flags;               // [2] sticky error, [4], [6], [7] as in StackParams, [8] launches of this kind, [9] workgroups
                                  // done, [11] next task
    unsigned char *xchg;          // two sets of kStackSetBytes
    unsigned act_shift;           // bytes from a set's begin to its copies
    int M, nphases, tasks, cus;
    unsigned act_used, mail_used;
    int polls;
    BatchPhase ph[kBatchMaxPhases];
    BatchLayer L[kBatchMaxLayers];
};
static_assert(sizeof(BatchParams) <= 4096, "kernel arguments");

// ---- kernel launchers (each validates nothing: the ABI layer has done it) -----------
hipError_t launch_wsum(const float *W, size_t n, double *partials, float *s_w_out, hipStream_t st);
hipError_t launch_pack(const float *W, int N, int K, const float *s_w, uint32_t *packed, hipStream_t st);
hipError_t launch_unpack(const uint32_t *packed, int N, int K, int8_t *T, hipStream_t st);
hipError_t launch_fill(void *p, size_t bytes, uint32_t word, hipStream_t st);   // whole 16-byte units, 16-byte aligned
hipError_t launch_zero_words(void *p, size_t n, hipStream_t st);
hipError_t launch_quantize(const _Float16 *x, int M, int K, int8_t *xq, float *s_x, int32_t *rowsum,
                           hipStream_t st);
hipError_t launch_ln_quantize(const _Float16 *x, int M, int K, const float *gamma, const float *beta, float eps,
                              int8_t *xq, float *s_x, int32_t *rowsum, hipStream_t st);
hipError_t launch_corr_down(const _Float16 *x, int M, int K, int G, const _Float16 *const *A, const int *rank,
                            _Float16 *const *h16, int8_t *xq, float *s_x, int32_t *rowsum, hipStream_t st);   // rows of whole 16 bytes
int prologue_slices(int K);
hipError_t launch_prologue(ProParams &p, hipStream_t st);
hipError_t launch_decode(DecodeParams &p, int d_in, hipStream_t st);
bool plan_short(ShortParams &p, size_t *lds_bytes);
hipError_t launch_short(const ShortParams &p, size_t lds_bytes, hipStream_t st);
bool batch_fits(int M, int K, int G, int rank, long long row_blocks);   // one phase: its largest rank, all its rows
bool plan_batch(BatchParams &p, size_t *lds_bytes);
hipError_t launch_batch(const BatchParams &p, size_t lds_bytes, hipStream_t st);
// Lets `kernel` be launched with up to `bytes` of dynamic LDS on the current device (the runtime keeps that per device).
inline hipError_t allow_lds(OncePerDevice &once, const void *kernel, size_t bytes)
{
    int dev = -1;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    return (hipError_t)once(dev, [&] { return (int)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); });
}
// What a plan or a launch of one of the persistent kernels came to.
enum class Launch { kRan, kNoFit, kRefused };
bool plan_fused(FusedParams &p, size_t *lds_bytes);
hipError_t launch_fused(const FusedParams &p, size_t lds_bytes, hipStream_t st);
bool plan_stack(StackParams &p, size_t *lds_bytes);
void set_stack_wait_limit(int tries);
int stack_wait_limit();
void set_stack_trace(unsigned long long *buf, size_t bytes, int first_phase);
hipError_t launch_stack(const StackParams &p, size_t lds_bytes, hipStream_t st);
struct PairOut {                 // extra outputs of a SwiGLU pair launch (both nullable)
    int32_t *acc_debug2;         // the up projection's int32 accumulators
    float *amax_out;             // per-token max |z|
};
hipError_t launch_prefill(const Workspace &ws, _Float16 *const *h16, int M, const hgf_layer *layers, int G,
                          void *const *ys, int32_t *acc_debug, hipStream_t st, const PairOut *pair_out = nullptr);

// differential attention, one decode step
size_t diff_attn_workspace_bytes(int B, int L_max, int n_heads, int d_h);
hipError_t launch_diff_attn(const void *q, const void *k, const void *v, const int32_t *lens, int B, int L_max,
                            int n_heads, int d_h, float lambda, void *out, void *workspace, hipStream_t st);

// base-3 packing (five ternary weights per byte)
constexpr int kB3Cols = 80;                            // columns of 16 packed bytes; rows are padded to whole ones
size_t b3_packed_bytes(int d_out, int d_in);
hipError_t launch_pack_b3(const float *W, int N, int K, const float *s_w, unsigned char *packed, hipStream_t st);
hipError_t launch_unpack_b3(const unsigned char *packed, int N, int K, int8_t *T, hipStream_t st);

}  // namespace hgf
