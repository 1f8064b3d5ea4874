// Offline weight path: absmean ternarisation and the 2-bit packed layout.
//
// Sec. 2.2 of the HGF paper (weight-quantisation definition): gamma_W is the mean of |W|
// over the whole matrix and T = Clip(Round(W / gamma_W), -1, 1).  The sum is taken in
// fp64 in a fixed order (per-block partial sums, then one block), rounded once to fp32
// and clamped to >= 1e-5; every element is then multiplied by the fp32 reciprocal and
// rounded half-to-even.
#include "hgf_internal.h"

namespace hgf {

namespace {

// Sum over the workgroup (a multiple of 64 threads, at most 1024) in a fixed order: a butterfly
// inside each wavefront, then the wavefronts' sums one after the other.  Valid in thread 0.
__device__ inline double block_sum_f64(double v, double *sh)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)blockDim.x / 64; ++i) s += sh[i];
    return s;
}

// |W| summed over one contiguous chunk per workgroup, a multiple of four elements long.  Bound by
// HBM: eight independent 16-byte requests per thread and round, where one 4-byte load per dependent
// add reached 2.8 TB/s.
__global__ __launch_bounds__(256) void wsum_partial_kernel(const float *__restrict__ W, size_t n, size_t chunk,
                                                           double *__restrict__ partials)
{
    __shared__ double sh[4];
    constexpr int UN = 8;
    const size_t lo = chunk * blockIdx.x;
    const size_t hi = lo + chunk < n ? lo + chunk : n;
    const size_t len = lo < hi ? hi - lo : 0;                 // (a chunk stays below 2^31 bytes: n <= HGF_MAX_DIM^2)
    const unsigned whole = (unsigned)(len / 4);               // 16-byte pieces; beyond them the requests read as zero
    const rsrc_t r = make_rsrc(W + (len ? lo : 0), whole * 16u);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (unsigned i = threadIdx.x; i < whole; i += 256 * UN) {
        v4f v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) v[u] = __builtin_bit_cast(v4f, buf_load16(r, (i + u * 256) * 16u));
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] += fabs((double)v[u][e]);
    }
    double t = (s[0] + s[1]) + (s[2] + s[3]);
    if (threadIdx.x < (unsigned)(len % 4)) t += fabs((double)W[lo + whole * 4 + threadIdx.x]);
    t = block_sum_f64(t, sh);
    if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

__global__ __launch_bounds__(kWsumBlocks) void wsum_final_kernel(const double *__restrict__ partials, size_t n,
                                                                 float *__restrict__ s_w)
{
    __shared__ double sh[kWsumBlocks / 64];
    const double s = block_sum_f64(partials[threadIdx.x], sh);
    if (threadIdx.x == 0) {
        float g = (float)(s / (double)n);
        *s_w = g < 1e-5f ? 1e-5f : g;
    }
}

__device__ inline uint32_t ternary_code(float w, float inv)
{
    float q = rintf(w * inv);
    q = fminf(fmaxf(q, -1.0f), 1.0f);
    return (uint32_t)((int)q + 1);
}

// Position of packed word `idx`: tile = idx/256; within the tile, lane l = (idx%256)/4 and
// word t = idx%4 hold row 32*rb + (l%32), columns 128*kt + 32*t + 16*(l/32) + 0..15.
__device__ inline void word_position(size_t idx, int KT, int &row, int &kbase)
{
    const size_t tile = idx >> 8;
    const int within = (int)(idx & 255);
    const int l = within >> 2, t = within & 3;
    const int rb = (int)(tile / KT), kt = (int)(tile % KT);
    row = rb * kTileRows + (l & 31);
    kbase = kt * kTileCols + t * 32 + (l >> 5) * 16;
}

// One wavefront per packed tile.  Bound by HBM (16 KiB read, 1 KiB written): every request takes two
// whole 512-byte row pieces, all sixteen are in flight together, and the tile leaves as one KiB.
// (One thread per packed word read 64 bytes per lane at a stride of a row and stored single words:
// 147 us for 11008 x 4096; sum and packing together 233.5 us then, 67.0 us now, both passes at about
// 5.8 TB/s because the second finds much of W in the 256 MB Infinity Cache.)
// Lane l holds columns 4c .. 4c+3 (c = l % 32) of row 2i + l/32: codes b = 0..3 of shift s = c % 4 in
// word t = c / 8, k-half (c / 4) % 2, so the four lanes of a quad share a word and OR their parts.
// TAIL: rows that are not a multiple of four columns (the code for their ends costs the others: 4096 x 4096
// 34.0 us with it, 33.3 without).
template <bool TAIL>
__global__ __launch_bounds__(256) void pack_kernel(const float *__restrict__ W, int N, int K, int KT,
                                                   const float *__restrict__ s_w,
                                                   uint32_t *__restrict__ packed, size_t ntiles)
{
    __shared__ __attribute__((aligned(16))) uint32_t words[4][256];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const size_t tile = (size_t)blockIdx.x * 4 + w;
    if (tile >= ntiles) return;
    const int rb = (int)(tile / KT), kt = (int)(tile % KT);
    const int row0 = rb * kTileRows, rows = min(kTileRows, N - row0);
    const int c = l & 31, k0 = kt * kTileCols + 4 * c;
    // the rows of the block behind one descriptor (at most 32 rows of HGF_MAX_DIM floats); rows start
    // at any multiple of four bytes, which is all a 16-byte request asks for
    const rsrc_t r = make_rsrc(W + (size_t)row0 * K, (unsigned)rows * K * 4u);
    // (the lane that holds a row's last one to three columns asks for the row's last four, in the same burst, and
    // moves them down: three more requests per row behind the first cost 0.4 us, 65 x 65 9.5 against 9.1)
    const bool last = TAIL && K >= 4 && k0 < K && k0 + 3 >= K;
    const int from = last ? K - 4 : k0;
    v4f v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 2 * i + (l >> 5);
        v[i] = __builtin_bit_cast(v4f, buf_load16(r, ((unsigned)row * K + from) * 4u, row < rows && from + 3 < K));
    }
    if (TAIL && kt == KT - 1 && K >= 4) {
        const int down = 4 - K % 4;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const v4f u = v[i];
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const float t = down == 1 ? u[e + 1] : (down == 2 ? u[e < 2 ? e + 2 : 3] : u[3]);
                v[i][e] = last ? t : u[e];
            }
        }
    } else if (TAIL && K < 4) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = 2 * i + (l >> 5);
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                const bool tail = row < rows && k0 + 3 >= K && k0 + e < K;
                const float t = __builtin_bit_cast(float, buf_load4(r, ((unsigned)row * K + k0 + e) * 4u, tail));
                v[i][e] = tail ? t : v[i][e];
            }
        }
    }
    const float inv = 1.0f / *s_w;
    const int word = ((c >> 2) & 1) * kTileRows * 4 + (c >> 3);      // + 4 * row
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = 2 * i + (l >> 5);
        uint32_t part = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)                // padding rows and columns decode to 0
            part |= ((row < rows && k0 + e < K) ? ternary_code(v[i][e], inv) : 1u) << (8 * e);
        part <<= 2 * (c & 3);
        part |= (uint32_t)dpp_move<0xB1>((int)part);
        part |= (uint32_t)dpp_move<0x4E>((int)part);
        if ((c & 3) == 0) words[w][word + 4 * row] = part;
    }
    // the wavefront's own words, from other lanes: LDS takes its requests in order, the fences keep the compiler
    // from reordering them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    reinterpret_cast<v4u *>(packed)[tile * 64 + l] = reinterpret_cast<const v4u *>(words[w])[l];
}

// One thread per packed word, writing its 16 values back as int8 -1/0/+1.
__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t *__restrict__ packed, int N, int K, int KT,
                                                     int8_t *__restrict__ T, size_t nwords)
{
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nwords) return;
    int row, kbase;
    word_position(idx, KT, row, kbase);
    if (row >= N) return;
    const uint32_t word = packed[idx];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int k = kbase + 4 * s + b;
            if (k < K) T[(size_t)row * K + k] = (int8_t)((int)((word >> (8 * b + 2 * s)) & 3u) - 1);
        }
    }
}

__global__ __launch_bounds__(256) void fill_kernel(uint4 *__restrict__ p, size_t n16, uint32_t word)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = make_uint4(word, word, word, word);
}

__global__ __launch_bounds__(256) void zero_words_kernel(uint32_t *__restrict__ p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

}  // namespace

// Zeroes n 4-byte words at any 4-byte aligned address (a kernel, so it may be captured in a graph).
hipError_t launch_zero_words(void *p, size_t n, hipStream_t st)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<uint32_t *>(p), n);
    return hipGetLastError();
}

hipError_t launch_wsum(const float *W, size_t n, double *partials, float *s_w_out, hipStream_t st)
{
    const size_t chunk = ((n + kWsumBlocks - 1) / kWsumBlocks + 3) / 4 * 4;
    hipLaunchKernelGGL(wsum_partial_kernel, dim3(kWsumBlocks), dim3(256), 0, st, W, n, chunk, partials);
    hipLaunchKernelGGL(wsum_final_kernel, dim3(1), dim3(kWsumBlocks), 0, st, partials, n, s_w_out);
    return hipGetLastError();
}

hipError_t launch_pack(const float *W, int N, int K, const float *s_w, uint32_t *packed, hipStream_t st)
{
    const int KT = round_up(K, kTileCols) / kTileCols;
    const size_t ntiles = (size_t)(round_up(N, kTileRows) / kTileRows) * KT;
    const dim3 grid((unsigned)((ntiles + 3) / 4)), block(256);
    if (K % 4 == 0)
        hipLaunchKernelGGL(pack_kernel<false>, grid, block, 0, st, W, N, K, KT, s_w, packed, ntiles);
    else
        hipLaunchKernelGGL(pack_kernel<true>, grid, block, 0, st, W, N, K, KT, s_w, packed, ntiles);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint32_t *packed, int N, int K, int8_t *T, hipStream_t st)
{
    const int KT = round_up(K, kTileCols) / kTileCols;
    const size_t nwords = (size_t)(round_up(N, kTileRows) / kTileRows) * KT * 256;
    hipLaunchKernelGGL(unpack_kernel, dim3((unsigned)((nwords + 255) / 256)), dim3(256), 0, st, packed, N, K, KT,
                       T, nwords);
    return hipGetLastError();
}

hipError_t launch_fill(void *p, size_t bytes, uint32_t word, hipStream_t st)
{
    const size_t n16 = bytes / 16;                               // callers pass multiples of 16
    unsigned blocks = (unsigned)((n16 + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel, dim3(blocks), dim3(256), 0, st, (uint4 *)p, n16, word);
    return hipGetLastError();
}

}  // namespace hgf
