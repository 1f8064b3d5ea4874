// Differential attention, one decode step (the block that consumes the HGF q/k/v projections).
//
// Sec. 2.4, Def. "Differential Attention": with Q = [Q1; Q2] and K = [K1; K2] split into two
// groups of heads,  O = (softmax(Q1 K1^T / sqrt(d_h)) - lambda softmax(Q2 K2^T / sqrt(d_h))) V.
// The appendix implementation fixes what the definition leaves open: q and k carry 2 n_heads
// heads of d_h = d_model / (2 n_heads) columns (the first n_heads are branch 1, the rest branch
// 2), v carries n_heads heads of the same d_h (V: d -> d/2), head h of both branches reads head
// h of v, the scores are scaled by 1/sqrt(d_h), and the difference is multiplied by 0.5.
//
// Decode: the newest token attends to every cached position 0 .. len-1 (itself included), so
// a step streams the K and V caches once: 6 len d_h bytes per head, nothing else of size.
// That is bandwidth-bound work with no reuse, so there are no matrix instructions here:
// coalesced 16-byte loads, dot products in the vector ALU, cross-lane reductions.
//   pass 1 (grid: chunks of 256 positions, heads, sequences): a workgroup loads its chunk
//     of K1 and K2 rows of one head in one burst, forms both branches' scores, maxima and
//     exponentials while the V rows arrive, and both exp-weighted sums of the V rows, which it
//     reads once for the two; it writes (max, sum, weighted V) per branch to the workspace;
//   pass 2 (grid: heads x sequences): merges the chunks (rescaling by exp(max_chunk - max)),
//     normalises, forms (a1 - lambda a2) * 0.5 and stores fp16.  Caches of one chunk need no
//     second launch: pass 1 does it.
#include "hgf_internal.h"

#include <type_traits>

namespace hgf {

namespace {

constexpr int kAttnChunk = 256;        // positions per workgroup of pass 1 (one per thread)

struct AttnParams {
    const _Float16 *q;                 // [B, 2 n_heads, d_h]
    const _Float16 *k;                 // [B, L_max, 2 n_heads, d_h]
    const _Float16 *v;                 // [B, L_max, n_heads, d_h]
    const int32_t *lens;               // [B]
    float *part;                       // [B, n_heads, chunks, 2, d_h + 2]
    _Float16 *out;                     // [B, n_heads, d_h]
    int B, L_max, n_heads, d_h, chunks;
    int heads_first, rotate;           // grid of pass 1: heads fastest, else chunks; see launch_diff_attn
    float lambda, scale;
};

// Sum over aligned groups of G lanes (G a power of two up to 16), in every lane of the group.
template <int G>
__device__ inline float group_sum(float v)
{
    auto mv = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, dpp_move<decltype(ctrl)::value>(__builtin_bit_cast(int, x)));
    };
    if (G > 1) v += mv(v, std::integral_constant<int, 0xB1>{});     // quad_perm [1,0,3,2]
    if (G > 2) v += mv(v, std::integral_constant<int, 0x4E>{});     // quad_perm [2,3,0,1]
    if (G > 4) v += mv(v, std::integral_constant<int, 0x141>{});    // row_half_mirror
    if (G > 8) v += mv(v, std::integral_constant<int, 0x140>{});    // row_mirror
    return v;
}

// V8: 16-byte pieces of a head row (d_h / 8).  Lane (ps = l / V8, pc = l % V8) takes piece pc of
// the positions ps, ps + P, ... of its wavefront's 64 positions (P = 64 / V8 per instruction).
// Bound by HBM.  Each wavefront is a softmax of its own over its 64 positions, in registers: the only
// meeting of the workgroup is the merge of its four (max, sum, weighted V) at the end.  The V8 lanes of
// a position hold the same score, so each of them takes the exponential of one of the lane's V8
// positions and hands it round (all V8 in every lane: 15.5 us for 512 positions of 32 heads of 64 over 8
// caches, 13.9 so), and V is requested when the registers of K are free again (90 instead of 124 at d_h =
// 64, 164 instead of 226 at 128).
template <int V8>
__global__ __launch_bounds__(256) void diff_attn_chunk_kernel(AttnParams p)
{
    constexpr int P = 64 / V8, IT = 64 / P, d_h = V8 * 8;
    __shared__ float accs[4][2][d_h];
    __shared__ float mx_s[4][2], sum_s[4][2];
    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = p.heads_first ? blockIdx.x : blockIdx.y, b = blockIdx.z;
    int chunk = p.heads_first ? blockIdx.y : blockIdx.x;
    if (p.rotate) chunk = (chunk + (V8 < 8 ? h * V8 / 8 : h) + b) % p.chunks;      // (by cache lines of heads, and by sequences)
    const int len = min(max(p.lens[b], 0), p.L_max);
    const int pos0 = chunk * kAttnChunk;
    if (pos0 >= len) {                  // nothing cached here (the merge reads only the chunks below len)
        if (p.chunks == 1 && tid < d_h) p.out[((size_t)b * p.n_heads + h) * d_h + tid] = (_Float16)0.f;
        return;
    }
    const int ps = l / V8, pc = l % V8;
    const size_t krow = (size_t)2 * p.n_heads * d_h, vrow = (size_t)p.n_heads * d_h;
    const rsrc_t kr = make_rsrc(p.k + (size_t)b * p.L_max * krow, (unsigned)((size_t)len * krow * 2));
    const rsrc_t vr = make_rsrc(p.v + (size_t)b * p.L_max * vrow, (unsigned)((size_t)len * vrow * 2));
    const _Float16 *qb = p.q + (size_t)b * krow;
    const v8h q1 = *reinterpret_cast<const v8h *>(qb + (size_t)h * d_h + pc * 8);
    const v8h q2 = *reinterpret_cast<const v8h *>(qb + (size_t)(p.n_heads + h) * d_h + pc * 8);
    // (rows past len lie beyond the descriptors: zeros)
    v4u k1[IT], k2[IT], vv[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const unsigned pos = (unsigned)(pos0 + w * 64 + it * P + ps);
        k1[it] = buf_load16_stream(kr, (unsigned)((pos * krow + (size_t)h * d_h + pc * 8) * 2));
        k2[it] = buf_load16_stream(kr, (unsigned)((pos * krow + (size_t)(p.n_heads + h) * d_h + pc * 8) * 2));
    }
    // ---- scores of both branches (each in all lanes of its position)
    float s[2][IT], mx[2] = {-INFINITY, -INFINITY}, sum[2];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const v8h x1 = __builtin_bit_cast(v8h, k1[it]), x2 = __builtin_bit_cast(v8h, k2[it]);
        float s1 = 0.f, s2 = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            s1 += (float)q1[e] * (float)x1[e];
            s2 += (float)q2[e] * (float)x2[e];
        }
        const bool valid = pos0 + w * 64 + it * P + ps < len;
        s[0][it] = valid ? group_sum<V8>(s1) * p.scale : -INFINITY;
        s[1][it] = valid ? group_sum<V8>(s2) * p.scale : -INFINITY;
        mx[0] = fmaxf(mx[0], s[0][it]);
        mx[1] = fmaxf(mx[1], s[1][it]);
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const unsigned pos = (unsigned)(pos0 + w * 64 + it * P + ps);
        vv[it] = buf_load16_stream(vr, (unsigned)((pos * vrow + (size_t)h * d_h + pc * 8) * 2));
    }
#pragma unroll
    for (int br = 0; br < 2; ++br) {
        mx[br] = wave_max(mx[br]);
        const float m = mx[br] == -INFINITY ? 0.f : mx[br];      // (no position here: every weight is exp(-inf) = 0)
        static_assert(IT == V8, "one exponential per lane");
        float mine = s[br][0];                                   // the weight of the lane's pc-th position
#pragma unroll
        for (int it = 1; it < IT; ++it) mine = pc == it ? s[br][it] : mine;
        mine = expf(mine - m);
#pragma unroll
        for (int it = 0; it < IT; ++it)
            s[br][it] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((ps * V8 + it) * 4, __builtin_bit_cast(int, mine)));
        sum[br] = group_sum<V8>(mine);
#pragma unroll
        for (int o = V8; o < 64; o <<= 1) sum[br] += __shfl_xor(sum[br], o, 64);
    }
    // ---- both branches' weighted sums of the V rows (read once)
    float a[2][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) a[0][e] = a[1][e] = 0.f;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        const v8h x = __builtin_bit_cast(v8h, vv[it]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a[0][e] += s[0][it] * (float)x[e];
            a[1][e] += s[1][it] * (float)x[e];
        }
    }
#pragma unroll
    for (int o = V8; o < 64; o <<= 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            a[0][e] += __shfl_xor(a[0][e], o, 64);
            a[1][e] += __shfl_xor(a[1][e], o, 64);
        }
    }
    if (ps == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            accs[w][0][pc * 8 + e] = a[0][e];
            accs[w][1][pc * 8 + e] = a[1][e];
        }
    }
    if (l < 2) {
        mx_s[w][l] = l == 0 ? mx[0] : mx[1];
        sum_s[w][l] = l == 0 ? sum[0] : sum[1];
    }
    __syncthreads();
    const int br = tid / d_h, d = tid % d_h;
    float acc = 0.f, total = 0.f, m = 0.f;
    if (br < 2) {
        m = fmaxf(fmaxf(mx_s[0][br], mx_s[1][br]), fmaxf(mx_s[2][br], mx_s[3][br]));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float f = sum_s[i][br] == 0.f ? 0.f : expf(mx_s[i][br] - m);     // (0: no positions there)
            acc += accs[i][br][d] * f;
            total += sum_s[i][br] * f;
        }
    }
    if (p.chunks == 1) {                // no merge follows
        if (br < 2) accs[0][br][d] = acc / total;                // (its own element: no other thread reads it before)
        __syncthreads();
        if (br == 0) p.out[((size_t)b * p.n_heads + h) * d_h + d] = (_Float16)((accs[0][0][d] - p.lambda * accs[0][1][d]) * 0.5f);
    } else if (br < 2) {
        float *out = p.part + ((((size_t)b * p.n_heads + h) * p.chunks + chunk) * 2 + br) * (d_h + 2);
        out[2 + d] = acc;
        if (d == 0) {
            out[0] = m;
            out[1] = total;
        }
    }
}

// One workgroup of eight wavefronts per head and sequence; wavefronts 0 and 1, one branch each, turn up
// to 64 chunks' (max, sum) at a time into weights (LDS), then four groups of 128 threads, one per
// column, take every fourth chunk's rows.  Bound by latency: a fixed number of
// trips to memory, where two loops over the chunks with a dependent load in each took 16.9 us at
// 16 chunks.
__global__ __launch_bounds__(512) void diff_attn_merge_kernel(AttnParams p)
{
    __shared__ float wgt[2][64], red[4][2][128], scale_s[2], sum_s[2];
    const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int d_h = p.d_h, d = tid & 127, part4 = tid >> 7;
    const float *part = p.part + (((size_t)b * p.n_heads + h) * p.chunks) * 2 * (d_h + 2);
    const int len = min(max(p.lens[b], 0), p.L_max);
    const int used = (len + kAttnChunk - 1) / kAttnChunk;
    float acc[2] = {0.f, 0.f};
    float run_m = -INFINITY, run_sum = 0.f;         // wavefronts 0 and 1: one branch each
    for (int c0 = 0; c0 < used; c0 += 64) {
        if (c0 > 0) __syncthreads();                // the weights of the batch before have been used
        const int n = min(64, used - c0);
        if (tid < 128) {
            const int br = tid >> 6, c = tid & 63;
            const float *q = part + ((size_t)(c0 + c) * 2 + br) * (d_h + 2);
            const float mc = c < n ? q[0] : -INFINITY, sc = c < n ? q[1] : 0.f;
            const float m = fmaxf(run_m, wave_max(mc));
            const float base = m == -INFINITY ? 0.f : m;
            const float f = expf(mc - base), keep = expf(run_m - base);
            float t = sc * f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
            run_sum = run_sum * keep + t;
            run_m = m;
            wgt[br][c] = f;
            if (c == 0) {
                scale_s[br] = keep;
                sum_s[br] = run_sum;
            }
        }
        __syncthreads();
        acc[0] *= scale_s[0];
        acc[1] *= scale_s[1];
        if (d < d_h) {
#pragma unroll 4
            for (int c = part4; c < n; c += 4) {
                const float *q = part + (size_t)(c0 + c) * 2 * (d_h + 2) + 2 + d;
                acc[0] += q[0] * wgt[0][c];
                acc[1] += q[d_h + 2] * wgt[1][c];
            }
        }
    }
    red[part4][0][d] = acc[0];
    red[part4][1][d] = acc[1];
    __syncthreads();
    if (part4 == 0 && d < d_h) {
        float o[2] = {0.f, 0.f};
        if (used > 0) {
#pragma unroll
            for (int br = 0; br < 2; ++br)
                o[br] = ((red[0][br][d] + red[1][br][d]) + (red[2][br][d] + red[3][br][d])) / sum_s[br];
        }
        p.out[((size_t)b * p.n_heads + h) * d_h + d] = (_Float16)((o[0] - p.lambda * o[1]) * 0.5f);
    }
}

}  // namespace

size_t diff_attn_workspace_bytes(int B, int L_max, int n_heads, int d_h)
{
    const size_t chunks = (size_t)(L_max + kAttnChunk - 1) / kAttnChunk;
    return (size_t)B * n_heads * chunks * 2 * (d_h + 2) * sizeof(float);
}

hipError_t launch_diff_attn(const void *q, const void *k, const void *v, const int32_t *lens, int B, int L_max,
                            int n_heads, int d_h, float lambda, void *out, void *workspace, hipStream_t st)
{
    AttnParams p;
    p.q = reinterpret_cast<const _Float16 *>(q);
    p.k = reinterpret_cast<const _Float16 *>(k);
    p.v = reinterpret_cast<const _Float16 *>(v);
    p.lens = lens;
    p.part = reinterpret_cast<float *>(workspace);
    p.out = reinterpret_cast<_Float16 *>(out);
    p.B = B;
    p.L_max = L_max;
    p.n_heads = n_heads;
    p.d_h = d_h;
    p.chunks = (L_max + kAttnChunk - 1) / kAttnChunk;
    p.lambda = lambda;
    p.scale = 1.0f / sqrtf((float)d_h);
    // Heads or chunks fastest.  Where heads share a cache line (128 bytes: d_h < 64), chunks: such heads then read
    // it on one XCD when the chunks are a multiple of eight.  From 128 columns on heads, which reads whole cache
    // rows; between, chunks for many workgroups, heads for few, for four chunks, and for long caches, whose
    // chunks alone fill the chip.  With chunks fastest an XCD would always get the same chunks, and caches that
    // are not full have only the first ones: the chunks are rotated from line to line and sequence to sequence.
    // (us, chunks rotated / heads fastest, caches read in turn that the Infinity Cache does not hold.  Full:
    // 8 of 4096 positions, 32 heads of 16 columns 39 / 77, of 32 47 / 75; 64 of 4096, 8 heads of 64 131 / 143; one of
    // 4096, 32 heads of 64 18.6 / 15.8; 4 of 8192, 16 heads of 128 75 / 68.  8 ragged caches of up to 4096, 32
    // heads, chunks not rotated / rotated / heads: 16 columns 34 / 28 / 46, 32 38 / 33 / 45, 64 52 / 44 / 44.  Of 802
    // sizes and fillings 12 are more than 3 % slower than the better of the two orders, taken throughout and
    // not rotated: at worst 4 caches of 8192, 30 % full, 16 heads of 32, 24.5 instead of 21.3.)
    // Only chunks can be more than the 65535 that a grid's other dimensions take, and only below 64 columns.
    p.heads_first = d_h >= 64 && p.chunks > 3 &&
                    (d_h > 64 || p.chunks == 4 || p.chunks >= 32 || (long long)B * n_heads * p.chunks < 2048);
    p.rotate = !p.heads_first;
    const dim3 grid = p.heads_first ? dim3(n_heads, p.chunks, B) : dim3(p.chunks, n_heads, B), block(256);
    switch (d_h / 8) {
        case 1: hipLaunchKernelGGL(diff_attn_chunk_kernel<1>, grid, block, 0, st, p); break;
        case 2: hipLaunchKernelGGL(diff_attn_chunk_kernel<2>, grid, block, 0, st, p); break;
        case 4: hipLaunchKernelGGL(diff_attn_chunk_kernel<4>, grid, block, 0, st, p); break;
        case 8: hipLaunchKernelGGL(diff_attn_chunk_kernel<8>, grid, block, 0, st, p); break;
        case 16: hipLaunchKernelGGL(diff_attn_chunk_kernel<16>, grid, block, 0, st, p); break;
        default: return hipErrorInvalidValue;
    }
    if (p.chunks > 1) hipLaunchKernelGGL(diff_attn_merge_kernel, dim3(n_heads, B), dim3(512), 0, st, p);
    return hipGetLastError();
}

}  // namespace hgf
