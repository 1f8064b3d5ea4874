// Preparation of a group of layers that read the same activations, for the direct path (and, where the
// prefill path's own is slower, for that): one launch
// that quantises the tokens and computes SiLU(A x) of every layer.
//
// Algorithm 1 of the HGF paper, steps 1-2 (per-token absmax int8 quantisation, Sec. 2.2.1, behind a
// LayerNorm where the layer has one) and steps 5-6 (H <- SiLU(X A) on the UN-quantised fp16
// activations).  Two roles share the grid; both only read x.
//
// Down-projection: a workgroup of eight wavefronts owns one tile of 16 ranks x 16 TT tokens of one
// layer and a slice of d_in: wavefront w takes the 64-column steps w, w+8, ... on the 16x16x32 f16
// MFMA (rows = rank indices, columns = tokens), and the eight partial tiles meet in LDS and are added
// in order.  Up to 2048 columns are one slice, SiLU(A x) leaves as fp16; longer rows are cut, because
// one compute unit takes in only some 0.1 MB per microsecond (all of d_in = 11008 in a workgroup: 19 us
// for 8 tokens, 32 us for 64), their slices leave as fp32 and the consumer adds them in order.
// Bound by latency: the launch is one or two memory round trips (6 us for a group of the 7B shape at 8
// tokens, 6.8 at 64, where all token tiles in one wavefront took 12.7).
//
// Quantiser: 64 to 512 threads per token by the row's length, the row in registers between the
// passes.  x_q is stored the way the consumer's MFMA operand wants it: per group of up to 32 tokens
// 16-byte pieces of 16 columns, [d_in / 16][token], so that a wavefront's request is contiguous.
// (500 tokens of 1408 columns behind a LayerNorm: 13.2 us with 256 threads per token and gamma and beta
// requested behind the reductions, 7.4 with 128 and requested with the row.)
#include "hgf_internal.h"

namespace hgf {

namespace {

constexpr int kProThreads = 512, kProWaves = kProThreads / 64;

// Eight (16) consecutive fp16 of a row whose address is any multiple of two bytes: the aligned dwords
// that hold them, shifted together.  `r` starts at a multiple of four bytes; `at`: byte offset of the
// first; the caller has checked that the dword behind the last whole one is inside as well when
// `at` is odd in units of two bytes.
template <int NW>      // words of two fp16
__device__ inline void load_unaligned(rsrc_t r, unsigned at, bool ok, unsigned (&out)[NW])
{
    unsigned d[NW + 1];
    const unsigned base = ok ? (at & ~3u) : kOob;
#pragma unroll
    for (int i = 0; i < NW; i += 4) {
        const v4u v = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(base + i * 4), 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) d[i + e] = v[e];
    }
    const unsigned odd = at & 2u;
    d[NW] = buf_load4(r, base + NW * 4, ok && odd);
#pragma unroll
    for (int i = 0; i < NW; ++i) out[i] = __builtin_amdgcn_alignbit(d[i + 1], d[i], odd * 8u);
}

// ---------------------------------------------------------------- quantiser

// T threads per token, NU 16-column units per thread kept in registers (longer rows are read again
// for every pass).
template <int T, int NU, bool VEC>
__device__ inline void quantize_tokens(const ProParams &p, const ProTokens &Q, int first)
{
    __shared__ double sh_d[kProWaves];
    __shared__ float sh_f[kProWaves];
    __shared__ int sh_i[kProWaves];
    constexpr int GW = T / 64;                      // wavefronts per token
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = threadIdx.x % T;
    const int w0 = w / GW * GW;
    const int m = first + w / GW;
    const bool live = m < p.M;                      // (a token group past the end still meets the others)
    const _Float16 *row = p.x + (size_t)(live ? m : 0) * p.K;
    const unsigned mis = (unsigned)(reinterpret_cast<uintptr_t>(row) & 2u);
    const rsrc_t r = make_rsrc(reinterpret_cast<const char *>(row) - mis, live ? (unsigned)p.K * 2u + mis : 0u);
    const int units = p.Kp / 16, chunks = (units + T * NU - 1) / (T * NU);

    auto total_d = [&](double v) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (GW == 1) return v;
        __syncthreads();
        if ((threadIdx.x & 63) == 0) sh_d[w] = v;
        __syncthreads();
        v = sh_d[w0];
        for (int i = 1; i < GW; ++i) v += sh_d[w0 + i];
        return v;
    };

    float v[NU][16];
    auto load = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = ((chunk * NU + u) * T + t) * 16;
            if (VEC) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const v8h x = __builtin_bit_cast(v8h, buf_load16(r, (unsigned)(col + h * 8) * 2u));
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[u][h * 8 + e] = (float)x[e];
                }
            } else {
                unsigned wd[8];
                const bool whole = col + 16 + (int)(mis >> 1) <= p.K;
                load_unaligned<8>(r, (unsigned)col * 2u + mis, whole, wd);
#pragma unroll
                for (int e = 0; e < 16; ++e) v[u][e] = (float)half_bits((unsigned short)(wd[e >> 1] >> (16 * (e & 1))));
                if (!whole && col < p.K) {          // the row's last columns, one by one
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        v[u][e] = (float)half_bits(buf_load2(r, (unsigned)(col + e) * 2u + mis, col + e < p.K));
                }
            }
        }
    };
    const bool ln = Q.gamma != nullptr;
    float mu = 0.f, rstd = 0.f;
    // gamma and beta of a chunk (a row in registers has them requested with it, ahead of the reductions)
    v4f ga[NU][4], be[NU][4];
    auto load_norm = [&](int chunk) __attribute__((always_inline)) {
        const rsrc_t gr = make_rsrc(Q.gamma, (unsigned)p.K * 4u), br = make_rsrc(Q.beta, Q.beta ? (unsigned)p.K * 4u : 0u);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = ((chunk * NU + u) * T + t) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                // (gamma and beta start at any multiple of four bytes, which is all the request asks for)
                const bool whole = col + q * 4 + 4 <= p.K;
                ga[u][q] = __builtin_bit_cast(v4f, buf_load16(gr, (unsigned)(col + q * 4) * 4u, whole));
                be[u][q] = __builtin_bit_cast(v4f, buf_load16(br, (unsigned)(col + q * 4) * 4u, whole));
            }
        }
        if (p.K % 4 == 0) return;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = ((chunk * NU + u) * T + t) * 16;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (col + q * 4 + 4 > p.K && col + q * 4 < p.K) {
#pragma unroll
                    for (int e = 0; e < 3; ++e) {
                        ga[u][q][e] = __builtin_bit_cast(float, buf_load4(gr, (unsigned)(col + q * 4 + e) * 4u, col + q * 4 + e < p.K));
                        be[u][q][e] = __builtin_bit_cast(float, buf_load4(br, (unsigned)(col + q * 4 + e) * 4u, col + q * 4 + e < p.K));
                    }
                }
            }
        }
    };
    auto normalise = [&](int chunk) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int col = ((chunk * NU + u) * T + t) * 16;
#pragma unroll
            for (int e = 0; e < 16; ++e) {          // in exactly this order, one rounding each; 0 past the row
                float y = v[u][e] - mu;
                y = y * rstd;
                y = y * ga[u][e / 4][e % 4];
                y = y + be[u][e / 4][e % 4];
                v[u][e] = col + e < p.K ? y : 0.f;
            }
        }
    };
    if (chunks == 1) {
        load(0);
        if (ln) load_norm(0);
    }
    if (ln) {
        // mean and mean squared deviation in fp64, each rounded once
        double s = 0.0;
        for (int c = 0; c < chunks; ++c) {
            if (chunks > 1) load(c);
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) s += (double)v[u][e];           // (zero past the row)
        }
        const double mean = total_d(s) / (double)p.K;
        double ss = 0.0;
        for (int c = 0; c < chunks; ++c) {
            if (chunks > 1) load(c);
#pragma unroll
            for (int u = 0; u < NU; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const double d = ((c * NU + u) * T + t) * 16 + e < p.K ? (double)v[u][e] - mean : 0.0;
                    ss += d * d;
                }
        }
        const double var = total_d(ss) / (double)p.K;
        mu = (float)mean;
        rstd = (float)(1.0 / sqrt(var + (double)Q.eps));
        if (chunks == 1) normalise(0);
    }
    float amax = 0.f;
    for (int c = 0; c < chunks; ++c) {
        if (chunks > 1) {
            load(c);
            if (ln) {
                load_norm(c);
                normalise(c);
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) amax = fmaxf(amax, fabsf(v[u][e]));
    }
    amax = wave_max(amax);
    if (GW > 1) {
        if ((threadIdx.x & 63) == 0) sh_f[w] = amax;
        __syncthreads();
        for (int i = 0; i < GW; ++i) amax = fmaxf(amax, sh_f[w0 + i]);
    }
    amax = fmaxf(amax, 1e-5f);
    const float inv = 127.0f / amax;
    int sum = 0;
    const int tg = m >> 5, rows = min(32, p.M - tg * 32);        // the token's group of 32 and its size
    int8_t *out = Q.xq + (p.by_rows ? (size_t)m * p.Kp : (size_t)tg * 32 * p.Kp + (m & 31) * 16);
    const int step = p.by_rows ? 16 : rows * 16;
    for (int c = 0; c < chunks; ++c) {
        if (chunks > 1) {
            load(c);
            if (ln) {
                load_norm(c);
                normalise(c);
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = (c * NU + u) * T + t;
            v4u o;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                unsigned word = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int q = quant1(v[u][d * 4 + b], inv);
                    sum += q;
                    word |= (unsigned)(q & 0xff) << (8 * b);
                }
                o[d] = word;
            }
            if (p.base3) {                          // (every byte to its digit's piece)
                if (live && unit < units) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int col = unit * 16 + e, b = col / 5, digit = col - b * 5;
                        Q.xq[(size_t)(((b >> 4) * 5 + digit) * p.M + m) * 16 + (b & 15)] = (int8_t)(o[e >> 2] >> (8 * (e & 3)));
                    }
                }
            } else if (live && unit < units) *reinterpret_cast<v4u *>(out + (size_t)unit * step) = o;
        }
    }
    sum = wave_sum(sum);
    if (GW > 1) {
        if ((threadIdx.x & 63) == 0) sh_i[w] = sum;
        __syncthreads();
        sum = 0;
        for (int i = 0; i < GW; ++i) sum += sh_i[w0 + i];
    }
    if (live && t == 0) {
        Q.s_x[m] = amax / 127.0f;
        Q.rowsum[m] = sum;
        if (p.amax_zero) p.amax_zero[m] = 0.0f;
    }
}

// ---------------------------------------------------------------- down-projection with SiLU

// Lane (i = l%16, kb = l/16) holds A[rt*16+i][k] and x[m][k], m = token tile's i-th, for the same eight
// k per MFMA: k = 64*step + 16*kb + 0..7 and + 8..15 (two MFMAs per 64 columns), so a row is read
// 128 contiguous bytes at a time.
template <int TT, bool VEC>
__device__ inline void corr_tile(const ProParams &p, int job)
{
    __shared__ v4f red[kProWaves][TT][64];
    int g = 0;
    while (g + 1 < p.G && job >= p.job_start[g + 1]) ++g;
    const ProLayer &L = p.L[g];
    const int local = job - p.job_start[g];
    const int sp = local % p.S, rest = local / p.S;
    const int rt = rest / p.token_tiles, m0 = (rest % p.token_tiles) * 16 * TT;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63, i = l & 15, kb = l >> 4;
    const int j = rt * 16 + i;
    const unsigned mis = (unsigned)(reinterpret_cast<uintptr_t>(L.A) & 2u);
    const rsrc_t ar = make_rsrc(reinterpret_cast<const char *>(L.A) - mis, (unsigned)L.rank * p.K * 2u + mis);
    // (the tokens of this tile behind a descriptor of their own: M * d_in fp16 may pass 4 GiB)
    const _Float16 *x0 = p.x + (size_t)m0 * p.K;
    const unsigned xmis = (unsigned)(reinterpret_cast<uintptr_t>(x0) & 2u);
    const int mrows = min(16 * TT, p.M - m0);
    const rsrc_t xr = make_rsrc(reinterpret_cast<const char *>(x0) - xmis, (unsigned)mrows * p.K * 2u + xmis);

    auto eight = [&](rsrc_t r, unsigned m, unsigned row, int k0, bool ok) __attribute__((always_inline)) {
        const unsigned at = (row * p.K + k0) * 2u + m;
        if (VEC) return __builtin_bit_cast(v8h, buf_load16(r, at, ok && k0 < p.K));
        unsigned d[4];
        const bool whole = ok && k0 + 8 + (int)((at & 2u) >> 1) <= p.K;
        load_unaligned<4>(r, at, whole, d);
        v8h v = __builtin_bit_cast(v8h, (v4u){d[0], d[1], d[2], d[3]});
        if (!whole && ok && k0 < p.K) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = half_bits(buf_load2(r, at + e * 2, k0 + e < p.K));
        }
        return v;
    };

    v4f acc[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) acc[tt] = (v4f){0.f, 0.f, 0.f, 0.f};
    const int all = (p.K + 63) / 64, per = (all + p.S - 1) / p.S, end = min((sp + 1) * per, all);
    constexpr int UN = 4;                           // 64-column steps requested together
    for (int s0 = sp * per + w; s0 < end; s0 += kProWaves * UN) {
        v8h a[UN][2], b[TT][UN][2];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k0 = (s0 + u * kProWaves) * 64 + kb * 16;      // (past d_in: zeros)
            const bool ok = j < L.rank && s0 + u * kProWaves < end;
            a[u][0] = eight(ar, mis, j, k0, ok);
            a[u][1] = eight(ar, mis, j, k0 + 8, ok);
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k0 = (s0 + u * kProWaves) * 64 + kb * 16;
                const bool ok = tt * 16 + i < mrows && s0 + u * kProWaves < end;
                b[tt][u][0] = eight(xr, xmis, tt * 16 + i, k0, ok);
                b[tt][u][1] = eight(xr, xmis, tt * 16 + i, k0 + 8, ok);
            }
        __builtin_amdgcn_sched_barrier(0);          // all requests before the first product waits
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u][0], b[tt][u][0], acc[tt], 0, 0, 0);
                acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u][1], b[tt][u][1], acc[tt], 0, 0, 0);
            }
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) red[w][tt][l] = acc[tt];
    __syncthreads();
    if (w >= TT) return;
    v4f h = red[0][w][l];
#pragma unroll
    for (int s = 1; s < kProWaves; ++s) h += red[s][w][l];
    // element v: rank rt*16 + 4*kb + v of token m0 + 16*w + i.  Ranks past the rank are zeros whatever x holds
    // (their sums are not: zero times an infinity)
    if (w * 16 + i >= mrows) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) h[v] = rt * 16 + 4 * kb + v < L.rank ? h[v] : 0.f;
    const size_t at = (size_t)(m0 + w * 16 + i) * L.hstride + rt * 16 + 4 * kb;
    if (p.S > 1) {
        *reinterpret_cast<v4f *>(L.hpart + (size_t)sp * p.M * L.hstride + at) = h;
    } else {
        v4h o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = (_Float16)silu(h[v]);
        *reinterpret_cast<v4h *>(L.h16 + at) = o;
    }
}

template <int TT, int T, int NU, bool VEC>
__global__ __launch_bounds__(kProThreads) void prologue_kernel(ProParams p)
{
    const int ncorr = p.job_start[p.G];
    if ((int)blockIdx.x < ncorr) {
        corr_tile<TT, VEC>(p, blockIdx.x);
        return;
    }
    const int q = (int)blockIdx.x - ncorr, per_set = (p.M + kProThreads / T - 1) / (kProThreads / T);
    quantize_tokens<T, NU, VEC>(p, p.Q[q / per_set], (q % per_set) * (kProThreads / T));
}

}  // namespace

int prologue_slices(int K) { return (K + 2047) / 2048; }

hipError_t launch_prologue(ProParams &p, hipStream_t st)
{
    p.Kp = round_up(p.K, p.base3 ? kB3Cols : kTileCols);
    // One token tile per workgroup while the workgroups find room side by side (a compute unit takes in 32
    // rows instead of 48: 64 tokens of 4096 columns, 128 ranks: 6.8 us against 8.3), two where there are many
    auto rank_tiles = [&](const ProLayer &L) { return L.rank == 0 ? 0 : (p.by_rows ? L.hstride / 16 : (L.rank + 15) / 16); };
    int tiles = 0;
    for (int g = 0; g < p.G; ++g) tiles += rank_tiles(p.L[g]);
    const int tt = p.M <= 16 || tiles * ((p.M + 15) / 16) * p.S <= 512 ? 1 : 2;
    p.token_tiles = (p.M + 16 * tt - 1) / (16 * tt);
    int jobs = 0;
    bool vec = p.K % 8 == 0 && (reinterpret_cast<uintptr_t>(p.x) % 16) == 0;
    for (int g = 0; g < p.G; ++g) {
        p.job_start[g] = jobs;
        if (p.L[g].rank > 0) {
            jobs += rank_tiles(p.L[g]) * p.token_tiles * p.S;
            vec = vec && (reinterpret_cast<uintptr_t>(p.L[g].A) % 16) == 0;
        }
    }
    p.job_start[p.G] = jobs;
    // threads per token: one 16-column unit each, a wavefront up to 1024 columns, 128 threads up to 2048, 256
    // up to 4096; two units and 512 threads up to 16384, beyond that the row is read once per pass.  (The
    // tokens of a workgroup lie side by side in x_q, so fewer threads per token also store longer pieces)
    const int T = p.Kp <= 1024 ? 64 : (p.Kp <= 2048 ? 128 : (p.Kp <= 4096 ? 256 : 512));
    const int per_wg = kProThreads / T;
    const dim3 grid(jobs + p.NQ * ((p.M + per_wg - 1) / per_wg)), block(kProThreads);
    if (grid.x == 0) return hipSuccess;             // no quantisation (a later launch of the same tokens), no correction path
#define HGF_PRO(TT_, T_, NU_)                                                                               \
    do {                                                                                                    \
        if (vec) hipLaunchKernelGGL((prologue_kernel<TT_, T_, NU_, true>), grid, block, 0, st, p);          \
        else hipLaunchKernelGGL((prologue_kernel<TT_, T_, NU_, false>), grid, block, 0, st, p);             \
    } while (0)
    if (tt == 1) {
        if (T == 64) HGF_PRO(1, 64, 1);
        else if (T == 128) HGF_PRO(1, 128, 1);
        else if (T == 256) HGF_PRO(1, 256, 1);
        else HGF_PRO(1, 512, 2);
    } else {
        if (T == 64) HGF_PRO(2, 64, 1);
        else if (T == 128) HGF_PRO(2, 128, 1);
        else if (T == 256) HGF_PRO(2, 256, 1);
        else HGF_PRO(2, 512, 2);
    }
#undef HGF_PRO
    return hipGetLastError();
}

}  // namespace hgf
