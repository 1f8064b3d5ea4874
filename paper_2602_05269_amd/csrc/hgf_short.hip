// Short rows: a group of layers that read the same activations in ONE launch, every workgroup for itself.
//
// Algorithm 1 of the HGF paper, steps 1-8.  Where rows are short, preparing the tokens (quantising them,
// SiLU(A x)) is less work than handing the result to another launch: a workgroup of eight wavefronts reads
// 8, 16 or 32 tokens, quantises them into LDS (behind a LayerNorm where the layer has one), computes SiLU(A x)
// of them into LDS and contracts, dequantises and gates its row-blocks.  Nothing passes through memory, nothing
// waits for another workgroup.
//
// Bound by latency: a launch (2.7 us in a chain of them), the trip for the tokens, and the instructions of one
// wavefront in between, some 2 ns each.  So a workgroup has as few tokens and row-blocks as leave one workgroup
// per compute unit (plan_short), the tokens and A x are requested before everything else, and what does not
// depend on them (gates) is computed while others wait.  us per call, two launches of the direct path before /
// this one (in a chain of the same call): 256 -> 256 at 8 tokens 6.5 / 5.1; three 512 -> 512 at 24 tokens 7.7 / 5.6,
// behind LayerNorms 8.7 / 6.7, at 500 tokens 13.0 / 10.2; pair 512 -> 1365 at 24 tokens 9.6 / 7.6; 512 -> 64 at 2048
// tokens 10.9 / 5.8.
//
// A x is added up in the order of the direct path's prologue (eight wavefronts, 64 columns each in turn), the
// rest in that of its main kernel: both give the same bits, so a layer's result does not depend on what else is
// in its group.
#include "hgf_internal.h"

namespace hgf {

namespace {

constexpr int kWaves = 8, kThreads = 64 * kWaves;

__device__ __forceinline__ void lds_barrier()
{
    // (not __syncthreads: requests to memory stay in flight across it)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

struct TokenWords {
    float s_x[32];
    int rowsum[32];
};

// Reductions over 2^log neighbouring lanes (16 to 64), with the result in each of them.
__device__ __forceinline__ float lanes_max(float v, int log)
{
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0xB1>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0x4E>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0x141>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<0x140>(__builtin_bit_cast(int, v))));
    if (log > 4) v = fmaxf(v, __shfl_xor(v, 16, 64));
    if (log > 5) v = fmaxf(v, __shfl_xor(v, 32, 64));
    return v;
}
__device__ __forceinline__ int lanes_sum(int v, int log)
{
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    v += dpp_move<0x140>(v);
    if (log > 4) v += __shfl_xor(v, 16, 64);
    if (log > 5) v += __shfl_xor(v, 32, 64);
    return v;
}
template <int CTRL>
__device__ __forceinline__ double dpp_move_d(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_move<CTRL>((int)(unsigned)b), hi = (unsigned)dpp_move<CTRL>((int)(unsigned)(b >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double lanes_sum_d(double v, int log)
{
    v += dpp_move_d<0xB1>(v);
    v += dpp_move_d<0x4E>(v);
    v += dpp_move_d<0x141>(v);
    v += dpp_move_d<0x140>(v);
    if (log > 4) v += __shfl_xor(v, 16, 64);
    if (log > 5) v += __shfl_xor(v, 32, 64);
    return v;
}

// Quantises the workgroup's tokens into LDS: unit u of 16 columns at u * ustride, 16 bytes per token slot.
// 2^plog slots (8 to 32), so 512 >> plog threads of one wavefront per token, NP pieces of 8 columns each, held in registers.
template <int NP, bool LN, bool VEC>
struct Tokens {
    int tlog, tok, t;
    bool live;
    v4u x[NP];
    v4f ga[LN ? NP : 1][2], be[LN ? NP : 1][2];

    __device__ __forceinline__ int column(int u) const { return (t + (u << tlog)) * 8; }
    // (at an odd multiple of two bytes the last dword holds one column more, which has to be the row's too)
    __device__ __forceinline__ bool whole_piece(const ShortParams &p, int col, unsigned at) const
    {
        return live && col + 8 + (int)(at >> 1 & 1u) <= p.K;
    }

    __device__ __forceinline__ void request(const ShortParams &p, const ShortLayer &L, int m0, int tokens)
    {
        tlog = 9 - p.plog;
        tok = threadIdx.x >> tlog;
        t = threadIdx.x & ((1 << tlog) - 1);
        live = tok < tokens;
        const _Float16 *x0 = p.x + (size_t)m0 * p.K;
        const unsigned mis = VEC ? 0u : (unsigned)(reinterpret_cast<uintptr_t>(x0) & 2u);
        const rsrc_t r = make_rsrc(reinterpret_cast<const char *>(x0) - mis, (unsigned)tokens * p.K * 2u + mis);
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int col = column(u);
            const unsigned at = ((unsigned)tok * p.K + col) * 2u + mis;
            if (VEC) {
                x[u] = buf_load16(r, at, live && col < p.K);
            } else {
                // the aligned dwords that hold the eight, shifted together
                const bool whole = whole_piece(p, col, at);
                const unsigned base = whole ? at & ~3u : kOob;
                const v4u d = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)base, 0, 0));
                const unsigned e = buf_load4(r, base + 16u, whole && (at & 2u));
                const unsigned sh = (at & 2u) * 8u;
                x[u] = (v4u){__builtin_amdgcn_alignbit(d[1], d[0], sh), __builtin_amdgcn_alignbit(d[2], d[1], sh),
                             __builtin_amdgcn_alignbit(d[3], d[2], sh), __builtin_amdgcn_alignbit(e, d[3], sh)};
            }
        }
        if (LN) {
            const rsrc_t gr = make_rsrc(L.gamma, (unsigned)p.K * 4u), br = make_rsrc(L.beta, L.beta ? (unsigned)p.K * 4u : 0u);
#pragma unroll
            for (int u = 0; u < NP; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) {       // (a request that runs past the row reads zeros there, element by element)
                    const unsigned at = (unsigned)(column(u) + 4 * h) * 4u;
                    ga[u][h] = __builtin_bit_cast(v4f, buf_load16(gr, at, at + 16u <= (unsigned)p.K * 4u));
                    be[u][h] = __builtin_bit_cast(v4f, buf_load16(br, at, at + 16u <= (unsigned)p.K * 4u));
                }
        }
        if (!VEC) {
            // a row's last columns, one by one
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const int col = column(u);
                if (live && col < p.K && !whole_piece(p, col, ((unsigned)tok * p.K + col) * 2u + mis)) {
                    unsigned short e[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) e[i] = buf_load2(r, ((unsigned)tok * p.K + col + i) * 2u + mis, col + i < p.K);
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[u][i] = e[2 * i] | (unsigned)e[2 * i + 1] << 16;
                }
                if (LN && p.K % 4 != 0) {
                    const rsrc_t gr = make_rsrc(L.gamma, (unsigned)p.K * 4u), br = make_rsrc(L.beta, L.beta ? (unsigned)p.K * 4u : 0u);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int c4 = col + 4 * h;
                        if (c4 < p.K && c4 + 4 > p.K) {
#pragma unroll
                            for (int i = 0; i < 3; ++i) {
                                ga[u][h][i] = __builtin_bit_cast(float, buf_load4(gr, (unsigned)(c4 + i) * 4u, c4 + i < p.K));
                                be[u][h][i] = __builtin_bit_cast(float, buf_load4(br, (unsigned)(c4 + i) * 4u, c4 + i < p.K));
                            }
                        }
                    }
                }
            }
        }
    }

    __device__ __forceinline__ float half_at(int u, int e) const
    {
        return (float)half_bits((unsigned short)(x[u][e >> 1] >> (16 * (e & 1))));
    }

    __device__ __forceinline__ void quantise(const ShortParams &p, const ShortLayer &L, unsigned char *xq, TokenWords &sh)
    {
        float v[LN ? NP : 1][8];
        float amax;
        bool odd = false;
        if (LN) {
            // mean and mean squared deviation in fp64, each rounded once; then fp32 in exactly this order, one
            // rounding each
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < NP; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) s += (double)half_at(u, e);          // (zero past the row)
            const double mean = lanes_sum_d(s, tlog) / (double)p.K;
            double ss = 0.0;
#pragma unroll
            for (int u = 0; u < NP; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const double d = column(u) + e < p.K ? (double)half_at(u, e) - mean : 0.0;
                    ss += d * d;
                }
            const double var = lanes_sum_d(ss, tlog) / (double)p.K;
            const float mu = (float)mean, rstd = (float)(1.0 / sqrt(var + (double)L.eps));
            amax = 0.f;
#pragma unroll
            for (int u = 0; u < NP; ++u)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float y = half_at(u, e) - mu;
                    y = y * rstd;
                    y = y * ga[u][e >> 2][e & 3];
                    y = y + be[u][e >> 2][e & 3];
                    v[u][e] = column(u) + e < p.K ? y : 0.f;
                    amax = fmaxf(amax, fabsf(v[u][e]));
                }
        } else {
            uint32_t mx = 0u;
#pragma unroll
            for (int u = 0; u < NP; ++u) mx = max_magnitudes(x[u], mx);
            odd = __builtin_amdgcn_ballot_w64(odd_magnitudes(mx)) != 0;
            if (odd) {
                amax = 0.f;
#pragma unroll
                for (int u = 0; u < NP; ++u) amax = max_odd(x[u], amax);
            } else {
                amax = larger_magnitude(mx);
            }
        }
        amax = lanes_max(amax, tlog);
        amax = fmaxf(amax, 1e-5f);
        const float inv = 127.0f / amax;
        int sum = 0;
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            uint2 q;
            if (LN) {                               // (the same, of fp32 values, which may pass 127 by a rounding)
                uint32_t w2[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t b[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        b[e] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_fmed3f(v[u][4 * h + e] * inv, -127.0f, 127.0f) + 12582912.0f);
                    w2[h] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u), __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), 0x05040100u);
                    sum = __builtin_amdgcn_sdot4((int)w2[h], 0x01010101, sum, false);
                }
                q = make_uint2(w2[0], w2[1]);
            } else {
                q = eight_codes(x[u], inv, odd, sum);
            }
            const int col = column(u);
            if (col < p.Kp) *reinterpret_cast<uint2 *>(xq + (col >> 4) * p.ustride + tok * 16 + (col & 8)) = q;
        }
        sum = lanes_sum(sum, tlog);
        if (t == 0) {
            sh.s_x[tok] = amax / 127.0f;
            sh.rowsum[tok] = sum;
        }
    }
};

// KS wavefronts share a row-block's k-tiles; 8 / KS row-blocks (PAIR: of each layer) per workgroup.
template <int KS, int NP, int UN, bool PAIR, bool LN, bool VEC>
__global__ __launch_bounds__(kThreads) void short_kernel(ShortParams p)
{
    constexpr int RB = kWaves / KS, NL = PAIR ? 2 : 1;
    constexpr int D = PAIR ? 3 : 4;                           // k-tiles in flight
    constexpr int PPW = KS == 1 ? 4 : (KS == 2 ? 2 : 1);      // quarters of its row-block's tile a wavefront finishes
    constexpr int JP = PAIR ? 2 : 4;                          // 16-rank steps of B requested ahead
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ TokenWords sh;

    const int l = threadIdx.x & 63, jl = l & 31, hf = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = w / KS, ks = w % KS;
    // (all row units of a token group, then the next group: the weights are little and in every L2)
    const int units = p.wg_start[p.G];
    const int group = (int)blockIdx.x / units, u = (int)blockIdx.x - group * units, m0 = group << p.plog;
    const int tokens = min(1 << p.plog, p.M - m0);
    ShortLayer L = p.L[0];
    int u0 = 0;
    if (!PAIR) {
#pragma unroll
        for (int i = 1; i < kMaxGroup; ++i)
            if (i < p.G && u >= p.wg_start[i]) {
                L = p.L[i];
                u0 = p.wg_start[i];
            }
    }
    const ShortLayer &L2 = PAIR ? p.L[1] : L;
    auto layer_of = [&](int g) -> const ShortLayer & { return PAIR && g == 1 ? L2 : L; };
    const int rb = (u - u0) * RB + rg;
    const bool rb_ok = rb < L.RBn;
    const int nb = rb * kTileRows;

    // ---- requests: the tokens first, then what does not depend on them
    Tokens<NP, LN, VEC> tk;
    tk.request(p, L, m0, tokens);
    __builtin_amdgcn_sched_barrier(0);
    // ---- A x: wavefront w takes the 64-column steps w, w + 8, ... of every rank tile and token tile (16 x 16);
    //      lane (i = l % 16, kb = l / 16) holds A[rt*16+i][k] and x[m][k] for the same eight k per MFMA.  The
    //      first step of the first two rank tiles is requested right behind the tokens.
    const int rt0 = (L.rank + 15) / 16, rt1 = PAIR ? (L2.rank + 15) / 16 : 0, RT = rt0 + rt1;
    const int TT = tokens > 16 ? 2 : 1, steps = (p.K + 63) / 64;
    v4f *part = reinterpret_cast<v4f *>(lds + p.part_off);
    const int ai = l & 15, akb = l >> 4;
    const _Float16 *x0 = p.x + (size_t)m0 * p.K;
    const unsigned xmis = VEC ? 0u : (unsigned)(reinterpret_cast<uintptr_t>(x0) & 2u);
    const rsrc_t xr = make_rsrc(reinterpret_cast<const char *>(x0) - xmis, (unsigned)tokens * p.K * 2u + xmis);
    auto eight = [&](rsrc_t r, unsigned mis, unsigned row, int k0, bool ok) __attribute__((always_inline)) {
        const unsigned at = (row * p.K + k0) * 2u + mis;
        if (VEC) return __builtin_bit_cast(v8h, buf_load16(r, at, ok && k0 < p.K));
        const bool whole = ok && k0 + 8 + (int)(at >> 1 & 1u) <= p.K;
        const unsigned base = whole ? at & ~3u : kOob;
        const v4u d = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)base, 0, 0));
        const unsigned e = buf_load4(r, base + 16u, whole && (at & 2u));
        const unsigned s = (at & 2u) * 8u;
        v8h v = __builtin_bit_cast(v8h, (v4u){__builtin_amdgcn_alignbit(d[1], d[0], s), __builtin_amdgcn_alignbit(d[2], d[1], s),
                                              __builtin_amdgcn_alignbit(d[3], d[2], s), __builtin_amdgcn_alignbit(e, d[3], s)});
        if (!whole && ok && k0 < p.K) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = half_bits(buf_load2(r, at + q * 2, k0 + q < p.K));
        }
        return v;
    };
    v8h aa[UN][2][2], ab[UN][2][2];
    auto ax_request = [&](int r0, int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < UN; ++n) {
            const int k0 = (s0 + n * kWaves) * 64 + akb * 16;       // (past d_in: zeros)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const bool second = PAIR && r0 + r >= rt0;
                const ShortLayer &Lr = second ? L2 : L;
                const int row = (r0 + r - (second ? rt0 : 0)) * 16 + ai;
                const unsigned mis = VEC ? 0u : (unsigned)(reinterpret_cast<uintptr_t>(Lr.A) & 2u);
                const rsrc_t ar = make_rsrc(reinterpret_cast<const char *>(Lr.A) - mis, (unsigned)Lr.rank * p.K * 2u + mis);
#pragma unroll
                for (int q = 0; q < 2; ++q) aa[n][r][q] = eight(ar, mis, row, k0 + 8 * q, r0 + r < RT && row < Lr.rank);
            }
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int q = 0; q < 2; ++q) ab[n][tt][q] = eight(xr, xmis, tt * 16 + ai, k0 + 8 * q, tt * 16 + ai < tokens);
        }
    };
    ax_request(0, w);
    __builtin_amdgcn_sched_barrier(0);
    rsrc_t wr[NL];
    v4u wq[D][NL];
#pragma unroll
    for (int g = 0; g < NL; ++g)
        wr[g] = make_rsrc(layer_of(g).packed + (size_t)(rb_ok ? rb : 0) * p.KT * 64, rb_ok ? (unsigned)p.KT * kTileBytes : 0u);
    auto request = [&](int d, int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < NL; ++g) wq[d][g] = buf_load16(wr[g], (unsigned)kt * kTileBytes + l * 16u);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(d, ks + d * KS);
    // the wavefront's rows of B as MFMA operands (rows whose pieces are not aligned are read when they are needed)
    const bool finishes = ks * PPW < 4;
    const int piece0 = ks * PPW & 3;
    v8h bq[NL][JP];
    float s_w[NL], alpha[NL][PPW][4];
    auto b_rsrc = [&](int g) { return make_rsrc(layer_of(g).B, layer_of(g).rank > 0 ? (unsigned)layer_of(g).N * layer_of(g).rank * 2u : 0u); };
    auto b_piece = [&](int g, int js) __attribute__((always_inline)) {
        const ShortLayer &Lg = layer_of(g);
        const int n = nb + jl, j = js * 16 + hf * 8;
        return __builtin_bit_cast(v8h, buf_load16(b_rsrc(g), ((unsigned)n * Lg.rank + j) * 2u, rb_ok && n < Lg.N && j < Lg.rank && Lg.b_aligned));
    };
#pragma unroll
    for (int g = 0; g < NL; ++g) {
        const ShortLayer &Lg = layer_of(g);
#pragma unroll
        for (int js = 0; js < JP; ++js) bq[g][js] = b_piece(g, js);
        const rsrc_t ar = make_rsrc(Lg.alpha, Lg.rank > 0 ? (unsigned)Lg.N * 2u : 0u);
#pragma unroll
        for (int c = 0; c < PPW; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int n = nb + 8 * (piece0 + c) + 4 * hf + v;
                alpha[g][c][v] = (float)half_bits(buf_load2(ar, (unsigned)n * 2u, finishes && n < Lg.N));
            }
        s_w[g] = *Lg.s_w;
    }
    __builtin_amdgcn_sched_barrier(0);

    tk.quantise(p, L, lds, sh);
    for (int r0 = 0; r0 < RT; r0 += 2) {
        v4f ax[2][2];
#pragma unroll
        for (int r = 0; r < 2; ++r) ax[r][0] = ax[r][1] = (v4f){0.f, 0.f, 0.f, 0.f};
        for (int s = w; s < steps; s += UN * kWaves) {
            if (r0 > 0 || s > w) ax_request(r0, s);
#pragma unroll
            for (int n = 0; n < UN; ++n)
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            ax[r][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aa[n][r][q], ab[n][tt][q], ax[r][tt], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
                if (r0 + r < RT && tt < TT) part[(((r0 + r) * TT + tt) * kWaves + w) * 64 + l] = ax[r][tt];
    }
    lds_barrier();

    // ---- SiLU of the sums, in the order of the wavefronts, as MFMA operands of 1 KiB (32 tokens x 16 ranks)
    unsigned char *const hl = lds + p.h_off;
    // (by the last wavefronts, so that those that finish quarters get to their gates meanwhile)
    for (int e = kThreads - 1 - (int)threadIdx.x; e < RT * TT * 64; e += kThreads) {
        const int tile = e >> 6, le = e & 63, r = tile / TT, tt = tile - r * TT;
        v4f h = part[tile * kWaves * 64 + le];
#pragma unroll
        for (int s = 1; s < kWaves; ++s) h += part[(tile * kWaves + s) * 64 + le];
        // element v: rank 16 r + 4 (le / 16) + v of token 16 tt + le % 16; past the rank zeros, whatever x holds
        const bool second = PAIR && r >= rt0;
        const int j = (r - (second ? rt0 : 0)) * 16 + 4 * (le >> 4), rank = second ? L2.rank : L.rank;
        v4h o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = (_Float16)silu(j + v < rank ? h[v] : 0.f);
        *reinterpret_cast<v4h *>(hl + r * 1024 + ((j >> 3 & 1) * 32 + 16 * tt + (le & 15)) * 16 + (j & 4) * 2) = o;
    }

    // ---- the contraction
    v16i acc[NL];
#pragma unroll
    for (int g = 0; g < NL; ++g) acc[g] = (v16i){};
    const unsigned char *xrow = lds + hf * p.ustride + (jl & ((1 << p.plog) - 1)) * 16;   // (slots past the tokens repeat)
    for (int k0 = ks; k0 < p.KT; k0 += D * KS) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int kt = k0 + d * KS;
            if (d > 0 && kt >= p.KT) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4i xv = *reinterpret_cast<const v4i *>(xrow + (kt * 8 + q * 2) * p.ustride);
#pragma unroll
                for (int g = 0; g < NL; ++g)
                    acc[g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(widen_codes(wq[d][g][q]), xv, acc[g], 0, 0, 0);
            }
            request(d, kt + D * KS);
        }
    }
    float gate[NL][PPW][4];
#pragma unroll
    for (int g = 0; g < NL; ++g)
#pragma unroll
        for (int c = 0; c < PPW; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) gate[g][c][v] = tanhf(alpha[g][c][v]);
    v4i *red = reinterpret_cast<v4i *>(lds + p.red_off);
    if (KS > 1) {
#pragma unroll
        for (int g = 0; g < NL; ++g)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                red[((g * kWaves + w) * 4 + c) * 64 + l] = (v4i){acc[g][4 * c], acc[g][4 * c + 1], acc[g][4 * c + 2], acc[g][4 * c + 3]};
    }
    lds_barrier();
    if (!finishes || nb >= L.N) return;

    // ---- correction up-projection, dequantise, gate, store.  Element v of quarter c is row 8c + 4hf + v of the
    //      tile, for the token of the lane.
    const int m = m0 + jl;
    const bool m_ok = jl < tokens;
    v16f corr[NL];
#pragma unroll
    for (int g = 0; g < NL; ++g) {
        const ShortLayer &Lg = layer_of(g);
        corr[g] = (v16f){};
        const unsigned char *hg = hl + (g ? rt0 : 0) * 1024 + l * 16;
#pragma unroll
        for (int js = 0; js < JP; ++js)
            if (Lg.b_aligned && js * 16 < Lg.rank)
                corr[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bq[g][js], *reinterpret_cast<const v8h *>(hg + js * 1024), corr[g], 0, 0, 0);
        for (int js = Lg.b_aligned ? JP : 0; js * 16 < Lg.rank; ++js) {
            const int n = nb + jl, j = js * 16 + hf * 8;
            const v8h b = Lg.b_aligned ? b_piece(g, js) : buf_load8h<false>(b_rsrc(g), (unsigned)n * Lg.rank + j, Lg.rank - j, n < Lg.N);
            corr[g] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, *reinterpret_cast<const v8h *>(hg + js * 1024), corr[g], 0, 0, 0);
        }
    }
    const float s_x = sh.s_x[jl];
    const int rs = sh.rowsum[jl];
    const int N = L.N;
    const bool nvec = N % 4 == 0;
    float zmax = 0.f;
#pragma unroll
    for (int c = 0; c < PPW; ++c) {
        const int q = piece0 + c, n = nb + 8 * q + 4 * hf;
        v4i a[NL];
        float y[NL][4];
#pragma unroll
        for (int g = 0; g < NL; ++g) {
            if (KS == 1) {
                a[g] = (v4i){acc[g][4 * c], acc[g][4 * c + 1], acc[g][4 * c + 2], acc[g][4 * c + 3]};
            } else {
                const v4i *pr = red + ((g * kWaves + rg * KS) * 4 + q) * 64 + l;
                a[g] = pr[0];
#pragma unroll
                for (int o = 1; o < KS; ++o) a[g] += pr[o * 256];
            }
            const float scale = s_x * s_w[g];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                // (a register array cannot be indexed by the wavefront's quarter: one of four is selected)
                const float cv = KS == 1 ? corr[g][4 * c + v]
                                         : (q == 0 ? corr[g][v] : (q == 1 ? corr[g][4 + v] : (q == 2 ? corr[g][8 + v] : corr[g][12 + v])));
                a[g][v] -= rs;
                y[g][v] = (float)a[g][v] * scale + gate[g][c][v] * cv;
            }
        }
        v4h o;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            o[v] = PAIR ? product_half(silu(y[0][v]), y[NL - 1][v]) : (_Float16)y[0][v];
            if (n + v < N) zmax = fmaxf(zmax, fabsf((float)o[v]));
        }
        if (!m_ok) continue;
        _Float16 *const out = PAIR ? L2.y : L.y;
        const size_t at = (size_t)m * N + n;
        if (nvec && n + 3 < N) {
            *reinterpret_cast<v4h *>(out + at) = o;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (n + v < N) out[at + v] = o[v];
        }
#pragma unroll
        for (int g = 0; g < NL; ++g) {
            int32_t *const dbg = layer_of(g).acc_debug;
            if (!dbg) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (n + v < N) dbg[at + v] = a[g][v];
        }
    }
    if (PAIR && p.amax_out) {
        zmax = fmaxf(zmax, __shfl_xor(zmax, 32, 64));
        if (hf == 0 && m_ok) atomicMax(reinterpret_cast<unsigned *>(p.amax_out) + m, __builtin_bit_cast(unsigned, zmax));
    }
}

// Which instantiations plan_short's shapes lead to.  Pieces: the columns of all token slots by 4096.  UN 2: rows beyond
// 512 columns, which are aligned and, behind a LayerNorm, have eight slots and two pieces at most; eight wavefronts
// per row-block have 16 slots at most, one wavefront stands behind a LayerNorm, pairs have two for 256 columns at most.
constexpr bool reached(int KS, int NP, int UN, bool pair, bool ln, bool vec)
{
    if (UN == 2) return vec && (ln ? NP == 2 && KS >= 4 : (KS == 8 && NP >= 2) || (KS == 4 && NP == 4));
    if (ln) return NP == 1 || (NP == 2 && vec && KS < 8);
    return KS == 8 ? NP < 4 : (KS == 4 || (KS == 2 && !(pair && NP == 4)));
}

template <int KS, int NP, int UN, bool PAIR, bool LN, bool VEC>
hipError_t launch_one(const ShortParams &p, size_t lds, hipStream_t st)
{
    if constexpr (reached(KS, NP, UN, PAIR, LN, VEC)) {
        static OncePerDevice once;
        const hipError_t attr = allow_lds(once, reinterpret_cast<const void *>(&short_kernel<KS, NP, UN, PAIR, LN, VEC>), kShortLdsMax);
        if (attr != hipSuccess) return attr;
        hipLaunchKernelGGL((short_kernel<KS, NP, UN, PAIR, LN, VEC>), dim3(p.wg_start[p.G] * p.token_groups), dim3(kThreads), lds, st, p);
        return hipGetLastError();
    } else {
        return hipErrorInvalidConfiguration;
    }
}

template <int KS, int NP, int UN>
hipError_t launch_kind(const ShortParams &p, size_t lds, hipStream_t st)
{
    if (p.pair) return p.vec ? launch_one<KS, NP, UN, true, false, true>(p, lds, st) : launch_one<KS, NP, UN, true, false, false>(p, lds, st);
    if (p.L[0].gamma) return p.vec ? launch_one<KS, NP, UN, false, true, true>(p, lds, st) : launch_one<KS, NP, UN, false, true, false>(p, lds, st);
    return p.vec ? launch_one<KS, NP, UN, false, false, true>(p, lds, st) : launch_one<KS, NP, UN, false, false, false>(p, lds, st);
}
template <int KS, int UN>
hipError_t launch_pieces(const ShortParams &p, size_t lds, hipStream_t st)
{
    const int columns = p.Kp << p.plog;             // of all token slots: 4096 per piece
    if (columns <= 4096) return launch_kind<KS, 1, UN>(p, lds, st);
    if (columns <= 8192) return launch_kind<KS, 2, UN>(p, lds, st);
    return launch_kind<KS, 4, UN>(p, lds, st);
}

}  // namespace

// Fills in the launch shape of a group whose layers, activations and outputs are set.  False: not a group of
// short rows.
bool plan_short(ShortParams &p, size_t *lds_bytes)
{
    p.Kp = round_up(p.K, kTileCols);
    p.KT = p.Kp / kTileCols;
    const bool ln = p.L[0].gamma != nullptr;
    p.vec = p.K % 8 == 0 && (reinterpret_cast<uintptr_t>(p.x) & 15u) == 0;
    int rt = 0;                                     // rank tiles of a workgroup
    for (int g = 0; g < p.G; ++g) {
        ShortLayer &L = p.L[g];
        const int r = (L.rank + 15) / 16;
        rt = p.pair ? rt + r : (r > rt ? r : rt);
        L.b_aligned = L.rank % 8 == 0 && (reinterpret_cast<uintptr_t>(L.B) & 15u) == 0;
        p.vec = p.vec && (L.rank == 0 || (reinterpret_cast<uintptr_t>(L.A) & 15u) == 0);
    }
    // Every workgroup reads all of A and takes two rank tiles at a time, so more ranks or columns are prepared
    // faster by workgroups of their own (us, two launches / one, 24 tokens, 512 rows: 2048 columns 16 ranks 10.2 / 9.1,
    // 32 ranks 10.5 / 10.9, none 7.6 / 6.6; 1024 columns 32 ranks 8.6 / 7.7, 64 ranks 8.9 / 11.0).  Rows at odd
    // addresses take three times the instructions (1365 columns 16 ranks 10.1 / 11.6; 511 8.9 / 7.2; 333 columns
    // behind a LayerNorm, 300 tokens 10.1 / 10.3).
    if (rt > 2 || (rt > 0 ? rt : 1) * p.K > 2048 || (!p.vec && p.K > (ln ? 256 : 512))) return false;
    // What a workgroup prepares and finishes is what it takes, so it has eight tokens of one row-block while that
    // needs no more than a workgroup per compute unit; then 16 tokens, then more row-blocks (512 -> 512, 32 ranks:
    // the shapes 6.2, 6.3, 6.7, 7.1 and 8.0 us at one workgroup per compute unit; with 384 workgroups the first
    // takes 8.6).  Behind a LayerNorm tokens are dear (6.7 with 8, 7.4 with 16, 10.2 with 32).
    // Two launches are as fast or faster (us, they / one) where a workgroup would have eight row-blocks of 32 tokens
    // (129 tokens, two 487 -> 3541 14.7 / 17.5; in the mean 1.01), for pairs of more than 256 columns with four (169 x
    // 286 -> 3674 14.6 / 16.5), behind a LayerNorm of more than 256 columns with eight below 256 tokens (88 x 472 -> 7523
    // 12.6 / 13.5, but three 500 x 512 -> 512 14.8 / 11.9), and where rows of B are read element by element for several
    // row-blocks (17 ranks: 32 tokens, two 536 -> 2940 9.3 / 10.3; 128 x 448 -> 5285 behind a LayerNorm 12.9 / 14.6).
    // (19 000 groups that the rule takes, of 5 to 3000 tokens, timed both ways: 0.80 in the mean, 1.09 at worst.)
    static const signed char plain[][2] = {{3, 8}, {4, 8}, {4, 4}, {5, 4}, {5, 2}}, norm[][2] = {{3, 8}, {3, 4}, {4, 4}, {4, 2}, {4, 1}};
    bool pieces = true;                             // rows of B of more than 16 ranks are whole aligned pieces
    for (int g = 0; g < p.G; ++g) pieces = pieces && (p.L[g].rank <= 16 || p.L[g].b_aligned);
    const bool several = p.K <= 256 || pieces;
    auto row_units = [&]() {                        // workgroups per token group
        int n = 0;
        for (int g = 0; g < (p.pair ? 1 : p.G); ++g) n += (p.L[g].RBn * p.KS + 7) / 8;
        return n;
    };
    bool fits = false;
    for (int i = 0; i < 5 && !fits; ++i) {
        p.plog = ln ? norm[i][0] : plain[i][0];
        p.KS = ln ? norm[i][1] : plain[i][1];
        p.token_groups = (p.M + (1 << p.plog) - 1) >> p.plog;
        fits = p.KT <= 4 * p.KS && (long long)p.Kp << p.plog <= (ln ? 8192 : 16384) &&
               (long long)p.token_groups * row_units() <= 256 && (p.KS == 8 || several) && !(p.pair && p.KS == 2 && p.Kp > 256) &&
               !(ln && p.KS == 1 && p.Kp > 256 && p.M < 256);
    }
    if (!fits) return false;
    const int tt = p.plog > 4 ? 2 : 1, per = 8 / p.KS;
    int units = 0;
    for (int g = 0; g < p.G; ++g) {
        p.wg_start[g] = units;
        if (!p.pair || g == 0) units += (p.L[g].RBn + per - 1) / per;
    }
    for (int g = p.G; g <= kMaxGroup; ++g) p.wg_start[g] = units;
    // bytes between units of 16 columns: the slots and what spreads the quantiser's 8-byte writes over the banks
    const int slots = 1 << p.plog;
    p.ustride = slots * 16 + (slots >= 32 ? 64 : (slots >= 16 ? 32 : 16));
    size_t off = (size_t)(p.Kp / 16) * p.ustride;
    p.part_off = (int)off;
    off += (size_t)rt * tt * kWaves * 1024;
    p.h_off = (int)off;
    off += (size_t)rt * 1024;
    p.red_off = (int)off;
    if (p.KS > 1) off += (size_t)(p.pair ? 2 : 1) * kWaves * 4096;
    *lds_bytes = off;
    return off <= kShortLdsMax;
}

hipError_t launch_short(const ShortParams &p, size_t lds_bytes, hipStream_t st)
{
    const bool one_step = p.K <= 512;               // 64 columns of A x for each of the eight wavefronts
    switch (p.KS) {
        case 1: return launch_pieces<1, 1>(p, lds_bytes, st);      // (four k-tiles and less)
        case 2: return launch_pieces<2, 1>(p, lds_bytes, st);      // (its 32 slots, or 16 behind a LayerNorm, are full at 512)
        case 4: return one_step ? launch_pieces<4, 1>(p, lds_bytes, st) : launch_pieces<4, 2>(p, lds_bytes, st);
        default: return one_step ? launch_pieces<8, 1>(p, lds_bytes, st) : launch_pieces<8, 2>(p, lds_bytes, st);
    }
}

}  // namespace hgf
