// Direct kernel: packed ternary weights x int8 activations, fused with dequantisation, the rank-r
// up-projection and the gate, for token counts whose 256-row prefill tiles would leave the chip idle.
//
// Algorithm 1 of the HGF paper, steps 3, 4, 7 and 8:
//   acc[m,n] = sum_k T[n,k] x_q[m,k]                       (exact int32)
//   y[m,n]   = acc * (s_x[m] s_w) + tanh(alpha[n]) * sum_j B[n,j] h[m,j]
// (the prologue has left x_q, s_x, the row sums and h = SiLU(A x)).
//
// Work split: a workgroup owns WR row-blocks of 32 rows x a group of 32 tokens and all of d_in;
// its KW wavefronts take the k-tiles round-robin and contract them on the 32x32x32 int8 MFMA (weight
// rows = matrix rows, tokens = matrix columns).  Both operands come straight from memory into the
// registers the MFMA reads: a tile of weights is one 16-byte request per lane (widened to int8 with
// a shift and a mask per four codes), and the prologue has stored x_q so that a group's operand for
// 32 columns is one contiguous request too (lanes without a token ask for nothing).  So the main loop
// has no LDS, no barrier and no wait but its own: D tiles are in flight per wavefront, a tile is consumed
// as it lands, the requests past the end are out of range.  The epilogue's operands (B rows, h) go to
// LDS with the first requests, as whole MFMA operands.  At the end the partial tiles meet in LDS and
// every wavefront finishes its share of the rows.  Codes are T+1: the per-token sum of x_q is subtracted once.
//
// Bound by HBM and, for small groups, latency.  Against a kernel that staged whole token rows in LDS
// behind a barrier and let one wavefront finish a row-block (us per launch, 7B-shape down projection at
// 64 tokens: 34.1 before, 13 with the tokens' operand from L2; 2048 -> 8192 twice at 16 tokens: 10.2
// and 7.1).  With the prologue, per pass: 8 up-gate pairs and down projections of the 7B shape at 64
// tokens 653 -> 404 us, 28 layers of d = 512 with LayerNorms at 500 tokens 516 -> 181 us (short rows in one launch).
//
// SwiGLU pair: the "two row-blocks" of a workgroup are the same row-block of the gate and of the up
// projection, so z = SiLU(y_gate) * y_up forms in registers.
#include "hgf_internal.h"

#include <type_traits>

namespace hgf {

namespace {

typedef __attribute__((address_space(3))) void *lds_ptr_t;

constexpr unsigned kOobStep = 0x80000000u;         // stays beyond every descriptor when step offsets are added

// B3: base-3 weights, rows of Kp / 5 bytes (Kp: a multiple of 80).  A k-tile is 32 bytes of every row =
// 160 columns, a lane's 16 bytes are five MFMA operands (digit 0 of its bytes, digit 1, ...), and the
// prologue has stored x_q to match.
// The wavefronts per SIMD that the registers have to leave room for: grids are a few workgroups per compute
// unit, and one more in residence can save a whole round (7B-shape up + gate at 64 tokens, 688 workgroups: 27
// us with room for two per compute unit in registers and in LDS, 23 us with three).
// ONCE: weights are requested as read once (non-temporal), for groups whose weights no second launch or
// token group finds in a cache.
constexpr int direct_waves(int D) { return D == 1 ? 4 : 3; }
template <int WR, int KW, int D, bool PAIR, bool B3 = false, bool ONCE = false>
__global__ __launch_bounds__(64 * KW, direct_waves(D)) void direct_kernel(DecodeParams p)
{
    static_assert(!PAIR || WR == 2, "a pair is one row-block of each layer");
    constexpr int NQ = B3 ? 5 : 4;                            // MFMAs per k-tile
    constexpr int TILES = PAIR ? 1 : WR;                      // output tiles of 32 rows x 32 tokens
    constexpr int PPW = 4 * TILES > KW ? 4 * TILES / KW : 1;  // quarter tiles a wavefront finishes (of one tile)
    static_assert(PPW <= 2, "a wavefront finishes one or two quarters of one tile");
    constexpr int NL = PAIR ? 2 : 1;                          // layers of a finished tile
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const int l = threadIdx.x & 63, jl = l & 31, hf = l >> 5;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Token groups of one row unit are eight workgroups apart, so they run on one XCD and its L2 hands
    // the weights to all of them.
    const int TU = (p.M + 31) / 32;
    const int blk = (int)blockIdx.x / (8 * TU), rem = (int)blockIdx.x % (8 * TU);
    const int u = blk * 8 + rem % 8, m0 = rem / 8 * 32;
    const int tokens = min(32, p.M - m0);
    if (u >= p.wg_start[p.G]) return;
    // this workgroup's layer: every candidate is read at a fixed kernel-argument offset (one batch of
    // scalar loads) and selected, instead of a dependent load at a computed offset
    DecLayer L = p.L[0];
    int u0 = 0;
    if (!PAIR) {
#pragma unroll
        for (int i = 1; i < kMaxGroup; ++i)
            if (i < p.G && u >= p.wg_start[i]) {
                L = p.L[i];
                u0 = p.wg_start[i];
            }
    }
    const DecLayer &L2 = PAIR ? p.L[1] : L;                   // the layer of "row-block 1"
    const int rb0 = PAIR ? u : (u - u0) * WR;
    auto layer_of = [&](int r) -> const DecLayer & { return PAIR && r == 1 ? L2 : L; };
    auto rb_of = [&](int r) { return PAIR ? rb0 : rb0 + r; };

    // ---- the main loop's operands
    rsrc_t wr[WR];
#pragma unroll
    for (int r = 0; r < WR; ++r) {
        const DecLayer &Lr = layer_of(r);
        const bool ok = rb_of(r) < Lr.RBn;
        if (B3) {
            const unsigned row_bytes = (unsigned)p.Kp / 5;
            wr[r] = make_rsrc(reinterpret_cast<const unsigned char *>(Lr.packed) + (size_t)(ok ? rb_of(r) : 0) * kTileRows * row_bytes,
                              ok ? (unsigned)min(kTileRows, Lr.N - rb_of(r) * kTileRows) * row_bytes : 0u);
        } else {
            wr[r] = make_rsrc(Lr.packed + (size_t)(ok ? rb_of(r) : 0) * p.KT * 64, ok ? (unsigned)p.KT * kTileBytes : 0u);
        }
    }
    const rsrc_t xr = make_rsrc(L.xq + (size_t)m0 * p.Kp, (unsigned)tokens * p.Kp);
    const unsigned xstep = (unsigned)tokens * (B3 ? 16u : 32u);   // bytes per MFMA (B3: of one half's tokens)
    const unsigned xoff = jl < tokens ? (unsigned)(hf * (B3 ? NQ : 1) * tokens + jl) * 16u : kOobStep;
    v4u wq[D][WR];
    v4u xq[D][NQ];
    const unsigned woff = B3 ? (unsigned)jl * ((unsigned)p.Kp / 5) + hf * 16u : l * 16u;
    auto request = [&](int d, int kt) __attribute__((always_inline)) {
        // (B3: past the last k-tile lies the next row.  In the last tile the second half may be one too: its
        // digits meet zeros, as x_q ends before)
#pragma unroll
        for (int r = 0; r < WR; ++r)
            wq[d][r] = B3 ? buf_load16(wr[r], (unsigned)kt * 32u + woff, kt < p.KT)
                   : ONCE ? buf_load16_stream(wr[r], (unsigned)kt * kTileBytes + woff)
                          : buf_load16(wr[r], (unsigned)kt * kTileBytes + woff);
#pragma unroll
        for (int q = 0; q < NQ; ++q) xq[d][q] = buf_load16(xr, xoff + (unsigned)(kt * (B3 ? 2 * NQ : NQ) + q) * xstep);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(d, w + d * KW);

    // ---- the epilogue's operands: rows of B and h as MFMA operands of 1 KiB (32 rows x 16 ranks) in LDS,
    //      dealt out over the wavefronts.  Ranks past the rank and rows past the end are zeros.
    //      The same LDS takes the partial tiles at the end, when the corrections have been formed: what a
    //      workgroup holds decides how many of them share a compute unit.
    constexpr int NB = WR;                                    // B blocks, then NL h blocks
    const int NH = p.S > 1 ? 0 : NL;
    const int JS = p.hsteps;                                  // 16-rank steps (of the wider layer of a pair)
    unsigned char *const ops = lds;
    for (int i = w; i < (NB + NH) * JS; i += KW) {
        const int blkno = i / JS, js = i - blkno * JS;
        const int j0 = js * 16 + hf * 8;
        unsigned char *const dst = ops + i * 1024;
        if (blkno < NB) {
            const bool second = blkno > 0;
            const DecLayer &Lr = second ? layer_of(1) : layer_of(0);
            const int n = (second ? rb_of(1) : rb_of(0)) * kTileRows + jl;
            const rsrc_t br = make_rsrc(Lr.B, Lr.rank > 0 ? (unsigned)Lr.N * Lr.rank * 2u : 0u);
            if (Lr.rank % 8 == 0 && Lr.b_aligned) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(br, (lds_ptr_t)dst, 16,
                                                         (int)(n < Lr.N && j0 < Lr.rank ? ((unsigned)n * Lr.rank + j0) * 2u : kOob), 0, 0, 0);
            } else {
                *reinterpret_cast<v8h *>(dst + l * 16) = buf_load8h<false>(br, (unsigned)n * Lr.rank + j0, Lr.rank - j0, n < Lr.N);
            }
        } else {
            const int m = m0 + jl;
            const DecLayer &Lr = blkno - NB > 0 ? layer_of(1) : layer_of(0);
            const rsrc_t hr = make_rsrc(Lr.h16, Lr.rank > 0 ? (unsigned)p.M * Lr.hstride * 2u : 0u);
            // (the prologue writes whole tiles of 16 ranks)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(hr, (lds_ptr_t)dst, 16,
                                                     (int)(m < p.M && js * 16 < Lr.rank ? ((unsigned)m * Lr.hstride + j0) * 2u : kOob), 0, 0, 0);
        }
    }
    // h from its slices (long d_in): a thread takes quadruples of ranks of one token, adds their slices in
    // order, SiLU, one fp16 rounding; as many quadruples at a time as eight requests allow
    auto stage_slices = [&](auto hs_) __attribute__((always_inline)) {
        constexpr int HS = decltype(hs_)::value, HV = 8 / HS;
#pragma unroll
        for (int g = 0; g < NL; ++g) {
            const DecLayer &Lg = layer_of(g);
            const int width = (Lg.rank + 15) / 16 * 4;        // quadruples per token (whole tiles of 16 ranks)
            const int quads = width * tokens;
            const unsigned slice = (unsigned)p.M * Lg.hstride * 4u;
            const rsrc_t hr = make_rsrc(Lg.hpart, Lg.rank > 0 ? (unsigned)p.S * slice : 0u);
            for (int i0 = threadIdx.x; i0 < quads; i0 += 64 * KW * HV) {
                v4f part[HV][HS];
                int tok[HV], j[HV];
#pragma unroll
                for (int v = 0; v < HV; ++v) {
                    const int i = i0 + v * 64 * KW;
                    tok[v] = i / width;
                    j[v] = (i - tok[v] * width) * 4;
#pragma unroll
                    for (int s = 0; s < HS; ++s)
                        part[v][s] = __builtin_bit_cast(v4f, buf_load16(hr, ((unsigned)(m0 + tok[v]) * Lg.hstride + j[v]) * 4u + s * slice,
                                                                        i < quads && s < p.S));
                }
#pragma unroll
                for (int v = 0; v < HV; ++v) {
                    v4f h = part[v][0];
#pragma unroll
                    for (int s = 1; s < HS; ++s) h += part[v][s];
                    for (int s = HS; s < p.S; ++s)
                        h += __builtin_bit_cast(v4f, buf_load16(hr, ((unsigned)(m0 + tok[v]) * Lg.hstride + j[v]) * 4u + s * slice,
                                                                i0 + v * 64 * KW < quads));
                    v4h o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (_Float16)silu(h[e]);
                    if (i0 + v * 64 * KW < quads)
                        *reinterpret_cast<v4h *>(ops + ((NB + g) * JS + (j[v] >> 4)) * 1024 +
                                                 ((j[v] >> 3 & 1) * 32 + tok[v]) * 16 + (j[v] & 4) * 2) = o;
                }
            }
        }
    };
    if (p.S > 4) stage_slices(std::integral_constant<int, 8>{});
    else if (p.S > 2) stage_slices(std::integral_constant<int, 4>{});
    else if (p.S > 1) stage_slices(std::integral_constant<int, 2>{});

    // what this wavefront finishes: quarters piece0 .. of row-block rt's tile
    const bool finishes = w * PPW < 4 * TILES;
    const int rt = finishes && !PAIR ? w * PPW / 4 : 0, piece0 = finishes ? w * PPW % 4 : 0;
    const int m = m0 + jl;
    const bool m_ok = m < p.M;
    const int nb = (PAIR ? rb0 : rb0 + rt) * kTileRows;       // first row of the tile
    float s_w[NL], alpha[NL][PPW][4];
#pragma unroll
    for (int g = 0; g < NL; ++g) {
        const DecLayer &Lg = layer_of(g);
        s_w[g] = *Lg.s_w;
        const rsrc_t ar = make_rsrc(Lg.alpha, Lg.rank > 0 ? (unsigned)Lg.N * 2u : 0u);
#pragma unroll
        for (int c = 0; c < PPW; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int n = nb + 8 * (piece0 + c) + 4 * hf + v;
                alpha[g][c][v] = (float)half_bits(buf_load2(ar, (unsigned)n * 2u, finishes && n < Lg.N));
            }
    }
    const float s_x = __builtin_bit_cast(float, buf_load4(make_rsrc(L.s_x, (unsigned)p.M * 4u), (unsigned)m * 4u, m_ok));
    const int rs = (int)buf_load4(make_rsrc(L.rowsum, (unsigned)p.M * 4u), (unsigned)m * 4u, m_ok);

    // ---- the contraction
    v16i acc[WR];
#pragma unroll
    for (int r = 0; r < WR; ++r) acc[r] = (v16i){};
    for (int k0 = w; k0 < p.KT; k0 += D * KW) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (d > 0 && k0 + d * KW >= p.KT) break;
            v4i digit[WR][5];
            if constexpr (B3) {
#pragma unroll
                for (int r = 0; r < WR; ++r) base3_digits(wq[d][r], digit[r]);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
#pragma unroll
                for (int r = 0; r < WR; ++r) {
                    const v4i a = B3 ? digit[r][q] : widen_codes(wq[d][r][q & 3]);
                    acc[r] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, __builtin_bit_cast(v4i, xq[d][q]), acc[r], 0, 0, 0);
                }
            }
            request(d, k0 + (d + D) * KW);
        }
    }

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");          // this wavefront's operands are in LDS
    __syncthreads();
    // ---- correction up-projection: corr[n,m] = sum_j B[n,j] h[m,j] on the f16 MFMA, of which the wavefront
    //      keeps the quarters it finishes (a register array cannot be indexed by them: one of four is selected)
    float cv[NL][PPW][4];
#pragma unroll
    for (int g = 0; g < NL; ++g) {
        v16f corr = {};
        const DecLayer &Lg = layer_of(g);
        if (finishes)
            for (int js = 0; js * 16 < Lg.rank; ++js) {
                const v8h b = *reinterpret_cast<const v8h *>(ops + ((PAIR ? g : rt) * JS + js) * 1024 + l * 16);
                const v8h h = *reinterpret_cast<const v8h *>(ops + ((NB + g) * JS + js) * 1024 + l * 16);
                corr = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, h, corr, 0, 0, 0);
            }
#pragma unroll
        for (int c = 0; c < PPW; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int q = piece0 + c;
                cv[g][c][v] = q == 0 ? corr[v] : (q == 1 ? corr[4 + v] : (q == 2 ? corr[8 + v] : corr[12 + v]));
            }
    }
    __syncthreads();                                          // everyone has read the operands

    // ---- the KW partial tiles meet in LDS (a tile as four pieces of 16 bytes per lane, piece by piece
    //      across the lanes: no bank conflicts)
    v4i *red = reinterpret_cast<v4i *>(lds);
#pragma unroll
    for (int r = 0; r < WR; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            red[((r * KW + w) * 4 + c) * 64 + l] = (v4i){acc[r][4 * c], acc[r][4 * c + 1], acc[r][4 * c + 2], acc[r][4 * c + 3]};
    __syncthreads();
    if (!finishes || nb >= L.N) return;

    // ---- dequantise, gate, store.  Element v of quarter c is row 8c + 4hf + v of the tile, for the
    //      token of the lane.
    const int N = L.N;
    const bool nvec = N % 4 == 0;
    float zmax = 0.f;
#pragma unroll
    for (int c = 0; c < PPW; ++c) {
        const int n = nb + 8 * (piece0 + c) + 4 * hf;
        v4i a[NL];
        float y[NL][4];
#pragma unroll
        for (int g = 0; g < NL; ++g) {
            const v4i *part = red + ((PAIR ? g : rt) * KW * 4 + piece0 + c) * 64 + l;
            a[g] = part[0];
#pragma unroll
            for (int o = 1; o < KW; ++o) a[g] += part[o * 256];
            const float scale = s_x * s_w[g];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                a[g][v] -= rs;
                y[g][v] = (float)a[g][v] * scale + tanhf(alpha[g][c][v]) * cv[g][c][v];
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
        // per token: the larger of the two lanes that hold its rows, then one atomic (non-negative
        // floats order like their bit patterns)
        zmax = fmaxf(zmax, __shfl_xor(zmax, 32, 64));
        if (hf == 0 && m_ok) atomicMax(reinterpret_cast<unsigned *>(p.amax_out) + m, __builtin_bit_cast(unsigned, zmax));
    }
}

template <int WR, int KW, int D, bool PAIR, bool B3 = false, bool ONCE = false>
hipError_t launch_shape(DecodeParams &p, hipStream_t st)
{
    int units = 0;
    for (int g = 0; g < p.G; ++g) {
        p.wg_start[g] = units;
        if (!PAIR || g == 0) units += PAIR ? p.L[g].RBn : (p.L[g].RBn + WR - 1) / WR;
    }
    for (int g = p.G; g <= kMaxGroup; ++g) p.wg_start[g] = units;
    const size_t red = (size_t)KW * WR * 4096, ops = (size_t)(WR + (PAIR ? 2 : 1)) * p.hsteps * 1024;
    const size_t lds = red > ops ? red : ops;
    static OncePerDevice once;
    const hipError_t attr = allow_lds(once, reinterpret_cast<const void *>(&direct_kernel<WR, KW, D, PAIR, B3, ONCE>), 160 * 1024);
    if (attr != hipSuccess) return attr;
    const int TU = (p.M + 31) / 32;
    hipLaunchKernelGGL((direct_kernel<WR, KW, D, PAIR, B3, ONCE>), dim3((units + 7) / 8 * 8 * TU), dim3(64 * KW), lds, st, p);
    return hipGetLastError();
}

}  // namespace

// Fills in the launch shape of a group whose layers, activations and outputs are set.
hipError_t launch_decode(DecodeParams &p, int d_in, hipStream_t st)
{
    p.Kp = round_up(d_in, p.base3 ? kB3Cols : kTileCols);
    p.KT = p.base3 ? (p.Kp + 2 * kB3Cols - 1) / (2 * kB3Cols) : p.Kp / kTileCols;
    p.hsteps = 0;
    int rbs = 0;
    for (int g = 0; g < p.G; ++g) {
        DecLayer &L = p.L[g];
        rbs += L.RBn;
        L.b_aligned = (reinterpret_cast<uintptr_t>(L.B) & 15u) == 0;
        if ((L.rank + 15) / 16 > p.hsteps) p.hsteps = (L.rank + 15) / 16;
    }
    // The shape: row-blocks of a workgroup, wavefronts, tiles in flight.  `tiles` output tiles of 32 x 32 are
    // dealt out to 256 compute units, so few tiles want many wavefronts along d_in and many tiles want a
    // workgroup that reads its tokens for two of them (us per group of layers, both launches: 7B-shape down,
    // 86 k-tiles, 128 tiles: 15.9 with eight wavefronts, 16.7 with four; 2048 -> 2048, 16 k-tiles, 64 tiles: 11.9
    // and 11.6; 7B-shape up + gate at 64 tokens, 1376 tiles: 35.0 for one row-block per workgroup, 30.7 for
    // two; 7B-shape down at 128 tokens, 512 tiles: two row-blocks with eight wavefronts 24.7, four wavefronts
    // 27.0; at 256 tokens 42.7 and 39.8).
    // (base-3, 344 row-blocks of 4096 columns: two k-tiles in flight 10.6, four 11.2; eight wavefronts 11.0)
    if (p.base3) return launch_shape<1, 4, 2, false, true>(p, st);
    const int groups = (p.M + 31) / 32, tiles = rbs * groups;
    if (p.pair) {
        if (p.G != 2 || p.L[0].N != p.L[1].N) return hipErrorInvalidValue;
        // (7B-shape, 344 row-blocks at 8 tokens: four wavefronts 21.6, eight 26.4; 512 -> 1365, 43: 10.7 and 10.4)
        // (one token group: the weights are the traffic, see below.  7B-shape at 4 tokens 21.4 with three tiles in
        // flight, 20.1 with two and read-once requests; 4096 -> 14336 at 5 tokens 20.9 and 19.6; with 256 row-blocks
        // of 16 k-tiles 13.3 and 13.7)
        if (groups == 1 && tiles > 512) return launch_shape<2, 4, 2, true, false, true>(p, st);
        return tiles > 512 ? launch_shape<2, 4, 3, true>(p, st) : launch_shape<2, 8, 3, true>(p, st);
    }
    // One token group: hardly anything but weights is read, so with many row-blocks what counts is how many
    // wavefronts are in flight, not how deep each reads ahead, and with many bytes that they are requested as
    // read once.  (us per pass, both launches, up to 350 MB of weights in turn, 5 .. 32 tokens; geometric mean
    // against the best of sixteen shapes, this one / four tiles in flight: up to 8 k-tiles and 1300
    // row-blocks 1.02 / 1.17; 9 to 24 and 257 to 800 1.01 / 1.07; longer and 513 to 800 1.02 / 1.08; up to
    // 1050 1.01 / 1.23; beyond 1.03 / 1.33.  Up + gate of the 7B shape, 688 row-blocks, 5 tokens: 19.8 -> 18.5,
    // without the read-once requests 19.0; three such layers 25.5 -> 22.4; 512 -> 32000 12.3 -> 9.6.)
    if (groups == 1) {
        if (p.KT >= 32 && tiles <= 256) return launch_shape<1, 8, 3, false>(p, st);
        if (p.KT > 8 && tiles <= (p.KT > 24 ? 512 : 256)) return launch_shape<1, 4, 4, false>(p, st);
        if (tiles <= (p.KT <= 8 ? 1300 : 800))
            return p.KT <= 24 ? launch_shape<1, 4, 1, false>(p, st) : launch_shape<1, 4, 1, false, false, true>(p, st);
        if (tiles <= 1050) return launch_shape<2, 4, 2, false, false, true>(p, st);
        return p.KT <= 4 ? launch_shape<2, 4, 1, false>(p, st) : launch_shape<2, 4, 1, false, false, true>(p, st);
    }
    if (tiles <= 256)
        return p.KT >= 32 ? launch_shape<1, 8, 3, false>(p, st) : launch_shape<1, 4, 4, false>(p, st);
    if (tiles <= 640) return launch_shape<2, 8, 3, false>(p, st);
    // (a wavefront with one k-tile has nothing to keep in flight behind it: registers for four workgroups
    // per compute unit instead of two, 1024 of them in one round.  2048 tiles of four k-tiles: 8.7 us, where
    // four in flight took 12.2)
    return p.KT <= 4 ? launch_shape<2, 4, 1, false>(p, st) : launch_shape<2, 4, 3, false>(p, st);
}

}  // namespace hgf
