// A list of layers for 5 to 16 tokens in ONE launch: a queue of tasks that the workgroups take in order.
//
// Algorithm 1 of the HGF paper, steps 1-8, phase by phase; a phase is a group of up to four layers that read the
// same activations.  Its tasks come in two kinds:
//
//   jobs   two tiles of 16 ranks by the tokens of A x over a slice of d_in (step 5), one for each half of the
//          workgroup's sixteen wavefronts; the fp32 sums go to an exchange region in the workspace
//   units  up to four row-blocks of 32 rows: the workgroup quantises the tokens into LDS for itself (steps 1-2),
//          contracts (step 3), collects the slices of A x, applies SiLU (step 6) and finishes its rows (steps 4, 7, 8)
//
// A workgroup takes the next task from a counter, so tasks begin in order, and a task waits only for tasks
// before it, which by then run or are done: the launch comes to its end however few of its workgroups the
// device holds at a time, whatever else runs.  (Every wait is bounded all the same.  On expiry the sticky word of
// the workspace is set, the workgroup's outputs from there on are NaN, its sums of A x too, and its tasks' words say
// so: who reads them gives up as well, as a NaN among the tokens alone would be lost in the quantiser.)
//
// Bound by latency: wavefronts spend 65 % (7B shape, 8 tokens) to 75 % (1.2B shape, 16) of their time at waits and
// barriers, 21 and 13 % ready and waiting to issue, 14 and 12 % issuing (shader counters).  A phase is a hop through
// memory (the last store to the next phase's tokens, 2 us), the tokens' trip and quantiser (2.5; its 4.5 instructions
// per element are the same in every workgroup, 5 to 7 for rows of 8192 and 11008 columns), contraction (0.5 to 1.5),
// and, beside these, A x and its exchange (5), then the finish (1.5).  Weights, gates and rows of A are asked for
// before the tokens are there.
// Two launches per group were bound by the launches (2.7 us each in a chain) and the same trips.  us per pass,
// before / now: twelve 1.2B-shape layers (48 groups) at 16 tokens 694 / 453, eight 7B-shape FFN blocks (16 groups) at
// 8 tokens 288 / 221; one such layer alone, its weights in cache, 47.2 / 55.0: a launch begins with
// 8 us that nothing hides (kBatchMinPhases).  The gain is the weights' trip from memory and phases that do not wait for
// each other; a chain of groups whose weights caches hold is left to two launches each (hgf_stack_forward).
// Beyond 16 tokens rows of 8192 columns do not fit LDS, and quantising them in every workgroup costs more than the
// launch (24 tokens, 2048 columns and up: 318 / 355), so there it stays two launches; so does a single group (2048 ->
// 2048 at 16 tokens 11.8 / 15.6).
//
// Hand-over.  Sums of A x: the region holds a sentinel (all ones) wherever nothing has been written; readers
// re-read with device scope until no word is the sentinel.  The two sets of regions are those of the whole-stack
// launch (lists of up to 4 tokens), under its protocol: they alternate by one launch counter, and each launch refills
// what the one before it used of the other.  Outputs of a layer: besides the caller's slot they go, with
// device scope, to a copy in the workspace, then the task's word is set; readers wait for
// the words of all tasks of the phase and then read the copy through their L2, as often as they like: its lines are
// written once in a launch, each by one workgroup (a row-block's outputs are whole lines: the copies begin at a
// multiple of 256 bytes wherever the workspace does), and nobody has read them before.
#include "hgf_internal.h"

#include <type_traits>

namespace hgf {

namespace {

constexpr int kWaves = 16, kThreads = 64 * kWaves;
constexpr unsigned kSentinel = 0xFFFFFFFFu;
constexpr unsigned kDone = 1, kVoid = 2;   // a task's word: outputs are there; a wait has expired before them
constexpr int kPolls = 1 << 18;        // bound of a wait for another workgroup (about a second; hgf_set_wait_limit)
constexpr int kD = 8;                  // weight tiles in flight per wavefront
constexpr size_t kLdsMax = 154 * 1024;   // (of 160 KiB; the words and the launch's description are static)

typedef unsigned int v2u __attribute__((ext_vector_type(2)));

// bytes between units of 16 columns: the slots and what spreads the quantiser's 8-byte writes over the banks
__host__ __device__ constexpr int unit_stride(int slots) { return slots * 16 + (slots >= 16 ? 32 : 16); }

struct Words {                         // LDS
    int ticket, epoch, failed;
    unsigned act_used, mail_used;      // of the other set
    float amax[kWaves];
    int sum[kWaves];
    float s_x[32];
    int rowsum[32];
    float s_w[4];
    alignas(16) float gate[128];       // of the units' rows
};

static_assert(kLdsMax + sizeof(Words) + sizeof(BatchParams) <= 160 * 1024, "a compute unit's LDS");

__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
__device__ __forceinline__ v4u load16_agent(rsrc_t r, unsigned off, bool ok = true)
{
    return __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(ok ? off : kOob), 0, 16));
}
__device__ __forceinline__ bool has_sentinel(v4u v)
{
    return v[0] == kSentinel || v[1] == kSentinel || v[2] == kSentinel || v[3] == kSentinel;
}
// Where the tokens of a phase are: the caller's rows, or the copy that earlier tasks have made of their
// outputs, [row-block][tokens, padded to even][32 rows].
struct Source {
    rsrc_t r;
    unsigned base, tstride, bstride;   // bytes: of the whole; from token to token; from 32 columns to the next 32
    __device__ __forceinline__ unsigned at(int tok, int col) const
    {
        return base + (unsigned)tok * tstride + (unsigned)(col >> 5) * bstride + (unsigned)(col & 31) * 2u;
    }
};

// Quantises the tokens (Sec. 2.2.1) into LDS: unit u of 16 columns at u * ustride, 16 bytes per token slot.  SL
// slots, so 1024 / SL threads per token, NP pieces of 8 columns each.
// CH times NP pieces: with two, the first ones are read again (through the L2) instead of held.
template <int SL, int NP, int CH>
__device__ __forceinline__ void quantise_tokens(const Source &S, int tx, int M, int K, int Kp, int ustride, unsigned char *xq, Words &sh)
{
    constexpr int T = kThreads / SL, LOG = T == 128 ? 7 : 6;
    const int tok = tx >> LOG, t = tx & (T - 1), l = tx & 63;
    const int w = __builtin_amdgcn_readfirstlane(tx >> 6);
    v4u x[NP];
    auto load = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int col = (t + (c * NP + u) * T) * 8;
            x[u] = buf_load16(S.r, S.at(tok, col), tok < M && col < K);
        }
    };
    bool odd = false;
    float amax = 0.f;
#pragma unroll
    for (int c = CH - 1; c >= 0; --c) {
        load(c);
        uint32_t mx = 0u;
#pragma unroll
        for (int u = 0; u < NP; ++u) mx = max_magnitudes(x[u], mx);
        if (__builtin_amdgcn_ballot_w64(odd_magnitudes(mx)) != 0) {
            odd = true;
#pragma unroll
            for (int u = 0; u < NP; ++u) amax = max_odd(x[u], amax);
        } else {
            amax = fmaxf(amax, larger_magnitude(mx));
        }
    }
    auto fmax_dpp = [&](int moved) { amax = fmaxf(amax, __builtin_bit_cast(float, moved)); };
    fmax_dpp(dpp_move<0xB1>(__builtin_bit_cast(int, amax)));
    fmax_dpp(dpp_move<0x4E>(__builtin_bit_cast(int, amax)));
    fmax_dpp(dpp_move<0x141>(__builtin_bit_cast(int, amax)));
    fmax_dpp(dpp_move<0x140>(__builtin_bit_cast(int, amax)));
    amax = fmaxf(amax, __shfl_xor(amax, 16, 64));
    amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
    if (T == 128) {                                 // two wavefronts share a token
        if (l == 0) sh.amax[w] = amax;
        lds_barrier();
        amax = fmaxf(amax, sh.amax[w ^ 1]);
    }
    amax = fmaxf(amax, 1e-5f);
    const float inv = 127.0f / amax;
    int sum = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        if (c > 0) load(c);
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const uint2 q = eight_codes(x[u], inv, odd, sum);
            const int col = (t + (c * NP + u) * T) * 8;
            if (col < Kp) *reinterpret_cast<uint2 *>(xq + (col >> 4) * ustride + tok * 16 + (col & 8)) = q;
        }
    }
    sum += dpp_move<0xB1>(sum);
    sum += dpp_move<0x4E>(sum);
    sum += dpp_move<0x141>(sum);
    sum += dpp_move<0x140>(sum);
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (T == 128) {
        if (l == 0) sh.sum[w] = sum;                // (added by who reads them, behind the next barrier)
        if (t == 0) sh.s_x[tok] = amax / 127.0f;
    } else if (t == 0) {
        sh.s_x[tok] = amax / 127.0f;
        sh.rowsum[tok] = sum;
    }
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <class T>
__device__ __forceinline__ T *uniform(T *v)
{
    const uint64_t b = reinterpret_cast<uint64_t>(v);
    return reinterpret_cast<T *>((uint64_t)(unsigned)uniform((int)(b >> 32)) << 32 | (unsigned)uniform((int)b));
}
// SiLU(A x) of four ranks per thread, the slices in order, into LDS as MFMA operands of 1 KiB (32 tokens x 16
// ranks); `first` and `step`: this thread among those that do it.  False: a wait has expired.
__device__ __forceinline__ bool gather_layer(const BatchLayer &LL, int first, int step, rsrc_t mail, int S, int M, int polls_max, bool given_up, unsigned char *hl)
{
    const int rank = uniform(LL.rank), hs = h_stride(rank), width = (rank + 15) / 16 * 4;
    const unsigned mail_off = (unsigned)uniform((int)LL.mail_off), slice = (unsigned)M * hs * 4u;
    bool late = given_up;
#pragma clang loop unroll(disable)
    for (int e = first; e < M * width; e += step) {
        const int tok = e / width, j = (e - tok * width) * 4;
        const unsigned at = mail_off + (unsigned)(tok * hs + j) * 4u;
        v4f part[kBatchSlices];
        int polls = 0;
#pragma clang loop unroll(disable)
        while (true) {
            bool ready = true;
#pragma unroll
            for (int s = 0; s < kBatchSlices; ++s) {
                const v4u raw = load16_agent(mail, at + (unsigned)s * slice, s < S);
                ready = ready && !has_sentinel(raw);
                part[s] = __builtin_bit_cast(v4f, raw);
            }
            if (ready || late) break;
            if (++polls >= polls_max) late = true;
            __builtin_amdgcn_s_sleep(1);
        }
        v4f h = part[0];
#pragma unroll
        for (int s = 1; s < kBatchSlices; ++s) h += part[s];
        v4h o;
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = (_Float16)silu(j + v < rank ? h[v] : 0.f);
        *reinterpret_cast<v4h *>(hl + (j >> 4) * 1024 + ((j >> 3 & 1) * 32 + tok) * 16 + (j & 4) * 2) = o;
    }
    return !late;
}

template <int SL>
__global__ __launch_bounds__(kThreads) void batch_kernel(const BatchParams p)
{
    constexpr int CO = 16;                                    // token columns of a finished tile
    constexpr int ustride = unit_stride(SL);
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ Words sh;
    __shared__ __attribute__((aligned(16))) unsigned char image[sizeof(BatchParams)];   // the launch's description: reads
                                                              // at offsets that depend on each other cost a tenth here
    const BatchParams &D = *reinterpret_cast<const BatchParams *>(image);
    const int M = p.M;

    for (unsigned e = threadIdx.x; e < sizeof(BatchParams) / 4; e += kThreads)
        reinterpret_cast<uint32_t *>(image)[e] =
            ((const __attribute__((address_space(4))) uint32_t *)__builtin_amdgcn_kernarg_segment_ptr())[e];
    if (threadIdx.x == 0) {
        sh.ticket = __hip_atomic_fetch_add(p.flags + 11, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.epoch = __hip_atomic_load(p.flags + 4, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.act_used = (unsigned)__hip_atomic_load(p.flags + 6, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.mail_used = (unsigned)__hip_atomic_load(p.flags + 7, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh.failed = 0;
    }
    lds_barrier();
    const unsigned epoch = (unsigned)uniform(sh.epoch);
    unsigned char *const mine = p.xchg + (size_t)(epoch & 1u) * kStackSetBytes, *const words = mine + kStackActBytes;
    const rsrc_t mail = make_rsrc(mine + kStackActBytes, (unsigned)kBatchMailBytes),
                 act = make_rsrc(mine + p.act_shift, (unsigned)kBatchActBytes);
    {   // this workgroup's share of what the launch before used of the other set
        unsigned char *const other = p.xchg + (size_t)((epoch & 1u) ^ 1u) * kStackSetBytes;
        const unsigned used[2] = {(unsigned)uniform((int)sh.act_used), (unsigned)uniform((int)sh.mail_used)};
        const v4u s4 = {kSentinel, kSentinel, kSentinel, kSentinel};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const rsrc_t r = make_rsrc(other + i * kStackActBytes, used[i]);
            for (unsigned v = blockIdx.x * kThreads + threadIdx.x; v < used[i] / 16u; v += gridDim.x * kThreads)
                __builtin_amdgcn_raw_buffer_store_b128(s4, r, (int)(v * 16u), 0, 16);
        }
    }
    int ph = 0;
    bool failed = false;

    while (true) {
        // (the thread's number anew for every task: what follows from it is computed where it is needed, not carried
        // through all of them in registers)
        int tx = threadIdx.x;
        asm volatile("" : "+v"(tx));
        const int l = tx & 63, jl = l & 31, hf = l >> 5;
        const int w = uniform(tx >> 6);
        const int ticket = uniform(sh.ticket);
        if (ticket >= p.tasks) break;
        while (ph + 1 < p.nphases && ticket >= uniform(D.ph[ph + 1].task0)) ++ph;
        const BatchPhase &P = D.ph[ph];
        const int K = uniform(P.K), first = uniform((int)P.first_layer), upt = uniform((int)P.upt), jobs = uniform(P.jobs), S = uniform((int)P.S);
        const int src_phase = uniform((int)P.src_phase);
        const int KT = (K + kTileCols - 1) / kTileCols, Kp = KT * kTileCols;
        const int local = ticket - uniform(P.task0), jtasks = (jobs + 1) / 2;

        Source src;
        if (src_phase < 0) {
            src.r = make_rsrc(uniform(P.x_ext), (unsigned)M * K * 2u);
            src.base = 0u;
            src.tstride = (unsigned)K * 2u;
            src.bstride = 64u;
        } else {
            src.r = act;
            src.base = (unsigned)uniform((int)P.src_off);
            src.tstride = 64u;
            src.bstride = (unsigned)(M + (M & 1)) * 64u;
        }
        // waits for the words of all unit tasks of the phase that makes the tokens
        auto tokens_ready = [&]() __attribute__((always_inline)) {
            if (src_phase < 0) return;
            if (w == 0) {
                const int n = uniform(D.ph[src_phase].unit_tasks);
                const rsrc_t wd = make_rsrc(words + src_phase * kBatchPhaseWords, (unsigned)n * 4u);
                int polls = 0;
#pragma clang loop unroll(disable)
                while (!failed) {
                    const v4u a = load16_agent(wd, (unsigned)l * 16u), b = n > 256 ? load16_agent(wd, 1024u + (unsigned)l * 16u) : a;
                    unsigned worst = 0u;                      // (past the last word lie zeros; the sentinel is the largest)
#pragma unroll
                    for (int e = 0; e < 4; ++e) worst = max(worst, max(a[e], b[e]));
                    if (__builtin_amdgcn_ballot_w64(worst > kVoid) == 0) {
                        failed = __builtin_amdgcn_ballot_w64(worst == kVoid) != 0;
                        break;
                    }
                    if (++polls >= p.polls) failed = true;
                    __builtin_amdgcn_s_sleep(1);
                }
                if (failed && l == 0) {
                    sh.failed = 1;
                    __hip_atomic_store(p.flags + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            lds_barrier();
        };
        int next = 0;                                         // (thread 0) the next task
        auto take_next = [&]() __attribute__((always_inline)) {
            if (tx == 0) next = __hip_atomic_fetch_add(p.flags + 11, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };

        if (local < jtasks) {
            // ---- two tiles of A x.  Half h of the wavefronts: wavefront i of eight takes the 64-column steps i, i + 8,
            //      ... of the slice; lane (i = l % 16, kb = l / 16) holds A[rt*16+i][k] and x[m][k] for the same eight k
            //      per MFMA (the sums in the order of the direct path's prologue)
            const int half = w >> 3, w8 = w & 7, i = l & 15, kb = l >> 4;
            const int job = 2 * local + half;
            const int e0 = uniform(P.job_end[0]), e1 = uniform(P.job_end[1]), e2 = uniform(P.job_end[2]);
            const int g = job < jobs ? (job >= e0) + (job >= e1) + (job >= e2) : 0;
            const int rel = job - (g == 0 ? 0 : (g == 1 ? e0 : (g == 2 ? e1 : e2)));
            const BatchLayer &L = D.L[first + g];
            const int rank = job < jobs ? uniform(L.rank) : 0, hs = h_stride(rank);
            const int sp = rel % S, rt = rel / S;
            const rsrc_t ar = make_rsrc(uniform(L.A), (unsigned)rank * K * 2u);
            const int all = (K + 63) / 64, per = (all + S - 1) / S, end = min((sp + 1) * per, all);
            constexpr int UN = 4;
            v8h a[UN][2], b[UN][2];
            const int row = rt * 16 + i, m = i;
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int s = sp * per + w8 + u * 8, k0 = s * 64 + kb * 16;
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    a[u][q] = __builtin_bit_cast(v8h, buf_load16(ar, ((unsigned)row * K + k0 + 8 * q) * 2u, s < end && k0 + 8 * q < K && row < rank));
            }
            tokens_ready();
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int s = sp * per + w8 + u * 8, k0 = s * 64 + kb * 16;
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    b[u][q] = __builtin_bit_cast(v8h, buf_load16(src.r, src.at(m, k0 + 8 * q), s < end && k0 + 8 * q < K && m < M));
            }
            v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < UN; ++u)
#pragma unroll
                for (int q = 0; q < 2; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u][q], b[u][q], acc, 0, 0, 0);
            take_next();
            v4f *part = reinterpret_cast<v4f *>(lds);
            part[w * 64 + l] = acc;
            lds_barrier();
            if (w8 == 0 && rank > 0) {
                v4f h = part[w * 64 + l];
#pragma unroll
                for (int s = 1; s < 8; ++s) h += part[(w + s) * 64 + l];
                if (sh.failed != 0) h = (v4f){NAN, NAN, NAN, NAN};    // (not the sentinel)
                // element v: rank 16 rt + 4 kb + v of token m
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, h), mail,
                                                       (int)(m < M ? L.mail_off + (unsigned)((sp * M + m) * hs + rt * 16 + 4 * kb) * 4u : kOob), 0, 16);
            }
        } else {
            // ---- up to four row-blocks.  Twelve wavefronts contract, KS of them unit i of n; the last four collect
            //      SiLU(A x) and the gates meanwhile.
            constexpr int CW = 12;
            const int t = local - jtasks, u0 = t * upt, n = min(upt, uniform(P.units) - u0);
            const int KS = n == 1 ? CW : (n == 2 ? CW / 2 : (n == 3 ? CW / 3 : CW / 4));
            const int e0 = uniform(P.unit_end[0]), e1 = uniform(P.unit_end[1]), e2 = uniform(P.unit_end[2]);
            auto layer_of = [&](int u) { return (u >= e0) + (u >= e1) + (u >= e2); };
            auto block_of = [&](int u, int g) { return u - (g == 0 ? 0 : (g == 1 ? e0 : (g == 2 ? e1 : e2))); };
            const int rg = w < CW ? w / KS : 0, ks = w - rg * KS;
            const bool contracts = w < CW && rg < n;
            const int g = layer_of(u0 + rg), rb = block_of(u0 + rg, g);
            const rsrc_t wr = make_rsrc(uniform(D.L[first + g].packed) + (size_t)rb * KT * 64, contracts ? (unsigned)KT * kTileBytes : 0u);
            v4u wq[kD];
#pragma unroll
            for (int d = 0; d < kD; ++d) wq[d] = buf_load16_stream(wr, (unsigned)(ks + d * KS) * kTileBytes + l * 16u);
            // gates of the units' rows (by wavefronts that have no weights to ask for)
            if (w >= CW && w < CW + 2) {
                const int gx = tx - CW * 64, i = gx >> 5, u = u0 + min(i, n - 1), gg = layer_of(u), row = block_of(u, gg) * kTileRows + (gx & 31);
                const BatchLayer &L = D.L[first + gg];
                float gate = 0.f;
                if (L.rank > 0 && row < L.N) gate = tanhf((float)L.alpha[row]);
                sh.gate[gx] = gate;
                if ((gx & 31) == 0) sh.s_w[i] = *L.s_w;
            }
            const int red_off = uniform(P.red_off), h_off = uniform(P.h_off), h_layer = uniform(P.h_layer);
            tokens_ready();
            unsigned char *const xq = lds;
            const int np = (Kp * SL + kThreads * 8 - 1) / (kThreads * 8);
            if (np <= 4) quantise_tokens<SL, 4, 1>(src, tx, M, K, Kp, ustride, xq, sh);
            else if (np <= 8) quantise_tokens<SL, 8, 1>(src, tx, M, K, Kp, ustride, xq, sh);
            else if (np <= 12) quantise_tokens<SL, 12, 1>(src, tx, M, K, Kp, ustride, xq, sh);
            else quantise_tokens<SL, 8, 2>(src, tx, M, K, Kp, ustride, xq, sh);
            lds_barrier();

            const int g0 = layer_of(u0), g1 = layer_of(u0 + n - 1);
            if (w >= CW) {
                // ---- SiLU(A x) of the units' layers
#pragma clang loop unroll(disable)
                for (int gg = g0; gg <= g1; ++gg)
                    if (!gather_layer(D.L[first + gg], tx - CW * 64, kThreads - CW * 64, mail, S, M, p.polls, failed, lds + h_off + (gg - g0) * h_layer)) {
                        sh.failed = 1;
                        __hip_atomic_store(p.flags + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
            }
            // what this wavefront finishes: a quarter (8 rows) of unit fi, whose rows of B it asks for here (the ranks
            // beyond 64 where the registers of the weights are free)
            const int fi = w >> 2, fq = w & 3;
            const bool finishes = fi < n;
            const int fg = layer_of(u0 + (finishes ? fi : 0)), frb = block_of(u0 + (finishes ? fi : 0), fg), nb = frb * kTileRows;
            const BatchLayer &FL = D.L[first + fg];
            const int rank = uniform(FL.rank), N = uniform(FL.N);
            v8h bq[8];
            const rsrc_t br = make_rsrc(uniform(FL.B), (unsigned)N * rank * 2u);
            auto b_request = [&](int js0, int js1) __attribute__((always_inline)) {
                const unsigned at = ((unsigned)(nb + jl) * rank + hf * 8) * 2u;
                const bool ok = finishes && nb + jl < N;
#pragma unroll
                for (int js = js0; js < js1; ++js)
                    bq[js] = __builtin_bit_cast(v8h, buf_load16(br, at + js * 32u, ok && js * 16 + hf * 8 < rank));
            };
            // (the weights have landed, as the tokens, requested after them, have: said here so that the contraction
            // does not wait for the rows of B)
            __builtin_amdgcn_s_waitcnt(0x0F70);
            b_request(0, 4);
            v4i *const red = reinterpret_cast<v4i *>(lds + red_off);
            v16i acc = (v16i){};
            if (w < CW) {
                // ---- the contraction
                const unsigned char *xrow = xq + hf * ustride + (jl & (SL - 1)) * 16;
                auto tile = [&](const v4u codes, int kt) __attribute__((always_inline)) {
                    v4i xv[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) asm("" : "=v"(xv[q]));
                    if (jl < SL) {                            // (the other columns are never read)
#pragma unroll
                        for (int q = 0; q < 4; ++q) xv[q] = *reinterpret_cast<const v4i *>(xrow + (kt * 8 + q * 2) * ustride);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(widen_codes(codes[q]), xv[q], acc, 0, 0, 0);
                };
                // the tiles in flight, in straight line (each waits for itself only), then what is left of long rows
#pragma unroll
                for (int d = 0; d < kD; ++d) {
                    if (ks + d * KS >= KT) break;
                    tile(wq[d], ks + d * KS);
                }
#pragma clang loop unroll(disable)
                for (int k0 = ks + kD * KS; k0 < KT; k0 += 4 * KS) {
                    v4u more[4];
#pragma unroll
                    for (int d = 0; d < 4; ++d) more[d] = buf_load16_stream(wr, (unsigned)(k0 + d * KS) * kTileBytes + l * 16u);
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        if (k0 + d * KS >= KT) break;
                        tile(more[d], k0 + d * KS);
                    }
                }
            }
            b_request(4, 8);
            if (red_off == 0) lds_barrier();                  // (the partial tiles take the tokens' place)
            if (w < CW && jl < CO) {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    red[(w * 4 + c) * 2 * CO + hf * CO + jl] = (v4i){acc[4 * c], acc[4 * c + 1], acc[4 * c + 2], acc[4 * c + 3]};
            }
            lds_barrier();
            failed = failed || sh.failed != 0;
            take_next();

            // ---- correction up-projection, dequantise, gate, store.  Element v: row 8 fq + 4 hf + v, token jl.
            if (finishes) {
                const bool m_ok = jl < M;
                float s_x = 0.f;
                int rs = 0;
                if (jl < SL) {
                    s_x = sh.s_x[jl];
                    rs = SL == 8 ? sh.sum[2 * jl] + sh.sum[2 * jl + 1] : sh.rowsum[jl];
                }
                const unsigned char *const hl = lds + h_off + (fg - g0) * h_layer + l * 16;
                v16f corr = (v16f){};
#pragma unroll
                for (int js = 0; js < 8; ++js)
                    if (js * 16 < rank) corr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bq[js], *reinterpret_cast<const v8h *>(hl + js * 1024), corr, 0, 0, 0);
                v4i a = (v4i){0, 0, 0, 0};
                if (jl < CO) {
                    const v4i *pr = red + (fi * KS * 4 + fq) * 2 * CO + hf * CO + jl;
                    auto add = [&](auto ks_) __attribute__((always_inline)) {
                        constexpr int kn = decltype(ks_)::value;
                        v4i part[kn];
#pragma unroll
                        for (int o = 0; o < kn; ++o) part[o] = pr[o * 8 * CO];
#pragma unroll
                        for (int o = 0; o < kn; ++o) a += part[o];
                    };
                    if (n == 1) add(std::integral_constant<int, CW>{});
                    else if (n == 2) add(std::integral_constant<int, CW / 2>{});
                    else if (n == 3) add(std::integral_constant<int, CW / 3>{});
                    else add(std::integral_constant<int, CW / 4>{});
                }
                const float scale = s_x * sh.s_w[fi];
                const v4f gate = *reinterpret_cast<const v4f *>(&sh.gate[fi * 32 + 8 * fq + 4 * hf]);
                const int nn = nb + 8 * fq + 4 * hf;
                v4h o;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float cv = fq == 0 ? corr[v] : (fq == 1 ? corr[4 + v] : (fq == 2 ? corr[8 + v] : corr[12 + v]));
                    o[v] = (_Float16)((float)(a[v] - rs) * scale + gate[v] * cv);
                    if (failed) o[v] = __builtin_bit_cast(_Float16, (unsigned short)0x7e00);
                }
                if (m_ok && nn < N) {
                    _Float16 *const out = uniform(FL.y) + (size_t)jl * N + nn;
                    if (N % 4 == 0) {
                        *reinterpret_cast<v4h *>(out) = o;
                    } else {
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (nn + v < N) out[v] = o[v];
                    }
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, o), act,
                                                          (int)((unsigned)uniform((int)FL.act_off) + (unsigned)(frb * (M + (M & 1)) + jl) * 64u + (unsigned)(8 * fq + 4 * hf) * 2u), 0, 16);
                }
            }
            // ---- the task's word, once all of its outputs are where every workgroup sees them
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lds_barrier();
            if (tx == 0)
                __hip_atomic_store(reinterpret_cast<unsigned *>(words + ph * kBatchPhaseWords) + t, failed ? kVoid : kDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (tx == 0) sh.ticket = next;
        lds_barrier();
    }

    // ---- the last workgroup to get here puts the counters back and advances the launch counter
    if (threadIdx.x == 0) {
        const int done = __hip_atomic_fetch_add(p.flags + 9, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (done == (int)gridDim.x - 1) {
            __hip_atomic_store(p.flags + 9, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p.flags + 11, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p.flags + 6, (int)p.act_used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p.flags + 7, (int)p.mail_used, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(p.flags + 8, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(p.flags + 4, (int)(epoch + 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace

static int token_slots(int M) { return M > 8 ? 16 : 8; }
// LDS of a phase: the tokens (at least what the jobs' sums need), the partial tiles where there is room beside, SiLU(A x)
static size_t phase_lds(int M, int K, int layers, int h_layer, int *h_off, int *red_off)
{
    const int SL = token_slots(M), Kp = round_up(K, kTileCols);
    const size_t red = size_t(12) * 2048, h = (size_t)layers * h_layer;
    size_t off = (size_t)(Kp / 16) * unit_stride(SL);
    if (off < 16 * 1024) off = 16 * 1024;
    *red_off = 0;
    if (off + red + h <= kLdsMax) {
        *red_off = (int)off;
        off += red;
    } else if (off < red) {
        off = red;
    }
    *h_off = (int)off;
    return off + h;
}
bool batch_fits(int M, int K, int G, int rank, long long row_blocks)
{
    int h, r;
    return M <= kBatchTokens && prologue_slices(K) <= kBatchSlices && row_blocks <= 4 * kBatchWords &&
           (size_t)round_up(K, kTileCols) * token_slots(M) <= size_t(16) * 8 * kThreads &&       // pieces of a thread
           phase_lds(M, K, G, (rank + 15) / 16 * 1024, &h, &r) <= kLdsMax;
}

// Fills in tasks, exchange offsets and LDS layout of a launch whose M, phases (x_ext or src_phase, K,
// first_layer, G) and layers (pointers, N, rank) are set.  False: does not fit (not where every phase does by itself and
// the exchange sets hold them all).
bool plan_batch(BatchParams &p, size_t *lds_bytes)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) {
        (void)hipGetLastError();
        return false;
    }
    const int Mp = p.M + (p.M & 1);
    p.polls = stack_wait_limit() > 0 ? stack_wait_limit() : kPolls;
    size_t act = 0, mail = p.nphases * kBatchPhaseWords;
    int tasks = 0;
    size_t lds = 0;
    for (int i = 0; i < p.nphases; ++i) {
        BatchPhase &P = p.ph[i];
        const int S = prologue_slices(P.K);
        if (S > kBatchSlices) return false;
        P.S = (unsigned char)S;
        int units = 0, jobs = 0, rank_max = 0;
        for (int g = 0; g < P.G; ++g) {
            BatchLayer &L = p.L[P.first_layer + g];
            const int rbs = (L.N + kTileRows - 1) / kTileRows;
            units += rbs;
            L.act_off = (unsigned)act;
            L.mail_off = (unsigned)mail;
            act += align256((size_t)rbs * Mp * 64);
            rank_max = L.rank > rank_max ? L.rank : rank_max;
            if (L.rank > 0) {
                jobs += (L.rank + 15) / 16 * S;
                mail += (size_t)S * p.M * h_stride(L.rank) * 4;
            }
            if (g < 3) {
                P.unit_end[g] = g + 1 < P.G ? units : 1 << 30;
                P.job_end[g] = g + 1 < P.G ? jobs : 1 << 30;
            }
        }
        if (units > 4 * kBatchWords) return false;
        if (P.src_phase >= 0) P.src_off = p.L[P.src_layer].act_off;
        P.units = units;
        P.jobs = jobs;
        for (int g = P.G; g < 3; ++g) P.unit_end[g] = P.job_end[g] = 1 << 30;
        const int jt = (jobs + 1) / 2;
        int upt = 1;
        while (upt < 4 && jt + (units + upt - 1) / upt > cus) ++upt;
        P.upt = (unsigned char)upt;
        P.unit_tasks = (units + upt - 1) / upt;
        if (P.unit_tasks > kBatchWords) return false;
        P.task0 = tasks;
        tasks += jt + P.unit_tasks;
        P.h_layer = (rank_max + 15) / 16 * 1024;
        const size_t need = phase_lds(p.M, P.K, P.G < upt ? P.G : upt, P.h_layer, &P.h_off, &P.red_off);
        if (need > lds) lds = need;
    }
    if (act > kBatchActBytes || mail > kBatchMailBytes) return false;
    p.tasks = tasks;
    p.act_used = (unsigned)(p.act_shift + act);
    p.mail_used = (unsigned)mail;
    p.cus = cus;
    *lds_bytes = lds;
    return lds <= kLdsMax;
}

template <int SL>
static hipError_t launch_slots(const BatchParams &p, size_t lds_bytes, hipStream_t st)
{
    static OncePerDevice once;
    const hipError_t attr = allow_lds(once, reinterpret_cast<const void *>(&batch_kernel<SL>), kLdsMax);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((batch_kernel<SL>), dim3(p.tasks < p.cus ? p.tasks : p.cus), dim3(kThreads), lds_bytes, st, p);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchParams &p, size_t lds_bytes, hipStream_t st)
{
    return token_slots(p.M) == 8 ? launch_slots<8>(p, lds_bytes, st) : launch_slots<16>(p, lds_bytes, st);
}

}  // namespace hgf
