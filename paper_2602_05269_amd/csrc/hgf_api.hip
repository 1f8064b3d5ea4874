// C ABI of libhgf: host-side argument validation, workspace carving and dispatch.
// Every check happens before the first HIP call, so the error paths run without a GPU.
#include "hgf_internal.h"

#include <algorithm>
#include <utility>
#include <vector>

namespace hgf {

Workspace carve_workspace(void *base, int M, int d_in, int d_out, int rank, int groups, bool with_stack)
{
    Workspace ws;
    char *p = reinterpret_cast<char *>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *r = p ? p + off : nullptr;
        off += align256(bytes);
        return r;
    };
    ws.flags = reinterpret_cast<int32_t *>(take(kZeroBytes));
    ws.mail = reinterpret_cast<unsigned char *>(take(2 * kMailBytes));
    ws.xchg = with_stack ? reinterpret_cast<unsigned char *>(take(2 * kStackSetBytes)) : nullptr;
    const int Kp = round_up(d_in, kTileCols);
    ws.xq = reinterpret_cast<int8_t *>(take((size_t)M * Kp));
    ws.s_x = reinterpret_cast<float *>(take((size_t)M * 4));
    ws.rowsum = reinterpret_cast<int32_t *>(take((size_t)M * 4));
    ws.h16_each = align256((size_t)M * h_stride(rank > 0 ? rank : 1) * 2);
    ws.h16 = reinterpret_cast<_Float16 *>(take(ws.h16_each * groups));
    const int Md = M < 64 ? M : 64;
    ws.spare_bytes = rank > 0 ? groups * align256((size_t)32 * Md * h_stride(rank) * sizeof(float)) : 0;
    ws.wsum = reinterpret_cast<double *>(take(size_t(kWsumBlocks) * 8));
    ws.spare = reinterpret_cast<unsigned char *>(take(ws.spare_bytes));
    (void)d_out;
    ws.bytes = off;
    return ws;
}

namespace {

bool dims_ok(int d_in, int d_out) { return d_in >= 1 && d_out >= 1 && d_in <= HGF_MAX_DIM && d_out <= HGF_MAX_DIM; }
bool tokens_ok(int M, int d_in, int d_out)
{
    if (M < 1) return false;
    const long long big = (long long)M * (d_in > d_out ? d_in : d_out);
    return big < (1LL << 31);
}
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

hgf_status check_layer(const hgf_layer *L, int M)
{
    if (!L) return HGF_ERR_NULL;
    if (!dims_ok(L->d_in, L->d_out) || L->rank < 0 || L->rank > HGF_MAX_RANK) return HGF_ERR_SHAPE;
    if (!tokens_ok(M, L->d_in, L->d_out)) return HGF_ERR_SHAPE;
    if (!L->W_packed || !L->s_w) return HGF_ERR_NULL;
    if (L->rank > 0 && (!L->A_f16 || !L->B_f16 || !L->alpha_f16)) return HGF_ERR_NULL;
    if (!aligned16(L->W_packed)) return HGF_ERR_ALIGN;
    if (L->ln_gamma && !(L->ln_eps >= 0.0f)) return HGF_ERR_SHAPE;
    return HGF_OK;
}

hgf_status from_hip(hipError_t e) { return e == hipSuccess ? HGF_OK : HGF_ERR_DEVICE; }

// Beyond 4096 columns, more tokens than a fifth of the columns: what stands behind a LayerNorm is prepared for the
// prefill kernel in two launches (run_large_group).
bool many_tokens_for_long_rows(int K, int M) { return K > 4096 && K < 5 * (long long)M; }

// Which of the two paths a group of layers takes.  The prefill kernel's tiles are 256 rows by 64 or 128
// tokens and walk all of d_in with one workgroup each, so a group that does not fill the chip with them
// costs about 10 + 0.55 k-tiles microseconds whatever its size.  The direct path costs by its output tiles of
// 32 x 32 and by its preparation.  Up to 2048 columns that leaves SiLU(A x) ready made and a token weighs
// half a tile; longer rows are cut into slices, which the workgroups of every output tile add for themselves,
// and a token weighs 1/4 of a tile and 0.3 for every 16 ranks of every layer.  Beyond 512 tokens, where the
// prefill kernel fills the chip with few rows, each weighs 1/4 more, of sliced rows 1 more.  In these units the
// paths cross near the figures below; beyond 6144 columns the prefill workgroups' walk is what counts.  The
// SwiGLU pair saves more on the prefill path (neither y is stored).  Layers behind LayerNorms are each a prefill
// group of their own with a longer preparation, so they are weighed one by one, their tokens with half a tile
// and 0.05 for every 16 ranks of sliced rows; where that preparation is two launches, 0.1, and tokens beyond 512
// a tile more (up to 6144 columns).  Layers without ranks on short rows (run_large_group) cost less on the prefill path.  Up to 40
// tokens the direct path takes every group.
// (2514 groups of 41 to 5000 tokens, 40 to 32768 columns, 32 to 32000 rows, 8 to 128 ranks, both paths timed: the
// choice is 0.2 % from the better path in the mean, where tiles + 1.5 tokens against limits between 1600 and 4200
// was 2 %.  us, direct / prefill: 512 -> 32000 behind a LayerNorm, 128 tokens 18.3 / 13.4; three layers 512 -> 4096,
// 192 tokens 14.9 / 12.3; three 2048 -> 2048 behind LayerNorms, 384 tokens 31.2 / 55.6; two 4096 -> 1024, 640 tokens
// 31.7 / 28.2; 11008 -> 4096, 384 tokens 53.9 / 60.6; many tokens: 3343 x 2880 -> 88 35.8 / 26.9, 1633 x 6760 -> 368
// as a pair 58.6 / 44.1, 3583 x 800 -> 72 behind a LayerNorm 33.7 / 28.2, but 2401 x 304 -> 392 12.5 / 14.1; prepared in two launches:
// 1385 x 5952 -> 728, 128 ranks 88 / 76, three 1409 x 4984 -> 72, 16 ranks 161 / 174, three 1741 x 7144 -> 32
// 198 / 249; without ranks: 142 x 456 ->
// 15616 behind a LayerNorm 14.1 / 10.9, 627 x 51 -> 2304 9.1 / 7.6, but 1258 x 56 -> 1152 behind one 10.6 / 11.4,
// 193 x 146 -> 3744 8.2 / 9.1.  All of these with the direct path's two launches: where short rows take one
// (plan_short), the line lies too low for many tokens, 1536 x 512 -> 512 7.9 / 10.8, 4096 x 512 -> 256 8.0 / 14.4,
// 8192 x 512 -> 64 7.0 / 21.0; below it the choice is right, three 768 x 512 -> 512 10.6 / 11.3.)
bool takes_direct_path(int M, const hgf_layer *layers, int G, bool pair)
{
    if (M <= 40) return true;
    const int K = layers[0].d_in;
    const long long tokens = M, groups = (tokens + 31) / 32;
    const bool ln = layers[0].ln_gamma != nullptr;            // (then every layer of the group has one)
    const bool sliced = prologue_slices(K) > 1;
    bool ranks = false;
    for (int g = 0; g < G; ++g) ranks = ranks || layers[g].rank > 0;
    int most;
    const bool two = ln && K <= 6144 && many_tokens_for_long_rows(K, M);
    if (ln) most = sliced ? (two ? 2200 : 2300) : (K > 512 ? 2200 : 2400);
    else most = sliced ? (K > 6144 ? 2800 : (pair ? 1900 : 2400)) : 1750;
    if (!ranks && K <= 512) most = K % 8 ? 1300 : (ln ? 2100 : most);
    const int more = ln ? (two ? 20 : (K > 512 && !sliced ? 5 : 0)) : (sliced ? 20 : 5);
    const long long beyond = tokens > 512 ? more * (tokens - 512) : 0;
    const long long each = (sliced && !ln ? 5 : 10) * tokens + beyond;
    const long long rank_tile = sliced ? (two ? 2 : (ln ? 1 : 6)) * tokens : 0;
    long long cost = each;                                    // in twentieths of a tile
    for (int g = 0; g < G; ++g) {
        cost += 20 * groups * ((layers[g].d_out + kTileRows - 1) / kTileRows) +
                rank_tile * (layers[g].rank > 16 ? (layers[g].rank + 15) / 16 : 1);
        if (!ln) continue;
        if (cost > 20 * most) return false;
        cost = each;
    }
    return ln || cost <= 20 * most;
}

// Profiling aid: event pairs recorded around main-kernel launches, by kind (0 decode, 1 prefill).
bool g_profile = false;
int g_launch_level = 3;      // 0: two launches per group, 1: one where a group has such a path, 2: one per stack, 3: the faster
std::vector<std::pair<hipEvent_t, hipEvent_t>> g_events[2];
std::vector<hipEvent_t> g_event_pool;

hipEvent_t take_event()
{
    hipEvent_t e = nullptr;
    if (!g_event_pool.empty()) {
        e = g_event_pool.back();
        g_event_pool.pop_back();
    } else if (hipEventCreate(&e) != hipSuccess) {
        e = nullptr;
    }
    return e;
}

// Records an event pair around a main-kernel launch when profiling is on.
struct ProfileScope {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    hipStream_t st;
    int kind;
    ProfileScope(int kind_, hipStream_t st_) : st(st_), kind(kind_)
    {
        if (!g_profile) return;
        e0 = take_event();
        e1 = take_event();
        if (e0 && e1) (void)hipEventRecord(e0, st);
    }
    ~ProfileScope()
    {
        if (e0 && e1) {
            (void)hipEventRecord(e1, st);
            g_events[kind].emplace_back(e0, e1);
        }
    }
};

// `n` quantisations of M tokens: the first has the workspace's own buffers, the others its spare region.
bool quantisations_fit(int M, int K, int n, const Workspace &ws)
{
    return (n - 1) * (align256((size_t)M * round_up(K, kTileCols)) + 2 * align256((size_t)M * 4)) <= ws.spare_bytes;
}

// Places what the prologue of a group writes (layers, sizes and NQ are set): the first quantisation
// in the workspace's own buffers, those of the other LayerNorms of the group and, where d_in is cut,
// the slices of A x in its spare region, as many of them as it holds (whole rows are slow: three layers
// 16384 -> 512 of 64 ranks at 384 tokens 88 us, in the seven slices that fit 66).  False: the quantisations
// do not fit.
bool place_prologue(ProParams &p, const hgf_layer *layers, const Workspace &ws)
{
    if (!quantisations_fit(p.M, p.K, p.NQ, ws)) return false;
    const size_t xq_bytes = align256((size_t)p.M * round_up(p.K, kTileCols)), word_bytes = align256((size_t)p.M * 4);
    size_t used = 0;
    for (int i = 0; i < p.NQ; ++i) {
        ProTokens &Q = p.Q[i];
        Q.xq = ws.xq;
        Q.s_x = ws.s_x;
        Q.rowsum = ws.rowsum;
        Q.gamma = layers[i].ln_gamma;
        Q.beta = layers[i].ln_beta;
        Q.eps = layers[i].ln_eps;
        if (i == 0) continue;
        Q.xq = reinterpret_cast<int8_t *>(ws.spare + used);
        Q.s_x = reinterpret_cast<float *>(ws.spare + used + xq_bytes);
        Q.rowsum = reinterpret_cast<int32_t *>(ws.spare + used + xq_bytes + word_bytes);
        used += xq_bytes + 2 * word_bytes;
    }
    size_t slice = 0;                                // of all layers
    for (int g = 0; g < p.G; ++g) slice += p.L[g].rank > 0 ? align256((size_t)p.M * p.L[g].hstride * 4) : 0;
    p.S = prologue_slices(p.K);
    if (p.S * slice > ws.spare_bytes - used) p.S = (int)((ws.spare_bytes - used) / slice);
    if (p.S < 1) p.S = 1;
    for (int g = 0; g < p.G; ++g) {
        p.L[g].hpart = p.S > 1 ? reinterpret_cast<float *>(ws.spare + used) : nullptr;
        if (p.L[g].rank > 0) used += align256((size_t)p.S * p.M * p.L[g].hstride * 4);
    }
    return true;
}

// Two [M, d] fp16 matrices that share no memory.
bool apart(int M, const void *a, int da, const void *b, int db)
{
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a), pb = reinterpret_cast<uintptr_t>(b);
    return pa + (size_t)M * da * 2 <= pb || pb + (size_t)M * db * 2 <= pa;
}

// A group that the task queue takes as a phase: up to 16 tokens, rows of whole aligned 16-byte pieces.
bool batchable(int M, const hgf_layer *layers, int G)
{
    if (M > kBatchTokens || g_launch_level < 1) return false;
    const int K = layers[0].d_in;
    int rank = 0;
    long long row_blocks = 0;
    for (int g = 0; g < G; ++g) {
        rank = layers[g].rank > rank ? layers[g].rank : rank;
        row_blocks += (layers[g].d_out + kTileRows - 1) / kTileRows;
    }
    if (K % 8 != 0 || !batch_fits(M, K, G, rank, row_blocks)) return false;
    for (int g = 0; g < G; ++g) {
        const hgf_layer &L = layers[g];
        if (L.ln_gamma) return false;
        if (L.rank > 0 && (L.rank % 8 != 0 || !aligned16(L.A_f16) || !aligned16(L.B_f16))) return false;
    }
    return true;
}
void set_batch_layer(BatchLayer &D, const hgf_layer &L, void *y)
{
    D.packed = reinterpret_cast<const v4u *>(L.W_packed);
    D.s_w = L.s_w;
    D.A = reinterpret_cast<const _Float16 *>(L.A_f16);
    D.B = reinterpret_cast<const _Float16 *>(L.B_f16);
    D.alpha = reinterpret_cast<const _Float16 *>(L.alpha_f16);
    D.y = reinterpret_cast<_Float16 *>(y);
    D.N = L.d_out;
    D.rank = L.rank;
}
void set_batch_workspace(BatchParams &bp, const Workspace &ws)
{
    bp.flags = ws.flags;
    bp.xchg = ws.xchg;
    // (a workspace is aligned to 16 bytes)
    bp.act_shift = (unsigned)((0 - reinterpret_cast<uintptr_t>(ws.xchg)) % kBatchActAlign);
}

// Fills in what the launch for short rows reads of a group.
void set_short(ShortParams &sp, const void *x, int M, const hgf_layer *layers, int G, void *const *ys, int32_t *acc_debug, bool pair,
               float *amax_out, int32_t *acc_debug2)
{
    sp.x = reinterpret_cast<const _Float16 *>(x);
    sp.M = M;
    sp.K = layers[0].d_in;
    sp.G = G;
    sp.pair = pair ? 1 : 0;
    sp.amax_out = pair ? amax_out : nullptr;
    for (int g = 0; g < G; ++g) {
        const hgf_layer &L = layers[g];
        ShortLayer &S = sp.L[g];
        S.packed = reinterpret_cast<const v4u *>(L.W_packed);
        S.s_w = L.s_w;
        S.A = reinterpret_cast<const _Float16 *>(L.A_f16);
        S.B = reinterpret_cast<const _Float16 *>(L.B_f16);
        S.alpha = reinterpret_cast<const _Float16 *>(L.alpha_f16);
        S.gamma = L.ln_gamma;
        S.beta = L.ln_beta;
        S.eps = L.ln_eps;
        S.y = reinterpret_cast<_Float16 *>(ys[g]);
        S.acc_debug = (pair && g == 1) ? acc_debug2 : acc_debug;
        S.N = L.d_out;
        S.RBn = round_up(L.d_out, kTileRows) / kTileRows;
        S.rank = L.rank;
    }
}

// Direct path: `G` layers that read the same activations `x` run as two launches: the prologue
// (quantisers + SiLU(A x) of every layer) and one grouped main kernel.
//
// `pair` (G == 2): the SwiGLU pair -- layers[0] is the gate projection, layers[1] the up
// projection; the one output ys[1] receives SiLU(y_gate) * y_up, amax_out (nullable) the
// per-token max of its magnitude, acc_debug2 (nullable) the up projection's accumulators.
hgf_status run_decode_group(const void *x, int M, const hgf_layer *layers, int G, void *const *ys,
                            int32_t *acc_debug, const Workspace &ws, hipStream_t st, bool pair = false,
                            float *amax_out = nullptr, int32_t *acc_debug2 = nullptr, bool base3 = false)
{
    const int K = layers[0].d_in;
    const bool ln = layers[0].ln_gamma != nullptr;   // (then every layer of the group has one)
    // Workgroups of a single launch read the tokens and write the outputs at their own pace: an output that lies over
    // the tokens takes two launches.
    bool free_tokens = true;
    for (int g = 0; g < G; ++g) free_tokens = free_tokens && (!ys[g] || apart(M, x, K, ys[g], layers[g].d_out));
    // The persistent launch.  Base-3 weights take it for one token from 768 columns on and for two from 1536, of more
    // than 2048 rows from 1536 and 1600 on (us in two launches and in one, weights from memory; one token: 4096 -> 11008
    // rank 128 16.3, 12.8; 11008 x 11008 24.9, 21.2; 2048 -> 8192 11.8, 11.3; rank 16: 768 -> 32 8.0, 7.8; 768 -> 2048
    // 8.7, 8.65; 768 -> 4096 8.5, 9.4; 1024 -> 8192 9.8, 11.1; 1536 -> 8192 10.9, 11.0; 256 -> 1024 7.6, 8.5; two tokens:
    // 11008 -> 4096 20.0, 16.4; rank 16: 1536 -> 1024 9.7, 9.1; 1536 -> 8192 11.05, 11.8; 1792 -> 8192 11.2, 11.9; 3072 ->
    // 8192 12.5, 12.1), up to 2^27 weights (8192 -> 28672 32.4, 29.2, but 28.5, 29.8 where layers are met again).
    // For three and four the tokens' conversion, which every workgroup repeats, takes what the launch saves
    // (2048 -> 8192 11.6, 12.3; 4096 -> 11008 15.9, 15.3; 5504 -> 28672 23.7, 25.1).
    const bool b3_in_one = base3 && M <= kMaxFusedB3M && K >= 768 * M && (layers[0].d_out <= 2048 || K >= (M == 1 ? 1536 : 1600)) &&
                           (size_t)K * layers[0].d_out <= (size_t)1 << 27;
    bool fused = !pair && !ln && free_tokens && g_launch_level >= 1 && M <= kMaxFusedM && K % 8 == 0 && K <= kMaxFusedK &&
                 aligned16(x) && (!base3 || b3_in_one);
    for (int g = 0; g < G; ++g)
        fused = fused && (layers[g].rank == 0 ||
                          (layers[g].rank % 8 == 0 && aligned16(layers[g].A_f16) && aligned16(layers[g].B_f16) &&
                           (reinterpret_cast<uintptr_t>(layers[g].alpha_f16) & 3u) == 0));
    // Short rows: one launch, every workgroup prepares its tokens itself
    if (free_tokens && !fused && !base3 && g_launch_level >= 1) {
        ShortParams sp;
        set_short(sp, x, M, layers, G, ys, acc_debug, pair, amax_out, acc_debug2);
        size_t lds_bytes = 0;
        if (plan_short(sp, &lds_bytes)) {
            if (sp.amax_out && launch_zero_words(sp.amax_out, (size_t)M, st) != hipSuccess) return HGF_ERR_DEVICE;
            ProfileScope prof(0, st);
            return from_hip(launch_short(sp, lds_bytes, st));
        }
    }
    if (fused) {
        FusedParams fp;
        fp.x = reinterpret_cast<const _Float16 *>(x);
        fp.M = M;
        fp.K = K;
        fp.G = G;
        fp.base3 = base3 ? 1 : 0;
        fp.flags = ws.flags;
        fp.mail = ws.mail;
        for (int g = 0; g < G; ++g) {
            const hgf_layer &L = layers[g];
            DecLayer &D = fp.L[g];
            D.packed = reinterpret_cast<const v4u *>(L.W_packed);
            D.s_w = L.s_w;
            D.B = reinterpret_cast<const _Float16 *>(L.B_f16);
            D.alpha = reinterpret_cast<const _Float16 *>(L.alpha_f16);
            D.h16 = nullptr;
            D.y = reinterpret_cast<_Float16 *>(ys[g]);
            D.acc_debug = acc_debug;
            D.N = L.d_out;
            D.RBn = round_up(L.d_out, kTileRows) / kTileRows;
            D.rank = L.rank;
            D.hstride = h_stride(L.rank > 0 ? L.rank : 1);
            fp.A[g] = reinterpret_cast<const _Float16 *>(L.A_f16);
        }
        size_t lds_bytes = 0;
        if (plan_fused(fp, &lds_bytes)) {
            ProfileScope prof(0, st);
            return from_hip(launch_fused(fp, lds_bytes, st));
        }
    }
    ProParams pp;
    pp.x = reinterpret_cast<const _Float16 *>(x);
    pp.amax_zero = pair ? amax_out : nullptr;
    pp.M = M;
    pp.K = K;
    pp.G = G;
    pp.NQ = ln ? G : 1;
    pp.base3 = base3 ? 1 : 0;
    pp.by_rows = 0;
    for (int g = 0; g < G; ++g) {
        const hgf_layer &L = layers[g];
        pp.L[g].A = reinterpret_cast<const _Float16 *>(L.A_f16);
        pp.L[g].h16 = reinterpret_cast<_Float16 *>(reinterpret_cast<char *>(ws.h16) + ws.h16_each * g);
        pp.L[g].rank = L.rank;
        pp.L[g].hstride = h_stride(L.rank > 0 ? L.rank : 1);
    }
    if (!place_prologue(pp, layers, ws)) return HGF_ERR_WORKSPACE;
    if (base3) {
        // x_q is whole units of 80 columns here, up to M * 79 bytes past the end of its region (M <= 4): over
        // s_x and rowsum (256 bytes each), which move to the SiLU(A x) of the group's layers that there are not
        pp.Q[0].s_x = reinterpret_cast<float *>(reinterpret_cast<char *>(ws.h16) + ws.h16_each);
        pp.Q[0].rowsum = reinterpret_cast<int32_t *>(reinterpret_cast<char *>(ws.h16) + 2 * ws.h16_each);
    }
    DecodeParams dp;
    dp.S = pp.S;
    dp.base3 = pp.base3;
    dp.M = M;
    dp.G = G;
    dp.pair = pair ? 1 : 0;
    dp.amax_out = pair ? amax_out : nullptr;
    for (int g = 0; g < G; ++g) {
        const hgf_layer &L = layers[g];
        DecLayer &D = dp.L[g];
        D.packed = reinterpret_cast<const v4u *>(L.W_packed);
        D.s_w = L.s_w;
        D.B = reinterpret_cast<const _Float16 *>(L.B_f16);
        D.alpha = reinterpret_cast<const _Float16 *>(L.alpha_f16);
        const ProTokens &Q = pp.Q[ln ? g : 0];
        D.h16 = pp.L[g].h16;
        D.hpart = pp.L[g].hpart;
        D.xq = Q.xq;
        D.s_x = Q.s_x;
        D.rowsum = Q.rowsum;
        D.y = reinterpret_cast<_Float16 *>(ys[g]);
        D.acc_debug = (pair && g == 1) ? acc_debug2 : acc_debug;
        D.N = L.d_out;
        D.RBn = round_up(L.d_out, kTileRows) / kTileRows;
        D.rank = L.rank;
        D.hstride = h_stride(L.rank > 0 ? L.rank : 1);
    }
    if (launch_prologue(pp, st) != hipSuccess) return HGF_ERR_DEVICE;
    ProfileScope prof(0, st);
    return from_hip(launch_decode(dp, K, st));
}

// Large M: per group of layers that read the same activations, one launch for the quantiser
// and the down-projections with SiLU of all layers (both read x), then one launch of the int8
// MFMA prefill kernel over the tiles of all layers.
hgf_status run_large_group(const void *x, int M, const hgf_layer *layers, int G, void *const *ys,
                           int32_t *acc_debug, const Workspace &ws, hipStream_t st, const PairOut *pair_out = nullptr)
{
    const _Float16 *xh = reinterpret_cast<const _Float16 *>(x);
    const int K = layers[0].d_in;
    const bool ln = layers[0].ln_gamma != nullptr;   // (here such a layer is always a group of its own)
    const _Float16 *A[kMaxGroup];
    _Float16 *h16[kMaxGroup];
    int rank[kMaxGroup];
    bool whole_rows = K % 8 == 0;                    // rows of x and A of whole 16-byte pieces
    bool ranks = false;
    for (int g = 0; g < G; ++g) {
        A[g] = reinterpret_cast<const _Float16 *>(layers[g].A_f16);
        rank[g] = layers[g].rank;
        h16[g] = reinterpret_cast<_Float16 *>(reinterpret_cast<char *>(ws.h16) + ws.h16_each * g);
        whole_rows = whole_rows && (rank[g] == 0 || aligned16(A[g]));
        ranks = ranks || rank[g] > 0;
    }
    // The direct path's prologue prepares rows that are not whole 16-byte pieces (one thread per (token, rank)
    // before: 1365 -> 2048, 32 ranks, 1000 tokens 161 us with the main kernel, 17 now; 4097 -> 4096 744 and 40)
    // and, as one launch instead of two, what stands behind a LayerNorm up to 2^23 elements (us, two launches /
    // one: 512 x 4096 59.2 / 45.4, 2048 x 3072 54.7 / 51.6, 2048 x 4096 131.3 / 133.4, 2048 x 8192 115.3 / 134.9).
    // Otherwise prepare_kernel's larger tiles of A x are the better ones (2048 x 3072: 35.4 against 44.3), and
    // beyond 4096 columns corr_down_kernel's are, unless the rows are much longer than there are tokens (1503 x 4472
    // 56.5 / 63.2, 1072 x 4496 for three layers of 128 ranks 158 / 182, 1030 x 4256 49.1 / 48.9, 964 x 5128 52.8 / 50.2,
    // 1093 x 6544 69.9 / 56.7).
    // Without ranks there is one launch either way, and short rows are quantised faster by a workgroup per
    // token (us, that / the prologue: odd rows 131 x 158 -> 8192 7.8 / 8.9, 4 x 307 x 947 -> 6192 19.2 / 19.1, 109 x
    // 4316 -> 6136 25.4 / 20.4; behind a LayerNorm 137 x 192 -> 8832 10.2 / 11.6, 1015 x 688 -> 1120 14.9 / 13.9).
    const bool short_rows = !ranks && K <= 512;
    const bool one_launch = ln && (long long)M * K < (1 << 23) && !many_tokens_for_long_rows(K, M);
    if (!short_rows && (!whole_rows || one_launch)) {
        ProParams pp;
        pp.x = xh;
        pp.amax_zero = pair_out ? pair_out->amax_out : nullptr;
        pp.M = M;
        pp.K = K;
        pp.S = 1;
        pp.base3 = 0;
        pp.by_rows = 1;
        pp.Q[0] = {ws.xq, ws.s_x, ws.rowsum, layers[0].ln_gamma, layers[0].ln_beta, layers[0].ln_eps};
        // one launch, or one per layer beyond 4 million tokens: a launch holds less than 2^32 threads (four
        // layers of 128 ranks reach them at 7.5 million tokens)
        const int at_once = M > (1 << 22) ? 1 : G;
        for (int g0 = 0; g0 < G; g0 += at_once) {
            pp.G = at_once;
            pp.NQ = g0 == 0 ? 1 : 0;
            for (int g = 0; g < at_once; ++g)
                pp.L[g] = {A[g0 + g], h16[g0 + g], nullptr, rank[g0 + g], h_stride(rank[g0 + g] > 0 ? rank[g0 + g] : 1)};
            if (launch_prologue(pp, st) != hipSuccess) return HGF_ERR_DEVICE;
        }
    } else {
        if (pair_out && pair_out->amax_out && launch_zero_words(pair_out->amax_out, (size_t)M, st) != hipSuccess)
            return HGF_ERR_DEVICE;
        if (ln && launch_ln_quantize(xh, M, K, layers[0].ln_gamma, layers[0].ln_beta, layers[0].ln_eps, ws.xq, ws.s_x,
                                     ws.rowsum, st) != hipSuccess)
            return HGF_ERR_DEVICE;
        if (!ln && !whole_rows && launch_quantize(xh, M, K, ws.xq, ws.s_x, ws.rowsum, st) != hipSuccess)
            return HGF_ERR_DEVICE;
        if (launch_corr_down(xh, M, K, G, A, rank, h16, ln || !whole_rows ? nullptr : ws.xq, ws.s_x, ws.rowsum, st) !=
            hipSuccess)
            return HGF_ERR_DEVICE;
    }
    ProfileScope prof(1, st);
    return from_hip(launch_prefill(ws, h16, M, layers, G, ys, acc_debug, st, pair_out));
}

// ---- the scratch of hgf_linear_forward_static: what the workspace argument brings to
//      hgf_linear_forward (launch counter, exchange buffers, x_q, scales, SiLU(A x), partial
//      sums), for callers that can bring none.  Every GPU the library runs on holds its own
//      copy of this array at its own address until the process ends; host code reaches it only
//      through the address hipGetSymbolAddress returns with that GPU current.
constexpr size_t kStaticScratchBytes = size_t(8) << 20;
constexpr int kMaxDevices = 64;
}  // namespace
}  // namespace hgf

static __device__ __align__(256) unsigned char scratch[hgf::kStaticScratchBytes];

namespace hgf {
namespace {

unsigned char *g_scratch_ptr[kMaxDevices];      // per device: the array's address there (null: not asked yet)

Workspace carve_static(void *base, int M, const hgf_layer *L)
{
    return carve_workspace(base, M, L->d_in, L->d_out, L->rank, /*groups=*/1, /*with_stack=*/false);
}

// The spare region of a call of one layer: what a workspace has for it or, where less, what is left of the
// static array (for sizes that the array serves).  Both entry points take this, so that they cut A x alike.
size_t single_spare(int M, const hgf_layer *L)
{
    const size_t whole = carve_workspace(nullptr, M, L->d_in, L->d_out, L->rank).spare_bytes;
    const Workspace s = carve_static(nullptr, M, L);
    if (s.bytes > kStaticScratchBytes) return whole;
    const size_t left = kStaticScratchBytes - s.bytes + s.spare_bytes;
    return left < whole ? left : whole;
}

// The device address of `scratch` on the current device, set up on first use: the address is
// looked up and the control words and exchange buffers are put into the state
// hgf_workspace_init leaves them in (fill kernels on `st`, ahead of the caller's work).
hgf_status static_scratch(hipStream_t st, unsigned char **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return HGF_ERR_DEVICE;
    }
    if (!g_scratch_ptr[dev]) {
        unsigned char *ptr = nullptr;
        if (hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return HGF_ERR_DEVICE;
        }
        const Workspace ws = carve_workspace(ptr, 1, 1, 1, 0, 1, false);
        if (launch_fill(ws.flags, align256(kZeroBytes), 0u, st) != hipSuccess ||
            launch_fill(ws.mail, 2 * kMailBytes, 0xFFFFFFFFu, st) != hipSuccess)
            return HGF_ERR_DEVICE;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return HGF_OK;
}

}  // namespace
}  // namespace hgf

using namespace hgf;

extern "C" {

const char *hgf_status_string(int status)
{
    switch (status) {
        case HGF_OK: return "HGF_OK";
        case HGF_ERR_NULL: return "HGF_ERR_NULL: a required pointer is NULL";
        case HGF_ERR_SHAPE: return "HGF_ERR_SHAPE: a dimension is out of range";
        case HGF_ERR_ALIGN: return "HGF_ERR_ALIGN: a buffer is not 16-byte aligned";
        case HGF_ERR_UNSUPPORTED: return "HGF_ERR_UNSUPPORTED";
        case HGF_ERR_WORKSPACE: return "HGF_ERR_WORKSPACE: workspace missing or too small";
        case HGF_ERR_DEVICE: return "HGF_ERR_DEVICE: the HIP runtime refused a launch";
        default: return "HGF: unknown status";
    }
}

int hgf_version(void) { return 100; }

int hgf_padded_k(int d_in) { return (d_in >= 1 && d_in <= HGF_MAX_DIM) ? round_up(d_in, kTileCols) : 0; }

size_t hgf_packed_weight_bytes(int d_out, int d_in)
{
    if (!dims_ok(d_in, d_out)) return 0;
    return (size_t)(round_up(d_out, kTileRows) / kTileRows) * (round_up(d_in, kTileCols) / kTileCols) * kTileBytes;
}

size_t hgf_workspace_bytes(int M_max, int d_in_max, int d_out_max, int rank_max)
{
    if (!dims_ok(d_in_max, d_out_max) || rank_max < 0 || rank_max > HGF_MAX_RANK) return 0;
    if (!tokens_ok(M_max, d_in_max, d_out_max)) return 0;
    return carve_workspace(nullptr, M_max, d_in_max, d_out_max, rank_max).bytes;
}

hgf_status hgf_workspace_init(void *workspace, size_t workspace_bytes, void *stream)
{
    if (!workspace) return HGF_ERR_NULL;
    if (!aligned16(workspace)) return HGF_ERR_ALIGN;
    const Workspace ws = carve_workspace(workspace, 1, 1, 1, 0);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (launch_fill(ws.flags, align256(kZeroBytes), 0u, st) != hipSuccess) return HGF_ERR_DEVICE;
    if (launch_fill(ws.mail, 2 * kMailBytes, 0xFFFFFFFFu, st) != hipSuccess) return HGF_ERR_DEVICE;
    return from_hip(launch_fill(ws.xchg, 2 * kStackSetBytes, 0xFFFFFFFFu, st));
}

hgf_status hgf_quantize_pack_weights(const float *W, int d_out, int d_in, void *packed_out, float *s_w_out,
                                     void *workspace, size_t workspace_bytes, void *stream)
{
    if (!W || !packed_out || !s_w_out) return HGF_ERR_NULL;
    if (!dims_ok(d_in, d_out)) return HGF_ERR_SHAPE;
    if (!aligned16(packed_out)) return HGF_ERR_ALIGN;
    if (!workspace) return HGF_ERR_WORKSPACE;
    const Workspace ws = carve_workspace(workspace, 1, 1, 1, 0);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (launch_wsum(W, (size_t)d_out * d_in, ws.wsum, s_w_out, st) != hipSuccess) return HGF_ERR_DEVICE;
    return from_hip(launch_pack(W, d_out, d_in, s_w_out, reinterpret_cast<uint32_t *>(packed_out), st));
}

hgf_status hgf_unpack_weights(const void *packed, int d_out, int d_in, int8_t *T_out, void *stream)
{
    if (!packed || !T_out) return HGF_ERR_NULL;
    if (!dims_ok(d_in, d_out)) return HGF_ERR_SHAPE;
    if (!aligned16(packed)) return HGF_ERR_ALIGN;
    return from_hip(launch_unpack(reinterpret_cast<const uint32_t *>(packed), d_out, d_in, T_out,
                                  reinterpret_cast<hipStream_t>(stream)));
}

hgf_status hgf_quantize_activations(const void *x_f16, int M, int d_in, int8_t *xq_out, float *s_x_out,
                                    int32_t *rowsum_out, void *stream)
{
    if (!x_f16 || !xq_out || !s_x_out) return HGF_ERR_NULL;
    if (!dims_ok(d_in, 1) || !tokens_ok(M, d_in, 1)) return HGF_ERR_SHAPE;
    if (!aligned16(x_f16) || !aligned16(xq_out)) return HGF_ERR_ALIGN;
    return from_hip(launch_quantize(reinterpret_cast<const _Float16 *>(x_f16), M, d_in, xq_out, s_x_out, rowsum_out,
                                    reinterpret_cast<hipStream_t>(stream)));
}

hgf_status hgf_layernorm_quantize_activations(const void *x_f16, int M, int d_in, const float *ln_gamma,
                                              const float *ln_beta, float ln_eps, int8_t *xq_out, float *s_x_out,
                                              int32_t *rowsum_out, void *stream)
{
    if (!x_f16 || !xq_out || !s_x_out || !ln_gamma) return HGF_ERR_NULL;
    if (!dims_ok(d_in, 1) || !tokens_ok(M, d_in, 1) || !(ln_eps >= 0.0f)) return HGF_ERR_SHAPE;
    if (!aligned16(x_f16) || !aligned16(xq_out)) return HGF_ERR_ALIGN;
    return from_hip(launch_ln_quantize(reinterpret_cast<const _Float16 *>(x_f16), M, d_in, ln_gamma, ln_beta, ln_eps,
                                       xq_out, s_x_out, rowsum_out, reinterpret_cast<hipStream_t>(stream)));
}

hgf_status hgf_linear_forward(const void *x_f16, int M, const hgf_layer *L, void *y_f16, int32_t *acc_debug,
                              void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x_f16 || !y_f16) return HGF_ERR_NULL;
    const hgf_status s = check_layer(L, M);
    if (s != HGF_OK) return s;
    if (!aligned16(x_f16) || !aligned16(y_f16) || (acc_debug && !aligned16(acc_debug))) return HGF_ERR_ALIGN;
    if (!workspace) return HGF_ERR_WORKSPACE;
    if (!aligned16(workspace)) return HGF_ERR_ALIGN;
    Workspace ws = carve_workspace(workspace, M, L->d_in, L->d_out, L->rank);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    ws.spare_bytes = single_spare(M, L);
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (takes_direct_path(M, L, 1, false)) {
        void *ys[1] = {y_f16};
        return run_decode_group(x_f16, M, L, 1, ys, acc_debug, ws, st);
    }
    void *ys1[1] = {y_f16};
    return run_large_group(x_f16, M, L, 1, ys1, acc_debug, ws, st);
}

hgf_status hgf_swiglu_forward(const void *x_f16, int M, const hgf_layer *gate, const hgf_layer *up, void *z_f16,
                              float *amax_out, int32_t *acc_debug_gate, int32_t *acc_debug_up, void *workspace,
                              size_t workspace_bytes, void *stream)
{
    if (!x_f16 || !z_f16) return HGF_ERR_NULL;
    hgf_status s = check_layer(gate, M);
    if (s == HGF_OK) s = check_layer(up, M);
    if (s != HGF_OK) return s;
    if (gate->d_in != up->d_in || gate->d_out != up->d_out) return HGF_ERR_SHAPE;
    if (gate->ln_gamma || up->ln_gamma) return HGF_ERR_UNSUPPORTED;   // (each would need a quantisation of its own)
    if (!aligned16(x_f16) || !aligned16(z_f16) || (acc_debug_gate && !aligned16(acc_debug_gate)) ||
        (acc_debug_up && !aligned16(acc_debug_up)) || (reinterpret_cast<uintptr_t>(amax_out) & 3u))
        return HGF_ERR_ALIGN;
    if (!workspace) return HGF_ERR_WORKSPACE;
    if (!aligned16(workspace)) return HGF_ERR_ALIGN;
    const int rank_max = gate->rank > up->rank ? gate->rank : up->rank;
    const Workspace ws = carve_workspace(workspace, M, gate->d_in, gate->d_out, rank_max);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    // the prefill kernel stages both layers' SiLU(A x) at one row width
    if (M > 40 && gate->rank > 0 && up->rank > 0 && h_stride(gate->rank) != h_stride(up->rank))
        return HGF_ERR_UNSUPPORTED;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const hgf_layer pairL[2] = {*gate, *up};
    void *ys[2] = {nullptr, z_f16};
    if (takes_direct_path(M, pairL, 2, true))
        return run_decode_group(x_f16, M, pairL, 2, ys, acc_debug_gate, ws, st, true, amax_out, acc_debug_up);
    const PairOut po = {acc_debug_up, amax_out};
    return run_large_group(x_f16, M, pairL, 2, ys, acc_debug_gate, ws, st, &po);
}

namespace {
bool attn_dims_ok(int B, int L_max, int n_heads, int d_h)
{
    if (B < 1 || L_max < 1 || n_heads < 1 || d_h < 8 || d_h > 128 || (d_h & (d_h - 1)) != 0) return false;
    // the caches are addressed with 32-bit byte offsets per sequence
    return (long long)L_max * 2 * n_heads * d_h * 2 < (1LL << 31) && (long long)B * n_heads < (1LL << 16);
}
}  // namespace

size_t hgf_diff_attention_workspace_bytes(int B, int L_max, int n_heads, int d_h)
{
    return attn_dims_ok(B, L_max, n_heads, d_h) ? diff_attn_workspace_bytes(B, L_max, n_heads, d_h) : 0;
}

hgf_status hgf_diff_attention_decode(const void *q_f16, const void *k_cache_f16, const void *v_cache_f16,
                                     const int32_t *lens, int B, int L_max, int n_heads, int d_h, float lambda,
                                     void *out_f16, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!q_f16 || !k_cache_f16 || !v_cache_f16 || !lens || !out_f16) return HGF_ERR_NULL;
    if (!attn_dims_ok(B, L_max, n_heads, d_h)) return HGF_ERR_SHAPE;
    if (!aligned16(q_f16) || !aligned16(k_cache_f16) || !aligned16(v_cache_f16) ||
        (reinterpret_cast<uintptr_t>(out_f16) & 1u) || (reinterpret_cast<uintptr_t>(lens) & 3u))
        return HGF_ERR_ALIGN;
    if (!workspace || workspace_bytes < diff_attn_workspace_bytes(B, L_max, n_heads, d_h)) return HGF_ERR_WORKSPACE;
    if (!aligned16(workspace)) return HGF_ERR_ALIGN;
    return from_hip(launch_diff_attn(q_f16, k_cache_f16, v_cache_f16, lens, B, L_max, n_heads, d_h, lambda, out_f16,
                                     workspace, reinterpret_cast<hipStream_t>(stream)));
}

size_t hgf_packed_weight_bytes_b3(int d_out, int d_in)
{
    if (!dims_ok(d_in, d_out)) return 0;
    return b3_packed_bytes(d_out, d_in);
}

hgf_status hgf_quantize_pack_weights_b3(const float *W, int d_out, int d_in, void *packed_out, float *s_w_out,
                                        void *workspace, size_t workspace_bytes, void *stream)
{
    if (!W || !packed_out || !s_w_out) return HGF_ERR_NULL;
    if (!dims_ok(d_in, d_out)) return HGF_ERR_SHAPE;
    if (!aligned16(packed_out)) return HGF_ERR_ALIGN;
    if (!workspace) return HGF_ERR_WORKSPACE;
    const Workspace ws = carve_workspace(workspace, 1, 1, 1, 0);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (launch_wsum(W, (size_t)d_out * d_in, ws.wsum, s_w_out, st) != hipSuccess) return HGF_ERR_DEVICE;
    return from_hip(launch_pack_b3(W, d_out, d_in, s_w_out, reinterpret_cast<unsigned char *>(packed_out), st));
}

hgf_status hgf_unpack_weights_b3(const void *packed, int d_out, int d_in, int8_t *T_out, void *stream)
{
    if (!packed || !T_out) return HGF_ERR_NULL;
    if (!dims_ok(d_in, d_out)) return HGF_ERR_SHAPE;
    if (!aligned16(packed)) return HGF_ERR_ALIGN;
    return from_hip(launch_unpack_b3(reinterpret_cast<const unsigned char *>(packed), d_out, d_in, T_out,
                                     reinterpret_cast<hipStream_t>(stream)));
}

hgf_status hgf_linear_forward_b3(const void *x_f16, int M, const hgf_layer *L, void *y_f16, int32_t *acc_debug,
                                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!x_f16 || !y_f16) return HGF_ERR_NULL;
    const hgf_status s = check_layer(L, M);
    if (s != HGF_OK) return s;
    if (!aligned16(x_f16) || !aligned16(y_f16)) return HGF_ERR_ALIGN;
    if (!workspace) return HGF_ERR_WORKSPACE;
    if (!aligned16(workspace)) return HGF_ERR_ALIGN;
    const Workspace ws = carve_workspace(workspace, M, L->d_in, L->d_out, L->rank);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    // up to four tokens (beyond them the 2-bit format is the faster one) of up to 20480 columns
    if (L->ln_gamma || M > 4 || round_up(L->d_in, kB3Cols) > 20480) return HGF_ERR_UNSUPPORTED;
    void *ys[1] = {y_f16};
    return run_decode_group(x_f16, M, L, 1, ys, acc_debug, ws, reinterpret_cast<hipStream_t>(stream), false, nullptr, nullptr, true);
}

size_t hgf_static_scratch_bytes(void) { return kStaticScratchBytes; }

size_t hgf_static_scratch_needed(int M, int d_in, int d_out, int rank)
{
    if (!dims_ok(d_in, d_out) || rank < 0 || rank > HGF_MAX_RANK || !tokens_ok(M, d_in, d_out)) return 0;
    return carve_workspace(nullptr, M, d_in, d_out, rank, 1, false).bytes;
}

hgf_status hgf_linear_forward_static(const void *x_f16, int M, const hgf_layer *L, void *y_f16, int32_t *acc_debug,
                                     void *stream)
{
    if (!x_f16 || !y_f16) return HGF_ERR_NULL;
    const hgf_status s = check_layer(L, M);
    if (s != HGF_OK) return s;
    if (!aligned16(x_f16) || !aligned16(y_f16) || (acc_debug && !aligned16(acc_debug))) return HGF_ERR_ALIGN;
    if (carve_static(nullptr, M, L).bytes > kStaticScratchBytes) return HGF_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    unsigned char *base = nullptr;
    const hgf_status ss = static_scratch(st, &base);
    if (ss != HGF_OK) return ss;
    Workspace ws = carve_static(base, M, L);
    ws.spare_bytes = single_spare(M, L);
    void *ys[1] = {y_f16};
    const bool profiling = g_profile;           // (the profiling aid creates events: not from here)
    g_profile = false;
    const hgf_status r = takes_direct_path(M, L, 1, false) ? run_decode_group(x_f16, M, L, 1, ys, acc_debug, ws, st)
                                          : run_large_group(x_f16, M, L, 1, ys, acc_debug, ws, st);
    g_profile = profiling;
    return r;
}

hgf_status hgf_stack_forward(const hgf_layer *layers, int n_layers, void *const *slots, int n_slots, int M,
                             void *workspace, size_t workspace_bytes, void *stream)
{
    if (!layers || !slots) return HGF_ERR_NULL;
    if (n_layers < 1 || n_slots < 1) return HGF_ERR_SHAPE;
    int d_in_max = 1, d_out_max = 1, rank_max = 0;
    for (int i = 0; i < n_layers; ++i) {
        const hgf_layer &L = layers[i];
        const hgf_status s = check_layer(&L, M);
        if (s != HGF_OK) return s;
        if (L.src_slot < 0 || L.src_slot >= n_slots || L.dst_slot < 0 || L.dst_slot >= n_slots ||
            L.src_slot == L.dst_slot)
            return HGF_ERR_SHAPE;
        if (!slots[L.src_slot] || !slots[L.dst_slot]) return HGF_ERR_NULL;
        if (!aligned16(slots[L.src_slot]) || !aligned16(slots[L.dst_slot])) return HGF_ERR_ALIGN;
        if (L.d_in > d_in_max) d_in_max = L.d_in;
        if (L.d_out > d_out_max) d_out_max = L.d_out;
        if (L.rank > rank_max) rank_max = L.rank;
    }
    if (!workspace) return HGF_ERR_WORKSPACE;
    if (!aligned16(workspace)) return HGF_ERR_ALIGN;
    const Workspace ws = carve_workspace(workspace, M, d_in_max, d_out_max, rank_max);
    if (workspace_bytes < ws.bytes) return HGF_ERR_WORKSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);

    // groups: consecutive layers reading the same slot with the same d_in, none of which writes
    // that slot or a slot another member writes (all with a LayerNorm of their own, or none)
    struct Group { int first, G; bool stackable, batch; };
    std::vector<Group> groups;
    for (int i = 0; i < n_layers;) {
        int G = 1;
        while (i + G < n_layers && G < kMaxGroup) {
            const hgf_layer &C = layers[i + G];
            bool ok = C.src_slot == layers[i].src_slot && C.d_in == layers[i].d_in &&
                      (C.ln_gamma != nullptr) == (layers[i].ln_gamma != nullptr);
            // layers with LayerNorms need a quantisation each: the direct path's prologue makes them in one launch
            // (and not where slots share memory: one after the other such layers see each other's outputs)
            if (ok && C.ln_gamma) {
                ok = takes_direct_path(M, layers + i, G + 1, false) && quantisations_fit(M, C.d_in, G + 1, ws);
                for (int j = i; ok && j < i + G; ++j)
                    ok = apart(M, slots[layers[j].dst_slot], layers[j].d_out, slots[C.src_slot], C.d_in) &&
                         apart(M, slots[layers[j].dst_slot], layers[j].d_out, slots[C.dst_slot], C.d_out);
            }
            for (int j = i; ok && j < i + G; ++j) ok = layers[j].dst_slot != C.dst_slot;
            if (!ok) break;
            ++G;
        }
        const int K = layers[i].d_in;
        bool stackable = g_launch_level >= 2 && M <= kMaxFusedM && K % 8 == 0 && K <= kMaxFusedK && !layers[i].ln_gamma;
        for (int g = 0; g < G && stackable; ++g) {
            const hgf_layer &L = layers[i + g];
            stackable = L.d_out % 8 == 0 &&
                        (L.rank == 0 || (L.rank % 8 == 0 && aligned16(L.A_f16) && aligned16(L.B_f16) &&
                                         (reinterpret_cast<uintptr_t>(L.alpha_f16) & 3u) == 0));
        }
        // a phase of the task queue, unless its rows are short.  (Such lists would gain from it too, which is left: us, d = 512
        // blocks of 16 ranks at 16 tokens, one launch a group / the queue: 8 groups 51.9 / 43.9, 32 groups 192.6 / 128.4.)
        bool batch = M > kMaxFusedM && batchable(M, layers + i, G);
        if (batch) {
            void *ys[kMaxGroup];
            for (int g = 0; g < G; ++g) ys[g] = slots[layers[i + g].dst_slot];
            ShortParams sp;
            set_short(sp, slots[layers[i].src_slot], M, layers + i, G, ys, nullptr, false, nullptr, nullptr);
            size_t lds_bytes = 0;
            batch = !plan_short(sp, &lds_bytes);
        }
        groups.push_back({i, G, stackable, batch});
        i += G;
    }

    auto run_group = [&](const Group &gr) -> hgf_status {
        const void *x = slots[layers[gr.first].src_slot];
        if (takes_direct_path(M, layers + gr.first, gr.G, false)) {
            void *ys[kMaxGroup];
            for (int g = 0; g < gr.G; ++g) ys[g] = slots[layers[gr.first + g].dst_slot];
            return run_decode_group(x, M, layers + gr.first, gr.G, ys, nullptr, ws, st);
        }
        void *ys[kMaxGroup];
        for (int g = 0; g < gr.G; ++g) ys[g] = slots[layers[gr.first + g].dst_slot];
        return run_large_group(x, M, layers + gr.first, gr.G, ys, nullptr, ws, st);
    };

    // Runs groups [a, b), all stackable, as one persistent launch.  kNoFit: they do not fit one
    // (nothing was enqueued; the groups then run one by one); kRefused: the runtime refused it.
    auto run_stack = [&](size_t a, size_t b) -> Launch {
        StackParams sp;
        sp.M = M;
        sp.nphases = (int)(b - a);
        sp.flags = ws.flags;
        sp.xchg = ws.xchg;
        int nl = 0;
        size_t act = 0;
        for (size_t gi = a; gi < b; ++gi) {
            const Group &gr = groups[gi];
            StackPhase &P = sp.ph[gi - a];
            P.K = layers[gr.first].d_in;
            P.first_layer = (short)nl;
            P.G = (short)gr.G;
            // the tokens: the latest earlier layer of this launch that writes the slot, else the slot itself
            const int src = layers[gr.first].src_slot;
            P.x_ext = reinterpret_cast<const _Float16 *>(slots[src]);
            P.src_off = 0;
            for (int j = 0; j < nl; ++j) {
                if (layers[groups[a].first + j].dst_slot == src) {
                    P.x_ext = nullptr;
                    P.src_off = sp.L[j].act_off;
                }
            }
            for (int g = 0; g < gr.G; ++g) {
                const hgf_layer &L = layers[gr.first + g];
                StackLayer &D = sp.L[nl++];
                D.packed = reinterpret_cast<const v4u *>(L.W_packed);
                D.s_w = L.s_w;
                D.A = reinterpret_cast<const _Float16 *>(L.A_f16);
                D.B = reinterpret_cast<const _Float16 *>(L.B_f16);
                D.alpha = reinterpret_cast<const _Float16 *>(L.alpha_f16);
                D.y = reinterpret_cast<_Float16 *>(slots[L.dst_slot]);
                D.N = L.d_out;
                D.rank = L.rank;
                D.act_off = (unsigned)act;
                D.reserved = 0;
                act += align256((size_t)M * L.d_out * 2);
            }
        }
        if (act > kStackActBytes) return Launch::kNoFit;
        sp.act_used = (unsigned)act;
        size_t lds_bytes = 0;
        if (!plan_stack(sp, &lds_bytes)) return Launch::kNoFit;
        ProfileScope prof(0, st);
        return launch_stack(sp, lds_bytes, st) == hipSuccess ? Launch::kRan : Launch::kRefused;
    };

    // The list's weights are more than the last-level cache holds (those that several layers share counted once).
    auto from_memory = [&]() {
        std::vector<std::pair<const void *, size_t>> w;
        for (int i = 0; i < n_layers; ++i) w.emplace_back(layers[i].W_packed, (size_t)layers[i].d_in * layers[i].d_out / 4);
        std::sort(w.begin(), w.end());
        size_t bytes = 0;
        for (size_t i = 0; i < w.size(); ++i)
            if (i == 0 || w[i].first != w[i - 1].first) bytes += w[i].second;
        return bytes >= kLastLevelCache;
    };

    // Runs groups [a, b') as one launch of the task queue, b' <= b as far as they fit: every slot that is written
    // in it shares no memory with another that is written or with one that is read as it was before the launch.
    // Without a launch: `ran` groups are not worth another attempt.
    auto run_batch = [&](size_t a, size_t b, size_t &ran) -> Launch {
        BatchParams bp;
        set_batch_workspace(bp, ws);
        bp.M = M;
        struct Range { const void *p; int d; bool written; } ranges[2 * kBatchMaxLayers];
        int nr = 0, nl = 0, np = 0;
        int depth[kBatchMaxPhases], deepest = 0, fresh = 0;     // phases that wait for each other; the first later one that does not
        size_t act = 0, mail = 0;
        const int Mp = M + (M & 1);
        for (size_t gi = a; gi < b && np < kBatchMaxPhases; ++gi) {
            const Group &gr = groups[gi];
            if (nl + gr.G > kBatchMaxLayers) break;
            const int K = layers[gr.first].d_in, src = layers[gr.first].src_slot;
            BatchPhase &P = bp.ph[np];
            P.x_ext = reinterpret_cast<const _Float16 *>(slots[src]);
            P.K = K;
            P.first_layer = (unsigned char)nl;
            P.G = (unsigned char)gr.G;
            P.src_phase = P.src_layer = -1;
            for (int q = 0; q < np; ++q)            // the latest earlier layer of this launch that writes the slot
                for (int j = 0; j < bp.ph[q].G; ++j) {
                    const int i = bp.ph[q].first_layer + j;
                    if (layers[groups[a].first + i].dst_slot == src) {
                        P.src_phase = (short)q;
                        P.src_layer = (short)i;
                    }
                }
            bool ok = P.src_phase < 0 || bp.L[P.src_layer].N == K;
            const int nr0 = nr;
            auto add = [&](const void *p, int d, bool written) {
                for (int i = 0; i < nr && ok; ++i) ok = (!written && !ranges[i].written) || apart(M, p, d, ranges[i].p, ranges[i].d);
                ranges[nr++] = {p, d, written};
            };
            if (P.src_phase < 0) add(slots[src], K, false);
            size_t act1 = act, mail1 = mail;
            for (int g = 0; g < gr.G; ++g) {
                const hgf_layer &L = layers[gr.first + g];
                add(slots[L.dst_slot], L.d_out, true);
                set_batch_layer(bp.L[nl + g], L, slots[L.dst_slot]);
                act1 += align256((size_t)((L.d_out + kTileRows - 1) / kTileRows) * Mp * 64);
                if (L.rank > 0) mail1 += (size_t)prologue_slices(K) * M * h_stride(L.rank) * 4;
            }
            if (!ok || act1 > kBatchActBytes || mail1 + (np + 1) * kBatchPhaseWords > kBatchMailBytes) {
                nr = nr0;
                break;
            }
            act = act1;
            mail = mail1;
            nl += gr.G;
            depth[np] = P.src_phase < 0 ? 1 : depth[P.src_phase] + 1;
            deepest = depth[np] > deepest ? depth[np] : deepest;
            if (P.src_phase < 0 && fresh == 0) fresh = np;
            ++np;
        }
        // (a launch begins with some 8 us that no earlier phase hides: us, two launches each / so, four phases of the
        // 1.2B shape at 16 tokens 47.2 / 55.0 where the weights are met again, 57.9 / 54.9 from memory, eight 102 / 86 and
        // 116 / 86; of the 7B shape at 8 tokens four 64.6 / 61.1 and 72.2 / 62.3)
        ran = 1;
        if (np < kBatchMinPhases) return Launch::kNoFit;
        // A run that is one chain has nothing to do while a phase waits: its two launches per group, whose tokens are
        // quantised once, are faster unless the weights come from memory, which the queue asks for ahead.  (us in the queue /
        // in two launches each, 196 lists of 6 to 16 phases repeated / behind flushed caches, in the mean: one chain 1.07
        // (1.33 at most) / 0.87, two phases beside the chain 0.92 / 0.74, four 0.78 / 0.66, eight 0.66 / 0.56; a chain of 64
        // phases of the 7B shape, 1.4 GB, at 8 tokens 0.79.)
        if (g_launch_level >= 3 && np - deepest < 2 && !from_memory()) {
            ran = fresh > 0 ? fresh : np;
            return Launch::kNoFit;
        }
        bp.nphases = np;
        size_t lds_bytes = 0;
        if (!plan_batch(bp, &lds_bytes)) return Launch::kNoFit;
        ran = np;
        ProfileScope prof(0, st);
        return launch_batch(bp, lds_bytes, st) == hipSuccess ? Launch::kRan : Launch::kRefused;
    };

    size_t gi = 0, queue_from = 0;
    while (gi < groups.size()) {
        if (groups[gi].batch && gi >= queue_from) {
            size_t ge = gi, ran = 1;
            while (ge < groups.size() && groups[ge].batch) ++ge;
            const Launch r = ge - gi >= (size_t)kBatchMinPhases ? run_batch(gi, ge, ran) : Launch::kNoFit;
            if (r == Launch::kRefused) return HGF_ERR_DEVICE;
            if (r == Launch::kRan) {
                gi += ran;
                continue;
            }
            queue_from = gi + ran;
        }
        // the longest run of stackable groups that fits one launch's description
        size_t ge = gi;
        int nl = 0;
        size_t act = 0;
        while (ge < groups.size() && groups[ge].stackable && (int)(ge - gi) < kStackMaxPhases &&
               nl + groups[ge].G <= kStackMaxLayers) {
            size_t add = 0;
            for (int g = 0; g < groups[ge].G; ++g) add += align256((size_t)M * layers[groups[ge].first + g].d_out * 2);
            if (act + add > kStackActBytes) break;
            act += add;
            nl += groups[ge].G;
            ++ge;
        }
        if (ge - gi >= 2) {
            const Launch r = run_stack(gi, ge);
            if (r == Launch::kRefused) return HGF_ERR_DEVICE;
            if (r == Launch::kRan) {
                gi = ge;
                continue;
            }
        }
        if (ge == gi) ge = gi + 1;
        for (; gi < ge; ++gi) {
            const hgf_status s = run_group(groups[gi]);
            if (s != HGF_OK) return s;
        }
    }
    return HGF_OK;
}

void hgf_profile_enable(int on) { g_profile = on != 0; }

hgf_status hgf_profile_collect(double *ms_out, long long *launches_out)
{
    if (!ms_out || !launches_out) return HGF_ERR_NULL;
    for (int kind = 0; kind < 2; ++kind) {
        double total = 0.0;
        long long n = 0;
        for (auto &pr : g_events[kind]) {
            float ms = 0.f;
            if (hipEventSynchronize(pr.second) == hipSuccess && hipEventElapsedTime(&ms, pr.first, pr.second) == hipSuccess) {
                total += ms;
                ++n;
            }
            g_event_pool.push_back(pr.first);
            g_event_pool.push_back(pr.second);
        }
        g_events[kind].clear();
        ms_out[kind] = total;
        launches_out[kind] = n;
    }
    return HGF_OK;
}

void hgf_set_single_launch(int level) { g_launch_level = level < 0 ? 0 : (level > 3 ? 3 : level); }

void hgf_set_wait_limit(int tries) { set_stack_wait_limit(tries); }

void hgf_set_stack_trace(void *device_buffer, size_t bytes, int first_phase)
{
    set_stack_trace(reinterpret_cast<unsigned long long *>(device_buffer), bytes, first_phase);
}

}  // extern "C"
