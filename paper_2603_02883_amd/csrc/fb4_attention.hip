// C ABI of the FB4 quantizer library, the attention-guided entry points (Sec. 3.3, 3.4, App. F): scores on the
// matrix cores, the per-tile choice, SeDA's main anchors and correlated tokens.  Declarations and contracts are in
// include/fb4.h.
#include <algorithm>

#include "fb4_common.hpp"
#include "fb4_salient.hpp"

using namespace fb4;

namespace {

// Blocks of 32 queries per wavefront of the long-group kernel.  A workgroup's time goes with b + 0.7 (0.7: what a step
// costs whatever the number of blocks; 24 groups x 16384 tokens x 128 channels take 1124 / 1215 / 1261 / 1555 us with
// 4 / 3 / 2 / 1), m workgroups on a compute unit take about 0.2 + 0.8 m times as long as one, and the last workgroup
// of a group has only the blocks that are left.  So long launches take 4 and short ones fewer, to reach more
// compute units.  us with 1 / 2 / 3 / 4, the choice starred: 16 x 400 x 72 4.4* / 5.4 / 6.4 / 7.7, 8 x 3000 x 72 16.6 / 17.8* /
// 22.4 / 27.6, 130 x 480 x 72 9.5 / 8.7 / 8.9* / 10.5, 24 x 4000 x 64 52.8 / 44.7 / 44.9* / 51.0, 272 x 1350 x 72 86.4 / 69.8 /
// 66.9 / 66.1*, 384 x 1024 x 128 120.8 / 96.7 / 90.5 / 84.5*.  With up to six (`most`, 80 to 96 channels) a workgroup's time goes
// with b + 1.05, m of them take about 0.33 + 0.67 m times as long, and m is 0.48 of the rounds that the load takes, a tenth of
// those that as many whole workgroups would, and the load itself for the rest: 1 / .. / 6 300 x 480 x 96 29.1 / 22.7 / 22.4 / 23.5 /
// 24.2* / 24.2, 130 x 480 x 96 12.7 / 11.9 / 10.5* / 12.3 / 11.6 / 11.2, 45 x 1744 x 96 34.9 / 31.7 / 28.6* / 33.2 / 32.8 / 29.4, 130 x
// 1350 x 96 64.0 / 49.8 / 48.0 / 47.6* / 50.6 / 52.2, 272 x 700 x 96 40.9 / 33.6 / 31.1 / 31.8* / 31.8 / 33.9, 1000 x 300 x 96 with 5 24.3
// and with 4 29.4 (646 shapes: 1.0 % above the best choice on average).  (256 compute units as on this card: the choice decides
// speed only.  That rows of up to 72 channels run three workgroups per compute unit and longer ones two is left out: the
// figures above come from both.)
uint32_t dma_blocks_per_wave(int64_t groups, uint32_t n_blk, uint32_t most)
{
    constexpr double kCus = 256.0;
    const bool six = most > 4;
    const double step = six ? 1.05 : 0.7, first = six ? 0.33 : 0.2;
    uint32_t best = most;
    double best_cost = 0.0;
    for (uint32_t b = most; b >= 1; --b) {
        const uint32_t full = n_blk / (2 * b), rest = n_blk - full * 2 * b;
        const double units = full * (b + step) + (rest ? (rest + 1) / 2 + step : 0.0);
        const double load = (double)groups * units / ((b + step) * kCus);
        const double whole = load > 1.0 ? (double)(int64_t)(load + 0.999) : 1.0;
        const double all = (double)((groups * (full + (rest ? 1 : 0)) + 255) / 256);   // (rounds of workgroups, the short ones too)
        const double m = six ? std::max(1.0, 0.48 * whole + 0.1 * all + 0.42 * load) : whole;
        const double cost = (b + step) * (first + (1.0 - first) * m);
        if (b == most || cost < best_cost) { best_cost = cost; best = b; }
    }
    return best;
}

}  // namespace

extern "C" {

int fb4_attention_scores(const void* q, const void* k, int64_t groups, int64_t tokens, int64_t dim, int mode,
                         float* scores, void* stream)
{
    if (groups < 0 || tokens < 0 || dim < 0 || (mode != 0 && mode != 1)) return FB4_ERR_INVALID_ARG;
    if (groups == 0 || tokens == 0) return FB4_OK;
    if (!q || !k || !scores || dim == 0) return FB4_ERR_INVALID_ARG;
    if ((dim % 8) || dim > 256 || !aligned(q, 16) || !aligned(k, 16) || !aligned(scores, 4)) return FB4_ERR_UNSUPPORTED;
    const bool small = tokens <= (int64_t)kScoreShortGroup;
    const int64_t per_wg = small ? 128 : 256;
    const int64_t bpg = (tokens + per_wg - 1) / per_wg;
    if (tokens * dim > 0x7FFFFFFFll || groups * bpg > 0x7FFFFFFFll) return FB4_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
#define FB4_SCORE_LAUNCH(d, relu, qb, keys) launch(attention_scores_kernel<d, relu, qb, keys>, grid, dim3(kScoreThreads), 0, s, qs, ks, (uint32_t)tokens, (uint32_t)dim, (uint32_t)bpg, grid.x, out)
#define FB4_SCORE_CASE(d, qb, keys)                          \
    case d:                                                  \
        if (mode) FB4_SCORE_LAUNCH(d, true, qb, keys);       \
        else FB4_SCORE_LAUNCH(d, false, qb, keys);           \
        break;
    if (small) {
        const uint32_t pieces = (uint32_t)(dim / 8);
        const uint32_t rows_per_task = tokens > 32 ? (uint32_t)tokens : (32u / (uint32_t)tokens) * (uint32_t)tokens;
        // One to four wavefronts per workgroup, at most 64 KiB of LDS: what puts most of them on a compute unit, up to
        // eight (24576 groups x 16 tokens x 128 channels: 37.7 us with four, 35.4 with eight, 38.0 with ten).
        const uint32_t per_wave = short_wave_bytes(rows_per_task, pieces);
        uint32_t waves = 1, most = 0;
        for (uint32_t w = 4; w >= 1; --w) {
            if (w * per_wave > 65536u) continue;
            const uint32_t n = std::min(163840u / (w * per_wave), 8u / w);
            if (n * w > most) { most = n * w; waves = w; }
        }
        const bool one_wave = scores_short_in_one_wave(groups, tokens, dim, most);
        // (row numbers are 32 bits in the one kernel, a launch takes fewer than 2^24 workgroups of the other: longer inputs
        // take several launches)
        const int64_t at_once = one_wave ? ((1ll << 30) / rows_per_task) * rows_per_task / tokens : 1ll << 23;
        for (int64_t g0 = 0; g0 < groups; g0 += at_once) {
            const int64_t n_groups = std::min(at_once, groups - g0);
            const uint16_t* qs = static_cast<const uint16_t*>(q) + (size_t)(g0 * tokens * dim);
            const uint16_t* ks = static_cast<const uint16_t*>(k) + (size_t)(g0 * tokens * dim);
            float* out = scores + g0 * tokens;
            if (!one_wave) {
                const dim3 grid((unsigned)n_groups);   // (bpg is 1)
                switch ((int)((dim + 31) / 32)) {
                    FB4_SCORE_CASE(1, 1, 32) FB4_SCORE_CASE(2, 1, 32) FB4_SCORE_CASE(3, 1, 32) FB4_SCORE_CASE(4, 1, 32)
                    FB4_SCORE_CASE(5, 1, 32) FB4_SCORE_CASE(6, 1, 32) FB4_SCORE_CASE(7, 1, 32) FB4_SCORE_CASE(8, 1, 32)
                }
                if (hipGetLastError() != hipSuccess) return FB4_ERR_HIP;
                continue;
            }
            const uint32_t n_rows = (uint32_t)(n_groups * tokens);
            const uint32_t n_tasks = (n_rows + rows_per_task - 1) / rows_per_task;
            if (n_tasks <= 256u) waves = 1;   // (a compute unit each: 64 groups x 32 x 112 2.90 us with four, 2.66 so)
            // every wavefront with the same number of tasks (6000 x 48 x 72: 16.3 us; with the last round ragged 17.5; for
            // 256 compute units, which decides speed only)
            const uint32_t rounds = (n_tasks + 256u * most - 1) / (256u * most);
            const dim3 sgrid((n_tasks + rounds * waves - 1) / (rounds * waves));
#define FB4_SHORT_CASE(p, n) case p: launch(attention_scores_short_kernel<p, n>, sgrid, dim3(64 * waves), waves * per_wave, s, qs, ks, n_rows, (uint32_t)tokens, rows_per_task, n_tasks, (uint32_t)mode, waves, sgrid.x, out); break;
#define FB4_SHORT_CASES(n)                                                                                                          \
    FB4_SHORT_CASE(1, n) FB4_SHORT_CASE(2, n) FB4_SHORT_CASE(3, n) FB4_SHORT_CASE(4, n) FB4_SHORT_CASE(5, n) FB4_SHORT_CASE(6, n)   \
    FB4_SHORT_CASE(7, n) FB4_SHORT_CASE(8, n) FB4_SHORT_CASE(9, n) FB4_SHORT_CASE(10, n) FB4_SHORT_CASE(11, n)                      \
    FB4_SHORT_CASE(12, n) FB4_SHORT_CASE(13, n) FB4_SHORT_CASE(14, n) FB4_SHORT_CASE(15, n) FB4_SHORT_CASE(16, n)
            if (tokens <= 32) {
                switch (pieces) {
                    FB4_SHORT_CASES(1)
                    FB4_SHORT_CASE(17, 1) FB4_SHORT_CASE(18, 1) FB4_SHORT_CASE(19, 1) FB4_SHORT_CASE(20, 1) FB4_SHORT_CASE(21, 1)
                    FB4_SHORT_CASE(22, 1) FB4_SHORT_CASE(23, 1) FB4_SHORT_CASE(24, 1) FB4_SHORT_CASE(25, 1) FB4_SHORT_CASE(26, 1)
                    FB4_SHORT_CASE(27, 1) FB4_SHORT_CASE(28, 1) FB4_SHORT_CASE(29, 1) FB4_SHORT_CASE(30, 1) FB4_SHORT_CASE(31, 1)
                    FB4_SHORT_CASE(32, 1)
                    default: return FB4_ERR_UNSUPPORTED;
                }
            } else {
                switch (pieces) {
                    FB4_SHORT_CASES(2)
                    default: return FB4_ERR_UNSUPPORTED;
                }
            }
#undef FB4_SHORT_CASES
#undef FB4_SHORT_CASE
            if (hipGetLastError() != hipSuccess) return FB4_ERR_HIP;
        }
        return FB4_OK;
    }
    if (dim <= 8 * kDmaMaxPieces) {   // (longer rows: too many registers for four blocks of queries)
        const uint32_t n_blk = (uint32_t)((tokens + 31) / 32);
        const uint32_t bpw = dma_blocks_per_wave(groups, n_blk, (uint32_t)dma_max_blocks((int)(dim / 8)));
        const uint32_t n_full = n_blk / (2 * bpw), n_wg = n_full + (n_blk % (2 * bpw) ? 1 : 0);
        const dim3 dgrid((unsigned)(groups * n_wg));
#define FB4_DMA_ARGS static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k), (uint32_t)groups, (uint32_t)tokens, n_full, bpw, scores
#define FB4_DMA_CASE(p)                                                                                                               \
    case p:                                                                                                                           \
        if (mode) launch(attention_scores_dma_kernel<p, true>, dgrid, dim3(kScoreThreads), 0, s, FB4_DMA_ARGS);         \
        else launch(attention_scores_dma_kernel<p, false>, dgrid, dim3(kScoreThreads), 0, s, FB4_DMA_ARGS);             \
        break;
        switch ((int)(dim / 8)) {
            FB4_DMA_CASE(1) FB4_DMA_CASE(2) FB4_DMA_CASE(3) FB4_DMA_CASE(4) FB4_DMA_CASE(5) FB4_DMA_CASE(6) FB4_DMA_CASE(7)
            FB4_DMA_CASE(8) FB4_DMA_CASE(9) FB4_DMA_CASE(10) FB4_DMA_CASE(11) FB4_DMA_CASE(12) FB4_DMA_CASE(13)
            FB4_DMA_CASE(14) FB4_DMA_CASE(15) FB4_DMA_CASE(16)
            default: return FB4_ERR_UNSUPPORTED;
        }
#undef FB4_DMA_CASE
#undef FB4_DMA_ARGS
        return hipGetLastError() == hipSuccess ? FB4_OK : FB4_ERR_HIP;
    }
    const dim3 grid((unsigned)(groups * bpg));
    const uint16_t *qs = static_cast<const uint16_t*>(q), *ks = static_cast<const uint16_t*>(k);
    float* out = scores;
    switch ((int)((dim + 31) / 32)) {
        FB4_SCORE_CASE(5, 2, 64) FB4_SCORE_CASE(6, 2, 64) FB4_SCORE_CASE(7, 2, 64) FB4_SCORE_CASE(8, 2, 64)
        default: return FB4_ERR_UNSUPPORTED;
    }
#undef FB4_SCORE_CASE
#undef FB4_SCORE_LAUNCH
    return hipGetLastError() == hipSuccess ? FB4_OK : FB4_ERR_HIP;
}

int fb4_select_salient_tokens(const float* scores, int64_t frames, int heads, int grid_h, int grid_w, int tile_h,
                              int tile_w, int32_t* rows_out, void* stream)
{
    if (frames < 0 || heads < 1 || grid_h < 1 || grid_w < 1 || tile_h < 1 || tile_w < 1) return FB4_ERR_INVALID_ARG;
    if (frames == 0) return FB4_OK;
    if (!scores || !rows_out) return FB4_ERR_INVALID_ARG;
    const int64_t tokens = (int64_t)grid_h * grid_w;
    if (tokens > (int64_t)kSelectMaxTokens || frames * tokens > 0x7FFFFFFFll || !aligned(scores, 4) || !aligned(rows_out, 4))
        return FB4_ERR_UNSUPPORTED;
    const int64_t th = std::min(tile_h, grid_h), tw = std::min(tile_w, grid_w), tile_rows = (grid_h + th - 1) / th;
    const uint32_t tile_columns = (uint32_t)((grid_w + tw - 1) / tw);
    const SelectShape shape = select_shape(frames, tile_rows, tile_columns, th * tw, th * grid_w);
    const int64_t per_frame = (tile_rows + shape.rows - 1) / shape.rows, workgroups = frames * per_frame;
    const bool small = std::min(shape.rows * th, (int64_t)grid_h) * grid_w <= 2048;   // (less LDS: more workgroups per compute unit)
    const int64_t at_once = 0xFFFFFFFFll / shape.threads;   // (a launch takes fewer than 2^32 threads)
    for (int64_t first = 0; first < workgroups; first += at_once) {
        const dim3 grid((unsigned)std::min(at_once, workgroups - first));
#define FB4_SELECT_LAUNCH(t, l, m, many) launch(select_salient_kernel<t, l, m, many>, grid, dim3(t), 0, static_cast<hipStream_t>(stream), scores, (uint32_t)heads, (uint32_t)grid_h, (uint32_t)grid_w, (uint32_t)tile_h, (uint32_t)tile_w, (uint32_t)tile_rows, tile_columns, (uint32_t)shape.rows, (uint32_t)per_frame, (uint32_t)first, rows_out)
#define FB4_SELECT_CASE(t, m)                                                              \
        if (shape.lanes == 16) FB4_SELECT_LAUNCH(t, 16, m, true);                          \
        else if (m == kSelectMaxTokens && heads < 24) FB4_SELECT_LAUNCH(t, 1, m, (m < kSelectMaxTokens)); \
        else FB4_SELECT_LAUNCH(t, 1, m, true);
        if (shape.threads == 128) { FB4_SELECT_CASE(128, 2048) }
        else if (shape.threads == 256) { if (small) { FB4_SELECT_CASE(256, 2048) } else { FB4_SELECT_CASE(256, kSelectMaxTokens) } }
        else { if (small) { FB4_SELECT_CASE(1024, 2048) } else { FB4_SELECT_CASE(1024, kSelectMaxTokens) } }
#undef FB4_SELECT_CASE
#undef FB4_SELECT_LAUNCH
        if (hipGetLastError() != hipSuccess) return FB4_ERR_HIP;
    }
    return FB4_OK;
}

int fb4_seda_assign(const void* q, const void* k, int joint, int64_t frames, int heads, int grid_h, int grid_w,
                    int64_t dim, const int32_t* anchors, int64_t n_anchors, int tile_h, int tile_w, int window,
                    int window_t, float threshold, int32_t* token_group, int32_t* anchor_group, float* window_scores,
                    void* stream)
{
    if (frames < 0 || heads < 1 || grid_h < 1 || grid_w < 1 || dim < 1 || n_anchors < 0 || window < 1 || window_t < 1 ||
        tile_h < 1 || tile_w < 1 || (joint != 0 && joint != 1))
        return FB4_ERR_INVALID_ARG;
    if (!(threshold == threshold)) return FB4_ERR_INVALID_ARG;
    if (!joint && window_t != 1) return FB4_ERR_INVALID_ARG;   // factorized attention has no scores across frames
    if (frames == 0) return FB4_OK;
    if (!token_group || !anchor_group || (n_anchors > 0 && (!q || !k || !anchors))) return FB4_ERR_INVALID_ARG;
    const int64_t tokens = (int64_t)grid_h * grid_w;
    if ((dim % 8) || window > 8 || window_t > 64 || !aligned(q, 16) || !aligned(k, 16) || !aligned(anchors, 4) ||
        !aligned(token_group, 4) || !aligned(anchor_group, 4) || (window_scores && !aligned(window_scores, 4)))
        return FB4_ERR_UNSUPPORTED;
    if (frames * tokens > 0x7FFFFFFFll || n_anchors > 0x7FFFFFFFll || tokens * dim > 0x7FFFFFFFll) return FB4_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint32_t n = (uint32_t)(frames * tokens);
    const uint32_t gh = (uint32_t)grid_h, gw = (uint32_t)grid_w, th = (uint32_t)tile_h, tw = (uint32_t)tile_w;
    const uint32_t n_prepare = (n + kPrepareRows - 1) / kPrepareRows;
    const bool one_buffer = token_group == anchor_group;
    auto own_groups = [&]() {
        if (n_anchors == 0) return;
        launch(seda_anchor_kernel, dim3((unsigned)((n_anchors + kAssignThreads - 1) / kAssignThreads)), dim3(kAssignThreads),
                           0, s, anchors, (uint32_t)n_anchors, (uint32_t)frames, gh, gw, th, tw, token_group, anchor_group);
    };
    if (n_anchors <= (int64_t)kPrepareMaxAnchors) {
        launch(seda_prepare_kernel, dim3(n_prepare), dim3(kAssignThreads), 0, s, anchors, (uint32_t)n_anchors, n,
                           (uint32_t)tokens, gw, th, tw, token_group, anchor_group);
    } else {
        launch(seda_fill_kernel, dim3((n + kAssignThreads - 1) / kAssignThreads), dim3(kAssignThreads), 0, s, token_group,
                           anchor_group, n);
        own_groups();
    }
    if (n_anchors > 0) {
        AssignParams p = {};
        p.frames = (uint32_t)frames; p.heads = (uint32_t)heads; p.grid_h = gh; p.grid_w = gw;
        p.dim = (uint32_t)dim; p.tile_h = th; p.tile_w = tw;
        p.window = (uint32_t)window; p.window_t = (uint32_t)window_t;
        p.stride_f = joint ? (uint64_t)tokens : (uint64_t)heads * tokens;
        p.stride_h = joint ? (uint64_t)frames * tokens : (uint64_t)tokens;
        p.threshold = threshold;
        const dim3 grid((unsigned)n_anchors, (unsigned)window_t);
        // As many lanes as a row has 16-byte pieces; with fewer heads than wavefronts at most 4, so that the wavefronts
        // that have a head take fewer steps.  us with 16 lanes for every row / now, 1024 anchors of 16 x 1024 tokens, 8 x 8
        // windows: 24 heads x 8 channels 25.9 / 10.0, x 32 channels 25.3 / 18.2, one head x 128 channels x 16 frames 77 / 27.
        int lanes = dim > 64 ? 16 : dim > 32 ? 8 : dim > 16 ? 4 : dim > 8 ? 2 : 1;
        if (heads < kAssignThreads / 64) lanes = std::min(lanes, 4);
#define FB4_MARK_LAUNCH(w, l) launch(seda_mark_kernel<w, l>, grid, dim3(kAssignThreads), 0, s, static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k), anchors, p, token_group, one_buffer ? nullptr : anchor_group, window_scores)
#define FB4_MARK_CASE(w)                                     \
        case w:                                              \
            if (lanes == 16) FB4_MARK_LAUNCH(w, 16);         \
            else if (lanes == 8) FB4_MARK_LAUNCH(w, 8);      \
            else if (lanes == 4) FB4_MARK_LAUNCH(w, 4);      \
            else if (lanes == 2) FB4_MARK_LAUNCH(w, 2);      \
            else FB4_MARK_LAUNCH(w, 1);                      \
            break;
        switch (window) {
            FB4_MARK_CASE(1) FB4_MARK_CASE(2) FB4_MARK_CASE(3) FB4_MARK_CASE(4)
            FB4_MARK_CASE(5) FB4_MARK_CASE(6) FB4_MARK_CASE(7) FB4_MARK_CASE(8)
        }
#undef FB4_MARK_CASE
#undef FB4_MARK_LAUNCH
        if (one_buffer) own_groups();
    }
    return hipGetLastError() == hipSuccess ? FB4_OK : FB4_ERR_HIP;
}

int fb4_seda_main_anchor(const float* temporal_scores, const void* qt, const void* kt, int64_t frames, int heads,
                         int grid_h, int grid_w, int64_t dim, const int32_t* candidates, int n_per_frame, int tile_h,
                         int tile_w, float prune_threshold, int32_t* main_anchor, int32_t* kept, float* prune_scores,
                         void* stream)
{
    if (frames < 0 || heads < 1 || grid_h < 1 || grid_w < 1 || dim < 1 || n_per_frame < 0 || tile_h < 1 || tile_w < 1)
        return FB4_ERR_INVALID_ARG;
    if (!(prune_threshold == prune_threshold)) return FB4_ERR_INVALID_ARG;
    if (!main_anchor) return FB4_ERR_INVALID_ARG;
    const int64_t tokens = (int64_t)grid_h * grid_w;
    const int64_t tiles = (int64_t)((grid_h + tile_h - 1) / tile_h) * ((grid_w + tile_w - 1) / tile_w);
    const int64_t n_cand = frames * n_per_frame;
    if (n_cand > 0 && (!temporal_scores || !qt || !kt || !candidates || !kept)) return FB4_ERR_INVALID_ARG;
    if ((dim % 8) || frames > (int64_t)kMainMaxFrames || !aligned(qt, 16) || !aligned(kt, 16) || !aligned(temporal_scores, 4) ||
        !aligned(candidates, 4) || !aligned(main_anchor, 4) || !aligned(kept, 4) || (prune_scores && !aligned(prune_scores, 4)))
        return FB4_ERR_UNSUPPORTED;
    if (frames * tokens > 0x7FFFFFFFll || n_cand > 0x7FFFFFFFll || frames * dim > 0x7FFFFFFFll) return FB4_ERR_UNSUPPORTED;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // A wavefront per frame, four at least.  Up to 16 while two workgroups per compute unit hold all tiles, else up to 8,
    // so that the next tiles do not wait for a whole workgroup of 16 (us with 4 / 8 / 16, 8 heads x 128 channels x 16
    // frames: 64 tiles 10.4 / 6.9 / 5.7, 256 tiles 14.5 / 9.2 / 7.3, 1024 tiles 45.5 / 36.6 / 44.2); a launch takes fewer
    // than 2^32 threads, so from 2^22 tiles on 4.
    const int64_t most = tiles <= 512 ? kMainMaxThreads : tiles <= (1 << 22) ? 512 : 256;
    const unsigned threads = (unsigned)std::min<int64_t>(std::max<int64_t>(frames, 4) * 64, most);
    // A tile's frames in parts, each with a workgroup that finds the tile's main anchor for itself, while a compute unit gets no
    // second one: what a compute unit has of loads in flight is what the pruning takes.  us, one part / so (graph, inputs changing):
    // 64 tiles x 16 frames x 24 heads x 128 channels 7.85 / 7.05, 16 tiles 7.25 / 6.4, 64 x 32 x 16 x 64 10.4 / 8.5, 4 x 32 x 8 x 128 7.8 /
    // 6.6.  Not for short rows (64 x 16 x 8 x 72 5.4 / 5.7, 65 x 12 x 12 x 64 5.65 / 6.2) nor where many tiles' parts come to different
    // XCDs (121 x 16 x 24 x 128 8.8 / 8.9), and not where `kept` overwrites the list that the other parts still read.  Two parts only
    // from 12 frames on (46 shapes there 0.88 on average, 35 with fewer frames 0.99 and up to 1.045).  500 shapes of 1 to 200 frames in
    // parts 0.83 of one part's time on average, at most 1.03; 500 in one part 1.00, at most 1.03.
    const uintptr_t from = reinterpret_cast<uintptr_t>(candidates), to = reinterpret_cast<uintptr_t>(kept);
    const bool in_place = from < to + n_cand * sizeof(int32_t) && to < from + n_cand * sizeof(int32_t);
    const bool worth = heads * dim >= 1024 && (tiles % 8 == 0 || tiles <= 32) && !in_place;
    int64_t most_parts = worth ? std::max<int64_t>(std::min<int64_t>(256 / tiles, frames), 1) : 1;   // (256 compute units)
    if (most_parts == 2 && frames < 12) most_parts = 1;
    const int64_t per_part = std::max<int64_t>((frames + most_parts - 1) / most_parts, 1);
    const int64_t parts = std::max<int64_t>((frames + per_part - 1) / per_part, 1);   // (each has a frame)
    launch(parts > 1 ? seda_main_anchor_kernel<true> : seda_main_anchor_kernel<false>, dim3((unsigned)tiles, (unsigned)parts), dim3(threads), 0, s, temporal_scores,
                       static_cast<const uint16_t*>(qt), static_cast<const uint16_t*>(kt), (uint32_t)frames, (uint32_t)heads,
                       (uint32_t)grid_h, (uint32_t)grid_w, (uint32_t)dim, candidates, (uint32_t)n_per_frame, (uint32_t)tile_h,
                       (uint32_t)tile_w, prune_threshold, main_anchor, kept, prune_scores, threads / 64u, (uint32_t)tiles,
                       main_anchor_split((uint32_t)per_part, (uint32_t)parts, threads / 64u, (uint32_t)heads));
    return hipGetLastError() == hipSuccess ? FB4_OK : FB4_ERR_HIP;
}

int fb4_seda_main_anchor_3d(const float* scores, int64_t frames, int heads, int grid_h, int grid_w, int tile_h,
                            int tile_w, int32_t* anchors, void* stream)
{
    if (frames < 1 || heads < 1 || grid_h < 1 || grid_w < 1 || tile_h < 1 || tile_w < 1) return FB4_ERR_INVALID_ARG;
    if (!scores || !anchors) return FB4_ERR_INVALID_ARG;
    const int64_t tokens = (int64_t)grid_h * grid_w;
    const int64_t tiles = (int64_t)((grid_h + tile_h - 1) / tile_h) * ((grid_w + tile_w - 1) / tile_w);
    if (frames * tokens > 0x7FFFFFFFll || !aligned(scores, 4) || !aligned(anchors, 4)) return FB4_ERR_UNSUPPORTED;
    launch(seda_main_anchor_3d_kernel, dim3((unsigned)tiles), dim3(kMainThreads), 0,
                       static_cast<hipStream_t>(stream), scores, (uint32_t)frames, (uint32_t)heads, (uint32_t)grid_h,
                       (uint32_t)grid_w, (uint32_t)tile_h, (uint32_t)tile_w, anchors);
    return hipGetLastError() == hipSuccess ? FB4_OK : FB4_ERR_HIP;
}

int fb4_probe_mfma_rate(int64_t workgroups, int64_t iterations, int random_operands, float* out, double* flop, void* stream)
{
    if (workgroups < 1 || workgroups > 65536 || iterations < 0 || iterations > 0x7FFFFFFFll || !out) return FB4_ERR_INVALID_ARG;
    if (!aligned(out, 4)) return FB4_ERR_UNSUPPORTED;
    launch(probe_mfma_rate_kernel, dim3((unsigned)workgroups), dim3(256), 0, static_cast<hipStream_t>(stream), out,
                       (uint32_t)iterations, (uint32_t)(random_operands != 0));
    // four wavefronts x 8 x 4 MFMAs of 32 x 32 x 16 per iteration, two operations per multiply-add
    if (flop) *flop = (double)workgroups * 4.0 * (double)iterations * 32.0 * (2.0 * 32 * 32 * 16);
    return hipGetLastError() == hipSuccess ? FB4_OK : FB4_ERR_HIP;
}

}  // extern "C"
