// Which MFMA GEMM kernel takes a call and in what passes: plain C++ without HIP, so that a host compiler can check it.
// Every choice leaves a row's sums as they are; these rules decide about time alone.
#pragma once

// Row tiles (of 32 rows) per work-group of k_gemm_rows, or 0: the few-row kernel takes the call.
// Up to 192 rows the few-row kernel needs one pass over the weights and every CU streams its own share of them;
// beyond that it re-streams them per pass (gate/up of the 8B shape, us, few-row against k_gemm_rows: 200 rows 83 / 60,
// 576 rows 150 / 114, 1000 rows 283 / 178).  Fewer than 128 work-groups leave half of the chip idle: then the
// few-row kernel's narrower n-blocks spread better.  Among the tiles the fewest rounds over the 256 CUs win, a
// round of 96, 128 or 160 rows costing 0.78 : 1 : 1.3 (measured at 640 and 1000 rows: 47, 59 and 78 us a
// round; the 160-row tile has registers for one weight chunk in flight only, the others for three).
inline int gemm_rows_tile(int M, int N, int split) {
    if (M <= 192) return 0;
    const int n_blocks = (N / 32 + 7) / 8, cost[3] = {78, 100, 130};
    int best = 0, best_cost = 0;
    for (int mt = 3; mt <= 5; ++mt) {
        const long long wgs = (long long)n_blocks * split * ((M + mt * 32 - 1) / (mt * 32));
        const long long c = (wgs + 255) / 256 * cost[mt - 3];
        if (wgs >= 128 && (best == 0 || c < best_cost)) { best = mt; best_cost = (int)c; }
    }
    return best;
}

// How the few-row kernel takes M rows: `passes` passes of `mt` row tiles of 32 rows.
struct GemmPass {
    int mt, passes;
    // Weights are loaded with the default cache policy where several passes read them: the passes of an n-block run
    // side by side on one XCD and find them in its L2.  One pass loads them non-temporally, so that they do not evict
    // the activations.  Non-temporal / default, us: QKV of a 1600-wide model, 512 rows 34.1 / 29.5, its attention output,
    // 1152 rows 33.0 / 26.8, its gate/up, 64 rows in two passes 20.7 / 17.4; gate/up of a 1024-wide model, 448 rows
    // 18.7 / 15.4.  No matrix of the widths 512, 1024, 1600 and 2048 is faster with non-temporal loads in several passes.
    bool cached;
};

// 32 ... 192 rows in steps of 32 take one pass; more rows (of matrices too small for k_gemm_rows) take passes of 160 or 192
// rows, whichever needs fewer.
// Small matrices, whose n-blocks leave more than half of the CUs idle, take shorter passes until 128 work-groups
// run: a work-group's time is its K walk times its row tiles
// (192 rows, K = 512, us, one pass / short passes: gate/up of 1536 channels 17 / 7.3, LM head of 2080 tokens 14.7 / 9.4,
// attention output 10 / 4.7).
inline GemmPass gemm_few_row_pass(int M, int N, int split, int wn) {
    const int tiles = (M + 31) / 32, blocks = (N / 32 + wn - 1) / wn * split;
    int mt = tiles;
    if (mt > 6) mt = (M + 191) / 192 < (M + 159) / 160 ? 6 : 5;
    while (mt > 1 && (long long)blocks * ((tiles + mt - 1) / mt) < 128) --mt;
    const int passes = (tiles + mt - 1) / mt;
    return GemmPass{mt, passes, passes > 1};
}
