// Which GEMM kernel takes a call and in what passes: plain C++ without HIP, so that a host compiler can check it.
// Every choice leaves a row's sums as they are; these rules decide about time alone.
#pragma once
#include <stdint.h>

// Row tiles per pass of the few-row kernel before short passes: 32 ... 192 rows in steps of 32 take one pass; more rows take
// passes of 160 or 192 rows, whichever needs fewer.
inline int gemm_full_pass(int M) {
    const int tiles = (M + 31) / 32;
    return tiles <= 6 ? tiles : (M + 191) / 192 < (M + 159) / 160 ? 6 : 5;
}

// The large tiles of k_gemm_rows, weight rows x activation rows.  The small ones, 256 x 96, 128 and 160, are named by their
// 3, 4 or 5 row tiles of 32.
enum GemmWideTile { GEMM_256x256 = 256256, GEMM_192x320 = 192320, GEMM_192x256 = 192256 };
// Tiles that walk one half of the k-slices and add their sums, so that two partial sums leave the kernel.
enum GemmHalvesTile { GEMM_HALVES_256x128 = 2256128, GEMM_HALVES_192x128 = 2192128 };

// One of the large tiles where it is the fastest way for M rows, or 0: gemm_rows_tile() and gemm_few_row_pass() choose.
// nch: chunks of 64 columns in a k-slice; wn: as below.
// Time of a launch = rounds over the 256 CUs x (fixed + chunks x a) + share of the chip's work-group slots x chunks x b, since
// a round that fills the chip only partly draws less power and clocks higher.  Fitted, ns, to gate/up of the 8B shape at 193
// to 2304 rows (64 chunks; one round of half the chip / of the whole chip, two rounds of it, us: 192 x 256 68 / 86, 171;
// 192 x 320 77 / 100, 195; 256 x 256 at 192 work-groups 89, at 512 and 768 - / - , 184 / 318).  Over the four matrices of the 8B and
// the 7B class and the LM head, 193 to 2304 rows, the choice was within 4 % of the fastest tile but for 8 % at down, 256 rows.
// At least 128 work-groups: fewer leave half of the chip idle, and the few-row kernel's narrower n-blocks spread better.
inline int gemm_wide_tile(int M, int N, int nch, int split, int wn, long long* time = nullptr) {
    if (M <= 192) return 0;
    struct Kind { int code, nt, mt, a, b; };
    static const Kind kinds[6] = {{GEMM_256x256, 8, 8, 840, 620}, {GEMM_192x320, 6, 10, 656, 750}, {GEMM_192x256, 6, 8, 625, 560},
                                  {0, 8, 4, 560, 250}, {0, 8, 5, 690, 230}, {0, 8, 3, 470, 190}};
    const long long fixed = 10000;
    int best = 0;
    long long best_time = -1;
    for (const Kind& k : kinds) {
        const long long wgs = (long long)((N / 32 + k.nt - 1) / k.nt) * split * ((M + k.mt * 32 - 1) / (k.mt * 32));
        const long long t = (wgs + 255) / 256 * (fixed + (long long)nch * k.a) + wgs * nch * k.b / 256;
        if (wgs >= 128 && (best_time < 0 || t < best_time)) { best = k.code; best_time = t; }
    }
    // the few-row kernel's passes of 160 or 192 rows
    const int mt = gemm_full_pass(M);
    const long long wgs = (long long)((N / 32 + wn - 1) / wn) * split * ((M + mt * 32 - 1) / (mt * 32));
    const long long few = (wgs + 255) / 256 * (4000 + (long long)nch * (mt == 6 ? 630 : 560)) * wn / 3;
    if (wgs >= 256 && few < best_time) { best = 0; best_time = few; }
    if (time) *time = best_time;
    return best;
}

// One of the tiles that walk half of the k-slices (fp32 partial sums only), or 0.  They hold two accumulators per output, so the
// tile is half as large and the kernel alone no faster (8B down, 1000 rows 97 us in eight slices / 102 in halves; 640 rows 70 /
// 75; 7B class down, 2304 rows 278 / 292); what they save is the other partial sums: 0.08 us to write and 0.16 us to read
// per MB each (norm of 1000 rows x 4096: 26 us with eight, 11 with two).  Time of a launch as above, with ns of their own.
inline int gemm_halves_tile(int M, int N, int nch, int split, int wn) {
    if (M <= 192 || split <= 2) return 0;
    struct Kind { int code, nt, mt, a, b; };
    static const Kind kinds[2] = {{GEMM_HALVES_256x128, 8, 4, 750, 250}, {GEMM_HALVES_192x128, 6, 4, 550, 170}};
    const long long fixed = 6000, kb = (long long)M * N * 4 / 1000, chunks = (long long)nch * ((split + 1) / 2);
    long long best_time = -1;
    gemm_wide_tile(M, N, nch, split, wn, &best_time);
    if (best_time < 0) return 0;
    best_time += split * kb * 24 / 100;
    int best = 0;
    for (const Kind& k : kinds) {
        const long long wgs = (long long)((N / 32 + k.nt - 1) / k.nt) * 2 * ((M + k.mt * 32 - 1) / (k.mt * 32));
        const long long t = (wgs + 255) / 256 * (fixed + chunks * k.a) + wgs * chunks * k.b / 256 + 2 * kb * 16 / 100;
        if (wgs >= 128 && t < best_time) { best = k.code; best_time = t; }
    }
    return best;
}

// Row tiles (of 32 rows) per work-group of k_gemm_rows with 256 weight rows, or 0: the few-row kernel takes the call, in
// n-blocks of wn tiles.  Asked where no large tile is the fastest.
// Up to 192 rows the few-row kernel needs one pass over the weights and every CU streams its own share of them;
// beyond that it re-streams them per pass (8B shape, 193 rows, us, few-row / 128 rows: gate/up 80 / 57, QKV 46 / 33, down 40 /
// 33).  Fewer than 128 work-groups leave half of the chip idle: then the
// few-row kernel's narrower n-blocks spread better.  Among the tiles the fewest rounds over the 256 CUs win, a
// round of 96, 128 or 160 rows costing 0.84 : 1 : 1.11 (gate/up at 256 to 640 rows: 48, 57 and 65 us a round).
// The few-row kernel's 96-row n-blocks, where they fill the chip, count along: a round of 160 or 192 rows costs 0.65 or
// 0.75 there (320 and 384 rows in two passes: 82 and 89 us).
// X, the activations, must start on 16 bytes (their rows then do: K is a multiple of 64): the kernels copy them to LDS in
// 16-byte pieces (launch_gemm_mfma sees to it that they do).
inline int gemm_rows_tile(const void* X, int M, int N, int split, int wn) {
    if (M <= 192 || ((uintptr_t)X & 15)) return 0;
    const int n_blocks = (N / 32 + 7) / 8, cost[3] = {84, 100, 111};
    int best = 0, best_cost = 0;
    for (int mt = 3; mt <= 5; ++mt) {
        const long long wgs = (long long)n_blocks * split * ((M + mt * 32 - 1) / (mt * 32));
        const long long c = (wgs + 255) / 256 * cost[mt - 3];
        if (wgs >= 128 && (best == 0 || c < best_cost)) { best = mt; best_cost = (int)c; }
    }
    const long long blocks = (long long)((N / 32 + wn - 1) / wn) * split;
    if (wn == 3 && blocks >= 256) {
        const int mt = gemm_full_pass(M);
        if ((blocks * ((M + mt * 32 - 1) / (mt * 32)) + 255) / 256 * (mt == 6 ? 75 : 65) < best_cost) return 0;
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

// Small matrices, whose n-blocks leave more than half of the CUs idle, take shorter passes until 128 work-groups
// run: a work-group's time is its K walk times its row tiles
// (192 rows, K = 512, us, one pass / short passes: gate/up of 1536 channels 17 / 7.3, LM head of 2080 tokens 14.7 / 9.4,
// attention output 10 / 4.7).
inline GemmPass gemm_few_row_pass(int M, int N, int split, int wn) {
    const int tiles = (M + 31) / 32, blocks = (N / 32 + wn - 1) / wn * split;
    int mt = gemm_full_pass(M);
    while (mt > 1 && (long long)blocks * ((tiles + mt - 1) / mt) < 128) --mt;
    const int passes = (tiles + mt - 1) / mt;
    return GemmPass{mt, passes, passes > 1};
}

// Plain GEMM: k_gemm_plain_small may take the call while k_gemm_plain's 64x64 tiles would give a CU at most one work-group.
// Unaligned operands (kernel-level entry points take any pointer) stay with the scalar loads.
#define GEMM_PLAIN_TILE 64
inline bool gemm_plain_small_tiles(const void* X, const void* W, int M, int N) {
    const long long tiles = (long long)((N + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) * ((M + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE);
    return tiles <= 256 && (((uintptr_t)X | (uintptr_t)W) & 15) == 0;
}

// It does for up to 64 rows, and for more rows up to 160 tiles: its 16 rows share nothing, so every 16 rows read the weights
// again (us, 64x64 tiles / small ones; up to 64 rows: 60 tiles 12.7 / 6.4, 125 tiles 43 / 30, 192 tiles 4096 wide 172 / 106 and 257 /
// 220; more rows: 120 tiles 13.2 / 11.7, 144 tiles 36 / 32, 160 tiles 54 / 45, 176 tiles 40 / 43, 192 tiles 20 / 25, 256
// tiles 40 / 60).
inline bool gemm_plain_small_wins(int M, int N) {
    return M <= 64 || (long long)((N + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) * ((M + GEMM_PLAIN_TILE - 1) / GEMM_PLAIN_TILE) <= 160;
}

// Attention: work-groups of four waves, two to a CU, where eight-wave ones would take more than one round over the 256 CUs
// (8B shape, us, eight waves / four: 576 work-groups of 64-row blocks 33.6 / 27.7, 640 at prefix 1152 59 / 48, 1000-row
// prompt 50 / 39, refresh of 512 rows 43 / 31; 160 work-groups 13.2 / 13.0, 32 at prefix 1000 18.2 / 19.0).
inline bool attn_two_per_cu(long long work_groups) { return work_groups > 256; }

// Plain attention, one wave per row and query head: whether a wave takes a SIMD's whole register file for loads in flight.  The 1024
// SIMDs have one wave each up to 1024 waves; two channels per lane (head size 128) hold twice the values, in bf16 at no gain.
// Rotary stage and attention, us, deep / not, prefix 384: head size 64, fp32 1024 waves 34.3 / 39.9, 1536 44.3 / 42.8, 4096 71 / 54,
// bf16 1024 waves 34.5 / 35.8, 1536 46.7 / 38.3; head size 128, fp32 512 waves 35.5 / 38.5, 768 40.1 / 40.7 (prefix 16: 29.4 / 25.6),
// 1024 45 / 42, 5120 122 / 94, bf16 256 waves 45 / 39, 5120 177 / 81.
inline bool attn_plain_deep(long long waves, int head_dim, int element_bytes) {
    return head_dim == 64 ? waves <= 1024 : element_bytes == 4 && waves <= 512;
}
