// The MFMA GEMM for forwards with many rows.  Shared by the translation units that instantiate it, one per epilogue.
#pragma once
#include "gemm_mfma.h"

// Work-group = WN x WM waves, one per SIMD, with the whole register file: wave (wn, wm) owns R adjacent n-tiles of 32 weight
// rows x TW adjacent row tiles, one chain of MFMAs per output over all columns of the k-slice, in the order of k_gemm_mfma:
// a row's sums are bit for bit those of the few-row kernel.
// Weights and activations go global -> LDS without passing through registers, in chunks of 64 columns and rings of NSW and
// NSX stages (whichever of LDS is left over goes to the weights, which come from HBM).  One barrier per chunk: chunk c has
// landed and everyone has read chunk c - 1, whose stages are loaded again in the four steps of 16 columns that follow.
//
// Bound by the matrix cores' power: a chunk of the 192 x 320 tile takes 1.43 us (1.41 PFLOP/s over the chip), without its
// loads 1.22 us (1.65; MFMAs alone on random operands, from registers, reach 1.65 to 1.75 and on zeros 2.3), and a
// launch about 10 us on top: ramp, first chunk, epilogue.  Why these tiles: bytes per operation are what the loads cost, and a
// grid that is a whole number of rounds over the 256 CUs (gemm_tile).  8B shape, us, before (256 x 128 in eight waves,
// two chains per output, which fill the register file at half the tile) / now: gate/up 512 rows 123 / 86, 576 rows 117 /
// 100, 640 rows 121 / 103, 1000 rows 186 / 171; QKV 640 rows 69.5 / 59, down 512 rows 61 / 50, 640 rows 77 / 66.
// HALF (fp32 partial sums): half of the k-slices one after the other, each a chain of its own, added as the consumers add partial
// sums: two leave the kernel instead of one per slice (gemm_tile).
// Fragments are read and loads issued one by one between MFMAs (all of a step's reads first and loads where the compiler left
// them: 1.58 us a chunk); eight waves on 256 x 256, two per SIMD, are no faster than four.
template <int WN, int WM, int R, int TW, int EPI, int NSX, int NSW, bool HALF>
__global__ __launch_bounds__(WN* WM * 64) void k_gemm_rows(const bf16_t* X, const uint4* Wp, void* outv, int M, int N, int K,
                                                           int k_len, size_t split_stride, int mask_id, int n_tiles_out,
                                                           int n_blocks, int n_split, int m_chunks, int n_slices) {
    constexpr int NW = WN * WM, KC = 64, KSTEPS = KC / 16, NB = WN * R, MT = WM * TW, ROWS = MT * 32;
    constexpr int WB = NB * KSTEPS * 1024, XB = ROWS * KC * 2, XBASE = NSW * WB;        // bytes of a stage; the activations' ring
    constexpr int WL = WB / 1024 / NW, XL = XB / 1024 / NW;                             // loads of a stage per wave
    static_assert(WB % (1024 * NW) == 0 && XB % (1024 * NW) == 0, "every wave issues the same loads");
    static_assert(NSX >= 2 && NSW >= NSX && XL * (NSX - 1) + WL * (NSW - 1) < 64, "ring depths");
    extern __shared__ uint4 smem_u4[];
    char* const smem = (char*)smem_u4;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave % WN, wm = wave / WN, lm = lane & 31, lh = lane >> 5;
    // Work-groups go to the 8 XCDs round-robin by their linear id.  Every XCD takes a contiguous range of
    // tiles, ordered by k-slice, n-block, row chunk: the row chunks of an n-block run side by side and share
    // its weights in that XCD's L2, and neighbouring n-blocks share the activations.
    int bx, by, bz;
    {
        const int total = n_blocks * m_chunks * n_split, id = blockIdx.x;
        const int xcd = id & 7, q = total >> 3, rem = total & 7;
        const int t = xcd * q + (xcd < rem ? xcd : rem) + (id >> 3);
        by = t % m_chunks;
        bx = (t / m_chunks) % n_blocks;
        bz = t / (m_chunks * n_blocks);
    }
    // HALF: this work-group walks one half of the n_slices k-slices, one after the other, and adds their sums
    const int nch = k_len / KC, first = HALF ? bz * ((n_slices + 1) >> 1) : bz;
    const int slices = HALF ? (bz == 0 ? (n_slices + 1) >> 1 : n_slices >> 1) : 1;
    const int m0 = by * ROWS, kbeg = first * k_len, nchunks = nch * slices;
    const int KS = K >> 4, NT = N >> 5;
    // Load i of this wave is piece wave + NW i of a stage, 1 KB: of the n-tiles' fragments, or eight rows of the
    // activations, the 16-byte piece s of row r in slot s ^ (r / 2 % 8) of its line, so that the 32 rows of a
    // fragment spread over all LDS banks.  n-tiles and rows past the end read the last one (never stored).
    const char* xrow0 = (const char*)(X + (size_t)m0 * K + kbeg);
    unsigned xoff[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        const int r = (wave + NW * i) * 8 + (lane >> 3), s = (lane & 7) ^ ((r >> 1) & 7);
        xoff[i] = (unsigned)(m0 + r < M ? r : M - 1 - m0) * (unsigned)(K * 2) + s * 16;
    }
    auto issue_w = [&](int i, int slot, int at) SSD_INLINE {        // at: the chunk, counted from kbeg, rotated within its slice
        const int p = wave + NW * i, t = bx * NB + p / KSTEPS, n = t < NT ? t : NT - 1;
        load_to_lds<false>(lds0 + slot * WB + p * 1024, lane * 16, Wp + ((size_t)n * KS + (kbeg >> 4) + at * KSTEPS + p % KSTEPS) * 64);
    };
    auto issue_x = [&](int i, int slot, int at) SSD_INLINE {
        load_to_lds<false>(lds0 + XBASE + slot * XB + (wave + NW * i) * 1024, xoff[i], xrow0 + (size_t)at * (KC * 2));
    };
    struct Walk { int at, done, slice; };                // the next chunk to load: where, how many of its slice before it
    auto begin = [&](int slice) SSD_INLINE { return slice * nch + gemm_k_start(bx * (NB * 32), first + slice, nch); };
    auto advance = [&](Walk& w) SSD_INLINE {
        if (HALF && ++w.done == nch) {
            w.done = 0;
            w.at = begin(++w.slice);
        } else {
            ++w.at;
            if (w.at == (w.slice + 1) * nch) w.at -= nch;
        }
    };
    Walk wx{begin(0), 0, 0}, ww = wx;

    floatx16 acc[R][TW];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < TW; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][t][i] = 0.f;
    floatx16 total[HALF ? R : 1][HALF ? TW : 1];         // the finished slices
    if constexpr (HALF)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < TW; ++t) total[r][t] = acc[r][t];
    auto close = [&]() SSD_INLINE {                      // the end of a slice
        if constexpr (HALF)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int t = 0; t < TW; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        total[r][t][i] += acc[r][t][i];
                        acc[r][t][i] = 0.f;
                    }
    };
    const int sw = (lm >> 1) & 7;
    struct Frags { bf16x8 w[R], x[TW]; } fa, fb;
    auto read1 = [&](Frags& f, auto jc, int slotx, int slotw, int ks) SSD_INLINE {       // fragment j of a step: weights, then rows
        constexpr int j = decltype(jc)::value;
        if constexpr (j < R) f.w[j] = *(const bf16x8*)(smem + slotw * WB + ((wn * R + j) * KSTEPS + ks) * 1024 + lane * 16);
        else f.x[j - R] = *(const bf16x8*)(smem + XBASE + slotx * XB + (wm * TW + j - R) * 4096 + lm * 128 + (((ks * 2 + lh) ^ sw) << 4));
    };
    // step q behind the barrier: its MFMAs; between them, one at a time so that a wave does not queue for the LDS or the
    // address unit while its matrix core idles, the next step's fragments (16 columns q of the chunk whose ring stages are rx,
    // rw) and its share of the loads into stages slotx, slotw: activations in step 0, weights in steps 1 to 3
    auto step = [&](auto qc, const Frags& f, Frags& g, int rx, int rw, int slotx, int slotw, bool more, bool loadx, bool loadw) SSD_INLINE {
        constexpr int q = decltype(qc)::value, NM = R * TW;
        constexpr int l0 = q == 0 ? 0 : q == 1 ? XL : XL + (q - 1) * WL / 3, l1 = q == 0 ? XL : XL + q * WL / 3;
        static_for<0, NM>([&](auto ic) SSD_INLINE {
            constexpr int i = decltype(ic)::value, r = i / TW, t = i % TW;
            acc[r][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w[r], f.x[t], acc[r][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i < R + TW) {
                if (more) read1(g, ic, rx, rw, q);
            }
            constexpr int a = l0 + i * (l1 - l0) / NM, b = l0 + (i + 1) * (l1 - l0) / NM;
            static_for<a, b>([&](auto kc) SSD_INLINE {
                constexpr int k = decltype(kc)::value;
                if constexpr (k < XL) { if (loadx) issue_x(k, slotx, wx.at); }
                else { if (loadw) issue_w(k - XL, slotw, ww.at); }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<NM, (NM > R + TW ? NM : R + TW)>([&](auto jc) SSD_INLINE { if (more) read1(g, jc, rx, rw, q); });
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int u = 0; u < NSW; ++u)
        if (u < nchunks) {
            if (u < NSX) {
#pragma unroll
                for (int i = 0; i < XL; ++i) issue_x(i, u, wx.at);
                advance(wx);
            }
#pragma unroll
            for (int i = 0; i < WL; ++i) issue_w(i, u, ww.at);
            advance(ww);
        }
    if (nchunks >= NSW) wait_and_meet<XL*(NSX - 1) + WL * (NSW - 1)>();
    else wait_and_meet<0>();
    static_for<0, R + TW>([&](auto jc) SSD_INLINE { read1(fa, jc, 0, 0, 0); });
    int sx = 0, sw_ = 0, in_slice = 0;
    constexpr std::integral_constant<int, 0> Q0{};
    constexpr std::integral_constant<int, 1> Q1{};
    constexpr std::integral_constant<int, 2> Q2{};
    constexpr std::integral_constant<int, 3> Q3{};
    // three steps of a chunk, whose first fragments are on their way
    auto three_steps = [&](int px, int pw, bool loadx, bool loadw) SSD_INLINE {
        step(Q1, fa, fb, sx, sw_, px, pw, true, loadx, loadw);
        step(Q2, fb, fa, sx, sw_, px, pw, true, loadx, loadw);
        step(Q3, fa, fb, sx, sw_, px, pw, true, loadx, loadw);
    };
    // from the barrier in front of chunk c on: the last step of chunk c - 1, whose stage is free, and three of chunk c
    auto period = [&](bool loadx, bool loadw) SSD_INLINE {
        const int px = sx, pw = sw_;
        sx = sx + 1 == NSX ? 0 : sx + 1;
        sw_ = sw_ + 1 == NSW ? 0 : sw_ + 1;
        step(Q0, fb, fa, sx, sw_, px, pw, true, loadx, loadw);
        if (HALF && ++in_slice == nch) {
            close();
            in_slice = 0;
        }
        three_steps(px, pw, loadx, loadw);
        advance(wx);
        advance(ww);
    };
    three_steps(0, 0, false, false);
    int c = 1;
    for (; c - 1 + NSW < nchunks; ++c) {
        wait_and_meet<(NSX - 2) * (XL + WL) + (NSW > NSX ? WL : 0)>();
        period(true, true);
    }
    for (; c < nchunks; ++c) {
        wait_and_meet<0>();
        period(c - 1 + NSX < nchunks, false);
    }
    step(Q0, fb, fa, 0, 0, 0, 0, false, false, false);
    close();
    __syncthreads();                                     // the epilogue reuses the ring

    // ---- epilogue.  Lane (lm, lh) holds, per tile, rows n = 8*(i/4) + 4*lh + i%4 of column m = lm.
    static_for<0, R * TW>([&](auto ic) SSD_INLINE {
        constexpr int j = decltype(ic)::value, r = j / TW, ti = j % TW;
        const int nt = bx * NB + wn * R + r, mt0 = m0 + (wm * TW + ti) * 32;
        const bool ok = nt < NT;                         // tiles and rows past the end are computed, but not stored
        const floatx16& v = HALF ? total[HALF ? r : 0][HALF ? ti : 0] : acc[r][ti];
        [[maybe_unused]] const int m = mt0 + lm;
        if constexpr (EPI == EPI_F32) {
            // through LDS into row order (4 KB per wave and parity of the tile), so that a store covers whole 128-byte
            // lines of 8 rows; piece s of row r lies in slot s ^ (r % 8)
            float4* t = (float4*)smem_u4 + (wave * 2 + (j & 1)) * 256;
            wave_lds_order();                            // every lane has read what is overwritten next
#pragma unroll
            for (int g = 0; g < 4; ++g)
                t[lm * 8 + ((g * 2 + lh) ^ (lm & 7))] = make_float4(v[g * 4], v[g * 4 + 1], v[g * 4 + 2], v[g * 4 + 3]);
            wave_lds_order();                            // other lanes wrote what is read next
            float* out = (float*)outv + (size_t)bz * split_stride + nt * 32 + (lane & 7) * 4;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r = g * 8 + (lane >> 3), row = mt0 + r;
                const float4 o = t[r * 8 + ((lane & 7) ^ (r & 7))];
                if (ok && row < M) *(float4*)(out + (size_t)row * N) = o;
            }
        } else if constexpr (EPI == EPI_SWIGLU) {
            bf16_t* out = (bf16_t*)outv;
            if (ok && m < M) {
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    float o[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[k] = swiglu(v[g * 4 + k], v[(g + 2) * 4 + k]);
                    *(uint2*)(out + (size_t)m * (N >> 1) + nt * 16 + g * 8 + lh * 4) = make_uint2(bf16_pair(o[0], o[1]), bf16_pair(o[2], o[3]));
                }
            }
        } else {
            float p[3];
            lm_tile_partial(v, nt, lh, mask_id, p);
            if (lh == 0 && ok && m < M) {
                float* o = (float*)outv + ((size_t)m * n_tiles_out + nt) * 3;
                o[0] = p[0]; o[1] = p[1]; o[2] = p[2];
            }
        }
    });
}

// HALF: a work-group per half of the a.split k-slices instead of one per slice
template <int WN, int WM, int R, int TW, int EPI, bool HALF = false>
static bool launch_rows(const GemmArgs& a) {
    constexpr int wst = WN * R * 4, xst = WM * TW * 4;                                  // KB of a stage
    constexpr int NSX = 2 * (wst + xst) + (wst + xst) <= 160 ? (160 / (wst + xst) >= 4 ? 4 : 160 / (wst + xst)) : 2;
    constexpr int left = (160 - NSX * xst) / wst, NSW = left > 4 ? 4 : left;
    constexpr size_t smem = (size_t)(NSX * xst + NSW * wst) * 1024;
    auto kern = k_gemm_rows<WN, WM, R, TW, EPI, NSX, NSW, HALF>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess)
            return false;
        attr_done = true;
    }
    const int n_blocks = (a.N / 32 + WN * R - 1) / (WN * R), m_chunks = (a.M + WM * TW * 32 - 1) / (WM * TW * 32);
    const int parts = HALF ? 2 : a.split;
    hipLaunchKernelGGL(kern, dim3(n_blocks * m_chunks * parts), dim3(WN * WM * 64), smem, a.st, a.X, a.Wp, a.out, a.M, a.N, a.K,
                       a.K / a.split, a.split_stride, a.mask_id, a.n_tiles_out, n_blocks, parts, m_chunks, a.split);
    return true;
}

template <int EPI>
static bool launch_tile(const GemmArgs& a, int tile) {
    if constexpr (EPI == EPI_F32) {
        if (tile == GEMM_HALVES_256x128) return launch_rows<2, 2, 4, 2, EPI, true>(a);
        if (tile == GEMM_HALVES_192x128) return launch_rows<2, 2, 3, 2, EPI, true>(a);
    }
    switch (tile) {
        case GEMM_256x256: return launch_rows<2, 2, 4, 4, EPI>(a);
        case GEMM_192x320: return launch_rows<2, 2, 3, 5, EPI>(a);
        case GEMM_192x256: return launch_rows<2, 2, 3, 4, EPI>(a);
        case GEMM_256x96: return launch_rows<4, 1, 2, 3, EPI>(a);
        case GEMM_256x128: return launch_rows<2, 2, 4, 2, EPI>(a);
        case GEMM_256x160: return launch_rows<4, 1, 2, 5, EPI>(a);
    }
    return false;
}
