// The MFMA GEMM for forwards with many rows: 256 weight rows x (32 MT) activation rows per work-group.
// Shared by the translation units that instantiate it, one per epilogue.
#pragma once
#include "gemm_mfma.h"

// Work-group = 8 waves, two per SIMD: 4 along the weight rows x the 2 k-slices of a chunk.  Wave (wn, wk) owns two
// n-tiles of 32 weight rows, all MT row tiles, and of every 64-column chunk the columns [32wk, 32wk + 32): the
// same two chains of MFMAs per output, over the same chunks in the same order, as in k_gemm_mfma, added at the
// end.  A row's sums are therefore bit for bit those of the few-row kernel.
//   weights      global -> registers, a ring of DW chunks, every fragment requested once per work-group;
//   activations  global -> LDS without passing through registers (16 bytes per lane), a ring of NST stages.  A
//                stage holds whole 128-byte lines, row by row; the 16-byte piece s of row r lies in slot
//                s ^ (r / 2 % 8) of its line, so that the 32 rows of a fragment spread over all LDS banks.
//                The loads are issued by inline assembly (no output registers): the compiler would make every
//                LDS read wait for the newest of them.  It does not count them either: the waits before
//                a stage is read are written out, and its own waits for weights come out as too long, never
//                as too short.
// One barrier per chunk c: it tells that chunk c + 1 is in LDS and that chunk c - 1 has been read by everyone.
// Fragments are read from LDS one 16-column step ahead of the MFMAs that use them.
//
// Bound: at 640 rows of the 8B gate/up shape 121 us (1.07 PFLOP/s; few-row kernel 168 us), 1000 rows 183 us (283 us).
// Without its loads (MFMAs, LDS reads and barriers on whatever LDS and registers hold) the kernel takes 76 and 108 us: the
// 32 KB of weights a work-group pulls through its L1 per chunk, next to 16 KB of activations, take the rest.  A large
// library product reaches 1.4 to 1.6 PFLOP/s on random operands and 2.1 on zeros on this chip.
// The two chains per output cap the tile: 256 x 128 outputs fill half of the register file.  Deeper rings (5 weight
// chunks, 5 or 6 activation stages), non-temporal weights, a raised wave priority around the MFMAs and a common
// start of all K walks made no difference, nor did gathering the SwiGLU outputs of a row tile in LDS for 256-byte
// stores (gate/up, 640 / 1000 / 2304 rows: 119.8 / 182.9 / 584 us either way).
template <int R, int MT, int EPI, int DW, int NST>
__global__ __launch_bounds__(512) void k_gemm_rows(const bf16_t* X, const uint4* Wp, void* outv, int M, int N, int K,
                                                   int k_len, size_t split_stride, int mask_id, int n_tiles_out,
                                                   int n_blocks, int n_split, int m_chunks) {
    constexpr int WN = 4, KC = 64, ROWS = MT * 32, SB = ROWS * KC * 2;      // SB: bytes of a stage
    constexpr int XL = SB / 1024, NX = XL / 8, NX_MORE = XL % 8;            // wave loads per stage; per wave
    constexpr int WF = R * 2;                                               // weight fragments per wave and chunk
    static_assert(R == 2, "the epilogue gives each of the two k-slice waves one of the two n-tiles");
    static_assert(NST >= 3 && DW >= 2 && DW <= 4, "ring depths");
    extern __shared__ uint4 smem_u4[];
    char* smem = (char*)smem_u4;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave & 3, wk = wave >> 2, lm = lane & 31, lh = lane >> 5;
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
    const int m0 = by * ROWS, kbeg = bz * k_len, nchunks = k_len / KC;
    const int KS = K >> 4, NT = N >> 5;
    int nt[R];
    bool nt_ok[R];
    const uint4* wbase[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        nt[r] = (bx * WN + wn) * R + r;
        nt_ok[r] = nt[r] < NT;                                              // tiles past the end: clamped, never stored
        if (!nt_ok[r]) nt[r] = NT - 1;
        wbase[r] = Wp + ((size_t)nt[r] * KS + (kbeg >> 4) + wk * 2) * 64;
    }
    const int rot = gemm_k_start(bx * (WN * R * 32), bz, nchunks);
    auto chunk_at = [&](int c) {
        c = c < nchunks - 1 ? c : nchunks - 1;
        c += rot;
        return c >= nchunks ? c - nchunks : c;
    };

    // this lane's byte offsets into the work-group's rows: load j of the wave covers 8 rows of a stage; rows past
    // the end read the last row (never stored)
    const char* xrow0 = (const char*)(X + (size_t)m0 * K + kbeg);
    unsigned xoff[NX + 1];
#pragma unroll
    for (int j = 0; j <= NX; ++j) {
        const int r = (wave + 8 * j) * 8 + (lane >> 3), s = (lane & 7) ^ ((r >> 1) & 7);
        xoff[j] = (unsigned)(m0 + r < M ? r : M - 1 - m0) * (unsigned)(K * 2) + s * 16;
    }
    auto issue_x1 = [&](int j, int slot, int c) {                            // load j of the wave
        const char* src = xrow0 + (size_t)chunk_at(c) * (KC * 2);
        const unsigned dst = lds0 + slot * SB + (wave + 8 * j) * 1024;
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(xoff[j]), "s"(src) : "memory", "m0");
    };
    uint4 w0[WF], w1[WF], w2[WF], w3[WF];
#define SSD_WSLOT(i) ((i) % DW == 0 ? w0 : (i) % DW == 1 ? w1 : (i) % DW == 2 ? w2 : w3)
    auto issue_w1 = [&](int f, uint4* dst, int c) {                          // fragment f = 2r + ks of chunk c
        dst[f] = (wbase[f >> 1] + (size_t)chunk_at(c) * (KC / 16) * 64 + (f & 1) * 64)[lane];
    };
    floatx16 acc[R][MT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][mt][i] = 0.f;
    const int sw = (lm >> 1) & 7;
    const int xr[2] = {lm * 128 + (((wk * 4 + lh) ^ sw) << 4), lm * 128 + (((wk * 4 + 2 + lh) ^ sw) << 4)};
    auto read_x = [&](bf16x8(&xf)[MT], int slot, int ks) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) xf[mt] = *(const bf16x8*)(smem + slot * SB + mt * 4096 + xr[ks]);
    };
    // Order of the loads: iteration i issues X(i + NST - 1), then W(i + DW - 1); the iterations before the first
    // do the same.  At the top of iteration c chunk c + 1 must have landed: what is issued behind it by then
    // is W of its own iteration and the NST - 3 iterations after that; before the first iteration, when chunk 1
    // must have landed, the weights issued so far are fewer.
    constexpr int NEWER = WF + (NST - 3) * (NX + WF);
    constexpr int NEWER0 = (NST - 3) * NX + (DW < NST - 1 ? DW - 1 : NST - 2) * WF;
    bf16x8 xa[MT], xb[MT];
    static_for<0, NST - 1>([&](auto ic) {
        constexpr int u = decltype(ic)::value, wi = u + DW - NST;
#pragma unroll
        for (int j = 0; j < NX; ++j) issue_x1(j, u, u);
        if (NX_MORE && wave < NX_MORE) issue_x1(NX, u, u);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (wi >= 0)
#pragma unroll
            for (int f = 0; f < WF; ++f) issue_w1(f, SSD_WSLOT(wi), wi);
        __builtin_amdgcn_sched_barrier(0);
    });
    static_assert(DW <= NST && DW >= NST - 2, "the first weight chunks are issued between the first activation chunks");
    auto landed = [&](auto newer) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(newer)::value) : "memory");
        __syncthreads();
    };
    landed(std::integral_constant<int, NEWER0>{});
    read_x(xa, 0, 0);
    auto step = [&](auto uc, int c, bool first) {
        constexpr int u = decltype(uc)::value;
        if (!first) landed(std::integral_constant<int, NEWER>{});
        read_x(xb, u % NST, 1);
        // the chunk's MFMAs, its loads spread between them: a load that waits for the address unit, which all waves
        // reach at the same time behind the barrier, then waits while MFMAs run
        constexpr int NM = 2 * R * MT, NL = NX + (NX_MORE ? 1 : 0) + WF;
        static_for<0, NM>([&](auto im) {
            constexpr int i = decltype(im)::value, ks = i / (R * MT), r = i / MT % R, mt = i % MT;
            const uint4 wv = SSD_WSLOT(u)[r * 2 + ks];
            acc[r][mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)&wv, ks == 0 ? xa[mt] : xb[mt], acc[r][mt], 0, 0, 0);
            if constexpr (i == R * MT - 1) {
                __builtin_amdgcn_sched_barrier(0);
                read_x(xa, (u + 1) % NST, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr int l = (i * NL) / (NM - 1);                           // loads before MFMA i + 1: l of NL
            static_for<((i - 1) * NL) / (NM - 1), l>([&](auto il) {
                constexpr int k = decltype(il)::value;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (k < NX)
                    issue_x1(k, (u + NST - 1) % NST, c + NST - 1);
                else if constexpr (k < NL - WF) {
                    if (wave < NX_MORE) issue_x1(NX, (u + NST - 1) % NST, c + NST - 1);
                } else
                    issue_w1(k - (NL - WF), SSD_WSLOT(u + DW - 1), c + DW - 1);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int UN = DW == NST ? DW : DW * NST / (DW % 2 == 0 && NST % 2 == 0 ? 2 : 1);   // slots repeat with this period
    int c = 0;
    bool first = true;
    for (; c + UN <= nchunks; c += UN) {
        static_for<0, UN>([&](auto ic) { constexpr int u = decltype(ic)::value; step(ic, c + u, u == 0 && first); });
        first = false;
    }
    static_for<0, UN - 1>([&](auto ic) {
        constexpr int u = decltype(ic)::value;
        if (c + u < nchunks) step(ic, c + u, u == 0 && first);
    });
#undef SSD_WSLOT
    // The counts of `landed` hold only while every weight load is really issued: the last ones, which no MFMA
    // reads, are kept.
#pragma unroll
    for (int i = 0; i < WF; ++i) {
        auto keep = [](const uint4& v) { asm volatile("" ::"v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w)); };
        keep(w0[i]);
        keep(w1[i]);
        if (DW > 2) keep(w2[i]);
        if (DW > 3) keep(w3[i]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                         // no load may land in the exchange area
    __syncthreads();

    // ---- epilogue: wave (wn, wk) finishes n-tile wk of its pair: it receives the other k-slice's sums of
    // that tile through LDS and hands over its own of the other (k-slice 0 plus k-slice 1), one row tile at a time
    // with two exchange buffers.  Lane (lm, lh) holds rows n = 8*(i/4) + 4*lh + i%4 of column m = lm.
    float4* const ex = (float4*)smem;                                        // [2][8 waves][4][64]
    const int my_nt = nt[wk ? 1 : 0];
    const bool my_ok = wk ? nt_ok[1] : nt_ok[0];
    static_for<0, MT>([&](auto im) {
        constexpr int mt = decltype(im)::value;
        float4* b = ex + (mt & 1) * 8 * 256;
        auto give = [&](const floatx16& a) {
#pragma unroll
            for (int g = 0; g < 4; ++g) b[wave * 256 + g * 64 + lane] = make_float4(a[g * 4], a[g * 4 + 1], a[g * 4 + 2], a[g * 4 + 3]);
        };
        floatx16 v;
        if (wk == 0) { give(acc[1][mt]); v = acc[0][mt]; } else { give(acc[0][mt]); v = acc[1][mt]; }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 o = b[(wave ^ 4) * 256 + g * 64 + lane];
            v[g * 4] += o.x; v[g * 4 + 1] += o.y; v[g * 4 + 2] += o.z; v[g * 4 + 3] += o.w;
        }
        [[maybe_unused]] const int m = m0 + mt * 32 + lm;
        if constexpr (EPI == EPI_F32) {
            // through LDS into row order, so that a store covers whole 128-byte lines of 8 rows instead of 32 bytes
            // of each of 32 (the L2 takes a fourth of the requests; 640 rows of the 8B shape, us: QKV 72.6 -> 69.5, down
            // 79.5 -> 77.2, attention output 31.1 -> 29.7); the area is the one the partner's sums came in, which only this wave reads, and
            // piece s of row r lies in slot s ^ (r % 8)
            float4* t = b + (wave ^ 4) * 256;
            wave_lds_order();                                            // every lane has read what is overwritten next
#pragma unroll
            for (int g = 0; g < 4; ++g)
                t[lm * 8 + ((g * 2 + lh) ^ (lm & 7))] = make_float4(v[g * 4], v[g * 4 + 1], v[g * 4 + 2], v[g * 4 + 3]);
            wave_lds_order();                                            // other lanes wrote what is read next
            float* out = (float*)outv + (size_t)bz * split_stride + my_nt * 32 + (lane & 7) * 4;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r = g * 8 + (lane >> 3), row = m0 + mt * 32 + r;
                const float4 o = t[r * 8 + ((lane & 7) ^ (r & 7))];
                if (my_ok && row < M) *(float4*)(out + (size_t)row * N) = o;
            }
        } else if constexpr (EPI == EPI_SWIGLU) {
            bf16_t* out = (bf16_t*)outv;
            if (my_ok && m < M) {
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    uint16_t o[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) o[j] = swiglu_bf16(v[g * 4 + j], v[(g + 2) * 4 + j]);
                    *(uint2*)(out + (size_t)m * (N >> 1) + my_nt * 16 + g * 8 + lh * 4) =
                        make_uint2((uint32_t)o[0] | ((uint32_t)o[1] << 16), (uint32_t)o[2] | ((uint32_t)o[3] << 16));
                }
            }
        } else {
            float p[3];
            lm_tile_partial(v, my_nt, lh, mask_id, p);
            if (lh == 0 && my_ok && m < M) {
                float* o = (float*)outv + ((size_t)m * n_tiles_out + my_nt) * 3;
                o[0] = p[0]; o[1] = p[1]; o[2] = p[2];
            }
        }
    });
}

template <int MT, int EPI, int DW, int NST>
static bool launch_rows(const GemmArgs& a) {
    constexpr int R = 2, ROWS = MT * 32;
    constexpr size_t ring = (size_t)NST * ROWS * 128, exch = 2 * 8 * 4096, smem = ring > exch ? ring : exch;
    static_assert(smem <= 160 * 1024, "LDS budget");
    auto kern = k_gemm_rows<R, MT, EPI, DW, NST>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess)
            return false;
        attr_done = true;
    }
    const int n_blocks = (a.N / 32 + 7) / 8, m_chunks = (a.M + ROWS - 1) / ROWS;
    hipLaunchKernelGGL(kern, dim3(n_blocks * m_chunks * a.split), dim3(512), smem, a.st, a.X, a.Wp, a.out, a.M, a.N, a.K,
                       a.K / a.split, a.split_stride, a.mask_id, a.n_tiles_out, n_blocks, a.split, m_chunks);
    return true;
}
