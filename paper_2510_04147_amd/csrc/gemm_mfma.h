// The MFMA GEMM kernel template and its launchers, shared by the translation units that instantiate it
// (gemm_f32_*, gemm_swiglu_*, gemm_lmhead_*: one per epilogue and work-group shape), so that they compile in parallel.
// See kernels_mfma.hip for the design.
#pragma once
#include <cstdlib>
#include <type_traits>

#include "gemm_rules.h"
#include "ssd_internal.h"

typedef uint16_t bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// for lambdas, whose captures have to stay in registers
#define SSD_INLINE __attribute__((always_inline))

// Compile-time loop: f(integral_constant<int, C>) for C in [BEGIN, END).  The ring slots of the
// GEMM pipeline are selected by these constants, so no register array is ever indexed by a
// run-time value (which would push it to scratch memory).
template <int BEGIN, int END, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (BEGIN < END) {
        f(std::integral_constant<int, BEGIN>{});
        static_for<BEGIN + 1, END>(f);
    }
}

// exp through the hardware's base-2 exponential (relative error about 1e-6): the epilogues and the softmax
// evaluate it once per output element, where the correctly rounded library routine costs as much as the
// arithmetic it follows; the results are rounded to bf16 or summed over a vocabulary afterwards.
__device__ __forceinline__ float fast_exp(float x) { return __expf(x); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// two values to bf16, to nearest even (one instruction)
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    const bf16x2 v = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint16_t f2bf_m(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// silu(gate) * up
__device__ __forceinline__ float swiglu(float g, float u) { return g * __builtin_amdgcn_rcpf(1.0f + fast_exp(-g)) * u; }

// The other half's value: lane l gets lane l ^ 32's (no trip through LDS, unlike a shuffle).
__device__ __forceinline__ unsigned other_half(unsigned v, int lh) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);     // [0]: the lower lanes' in both halves, [1]: the upper lanes'
    return lh ? r[0] : r[1];
}
__device__ __forceinline__ float other_half(float v, int lh) { return __uint_as_float(other_half(__float_as_uint(v), lh)); }

// LM head: (max, arg-max as float bits, sum of exp) of one row over the 32 vocabulary rows of tile nt; lane (lm, lh)
// holds n = 8*(i/4) + 4*lh + i%4 of row lm.  The mask token takes no part.  Bound by instructions: the maximum first, its
// lowest position from the equal ones (384 rows, us, with a compare and two selects per value and shuffles through LDS /
// this: 32000 tokens, K = 1600 55.2 / 46.5, K = 2048 65.9 / 56.8).
__device__ __forceinline__ void lm_tile_partial(const floatx16& acc, int nt, int lh, int mask_id, float* p) {
    floatx16 v = acc;
    if (nt == mask_id >> 5) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (nt * 32 + (i >> 2) * 8 + lh * 4 + (i & 3) == mask_id) v[i] = -INFINITY;
    }
    float bm = -INFINITY;                                    // a NaN is never the maximum
#pragma unroll
    for (int i = 0; i < 16; ++i) bm = fmaxf(bm, v[i]);
    bm = fmaxf(bm, other_half(bm, lh));
    int bi = 0x7fffffff;
#pragma unroll
    for (int i = 15; i >= 0; --i) bi = v[i] == bm ? (i >> 2) * 8 + (i & 3) : bi;
    bi = bi == 0x7fffffff || bm == -INFINITY ? 0x7fffffff : nt * 32 + lh * 4 + bi;
    bi = min(bi, (int)other_half((unsigned)bi, lh));
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) se += fast_exp(v[i] - bm);
    p[0] = bm;
    p[1] = __int_as_float(bi);
    p[2] = se + other_half(se, lh);
}

// First chunk of a work-group's K walk: groups of work-groups start at different chunks, which spreads the grid's weight
// streams over the HBM channels.  One start per 768 weight rows (a multiple of every n-block width: three to twelve
// neighbouring n-blocks; a matrix of at most 768 rows has one) and k-slice, so that the kernels for few and for many
// rows sum in the same order.
__device__ __forceinline__ int gemm_k_start(int row, int bz, int nchunks) {
    return (int)(((unsigned)(row / 768) * 5u + (unsigned)bz * 3u) % (unsigned)nchunks);
}

// Between accesses to LDS by different lanes of one wave.  No instruction: a wave's LDS accesses complete in order, but the
// compiler orders them by address within a lane only.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16 bytes per lane from src + off (per lane) to LDS address dst + 16 lane, without passing through registers.  The compiler
// does not count these loads: whoever reads what they bring writes the wait out.  NT: non-temporal.
template <bool NT>
__device__ __forceinline__ void load_to_lds(unsigned dst, unsigned off, const void* src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t.if %3\n\tglobal_load_lds_dwordx4 %1, %2 nt\n\t.else\n\tglobal_load_lds_dwordx4 %1, %2\n\t.endif"
                 ::"s"(dst), "v"(off), "s"(src), "n"(NT ? 1 : 0) : "memory", "m0");
}
// At most N of this wave's loads outstanding and none of its LDS accesses, then the barrier of the work-group.
template <int N>
__device__ __forceinline__ void wait_and_meet() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// ------------------------------------------------------------------------
// GEMM for few rows.  Work-group = WN x WM waves.  Wave (wn, wm) owns one n-tile of 32 weight rows, the row tiles wm,
// wm + WM, ... of MT and, of the work-group's k-slice, every column: one chain of MFMAs per output, in chunks of KC = 64
// columns.  k_gemm_rows builds the same chains, so a row's sums are bit for bit the same in both.
//
// Weights and activations go global -> LDS without passing through registers into a ring of NST stages.  From the barrier in
// front of chunk c on, whose stage has landed and with which everyone has read chunk c - 1, chunk c - 1 + NST is loaded into
// the stage of chunk c - 1, a fourth of its loads in front of each of four steps of 16 columns; fragments are
// read from LDS one step ahead of the MFMAs that use them.
// The K walk starts at a chunk that depends on the k-slice and on the group of
// 768 weight rows (gemm_k_start) and wraps, which spreads the grid's weight
// streams over the HBM channels; the order depends on the n-tile only, so a
// row's summation order is the same in every forward.
// CACHED: weight loads with the default cache policy (GemmPass).
//
// Bound by the line requests a CU keeps in flight: the weight stream and the activations, which every work-group reads whole
// from L2, queue for them.  160 rows of the 8B shape, inside the forward, us (with two chains per output in two waves,
// weights in register rings and activations staged through registers / this): gate/up 48.2 / 46.6, QKV 28.1 / 27.6,
// down 27.4 / 26.3, attention output 15.5 / 14.9; 40 rows 32.4 / 32.8, 18.8 / 18.9, 19.0 / 18.8, 9.6 / 9.0.  Four stages:
// five take 51.0 for gate/up at 160 rows, three 47.8 there but 27.4 for down; all of a chunk's loads
// behind the barrier in one go 52.0, one wave per n-tile for all rows (WM = 1) 52.3.
// ------------------------------------------------------------------------
template <int WN, int WM, int MT, int EPI, bool CACHED, int NST>
__global__ __launch_bounds__(WN* WM * 64) void k_gemm_mfma(const bf16_t* X, const uint4* Wp, void* outv, int M, int N,
                                                           int K, int k_len, size_t split_stride, int mask_id,
                                                           int n_tiles_out, int n_blocks, int n_split, int m_chunks_total) {
    constexpr int NW = WN * WM, KC = 64, KSTEPS = KC / 16, ROWS = MT * 32, TW = (MT + WM - 1) / WM;
    constexpr int WB = WN * KSTEPS * 1024, SB = WB + ROWS * KC * 2;             // bytes of a stage: weights, activations
    constexpr int PIECES = SB / 1024, PMIN = PIECES / NW, PMORE = PIECES % NW;  // loads of a stage; per wave
    static_assert(NST >= 2 && PMIN * (NST - 1) < 64, "ring depth");
    extern __shared__ uint4 smem_u4[];
    char* const smem = (char*)smem_u4;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave % WN, wm = wave / WN, lm = lane & 31, lh = lane >> 5;
    // The grid is one-dimensional; work-groups go to the 8 XCDs round-robin by their linear id, and every
    // XCD has an L2 of its own.  The id is decoded so that with split-K all work-groups of an XCD take the
    // same k-slice, i.e. read the same slice of the activations and find it in that XCD's L2, and so that
    // the row chunks of one n-block (forwards with more rows than one pass holds) are neighbours on one
    // XCD and stream the same weights at the same time.  A tile's result does not depend on where it runs.
    int bx, bz, by;
    {
        const int split = n_split, mch = m_chunks_total;
        const int id = blockIdx.x;
        if (split <= 8 && 8 % split == 0 && n_blocks % (8 / split) == 0) {
            const int xcd = id & 7, t = id >> 3, per = 8 / split;
            bz = xcd % split;
            by = t % mch;
            bx = (t / mch) * per + xcd / split;
        } else {
            bz = id % split;
            by = (id / split) % mch;
            bx = id / (split * mch);
        }
    }
    const int m0 = by * ROWS;
    const int kbeg = bz * k_len, nchunks = k_len / KC;
    const int KS = K >> 4, NT = N >> 5;
    const int nt = bx * WN + wn;                         // this wave's n-tile (past the end: never stored)
    const bool nt_ok = nt < NT;

    const int rot = gemm_k_start(bx * (WN * 32), bz, nchunks);
    // Load i of this wave is piece wave + NW i of a stage: 1 KB each, first the n-tiles' fragments, then eight rows of the
    // activations per piece, the 16-byte piece s of row r in slot s ^ (r / 2 % 8) of its line, so that the 32 rows of a
    // fragment spread over all LDS banks.  n-tiles and rows past the end read the last one (never stored).
    const char* xrow0 = (const char*)(X + (size_t)m0 * K + kbeg);
    unsigned xoff[PMIN + 1];
#pragma unroll
    for (int i = 0; i <= PMIN; ++i) {
        const int p = wave + NW * i - WN * KSTEPS;
        const int r = p * 8 + (lane >> 3), s = (lane & 7) ^ ((r >> 1) & 7);
        xoff[i] = p < 0 ? lane * 16 : (unsigned)(m0 + r < M ? r : M - 1 - m0) * (unsigned)(K * 2) + s * 16;
    }
    auto issue1 = [&](int i, int slot, int at) SSD_INLINE {         // at: the chunk, rotated
        const int p = wave + NW * i;
        const unsigned dst = lds0 + slot * SB + p * 1024;
        const int t = p / KSTEPS;
        if (NW * i + NW <= WN * KSTEPS || (NW * i < WN * KSTEPS && p < WN * KSTEPS)) {
            const int n = bx * WN + t < NT ? bx * WN + t : NT - 1;
            load_to_lds<!CACHED>(dst, xoff[i], Wp + ((size_t)n * KS + (kbeg >> 4) + at * KSTEPS + p % KSTEPS) * 64);
        } else
            load_to_lds<false>(dst, xoff[i], xrow0 + (size_t)at * (KC * 2));
    };
    int at = rot;                                        // the next chunk to load, rotated
    floatx16 acc[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    const bool full = MT % WM == 0 || wm < MT % WM;      // this wave has TW row tiles, else TW - 1
    const int sw = (lm >> 1) & 7;
    struct Frags { bf16x8 w, x[TW]; } fa, fb;
    auto read = [&](Frags& f, int slot, int ks) SSD_INLINE {
        const char* s = smem + slot * SB;
        f.w = *(const bf16x8*)(s + (wn * KSTEPS + ks) * 1024 + lane * 16);
#pragma unroll
        for (int t = 0; t < TW; ++t)
            if (t < TW - 1 || full)
                f.x[t] = *(const bf16x8*)(s + WB + (wm + WM * t) * 4096 + lm * 128 + (((ks * 2 + lh) ^ sw) << 4));
    };
    auto multiply = [&](const Frags& f) SSD_INLINE {
#pragma unroll
        for (int t = 0; t < TW; ++t)
            if (t < TW - 1 || full) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.w, f.x[t], acc[t], 0, 0, 0);
    };
    auto issue = [&](int i, int slot) SSD_INLINE {       // i up to PMIN; some waves have one load more than others
        if (i < PMIN || wave < PMORE) issue1(i, slot, at);
    };
    auto after = [&](int at) SSD_INLINE { return at + 1 == nchunks ? 0 : at + 1; };
    constexpr int PER = PMIN + (PMORE ? 1 : 0);
    // step q behind the barrier: its share of the loads, then its MFMAs
    auto step = [&](auto qc, const Frags& f, int slot, bool load) SSD_INLINE {
        constexpr int q = decltype(qc)::value;
        __builtin_amdgcn_sched_barrier(0);
        if (load)
            static_for<q * PER / 4, (q + 1) * PER / 4>([&](auto ic) SSD_INLINE { issue(decltype(ic)::value, slot); });
        __builtin_amdgcn_sched_barrier(0);
        multiply(f);
        __builtin_amdgcn_sched_barrier(0);
    };
    int slot = 0;
    // three steps of a chunk, whose first fragments are on their way
    auto three_steps = [&](int prev, bool load) SSD_INLINE {
        read(fb, slot, 1);
        step(std::integral_constant<int, 1>{}, fa, prev, load);
        read(fa, slot, 2);
        step(std::integral_constant<int, 2>{}, fb, prev, load);
        read(fb, slot, 3);
        step(std::integral_constant<int, 3>{}, fa, prev, load);
    };
    // from the barrier in front of a chunk on: the last step of the chunk before, whose stage is free, and three of its own
    auto period = [&](bool load) SSD_INLINE {
        const int prev = slot;
        slot = slot + 1 == NST ? 0 : slot + 1;
        read(fa, slot, 0);
        step(std::integral_constant<int, 0>{}, fb, prev, load);
        three_steps(prev, load);
        at = after(at);
    };
#pragma unroll
    for (int u = 0; u < NST; ++u)
        if (u < nchunks) {
#pragma unroll
            for (int i = 0; i < PER; ++i) issue(i, u);
            at = after(at);
        }
    // the oldest chunk on its way has landed, B behind it may be outstanding
    auto landed = [&](auto bc) SSD_INLINE {
        constexpr int B = decltype(bc)::value;
        if (PMORE && wave < PMORE) wait_and_meet<(PMIN + 1) * B>();
        else wait_and_meet<PMIN * B>();
    };
    if (nchunks >= NST) landed(std::integral_constant<int, NST - 1>{});
    else landed(std::integral_constant<int, 0>{});
    read(fa, 0, 0);
    three_steps(0, false);
    int c = 1;
    for (; c - 1 + NST < nchunks; ++c) {
        landed(std::integral_constant<int, NST - 2>{});
        period(true);
    }
    for (; c < nchunks; ++c) {
        landed(std::integral_constant<int, 0>{});
        period(false);
    }
    step(std::integral_constant<int, 0>{}, fb, 0, false);
    __syncthreads();                                     // the epilogue reuses the ring

    // ---- epilogues.  Lane (lm, lh) holds, per tile, rows n = 8*(i/4) + 4*lh + i%4 of column m = lm;
    // g = i/4 selects a group of four consecutive n.
    if constexpr (EPI == EPI_F32) {
        // through LDS into row order (every wave has read its last fragments: an area of 4 KB per wave and parity of the
        // row tile), so that a store covers whole 128-byte lines of 8 rows; piece s of row r lies in slot s ^ (r % 8)
        float* out = (float*)outv + (size_t)bz * split_stride + (size_t)nt * 32 + (lane & 7) * 4;
#pragma unroll
        for (int i = 0; i < TW; ++i) {
            if (i == TW - 1 && !full) continue;
            const int mt = wm + WM * i;
            float4* t = (float4*)smem_u4 + (wave * 2 + (i & 1)) * 256;
            wave_lds_order();                            // every lane has read what is overwritten next
#pragma unroll
            for (int g = 0; g < 4; ++g)
                t[lm * 8 + ((g * 2 + lh) ^ (lm & 7))] = make_float4(acc[i][g * 4], acc[i][g * 4 + 1], acc[i][g * 4 + 2], acc[i][g * 4 + 3]);
            wave_lds_order();                            // other lanes wrote what is read next
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int r = g * 8 + (lane >> 3), m = m0 + mt * 32 + r;
                const float4 o = t[r * 8 + ((lane & 7) ^ (r & 7))];
                if (nt_ok && m < M) *(float4*)(out + (size_t)m * N) = o;
            }
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
        // A tile holds 16 channels: rows 0..15 gate, rows 16..31 up, so groups g and g + 2 of a lane are
        // gate and up of the same four channels.
        bf16_t* out = (bf16_t*)outv;
        const int F = N >> 1;                            // output channels = row stride of the output
#pragma unroll
        for (int i = 0; i < TW; ++i) {
            if (i == TW - 1 && !full) continue;
            const int mt = wm + WM * i;
            const int m = m0 + mt * 32 + lm;
            if (!nt_ok || m >= M) continue;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                float o[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) o[j] = swiglu(acc[i][g * 4 + j], acc[i][(g + 2) * 4 + j]);
                *(uint2*)(out + (size_t)m * F + nt * 16 + g * 8 + lh * 4) = make_uint2(bf16_pair(o[0], o[1]), bf16_pair(o[2], o[3]));
            }
        }
    } else {
        // LM head: per (row, n-tile) partial over the tile's 32 vocabulary rows
        float* out = (float*)outv;
#pragma unroll
        for (int i = 0; i < TW; ++i) {
            if (i == TW - 1 && !full) continue;
            const int mt = wm + WM * i;
            float p[3];
            lm_tile_partial(acc[i], nt, lh, mask_id, p);
            const int m = m0 + mt * 32 + lm;
            if (lh == 0 && m < M && nt_ok) {
                float* o = out + ((size_t)m * n_tiles_out + nt) * 3;
                o[0] = p[0];
                o[1] = p[1];
                o[2] = p[2];
            }
        }
    }
}

// ------------------------------------------------------------------------
// launcher
// ------------------------------------------------------------------------

// the launchers of the work-group shapes, one translation unit each (they compile in parallel)
struct GemmArgs {
    const bf16_t* X;
    const uint4* Wp;
    void* out;
    int M, N, K, split;
    size_t split_stride;
    int mask_id, n_tiles_out;
    GemmPass pass;                        // the few-row kernel's
    hipStream_t st;
};

template <int WN, int MT, int EPI, bool CACHED, int NST = 4>
static bool launch_one(const GemmArgs& a) {
    constexpr int WM = MT > 1 ? 2 : 1;
    constexpr size_t stage = (size_t)(WN + MT) * 4096;
    // four stages; a grid of several rounds over the chip (the LM head) takes as many as leave room for a second work-group on
    // the CU (8B, 160 rows 213.5 -> 211.2 us, 40 rows 162 -> 160; 250 work-groups, 1600 wide, 96 rows: 24.5 with four, 27.3 so)
    constexpr int fit = (int)(80 * 1024 / stage), PAIR = fit > 4 ? 4 : fit < 2 ? 2 : fit;
    if constexpr (EPI == EPI_LMHEAD && NST == 4 && PAIR < 4)
        if ((a.N / 32 + WN - 1) / WN * a.pass.passes * a.split > 256) return launch_one<WN, MT, EPI, CACHED, PAIR>(a);
    constexpr size_t rbytes = EPI == EPI_F32 ? (size_t)WN * WM * 2 * 4096 : 0;          // the epilogue's row-order areas
    constexpr size_t smem = NST * stage > rbytes ? NST * stage : rbytes;
    static_assert(smem <= 160 * 1024, "LDS budget");
    auto kern = k_gemm_mfma<WN, WM, MT, EPI, CACHED, NST>;
    static bool attr_done = false;
    if (!attr_done) {
        if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) != hipSuccess)
            return false;
        attr_done = true;
    }
    const int n_blocks = (a.N / 32 + WN - 1) / WN;
    dim3 grid(n_blocks * a.pass.passes * a.split);
    hipLaunchKernelGGL(kern, grid, dim3(WN * WM * 64), smem, a.st, a.X, a.Wp, a.out, a.M, a.N, a.K, a.K / a.split,
                       a.split_stride, a.mask_id, a.n_tiles_out, n_blocks, a.split, a.pass.passes);
    return true;
}

// Row tiles of 32 rows per pass: 1 (a stepwise forward of one block) to 6; other row counts round up
// (rows past the end repeat the last one and are never stored).  The rows of a pass share nothing but the weight fragments,
// so a row's sums do not depend on the tile it is computed in.
template <int WN, int EPI, bool CACHED>
static bool launch_mt(const GemmArgs& a) {
    switch (a.pass.mt) {
        case 1: return launch_one<WN, 1, EPI, CACHED>(a);
        case 2: return launch_one<WN, 2, EPI, CACHED>(a);
        case 3: return launch_one<WN, 3, EPI, CACHED>(a);
        case 4: return launch_one<WN, 4, EPI, CACHED>(a);
        case 5: return launch_one<WN, 5, EPI, CACHED>(a);
        case 6: return launch_one<WN, 6, EPI, CACHED>(a);
    }
    return false;
}

template <int WN, int EPI>
static bool launch_shape(const GemmArgs& a) {
    return a.pass.cached ? launch_mt<WN, EPI, true>(a) : launch_mt<WN, EPI, false>(a);
}

bool gemm_f32_wn3(const GemmArgs& a);     // wide outputs (QKV): 96-row n-blocks
bool gemm_f32_wn2(const GemmArgs& a);     // narrow outputs, short K (attention output): 64-row n-blocks
bool gemm_f32_wn4(const GemmArgs& a);     // narrow outputs, long K (down) and everything else: 128-row n-blocks
bool gemm_swiglu_wn3(const GemmArgs& a);
bool gemm_swiglu_wn4(const GemmArgs& a);
bool gemm_lmhead_wn4(const GemmArgs& a);
// the kernel for many rows (gemm_rows.h) with the tile that gemm_tile() says
bool gemm_rows_f32(const GemmArgs& a, int tile);
bool gemm_rows_swiglu(const GemmArgs& a, int tile);
bool gemm_rows_lmhead(const GemmArgs& a, int tile);

// Split along K across work-groups: a function of the weight shape only.
static int pick_split(int K, int kc, int want) {
    int s = want;
    while (s > 1 && (K % (s * kc)) != 0) --s;
    return s < 1 ? 1 : s;
}
