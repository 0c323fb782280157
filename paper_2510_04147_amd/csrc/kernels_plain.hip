// Plain (FMA, no matrix cores) kernels for every step of the forward, for fp32
// and bf16 storage.  They are the complete path for fp32 models and the
// fallback / cross-check for bf16.  Every reduction runs in a fixed order that
// depends only on the reduced extent, never on how many rows a launch holds,
// so a row's result is bit-identical whether it is computed in a 1-node or an
// (N+1)-node forward: that is what makes the batched verification (Eq. 5)
// reproduce stepwise decoding exactly.
#include <type_traits>

#include "gemm_rules.h"
#include "ssd_internal.h"

typedef uint16_t bf16_t;

__device__ __forceinline__ float ld_f(const float* p) { return *p; }
__device__ __forceinline__ float ld_f(const bf16_t* p) { return __uint_as_float(((uint32_t)*p) << 16); }
__device__ __forceinline__ float4 ld4_f(const float* p) {
    const float4 v = *(const float4*)p;
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ float4 ld4_f(const bf16_t* p) {
    const uint2 v = *(const uint2*)p;
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xffff0000u));
}
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t x = __float_as_uint(f);
    if ((x & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((x >> 16) | 0x40);   // NaN stays NaN
    x += 0x7fffu + ((x >> 16) & 1u);                                            // round to nearest even
    return (uint16_t)(x >> 16);
}
__device__ __forceinline__ void st_f(float* p, float v) { *p = v; }
__device__ __forceinline__ void st_f(bf16_t* p, float v) { *p = f2bf(v); }

// Reductions over the wave's 64 lanes, the result in every lane, without the LDS (a shuffle costs a trip through it): within
// rows of 16 lanes by DPP (pairs, pairs of pairs, mirrored halves), across rows by the swaps of 16 and 32 lanes.
template <int CTRL>
__device__ __forceinline__ int dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true); }
template <class F>
__device__ __forceinline__ int wave_reduce(int v, F&& f) {
    v = f(v, dpp<0xB1>(v));                              // lanes 1 0 3 2
    v = f(v, dpp<0x4E>(v));                              // lanes 2 3 0 1
    v = f(v, dpp<0x141>(v));                             // the other four of eight
    v = f(v, dpp<0x140>(v));                             // the other eight of sixteen
    const auto r16 = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = f((int)r16[0], (int)r16[1]);
    const auto r32 = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return f((int)r32[0], (int)r32[1]);
}
__device__ __forceinline__ float wave_sum(float v) {
    return __int_as_float(wave_reduce(__float_as_int(v), [](int a, int b) { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }));
}
__device__ __forceinline__ float wave_max(float v) {
    return __int_as_float(wave_reduce(__float_as_int(v), [](int a, int b) { return __float_as_int(fmaxf(__int_as_float(a), __int_as_float(b))); }));
}
__device__ __forceinline__ int wave_min(int v) { return wave_reduce(v, [](int a, int b) { return a < b ? a : b; }); }
__device__ __forceinline__ float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }
// How many of the lanes in `set` are ahead of this one: higher value, or equal and lower lane.
__device__ __forceinline__ int rank_among(float c, unsigned long long set, int lane) {
    int rank = 0;
    while (set) {                                        // uniform over the wave
        const int l = __ffsll(set) - 1;
        set &= set - 1;
        const float o = lane_value(c, l);
        rank += o > c || (o == c && l < lane);
    }
    return rank;
}

// a2/a6/a9: h += split-K partial sums (the sum of the first half of them, then the second's: a GEMM that walks half of the
// slices itself leaves two), then RMSNorm.
// One work-group of NORM_T threads per row; every thread owns up to NORM_J float4 groups of the
// row and issues all partial-sum loads of a group before the first add, so a 4096-wide row has
// its whole input (the row and every partial sum) in flight at once.
#define NORM_T 1024
#define NORM_J 2   // 1024 threads x 2 float4 = rows up to 8192 wide
__device__ __forceinline__ void st4(float* p, float a, float b, float c, float d) { *(float4*)p = make_float4(a, b, c, d); }
__device__ __forceinline__ void st4(bf16_t* p, float a, float b, float c, float d) {
    *(uint2*)p = make_uint2((uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16), (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16));
}

// NP < 0: the row is the embedding e.
template <typename T, int NP>
__device__ __forceinline__ void norm_row(float* hr, const float* pr, size_t part_stride, const float* gain, T* xr,
                                         int d, float eps, const T* e = nullptr) {
    const int n4 = d >> 2;
    float4 v[NORM_J], g[NORM_J];
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < NORM_J; ++j) {
        const int i4 = threadIdx.x + j * NORM_T;
        if (i4 < n4) {
            v[j] = NP < 0 ? (((uintptr_t)e & 15) == 0 ? ld4_f(e + 4 * i4) : make_float4(ld_f(e + 4 * i4), ld_f(e + 4 * i4 + 1), ld_f(e + 4 * i4 + 2), ld_f(e + 4 * i4 + 3))) : ((const float4*)hr)[i4];
            g[j] = ((const float4*)gain)[i4];                // not behind the reduction's barrier (1000 rows 20.1 -> 19.2 us)
            float4 pv[NP > 0 ? NP : 1];
#pragma unroll
            for (int s = 0; s < NP; ++s) pv[s] = ((const float4*)(pr + s * part_stride))[i4];
            // the sum of the first half of them, then the second's
            constexpr int HALF = (NP + 1) / 2;
            auto add = [](float4& x, const float4& y) { x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w; };
            if constexpr (NP > 0) {
                float4 t = pv[0];
#pragma unroll
                for (int s = 1; s < HALF; ++s) add(t, pv[s]);
                add(v[j], t);
            }
            if constexpr (NP > 1) {
                float4 t = pv[HALF];
#pragma unroll
                for (int s = HALF + 1; s < NP; ++s) add(t, pv[s]);
                add(v[j], t);
            }
            if (NP != 0) ((float4*)hr)[i4] = v[j];
            ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
        }
    }
    __shared__ float red[NORM_T / 64];
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < NORM_T / 64; ++w) tot += red[w];
    const float r = 1.0f / sqrtf(tot / (float)d + eps);
#pragma unroll
    for (int j = 0; j < NORM_J; ++j) {
        const int i4 = threadIdx.x + j * NORM_T;
        if (i4 < n4) {
            st4(xr + 4 * i4, v[j].x * r * g[j].x, v[j].y * r * g[j].y, v[j].z * r * g[j].z, v[j].w * r * g[j].w);
        }
    }
}

template <typename T>
__global__ __launch_bounds__(NORM_T) void k_norm(float* __restrict__ h, const float* __restrict__ part, int n_part,
                                              size_t part_stride, const float* __restrict__ gain,
                                              T* __restrict__ xn, int d, float eps) {
    const int row = blockIdx.x;
    float* hr = h + (size_t)row * d;
    const float* pr = part + (size_t)row * d;
    T* xr = xn + (size_t)row * d;
    switch (n_part) {
        case 0: norm_row<T, 0>(hr, pr, part_stride, gain, xr, d, eps); break;
        case 1: norm_row<T, 1>(hr, pr, part_stride, gain, xr, d, eps); break;
        case 2: norm_row<T, 2>(hr, pr, part_stride, gain, xr, d, eps); break;
        case 4: norm_row<T, 4>(hr, pr, part_stride, gain, xr, d, eps); break;
        case 8: norm_row<T, 8>(hr, pr, part_stride, gain, xr, d, eps); break;
        default: {
            // any other split count: fold the partial sums into h first, by halves
            for (int i = threadIdx.x; i < d; i += NORM_T) {
                float v = hr[i];
                const int half = (n_part + 1) >> 1;
                for (int s = 0; s < n_part; s = s == 0 && n_part > 1 ? half : n_part) {
                    float t = pr[s * part_stride + i];
                    for (int u = s + 1; u < (s == 0 ? half : n_part); ++u) t += pr[u * part_stride + i];
                    v += t;
                }
                hr[i] = v;
            }
            __syncthreads();
            norm_row<T, 0>(hr, pr, part_stride, gain, xr, d, eps);
        }
    }
}

// ------------------------------------------------------------------------
// The forward's descriptor, raw tokens and block states from pinned host memory: what is used of them, in one trip by one
// work-group.  A copy of the header, 25 KB, goes through the copy engine, and the kernels wait for it on both sides; every block
// state is a copy of its own (a forward of the fp32 parity model, 32 rows, 101 us; with this and the fused kernel below 82; of
// the small bf16 model, two sequences of four nodes, 140 / 118).  One work-group is enough for long prompts too (KV pass of one 512
// wide bf16 layer, copies and three kernels / this and the fused one, us: 1000 tokens 44 / 23, 4096 79 / 51, 16384 228 / 127).
// ------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_stage(const int* __restrict__ src, StageLayout lay, int* __restrict__ fwd,
                                                int* __restrict__ raw_tok, int* __restrict__ state) {
    // segment s of the source: lay.n[s] words from lay.from[s]
    for (int i = threadIdx.x; i < lay.total; i += 1024) {
        int j = i, s = 0;
        while (j >= lay.n[s]) j -= lay.n[s++];
        const int v = src[lay.from[s] + j];
        if (s < 3) fwd[lay.from[s] + j] = v;              // the header's front, groups, nodes: same place as in the source
        else if (s == 3) raw_tok[j] = v;
        else {
            constexpr int W = sizeof(SeqState) / 4;
            state[lay.seq[j / W] * W + j % W] = v;
        }
    }
}

// ------------------------------------------------------------------------
// a0 + a1 + a2 of the first layer: tree build, embedding gather into the fp32 residual stream, RMSNorm.  One work-group per
// row.  Node j of a decode group is the block state with drafts 1..j written in (Section 3.2.3).  Bound by latency, a trip to
// memory each for node, state and embedding (32 rows x 256, us, three kernels / this: 2.6 + 2.3 + 2.7 / 3.8).
// EMBED = false: the tree build alone.
// ------------------------------------------------------------------------
template <typename T, bool EMBED>
__global__ __launch_bounds__(EMBED ? NORM_T : 64) void k_rows(const FwdHeader* __restrict__ fw, int n_nodes, const SeqState* __restrict__ state,
                                                             const int* __restrict__ raw_tok, NodeDesc* __restrict__ row_desc,
                                                             int* __restrict__ out_tok, int mask_id, int max_seq_len,
                                                             const float* __restrict__ ref_conf, const int* __restrict__ ref_arg,
                                                             const T* __restrict__ embed, float* __restrict__ h,
                                                             const float* __restrict__ gain, T* __restrict__ xn, int d, int V, float eps) {
    __shared__ int sh_tok;
    const int row = blockIdx.x, lane = threadIdx.x & 63;
    if (threadIdx.x < 64) {
        // the node that holds the row: nodes lie in row order
        int ni = 0;
        for (int n0 = 0; n0 < n_nodes; n0 += 64) {
            const unsigned long long at_or_before = __ballot(n0 + lane < n_nodes && fw->nodes[min(n0 + lane, n_nodes - 1)].row0 <= row);
            if (at_or_before) ni = n0 + 63 - __clzll(at_or_before);
        }
        const NodeDesc nd = fw->nodes[ni];
        const GroupDesc g = fw->groups[nd.group];
        const SeqState* s = &state[nd.seq];
        const int p = row - nd.row0;
        int tok;
        if (g.mode == GM_RAW) {
            tok = raw_tok[g.raw_off + p];
        } else if (g.mode == GM_APPEND) {
            tok = s->tok[p];
            if (g.out_off >= 0 && lane == 0) out_tok[(size_t)nd.seq * max_seq_len + g.out_off + p] = tok;
        } else if (g.from_refresh) {
            // A block nobody has predicted yet, with drafts read off the last refresh (Section 3.2.2 with the cache of
            // Section 4.1): node j holds the j positions the refresh was most confident of.  One lane per position.
            const size_t base = (size_t)nd.seq * max_seq_len + nd.S;
            const float c = lane < nd.blen ? ref_conf[base + lane] : -1.f;
            const int rank = rank_among(c, nd.blen >= 64 ? ~0ull : (1ull << nd.blen) - 1ull, lane);
            tok = __builtin_amdgcn_readlane(rank, p) < nd.j ? ref_arg[base + p] : mask_id;
        } else if (g.fresh) {
            tok = mask_id;
        } else {
            // the drafts: lane j holds draft j + 1; a mix-order node skips draft j and holds draft j + 1 instead (Section 5.2)
            const int dpos = lane <= SSD_MAX_DRAFT ? s->draft_pos[lane] : -1, dtok = lane <= SSD_MAX_DRAFT ? s->draft_tok[lane] : 0;
            tok = s->tok[p];
            const unsigned long long in = __ballot((lane < nd.j || lane == nd.extra) && lane <= SSD_MAX_DRAFT && dpos == p);
            if (in) tok = __builtin_amdgcn_readlane(dtok, 63 - __clzll(in));
        }
        if (threadIdx.x == 0) {
            row_desc[row] = nd;
            sh_tok = tok;
        }
    }
    if constexpr (EMBED) {
        __syncthreads();
        // ids are validated on the host or produced by the arg-max; the clamp keeps the gather in bounds whatever a corrupted
        // state holds
        const T* e = embed + (size_t)min(max(sh_tok, 0), V - 1) * d;
        norm_row<T, -1>(h + (size_t)row * d, nullptr, 0, gain, xn + (size_t)row * d, d, eps, e);
    }
}

// Rotary embedding (rotate-half pairing) of Q and K from the fp32 projection (the sum of its
// split-K partial sums, by halves), conversion to the operand type, the fragment-order copies
// of the nodes' own keys and values, and the cache write for nodes that own finished tokens.
// One work-group per (node, 32-row tile, head of Q, K or V): 32 rows x 8 column groups.  Bound by the partial sums'
// bytes; with a split's loads in flight together and the cached values written four positions at a time
// 1000 rows of the 8B shape take 30.5 us (one group after the other, single values: 36.7), 576 rows 13.4 (16.6).
template <typename T, int DH>
__global__ __launch_bounds__(256) void k_rope(const FwdHeader* __restrict__ fw, const float* __restrict__ part,
                                              int n_part, size_t part_stride, const float* __restrict__ cosT,
                                              const float* __restrict__ sinT, T* __restrict__ q,
                                              T* __restrict__ kown, T* __restrict__ vown, int vt_rows,
                                              T* __restrict__ kcache, T* __restrict__ vcache, int Hq, int Hkv,
                                              int layer, int max_seqs, int seq_stride) {
    constexpr int HALF = DH / 2, PT = HALF / 8;          // q/k: values of each rotary half per thread
    constexpr int VPT = DH / 8;                          // v: values per thread
    const NodeDesc nd = fw->nodes[blockIdx.x];
    const int r0 = blockIdx.y * 32;
    if (r0 >= nd.blen) return;
    const int hh = blockIdx.z, tid = threadIdx.x, r = tid >> 3, cg = tid & 7;
    const bool rvalid = r0 + r < nd.blen;
    const int row = nd.row0 + (rvalid ? r0 + r : 0);
    const int pos = nd.S + (rvalid ? r0 + r : 0);
    const int nq = Hq * DH, nkv = Hkv * DH, nqkv = nq + 2 * nkv;
    const float* src = part + (size_t)row * nqkv;
    const size_t cbase = (((size_t)layer * max_seqs + nd.seq) * Hkv) * (size_t)seq_stride * DH;
    // G groups of four values, group j from column col[j], partial sums added by halves; a split's groups are in flight together,
    // and two or three splits where there are two or four
    auto load = [&](auto gc, const int* col, float* dst) {
        constexpr int G = decltype(gc)::value;
        float4 a[G], b[G], t[G];
        auto get = [&](float4(&v)[G], int sp) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < G; ++j) v[j] = *(const float4*)(src + sp * part_stride + col[j]);
        };
        auto add = [&](float4(&v)[G], const float4(&w)[G]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < G; ++j) { v[j].x += w[j].x; v[j].y += w[j].y; v[j].z += w[j].z; v[j].w += w[j].w; }
        };
        get(a, 0);
        if (n_part == 2) {
            get(b, 1);
            add(a, b);
        } else if (n_part == 4) {
            get(b, 1);
            get(t, 2);
            add(a, b);
            get(b, 3);
            add(t, b);
            add(a, t);
        } else if (n_part > 1) {
            const int half = (n_part + 1) >> 1;
            for (int sp = 1; sp < half; ++sp) { get(b, sp); add(a, b); }
            get(t, half);
            for (int sp = half + 1; sp < n_part; ++sp) { get(b, sp); add(t, b); }
            add(a, t);
        }
#pragma unroll
        for (int j = 0; j < G; ++j) { dst[4 * j] = a[j].x; dst[4 * j + 1] = a[j].y; dst[4 * j + 2] = a[j].z; dst[4 * j + 3] = a[j].w; }
    };
    if (hh < Hq + Hkv) {
        const int i0 = cg * PT;
        float x[2 * PT], cs[PT], sn[PT], o1[PT], o2[PT];
        int cols[PT / 2];
#pragma unroll
        for (int j = 0; j < PT / 4; ++j) {
            cols[j] = hh * DH + i0 + 4 * j;
            cols[PT / 4 + j] = cols[j] + HALF;
            const float4 c = ld4_f(cosT + (size_t)pos * HALF + i0 + 4 * j), n = ld4_f(sinT + (size_t)pos * HALF + i0 + 4 * j);
            cs[4 * j] = c.x; cs[4 * j + 1] = c.y; cs[4 * j + 2] = c.z; cs[4 * j + 3] = c.w;
            sn[4 * j] = n.x; sn[4 * j + 1] = n.y; sn[4 * j + 2] = n.z; sn[4 * j + 3] = n.w;
        }
        load(std::integral_constant<int, PT / 2>{}, cols, x);
#pragma unroll
        for (int j = 0; j < PT; ++j) rope_pair(x[j], x[PT + j], cs[j], sn[j], o1[j], o2[j]);
        if (rvalid) {
            if (hh < Hq) {
                T* dst = q + (size_t)row * nq + hh * DH;
#pragma unroll
                for (int j = 0; j < PT; j += 4) {
                    st4(dst + i0 + j, o1[j], o1[j + 1], o1[j + 2], o1[j + 3]);
                    st4(dst + i0 + HALF + j, o2[j], o2[j + 1], o2[j + 2], o2[j + 3]);
                }
            } else {
                // four consecutive channels starting at a multiple of four stay contiguous in fragment order
                const int kvh = hh - Hq;
                T* ko = kown + (size_t)kvh * vt_rows * DH;
                T* kc = kcache + cbase + (size_t)kvh * seq_stride * DH;
                const int prow = nd.vrow0 + r0 + r;
#pragma unroll
                for (int j = 0; j < PT; j += 4) {
                    st4(ko + kfrag_off(prow, i0 + j, DH), o1[j], o1[j + 1], o1[j + 2], o1[j + 3]);
                    st4(ko + kfrag_off(prow, i0 + HALF + j, DH), o2[j], o2[j + 1], o2[j + 2], o2[j + 3]);
                }
                if (nd.write_kv) {
#pragma unroll
                    for (int j = 0; j < PT; j += 4) {
                        st4(kc + kfrag_off(pos, i0 + j, DH), o1[j], o1[j + 1], o1[j + 2], o1[j + 3]);
                        st4(kc + kfrag_off(pos, i0 + HALF + j, DH), o2[j], o2[j + 1], o2[j + 2], o2[j + 3]);
                    }
                }
            }
        }
    } else {
        const int vh = hh - Hq - Hkv, c0 = cg * VPT;
        __shared__ float tile[32][DH + 1];
        float x[VPT];
        int cols[VPT / 4];
#pragma unroll
        for (int j = 0; j < VPT / 4; ++j) cols[j] = nq + nkv + vh * DH + c0 + 4 * j;
        load(std::integral_constant<int, VPT / 4>{}, cols, x);
#pragma unroll
        for (int j = 0; j < VPT; ++j) tile[r][c0 + j] = rvalid ? x[j] : 0.f;
        __syncthreads();
        // thread -> (channel, group of rows): four consecutive positions starting at a multiple of four
        // stay contiguous in fragment order; a node's rows start 64-aligned, rows past its end get zeros
        constexpr int TPC = 256 / DH, RPT = 32 / TPC;    // threads per channel, rows per thread
        const int col = tid / TPC, rg = (tid % TPC) * RPT;
        T* vd = vown + (size_t)vh * vt_rows * DH;
#pragma unroll
        for (int j = 0; j < RPT; j += 4)
            st4(vd + vfrag_off(nd.vrow0 + r0 + rg + j, col, DH), tile[rg + j][col], tile[rg + j + 1][col],
                tile[rg + j + 2][col], tile[rg + j + 3][col]);
        if (nd.write_kv) {
            T* vc = vcache + cbase + (size_t)vh * seq_stride * DH;
            const int p0 = nd.S + r0 + rg, cnt = min(RPT, nd.blen - r0 - rg);
            int j = 0;
            while (j < cnt) {
                // four positions at a time from a multiple of four on, singly in front of it and behind the last four
                if (((p0 + j) & 3) == 0 && j + 4 <= cnt) {
                    st4(vc + vfrag_off(p0 + j, col, DH), tile[rg + j][col], tile[rg + j + 1][col], tile[rg + j + 2][col], tile[rg + j + 3][col]);
                    j += 4;
                } else {
                    st_f(vc + vfrag_off(p0 + j, col, DH), tile[rg + j][col]);
                    ++j;
                }
            }
        }
    }
}

// a4 (plain): one wave per (row, query head).  Keys = the sequence's cached
// prefix [0,S), its cached suffix behind the block if it has one, then the node's own rows; online softmax in fp32 over
// key tiles of 64 in position order.  Keys and values are read 16 bytes per lane; a row's chain of
// FMAs stays in channel and key order, whatever the variant.
// DEEP: for launches that give a SIMD at most one wave, bound by latency.  A tile's values and the next tile's keys are in flight
// while its scores are computed, which takes the SIMD's whole register file (64 cached keys and a block of 32, head size 64, 4
// heads, us, node looked up by two trips, keys and values one trip after the other / this: 7.5 / 5.4).  Otherwise a tile's keys, 64
// channels at a time, then its values, 32 keys at a time: 115 to 144 registers, three or four waves to a SIMD that hide each
// other's trips (both times: attn_plain_deep).
template <typename T, int DH, bool DEEP>
__global__ __launch_bounds__(64) void k_attn_plain(const NodeDesc* __restrict__ row_desc, const T* __restrict__ q,
                                                   const T* __restrict__ kown, const T* __restrict__ vown,
                                                   const T* __restrict__ kcache, const T* __restrict__ vcache,
                                                   T* __restrict__ out, int Hq, int Hkv, int layer, int max_seqs,
                                                   int seq_stride, int vt_rows) {
    constexpr int CH = DH / 64;                              // channels per lane: lane, lane + 64
    const int row = blockIdx.x, head = blockIdx.y, lane = threadIdx.x;
    __shared__ __attribute__((aligned(16))) float qs[DH];
    const int kvh = head / (Hq / Hkv), nq = Hq * DH;
    float q0[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) q0[c] = ld_f(q + (size_t)row * nq + head * DH + c * 64 + lane);
    const NodeDesc nd = row_desc[row];
#pragma unroll
    for (int c = 0; c < CH; ++c) qs[c * 64 + lane] = q0[c];
    __syncthreads();
    const size_t cbase = ((((size_t)layer * max_seqs + nd.seq) * Hkv) + kvh) * (size_t)seq_stride * DH;
    const T* kc = kcache + cbase;
    const T* vc = vcache + cbase;
    const T* ko = kown + (size_t)kvh * vt_rows * DH;
    const T* vo = vown + (size_t)kvh * vt_rows * DH;
    // keys: the cached prefix [0, S), the cached suffix [S + blen, T) if the sequence has one, the node's own rows
    const int n_suf = max(nd.T - (nd.S + nd.blen), 0), n_cache = nd.S + n_suf;
    const int n_keys = n_cache + nd.blen;
    auto cache_pos = [&](int j) { return j < nd.S ? j : j + nd.blen; };
    constexpr int KG = DEEP ? DH / 4 : 16;                   // groups of four channels of a key that are loaded together
    auto load_k = [&](float4(&kv)[KG], int t0, int g0) __attribute__((always_inline)) {
        const int j = min(t0 + lane, n_keys - 1);            // past the last key: that one, not counted
        const bool pre = j < n_cache;
        const T* kp = pre ? kc : ko;
        const int p = pre ? cache_pos(j) : nd.vrow0 + j - n_cache;
#pragma unroll
        for (int i = 0; i < KG; ++i) kv[i] = ld4_f(kp + kfrag_off(p, (g0 + i) * 4, DH));
    };
    // where key jk lies, and how many keys from it on lie at consecutive positions (uniform over the wave)
    auto place = [&](int jk, int end, const T*& vp, int& pp) __attribute__((always_inline)) {
        const bool pre = jk < n_cache;
        vp = pre ? vc : vo;
        pp = pre ? cache_pos(jk) : nd.vrow0 + jk - n_cache;
        return min(end - jk, jk < nd.S ? nd.S - jk : pre ? n_cache - jk : n_keys - jk);
    };
    // 32 keys at consecutive positions from a multiple of four on: four of a channel lie together
    auto load32 = [&](float4(&v)[8][CH], const T* vp, int pp) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < 8; ++g)
#pragma unroll
            for (int c = 0; c < CH; ++c) v[g][c] = ld4_f(vp + vfrag_off(pp + 4 * g, c * 64 + lane, DH));
    };
    auto load_v = [&](float4(&v)[8][CH], int jk, int end) __attribute__((always_inline)) {
        if (jk >= end) return false;
        const T* vp;
        int pp;
        if (place(jk, end, vp, pp) < 32 || (pp & 3)) return false;
        load32(v, vp, pp);
        return true;
    };
    const float scale = 1.0f / sqrtf((float)DH);
    float m = -INFINITY, l = 0.f, o[CH] = {};
    constexpr bool AHEAD = DEEP && DH == 64;                 // 128 channels: no registers for the next tile's keys
    float4 kv[KG], kn[AHEAD ? KG : 1], va[8][CH], vb[8][CH];
    if constexpr (DEEP) load_k(kv, 0, 0);
    for (int t0 = 0; t0 < n_keys; t0 += 64) {
        const int end = min(t0 + 64, n_keys);
        bool fast_a = false, fast_b = false;
        if constexpr (DEEP) {
            fast_a = load_v(va, t0, end);
            fast_b = load_v(vb, t0 + 32, end);
        }
        if constexpr (AHEAD)
            if (t0 + 64 < n_keys) load_k(kn, t0 + 64, 0);
        const int j = t0 + lane;
        float acc = 0.f;
#pragma unroll 1
        for (int g0 = 0; g0 < DH / 4; g0 += KG) {
            if constexpr (!DEEP) load_k(kv, t0, g0);
#pragma unroll
            for (int i = 0; i < KG; ++i) {
                const float4 qv = *(const float4*)&qs[(g0 + i) * 4];
                acc += qv.x * kv[i].x; acc += qv.y * kv[i].y; acc += qv.z * kv[i].z; acc += qv.w * kv[i].w;
            }
        }
        const float s = j < n_keys ? acc * scale : -INFINITY;
        const float m_new = fmaxf(m, wave_max(s));
        const float p = j < n_keys ? expf(s - m_new) : 0.f;
        const float corr = expf(m - m_new);
        l = l * corr + wave_sum(p);
#pragma unroll
        for (int c = 0; c < CH; ++c) o[c] *= corr;
        auto weight = [&](int jj) { return lane_value(p, jj); };
        auto add32 = [&](const float4(&v)[8][CH], int jj) __attribute__((always_inline)) {
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const float w0 = weight(jj + 4 * g), w1 = weight(jj + 4 * g + 1), w2 = weight(jj + 4 * g + 2), w3 = weight(jj + 4 * g + 3);
#pragma unroll
                for (int c = 0; c < CH; ++c) { o[c] += w0 * v[g][c].x; o[c] += w1 * v[g][c].y; o[c] += w2 * v[g][c].z; o[c] += w3 * v[g][c].w; }
            }
        };
        // the tile's keys [jj, stop) whose values are not on their way
        auto walk = [&](int jj, int stop) __attribute__((always_inline)) {
            while (jj < stop) {
                const T* vp;
                int pp;
                const int run = place(t0 + jj, t0 + stop, vp, pp);
                if (!DEEP && run >= 32 && (pp & 3) == 0) {
                    load32(va, vp, pp);
                    add32(va, jj);
                    jj += 32;
                } else if (run >= 8) {
                    float a[8][CH];
#pragma unroll
                    for (int g = 0; g < 8; ++g)
#pragma unroll
                        for (int c = 0; c < CH; ++c) a[g][c] = ld_f(vp + vfrag_off(pp + g, c * 64 + lane, DH));
#pragma unroll
                    for (int g = 0; g < 8; ++g)
#pragma unroll
                        for (int c = 0; c < CH; ++c) o[c] += weight(jj + g) * a[g][c];
                    jj += 8;
                } else {
#pragma unroll
                    for (int c = 0; c < CH; ++c) o[c] += weight(jj) * ld_f(vp + vfrag_off(pp, c * 64 + lane, DH));
                    ++jj;
                }
            }
        };
        if constexpr (DEEP) {
            if (fast_a) add32(va, 0);
            else walk(0, min(32, n_keys - t0));
            if (fast_b) add32(vb, 32);
            else walk(32, min(64, n_keys - t0));
        } else walk(0, min(64, n_keys - t0));
        m = m_new;
        if (DEEP && t0 + 64 < n_keys) {
            if constexpr (AHEAD)
#pragma unroll
                for (int i = 0; i < KG; ++i) kv[i] = kn[i];
            else load_k(kv, t0 + 64, 0);
        }
    }
    T* op = out + (size_t)row * nq + head * DH;
#pragma unroll
    for (int c = 0; c < CH; ++c) st_f(op + c * 64 + lane, o[c] / l);
}

// ------------------------------------------------------------------------
// Plain GEMM  out[M,N] = X[M,K] * W[N,K]^T  in fp32 (bf16 operands widened), on the fp32 matrix cores.
// The order of an output's sum, the same in both kernels: the columns in steps of 16, the steps in eight chains of ceil(steps
// / 8) consecutive ones, a step as four 16x16x4 MFMAs, MFMA i over its columns 4q + i, q = 0 ... 3; the chains are
// added in order.  A lane's operands of a step's four MFMAs are four consecutive columns of one row: one 16-byte load,
// straight from memory into the registers that the matrix core reads.  Columns past K (a multiple of 8) count as zeros.
// ------------------------------------------------------------------------
#define PBM GEMM_PLAIN_TILE
#define PBN GEMM_PLAIN_TILE
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Four consecutive values as they lie in memory, to wait in registers.
template <typename T> struct Four;
template <> struct Four<float> { typedef float4 type; };
template <> struct Four<bf16_t> { typedef uint2 type; };
__device__ __forceinline__ float4 widen(const float4& v) { return v; }
__device__ __forceinline__ float4 widen(const uint2& v) {
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xffff0000u));
}
// The four from p on, or zeros.  VEC: the address is a multiple of four elements.
template <bool VEC>
__device__ __forceinline__ float4 get_four(const float* p, bool ok) {
    if (!ok) return make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (VEC) return *(const float4*)p;
    else return make_float4(p[0], p[1], p[2], p[3]);
}
template <bool VEC>
__device__ __forceinline__ uint2 get_four(const bf16_t* p, bool ok) {
    if (!ok) return make_uint2(0, 0);
    if constexpr (VEC) return *(const uint2*)p;
    else return make_uint2(p[0] | ((uint32_t)p[1] << 16), p[2] | ((uint32_t)p[3] << 16));
}
// One step of one chain: lane (q, j) = (lane / 16, lane % 16) holds columns 4q ... 4q + 3 of weight row j and of row j of X;
// it ends up with weight rows 4q ... 4q + 3 of row j.
__device__ __forceinline__ floatx4 mfma_step(const float4& w, const float4& x, floatx4 acc) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, x.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, x.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, x.z, acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, x.w, acc, 0, 0, 0);
}

// Fused LM-head reduction over 16 adjacent lanes that hold NJ consecutive logits each, from vocabulary row n0 of this
// lane on: max logit, its lowest index, sum of exp(logit - max).  The mask token takes no part.
template <int NJ>
__device__ __forceinline__ void lm_row_partial(const float (&v)[NJ], int n0, int N, int mask_id, bool store, float* o) {
    float bm = -INFINITY;
    int bi = 0x7fffffff;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int n = n0 + j;
        if (n < N && n != mask_id && v[j] > bm) { bm = v[j]; bi = n; }
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        const float om = __shfl_xor(bm, off, 64);
        const int oi = __shfl_xor(bi, off, 64);
        if (om > bm || (om == bm && oi < bi)) { bm = om; bi = oi; }
    }
    float se = 0.f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int n = n0 + j;
        if (n < N && n != mask_id) se += expf(v[j] - bm);
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) se += __shfl_xor(se, off, 64);
    if (store) {
        o[0] = bm;
        o[1] = __int_as_float(bi);
        o[2] = se;
    }
}

// 64x64 tile per work-group, 2x2 waves of 32x32: 2x2 MFMA tiles.  LINE steps' operands are loaded while the LINE steps before them
// are multiplied: in bf16 the four steps of a 128-byte line, which one at a time fetch it four times once the work-groups of a CU
// need more lines than its L1 holds.  Bound: the caches; every operand is requested by the two waves that need it.  160 rows, K = 12288,
// N = 4096, us, fp32, FMAs through LDS / this: 697 / 462; bf16, FMAs / one step at a time / this: 192 rows 763 / 737 / 368, gate/up
// of 18944 channels, K = 3584, 256 rows 1485 / 1600 / 862.  (fp32 by lines of two steps: 407 against 486 where the grid is one
// round, 1807 against 1587 where it is several.)
template <typename T, int EPI, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_plain(const T* __restrict__ X, const T* __restrict__ W,
                                                    void* __restrict__ outv, int M, int N, int K, int up_off,
                                                    int mask_id, int n_tiles) {
    constexpr int NU = EPI == EPI_SWIGLU ? 2 : 1;         // gate rows and up rows
    __shared__ float lg[EPI == EPI_LMHEAD ? PBM : 1][EPI == EPI_LMHEAD ? PBN + 4 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, j = lane & 15;
    const int m0 = blockIdx.y * PBM + (wave >> 1) * 32, n0 = blockIdx.x * PBN + (wave & 1) * 32;
    floatx4 acc[NU][2][2], tot[NU][2][2];                 // [gate, up][n-tile][m-tile]: a chain, the chains before it
    constexpr int LINE = sizeof(T) == 2 ? 4 : 1;          // steps whose operands are loaded together
    typename Four<T>::type w[2][LINE][NU][2], x[2][LINE][2];
    const T *xr[2], *wr[NU][2];                           // rows past the end read the last one (never stored)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        xr[t] = X + (size_t)min(m0 + t * 16 + j, M - 1) * K;
#pragma unroll
        for (int u = 0; u < NU; ++u) wr[u][t] = W + (size_t)(u * up_off + min(n0 + t * 16 + j, N - 1)) * K;
    }
    auto load = [&](int buf, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LINE; ++i) {
            const int k = (s + i) * 16 + q * 4;
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                x[buf][i][t] = get_four<VEC>(xr[t] + k, k < K);
#pragma unroll
                for (int u = 0; u < NU; ++u) w[buf][i][u][t] = get_four<VEC>(wr[u][t] + k, k < K);
            }
        }
    };
    const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    const int steps = (K + 15) >> 4, len = (steps + 7) >> 3;
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[u][a][b] = tot[u][a][b] = zero;
    auto close = [&]() __attribute__((always_inline)) {   // the end of a chain
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) { tot[u][a][b] += acc[u][a][b]; acc[u][a][b] = zero; }
    };
    load(0, 0);
    int left = len;
    for (int s0 = 0; s0 < steps; s0 += 2 * LINE)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int s = s0 + c * LINE;
            if (s >= steps) break;
            load(c ^ 1, s + LINE);                        // past the end: zeros, unused
#pragma unroll
            for (int i = 0; i < LINE; ++i) {
                if (s + i >= steps) break;
#pragma unroll
                for (int u = 0; u < NU; ++u)
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int b = 0; b < 2; ++b) acc[u][a][b] = mfma_step(widen(w[c][i][u][a]), widen(x[c][i][b]), acc[u][a][b]);
                if (--left == 0) { close(); left = len; }
            }
        }
    close();
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            floatx4 v[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) v[u] = tot[u][a][b];
            const int m = m0 + b * 16 + j, n = n0 + a * 16 + q * 4;
            if constexpr (EPI == EPI_LMHEAD) {
#pragma unroll
                for (int i = 0; i < 4; ++i) lg[(wave >> 1) * 32 + b * 16 + j][(wave & 1) * 32 + a * 16 + q * 4 + i] = v[0][i];
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (m >= M || n + i >= N) continue;
                    if constexpr (EPI == EPI_F32) ((float*)outv)[(size_t)m * N + n + i] = v[0][i];
                    else st_f((T*)outv + (size_t)m * N + n + i, v[0][i] / (1.0f + expf(-v[0][i])) * v[NU - 1][i]);
                }
            }
        }
    if constexpr (EPI == EPI_LMHEAD) {
        // per row, over this tile's 64 vocabulary columns; the 16 threads of a row are 16 adjacent lanes
        __syncthreads();
        float* out = (float*)outv;
        const int tx = tid & 15;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = (tid >> 4) * 4 + i, m = blockIdx.y * PBM + r;
            const float v[4] = {lg[r][tx * 4], lg[r][tx * 4 + 1], lg[r][tx * 4 + 2], lg[r][tx * 4 + 3]};
            lm_row_partial<4>(v, blockIdx.x * PBN + tx * 4, N, mask_id, tx == 0 && m < M, out + ((size_t)m * n_tiles + blockIdx.x) * 3);
        }
    }
}

// The same sums for launches whose 64x64 tiles would leave most of the chip idle (small models, few rows): 16 rows x 16
// outputs per work-group (LM head: 16 x 64, the width of a partial), one wave per chain; gate and up rows, and two halves of the
// LM head's columns, have waves of their own.  Bound: launch, one trip to memory, a chain's MFMAs; four steps' loads are in
// flight together (K up to 512 in one trip).  Operands must be 16-byte aligned.
// Measured, fp32, 32 rows (K x N, us, FMAs of 8x16 tiles through LDS / this): 256 x 768 5.5 / 3.6, 256 and 768 x 256 8.7 / 4.5,
// gate/up 256 x 768 6.7 / 4.6, LM head 256 x 1024 9.0 / 6.2; four chains instead of eight, twice the steps each: 4.6, 6.1, 6.6, 10.5.
// bf16 waits in registers as it lies in memory (36 to 49 instead of 52 to 74; gate/up 512 x 1536, us, FMAs / widened at once / this:
// 96 rows 13.6 / 15.2 / 13.3, 256 rows 28.5 / 32.2 / 24.5).
template <typename T, int EPI>
__global__ __launch_bounds__(EPI == EPI_F32 ? 512 : 1024) void k_gemm_plain_small(
    const T* __restrict__ X, const T* __restrict__ W, void* __restrict__ outv, int M, int N, int K, int up_off, int mask_id,
    int n_tiles) {
    constexpr int NG = EPI == EPI_F32 ? 1 : EPI == EPI_SWIGLU ? 2 : 4;       // groups of 16 weight rows
    constexpr int GW = EPI == EPI_LMHEAD ? 2 : 1, TN = EPI == EPI_LMHEAD ? 64 : 16, BATCH = 4;     // groups per wave
    __shared__ __attribute__((aligned(16))) float part[NG][8][16][20];       // [group][chain][row][16 outputs, padded]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, chain = wave & 7, h = wave >> 3, q = lane >> 4, j = lane & 15;
    const int m0 = blockIdx.y * 16, n0 = blockIdx.x * TN;
    const int steps = (K + 15) >> 4, len = (steps + 7) >> 3, s0 = chain * len, cnt = min(len, steps - s0);
    const T* xr = X + (size_t)min(m0 + j, M - 1) * K + s0 * 16 + q * 4;      // rows past the end: the last one, never stored
    const T* wr[GW];
#pragma unroll
    for (int g = 0; g < GW; ++g) {
        const int n = EPI == EPI_SWIGLU ? h * up_off + min(n0 + j, N - 1) : min(n0 + (h * GW + g) * 16 + j, N - 1);
        wr[g] = W + (size_t)n * K + s0 * 16 + q * 4;
    }
    const int kleft = K - s0 * 16 - q * 4;                                   // this lane's columns are below K while > 0
    floatx4 acc[GW];
#pragma unroll
    for (int g = 0; g < GW; ++g) acc[g] = {0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < cnt; s += BATCH) {
        typename Four<T>::type w[GW][BATCH], x[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            if (s + i < cnt) {
                const bool ok = (s + i) * 16 < kleft;
                x[i] = get_four<true>(xr + (s + i) * 16, ok);
#pragma unroll
                for (int g = 0; g < GW; ++g) w[g][i] = get_four<true>(wr[g] + (s + i) * 16, ok);
            }
#pragma unroll
        for (int i = 0; i < BATCH; ++i)
            if (s + i < cnt)
#pragma unroll
                for (int g = 0; g < GW; ++g) acc[g] = mfma_step(widen(w[g][i]), widen(x[i]), acc[g]);
    }
#pragma unroll
    for (int g = 0; g < GW; ++g) *(floatx4*)&part[h * GW + g][chain][j][q * 4] = acc[g];
    __syncthreads();
    if (tid >= 256) return;
    const int r = tid >> 4, c = tid & 15, m = m0 + r;
    auto sum = [&](int g, int col) {
        float v = 0.f;
#pragma unroll
        for (int p = 0; p < 8; ++p) v += part[g][p][r][col];
        return v;
    };
    if constexpr (EPI == EPI_LMHEAD) {
        const int g = c >> 2, col = (c & 3) * 4;
        const float v[4] = {sum(g, col), sum(g, col + 1), sum(g, col + 2), sum(g, col + 3)};
        lm_row_partial<4>(v, n0 + c * 4, N, mask_id, c == 0 && m < M, (float*)outv + ((size_t)m * n_tiles + blockIdx.x) * 3);
    } else {
        const int n = n0 + c;
        if (m >= M || n >= N) return;
        if constexpr (EPI == EPI_F32) ((float*)outv)[(size_t)m * N + n] = sum(0, c);
        else {
            const float g = sum(0, c);
            st_f((T*)outv + (size_t)m * N + n, g / (1.0f + expf(-g)) * sum(NG - 1, c));
        }
    }
}

// Merge the per-tile (max, arg, sumexp) triples of a row: the maximum first, then every tile's sum scaled to it, added in an
// order that depends on the tile count alone (tile t by thread t mod 256, ascending; the lanes of a wave; the four waves).
// Ties keep the lowest token id.  Bound by latency: folding pairs of triples lane by lane through LDS took two exponentials
// and three shuffles a step (us before / now: 1024 tokens, 32 rows 3.9 / 2.5; 2080 tokens, 192 rows 5.0 / 2.6).
__global__ __launch_bounds__(256) void k_lm_merge(const float* __restrict__ part, int n_tiles,
                                                  float* __restrict__ row_max, int* __restrict__ row_arg,
                                                  float* __restrict__ row_conf, int V, int mask_id) {
    __shared__ float sm[4], ss[4];
    __shared__ int sa[4];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* p = part + (size_t)row * n_tiles * 3;
    float m = -INFINITY;
    for (int t = tid; t < n_tiles; t += 256) m = fmaxf(m, p[3 * t]);
    m = wave_max(m);
    if (lane == 0) sm[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
    float s = 0.f;
    int a = 0x7fffffff;
    for (int t = tid; t < n_tiles; t += 256) {
        const float tm = p[3 * t];
        const int ta = __float_as_int(p[3 * t + 1]);
        const float ts = p[3 * t + 2];
        if (tm == m && ta < a) a = ta;
        if (ts != 0.f) s += ts * expf(tm - m);           // 0: a tile without tokens
    }
    s = wave_sum(s);
    a = wave_min(a);
    if (lane == 0) { ss[wave] = s; sa[wave] = a; }
    __syncthreads();
    if (tid == 0) {
        s = ((ss[0] + ss[1]) + ss[2]) + ss[3];
        a = min(min(sa[0], sa[1]), min(sa[2], sa[3]));
        // Non-finite logits (NaN weights) leave no arg-max: fall back to the lowest valid id and
        // confidence 0 so that every later step stays well defined and in bounds.
        if ((unsigned)a >= (unsigned)V) a = mask_id == 0 ? 1 : 0;
        float conf = 1.0f / s;             // softmax probability of the arg-max (Section 3.2.2)
        if (!(conf >= 0.f && conf <= 1.f)) conf = 0.f;
        row_max[row] = m;
        row_arg[row] = a;
        row_conf[row] = conf;
    }
}

// ------------------------------------------------------------------------
// a11: acceptance (Section 3.2.4).  One wave per decode group, one lane per
// block position.  Walks the chain: node m's stepwise choice (most confident
// masked position, ties to the lowest position) must equal draft m+1 in
// position and token; stops at the first mismatch; accepts the matched drafts
// plus the choice of the node it stopped at; ranks that node's remaining
// masked positions by confidence for the next drafts; commits to the state.
// With mix-order nodes in the group (Section 5.2) a mismatch whose choice is
// draft m+2 accepts that draft and ends at the node holding drafts 1..m, m+2.
// Bound by latency: the confidences and tokens of all nodes come in one trip and wait in LDS, a choice is a reduction without
// LDS, ranks count over the open positions alone (us, a trip and shuffles per node and 64 shuffles per ranking / this: one
// node of 32 positions 6.9 / 3.9, two sequences of four nodes 11.1 / 5.2).
// ------------------------------------------------------------------------
#define ACCEPT_NODES (2 * SSD_MAX_DRAFT + 1)              // a chain and its mix-order nodes
__global__ __launch_bounds__(64) void k_accept(const FwdHeader* __restrict__ fw, SeqState* __restrict__ state,
                                               const float* __restrict__ row_conf, const int* __restrict__ row_arg,
                                               const float* __restrict__ row_max, StepResult* __restrict__ result,
                                               int* __restrict__ out_tok, int max_seq_len, int blockB, int maxDraft,
                                               int mask_id, float* __restrict__ ref_conf, int* __restrict__ ref_arg) {
    const int gi = blockIdx.x, lane = threadIdx.x;
    const GroupDesc g = fw->groups[gi];
    const ssd_step_out out = fw->out;
    if (g.mode == GM_RAW && g.keep_ref) {
        // rows of a cache refresh behind the current block: their predictions are the drafts later blocks
        // start from (Section 3.2.2: candidates from the next block; Section 4.1: the refresh covers all positions)
        for (int p = lane; p < g.blen; p += 64) {
            ref_conf[(size_t)g.seq * max_seq_len + g.S + p] = row_conf[g.row0 + p];
            ref_arg[(size_t)g.seq * max_seq_len + g.S + p] = row_arg[g.row0 + p];
        }
        return;
    }
    if (g.mode != GM_DECODE || g.spec_of1 != 0) return;   // a speculative group is its master's business
    SeqState* s = &state[g.seq];
    // drafts = chain nodes - 1, or one per chain node if the node holding all of them was left out
    const int nd = g.leafless ? g.n_chain : g.n_chain - 1;
    const int blen = g.blen;
    __shared__ int sh_pos[64], sh_tok[64];
    // drafts read off the last refresh: the block's positions by descending confidence; lane k gets draft k
    auto drafts_from_refresh = [&](int S_blk, int blen_blk, int& dpos, int& dtok) {
        const size_t base = (size_t)g.seq * max_seq_len + S_blk;
        const float cr = lane < blen_blk ? ref_conf[base + lane] : -1.f;
        const int rank = rank_among(cr, blen_blk >= 64 ? ~0ull : (1ull << blen_blk) - 1ull, lane);
        __syncthreads();
        if (lane < blen_blk) { sh_pos[rank] = lane; sh_tok[rank] = ref_arg[base + lane]; }
        __syncthreads();
        dpos = lane < blen_blk ? sh_pos[lane] : -1;
        dtok = lane < blen_blk ? sh_tok[lane] : -1;
    };
    int my_dpos = lane <= SSD_MAX_DRAFT ? s->draft_pos[lane] : -1;
    int my_dtok = lane <= SSD_MAX_DRAFT ? s->draft_tok[lane] : -1;
    if (g.from_refresh) drafts_from_refresh(g.S, blen, my_dpos, my_dtok);
    // a fresh block starts all masked with no drafts (Algorithm 1, start of a block); its state is written here,
    // at the end of the forward, so that a KV-append group of the same sequence in the same forward
    // still reads the finished block's tokens
    unsigned long long cur = g.fresh ? (blen >= 64 ? ~0ull : ((1ull << blen) - 1ull)) : s->masked;
    __syncthreads();

    __shared__ float node_conf[ACCEPT_NODES][64];
    __shared__ int node_arg[ACCEPT_NODES][64];
    if (lane < blen) {
        const int n_nodes = min(g.n_nodes, ACCEPT_NODES);
        for (int j0 = 0; j0 < n_nodes; j0 += 8) {
            float cf[8], mx[8];
            int ar[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = g.row0 + min(j0 + i, n_nodes - 1) * blen + lane;
                cf[i] = row_conf[row];
                ar[i] = row_arg[row];
                mx[i] = row_max[row];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = j0 + i;
                if (j >= n_nodes) break;
                node_conf[j][lane] = cf[i];
                node_arg[j][lane] = ar[i];
                if (j >= g.n_chain || j > maxDraft) continue;
                const size_t o = ((size_t)gi * (maxDraft + 1) + j) * blockB + lane;
                if (out.row_maxlogit) out.row_maxlogit[o] = mx[i];
                if (out.row_argmax) out.row_argmax[o] = ar[i];
                if (out.row_conf) out.row_conf[o] = cf[i];
            }
        }
    }
    __syncthreads();

    // stepwise choice of a node over the positions still masked in `cur`: highest confidence (not a number counts as 0), ties
    // to the lowest position; leaves this lane's confidence in c.  conf: of position `lane`
    int pstar = 0, tstar = 0;
    float c = -1.f;
    auto choose_from = [&](float conf, int bl) {
        const bool valid = lane < bl && ((cur >> lane) & 1ull);
        c = valid ? (conf == conf ? conf : 0.f) : -INFINITY;
        const float top = wave_max(c);
        const unsigned long long best = __ballot(valid && c == top);
        pstar = best ? __ffsll(best) - 1 : 0;
    };
    auto choose_at = [&](int row0, int bl) {              // rows row0 + lane
        choose_from(lane < bl ? row_conf[row0 + lane] : 0.f, bl);
        tstar = __builtin_amdgcn_readfirstlane(row_arg[row0 + pstar]);
    };
    auto choose = [&](int node) {
        choose_from(lane < blen ? node_conf[node][lane] : 0.f, blen);
        tstar = __builtin_amdgcn_readfirstlane(node_arg[node][pstar]);
    };
    int m = 0;
    bool complete = false;
    while (true) {
        if (cur == 0ull) { complete = true; break; }     // the drafts covered every masked position
        choose(m);
        const int dp = __builtin_amdgcn_readlane(my_dpos, m), dt = __builtin_amdgcn_readlane(my_dtok, m);
        if (m < nd && pstar == dp && tstar == dt) {
            cur &= ~(1ull << pstar);
            ++m;
            continue;
        }
        break;
    }
    StepResult* r = &result[g.seq];
    if (complete) {
        // Every draft verified and the block is finished (Section 3.2.2, the round across the block
        // boundary).  Its tokens go to the output (exact cache: its KV was written by the leaf in this
        // forward).  The group behind it, if any, holds the next block: all masked, then with the drafts
        // the last refresh gives it written in.  The walk goes on there: its matched drafts and the
        // choice of the node it stops at are further accepted tokens (positions counted on from this
        // block's length), and that node's other positions give the next drafts.
        if (g.fresh) s->tok[lane] = mask_id;
        __syncthreads();
        if (lane < m) {
            r->acc_pos[lane] = my_dpos;
            r->acc_tok[lane] = my_dtok;
            s->tok[my_dpos] = my_dtok;
            if (out.acc_pos) out.acc_pos[(size_t)gi * (maxDraft + 1) + lane] = my_dpos;
            if (out.acc_tok) out.acc_tok[(size_t)gi * (maxDraft + 1) + lane] = my_dtok;
        }
        __syncthreads();
        if (g.out_off >= 0 && lane < blen) out_tok[(size_t)g.seq * max_seq_len + g.out_off + lane] = s->tok[lane];
        __syncthreads();
        int n_acc = m, n_next = 0, n_in_next = 0;
        unsigned long long rem = 0ull;
        if (g.spec_next1 != 0) {
            const GroupDesc g2 = fw->groups[g.spec_next1 - 1];
            const int blen2 = g2.blen, nd2 = g2.n_chain - 1;
            int dpos2 = -1, dtok2 = -1;
            if (g2.from_refresh) drafts_from_refresh(g2.S, blen2, dpos2, dtok2);
            cur = blen2 >= 64 ? ~0ull : ((1ull << blen2) - 1ull);
            int k = 0;
            while (true) {
                choose_at(g2.row0 + k * blen2, blen2);
                const int dp = __builtin_amdgcn_readlane(dpos2, k), dt = __builtin_amdgcn_readlane(dtok2, k);
                if (k < nd2 && pstar == dp && tstar == dt) {
                    cur &= ~(1ull << pstar);
                    ++k;
                    continue;
                }
                break;
            }
            rem = cur & ~(1ull << pstar);
            const int n_rem = __popcll(rem);
            n_next = min(g2.n_draft_next, g2.allow_full ? n_rem : max(n_rem - 1, 0));
            const bool mine = (rem >> lane) & 1ull;
            const int rank = n_next > 0 ? rank_among(c, rem, lane) : 0;
            const int my_tok = row_arg[g2.row0 + k * blen2 + (lane < blen2 ? lane : 0)];
            if (mine && rank < n_next) {
                r->next_pos[rank] = lane;
                r->next_tok[rank] = my_tok;
                s->draft_pos[rank] = lane;
                s->draft_tok[rank] = my_tok;
                if (out.next_pos) out.next_pos[(size_t)gi * maxDraft + rank] = lane;
                if (out.next_tok) out.next_tok[(size_t)gi * maxDraft + rank] = my_tok;
            }
            s->tok[lane] = mask_id;
            __syncthreads();
            if (lane <= k) {
                // the next block's matched drafts, then the choice of the node the walk stopped at
                const int ap = lane < k ? dpos2 : pstar, at = lane < k ? dtok2 : tstar;
                s->tok[ap] = at;
                r->acc_pos[m + lane] = blen + ap;
                r->acc_tok[m + lane] = at;
                if (out.acc_pos) out.acc_pos[(size_t)gi * (maxDraft + 1) + m + lane] = blen + ap;
                if (out.acc_tok) out.acc_tok[(size_t)gi * (maxDraft + 1) + m + lane] = at;
            }
            n_in_next = k + 1;
            n_acc = m + n_in_next;
        }
        if (lane == 0) {
            r->n_accept = n_acc;
            r->n_next = n_next;
            r->completed = 1;
            r->n_in_next = n_in_next;
            s->masked = rem;
            s->n_draft = n_next;
            if (out.n_accept) out.n_accept[gi] = n_acc;
            if (out.n_next) out.n_next[gi] = n_next;
        }
        return;
    }
    // mix order (Section 5.2): the choice is the draft after the expected one -> accept it and take
    // one more token from the node that holds drafts 1..m and m+2; that node has no children
    int last = m, res_pos = -1, res_tok = -1;
    if (g.n_nodes > g.n_chain && m + 1 < nd) {
        const int dp2 = __builtin_amdgcn_readlane(my_dpos, m + 1), dt2 = __builtin_amdgcn_readlane(my_dtok, m + 1);
        if (pstar == dp2 && tstar == dt2) {
            res_pos = pstar;
            res_tok = tstar;
            cur &= ~(1ull << pstar);
            last = g.n_chain + m;
            choose(last);
        }
    }
    const int n_acc = m + 1 + (res_pos >= 0 ? 1 : 0);
    const unsigned long long rem = cur & ~(1ull << pstar);
    const int n_rem = __popcll(rem);
    // the leaf keeps one masked position to predict, unless a next block exists for it to reach into
    const int n_next = min(g.n_draft_next, g.allow_full ? n_rem : max(n_rem - 1, 0));
    const bool mine = (rem >> lane) & 1ull;
    const int rank = n_next > 0 ? rank_among(c, rem, lane) : 0;
    const int my_tok = node_arg[last][lane < blen ? lane : 0];
    if (mine && rank < n_next) {
        r->next_pos[rank] = lane;
        r->next_tok[rank] = my_tok;
        s->draft_pos[rank] = lane;
        s->draft_tok[rank] = my_tok;
        if (out.next_pos) out.next_pos[(size_t)gi * maxDraft + rank] = lane;
        if (out.next_tok) out.next_tok[(size_t)gi * maxDraft + rank] = my_tok;
    }
    if (g.fresh) s->tok[lane] = mask_id;                  // SSD_MAX_BLOCK = 64 = one lane per position
    __syncthreads();
    if (lane < n_acc) {
        // the matched drafts, then (mix order) the out-of-order draft, then the last node's own choice
        const int ap = lane < m ? my_dpos : (lane == n_acc - 1 ? pstar : res_pos);
        const int at = lane < m ? my_dtok : (lane == n_acc - 1 ? tstar : res_tok);
        r->acc_pos[lane] = ap;
        r->acc_tok[lane] = at;
        s->tok[ap] = at;
        if (out.acc_pos) out.acc_pos[(size_t)gi * (maxDraft + 1) + lane] = ap;
        if (out.acc_tok) out.acc_tok[(size_t)gi * (maxDraft + 1) + lane] = at;
    }
    if (lane == 0) {
        r->n_accept = n_acc;
        r->n_next = n_next;
        r->completed = 0;
        r->n_in_next = 0;
        s->masked = rem;
        s->n_draft = n_next;
        if (out.n_accept) out.n_accept[gi] = n_acc;
        if (out.n_next) out.n_next[gi] = n_next;
    }
}

// ------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------
void launch_stage(const ssd_ctx* c, const void* pinned, const StageLayout& lay, hipStream_t st) {
    k_stage<<<1, 1024, 0, st>>>((const int*)pinned, lay, (int*)c->b.fwd, c->b.raw_tok, (int*)c->b.state);
}

template <typename T, bool EMBED>
static void rows_t(const ssd_ctx* c, int M, int n_nodes, const float* gain, hipStream_t st) {
    k_rows<T, EMBED><<<M, EMBED ? NORM_T : 64, 0, st>>>(c->b.fwd, n_nodes, c->b.state, c->b.raw_tok, c->b.row_desc, c->b.out_tok,
                                                       c->dm.mask_id, c->dm.max_seq_len, c->b.ref_conf, c->b.ref_arg,
                                                       (const T*)c->embed, c->b.h, gain, (T*)c->b.xn, c->dm.d, c->dm.V, c->dm.eps);
}

void launch_rows(const ssd_ctx* c, int M, int n_nodes, const float* gain, hipStream_t st) {
    if (c->dm.dtype == SSD_F32) gain ? rows_t<float, true>(c, M, n_nodes, gain, st) : rows_t<float, false>(c, M, n_nodes, gain, st);
    else gain ? rows_t<bf16_t, true>(c, M, n_nodes, gain, st) : rows_t<bf16_t, false>(c, M, n_nodes, gain, st);
}

void launch_norm(const ssd_ctx* c, int M, const float* gain, int n_part, hipStream_t st) {
    const size_t stride = (size_t)c->dm.max_rows * c->part_cols;
    if (c->dm.dtype == SSD_F32)
        k_norm<float><<<M, NORM_T, 0, st>>>(c->b.h, c->b.part, n_part, stride, gain, (float*)c->b.xn, c->dm.d, c->dm.eps);
    else
        k_norm<bf16_t><<<M, NORM_T, 0, st>>>(c->b.h, c->b.part, n_part, stride, gain, (bf16_t*)c->b.xn, c->dm.d,
                                          c->dm.eps);
}

void launch_rope(const ssd_ctx* c, int n_nodes, int max_blen, int layer, int n_part, hipStream_t st) {
    const Dims& d = c->dm;
    const size_t ps = (size_t)d.max_rows * c->part_cols;
    dim3 grid(n_nodes, (max_blen + 31) / 32, d.Hq + 2 * d.Hkv);
#define SSD_ROPE_ARGS(T)                                                                                           \
    c->b.fwd, c->b.part, n_part, ps, c->b.rope_cos, c->b.rope_sin, (T*)c->b.q, (T*)c->b.kown, (T*)c->b.vown,        \
        d.vt_rows(), (T*)c->b.kcache, (T*)c->b.vcache, d.Hq, d.Hkv, layer, d.max_seqs, d.seq_stride()
    if (d.dtype == SSD_F32) {
        if (d.dh == 128) k_rope<float, 128><<<grid, 256, 0, st>>>(SSD_ROPE_ARGS(float));
        else k_rope<float, 64><<<grid, 256, 0, st>>>(SSD_ROPE_ARGS(float));
    } else {
        if (d.dh == 128) k_rope<bf16_t, 128><<<grid, 256, 0, st>>>(SSD_ROPE_ARGS(bf16_t));
        else k_rope<bf16_t, 64><<<grid, 256, 0, st>>>(SSD_ROPE_ARGS(bf16_t));
    }
#undef SSD_ROPE_ARGS
}

template <typename T>
static void attn_plain_t(const ssd_ctx* c, int M, int layer, hipStream_t st) {
    const Dims& d = c->dm;
    const dim3 grid(M, d.Hq);
    auto run = [&](auto dh, auto deep) {
        k_attn_plain<T, decltype(dh)::value, decltype(deep)::value><<<grid, 64, 0, st>>>(c->b.row_desc, (const T*)c->b.q, (const T*)c->b.kown, (const T*)c->b.vown,
                                                                  (const T*)c->b.kcache, (const T*)c->b.vcache, (T*)c->b.attn, d.Hq, d.Hkv,
                                                                  layer, d.max_seqs, d.seq_stride(), d.vt_rows());
    };
    const bool deep = attn_plain_deep((long long)M * d.Hq, d.dh, sizeof(T));
    if (d.dh == 64) deep ? run(std::integral_constant<int, 64>{}, std::true_type{}) : run(std::integral_constant<int, 64>{}, std::false_type{});
    else if constexpr (sizeof(T) == 4) deep ? run(std::integral_constant<int, 128>{}, std::true_type{}) : run(std::integral_constant<int, 128>{}, std::false_type{});
    else run(std::integral_constant<int, 128>{}, std::false_type{});
}

void launch_attn_plain(const ssd_ctx* c, int M, int layer, hipStream_t st) {
    if (c->dm.dtype == SSD_F32) attn_plain_t<float>(c, M, layer, st);
    else attn_plain_t<bf16_t>(c, M, layer, st);
}

template <typename T>
static void gemm_plain_t(const ssd_ctx* c, int epi, const T* X, const T* W, void* out, int M, int N, int K,
                         hipStream_t st) {
    const unsigned tiles = (N + PBN - 1) / PBN;
    const int mask = c->dm.mask_id;
    if (gemm_plain_small_tiles(X, W, M, N) && gemm_plain_small_wins(M, N)) {
        const unsigned gy = (M + 15) / 16;
        const dim3 grid((N + 15) / 16, gy);
        if (epi == EPI_F32) k_gemm_plain_small<T, EPI_F32><<<grid, 512, 0, st>>>(X, W, out, M, N, K, 0, -1, 0);
        else if (epi == EPI_SWIGLU) k_gemm_plain_small<T, EPI_SWIGLU><<<grid, 1024, 0, st>>>(X, W, out, M, N, K, N, -1, 0);
        else k_gemm_plain_small<T, EPI_LMHEAD><<<dim3(tiles, gy), 1024, 0, st>>>(X, W, out, M, N, K, 0, mask, (int)tiles);
        return;
    }
    const dim3 grid(tiles, (M + PBM - 1) / PBM);
    auto run = [&](auto vec) {
        constexpr bool VEC = decltype(vec)::value;
        if (epi == EPI_F32) k_gemm_plain<T, EPI_F32, VEC><<<grid, 256, 0, st>>>(X, W, out, M, N, K, 0, -1, 0);
        else if (epi == EPI_SWIGLU) k_gemm_plain<T, EPI_SWIGLU, VEC><<<grid, 256, 0, st>>>(X, W, out, M, N, K, N, -1, 0);
        else k_gemm_plain<T, EPI_LMHEAD, VEC><<<grid, 256, 0, st>>>(X, W, out, M, N, K, 0, mask, (int)tiles);
    };
    // four elements of a row, which starts at a multiple of eight elements, as one load where the matrices are aligned
    if ((((uintptr_t)X | (uintptr_t)W) & 15) == 0) run(std::true_type{});
    else run(std::false_type{});
}

void launch_gemm_plain(const ssd_ctx* c, int epi, const void* X, const void* W, void* out, int M, int N, int K,
                       hipStream_t st) {
    if (c->dm.dtype == SSD_F32)
        gemm_plain_t<float>(c, epi, (const float*)X, (const float*)W, out, M, N, K, st);
    else
        gemm_plain_t<bf16_t>(c, epi, (const bf16_t*)X, (const bf16_t*)W, out, M, N, K, st);
}

int lm_tiles_plain(int V) { return (V + PBN - 1) / PBN; }

void launch_lm_merge(const ssd_ctx* c, int M, int n_tiles, hipStream_t st) {
    launch_lm_merge_to(c, M, n_tiles, c->b.lm_part, c->b.row_max, c->b.row_arg, c->b.row_conf, st);
}

void launch_lm_merge_to(const ssd_ctx* c, int M, int n_tiles, const float* part, float* row_max, int* row_arg,
                        float* row_conf, hipStream_t st) {
    k_lm_merge<<<M, 256, 0, st>>>(part, n_tiles, row_max, row_arg, row_conf, c->dm.V, c->dm.mask_id);
}

void launch_accept(const ssd_ctx* c, int n_groups, hipStream_t st) {
    k_accept<<<n_groups, 64, 0, st>>>(c->b.fwd, c->b.state, c->b.row_conf, c->b.row_arg, c->b.row_max, c->results_to_host ? c->host_result_dev : c->b.result,
                                      c->b.out_tok, c->dm.max_seq_len, c->dm.block, c->dm.max_draft, c->dm.mask_id,
                                      c->b.ref_conf, c->b.ref_arg);
}

// Helpers of the kernel-level entry points.
__global__ void k_sum_partials(const float* __restrict__ part, int n_part, size_t part_stride, float* __restrict__ out,
                               size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int half = (n_part + 1) >> 1;
    float v = part[i], u = 0.f;
    for (int s = 1; s < half; ++s) v += part[s * part_stride + i];
    if (half < n_part) {
        u = part[half * part_stride + i];
        for (int s = half + 1; s < n_part; ++s) u += part[s * part_stride + i];
        v += u;
    }
    out[i] = v;
}

__global__ __launch_bounds__(256) void k_token_rank(const float* __restrict__ logits, int V, int mask_id, RankPairs pairs,
                                                    int* __restrict__ rank) {
    const int i = blockIdx.x;
    const float* row = logits + (size_t)pairs.pos[i] * V;
    const int t = pairs.tok[i];
    const float lt = row[t];
    int ahead = 0;
    for (int v = threadIdx.x; v < V; v += 256)
        ahead += v != mask_id && (row[v] > lt || (row[v] == lt && v < t));
    __shared__ int part[4];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ahead += __shfl_xor(ahead, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ahead;
    __syncthreads();
    if (threadIdx.x == 0) rank[i] = part[0] + part[1] + part[2] + part[3];
}

void launch_token_rank(const float* logits, int V, int mask_id, const RankPairs& pairs, int* rank, hipStream_t st) {
    if (pairs.n > 0) k_token_rank<<<pairs.n, 256, 0, st>>>(logits, V, mask_id, pairs, rank);
}

__global__ void k_int_to_float(const int* __restrict__ src, float* __restrict__ dst, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (float)src[i];
}

void launch_sum_partials(const ssd_ctx* c, int M, int N, int n_part, float* out, hipStream_t st) {
    const size_t n = (size_t)M * N;
    k_sum_partials<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(c->b.part, n_part,
                                                                (size_t)c->dm.max_rows * c->part_cols, out, n);
}

// Kernel-level entry points: caller-supplied keys and values (row-major [n, Hkv, dh], keys after the
// rotary embedding) into a sequence's cache slot at positions [pos0, pos0 + n), fragment order.
template <typename T>
__global__ void k_write_cache(const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ kcache,
                              T* __restrict__ vcache, int Hkv, int dh, int pos0, size_t slot_base, int seq_stride) {
    const int r = blockIdx.x, kvh = blockIdx.y;
    const size_t hb = slot_base + (size_t)kvh * seq_stride * dh;
    for (int ch = threadIdx.x; ch < dh; ch += blockDim.x) {
        const size_t src = ((size_t)r * Hkv + kvh) * dh + ch;
        kcache[hb + kfrag_off(pos0 + r, ch, dh)] = k[src];
        vcache[hb + vfrag_off(pos0 + r, ch, dh)] = v[src];
    }
}

void launch_write_cache(const ssd_ctx* c, int seq, int layer, int pos0, int n, const void* k, const void* v, hipStream_t st) {
    const Dims& d = c->dm;
    const size_t slot = (((size_t)layer * d.max_seqs + seq) * d.Hkv) * (size_t)d.seq_stride() * d.dh;
    dim3 grid(n, d.Hkv);
    if (d.dtype == SSD_F32)
        k_write_cache<float><<<grid, 128, 0, st>>>((const float*)k, (const float*)v, (float*)c->b.kcache, (float*)c->b.vcache,
                                                   d.Hkv, d.dh, pos0, slot, d.seq_stride());
    else
        k_write_cache<bf16_t><<<grid, 128, 0, st>>>((const bf16_t*)k, (const bf16_t*)v, (bf16_t*)c->b.kcache,
                                                    (bf16_t*)c->b.vcache, d.Hkv, d.dh, pos0, slot, d.seq_stride());
}

// The nodes' own keys and values of a forward, from fragment order back to row-major [M, Hkv, dh].
template <typename T>
__global__ void k_read_own_kv(const NodeDesc* __restrict__ row_desc,
                              const T* __restrict__ kown, const T* __restrict__ vown, T* __restrict__ k,
                              T* __restrict__ v, int Hkv, int dh, int vt_rows) {
    const int row = blockIdx.x, kvh = blockIdx.y;
    const NodeDesc nd = row_desc[row];
    const int prow = nd.vrow0 + (row - nd.row0);
    const size_t hb = (size_t)kvh * vt_rows * dh;
    for (int ch = threadIdx.x; ch < dh; ch += blockDim.x) {
        const size_t dst = ((size_t)row * Hkv + kvh) * dh + ch;
        k[dst] = kown[hb + kfrag_off(prow, ch, dh)];
        v[dst] = vown[hb + vfrag_off(prow, ch, dh)];
    }
}

void launch_read_own_kv(const ssd_ctx* c, int M, void* k, void* v, hipStream_t st) {
    const Dims& d = c->dm;
    dim3 grid(M, d.Hkv);
    if (d.dtype == SSD_F32)
        k_read_own_kv<float><<<grid, 128, 0, st>>>(c->b.row_desc, (const float*)c->b.kown, (const float*)c->b.vown,
                                                   (float*)k, (float*)v, d.Hkv, d.dh, d.vt_rows());
    else
        k_read_own_kv<bf16_t><<<grid, 128, 0, st>>>(c->b.row_desc, (const bf16_t*)c->b.kown,
                                                    (const bf16_t*)c->b.vown, (bf16_t*)k, (bf16_t*)v, d.Hkv, d.dh, d.vt_rows());
}

void launch_int_to_float(const int* src, float* dst, int n, hipStream_t st) {
    k_int_to_float<<<(n + 255) / 256, 256, 0, st>>>(src, dst, n);
}
