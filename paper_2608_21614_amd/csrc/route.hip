// route.hip -- router scores and top-k gate (SAEM Section II-A: top-k gating by
// a router), and the decode front end (scores + top-k + repacking).
//
// Scores run on MFMA (v_mfma_f32_16x16x32_bf16, or v_mfma_f32_16x16x4_f32 for
// fp32 inputs): router rows are the M side, 16 tokens the N side.
//
//  * T > 64 (prefill): k_router_scores, one workgroup per 8, 16 or 32 tokens x 16, 32 or 64
//    experts whose 16 waves split K and add their partial tiles in a fixed order, writes the
//    scores.  With all of a token's scores in one workgroup (up to 64 experts) it also picks the
//    top-k; else, and from the caller's scores, k_route_finish does, one wave per token.
//  * T <= 64 (decode): k_router_partial spreads the scores over one workgroup
//    per K slice (a single CU cannot stream the batch and the router fast
//    enough), then k_route_finish adds each token's slices in order and runs its
//    top-k.  The fused forward and moe_route_topk use the same two kernels, so both
//    give bit-identical scores.
#include "block_ops.hpp"
#include "kernels.hpp"

namespace saem {
namespace {

// Top-k gate of token t by one wave, lane l holding the scores of experts l, l + 64, ...
// (open: those that exist).  k rounds of a wave maximum over integer keys with the scores'
// order, and a ballot per slot for the lowest id that has it.  The gate of choice j is
// exp(s_j - s_0) / sum_j' exp(s_j' - s_0), summed in j order; a score equal to the top one
// contributes exactly 1 (so all-equal rows, -inf included, get 1/k).  (NaN scores:
// undefined selection, never an index outside [-1, E).)
template <int NS>
__device__ __forceinline__ void topk_wave(const float (&v)[NS], bool (&open)[NS], int k, int t,
                                          int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    const int lane = lane_id();
    int key[NS];
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) key[sl] = score_key(v[sl]);
    float selv[8];
    int sele[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        selv[j] = 0.f;
        sele[j] = -1;
        if (j >= k) continue;  // uniform
        int kb = INT_MIN;
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) kb = open[sl] ? max(kb, key[sl]) : kb;
        const int m = wave_max_i32(kb);
        // lowest id with that key: slot sl holds ids 64 sl .. 64 sl + 63, one per lane
        int es = 0, el = 0;
        bool found = false;  // always found in the end: k <= E
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) {
            const unsigned long long b = __ballot(open[sl] && key[sl] == m);
            if (!found && b) {
                found = true;
                es = sl;
                el = __ffsll((long long)b) - 1;
            }
        }
#pragma unroll
        for (int sl = 0; sl < NS; ++sl)
            if (es == sl && lane == el) open[sl] = false;
        float ve = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[0]), el));
#pragma unroll
        for (int sl = 1; sl < NS; ++sl)
            if (es == sl) ve = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[sl]), el));
        selv[j] = ve;
        sele[j] = kWave * es + el;
    }
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < k) sum += (selv[j] == selv[0]) ? 1.0f : expf(selv[j] - selv[0]);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < k && lane == j) {
            const float term = (selv[j] == selv[0]) ? 1.0f : expf(selv[j] - selv[0]);
            topk_idx[(size_t)t * k + j] = sele[j];
            topk_w[(size_t)t * k + j] = term / sum;
        }
}

// Prefill scores of 16 tokens x 16 M experts by a workgroup of 16 waves; wave w takes the
// 32-wide K steps w, w + 16, ...  Router rows are the MFMA M side, the tokens the N side;
// the waves' partial tiles meet in LDS and are added in wave order, so the fp32 scores do
// not depend on timing.
//
// Latency bounds it: a CU keeps about 64 KB of loads in flight, and a workgroup asks for
// (tokens + experts) x H, so the tile is chosen by that (launch_prefill).  One kernel of 8
// tokens a workgroup, each streaming the whole router, took 25 us at 150 tokens x 128
// experts x H 2048 (19 workgroups), 14 to 16 at 2048 x 64, 53 at 8192 x 64 and 122 at 5305 x
// 223 x H 2176; this one (with the top-k) takes 5.7 + 4.6, 14 to 16, 22 and 38 + 11.
constexpr int kScoreWaves = 16;

template <typename Elt, int M, int TT, bool kTopk>
__global__ void __launch_bounds__(kScoreWaves* kWave)
    k_router_scores(int T, int H, int E, int rows, const Elt* __restrict__ x, const Elt* __restrict__ wr,
                    const float* __restrict__ bias, float* __restrict__ logits, int k, int32_t* __restrict__ topk_idx,
                    float* __restrict__ topk_w) {
    constexpr int U = (sizeof(Elt) == 2 ? 4 : 2) / TT;  // K steps per load batch
    constexpr int kPitch = 16 * M + 4;  // floats of a partial row: the 16 row lanes' 16-byte writes spread over the banks
    __shared__ __attribute__((aligned(16))) float red[kScoreWaves * 16 * TT * kPitch];
    __shared__ float s_lg[kTopk ? 16 * TT : 1][kTopk ? 16 * M + 1 : 1];
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int r = lane & 15, kq = (lane >> 4) * 8;
    const int t0 = blockIdx.x * rows, e0 = blockIdx.y * 16 * M;
    T = min(T, t0 + rows);  // rows <= 16 TT: the MFMA tile's rows past it stay zero
    const Elt* xp[TT];
    const Elt* wp[M];
    f32x4 acc[TT][M];
#pragma unroll
    for (int j = 0; j < TT; ++j) xp[j] = (t0 + 16 * j + r < T) ? x + (size_t)(t0 + 16 * j + r) * H + kq : nullptr;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int e = e0 + 16 * m + r;
        wp[m] = (e < E) ? wr + (size_t)e * H + kq : nullptr;
#pragma unroll
        for (int j = 0; j < TT; ++j) acc[j][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int nsteps = H / 32;
    for (int i = wave; i < nsteps; i += U * kScoreWaves) {
        Frag8<Elt> A[U][M], B[U][TT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = i + kScoreWaves * u;
            const bool ok = s < nsteps;
#pragma unroll
            for (int j = 0; j < TT; ++j) B[u][j] = (ok && xp[j]) ? load_frag(xp[j] + s * 32) : zero_frag<Elt>();
#pragma unroll
            for (int m = 0; m < M; ++m) A[u][m] = (ok && wp[m]) ? load_frag(wp[m] + s * 32) : zero_frag<Elt>();
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < TT; ++j)
#pragma unroll
                for (int m = 0; m < M; ++m) acc[j][m] = mma_frag(A[u][m], B[u][j], acc[j][m]);
    }
    // lane holds experts 16 m + 4 (lane / 16) + 0..3 of token row 16 j + r
#pragma unroll
    for (int j = 0; j < TT; ++j)
#pragma unroll
        for (int m = 0; m < M; ++m)
            *reinterpret_cast<f32x4*>(red + ((wave * TT + j) * 16 + r) * kPitch + 16 * m + 4 * (lane >> 4)) = acc[j][m];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 16 * TT * 16 * M; idx += kScoreWaves * kWave) {
        const int row = idx / (16 * M), el = idx % (16 * M);
        const int t = t0 + row, e = e0 + el;
        if (t >= T || e >= E) continue;
        float v = red[row * kPitch + el];
#pragma unroll
        for (int p = 1; p < kScoreWaves; ++p) v += red[(p * 16 * TT + row) * kPitch + el];
        v += bias ? bias[e] : 0.f;
        logits[(size_t)t * E + e] = v;
        if constexpr (kTopk) s_lg[row][el] = v;
    }
    if constexpr (kTopk) {
        __syncthreads();
        for (int row = wave; row < 16 * TT && t0 + row < T; row += kScoreWaves) {
            bool open[1] = {lane < E};
            const float v[1] = {lane < E ? s_lg[row][lane] : 0.f};
            topk_wave<1>(v, open, k, t0 + row, topk_idx, topk_w);
        }
    }
}

// Decode batches: part[slice][t][e] = sum over the slice's K steps of x[t] . w_router[e].
// One workgroup per (K slice, chunk of 16 kPartM experts); wave w covers tokens
// 16w .. 16w+15; MFMA on bf16 (16x16x32) or fp32 (16x16x4) operands.  Latency bounds it, and a
// CU keeps about 64 KB of loads in flight, which a workgroup with 64 experts exceeds: chunks of
// 64 / 32 / 16 experts take 7.2 / 4.8 / 4.7 us for 64 tokens x 128 experts x H 2048, 6.4 / 4.7 /
// 4.7 for 64 x 60, 4.8 / 3.4 / 2.8 for one token x 128.
constexpr int kPartM = 1;

template <typename Elt>
__global__ void __launch_bounds__(256)
    k_router_partial(int T, int H, int E, const void* __restrict__ x, const void* __restrict__ wr, int nsl,
                     float* __restrict__ part) {
    constexpr int M = kPartM;
    const int slice = blockIdx.x;
    const int nst = H / 32, s0 = slice * nst / nsl, s1 = (slice + 1) * nst / nsl;
    float* out = part + (size_t)slice * 64 * E;
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int r = lane & 15, kq = (lane >> 4) * 8;
    if (16 * wave >= T) return;
    const int tok = 16 * wave + r;
    const Elt* xp = (tok < T) ? static_cast<const Elt*>(x) + (size_t)tok * H + kq : nullptr;
    const int c0 = blockIdx.y * 16 * M;
    f32x4 acc[M];
    const Elt* wp[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int e = c0 + 16 * m + r;
        wp[m] = (e < E) ? static_cast<const Elt*>(wr) + (size_t)e * H + kq : nullptr;
    }
    for (int s = s0; s < s1; s += 4) {
        Frag8<Elt> A[4][M], B[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool ok = s + u < s1;
            B[u] = (ok && xp) ? load_frag(xp + (s + u) * 32) : zero_frag<Elt>();
#pragma unroll
            for (int m = 0; m < M; ++m) A[u][m] = (ok && wp[m]) ? load_frag(wp[m] + (s + u) * 32) : zero_frag<Elt>();
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (c0 + 16 * m < E) acc[m] = mma_frag(A[u][m], B[u], acc[m]);
    }
    if (tok < T) {
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = c0 + 16 * m + 4 * (lane >> 4) + i;
                if (e < E) out[tok * E + e] = acc[m][i];
            }
    }
}

// Top-k gate, one wave per token.  At decode the wave first adds the token's K-sliced
// partial scores in slice order (+ bias) and writes them to logits; at prefill, and with
// the caller's scores, it reads logits.
// NS: expert slots per lane (E <= 64 NS).  kLogitsIn: the scores are in logits (without the
// slices' registers a CU holds two to four times the waves).
template <int NS, bool kLogitsIn>
__global__ void __launch_bounds__(256)
    k_route_finish(int T, int E, int k, const float* __restrict__ part, int nsl, const float* __restrict__ bias,
                   float* __restrict__ logits, int32_t* __restrict__ topk_idx, float* __restrict__ topk_w) {
    const int lane = lane_id();
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t >= T) return;  // the whole wave
    float v[NS];
    bool open[NS];
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
        open[sl] = lane + kWave * sl < E;
        v[sl] = 0.f;
    }
    if constexpr (kLogitsIn) {
#pragma unroll
        for (int sl = 0; sl < NS; ++sl)
            if (open[sl]) v[sl] = logits[(size_t)t * E + lane + kWave * sl];
    } else {
        // all slots' loads of a batch of 16 slices in flight together, bias included
        float bv[NS];
#pragma unroll
        for (int sl = 0; sl < NS; ++sl) bv[sl] = (open[sl] && bias) ? bias[lane + kWave * sl] : 0.f;
        for (int b = 0; b < nsl; b += 16) {
            float q[NS][16];
#pragma unroll
            for (int sl = 0; sl < NS; ++sl) {
                const float* p = part + (size_t)t * E + (open[sl] ? lane + kWave * sl : 0);
#pragma unroll
                for (int j = 0; j < 16; ++j) q[sl][j] = (b + j < nsl) ? p[(size_t)(b + j) * 64 * E] : 0.f;
            }
#pragma unroll
            for (int sl = 0; sl < NS; ++sl)
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (b + j < nsl) v[sl] = (b + j == 0) ? q[sl][j] : v[sl] + q[sl][j];
        }
#pragma unroll
        for (int sl = 0; sl < NS; ++sl)
            if (open[sl]) {
                v[sl] += bv[sl];
                logits[(size_t)t * E + lane + kWave * sl] = v[sl];
            }
    }
    topk_wave<NS>(v, open, k, t, topk_idx, topk_w);
}

void launch_finish(const Shape& s, const float* part, int nsl, const float* bias, float* logits, bool logits_in,
                   int32_t* topk_idx, float* topk_w, hipStream_t st) {
    const dim3 grid((s.T + 3) / 4);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, s.T, s.E, s.k, part, nsl, bias, logits, topk_idx, topk_w);
    };
    if (s.E <= 64) logits_in ? go(k_route_finish<1, true>) : go(k_route_finish<1, false>);
    else if (s.E <= 128) logits_in ? go(k_route_finish<2, true>) : go(k_route_finish<2, false>);
    else logits_in ? go(k_route_finish<4, true>) : go(k_route_finish<4, false>);
}

// Prefill routing.  A CU draws about 64 KB per microsecond of such loads, so what counts is
// the bytes of the fullest CU: (tokens + experts of a workgroup) x H, times its workgroups.
//  * Up to 64 experts a workgroup can have all scores of its tokens and pick their top-k itself,
//    for 8 tokens (half an MFMA tile) while every CU gets at most one workgroup, then 16, then 32.
//    In us at H 2048, 8 / 16 / 32 tokens a workgroup:
//      64 experts, bf16: 2047 tokens 13.0 / 14.7 / 19.7;   2049: 22.1 / 14.6 / 19.6;   4095:
//      24.2 / 15.3 / 20.2;   4097: 32.8 / 24.4 / 20.4;   8191: 46.5 / 28.4 / 21.0;   12000: 68 / 41 / 38
//    Up to 16 experts take little enough LDS for several workgroups on a CU, so 16 tokens stay ahead:
//      8 experts, bf16: 2047 tokens 6.2 / 7.5 / 10.7;   8193: 14.8 / 11.3 / 13.1;   16384: 24 / 18 / 22
//  * The smaller loads of tiles over fewer experts pay for a second launch (the top-k) where a
//    workgroup's rows are many bytes.  All experts at once / tiles and top-k, in us:
//      at most one 8-token workgroup per CU: bf16 168 KB 9.5 / 9.0, 200 KB (17 experts, H 4096)
//        10.6 / 12.5, 216 KB (64, H 1536) 10.6 / 8.3; fp32 100 KB (17, H 1024) 9.4 / 10.2, 150 KB
//        (17, H 1536) 12.0 / 11.1, 246 KB (33, H 1536) 18.2 / 11.5, 576 KB (64, H 2048) 23 / 13
//      one 16-token workgroup: bf16 320 KB 15 / 17, fp32 400 KB 24 / 21 to 26, 640 KB 28 / 28,
//        784 KB (33, H 4096) 42 / 35
//  * More than 64 experts: the largest tile that still gives every CU a workgroup, then the
//    top-k in a launch of its own.
template <typename Elt>
hipError_t launch_prefill(const Shape& s, const void* x, const void* w_router, const float* bias, float* logits,
                          int32_t* topk_idx, float* topk_w, hipStream_t st) {
    int cus = 0;
    if (hipError_t e = device_cus(&cus); e != hipSuccess) return e;
    auto tiles = [&](int n, int tile) { return (n + tile - 1) / tile; };
    auto go = [&](auto kernel, int rows, int m) {
        hipLaunchKernelGGL(kernel, dim3(tiles(s.T, rows), tiles(s.E, 16 * m)), dim3(kScoreWaves * kWave), 0, st, s.T,
                           s.H, s.E, rows, static_cast<const Elt*>(x), static_cast<const Elt*>(w_router), bias, logits,
                           s.k, topk_idx, topk_w);
    };
    const int rows = s.T <= 8 * cus ? 8 : (s.T <= 16 * cus || s.E <= 16 ? 16 : 32);
    const size_t bytes = (size_t)(s.E + rows) * s.H * sizeof(Elt);  // a workgroup's, with all experts
    const size_t limit = rows == 8 ? (sizeof(Elt) == 2 ? 200 : 144) << 10 : (rows == 16 ? 640 << 10 : SIZE_MAX);
    if (s.E <= 16 || (s.E <= 64 && bytes <= limit)) {
        if (rows == 32) {
            if (s.E <= 32) go(k_router_scores<Elt, 2, 2, true>, rows, 2);
            else go(k_router_scores<Elt, 4, 2, true>, rows, 4);
        } else {
            if (s.E <= 16) go(k_router_scores<Elt, 1, 1, true>, rows, 1);
            else if (s.E <= 32) go(k_router_scores<Elt, 2, 1, true>, rows, 2);
            else go(k_router_scores<Elt, 4, 1, true>, rows, 4);
        }
        return hipGetLastError();
    }
    if (tiles(s.T, 32) * tiles(s.E, 64) >= cus) go(k_router_scores<Elt, 4, 2, false>, 32, 4);
    else if (tiles(s.T, 16) * tiles(s.E, 64) >= cus) go(k_router_scores<Elt, 4, 1, false>, 16, 4);
    else if (tiles(s.T, 16) * tiles(s.E, 32) >= cus) go(k_router_scores<Elt, 2, 1, false>, 16, 2);
    else go(k_router_scores<Elt, 1, 1, false>, 16, 1);
    launch_finish(s, nullptr, 0, nullptr, logits, true, topk_idx, topk_w, st);
    return hipGetLastError();
}

}  // namespace

bool front_small_fits(const Shape& s) { return s.T <= 64; }

int router_slices(const Shape& s) {
    if (!front_small_fits(s)) return 0;
    const int n = (s.H / 32) / 4;  // about 4 K steps of 32 per workgroup
    return n < 1 ? 1 : (n > 64 ? 64 : n);
}

hipError_t launch_route_topk(const Shape& s, const void* x, const void* w_router, const float* bias, float* logits,
                             bool logits_in, int32_t* topk_idx, float* topk_w, float* part, hipStream_t st) {
    if (s.T == 0) return hipSuccess;
    if (!front_small_fits(s)) {
        if (!logits_in)
            return s.bf16 ? launch_prefill<uint16_t>(s, x, w_router, bias, logits, topk_idx, topk_w, st)
                          : launch_prefill<float>(s, x, w_router, bias, logits, topk_idx, topk_w, st);
        launch_finish(s, nullptr, 0, nullptr, logits, true, topk_idx, topk_w, st);
        return hipGetLastError();
    }
    const int nsl = router_slices(s);
    if (!logits_in) {
        const dim3 grid(nsl, (s.E + 16 * kPartM - 1) / (16 * kPartM));
        if (s.bf16)
            hipLaunchKernelGGL((k_router_partial<uint16_t>), grid, dim3(256), 0, st, s.T, s.H, s.E, x, w_router, nsl,
                               part);
        else
            hipLaunchKernelGGL((k_router_partial<float>), grid, dim3(256), 0, st, s.T, s.H, s.E, x, w_router, nsl,
                               part);
    }
    launch_finish(s, part, nsl, bias, logits, logits_in, topk_idx, topk_w, st);
    return hipGetLastError();
}

}  // namespace saem
