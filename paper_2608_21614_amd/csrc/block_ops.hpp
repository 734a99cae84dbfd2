// block_ops.hpp -- building blocks of the routing front end: order-preserving score
// keys, wave-wide maxima, and the chunked counting sort that repacks the (token,
// expert) pairs.
#pragma once

#include <limits.h>
#include <math.h>

#include "common.hpp"

namespace saem {

constexpr int kFrontThreads = 1024;            // 16 waves

// Integer key with the order of the float scores: equal keys iff equal scores
// (-0 is folded into +0), larger key iff larger score.
__device__ __forceinline__ int score_key(float f) {
    int b = __float_as_int(f);
    if (b == (int)0x80000000) b = 0;
    return b >= 0 ? b : (b ^ 0x7fffffff);
}

// Maximum over the wave: DPP within each row of 16 lanes (each step folds into
// one v_max_i32 with a DPP operand), then the four row maxima on the scalar unit.
__device__ __forceinline__ int wave_max_i32(int v) {
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));   // quad_perm 1,0,3,2
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));   // quad_perm 2,3,0,1
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xF, 0xF, true));  // row_ror 4
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true));  // row_ror 8
    const int r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const int r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    return max(max(r0, r1), max(r2, r3));
}

// LDS ints the repack needs with NT threads.
template <int NT>
constexpr int repack_lds_ints() {
    return 4 * 256 + (NT / 64) * 256 + 4;
}

// Expert-aligned repacking of the T*k pairs in chunks of NT pairs (chunk c =
// pairs [c NT, (c + 1) NT)); a workgroup of NT threads scatters the chunks
// [c_begin, c_end) in order:
//   1. it counts all pairs per expert, and separately the pairs before c_begin,
//      with LDS atomics (order-free; the ids are a few tens of KB and stay in L2);
//   2. one wave scans the counts in group order -- resident experts by id, then
//      offloaded experts by id -- into segment starts and n_res; the first
//      chunk's pairs of expert e start after the earlier chunks' pairs of e;
//   3. one pair per thread per chunk: inside a wave the lanes holding the same
//      expert are found with 8 ballots over the bits of the expert id, a lane's
//      rank is the popcount of the matching lanes below it, and each wave adds
//      the counts of the waves before it (LDS); after the chunk every expert's
//      start moves past the chunk's pairs.  Pairs keep their index order inside
//      an expert: a stable counting sort with no global atomics, and the same
//      result for any split of the chunks over workgroups.
// The workgroup with c_begin == 0 also writes counts, seg_start and n_res.
// ids outside [0, E) are dropped (inv_perm = -1); the packed rows they leave
// over at the end, [sum(counts), T*k), get perm = -1.
// kLocal: nothing is written to memory; the workgroup takes all chunks and leaves the
// permutation in s_perm (T*k ints of LDS), for its own use.  Returns n_res.
template <int NT, bool kLocal = false>
__device__ inline int repack_chunks(int T, int E, int k, int slots, int c_begin, int c_end,
                                     const int32_t* __restrict__ idx, const int32_t* __restrict__ expert_slot,
                                     int32_t* __restrict__ counts, int32_t* __restrict__ seg_start,
                                     int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                                     int32_t* __restrict__ n_res, int* lds, int* s_perm = nullptr) {
    int* s_cnt = lds;
    int* s_pre = lds + 256;
    int* s_base = lds + 512;
    int* s_res = lds + 768;
    constexpr int NW = NT / 64;
    int* s_wcnt = lds + 1024;               // [NW][256]
    int* s_nres = lds + 1024 + NW * 256;
    const int tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
    const int P = T * k;
    const int c0 = c_begin * NT;

    for (int e = tid; e < 256; e += NT) {
        s_cnt[e] = 0;
        s_pre[e] = 0;
        s_res[e] = (e < E) ? (is_resident(expert_slot[e], slots) ? 1 : 0) : 0;
    }
    __syncthreads();
    for (int q = tid; q < P; q += NT) {
        const int e = idx[q];
        if (e >= 0 && e < E) {
            atomicAdd(&s_cnt[e], 1);
            if (q < c0) atomicAdd(&s_pre[e], 1);
        }
    }
    __syncthreads();
    if (wave == 0) {
        int rs = 0, os = 0;  // lane owns experts 4 lane .. 4 lane + 3
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 4 * lane + i;
            if (e < E) {
                if (s_res[e]) rs += s_cnt[e];
                else os += s_cnt[e];
            }
        }
        int rinc = rs, oinc = os;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int a = __shfl_up(rinc, off, 64);
            const int b = __shfl_up(oinc, off, 64);
            if (lane >= off) {
                rinc += a;
                oinc += b;
            }
        }
        const int rtot = __shfl(rinc, 63, 64);
        const int otot = __shfl(oinc, 63, 64);
        int rp = rinc - rs, op = rtot + (oinc - os);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = 4 * lane + i;
            if (e < E) {
                if (s_res[e]) {
                    s_base[e] = rp;
                    rp += s_cnt[e];
                } else {
                    s_base[e] = op;
                    op += s_cnt[e];
                }
            }
        }
        if (lane == 0) {
            s_nres[0] = rtot;
            s_nres[1] = rtot + otot;  // valid pairs: the packed rows that get a pair
        }
    }
    __syncthreads();
    const int total_res = s_nres[0];
    if (kLocal) {
        for (int p = s_nres[1] + tid; p < P; p += NT) s_perm[p] = -1;
    } else if (c_begin == 0) {
        for (int e = tid; e < E; e += NT) {
            counts[e] = s_cnt[e];
            seg_start[e] = s_base[e];
        }
        if (tid == 0) *n_res = s_nres[0];
        // rows past the valid pairs (there are some only when ids outside [0, E) were
        // dropped) get no pair: mark them, so no reader takes a stale entry for one
        for (int p = s_nres[1] + tid; p < P; p += NT) perm[p] = -1;
    }
    for (int e = tid; e < E; e += NT) s_base[e] += s_pre[e];

    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    for (int c = c_begin; c < c_end; ++c) {
        for (int i = tid; i < NW * 256; i += NT) s_wcnt[i] = 0;
        __syncthreads();
        const int q = c * NT + tid;
        const int e = (q < P) ? idx[q] : -1;
        const bool valid = (e >= 0 && e < E);
        unsigned long long m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = valid && ((e >> b) & 1);
            const unsigned long long bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const int rank = __popcll(m & lt_mask);
        if (valid && rank == 0) s_wcnt[wave * 256 + e] = __popcll(m);
        __syncthreads();
        if (valid) {
            int p = s_base[e] + rank;
            for (int w = 0; w < wave; ++w) p += s_wcnt[w * 256 + e];
            if (kLocal) {
                s_perm[p] = q;
            } else {
                perm[p] = q;
                inv_perm[q] = p;
            }
        } else if (q < P && !kLocal) {
            inv_perm[q] = -1;
        }
        __syncthreads();
        for (int ee = tid; ee < E; ee += NT) {
            int sum = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += s_wcnt[w * 256 + ee];
            s_base[ee] += sum;
        }
        __syncthreads();
    }
    return total_res;
}

}  // namespace saem
