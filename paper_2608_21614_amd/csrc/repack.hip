// repack.hip -- expert-aligned token repacking with the residency split
// (SAEM Section IV-E.1; partition by residency map, Section IV-D.2).
//
// A stable counting sort over the T*k pairs (repack_chunks in block_ops.hpp).
// Up to 512 pairs (a decode batch): one workgroup of 256 threads; when the offloaded
// rows are packed too, further workgroups sort for themselves (the result stays in LDS)
// and pack them in the same launch.  Otherwise
// chunks of 1024 pairs, split into contiguous ranges over up to kRepackGroups
// workgroups of 1024 threads; every workgroup counts the whole batch itself, so
// none waits for another, and the result does not depend on the split.  A
// second small kernel then packs the offloaded rows (moe_repack on its own; the fused
// forward packs them elsewhere).
#include "block_ops.hpp"
#include "kernels.hpp"

namespace saem {
namespace {

// Workgroups of one repack: each counts all T*k ids, so more groups cost L2 reads
// (groups x T*k) and fewer cost chunk passes (chunks / groups in sequence).
constexpr int kRepackGroups = 128;

template <int NT>
__global__ void __launch_bounds__(NT)
    k_repack(int T, int E, int k, int slots, int chunks, const int32_t* __restrict__ topk_idx,
             const int32_t* __restrict__ expert_slot, int32_t* __restrict__ counts, int32_t* __restrict__ seg_start,
             int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, int32_t* __restrict__ n_res) {
    __shared__ int s_lds[repack_lds_ints<NT>()];
    const int g = blockIdx.x, G = gridDim.x;
    const int c_begin = (int)((long long)chunks * g / G), c_end = (int)((long long)chunks * (g + 1) / G);
    repack_chunks<NT>(T, E, k, slots, c_begin, c_end, topk_idx, expert_slot, counts, seg_start, perm, inv_perm, n_res,
                      s_lds);
}

// off_rows[p - n_res] = x[q / k] and off_w[p - n_res] = topk_w[q] for packed row p of pair q,
// by one workgroup.
__device__ void pack_row(int q, int P, int k, int row_bytes, const uint8_t* __restrict__ x,
                         const float* __restrict__ topk_w, uint8_t* __restrict__ off_rows, float* __restrict__ off_w,
                         int at) {
    if (q < 0 || q >= P) return;  // rows of dropped pairs are left as they are
    if (off_rows) {
        const u32x4* src = reinterpret_cast<const u32x4*>(x + (size_t)(q / k) * row_bytes);
        u32x4* dst = reinterpret_cast<u32x4*>(off_rows + (size_t)at * row_bytes);
        for (int c = threadIdx.x; c < row_bytes / 16; c += blockDim.x) dst[c] = src[c];
    }
    if (off_w && threadIdx.x == 0) off_w[at] = topk_w[q];
}

// A decode batch repacked and its offloaded rows packed: workgroup 0 writes the repack's
// outputs, workgroup 1 + i packs row n_res + i (several rows a workgroup had made many wide rows
// a chain of copies).  Both are chains of a few memory round trips, so one launch instead of two
// takes no more than the repack alone.  In us, two launches, one with 128 pack workgroups, and now:
//   64 tokens, 256 pairs, H 2048, bf16:    6.4,  5.0,  4.7
//   64 tokens, 512 pairs, H 8192, bf16:    8.8,  9.2,  7.2
//   64 tokens, 512 pairs, H 16384, fp32:  14.9, 25.1, 13.1
__global__ void __launch_bounds__(256)
    k_repack_pack(int T, int E, int k, int slots, int chunks, const int32_t* __restrict__ topk_idx,
                  const int32_t* __restrict__ expert_slot, int32_t* __restrict__ counts,
                  int32_t* __restrict__ seg_start, int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm,
                  int32_t* __restrict__ n_res, int row_bytes, const uint8_t* __restrict__ x,
                  const float* __restrict__ topk_w, uint8_t* __restrict__ off_rows, float* __restrict__ off_w) {
    __shared__ int s_lds[repack_lds_ints<256>()];
    __shared__ int s_perm[512];
    if (blockIdx.x == 0) {
        repack_chunks<256>(T, E, k, slots, 0, chunks, topk_idx, expert_slot, counts, seg_start, perm, inv_perm, n_res,
                           s_lds);
        return;
    }
    const int nres = repack_chunks<256, true>(T, E, k, slots, 0, chunks, topk_idx, expert_slot, nullptr, nullptr,
                                              nullptr, nullptr, nullptr, s_lds, s_perm);
    const int P = T * k, row = (int)blockIdx.x - 1;
    if (nres + row < P) pack_row(s_perm[nres + row], P, k, row_bytes, x, topk_w, off_rows, off_w, row);
}

__global__ void __launch_bounds__(256)
    k_offload_pack(int T, int k, int row_bytes, const uint8_t* __restrict__ x, const float* __restrict__ topk_w,
                   const int32_t* __restrict__ perm, const int32_t* __restrict__ n_res_p,
                   uint8_t* __restrict__ off_rows,
                   float* __restrict__ off_w) {
    const int P = T * k;
    const int nres = *n_res_p;
    for (int p = nres + (int)blockIdx.x; p < P; p += gridDim.x)
        pack_row(perm[p], P, k, row_bytes, x, topk_w, off_rows, off_w, p - nres);
}

}  // namespace

hipError_t launch_repack(const Shape& s, const int32_t* topk_idx, const int32_t* expert_slot, int32_t* counts,
                         int32_t* seg_start, int32_t* perm, int32_t* inv_perm, int32_t* n_res, const void* x,
                         const float* topk_w, void* off_rows, float* off_w, hipStream_t st) {
    const int P = s.T * s.k;
    const bool pack = P > 0 && (off_rows || off_w);
    const int row_bytes = s.H * (s.bf16 ? 2 : 4);
    const uint8_t* xb = static_cast<const uint8_t*>(x);
    uint8_t* ob = static_cast<uint8_t*>(off_rows);
    if (P <= 512) {  // a decode batch: up to two chunks of 256
        const int chunks = (P + 255) / 256;
        if (pack)
            hipLaunchKernelGGL(k_repack_pack, dim3(1 + P), dim3(256), 0, st, s.T, s.E, s.k, s.slots,
                               chunks, topk_idx, expert_slot, counts, seg_start, perm, inv_perm, n_res, row_bytes, xb,
                               topk_w, ob, off_w);
        else
            hipLaunchKernelGGL(k_repack<256>, dim3(1), dim3(256), 0, st, s.T, s.E, s.k, s.slots, chunks, topk_idx,
                               expert_slot, counts, seg_start, perm, inv_perm, n_res);
        return hipGetLastError();
    }
    const int chunks = (P + kFrontThreads - 1) / kFrontThreads;
    const int groups = chunks < kRepackGroups ? chunks : kRepackGroups;
    hipLaunchKernelGGL(k_repack<kFrontThreads>, dim3((unsigned)groups), dim3(kFrontThreads), 0, st, s.T, s.E, s.k,
                       s.slots, chunks, topk_idx, expert_slot, counts, seg_start, perm, inv_perm, n_res);
    if (pack)
        hipLaunchKernelGGL(k_offload_pack, dim3(P < 1024 ? P : 1024), dim3(256), 0, st, s.T, s.k, row_bytes, xb, topk_w,
                           perm, n_res, ob, off_w);
    return hipGetLastError();
}

}  // namespace saem
