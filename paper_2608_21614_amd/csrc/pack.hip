// pack.hip -- expert weights into the MFMA tile layout.
//
// A K-contiguous matrix W[R][K] (R % 16 == 0, K % 32 == 0) is stored as blocks
// of 16 rows x 32 columns; block (rt, s) covers rows 16*rt .. 16*rt+15 and
// columns 32*s .. 32*s+31 and sits at element offset (rt * K/32 + s) * 512.
// Inside a block, element 8*l + i holds W[16*rt + l%16][32*s + 8*(l/16) + i]:
// lane l of a wave reads its MFMA A operand (row l%16, 8 consecutive K values)
// as one 16-byte load, and a wave reads a whole block as 1 KB of contiguous
// memory.  Expert weights are packed once, when they are loaded into a slot
// (the fixed per-layer expert slots of SAEM Section IV-C.1); every forward then
// streams them with fully contiguous wave loads.
#include "common.hpp"
#include "kernels.hpp"

namespace saem {
namespace {

// A wave moves two neighbouring 16 x 32 blocks (elt = 2 or 4 bytes), so that it reads whole
// 128-byte lines of the rows; lane l stores pieces l, l + 64, ... of 16 bytes of a block, so that
// every store instruction of the wave writes 1 KB in one run, and past the caches, since nothing
// reads the lines soon.  HBM bounds it: one expert of H 4096, F 14336 (as much written as read),
//   bf16, 2 x 352 MB: half lines read and plain stores 127.5 us, non-temporal stores 122.3,
//     with whole lines 120; non-temporal loads as well 131;
//   fp32, 2 x 705 MB: 8 elements a lane with plain stores 255, non-temporal ones (half a line
//     each) 520, one run per store 231.
template <typename T>
__global__ void __launch_bounds__(256)
    k_pack(const T* __restrict__ src, T* __restrict__ dst, long long rows, long long K) {
    constexpr int kV = (int)sizeof(T) / 2;  // 16-byte pieces of 8 elements
    const long long nsteps = K / 32, pairs = (nsteps + 1) / 2;
    const long long work = rows / 16 * pairs * 64;
    for (long long c = (long long)blockIdx.x * 256 + threadIdx.x; c < work; c += (long long)gridDim.x * 256) {
        const long long p = c / 64, l = c % 64;
        const long long rt = p / pairs, s = 2 * (p % pairs);
        const bool two = s + 1 < nsteps;
        u32x4 v[2][kV];
        u32x4* out = reinterpret_cast<u32x4*>(dst + (rt * nsteps + s) * 512) + l;
#pragma unroll
        for (int i = 0; i < kV; ++i) {
            // piece j of a block: part j % kV of the 8 elements that an MFMA reads with lane j / kV
            const int j = (int)l + 64 * i, r = j / kV;
            const u32x4* in =
                reinterpret_cast<const u32x4*>(src + (16 * rt + (r & 15)) * K + 32 * s + 8 * (r >> 4)) + j % kV;
            v[0][i] = in[0];
            if (two) v[1][i] = in[4 * kV];
        }
#pragma unroll
        for (int i = 0; i < kV; ++i) {
            __builtin_nontemporal_store(v[0][i], out + 64 * i);
            if (two) __builtin_nontemporal_store(v[1][i], out + 64 * kV + 64 * i);
        }
    }
}

}  // namespace

hipError_t launch_pack_weights(const void* src, void* dst, long long rows, long long K, bool bf16, hipStream_t st) {
    const long long work = rows / 16 * ((K / 32 + 1) / 2) * 64;
    if (work == 0) return hipSuccess;
    long long grid = (work + 255) / 256;
    if (grid > 65536) grid = 65536;
    if (bf16)
        hipLaunchKernelGGL(k_pack<uint16_t>, dim3((unsigned)grid), dim3(256), 0, st, static_cast<const uint16_t*>(src),
                           static_cast<uint16_t*>(dst), rows, K);
    else
        hipLaunchKernelGGL(k_pack<float>, dim3((unsigned)grid), dim3(256), 0, st, static_cast<const float*>(src),
                           static_cast<float*>(dst), rows, K);
    return hipGetLastError();
}

}  // namespace saem
