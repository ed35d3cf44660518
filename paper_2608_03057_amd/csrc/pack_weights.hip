// Relayout of the stored 8-bit weight buffer into the MFMA operand order
// read by the packed-weight kernels (one-time, like the bit planes).
//
// Unit (nb, ks) of 1 KB holds, for lane l = 0..63 at bytes 16*l .. 16*l+15,
// W[32*nb + l%32][32*ks + 16*(l/32) .. +15]; units are ordered nb-major,
// KS = 4 * ceil(K / 128) units per 32-row block, and every byte past row N
// or column K is zero.  The codes are copied unchanged: masking to b bits
// happens in the kernels, so this one buffer serves every precision.
#include "rows.h"
#include "tasq_internal.h"

namespace tasq {

// One wave per (32-row block, 128-byte K block): four chunk loads per lane in
// flight, then four 1 KB units written whole.  A copy in other order, bound
// by memory; byte loads (sixteen per chunk) held it at 0.9 TB/s of reads and
// writes.
// 4608x1152 14.0 -> 5.1 us; 10240x3456 took 76 us, 10240x6720 now takes 28.7
// (4.8 TB/s).
__global__ void __launch_bounds__(256) k_pack_weights(const int8_t *__restrict__ W, int N, int K,
                                                      int KB, int blocks,
                                                      int8_t *__restrict__ packed)
{
    const int blk = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blk >= blocks)
        return;
    const int nb = blk / KB, kb = blk - nb * KB;
    const int lane = threadIdx.x & 63, row = lane & 31;
    Window w;
    w.init(W, N, 32 * nb, 32, K);
    const bool ok = 32 * nb + row < N;
    const int k0 = 128 * kb + 16 * (lane >> 5);
    const uint32_t off = w.lead + (uint32_t)row * (uint32_t)K + (uint32_t)k0;
    Chunk5 c[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        c[u].load(w.r, ok && k0 + 32 * u < K ? off + 32u * u : kOOB);
    v4i *out = reinterpret_cast<v4i *>(packed) + (size_t)blk * 256 + lane;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        out[64 * u] = keep_bytes(c[u].bytes(off), K - k0 - 32 * u);
}

hipError_t launch_pack_weights(const int8_t *W, int N, int K, int8_t *packed,
                               hipStream_t stream)
{
    return launch_pack_units(N, K, [&](long long nb, int rows, int KB, int units) {
        hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)(units + 3) / 4), dim3(256), 0, stream,
                           W + (size_t)nb * 32 * (size_t)K, rows, K, KB, units,
                           packed + (size_t)nb * (size_t)KB * 4096);
        return hipGetLastError();
    });
}

}  // namespace tasq
