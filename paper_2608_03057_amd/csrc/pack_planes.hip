// Bit-plane relayout of the stored weight buffer (one-time).
//
// Plane q holds bit p = 7 - q of each code (App. G.2: plane p is bit p of the
// two's-complement code; most significant plane first).  The words of one
// 32-channel block nb are stored together, plane after plane, so the top b
// planes of a block are one contiguous run of b * ceil(K/128) * 512 bytes:
//   planes[nb][q][kb][r][w][f],  channel n = 32 nb + 16 f + r  (r < 16),
// word w < 4 of the 128 codes W[n][128 kb ..].  The 128 codes of a block
// split into four sub-steps of 32 (s), each into two halves of 16 (h) of four
// groups (i) of four bytes (c); word w = 2h + t holds half h of sub-steps 2t
// and 2t+1, element (s, h, i, c) at bit (8c + g + p) mod 32 with
// g = 4(s % 2) + i.  Rotating each plane's word left by p puts the b planes'
// bits of one group g on disjoint positions, so the reader merges them with
// one AND-OR per plane and one rotate right by g yields bit p of each of the
// group's four bytes.  The words of channels n and n + 16 (f = 0, 1) sit side
// by side, so the weight-streaming kernel reads both with one 8-byte load.
// Words of channels past N and codes past K are zero.
#include "rows.h"
#include "tasq_internal.h"

namespace tasq {

// One wave per (32-channel block, K block), two word positions (r, w, f) per
// lane: a position's 32 codes are two chunks, and a plane's bits of four
// codes are one dword rotated to their group and masked, so a group costs
// one rotate and one AND-OR per plane (nine instructions; bit by bit it was
// about a hundred).  Bound by memory: 4608x1152 9.4 -> 4.3 us; 10240x3456
// took 41 us (1.7 TB/s), 10240x6720 now takes 25.0 (5.5 TB/s).
//
// FAR: K so large that 32 rows pass the 2 GiB of a window; the chunks are
// then read by 64-bit addresses.
template <bool FAR>
__global__ void __launch_bounds__(256) k_pack_planes(const int8_t *__restrict__ W, int N, int K,
                                                     int KB, int blocks,
                                                     uint32_t *__restrict__ planes)
{
    const int blk = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blk >= blocks)
        return;
    const int nb = blk / KB, kb = blk - nb * KB;
    Window win;
    if constexpr (!FAR)
        win.init(W, N, 32 * nb, 32, K);
    Chunk5 c[2][2] = {};
    uint32_t off[2];
    int k0[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        const int pos = (threadIdx.x & 63) + 64 * v;    // 8 r + 2 w + f
        const int f = pos & 1, w = (pos >> 1) & 3, r = pos >> 3;
        const int row = 16 * f + r;
        k0[v] = 128 * kb + 64 * (w & 1) + 16 * (w >> 1);
        const int8_t *p = W + (size_t)(32 * nb + row) * (size_t)K + k0[v];
        if constexpr (FAR)
            off[v] = (uint32_t)reinterpret_cast<uintptr_t>(p);
        else
            off[v] = win.lead + (uint32_t)row * (uint32_t)K + (uint32_t)k0[v];
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {                // the word's two sub-steps
            const bool ok = 32 * nb + row < N && k0[v] + 32 * sl < K;
            if constexpr (!FAR)
                c[v][sl].load(win.r, ok ? off[v] + 32u * sl : kOOB);
            else if (ok)
                c[v][sl].load_at(p + 32 * sl, W + (size_t)N * (size_t)K);
        }
    }
    uint32_t *out = planes + ((size_t)nb * 8 * (size_t)KB + (size_t)kb) * 128 + (threadIdx.x & 63);
#pragma unroll
    for (int v = 0; v < 2; ++v) {
        uint32_t pw[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
            const v4i x = keep_bytes(c[v][sl].bytes(off[v]), K - k0[v] - 32 * sl);
            const uint32_t d[4] = {(uint32_t)x.x, (uint32_t)x.y, (uint32_t)x.z, (uint32_t)x.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int g = 4 * sl + i;
                // rotate left by g: bit p of byte c moves to 8c + p + g
                const uint32_t rot = __builtin_amdgcn_alignbit(d[i], d[i], (32 - g) & 31);
#pragma unroll
                for (int p = 0; p < 8; ++p)
                    pw[p] |= rot & (0x01010101u << ((p + g) & 7));
            }
        }
#pragma unroll
        for (int p = 0; p < 8; ++p)
            out[(size_t)(7 - p) * (size_t)KB * 128 + 64 * v] = pw[p];
    }
}

hipError_t launch_pack_planes(const int8_t *W, int N, int K, uint32_t *planes,
                              hipStream_t stream)
{
    const auto kernel = window_fits(32, K) ? &k_pack_planes<false> : &k_pack_planes<true>;
    return launch_pack_units(N, K, [&](long long nb, int rows, int KB, int units) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(units + 3) / 4), dim3(256), 0, stream,
                           W + (size_t)nb * 32 * (size_t)K, rows, K, KB, units,
                           planes + (size_t)nb * 8 * (size_t)KB * 128);
        return hipGetLastError();
    });
}

}  // namespace tasq
