// Masked int8 GEMM with the K range of each output tile shared by groups of
// waves, for layers with too few tiles to keep the compute units busy.
#include "gemm_core.h"

namespace tasq {

// KG groups of a tile configuration's waves share one output tile: group g
// accumulates the K tiles g * nkg .. (g + 1) * nkg - 1 in LDS stages of its
// own, then group 0 adds the others' exact int32 partials, handed over
// through those stages in a fixed order, and writes the tile.  What bounds a
// layer of few tiles is the chain of a tile's K tiles, about 0.5 us each
// (64x64) with one workgroup on a compute unit; groups walk it side by side
// until the compute unit's loads in flight (some 64 KB) are the limit.
// 128x4608 -> 1152 14.1 -> 10.7 us, 2000x4608 -> 1152 26.5 -> 22.6.
template <class C, int KG>
constexpr int kg_lds()
{
    return KG * (C::SMA + C::NSTAGE * C::BN * C::CPR);
}

// Tile t of layer d.
template <class C, int KG, bool ALIGNED, int KIND>
__device__ __forceinline__ void kg_tile(const LayerDesc &d, int t, int bits, v4i *sm)
{
    constexpr int SB = C::NSTAGE * C::BN * C::CPR;
    static_assert((C::SMA + SB) * 16 >= C::BM * C::BN * 4, "a group's partial tile fits its stages");
    const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / C::NT);
    v4i *const smA = sm + group * (C::SMA + SB), *const smB = smA + C::SMA;
    int tm, tn;
    tile_coords(t, d.tiles_m, d.tiles_n, tm, tn);
    const int m0 = tm * C::BM, n0 = tn * C::BN;
    const int ktot = KIND == KIND_CONV3X3 && !ALIGNED ? 9 * ((d.C + 15) & ~15) : d.K;
    // Every group walks the same number of K tiles (the barriers are the
    // workgroup's); those past its range read zero weights.
    const int nkg = ((ktot + C::BK - 1) / C::BK + KG - 1) / KG;
    const int kb = group * nkg * C::BK, ke = min(ktot, kb + nkg * C::BK);
    v16i acc[C::FM][C::FN];
    ColLoads<C> cl;
    mainloop<C, ALIGNED, KIND, false>(d, keep_mask_dword(bits), m0, n0, kb, ke, nkg, acc, smA,
                                      smB, [&] { cols_request<C, true>(d, n0, bits, cl); });
    __syncthreads();                // every wave is done with the stages
    const int tid = threadIdx.x % C::NT;
    if (group > 0) {
        int *p = reinterpret_cast<int *>(smA) + tid;
#pragma unroll
        for (int i = 0; i < C::FM; ++i)
#pragma unroll
            for (int j = 0; j < C::FN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    p[((i * C::FN + j) * 16 + v) * C::NT] = acc[i][j][v];
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
        for (int g = 1; g < KG; ++g) {
            const int *p = reinterpret_cast<const int *>(sm + g * (C::SMA + SB)) + tid;
#pragma unroll
            for (int i = 0; i < C::FM; ++i)
#pragma unroll
                for (int j = 0; j < C::FN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[i][j][v] += p[((i * C::FN + j) * 16 + v) * C::NT];
        }
    }
    epilogue_stage<C, KG * C::NT>(d, m0, n0, reinterpret_cast<char *>(sm));
    if (group == 0) {
        EpiCols<C> ec;
        cols_finish<C, true>(d, m0, n0, cl, ec);
        epilogue_write<C>(d, acc, ec, reinterpret_cast<char *>(sm));
    }
}

template <class C, int KG, bool ALIGNED, int KIND>
__global__ void __launch_bounds__(C::NT * KG, C::OCC) k_masked_gemm_kg(LayerDesc d)
{
    __shared__ v4i sm[kg_lds<C, KG>()];
    pin(d);
    kg_tile<C, KG, ALIGNED, KIND>(d, xcd_remap(blockIdx.x, gridDim.x), d.bits, sm);
}

// A grouped step of linear layers (k_masked_gemm_grouped) whose tiles share K
// the same way, for steps of few tiles, which the chain of the deepest layer's
// K tiles bounds: one PixArt-shaped block at 100 tokens 17.5 -> 14.0 us per
// step, at 256 tokens 20.6 -> 16.0.
template <class C, int KG>
__global__ void __launch_bounds__(C::NT * KG, C::OCC)
k_masked_gemm_kg_grouped(const LayerDesc *__restrict__ descs, int L,
                         const uint8_t *__restrict__ table, int S, int stage, int rounds)
{
    __shared__ v4i sm[kg_lds<C, KG>()];
    const GroupedUnit u = grouped_unit(descs, L, rounds);
    LayerDesc d = descs[u.layer];
    pin(d);
    const int bits = table_bits(table, d.layer * S + stage);
    kg_tile<C, KG, true, KIND_LINEAR>(d, u.tile, bits, sm);
}

template <class C, int KG>
hipError_t launch_kg_cfg(const LayerDesc &din, bool aligned, hipStream_t stream)
{
    LayerDesc d = din;
    fill_tiles<C>(d);
    const long long grid = (long long)d.tiles_m * d.tiles_n;
    if (grid > 0x7fffffffLL)
        return hipErrorInvalidValue;
    dim3 g((unsigned)grid), b(C::NT * KG);
    if (d.kind == KIND_CONV3X3 && aligned)
        hipLaunchKernelGGL((k_masked_gemm_kg<C, KG, true, KIND_CONV3X3>), g, b, 0, stream, d);
    else if (d.kind == KIND_CONV3X3)
        hipLaunchKernelGGL((k_masked_gemm_kg<C, KG, false, KIND_CONV3X3>), g, b, 0, stream, d);
    else if (aligned)
        hipLaunchKernelGGL((k_masked_gemm_kg<C, KG, true, KIND_LINEAR>), g, b, 0, stream, d);
    else
        hipLaunchKernelGGL((k_masked_gemm_kg<C, KG, false, KIND_LINEAR>), g, b, 0, stream, d);
    return hipGetLastError();
}

hipError_t launch_kgroups(const LayerDesc &d, KGroupTile tile, bool aligned, hipStream_t stream)
{
    using C64 = Cfg<64, 64, 128, 2, 2, 2, 4>;
    using C128 = Cfg<128, 128, 128, 2, 2, 2, 2>;
    switch (tile) {
    case KG_64x64_2: return launch_kg_cfg<C64, 2>(d, aligned, stream);
    case KG_64x64_4: return launch_kg_cfg<C64, 4>(d, aligned, stream);
    case KG_128x128_2: return launch_kg_cfg<C128, 2>(d, aligned, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_kgroups_2x64(const LayerDesc *d_descs, int L, int total_tiles,
                               const uint8_t *d_table, int S, int stage, bool any_conv,
                               bool rounds, hipStream_t stream)
{
    using C = Cfg<64, 64, 128, 2, 2, 2, 4>;
    if (any_conv)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_masked_gemm_kg_grouped<C, 2>), dim3((unsigned)total_tiles),
                       dim3(C::NT * 2), 0, stream, d_descs, L, d_table, S, stage, rounds ? 1 : 0);
    return hipGetLastError();
}

}  // namespace tasq
