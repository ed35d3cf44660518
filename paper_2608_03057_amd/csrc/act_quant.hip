// Asymmetric 8-bit activation quantizer (App. A.1.2, Eqs. act_quant and
// act_scale) feeding the masked GEMM, and the per-precision channel sums of
// the masked weight that its zero point needs.
//
//   alpha = (max(x) - min(x)) / 255,  z = -min(x) / alpha  (per tensor),
//   Q = clamp(round_to_nearest(x / alpha + z), 0, 255),
//   stored as the signed code Q - 128 (int8), the operand of the int8 MFMA.
//
// With x_hat = alpha (Q - z) the layer output is
//   sum_k x_hat_k * sw[n] W_b[n][k] = alpha sw[n] (acc[n] + (128 - z) colsum_b[n]),
//   acc[n] = sum_k (Q_k - 128) W_b[n][k],  colsum_b[n] = sum_k W_b[n][k],
// which the GEMM epilogue evaluates.  The codes are decided in IEEE single
// precision (correctly rounded division, then addition, ties to even);
// when max == min, alpha = 1 and z = -min (every code 0, dequantising to min).
//
// Two launches: per-workgroup ranges into the params buffer's partial slots,
// then a pass in which every workgroup folds those partials and writes its
// share of the codes.  No atomics and no buffer to clear beforehand.  The
// batched form runs the passes of many tensors in few launches.
#include <type_traits>
#include <vector>

#include "quant.h"
#include "rows.h"
#include "tasq_internal.h"

namespace tasq {

namespace {

// Order-preserving map of a finite float to uint32, so that min / max are
// unsigned integer min / max, whatever order the partial ranges are folded in.
__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float order_value(uint32_t k)
{
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(u);
}

// Per-workgroup range of x as order keys: workgroup g of G writes its
// minimum key to part[2g] and its maximum key to part[2g + 1] (no atomics:
// the quantizer folds the partial ranges).  The first 4*n4 elements are read
// as float4 (n4 = 0 when x is not 16-byte aligned), four loads in flight per
// thread.
__device__ __forceinline__ void act_range(const float *__restrict__ x, long long n, long long n4,
                                          uint32_t *__restrict__ part, int g, int G)
{
    __shared__ uint32_t smin[4], smax[4];
    float mn = __builtin_huge_valf(), mx = -__builtin_huge_valf();
    const long long stride = (long long)G * blockDim.x;
    const float4 *x4 = reinterpret_cast<const float4 *>(x);
    long long i = (long long)g * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n4; i += 4 * stride) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = x4[i + u * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            mn = fminf(fminf(mn, v[u].x), fminf(v[u].y, fminf(v[u].z, v[u].w)));
            mx = fmaxf(fmaxf(mx, v[u].x), fmaxf(v[u].y, fmaxf(v[u].z, v[u].w)));
        }
    }
    for (; i < n4; i += stride) {
        const float4 v = x4[i];
        mn = fminf(fminf(mn, v.x), fminf(v.y, fminf(v.z, v.w)));
        mx = fmaxf(fmaxf(mx, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
    }
    for (long long t = (n4 << 2) + (long long)g * blockDim.x + threadIdx.x; t < n; t += stride) {
        mn = fminf(mn, x[t]);
        mx = fmaxf(mx, x[t]);
    }
    // Keys order -0 below +0, so the fold below is independent of the order
    // in which the partial ranges meet.
    uint32_t kmn = order_key(mn), kmx = order_key(mx);
    for (int off = 32; off > 0; off >>= 1) {
        kmn = min(kmn, (uint32_t)__shfl_xor((int)kmn, off));
        kmx = max(kmx, (uint32_t)__shfl_xor((int)kmx, off));
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        smin[wave] = kmn;
        smax[wave] = kmx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) {
            kmn = min(kmn, smin[w]);
            kmx = max(kmx, smax[w]);
        }
        part[2 * g] = kmn;
        part[2 * g + 1] = kmx;
    }
}

__global__ void __launch_bounds__(256) k_act_range(const float *__restrict__ x, long long n,
                                                   long long n4, uint32_t *__restrict__ part)
{
    act_range(x, n, n4, part, blockIdx.x, gridDim.x);
}

__device__ __forceinline__ void scale_of(uint32_t kmn, uint32_t kmx, float &alpha, float &z)
{
    const float mn = order_value(kmn), mx = order_value(kmx);
    if (mx == mn) {
        alpha = 1.0f;
        z = -mn;
    } else {
        alpha = __fdiv_rn(mx - mn, 255.0f);
        z = __fdiv_rn(-mn, alpha);
    }
}

// Codes of elements first, first + step, .. below n (vector part: groups of
// four), div the division by alpha.
template <class Div>
__device__ __forceinline__ void act_codes(const float *__restrict__ x, long long n, long long n4,
                                          int8_t *__restrict__ q, float z, long long first,
                                          long long stride, const Div &div)
{
    auto code = [&](float v) { return rintf(__fadd_rn(div(v), z)); };
    auto codes = [&](float4 v) { return pack_codes(code(v.x), code(v.y), code(v.z), code(v.w)); };
    const float4 *x4 = reinterpret_cast<const float4 *>(x);
    uint32_t *q4 = reinterpret_cast<uint32_t *>(q);
    long long i = first;
    for (; i + 3 * stride < n4; i += 4 * stride) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = x4[i + u * stride];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            q4[i + u * stride] = codes(v[u]);
    }
    for (; i < n4; i += stride)
        q4[i] = codes(x4[i]);
    for (long long t = (n4 << 2) + first; t < n; t += stride)
        q[t] = (int8_t)pack_codes(code(x[t]), 0.f, 0.f, 0.f);
}

// Every workgroup (g of Q) folds the G partial ranges (a few KB, cache
// resident) into alpha and z, then writes the codes of its share; workgroup
// 0 also publishes alpha and z.  n4 as in act_range, with q 4-byte aligned
// whenever n4 > 0.
__device__ __forceinline__ void act_quantize(const float *__restrict__ x, long long n,
                                             long long n4, int8_t *__restrict__ q, float *params,
                                             int G, int g, int Q)
{
    __shared__ uint32_t smin[4], smax[4];
    const uint32_t *part = reinterpret_cast<const uint32_t *>(params + kActHeader);
    uint32_t kmn = 0xffffffffu, kmx = 0u;
    for (int g = threadIdx.x; g < G; g += blockDim.x) {
        kmn = min(kmn, part[2 * g]);
        kmx = max(kmx, part[2 * g + 1]);
    }
    for (int off = 32; off > 0; off >>= 1) {
        kmn = min(kmn, (uint32_t)__shfl_xor((int)kmn, off));
        kmx = max(kmx, (uint32_t)__shfl_xor((int)kmx, off));
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) {
        smin[wave] = kmn;
        smax[wave] = kmx;
    }
    __syncthreads();
    kmn = min(min(smin[0], smin[1]), min(smin[2], smin[3]));
    kmx = max(max(smax[0], smax[1]), max(smax[2], smax[3]));
    float alpha, z;
    scale_of(kmn, kmx, alpha, z);
    if (g == 0 && threadIdx.x == 0) {
        params[0] = alpha;
        params[1] = z;
    }
    const long long stride = (long long)Q * blockDim.x;
    const long long first = (long long)g * blockDim.x + threadIdx.x;
    const Divider div(alpha);
    if (div.exact)
        act_codes(x, n, n4, q, z, first, stride, div);
    else
        act_codes(x, n, n4, q, z, first, stride, [&](float v) { return __fdiv_rn(v, alpha); });
}

__global__ void __launch_bounds__(256) k_act_quantize(const float *__restrict__ x, long long n,
                                                      long long n4, int8_t *__restrict__ q,
                                                      float *params, int G)
{
    act_quantize(x, n, n4, q, params, G, blockIdx.x, gridDim.x);
}

// Many tensors in one launch: each task is one tensor's range pass or its
// code pass, run by a contiguous run of the launch's workgroups exactly as
// the single-tensor kernels run it, so the codes and scales are those of the
// single-tensor calls.  The task list travels in the kernel arguments.
struct ActTask {
    const float *x;
    int8_t *q;
    float *params;
    long long n, n4;
    int first;      // first workgroup of the task in the launch
    int wgs;        // its workgroups
    int parts;      // workgroups (partial ranges) of the tensor's range pass
    int quant;      // 0: range pass, 1: code pass
};
constexpr int kActBatchTasks = 16;
struct ActLaunch {
    ActTask t[kActBatchTasks];
    int ntasks;
};

__global__ void __launch_bounds__(256) k_act_batch(const ActLaunch L)
{
    int i = 0;
    while (i + 1 < L.ntasks && (int)blockIdx.x >= L.t[i + 1].first)
        ++i;
    const ActTask &t = L.t[i];
    const int g = (int)blockIdx.x - t.first;
    if (t.quant)
        act_quantize(t.x, t.n, t.n4, t.q, t.params, t.parts, g, t.wgs);
    else
        act_range(t.x, t.n, t.n4, reinterpret_cast<uint32_t *>(t.params + kActHeader), g,
                  t.parts);
}

// ------------------------------------------------- low-rank down projection
//
// T = x~ D^T for the 16-bit low-rank branch: x~ is x rounded to bfloat16
// (nearest, ties to even), D [r x K] bfloat16, T fp32 [M x r], r <= 32.
// One workgroup per block of 16 or 32 rows (grid-stride over blocks); its 16
// waves take interleaved 32-wide K steps, each a v_mfma_f32_16x16x32_bf16 per
// 16 rows and 16 columns of D^T, with lane l feeding row l%16 of x and column
// l%16 of D^T (columns past r are zero), 8 elements from 8*(l/16).
// The waves' partial blocks are summed through LDS in a fixed order, so T
// does not depend on timing.  The same pass can fold the range of x (one
// partial per workgroup, as k_act_range), so that quantizing the codes and
// projecting share one read of x.  Bound by the loads in flight per compute
// unit, D's from L2 counting as much as x's: blocks of 16 rows up to one
// workgroup per compute unit (32-row blocks left half the chip idle at 4096
// rows), of 32 beyond, which read D half as often (8192x2240, rank 32: 15.0 us,
// 19.0 with 16-row blocks).  Whole 128-byte lines of a row either way.  us,
// one 32x32x16 product per block and step / now, rank 32: 4096x2240 15.1 /
// 10.4, 300x4608 26.2 / 18.1, 16384x4608 77.1 / 58.1.

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kDownWaves = 16;

__device__ __forceinline__ uint32_t bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ v4u pack_bf16(float4 lo, float4 hi)
{
    return v4u{bf16_rne(lo.x) | (bf16_rne(lo.y) << 16), bf16_rne(lo.z) | (bf16_rne(lo.w) << 16),
               bf16_rne(hi.x) | (bf16_rne(hi.y) << 16), bf16_rne(hi.z) | (bf16_rne(hi.w) << 16)};
}

__device__ __forceinline__ void fold_range(float4 v, float &mn, float &mx)
{
    mn = fminf(fminf(mn, v.x), fminf(v.y, fminf(v.z, v.w)));
    mx = fmaxf(fmaxf(mx, v.x), fmaxf(v.y, fmaxf(v.z, v.w)));
}

// NF, NB: 16-wide column and row fragments of a block.
// FAST: K % 8 == 0 and x, D 16-byte aligned, so an in-range K step covers
// all 8 elements of a lane; each wave then issues the loads of 4 of its row
// fragments' K steps before their MFMAs (enough bytes in flight with one workgroup per
// CU).  Otherwise every element is loaded on its own with bounds checks.
template <bool RANGE, bool FAST, int NF, int NB>
__global__ void __launch_bounds__(64 * kDownWaves)
k_lowrank_down(const float *__restrict__ x, int M, int K, const uint16_t *__restrict__ D, int r,
               float *__restrict__ T, uint32_t *__restrict__ part)
{
    __shared__ float red[kDownWaves][NB * NF * 4][64];
    __shared__ uint32_t smin[kDownWaves], smax[kDownWaves];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, quarter = lane >> 4;
    const int nsteps = (K + 31) / 32;
    const int nblocks = (M + 16 * NB - 1) / (16 * NB);
    float mn = __builtin_huge_valf(), mx = -__builtin_huge_valf();

    for (int rb = blockIdx.x; rb < nblocks; rb += gridDim.x) {
        const float *xr[NB];        // the rows of x and of D (columns of D^T)
        const uint16_t *dr[NF];     // that this lane feeds
        bool rok[NB], dok[NF];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int row = (rb * NB + i) * 16 + j;
            rok[i] = row < M;
            xr[i] = x + (size_t)(rok[i] ? row : 0) * (size_t)K;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            dok[f] = 16 * f + j < r;
            dr[f] = D + (size_t)(dok[f] ? 16 * f + j : 0) * (size_t)K;
        }
        v4f acc[NB][NF] = {};
        auto step = [&](v4u aw, v4u bw, v4f &c) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, aw),
                                                        __builtin_bit_cast(v8bf, bw), c, 0, 0, 0);
        };
        if constexpr (FAST) {
            constexpr int U = 4 / NB;
            for (int s0 = wave; s0 < nsteps; s0 += U * kDownWaves) {
                float4 lo[U][NB], hi[U][NB];
                v4u bw[U][NF];
                bool kin[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int k = 32 * (s0 + u * kDownWaves) + 8 * quarter;
                    kin[u] = k < K;
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        lo[u][i] = make_float4(0.f, 0.f, 0.f, 0.f);
                        hi[u][i] = lo[u][i];
                        if (rok[i] && kin[u]) {
                            const float4 *p = reinterpret_cast<const float4 *>(xr[i] + k);
                            lo[u][i] = p[0];
                            hi[u][i] = p[1];
                        }
                    }
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        bw[u][f] = v4u{0, 0, 0, 0};
                        if (dok[f] && kin[u])
                            bw[u][f] = *reinterpret_cast<const v4u *>(dr[f] + k);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        if (RANGE && rok[i] && kin[u]) {
                            fold_range(lo[u][i], mn, mx);
                            fold_range(hi[u][i], mn, mx);
                        }
                        const v4u aw = pack_bf16(lo[u][i], hi[u][i]);
#pragma unroll
                        for (int f = 0; f < NF; ++f)
                            step(aw, bw[u][f], acc[i][f]);
                    }
            }
        } else {
            for (int s = wave; s < nsteps; s += kDownWaves) {
                const int k = 32 * s + 8 * quarter;
                v4u bw[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    uint32_t dv[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        dv[e] = dok[f] && k + e < K ? (uint32_t)dr[f][k + e] : 0u;
                    bw[f] = v4u{dv[0] | (dv[1] << 16), dv[2] | (dv[3] << 16),
                                dv[4] | (dv[5] << 16), dv[6] | (dv[7] << 16)};
                }
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    float xv[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const bool ok = rok[i] && k + e < K;
                        xv[e] = ok ? xr[i][k + e] : 0.f;
                        if (ok) {
                            mn = fminf(mn, xv[e]);
                            mx = fmaxf(mx, xv[e]);
                        }
                    }
                    const v4u aw = pack_bf16(make_float4(xv[0], xv[1], xv[2], xv[3]),
                                             make_float4(xv[4], xv[5], xv[6], xv[7]));
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        step(aw, bw[f], acc[i][f]);
                }
            }
        }
        // Register v of lane l is row 4*(l/16) + v, column l%16.
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[wave][(i * NF + f) * 4 + v][lane] = acc[i][f][v];
        __syncthreads();
        for (int e = threadIdx.x; e < NB * NF * 4 * 64; e += 64 * kDownWaves) {
            const int v = e >> 6, l = e & 63, frag = v >> 2;
            const int orow = (rb * NB + frag / NF) * 16 + 4 * (l >> 4) + (v & 3);
            const int ocol = 16 * (frag % NF) + (l & 15);
            float sum = red[0][v][l];
#pragma unroll
            for (int w = 1; w < kDownWaves; ++w)
                sum += red[w][v][l];
            if (orow < M && ocol < r)
                T[(size_t)orow * (size_t)r + ocol] = sum;
        }
        __syncthreads();
    }
    if (RANGE) {
        uint32_t kmn = order_key(mn), kmx = order_key(mx);
        for (int off = 32; off > 0; off >>= 1) {
            kmn = min(kmn, (uint32_t)__shfl_xor((int)kmn, off));
            kmx = max(kmx, (uint32_t)__shfl_xor((int)kmx, off));
        }
        if (lane == 0) {
            smin[wave] = kmn;
            smax[wave] = kmx;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kDownWaves; ++w) {
                kmn = min(kmn, smin[w]);
                kmx = max(kmx, smax[w]);
            }
            part[2 * blockIdx.x] = kmn;
            part[2 * blockIdx.x + 1] = kmx;
        }
    }
}

// Channel sums of the masked weight at every b in one pass: LPR lanes per
// row, a 16-byte chunk each, and per dword and b one AND and one four-byte
// dot product with ones (v_dot4_i32_i8).  Bound by the latency of a row's
// loads: a byte per lane and load held it at 0.6-0.95 TB/s.  4608x1152
// 9.4 -> 5.5 us; 10240x3456 took 37 us, 10240x6720 now takes 19.2 (3.6 TB/s).
template <int LPR>
__global__ void __launch_bounds__(256) k_weight_colsums(const int8_t *__restrict__ W, int N, int K,
                                                        int32_t *__restrict__ colsums)
{
    constexpr int RPW = 64 / LPR, U = 2;
    const int lane = threadIdx.x & 63, j = lane % LPR, sub = lane / LPR;
    const int n0 = (blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * RPW;
    if (n0 >= N)
        return;
    Window w;
    w.init(W, N, n0, RPW, K);
    const uint32_t off = w.lead + (uint32_t)sub * (uint32_t)K;
    int s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int k0 = 16 * j; k0 < K; k0 += 16 * LPR * U) {
        Chunk5 c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + 16 * LPR * u;
            c[u].load(w.r, k < K ? off + (uint32_t)k : kOOB);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const v4i v = keep_bytes(c[u].bytes(off), K - k0 - 16 * LPR * u);
#pragma unroll
            for (int b = 1; b <= 8; ++b) {
                const int m = (int)keep_mask_dword(b);
                int t = s[b - 1];
                t = __builtin_amdgcn_sdot4(v.x & m, 0x01010101, t, false);
                t = __builtin_amdgcn_sdot4(v.y & m, 0x01010101, t, false);
                t = __builtin_amdgcn_sdot4(v.z & m, 0x01010101, t, false);
                s[b - 1] = __builtin_amdgcn_sdot4(v.w & m, 0x01010101, t, false);
            }
        }
    }
#pragma unroll
    for (int b = 0; b < 8; ++b)
        for (int o = LPR / 2; o > 0; o >>= 1)
            s[b] += __shfl_xor(s[b], o);
    if (j == 0 && n0 + sub < N) {
#pragma unroll
        for (int b = 0; b < 8; ++b)
            colsums[(long long)b * N + n0 + sub] = s[b];
    }
}

int grid_for(long long items, int per_block, int cap)
{
    long long g = (items + per_block - 1) / per_block;
    if (g > cap)
        g = cap;
    return g < 1 ? 1 : (int)g;
}

}  // namespace

hipError_t launch_quantize_activations(const float *x, long long n, int8_t *q, float *params,
                                       hipStream_t stream)
{
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(q) & 3) == 0;
    const long long n4 = vec ? n >> 2 : 0;
    const long long items = vec ? (n + 3) / 4 : n;
    // Range: at most kActPartials workgroups, four float4 per thread per pass.
    const int G = grid_for(items, 256 * 4, kActPartials);
    uint32_t *part = reinterpret_cast<uint32_t *>(params + kActHeader);
    hipLaunchKernelGGL(k_act_range, dim3(G), dim3(256), 0, stream, x, n, n4, part);
    hipLaunchKernelGGL(k_act_quantize, dim3(grid_for(items, 256, 1024)), dim3(256), 0, stream, x,
                       n, n4, q, params, G);
    return hipGetLastError();
}

// Groups of consecutive tensors (at most half a launch's tasks, and about
// 192 MB of x unless a single tensor is larger) run their code pass in the
// launch after their range pass, beside the next group's range pass:
// ceil(n / group) + 1 launches instead of 2 n, and each x is read the second
// time while it is still in the last-level cache (256 MB).  us, groups of 128 /
// 192 / 400 MB: SANA block of 3000 tokens 65.9 / 60.7 / 59.4, PixArt block of
// 8192 116 / 116 / 113, SANA block of 8192 171 / 172 / 180.
hipError_t launch_quantize_activations_batch(const ActJob *jobs, int n, hipStream_t stream)
{
    constexpr long long kGroupBytes = 192LL << 20;
    constexpr int kGroupTasks = kActBatchTasks / 2;
    struct Prep {
        ActTask range, quant;
    };
    std::vector<Prep> prep;
    prep.reserve((size_t)n);
    for (int j = 0; j < n; ++j) {
        const ActJob &a = jobs[j];
        const long long cnt = (long long)a.M * a.K;
        if (cnt == 0)
            continue;
        const bool vec = (reinterpret_cast<uintptr_t>(a.x) & 15) == 0 &&
                         (reinterpret_cast<uintptr_t>(a.q) & 3) == 0;
        const long long n4 = vec ? cnt >> 2 : 0;
        const long long items = vec ? (cnt + 3) / 4 : cnt;
        const int G = grid_for(items, 256 * 4, kActPartials);
        ActTask r = {a.x, a.q, a.params, cnt, n4, 0, G, G, 0};
        ActTask q = r;
        q.wgs = grid_for(items, 256, 1024);
        q.quant = 1;
        prep.push_back({r, q});
    }
    // group boundaries
    std::vector<int> bounds{0};
    long long bytes = 0;
    for (int j = 0; j < (int)prep.size(); ++j) {
        const long long b = prep[j].range.n * 4;
        const int in_group = j - bounds.back();
        if (in_group > 0 && (in_group == kGroupTasks || bytes + b > kGroupBytes)) {
            bounds.push_back(j);
            bytes = 0;
        }
        bytes += b;
    }
    bounds.push_back((int)prep.size());
    const int ng = (int)bounds.size() - 1;
    for (int k = 0; k <= ng && !prep.empty(); ++k) {
        ActLaunch L = {};
        int wg = 0;
        auto add = [&](ActTask t) {
            t.first = wg;
            wg += t.wgs;
            L.t[L.ntasks++] = t;
        };
        if (k > 0)
            for (int j = bounds[k - 1]; j < bounds[k]; ++j)
                add(prep[j].quant);
        if (k < ng)
            for (int j = bounds[k]; j < bounds[k + 1]; ++j)
                add(prep[j].range);
        hipLaunchKernelGGL(k_act_batch, dim3(wg), dim3(256), 0, stream, L);
        if (hipError_t e = hipGetLastError(); e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_lowrank_down(const float *x, int M, int K, const uint16_t *D, int r, float *T,
                               uint32_t *part, int *groups, hipStream_t stream)
{
    const bool fast = (K % 8) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(D) & 15) == 0;
    const bool wide = M > 16 * 256;     // more 16-row blocks than compute units
    const int G = grid_for(M, wide ? 32 : 16, kActPartials);
    if (groups)
        *groups = G;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(G), dim3(64 * kDownWaves), 0, stream, x, M, K, D, r, T,
                           part);
        return hipGetLastError();
    };
    auto with_rows = [&](auto nf, auto nb) {
        constexpr int NF = decltype(nf)::value, NB = decltype(nb)::value;
        if (part)
            return launch(fast ? &k_lowrank_down<true, true, NF, NB>
                               : &k_lowrank_down<true, false, NF, NB>);
        return launch(fast ? &k_lowrank_down<false, true, NF, NB>
                           : &k_lowrank_down<false, false, NF, NB>);
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    if (r <= 16)
        return wide ? with_rows(One{}, Two{}) : with_rows(One{}, One{});
    return wide ? with_rows(Two{}, Two{}) : with_rows(Two{}, One{});
}

hipError_t launch_quantize_activations_lowrank(const float *x, int M, int K, int8_t *q,
                                               float *params, const uint16_t *D, int r, float *T,
                                               hipStream_t stream)
{
    int G = 0;
    uint32_t *part = reinterpret_cast<uint32_t *>(params + kActHeader);
    hipError_t e = launch_lowrank_down(x, M, K, D, r, T, part, &G, stream);
    if (e != hipSuccess)
        return e;
    const long long n = (long long)M * K;
    const bool vec = (reinterpret_cast<uintptr_t>(x) & 15) == 0 &&
                     (reinterpret_cast<uintptr_t>(q) & 3) == 0;
    const long long n4 = vec ? n >> 2 : 0;
    const long long items = vec ? (n + 3) / 4 : n;
    hipLaunchKernelGGL(k_act_quantize, dim3(grid_for(items, 256, 1024)), dim3(256), 0, stream, x,
                       n, n4, q, params, G);
    return hipGetLastError();
}

hipError_t launch_weight_colsums(const int8_t *W, int N, int K, int32_t *colsums,
                                 hipStream_t stream)
{
    // Rows of 2048 weights and more keep a whole wave's lanes busy.
    if (K >= 2048)
        hipLaunchKernelGGL(k_weight_colsums<64>, dim3((unsigned)((N + 3LL) / 4)), dim3(256), 0,
                           stream, W, N, K, colsums);
    else
        hipLaunchKernelGGL(k_weight_colsums<16>, dim3((unsigned)((N + 15LL) / 16)), dim3(256), 0,
                           stream, W, N, K, colsums);
    return hipGetLastError();
}

}  // namespace tasq
