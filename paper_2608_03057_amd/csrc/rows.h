// Bounded loads of int8 matrix rows, aligned or not.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace tasq {

typedef int v4i __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- buffers

// Raw buffer resources: a load whose byte offset is at or past num_records
// returns zero and such a store is dropped, which bounds every access to
// its operand without per-element checks.  Offsets are 32-bit; the host
// keeps every operand below 2 GiB and kOOB marks a lane with nothing to do.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOOB = 0x80000000u;

__device__ __forceinline__ rsrc_t make_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             0x00020000);
}

__device__ __forceinline__ v4i ld16(rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// Rows of an int8 matrix at any byte alignment.  A 16-byte chunk at byte o of
// the rows' window is taken as the five aligned dwords from o & ~3 on and
// funnel-shifted into place (four v_alignbyte_b32) on its way to LDS.  The
// window starts at the dword holding the first byte and ends with the dword
// holding the last one, so every dword it reads holds a byte of the matrix;
// the others are dropped by the buffer bounds.  It is set per output tile,
// so the matrix itself may exceed the 2 GiB of a buffer offset.
//
// Bound by instruction issue and latency like the aligned path: the extra
// dword load and shifts hide behind the matrix work of the other waves.
// A call in a row of calls, against byte-by-byte loads (sixteen per chunk):
// 777x1153 -> 1111 12.6 us (62.5 before, both with 64x64 tiles; 8.3 with K
// shared by wave groups as well), 8192x1151 -> 3456 64.2 us (361.7), a 20x30 conv
// 1275 -> 1280 64.9 us (1217).
//
// window_fits: rows * K bytes, the partial dwords at both ends and every
// offset into them stay below kOOB.
constexpr bool window_fits(long long rows, long long K)
{
    return rows * K + 8 < (long long)kOOB;
}

struct Window {
    rsrc_t r;
    uint32_t lead;              // bytes before the first row in its dword

    __device__ __forceinline__ void init(const int8_t *base, int rows, int first, int count,
                                         int K)
    {
        const int8_t *p = base + (size_t)first * (size_t)K;
        lead = (uint32_t)(reinterpret_cast<uintptr_t>(p) & 3u);
        const int n = min(rows - first, count);
        const uint32_t bytes = n > 0 ? lead + (uint32_t)n * (uint32_t)K : 0u;
        r = make_rsrc(p - lead, (bytes + 3u) & ~3u);
    }
};

struct Chunk5 {
    v4i lo;
    uint32_t hi;

    __device__ __forceinline__ void load(rsrc_t r, uint32_t off)
    {
        lo = ld16(r, off & ~3u);
        hi = __builtin_amdgcn_raw_buffer_load_b32(r, (off & ~3u) + 16u, 0, 0);
    }

    // The same dwords by address, for rows that no window holds: p < end, and
    // dwords that begin at or after end, the end of the matrix, are not read.
    __device__ __forceinline__ void load_at(const int8_t *p, const int8_t *end)
    {
        const uintptr_t a = reinterpret_cast<uintptr_t>(p) & ~(uintptr_t)3;
        const uintptr_t e = reinterpret_cast<uintptr_t>(end);
        const uint32_t *q = reinterpret_cast<const uint32_t *>(a);
        lo.x = (int)q[0];
        lo.y = a + 4 < e ? (int)q[1] : 0;
        lo.z = a + 8 < e ? (int)q[2] : 0;
        lo.w = a + 12 < e ? (int)q[3] : 0;
        hi = a + 16 < e ? q[4] : 0u;
    }

    // The 16 bytes from byte off % 4 of the five dwords on.
    __device__ __forceinline__ v4i bytes(uint32_t off) const
    {
        const uint32_t a = (uint32_t)lo.x, b = (uint32_t)lo.y, c = (uint32_t)lo.z,
                       d = (uint32_t)lo.w;
        return v4i{(int)__builtin_amdgcn_alignbyte(b, a, off),
                   (int)__builtin_amdgcn_alignbyte(c, b, off),
                   (int)__builtin_amdgcn_alignbyte(d, c, off),
                   (int)__builtin_amdgcn_alignbyte(hi, d, off)};
    }
};

// Launches of a packer over an N x K weight in blocks of 32 rows: f(nb, rows,
// KB, units) packs `rows` rows from block nb on, `units` (32-row, 128-byte)
// units of a wave each.  One launch takes at most 2^22 units or one block of
// rows, so that its unit and row numbers stay in 32 bits and its threads below
// the 2^32 of a grid.
template <class F>
inline hipError_t launch_pack_units(long long N, long long K, F f)
{
    const long long KB = (K + 127) / 128, NB = (N + 31) / 32;
    const long long most = (1LL << 22) / KB, step = most > 1 ? most : 1;
    for (long long nb = 0; nb < NB; nb += step) {
        const long long blocks = NB - nb < step ? NB - nb : step;
        const long long left = N - 32 * nb, rows = left < 32 * blocks ? left : 32 * blocks;
        if (hipError_t e = f(nb, (int)rows, (int)KB, (int)(blocks * KB)))
            return e;
    }
    return hipSuccess;
}

// Keeps the first `valid` bytes of a chunk.
__device__ __forceinline__ v4i keep_bytes(v4i v, int valid)
{
    auto mask = [&](int w) {
        const int n = valid - 4 * w;
        return n >= 4 ? -1 : n <= 0 ? 0 : (1 << (8 * n)) - 1;
    };
    v.x &= mask(0);
    v.y &= mask(1);
    v.z &= mask(2);
    v.w &= mask(3);
    return v;
}

}  // namespace tasq
