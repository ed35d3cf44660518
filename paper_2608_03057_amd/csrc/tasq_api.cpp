// C ABI of the TASQ masked quantized linear layer: argument validation,
// variant/tile choice, launches, schedule runner.  See include/tasq.h for the
// contract of every entry point.
#include "tasq.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "tasq_internal.h"

using tasq::LayerDesc;

namespace {

constexpr size_t kWsAlign = 256;

// XCDs of the device; the grouped GEMM kernels give each one a contiguous
// run of work units (xcd_remap in gemm_core.h).
constexpr int kXcds = 8;
constexpr int kComputeUnits = 256;
constexpr double kImbalanceLimit = 1.10;

// Cost of a 256x256 tile of the persistent step in bytes of K: its K plus a
// fixed part for its epilogue and the next tile's prologue.  The 28-block
// PixArt-shaped step (4.13 ms, 147 tiles per compute unit, 12.2 K tiles of
// 128 each on average) spends about 0.66 ms in tile ends, 4.5 us per tile,
// against 1.9 us per K tile: about 300 bytes of K.
constexpr double kTileFixedK = 384.0;

// Persistent steps of up to this many tiles run over lists of units, which the
// host deals out on each call, where these cut the busiest workgroup's cost to
// 0.87 of the runs'.  us per step, runs / lists: 1 PixArt block at 4096 tokens
// (672 tiles) 107 / 83, 6 at 700 (756) 109.5 / 97.6, 1 SANA block at 3000 (1068)
// 197.8 / 179.4, 2 PixArt blocks at 4096 (1344) 165.2 / 157.3; but 6 at 2048
// (2016) 225.3 / 231.1: six tiles per workgroup and more even out, and layers
// in turn keep the stores of shallow tiles under the matrix work of deep ones.
// The line of 0.87: at 0.85 16 SANA blocks at 256 tokens 370 / 330 and 8 PixArt
// blocks at 700 120.9 / 120.9, at 0.873 8 PixArt blocks at 1024 159.3 / 168.5 and 16 at
// 500 184.8 / 188.4 (a run there is an XCD's own block or two, its tail of deep
// tiles alone with the memory), at 0.886 4 blocks at 2048 164.4 / 161.1.
constexpr long long kListMaxUnits = 1536;
constexpr double kListGain = 0.87;
constexpr long long kStepCostMaxTiles = 4096;   // pick_step_tile
// A tile of theirs takes about 8.5 us plus 1.6 per K tile of 128 bytes.
constexpr double kListFixedK = 680.0;

// The XCD runs of a persistent launch: contiguous in the work-unit order
// (neighbouring tiles share operands in one L2) and cut at about equal cost,
// a tile costing its K plus kTileFixedK.  Equal counts of tiles would give
// the XCD whose run ends a block later in the 28-block PixArt-shaped step
// (more 4608-deep tiles) 3% more work than the mean.
tasq::XcdRuns cost_runs(const std::vector<LayerDesc> &descs, long long total)
{
    double all = 0;
    for (const LayerDesc &d : descs)
        all += (double)d.tiles_m * d.tiles_n * ((double)d.K + kTileFixedK);
    tasq::XcdRuns r = {};
    int x = 1;
    double cum = 0;
    for (const LayerDesc &d : descs) {
        const long long n = (long long)d.tiles_m * d.tiles_n;
        const double c = (double)d.K + kTileFixedK;
        while (x < kXcds && cum + (double)n * c >= all * x / kXcds) {
            long long take = (long long)((all * x / kXcds - cum) / c + 0.5);
            take = take < 0 ? 0 : take > n ? n : take;
            r.begin[x] = (int)(d.tile_begin + take);
            ++x;
        }
        cum += (double)n * c;
    }
    for (; x < kXcds; ++x)
        r.begin[x] = (int)total;
    r.begin[kXcds] = (int)total;
    for (int i = 1; i <= kXcds; ++i)
        if (r.begin[i] < r.begin[i - 1])
            r.begin[i] = r.begin[i - 1];
    return r;
}

// Cost of the busiest workgroup of a persistent launch over `runs`.
double runs_makespan(const std::vector<LayerDesc> &descs, const tasq::XcdRuns &runs)
{
    constexpr int wgs = tasq::kListWorkgroups / kXcds;
    double mx = 0;
    size_t l = 0;
    for (int x = 0; x < kXcds; ++x) {
        double load[wgs] = {0};
        for (int u = runs.begin[x], j = 0; u < runs.begin[x + 1]; ++u, j = (j + 1) % wgs) {
            while (l + 1 < descs.size() && descs[l + 1].tile_begin <= u)
                ++l;
            load[j] += descs[l].K + kListFixedK;
        }
        mx = std::max(mx, *std::max_element(load, load + wgs));
    }
    return mx;
}

// Work units of a persistent step as one list per workgroup (ListWalk): the
// layers from the deepest K down, each cut into one contiguous run of tiles
// per XCD (tiles that share operands meet in one L2), and within an XCD each
// next tile to the workgroup with the least work so far.  A step of few tiles
// per workgroup whose layers differ in K ends when the workgroup that drew a
// deep tile late is done: the busiest over the UNet block's linear layers (804
// tiles of 256x256, K 640..5120) has 1.42 times the mean work in layer order
// and 1.09 times with lists.
// Returns the cost of the busiest workgroup.
// It is computed on every call, before the first launch, so costs are whole
// numbers in flat arrays (20 us for the 804 tiles above; 120 with a growing list
// per workgroup).
double unit_lists(const std::vector<LayerDesc> &descs, std::vector<uint16_t> &order)
{
    constexpr int W = tasq::kListWorkgroups, wgs = W / kXcds;
    std::vector<const LayerDesc *> by_k;
    by_k.reserve(descs.size());
    for (const LayerDesc &d : descs)
        by_k.push_back(&d);
    std::stable_sort(by_k.begin(), by_k.end(),
                     [](const LayerDesc *a, const LayerDesc *b) { return a->K > b->K; });
    int load[W] = {0}, rows[W] = {0};
    long long xload[kXcds] = {0};
    order.assign((size_t)4 * W, (uint16_t)tasq::kNoUnit);
    for (const LayerDesc *d : by_k) {
        const int n = d->tiles_m * d->tiles_n;
        const int cost = d->K + (int)kListFixedK;
        // An eighth of the layer per XCD, the odd tiles to those with the
        // least work so far.
        int take[kXcds];
        for (int x = 0; x < kXcds; ++x) {
            take[x] = n / kXcds;
            xload[x] += (long long)take[x] * cost;
        }
        for (int i = 0; i < n % kXcds; ++i) {
            const int x = (int)(std::min_element(xload, xload + kXcds) - xload);
            ++take[x];
            xload[x] += cost;
        }
        int u = d->tile_begin;
        for (int x = 0; x < kXcds; ++x)
            for (int i = 0; i < take[x]; ++i, ++u) {
                int *const w = load + x * wgs;
                int least = w[0];
                for (int j = 1; j < wgs; ++j)
                    least = w[j] < least ? w[j] : least;
                int j = 0;
                while (w[j] != least)
                    ++j;
                w[j] += cost;
                const int block = j * kXcds + x;    // workgroup j of XCD x
                const size_t at = (size_t)rows[block]++ * W + block;
                if (at + W >= order.size())         // keeps a row of kNoUnit at the end
                    order.resize(order.size() + 4 * W, (uint16_t)tasq::kNoUnit);
                order[at] = (uint16_t)u;
            }
    }
    order.resize((size_t)(*std::max_element(rows, rows + W) + 1) * W);
    return *std::max_element(load, load + W);
}

// Heaviest XCD run over the mean, for the per-layer tile order, a tile
// costing about its K plus a fixed part for loading and writing the tile.
double xcd_imbalance(const std::vector<LayerDesc> &descs, long long G)
{
    const long long per = (G + kXcds - 1) / kXcds;
    long long tall = G % kXcds;
    if (tall == 0)
        tall = kXcds;
    double work[kXcds] = {0};
    size_t l = 0;
    long long used = 0;          // tiles of layer l already assigned
    double total = 0;
    for (int x = 0; x < kXcds; ++x) {
        long long cnt = x < tall ? per : per - 1;
        while (cnt > 0 && l < descs.size()) {
            const long long n = (long long)descs[l].tiles_m * descs[l].tiles_n - used;
            const long long take = n < cnt ? n : cnt;
            const double w = (double)take * ((double)descs[l].K + 1024.0);
            work[x] += w;
            total += w;
            cnt -= take;
            used += take;
            if (used == (long long)descs[l].tiles_m * descs[l].tiles_n) {
                ++l;
                used = 0;
            }
        }
    }
    double mx = 0;
    for (double w : work)
        mx = w > mx ? w : mx;
    return total > 0 ? mx / (total / kXcds) : 1.0;
}

long long grouped_tiles(const std::vector<LayerDesc> &descs, const tasq::TileShape &ts)
{
    long long n = 0;
    for (const LayerDesc &d : descs)
        n += (long long)((d.M + ts.bm - 1) / ts.bm) * ((d.N + ts.bn - 1) / ts.bn);
    return n;
}

constexpr size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

int variant_of_opts(const tasq_opts *o) { return o ? o->variant : TASQ_VARIANT_AUTO; }

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_dims(long long M, long long N, long long K)
{
    if (M < 0 || N < 0 || K < 0)
        return TASQ_ERR_DIM;
    if (K > TASQ_MAX_K)
        return TASQ_ERR_OVERFLOW;
    return TASQ_OK;
}

// The variant value, split_k and the alignment of the optional buffers.
// Whether the layer has the weight copy its variant reads is checked per
// layer (check_weights).
int check_variant(const tasq_opts *o)
{
    const int v = variant_of_opts(o);
    if (v != TASQ_VARIANT_AUTO && v != TASQ_VARIANT_MASKED_I8 && v != TASQ_VARIANT_BITPLANE &&
        v != TASQ_VARIANT_PACKED)
        return TASQ_ERR_KIND;
    if (o && o->split_k < 0)
        return TASQ_ERR_RANGE;
    if (o && o->W_packed && !aligned16(o->W_packed))
        return TASQ_ERR_ALIGN;
    if (o && o->workspace && (reinterpret_cast<uintptr_t>(o->workspace) % kWsAlign) != 0)
        return TASQ_ERR_ALIGN;
    return TASQ_OK;
}

// Tuning overrides carried in tasq_opts (0 = the library's choice).
int forced_tile(const tasq_opts *o) { return o && o->tile > 0 ? o->tile - 1 : -1; }

int forced_ptile(const tasq_opts *o) { return o && o->packed_tile > 0 ? o->packed_tile - 1 : -1; }

int check_tuning(const tasq_opts *o)
{
    if (!o)
        return TASQ_OK;
    if (o->tile < 0 || o->tile > tasq::TILE_COUNT || o->packed_tile < 0 ||
        o->packed_tile > tasq::PTILE_COUNT || o->persistent < 0 || o->persistent > 2 ||
        o->persistent_wgs < 0 || o->persistent_wgs > 1024 || o->persistent_parties < 0 ||
        o->persistent_parties > 1024)
        return TASQ_ERR_RANGE;
    return TASQ_OK;
}

// The grouped step over linear layers without low-rank or weight-zero-point
// terms runs as a persistent launch (one workgroup per compute unit, tile
// boundaries overlapped) with the 256x256 tile where pick_step_tile's estimate
// says so, otherwise once there are at least two tiles per compute unit, unless
// the caller forces it off or on.
bool use_persistent(const tasq_opts *o, bool big_tile, long long total)
{
    if (o && o->persistent)
        return o->persistent == 2;
    return big_tile && total >= 2LL * kComputeUnits;
}

int persistent_wgs_per_xcd(const tasq_opts *o)
{
    return o && o->persistent_wgs > 0 ? o->persistent_wgs : kComputeUnits / kXcds;
}

// Parts of each XCD's run walked side by side by the persistent launch;
// falls back to 1 when the requested count does not divide the workgroups
// per XCD.
int persistent_parties(const tasq_opts *o, int wgs_per_xcd)
{
    const int p = o && o->persistent_parties > 0 ? o->persistent_parties : 1;
    return wgs_per_xcd % p == 0 ? p : 1;
}

// Packed-weight tile of a single launch, from sweeps of every tile over the
// DiT/UNet layer shapes and a grid of K 1152..8192 at 288 to 1280 tiles: 64x64
// tiles below 200 of 128x256, the 4-wave 128x256 tile (two workgroups per CU,
// one's stores under the other's matrix work) from there, and 256x256
//   * from 140 of them up to one per compute unit: even half a round of them
//     beats 2-3 of smaller ones from about there;
//   * above that where K is over 2048 and the last round has 140 tiles or
//     more: a 128x256 tile reads each weight twice as often, which K pays for,
//     most on buffers that are new to the chip, while the stores it hides
//     don't grow with K;
//   * for the largest layers.
// us, 128x256 / 256x256, the same buffers each call and then new ones: 8192x1152
// -> 3456 (448 tiles of 256x256) 43.0 / 47.7 and 45.1 / 48.0, 8192x1152 -> 4608
// (576) 55.3 / 67.1 and 56.1 / 67.4, 6000x2240 -> 6720 (648) 101 / 109 and 100 /
// 108, 16384x5600 -> 2240 (576) 206 / 223 and 231 / 234; 4096x2240 -> 6720 (432)
// 73.8 / 74.9 and 84.6 / 75.4, 4096x3072 -> 6720 (432) 88.7 / 89.6 and 105 / 92.4,
// 4096x4608 -> 6720 128 / 124 and 151 / 130; on the same buffers 4096x2240 -> 2240
// (144) 36.1 / 33.7, 8192x8192 -> 8192 462 / 435.  Above a round, 128x256 over
// 256x256 on the grid: K up to 2048 0.79 to 0.98, and 0.81 to 1.01 on new
// buffers (2048x2048 -> 16128 1.13, 1200x1152 -> 24000 1.08); deeper with a shorter last round 0.84 to
// 0.98 and 0.92 to 1.04; deeper with 140 tiles or more in it 0.95 to 1.10 and
// 1.00 to 1.23.  Right after a 512 MB fill, which leaves the caches full of
// written lines, 128x256 tiles are slower by up to 12% (8192x1152 -> 3456 62 /
// 55).
// A conv's taps need more registers than the 128x256 tile leaves (its conv
// kernel spills): 256x256 from 140 tiles up whatever their number (us, 128x256 /
// 256x256: 96x96 pixels 1280 -> 2560 434 / 303, 160x160 640 -> 640 187 / 153,
// 128x128 320 -> 1280 99.5 / 91.6).
int pick_packed_tile(const tasq_opts *o, long long M, long long N, long long K, bool conv)
{
    const int f = forced_ptile(o);
    if (f >= 0)
        return f;
    const long long t256 = ((M + 255) / 256) * ((N + 255) / 256);
    const long long t128x256 = ((M + 127) / 128) * ((N + 255) / 256);
    const long long last = t256 % kComputeUnits;
    const bool deep = K > 2048 && (last == 0 || last >= 140);
    if ((t256 >= 140 && (conv || t256 <= kComputeUnits || deep)) || M * N * K >= (1LL << 38))
        return tasq::PTILE_256x256_K128_W8;
    if (t128x256 >= 200)
        return tasq::PTILE_128x256_K128_W4;
    return tasq::PTILE_64x64_K128_W4;
}

// Packed-weight tile of the grouped per-step launch.
int pick_packed_grouped_tile(const tasq_opts *o)
{
    const int f = forced_ptile(o);
    return f >= 0 ? f : tasq::PTILE_256x256_K128_W8;
}

// Estimated time in us of nk K tiles (128 bytes) over output tiles of the
// row-major GEMM kernels, fitted to a sweep of the DiT/UNet layer shapes
// (M 1024..16384, K 320..11200; most within 10%).
//   256x256 (persistent walk, one workgroup per compute unit): rounds of
//     8.5 + 1.35 nk;
//   128x128 (two workgroups per compute unit): rounds of 512 tiles of 4 +
//     1.15 nk, which overlap from two rounds on; a last round of at most one
//     workgroup per compute unit runs at 0.65 nk.
// With a low-rank branch of rank 32 a round ends 3.5 and 3.0 us later (its
// operands staged and multiplied; a round of half the slots is as long), which
// moves the line (us, 128x128 / 256x256: 3000x1152 -> 3456 25.6 / 23.5, 777x1280 ->
// 10240 24.7 / 22.1).  At rank 16 and with weight zero points both grow by less
// and alike, and the line stays.
double cost_256(long long tiles, long long nk, bool rank32)
{
    const double end = rank32 ? 12.0 : 8.5;
    return (double)((tiles + kComputeUnits - 1) / kComputeUnits) * (end + 1.35 * nk);
}

double cost_128(long long tiles, long long nk, bool rank32)
{
    const long long slots = 2 * kComputeUnits, full = tiles / slots, rem = tiles % slots;
    const double end = rank32 ? 7.0 : 4.0;
    if (full >= 2)
        return (double)tiles / slots * (end + 1.15 * nk);
    const double last = rem == 0 ? 0.0 : rem <= kComputeUnits ? 0.65 * nk : 1.15 * nk;
    if (!full)
        return end + last;
    return end + 1.15 * nk + last + (rem && rank32 ? 3.0 : 0.0);
}

// Tile used for a single (non-grouped) launch: 64x64 tiles, so that more
// workgroups cover the 256 compute units, while 128x128 would give fewer
// than 200; above that the cheaper of 128x128 and the persistent 256x256
// walk.  us, 128x128 / 256x256: 4096x640 -> 5120 (320 tiles of 256x256, a
// second round a quarter full) 23.7 / 30.9, 2048x1280 -> 10240 (320) 34.2 /
// 42.4, 8192x1152 -> 3456 (448) 48.9 / 46.9, 4096x2240 -> 2240 (144) 40.0 /
// 33.8, 4096x2240 -> 11200 (704) 124.6 / 104.6.
// From 140 to 256 tiles of 256x256 with K above 1024 always the walk: the
// estimates come from operands that stay in the caches, where the two are
// within 7%, and 128x128 tiles read each operand twice as often, which shows
// on operands that are new to the chip.  us, 128x128 / 256x256, the same
// buffers each call and then new ones: 1024x1280 -> 10240 (160 tiles) 22.1 /
// 22.7 and 28.7 / 23.8, 8192x1152 -> 1152 (160) 21.2 / 20.7 and 22.8 / 21.1,
// 2048x1152 -> 4608 (144) 20.3 / 21.0 and 22.1 / 20.8, 4096x1152 -> 3456 (224)
// 25.3 / 25.1 and 31.1 / 26.2.  With a short K 128x128 is as good or better on
// both: 3000x320 -> 4096 (192) 14.7 / 16.0 and 14.9 / 16.3, 3000x640 -> 5120
// (240) 19.2 / 20.7 and 19.9 / 21.6.
// Byte-aligned operands have no persistent walk: 256x256 tiles from 140 up
// (8192x1151 -> 3456 64 us against 69), and none for a conv, whose chunks'
// taps and shifts need more registers than that tile leaves (96x96 pixels
// 650 -> 650: 93.8 us with 128x128 tiles, 152 with 256x256, 95.9 with 64x64).
int pick_tile(const tasq_opts *o, long long M, long long N, long long K, bool aligned, bool conv,
              bool rank32)
{
    const int f = forced_tile(o);
    if (f >= 0)
        return f;
    const long long t256 = ((M + 255) / 256) * ((N + 255) / 256);
    const long long t128 = ((M + 127) / 128) * ((N + 127) / 128);
    const long long nk = (K + 127) / 128;
    const bool one_round = t256 >= 140 && t256 <= kComputeUnits && K > 1024;
    const bool big = aligned && !conv ? one_round || cost_256(t256, nk, rank32) <
                                                         cost_128(t128, nk, rank32)
                                      : t256 >= 140 && (aligned || !conv);
    if (t128 >= 200 && big)
        return tasq::TILE_256x256_K128_W8_PF1;
    if (t128 >= 200)
        return tasq::TILE_128x128_K128_W4_PF2;
    return tasq::TILE_64x64_K128_W4_PF2;
}

// Wave groups sharing each tile's K range (kgroups.hip), for a single layer
// whose tiles leave compute units short of waves.  us, plain / grouped:
// 128x128 tiles, two groups: 2000x4608 -> 1152 (144 tiles) 26.5 / 22.6, 64x64
// pixels 640 -> 640 3x3 (160) 38.6 / 32.5, 2048x2048 -> 2048 (256) 15.2 / 14.2,
// but 4942x861 -> 640 (195, K too short) 12.5 / 12.9.  64x64 tiles, four
// groups: 128x4608 -> 1152 (36) 14.1 / 10.7, 300x4608 -> 1152 (90) 14.2 / 11.2,
// 18x25 pixels 640 -> 640 (80) 21.5 / 15.6; two groups: 1000x2560 -> 640 (160)
// 9.3 / 8.1, 32x32 pixels 1280 -> 1280 (320) 57.6 / 49.0, 777x1153 -> 1111 (234)
// 9.6 / 8.9.  Beyond those counts the groups only contend for the compute
// unit's loads (1024x1280 -> 3840, 960 tiles of 64x64: 11.9 / 13.7).
tasq::KGroupTile pick_kgroups(const tasq_opts *o, long long M, long long N, long long K)
{
    if (forced_tile(o) >= 0)
        return tasq::KG_NONE;
    const long long t128 = ((M + 127) / 128) * ((N + 127) / 128);
    const long long t64 = ((M + 63) / 64) * ((N + 63) / 64);
    const long long nk = (K + 127) / 128;
    if (t128 >= 130 && t128 <= kComputeUnits && nk >= 14)
        return tasq::KG_128x128_2;
    if (t64 <= kComputeUnits / 2 && nk >= 8)
        return tasq::KG_64x64_4;
    if (t64 <= kComputeUnits + kComputeUnits / 4 && nk >= 8)
        return tasq::KG_64x64_2;
    return tasq::KG_NONE;
}

// Split-K of single-layer calls with the row-major weight.  A layer with few
// output tiles and a long K leaves most of the chip idle while each
// workgroup walks all of K; cutting K into s ranges gives s times the
// workgroups, at the price of writing and re-reading s int32 partial
// outputs (summed in a fixed order, so the result is exact and identical).
// Measured on the DiT/UNet shapes (cache flushed before each launch), the
// partial traffic outweighs the gain unless K is long and the 256x256 tiles
// few: the SDXL-Turbo 3x3 conv (K = 11520, 20 tiles) runs 75 -> 44 us with
// 10 ranges, while K <= 5600 layers ran 0-3x slower split.
constexpr int kSplitMinChunk = 1024;     // at least this much K per split
constexpr int kSplitMinK = 8192;
constexpr int kSplitMaxTiles = 64;

int auto_splits(long long M, long long N, long long K)
{
    const long long t256 = ((M + 255) / 256) * ((N + 255) / 256);
    if (t256 > kSplitMaxTiles || t256 == 0 || K < kSplitMinK)
        return 1;
    long long s = kComputeUnits / t256;
    const long long smax = K / kSplitMinChunk;
    if (s > smax)
        s = smax;
    return s >= 2 ? (int)s : 1;
}

// K range per split (a multiple of 128, the largest BK) and the resulting
// number of non-empty splits.
void split_geometry(int K, int s, int &kchunk, int &splits)
{
    const int per = (K + s - 1) / s;
    kchunk = (per + 127) / 128 * 128;
    splits = (K + kchunk - 1) / kchunk;
}

// Split-K partials of the largest layer a schedule would split (0 when
// none would): the schedule workspace keeps room for them after the device
// layer list and the bit table.
size_t max_split_bytes(const tasq_layer *layers, int L)
{
    unsigned long long mx = 0;
    for (int l = 0; l < L; ++l) {
        const tasq_layer &t = layers[l];
        if (t.M <= 0 || t.N <= 0 || t.K <= 128)
            continue;
        const int s = auto_splits(t.M, t.N, t.K);
        if (s < 2)
            continue;
        int kchunk, splits;
        split_geometry(t.K, s, kchunk, splits);
        const unsigned long long need = 4ULL * splits * (unsigned long long)t.M * t.N;
        if (need < (1ULL << 31) && need > mx)
            mx = need;
    }
    return (size_t)mx;
}

// Room of a layer in the schedule's workspace, for its descriptor and a share
// of the unit lists.
constexpr size_t kLayerRoom = 1408;
static_assert(sizeof(LayerDesc) <= kLayerRoom && sizeof(LayerDesc) % 4 == 0);

constexpr size_t schedule_partials_offset(int L)
{
    return round_up((size_t)L * kLayerRoom, kWsAlign) + round_up((size_t)L * 64, kWsAlign);
}

// Estimated us of a layer cut into s ranges of K, fitted to 60 layers
// (convs of 8x8 to 64x96 pixels, linear layers of 65 to 4096 rows, K 8192..32768;
// most within 15%): rounds of the chip's workgroups, a range's nk K tiles each,
// and the partial outputs written and read again, 0.42 to 0.47 us per MB.  A
// linear layer's 128x128 tiles read its operands at 12 TB/s at best (a conv's
// taps find theirs again nearby).
double split_cost(int tile, long long M, long long N, int K, int s, bool conv)
{
    int kchunk, splits;
    split_geometry(K, s, kchunk, splits);
    const int b = tile == tasq::TILE_256x256_K128_W8_PF1 ? 256 : 128;
    const double tiles = (double)((M + b - 1) / b) * ((N + b - 1) / b);
    const double wgs = tiles * splits, nk = kchunk / 128, mb = 4e-6 * M * N * splits;
    if (b == 256)
        return std::ceil(wgs / kComputeUnits) * (6.0 + 1.5 * nk) + 0.42 * mb;
    const double rounds = wgs <= kComputeUnits
                              ? 5.8 + 0.67 * nk
                              : std::max(1.0, wgs / (2 * kComputeUnits)) * (2.0 + 1.1 * nk);
    const double reads = conv ? 0.0 : tiles * 256 * K / 12e6;
    return std::max(rounds, reads) + 0.47 * mb;
}

// Tile and ranges of a split layer, s >= 2 as the caller forces it, 0 = the
// library's choice among two: 128x128 tiles with as many ranges as fill the two
// workgroups per compute unit, or 256x256 tiles with as many as fill one, which
// the workspace is sized for.  The first has fewer workgroups per range to
// feed and fewer partials, the second reads its operands half as often.
// us, 128x128 / 256x256: 32x32 pixels 1280 -> 1280 32.5 (6 ranges) / 37.6 (10),
// 48x48 1280 -> 1280 62.6 (2) / 57.7 (5), 48x48 2560 -> 1280 110.8 / 90.0, 40x40
// 2560 -> 1280 80.3 (3) / 71.6 (7), 64x64 1280 -> 640 51.2 (3) / 57.3 (5), linear
// 1024x32768 -> 1024 59.5 (8) / 52.3 (16), 4096x32768 -> 1024 162.8 (2) / 136.2 (4).
struct SplitForm {
    int tile, s;
};

SplitForm pick_split(const tasq_opts *o, long long M, long long N, int K, int s, bool conv)
{
    const long long t128 = ((M + 127) / 128) * ((N + 127) / 128);
    const int most = s ? s : auto_splits(M, N, K);
    const int fill = s ? s : (int)std::min<long long>(std::max(2LL, 2LL * kComputeUnits / t128),
                                                      most);
    const SplitForm small = {tasq::TILE_128x128_K128_W4_PF2, fill};
    const SplitForm big = {tasq::TILE_256x256_K128_W8_PF1, most};
    if (const int f = forced_tile(o); f >= 0)
        return {f, fill};
    return split_cost(big.tile, M, N, K, big.s, conv) < split_cost(small.tile, M, N, K, small.s, conv)
               ? big
               : small;
}

// Tiles of the grouped per-step launch.
enum StepTile { STEP_256, STEP_128, STEP_64, STEP_64_2 };

// The tiles of the grouped step over linear layers, by an estimate in us of
// each form's time: the longest tile on its own, or all tiles' work spread
// over the chip and a share of the longest one for the uneven end.  nk is a
// layer's K tiles of 128 bytes; the constants are fitted to 45 steps of 1 to
// 20 blocks of the DiT shapes at 65 to 4096 tokens (most within 15%).
//   256x256 (persistent, lists): tiles of 8.5 + 1.6 nk, 256 at a time;
//   128x128: 4 + 1.15 nk, 512 at a time;
//   64x64: 1050 K tiles per us, each tile costing nk + 1;
//   64x64 with K shared by two wave groups: 28% less of them, half the chain.
// us per step, 256 / 128 / 64 / 64 in two groups:
//   1 PixArt block, 100 tokens 45 / 25.5 / 17.5 / 14.0
//   1 PixArt block, 700 tokens 48.5 / 32.0 / 25.9 / 32.3
//   2 PixArt blocks, 700 tokens 55.2 / 41.5 / 47.2 / 57.4
//   1 PixArt block, 2048 tokens 59 / 50 / 63 / 78
//   UNet block (conv apart) 79 / 82 / 115 / 136
//   1 SANA block, 1024 tokens 72 / 87 / 120 / 129
//   6 PixArt blocks, 1024 tokens 127 / 141 / 188 / 227
// The former rule, 256x256 unless one tile outweighed a compute unit's share
// of the step and 128x128 then, took 28 us on the first, 62 on the fourth, 99
// on the fifth and 91.6 on the sixth.
// Many tiles per compute unit leave no uneven end, and steps with a conv
// (which has no persistent form), forced tiles or a forced form keep to the
// former rule.
StepTile pick_step_tile(const tasq_opts *o, const std::vector<LayerDesc> &descs, bool any_conv)
{
    double total = 0, longest = 0, t256 = 0;
    for (const LayerDesc &d : descs) {
        total += 2.0 * d.M * (double)d.N * d.K;
        longest = std::max(longest, (double)d.K);
        t256 += (double)((d.M + 255) / 256) * ((d.N + 255) / 256);
    }
    if (any_conv || (o && o->persistent) || t256 > kStepCostMaxTiles)
        return 2.0 * 256 * 256 * longest > total / kComputeUnits ? STEP_128 : STEP_256;
    double w256 = 0, w128 = 0, w64 = 0;
    for (const LayerDesc &d : descs) {
        const double nk = (d.K + 127) / 128;
        auto tiles = [&](int b) {
            return (double)((d.M + b - 1) / b) * ((d.N + b - 1) / b);
        };
        w256 += tiles(256) * (8.5 + 1.6 * nk) / kComputeUnits;
        w128 += tiles(128) * (4.0 + 1.15 * nk) / (2 * kComputeUnits);
        w64 += tiles(64) * (1.0 + nk) / 1050.0;
    }
    const double nk = std::ceil(longest / 128);
    const double a256 = 6.0 + 1.15 * nk, a128 = 4.0 + 0.65 * nk;
    const double a64 = 3.0 + 0.48 * nk, a64_2 = 3.0 + 0.28 * nk;
    w256 *= 1.12;
    const double cost[] = {std::max(a256, w256) + 0.35 * std::min(a256, w256),
                           std::max(a128, w128 + 0.55 * a128), std::max(a64, w64 + 0.3 * a64),
                           std::max(a64_2, 1.28 * w64 + 0.3 * a64_2)};
    return (StepTile)(std::min_element(cost, cost + 4) - cost);
}

bool use_bitplane(const tasq_opts *o) { return o && o->variant == TASQ_VARIANT_BITPLANE; }

// The buffer-offset fast path also needs each input below 2 GiB.
bool fits_buffers(const LayerDesc &d)
{
    const long long xb = d.kind == tasq::KIND_CONV3X3 ? (long long)d.H * d.Wd * d.C
                                                       : (long long)d.M * d.K;
    return xb < (1LL << 31) && (long long)d.N * d.K < (1LL << 31);
}

// The packed buffer is addressed with 32-bit offsets.
bool packed_fits(const LayerDesc &d)
{
    return tasq::packed_weight_bytes_host(d.N, d.K) < (1ULL << 31);
}

// The planes are addressed with 32-bit offsets by the weight-streaming kernel.
bool planes_fit(const LayerDesc &d)
{
    return tasq::planes_bytes_host(d.N, d.K) < (1ULL << 31);
}

// Activation operand on the 16-byte buffer fast path.
bool x_aligned(const LayerDesc &d)
{
    const int inner = d.kind == tasq::KIND_CONV3X3 ? d.C : d.K;
    return inner % 16 == 0 && aligned16(d.X) && fits_buffers(d);
}

// A linear layer that the weight-streaming kernels take: few tokens and
// 16-byte activation rows.
bool skinny_shape(const LayerDesc &d)
{
    return d.kind == tasq::KIND_LINEAR && d.M <= tasq::kSkinnyMaxM && x_aligned(d);
}

// Which stored copy of the weight a layer reads.
enum WeightSrc { SRC_NONE = 0, SRC_ROWS, SRC_PACKED, SRC_PLANES };

// The variant names the copy; AUTO picks by shape from what is present.
// With few tokens the layer is a weight stream whose time follows the
// bytes read, so AUTO reads the top b planes there (App. G.2: only the
// surviving planes are fetched).  Measured on the 112-layer PixArt-shaped
// schedule (ms per denoising step, TASQ table of mean 4.94 bits / static
// b = 8): at M = 16 planes 0.058 / 0.093, packed int8 0.095 / 0.095, int8
// rows 0.108 / 0.101; at M = 32 planes 0.088 / 0.117, packed 0.111 / 0.111;
// at M = 64 planes 0.152 / 0.169, packed 0.181 / 0.181.  The plane stream
// wins at every b below 8; at b = 8 it reads as many bytes as the int8 copy
// and the two streams are within 7% of each other either way, so there AUTO
// keeps the packed copy when one is given.  For M in the
// thousands the weights are a few percent of the traffic and rebuilding the
// bytes from planes per output tile costs more than it saves, so AUTO takes
// the int8 copies, and the bit-plane GEMM only when no other copy is given.
// Between the two int8 copies (both given):
//   * a single layer takes the packed copy when it has more than one
//     256x256 tile per two compute units, the rows otherwise.  us of a call
//     in a row of calls (b = 5), rows / packed: 1024x1280 -> 3840 (60 tiles)
//     10.0 / 11.0, 1500x1152 -> 4608 (108) 13.0 / 13.9, 4096x640 -> 1920 (128)
//     11.1 / 11.6, 4096x2240 -> 2240 (144) 29.7 / 29.7, 8192x1152 -> 1152 (160)
//     20.2 / 18.3, 8192x1152 -> 3456 (448) 46.2 / 43.5, 8192x1152 -> 4608 (576)
//     66.6 / 54.9, 4096x2240 -> 11200 (704) 112.8 / 113.7, 16384x1152 -> 4608
//     (1152) 110.7 / 104.3.  The line leaves out some deep layers below it
//     (3000x5600 -> 2240, 108 tiles, 53.6 / 44.6) and the largest ones, where
//     the rows' walk is ahead by 1 to 5% (16384x2240 -> 6720, 1728 tiles, 257 /
//     269);
//   * on byte-aligned activations (a K that is no multiple of 16, an odd
//     address) a linear layer takes the packed copy, whose weights need no
//     shifts (rows / packed: 4942x861 -> 640 15.6 / 12.4, 4096x2241 -> 2240
//     48.1 / 39.1), and a conv the rows, because the packed K order lets a
//     chunk cross taps (20x30 1275 -> 1280: 65 against more than 1000);
//   * a schedule takes the rows, whose grouped step runs as the persistent
//     launch: 4.23 ms per denoising step of the 28-block PixArt-shaped
//     schedule against 4.59 ms for the grouped packed-weight launch.
// any_below8: the layer runs at some b below 8 (its b for a single call; any
// entry of its table row for a schedule).
WeightSrc weight_source(const LayerDesc &d, const tasq_opts *o, bool any_below8,
                        bool in_schedule)
{
    const bool rows = d.W != nullptr, packed = d.Wp != nullptr, planes = d.P != nullptr;
    switch (variant_of_opts(o)) {
    case TASQ_VARIANT_BITPLANE:
        return planes && d.kind == tasq::KIND_LINEAR ? SRC_PLANES : SRC_NONE;
    case TASQ_VARIANT_PACKED:
        return packed ? SRC_PACKED : SRC_NONE;
    case TASQ_VARIANT_MASKED_I8:
        return rows ? SRC_ROWS : SRC_NONE;
    default:
        break;
    }
    const bool linear = d.kind == tasq::KIND_LINEAR;
    if (planes && linear && skinny_shape(d) && planes_fit(d) && (any_below8 || !packed))
        return SRC_PLANES;
    if (packed && rows && !skinny_shape(d)) {
        if (in_schedule)
            return aligned16(d.W) ? SRC_ROWS : SRC_PACKED;
        if (!x_aligned(d))
            return linear ? SRC_PACKED : SRC_ROWS;
        const long long tiles = (long long)((d.M + 255) / 256) * ((d.N + 255) / 256);
        return tiles > kComputeUnits / 2 ? SRC_PACKED : SRC_ROWS;
    }
    if (packed)
        return SRC_PACKED;
    if (rows)
        return SRC_ROWS;
    if (planes && linear)
        return SRC_PLANES;
    return SRC_NONE;
}

// Weight-streaming path for skinny activations: linear layers with M <= 64
// and 16-byte activation rows, reading the weight copy `src`.  Returns false
// when that copy cannot be streamed.
bool skinny_source(const LayerDesc &d, WeightSrc src, tasq::SkinnyWeights &out)
{
    if (!skinny_shape(d))
        return false;
    switch (src) {
    case SRC_PLANES:
        out = tasq::SKINNY_PLANES;
        return planes_fit(d);
    case SRC_PACKED:
        out = tasq::SKINNY_PACKED;
        return packed_fits(d);
    case SRC_ROWS:
        out = tasq::SKINNY_ROWS;
        return aligned16(d.W);
    default:
        return false;
    }
}

int launch_layer(const LayerDesc &d, const tasq_opts *o, hipStream_t stream,
                 bool allow_split = false)
{
    if (d.M == 0 || d.N == 0)
        return TASQ_OK;
    hipError_t e;
    const WeightSrc wsrc = weight_source(d, o, d.bits < 8, false);
    tasq::SkinnyWeights src;
    if (skinny_source(d, wsrc, src)) {
        e = tasq::launch_skinny(d, src, stream);
        return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
    }
    if (wsrc == SRC_PACKED && packed_fits(d)) {
        e = tasq::packed_tile_ops(
                pick_packed_tile(o, d.M, d.N, d.K, d.kind == tasq::KIND_CONV3X3))
                .single(d, x_aligned(d), stream);
        return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
    }
    if (wsrc == SRC_PLANES) {
        e = tasq::tile_ops(tasq::TILE_64x64_K128_W4_PF2).planes(
            d, (d.K % 16) == 0 && aligned16(d.X) && fits_buffers(d), stream);
    } else {
        bool aligned;
        if (d.kind == tasq::KIND_CONV3X3)
            aligned = (d.C % 16) == 0 && aligned16(d.X) && aligned16(d.W);
        else
            aligned = (d.K % 16) == 0 && aligned16(d.X) && aligned16(d.W);
        aligned = aligned && fits_buffers(d);
        // Split-K: forced (split_k >= 2, needs the workspace) or chosen
        // (split_k == 0, only with a workspace of tasq_workspace_bytes).
        const int req = o ? o->split_k : 0;
        int splits = 1, kchunk = 0, split_tile = 0;
        if (allow_split && req != 1 && d.K > 128) {
            const unsigned long long room = o && o->workspace ? o->workspace_bytes : 0;
            int s = req;
            if (req == 0) {
                const size_t whole = tasq_workspace_bytes(d.M, d.N, d.K);
                s = whole && room >= whole ? 0 : 1;
            }
            if (s != 1) {
                const SplitForm form =
                    pick_split(o, d.M, d.N, d.K, s, d.kind == tasq::KIND_CONV3X3);
                split_tile = form.tile;
                split_geometry(d.K, form.s, kchunk, splits);
                const unsigned long long need = 4ULL * splits * (unsigned long long)d.M * d.N;
                const bool ws_ok = room >= need && need < (1ULL << 31);
                if (!ws_ok && req >= 2)
                    return TASQ_ERR_WORKSPACE;
                if (!ws_ok || !aligned)
                    splits = 1;
            }
        }
        if (splits > 1) {
            int32_t *part = static_cast<int32_t *>(o->workspace);
            e = tasq::tile_ops(split_tile).split(d, part, splits, kchunk, stream);
            if (e == hipSuccess)
                e = tasq::launch_split_finish(d, part, splits, stream);
        } else {
            const tasq::KGroupTile kg = pick_kgroups(o, d.M, d.N, d.K);
            const bool conv = d.kind == tasq::KIND_CONV3X3;
            e = kg != tasq::KG_NONE
                    ? tasq::launch_kgroups(d, kg, aligned, stream)
                    : tasq::tile_ops(pick_tile(o, d.M, d.N, d.K, aligned, conv,
                                               d.y && d.lr_T && d.lr_r > 16))
                          .single(d, aligned, stream);
        }
    }
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

LayerDesc make_desc(const tasq_layer &L, const tasq_opts *o)
{
    LayerDesc d;
    std::memset(&d, 0, sizeof d);
    d.X = L.X;
    d.W = L.W;
    d.P = L.W_planes ? L.W_planes : (o ? o->W_planes : nullptr);
    d.Wp = L.W_packed ? L.W_packed : (o ? o->W_packed : nullptr);
    d.act = L.act_params ? L.act_params : (o ? o->act_params : nullptr);
    d.colsums = L.colsums ? L.colsums : (o ? o->colsums : nullptr);
    d.wz = L.w_zero ? L.w_zero : (o ? o->w_zero : nullptr);
    d.xrs = L.w_zero ? L.x_rowsums : (o ? o->x_rowsums : nullptr);
    if (L.lowrank_T) {
        d.lr_T = L.lowrank_T;
        d.lr_U = L.lowrank_up;
        d.lr_r = L.lowrank_rank;
    } else if (o && o->lowrank_T) {
        d.lr_T = o->lowrank_T;
        d.lr_U = o->lowrank_up;
        d.lr_r = o->lowrank_rank;
    }
    d.sw = L.sw;
    d.bias = L.bias;
    d.acc = L.acc;
    d.y = L.y;
    d.sx = L.sx;
    d.M = L.M;
    d.N = L.N;
    d.K = L.K;
    d.kind = L.kind;
    d.H = L.H;
    d.Wd = L.Wd;
    d.C = L.C;
    return d;
}

// The layer has the weight copy its variant reads: the planes (BITPLANE),
// the packed buffer (PACKED), the rows (MASKED_I8), or under AUTO any copy
// that serves the layer kind (the planes serve linear layers only).  The
// named copy must be present even when the layer is empty.
int check_weights(const tasq_layer &L, const tasq_opts &o, bool needs_w)
{
    const int v = o.variant;
    if (v == TASQ_VARIANT_BITPLANE && !o.W_planes)
        return TASQ_ERR_LAYOUT;
    if (v == TASQ_VARIANT_PACKED && !o.W_packed)
        return TASQ_ERR_LAYOUT;
    if (!needs_w || v == TASQ_VARIANT_BITPLANE || v == TASQ_VARIANT_PACKED)
        return TASQ_OK;
    if (v == TASQ_VARIANT_MASKED_I8)
        return L.W ? TASQ_OK : TASQ_ERR_NULL;
    const bool planes_serve = o.W_planes && L.kind == TASQ_KIND_LINEAR;
    return L.W || o.W_packed || planes_serve ? TASQ_OK : TASQ_ERR_NULL;
}

// Validation shared by single calls and schedule layers.
int validate_layer(const tasq_layer &L, const tasq_opts *o)
{
    if (L.kind != TASQ_KIND_LINEAR && L.kind != TASQ_KIND_CONV3X3)
        return TASQ_ERR_KIND;
    // A pointer is required only where its array has elements.
    const bool has_out = L.M > 0 && L.N > 0;
    if (L.M > 0 && L.K > 0 && !L.X)
        return TASQ_ERR_NULL;
    if (has_out && !L.acc && !L.y)
        return TASQ_ERR_NULL;
    if (has_out && L.y && !L.sw)
        return TASQ_ERR_NULL;
    tasq_opts local = o ? *o : tasq_opts{};
    if (L.W_planes)
        local.W_planes = L.W_planes;
    if (L.W_packed)
        local.W_packed = L.W_packed;
    if (L.act_params)
        local.act_params = L.act_params;
    if (L.colsums)
        local.colsums = L.colsums;
    // Asymmetric activations need the channel sums for the zero point.
    if (has_out && L.y && local.act_params && !local.colsums)
        return TASQ_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(local.act_params) & 3) ||
        (reinterpret_cast<uintptr_t>(local.colsums) & 3))
        return TASQ_ERR_ALIGN;
    // Weight zero points: the layer's own fields, else the call's.
    if (L.w_zero) {
        local.w_zero = L.w_zero;
        local.x_rowsums = L.x_rowsums;
    }
    if (has_out && L.y && local.w_zero) {
        if (!local.x_rowsums)
            return TASQ_ERR_NULL;
        if ((reinterpret_cast<uintptr_t>(local.w_zero) & 3) ||
            (reinterpret_cast<uintptr_t>(local.x_rowsums) & 3))
            return TASQ_ERR_ALIGN;
        if (L.kind == TASQ_KIND_CONV3X3)
            return TASQ_ERR_LAYOUT;
    }
    // Low-rank branch: the layer's own fields, else the call's.
    if (L.lowrank_T) {
        local.lowrank_T = L.lowrank_T;
        local.lowrank_up = L.lowrank_up;
        local.lowrank_rank = L.lowrank_rank;
    }
    if (has_out && L.y && local.lowrank_T) {
        if (!local.lowrank_up)
            return TASQ_ERR_NULL;
        if (local.lowrank_rank != 16 && local.lowrank_rank != 32)
            return TASQ_ERR_DIM;
        if ((reinterpret_cast<uintptr_t>(local.lowrank_T) & 15) ||
            (reinterpret_cast<uintptr_t>(local.lowrank_up) & 15))
            return TASQ_ERR_ALIGN;
        if (L.kind == TASQ_KIND_CONV3X3)
            return TASQ_ERR_LAYOUT;
        // Staged through 32-bit buffer offsets, with a tile's rows past M.
        if (((long long)L.M + 256) * local.lowrank_rank * 4 >= (1LL << 31) ||
            ((long long)L.N + 256) * local.lowrank_rank * 2 >= (1LL << 31))
            return TASQ_ERR_DIM;
    }
    const bool needs_w = L.N > 0 && L.K > 0;
    if (int rc = check_variant(&local))
        return rc;
    if (int rc = check_weights(L, local, needs_w))
        return rc;
    if (L.kind == TASQ_KIND_CONV3X3) {
        if (L.H < 0 || L.Wd < 0 || L.C < 0 || L.N < 0)
            return TASQ_ERR_DIM;
        if ((long long)L.M != (long long)L.H * L.Wd || (long long)L.K != 9LL * L.C)
            return TASQ_ERR_DIM;
        if (use_bitplane(&local))
            return TASQ_ERR_LAYOUT;     // the bit-plane kernel covers linear layers
        // A padded tap holds code 0, which dequantises to alpha (128 - z), not
        // to zero: asymmetric codes would need a per-pixel zero-point term.
        if (local.act_params)
            return TASQ_ERR_LAYOUT;
    }
    if (int rc = check_dims(L.M, L.N, L.K))
        return rc;
    // Without the row-major copy the packed buffer must be addressable.
    if (local.W_packed && !L.W && !use_bitplane(&local) &&
        tasq::packed_weight_bytes_host(L.N, L.K) >= (1ULL << 31))
        return TASQ_ERR_DIM;
    // Outputs are written through 32-bit buffer offsets (see gemm_core.h).
    if (((long long)L.M + 256) * (long long)L.N * 4 >= (1LL << 31))
        return TASQ_ERR_DIM;
    return TASQ_OK;
}


// Device-side layer list and bit table of tasq_run_schedule_noalloc: one
// copy per GPU the library runs on, held until the process ends.  Host code
// never uses the name itself (a host-side stand-in, not a device address):
// static_scratch() looks the address up once per device with that device
// current, and only that pointer reaches kernels and copies.
constexpr size_t kStaticScratchBytes = schedule_partials_offset(TASQ_STATIC_MAX_LAYERS);
static_assert(kStaticScratchBytes == TASQ_STATIC_SCRATCH_BYTES,
              "TASQ_STATIC_SCRATCH_BYTES must match the layer-list layout");
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices];

// Device address of this stream's GPU's scratch array.
int static_scratch(hipStream_t stream, void **out)
{
    int cur = 0, dev = 0;
    if (hipGetDevice(&cur) != hipSuccess)
        return TASQ_ERR_HIP;
    dev = cur;
    if (stream && hipStreamGetDevice(stream, &dev) != hipSuccess)
        return TASQ_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices)
        return TASQ_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        if (dev != cur && hipSetDevice(dev) != hipSuccess)
            return TASQ_ERR_HIP;
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (dev != cur && hipSetDevice(cur) != hipSuccess)
            return TASQ_ERR_HIP;
        if (e != hipSuccess || !p)
            return TASQ_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TASQ_OK;
}

// Host bytes to device memory, stream-ordered: by value in the arguments of
// up to kUploadLaunches small launches, or as one copy; under capture always by
// value, because a captured copy reads its source again at every replay, when
// the host lists are gone.  A copy from pageable
// memory is staged by the runtime and costs the caller as much as several
// launches: 20 layers of a 16-token schedule, 4 steps, 22.6 us of host time
// against 28.6 with two copies; one layer, 1 step, 11.2 against 15.9.
constexpr size_t kUploadChunk = 3584;      // kernel arguments end at 4 KB
constexpr size_t kUploadLaunches = 2;

struct UploadChunk {
    uint4 v[kUploadChunk / 16];
};

__global__ void k_upload(uint4 *dst, int n, UploadChunk c)
{
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        dst[i] = c.v[i];
}

// dst 16-byte aligned, bytes a multiple of 16.
hipError_t upload(void *dst, const void *src, size_t bytes, hipStream_t stream)
{
    if (bytes > kUploadLaunches * kUploadChunk) {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipError_t e = hipStreamIsCapturing(stream, &capture))
            return e;
        if (capture == hipStreamCaptureStatusNone)
            return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, stream);
    }
    for (size_t off = 0; off < bytes; off += kUploadChunk) {
        const size_t n = std::min(bytes - off, kUploadChunk);
        UploadChunk c;
        std::memcpy(c.v, static_cast<const char *>(src) + off, n);
        hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, stream,
                           reinterpret_cast<uint4 *>(static_cast<char *>(dst) + off),
                           (int)(n / 16), c);
        if (hipError_t e = hipGetLastError())
            return e;
    }
    return hipSuccess;
}

}  // namespace

extern "C" {

const char *tasq_status_string(int status)
{
    switch (status) {
    case TASQ_OK: return "ok";
    case TASQ_ERR_NULL: return "required pointer is NULL or no output requested";
    case TASQ_ERR_DIM: return "bad dimension";
    case TASQ_ERR_BITS: return "effective bits outside [1, 8]";
    case TASQ_ERR_OVERFLOW: return "K too large for exact int32 accumulation";
    case TASQ_ERR_RANGE: return "bad stage/step range or count, or a buffer shared by two jobs";
    case TASQ_ERR_LAYOUT: return "requested variant needs a weight layout that is absent";
    case TASQ_ERR_WORKSPACE:
        return "workspace missing or too small (noalloc schedule: more layers than its scratch holds)";
    case TASQ_ERR_HIP: return "HIP runtime or launch failure";
    case TASQ_ERR_KIND: return "unknown layer kind or variant";
    case TASQ_ERR_ALIGN: return "workspace not 256-byte aligned or packed weight not 16-byte aligned";
    default: return "unknown status";
    }
}

int tasq_stage_of_step(int t, int S, int T)
{
    if (S < 1 || T < 1 || S > T || t < 0 || t >= T)
        return TASQ_ERR_RANGE;
    return (int)(((long long)t * S) / T);
}

size_t tasq_planes_bytes(int N, int K)
{
    return (size_t)tasq::planes_bytes_host(N, K);
}

size_t tasq_workspace_bytes(int M, int N, int K)
{
    if (M <= 0 || N <= 0 || K <= 128)
        return 0;
    const int s = auto_splits(M, N, K);
    if (s < 2)
        return 0;
    int kchunk, splits;
    split_geometry(K, s, kchunk, splits);
    const unsigned long long need = 4ULL * splits * (unsigned long long)M * N;
    return need < (1ULL << 31) ? (size_t)need : 0;
}

int tasq_masked_linear(const int8_t *X, const int8_t *W, float sx, const float *sw,
                       const float *bias, int M, int N, int K, int b, int32_t *acc_out,
                       float *y_out, const tasq_opts *opts, void *stream)
{
    tasq_layer L;
    std::memset(&L, 0, sizeof L);
    L.kind = TASQ_KIND_LINEAR;
    L.M = M;
    L.N = N;
    L.K = K;
    L.sx = sx;
    L.X = X;
    L.W = W;
    L.sw = sw;
    L.bias = bias;
    L.acc = acc_out;
    L.y = y_out;
    if (int rc = check_tuning(opts))
        return rc;
    if (int rc = validate_layer(L, opts))
        return rc;
    if (b < 1 || b > 8)
        return TASQ_ERR_BITS;
    LayerDesc d = make_desc(L, opts);
    d.bits = b;
    return launch_layer(d, opts, static_cast<hipStream_t>(stream), true);
}

int tasq_masked_conv3x3(const int8_t *X, const int8_t *W, float sx, const float *sw,
                        const float *bias, int H, int Wd, int C, int N, int b,
                        int32_t *acc_out, float *y_out, const tasq_opts *opts, void *stream)
{
    if (H < 0 || Wd < 0 || C < 0 || N < 0)
        return TASQ_ERR_DIM;
    const long long M = (long long)H * Wd, K = 9LL * C;
    if (M > 0x7fffffffLL)
        return TASQ_ERR_DIM;
    if (K > TASQ_MAX_K)
        return TASQ_ERR_OVERFLOW;
    tasq_layer L;
    std::memset(&L, 0, sizeof L);
    L.kind = TASQ_KIND_CONV3X3;
    L.M = (int)M;
    L.N = N;
    L.K = (int)K;
    L.H = H;
    L.Wd = Wd;
    L.C = C;
    L.sx = sx;
    L.X = X;
    L.W = W;
    L.sw = sw;
    L.bias = bias;
    L.acc = acc_out;
    L.y = y_out;
    if (int rc = check_tuning(opts))
        return rc;
    if (int rc = validate_layer(L, opts))
        return rc;
    if (b < 1 || b > 8)
        return TASQ_ERR_BITS;
    LayerDesc d = make_desc(L, opts);
    d.bits = b;
    return launch_layer(d, opts, static_cast<hipStream_t>(stream), true);
}

int tasq_pack_planes(const int8_t *W, int N, int K, uint32_t *planes_out, void *stream)
{
    if (!W || !planes_out)
        return TASQ_ERR_NULL;
    if (N < 0 || K < 0)
        return TASQ_ERR_DIM;
    if (N == 0 || K == 0)
        return TASQ_OK;
    hipError_t e = tasq::launch_pack_planes(W, N, K, planes_out, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

int tasq_pack_weights(const int8_t *W, int N, int K, int8_t *packed_out, void *stream)
{
    if (N < 0 || K < 0)
        return TASQ_ERR_DIM;
    if (K > TASQ_MAX_K)
        return TASQ_ERR_OVERFLOW;
    if (N == 0 || K == 0)
        return TASQ_OK;
    if (!W || !packed_out)
        return TASQ_ERR_NULL;
    if (!aligned16(packed_out))
        return TASQ_ERR_ALIGN;
    hipError_t e = tasq::launch_pack_weights(W, N, K, packed_out, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

int tasq_quantize_activations(const float *x, int M, int K, int8_t *X_out, float *act_params,
                              void *stream)
{
    if (M < 0 || K < 0)
        return TASQ_ERR_DIM;
    const long long n = (long long)M * K;
    if (n == 0)
        return TASQ_OK;
    if (!x || !X_out || !act_params)
        return TASQ_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(x) & 3) || (reinterpret_cast<uintptr_t>(act_params) & 3))
        return TASQ_ERR_ALIGN;
    hipError_t e = tasq::launch_quantize_activations(x, n, X_out, act_params,
                                                     static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

// The lists of a batch are std::vectors: running out of host memory is returned
// as TASQ_ERR_HIP, not thrown across the C ABI (here and in
// tasq_quantize_weights_batch).
int tasq_quantize_activations_batch(const tasq_act_job *jobs, int n, void *stream)
try {
    if (n < 0)
        return TASQ_ERR_RANGE;
    if (n == 0)
        return TASQ_OK;
    if (!jobs)
        return TASQ_ERR_NULL;
    std::vector<tasq::ActJob> js;
    std::vector<const float *> bufs;
    js.reserve((size_t)n);
    bufs.reserve((size_t)n);
    for (int j = 0; j < n; ++j) {
        const tasq_act_job &a = jobs[j];
        if (a.M < 0 || a.K < 0)
            return TASQ_ERR_DIM;
        if ((long long)a.M * a.K == 0)
            continue;
        if (!a.x || !a.X_out || !a.act_params)
            return TASQ_ERR_NULL;
        if ((reinterpret_cast<uintptr_t>(a.x) & 3) || (reinterpret_cast<uintptr_t>(a.act_params) & 3))
            return TASQ_ERR_ALIGN;
        js.push_back({a.x, a.M, a.K, a.X_out, a.act_params});
        bufs.push_back(a.act_params);
    }
    std::sort(bufs.begin(), bufs.end());
    if (std::adjacent_find(bufs.begin(), bufs.end()) != bufs.end())
        return TASQ_ERR_RANGE;
    hipError_t e = tasq::launch_quantize_activations_batch(js.data(), (int)js.size(),
                                                           static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
} catch (const std::bad_alloc &) {
    return TASQ_ERR_HIP;
}

int tasq_quantize_weights(const float *W, int N, int K, int8_t *W_out, float *alpha_out,
                          float *z_out, float *sw_out, void *stream)
{
    if (N < 0 || K < 0 || (N > 0 && K == 0))
        return TASQ_ERR_DIM;
    if (K > TASQ_MAX_K)
        return TASQ_ERR_OVERFLOW;
    if (N == 0)
        return TASQ_OK;
    if (!W || !W_out || !alpha_out || !z_out || !sw_out)
        return TASQ_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(W) & 3) || (reinterpret_cast<uintptr_t>(alpha_out) & 3) ||
        (reinterpret_cast<uintptr_t>(z_out) & 3) || (reinterpret_cast<uintptr_t>(sw_out) & 3))
        return TASQ_ERR_ALIGN;
    hipError_t e = tasq::launch_quantize_weights(W, N, K, W_out, alpha_out, z_out, sw_out,
                                                 static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

int tasq_row_sums(const int8_t *X, int M, int K, int32_t *out, void *stream)
{
    if (M < 0 || K < 0)
        return TASQ_ERR_DIM;
    if (K > TASQ_MAX_K)
        return TASQ_ERR_OVERFLOW;
    if (M == 0)
        return TASQ_OK;
    if (!out || (K > 0 && !X))
        return TASQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(out) & 3)
        return TASQ_ERR_ALIGN;
    hipError_t e = tasq::launch_row_sums(X, M, K, out, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

static int check_lowrank_down(const float *x, int M, int K, const uint16_t *down, int r,
                              const float *T_out)
{
    if (M < 0 || K < 0 || (r != 16 && r != 32))
        return TASQ_ERR_DIM;
    if ((long long)M * r * 4 >= (1LL << 31) || K > (1 << 30) / 32)
        return TASQ_ERR_DIM;
    if (M == 0)
        return TASQ_OK;
    if (!T_out || (K > 0 && (!x || !down)))
        return TASQ_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(x) & 3) || (reinterpret_cast<uintptr_t>(down) & 1) ||
        (reinterpret_cast<uintptr_t>(T_out) & 3))
        return TASQ_ERR_ALIGN;
    return TASQ_OK;
}

int tasq_lowrank_down(const float *x, int M, int K, const uint16_t *down, int r, float *T_out,
                      void *stream)
{
    if (int rc = check_lowrank_down(x, M, K, down, r, T_out))
        return rc;
    if (M == 0)
        return TASQ_OK;
    hipError_t e = tasq::launch_lowrank_down(x, M, K, down, r, T_out, nullptr, nullptr,
                                             static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

int tasq_quantize_activations_lowrank(const float *x, int M, int K, int8_t *X_out,
                                      float *act_params, const uint16_t *down, int r,
                                      float *T_out, void *stream)
{
    if (int rc = check_lowrank_down(x, M, K, down, r, T_out))
        return rc;
    if (M == 0)
        return TASQ_OK;
    if (K == 0) {       // no codes to write; the projection is zero
        hipError_t e = tasq::launch_lowrank_down(x, M, K, down, r, T_out, nullptr, nullptr,
                                                 static_cast<hipStream_t>(stream));
        return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
    }
    if (!X_out || !act_params)
        return TASQ_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(act_params) & 3)
        return TASQ_ERR_ALIGN;
    hipError_t e = tasq::launch_quantize_activations_lowrank(
        x, M, K, X_out, act_params, down, r, T_out, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

int tasq_weight_colsums(const int8_t *W, int N, int K, int32_t *colsums_out, void *stream)
{
    if (N < 0 || K < 0)
        return TASQ_ERR_DIM;
    if (K > TASQ_MAX_K)
        return TASQ_ERR_OVERFLOW;
    if (N == 0)
        return TASQ_OK;
    if (!colsums_out || (K > 0 && !W))
        return TASQ_ERR_NULL;
    hipError_t e = tasq::launch_weight_colsums(W, N, K, colsums_out,
                                               static_cast<hipStream_t>(stream));
    return e == hipSuccess ? TASQ_OK : TASQ_ERR_HIP;
}

size_t tasq_packed_weight_bytes(int N, int K)
{
    return (size_t)tasq::packed_weight_bytes_host(N, K);
}

size_t tasq_schedule_workspace_bytes(const tasq_layer *layers, int L)
{
    if (L <= 0)
        return 0;
    return schedule_partials_offset(L) + (layers ? round_up(max_split_bytes(layers, L), kWsAlign)
                                                 : 0);
}

// step_events[i] (caller-created hipEvent_t), when the caller asked for them.
static int record_step_event(const tasq_opts *o, int i, hipStream_t st)
{
    if (!o || !o->step_events)
        return TASQ_OK;
    return hipEventRecord(static_cast<hipEvent_t>(o->step_events[i]), st) == hipSuccess
               ? TASQ_OK
               : TASQ_ERR_HIP;
}

// static_ws: the per-device scratch array (tasq_run_schedule_noalloc) in
// place of the caller's workspace; it holds the layer list and the table
// only, so layers that a workspace schedule would split-K run unsplit.
static int run_schedule_impl(const tasq_layer *layers, int L, const uint8_t *b_table, int S,
                             int T, int t_begin, int t_end, const tasq_opts *opts, void *stream,
                             bool use_static)
{
    if (L < 0)
        return TASQ_ERR_RANGE;
    if (L > 0 && (!layers || !b_table))
        return TASQ_ERR_NULL;
    if (S < 1 || T < 1 || S > T || t_begin < 0 || t_begin > t_end || t_end > T)
        return TASQ_ERR_RANGE;
    if (S > 64)
        return TASQ_ERR_RANGE;
    if (opts && opts->workspace && (reinterpret_cast<uintptr_t>(opts->workspace) % kWsAlign))
        return TASQ_ERR_ALIGN;
    if (int rc = check_tuning(opts))
        return rc;
    for (int l = 0; l < L; ++l) {
        if (int rc = validate_layer(layers[l], opts))
            return rc;
        for (int s = 0; s < S; ++s) {
            const int b = b_table[(size_t)l * S + s];
            if (b < 1 || b > 8)
                return TASQ_ERR_BITS;
        }
    }
    if (use_static && L > TASQ_STATIC_MAX_LAYERS)
        return TASQ_ERR_WORKSPACE;
    if (L == 0 || t_begin == t_end)
        return TASQ_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    void *static_ws = nullptr;
    if (use_static) {
        if (int rc = static_scratch(st, &static_ws))
            return rc;
    }

    std::vector<LayerDesc> descs(L);
    for (int l = 0; l < L; ++l)
        descs[l] = make_desc(layers[l], opts);

    // Grouped path: one launch per step over every layer's tiles, with the
    // layer list and bit table resident in the caller's workspace.
    // Grouped launches need the workspace for the device-side layer list.
    // Three kinds, each over every layer's work units in one launch per step:
    //  - weight streaming, when every layer is skinny (M <= 64) with the same
    //    weight source: one unit per 32 output channels;
    //  - packed-weight GEMM, when every layer has a packed weight;
    //  - staged GEMM, when every layer has its aligned row-major weight.
    // Otherwise each layer is launched on its own.
    const size_t need = use_static ? schedule_partials_offset(L)
                                   : tasq_schedule_workspace_bytes(layers, L);
    char *const ws = use_static ? static_cast<char *>(static_ws)
                                : static_cast<char *>(opts ? opts->workspace : nullptr);
    const size_t ws_bytes = use_static ? kStaticScratchBytes : (opts ? opts->workspace_bytes : 0);
    const bool have_ws = ws && ws_bytes >= need;
    // The weight copy each layer reads (AUTO: by shape, see weight_source),
    // with "some b below 8" taken over the stages the steps touch.
    const int s_first = tasq_stage_of_step(t_begin, S, T);
    const int s_last = tasq_stage_of_step(t_end - 1, S, T);
    std::vector<WeightSrc> wsrc(L);
    for (int l = 0; l < L; ++l) {
        bool below8 = false;
        for (int s = s_first; s <= s_last; ++s)
            below8 = below8 || b_table[(size_t)l * S + s] < 8;
        wsrc[l] = weight_source(descs[l], opts, below8, true);
    }
    // Only layers with a product to compute (M, N and K all positive) take
    // part in a grouped launch and decide its form; a layer with outputs
    // but K = 0 writes its bias (or zero) through the single-layer launcher
    // each step, and a layer without outputs has nothing to do.
    auto multiplies = [](const LayerDesc &d) { return d.M > 0 && d.N > 0 && d.K > 0; };
    // AUTO names each layer's best copy on its own, which can differ from
    // layer to layer (a layer at b = 8 in every stage takes the packed copy,
    // the others the planes).  One launch per step reads one kind, and
    // beats a launch per layer by far more than the copies differ (112
    // layers at 16 tokens, one stage: 0.06 ms per step against 0.53): the
    // first kind that every layer has, in AUTO's order.
    if (have_ws && variant_of_opts(opts) == TASQ_VARIANT_AUTO) {
        bool mixed = false, streams = true;
        WeightSrc first = SRC_NONE;
        for (int l = 0; l < L; ++l) {
            if (!multiplies(descs[l]))
                continue;
            streams = streams && skinny_shape(descs[l]);
            mixed = mixed || (first != SRC_NONE && wsrc[l] != first);
            first = first == SRC_NONE ? wsrc[l] : first;
        }
        if (mixed && streams) {
            for (const WeightSrc c : {SRC_PLANES, SRC_PACKED, SRC_ROWS}) {
                bool every = true;
                for (int l = 0; l < L; ++l) {
                    const LayerDesc &d = descs[l];
                    const void *copy = c == SRC_PLANES ? (const void *)d.P
                                       : c == SRC_PACKED ? (const void *)d.Wp
                                                         : (const void *)d.W;
                    tasq::SkinnyWeights sl;
                    every = every && (!multiplies(d) || (copy && skinny_source(d, c, sl)));
                }
                if (every) {
                    std::fill(wsrc.begin(), wsrc.end(), c);
                    break;
                }
            }
        }
    }
    tasq::SkinnyWeights src = tasq::SKINNY_ROWS;
    bool all_skinny = have_ws;
    bool seen = false;
    int max_m = 0;
    for (int l = 0; all_skinny && l < L; ++l) {
        if (!multiplies(descs[l]))
            continue;
        tasq::SkinnyWeights sl;
        all_skinny = skinny_source(descs[l], wsrc[l], sl) && (!seen || sl == src);
        src = sl;
        seen = true;
        max_m = descs[l].M > max_m ? descs[l].M : max_m;
    }
    bool all_packed = true;
    for (int l = 0; l < L; ++l)
        all_packed = all_packed && (!multiplies(descs[l]) ||
                                    (wsrc[l] == SRC_PACKED && packed_fits(descs[l])));
    const int v = variant_of_opts(opts);
    bool grouped = have_ws && v != TASQ_VARIANT_BITPLANE;
    for (int l = 0; grouped && l < L; ++l) {
        const LayerDesc &d = descs[l];
        if (!multiplies(d))
            continue;
        const bool staged = v != TASQ_VARIANT_PACKED && wsrc[l] != SRC_PLANES && d.W &&
                            aligned16(d.W);
        grouped = x_aligned(d) && (all_packed || staged);
    }
    if (all_skinny || grouped) {
        for (int l = 0; l < L; ++l)
            descs[l].layer = l;
        // A layer whose one 256x256 tile costs more than a compute unit's
        // even share of the step, and that split-K can cut (a long K on few
        // tiles: the 3x3 conv of the UNet block), is launched on its own
        // each step, split-K over the partials room of the workspace, ahead
        // of the grouped launch over the other layers; inside the grouped
        // launch its tiles would set the step time and force small tiles on
        // every layer (SDXL-Turbo-shaped block: 174.5 us per step grouped,
        // 99.1 + 39.1 us split this way).
        std::vector<LayerDesc> solo;
        {
            std::vector<LayerDesc> rest;
            for (const LayerDesc &d : descs) {
                if (multiplies(d))
                    rest.push_back(d);
                else if (d.M > 0 && d.N > 0)
                    solo.push_back(d);
            }
            descs.swap(rest);
        }
        if (!all_skinny && !all_packed) {
            double ops = 0;
            for (const LayerDesc &d : descs)
                ops += 2.0 * d.M * (double)d.N * d.K;
            std::vector<LayerDesc> rest, split;
            for (const LayerDesc &d : descs) {
                const bool long_tile = 2.0 * 256 * 256 * (double)d.K > ops / kComputeUnits;
                if (long_tile && auto_splits(d.M, d.N, d.K) > 1)
                    split.push_back(d);
                else
                    rest.push_back(d);
            }
            if (!rest.empty() && !split.empty()) {
                descs.swap(rest);
                solo.insert(solo.end(), split.begin(), split.end());
            }
        }
        // Weight streaming: the workgroups of the deepest layers first.  A
        // workgroup streams all of its layer's K, so the 4608-deep layers'
        // workgroups run four times as long as the 1152-deep ones; launched
        // last (in layer order) they leave the end of the step to a few
        // compute units (28-block PixArt-shaped step at 16 tokens, planes:
        // 0.0581 ms ordered by K, 0.0638 ms in layer order).
        if (all_skinny)
            std::stable_sort(descs.begin(), descs.end(),
                             [](const LayerDesc &x, const LayerDesc &y) { return x.K > y.K; });
        const int LG = (int)descs.size();
        bool any_conv = false;
        for (int l = 0; l < LG; ++l)
            any_conv = any_conv || descs[l].kind == tasq::KIND_CONV3X3;
        tasq::TileShape ts = {32, 32, 128};
        hipError_t (*launch_step)(const LayerDesc *, int, int, const uint8_t *, int, int, bool,
                                  bool, hipStream_t) = nullptr;
        hipError_t (*launch_persistent)(const LayerDesc *, int, int, const tasq::XcdRuns &,
                                        const uint8_t *, int, int, int, int,
                                        hipStream_t) = nullptr;
        hipError_t (*launch_lists)(const LayerDesc *, int, const uint16_t *, const uint8_t *, int,
                                   int, hipStream_t) = nullptr;
        bool persistent_pays = false;     // chosen as a persistent launch by cost
        bool big_tile = false;      // the 256x256 tile, which AUTO runs persistent
        bool extras = false;
        for (int l = 0; l < LG; ++l)
            extras = extras || descs[l].lr_T != nullptr || descs[l].wz != nullptr;
        if (all_skinny) {
            // one unit per 32 output channels, all tokens
            ts = {tasq::kSkinnyMaxM, 32, 128};
        } else if (all_packed) {
            const int ptile = pick_packed_grouped_tile(opts);
            const tasq::PackedTileOps &ops = tasq::packed_tile_ops(ptile);
            ts = ops.shape;
            launch_step = ops.grouped;
            if (!any_conv && !extras)
                launch_persistent = ops.persistent;
            big_tile = ptile == tasq::PTILE_256x256_K128_W8;
        } else {
            const int f = forced_tile(opts);
            const StepTile step = f >= 0 ? STEP_256 : pick_step_tile(opts, descs, any_conv);
            constexpr int tile_of[] = {tasq::TILE_256x256_K128_W8_PF1,
                                       tasq::TILE_128x128_K128_W4_PF2,
                                       tasq::TILE_64x64_K128_W4_PF2,
                                       tasq::TILE_64x64_K128_W4_PF2};
            const int tile = f >= 0 ? f : tile_of[step];
            const tasq::TileOps &ops = tasq::tile_ops(tile);
            ts = ops.shape;
            launch_step = step == STEP_64_2 ? tasq::launch_kgroups_2x64 : ops.grouped;
            if (!any_conv) {
                launch_persistent = extras ? ops.persistent_extras : ops.persistent;
                launch_lists = extras ? ops.lists_extras : ops.lists;
            }
            big_tile = tile == tasq::TILE_256x256_K128_W8_PF1;
            persistent_pays = f < 0 && !any_conv && step == STEP_256 && !(opts && opts->persistent);
        }
        // The one-workgroup-per-tile launches run the deepest layers first too,
        // so that no deep tile starts when the others are done (us per step of
        // one block in 128x128 tiles, layer order / by K: 1024 tokens 41.9 /
        // 35.1, 2048 64.7 / 49.9).
        const bool persistent_step =
            launch_persistent && (persistent_pays ||
                                  use_persistent(opts, big_tile, grouped_tiles(descs, ts)));
        if (!all_skinny && !persistent_step)
            std::stable_sort(descs.begin(), descs.end(),
                             [](const LayerDesc &x, const LayerDesc &y) { return x.K > y.K; });
        long long total = 0;
        for (int l = 0; l < LG; ++l) {
            LayerDesc &d = descs[l];
            d.tiles_m = (d.M + ts.bm - 1) / ts.bm;
            d.tiles_n = (d.N + ts.bn - 1) / ts.bn;
            d.tile_begin = (int)total;
            total += (long long)d.tiles_m * d.tiles_n;
            if (total > 0x7fffffffLL)
                return TASQ_ERR_DIM;
        }
        if (total == 0 && solo.empty())
            return TASQ_OK;
        if (!persistent_step)
            launch_persistent = nullptr;
        const int wgs_per_xcd = persistent_wgs_per_xcd(opts);
        const int parties = persistent_parties(opts, wgs_per_xcd);
        // The GEMM kernels give each XCD one contiguous run of the work
        // units (for L2 locality): the persistent launch runs of about equal
        // cost (cost_runs), the one-workgroup-per-tile launches runs equal in
        // count.  For the latter, when the layers' tiles differ in cost (K)
        // and the layer order leaves one run much heavier than the others,
        // every XCD takes an eighth of every layer instead (grouped_unit;
        // measured slower than contiguous runs for the persistent step: 4.27
        // against 4.15 ms).
        const bool rounds = !all_skinny && !launch_persistent &&
                            xcd_imbalance(descs, total) > kImbalanceLimit;
        const tasq::XcdRuns runs = cost_runs(descs, total);
        // The persistent step over lists of units where they spare the
        // busiest workgroup enough of its work, and where they fit the part
        // of the layer list's room that the descriptors leave unused.
        const size_t desc_bytes = (size_t)LG * sizeof(LayerDesc);
        const size_t order_at = round_up(desc_bytes + (size_t)L * S, 16);
        std::vector<uint16_t> order;
        if (!launch_persistent || total > kListMaxUnits ||
            (opts && (opts->persistent_wgs || opts->persistent_parties)))
            launch_lists = nullptr;
        if (launch_lists) {
            if (unit_lists(descs, order) > kListGain * runs_makespan(descs, runs) ||
                order_at + 2 * order.size() > schedule_partials_offset(L)) {
                order.clear();
                launch_lists = nullptr;
            }
        }
        // The descriptors, the table, then the lists, in one block of the
        // workspace.
        std::vector<uint8_t> block(order_at + round_up(2 * order.size(), 16), 0);
        std::memcpy(block.data(), descs.data(), desc_bytes);
        std::memcpy(block.data() + desc_bytes, b_table, (size_t)L * S);
        if (!order.empty())
            std::memcpy(block.data() + order_at, order.data(), 2 * order.size());
        LayerDesc *d_descs = reinterpret_cast<LayerDesc *>(ws);
        uint8_t *d_table = reinterpret_cast<uint8_t *>(ws) + desc_bytes;
        const uint16_t *d_order = reinterpret_cast<uint16_t *>(ws + order_at);
        if (upload(ws, block.data(), block.size(), st) != hipSuccess)
            return TASQ_ERR_HIP;
        // Schedules ignore split_k: a layer launched on its own takes the
        // automatic split over the partials room, which
        // tasq_schedule_workspace_bytes reserved for it.
        tasq_opts sopts = opts ? *opts : tasq_opts{};
        sopts.split_k = 0;
        sopts.step_events = nullptr;
        sopts.workspace = use_static ? nullptr : ws + schedule_partials_offset(L);
        sopts.workspace_bytes = use_static ? 0 : ws_bytes - schedule_partials_offset(L);
        for (int t = t_begin; t < t_end; ++t) {
            const int s = tasq_stage_of_step(t, S, T);
            if (int rc = record_step_event(opts, 2 * (t - t_begin), st))
                return rc;
            for (LayerDesc d : solo) {
                d.bits = b_table[(size_t)d.layer * S + s];
                if (int rc = launch_layer(d, &sopts, st, true))
                    return rc;
            }
            if (total == 0) {
                if (int rc = record_step_event(opts, 2 * (t - t_begin) + 1, st))
                    return rc;
                continue;
            }
            const hipError_t e =
                all_skinny ? tasq::launch_skinny_grouped(d_descs, LG, (int)total, max_m, src,
                                                         d_table, S, s, st)
                : launch_lists ? launch_lists(d_descs, LG, d_order, d_table, S, s, st)
                : launch_persistent
                    ? launch_persistent(d_descs, LG, (int)total, runs, d_table, S, s,
                                        wgs_per_xcd, parties, st)
                    : launch_step(d_descs, LG, (int)total, d_table, S, s, any_conv,
                                  rounds, st);
            if (e != hipSuccess)
                return TASQ_ERR_HIP;
            if (int rc = record_step_event(opts, 2 * (t - t_begin) + 1, st))
                return rc;
        }
        return TASQ_OK;
    }

    for (int t = t_begin; t < t_end; ++t) {
        const int s = tasq_stage_of_step(t, S, T);
        if (int rc = record_step_event(opts, 2 * (t - t_begin), st))
            return rc;
        for (int l = 0; l < L; ++l) {
            descs[l].bits = b_table[(size_t)l * S + s];
            if (int rc = launch_layer(descs[l], opts, st))
                return rc;
        }
        if (int rc = record_step_event(opts, 2 * (t - t_begin) + 1, st))
            return rc;
    }
    return TASQ_OK;
}

// The host-side lists (layer descriptors, unit lists, the table copy) are
// std::vectors: running out of host memory is returned as TASQ_ERR_HIP, not
// thrown across the C ABI.
int tasq_run_schedule(const tasq_layer *layers, int L, const uint8_t *b_table, int S, int T,
                      int t_begin, int t_end, const tasq_opts *opts, void *stream)
{
    try {
        return run_schedule_impl(layers, L, b_table, S, T, t_begin, t_end, opts, stream, false);
    } catch (const std::bad_alloc &) {
        return TASQ_ERR_HIP;
    }
}

int tasq_run_schedule_noalloc(const tasq_layer *layers, int L, const uint8_t *b_table, int S,
                              int T, int t_begin, int t_end, const tasq_opts *opts, void *stream)
{
    try {
        return run_schedule_impl(layers, L, b_table, S, T, t_begin, t_end, opts, stream, true);
    } catch (const std::bad_alloc &) {
        return TASQ_ERR_HIP;
    }
}

}  // extern "C"
