// Arithmetic shared by the matrix-core kernels and their launchers that depends on sizes only: plain C++, so that it can be
// checked on a CPU at sizes no test would allocate.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

#if defined(__HIPCC__)
#define MOC_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MOC_HOST_DEVICE inline
#endif

namespace moc {

// Offset of the last readable k row of a slice of `bk` rows in a k-major operand, `left` >= 1 rows before the end of the
// contraction: the k-row offsets of a slice are clamped to it.  The rows are clamped before the product is formed: left * ld does not
// fit 32 bits for contractions over a few hundred thousand tokens, bk * ld does (checked on the host).
MOC_HOST_DEVICE int last_row_offset(int left, int bk, int ld) { return ((left < bk ? left : bk) - 1) * ld; }

constexpr int kMfmaBK = 32;      // k-slice of the bf16 kernel

// Tile shapes of the bf16 matrix-core kernel and what a launch of each costs, in microseconds: `o` once per round of
// tiles (launch, first loads, epilogue), `lo` .. `hi` per 32-k slice with few .. all compute units busy (the chip is
// power-limited with the large tiles, so a full round runs slower), `co` per slice and workgroup where several
// workgroups share a compute unit (`resident` of them; 1 = one persistent workgroup per compute unit).
// Measured with 64 .. 768 tiles at contractions of 768, 2048 and 5472; the three operand layouts agree within 5 %.  Longer contractions are
// underestimated: 2047 x 2048 over 2 * 5464 on 128 x 128 tiles takes 126 us, the formula says 100 (over 5464: 68, 53).
struct GemmTile {
    int bm, bn, sets, resident;      // sets: k-slices in flight in registers
    double o, lo, hi, co;
};
constexpr int kGemmTiles = 8;
constexpr GemmTile kGemmTile[kGemmTiles] = {
    {256, 256, 3, 1, 12.0, 0.592, 0.851, 0.0}, {256, 192, 3, 1, 11.5, 0.457, 0.680, 0.0}, {192, 256, 3, 1, 11.0, 0.457, 0.668, 0.0},
    {256, 128, 3, 1, 9.0, 0.373, 0.484, 0.0},  {128, 192, 3, 1, 7.0, 0.283, 0.378, 0.0},  {192, 128, 3, 1, 7.0, 0.290, 0.385, 0.0},
    {128, 128, 3, 3, 5.7, 0.222, 0.275, 0.275}, {64, 128, 5, 4, 4.7, 0.216, 0.225, 0.200}};
// The same for products over the channels (down, dX) with 1.4 M results or rows of 2048 and 8 MB of weights or more, which do not stay in a
// cache until they are read: measured with operands from memory, 32 to 6000 rows, d 512 to 4096.  The table above, measured with warm
// operands, made such products up to 1.8 times as long as the best choice (2047 x 2048 over 2 * 5464 121 us against 80, 1024 x 4096 over 10928 121
// against 80), this one 1.01 times on average (502 products of 40 to 2600 rows; three of them 1.02 to 1.03 times what the table above takes).  Below 8 MB the warm table holds: 4096 x 768 over 2 * 2048, cold 46 us whole and 40 in shares, runs
// in 40 and 42 inside a training step.
constexpr GemmTile kGemmTileLong[kGemmTiles] = {
    {256, 256, 3, 1, 12.0, 0.595, 0.850, 0.0}, {256, 192, 3, 1, 11.5, 0.510, 0.673, 0.0}, {192, 256, 3, 1, 11.0, 0.457, 0.668, 0.0},
    {256, 128, 3, 1, 9.0, 0.373, 0.484, 0.0},  {128, 192, 3, 1, 7.0, 0.299, 0.475, 0.0},  {192, 128, 3, 1, 8.0, 0.330, 0.381, 0.0},
    {128, 128, 3, 3, 5.5, 0.241, 0.308, 0.297}, {64, 128, 5, 4, 4.9, 0.214, 0.257, 0.211}};
// The lines: with this table / with the warm one, whole forward or backward, weights from memory, d 640 to 1536.  By results: 14 to 20 << 16 0.90 to 1.06, mean
// 1.00 over 48 layers; 21 to 31 << 16 0.85 to 1.05, mean 0.94.  By bytes: 5 to 8 MB forward 0.99 to 1.01; backward 0.86 to 0.99 from 1700 to 3600 rows of 768 x
// 2048, 1.02 and 1.03 at 4096 and 5000.
inline bool long_product(int M, int N, int Kc, int Kc2) {
    return 2 * ((int64_t)Kc + Kc2) * N >= 8000000 && (N >= 2048 || (int64_t)M * N >= 21 << 16);
}
// every shape; 256x256, 256x192, 128x128; and 256x128, 64x128; 192x128, 128x128, 64x128
constexpr unsigned kTilesAll = 0xFF, kTilesBasic = 0x43, kTilesGroup = 0xCB, kTilesShares = 0xE0;
// With a k-major B, the large tiles of gemm_pingpong.h take every product that 192x256 or 256x128 would be chosen for but those of operands
// past 4 GiB, which 256x256 and 256x192 serve as well (and which MOC_GEMM_TILE names): not built.
constexpr unsigned kTilesKm = kTilesAll & ~0x0Cu, kTilesKmGroup = kTilesGroup & ~0x0Cu;
constexpr int kTile128 = 6;

inline int64_t tile_count(int M, int N, const GemmTile& t) {
    return (int64_t)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
}
inline int slice_count(int Kc, int Kc2) { return (Kc + kMfmaBK - 1) / kMfmaBK + (Kc2 + kMfmaBK - 1) / kMfmaBK; }

inline double gemm_cost(const GemmTile& t, int64_t tiles, int nk, int cus) {
    const int64_t n = tiles % cus;
    const double f = std::max(0.0, ((double)n / cus - 0.25) / 0.75);
    const double partial = n ? t.o + nk * (t.lo + (t.hi - t.lo) * f * f) : 0.0;      // a round that leaves compute units idle
    if (t.resident == 1 || tiles <= cus) return (double)(tiles / cus) * (t.o + nk * t.hi) + partial;
    const double w = 0.6 * tiles / cus + 0.4 * ((tiles + cus - 1) / cus);             // workgroups on the busiest compute unit, softened
    return 1.5 + t.o * ((tiles + (int64_t)cus * t.resident - 1) / ((int64_t)cus * t.resident)) + nk * t.co * w;
}

// The cheapest of the tile shapes in `mask` (the one named by `forced` if that is not negative); tiles_of(tile) counts the tiles of
// the launch.
template <class TilesOf>
int cheapest_tile(unsigned mask, const TilesOf& tiles_of, int nk, int cus, int forced = -1, double* cost_out = nullptr, const GemmTile* table = kGemmTile) {
    int best = -1;
    double best_cost = 0.0;
    for (int c = 0; c < kGemmTiles; ++c) {
        if (!((mask >> c) & 1u) || (forced >= 0 && c != forced)) continue;
        const double cost = gemm_cost(table[c], tiles_of(table[c]), nk, cus);
        if (best < 0 || cost < best_cost) { best = c; best_cost = cost; }
    }
    if (cost_out) *cost_out = best_cost;
    return best;
}

// Shares of a split contraction (run_gemm_shares): tile -1 where the whole product, of `whole_cost`, is not dearer.  The shares' way
// through memory, written and read once at about 4 TB/s, and the second launch are counted.
struct SharePlan {
    int tile, shares;
};
// (long products, see kGemmTileLong: as measured together with the products, the last-level cache holds the shares)
inline double shares_traffic_cost(int64_t out, int shares, int elem, bool lng) {
    return lng ? 3.3 + (8.0 * shares + elem) * out / 11.5e6 : 3.5 + (8.0 * shares + elem) * out / 4.0e6;
}
inline SharePlan plan_shares(int M, int N, int nk, int elem, size_t scratch_bytes, int cus, double whole_cost, double* cost_out, bool lng) {
    const GemmTile* table = lng ? kGemmTileLong : kGemmTile;
    const int64_t out = (int64_t)M * N;
    SharePlan best{-1, 0};
    double best_cost = (lng ? 1.0 : 0.95) * whole_cost;
    for (int c = 0; c < kGemmTiles; ++c) {
        if (!((kTilesShares >> c) & 1u)) continue;
        // A single row of tiles reads every weight once, from memory, and one workgroup to a compute unit has too little of them under way: 192 x 128 in
        // eight shares against what is chosen now, whole call of 129 to 192 rows: dX 2048 x 8192 93.5 .. 104.8 -> 85.4 .. 92.0 us, 2560 x 6826 106.8 .. 114.5
        // -> 103.0 .. 109.0, 3072 x 8192 131.5 .. 145.8 -> 127.8 .. 138.9, down 2560 x 6826 64.6 .. 71.5 -> 60.6 .. 66.7, the others 0.97 to 1.00.
        if (lng && table[c].resident == 1 && M <= table[c].bm) continue;
        for (int z = 2; z <= 8 && nk / z >= 8 && (size_t)z * out * sizeof(float) <= scratch_bytes; ++z) {
            const double cost = gemm_cost(table[c], z * tile_count(M, N, table[c]), (nk + z - 1) / z, cus) + shares_traffic_cost(out, z, elem, lng);
            if (cost < best_cost) { best = SharePlan{c, z}; best_cost = cost; }
        }
    }
    if (cost_out && best.tile >= 0) *cost_out = best_cost;
    return best;
}

// The large tiles of gemm_pingpong.h and their cost in microseconds: kPpLaunch once, `o` per round of tiles, `lo` .. `hi` per 64-k slice
// with few .. all compute units busy.  Measured with 64 .. 704 tiles at contractions of 512, 2048 and 8192; the operand layouts agree
// within 5 %, the formula with the measurements within 6 %.
constexpr int kPpBK = 64;
// The library's dense operands [rows, F] are laid out in rows of a multiple of this and are zero from column F on, so that contractions
// over the columns may run to the end of the last slice of any kernel (GemmProblem::a_zero_padded).
constexpr int kColPad = 64;
static_assert(kColPad % kMfmaBK == 0 && kColPad % kPpBK == 0, "whole slices");
struct PpTile {
    int bm, bn;
    double o, lo, hi;
};
constexpr int kPpTiles = 5;
constexpr double kPpLaunch = 6.8;
constexpr PpTile kPpTile[kPpTiles] = {
    {256, 256, 3.2, 1.04, 1.37}, {192, 256, 1.8, 0.84, 1.05}, {256, 192, 2.0, 0.86, 1.07}, {128, 256, 1.4, 0.69, 0.79}, {256, 128, 1.4, 0.68, 0.78}};

constexpr PpTile kPpTileLong[kPpTiles] = {      // see kGemmTileLong
    {256, 256, 3.2, 1.01, 1.26}, {192, 256, 2.0, 0.87, 1.02}, {256, 192, 2.0, 0.97, 1.13}, {128, 256, 1.4, 0.71, 0.82}, {256, 128, 1.3, 0.72, 0.84}};

// A product as the kernel of gemm_pingpong.h sees it: leading dimensions, layouts (km: k-major) and zero padding of the operands as in
// GemmProblem, and its result: columns stored, row pitch, distance of the shares of a split contraction, bytes of an element.
struct PpSizes {
    int M, N, Kc, Kc2;
    int64_t lda, ldb;
    bool akm, bkm, a_zero_padded;
    int64_t out_n, ldc, stride;
    int elem;
};
// Whether sizes let the kernel take it: contraction ends that the range check or A's zeros cover; byte offsets within an operand in 32 bits,
// to the end of the last tile (256 rows or columns) and slice; whole 16-byte pieces of output rows.
inline bool pp_sizes_ok(const PpSizes& s) {
    const auto whole = [](int k) { return k % kPpBK == 0; };
    // both k-contiguous: the slice past the end would be the next rows' values
    if (!s.akm && !s.bkm && !(whole(s.Kc) && whole(s.Kc2))) return false;
    const int longest = std::max(s.Kc, s.Kc2);
    if (!s.akm && s.bkm && !(whole(s.Kc) && whole(s.Kc2)) &&
        !(s.a_zero_padded && s.lda >= ((int64_t)longest + kColPad - 1) / kColPad * kColPad)) return false;
    if (s.akm && (!s.bkm || s.Kc2 != 0)) return false;      // (the kernel has one count of A's readable bytes, which with k-major rows depends on the contraction)
    const int64_t k = (int64_t)longest + 2 * kPpBK, lim = (1ll << 32) - 65536;
    const auto bytes = [&](bool km, int rows, int64_t ld) { return ((km ? k : (int64_t)rows + 256) * ld + 256 + k) * 2; };
    if (bytes(s.akm, s.M, s.lda) >= lim || bytes(s.bkm, s.N, s.ldb) >= lim) return false;
    return s.out_n * s.elem % 16 == 0 && s.ldc * s.elem % 16 == 0 && s.stride * s.elem % 16 == 0 && 256 * s.ldc * s.elem < (1ll << 31);
}

// Weight gradients of experts: rows of tiles in a band where an XCD takes `tiles` neighbouring tiles of a problem, the height at which these touch the
// fewest operand panels, which come from beyond its L2 (four tiles: a 2 x 2 block instead of a column, see pp_owners).  Four at most: with
// eight, which the count prefers by 6 % for 29 tiles of 192 x 256, three experts of 2048 x 5461 take 155 us instead of 147.
inline int pp_band_height(int bm, int bn, int tiles) {
    int best = 1;
    for (int h = 2; h <= 4; h *= 2)
        if (h * bm + tiles * bn / h < best * bm + tiles * bn / best) best = h;
    return best;
}
// Problems (in the order of their contraction lengths, `slices` to a tile, all of as many tiles) to whole XCDs of `width` workgroups, the longest
// first to the XCD with the least work; false, and owner[] untouched, where the busiest workgroup has over 3 % more to do than with an eighth of
// every problem on every XCD.  Eight experts of 768 x 2048 with 2000 to 6000 rows (24 weight gradients of 32 tiles): an eighth of each means
// panels of eight problems a round from beyond every L2, 5 TB/s of them: 310 us in bands of four tile rows, 296 in bands of two, 277 whole.
// The backward of six experts of 512 x 1376 (18 problems on eight XCDs), 2048 to 32768 rows: 0.93 to 0.98 of the time with eighths; of four (12 problems)
// 0.97 to 0.99 from 16384 rows on, 0.97 to 1.03 below.
inline bool pp_owners(int n, const int* slices, const int* tiles, int width, int* owner) {
    constexpr int kMost = 24, kWidth = 64;
    if (n < 8 || n > kMost || width > kWidth || tiles[0] > 4 * width) return false;
    for (int z = 1; z < n; ++z)
        if (tiles[z] != tiles[0]) return false;
    int to[kMost];
    int64_t load[8] = {};
    for (int z = 0; z < n; ++z) {
        to[z] = (int)(std::min_element(load, load + 8) - load);
        load[to[z]] += slices[z] + 2;      // (two slices' time to write a tile)
    }
    // the busiest workgroup, dealt as the kernel does: every second round backwards
    const auto busiest = [&](bool whole) {
        int64_t most = 0;
        for (int x = 0; x < 8; ++x) {
            int64_t wg[kWidth] = {};
            int at = 0;
            for (int z = 0; z < n; ++z) {
                const int count = !whole ? tiles[z] * (x + 1) / 8 - tiles[z] * x / 8 : to[z] == x ? tiles[z] : 0;
                for (int i = 0; i < count; ++i, ++at) wg[(at / width) & 1 ? width - 1 - at % width : at % width] += slices[z] + 2;
            }
            for (int i = 0; i < width; ++i) most = std::max(most, wg[i]);
        }
        return most;
    };
    if (100 * busiest(true) > 103 * busiest(false)) return false;
    std::copy(to, to + n, owner);
    return true;
}
inline int64_t tile_count(int M, int N, const PpTile& t) { return (int64_t)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }
inline int pp_slice_count(int Kc, int Kc2) { return (Kc + kPpBK - 1) / kPpBK + (Kc2 + kPpBK - 1) / kPpBK; }
inline double pp_cost(const PpTile& t, int64_t tiles, int nk, int cus) {
    const int64_t n = tiles % cus;
    const double f = std::max(0.0, ((double)n / cus - 0.25) / 0.75);
    return kPpLaunch + (double)(tiles / cus) * (t.o + nk * t.hi) + (n ? t.o + nk * (t.lo + (t.hi - t.lo) * f * f) : 0.0);
}
template <class TilesOf> int cheapest_pp_tile(const TilesOf& tiles_of, int nk, int cus, double* cost_out, const PpTile* table = kPpTile) {
    int best = 0;
    for (int c = 0; c < kPpTiles; ++c) {
        const double cost = pp_cost(table[c], tiles_of(table[c]), nk, cus);
        if (c == 0 || cost < *cost_out) { best = c; *cost_out = cost; }
    }
    return best;
}
// As plan_shares, for the large tiles; at least four slices to a share.
inline SharePlan plan_pp_shares(int M, int N, int nk, int elem, size_t scratch_bytes, int cus, double whole_cost, double* cost_out, bool lng) {
    const PpTile* table = lng ? kPpTileLong : kPpTile;
    const int64_t out = (int64_t)M * N;
    SharePlan best{-1, 0};
    double best_cost = (lng ? 1.0 : 0.95) * whole_cost;
    for (int c = 0; c < kPpTiles; ++c)
        for (int z = 2; z <= 16 && nk / z >= 4 && (size_t)z * out * sizeof(float) <= scratch_bytes; ++z) {
            const double cost = pp_cost(table[c], z * tile_count(M, N, table[c]), (nk + z - 1) / z, cus) + shares_traffic_cost(out, z, elem, lng);
            if (cost < best_cost) { best = SharePlan{c, z}; best_cost = cost; }
        }
    if (best.tile >= 0) *cost_out = best_cost;
    return best;
}

// Memory that a workspace holds for the shares of down (Kc2 = 0) or dX, bf16; what else is free at that time counts towards it.  Eight shares, or as
// many as the contraction has groups of eight slices for (plan_shares), up to what the routes use over d 64 .. 8192, F d/2 .. 8 d and 16 to 12000
// tokens with as much as they like: 12 MB (down) and 21 MB (dX) below the line of long_product, 64 MB (a round of 256 x 256 tiles) above it, where
// the weight gradients' last rows take up to 72 MB.  Grows with the tokens for a layer, so that a workspace for many serves fewer.
inline size_t share_scratch_wanted(int T, int d, int Kc, int Kc2) {
    const int most = std::min(8, slice_count(Kc, Kc2) / 8);
    const size_t cap = long_product(T, d, Kc, Kc2) ? (Kc2 ? 72 : 64) : (Kc2 ? 21 : 12);
    return most < 2 ? 0 : std::min((size_t)most * T * d * sizeof(float), cap << 20);
}

// How a product runs: whole on a tile of gemm_mfma.h (`mask`; `forced` see cheapest_tile) or, with pp, of gemm_pingpong.h, or, with scratch
// for it, with every tile's k-slices cut into shares that run as workgroups of their own and are summed afterwards.  The cheapest
// by the cost models.
struct GemmRoute {
    bool pp = false;
    int tile = 0, shares = 1;
};
inline GemmRoute gemm_route(unsigned mask, int M, int N, int Kc, int Kc2, int elem, bool pp, size_t scratch_bytes, int cus, int forced = -1) {
    const int nk = slice_count(Kc, Kc2), nk64 = pp_slice_count(Kc, Kc2);
    const bool lng = scratch_bytes && long_product(M, N, Kc, Kc2);
    GemmRoute r;
    double cost = 0.0;
    r.tile = cheapest_tile(mask, [&](const GemmTile& t) { return tile_count(M, N, t); }, nk, cus, forced, &cost, lng ? kGemmTileLong : kGemmTile);
    if (scratch_bytes) {
        const SharePlan p = plan_shares(M, N, nk, elem, scratch_bytes, cus, cost, &cost, lng);
        if (p.tile >= 0) r = GemmRoute{false, p.tile, p.shares};
    }
    if (!pp) return r;
    double pp_whole = 0.0;
    const int t = cheapest_pp_tile([&](const PpTile& p) { return tile_count(M, N, p); }, nk64, cus, &pp_whole, lng ? kPpTileLong : kPpTile);
    if (pp_whole < cost) {
        r = GemmRoute{true, t, 1};
        cost = pp_whole;
    }
    if (scratch_bytes) {
        const SharePlan p = plan_pp_shares(M, N, nk64, elem, scratch_bytes, cus, cost, &cost, lng);
        if (p.tile >= 0) r = GemmRoute{true, p.tile, p.shares};
    }
    return r;
}
// The same for several products in one launch, `tiles_of(tile)` tiles altogether; never in shares.
template <class TilesOf, class PpTilesOf>
GemmRoute group_route(unsigned mask, const TilesOf& tiles_of, const PpTilesOf& pp_tiles_of, int nk, int nk64, bool pp, int cus, int forced, double* cost) {
    GemmRoute r;
    r.tile = cheapest_tile(mask, tiles_of, nk, cus, forced, cost);
    if (!pp) return r;
    double pp_cost = 0.0;
    const int t = cheapest_pp_tile(pp_tiles_of, nk64, cus, &pp_cost);
    if (pp_cost < *cost) {
        r = GemmRoute{true, t, 1};
        *cost = pp_cost;
    }
    return r;
}

// Two products of one shape, both operands k-contiguous: in one launch where the two together cost less than apart, which they do unless both
// fill whole rounds of tiles.
struct PairRoute {
    bool together;
    GemmRoute route;      // of the one launch
};
inline PairRoute pair_route(int M, int N, int Kc, bool pp, int cus, int forced = -1) {
    double cost = 0.0, single = 0.0;
    PairRoute r;
    r.route = group_route(kTilesAll, [&](const GemmTile& t) { return 2 * tile_count(M, N, t); }, [&](const PpTile& t) { return 2 * tile_count(M, N, t); },
                          slice_count(Kc, 0), pp_slice_count(Kc, 0), pp, cus, forced, &cost);
    (void)cheapest_tile(kTilesAll, [&](const GemmTile& t) { return tile_count(M, N, t); }, slice_count(Kc, 0), cus, forced, &single);
    r.together = cost < 2.0 * single;
    return r;
}
// Three products of one shape, k-major, in one launch.
inline GemmRoute batch3_route(int M, int N, int Kc, bool pp, int cus, int forced = -1) {
    double cost = 0.0;
    return group_route(kTilesKm, [&](const GemmTile& t) { return 3 * tile_count(M, N, t); }, [&](const PpTile& t) { return 3 * tile_count(M, N, t); },
                       slice_count(Kc, 0), pp_slice_count(Kc, 0), pp, cus, forced, &cost);
}
// Weight gradients of many tokens whose tiles fill whole rounds and a little of another: the first `rows` rows, whole rounds, in one launch on
// tile `main`, the others in a second one on tile `rest` with their contraction in shares, summed by a third.  rows = 0 where that is not cheaper
// than the one launch of batch3_route.  The costs are those of k-major operands from memory (the same shapes and formula as kPpTile).
// The layer step of 8192 tokens, 2048 x 5461 (504 tiles in two rounds, then 85 rows in ten shares): 1393 -> 1325 us.
constexpr PpTile kPpTileWeights[kPpTiles] = {
    {256, 256, 3.2, 1.09, 1.40}, {192, 256, 1.8, 1.04, 1.27}, {256, 192, 2.0, 1.02, 1.19}, {128, 256, 1.4, 0.80, 0.85}, {256, 128, 1.4, 0.80, 0.85}};
struct Batch3Split {
    int rows = 0, main = 0, rest = 0, shares = 0;
};
// What the second and third launch cost beside what the tables say, from the step with and without them at d 768 to 4096 and 500 to 8192 tokens: where the
// tables promise 4 to 9.2 us, it was 4 us longer to 1 shorter (1536 x 4096, 1900 to 2400 tokens, 2048 x 5461, 1500 to 1984), where 9.8 to 16, 0 to 4 shorter
// (2048 x 5461, 2047 to 2400), 35, 13 to 20, 51, 35 shorter.  So 9.5 us are taken off.
constexpr double kBatch3Extra = 9.5;
inline Batch3Split batch3_split(int M, int N, int Kc, const GemmRoute& whole, size_t scratch_bytes, int cus) {
    const int nk = pp_slice_count(Kc, 0);
    Batch3Split best;
    if (!whole.pp || N % 4 != 0) return best;
    double cost = pp_cost(kPpTileWeights[whole.tile], 3 * tile_count(M, N, kPpTileWeights[whole.tile]), nk, cus) - kBatch3Extra;
    for (int c = 0; c < kPpTiles; ++c) {
        const PpTile& t = kPpTileWeights[c];
        const int tiles_n = (N + t.bn - 1) / t.bn, strips = (M + t.bm - 1) / t.bm;
        for (int r = 1; r <= 8; ++r) {
            const int full = r * cus / (3 * tiles_n);      // strips of tile rows that r rounds hold
            if (full < 1 || full >= strips) continue;
            const int rows = full * t.bm, left = M - rows;
            const double main = pp_cost(t, (int64_t)3 * full * tiles_n, nk, cus);
            if (main + kPpLaunch >= cost) break;
            for (int q : {0, 3})
                for (int z = 2; z <= 16 && nk / z >= 4 && (size_t)3 * z * left * N * sizeof(float) <= scratch_bytes; ++z) {
                    const double c2 = main + pp_cost(kPpTileWeights[q], (int64_t)3 * z * tile_count(left, N, kPpTileWeights[q]), (nk + z - 1) / z, cus) +
                                      shares_traffic_cost((int64_t)3 * left * N, z, 2, true);
                    if (c2 < cost) {
                        best = Batch3Split{rows, c, q, z};
                        cost = c2;
                    }
                }
        }
    }
    return best;
}
// Products of M[z] x N with contractions Kc[z], Kc2[z] (experts) in one launch; those without rows count for nothing.
inline GemmRoute grouped_route(unsigned mask, int n, const int* M, int N, const int* Kc, const int* Kc2, bool pp, int cus, int forced, double* cost) {
    int64_t rows = 0, slices = 0, slices64 = 0;
    for (int z = 0; z < n; ++z) {
        if (M[z] == 0) continue;
        rows += M[z];
        slices += (int64_t)M[z] * slice_count(Kc[z], Kc2[z]);
        slices64 += (int64_t)M[z] * pp_slice_count(Kc[z], Kc2[z]);
    }
    if (rows == 0) return GemmRoute{};
    const auto tiles_of = [&](const auto& t) {
        int64_t tiles = 0;
        for (int z = 0; z < n; ++z) tiles += tile_count(M[z], N, t);
        return tiles;
    };
    return group_route(mask, tiles_of, tiles_of, (int)(slices / rows), (int)(slices64 / rows), pp, cus, forced, cost);
}
// Two products per expert with the same contraction in one launch on large tiles: the tile, or -1 where two launches are not dearer.
inline int grouped_pair_tile(int n, const int* M, int N, int Kc, int cus, int forced = -1) {
    const auto tiles_of = [&](const auto& t) {
        int64_t tiles = 0;
        for (int z = 0; z < n; ++z) tiles += tile_count(M[z], N, t);
        return tiles;
    };
    double single = 0.0, both = 0.0;
    (void)group_route(kTilesGroup, tiles_of, tiles_of, slice_count(Kc, 0), pp_slice_count(Kc, 0), true, cus, forced, &single);
    const int t = cheapest_pp_tile([&](const PpTile& p) { return 2 * tiles_of(p); }, pp_slice_count(Kc, 0), cus, &both);
    return both < 2.0 * single ? t : -1;
}

// The streamed gate of bf16 decode (decode_gate_stream_kernel), whose workgroups have ceil(F / workgroups) rows each, in blocks of 16.
//
// Non-temporal loads where the layers of a model do not stay in the 256 MB last-level cache until the next token: from 24 MB of W_gate on for
// certain (twelve matrices, four layers), with the hint / without, whole call: weights from memory 34 MB 0.93 to 0.98, 67 MB and more 0.85 to 0.97;
// three layers in turn 34 MB 0.97 to 1.06, more as above.  Between 12 and 24 MB what three layers in turn lose weighs against what a
// model's weights win: d > 2048 1.00 to 1.03 and 0.96 to 0.97, shorter rows 1.01 to 1.06 and 0.95 to 0.99.  Below: 1.00 to 1.07 and 0.96 to 1.02.
inline bool gate_stream_nontemporal(int d, int F) { return 2ll * d * F >= (d > 2048 ? 12000000 : 24000000); }
// From five tokens on it takes 0.44 to 0.93 of the dot products' time (d 512 .. 4096, F d/4 .. 8 d).  For two to four tokens, against one row
// (grouped: one group) to a wavefront (workgroup), weights from memory, d 512 .. 4096, F 512 .. 12288, mean over two, three and four:
//   row-wide: 0.89 to 1.02 with the hint.  Otherwise a compute unit's share of W_gate is requested at once by either kernel, and the dot products
//     are as fast or faster (d > 1024: 0.98 to 1.10) except where their sums over a wavefront weigh most, in short rows: d <= 1024
//     0.95 to 1.03 from five rows a workgroup on, below 1.01 to 1.04.
//   grouped: 0.87 to 0.98 where a workgroup has one block of rows (up to 2048 x 4096: 1.01); with part of a second one 0.97 to 1.04 for
//     d <= 1024 and d > 2048, 1.00 to 1.08 in between.
inline bool gate_stream_pays(int B, int d, int F, bool grouped, int workgroups) {
    if (B < 2) return false;
    if (B > 4) return true;
    const int rows = (F + workgroups - 1) / workgroups;
    if (grouped) return d <= 1024 || d > 2048 || rows <= 16;
    return gate_stream_nontemporal(d, F) || (d <= 1024 && rows >= 5);
}

// bf16 decode with both projections as streams (decode_dense.h) instead of gathers, by what the gathers would request of a matrix, B K / F
// times its rows.  Whole call, this / gather, weights from memory:
//   row-wide, 5 to 16 tokens, at 1.2 times: d 1024 to 2048 and 4096 0.88 to 1.00, where 1.0 times is 0.94 to 1.06.  Between 2048 and 4096 the down projection
//     has eight ranges of channels and so leaves an eighth to a half of the compute units idle, which costs the more the more tokens a gathered row serves:
//     at 1.2 times 2560 x 6816 1.02 (5 tokens) to 1.08 (16), 3072 x 8192 0.96 to 1.07, 3584 x 9552 0.90 to 1.02; on the line drawn for them (2560: 1.38 to
//     1.88 times, 3072: 1.34 to 1.64) 0.92 to 1.01.
//     Long columns (F > 4 d), whose values every slice reads: 1.2 times 0.93 to 1.08, 1.6 times 0.85 to 0.99, 2 times 0.78 to 0.93.
//     Fewer tokens, whose gathers repeat less: 2 times 0.93 to 1.08, 4 times 0.73 to 0.86.
//   grouped, where no selection runs beside it: 2.5 times 0.94 to 1.05, 3.25 times 0.60 to 0.98.
//   layers below 12 MB a matrix, where the launches weigh: 512 x 1376 to 1024 x 2752 3.2 times 1.01 to 1.02, 6 times 0.88 to 0.99; wide rows (2560
//     x 640) gain nothing.
constexpr int kDownNarrowMaxD = 2048;      // up to here the down projection takes slices of 64 columns, above of 128
inline bool decode_dense_pays(int B, int d, int F, int K, bool grouped) {
    const int64_t requested = (int64_t)B * K, bytes = 2ll * d * F;
    if (bytes < 12000000) return B > 4 && d <= 2048 && requested >= 6ll * F;
    if (B <= 4) return !grouped && bytes >= 24000000 && requested >= 3ll * F;
    if (grouped) return requested >= 3ll * F;
    if (F > 4 * d) return requested >= 2ll * F;
    const int idle = d > kDownNarrowMaxD ? 32 - (d + 127) / 128 : 0;      // of 32 slices, eight compute units each
    return 1440 * requested >= (int64_t)(1728 + 5 * idle * B) * F;        // 1.2 times, and 1/288 more for every token and idle slice
}

// Channel shares per token in the gather stage of decode: shares x tokens fills the 256 CUs once (one
// 512-thread workgroup per CU), and a multiple of 8 shares lets the kernel keep each share on one XCD.
inline int decode_splits(int B, int K) {
    const int by_batch = std::max(8, 256 / B / 8 * 8);
    const int by_k = (K + 7) / 8;
    return std::max(1, std::min(by_batch, by_k));
}
// Ranges of channels of the streamed down projection: as many workgroups as the device has compute units, at least a step of 32 channels for every
// wavefront, no more than the workspace has partial outputs for; whole eights, so that a range stays on one XCD (1536 x 4096 23.0 us with 8
// ranges, 24.0 with the 10 that fill the chip).
inline int down_stream_ranges(int B, int d, int F, int K, int workgroups) {
    const int cols = d <= kDownNarrowMaxD ? 64 : 128, slices = (d + cols - 1) / cols;
    const int P = std::min({std::max(1, workgroups / slices), (F + 127) / 128, decode_splits(B, K)});
    return P > 8 ? P / 8 * 8 : P;
}

// fp32 tile shapes of gemm_f32.h: 64 x 64 once that gives every compute unit a workgroup (a wavefront then feeds four MFMAs from four
// fragment reads); below that 32 x 32, with the k-slices split over the wavefronts (16 x 32 or 32 x 32) when the contraction is long
// (several 128-k slices) or the tiles are still fewer than the compute units.  `one_sum` asks for one sum in one order of k (the gate
// product, so that the selection does not depend on the tile choice).
enum class F32Tile { k64x64, k32x32, k32x32Split, k16x32Split };
inline F32Tile f32_tile(int M, int N, int batch, int64_t contraction, bool one_sum, int cus) {
    const int64_t t64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64) * batch, t32 = (int64_t)((M + 31) / 32) * ((N + 31) / 32) * batch;
    if (t64 >= cus) return F32Tile::k64x64;
    if (one_sum || (t32 >= cus && contraction <= 1024)) return F32Tile::k32x32;
    return t32 < cus ? F32Tile::k16x32Split : F32Tile::k32x32Split;
}
// Cost in microseconds of a launch of `tiles` 32 x 32 tiles (k-slices of 64, three workgroups to a compute unit) or 16 x 32 tiles whose slices
// of 128 are split over the wavefronts (two), `slices` to a tile: workgroups of one compute unit share its matrix cores and hide each other's
// latency.  Measured at 64 to 1024 rows, d 512 and 768, contractions of 1376 to 4096; within 10 %.
inline double f32_cost(bool k32, int64_t tiles, int slices, int cus) {
    const int64_t w = (tiles + cus - 1) / cus, most = k32 ? 3 : 2, rest = w % most;
    const auto round = [&](int64_t n) { return k32 ? 3.0 + slices * (0.25 + 0.3 * n) : 2.7 + slices * (0.32 + 0.34 * n); };
    return (w / most) * round(most) + (rest ? round(rest) : 0.0);
}
// Contraction in shares that run as workgroups of their own and are summed by a second launch (3.2 us and the shares' way through memory); shares
// = 1 where that is not cheaper than whole tiles.  A result is the sum of no fewer partial sums than before: the split tiles add four, a share of
// a 32 x 32 tile has two, of which three shares are asked for.  us, the tiles of f32_tile / the shares chosen here: 64 x 768 over 4096 21.9 / 13.3,
// 256 x 512 over 2752 16.5 / 15.4, 256 x 768 over 2048 and 4096 19.5 / 16.8 and 33.2 / 24.4, 512 x 768 35.5 / 26.8 and 64.8 / 42.9.
struct F32Shares {
    F32Tile tile;
    int shares;
};
inline F32Shares f32_shares(int M, int N, int Kc, int Kc2, size_t scratch_bytes, int cus) {
    const F32Tile whole = f32_tile(M, N, 1, (int64_t)Kc + Kc2, false, cus);
    F32Shares best{whole, 1};
    if (whole != F32Tile::k16x32Split && whole != F32Tile::k32x32Split) return best;
    const int64_t n32 = (int64_t)((M + 31) / 32) * ((N + 31) / 32), n16 = (int64_t)((M + 15) / 16) * ((N + 31) / 32), out = (int64_t)M * N;
    const int s32 = (Kc + 63) / 64 + (Kc2 + 63) / 64, s16 = (Kc + 127) / 128 + (Kc2 + 127) / 128;
    // (32 x 32 split tiles: one workgroup per compute unit)
    double cost = 0.97 * (whole == F32Tile::k16x32Split ? f32_cost(false, n16, s16, cus) : 2.7 + s16 * 1.05 * ((n32 + cus - 1) / cus));
    for (int z = 2; z <= 8 && (size_t)z * out * sizeof(float) <= scratch_bytes; ++z) {
        const double sum = 3.2 + (z + 1) * out / 1.0e6;
        if (s16 / z >= 2) {
            const double c = f32_cost(false, z * n16, (s16 + z - 1) / z, cus) + sum;
            if (c < cost) { best = F32Shares{F32Tile::k16x32Split, z}; cost = c; }
        }
        if (z >= 3 && s32 / z >= 2) {
            const double c = f32_cost(true, z * n32, (s32 + z - 1) / z, cus) + sum;
            if (c < cost) { best = F32Shares{F32Tile::k32x32, z}; cost = c; }
        }
    }
    return best;
}

}  // namespace moc
