// bf16 x bf16 -> fp32 GEMM for large tiles: two groups of four wavefronts that take turns at the matrix cores.
//
//   C[m, n] = sum_k A(m, k) B(n, k)   (+ a second operand pair accumulated into the same tile)
//
// Operands as in gemm_mfma.h: k-contiguous (KC) or k-major (KM), in the layout they have in memory.
//
// Bound: the matrix cores, as far as the hand-over and the rounds of tiles let them work, at the clock the power limit leaves (2.0 to
// 2.2 GHz).  Counted (SQ_VALU_MFMA_BUSY_CYCLES of all SIMD cycles): 0.70 for one full round of 256 tiles, 8192 x 2048 x 5461 and 2 * 5461;
// 0.61 and 0.58 for 2.75 and 5.5 rounds, 8192 x 5461 x 2048 to bf16 and as gate + up; 0.68 for two rounds of three products, 5376 x 2048 x 8192 (0.55 when
// 5461 rows ran on 192 x 256 tiles in 2.72 rounds).  What the kernel of gemm_mfma.h (0.47 to 0.61) loses against that is the way of the operands: one
// wavefront per SIMD has to fit the global loads, the writes to LDS and the fragment reads between its own MFMAs.  Here
//  - operands go from memory to LDS without passing through registers (buffer_load ... lds, 1 KB per instruction), so there are no
//    staging registers and no LDS writes to issue; what lies past the end of an operand is delivered as zeros by the buffer's range
//    check, so ragged rows, columns and contraction ends need no code;
//  - a compute unit holds eight wavefronts, two per SIMD, in two groups that run half a phase apart: while one group issues its
//    fragment reads and loads, the other has the matrix cores.  Barriers hand them over.  Without the offset, the same code
//    takes 611 instead of 533 us for 8192 x 11008 x 4096 (bf16 result), 218 instead of 183 us for 4096 x 4096 x 8192.
//
// A k-slice is 64 wide.  A tile's slice is loaded as four half tiles, the first and second half of its rows of A and of B; a
// wavefront owns a block in every quadrant of the tile, so each half tile is read by every wavefront in ONE phase and its place in
// LDS can be filled again from the next phase on.  Two slices live in LDS; four phases a slice, one quadrant's products each:
//
//     phase       1      2      3      4      5      6      7      8
//     reads      A0     B1     A1     B1'    A0'    B0'    A1'    B0''      (' the odd slice, '' the next even one)
//     products   00     01     11     10     01'    00'    10'    11'
//     loads      B0''   A0''   B1''   A1''   B1'''  A0'''  B0'''  A1'''     (two slices on, into the place read one phase ago)
//
// Every half tile is requested seven phases (1.75 slices) before it is read, and a wait never asks for more than the oldest
// request.  The requests run on into the workgroup's next tile, whose first two slices arrive while the tile is written out.
// Hand-over: a wavefront waits for its own fragment reads and for its own part of the next half tile at the end of the
// reading half of a phase, before the barrier.  So behind that barrier (a) everybody's part of the half tile has arrived and (b) nobody
// reads the place any more that the other group's next loads fill.
//
// Measured (one MI355X, 256 x 256 tiles, us; before: the best tile of gemm_mfma.h): 8192 x 5461 x 2048 to bf16 178 -> 151,
// 8192 x 11008 x 4096 to bf16 655 -> 533, 8192 x 2048 x 5461 (B k-major) 148 -> 126, 8192 x 2048 x 2*5461 297 -> 248.
#pragma once
#include <type_traits>

#include "common.h"
#include "gemm_mfma.h"
#include "gemm_plan.h"
#include "kernel_attrs.h"
#include "lds_dma.h"

namespace moc {

constexpr int kPpWaves = 8, kPpThreads = kPpWaves * 64;
constexpr int kPpStageBytes = 4096;      // per wavefront, for turning accumulators into rows

// Wavefronts form a WGM x (8 / WGM) grid over every quadrant; group 0 has the upper half of the rows of each.
template <int BM, int BN> struct PpCfg {
    static constexpr int HA = BM / 2, HB = BN / 2;                   // rows of a half tile
    static constexpr int WGM = BN == 256 ? 2 : 4, WGN = kPpWaves / WGM;
    static constexpr int WA = HA / WGM, WB = HB / WGN;               // rows a wavefront reads of it
    static constexpr int TA = WA / 16, TB = WB / 16;
    static_assert(WA % 16 == 0 && WB % 16 == 0 && TA >= 1 && TB >= 1, "wave tile must consist of 16x16 blocks");
    static constexpr int kA = HA * kPpBK * 2, kB = HB * kPpBK * 2;   // bytes of a half tile
    static constexpr int NA = (HA + 63) / 64, NB = (HB + 63) / 64;   // 1 KB loads per wavefront and half tile; 96 rows: the second of half a KB
    static constexpr int kBufs = 4 * (kA + kB);
    static constexpr int kLds = kBufs + kPpWaves * kPpStageBytes;
    static_assert(4 * kA <= 65536 && 4 * kB <= 65536 && kLds <= 160 * 1024, "");
};

__device__ __forceinline__ void pp_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
}

// The half tile of HR rows x 64 k of one operand: its layout in LDS, the loads that fill it and the fragments read from it.
//   KC: [row][64 k], 128 bytes a row, the position of a 16-byte chunk XORed with bits 1..3 of the row;
//   KM: [k][HR rows] as in memory, the position of a 64-byte piece XORed with the k row and of a 32-byte piece with bit 3 of the k row
//       (96 rows: 192 bytes a k row, which spreads the 64-byte pieces by itself).
// Both so that the lanes that an LDS read serves together meet different banks.  (Counted: 2 to 15 % of the LDS cycles are conflicts, in inverse
// proportion to the number of slices: they are the epilogue's.)
template <bool KM, int HR, int TR> struct PpHalf {
    static constexpr int kPitch = HR * 2;                 // KM
    static constexpr int kAddrs = KM ? TR : 2;
    typedef __attribute__((address_space(3))) const bf16x8_t* frag_ptr;
    typedef __attribute__((address_space(3))) s16x4_t* tr_ptr;
    uint32_t addr[kAddrs];

    static __device__ __forceinline__ int chunk_xor(int row_or_k) {
        if (!KM) return (row_or_k >> 1) & 7;
        const int flip = ((row_or_k >> 3) & 1) << 1;
        return HR == 128 ? ((row_or_k & 3) << 2) ^ flip : HR == 64 ? (((row_or_k >> 1) & 1) << 2) ^ flip : flip;
    }
    // base: LDS byte address of the operand's half tiles; row0: the wavefront's first row
    __device__ __forceinline__ void init(uint32_t base, int row0, int lane) {
        if constexpr (!KM) {
            const int row = row0 + (lane & 15);
#pragma unroll
            for (int k = 0; k < 2; ++k) addr[k] = base + row * 128 + (((k * 4 + (lane >> 4)) ^ chunk_xor(row)) << 4);
        } else {
            const int krow = 8 * (lane >> 4) + ((lane & 15) >> 2);      // see read_fragment (gemm_mfma.h) for the transposing read
#pragma unroll
            for (int i = 0; i < TR; ++i) {
                const int col = row0 + i * 16 + (lane & 3) * 4;
                addr[i] = base + krow * kPitch + (((col >> 3) ^ chunk_xor(krow)) << 4) + (col & 7) * 2;
            }
        }
    }
    // fragment of 16 rows x 32 k: row block i, k step k, of the half tile at byte `off`: lane l gets row l % 16, k 8 (l / 16) .. + 8
    __device__ __forceinline__ bf16x8_t read(uint32_t off, int i, int k) const {
        if constexpr (!KM) {
            return *reinterpret_cast<frag_ptr>(addr[k] + off + i * 16 * 128);
        } else {
            const uint32_t p = addr[i] + off + k * 32 * kPitch;      // (neither 32 nor 4 k rows change the XOR)
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<tr_ptr>(p));
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<tr_ptr>(p + 4 * kPitch));
            typedef short s16x8_t __attribute__((ext_vector_type(8)));
            const s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8_t, v);
        }
    }
    // byte offset in memory, from the half tile's first element, of the 16-byte chunk number c of the half tile in LDS
    static __device__ __forceinline__ uint32_t source(int c, uint32_t ld) {
        constexpr int CPR = KM ? HR / 8 : 8;
        const int r = c / CPR;
        return (uint32_t)r * ld * 2u + (uint32_t)(((c % CPR) ^ chunk_xor(r)) << 4);
    }
};

// Where the products go: row-major, ldc and N multiples of 8 (of 4 for fp32), share z of a split contraction at p + z * stride.
struct PpOut {
    void* p;
    int64_t ldc, stride;
    int N;
    int f32;
};

// Up to NB problems in one launch that agree in N, both leading dimensions and the layouts; problem z has tiles[z] tiles, tiles_n to a
// row of tiles.  With nsplit > 1 (pp_shares) item i is share i / tiles of tile i % tiles: the shares are ranges of whole slices.
//
// The items are the tiles, dealt to the XCDs as follows; an XCD's workgroups take its items in turn.
//   NB <= 3: the tiles of all problems in a row, XCD x takes the x-th eighth (neighbouring tiles share operand panels in its L2).
//   NB > 3 (experts, whose row counts differ): XCD x takes the x-th eighth of EVERY problem, in the order of the problems, which the host
//     sorts by the length of the contraction, and every second round of its workgroups goes backwards, so that long and short
//     contractions add up alike.  Weight gradients go to one XCD whole (owner) where the XCDs' loads are as even that way (pp_owners): its
//     L2 then serves every operand panel to all tiles.  Eight experts of 768 x 2048 with 2000 to 6000 rows each (24 weight gradients): 370 us with
//     the whole list cut into eighths, where one XCD got one expert.
template <int NB> struct PpWork {
    static constexpr bool kSpread = NB > 3;
    MfmaProblem pr[NB];
    PpOut out[NB];
    int tiles[NB];
    int cum[kSpread ? 8 : 1][NB + 1];      // items before problem z: of XCD x, or of all
    int nprob, tiles_n, nsplit;
    // weight gradients with kSpread: rows of tiles in a band, and the XCD that has all tiles of problem z, or -1 (words, which the scalar cache can load)
    int height = 4;
    int owner[kSpread ? NB : 1];
};

// F32: 0 = every result bf16, 1 = every result fp32, 2 = as PpOut says.
// Shares are for one problem, or for three with fp32 results: the other kernels are built without the divisions that find an item's share (gate
// + up of 4096 x 768 x 2048, 12 slices a tile: 31.8 us with them, 31.5 without).
template <int F32, int NB> constexpr bool pp_shares = NB == 1 || (NB == 3 && F32 == 1);
template <int BM, int BN, bool AKM, bool BKM, int F32, int NB>
__global__ __launch_bounds__(kPpThreads, 2) void gemm_bf16_pp_kernel(PpWork<NB> w) {
    using C = PpCfg<BM, BN>;
    constexpr int TA = C::TA, TB = C::TB;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / C::WGN, wn = wave % C::WGN;
    const int group = wave >> 2;
    constexpr bool kSpread = PpWork<NB>::kSpread, kOwners = kSpread && AKM && BKM, kShares = pp_shares<F32, NB>;
    const int xcd = blockIdx.x & 7;
    const int* const cum = w.cum[kSpread ? xcd : 0];
    const int tiles = cum[NB], total = tiles * (kShares ? w.nsplit : 1);      // (cum[NB] is the total also with fewer problems; of this XCD if kSpread)
    const uint32_t lda = (uint32_t)w.pr[0].A.ld, ldb = (uint32_t)w.pr[0].B.ld;

    const uint32_t lds_a = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem);
    const uint32_t lds_b = lds_a + 4 * C::kA;
    using HalfA = PpHalf<AKM, C::HA, TA>;
    using HalfB = PpHalf<BKM, C::HB, TB>;
    HalfA ha;
    HalfB hb;
    ha.init(lds_a, wm * C::WA, lane);
    hb.init(lds_b, wn * C::WB, lane);
    // a wavefront loads HA / 8 (HB / 8) KB of a half tile: chunk numbers wave * HA + lane, + 64
    uint32_t src_a[C::NA], src_b[C::NB];
#pragma unroll
    for (int i = 0; i < C::NA; ++i) src_a[i] = HalfA::source(wave * C::HA + i * 64 + lane, lda);
#pragma unroll
    for (int i = 0; i < C::NB; ++i) src_b[i] = HalfB::source(wave * C::HB + i * 64 + lane, ldb);

    // ---- items: problem z, tile origin, range of slices
    struct Item {
        int z, share, m0, n0;
    };
    // position of this workgroup's item number r in the list that cum counts, or -1 after its last
    auto position = [&](int r) {
        if (kSpread) {
            const int width = (int)gridDim.x >> 3, local = (int)blockIdx.x >> 3;
            const int p = r * width + ((r & 1) ? width - 1 - local : local);
            return p < total ? p : -1;      // (only the last round is part-filled)
        }
        const int item = (int)blockIdx.x + r * (int)gridDim.x;
        return item < total ? xcd_contiguous_index(item, total) : -1;
    };
    auto item_at = [&](int mapped) {
        Item t;
        t.share = 0;
        if (kShares && w.nsplit > 1) {
            t.share = mapped / tiles;
            mapped -= t.share * tiles;
        }
        t.z = 0;
#pragma unroll
        for (int z = 1; z < NB; ++z) t.z += mapped >= cum[z];
        int logical = mapped - cum[t.z];
        if (kSpread && (!kOwners || w.owner[t.z] < 0)) logical += w.tiles[t.z] * xcd / 8;
        const int tiles_m = w.tiles[t.z] / w.tiles_n;
        const int height = kOwners ? w.height : w.tiles_n >= 32 ? 8 : 4;      // band height, see gemm_bf16_mfma_tiles
        const int band = logical / (height * w.tiles_n);
        const int first_m = band * height;
        const int rows = min(tiles_m - first_m, height);
        const int in_band = logical - first_m * w.tiles_n;
        t.m0 = (first_m + in_band % rows) * BM;
        t.n0 = (in_band / rows) * BN;
        return t;
    };
    // ---- the stream of slices to load: base pointers, readable bytes and offsets of the present segment, slices left in it
    struct Stream {
        const bf16_t *a, *b, *a2, *b2;
        uint32_t a_bytes, b_bytes, b_bytes2, oa, ob, oa2, ob2;
        int left, left2;
    };
    auto begin = [&](const Item& t, int& slices) {
        const MfmaProblem& pr = w.pr[t.z];
        const int nk0 = (pr.Kc + kPpBK - 1) / kPpBK, nk = nk0 + (pr.Kc2 + kPpBK - 1) / kPpBK;
        const int from = kShares ? nk * t.share / w.nsplit : 0, to = kShares ? nk * (t.share + 1) / w.nsplit : nk;
        slices = to - from;
        Stream s;
        s.a_bytes = (uint32_t)(AKM ? pr.Kc : pr.M) * lda * 2u;
        s.b_bytes = (uint32_t)(BKM ? pr.Kc : pr.N) * ldb * 2u;
        s.b_bytes2 = (uint32_t)(BKM ? pr.Kc2 : pr.N) * ldb * 2u;
        s.a2 = pr.A.p2;
        s.b2 = pr.B.p2;
        s.oa2 = (uint32_t)t.m0 * (AKM ? 1u : lda) * 2u;
        s.ob2 = (uint32_t)t.n0 * (BKM ? 1u : ldb) * 2u;
        const bool second = from >= nk0;      // a share that starts in the second segment
        const uint32_t k = (uint32_t)(second ? from - nk0 : from) * kPpBK;
        s.a = second ? pr.A.p2 : pr.A.p;
        s.b = second ? pr.B.p2 : pr.B.p;
        if (second) s.b_bytes = s.b_bytes2;
        s.oa = s.oa2 + k * (AKM ? lda : 1u) * 2u;
        s.ob = s.ob2 + k * (BKM ? ldb : 1u) * 2u;
        s.left = min(nk0, to) - from;
        s.left2 = max(0, to - nk0);
        if (second) {
            s.left = to - from;
            s.left2 = 0;
        }
        return s;
    };
    struct Slice {
        u32x4_t ra, rb;
        uint32_t oa, ob;
    };
    // the next slice of the stream; past its end the descriptors are empty and loads bring zeros without reading
    auto advance = [&](Stream& s) {
        Slice r;
        r.ra = buffer_desc(s.a, s.left > 0 ? s.a_bytes : 0u);
        r.rb = buffer_desc(s.b, s.left > 0 ? s.b_bytes : 0u);
        r.oa = s.oa;
        r.ob = s.ob;
        s.oa += kPpBK * 2u * (AKM ? lda : 1u);
        s.ob += kPpBK * 2u * (BKM ? ldb : 1u);
        if (--s.left == 0) {
            s.a = s.a2;
            s.b = s.b2;
            s.b_bytes = s.b_bytes2;
            s.oa = s.oa2;
            s.ob = s.ob2;
            s.left = s.left2;
            s.left2 = 0;
        }
        return r;
    };
    auto place_a = [&](int buf, int h) { return (uint32_t)((buf * 2 + h) * C::kA); };
    auto place_b = [&](int buf, int h) { return (uint32_t)((buf * 2 + h) * C::kB); };
    auto load_a = [&](const Slice& s, int buf, int h) {
        const uint32_t o = s.oa + (h ? (uint32_t)C::HA * 2u * (AKM ? 1u : lda) : 0u);
#pragma unroll
        for (int i = 0; i < C::NA; ++i)
            if (i * 64 + 64 <= C::HA || lane < C::HA % 64) lds_load16(src_a[i] + o, s.ra, lds_a + place_a(buf, h) + (wave * C::HA + i * 64) * 16);
    };
    auto load_b = [&](const Slice& s, int buf, int h) {
        const uint32_t o = s.ob + (h ? (uint32_t)C::HB * 2u * (BKM ? 1u : ldb) : 0u);
#pragma unroll
        for (int i = 0; i < C::NB; ++i)
            if (i * 64 + 64 <= C::HB || lane < C::HB % 64) lds_load16(src_b[i] + o, s.rb, lds_b + place_b(buf, h) + (wave * C::HB + i * 64) * 16);
    };

    f32x4_t acc[2][2][TA][TB];      // [half of A][half of B]
    bf16x8_t fa[TA][2], fb[2][TB][2];
    auto read_a = [&](int buf, int h) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < TA; ++i) fa[i][k] = ha.read(place_a(buf, h), i, k);
    };
    auto read_b = [&](int buf, int h) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < TB; ++j) fb[h][j][k] = hb.read(place_b(buf, h), j, k);
    };
    // Products of quadrant (hm, hn); `zero`: the tile's first, which start from zero.
    auto multiply = [&](int hm, int hn, bool zero) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < TB; ++j) {
                    const f32x4_t c = zero && k == 0 ? f32x4_t{0.0f, 0.0f, 0.0f, 0.0f} : acc[hm][hn][i][j];
                    acc[hm][hn][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[hn][j][k], fa[i][k], c, 0, 0, 0);
                }
    };

    int turn = 0, item = position(0);
    if (item < 0) return;
    int slices, next_slices = 0;
    Item cur = item_at(item), nxt = cur;
    Stream st = begin(cur, slices);
    {
        const Slice s0 = advance(st), s1 = advance(st);
        load_b(s0, 0, 0); load_a(s0, 0, 0); load_b(s0, 0, 1); load_a(s0, 0, 1);
        load_b(s1, 1, 1); load_a(s1, 1, 0); load_b(s1, 1, 0); load_a(s1, 1, 1);
    }
    constexpr int VM = 3 * (C::NA + C::NB);      // vector memory instructions of the last six phases
    constexpr int kStores32 = 2 * C::WA * 2 * C::WB * 4 / 1024, kStores16 = kStores32 / 2;      // of an epilogue
    static_assert(VM + kStores32 < 64, "");
    wait_counts<VM + C::NA, true>();
    pp_barrier();
    read_b(0, 0);
    wait_counts<VM, true>();
    pp_barrier();
    int stores = 0;                              // of the tile before, still among the counted
    if (group == 1) pp_barrier();                // half a phase behind
    for (;;) {
        const int next_item = position(++turn);
        const bool more = next_item >= 0;
        const int pairs = (slices + 1) >> 1;
        // Two slices.  In a tile's first pair the products start from zero and, as the previous tile's stores went out after the loads
        // that phases 1 .. 6 wait for, these waits let the stores be.
        auto pair = [&](auto first, bool last) {
            constexpr bool FIRST = decltype(first)::value;
            if (last) {
                if (more) {
                    nxt = item_at(next_item);
                    st = begin(nxt, next_slices);
                }
            }
            const bool two = !(last && (slices & 1));
            const Slice s0 = advance(st), s1 = advance(st);
            auto hand_over = [&](bool early) {
                if constexpr (FIRST) {
                    if (early && F32 != 0 && stores == kStores32) wait_counts<VM + kStores32, true>();
                    else if (early && F32 != 1 && stores == kStores16) wait_counts<VM + kStores16, true>();
                    else wait_counts<VM, true>();
                } else {
                    wait_counts<VM, true>();
                }
                pp_barrier();
            };
            read_a(0, 0); load_b(s0, 0, 0); hand_over(true);  multiply(0, 0, FIRST); pp_barrier();
            read_b(0, 1); load_a(s0, 0, 0); hand_over(true);  multiply(0, 1, FIRST); pp_barrier();
            read_a(0, 1); load_b(s0, 0, 1); hand_over(true);  multiply(1, 1, FIRST); pp_barrier();
            read_b(1, 1); load_a(s0, 0, 1); hand_over(true);  multiply(1, 0, FIRST); pp_barrier();
            read_a(1, 0); load_b(s1, 1, 1); hand_over(true);  if (two) multiply(0, 1, false); pp_barrier();
            read_b(1, 0); load_a(s1, 1, 0); hand_over(true);  if (two) multiply(0, 0, false); pp_barrier();
            read_a(1, 1); load_b(s1, 1, 0); hand_over(false); if (two) multiply(1, 0, false); pp_barrier();
            read_b(0, 0); load_a(s1, 1, 1); hand_over(false); if (two) multiply(1, 1, false); pp_barrier();
        };
        pair(std::true_type{}, pairs == 1);
        for (int p = 1; p < pairs; ++p) pair(std::false_type{}, p + 1 == pairs);

        // ---- epilogue.  acc[.][.][i][j][r] is C[m, n] with m = .. + lane % 16 and n = .. + 4 (lane / 16) + r.  Every wavefront turns blocks
        //      of 16 or 32 rows around in its own piece of LDS and stores whole row segments, 16 bytes per lane.  The number of
        //      store instructions does not depend on the edges (the range check drops rows past the last, an offset out
        //      of range columns past the last), because the waits above count them.
        const PpOut& out = w.out[cur.z];
        const int rows = min(w.pr[cur.z].M - cur.m0, BM);
        auto write = [&](auto zero) {
            using T = decltype(zero);
            constexpr bool f32 = std::is_same<T, float>::value;
            constexpr int ES = sizeof(T);
            constexpr int RB = f32 && C::WB == 48 ? 1 : 2;                   // 16-row blocks at a time
            constexpr int CPR = C::WB * ES / 16;                             // 16-byte chunks per row
            constexpr int PITCH = f32 && C::WB == 32 ? 128 : C::WB * ES + 16;      // (128: positions XORed with the row instead of padding)
            static_assert(RB * 16 * PITCH <= kPpStageBytes && (RB * 16 * CPR) % 64 == 0 && (2 * TA) % RB == 0, "");
            const auto place = [](int row, int bytes) {
                return row * PITCH + (PITCH == 128 ? bytes ^ ((row & 7) << 4) : bytes);
            };
            unsigned char* area = smem + C::kBufs + wave * kPpStageBytes;
            const uint32_t pitch = (uint32_t)out.ldc * ES;
            const auto desc = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<unsigned char*>(out.p) + ((int64_t)cur.share * out.stride + (int64_t)cur.m0 * out.ldc) * ES, 0, rows * pitch, 0x00020000);
#pragma unroll
            for (int hn = 0; hn < 2; ++hn)
#pragma unroll
                for (int b = 0; b < 2 * TA; b += RB) {
#pragma unroll
                    for (int i = 0; i < RB; ++i)
#pragma unroll
                        for (int j = 0; j < TB; ++j) {
                            const f32x4_t v = acc[(b + i) / TA][hn][(b + i) % TA][j];
                            unsigned char* q = area + place(i * 16 + (lane & 15), (j * 16 + 4 * (lane >> 4)) * ES);
                            if constexpr (f32) *reinterpret_cast<f32x4_t*>(q) = v;
                            else *reinterpret_cast<u32x2_t*>(q) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                        }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                    for (int it = 0; it < RB * 16 * CPR / 64; ++it) {
                        const int c = it * 64 + lane, row = c / CPR, ch = c % CPR;
                        const u32x4_t v = *reinterpret_cast<const u32x4_t*>(area + place(row, ch * 16));
                        const int blk = b + row / 16;
                        const int m = (blk / TA) * C::HA + wm * C::WA + (blk % TA) * 16 + (row & 15);
                        const int n = cur.n0 + hn * C::HB + wn * C::WB + ch * (16 / ES);
                        const uint32_t off = n < out.N ? (uint32_t)m * pitch + (uint32_t)n * ES : 0xFFFFFF00u;
                        __builtin_amdgcn_raw_buffer_store_b128(v, desc, off, 0, 0);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            stores = f32 ? kStores32 : kStores16;
        };
        if (F32 == 1 || (F32 == 2 && out.f32)) write(0.0f);
        else write(bf16_t{});
        if (!more) break;
        cur = nxt;
        slices = next_slices;
        item = next_item;
    }
    if (group == 0) pp_barrier();
    wait_counts<0, true>();      // nothing may still be on its way to LDS when the workgroup ends
}

inline PpSizes pp_sizes(const MfmaProblem& p, const PpOut& o) {
    return PpSizes{p.M, p.N, p.Kc, p.Kc2, p.A.ld, p.B.ld, p.A.km, p.B.km, p.a_zero_padded, o.N, o.ldc, o.stride, o.f32 ? 4 : 2};
}
inline bool pp_problem_ok(const MfmaProblem& p, const PpOut& o) {
    return mfma_problem_ok(p) && (reinterpret_cast<uintptr_t>(o.p) & 15) == 0 && pp_sizes_ok(pp_sizes(p, o));
}

// w.tiles, w.cum and w.tiles_n are filled in here; `wgs` workgroups at most (a multiple of 8; 0: one per item), each walking over its items.
template <int BM, int BN, bool AKM, bool BKM, int F32, int NB> inline hipError_t launch_gemm_bf16_pp(PpWork<NB>& w, int wgs, hipStream_t st) {
    using C = PpCfg<BM, BN>;
    auto kern = gemm_bf16_pp_kernel<BM, BN, AKM, BKM, F32, NB>;
    LdsAttr<gemm_bf16_pp_kernel<BM, BN, AKM, BKM, F32, NB>, C::kLds>::use();
    w.tiles_n = (w.pr[0].N + BN - 1) / BN;
    for (int z = 0; z < NB; ++z) w.tiles[z] = z < w.nprob ? (w.pr[z].M + BM - 1) / BM * w.tiles_n : 0;
    constexpr int kLists = PpWork<NB>::kSpread ? 8 : 1;
    int longest = 0;
    constexpr bool kOwners = kLists > 1 && AKM && BKM;
    if constexpr (kOwners) {
        w.height = pp_band_height(BM, BN, *std::max_element(w.tiles, w.tiles + NB) / 8);
        std::fill(w.owner, w.owner + NB, -1);
        int slices[NB];
        for (int z = 0; z < w.nprob; ++z) slices[z] = pp_slice_count(w.pr[z].Kc, w.pr[z].Kc2);
        if (pp_owners(w.nprob, slices, w.tiles, std::max(1, wgs / 8), w.owner)) w.height = pp_band_height(BM, BN, std::min(w.tiles[0], wgs / 8));
    }
    for (int x = 0; x < kLists; ++x) {
        w.cum[x][0] = 0;
        for (int z = 0; z < NB; ++z) {
            int n = w.tiles[z] * (x + 1) / kLists - w.tiles[z] * x / kLists;
            if (kOwners && w.owner[z] >= 0) n = w.owner[z] == x ? w.tiles[z] : 0;
            w.cum[x][z + 1] = w.cum[x][z] + n;
        }
        longest = std::max(longest, w.cum[x][NB]);
    }
    if (!pp_shares<F32, NB> && w.nsplit != 1) return hipErrorInvalidValue;
    const int total = kLists * longest * w.nsplit;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(kern, dim3(mfma_grid(total, wgs)), dim3(kPpThreads), C::kLds, st, w);
    return hipGetLastError();
}

}  // namespace moc
