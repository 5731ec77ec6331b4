// fp32 GEMM on the gfx950 matrix cores (v_mfma_f32_16x16x4_f32: fp32 inputs, fp32 products and sums).
//
//   C[m, n] = sum_k A(m, k) B(n, k)   (+ a second operand pair accumulated into the same tile)
//
// Same operand layouts as the bf16 kernel (k-contiguous or k-major, gemm_generic.h), staged as they lie in
// memory: k-contiguous tiles as [row][BK + 4] floats, k-major tiles as [k][ROWS + 4] floats.  Both pitches
// spread what one fragment read touches over all 64 banks: 16 rows of 16 bytes, or 16 rows of k 0, 4, 8 and 12.
//
// What bounds it: at the sizes fp32 is used for (a few hundred tokens, d of 512 to 768) a product has less than
// one GFLOP, 2 to 5 us of matrix-core time for the chip, so the launch, the load latency and the length of a
// wavefront's chain of MFMAs decide.  Hence small tiles (enough workgroups for all compute units), four k-slices of
// 32 to 128 in flight in registers ahead of two LDS stages, and, where even 32 x 32 tiles do not fill the chip
// and the contraction is long, KW = 4: the four wavefronts of a workgroup take a quarter of every k-slice each and
// their tiles are added through LDS in a fixed order.  With KW = 1 a result is one sum from zero in
// one order of k for every tile shape: groups of 16 ascending, a group's k as 0 4 8 12, 1 5 9 13, 2 6 10 14, 3 7 11 15.
//
// Contractions whose tiles leave compute units idle run in shares (f32_shares).
//
// Measured at T 256, d 512, F 1376 (forward + backward, ten products in five launches and a sum of shares; medians of a profile, which adds about 10 % to
// launches of this length): gate + up 15.7 us, down 10.6, dZ' 11.7, three weight gradients 22.1, dX 13.4 + 4.4, against 125, 222, 63, 143 and 424 us on
// the fp32-FMA kernel of gemm_generic.h, which has 32 to 88 workgroups and waits for every 16-k slice; about 72 TFLOP/s at the margin (142 on a large
// library product), the rest launch and first loads.
#pragma once
#include "common.h"
#include "gemm_generic.h"
#include "gemm_plan.h"
#include "kernel_attrs.h"

namespace moc {

// NB problems of one shape and layout in one launch (blockIdx.y).
template <class Epi, int NB> struct F32Batch {
    GemmProblem<float> pr[NB];
    Epi epi[NB];
};

constexpr int kF32Sets = 4;      // k-slices in flight in registers

template <int BM, int BN, int KW, bool AKM, bool BKM> struct F32Cfg {
    static constexpr int BK = KW > 1 ? 128 : (BM < 64 ? 64 : 32);
    static constexpr int kPitchA = (AKM ? BM : BK) + 4, kPitchB = (BKM ? BN : BK) + 4;       // floats
    static constexpr int kFloatsA = (AKM ? BK : BM) * kPitchA, kFloatsB = (BKM ? BK : BN) * kPitchB;
    static constexpr int kStage = kFloatsA + kFloatsB;
    static constexpr int kLds = 2 * kStage * (int)sizeof(float);
};

// (three workgroups per compute unit for the small-slice tiles: the weight-gradient launch then runs in one round)
// With SPLIT (one problem) blockIdx.y is a share of the tile's k-slices, whose sums go to epi.share(blockIdx.y).
template <int BM, int BN, int KW, bool AKM, bool BKM, class Epi, int NB, bool SPLIT = false>
__global__ __launch_bounds__(256, KW == 1 ? 3 : 2) void gemm_f32_mfma_kernel(F32Batch<Epi, NB> batch, int tiles_n) {
    using Cfg = F32Cfg<BM, BN, KW, AKM, BKM>;
    static_assert(KW == 1 || KW == 4, "the wavefronts split the tile 2 x 2 or the k-slice in four");
    constexpr int BK = Cfg::BK, NT = 256;
    constexpr int WM = KW == 1 ? BM / 2 : BM, WN = KW == 1 ? BN / 2 : BN;
    constexpr int TM = WM / 16, TN = WN / 16;
    constexpr int LA = BM * BK / 4 / NT, LB = BN * BK / 4 / NT;      // 16-byte chunks per thread and slice
    extern __shared__ __align__(16) float f32_smem[];
    const GemmProblem<float>& pr = batch.pr[NB == 1 ? 0 : blockIdx.y];
    static_assert(!SPLIT || NB == 1, "");
    const Epi epi = [&] {
        if constexpr (SPLIT) return batch.epi[0].share(blockIdx.y);
        else return batch.epi[NB == 1 ? 0 : blockIdx.y];
    }();
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int M = pr.M, N = pr.N;
    const int m0 = (blockIdx.x / tiles_n) * BM, n0 = (blockIdx.x % tiles_n) * BN;
    const int wm0 = KW == 1 ? (wave >> 1) * WM : 0, wn0 = KW == 1 ? (wave & 1) * WN : 0;
    const int k_wave = KW == 1 ? 0 : wave * (BK / KW);               // first k of this wavefront inside a slice
    const int nk0 = (pr.Kc + BK - 1) / BK, nk_all = nk0 + (pr.Kc2 + BK - 1) / BK;
    const int ks = SPLIT ? nk_all * (int)blockIdx.y / (int)gridDim.y : 0, nk = SPLIT ? nk_all * ((int)blockIdx.y + 1) / (int)gridDim.y : nk_all;      // slices ks .. nk - 1

    f32x4_t ga[kF32Sets][LA], gb[kF32Sets][LB];
    // one operand's chunks of k-slice kt -> registers.  Branch-free: rows and k past the end are clamped to readable
    // ones (a predicated load would make the wavefront wait for its predecessors); rows past the edge give results
    // that the epilogue drops, k past the end is zeroed when the slice goes to LDS.
    int a_off[LA], b_off[LB], a_koff[LA], b_koff[LB];      // element offsets of the chunks: row part, k part inside a slice
    auto offsets = [&](auto km_c, auto rows_c, const GemmOperand<float>& o, int row0, int rows, int* off, int* koff) {
        constexpr bool KM = decltype(km_c)::value;
        constexpr int ROWS = decltype(rows_c)::value, L = ROWS * BK / 4 / NT;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const int c = tid + i * NT;
            off[i] = KM ? min(row0 + (c % (ROWS / 4)) * 4, o.ext - 4) : min(row0 + c / (BK / 4), rows - 1) * (int)o.ld;
            koff[i] = KM ? c / (ROWS / 4) * (int)o.ld : (c % (BK / 4)) * 4;
        }
    };
    offsets(std::integral_constant<bool, AKM>{}, std::integral_constant<int, BM>{}, pr.A, m0, M, a_off, a_koff);
    offsets(std::integral_constant<bool, BKM>{}, std::integral_constant<int, BN>{}, pr.B, n0, N, b_off, b_koff);
    int a_all[LA], b_all[LB];
#pragma unroll
    for (int i = 0; i < LA; ++i) a_all[i] = a_off[i] + a_koff[i];
#pragma unroll
    for (int i = 0; i < LB; ++i) b_all[i] = b_off[i] + b_koff[i];
    auto fetch = [&](auto buf_c, int kt) {
        constexpr int buf = decltype(buf_c)::value;
        kt = min(kt, nk - 1);
        const bool seg = kt >= nk0;
        const int k0 = (seg ? kt - nk0 : kt) * BK, left = (seg ? pr.Kc2 : pr.Kc) - k0;      // left >= 1
        const float* pa = (seg ? pr.A.p2 : pr.A.p) + (AKM ? k0 * pr.A.ld : (int64_t)k0);
        const float* pb = (seg ? pr.B.p2 : pr.B.p) + (BKM ? k0 * pr.B.ld : (int64_t)k0);
        const int a_last = AKM ? last_row_offset(left, BK, (int)pr.A.ld) : ((left + 3) & ~3) - 4;
        const int b_last = BKM ? last_row_offset(left, BK, (int)pr.B.ld) : ((left + 3) & ~3) - 4;
        auto load = [&](auto cut_c) {                                // (whole slices: nothing to compute per chunk)
            constexpr bool CUT = decltype(cut_c)::value;
#pragma unroll
            for (int i = 0; i < LA; ++i) ga[buf][i] = *reinterpret_cast<const f32x4_t*>(pa + (uint32_t)(CUT ? a_off[i] + min(a_koff[i], a_last) : a_all[i]));
#pragma unroll
            for (int i = 0; i < LB; ++i) gb[buf][i] = *reinterpret_cast<const f32x4_t*>(pb + (uint32_t)(CUT ? b_off[i] + min(b_koff[i], b_last) : b_all[i]));
        };
        if (left >= BK) load(std::false_type{});
        else load(std::true_type{});
    };
    // `left`: k of the slice that count, the rest is zeroed (CUT is the uniform "left < BK")
    auto stash_operand = [&](auto km_c, auto rows_c, auto pitch_c, auto cut_c, float* base, const f32x4_t* g, int left) {
        constexpr bool KM = decltype(km_c)::value, CUT = decltype(cut_c)::value;
        constexpr int ROWS = decltype(rows_c)::value, PITCH = decltype(pitch_c)::value, L = ROWS * BK / 4 / NT;
#pragma unroll
        for (int i = 0; i < L; ++i) {
            const int c = tid + i * NT;
            f32x4_t v = g[i];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (CUT && (KM ? c / (ROWS / 4) : (c % (BK / 4)) * 4 + e) >= left) v[e] = 0.0f;
            *reinterpret_cast<f32x4_t*>(KM ? base + (c / (ROWS / 4)) * PITCH + (c % (ROWS / 4)) * 4
                                           : base + (c / (BK / 4)) * PITCH + (c % (BK / 4)) * 4) = v;
        }
    };
    auto stash = [&](auto buf_c, int kt) {                           // register set s goes to LDS stage s % 2
        constexpr int buf = decltype(buf_c)::value;
        float* a = f32_smem + (buf & 1) * Cfg::kStage;
        const int left = kt >= nk0 ? pr.Kc2 - (kt - nk0) * BK : pr.Kc - kt * BK;
        auto both = [&](auto cut_c) {
            stash_operand(std::integral_constant<bool, AKM>{}, std::integral_constant<int, BM>{},
                          std::integral_constant<int, Cfg::kPitchA>{}, cut_c, a, ga[buf], left);
            stash_operand(std::integral_constant<bool, BKM>{}, std::integral_constant<int, BN>{},
                          std::integral_constant<int, Cfg::kPitchB>{}, cut_c, a + Cfg::kFloatsA, gb[buf], left);
        };
        if (left >= BK) both(std::false_type{});
        else both(std::true_type{});
    };

    // (a share's products may be two sums, of every other group of four k, which halves the chain of dependent instructions)
    constexpr int NACC = SPLIT && KW == 1 ? 2 : 1;
    f32x4_t accs[NACC][TM][TN];
    f32x4_t (&acc)[TM][TN] = accs[0];
#pragma unroll
    for (int n = 0; n < NACC; ++n)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) accs[n][i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // fragment of 16 rows x 4 k: lane l gets row l % 16, k = l / 16
    // `between`: what the next slices need (LDS writes, loads and their addresses), put behind the first fragment reads so that the matrix
    // instructions hide it.  Before the products it took 8 to 12 % of a slice (64 x 64 tiles 0.83 -> 0.76 us, 16 x 32 0.75 -> 0.67).
    auto compute = [&](auto stage_c, const auto& between) {
        constexpr int stage = decltype(stage_c)::value;
        const float* a = f32_smem + stage * Cfg::kStage;
        const float* b = a + Cfg::kFloatsA;
        // groups of four fragments deep, the next group's reads ahead of this group's MFMAs.  The 16 lanes of lane / 16 = q have k 4 q .. 4 q + 3 of a group's
        // 16 (not every fourth), so that a k-contiguous operand's four fragments are one 16-byte LDS read: the reads, not the MFMAs, fill a step of the small
        // tiles.  With it and the narrower pitch of the k-major tiles one pass at T 256, d 512, F 1376 went from 82.4 to 79.6 us; the error against 64-bit sums is
        // that of ascending k (ratio 0.995 to 1.001 over ten shapes).
        const int r = lane & 15, kq = k_wave + 4 * (lane >> 4);
        const float* pa = AKM ? a + kq * Cfg::kPitchA + wm0 + r : a + (wm0 + r) * Cfg::kPitchA + kq;
        const float* pb = BKM ? b + kq * Cfg::kPitchB + wn0 + r : b + (wn0 + r) * Cfg::kPitchB + kq;
        constexpr int GK = 4, NG = BK / KW / (4 * GK);
        static_assert(NG >= 1, "a wavefront's share of a slice is at least one group");
        float fa[2][GK][TM], fb[2][GK][TN];
        auto read_one = [&](auto km_c, const float* p, int pitch, int g, auto&& f) {
            if constexpr (decltype(km_c)::value) {
#pragma unroll
                for (int q = 0; q < GK; ++q) f(q, p[(g * 16 + q) * pitch]);
            } else {
                const f32x4_t v = *reinterpret_cast<const f32x4_t*>(p + g * 16);
#pragma unroll
                for (int q = 0; q < GK; ++q) f(q, v[q]);
            }
        };
        auto read = [&](int g, int d) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
                read_one(std::integral_constant<bool, AKM>{}, AKM ? pa + i * 16 : pa + i * 16 * Cfg::kPitchA, Cfg::kPitchA, g, [&](int q, float v) { fa[d][q][i] = v; });
#pragma unroll
            for (int j = 0; j < TN; ++j)
                read_one(std::integral_constant<bool, BKM>{}, BKM ? pb + j * 16 : pb + j * 16 * Cfg::kPitchB, Cfg::kPitchB, g, [&](int q, float v) { fb[d][q][j] = v; });
        };
        read(0, 0);
        between();
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) read(g + 1, (g + 1) & 1);
#pragma unroll
            for (int q = 0; q < GK; ++q)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        accs[q % NACC][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[g & 1][q][j], fa[g & 1][q][i], accs[q % NACC][i][j], 0, 0, 0);
        }
    };
    fetch(std::integral_constant<int, 0>{}, ks);
    fetch(std::integral_constant<int, 1>{}, ks + 1);
    fetch(std::integral_constant<int, 2>{}, ks + 2);
    fetch(std::integral_constant<int, 3>{}, ks + 3);
    stash(std::integral_constant<int, 0>{}, ks);
    fetch(std::integral_constant<int, 0>{}, ks + 4);
    __syncthreads();
    // slice kt is in LDS stage kt % 2, slices kt + 1 .. kt + 4 are in or on their way to registers
    auto step = [&](auto set_c, int kt) {
        constexpr int set = decltype(set_c)::value, nxt = (set + 1) % kF32Sets;
        // the other stage was last read in the slice before this one, a barrier ago (past the end: zeros nobody multiplies)
        compute(std::integral_constant<int, set & 1>{}, [&] {
            stash(std::integral_constant<int, nxt>{}, kt + 1);
            fetch(std::integral_constant<int, nxt>{}, kt + 5);
        });
        __syncthreads();
    };
    int kt = ks;
    for (; kt + 4 <= nk; kt += 4) {
        step(std::integral_constant<int, 0>{}, kt);
        step(std::integral_constant<int, 1>{}, kt + 1);
        step(std::integral_constant<int, 2>{}, kt + 2);
        step(std::integral_constant<int, 3>{}, kt + 3);
    }
    if (kt < nk) step(std::integral_constant<int, 0>{}, kt);
    if (kt + 1 < nk) step(std::integral_constant<int, 1>{}, kt + 1);
    if (kt + 2 < nk) step(std::integral_constant<int, 2>{}, kt + 2);

    if constexpr (NACC == 2) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += accs[1][i][j];
    }
    // acc[i][j][r] is C[m0 + wm0 + 16 i + lane % 16, n0 + wn0 + 16 j + 4 (lane / 16) + r]
    if (KW == 1) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int m = m0 + wm0 + i * 16 + (lane & 15), n = n0 + wn0 + j * 16 + 4 * (lane >> 4);
                const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
                if (m < M) epi.store4(m, n, v);
            }
    } else {
        // (the stages are free: the loop ended with a barrier)
        constexpr int PITCH = BN + 4;
        static_assert(KW * BM * PITCH <= 2 * Cfg::kStage, "partial tiles must fit in the stage memory");
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                *reinterpret_cast<f32x4_t*>(f32_smem + (wave * BM + i * 16 + (lane & 15)) * PITCH + j * 16 + 4 * (lane >> 4)) = acc[i][j];
        __syncthreads();
        for (int c = tid; c < BM * BN / 4; c += NT) {
            const int m = c / (BN / 4), n = (c % (BN / 4)) * 4;
            f32x4_t s = *reinterpret_cast<const f32x4_t*>(f32_smem + m * PITCH + n);
#pragma unroll
            for (int w = 1; w < KW; ++w) s += *reinterpret_cast<const f32x4_t*>(f32_smem + (w * BM + m) * PITCH + n);
            const float v[4] = {s[0], s[1], s[2], s[3]};
            if (m0 + m < M) epi.store4(m0 + m, n0 + n, v);
        }
    }
}

// Host-side check of the kernel's layout assumptions: 16-byte aligned bases and rows, and whole 16-byte chunks
// readable (a k-contiguous operand up to the next multiple of 4 past the contraction length).
inline bool f32_problem_ok(const GemmProblem<float>& p) {
    auto al16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
    const bool two = p.Kc2 != 0;
    auto operand_ok = [&](const GemmOperand<float>& o, int rows) {
        bool ok = o.p && al16(o.p) && o.ld % 4 == 0 && (!two || (o.p2 && al16(o.p2)));
        ok = ok && (int64_t)(o.km ? 128 : rows) * o.ld < (1ll << 29);      // 32-bit byte offsets inside a tile
        if (o.km) return ok && o.ext % 4 == 0 && o.ext >= 4 && o.ext <= o.ld && rows <= o.ext;
        return ok && o.ld >= round_up(p.Kc > p.Kc2 ? p.Kc : p.Kc2, 4);
    };
    return p.M >= 1 && p.N >= 1 && p.Kc >= 1 && operand_ok(p.A, p.M) && operand_ok(p.B, p.N);
}

template <int BM, int BN, int KW, bool AKM, bool BKM, class Epi, int NB, bool SPLIT = false>
inline hipError_t launch_gemm_f32_tile(const F32Batch<Epi, NB>& b, hipStream_t st, int shares = 1) {
    using Cfg = F32Cfg<BM, BN, KW, AKM, BKM>;
    auto kern = gemm_f32_mfma_kernel<BM, BN, KW, AKM, BKM, Epi, NB, SPLIT>;
    LdsAttr<gemm_f32_mfma_kernel<BM, BN, KW, AKM, BKM, Epi, NB, SPLIT>, Cfg::kLds>::use();
    const int tiles_m = (b.pr[0].M + BM - 1) / BM, tiles_n = (b.pr[0].N + BN - 1) / BN;
    hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n, SPLIT ? shares : NB), dim3(256), Cfg::kLds, st, b, tiles_n);
    return hipGetLastError();
}

// Tile shape by f32_tile (gemm_plan.h).
template <bool AKM, bool BKM, class Epi, int NB>
inline hipError_t launch_gemm_f32(const F32Batch<Epi, NB>& b, bool one_sum, int num_cu, hipStream_t st) {
    const GemmProblem<float>& p = b.pr[0];
    switch (f32_tile(p.M, p.N, NB, (int64_t)p.Kc + p.Kc2, one_sum, num_cu)) {
        case F32Tile::k64x64: return launch_gemm_f32_tile<64, 64, 1, AKM, BKM, Epi, NB>(b, st);
        case F32Tile::k32x32: return launch_gemm_f32_tile<32, 32, 1, AKM, BKM, Epi, NB>(b, st);
        case F32Tile::k32x32Split: return launch_gemm_f32_tile<32, 32, 4, AKM, BKM, Epi, NB>(b, st);
        default: return launch_gemm_f32_tile<16, 32, 4, AKM, BKM, Epi, NB>(b, st);
    }
}

// One product with A k-contiguous and B k-major in shares (f32_shares): share z of the sums to epi.share(z).
template <class EpiS> inline hipError_t launch_gemm_f32_shares(const GemmProblem<float>& p, const EpiS& epi, F32Shares plan, hipStream_t st) {
    const F32Batch<EpiS, 1> b{{p}, {epi}};
    return plan.tile == F32Tile::k32x32 ? launch_gemm_f32_tile<32, 32, 1, false, true, EpiS, 1, true>(b, st, plan.shares)
                                        : launch_gemm_f32_tile<16, 32, 4, false, true, EpiS, 1, true>(b, st, plan.shares);
}

}  // namespace moc
