// Decode path of the MoC layer (row-wide, keyed and grouped selection): kernel sequences and their
// C entry points.
#include "api_common.h"
#include "api_launch.h"
#include <atomic>
#include <random>

#include "decode_dense.h"
#include "decode_kernels.h"
#include "decode_persist.h"
#include "decode_rows.h"
#include "decode_select_gather.h"

using namespace moc;
using namespace mocapi;

namespace {

// ------------------------------------------------------------------------------ decode
template <class E, int BT>
moc_status decode_gate(const Dims& D, const E* x, const E* wg, float* g, hipStream_t st) {
    const size_t lds = (size_t)BT * D.d * sizeof(E);
    if (lds > 160 * 1024 - 64) return fail(MOC_ERR_UNSUPPORTED, "decode: d = %d too large for LDS staging", D.d);
    auto kern = decode_gate_kernel<E, BT>;
    LdsAttr<decode_gate_kernel<E, BT>, kMaxDynLds>::use();
    Span span("decode_gate", st);
    const int per_cu = lds > 80 * 1024 ? 1 : (lds > 40 * 1024 ? 2 : 4);
    const int grid = std::min((D.F + 3) / 4, 256 * per_cu);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, x, wg, D.T, D.d, D.F, g, (int64_t)D.ldF);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

// Gate projection fused with the grouped selection (MoC_{a:b}) on the vector ALU.
template <class E, int BT, int GB>
moc_status decode_gate_group(const Dims& D, const E* x, const E* wg, int ga, int32_t* idx, float* gsel, hipStream_t st) {
    const size_t lds = (size_t)BT * D.d * sizeof(E);
    if (lds > 156 * 1024) return fail(MOC_ERR_UNSUPPORTED, "decode: d = %d too large for LDS staging", D.d);
    auto kern = decode_gate_group_kernel<E, BT, GB>;
    LdsAttr<decode_gate_group_kernel<E, BT, GB>, 156 * 1024>::use();
    Span span("decode_gate_select", st);
    const int per_cu = lds > 76 * 1024 ? 1 : (lds > 36 * 1024 ? 2 : (lds > 16 * 1024 ? 4 : 8));
    const int grid = std::min(D.F / GB, 256 * per_cu);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, x, wg, D.T, D.d, D.F, ga, D.K, idx, gsel);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

template <class E, int BT>
moc_status decode_gate_group_b(const Dims& D, const E* x, const E* wg, int ga, int gb, int32_t* idx, float* gsel,
                               hipStream_t st) {
    if (gb == 4) return decode_gate_group<E, BT, 4>(D, x, wg, ga, idx, gsel, st);
    if (gb == 8) return decode_gate_group<E, BT, 8>(D, x, wg, ga, idx, gsel, st);
    return decode_gate_group<E, BT, 16>(D, x, wg, ga, idx, gsel, st);
}

int gate_stream_workgroups() { return std::max(1, device_cu_count()); }

template <int GB, int NS, bool NT>
moc_status launch_decode_gate_stream_nt(const Dims& D, const bf16_t* x, const bf16_t* wg, float* g, int ga, int32_t* idx, float* gsel,
                                        hipStream_t st) {
    auto kern = decode_gate_stream_kernel<GB, NS, NT>;
    constexpr int lds = GateStreamCfg<GB, NS>::kLds;
    LdsAttr<decode_gate_stream_kernel<GB, NS, NT>, lds>::use();
    Span span(GB == 0 ? "decode_gate" : "decode_gate_select", st);
    const int unit = GB == 0 ? 4 : GB;
    hipLaunchKernelGGL(kern, dim3(std::min(gate_stream_workgroups(), (D.F + unit - 1) / unit)), dim3(kGateStreamWaves * 64), lds, st,
                       x, wg, D.T, D.d, D.F, g, (int64_t)D.ldF, ga, D.K, idx, gsel);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}
template <int GB, int NS>
moc_status launch_decode_gate_stream_ns(const Dims& D, const bf16_t* x, const bf16_t* wg, float* g, int ga, int32_t* idx, float* gsel,
                                        hipStream_t st) {
    return gate_stream_nontemporal(D.d, D.F) ? launch_decode_gate_stream_nt<GB, NS, true>(D, x, wg, g, ga, idx, gsel, st)
                                             : launch_decode_gate_stream_nt<GB, NS, false>(D, x, wg, g, ga, idx, gsel, st);
}
template <int GB>
moc_status launch_decode_gate_stream(const Dims& D, const bf16_t* x, const bf16_t* wg, float* g, int ga, int32_t* idx, float* gsel,
                                     hipStream_t st) {
    const int steps = (D.d / 64 + kGateStreamWaves - 1) / kGateStreamWaves;
    if (steps <= 1) return launch_decode_gate_stream_ns<GB, 1>(D, x, wg, g, ga, idx, gsel, st);
    if (steps <= 2) return launch_decode_gate_stream_ns<GB, 2>(D, x, wg, g, ga, idx, gsel, st);
    if (steps <= 4) return launch_decode_gate_stream_ns<GB, 4>(D, x, wg, g, ga, idx, gsel, st);
    return launch_decode_gate_stream_ns<GB, 8>(D, x, wg, g, ga, idx, gsel, st);
}

// ------------------------------------------------- both projections as streams (decode_dense.h)
constexpr int kSelectUpMaxLds = 156 * 1024;      // (the kernel has up to 512 bytes of static LDS)
template <int NCH, int NS, bool NT>
moc_status launch_select_up_stream(const Dims& D, const TopkArgs<float>& a, const bf16_t* x, const bf16_t* wu, float* u, uint32_t* arrived, hipStream_t st) {
    auto kern = decode_select_up_stream_kernel<NCH, NS, NT>;
    LdsAttr<decode_select_up_stream_kernel<NCH, NS, NT>, kSelectUpMaxLds>::use();
    const size_t lds = std::max((size_t)GateStreamCfg<0, NS>::kLds, NCH > 0 ? topk_reg_dyn_lds(D.K, 0, sizeof(float), false) : 0);
    Span span("decode_select_up_stream", st);
    hipLaunchKernelGGL(kern, dim3(D.T + std::min(std::max(1, gate_stream_workgroups() - D.T), (D.F + 3) / 4)), dim3(kGateStreamWaves * 64), lds, st,
                       a, x, wu, D.T, D.d, u, arrived);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}
template <int NCH, int NS>
moc_status launch_select_up_stream_nt(const Dims& D, const TopkArgs<float>& a, const bf16_t* x, const bf16_t* wu, float* u, uint32_t* arrived, hipStream_t st) {
    return gate_stream_nontemporal(D.d, D.F) ? launch_select_up_stream<NCH, NS, true>(D, a, x, wu, u, arrived, st)
                                             : launch_select_up_stream<NCH, NS, false>(D, a, x, wu, u, arrived, st);
}
template <int NCH>
moc_status launch_select_up_stream_ns(const Dims& D, const TopkArgs<float>& a, const bf16_t* x, const bf16_t* wu, float* u, uint32_t* arrived, hipStream_t st) {
    const int steps = (D.d / 64 + kGateStreamWaves - 1) / kGateStreamWaves;
    if (steps <= 1) return launch_select_up_stream_nt<NCH, 1>(D, a, x, wu, u, arrived, st);
    if (steps <= 2) return launch_select_up_stream_nt<NCH, 2>(D, a, x, wu, u, arrived, st);
    if (steps <= 4) return launch_select_up_stream_nt<NCH, 4>(D, a, x, wu, u, arrived, st);
    return launch_select_up_stream_nt<NCH, 8>(D, a, x, wu, u, arrived, st);
}
// Slices of 64 columns (kDownNarrowMaxD) where those of 128 would need many ranges, whose shares are added: d 512 6.8 us against 9.2, 2048 12.3 against 15.1;
// at 4096 the twice as many slices read SiLU(g) and u twice as often, 30.0 against 24.8.
static_assert(kDownNarrowMaxD <= kDownArrived * DownStreamCfg<4>::kCols && kGateStreamMaxD <= kDownArrived * DownStreamCfg<8>::kCols, "a counter to a slice");
static_assert(kDownArrived * sizeof(uint32_t) <= kDecodeArrivedBytes, "workspace reserve for the counters");
template <int CT, bool NT>
moc_status launch_down_stream(const Dims& D, const DecodeWs& W, const bf16_t* wd, bf16_t* y, hipStream_t st) {
    auto kern = decode_down_stream_kernel<CT, NT>;
    LdsAttr<decode_down_stream_kernel<CT, NT>, DownStreamCfg<CT>::kLds>::use();
    Span span("decode_down_stream", st);
    const int slices = (D.d + 16 * CT - 1) / (16 * CT);
    const int P = down_stream_ranges(D.T, D.d, D.F, D.K, gate_stream_workgroups());
    const int per = round_up((D.F + 4 * P - 1) / (4 * P), 4);
    hipLaunchKernelGGL(kern, dim3(P, slices), dim3(256), DownStreamCfg<CT>::kLds, st, W.sd, W.ud, (int64_t)D.ldF, wd, D.T, D.d, D.F, per, W.part,
                       W.arrived, y);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}
// After the gate: selection (row-wide; grouped selection happened in the gate) and up projection, then the down projection, which adds its own shares.
moc_status decode_dense(const Dims& D, const DecodeWs& W, const bf16_t* x, const bf16_t* wu, const bf16_t* wd, bf16_t* y, int32_t* idx, int gb,
                        int key_mode, hipStream_t st) {
    moc_status s;
    // (gsel is what grouped selection has left; a row's selection leaves SiLU(g) only)
    TopkArgs<float> a{W.g, D.ldF, D.F, D.K, idx, gb != 0 ? W.gsel : nullptr, nullptr, nullptr, 0, nullptr, nullptr, 0, nullptr, cut_far(D.F, D.K), W.sd};
    if (gb != 0) {
        s = launch_select_up_stream_ns<0>(D, a, x, wu, W.ud, W.arrived, st);
    } else {
        if (key_mode != 0) {
            if ((s = launch_key_transform(W.g, W.gkeys, (int64_t)D.T * D.ldF, key_mode, st)) != MOC_OK) return s;
            a.g = W.gkeys;
            a.g_raw = W.g;
        }
        constexpr int kChunk = 4 * kGateStreamWaves * 64;
        if (D.F <= 3 * kChunk) s = launch_select_up_stream_ns<3>(D, a, x, wu, W.ud, W.arrived, st);
        else if (D.F <= 6 * kChunk) s = launch_select_up_stream_ns<6>(D, a, x, wu, W.ud, W.arrived, st);
        else s = launch_select_up_stream_ns<16>(D, a, x, wu, W.ud, W.arrived, st);
    }
    if (s != MOC_OK) return s;
    if (D.d <= kDownNarrowMaxD) return gate_stream_nontemporal(D.d, D.F) ? launch_down_stream<4, true>(D, W, wd, y, st) : launch_down_stream<4, false>(D, W, wd, y, st);
    return gate_stream_nontemporal(D.d, D.F) ? launch_down_stream<8, true>(D, W, wd, y, st) : launch_down_stream<8, false>(D, W, wd, y, st);
}

template <class E, int BT, int GA>
moc_status launch_decode_fused_t(const Dims& D, const E* x, const E* wg, const E* wu, const E* wd, int32_t* idx,
                                 float* part, int P, hipStream_t st) {
    const size_t lds = (size_t)BT * D.d * sizeof(E);
    auto kern = decode_fused_group_kernel<E, BT, GA>;
    LdsAttr<decode_fused_group_kernel<E, BT, GA>, 64 * 1024>::use();
    Span span("decode_fused_gate_select_gather", st);
    hipLaunchKernelGGL(kern, dim3(P), dim3(512), lds, st, x, wg, wu, wd, D.T, D.d, D.F, D.K, idx, part);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

template <class E>
moc_status launch_decode_fused(const Dims& D, const E* x, const E* wg, const E* wu, const E* wd, int ga, int32_t* idx,
                               float* part, int P, hipStream_t st) {
    if (ga == 1) return launch_decode_fused_t<E, 1, 1>(D, x, wg, wu, wd, idx, part, P, st);
    return launch_decode_fused_t<E, 1, 2>(D, x, wg, wu, wd, idx, part, P, st);
}

// ------------------------------------------------------- row-wide decode in one persistent launch
static_assert(sizeof(DecodeSync) <= kDecodeArrivedAt, "workspace reserve for the decode flags");

// Host call counter that makes the flag epochs of different calls differ (decode_persist.h); seeded
// randomly so that flags left in reused memory by another process cannot match either.
std::atomic<uint32_t> g_decode_salt{std::random_device{}()};

constexpr int kPersistentDynLds = 158 * 1024;      // the persistent kernels also hold about 1.2 KB of static LDS

struct DecodePlan {
    bool ok = false;
    int variant = 0;              // 0: row per wavefront, one token; 1: row per wavefront, up to 4; 2: MFMA gate, up to 16
    int nt = 0, nch = 0, bt = 0;
    int nwg = 0, P = 1, C = 1, rmax = 1;
    int off_own = 0, off_over = 0;
    size_t lds = 0;
};

// The single-launch kernel serves the row-wide Top-K on the raw gate when the shape fits its
// assumptions (whole weight rows in registers, the gate row of a token in one workgroup's registers,
// 16-byte column segments); everything else stays on the separate launches.
template <class E>
DecodePlan plan_persistent(const Dims& D, int num_cu) {
    DecodePlan pl;
    constexpr int CN = Chunk<E>::N;
    const int B = D.T, d = D.d, F = D.F;
    const bool bf16 = std::is_same<E, bf16_t>::value;
    if (num_cu < kDecMaxB || options().force_generic || !options().decode_persistent) return pl;   // workgroup b selects for token b
    if (d % CN != 0 || d > 64 * CN * 8) return pl;
    if (B <= 4) {
        pl.variant = B == 1 ? 0 : 1;
        pl.bt = B == 1 ? 1 : 4;
        pl.nt = 1024;
    } else {
        if (!bf16 || d % 1024 != 0) return pl;
        pl.variant = 2;
        pl.bt = 16;
        pl.nt = 768;
    }
    const int nwv = pl.nt / 64;
    const int nch = (F + pl.nt * 4 - 1) / (pl.nt * 4);
    pl.nch = nch <= 3 ? 3 : (nch <= 4 ? 4 : 8);
    if (nch > 8) return pl;
    pl.nwg = std::min(num_cu, kDecMaxWG);
    // x, own gate values, phase-overlaid area
    const size_t xbytes = pl.variant == 2 ? (size_t)16 * (d * 2 + 16) : (size_t)pl.bt * d * sizeof(E);
    size_t own;
    if (pl.variant == 2) {
        const int nblk = (F + 47) / 48;
        pl.rmax = (nblk + pl.nwg - 1) / pl.nwg;
        own = (size_t)pl.rmax * 48 * 17 * sizeof(float);
    } else {
        pl.rmax = (F + pl.nwg * nwv - 1) / (pl.nwg * nwv);
        own = (size_t)nwv * pl.rmax * pl.bt * sizeof(float);
    }
    pl.off_own = (int)round_up_sz(xbytes, 16);
    pl.off_over = (int)round_up_sz(pl.off_own + own, 16);
    const size_t over = std::max(kDecSelLds, pl.variant == 2 ? (size_t)12 * 256 * sizeof(float) : (size_t)0);
    // down projection: C column slices of LPR 16-byte chunks each, P channel ranges
    const int total = (int)((size_t)d * sizeof(E) / 16);
    const int tb = pl.bt > 8 ? 8 : pl.bt;
    int best_lpr = 0;
    size_t best_vol = 0;
    bool best_good = false;
    for (int lpr = 64; lpr >= 1; lpr >>= 1) {
        if (total % lpr != 0) continue;
        const int C = total / lpr;
        if (C > pl.nwg) continue;
        // the last B workgroups write the index lists: they get no share of the down projection if possible
        const int P = std::max(1, std::min(std::max(pl.nwg - B, C) / C, F));
        const int seg = d / C;
        const size_t vol = (size_t)P * B * d * sizeof(float), last = (size_t)P * B * seg * sizeof(float);
        const size_t dl = round_up_sz(((size_t)(F + P - 1) / P + 1) * 8, 16) + (size_t)nwv * tb * seg * sizeof(float);
        if (dl > (size_t)kPersistentDynLds || vol > kDecodePartBudget) continue;
        const bool good = last <= 96 * 1024;
        if (best_lpr == 0 || (good && !best_good) || (good == best_good && !good && vol < best_vol)) {
            if (best_lpr != 0 && best_good) continue;        // keep the first (widest) good split
            best_lpr = lpr; best_vol = vol; best_good = good;
        }
    }
    if (best_lpr == 0) return pl;
    pl.C = total / best_lpr;
    pl.P = std::max(1, std::min(std::max(pl.nwg - B, pl.C) / pl.C, F));
    const size_t dl = round_up_sz(((size_t)(F + pl.P - 1) / pl.P + 1) * 8, 16) + (size_t)nwv * tb * (d / pl.C) * sizeof(float);
    // more than half of a compute unit's LDS, so that the dispatcher places one workgroup per unit
    pl.lds = std::max(std::max((size_t)pl.off_over + over, dl), (size_t)84 * 1024);
    if (pl.lds > (size_t)kPersistentDynLds) return pl;
    pl.ok = true;
    return pl;
}

template <class E, int BT, int NCH>
moc_status launch_persistent_rows(const DecodePlan& pl, const DecArgs<E>& a, hipStream_t st) {
    auto kern = decode_persistent_kernel<E, BT, 1024, NCH>;
    LdsAttr<decode_persistent_kernel<E, BT, 1024, NCH>, kPersistentDynLds>::use();
    Span span("decode_persistent", st);
    hipLaunchKernelGGL(kern, dim3(pl.nwg), dim3(1024), pl.lds, st, a);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

template <int NCH>
moc_status launch_persistent_mfma(const DecodePlan& pl, const DecArgs<bf16_t>& a, hipStream_t st) {
    auto kern = decode_persistent_mfma_kernel<NCH>;
    LdsAttr<decode_persistent_mfma_kernel<NCH>, kPersistentDynLds>::use();
    Span span("decode_persistent", st);
    hipLaunchKernelGGL(kern, dim3(pl.nwg), dim3(768), pl.lds, st, a);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

template <class E>
moc_status decode_persistent(const DecodePlan& pl, const Dims& D, const DecodeWs& W, const E* x, const E* wg, const E* wu,
                             const E* wd, E* y, int32_t* idx, hipStream_t st) {
    DecArgs<E> a;
    a.x = x; a.wg = wg; a.wu = wu; a.wd = wd; a.y = y; a.idx = idx;
    a.B = D.T; a.d = D.d; a.F = D.F; a.K = D.K; a.ldF = D.ldF;
    a.g2 = W.g2; a.zt = W.zt; a.part = W.part2;
    a.sync = static_cast<DecodeSync*>(W.sync);
    a.salt = g_decode_salt.fetch_add(1, std::memory_order_relaxed);
    a.P = pl.P; a.C = pl.C; a.rmax = pl.rmax; a.off_own = pl.off_own; a.off_over = pl.off_over;
    if (pl.variant == 0)
        return pl.nch == 3   ? launch_persistent_rows<E, 1, 3>(pl, a, st)
               : pl.nch == 4 ? launch_persistent_rows<E, 1, 4>(pl, a, st)
                             : launch_persistent_rows<E, 1, 8>(pl, a, st);
    if (pl.variant == 1)
        return pl.nch == 3   ? launch_persistent_rows<E, 4, 3>(pl, a, st)
               : pl.nch == 4 ? launch_persistent_rows<E, 4, 4>(pl, a, st)
                             : launch_persistent_rows<E, 4, 8>(pl, a, st);
    if constexpr (std::is_same<E, bf16_t>::value)
        return pl.nch == 3   ? launch_persistent_mfma<3>(pl, a, st)
               : pl.nch == 4 ? launch_persistent_mfma<4>(pl, a, st)
                             : launch_persistent_mfma<8>(pl, a, st);
    return fail(MOC_ERR_UNSUPPORTED, "decode: no single-launch kernel for this shape");
}

// ga:gb = 0:0 is the row-wide Top-K; otherwise the grouped selection of MoC_{a:b}, which is decided
// inside the gate kernel (a group's channels meet in one workgroup) and needs no selection launch.
// Selection + gather of row-wide decode in one launch (decode_select_gather.h).
constexpr int kSelectGatherMaxLds = 156 * 1024;
template <class E, int NCH>
moc_status launch_select_gather_nch(const Dims& D, const E* x, const E* wu, const E* wd, const float* g, int32_t* idx, float* part,
                                    int P, hipStream_t st) {
    constexpr int NIT = 8;
    auto kern = decode_select_gather_kernel<E, NIT, NCH>;
    LdsAttr<decode_select_gather_kernel<E, NIT, NCH>, kSelectGatherMaxLds>::use();      // (the kernel has 160 bytes of static LDS)
    Span span("decode_select_gather", st);
    hipLaunchKernelGGL(kern, dim3(P * D.T), dim3(512), decode_select_gather_lds<E>(D.d), st, x, wu, wd, g, (int64_t)D.ldF, D.F, D.d,
                       D.K, P, D.T, idx, part);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}
template <class E>
moc_status launch_select_gather(const Dims& D, const E* x, const E* wu, const E* wd, const float* g, int32_t* idx, float* part, int P,
                                hipStream_t st) {
    if (D.F <= 2 * 2048) return launch_select_gather_nch<E, 2>(D, x, wu, wd, g, idx, part, P, st);
    if (D.F <= 6 * 2048) return launch_select_gather_nch<E, 6>(D, x, wu, wd, g, idx, part, P, st);
    return launch_select_gather_nch<E, 16>(D, x, wu, wd, g, idx, part, P, st);
}

// Selection + up projection, then the down projection, of row-wide decode (decode_rows.h).
template <class E, int NCH>
moc_status launch_select_up_nch(const Dims& D, const E* x, const E* wu, const float* g, const float* graw, int P, int32_t* idx,
                                float* z, hipStream_t st) {
    Span span("decode_select_up", st);
    hipLaunchKernelGGL((decode_select_up_kernel<E, NCH>), dim3(P * D.T), dim3(kRowsNT), 0, st, x, wu, g, graw, (int64_t)D.ldF, D.F, D.d, D.K,
                       cut_far(D.F, D.K), P, D.T, idx, z);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}
template <class E>
moc_status launch_down_cols(const Dims& D, const E* wd, const int32_t* idx, const float* z, E* y, hipStream_t st) {
    Span span("decode_down", st);
    const int slices = (D.d * (int)sizeof(E) + 63) / 64;
    hipLaunchKernelGGL((decode_down_cols_kernel<E>), dim3(slices * D.T), dim3(1024), 0, st, wd, idx, z, D.d, D.F, D.K, slices, D.T, y);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}
// Whether up to four tokens take the three launches: they save the selection's and the partial outputs' time, while the gather of
// decode_updown_kernel, both rows of a channel in flight together, streams faster and serves a channel that several tokens selected from L2.
// Measured over d 512, 1024, 2048, 4096, 8192 (F of 8/3 d, 8192 at the last), both types, one to four tokens, K/F of 1/50 .. 1, as time of
// this / gather: one token K/F 1/4 0.83 .. 0.93 (fused gather), 1/2 0.84 .. 1.00, 3/4 0.86 .. 1.23; two to four tokens 1/4 0.83 .. 1.01,
// 1/2 0.87 .. 1.21, 3/4 0.85 .. 1.38.  Below 8.5 MB of selected rows the launches decide (0.78 .. 0.98 up to 3/4; K = F has a selection
// of its own, 1.02 .. 1.10).  Against the gather in two launches (rows too long for the fused one): 0.75 .. 1.05 up to 16 KB a row, for
// longer rows 0.84 .. 1.03 at 1/8 and 0.98 .. 1.13 at 1/4.
template <class E> bool decode_rows_pays(const Dims& D, bool gather_fused) {
    const int64_t row = D.d * (int64_t)sizeof(E);
    if (D.T > 4) return false;
    if (!gather_fused) return row <= 16384 || 5 * D.K <= D.F;
    if (2 * D.T * D.K * row <= 8500000 && D.K < D.F) return true;
    return D.T == 1 ? 2 * D.K <= D.F : 3 * D.K <= D.F;
}
template <class E>
moc_status decode_rows(const Dims& D, const DecodeWs& W, const E* x, const E* wu, const E* wd, E* y, int32_t* idx, int key_mode,
                       hipStream_t st) {
    // ranges of channels: about five selected channels for the eight wavefronts of a workgroup, and one workgroup per compute unit over
    // all tokens (two slow each other down: 25.0 against 23.8 us for three tokens at 2048 x 5461) unless the ranges would become too long
    int P = std::min((D.K + 4) / 5, 256 / D.T);
    P = std::max(P, (D.F + kRowsMaxRange - 1) / kRowsMaxRange);
    if (P > 8) P = round_up(P, 8);
    moc_status s;
    const float* g = W.g;
    if (key_mode != 0) {
        if ((s = launch_key_transform(W.g, W.gkeys, (int64_t)D.T * D.ldF, key_mode, st)) != MOC_OK) return s;
        g = W.gkeys;
    }
    const int nch = (D.F + 4 * kRowsNT - 1) / (4 * kRowsNT);
    if (nch <= 1) s = launch_select_up_nch<E, 1>(D, x, wu, g, W.g, P, idx, W.z, st);
    else if (nch <= 2) s = launch_select_up_nch<E, 2>(D, x, wu, g, W.g, P, idx, W.z, st);
    else if (nch <= 3) s = launch_select_up_nch<E, 3>(D, x, wu, g, W.g, P, idx, W.z, st);
    else if (nch <= 6) s = launch_select_up_nch<E, 6>(D, x, wu, g, W.g, P, idx, W.z, st);
    else s = launch_select_up_nch<E, 16>(D, x, wu, g, W.g, P, idx, W.z, st);
    if (s != MOC_OK) return s;
    return launch_down_cols<E>(D, wd, idx, W.z, y, st);
}

template <class E>
moc_status decode_impl(const Dims& D, const E* x, const E* wg, const E* wu, const E* wd, E* y, int32_t* idx_out,
                       void* ws, hipStream_t st, int ga = 0, int gb = 0, int key_mode = 0) {
    DecodeWs W(ws, D);
    const int B = D.T;
    int32_t* idx = idx_out ? idx_out : W.idx;
    moc_status s;
    // the gather stage stages one token's x in LDS: refuse a d it cannot hold before anything is launched
    // (the gate stage checks its own staging in its launcher, which is the first launch)
    constexpr int NIT = 8;
    const size_t fused_lds = (size_t)D.d * sizeof(E) + (size_t)8 * D.d * sizeof(float);
    const bool gather_fused = D.d <= 64 * Chunk<E>::N * NIT && fused_lds <= 160 * 1024 - 64;
    if (!gather_fused && (size_t)D.d * sizeof(E) > 64 * 1024) return fail(MOC_ERR_UNSUPPORTED, "decode: d = %d too large", D.d);
    if (gb == 0 && key_mode == 0) {
        // row-wide Top-K on the raw gate: gate, selection, up and down projection in one launch
        const DecodePlan pl = plan_persistent<E>(D, device_cu_count());
        if (pl.ok) return decode_persistent<E>(pl, D, W, x, wg, wu, wd, y, idx, st);
    }
    // MOC_DECODE_FUSED=0 keeps grouped decode on the separate gate+select and gather launches;
    // MOC_DECODE_FUSED_P=n sets the workgroup count of the single-launch kernel.
    if (gb == 8 && (ga == 1 || ga == 2) && B == 1 && D.d <= 8 * 64 * Chunk<E>::N && options().decode_fused &&
        !options().force_generic) {
        // MoC_{a:8}, one token: gate, selection and gather in one launch, then the deterministic
        // reduction.  Two workgroups are resident per CU; the groups are dealt out evenly.
        const int ngroups = D.F / 8;
        const int rounds = (ngroups + kDecodeFusedMaxP - 1) / kDecodeFusedMaxP;
        const int want = options().decode_fused_p > 0 ? options().decode_fused_p : (ngroups + rounds - 1) / rounds;
        const int P = std::min(ngroups, std::max(1, std::min(kDecodeFusedMaxP, want)));
        if ((s = launch_decode_fused<E>(D, x, wg, wu, wd, ga, idx, W.part, P, st)) != MOC_OK) return s;
        Span span("decode_reduce", st);
        const int64_t n = (int64_t)B * D.d;
        hipLaunchKernelGGL((decode_reduce_kernel<E>), dim3((unsigned)((n + 63) / 64)), dim3(1024), 0, st, W.part, P, n, y);
        HIP_TRY(hipGetLastError());
        return MOC_OK;
    }
    // bf16 from two tokens on: the streamed gate on the matrix cores where gate_stream_pays says so.
    const bool gate_stream = std::is_same<E, bf16_t>::value && !options().force_generic && D.d % 64 == 0 && D.d <= kGateStreamMaxD &&
                             gate_stream_pays(B, D.d, D.F, gb != 0, gate_stream_workgroups());
    const bool dense = gate_stream && !options().decode_select_gather && decode_dense_pays(B, D.d, D.F, D.K, gb != 0) &&
                       (gb != 0 || topk_reg_dyn_lds(D.K, 0, sizeof(float), false) <= (size_t)kSelectUpMaxLds);
    if (gate_stream) {
        const bf16_t* xb = reinterpret_cast<const bf16_t*>(x);
        const bf16_t* wb = reinterpret_cast<const bf16_t*>(wg);
        if (gb == 0) s = launch_decode_gate_stream<0>(D, xb, wb, W.g, 0, idx, W.gsel, st);
        else if (gb == 4) s = launch_decode_gate_stream<4>(D, xb, wb, W.g, ga, idx, W.gsel, st);
        else if (gb == 8) s = launch_decode_gate_stream<8>(D, xb, wb, W.g, ga, idx, W.gsel, st);
        else s = launch_decode_gate_stream<16>(D, xb, wb, W.g, ga, idx, W.gsel, st);
    } else if (gb == 0) {
        if (B == 1) s = decode_gate<E, 1>(D, x, wg, W.g, st);
        else if (B <= 4) s = decode_gate<E, 4>(D, x, wg, W.g, st);
        else s = decode_gate<E, 16>(D, x, wg, W.g, st);
    } else {
        if (B == 1) s = decode_gate_group_b<E, 1>(D, x, wg, ga, gb, idx, W.gsel, st);
        else if (B <= 4) s = decode_gate_group_b<E, 4>(D, x, wg, ga, gb, idx, W.gsel, st);
        else s = decode_gate_group_b<E, 16>(D, x, wg, ga, gb, idx, W.gsel, st);
    }
    if (s != MOC_OK) return s;
    if constexpr (std::is_same<E, bf16_t>::value)
        if (dense) return decode_dense(D, W, x, wu, wd, y, idx, gb, key_mode, st);
    if (gb == 0 && decode_rows_pays<E>(D, gather_fused) && !options().decode_select_gather) return decode_rows<E>(D, W, x, wu, wd, y, idx, key_mode, st);
    const int P = decode_splits(B, D.K);
    if (gb == 0 && key_mode == 0 && gather_fused && options().decode_select_gather && (D.F + P - 1) / P <= kDsgMaxRange &&
        decode_select_gather_lds<E>(D.d) <= (size_t)kSelectGatherMaxLds) {
        // selection and gather in one launch: every workgroup finds its token's threshold itself
        if ((s = launch_select_gather<E>(D, x, wu, wd, W.g, idx, W.part, P, st)) != MOC_OK) return s;
        Span span("decode_reduce", st);
        const int64_t n = (int64_t)B * D.d;
        hipLaunchKernelGGL((decode_reduce_kernel<E>), dim3((unsigned)((n + 63) / 64)), dim3(1024), 0, st, W.part, P, n, y);
        HIP_TRY(hipGetLastError());
        return MOC_OK;
    }
    if (gb == 0) {
        TopkArgs<float> a{W.g, D.ldF, D.F, D.K, idx, W.gsel, nullptr, nullptr, 0, nullptr, nullptr, 0, nullptr};
        if (key_mode != 0) {
            if ((s = launch_key_transform(W.g, W.gkeys, (int64_t)B * D.ldF, key_mode, st)) != MOC_OK) return s;
            a.g = W.gkeys;
            a.g_raw = W.g;
        }
        if ((s = run_topk<float, 1024, false>("decode_topk", a, B, st)) != MOC_OK) return s;
    }
    if (gather_fused) {
        auto kern = B > 1 ? decode_updown_kernel<E, NIT, true> : decode_updown_kernel<E, NIT, false>;
        LdsAttr<decode_updown_kernel<E, NIT, true>, kMaxDynLds>::use();
        LdsAttr<decode_updown_kernel<E, NIT, false>, kMaxDynLds>::use();
        Span span("decode_updown", st);
        hipLaunchKernelGGL(kern, dim3(P * B), dim3(512), fused_lds, st, x, wu, wd, idx, W.gsel, D.d, D.K, P, B, W.part);
        HIP_TRY(hipGetLastError());
    } else {
        {
            const size_t lds = (size_t)D.d * sizeof(E);
            Span span("decode_up", st);
            const int gx = std::max(1, std::min((D.K + 3) / 4, 1024 / B));
            hipLaunchKernelGGL((decode_up_kernel<E>), dim3(gx, B), dim3(256), lds, st, x, wu, idx, W.gsel, D.d, D.K, W.z);
            HIP_TRY(hipGetLastError());
        }
        Span span("decode_down", st);
        constexpr int SLICE = 64 * Chunk<E>::N * 4;
        hipLaunchKernelGGL((decode_down_kernel<E, 4>), dim3(P, B, (D.d + SLICE - 1) / SLICE), dim3(256), 0, st, wd, idx,
                           W.z, D.d, D.K, P, W.part);
        HIP_TRY(hipGetLastError());
    }
    {
        Span span("decode_reduce", st);
        const int64_t n = (int64_t)B * D.d;
        hipLaunchKernelGGL((decode_reduce_kernel<E>), dim3((unsigned)((n + 63) / 64)), dim3(1024), 0, st, W.part, P, n,
                           y);
        HIP_TRY(hipGetLastError());
    }
    return MOC_OK;
}

}  // namespace

extern "C" {

moc_status moc_ffn_decode(const moc_shape* shape, const void* x, const void* wg, const void* wu, const void* wd,
                          void* y, int32_t* idx_or_null, void* ws, size_t ws_bytes, void* hip_stream) {
    moc_status s = check_shape(shape, true);
    if (s != MOC_OK) return s;
    CHECK_PTR(x); CHECK_PTR(wg); CHECK_PTR(wu); CHECK_PTR(wd); CHECK_PTR(y);
    if (idx_or_null && !aligned16(idx_or_null)) return fail(MOC_ERR_BAD_ARG, "idx is not 16-byte aligned");
    CHECK_WS(MOC_OP_DECODE);
    Dims D(*shape);
    MOC_SETUP();
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (shape->dtype == MOC_BF16)
        return decode_impl<bf16_t>(D, (const bf16_t*)x, (const bf16_t*)wg, (const bf16_t*)wu, (const bf16_t*)wd,
                                   (bf16_t*)y, idx_or_null, ws, st);
    return decode_impl<float>(D, (const float*)x, (const float*)wg, (const float*)wu, (const float*)wd, (float*)y,
                              idx_or_null, ws, st);
}

moc_status moc_ffn_decode_static(const moc_shape* shape, const void* x, const void* wg, const void* wu, const void* wd,
                                 void* y, int32_t* idx_or_null, void* hip_stream) {
    moc_status s = check_shape(shape, true);
    if (s != MOC_OK) return s;
    CHECK_PTR(x); CHECK_PTR(wg); CHECK_PTR(wu); CHECK_PTR(wd); CHECK_PTR(y);
    if (idx_or_null && !aligned16(idx_or_null)) return fail(MOC_ERR_BAD_ARG, "idx is not 16-byte aligned");
    const size_t need = moc_workspace_bytes(shape, MOC_OP_DECODE);
    if (need > kStaticScratchBytes)
        return fail(MOC_ERR_UNSUPPORTED, "decode scratch for this shape is %zu bytes, the static buffer holds %zu", need,
                    kStaticScratchBytes);
    void* ws = nullptr;                     // this device's copy of the static scratch array
    if ((s = ensure_init(&ws)) != MOC_OK) return s;
    Dims D(*shape);
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (shape->dtype == MOC_BF16)
        return decode_impl<bf16_t>(D, (const bf16_t*)x, (const bf16_t*)wg, (const bf16_t*)wu, (const bf16_t*)wd,
                                   (bf16_t*)y, idx_or_null, ws, st);
    return decode_impl<float>(D, (const float*)x, (const float*)wg, (const float*)wu, (const float*)wd, (float*)y,
                              idx_or_null, ws, st);
}

moc_status moc_ffn_decode_keyed(const moc_shape* shape, int32_t key_mode, const void* x, const void* wg, const void* wu,
                                const void* wd, void* y, int32_t* idx_or_null, void* ws, size_t ws_bytes, void* hip_stream) {
    moc_status s = check_shape(shape, true);
    if (s != MOC_OK) return s;
    if ((s = check_key_mode(key_mode)) != MOC_OK) return s;
    CHECK_PTR(x); CHECK_PTR(wg); CHECK_PTR(wu); CHECK_PTR(wd); CHECK_PTR(y);
    if (idx_or_null && !aligned16(idx_or_null)) return fail(MOC_ERR_BAD_ARG, "idx is not 16-byte aligned");
    CHECK_WS(MOC_OP_DECODE);
    Dims D(*shape);
    MOC_SETUP();
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (shape->dtype == MOC_BF16)
        return decode_impl<bf16_t>(D, (const bf16_t*)x, (const bf16_t*)wg, (const bf16_t*)wu, (const bf16_t*)wd,
                                   (bf16_t*)y, idx_or_null, ws, st, 0, 0, key_mode);
    return decode_impl<float>(D, (const float*)x, (const float*)wg, (const float*)wu, (const float*)wd, (float*)y,
                              idx_or_null, ws, st, 0, 0, key_mode);
}

moc_status moc_ffn_decode_grouped(const moc_shape* shape, int32_t ga, int32_t gb, const void* x, const void* wg,
                                  const void* wu, const void* wd, void* y, int32_t* idx_or_null, void* ws,
                                  size_t ws_bytes, void* hip_stream) {
    moc_status s = check_shape(shape, true);
    if (s != MOC_OK) return s;
    if ((s = check_group(shape->F, shape->K, ga, gb)) != MOC_OK) return s;
    CHECK_PTR(x); CHECK_PTR(wg); CHECK_PTR(wu); CHECK_PTR(wd); CHECK_PTR(y);
    if (idx_or_null && !aligned16(idx_or_null)) return fail(MOC_ERR_BAD_ARG, "idx is not 16-byte aligned");
    CHECK_WS(MOC_OP_DECODE);
    Dims D(*shape);
    MOC_SETUP();
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (shape->dtype == MOC_BF16)
        return decode_impl<bf16_t>(D, (const bf16_t*)x, (const bf16_t*)wg, (const bf16_t*)wu, (const bf16_t*)wd,
                                   (bf16_t*)y, idx_or_null, ws, st, ga, gb);
    return decode_impl<float>(D, (const float*)x, (const float*)wg, (const float*)wu, (const float*)wd, (float*)y,
                              idx_or_null, ws, st, ga, gb);
}

}  // extern "C"
