// Row-wide decode of up to four tokens after the gate: selection and up projection in one launch
// (decode_select_up_kernel), down projection in another (decode_down_cols_kernel), which writes y itself.
//
// What bounds it: at one token of the 7B shape the selected rows are 22.5 MB, 4 us of HBM time; the rest is a chain of
// dependent steps on one gate row.  So the chain is kept short rather than the work small: every workgroup of the first
// kernel finds its token's threshold itself (no launch, no index list between selection and gather), and the down
// projection is split over columns instead of channels, so that no partial outputs go through memory.
#pragma once
#include "decode_kernels.h"
#include "row_cut.h"

namespace moc {

constexpr int kRowsNT = 512;                 // threads of the selection workgroup
constexpr int kRowsMaxRange = 128;           // channels of one workgroup's share
// Workgroup (p, b): finds token b's cut, then u_j = x[b] . wu[j] and z'_j = SiLU(g_j) u_j for the selected channels j of
// the p-th range of channels, a wavefront per channel, and writes (j, z'_j) to their slots of idx[b, :], z[b, :] (slot =
// selected channels before j).  The rank of a range's first slot needs no other workgroup: every workgroup holds the whole
// gate row.  Workgroups of one range are placed on one XCD, whose L2 serves the rows that several tokens selected.
// g holds what is ranked, graw the gate itself (the same array unless the Top-K is keyed).
template <class E, int NCH>
__global__ __launch_bounds__(kRowsNT, NCH <= 6 ? 4 : 2) void decode_select_up_kernel(const E* __restrict__ x, const E* __restrict__ wu,
                                                                   const float* __restrict__ g, const float* __restrict__ graw,
                                                                   int64_t ldg, int F, int d, int K, float far, int P, int B,
                                                                   int32_t* __restrict__ idx, float* __restrict__ z) {
    constexpr int CN = Chunk<E>::N, NIT = 8, NW = kRowsNT / 64;
    __shared__ RowCutLds<kRowsNT> L;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int p, b;
    if (P % 8 == 0) {
        const int slot = blockIdx.x >> 3;
        p = (blockIdx.x & 7) + 8 * (slot / B);
        b = slot % B;
    } else {
        p = blockIdx.x / B;
        b = blockIdx.x % B;
    }
    const int range = (F + P - 1) / P, c0 = min(F, p * range), cn = min(F, c0 + range) - c0;
    const float* grow = g + b * ldg;
    const E* xrow = x + (int64_t)b * d;

    f32x4_t gv[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) gv[c] = *reinterpret_cast<const f32x4_t*>(grow + min(c * 4 * kRowsNT + tid * 4, ((F + 3) & ~3) - 4));
    float own[2], own_raw[2];                                // the range's channels
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        own[q] = grow[min(c0 + q * 64 + lane, F - 1)];
        own_raw[q] = graw[b * ldg + min(c0 + q * 64 + lane, F - 1)];
    }
    float v[NCH][4];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[c][e] = gv[c][e];
        if ((c + 1) * 4 * kRowsNT > F) {                     // only the chunks that reach past the row (uniform)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c * 4 * kRowsNT + tid * 4 + e >= F) v[c][e] = -__builtin_inff();
        }
    }
    const RowCut cut = row_cut<kRowsNT, NCH, true>(v, F, K, far, L, c0);
    const int below = cut.before;
    uint64_t mask[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) mask[q] = __ballot(q * 64 + lane < cn && cut.in(own[q], c0 + q * 64 + lane));
    const int n0 = __popcll(mask[0]), n = n0 + __popcll(mask[1]);
    for (int s = wave; s < n; s += NW) {                     // s-th selected channel of the range
        uint64_t m = s < n0 ? mask[0] : mask[1];
        for (int q = s < n0 ? s : s - n0; q > 0; --q) m &= m - 1;
        const int bit = __ffsll((unsigned long long)m) - 1;
        const int j = c0 + (s < n0 ? 0 : 64) + bit;
        const float gj = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(s < n0 ? own_raw[0] : own_raw[1]), bit));
        const E* wrow = wu + (int64_t)j * d;
        float dot = 0.0f;
        for (int k0 = 0; k0 < d; k0 += 64 * CN * NIT) {
            u32x4_t ru[NIT], xr[NIT];
#pragma unroll
            for (int i = 0; i < NIT; ++i) {
                const int k = k0 + (i * 64 + lane) * CN;
                ru[i] = u32x4_t{0, 0, 0, 0};
                if (k < d) ru[i] = *reinterpret_cast<const u32x4_t*>(wrow + k);
            }
#pragma unroll
            for (int i = 0; i < NIT; ++i) xr[i] = *reinterpret_cast<const u32x4_t*>(xrow + min(k0 + (i * 64 + lane) * CN, d - CN));
#pragma unroll
            for (int i = 0; i < NIT; ++i) dot = Chunk<E>::dot(ru[i], xr[i], dot);
        }
        dot = wave_sum(dot);
        const int slot = below + s;
        if (lane == 0 && slot < K) {
            idx[(int64_t)b * K + slot] = j;
            z[(int64_t)b * K + slot] = silu_f32(gj) * dot;
        }
    }
}

// y[b, c] = sum over token b's selected channels of z[b, s] * wd[idx[b, s], c] for a 64-byte slice of columns c per
// workgroup: four lanes cover a row's segment, a wavefront 16 rows, the workgroup 256 rows at a time, all of a step's loads
// in flight together; row sums meet in registers, then in LDS.  Neighbouring slices (the two halves of a 128-byte line) and
// the tokens of a slice share an XCD.
template <class E>
__global__ __launch_bounds__(1024) void decode_down_cols_kernel(const E* __restrict__ wd, const int32_t* __restrict__ idx,
                                                                const float* __restrict__ z, int d, int F, int K, int slices, int B,
                                                                E* __restrict__ y) {
    constexpr int CN = Chunk<E>::N, U = 4;
    __shared__ float red[16][4 * CN];
    int s, b;
    if (slices % 8 == 0) {
        const int q = blockIdx.x >> 3;
        s = (blockIdx.x & 7) * (slices / 8) + q / B;
        b = q % B;
    } else {
        s = blockIdx.x / B;
        b = blockIdx.x % B;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = (s * 4 + (lane & 3)) * CN;
    const int colc = min(col, d - CN);                       // (a slice that hangs over the edge re-reads the last chunk)
    const int32_t* ib = idx + (int64_t)b * K;
    const float* zb = z + (int64_t)b * K;
    float acc[CN];
#pragma unroll
    for (int e = 0; e < CN; ++e) acc[e] = 0.0f;
    for (int r0 = wave * 16 + (lane >> 2); r0 < K; r0 += 256 * U) {
        int j[U];
        float zz[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = r0 + u * 256;
            j[u] = min((uint32_t)ib[min(r, K - 1)], (uint32_t)(F - 1));      // (every slot holds a channel: the bound only guards the loads)
            zz[u] = r < K ? zb[min(r, K - 1)] : 0.0f;
        }
        u32x4_t w[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u == 0 || r0 + u * 256 < K) w[u] = *reinterpret_cast<const u32x4_t*>(wd + (int64_t)j[u] * d + colc);
            else w[u] = u32x4_t{0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float f[CN];
            Chunk<E>::unpack(w[u], f);
#pragma unroll
            for (int e = 0; e < CN; ++e) acc[e] = fmaf(zz[u], f[e], acc[e]);
        }
    }
#pragma unroll
    for (int o = 4; o < 64; o <<= 1)
#pragma unroll
        for (int e = 0; e < CN; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
    if (lane < 4) {
#pragma unroll
        for (int e = 0; e < CN; ++e) red[wave][lane * CN + e] = acc[e];
    }
    __syncthreads();
    if (tid < 4 * CN && s * 4 * CN + tid < d) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += red[w][tid];
        Elem<E>::store(y + (int64_t)b * d + s * 4 * CN + tid, t);
    }
}

}  // namespace moc
