// Decode of so many tokens that together they request most channels several times: the up and the down projection stream their whole
// matrices once for all tokens, as products on the matrix cores, instead of gathering every token's rows (decode_dense_pays, gemm_plan.h).
//
// Bound: the streams of W_up and W_down.  The gather (decode_updown_kernel) requests a row once per token that selected it: with 16 tokens
// and K = F/8 twice the bytes of both matrices, of which L2 absorbs a third.  Two launches after the gate:
//  - u = x W_up for every channel, on the walk of the streamed gate; as it does not need the selection, the row Top-K of all tokens runs
//    beside it in workgroups of its own.  These leave SiLU(g) of every channel, or kNotSelected, in a dense row;
//  - y = Z' W_down (decode_down_stream_kernel), which adds its own shares.
// 4096 x 11008, 16 tokens, K = F/8, us of a profile: selection 8.7 + gather 42.1 + sum 4.7 -> 19.1 + 24.8, the call 73.4 -> 62.3; K = F/5 82.8 ->
// 62.3, 2:8 77.9 -> 64.2, K = F 185.6 -> 62.8; 2048 x 5461, K = F/8 33.6 -> 30.8.
#pragma once
#include "decode_kernels.h"
#include "gemm_mfma.h"
#include "topk.h"

namespace moc {

// Workgroups 0 .. B - 1: the row of token blockIdx.x (row Top-K; NCH = 0, grouped selection, which the gate has made: from idx and gsel); the
// others: u.  Also clears the counters of the next launch.
constexpr int kDownArrived = 64;
template <int NCH, int NS, bool NT>
__global__ __launch_bounds__(kGateStreamWaves * 64, 2) void decode_select_up_stream_kernel(TopkArgs<float> a, const bf16_t* __restrict__ x,
                                                                                           const bf16_t* __restrict__ wu, int B, int d,
                                                                                           float* __restrict__ u, uint32_t* __restrict__ arrived) {
    extern __shared__ __align__(16) unsigned char dec_smem[];
    constexpr int NTH = kGateStreamWaves * 64;
    const int b = blockIdx.x;
    if (b >= B) {
        decode_stream_rows<0, NS, NT>(x, wu, B, d, a.F, u, a.ldg, 0, 0, nullptr, nullptr, b - B, gridDim.x - B, dec_smem);
        return;
    }
    if (b == 0 && threadIdx.x < kDownArrived) arrived[threadIdx.x] = 0;
    if constexpr (NCH > 0) {
        topk_row_body<float, NTH, NCH, false, true>(a, b, dec_smem);
    } else {
        float* const row = a.sd + b * a.ldg;
        for (int j = 4 * threadIdx.x; j < a.ldg; j += 4 * NTH) *reinterpret_cast<f32x4_t*>(row + j) = f32x4_t{kNotSelected, kNotSelected, kNotSelected, kNotSelected};
        __syncthreads();                                     // (one workgroup's stores to one place stay in order)
        for (int s = threadIdx.x; s < a.K; s += NTH) row[min((uint32_t)a.idx[(int64_t)b * a.K + s], (uint32_t)(a.F - 1))] = silu_f32(a.gsel_f32[(int64_t)b * a.K + s]);
    }
}

// y[b, c] = sum over the channels j that token b selected of z'[b, j] W_down[j, c], z' = SiLU(g) u.
// Workgroup (p, slice of 16 CT columns): its four wavefronts have a quarter of the p-th range of channels each and walk over it 32 at a
// time.  W_down goes to LDS as in the gate (32 rows of the slice a piece, with these channels' SiLU(g) and u of all tokens; a wavefront
// reads only what it loaded) and from there by transposing reads into v_mfma_f32_16x16x32_bf16, as D[column][token].  z' stays in 32 bits: it
// is cut into three bf16 (by truncation, 8 + 8 + 8 bits, which is exact), so a product takes three matrix instructions, whose time the
// stream hides.  A loop of one step: unrolled over the steps of a range, with z' in registers, the code's way into the instruction cache took
// longer than the data of small layers (512 x 1376: 8.1 us).
// A selected channel's value times a row of W_down with an infinity or a NaN is what it is; the zeros that stand for tokens that did not select
// the channel must not meet such a row, so a piece that holds one goes through fused multiply-adds that leave these tokens out.
// The ranges of one p share an XCD, whose L2 then serves SiLU(g) and u to all slices.
template <int CT> struct DownStreamCfg {
    static constexpr int kWaves = 4, kSlots = 3;             // (pieces of a wavefront under way)
    static constexpr int kCols = 16 * CT, kPitch = kCols * 2, kRows = 32 * kPitch, kPiece = kRows + 4096, kLoads = kRows / 1024 + 4;
    static constexpr int kLds = kWaves * kSlots * kPiece;
};
template <int CT, bool NT>
__global__ __launch_bounds__(DownStreamCfg<CT>::kWaves * 64, 1) void decode_down_stream_kernel(const float* __restrict__ sd, const float* __restrict__ u,
                                                                                              int64_t ldg, const bf16_t* __restrict__ wd, int B, int d, int F,
                                                                                              int per, float* __restrict__ part,
                                                                                              uint32_t* __restrict__ arrived, bf16_t* __restrict__ y) {
    using C = DownStreamCfg<CT>;
    constexpr int NW = C::kWaves;
    extern __shared__ __align__(16) unsigned char dec_smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int p = blockIdx.x, P = gridDim.x, slice = blockIdx.y;
    const int col0 = slice * C::kCols;
    const int k0 = min(F, (p * NW + wave) * per), k1 = min(F, k0 + per);      // this wavefront's channels
    const uint32_t pitch = (uint32_t)d * 2u;
    const int token = lane & 15, kq = 8 * (lane >> 4);

    // the position of a 16-byte chunk of a row is XORed with the row (see PpHalf, gemm_pingpong.h), so that a transposing read meets all banks
    const auto chunk_xor = [](int row) {
        const int flip = ((row >> 3) & 1) << 1;
        return CT == 8 ? ((row & 3) << 2) ^ flip : (((row >> 1) & 1) << 2) ^ flip;
    };
    constexpr int NR = C::kLoads - 4;
    uint32_t src[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int c = i * 64 + lane, row = c / (2 * CT), chunk = (c % (2 * CT)) ^ chunk_xor(row);
        src[i] = (uint32_t)row * pitch + (uint32_t)col0 * 2u + (uint32_t)chunk * 16u;
    }
    // 32 channels of eight tokens an instruction, chunk positions XORed with the token
    const uint32_t src_z = (uint32_t)(lane >> 3) * (uint32_t)ldg * 4u + (uint32_t)((lane ^ (lane >> 3)) & 7) * 16u;
    const uint32_t zbytes = (uint32_t)B * (uint32_t)ldg * 4u;      // (tokens from B up: zeros)
    const uint32_t ring = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)dec_smem) +
                          (uint32_t)wave * C::kSlots * C::kPiece;
    auto request = [&](int k, uint32_t slot) {               // 32 channels from k on; rows past the range: zeros
        const uint32_t left = (uint32_t)max(k1 - k, 0);
        const u32x4_t desc = buffer_desc(wd + (int64_t)k * d, left * pitch);
        const u32x4_t ds = buffer_desc(sd, left ? zbytes : 0u), du = buffer_desc(u, left ? zbytes : 0u);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t o = src_z + ((uint32_t)(8 * h) * (uint32_t)ldg + (uint32_t)k) * 4u;
            lds_load16(o, ds, ring + slot + C::kRows + h * 1024);
            lds_load16(o, du, ring + slot + C::kRows + 2048 + h * 1024);
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) lds_load16<NT>(src[i], desc, ring + slot + i * 1024);
    };
    typedef __attribute__((address_space(3))) s16x4_t* tr_ptr;
    typedef __attribute__((address_space(3))) const f32x4_t* z_ptr;
    uint32_t frag[CT], zfrag[2];
    {
        const int row = kq + ((lane & 15) >> 2);
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const int col = j * 16 + (lane & 3) * 4;
            frag[j] = ring + row * C::kPitch + (((col >> 3) ^ chunk_xor(row)) << 4) + (col & 7) * 2;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) zfrag[h] = ring + C::kRows + token * 128 + (((kq / 4 + h) ^ (token & 7)) << 4);
    }
    f32x4_t acc[CT];
#pragma unroll
    for (int j = 0; j < CT; ++j) acc[j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < C::kSlots; ++s) request(k0 + 32 * s, s * C::kPiece);
    uint32_t slot = 0;
#pragma unroll 1
    for (int k = k0; k < k1; k += 32) {
        wait_counts<(C::kSlots - 1) * C::kLoads, false>();
        bf16x8_t w[CT];
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const uint32_t q = frag[j] + slot;
            const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<tr_ptr>(q));
            const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<tr_ptr>(q + 4 * C::kPitch));
            typedef short s16x8_t __attribute__((ext_vector_type(8)));
            w[j] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
        f32x4_t sv[2], uv[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            sv[h] = *reinterpret_cast<z_ptr>(zfrag[h] + slot);
            uv[h] = *reinterpret_cast<z_ptr>(zfrag[h] + slot + 2048);
        }
        wait_counts<63, true>();
        request(k + 32 * C::kSlots, slot);
        slot = slot == (C::kSlots - 1) * C::kPiece ? 0 : slot + C::kPiece;
        uint32_t odd = 0;                                    // (an exponent of all ones carries into the sign)
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            const u32x4_t v = __builtin_bit_cast(u32x4_t, w[j]);
#pragma unroll
            for (int e = 0; e < 4; ++e) odd |= (v[e] & 0x7FFF7FFFu) + 0x00800080u;
        }
        if (__any((odd & 0x80008000u) != 0)) {
#pragma unroll 1
            for (int row = k; row < min(k + 32, k1); ++row) {
                const int64_t at = (int64_t)min(token, B - 1) * ldg + row;
                const float s = sd[at], zv = s * u[at];
                const bf16_t* const wrow = wd + (int64_t)row * d;
#pragma unroll
                for (int j = 0; j < CT; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float t = fmaf(zv, bf16_to_f32(wrow[min(col0 + j * 16 + 4 * (lane >> 4) + r, d - 1)]), acc[j][r]);
                        acc[j][r] = s != kNotSelected ? t : acc[j][r];
                    }
            }
            continue;
        }
        uint32_t zp[3][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t b[3][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int e = 2 * q + h;
                const float s = sv[e / 4][e % 4];
                const bool in = (s != kNotSelected) & (k + kq + e < k1);
                float v = s * uv[e / 4][e % 4];
                v = in ? v : 0.0f;
                const uint32_t top = __float_as_uint(v) & 0xFFFF0000u;
                const bool finite = (top & 0x7F800000u) != 0x7F800000u;
                const float rest = finite ? v - __uint_as_float(top) : 0.0f;
                const uint32_t mid = __float_as_uint(rest) & 0xFFFF0000u;
                b[0][h] = top;
                b[1][h] = mid;
                b[2][h] = __float_as_uint(rest - __uint_as_float(mid));
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) zp[i][q] = (b[i][0] >> 16) | (b[i][1] & 0xFFFF0000u);
        }
#pragma unroll
        for (int i = 2; i >= 0; --i) {
            const bf16x8_t zf = __builtin_bit_cast(bf16x8_t, u32x4_t{zp[i][0], zp[i][1], zp[i][2], zp[i][3]});
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j], zf, acc[j], 0, 0, 0);
        }
    }
    wait_counts<0, true>();                                  // the ring is free
    __syncthreads();
    float* red = reinterpret_cast<float*>(dec_smem);         // [NW][16 tokens][kCols]
    static_assert(NW * 16 * C::kCols * 4 <= C::kLds, "");
#pragma unroll
    for (int j = 0; j < CT; ++j)
        *reinterpret_cast<f32x4_t*>(red + (wave * 16 + token) * C::kCols + j * 16 + 4 * (lane >> 4)) = acc[j];
    __syncthreads();
    // The workgroup's share goes past L2, and the last workgroup of the slice to arrive adds all of them, in their order.
    const auto each = [&](const auto& f) {                   // f(four columns of a token)
        for (int i = threadIdx.x; i < 16 * C::kCols / 4; i += NW * 64) {
            const int b = i / (C::kCols / 4), c = i % (C::kCols / 4) * 4;
            if (b < B && col0 + c < d) f(b, c);
        }
    };
    const auto sum = [&](int b, int c) {
        f32x4_t s = *reinterpret_cast<const f32x4_t*>(red + b * C::kCols + c);
#pragma unroll
        for (int w = 1; w < NW; ++w) s += *reinterpret_cast<const f32x4_t*>(red + (w * 16 + b) * C::kCols + c);
        return s;
    };
    const auto store = [&](int b, int c, f32x4_t s) {
        *reinterpret_cast<u32x2_t*>(y + (int64_t)b * d + col0 + c) = u32x2_t{pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3])};
    };
    if (P == 1) {
        each([&](int b, int c) { store(b, c, sum(b, c)); });
        return;
    }
    constexpr int kPast = 17;                                // sc0 sc1: past the caches that the XCDs do not share
    const auto pbuf = __builtin_amdgcn_make_buffer_rsrc(part, 0, (uint32_t)P * (uint32_t)B * (uint32_t)d * 4u, 0x00020000);
    const auto share = [&](int q, int b, int c) { return (((uint32_t)q * (uint32_t)B + (uint32_t)b) * (uint32_t)d + (uint32_t)(col0 + c)) * 4u; };
    each([&](int b, int c) { __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, sum(b, c)), pbuf, share(p, b, c), 0, kPast); });
    wait_counts<0, true>();                                  // every wavefront's stores have been written through
    __syncthreads();
    __shared__ uint32_t before;
    if (threadIdx.x == 0) before = __hip_atomic_fetch_add(arrived + slice, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (before != (uint32_t)(P - 1)) return;
    each([&](int b, int c) {
        f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
        for (int q = 0; q < P; ++q) s += __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(pbuf, share(q, b, c), 0, kPast));
        store(b, c, s);
    });
}

}  // namespace moc
