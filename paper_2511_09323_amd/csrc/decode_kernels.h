// Decode path (paper section "Accelerated inference"): g = x W_gate over every channel, Top-K per
// token, then u_j = x . W_up[:, j] and y += SiLU(g_j) u_j w_j only for the selected channels j.
// All three weights are channel-major [F, d], so one channel is one contiguous row in each.
//
// The kernels stream weight rows with 16-byte loads, one wavefront per row (or row segment), and
// keep x in LDS.  All are bandwidth-bound; the arithmetic is fp32 FMA on the vector ALU.
#pragma once
#include "common.h"
#include "group_select.h"
#include "kernel_attrs.h"
#include "lds_dma.h"

namespace moc {

template <class E> struct Chunk;   // 16 bytes of E as floats
template <> struct Chunk<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void unpack(u32x4_t t, float* v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(t[i]);
    }
    static __device__ __forceinline__ void load(const float* p, float* v) {
        unpack(*reinterpret_cast<const u32x4_t*>(p), v);
    }
    // acc + sum of the products of the elements of two chunks
    static __device__ __forceinline__ float dot(u32x4_t a, u32x4_t b, float acc) {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), acc);
        return acc;
    }
};
template <> struct Chunk<bf16_t> {
    static constexpr int N = 8;
    static __device__ __forceinline__ void unpack(u32x4_t t, float* v) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(t[i] << 16);
            v[2 * i + 1] = __uint_as_float(t[i] & 0xFFFF0000u);
        }
    }
    static __device__ __forceinline__ void load(const bf16_t* p, float* v) {
        unpack(*reinterpret_cast<const u32x4_t*>(p), v);
    }
    // (v_dot2c_f32_bf16 would halve the instruction count but measured slower here.)
    static __device__ __forceinline__ float dot(u32x4_t a, u32x4_t b, float acc) {
        float w[N], x[N];
        unpack(a, w);
        unpack(b, x);
#pragma unroll
        for (int i = 0; i < N; ++i) acc = fmaf(w[i], x[i], acc);
        return acc;
    }
};

// g[b, j] = x[b] . wg[j]  for every channel j and every token b < B (B <= BT).
// x is staged in LDS ([BT, d] of E); each wavefront walks rows j = global wave id, += total waves.
template <class E, int BT>
__global__ __launch_bounds__(256) void decode_gate_kernel(const E* __restrict__ x, const E* __restrict__ wg, int B,
                                                          int d, int F, float* __restrict__ g, int64_t ldg) {
    constexpr int CN = Chunk<E>::N;
    extern __shared__ __align__(16) unsigned char dec_smem[];
    E* xs = reinterpret_cast<E*>(dec_smem);
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), nwave = gridDim.x * 4;
    constexpr int UN = 8;      // 16-byte chunks of a row per lane: rows of up to 64 * CN * UN elements in one go
    const bool whole_rows = d <= 64 * CN * UN;
    u32x4_t cur[UN], nxt[UN];
    auto fetch = [&](u32x4_t (&r)[UN], int j) {
        const E* wrow = wg + (int64_t)j * d;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = (u * 64 + lane) * CN;
            r[u] = u32x4_t{0, 0, 0, 0};
            if (k < d) r[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wrow + k));
        }
    };
    if (whole_rows && wave < F) fetch(cur, wave);          // in flight while x is staged
    for (int i = threadIdx.x * CN; i < BT * d; i += 256 * CN) {
        int b = i / d;
        u32x4_t v = {0, 0, 0, 0};
        if (b < B) v = *reinterpret_cast<const u32x4_t*>(x + i);
        *reinterpret_cast<u32x4_t*>(xs + i) = v;
    }
    __syncthreads();
    if (whole_rows) {
        // whole row in registers; the next row's loads are issued before this row is reduced
        for (int j = wave; j < F; j += nwave) {
            const bool more = j + nwave < F;
            if (more) fetch(nxt, j + nwave);
            float acc[BT];
#pragma unroll
            for (int b = 0; b < BT; ++b) acc[b] = 0.0f;
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = (u * 64 + lane) * CN;
                if (k < d) {
#pragma unroll
                    for (int b = 0; b < BT; ++b)
                        acc[b] = Chunk<E>::dot(cur[u], *reinterpret_cast<const u32x4_t*>(xs + b * d + k), acc[b]);
                }
            }
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                float s = wave_sum(acc[b]);
                if (lane == 0 && b < B) g[(int64_t)b * ldg + j] = s;
            }
            if (more) {
#pragma unroll
                for (int u = 0; u < UN; ++u) cur[u] = nxt[u];
            }
        }
        return;
    }
    for (int j = wave; j < F; j += nwave) {
        const E* wrow = wg + (int64_t)j * d;
        float acc[BT];
#pragma unroll
        for (int b = 0; b < BT; ++b) acc[b] = 0.0f;
        for (int k0 = lane * CN; k0 < d; k0 += 64 * CN * UN) {
            u32x4_t raw[UN];
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = k0 + u * 64 * CN;
                raw[u] = u32x4_t{0, 0, 0, 0};
                if (k < d) raw[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wrow + k));
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                const int k = k0 + u * 64 * CN;
                if (k < d) {
#pragma unroll
                    for (int b = 0; b < BT; ++b)
                        acc[b] = Chunk<E>::dot(raw[u], *reinterpret_cast<const u32x4_t*>(xs + b * d + k), acc[b]);
                }
            }
        }
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            float s = wave_sum(acc[b]);
            if (lane == 0 && b < B) g[(int64_t)b * ldg + j] = s;
        }
    }
}

// Grouped selection of MoC_{a:b} for one group and one token: vals[i * stride] are the gate values of
// channels c0 .. c0 + GB - 1; the kept channels go to slots q*ga .. q*ga + ga - 1 of the token's row.
template <int GB>
__device__ __forceinline__ void decode_group_select(const float* vals, int stride, int c0, int q, int ga,
                                                    int32_t* idx_row, float* gsel_row) {
    float v[GB];
#pragma unroll
    for (int i = 0; i < GB; ++i) v[i] = vals[i * stride];
    int rank[GB];
    group_ranks<GB>(v, rank);
    int r = 0;
#pragma unroll
    for (int i = 0; i < GB; ++i) {
        if (rank[i] < ga && r < ga) {                  // r < ga only matters for non-finite input
            idx_row[q * ga + r] = c0 + i;
            gsel_row[q * ga + r] = v[i];
            ++r;
        }
    }
}

// Gate projection fused with the grouped selection of MoC_{a:b}: a workgroup owns one group of GB
// consecutive channels at a time (wave w computes rows w, w + 4, ... of the group), the GB x B gate
// values meet in LDS and thread b selects for token b.  No gate row is written to memory.
template <class E, int BT, int GB>
__global__ __launch_bounds__(256) void decode_gate_group_kernel(const E* __restrict__ x, const E* __restrict__ wg,
                                                                int B, int d, int F, int ga, int K,
                                                                int32_t* __restrict__ idx, float* __restrict__ gsel) {
    constexpr int CN = Chunk<E>::N;
    extern __shared__ __align__(16) unsigned char dec_smem[];
    E* xs = reinterpret_cast<E*>(dec_smem);
    __shared__ float gl[2][GB][BT];
    for (int i = threadIdx.x * CN; i < BT * d; i += 256 * CN) {
        int b = i / d;
        u32x4_t v = {0, 0, 0, 0};
        if (b < B) v = *reinterpret_cast<const u32x4_t*>(x + i);
        *reinterpret_cast<u32x4_t*>(xs + i) = v;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int UN = 8;      // 16-byte chunks of the row in flight per lane
    int it = 0;
    for (int q = blockIdx.x; q < F / GB; q += gridDim.x, ++it) {
        for (int rr = wave; rr < GB; rr += 4) {
            const E* wrow = wg + (int64_t)(q * GB + rr) * d;
            float acc[BT];
#pragma unroll
            for (int b = 0; b < BT; ++b) acc[b] = 0.0f;
            for (int k0 = lane * CN; k0 < d; k0 += 64 * CN * UN) {
                u32x4_t raw[UN];
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int k = k0 + u * 64 * CN;
                    raw[u] = u32x4_t{0, 0, 0, 0};
                    if (k < d) raw[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wrow + k));
                }
#pragma unroll
                for (int u = 0; u < UN; ++u) {
                    const int k = k0 + u * 64 * CN;
                    if (k < d) {
#pragma unroll
                        for (int b = 0; b < BT; ++b)
                            acc[b] = Chunk<E>::dot(raw[u], *reinterpret_cast<const u32x4_t*>(xs + b * d + k), acc[b]);
                    }
                }
            }
#pragma unroll
            for (int b = 0; b < BT; ++b) {
                float s = wave_sum(acc[b]);
                if (lane == 0) gl[it & 1][rr][b] = s;
            }
        }
        __syncthreads();       // gl[it & 1] complete; gl[(it + 1) & 1] is free again (read two barriers ago)
        if (threadIdx.x < B)
            decode_group_select<GB>(&gl[it & 1][0][threadIdx.x], BT, q * GB, q, ga, idx + (int64_t)threadIdx.x * K,
                                    gsel + (int64_t)threadIdx.x * K);
    }
}

// Gate projection for batches of 2..16 tokens on the matrix cores (bf16 only):
//   g[b, j] = x[b] . wg[j]  as D[row j][token b] tiles of v_mfma_f32_16x16x32_bf16.
// Bound: the stream of W_gate, which every compute unit must keep full from its first to its last cycle.  So
//  - the rows are dealt evenly to one workgroup per compute unit (in units of four rows, or of a group), which walks over them
//    16 at a time;
//  - the eight wavefronts of a workgroup each have an eighth of the contraction (at most NS steps of 64 k), so that x stays in
//    registers, MFMA-ready, and nothing is staged before the first product;
//  - W_gate goes to LDS directly (lds_load16), in pieces of 16 rows x P steps, two pieces of every wavefront under way: one instruction
//    reads 512 bytes of a row where d allows, while loads in the order the MFMA wants would read 64 bytes of each of 16 rows.
//    A wavefront reads only what it loaded, so nothing but its own counter orders the two;
//  - rows past the workgroup's last, steps past d and tokens from B up are zeros of the buffer's range check, not branches.
// The partial tiles meet in LDS, one barrier per 16 rows; the wavefronts take turns in adding them.
// 4096 x 11008 (90 MB), averages of a profile with eight sets of weights in turn: 16 tokens 22.3 -> 19.2 us (4.8 TB/s), with the selection of a:8
// and four tokens 25.8, 16 tokens 23.2 -> 19.9 over both; before, one workgroup per 48 (16) rows staged x in LDS and read W_gate in MFMA
// order.  The same walk with loads to registers, 64 bytes of a row each, against this, the least of the launches: 20.8 / 17.8.
// GB = 0 writes the gate rows g[B, ldg]; GB = 4, 8, 16 selects the a largest of every GB channels instead (MoC_{a:b}; a workgroup's
// rows are a whole number of groups) and writes idx / gsel [B, K] only.  NT: see gate_stream_nontemporal.  Needs d % 64 == 0, d <= 512 NS,
// 16-byte aligned operands.
typedef __bf16 dec_bf16x8_t __attribute__((ext_vector_type(8)));
constexpr int kGateStreamWaves = 8, kGateStreamMaxD = 8 * 64 * kGateStreamWaves;
template <int GB, int NS> struct GateStreamCfg {
    static constexpr int P = NS < 4 ? NS : 4;                // steps of a piece
    static constexpr int PB = NS / P;                        // pieces of a block of 16 rows
    static constexpr int kPiece = 16 * P * 128;              // bytes
    static constexpr int kRing = kGateStreamWaves * 2 * kPiece, kRed = 2 * kGateStreamWaves * 256 * 4;
    static constexpr int kLds = kRing + kRed + (GB == 0 ? 0 : 16 * 17 * 4);
    static_assert(PB <= 2 && kLds <= kMaxDynLds, "");
};
// (workgroup wgi of wgn: the same walk also computes u over W_up, decode_dense.h)
template <int GB, int NS, bool NT>
__device__ __forceinline__ void decode_stream_rows(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg, int B, int d, int F,
                                                   float* __restrict__ g, int64_t ldg, int ga, int K, int32_t* __restrict__ idx,
                                                   float* __restrict__ gsel, int wgi, int wgn, unsigned char* dec_smem) {
    using C = GateStreamCfg<GB, NS>;
    constexpr int NW = kGateStreamWaves, P = C::P, PB = C::PB;
    constexpr int UNIT = GB == 0 ? 4 : GB;
    float (*red)[NW][256] = reinterpret_cast<float (*)[NW][256]>(dec_smem + C::kRing);
    float* tile = reinterpret_cast<float*>(dec_smem + C::kRing + C::kRed);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t units = (F + UNIT - 1) / UNIT;
    const int row0 = (int)(units * wgi / wgn) * UNIT;
    const int rows = min(F, (int)(units * (wgi + 1) / wgn) * UNIT) - row0;
    // this wavefront's steps of 64 k
    const int steps = d / 64, per = (steps + NW - 1) / NW;
    const int first = min(wave * per, steps), mine = min(per, steps - first);
    constexpr uint32_t kNowhere = 0xF0000000u;      // past the end of every buffer: zeros
    const uint32_t pitch = (uint32_t)d * 2u;
    u32x4_t xf[NS][2];
    {
        const auto xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(x), 0, (uint32_t)B * pitch, 0x00020000);
        const uint32_t off = (uint32_t)(lane & 15) * pitch + (uint32_t)first * 128u + (uint32_t)(lane >> 4) * 16u;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint32_t o = s < mine ? off : kNowhere;
            xf[s][0] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, o + s * 128, 0, 0);
            xf[s][1] = __builtin_amdgcn_raw_buffer_load_b128(xbuf, o + s * 128 + 64, 0, 0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // A piece in LDS: [16 rows][8 P chunks of 16 bytes], the position of a chunk XORed with the row, so that the 16 rows that an LDS
    // read takes one chunk of lie in different banks.
    const auto chunk_xor = [](int row) { return P == 1 ? (row >> 1) & 7 : row & 15; };
    uint32_t src[PB][2 * P];
#pragma unroll
    for (int i = 0; i < 2 * P; ++i) {
        const int c = i * 64 + lane, row = c / (8 * P), chunk = (c % (8 * P)) ^ chunk_xor(row);
#pragma unroll
        for (int part = 0; part < PB; ++part)
            src[part][i] = part * P + chunk / 8 < mine ? (uint32_t)row * pitch + (uint32_t)(first + part * P) * 128u + (uint32_t)chunk * 16u : kNowhere;
    }
    const uint32_t ring = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)dec_smem) +
                          (uint32_t)wave * 2 * C::kPiece;
    auto request = [&](int block, int part, int slot) {      // blocks past the last: no bytes to read, zeros
        const int left = max(rows - block * 16, 0);
        const u32x4_t desc = buffer_desc(wg + (int64_t)(row0 + block * 16) * d, (uint32_t)left * pitch);
#pragma unroll
        for (int i = 0; i < 2 * P; ++i) lds_load16<NT>(src[part][i], desc, ring + slot * C::kPiece + i * 1024);
    };
    typedef __attribute__((address_space(3))) const u32x4_t* frag_ptr;
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
    // Products of one piece; the ring slot is requested again as soon as its fragments are in registers.
    auto consume = [&](int part, int slot, int next_block) {
        wait_counts<2 * P, false>();                // (all but the other slot's requests have arrived)
        u32x4_t f[P][2];
        const int row = lane & 15;
#pragma unroll
        for (int s = 0; s < P; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                f[s][h] = *reinterpret_cast<frag_ptr>(ring + slot * C::kPiece + row * P * 128 +
                                                      (((s * 8 + h * 4 + (lane >> 4)) ^ chunk_xor(row)) << 4));
        wait_counts<63, true>();
        request(next_block, part, slot);
#pragma unroll
        for (int s = 0; s < P; ++s)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(dec_bf16x8_t, f[s][h]),
                                                              __builtin_bit_cast(dec_bf16x8_t, xf[part * P + s][h]), acc, 0, 0, 0);
    };
    // acc[e] = D[row 4 (lane / 16) + e][token lane % 16] over this wavefront's share of k
    auto finish = [&](int block) {
        float (&part)[NW][256] = red[block & 1];
        *reinterpret_cast<f32x4_t*>(&part[wave][lane * 4]) = acc;
        acc = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        wait_counts<63, true>();
        __builtin_amdgcn_s_barrier();               // (the requests stay under way)
        asm volatile("" ::: "memory");
        // Until the next block's barrier the adding wavefront has `part`, and `tile`, to itself.
        if (wave != (block & (NW - 1))) return;
        f32x4_t s = *reinterpret_cast<const f32x4_t*>(&part[0][lane * 4]);
#pragma unroll
        for (int o = 1; o < NW; ++o) s += *reinterpret_cast<const f32x4_t*>(&part[o][lane * 4]);
        const int b = lane & 15, in_block = 4 * (lane >> 4);
        if constexpr (GB == 0) {
            const int r = block * 16 + in_block;
            float* q = g + (int64_t)b * ldg + row0 + r;
            if (b < B) {
                if (r + 3 < rows) *reinterpret_cast<f32x4_t*>(q) = s;
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (r + e < rows) q[e] = s[e];
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) tile[(in_block + e) * 17 + b] = s[e];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int group = lane >> 4, r = block * 16 + group * GB;
            if (group < 16 / GB && b < B && r < rows)
                decode_group_select<GB>(tile + group * GB * 17 + b, 17, row0 + r, (row0 + r) / GB, ga, idx + (int64_t)b * K,
                                        gsel + (int64_t)b * K);
        }
    };
    request(0, 0, 0);
    if (PB == 2) request(0, PB - 1, 1);
    else request(1, 0, 1);
    // x has arrived before the loop: the compiler, which does not count the requests, would wait for them inside it
#pragma unroll
    for (int s = 0; s < NS; ++s) asm volatile("" : "+v"(xf[s][0]), "+v"(xf[s][1]));
    const int blocks = (rows + 15) / 16;
    if constexpr (PB == 2) {
        for (int block = 0; block < blocks; ++block) {
            consume(0, 0, block + 1);
            consume(1, 1, block + 1);
            finish(block);
        }
    } else {
        for (int block = 0; block < blocks; block += 2) {
            consume(0, 0, block + 2);
            finish(block);
            if (block + 1 == blocks) break;
            consume(0, 1, block + 3);
            finish(block + 1);
        }
    }
    wait_counts<0, true>();                         // nothing may still be on its way to LDS when the workgroup ends
}
template <int GB, int NS, bool NT>
__global__ __launch_bounds__(kGateStreamWaves * 64, 2) void decode_gate_stream_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ wg, int B, int d, int F, float* __restrict__ g, int64_t ldg, int ga,
    int K, int32_t* __restrict__ idx, float* __restrict__ gsel) {
    extern __shared__ __align__(16) unsigned char dec_smem[];
    decode_stream_rows<GB, NS, NT>(x, wg, B, d, F, g, ldg, ga, K, idx, gsel, blockIdx.x, gridDim.x, dec_smem);
}

// z[b, s] = SiLU(gsel[b, s]) * (x[b] . wu[idx[b, s]])  for every selected (token, channel) pair.
// grid = (row groups, B); x[b] is staged in LDS.
template <class E>
__global__ __launch_bounds__(256) void decode_up_kernel(const E* __restrict__ x, const E* __restrict__ wu,
                                                        const int32_t* __restrict__ idx,
                                                        const float* __restrict__ gsel, int d, int K,
                                                        float* __restrict__ z) {
    constexpr int CN = Chunk<E>::N;
    extern __shared__ __align__(16) unsigned char dec_smem[];
    E* xs = reinterpret_cast<E*>(dec_smem);
    const int b = blockIdx.y;
    for (int i = threadIdx.x * CN; i < d; i += 256 * CN)
        *reinterpret_cast<u32x4_t*>(xs + i) = *reinterpret_cast<const u32x4_t*>(x + (int64_t)b * d + i);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * 4 + (threadIdx.x >> 6), nwave = gridDim.x * 4;
    for (int s = wave; s < K; s += nwave) {
        const int j = idx[(int64_t)b * K + s];
        const E* wrow = wu + (int64_t)j * d;
        float acc = 0.0f;
        for (int k = lane * CN; k < d; k += 64 * CN) {
            float w[CN], xv[CN];
            Chunk<E>::load(wrow + k, w);
            Chunk<E>::load(xs + k, xv);
#pragma unroll
            for (int e = 0; e < CN; ++e) acc = fmaf(w[e], xv[e], acc);
        }
        acc = wave_sum(acc);
        if (lane == 0) z[(int64_t)b * K + s] = silu_f32(gsel[(int64_t)b * K + s]) * acc;
    }
}

// part[p, b, c] = sum over the p-th share of token b's selected channels of z[b, s] * wd[idx[b, s], c]
// for the 64*CN*DIT-wide slice of columns c chosen by blockIdx.z.  grid = (P, B, slices).
template <class E, int DIT>
__global__ __launch_bounds__(256) void decode_down_kernel(const E* __restrict__ wd, const int32_t* __restrict__ idx,
                                                          const float* __restrict__ z, int d, int K, int P,
                                                          float* __restrict__ part) {
    constexpr int CN = Chunk<E>::N;
    constexpr int SLICE = 64 * CN * DIT;
    __shared__ float red[4][SLICE];
    const int p = blockIdx.x, b = blockIdx.y, c0 = blockIdx.z * SLICE;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = (K + P - 1) / P;
    const int s_begin = p * per, s_end = min(K, s_begin + per);
    float acc[DIT][CN];
#pragma unroll
    for (int i = 0; i < DIT; ++i)
#pragma unroll
        for (int e = 0; e < CN; ++e) acc[i][e] = 0.0f;
    for (int s = s_begin + wave; s < s_end; s += 4) {
        const int j = idx[(int64_t)b * K + s];
        const float zz = z[(int64_t)b * K + s];
        const E* wrow = wd + (int64_t)j * d + c0;
#pragma unroll
        for (int i = 0; i < DIT; ++i) {
            const int c = i * 64 * CN + lane * CN;
            if (c0 + c < d) {
                float w[CN];
                Chunk<E>::load(wrow + c, w);
#pragma unroll
                for (int e = 0; e < CN; ++e) acc[i][e] = fmaf(zz, w[e], acc[i][e]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < DIT; ++i)
#pragma unroll
        for (int e = 0; e < CN; ++e) red[wave][i * 64 * CN + lane * CN + e] = acc[i][e];
    __syncthreads();
    for (int c = threadIdx.x; c < SLICE; c += 256) {
        if (c0 + c < d)
            part[((int64_t)p * gridDim.y + b) * d + c0 + c] = red[0][c] + red[1][c] + red[2][c] + red[3][c];
    }
}

// Fused gather stage for one token per workgroup column: for the p-th share of token b's selected
// channels, u = x[b] . wu[j], z' = SiLU(g) u, and part[p, b, :] = sum z' wd[j, :].  A wavefront
// owns a channel at a time and has both of its rows (one of wu, one of wd, NIT 16-byte chunks per
// lane each) in flight before it waits.  P * B workgroups of 512 threads; needs d <= 64 * CN * NIT.
// Workgroup w of the P * B launched handles (share p, token b).  idx rows ascend, so share p of every
// token covers about the same channel range: when P is a multiple of 8 the workgroups of one share
// are placed on one XCD (w % 8), whose L2 then serves the rows that several tokens selected
// (SHARED = true also drops the non-temporal hint so that those rows stay in L2).
template <class E, int NIT, bool SHARED>
__global__ __launch_bounds__(512) void decode_updown_kernel(const E* __restrict__ x, const E* __restrict__ wu,
                                                            const E* __restrict__ wd,
                                                            const int32_t* __restrict__ idx,
                                                            const float* __restrict__ gsel, int d, int K, int P, int B,
                                                            float* __restrict__ part) {
    constexpr int CN = Chunk<E>::N;
    constexpr int NWV = 8;
    extern __shared__ __align__(16) unsigned char dec_smem[];
    E* xs = reinterpret_cast<E*>(dec_smem);
    float* red = reinterpret_cast<float*>(dec_smem + (size_t)d * sizeof(E));     // [NWV][d]
    int p, b;
    if (SHARED && P % 8 == 0) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        p = xcd + 8 * (slot / B);
        b = slot % B;
    } else {
        p = blockIdx.x / B;
        b = blockIdx.x % B;
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per = (K + P - 1) / P;
    const int s_begin = p * per, s_end = min(K, s_begin + per);
    float acc[NIT][CN];
#pragma unroll
    for (int i = 0; i < NIT; ++i)
#pragma unroll
        for (int e = 0; e < CN; ++e) acc[i][e] = 0.0f;
    u32x4_t ru[NIT], rd[NIT];
    float gj = 0.0f;
    // Channel and gate value of this wavefront's next 64 slots, one per lane, so that a row's address waits for no load.  Call, read per
    // slot / this: 4096 x 11008, 2:8 with 16 tokens 88.8 / 79.2 us, with 4 tokens 49.8 / 49.1, row-wide with 16 tokens 75.1 / 74.5.
    int lane_j = 0;
    float lane_g = 0.0f;
    auto fetch_slots = [&](int s) {
        const int q = s + lane * NWV;
        if (q < s_end) {
            lane_j = idx[(int64_t)b * K + q];
            lane_g = gsel[(int64_t)b * K + q];
        }
    };
    // rows of the n-th of those slots (both matrices) -> registers; all loads are issued before any is used
    auto fetch_rows = [&](int n) {
        const int j = __builtin_amdgcn_readlane(lane_j, n);
        gj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lane_g), n));
        const E* urow = wu + (int64_t)j * d;
        const E* drow = wd + (int64_t)j * d;
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int k = i * 64 * CN + lane * CN;
            ru[i] = u32x4_t{0, 0, 0, 0};
            if (k < d) ru[i] = SHARED ? *reinterpret_cast<const u32x4_t*>(urow + k)
                                      : __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(urow + k));
        }
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int k = i * 64 * CN + lane * CN;
            rd[i] = u32x4_t{0, 0, 0, 0};
            if (k < d) rd[i] = SHARED ? *reinterpret_cast<const u32x4_t*>(drow + k)
                                      : __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(drow + k));
        }
    };
    int s = s_begin + wave, n = 0;
    if (s < s_end) {                       // in flight while x is staged
        fetch_slots(s);
        fetch_rows(0);
    }
    for (int i = threadIdx.x * CN; i < d; i += 512 * CN)
        *reinterpret_cast<u32x4_t*>(xs + i) = *reinterpret_cast<const u32x4_t*>(x + (int64_t)b * d + i);
    __syncthreads();
    while (s < s_end) {
        float dot = 0.0f;
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            const int k = i * 64 * CN + lane * CN;
            if (k < d) {
                dot = Chunk<E>::dot(ru[i], *reinterpret_cast<const u32x4_t*>(xs + k), dot);
            }
        }
        dot = wave_sum(dot);
        const float zz = silu_f32(gj) * dot;
#pragma unroll
        for (int i = 0; i < NIT; ++i) {
            float w[CN];
            Chunk<E>::unpack(rd[i], w);
#pragma unroll
            for (int e = 0; e < CN; ++e) acc[i][e] = fmaf(zz, w[e], acc[i][e]);
        }
        s += NWV;
        if (s < s_end) {
            if (++n == 64) {
                fetch_slots(s);
                n = 0;
            }
            fetch_rows(n);
        }
    }
#pragma unroll
    for (int i = 0; i < NIT; ++i) {
        const int k = i * 64 * CN + lane * CN;
        if (k < d) {
#pragma unroll
            for (int e = 0; e < CN; ++e) red[wave * d + k + e] = acc[i][e];
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < d; c += 512) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) s += red[w * d + c];
        part[((int64_t)p * B + b) * d + c] = s;
    }
}

// Whole decode step of MoC_{a:8} (a = GA = 1 or 2) in one launch, for up to BT tokens (the host uses it
// for single tokens only: with more tokens per workgroup the separate launches measured faster).  The grouped
// selection is local to 8 consecutive channels, so a workgroup that has computed the gate values of
// a group knows the group's kept channels at once and can fetch their W_up / W_down rows itself: no
// launch boundary between gate, selection and gather.  512 threads; per group
//   gate:   wave w reads row 8q + w of W_gate (prefetched during the previous group) and reduces its
//           dot products with the BT staged tokens;
//   select: after one barrier every thread ranks the 8 x BT gate values (same rule as
//           group_select_kernel) and knows the BT*GA (token, channel) pairs;
//   gather: wave w reads slice w (d/8 elements) of both rows of every pair, together with the next
//           group's gate row; partial dots with x meet in LDS (second barrier); then
//           acc[token][own columns] += SiLU(g) u W_down[j][own columns].
// part[p, b, :] gets the workgroup's partial output (p = blockIdx.x); decode_reduce_kernel sums them.
// Needs d % CN == 0 and d <= 8 * 64 * CN (one 16-byte chunk per lane and slice).
template <class E, int BT, int GA>
__global__ __launch_bounds__(512) void decode_fused_group_kernel(const E* __restrict__ x, const E* __restrict__ wg,
                                                                 const E* __restrict__ wu, const E* __restrict__ wd,
                                                                 int B, int d, int F, int K, int32_t* __restrict__ idx,
                                                                 float* __restrict__ part) {
    constexpr int CN = Chunk<E>::N;
    constexpr int GB = 8, NWV = 8, NE = BT * GA;
    static_assert(GA == 1 || GA == 2, "the ordered pair below covers one or two kept channels");
    constexpr int UN = 8;                       // 16-byte chunks of a gate row per lane
    extern __shared__ __align__(16) unsigned char dec_smem[];
    E* xs = reinterpret_cast<E*>(dec_smem);     // [BT][d]
    __shared__ float gl[2][GB][BT];
    __shared__ float dl[2][NE][NWV];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ngroups = F / GB;
    int q = blockIdx.x;
    u32x4_t raw[UN];
    auto fetch_gate = [&](int qq) {
        const E* wrow = wg + (int64_t)(qq * GB + wave) * d;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = (u * 64 + lane) * CN;
            raw[u] = u32x4_t{0, 0, 0, 0};
            if (k < d) raw[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wrow + k));
        }
    };
    if (q < ngroups) fetch_gate(q);             // in flight while x is staged
    for (int i = tid * CN; i < BT * d; i += 512 * CN) {
        const int b = i / d;
        u32x4_t v = {0, 0, 0, 0};
        if (b < B) v = *reinterpret_cast<const u32x4_t*>(x + i);
        *reinterpret_cast<u32x4_t*>(xs + i) = v;
    }
    __syncthreads();
    const int kslice = (wave * 64 + lane) * CN;  // this thread's columns in the gather stage
    const bool have_slice = kslice < d;
    float acc[BT][CN];
#pragma unroll
    for (int b = 0; b < BT; ++b)
#pragma unroll
        for (int e = 0; e < CN; ++e) acc[b][e] = 0.0f;
    int it = 0;
    for (; q < ngroups; q += gridDim.x, ++it) {
        // ---- gate values of this wave's row for every token
        float ga_[BT];
#pragma unroll
        for (int b = 0; b < BT; ++b) ga_[b] = 0.0f;
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int k = (u * 64 + lane) * CN;
            if (k < d) {
#pragma unroll
                for (int b = 0; b < BT; ++b)
                    ga_[b] = Chunk<E>::dot(raw[u], *reinterpret_cast<const u32x4_t*>(xs + b * d + k), ga_[b]);
            }
        }
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            const float s = wave_sum(ga_[b]);
            if (lane == 0) gl[it & 1][wave][b] = s;
        }
        __syncthreads();
        // ---- selection (every thread, same result) and the loads that depend on it
        int jsel[NE];
        float gsel[NE];
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            float v[GB];
#pragma unroll
            for (int i = 0; i < GB; ++i) v[i] = gl[it & 1][i][b];
            int rank[GB];
            group_ranks<GB>(v, rank);
            // kept channels in ascending order: with GA <= 2 they are the lowest and the highest kept index
            int lo = -1, hi = 0;
#pragma unroll
            for (int i = 0; i < GB; ++i) {
                if (rank[i] < GA) {
                    if (lo < 0) lo = i;
                    hi = i;
                }
            }
            if (lo < 0) lo = 0;                                  // only for non-finite input
            float vlo = v[0], vhi = v[0];
#pragma unroll
            for (int i = 1; i < GB; ++i) {
                vlo = (i == lo) ? v[i] : vlo;
                vhi = (i == hi) ? v[i] : vhi;
            }
            jsel[b * GA] = q * GB + lo;
            gsel[b * GA] = vlo;
            if (GA == 2) {
                jsel[b * GA + 1] = q * GB + hi;
                gsel[b * GA + 1] = vhi;
            }
        }
        if (tid < B * GA) {
            // tid = b * GA + r
#pragma unroll
            for (int e = 0; e < NE; ++e)
                if (tid == e) idx[(int64_t)(e / GA) * K + q * GA + (e % GA)] = jsel[e];
        }
        u32x4_t ru[NE], rd[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            ru[e] = u32x4_t{0, 0, 0, 0};
            rd[e] = u32x4_t{0, 0, 0, 0};
            if (have_slice && e / GA < B) {
                ru[e] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wu + (int64_t)jsel[e] * d + kslice));
                rd[e] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(wd + (int64_t)jsel[e] * d + kslice));
            }
        }
        if (q + (int)gridDim.x < ngroups) fetch_gate(q + gridDim.x);     // next group's gate row, in flight with the gather
        // ---- partial dots of the up projection over this wave's slice
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            float dot = 0.0f;
            if (have_slice) {
                dot = Chunk<E>::dot(ru[e], *reinterpret_cast<const u32x4_t*>(xs + (e / GA) * d + kslice), dot);
            }
            dot = wave_sum(dot);
            if (lane == 0) dl[it & 1][e][wave] = dot;
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            float u = 0.0f;
#pragma unroll
            for (int w = 0; w < NWV; ++w) u += dl[it & 1][e][w];
            const float zz = silu_f32(gsel[e]) * u;
            float w[CN];
            Chunk<E>::unpack(rd[e], w);
#pragma unroll
            for (int c = 0; c < CN; ++c) acc[e / GA][c] = fmaf(zz, w[c], acc[e / GA][c]);
        }
    }
    if (have_slice) {
#pragma unroll
        for (int b = 0; b < BT; ++b) {
            if (b < B) {
                float* dst = part + ((int64_t)blockIdx.x * B + b) * d + kslice;
#pragma unroll
                for (int c = 0; c < CN; c += 4)
                    *reinterpret_cast<f32x4_t*>(dst + c) = f32x4_t{acc[b][c], acc[b][c + 1], acc[b][c + 2], acc[b][c + 3]};
            }
        }
    }
}

// y[b, c] = sum_p part[p, b, c] in a fixed order (deterministic).  A 1024-thread workgroup owns 64
// columns; its sixteen wavefronts each sum a sixteenth of the P partials with the loads in flight
// together, and the sixteen sums are combined through LDS.
template <class E>
__global__ __launch_bounds__(1024) void decode_reduce_kernel(const float* __restrict__ part, int P, int64_t n,
                                                             E* __restrict__ y) {
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const int per = (P + 15) / 16;
    const int p0 = q * per, p1 = min(P, p0 + per);
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
    if (c < n) {
        int p = p0;
        for (; p + 3 < p1; p += 4) {
            const float a0 = part[(int64_t)p * n + c], a1 = part[(int64_t)(p + 1) * n + c];
            const float a2 = part[(int64_t)(p + 2) * n + c], a3 = part[(int64_t)(p + 3) * n + c];
            s0 += a0; s1 += a1; s2 += a2; s3 += a3;
        }
        for (; p < p1; ++p) s0 += part[(int64_t)p * n + c];
    }
    red[q][lane] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (q == 0 && c < n) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += red[w][lane];
        Elem<E>::store(y + c, t);
    }
}

}  // namespace moc
