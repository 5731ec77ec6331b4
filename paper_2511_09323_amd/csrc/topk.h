// Row-wise Top-K selection over the fp32 gate (the mask M = TopK(G) of the paper's section
// "Mixture-of-Channels architecture"): exactly K channels per row, the largest signed values,
// equal values ordered by channel index (lower first), -0.0 equal to +0.0.
//
// One workgroup per row.  topk_rows_kernel keeps the whole row in registers (all global loads are issued before anything
// waits on them) and finds the K-th largest value by row_cut.h; topk_rows_lds_kernel parks order-preserving keys in LDS
// instead, finds the K-th with a most-significant-digit-first radix select and serves rows that are too long for registers or
// not 16-byte aligned.  A final ordered pass ranks the selected channels with wavefront ballots, so the output ascends by
// channel without any sort.
//
// FUSED = true is the training forward: besides idx and the gate values it gathers U at the
// selected channels and writes the dense activation row Z' = SiLU(G) . M . U (Eq. MoC-2), zeros
// on unselected channels and on the padding up to ldz.
#pragma once
#include "common.h"
#include "row_cut.h"

namespace moc {

constexpr int kTopkBins = 2048;

template <class E> __device__ __forceinline__ void store_vec4_any(E* p, const float v[4]);
template <> __device__ __forceinline__ void store_vec4_any<float>(float* p, const float v[4]) {
    *reinterpret_cast<f32x4_t*>(p) = f32x4_t{v[0], v[1], v[2], v[3]};
}
template <> __device__ __forceinline__ void store_vec4_any<bf16_t>(bf16_t* p, const float v[4]) {
    *reinterpret_cast<u32x2_t*>(p) = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}

template <class E> struct TopkArgs {
    const float* g;     // [T, ldg] fp32 gate
    int64_t ldg;
    int F, K;
    int32_t* idx;       // [T, K]
    float* gsel_f32;    // [T, K] or null: selected gate values, fp32
    E* gvals;           // [T, K] or null: selected gate values, E
    // FUSED only:
    const E* u;         // [T, ldu] dense up projection
    int64_t ldu;
    E* uvals;           // [T, K]
    E* zd;              // [T, ldz] dense masked activation
    int64_t ldz;
    // Keyed selection (Top-K position variants): g then holds the transformed keys the ranking is
    // done on, and the gate values themselves are fetched from here ([T, ldg] like g); null otherwise.
    const float* g_raw;
    float far = 0.0f;   // cut_far(F, K), set by the launcher of the register-resident kernel
    float* sd = nullptr;      // DENSE only: [T, ldg], SiLU(g) of selected channels, kNotSelected elsewhere and on the padding of the row
};

// Selection keys of the Top-K position variants: mode 1 ranks SiLU(g) (ablation row "After SiLU"),
// mode 2 ranks |SiLU(g)| (the selection of the proof of Theorem 1).  Element-wise, [T, ld] fp32.
static __global__ void topk_key_transform_kernel(const float* __restrict__ g, float* __restrict__ keys, int64_t n, int mode) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float s = silu_f32(g[i]);
        keys[i] = mode == 2 ? fabsf(s) : s;
    }
}

// Exclusive scan of one value per thread across the workgroup, in thread order.
// red must hold NT/64 ints.  Returns the exclusive prefix; total goes to *total.
template <int NT> __device__ __forceinline__ int block_exclusive_scan(int v, int* red, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) red[wave] = inc;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        int r = red[w];
        if (w < wave) base += r;
        tot += r;
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

template <class E, int NT, int VEC, bool FUSED>
__global__ __launch_bounds__(NT) void topk_rows_lds_kernel(TopkArgs<E> a) {
    constexpr int NW = NT / 64;
    constexpr int CHUNK = NT * VEC;
    extern __shared__ __align__(16) unsigned char topk_smem[];
    const int F = a.F, K = a.K;
    const int nchunk = (F + CHUNK - 1) / CHUNK;
    uint32_t* keys = reinterpret_cast<uint32_t*>(topk_smem);           // nchunk * CHUNK
    uint32_t* hist = keys + nchunk * CHUNK;                            // kTopkBins
    int* cnt_gt = reinterpret_cast<int*>(hist + kTopkBins);            // nchunk * NW
    int* cnt_eq = cnt_gt + nchunk * NW;                                // nchunk * NW
    int* red = cnt_eq + nchunk * NW;                                   // NW
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_need;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const float* grow = a.g + row * a.ldg;

    // ---- load the row, build keys
    for (int i = tid; i < kTopkBins; i += NT) hist[i] = 0;
    __syncthreads();
    for (int c = 0; c < nchunk; ++c) {
        const int j0 = c * CHUNK + tid * VEC;
        uint32_t k[VEC];
        if (VEC == 4 && j0 + 3 < F) {
            f32x4_t v = *reinterpret_cast<const f32x4_t*>(grow + j0);
#pragma unroll
            for (int e = 0; e < VEC; ++e) k[e] = float_key(v[e]);
        } else {
#pragma unroll
            for (int e = 0; e < VEC; ++e) k[e] = (j0 + e < F) ? float_key(grow[j0 + e]) : 0u;
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            keys[j0 + e] = k[e];
            if (j0 + e < F) atomicAdd(&hist[k[e] >> 21], 1u);
        }
    }
    __syncthreads();

    // ---- three digit passes, most significant first.  After a pass: prefix = the digits fixed so
    //      far of the K-th largest key, need = how many elements are still wanted among those
    //      whose key starts with that prefix.
    uint32_t prefix = 0;
    int need = K;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : (pass == 1 ? 10 : 0);
        const int nbins = pass == 2 ? 1024 : 2048;
        if (pass > 0) {
            for (int i = tid; i < kTopkBins; i += NT) hist[i] = 0;
            __syncthreads();
            const int pshift = pass == 1 ? 21 : 10;
            for (int c = 0; c < nchunk; ++c) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const int j = c * CHUNK + tid * VEC + e;
                    const uint32_t k = keys[j];
                    if (j < F && (k >> pshift) == prefix) atomicAdd(&hist[(k >> shift) & (nbins - 1)], 1u);
                }
            }
            __syncthreads();
        }
        // descending scan over bins: thread t owns bins [nbins-1 - t*per - (per-1), nbins-1 - t*per]
        const int per = (nbins + NT - 1) / NT;
        int local = 0;
        for (int q = 0; q < per; ++q) {
            int b = nbins - 1 - (tid * per + q);
            if (b >= 0) local += (int)hist[b];
        }
        int total;
        int above = block_exclusive_scan<NT>(local, red, &total);
        if (above < need && above + local >= need) {   // the crossing bin is one of mine
            int run = above;
            for (int q = 0; q < per; ++q) {
                int b = nbins - 1 - (tid * per + q);
                if (b < 0) break;
                int h = (int)hist[b];
                if (run + h >= need) {
                    sh_prefix = (prefix << (pass == 0 ? 0 : (pass == 1 ? 11 : 10))) | (uint32_t)b;
                    sh_need = need - run;
                    break;
                }
                run += h;
            }
        }
        __syncthreads();
        prefix = sh_prefix;
        need = sh_need;
        __syncthreads();
    }
    const uint32_t tau = prefix;   // key of the K-th largest element; `need` of the keys equal to
                                   // tau are selected (lowest channels first), all keys above are.

    // ---- ordered pass 1: per (chunk, wave) counts of keys > tau and keys == tau
    for (int c = 0; c < nchunk; ++c) {
        int ngt = 0, neq = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const int j = c * CHUNK + tid * VEC + e;
            const uint32_t k = keys[j];
            const bool in = j < F;
            ngt += __popcll(__ballot(in && k > tau));
            neq += __popcll(__ballot(in && k == tau));
        }
        if (lane == 0) {
            cnt_gt[c * NW + wave] = ngt;
            cnt_eq[c * NW + wave] = neq;
        }
    }
    __syncthreads();
    // exclusive scan of the two small tables in (chunk, wave) order, by wave 0
    if (wave == 0) {
        const int n = nchunk * NW;
        const int per = (n + 63) / 64;
        int sg = 0, se = 0;
        for (int q = 0; q < per; ++q) {
            int i = lane * per + q;
            if (i < n) { sg += cnt_gt[i]; se += cnt_eq[i]; }
        }
        int ig = sg, ie = se;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            int tg = __shfl_up(ig, o, 64), te = __shfl_up(ie, o, 64);
            if (lane >= o) { ig += tg; ie += te; }
        }
        int rg = ig - sg, re = ie - se;
        for (int q = 0; q < per; ++q) {
            int i = lane * per + q;
            if (i < n) {
                int g0 = cnt_gt[i], e0 = cnt_eq[i];
                cnt_gt[i] = rg; cnt_eq[i] = re;
                rg += g0; re += e0;
            }
        }
    }
    __syncthreads();

    // ---- ordered pass 2: rank and write
    int32_t* idx_row = a.idx + row * K;
    const int64_t ldz_pad = FUSED ? a.ldz : 0;
    const int out_chunks = FUSED ? (int)((ldz_pad + CHUNK - 1) / CHUNK) : nchunk;
    for (int c = 0; c < out_chunks; ++c) {
        const int j0 = c * CHUNK + tid * VEC;
        int gt_before = 0, eq_before = 0;
        uint32_t k[VEC];
        bool isgt[VEC], iseq[VEC];
        if (c < nchunk) {
            gt_before = cnt_gt[c * NW + wave];
            eq_before = cnt_eq[c * NW + wave];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                k[e] = keys[j0 + e];
                const bool in = j0 + e < F;
                isgt[e] = in && k[e] > tau;
                iseq[e] = in && k[e] == tau;
                gt_before += mbcnt(__ballot(isgt[e]));
                eq_before += mbcnt(__ballot(iseq[e]));
            }
        } else {
#pragma unroll
            for (int e = 0; e < VEC; ++e) { isgt[e] = iseq[e] = false; k[e] = 0; }
        }
        float z[VEC];
        float uu[VEC];
        if (FUSED) {
            const E* urow = a.u + row * a.ldu;
#pragma unroll
            for (int e = 0; e < VEC; ++e) uu[e] = (j0 + e < F) ? Elem<E>::load(urow + j0 + e) : 0.0f;
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const bool sel = isgt[e] || (iseq[e] && eq_before < need);
            z[e] = 0.0f;
            if (sel) {
                const int slot = gt_before + min(eq_before, need);
                const float g = a.g_raw ? a.g_raw[row * a.ldg + j0 + e] : key_float(k[e]);
                idx_row[slot] = j0 + e;
                if (a.gsel_f32) a.gsel_f32[row * K + slot] = g;
                if (a.gvals) Elem<E>::store(a.gvals + row * K + slot, g);
                if (FUSED) {
                    Elem<E>::store(a.uvals + row * K + slot, uu[e]);
                    z[e] = silu_f32(g) * uu[e];
                }
            }
            gt_before += isgt[e] ? 1 : 0;
            eq_before += iseq[e] ? 1 : 0;
        }
        if (FUSED) {
            E* zrow = a.zd + row * a.ldz;
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                if (j0 + e < ldz_pad) Elem<E>::store(zrow + j0 + e, z[e]);
        }
    }
}

// ---------------------------------------------------------------- K = F: nothing to select
// Bound by its stores; workgroup (t, p) writes channels p * kAllSpan .. of row t, padding of Z' included.  8192 rows of 5461: 193 us (297
// with a radix select, 465 with a cut and the gather of the row kernel).
constexpr int kAllSpan = 1024;
template <class E, bool FUSED>
__global__ __launch_bounds__(256) void select_all_kernel(TopkArgs<E> a) {
    constexpr int U = kAllSpan / 256;
    const int64_t row = blockIdx.x;
    const float* grow = (a.g_raw ? a.g_raw : a.g) + row * a.ldg;
    const int j0 = blockIdx.y * kAllSpan + threadIdx.x;
    float g[U], u[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int j = min(j0 + q * 256, a.F - 1);
        g[q] = a.g_raw ? grow[j] : grow[j] + 0.0f;           // (-0.0 is stored as +0.0)
        if (FUSED) u[q] = Elem<E>::load(a.u + row * a.ldu + j);
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int j = j0 + q * 256;
        if (j < a.F) {
            a.idx[row * a.F + j] = j;
            if (a.gsel_f32) a.gsel_f32[row * a.F + j] = g[q];
            if (a.gvals) Elem<E>::store(a.gvals + row * a.F + j, g[q]);
            if (FUSED) Elem<E>::store(a.uvals + row * a.F + j, u[q]);
        }
        if (FUSED && j < a.ldz) Elem<E>::store(a.zd + row * a.ldz + j, j < a.F ? silu_f32(g[q]) * u[q] : 0.0f);
    }
}

// ---------------------------------------------------------------- register-resident variant
// The selected set without the index list: a channel j with key k belongs to it iff k > tau, or k == tau and j <= cut
// (cut = INT_MAX when every key equal to tau is in).
struct TopkThreshold {
    uint32_t tau;
    int cut;
};

__device__ __forceinline__ bool topk_member(uint32_t key, int j, TopkThreshold t) {
    return key > t.tau || (key == t.tau && j <= t.cut);
}

// Row of up to NCH * NT * 4 channels; thread t holds channels c*NT*4 + t*4 .. +3 of every chunk c.
// Bound by vector instructions as long as a value costs more than about 25 of them, then by memory.  The cut comes from
// row_cut.h; channels are ranked with one ballot sweep (one compare per value; where equal values straddle the cut, those past it are
// marked before) whose per-lane prefixes stay in registers.  Selected channels are staged in LDS at their output slot, so that the
// compact outputs are written slot by slot (coalesced, SiLU evaluated K times instead of under divergence for every channel)
// and the dense Z' row is assembled in LDS and streamed out with 16-byte stores.  Dynamic LDS: topk_reg_dyn_lds().
template <class E, int NT, int NCH, bool FUSED, bool DENSE = false>
__device__ __forceinline__ void topk_row_body(const TopkArgs<E>& a, int64_t row, unsigned char* topk_dyn) {
    constexpr int NW = NT / 64;
    constexpr int CHUNK = NT * 4;
    __shared__ int tab[NCH * NW];
    const int F = a.F, K = a.K;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* grow = a.g + row * a.ldg;

    // ---- all loads of the row up front
    f32x4_t gv[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        // ldg is a multiple of 4, so the aligned 16-byte block that holds channel j0 < F lies inside
        // the row pitch; what it holds past F is masked out below
        // Threads past the end of the row re-read its last block instead of branching.
        const int j0 = min(c * CHUNK + tid * 4, ((F + 3) & ~3) - 4);
        gv[c] = *reinterpret_cast<const f32x4_t*>(grow + j0);
    }
    float v[NCH][4];
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[c][e] = gv[c][e];
        if ((c + 1) * CHUNK > F) {                          // only the chunks that reach past the row (uniform)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c * CHUNK + tid * 4 + e >= F) v[c][e] = -__builtin_inff();
        }
    }
    // ---- slot lists and the dense row; they take over the LDS of the cut
    u32x2_t* rec = reinterpret_cast<u32x2_t*>(topk_dyn);              // [K] records {channel, value}
    E* zrow = reinterpret_cast<E*>(topk_dyn + ((size_t)2 * K * 4 + 15) / 16 * 16);   // [ldz] (FUSED)
    const RowCut cut = row_cut<NT, NCH, false>(v, F, K, a.far, *reinterpret_cast<RowCutLds<NT>*>(topk_dyn));
    // values equal to tau on both sides of the cut, or NaN (uniform): decided once, a value that is out becomes a NaN
    const bool keyed = cut.end != 0;
    if (cut.last != 0x7FFFFFFF && !keyed) {
        int jv = tid * 4;
        asm volatile("" : "+v"(jv));
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (v[c][e] == cut.tau && c * CHUNK + jv + e > cut.last) v[c][e] = __builtin_nanf("");
    }

    // ---- one ballot sweep: per-lane prefixes in registers, per-wave totals to LDS
    int pg[NCH];
    int jb = tid * 4;
    asm volatile("" : "+v"(jb));                            // (channel numbers are formed where they are used, not kept in registers)
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        int lg = 0, ngt = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bool in = v[c][e] >= cut.tau;
            if (keyed) in = cut.in(v[c][e], c * CHUNK + jb + e);
            const uint64_t bg = __ballot(in);
            lg += mbcnt(bg);
            ngt += __popcll(bg);
        }
        pg[c] = lg;
        if (lane == 0) tab[c * NW + wave] = ngt;
    }
    if constexpr (DENSE) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int j0 = c * CHUNK + jb;
            if (j0 >= a.ldg) break;                         // (ldg is a multiple of 4)
            f32x4_t g = a.g_raw ? *reinterpret_cast<const f32x4_t*>(a.g_raw + row * a.ldg + j0) : f32x4_t{v[c][0], v[c][1], v[c][2], v[c][3]};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                bool in = v[c][e] >= cut.tau;
                if (keyed) in = cut.in(v[c][e], j0 + e);
                g[e] = in ? silu_f32(g[e]) : kNotSelected;
            }
            *reinterpret_cast<f32x4_t*>(a.sd + row * a.ldg + j0) = g;
        }
    }
    __syncthreads();
    // exclusive prefix of the totals in (chunk, wavefront) order: the first n lanes of every wavefront hold one total each
    constexpr int n = NCH * NW;
    int base[NCH];
    if constexpr (n <= 64) {
        const int t = lane < n ? tab[lane] : 0;
        const int ex = wave_inclusive_sum(t) - t;
#pragma unroll
        for (int c = 0; c < NCH; ++c) base[c] = __builtin_amdgcn_readlane(ex, c * NW + __builtin_amdgcn_readfirstlane(wave));
    } else {
        int run = 0;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                if (w == wave) base[c] = run;
                run += tab[c * NW + w];
            }
    }
    if (FUSED) {                                            // (the cut's LDS is dead since the last barrier)
        constexpr int PER = 16 / (int)sizeof(E);
        for (int i = tid * PER; i < (int)a.ldz; i += NT * PER) *reinterpret_cast<u32x4_t*>(zrow + i) = u32x4_t{0, 0, 0, 0};
    }
    asm volatile("" : "+v"(jb));
    // ---- rank: every selected channel drops (channel, gate value) into LDS at its
    //      output slot (number of selected channels before it)
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int j0 = c * CHUNK + jb;
        int slot = base[c] + pg[c];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bool in = v[c][e] >= cut.tau;
            if (keyed) in = cut.in(v[c][e], j0 + e);
            if (in) {
                rec[min(slot, K - 1)] = u32x2_t{(uint32_t)(j0 + e), __float_as_uint(v[c][e])};
                ++slot;
            }
        }
    }
    __syncthreads();
    // ---- write the compact outputs slot by slot (coalesced) and scatter z' into the dense row; the gathered loads of up to four slots of a
    //      thread go out together (8192 rows of 5461: K 4000 255 us, 280 with a slot at a time, K 683 88.8 and 90.3)
    auto write_slots = [&](auto slots_c) {
        constexpr int NS = decltype(slots_c)::value;
        for (int s0 = tid; s0 < K; s0 += NS * NT) {
            int j[NS];
            float g[NS], u[NS];
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const u32x2_t r = rec[min(s0 + q * NT, K - 1)];
                j[q] = (int)min(r[0], (uint32_t)(F - 1));     // (every slot holds a channel: the bound only guards the loads)
                g[q] = a.g_raw ? a.g_raw[row * a.ldg + j[q]] : __uint_as_float(r[1]) + 0.0f;      // (-0.0 is stored as +0.0)
                if (FUSED) u[q] = Elem<E>::load(a.u + row * a.ldu + j[q]);
            }
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const int sl = s0 + q * NT;
                if (sl >= K) break;
                a.idx[row * K + sl] = j[q];
                if (a.gsel_f32) a.gsel_f32[row * K + sl] = g[q];
                if (a.gvals) Elem<E>::store(a.gvals + row * K + sl, g[q]);
                if (FUSED) {
                    Elem<E>::store(a.uvals + row * K + sl, u[q]);
                    Elem<E>::store(zrow + j[q], silu_f32(g[q]) * u[q]);
                }
            }
        }
    };
    if (K <= NT) write_slots(std::integral_constant<int, 1>{});
    else if (K <= 2 * NT) write_slots(std::integral_constant<int, 2>{});
    else write_slots(std::integral_constant<int, 4>{});
    if (FUSED) {
        __syncthreads();
        constexpr int PER = 16 / (int)sizeof(E);
        E* zout = a.zd + row * a.ldz;
        for (int i = tid * PER; i < (int)a.ldz; i += NT * PER)
            *reinterpret_cast<u32x4_t*>(zout + i) = *reinterpret_cast<const u32x4_t*>(zrow + i);
    }
}

// Eight wavefronts per SIMD up to six chunks: rows come and go, and what one waits for the others compute.  With U gathered at the
// selected channels (instead of the whole row in registers) that costs up to four spilled registers in the rare general step.  Rows of 11008,
// K 1376, 8192 of them: 205 us with four wavefronts, 155 with eight (5.2 TB/s, the rate of a copy); 5461 / 683: 102 and 92.
template <class E, int NT, int NCH, bool FUSED>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : NCH <= 6 ? 8 : NCH <= 8 ? 6 : 4) void topk_rows_kernel(TopkArgs<E> a) {
    extern __shared__ __align__(16) unsigned char topk_dyn[];
    topk_row_body<E, NT, NCH, FUSED>(a, blockIdx.x, topk_dyn);
}

// Dynamic LDS of topk_rows_kernel: the bins and lists of the cut, reused for the slot records and, in
// the fused forward, the dense row.
inline size_t topk_reg_dyn_lds(int K, int64_t ldz, size_t elem, bool fused) {
    size_t lists = (size_t)2 * K * 4;
    lists = (lists + 15) / 16 * 16;
    if (fused) lists += (size_t)ldz * elem;
    const size_t cut = sizeof(RowCutLds<1024>);      // (the largest of them)
    return lists > cut ? lists : cut;
}

inline size_t topk_lds_bytes(int F, int NT, int VEC) {
    const int chunk = NT * VEC;
    const int nchunk = (F + chunk - 1) / chunk;
    return (size_t)nchunk * chunk * 4 + kTopkBins * 4 + (size_t)2 * nchunk * (NT / 64) * 4 + (NT / 64) * 4;
}

}  // namespace moc
