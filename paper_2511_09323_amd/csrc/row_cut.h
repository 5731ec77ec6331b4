// The cut of one row's Top-K, found by a workgroup that holds the row in registers: shared by the training forward's row
// selection (topk.h) and by decode (decode_rows.h).
//
// Method: one histogram over 2048 bins of equal width between 0 and the row's maximum, or a bound on the K-th value where outliers lie
// far above it (a product, a conversion, a clamp and an LDS atomic per value), a scan from the top for the bin that holds the K-th value,
// and a direct ranking of that bin's few values by every wavefront.  Where more than a third of the row is selected, half of the
// bins lie below zero.  Values spread over linear bins, so the atomics hardly collide and the bin of the cut holds a handful of values: at the
// 7B shape (11008 gates around zero, K = 1376) about five.  Everything else -- fewer than
// K non-negative values, more than 64 values in the bin (ties), infinities -- goes on with what holds the cut (a bin, the positive ones,
// zeros, the negative ones, an infinity) by up to two general steps.  Rows that these do not resolve (values spread over many
// powers of two) or whose cut lies among NaN (+NaN above +inf, -NaN below -inf) are cut by a radix select on float_key.
// What bounds it: instructions per value (one row occupies one workgroup, often one compute unit) and the dependent steps
// between barriers; about nine instructions per value and six barriers.  The radix select it replaces (three histograms over key digits,
// colliding atomics on the exponent digit, thirteen barriers) took 8.8 us for one decode row of 11008 as a launch of its own and
// 225 us for 8192 such rows in the training forward, against 4.9 us inside the decode gather and 155 us here.
// Other rows, 8192 of 11008, K 1376, in a forward at d 64 (this / the radix select; 182 / 229 us for Gaussian rows): one value of 1000
// standard deviations 180 / 220, hundreds of ties at the cut 202 / 260, all zero 176 / 1013, all negative 225 / 334, 95 % -inf 211 / 999,
// K 5504 372 / 467.  The paths for these cost Gaussian rows an eighth more scalar instructions and
// branches (the vector instructions are as many): nothing in the forward, 45.0 -> 47.5 us for 16384 rows of 2048 on their own (67 with the
// radix select).  Slower than it: values spread evenly over 200 powers of two, 551 / 225.
#pragma once
#include "common.h"

namespace moc {

constexpr int kCutBins = 2048;

// Channel j with value v is selected iff v > tau, or v == tau and j <= last; with `end` set (rows with NaN, or K = F; last < INT_MAX)
// the same of keys, for the channels below end.
struct RowCut {
    float tau;
    int last;      // INT_MAX: every value equal to tau is selected
    int before;    // BEFORE: selected channels below c0
    int end = 0;
    uint32_t key = 0;
    __device__ __forceinline__ bool in(float v, int j) const {
        if (end) return j < end && (float_key(v) > key || (float_key(v) == key && j <= last));
        return v > tau || (v == tau && j <= last);
    }
};

template <int NT> struct RowCutLds {
    uint32_t count[64 + kCutBins];      // a word per lane for what lies below the bins, then the bins
    float cand_v[64];
    int cand_j[64];
    float red_f[2][NT / 64];
    int red_i[NT / 64], red_b[NT / 64];
    int bin, need, cnt, ncand;
};

// The bins end at the maximum or, where outliers lie above the rest, at 1.5 / K of the sum S of the positive values (the K-th value is at most
// S / K; 1.5 because S comes from a quarter of the row) or ten times their mean over the row, whichever is larger: what lies above shares
// the last bin.  This is the factor for the sum of that quarter.
inline float cut_far(int F, int K) { return fmaxf(6.0f / (float)K, 40.0f / (float)F); }

// v[c][e] is the value of channel c * 4 NT + tid * 4 + e; what lies past the row's end (F) holds -inf.  1 <= K <= F.
// far: cut_far(F, K).  BEFORE: also counts the selected channels below c0 (on the way, from the bins).
// Exactly K channels are selected, whatever the values.  L may be overwritten after a barrier.
template <int NT, int NCH, bool BEFORE>
__device__ __forceinline__ RowCut row_cut(const float (&v)[NCH][4], int F, int K, float far, RowCutLds<NT>& L, int c0 = 0) {
    constexpr int NW = NT / 64, BPT = kCutBins / NT;
    static_assert(BPT == 2 || BPT == 4 || BPT == 8, "256, 512 or 1024 threads");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float kInf = __builtin_inff();
    uint32_t* const hist = L.count + 64;
    // a copy the compiler does not recognise: channel numbers are formed where they are used instead of kept in registers
    auto opaque = [](int t) {
        asm volatile("" : "+v"(t));
        return t;
    };
    // the same of a value, so that what is formed from it is not kept from one pass to the next
    auto opaque_value = [](float t) {
        asm volatile("" : "+v"(t));
        return t;
    };

    if (K == F) return RowCut{0.0f, F - 1, min(c0, F), F, 0u};      // (every key is above or equal to 0)

    auto clear_bins = [&](int base) {
        if (BPT == 2) *reinterpret_cast<u32x2_t*>(hist + base) = u32x2_t{0, 0};
        else
#pragma unroll
            for (int q = 0; q < BPT; q += 4) *reinterpret_cast<u32x4_t*>(hist + base + q) = u32x4_t{0, 0, 0, 0};
    };
    // the maximum as an integer: the same as the floats' where one is not negative, and a NaN shows above infinity
    auto bits_max = [](float a, float b) { return __int_as_float(max(__float_as_int(a), __float_as_int(b))); };
    float vmax = __int_as_float((int)0x80000000);
#pragma unroll
    for (int c = 0; c < NCH; ++c) vmax = bits_max(bits_max(bits_max(vmax, v[c][0]), v[c][1]), bits_max(v[c][2], v[c][3]));
    vmax = __int_as_float(wave_reduce_last(__float_as_int(vmax), (int)0x80000000, [](int a, int b) { return max(a, b); }));
    float pos = 0.0f;                                        // sum of the positive values, from a quarter of the row
#pragma unroll
    for (int c = 0; c < NCH; ++c) pos += __int_as_float(max(__float_as_int(v[c][0]), 0));
    pos = __int_as_float(wave_reduce_last(__float_as_int(pos), 0, [](int a, int b) { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }));
    clear_bins(BPT * tid);
    if (lane == 63) { L.red_f[0][wave] = vmax; L.red_f[1][wave] = pos; }
    if (tid == 0) { L.bin = 0; L.need = K; L.cnt = 0; L.ncand = 0; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NW; ++w) vmax = bits_max(vmax, L.red_f[0][w]);
    // (decisions are taken on scalar copies of what all lanes hold: branches instead of lane masks)
    vmax = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(vmax)));
    pos = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) pos += L.red_f[1][w];

    // Scans the bins from the top for the one in which the running count reaches `need`; L.bin, L.need (what is still wanted in
    // that bin) and L.cnt (its size) are set, the bins are cleared and the total of all bins is returned.
    auto scan = [&](int need) {
        __syncthreads();
        const int base = kCutBins - BPT * (tid + 1);         // thread order is descending bin order
        uint32_t h[BPT];
        if (BPT == 2) {
            const u32x2_t t = *reinterpret_cast<const u32x2_t*>(hist + base);
            h[0] = t[0]; h[1] = t[1];
        } else {
#pragma unroll
            for (int q = 0; q < BPT; q += 4) {
                const u32x4_t t = *reinterpret_cast<const u32x4_t*>(hist + base + q);
                h[q] = t[0]; h[q + 1] = t[1]; h[q + 2] = t[2]; h[q + 3] = t[3];
            }
        }
        int local = 0;
#pragma unroll
        for (int q = 0; q < BPT; ++q) local += (int)h[q];
        int inc = wave_inclusive_sum(local);
        if (lane == 63) L.red_i[wave] = inc;
        clear_bins(base);                                    // (this thread's own, for a repetition)
        __syncthreads();
        int total = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            inc += w < wave ? L.red_i[w] : 0;
            total += L.red_i[w];
        }
        int run = inc - local;
        if (run < need && inc >= need) {                     // the bin is one of mine
            int fb = -1, fneed = 0, fh = 0;
#pragma unroll
            for (int q = BPT - 1; q >= 0; --q) {
                if (fb < 0 && run + (int)h[q] >= need) { fb = base + q; fneed = need - run; fh = (int)h[q]; }
                run += (int)h[q];
            }
            L.bin = fb;
            L.need = fneed;
            L.cnt = fh;
        }
        __syncthreads();
        return total;
    };
    auto keep = [&](float t, int j) {
        const int p = atomicAdd(&L.ncand, 1);
        if (p < 64) { L.cand_v[p] = t; L.cand_j[p] = j; }
    };
    // the cut among the cnt <= 64 kept values: the need-th in the order (value descending, channel ascending)
    // (`above`: this thread's values above the kept ones with channels below c0)
    auto rank_kept = [&](int cnt, int need, int above) {
        if (BEFORE) {
            above = (int)wave_sum((float)above);             // exact: counts are far below 2^24
            if (lane == 0) L.red_b[wave] = above;
        }
        __syncthreads();
        const int i = min(lane, max(cnt, 1) - 1);
        const float cv = L.cand_v[i];
        const int cj = L.cand_j[i];
        int rank = 0;
        for (int q = 0; q < cnt; ++q) {
            const float ov = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cv), q));
            const int oj = __builtin_amdgcn_readlane(cj, q);
            rank += (ov > cv || (ov == cv && oj < cj)) ? 1 : 0;
        }
        const uint64_t m = __ballot(lane < cnt && rank == need - 1);
        const int src = m ? __ffsll((unsigned long long)m) - 1 : 0;
        const float tau = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(cv), src));
        const bool cut_ties = __ballot(lane < cnt && cv == tau && rank >= need) != 0;
        int before = 0;
        if (BEFORE) {
            before = __popcll(__ballot(lane < cnt && rank < need && cj < c0));
#pragma unroll
            for (int w = 0; w < NW; ++w) before += L.red_b[w];
        }
        return RowCut{tau, cut_ties ? (int)__builtin_amdgcn_readlane(cj, src) : 0x7FFFFFFF, before};
    };

    int need = K, fb = 0;
    float scale0 = 0.0f, zero_bin = 0.0f;
    auto bin_at = [&](float t) { return cvt_i32(fmaf(t, scale0, zero_bin)); };
    if (__float_as_int(vmax) > __float_as_int(1e-30f) && __float_as_int(vmax) < __float_as_int(1e38f)) {
        const float end = pos * far;
        const float range = end > 1e-30f ? fminf(end, vmax) : vmax;      // (nothing positive in that quarter: up to the maximum)
        // From zero upwards, or from -range upwards where more than a third of the row is selected and the cut may lie below zero.
        zero_bin = 3 * K > F ? kCutBins / 2 : 0.0f;
        scale0 = ((float)kCutBins - 2.0f - zero_bin) * __builtin_amdgcn_rcpf(range);      // bin_at(v) < 2047 for every v <= range
        // (no branch per value: those below count into the lane's own word in front of the bins; what truncates to bin 0 from
        // below spoils that bin, which is therefore not used)
        const int floor_bin = -1 - lane;
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) atomicAdd(hist + clamp_i32(bin_at(v[c][e]), floor_bin, kCutBins - 1), 1u);
        const int total = __builtin_amdgcn_readfirstlane(scan(need)), bin = __builtin_amdgcn_readfirstlane(L.bin);
        fb = total >= need ? bin : 0;
        const int cnt = __builtin_amdgcn_readfirstlane(L.cnt);
        if (fb > 0) {
            need = __builtin_amdgcn_readfirstlane(L.need);
            if (cnt <= 64 && fb < kCutBins - 1) {
                asm volatile("" : "+v"(scale0));             // (keeps the compiler from holding every value's bin in a register)
                uint32_t near = 1;
                int above = 0;
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    int x[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        x[e] = bin_at(v[c][e]);      // (down to the lowest integer: no difference of it is formed)
                        near = min(near, (uint32_t)x[e] ^ (uint32_t)fb);
                    }
                    if (BEFORE && c * 4 * NT < c0) {         // (uniform; only the chunk that holds c0 needs the channel test)
                        const int stop = c0 - (c * 4 * NT + tid * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) above += (x[e] > fb && e < stop) ? 1 : 0;
                    }
                }
                if (near == 0) {
                    const int jb = opaque(tid * 4);
                    asm volatile("" : "+v"(scale0));
#pragma unroll
                    for (int c = 0; c < NCH; ++c)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (bin_at(v[c][e]) == fb) keep(v[c][e], c * 4 * NT + jb + e);
                }
                return rank_kept(cnt, need, above);
            }
        }
    }
    // f(value, channel) for this thread's values; every pass of the steps below forms what it needs anew
    auto each = [&](const auto& f) {
        const int jb = opaque(tid * 4);
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) f(opaque_value(v[c][e]), c * 4 * NT + jb + e);
    };
    // how many values of the row satisfy p, and how many q (each at most 32768): first * 2^16 + second
    auto count2 = [&](const auto& p, const auto& q) {
        uint32_t np = 0, n = 0;
        each([&](float t, int j) {
            np += p(t, j) ? 1u : 0u;
            n += q(t, j) ? 1u : 0u;
        });
        n = (uint32_t)wave_inclusive_sum((int)(n + (np << 16)));
        __syncthreads();
        if (lane == 63) L.red_i[wave] = (int)n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) n += (uint32_t)L.red_i[w];
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
    };
    auto count = [&](const auto& p) { return (int)count2([](float, int) { return false; }, p); };
    // the channel of the n-th value in question, in one pass: the values of every (chunk, wavefront) are counted, the one that holds the
    // n-th is found from the counts, and its wavefront looks the channel up.  (The counts take the place of the bins.)
    auto nth_channel = [&](int n, const auto& pred) {
        constexpr int NG = NCH * NW;
        const int jb = opaque(tid * 4);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            int m = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) m += __popcll(__ballot(pred(v[c][e], c * 4 * NT + jb + e)));
            if (lane == 0) hist[c * NW + wave] = (uint32_t)m;
        }
        if (tid == 0) L.bin = F - 1;
        __syncthreads();
        int group = -1, left = n;                            // the group and what is still wanted in it
#pragma unroll
        for (int q = 0; q < NG; q += 64) {
            const int m = q + lane < NG ? (int)hist[q + lane] : 0;
            const int inc = wave_inclusive_sum(m);
            const uint64_t reached = __ballot(inc >= left);
            if (group < 0) {
                if (reached) {
                    const int at = __ffsll((unsigned long long)reached) - 1;
                    left -= __builtin_amdgcn_readlane(inc - m, at);
                    group = q + at;
                } else {
                    left -= __builtin_amdgcn_readlane(inc, 63);
                }
            }
        }
        if (group >= 0 && group % NW == wave) {
#pragma unroll
            for (int c = 0; c < NCH; ++c)
                if (c == group / NW) {
                    const int j0 = c * 4 * NT + opaque(tid * 4);
                    bool in[4];
                    int rank = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        in[e] = pred(opaque_value(v[c][e]), j0 + e);
                        rank += mbcnt(__ballot(in[e]));
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (in[e] && ++rank == left) L.bin = j0 + e;
                }
        }
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(L.bin);
    };
    const bool nan = __float_as_int(vmax) > 0x7F800000;      // +NaN lies above +inf
    auto finish = [&](RowCut cut) {
        if (nan) {
            cut.end = F;
            cut.key = float_key(cut.tau);
            cut.last = min(cut.last, F - 1);
        }
        if (BEFORE) cut.before = count([&](float t, int j) { return j < c0 && cut.in(t, j); });
        return cut;
    };
    // ---- general step on the closed range [lo, hi] of the values in question: every value above hi is selected, `need` of those
    //      inside are.  A repetition takes at least the range's two ends apart, so it ends.
    float lo, hi;
    auto range_of = [&](const auto& in_question) {
        float a = kInf, b = -kInf;
        each([&](float t, int) {
            if (in_question(t)) { a = fminf(a, t); b = fmaxf(b, t); }
        });
        a = wave_min(a);
        b = wave_max(b);
        __syncthreads();
        if (lane == 0) { L.red_f[0][wave] = a; L.red_f[1][wave] = b; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) { a = fminf(a, L.red_f[0][w]); b = fmaxf(b, L.red_f[1][w]); }
        lo = a;
        hi = b;
    };
    // ---- the values in question: those of the cut's bin or, without one, +inf, the positive ones, zeros, the negative ones or -inf, whichever
    //      hold the cut once +NaN and what lies above are selected
    bool found = fb > 0;
    lo = hi = 0.0f;
    if (found) {
        range_of([&](float t) { return min(bin_at(t), kCutBins - 1) == fb; });
    } else {
        need = K;
        if (nan) need -= count([](float t, int) { return __float_as_int(t) > 0x7F800000; });
        if (__float_as_int(vmax) >= 0x7F800000 && need > 0) {
            const int n = count([&](float t, int) { return t == kInf; });
            found = need <= n;
            if (found) lo = hi = kInf;
            else need -= n;
        }
        const bool below = __float_as_int(vmax) < 0;         // no value above -0.0, which is one of the negative ones then
#pragma unroll 1
        for (int q = below ? 1 : 0; q < 2 && !found && need > 0; ++q) {
            const float a = q ? -kInf : 0.0f, b = q ? (below ? 0x1p-149f : 0.0f) : kInf;
            const uint32_t n = count2([&](float t, int) { return t > a && t < b; }, [&](float t, int j) { return t == a && j < F; });
            const int inside = (int)(n >> 16), equal = (int)(n & 0xFFFF);
            if (need <= inside) {
                if (q == 0 && scale0 != 0.0f) break;         // positive ones that the bins did not tell apart: by keys
                found = true;
                range_of([&](float t) { return t > a && t < b; });
            } else {
                need -= inside;
                found = need <= equal;
                if (found) lo = hi = a;
                else need -= equal;
            }
        }
    }
#pragma unroll 1
    for (int it = 0; found && it < 3; ++it) {
        if (lo == hi) return finish(RowCut{lo, nth_channel(need, [&](float t, int j) { return t == lo && j < F; }), 0});
        if (it == 2) break;
        // monotonic in t, lo falls into bin 0 and hi into the last ones (`pre` keeps the factor finite for tiny ranges)
        const float pre = hi - lo < 1e-30f ? 0x1p100f : 1.0f;
        const float scale = (float)kCutBins / ((hi - lo) * pre);
        auto bin_of = [&](float t) { return min(kCutBins - 1, (int)fminf((t - lo) * pre * scale, 4096.0f)); };
        each([&](float t, int) {
            if (t >= lo && t <= hi) atomicAdd(hist + bin_of(t), 1u);
        });
        (void)scan(need);
        fb = L.bin;
        need = L.need;
        const int cnt = L.cnt;
        if (cnt <= 64) {
            each([&](float t, int j) {
                if (t >= lo && t <= hi && bin_of(t) == fb) keep(t, j);
            });
            return finish(rank_kept(cnt, need, 0));
        }
        const float l0 = lo, h0 = hi;
        range_of([&](float t) { return t >= l0 && t <= h0 && min(kCutBins - 1, (int)fminf((t - l0) * pre * scale, 4096.0f)) == fb; });
    }
    // ---- values that two more steps do not tell apart (spread over many powers of two), a cut among NaN: by the digits of their keys
    uint32_t key = 0;
    need = K;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0, bits = pass == 2 ? 10 : 11;
        each([&](float t, int j) {
            const uint32_t k = float_key(t);
            if (j < F && (pass == 0 || k >> (shift + bits) == key)) atomicAdd(hist + (k >> shift & ((1u << bits) - 1)), 1u);
        });
        (void)scan(need);
        key = key << bits | (uint32_t)L.bin;
        need = L.need;
    }
    RowCut cut{0.0f, nth_channel(need, [&](float t, int j) { return j < F && float_key(t) == key; }), 0, F, key};
    if (BEFORE) cut.before = count([&](float t, int j) { return j < c0 && cut.in(t, j); });
    return cut;
}

}  // namespace moc
