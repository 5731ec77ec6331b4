// Launch helpers shared by the entry-point files: GEMM dispatch (tile choice, MFMA or generic
// kernel, batched / paired / grouped launches), the row Top-K and grouped-selection launchers.
#pragma once
#include <algorithm>
#include <type_traits>

#include "api_common.h"
#include "epilogue.h"
#include "gemm_f32.h"
#include "gemm_generic.h"
#include "gemm_mfma.h"
#include "gemm_pingpong.h"
#include "group_select.h"
#include "kernel_attrs.h"
#include "topk.h"

namespace mocapi {
using namespace moc;

// ------------------------------------------------------------------------ GEMM dispatch
// Workgroups of a persistent GEMM launch: one per compute unit (the kernels' LDS use allows no more),
// or 0 (one workgroup per tile) with MOC_GEMM_PERSISTENT=0.
inline int persistent_workgroups() { return options().gemm_persistent ? device_cu_count() : 0; }

inline int forced_tile() { return options().tile == 256 ? 0 : options().tile == 192 ? 1 : options().tile == 128 ? kTile128 : -1; }

// The cheapest of the tile shapes in MASK on this device (gemm_plan.h); MOC_GEMM_TILE forces one.
template <unsigned MASK, class TilesOf> int choose_tile(const TilesOf& tiles_of, int nk, double* cost_out = nullptr) {
    return cheapest_tile(MASK, tiles_of, nk, std::max(1, device_cu_count()), forced_tile(), cost_out);
}

// f(tile index as a compile-time constant) for the tile shape `t` of MASK.
template <unsigned MASK, int C = 0, class F> hipError_t with_tile(int t, const F& f) {
    if constexpr (C < kGemmTiles) {
        if constexpr ((MASK >> C) & 1u)
            if (t == C) return f(std::integral_constant<int, C>{});
        return with_tile<MASK, C + 1>(t, f);
    } else {
        return hipErrorInvalidValue;
    }
}
// One persistent workgroup per compute unit for the tiles that fill one, a workgroup per tile for the others.
template <int C> int tile_workgroups() { return kGemmTile[C].resident == 1 ? persistent_workgroups() : 0; }

inline bool gemm_has_tail(const MfmaProblem& pr) { return pr.Kc % kMfmaBK != 0 || pr.Kc2 % kMfmaBK != 0; }
// Whether a contraction tail can run as "padded" (TAILMODE 2, see gemm_mfma.h).
inline bool gemm_padded(const MfmaProblem& pr) {
    return pr.a_zero_padded && pr.B.km && (pr.A.km || pr.A.ld >= round_up(std::max(pr.Kc, pr.Kc2), kMfmaBK));
}

inline StreamKArgs streamk_args(const StreamKArea& a, int nk) {
    return StreamKArgs{a.part, a.flag, next_streamk_tag(), std::max(1, nk / 8), std::max(0, options().gemm_streamk_spin)};
}
inline int streamk_workgroups() { return std::min(persistent_workgroups(), kStreamKSlots) / 8 * 8; }

// Memory of a launch's workspace that holds nothing while a product runs, for the shares of a split contraction.
struct ShareScratch {
    float* p = nullptr;
    size_t bytes = 0;
};

// f(tile index as a compile-time constant) for the large tile `t`.
template <int C = 0, class F> hipError_t with_pp_tile(int t, const F& f) {
    if constexpr (C < kPpTiles) {
        if (t == C) return f(std::integral_constant<int, C>{});
        return with_pp_tile<C + 1>(t, f);
    } else {
        return hipErrorInvalidValue;
    }
}
template <class T> PpOut pp_out(const EpiStore<T>& e) { return PpOut{e.C, e.ldc, 0, e.N, std::is_same<T, float>::value}; }
// Whether the kernel of gemm_pingpong.h takes the problem (a tile shape named by the environment is one of gemm_mfma.h).
template <class Epi> bool pp_takes(const MfmaProblem&, const Epi&) { return false; }
template <class T> bool pp_takes(const MfmaProblem& pr, const EpiStore<T>& epi) {
    return !options().force_generic && options().tile == 0 && epi.pad_to == 0 && pp_problem_ok(pr, pp_out(epi));
}

// One product (its contraction in `shares` shares) on large tiles.
template <bool AKM, bool BKM, bool F32> hipError_t launch_pp(int tile, const MfmaProblem& pr, const PpOut& out, int shares, hipStream_t st) {
    PpWork<1> w;
    w.pr[0] = pr;
    w.out[0] = out;
    w.nprob = 1;
    w.nsplit = shares;
    return with_pp_tile(tile, [&](auto c) {
        constexpr PpTile t = kPpTile[decltype(c)::value];
        return launch_gemm_bf16_pp<t.bm, t.bn, AKM, BKM, F32 ? 1 : 0, 1>(w, persistent_workgroups(), st);
    });
}

// Can the product be cut into shares: A k-contiguous and padded, B k-major, stored contiguously, memory for the shares.
template <class E> bool can_share(const GemmProblem<E>& pr, const EpiStore<E>& epi, const ShareScratch& sc) {
    return sc.p && epi.ldc == epi.N && epi.N == pr.N && epi.N % 4 == 0 && options().tile == 0 && gemm_padded(pr);
}

// Bytes of scratch the shares of a product may take, 0 if it cannot be cut.
template <class E, class Epi> size_t share_bytes(const GemmProblem<E>& pr, const Epi& epi, const ShareScratch& sc) {
    if constexpr (std::is_same<Epi, EpiStore<E>>::value) return can_share(pr, epi, sc) ? sc.bytes : 0;
    return 0;
}

template <class E>
moc_status run_gemm_shares(const char* name, const GemmProblem<E>& pr, const EpiStore<E>& epi, hipStream_t st, const ShareScratch& sc,
                           const GemmRoute& r) {
    const int64_t out = (int64_t)pr.M * pr.N;
    hipError_t e;
    if (r.pp) {
        e = launch_pp<false, true, true>(r.tile, pr, PpOut{sc.p, pr.N, out, pr.N, 1}, r.shares, st);
    } else {
        const EpiShare es{sc.p, pr.N, out, pr.N};
        e = with_tile<kTilesShares>(r.tile, [&](auto c) {
            constexpr GemmTile t = kGemmTile[decltype(c)::value];
            return launch_gemm_bf16_mfma_split<t.bm, t.bn, false, true, 2, EpiShare, 4, t.sets>(pr, es, r.shares, st);
        });
    }
    if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
    const int64_t n4 = out / 4;
    hipLaunchKernelGGL((reduce_shares_kernel<E>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, sc.p, r.shares, out, n4, epi.C);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

// Runs C = A B^T (+ second segment) with the epilogue `epi`.  AKM / BKM state the operand layouts
// at compile time (they must match pr.A.km / pr.B.km).  bf16 and fp32 problems that satisfy the assumptions of a matrix-core
// kernel go there, everything else to the generic kernel.
// `sk`, if given and carved, lets a product whose whole tiles would leave part of the chip idle in their last
// round split its work along the contraction instead (256 x 256 tiles, contraction a multiple of 32); `scratch` is memory for
// run_gemm_shares; `one_sum` see launch_gemm_f32.
template <class E, bool AKM, bool BKM, class Epi>
moc_status run_gemm(const char* name, const GemmProblem<E>& pr, const Epi& epi, hipStream_t st, const StreamKArea* sk = nullptr,
                    bool one_sum = false, const ShareScratch& scratch = ShareScratch{}) {
    Span span(name, st);
    if constexpr (std::is_same<E, bf16_t>::value && !(AKM && BKM)) {      // (k-major x k-major products: run_gemm_batch3, run_gemm_grouped)
        if (!options().force_generic && mfma_problem_ok(pr)) {
            const int nk = slice_count(pr.Kc, pr.Kc2);
            const bool tail = gemm_has_tail(pr), padded = gemm_padded(pr);
            if (sk && sk->part && options().gemm_streamk && options().tile == 0 && !tail) {
                const int wgs = streamk_workgroups();
                if (streamk_pays(tile_count(pr.M, pr.N, kGemmTile[0]), nk, wgs)) {
                    hipError_t e = launch_gemm_bf16_mfma_streamk<256, 256, AKM, BKM, 0, Epi, 4, 3>(pr, epi, streamk_args(*sk, nk), wgs, st);
                    if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                    return MOC_OK;
                }
            }
            constexpr bool kStore = std::is_same<Epi, EpiStore<bf16_t>>::value || std::is_same<Epi, EpiStore<float>>::value;
            constexpr unsigned kMask = !kStore ? kTilesBasic : BKM ? kTilesKm : kTilesAll;
            constexpr bool kShares = !AKM && BKM && std::is_same<Epi, EpiStore<E>>::value;
            const GemmRoute route = gemm_route(kMask, pr.M, pr.N, pr.Kc, pr.Kc2, sizeof(E), pp_takes(pr, epi), kShares ? share_bytes(pr, epi, scratch) : 0,
                                               std::max(1, device_cu_count()), forced_tile());
            if constexpr (kShares)
                if (route.shares > 1) return run_gemm_shares<E>(name, pr, epi, st, scratch, route);
            if constexpr (kStore) {
                if (route.pp) {
                    const hipError_t e = launch_pp<AKM, BKM, std::is_same<Epi, EpiStore<float>>::value>(route.tile, pr, pp_out(epi), 1, st);
                    if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                    return MOC_OK;
                }
            }
            const int best = route.tile;
            hipError_t e;
            if (!tail)
                e = with_tile<kMask>(best, [&](auto c) {
                    constexpr int C = decltype(c)::value;
                    constexpr GemmTile t = kGemmTile[C];
                    return launch_gemm_bf16_mfma<t.bm, t.bn, AKM, BKM, 0, Epi, 4, t.sets>(pr, epi, st, tile_workgroups<C>());
                });
            else if (BKM && padded)
                e = with_tile<kMask>(best, [&](auto c) {
                    constexpr int C = decltype(c)::value;
                    constexpr GemmTile t = kGemmTile[C];
                    return launch_gemm_bf16_mfma<t.bm, t.bn, AKM, BKM, BKM ? 2 : 1, Epi, 4, t.sets>(pr, epi, st, tile_workgroups<C>());
                });
            else {    // a contraction tail without padding (d % 32 != 0); the smaller shapes were measured without one only
                const int basic = choose_tile<kTilesBasic>([&](const GemmTile& t) { return tile_count(pr.M, pr.N, t); }, nk);
                e = with_tile<kTilesBasic>(basic, [&](auto c) {
                    constexpr int C = decltype(c)::value;
                    constexpr GemmTile t = kGemmTile[C];
                    return launch_gemm_bf16_mfma<t.bm, t.bn, AKM, BKM, 1, Epi, 4, t.sets>(pr, epi, st, tile_workgroups<C>());
                });
            }
            if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
            return MOC_OK;
        }
    }
    if constexpr (std::is_same<E, float>::value) {
        if (!options().force_generic && f32_problem_ok(pr)) {
            if constexpr (!AKM && BKM && std::is_same<Epi, EpiStore<float>>::value) {
                if (!one_sum && scratch.p && epi.ldc == epi.N && epi.N == pr.N && epi.N % 4 == 0 && epi.pad_to == 0) {
                    const F32Shares plan = f32_shares(pr.M, pr.N, pr.Kc, pr.Kc2, scratch.bytes, std::max(1, device_cu_count()));
                    const int64_t out = (int64_t)pr.M * pr.N, n4 = out / 4;
                    if (plan.shares > 1) {
                        const hipError_t e = launch_gemm_f32_shares(pr, EpiShare{scratch.p, pr.N, out, pr.N}, plan, st);
                        if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                        hipLaunchKernelGGL((reduce_shares_kernel<float>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, scratch.p, plan.shares, out, n4, epi.C);
                        HIP_TRY(hipGetLastError());
                        return MOC_OK;
                    }
                }
            }
            hipError_t e = launch_gemm_f32<AKM, BKM, Epi, 1>(F32Batch<Epi, 1>{{pr}, {epi}}, one_sum, device_cu_count(), st);
            if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
            return MOC_OK;
        }
    }
    launch_gemm_generic<E, Epi>(pr, epi, st);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

// Several products in one launch on large tiles: they agree in their columns and leading dimensions, and the kernel takes every one of them.
template <class T> bool pp_group_takes(int n, const MfmaProblem* pr, const EpiStore<T>* epi) {
    for (int z = 0; z < n; ++z)
        if (pr[z].M != 0 && !(pp_takes(pr[z], epi[z]) && pr[z].N == pr[0].N && pr[z].A.ld == pr[0].A.ld && pr[z].B.ld == pr[0].B.ld)) return false;
    return true;
}
template <bool AKM, bool BKM, int F32, int NB> hipError_t launch_pp_group(int tile, PpWork<NB>& w, hipStream_t st) {
    w.nsplit = 1;
    return with_pp_tile(tile, [&](auto c) {
        constexpr PpTile t = kPpTile[decltype(c)::value];
        return launch_gemm_bf16_pp<t.bm, t.bn, AKM, BKM, F32, NB>(w, persistent_workgroups(), st);
    });
}

// Three independent products of one shape (both operands k-major, plain stores) in one launch when
// a matrix-core kernel takes them; otherwise one run_gemm each.  Same tile choice as run_gemm, over the
// tiles of all three.
template <class E>
moc_status run_gemm_batch3(const char* name, const char* const names[3], const GemmProblem<E> pr[3], const EpiStore<E> epi[3],
                           hipStream_t st, const StreamKArea* sk = nullptr, const ShareScratch& scratch = ShareScratch{}) {
    if constexpr (std::is_same<E, bf16_t>::value) {
        const bool same = pr[0].M == pr[1].M && pr[0].M == pr[2].M && pr[0].N == pr[1].N && pr[0].N == pr[2].N &&
                          pr[0].Kc == pr[1].Kc && pr[0].Kc == pr[2].Kc && pr[0].Kc2 == 0 && pr[1].Kc2 == 0 && pr[2].Kc2 == 0;
        const bool tail = gemm_has_tail(pr[0]);
        const bool padded = gemm_padded(pr[0]) && gemm_padded(pr[1]) && gemm_padded(pr[2]);
        if (same && (!tail || padded) && !options().force_generic && mfma_problem_ok(pr[0]) && mfma_problem_ok(pr[1]) && mfma_problem_ok(pr[2])) {
            const int nk = slice_count(pr[0].Kc, 0);
            const bool pp = pp_group_takes(3, pr, epi) && !(sk && sk->part && options().gemm_streamk);
            const GemmRoute route = batch3_route(pr[0].M, pr[0].N, pr[0].Kc, pp, std::max(1, device_cu_count()), forced_tile());
            if (route.pp) {
                Span span(name, st);
                const int M = pr[0].M, N = pr[0].N;
                const bool tight = epi[0].ldc == N && epi[1].ldc == N && epi[2].ldc == N && epi[0].N == N && epi[1].N == N && epi[2].N == N;
                const Batch3Split split = tight && scratch.p && persistent_workgroups() ? batch3_split(M, N, pr[0].Kc, route, scratch.bytes, std::max(1, device_cu_count()))
                                                                                        : Batch3Split{};
                PpWork<3> w;
                for (int i = 0; i < 3; ++i) { w.pr[i] = pr[i]; w.out[i] = pp_out(epi[i]); }
                w.nprob = 3;
                if (split.rows)
                    for (int i = 0; i < 3; ++i) w.pr[i].M = split.rows;
                hipError_t e = launch_pp_group<true, true, 0, 3>(split.rows ? split.main : route.tile, w, st);
                if (e == hipSuccess && split.rows) {
                    // the rows behind the whole rounds, their contraction in shares
                    const int left = M - split.rows;
                    const int64_t out = (int64_t)left * N, n4 = out / 4;
                    ReduceOuts<bf16_t> outs;
                    for (int i = 0; i < 3; ++i) {
                        w.pr[i].M = left;
                        w.pr[i].A.p += split.rows;
                        w.pr[i].A.ext -= split.rows;
                        w.out[i] = PpOut{scratch.p + (int64_t)i * split.shares * out, N, out, N, 1};
                        outs.p[i] = epi[i].C + (int64_t)split.rows * N;
                    }
                    w.nsplit = split.shares;
                    e = split.rest == 0 ? launch_gemm_bf16_pp<256, 256, true, true, 1, 3>(w, persistent_workgroups(), st)
                                        : launch_gemm_bf16_pp<128, 256, true, true, 1, 3>(w, persistent_workgroups(), st);
                    if (e == hipSuccess) {
                        hipLaunchKernelGGL((reduce_shares_batch_kernel<bf16_t>), dim3((unsigned)((n4 + 255) / 256), 3), dim3(256), 0, st, scratch.p, split.shares,
                                           out, n4, outs);
                        e = hipGetLastError();
                    }
                }
                if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                return MOC_OK;
            }
            const int best = route.tile;
            MfmaBatch<EpiStore<E>, 3> b;
            for (int i = 0; i < 3; ++i) { b.pr[i] = pr[i]; b.epi[i] = epi[i]; }
            Span span(name, st);
            if (sk && sk->part && options().gemm_streamk && options().tile == 0 && !tail) {
                const int wgs = streamk_workgroups();
                if (streamk_pays(3 * tile_count(pr[0].M, pr[0].N, kGemmTile[0]), nk, wgs)) {
                    hipError_t e = launch_gemm_bf16_mfma_batch_streamk<256, 256, true, true, 0, EpiStore<E>, 3, 4, 3>(b, streamk_args(*sk, nk), wgs, st);
                    if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                    return MOC_OK;
                }
            }
            auto launch = [&](auto mode) {
                return with_tile<kTilesKm>(best, [&](auto c) {
                    constexpr int C = decltype(c)::value;
                    constexpr GemmTile t = kGemmTile[C];
                    return launch_gemm_bf16_mfma_batch<t.bm, t.bn, true, true, decltype(mode)::value, EpiStore<E>, 3, 4, t.sets>(b, st, tile_workgroups<C>());
                });
            };
            const hipError_t e = tail ? launch(std::integral_constant<int, 2>{}) : launch(std::integral_constant<int, 0>{});
            if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
            return MOC_OK;
        }
    }
    if constexpr (std::is_same<E, float>::value) {
        if (!options().force_generic && f32_problem_ok(pr[0]) && f32_problem_ok(pr[1]) && f32_problem_ok(pr[2])) {
            Span span(name, st);
            hipError_t e = launch_gemm_f32<true, true, EpiStore<E>, 3>(F32Batch<EpiStore<E>, 3>{{pr[0], pr[1], pr[2]}, {epi[0], epi[1], epi[2]}},
                                                                       false, device_cu_count(), st);
            if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
            return MOC_OK;
        }
    }
    for (int i = 0; i < 3; ++i) {
        moc_status s = run_gemm<E, true, true>(names[i], pr[i], epi[i], st, sk);
        if (s != MOC_OK) return s;
    }
    return MOC_OK;
}

// Two independent products of one shape (both operands k-contiguous; bf16: contraction a multiple of 32)
// with different epilogues in one launch when a matrix-core kernel takes them; otherwise one run_gemm each.
template <class E, class EpiA, class EpiB>
moc_status run_gemm_pair(const char* name, const char* name_a, const char* name_b, const GemmProblem<E>& pa, const EpiA& ea,
                         const GemmProblem<E>& pb, const EpiB& eb, hipStream_t st, const StreamKArea* sk = nullptr) {
    if constexpr (std::is_same<E, bf16_t>::value) {
        const bool same = pa.M == pb.M && pa.N == pb.N && pa.Kc == pb.Kc && pa.Kc % kMfmaBK == 0 && pa.Kc2 == 0 && pb.Kc2 == 0;
        if (same && !options().force_generic && mfma_problem_ok(pa) && mfma_problem_ok(pb)) {
            constexpr bool kGateUp = std::is_same<EpiA, EpiStore<float>>::value && std::is_same<EpiB, EpiStore<bf16_t>>::value;
            const bool pp = kGateUp && pp_takes(pa, ea) && pp_takes(pb, eb) && pa.A.ld == pb.A.ld && pa.B.ld == pb.B.ld &&
                            !(sk && sk->part && options().gemm_streamk);
            const PairRoute pair = pair_route(pa.M, pa.N, pa.Kc, pp, std::max(1, device_cu_count()), forced_tile());
            const GemmRoute route = pair.route;
            if constexpr (kGateUp) {
                if (pair.together && route.pp) {
                    Span span(name, st);
                    PpWork<2> w;
                    w.pr[0] = pa; w.out[0] = pp_out(ea);
                    w.pr[1] = pb; w.out[1] = pp_out(eb);
                    w.nprob = 2;
                    const hipError_t e = launch_pp_group<false, false, 2, 2>(route.tile, w, st);
                    if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                    return MOC_OK;
                }
            }
            const int best = route.tile;
            if (pair.together && !route.pp) {
                Span span(name, st);
                const hipError_t e = with_tile<kTilesAll>(best, [&](auto c) {
                    constexpr GemmTile t = kGemmTile[decltype(c)::value];
                    return launch_gemm_bf16_mfma_pair<t.bm, t.bn, false, false, 0, EpiA, EpiB, 4, t.sets>(pa, ea, pb, eb, st);
                });
                if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                return MOC_OK;
            }
        }
    }
    if constexpr (std::is_same<E, float>::value && std::is_same<EpiA, EpiB>::value) {
        if (!options().force_generic && f32_problem_ok(pa) && f32_problem_ok(pb)) {
            Span span(name, st);
            hipError_t e = launch_gemm_f32<false, false, EpiA, 2>(F32Batch<EpiA, 2>{{pa, pb}, {ea, eb}}, true, device_cu_count(), st);
            if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
            return MOC_OK;
        }
    }
    moc_status s = run_gemm<E, false, false>(name_a, pa, ea, st, sk, true);
    if (s != MOC_OK) return s;
    return run_gemm<E, false, false>(name_b, pb, eb, st, sk);
}

// Up to NB products that differ only in their row counts (and, for weight gradients, in their
// contraction lengths) in one launch: one per expert of an MoE layer.  Problems with M = 0 are
// skipped.  Falls back to one run_gemm per problem when the MFMA kernel cannot take all of them (`one_sum` see launch_gemm_f32).
template <class E, bool AKM, bool BKM, class Epi, int NB>
moc_status run_gemm_grouped(const char* name, int nprob, const GemmProblem<E>* pr, const Epi* epi, hipStream_t st, bool one_sum = false) {
    if constexpr (std::is_same<E, bf16_t>::value) {
        bool ok = !options().force_generic && nprob <= NB;
        bool tail = false, padded = true;
        int64_t total_m = 0;
        int rows[NB], k[NB], k2[NB];
        for (int z = 0; z < nprob && ok; ++z) {
            rows[z] = pr[z].M; k[z] = pr[z].Kc; k2[z] = pr[z].Kc2;
            if (pr[z].M == 0) continue;
            ok = mfma_problem_ok(pr[z]) && pr[z].N == pr[0].N && (pr[z].Kc2 == 0) == (pr[0].Kc2 == 0);
            tail = tail || gemm_has_tail(pr[z]);
            padded = padded && gemm_padded(pr[z]);
            total_m += pr[z].M;
        }
        if (ok && total_m > 0 && !(BKM && tail && !padded)) {
            const int cus = std::max(1, device_cu_count());
            constexpr unsigned kMask = BKM ? kTilesKmGroup : kTilesGroup;
            double cost = 0.0;
            const GemmRoute route = grouped_route(kMask, nprob, rows, pr[0].N, k, k2, pp_group_takes(nprob, pr, epi), cus, forced_tile(), &cost);
            if (route.pp) {
                Span span(name, st);
                PpWork<NB> w;
                int order[NB];
                for (int z = 0; z < nprob; ++z) order[z] = z;
                std::stable_sort(order, order + nprob, [&](int a, int b) { return pr[a].Kc + pr[a].Kc2 > pr[b].Kc + pr[b].Kc2; });
                for (int z = 0; z < nprob; ++z) { w.pr[z] = pr[order[z]]; w.out[z] = pp_out(epi[order[z]]); }
                w.nprob = nprob;
                const hipError_t e = launch_pp_group<AKM, BKM, std::is_same<Epi, EpiStore<float>>::value ? 1 : 0, NB>(route.tile, w, st);
                if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
                return MOC_OK;
            }
            const int best = route.tile;
            MfmaGroup<Epi, NB> g;
            for (int z = 0; z < nprob; ++z) { g.pr[z] = pr[z]; g.epi[z] = epi[z]; }
            Span span(name, st);
            hipError_t e;
            if constexpr (BKM) {
                // (the padded mode also serves contractions without a tail: one set of kernels)
                e = with_tile<kMask>(best, [&](auto c) {
                    constexpr GemmTile t = kGemmTile[decltype(c)::value];
                    return launch_gemm_bf16_mfma_group<t.bm, t.bn, AKM, BKM, 2, Epi, NB, 4, t.sets>(g, nprob, st);
                });
            } else {
                e = tail ? with_tile<kTilesBasic>(grouped_route(kTilesBasic, nprob, rows, pr[0].N, k, k2, false, cus, forced_tile(), &cost).tile, [&](auto c) {
                               constexpr GemmTile t = kGemmTile[decltype(c)::value];
                               return launch_gemm_bf16_mfma_group<t.bm, t.bn, AKM, BKM, 1, Epi, NB, 4, t.sets>(g, nprob, st);
                           })
                         : with_tile<kMask>(best, [&](auto c) {
                               constexpr GemmTile t = kGemmTile[decltype(c)::value];
                               return launch_gemm_bf16_mfma_group<t.bm, t.bn, AKM, BKM, 0, Epi, NB, 4, t.sets>(g, nprob, st);
                           });
            }
            if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
            return MOC_OK;
        }
    }
    for (int z = 0; z < nprob; ++z) {
        if (pr[z].M == 0) continue;
        moc_status s = run_gemm<E, AKM, BKM>(name, pr[z], epi[z], st, nullptr, one_sum);
        if (s != MOC_OK) return s;
    }
    return MOC_OK;
}

// The gate (fp32 result) and up projection of all experts in one launch on large tiles, an expert's two products next to each other
// because they share its rows of x; fills `done` unless the kernel does not take them or single launches are cheaper.
template <int NB>
moc_status run_gate_up_grouped(const char* name, int nprob, const MfmaProblem* gate, const EpiStore<float>* eg, const MfmaProblem* up,
                               const EpiStore<bf16_t>* eu, hipStream_t st, bool* done) {
    *done = false;
    bool ok = nprob <= NB && pp_group_takes(nprob, gate, eg) && pp_group_takes(nprob, up, eu) && gate[0].A.ld == up[0].A.ld && gate[0].B.ld == up[0].B.ld;
    int64_t rows = 0;
    int m[NB];
    for (int z = 0; z < nprob && ok; ++z) {
        m[z] = gate[z].M;
        ok = ok && gate[z].M == up[z].M && gate[z].N == up[z].N && gate[z].Kc == gate[0].Kc && up[z].Kc == gate[0].Kc && gate[z].Kc2 == 0 && up[z].Kc2 == 0;
        rows += gate[z].M;
    }
    if (!ok || rows == 0) return MOC_OK;
    const int t = grouped_pair_tile(nprob, m, gate[0].N, gate[0].Kc, std::max(1, device_cu_count()), forced_tile());
    if (t < 0) return MOC_OK;
    Span span(name, st);
    PpWork<2 * NB> w;
    for (int z = 0; z < nprob; ++z) {
        w.pr[2 * z] = gate[z]; w.out[2 * z] = pp_out(eg[z]);
        w.pr[2 * z + 1] = up[z]; w.out[2 * z + 1] = pp_out(eu[z]);
    }
    w.nprob = 2 * nprob;
    const hipError_t e = launch_pp_group<false, false, 2, 2 * NB>(t, w, st);
    if (e != hipSuccess) return fail(MOC_ERR_HIP, "%s launch: %s", name, hipGetErrorString(e));
    *done = true;
    return MOC_OK;
}

// LDS-resident Top-K: any row length up to the LDS capacity, any alignment.
template <class E, int NT, int VEC, bool FUSED>
moc_status run_topk_lds(const char* name, const TopkArgs<E>& a, int T, hipStream_t st) {
    const size_t lds = topk_lds_bytes(a.F, NT, VEC);
    if (lds > 160 * 1024 - 64) return fail(MOC_ERR_UNSUPPORTED, "F = %d needs %zu bytes of LDS for Top-K", a.F, lds);
    auto kern = topk_rows_lds_kernel<E, NT, VEC, FUSED>;
    LdsAttr<topk_rows_lds_kernel<E, NT, VEC, FUSED>, kMaxDynLds>::use();
    Span span(name, st);
    hipLaunchKernelGGL(kern, dim3(T), dim3(NT), lds, st, a);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

constexpr size_t kTopkRegDynMax = 96 * 1024;     // slot lists + dense row of the register-resident kernel

template <class E, int NT, int NCH, bool FUSED>
moc_status launch_topk_reg(const char* name, const TopkArgs<E>& a, int T, hipStream_t st) {
    const size_t dyn = topk_reg_dyn_lds(a.K, FUSED ? a.ldz : 0, sizeof(E), FUSED);
    auto kern = topk_rows_kernel<E, NT, NCH, FUSED>;
    LdsAttr<topk_rows_kernel<E, NT, NCH, FUSED>, (int)kTopkRegDynMax>::use();
    Span span(name, st);
    TopkArgs<E> args = a;
    args.far = cut_far(a.F, a.K);
    hipLaunchKernelGGL(kern, dim3(T), dim3(NT), dyn, st, args);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

// Row Top-K with NT threads per row.  Rows that are 16-byte aligned and short enough stay in
// registers; everything else goes through the LDS-resident kernel.
template <class E, int NT, bool FUSED>
moc_status run_topk(const char* name, const TopkArgs<E>& a, int T, hipStream_t st) {
    if (a.K == a.F) {
        Span span(name, st);
        const unsigned parts = (unsigned)(((FUSED ? a.ldz : a.F) + kAllSpan - 1) / kAllSpan);
        hipLaunchKernelGGL((select_all_kernel<E, FUSED>), dim3(T, parts), dim3(256), 0, st, a);
        HIP_TRY(hipGetLastError());
        return MOC_OK;
    }
    const bool aligned = a.ldg % 4 == 0 && aligned16(a.g);
    const int cover = FUSED ? (int)std::max<int64_t>(a.F, a.ldz) : a.F;
    const int nch = (cover + NT * 4 - 1) / (NT * 4);
    // very large K (slot lists beyond the LDS budget of the register kernel) goes to the LDS-resident kernel
    const bool lists_fit = topk_reg_dyn_lds(a.K, FUSED ? a.ldz : 0, sizeof(E), FUSED) <= kTopkRegDynMax;
    if (aligned && lists_fit) {
        if (nch <= 1) return launch_topk_reg<E, NT, 1, FUSED>(name, a, T, st);
        if (nch <= 2) return launch_topk_reg<E, NT, 2, FUSED>(name, a, T, st);
        if (nch <= 3) return launch_topk_reg<E, NT, 3, FUSED>(name, a, T, st);
        if constexpr (NT < 1024) {
            if (nch <= 4) return launch_topk_reg<E, NT, 4, FUSED>(name, a, T, st);
            if (nch <= 6) return launch_topk_reg<E, NT, 6, FUSED>(name, a, T, st);
            if (nch <= 8) return launch_topk_reg<E, NT, 8, FUSED>(name, a, T, st);
            if constexpr (NT == 256)
                if (nch <= 11) return launch_topk_reg<E, NT, 11, FUSED>(name, a, T, st);
        }
        return run_topk_lds<E, NT, 4, FUSED>(name, a, T, st);
    }
    if (aligned) return run_topk_lds<E, NT, 4, FUSED>(name, a, T, st);
    if (FUSED) return fail(MOC_ERR_BAD_ARG, "%s: unaligned workspace", name);
    return run_topk_lds<E, NT, 1, FUSED>(name, a, T, st);
}

// Grouped Top-K of MoC_{a:b}: one thread per group of gb channels.
template <class E, bool FUSED>
moc_status run_group_select(const char* name, const TopkArgs<E>& a, int T, int ga, int gb, hipStream_t st) {
    const int vec_ok = a.ldg % 4 == 0 && aligned16(a.g);
    if (FUSED && (!vec_ok || a.ldz % 64 != 0 || a.ldu % 64 != 0)) return fail(MOC_ERR_BAD_ARG, "%s: unaligned workspace", name);
    const int64_t groups = (int64_t)T * ((FUSED ? a.ldz : (int64_t)a.F) / gb);
    const unsigned grid = (unsigned)((groups + 255) / 256);
    Span span(name, st);
    if (gb == 4) hipLaunchKernelGGL((group_select_kernel<E, 4, FUSED>), dim3(grid), dim3(256), 0, st, a, T, ga, vec_ok);
    else if (gb == 8) hipLaunchKernelGGL((group_select_kernel<E, 8, FUSED>), dim3(grid), dim3(256), 0, st, a, T, ga, vec_ok);
    else hipLaunchKernelGGL((group_select_kernel<E, 16, FUSED>), dim3(grid), dim3(256), 0, st, a, T, ga, vec_ok);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

// keys = SiLU(g) or |SiLU(g)| over n contiguous fp32 values (Top-K position variants)
inline moc_status launch_key_transform(const float* g, float* keys, int64_t n, int key_mode, hipStream_t st) {
    Span span("topk_key_transform", st);
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 16384));
    hipLaunchKernelGGL(topk_key_transform_kernel, dim3(grid), dim3(256), 0, st, g, keys, n, key_mode);
    HIP_TRY(hipGetLastError());
    return MOC_OK;
}

// D = Z' W_down (Eq. MoC-2 / FFN-2): Z' is [T, ldF] with zeros past F, W_down [F, d] is read k-major.
template <class E>
moc_status down_projection(const Dims& D, const E* Zd, const E* wd, E* y, hipStream_t st, const ShareScratch& scratch = ShareScratch{}) {
    GemmProblem<E> pr{kc_operand<E>(Zd, D.ldF), km_operand<E>(wd, D.d, D.d), D.T, D.d, D.F, 0, true};
    return run_gemm<E, false, true>("gemm_down", pr, EpiStore<E>{y, D.d, D.d, 0}, st, nullptr, false, scratch);
}

}  // namespace mocapi
