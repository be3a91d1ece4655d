// pd_direct.hip -- launches of the direct horizon sums (pd_direct.hpp,
// pd_direct2.hpp), compiled in parallel units: PD_INST_T = float or double,
// PD_DIR_PART = 0 .. 2 the 3D LPS kernels at radius 2 .. 4, 3 and 4 the 3D
// bond-based ones (radius 2 and 3 with the dispatch and the element-wise
// kernels; radius 4), 5 the 2D force, 6 the 2D adjoint and damage count, 7 the
// nonlinear model.
#include <algorithm>

#include "pd_direct2.hpp"
#include "pd_direct_api.hpp"

#ifndef PD_INST_T
#error "PD_INST_T must be defined (float or double)"
#endif
#ifndef PD_DIR_PART
#error "PD_DIR_PART must be defined (0 .. 7)"
#endif

namespace pdd {

using pdi::allow_lds;
using pdi::finish_reduction;
using pdi::ProfScope;

// ------------------------------------------------------------ 3D launches
// g0: the interior static value the epilogue takes from scalar registers.
template <class T, class Op, class Ep, int MT>
pd_status launch3(pd_plan p, const D3In<T>& in, double ka, T g0, const Ep& ep, const char* name, hipStream_t st) {
    using S3 = Shape3<T, Op, MT>;
    const Geo& g = p->geo;
    D3Args<T, Ep, MT> a{};
    a.in = in;
    a.partials = p->partials;
    a.g0 = g0;
    a.ep = ep;
    constexpr TapIds<MT> ids = kTapIds<MT>;
    for (int r2 = 1; r2 <= MT * MT; ++r2) {
        for (int pr = 1; pr <= MT * MT; ++pr)
            if (ids.c[r2][pr] >= 0) a.tp.c[ids.c[r2][pr]] = T(p->dir_c[r2] * pr);
        for (int k = 1; k <= MT; ++k)
            if (ids.a[r2][k] >= 0) a.tp.a[ids.a[r2][k]] = T(ka * p->dir_a[r2] * k);
    }
    auto go = [&](auto shape) -> pd_status {
        using S = decltype(shape);
        D3Geo& d = a.g;
        d.b1 = g.b1; d.b2 = g.b2; d.b3 = g.b3;
        d.ntx = (g.b1 + S::TX - 1) / S::TX;
        d.nty = (g.b2 + S::TY - 1) / S::TY;
        d.zc = p->dir_planes > 0 ? std::min(p->dir_planes, g.b3) : chunk3(g, MT, S::TX, S::TY, S3::RES, S3::LAT);
        d.nzc = (g.b3 + d.zc - 1) / d.zc;
        const long nblk = (long)d.ntx * d.nty * d.nzc;
        if (nblk > 0x7fffffffL) return PD_EUNSUPPORTED;
        if (Ep::NRED > 0 && nblk * Ep::NRED > p->partials_cap) return PD_EINVAL;
        constexpr size_t lds = S::template lds<T, Op, MT>();
        if (lds > (size_t)p->max_lds) return PD_EUNSUPPORTED;
        auto kern = k_dir3<T, Op, Ep, MT, S>;
        allow_lds(kern, lds);
        ProfScope ps(p, st);
        hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(S::NT), lds, st, a);
        if (p->prof) {
            char nm[32];
            std::snprintf(nm, sizeof nm, "%s_m%d", name, MT);
            ps.done(nm, ep.nbytes() * (double)g.nb);
        }
        if (pd_status s = pdh::check(hipGetLastError()); s != PD_OK) return s;
        if (Ep::NRED > 0) return finish_reduction(p, nblk, Ep::NRED, st);
        return PD_OK;
    };
    if constexpr (S3::PAIR) {
        // rows of an odd length: the last thread of a row has one node
        if (g.b1 % 2 != 0) return go(typename S3::template S<false>{});
    }
    return go(typename S3::template S<true>{});
}

template <class T, bool LPS, int MT, int KIND>
pd_status force3(pd_plan p, const Eval<T>& e, hipStream_t st) {
    EpForce<T, LPS, KIND> ep{};
    ep.c = pdi::ctx<T>(p);
    ep.mode = e.mode;
    ep.ka = T(p->ka);
    ep.u = e.u; ep.theta = e.theta;
    ep.L = e.L; ep.v = e.v; ep.F = e.F; ep.b = e.b; ep.w = e.w;
    ep.c1 = e.c1; ep.c2 = e.c2; ep.rho = e.rho; ep.dt = e.dt;
    ep.u_next = e.u_next;
    ep.nanflag = e.nanflag;
    ep.vh_in = e.vh_in; ep.vh_out = e.vh_out; ep.next = e.next;
    ep.has = (e.b ? 1 : 0) | (e.w ? 2 : 0);
    D3In<T> in{{e.u, e.u + p->nb, e.u + 2 * p->nb, e.theta}, p->chiB};
    const T g0 = ep.c.sint[0];   // G_xx = G_yy = G_zz; the odd sums vanish
    if constexpr (LPS) return launch3<T, OpB, EpForce<T, LPS, KIND>, MT>(p, in, p->ka, g0, ep, "dir3_lps", st);
    else return launch3<T, OpC, EpForce<T, LPS, KIND>, MT>(p, in, 0.0, g0, ep, "dir3_bb", st);
}
// Force sums at radius MT, and the dilatation; each compiled in one unit.
template <class T, bool LPS, int MT>
pd_status force3_at(pd_plan p, const Eval<T>& e, hipStream_t st) {
    if (e.mode >= 2) return force3<T, LPS, MT, SOLVER>(p, e, st);
    if (e.mode == 0) return force3<T, LPS, MT, FORCE>(p, e, st);
    if (e.energy) return force3<T, LPS, MT, ENERGY>(p, e, st);
    return e.vh_in && e.vh_out ? force3<T, LPS, MT, INNER>(p, e, st) : force3<T, LPS, MT, STEP>(p, e, st);
}
template <class T, int MT>
pd_status theta3_at(pd_plan p, const T* u, T* theta, hipStream_t st) {
    EpTheta<T> ep{};
    ep.c = pdi::ctx<T>(p);
    ep.u = u;
    ep.theta = theta;
    D3In<T> in{{u, u + p->nb, u + 2 * p->nb, nullptr}, p->chiB};
    const T g0 = T(3) / ep.c.sint[9];   // 3 / m
    return launch3<T, OpA, EpTheta<T>, MT>(p, in, 1.0, g0, ep, "dir3_theta", st);
}

using R = PD_INST_T;
#if PD_DIR_PART <= 2
template pd_status force3_at<R, true, PD_DIR_PART + 2>(pd_plan, const Eval<R>&, hipStream_t);
template pd_status theta3_at<R, PD_DIR_PART + 2>(pd_plan, const R*, R*, hipStream_t);
#elif PD_DIR_PART == 4
template pd_status force3_at<R, false, 4>(pd_plan, const Eval<R>&, hipStream_t);
#elif PD_DIR_PART == 3
extern template pd_status force3_at<R, true, 2>(pd_plan, const Eval<R>&, hipStream_t);
extern template pd_status force3_at<R, true, 3>(pd_plan, const Eval<R>&, hipStream_t);
extern template pd_status force3_at<R, true, 4>(pd_plan, const Eval<R>&, hipStream_t);
extern template pd_status force3_at<R, false, 4>(pd_plan, const Eval<R>&, hipStream_t);
extern template pd_status theta3_at<R, 2>(pd_plan, const R*, R*, hipStream_t);
extern template pd_status theta3_at<R, 3>(pd_plan, const R*, R*, hipStream_t);
extern template pd_status theta3_at<R, 4>(pd_plan, const R*, R*, hipStream_t);

template <class T>
pd_status dir3_theta(pd_plan p, const T* u, T* theta, hipStream_t st) {
    switch (p->dir_mt) {
        case 2: return theta3_at<T, 2>(p, u, theta, st);
        case 3: return theta3_at<T, 3>(p, u, theta, st);
        case 4: return theta3_at<T, 4>(p, u, theta, st);
        default: return PD_EUNSUPPORTED;
    }
}
template <class T>
pd_status dir3_force(pd_plan p, const Eval<T>& e, hipStream_t st) {
    const bool lps = p->kern.model == PD_LPS_LINEAR;
    switch (p->dir_mt) {
        case 2: return lps ? force3_at<T, true, 2>(p, e, st) : force3_at<T, false, 2>(p, e, st);
        case 3: return lps ? force3_at<T, true, 3>(p, e, st) : force3_at<T, false, 3>(p, e, st);
        case 4: return lps ? force3_at<T, true, 4>(p, e, st) : force3_at<T, false, 4>(p, e, st);
        default: return PD_EUNSUPPORTED;
    }
}
template pd_status dir3_theta<PD_INST_T>(pd_plan, const PD_INST_T*, PD_INST_T*, hipStream_t);
template pd_status dir3_force<PD_INST_T>(pd_plan, const Eval<PD_INST_T>&, hipStream_t);

template <class T>
pd_status dir_drift(pd_plan p, const T* u, T* u_out, const T* v, const T* F, const T* w, T dt, T c2,
                    const uint8_t* lam, uint8_t* lam_out, const T* W, T Wc, int fail, hipStream_t st) {
    ProfScope ps(p, st);
    const long n = p->nb;
    const unsigned nblk = (unsigned)std::max<long>(1, std::min<long>((n + 255) / 256, 8192L));
    auto go = [&](auto Dc) {
        hipLaunchKernelGGL((k_drift<T, decltype(Dc)::value>), dim3(nblk), dim3(256), 0, st, n, p->chiB, u, u_out, v, F,
                           w, dt, c2, lam, lam_out, W, Wc, fail);
    };
    if (p->dim == 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 3>{});
    if (p->prof)
        ps.done("drift", (double)n * (p->dim * sizeof(T) * (w ? 5.0 : 4.0) + 1.0 +
                                      (lam ? 2.0 + (fail ? sizeof(T) : 0) : 0.0)));
    return pdh::check(hipGetLastError());
}
template pd_status dir_drift<PD_INST_T>(pd_plan, const PD_INST_T*, PD_INST_T*, const PD_INST_T*, const PD_INST_T*,
                                        const PD_INST_T*, PD_INST_T, PD_INST_T, const uint8_t*, uint8_t*,
                                        const PD_INST_T*, PD_INST_T, int, hipStream_t);

#if PD_DIR_FIRST   // once: not per type
// Most blocks of a launch with a reduction: plate tiles of 32 x 8 nodes, or
// four rounds of seven resident blocks per CU and one more of tiles (chunk3).
void dir_launch_shape(pd_plan p) {
    const Geo& g = p->geo;
    const long tiles = (long)((g.b1 + 31) / 32) * ((g.b2 + 7) / 8);
    p->dir_blocks = p->dim == 2 ? tiles : std::max(4L * 256 * 7, tiles) + tiles;
}
#endif
#endif

// ------------------------------------------------------------ 2D launches
template <class T, int M>
Radial<T, M> radial(pd_plan p, double scale = 1.0) {
    Radial<T, M> r;
    for (int q = 0; q <= M * M; ++q) r.k[q] = T(p->dir_c[q] * scale);
    return r;
}
inline D2Geo geo2(pd_plan p) { return D2Geo{p->geo.b1, p->geo.b2, p->nb}; }
template <class TL>
dim3 grid2(pd_plan p) {
    return dim3((unsigned)((p->geo.b1 + TL::TX - 1) / TL::TX), (unsigned)((p->geo.b2 + TL::TY - 1) / TL::TY));
}
// The radii compiled for the plate kernels; f(integral_constant<M>).
template <class F>
pd_status by_radius2(pd_plan p, F&& f) {
    switch (p->dir_mt) {
        case 2: return f(std::integral_constant<int, 2>{});
        case 3: return f(std::integral_constant<int, 3>{});
        case 4: return f(std::integral_constant<int, 4>{});
        case 5: return f(std::integral_constant<int, 5>{});
        case 6: return f(std::integral_constant<int, 6>{});
        case 8: return f(std::integral_constant<int, 8>{});
        default: return PD_EUNSUPPORTED;
    }
}
// Tile of 32 x 8 nodes, one per thread, for every size: many short blocks.
// (Verlet step of a 64 x 64 plate, M = 3 in FP32: 4.2 us; 64 x 8 nodes with
// two per thread 5.3; 1000 x 400, M = 4: 10.4 and 10.9 us; 601 x 241, M = 6 in
// FP64: 14.3 and 15.3 us.  The pair reads fewer LDS words per node but halves
// the waves, and a plate has few.)
template <class T, int M> using Plate = Tile2<T, M, 32, 8, 1>;

#if PD_DIR_PART == 5
template <class T, int M, class TL, bool WE, int NR>
pd_status run2(pd_plan p, const Args2<T>& A, hipStream_t st) {
    const dim3 grid = grid2<TL>(p);
    const long nblk = (long)grid.x * grid.y;
    if (NR > 0 && nblk * NR > p->partials_cap) return PD_EINVAL;
    constexpr size_t lds = 3 * TL::PL * sizeof(T);
    if (lds > (size_t)p->max_lds) return PD_EUNSUPPORTED;
    auto kern = k_dir2<T, M, TL, WE, NR>;
    allow_lds(kern, lds);
    ProfScope ps(p, st);
    hipLaunchKernelGGL(kern, grid, dim3(TL::NT), lds, st, geo2(p), radial<T, M>(p), A, p->partials);
    if (p->prof) {
        char nm[32];
        std::snprintf(nm, sizeof nm, "dir2_m%d", M);
        const double t = sizeof(T);
        double by = 2 * t + 1 + (A.wt.lam ? 1 : 0) + (A.wt.s ? t : 0) + (A.Wo ? t : 0) + (A.b ? 2 * t : 0);
        if (A.mode == 1) by += 2 * t * (2 + (A.vh_in ? 0 : 1) + (A.vh_out ? 0 : 1) + A.next) + (A.next && A.lam_next ? 1 : 0);
        else by += 2 * t;
        ps.done(nm, by * (double)p->nb);
    }
    if (pd_status s = pdh::check(hipGetLastError()); s != PD_OK) return s;
    return NR > 0 ? finish_reduction(p, nblk, NR, st) : PD_OK;
}

template <class T>
pd_status dir2_force(pd_plan p, const Eval<T>& e, hipStream_t st) {
    Args2<T> A{};
    A.mode = e.mode;
    A.wt = Weight<T>{p->chiB, e.lam, e.s};
    A.u = e.u;
    A.L = e.L; A.Wo = e.W;
    A.v = e.v; A.F = e.F; A.b = e.b; A.w = e.w;
    A.c1 = e.c1; A.c2 = e.c2; A.dt = e.dt; A.rho = e.rho;
    A.vh_in = e.vh_in; A.vh_out = e.vh_out; A.next = e.next;
    A.u_next = e.u_next; A.lam_next = e.lam_next;
    A.Wc = e.Wc; A.fail = e.fail;
    A.nanflag = e.nanflag;
    return by_radius2(p, [&](auto mc) -> pd_status {
        constexpr int M = decltype(mc)::value;
        auto go = [&](auto we, auto nr) -> pd_status {
            constexpr bool WE = decltype(we)::value;
            constexpr int NR = decltype(nr)::value;
            return run2<T, M, Plate<T, M>, WE, NR>(p, A, st);
        };
        if (e.mode >= 2) return go(std::false_type{}, std::integral_constant<int, 1>{});
        if (e.energy && e.W) return go(std::true_type{}, std::integral_constant<int, 4>{});
        if (e.energy) return go(std::false_type{}, std::integral_constant<int, 4>{});
        if (e.W) return go(std::true_type{}, std::integral_constant<int, 0>{});
        return go(std::false_type{}, std::integral_constant<int, 0>{});
    });
}
template pd_status dir2_force<PD_INST_T>(pd_plan, const Eval<PD_INST_T>&, hipStream_t);
#elif PD_DIR_PART == 6
template <class T>
pd_status run_adj(pd_plan p, const ArgsAdj<T>& A, hipStream_t st) {
    return by_radius2(p, [&](auto mc) -> pd_status {
        constexpr int M = decltype(mc)::value;
        using TL = Plate<T, M>;
        constexpr size_t lds = 5 * TL::PL * sizeof(T);
        if (lds > (size_t)p->max_lds) return PD_EUNSUPPORTED;
        auto kern = k_adj2<T, M, TL>;
        allow_lds(kern, lds);
        ProfScope ps(p, st);
        hipLaunchKernelGGL(kern, grid2<TL>(p), dim3(TL::NT), lds, st, geo2(p), radial<T, M>(p), A);
        if (p->prof) {
            char nm[32];
            std::snprintf(nm, sizeof nm, "adj2_m%d", M);
            const double t = sizeof(T);
            double by = 2 * t + 1 + (A.wt.s ? t : 0) + (A.wbar ? 2 * t + (A.u2 ? 2 * t : 0) + (A.acc ? 2 : 1) * t : 0);
            by += A.stage == 0 ? (A.ubar ? 2 * t : 0) : (A.stage == 1 ? 6 * t : 8 * t + (A.bb ? 4 * t : 0));
            ps.done(nm, by * (double)p->nb);
        }
        return pdh::check(hipGetLastError());
    });
}

template <class T>
pd_status dir2_adjoint(pd_plan p, const T* u, const T* u2, const T* s, const T* g, T* ubar, T* wbar, T wscale,
                       int acc, hipStream_t st) {
    ArgsAdj<T> A{};
    A.wt = Weight<T>{p->chiB, nullptr, s};
    A.u = u; A.u2 = u2; A.g = g;
    A.ubar = ubar; A.wbar = wbar; A.wscale = wscale; A.acc = acc;
    return run_adj<T>(p, A, st);
}

template <class T>
pd_status dir2_verlet_adjoint(pd_plan p, const T* un, const T* unp1, const T* s, T* ub, T* vb, T* sb, T* bb, T c1,
                              T c2, T dt, T* ut, T* tmp, hipStream_t st) {
    ArgsAdj<T> A{};
    A.wt = Weight<T>{p->chiB, nullptr, p->kern.weight == PD_WEIGHT_SCALE ? s : nullptr};
    A.u = un; A.u2 = unp1; A.g = vb;
    A.wbar = sb; A.wscale = c1; A.acc = 1;
    A.stage = 1;
    A.ub = ub; A.vb = vb; A.bb = bb; A.ut = ut; A.tmp = tmp;
    A.c1 = c1; A.c2 = c2; A.dt = dt;
    if (pd_status r = run_adj<T>(p, A, st); r != PD_OK) return r;
    A.u2 = nullptr;
    A.g = ut;
    A.wscale = c2;
    A.stage = 2;
    return run_adj<T>(p, A, st);
}

template <class T>
pd_status dir2_damage(pd_plan p, const uint8_t* lam, T* d, hipStream_t st) {
    const int M = p->dir_mt;
    DiscRows rows{};
    for (int b = -M; b <= M; ++b)
        for (int a = -M; a <= M; ++a) {
            const int r2 = a * a + b * b;
            if (r2 == 0 || (r2 <= M * M && p->dir_c[r2] != 0.0)) rows.mask[b + M] |= 1u << (a + M);
        }
    ProfScope ps(p, st);
    hipLaunchKernelGGL((k_damage2<T>), dim3((unsigned)((p->geo.b1 + 63) / 64), (unsigned)((p->geo.b2 + 7) / 8)),
                       dim3(256), 0, st, geo2(p), M, rows, pdi::ctx<T>(p), p->beta_comp, lam, d);
    if (p->prof) ps.done("damage2", (double)p->nb * (2.0 + sizeof(T)));
    return pdh::check(hipGetLastError());
}
template pd_status dir2_adjoint<R>(pd_plan, const R*, const R*, const R*, const R*, R*, R*, R, int, hipStream_t);
template pd_status dir2_verlet_adjoint<R>(pd_plan, const R*, const R*, const R*, R*, R*, R*, R*, R, R, R, R*, R*,
                                          hipStream_t);
template pd_status dir2_damage<R>(pd_plan, const uint8_t*, R*, hipStream_t);
#elif PD_DIR_PART == 7
template <class T>
pd_status dir_nbb(pd_plan p, const T* u, T* L, hipStream_t st) {
    const Geo& g = p->geo;
    ProfScope ps(p, st);
    pd_status s = PD_EUNSUPPORTED;
    // c per bond, not per o_i o_j, for the spacing as the kernel holds it
    const double dxT = (double)T(p->dx[0]), inv = 1.0 / (dxT * dxT);
    if (p->dim == 2) {
        s = by_radius2(p, [&](auto mc) -> pd_status {
            constexpr int M = decltype(mc)::value;
            using TL = Plate<T, M>;
            constexpr size_t lds = 3 * TL::PL * sizeof(T);
            if (lds > (size_t)p->max_lds) return PD_EUNSUPPORTED;
            auto kern = k_nbb2<T, M, TL>;
            allow_lds(kern, lds);
            hipLaunchKernelGGL(kern, grid2<TL>(p), dim3(TL::NT), lds, st, geo2(p), radial<T, M>(p, inv), T(p->dx[0]),
                               p->chiB, u, L);
            return pdh::check(hipGetLastError());
        });
    } else {
        auto go = [&](auto mc) -> pd_status {
            constexpr int M = decltype(mc)::value;
            using TL = Tile3;
            constexpr size_t lds = sizeof(T) * 4 * (TL::TX + 2 * ((M + TL::NX - 1) / TL::NX * TL::NX)) *
                                   (TL::TY + 2 * M) * (TL::TZ + 2 * M);
            if (lds > (size_t)p->max_lds) return PD_EUNSUPPORTED;
            auto kern = k_nbb3<T, M>;
            allow_lds(kern, lds);
            dim3 grid((g.b1 + TL::TX - 1) / TL::TX, (g.b2 + TL::TY - 1) / TL::TY, (g.b3 + TL::TZ - 1) / TL::TZ);
            hipLaunchKernelGGL(kern, grid, dim3(TL::NT), lds, st, g.b1, g.b2, g.b3, radial<T, M>(p, inv), T(p->dx[0]),
                               p->chiB, u, L);
            return pdh::check(hipGetLastError());
        };
        if (p->dir_mt == 2) s = go(std::integral_constant<int, 2>{});
        else if (p->dir_mt == 3) s = go(std::integral_constant<int, 3>{});
    }
    if (p->prof) ps.done(p->dim == 2 ? "nbb2" : "nbb3", (double)p->nb * (2.0 * p->dim * sizeof(T) + 1.0));
    return s;
}
template pd_status dir_nbb<PD_INST_T>(pd_plan, const PD_INST_T*, PD_INST_T*, hipStream_t);
#endif

}  // namespace pdd
