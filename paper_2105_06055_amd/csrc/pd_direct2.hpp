// pd_direct2.hpp -- direct bond sums per node (internal): the 2D bond-based
// plate (force, energy density, Verlet, adjoint, damage count) and the
// nonlinear bond-based model in 2D and 3D.
//
// Where the bond weights change per node (integrity, micromodulus scale), or
// the bond force is not linear, nothing folds; a node sums its bonds one by
// one in terms of the differences eta = u(x + o) - u(x):
//   s = phi(x + o) c(r) (o . eta),   L += s o,   W += s (o . eta) / 2.
// A block loads a tile of nodes and its halo of M nodes once into LDS; each
// thread takes NX consecutive nodes and reads each row of the horizon disc as
// a window of NX + 2R values.  Offsets and the order of the bonds are
// compile-time constants, the radial factors are kernel arguments in scalar
// registers.  A plate of 400,000 nodes (48 bonds) stays in the caches, so one
// launch per step replaces four passes over padded spectra.  On such plates
// all blocks are resident at once and a block's latency (load, rows of LDS
// reads and sums in turn, store) bounds the launch: ~9 instructions a bond
// issue at 0.48 per CU and cycle (1000 x 400, four spacings, 13 us), LDS reads
// fill 22 % of the cycles.  Measured against the transform passes: 20 FP32
// fracture steps of the 1000 x 400 plate 1458 -> 275 us, 20 FP64 steps of a 601
// x 241 plate at six spacings 3910 -> 357 us, 10 steps forward and backward on
// the 512 x 512 plate 3250 -> 728 us, the force of a 64 x 64 plate 22.5 -> 9.3
// us.
#pragma once

#include "pd_direct.hpp"

namespace pdd {

struct D2Geo {
    int b1, b2;
    long nb;
};
template <class T, int M>
struct Radial {
    T k[M * M + 1];
};

// nodal weight phi = chi_B [lam] [s]
template <class T>
struct Weight {
    const uint8_t* chiB;
    const uint8_t* lam;
    const T* s;
    __device__ __forceinline__ T at(uint32_t i) const {
        bool on = chiB[i] != 0;
        if (lam) on = on && lam[i] != 0;
        T ph = on ? T(1) : T(0);
        if (s) ph *= s[i];
        return ph;
    }
};

template <class T, int N>
struct Node {
    T v[N];
};

// Tile of TX x TY nodes, NX per thread; rows of W values, HY rows.
template <class T, int M, int TX_, int TY_, int NX_>
struct Tile2 {
    static constexpr int TX = TX_, TY = TY_, NX = NX_, NT = TX / NX * TY;
    static constexpr int H = (M + NX - 1) / NX * NX, W = TX + 2 * H, HY = TY + 2 * M, FX = TX + 2 * M;
    static constexpr int PL = W * HY;
    // The tile with its halo: get(in, i) loads the values of box node i (0 and
    // unused where !in), put(slot, value) stores them; all loads of a thread
    // are issued before its first store.
    static constexpr int NE = (FX * HY + NT - 1) / NT;
    template <class G, class P>
    __device__ __forceinline__ static void fill(const D2Geo& g, int x0, int y0, G&& get, P&& put) {
        decltype(get(false, 0u)) v[NE];
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const int e = threadIdx.x + NT * k, r = e / FX, cx = e - r * FX, gx = x0 - M + cx, gy = y0 - M + r;
            const bool in = e < FX * HY && gx >= 0 && gx < g.b1 && gy >= 0 && gy < g.b2;
            v[k] = get(in, in ? (uint32_t)(gy * g.b1 + gx) : 0u);
        }
#pragma unroll
        for (int k = 0; k < NE; ++k) {
            const int e = threadIdx.x + NT * k, r = e / FX, cx = e - r * FX;
            if (e < FX * HY) put(r * W + cx + (H - M), v[k]);
        }
    }
    // row window: values at columns -RA .. NX - 1 + RA around the thread's
    // nodes (RA: R rounded up to NX)
    template <int R>
    __device__ __forceinline__ static void row(lds_ptr<T> p, T (&w)[NX + 2 * ((R + NX - 1) / NX * NX)]) {
        constexpr int RA = (R + NX - 1) / NX * NX;
#pragma unroll
        for (int k = 0; k < (NX + 2 * RA) / NX; ++k) {
            const typename Vec<T, NX>::A a = *(lds_ptr<typename Vec<T, NX>::A>)(p - RA + k * NX);
#pragma unroll
            for (int n = 0; n < NX; ++n) w[k * NX + n] = a[n];
        }
    }
};

// Type of the sums over the rows of a disc.  The sum along a row is short, the
// one over the rows runs through terms of b times a row's, which cancel between
// b and -b: in FP32 it made an unweighted force of eight spacings less accurate
// than the transforms (L2 error 7.1e-8 against 4.5e-8; in FP64 3.7e-8).  Two
// conversions and two FP64 adds a row.  The kernels with the energy density
// keep T: their error is below the weighted transforms' (4 spacings 5.9e-8
// against 8.9e-8).
template <class T, bool WIDE>
struct RowSum {
    using type = std::conditional_t<WIDE, double, T>;
};

// ------------------------------------------------------------ force, 2D
template <class T>
struct Args2 {
    int mode;
    Weight<T> wt;
    const T* u;
    T* L; T* Wo;
    T* v; T* F; const T* b; const T* w;
    T c1, c2, dt, rho;
    int vh_in, vh_out, next;
    T* u_next; uint8_t* lam_next;
    T Wc;
    int fail;
    double* nanflag;
};

// WE: with the energy density.  NR: reductions (0, 1: modes 2 and 3, 4: the
// energy sums of mode 1).  Modes as pdd::Eval.
template <class T, int M, class TL, bool WE, int NR>
__global__ void __launch_bounds__(TL::NT) k_dir2(D2Geo g, Radial<T, M> tp, Args2<T> A, double* __restrict__ partials) {
    constexpr int NX = TL::NX, W = TL::W, PL = TL::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];   // 3 PL values
    lds_ptr<T> s0 = as_lds(reinterpret_cast<T*>(smem_raw)), s1 = s0 + PL, sp = s0 + 2 * PL;
    const int x0 = blockIdx.x * TL::TX, y0 = blockIdx.y * TL::TY;
    TL::fill(
        g, x0, y0,
        [&](bool in, uint32_t i) {
            const T a = A.u[i], b = A.u[g.nb + i], ph = A.wt.at(i);
            return Node<T, 3>{{in ? a : T(0), in ? b : T(0), in ? ph : T(0)}};
        },
        [&](int slot, const Node<T, 3>& q) {
            s0[slot] = q.v[0];
            s1[slot] = q.v[1];
            sp[slot] = q.v[2];
        });
    const int tx = threadIdx.x % (TL::TX / NX), ty = threadIdx.x / (TL::TX / NX);
    const int x = x0 + tx * NX, y = y0 + ty;
    const int nx = y < g.b2 ? min(max(g.b1 - x, 0), NX) : 0;
    const uint32_t off = nx > 0 ? (uint32_t)(y * g.b1 + x) : 0u;
    // the node's other fields, in flight during the fill and the sums
    uint8_t cb[NX];
    T vv[2][NX], FF[2][NX], bb[2][NX];
    ldn<NX>(A.wt.chiB, 0, off, nx, cb);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        if (NR != 1 && A.mode == 1) {
            ldn<NX>(A.v + d * g.nb, 0, off, nx, vv[d]);
            if (!A.vh_in) ldn<NX>(A.F + d * g.nb, 0, off, nx, FF[d]);
        }
        if (A.b) ldn<NX>(A.b + d * g.nb, 0, off, nx, bb[d]);
        else {
#pragma unroll
            for (int n = 0; n < NX; ++n) bb[d][n] = T(0);
        }
    }
    __syncthreads();
    const int c = (ty + M) * W + tx * NX + TL::H;
    using TS = typename RowSum<T, !WE>::type;
    T u0[NX], u1[NX], ph[NX], en[NX];
    TS a0[NX], a1[NX];
#pragma unroll
    for (int n = 0; n < NX; ++n) {
        u0[n] = s0[c + n];
        u1[n] = s1[c + n];
        ph[n] = sp[c + n];
        a0[n] = a1[n] = TS(0);
        en[n] = T(0);
    }
    each<0, 2 * M + 1>([&](auto rc) {
        constexpr int b = decltype(rc)::value - M, R = isqrt(M * M - b * b), RA = (R + NX - 1) / NX * NX;
        pin(a0);
        pin(a1);
        if constexpr (WE) pin(en);
        row_fence();
        T w0[NX + 2 * RA], w1[NX + 2 * RA], wp[NX + 2 * RA];
        TL::template row<R>(s0 + c + b * W, w0);
        TL::template row<R>(s1 + c + b * W, w1);
        TL::template row<R>(sp + c + b * W, wp);
        // sums along the row (short chains round less; that of s enters L_y
        // times b)
        T rs[NX], ra[NX], re[NX];
#pragma unroll
        for (int n = 0; n < NX; ++n) rs[n] = ra[n] = re[n] = T(0);
        each<0, 2 * R + 1>([&](auto ac) {
            constexpr int a = decltype(ac)::value - R, r2 = a * a + b * b;
            if constexpr (r2 > 0) {
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    T e = T(0);
                    if constexpr (a != 0) e += T(a) * (w0[RA + n + a] - u0[n]);
                    if constexpr (b != 0) e += T(b) * (w1[RA + n + a] - u1[n]);
                    const T s = tp.k[r2] * wp[RA + n + a] * e;
                    if constexpr (a != 0) ra[n] += T(a) * s;
                    if constexpr (b != 0) rs[n] += s;
                    if constexpr (WE) re[n] += s * e;
                }
            }
        });
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            if constexpr (R > 0) a0[n] += TS(ra[n]);
            if constexpr (b != 0) a1[n] += TS(b) * TS(rs[n]);
            if constexpr (WE) en[n] += re[n];
        }
    });
    double red[NR > 0 ? NR : 1];
#pragma unroll
    for (int r = 0; r < (NR > 0 ? NR : 1); ++r) red[r] = 0.0;
    if (nx > 0) {
        T L[2][NX], Wn[NX];
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            L[0][n] = ph[n] * T(a0[n]);
            L[1][n] = ph[n] * T(a1[n]);
            Wn[n] = T(0.5) * ph[n] * en[n];
        }
        if constexpr (WE) {
            if (A.Wo) stn<NX>(A.Wo, 0, off, nx, Wn);
        }
        if constexpr (NR == 1) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                T out[NX];
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    const bool o = omega_bit(cb[n], d) && n < nx;
                    if (A.mode == 2) {
                        out[n] = o ? -L[d][n] : T(0);
                        red[0] += o ? double(d ? u1[n] : u0[n]) * double(out[n]) : 0.0;
                    } else {
                        out[n] = o ? L[d][n] + bb[d][n] : T(0);
                        red[0] += double(out[n]) * double(out[n]);
                    }
                }
                stn<NX>(A.L + d * g.nb, 0, off, nx, out);
            }
        } else if (A.mode == 0) {
            stn<NX>(A.L, 0, off, nx, L[0]);
            stn<NX>(A.L + g.nb, 0, off, nx, L[1]);
        } else {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                T vo[NX], fo[NX];
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    const bool o = omega_bit(cb[n], d);
                    const T Fn = L[d][n] + bb[d][n];
                    const T Fo = A.vh_in ? T(0) : FF[d][n];
                    const T vf = vv[d][n] + A.c1 * (Fo + Fn);
                    const T vn = o ? vf : T(0);
                    if (n < nx) flag_nonfinite(A.nanflag, Fn, vn);
                    fo[n] = Fn;
                    vo[n] = A.vh_out ? (o ? vn + A.c1 * Fn : T(0)) : vn;
                    if constexpr (NR == 4) {
                        if (n < nx) {
                            const double un = double(d ? u1[n] : u0[n]);
                            red[0] += 0.5 * double(A.rho) * double(vn) * double(vn);
                            red[1] += -0.5 * un * double(L[d][n]);
                            red[2] += -double(bb[d][n]) * un;
                            red[3] += o ? double(Fn) * double(Fn) : 0.0;
                        }
                    }
                }
                stn<NX>(A.v + d * g.nb, 0, off, nx, vo);
                if (!A.vh_out) stn<NX>(A.F + d * g.nb, 0, off, nx, fo);
                if (A.next) {
                    T wk[NX];
                    if (A.w) ldn<NX>(A.w + d * g.nb, 0, off, nx, wk);
#pragma unroll
                    for (int n = 0; n < NX; ++n) {
                        const T un = d ? u1[n] : u0[n];
                        const T x = A.vh_out ? mad(A.dt, vo[n], un) : position_update(un, A.dt, vo[n], A.c2, fo[n]);
                        wk[n] = omega_bit(cb[n], d) ? x : (A.w ? wk[n] : T(0));
                    }
                    stn<NX>(A.u_next + d * g.nb, 0, off, nx, wk);
                }
            }
            if (A.next && A.lam_next) {
                uint8_t ln[NX];
                ldn<NX>(A.wt.lam, 0, off, nx, ln);
                if constexpr (WE) {
                    if (A.fail) {
#pragma unroll
                        for (int n = 0; n < NX; ++n) ln[n] = (ln[n] != 0 && Wn[n] <= A.Wc) ? 1 : 0;
                    }
                }
                stn<NX>(A.lam_next, 0, off, nx, ln);
            }
        }
    }
    if constexpr (NR > 0) {
        __syncthreads();
        block_reduce_store<NR>(red, partials + ((long)blockIdx.y * gridDim.x + blockIdx.x) * NR,
                               reinterpret_cast<double*>(smem_raw));
    }
}

// ------------------------------------------------------------ adjoint, 2D
// u_bar = phi sum phi' c (o . gamma) o, gamma = g' - g;
// w_bar = -chi_B sum phi' c (o . eta)(o . gamma)  (the derivative of <g, L>
// with respect to the weight at this node, from its bonds as either end).
template <class T>
struct ArgsAdj {
    Weight<T> wt;
    const T* u; const T* u2;      // primal field u (+ u2)
    const T* g;                   // cotangent; masked by chi_Omega in stage 1
    T* ubar;
    T* wbar;
    T wscale;
    int acc;
    // reverse Verlet step: stage 0 a plain adjoint; stage 1: ut = chi_O (ub +
    // c1 L a), tmp = c1 L a + ut; stage 2: ub = tmp + c2 L ut, vb = a + dt ut,
    // bb += c2 ut + 2 c1 a with a = chi_O vb
    int stage;
    T* ub; T* vb; T* bb; T* ut; T* tmp;
    T c1, c2, dt;
};
template <class T, int M, class TL>
__global__ void __launch_bounds__(TL::NT) k_adj2(D2Geo g, Radial<T, M> tp, ArgsAdj<T> A) {
    constexpr int NX = TL::NX, W = TL::W, PL = TL::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];   // 5 PL values
    lds_ptr<T> s0 = as_lds(reinterpret_cast<T*>(smem_raw)), s1 = s0 + PL, q0 = s0 + 2 * PL, q1 = s0 + 3 * PL, sp = s0 + 4 * PL;
    const int x0 = blockIdx.x * TL::TX, y0 = blockIdx.y * TL::TY;
    TL::fill(
        g, x0, y0,
        [&](bool in, uint32_t i) {
        T a = T(0), b = T(0);
        if (A.wbar) {
            a = A.u[i];
            b = A.u[g.nb + i];
            if (A.u2) {
                a += A.u2[i];
                b += A.u2[g.nb + i];
            }
        }
        T ga = A.g[i], gb = A.g[g.nb + i];
        if (A.stage == 1) {
            const uint8_t cbi = A.wt.chiB[i];
            ga = omega_bit(cbi, 0) ? ga : T(0);
            gb = omega_bit(cbi, 1) ? gb : T(0);
        }
        const T ph = A.wt.at(i);
        return Node<T, 5>{{in ? a : T(0), in ? b : T(0), in ? ga : T(0), in ? gb : T(0), in ? ph : T(0)}};
        },
        [&](int slot, const Node<T, 5>& q) {
            s0[slot] = q.v[0];
            s1[slot] = q.v[1];
            q0[slot] = q.v[2];
            q1[slot] = q.v[3];
            sp[slot] = q.v[4];
        });
    __syncthreads();
    const int tx = threadIdx.x % (TL::TX / NX), ty = threadIdx.x / (TL::TX / NX);
    const int x = x0 + tx * NX, y = y0 + ty;
    const int nx = y < g.b2 ? min(max(g.b1 - x, 0), NX) : 0;
    const uint32_t off = nx > 0 ? (uint32_t)(y * g.b1 + x) : 0u;
    const int c = (ty + M) * W + tx * NX + TL::H;
    T u0[NX], u1[NX], g0[NX], g1[NX], a0[NX], a1[NX], pb[NX];
#pragma unroll
    for (int n = 0; n < NX; ++n) {
        u0[n] = s0[c + n]; u1[n] = s1[c + n];
        g0[n] = q0[c + n]; g1[n] = q1[c + n];
        a0[n] = a1[n] = pb[n] = T(0);
    }
    each<0, 2 * M + 1>([&](auto rc) {
        constexpr int b = decltype(rc)::value - M, R = isqrt(M * M - b * b), RA = (R + NX - 1) / NX * NX;
        pin(a0);
        pin(a1);
        pin(pb);
        row_fence();
        T w0[NX + 2 * RA], w1[NX + 2 * RA], h0[NX + 2 * RA], h1[NX + 2 * RA], wp[NX + 2 * RA];
        TL::template row<R>(s0 + c + b * W, w0);
        TL::template row<R>(s1 + c + b * W, w1);
        TL::template row<R>(q0 + c + b * W, h0);
        TL::template row<R>(q1 + c + b * W, h1);
        TL::template row<R>(sp + c + b * W, wp);
        T rs[NX], ra[NX], rp[NX];   // sums along the row
#pragma unroll
        for (int n = 0; n < NX; ++n) rs[n] = ra[n] = rp[n] = T(0);
        each<0, 2 * R + 1>([&](auto ac) {
            constexpr int a = decltype(ac)::value - R, r2 = a * a + b * b;
            if constexpr (r2 > 0) {
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    T e = T(0), f = T(0);
                    if constexpr (a != 0) {
                        e += T(a) * (w0[RA + n + a] - u0[n]);
                        f += T(a) * (h0[RA + n + a] - g0[n]);
                    }
                    if constexpr (b != 0) {
                        e += T(b) * (w1[RA + n + a] - u1[n]);
                        f += T(b) * (h1[RA + n + a] - g1[n]);
                    }
                    const T s = tp.k[r2] * wp[RA + n + a] * f;
                    if constexpr (a != 0) ra[n] += T(a) * s;
                    if constexpr (b != 0) rs[n] += s;
                    rp[n] += s * e;
                }
            }
        });
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            if constexpr (R > 0) a0[n] += ra[n];
            if constexpr (b != 0) a1[n] += T(b) * rs[n];
            pb[n] += rp[n];
        }
    });
    if (nx <= 0) return;
    uint8_t cb[NX];
    ldn<NX>(A.wt.chiB, 0, off, nx, cb);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        T Lg[NX];
#pragma unroll
        for (int n = 0; n < NX; ++n) Lg[n] = sp[c + n] * (d ? a1[n] : a0[n]);
        if (A.stage == 0) {
            if (A.ubar) stn<NX>(A.ubar + d * g.nb, 0, off, nx, Lg);
        } else if (A.stage == 1) {
            T ub[NX], ut[NX];
            ldn<NX>(A.ub + d * g.nb, 0, off, nx, ub);
#pragma unroll
            for (int n = 0; n < NX; ++n) {
                ut[n] = omega_bit(cb[n], d) ? ub[n] + A.c1 * Lg[n] : T(0);
                ub[n] = A.c1 * Lg[n] + ut[n];
            }
            stn<NX>(A.ut + d * g.nb, 0, off, nx, ut);
            stn<NX>(A.tmp + d * g.nb, 0, off, nx, ub);
        } else {
            T tp_[NX], vb[NX], bb[NX];
            ldn<NX>(A.tmp + d * g.nb, 0, off, nx, tp_);
            ldn<NX>(A.vb + d * g.nb, 0, off, nx, vb);
            if (A.bb) ldn<NX>(A.bb + d * g.nb, 0, off, nx, bb);
#pragma unroll
            for (int n = 0; n < NX; ++n) {
                const T a = omega_bit(cb[n], d) ? vb[n] : T(0), ut = d ? g1[n] : g0[n];
                tp_[n] += A.c2 * Lg[n];
                vb[n] = a + A.dt * ut;
                if (A.bb) bb[n] += A.c2 * ut + T(2) * A.c1 * a;
            }
            stn<NX>(A.ub + d * g.nb, 0, off, nx, tp_);
            stn<NX>(A.vb + d * g.nb, 0, off, nx, vb);
            if (A.bb) stn<NX>(A.bb + d * g.nb, 0, off, nx, bb);
        }
    }
    if (A.wbar) {
        T wb[NX];
        if (A.acc) ldn<NX>(A.wbar, 0, off, nx, wb);
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            const T add = cb[n] ? -A.wscale * pb[n] : T(0);
            wb[n] = A.acc ? wb[n] + add : add;
        }
        stn<NX>(A.wbar, 0, off, nx, wb);
    }
}

// ------------------------------------------------------------ damage count
// cnt = number of intact partners within the horizon, itself included,
// d = 1 - phi cnt / beta on the body.  A block takes 64 x 8 nodes; the state of
// a row of the tile and its halo is a ballot of its lanes, kept as bits in
// LDS, so that a row of the horizon disc is two words, a shift, a mask and a
// bit count, not a read per bond (196 bonds at eight spacings: 408 x 713 nodes
// in FP32 30.0 us with a read per bond; the bound is now the launch).
struct DiscRows {
    uint32_t mask[17];   // row b of the disc, b < 2 M + 1: bit a set where offset (a - M, b - M) is in it
};
template <class T>
__global__ void __launch_bounds__(256) k_damage2(D2Geo g, int M, DiscRows rows, NodeCtx<T> c, int beta_comp,
                                                 const uint8_t* __restrict__ lam, T* __restrict__ d) {
    constexpr int TY = 8, HR = TY + 16, NK = HR / 4;
    __shared__ uint32_t bits[HR][4];   // columns x0 - M .. x0 - M + 95
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, HY = TY + 2 * M;
    const int x0 = blockIdx.x * 64, y0 = blockIdx.y * TY, x = x0 + lane;
    uint8_t on[NK][2];
#pragma unroll
    for (int k = 0; k < NK; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = wave + 4 * k, gx = x - M + 64 * h, gy = y0 - M + r;
            const bool in = r < HY && (h == 0 || lane < 2 * M) && gx >= 0 && gx < g.b1 && gy >= 0 && gy < g.b2;
            on[k][h] = 0;
            if (in) {
                const uint32_t i = (uint32_t)(gy * g.b1 + gx);
                const uint8_t body = c.chiB[i], whole = lam[i];
                on[k][h] = (body != 0) & (whole != 0);
            }
        }
#pragma unroll
    for (int k = 0; k < NK; ++k) {
        const uint64_t m0 = __ballot(on[k][0]), m1 = __ballot(on[k][1]);
        if (lane == 0) {
            uint32_t* w = bits[wave + 4 * k];
            w[0] = (uint32_t)m0;
            w[1] = (uint32_t)(m0 >> 32);
            w[2] = (uint32_t)m1;
        }
    }
    __syncthreads();
    const int w = lane >> 5, sh = lane & 31;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int ty = wave + 4 * h, y = y0 + ty;
        if (x >= g.b1 || y >= g.b2) continue;
        auto window = [&](int r) {
            const uint64_t v = bits[r][w] | (uint64_t)bits[r][w + 1] << 32;
            return (uint32_t)(v >> sh);
        };
        int cnt = 0;
#pragma unroll
        for (int b = 0; b < 17; ++b) cnt += __popc(window(ty + b) & rows.mask[b]);   // (no bits beyond 2 M)
        const int phi = (window(ty + M) >> M) & 1;
        const uint32_t i = (uint32_t)(y * g.b1 + x);
        const uint8_t cb = c.chiB[i];
        const long beta = (long)rint(c.st(beta_comp, Nd{0, i}, cb)) + (cb ? 1 : 0);
        d[i] = cb ? T(1.0 - double((long)phi * cnt) / double(beta > 0 ? beta : 1)) : T(0);
    }
}

// ------------------------------------------------------------ nonlinear
// f = c (2 xi . eta + eta . eta)(xi + eta) / 2 per bond, xi = dx o.  dx comes
// rounded to T and the radial factors are c dx^2 over its square, so that the
// linear part of f, c dx^2 (o . eta) o, does not see the rounding; with the
// factors c the FP32 forces were off by the spacing's error twice (128^3 block:
// L2 error 1.2e-7, now 6e-8).
template <class T, int M, class TL>
__global__ void __launch_bounds__(TL::NT) k_nbb2(D2Geo g, Radial<T, M> tp, T dx, const uint8_t* __restrict__ chiB,
                                                 const T* __restrict__ u, T* __restrict__ L) {
    constexpr int NX = TL::NX, W = TL::W, PL = TL::PL;
    extern __shared__ __align__(16) unsigned char smem_raw[];   // 3 PL values
    lds_ptr<T> s0 = as_lds(reinterpret_cast<T*>(smem_raw)), s1 = s0 + PL, sp = s0 + 2 * PL;
    const int x0 = blockIdx.x * TL::TX, y0 = blockIdx.y * TL::TY;
    TL::fill(
        g, x0, y0,
        [&](bool in, uint32_t i) {
            const T a = u[i], b = u[g.nb + i], ph = chiB[i] ? T(1) : T(0);
            return Node<T, 3>{{in ? a : T(0), in ? b : T(0), in ? ph : T(0)}};
        },
        [&](int slot, const Node<T, 3>& q) {
            s0[slot] = q.v[0];
            s1[slot] = q.v[1];
            sp[slot] = q.v[2];
        });
    __syncthreads();
    const int tx = threadIdx.x % (TL::TX / NX), ty = threadIdx.x / (TL::TX / NX);
    const int x = x0 + tx * NX, y = y0 + ty;
    const int nx = y < g.b2 ? min(max(g.b1 - x, 0), NX) : 0;
    const uint32_t off = nx > 0 ? (uint32_t)(y * g.b1 + x) : 0u;
    const int c = (ty + M) * W + tx * NX + TL::H;
    const T dx2 = T(2) * dx;
    using TS = typename RowSum<T, true>::type;
    T u0[NX], u1[NX];
    TS o0[NX], o1[NX], e0[NX], e1[NX];
#pragma unroll
    for (int n = 0; n < NX; ++n) {
        u0[n] = s0[c + n]; u1[n] = s1[c + n];
        o0[n] = o1[n] = e0[n] = e1[n] = TS(0);
    }
    each<0, 2 * M + 1>([&](auto rc) {
        constexpr int b = decltype(rc)::value - M, R = isqrt(M * M - b * b), RA = (R + NX - 1) / NX * NX;
        pin(o0);
        pin(o1);
        pin(e0);
        pin(e1);
        row_fence();
        T w0[NX + 2 * RA], w1[NX + 2 * RA], wp[NX + 2 * RA];
        TL::template row<R>(s0 + c + b * W, w0);
        TL::template row<R>(s1 + c + b * W, w1);
        TL::template row<R>(sp + c + b * W, wp);
        T rs[NX], ra[NX], r0[NX], r1[NX];   // sums along the row
#pragma unroll
        for (int n = 0; n < NX; ++n) rs[n] = ra[n] = r0[n] = r1[n] = T(0);
        each<0, 2 * R + 1>([&](auto ac) {
            constexpr int a = decltype(ac)::value - R, r2 = a * a + b * b;
            if constexpr (r2 > 0) {
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    const T h0 = w0[RA + n + a] - u0[n], h1 = w1[RA + n + a] - u1[n];
                    const T e = T(a) * h0 + T(b) * h1;
                    const T s = tp.k[r2] * wp[RA + n + a] * (dx2 * e + h0 * h0 + h1 * h1);
                    if constexpr (a != 0) ra[n] += T(a) * s;
                    if constexpr (b != 0) rs[n] += s;
                    r0[n] += s * h0;
                    r1[n] += s * h1;
                }
            }
        });
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            if constexpr (R > 0) o0[n] += TS(ra[n]);
            if constexpr (b != 0) o1[n] += TS(b) * TS(rs[n]);
            e0[n] += TS(r0[n]);
            e1[n] += TS(r1[n]);
        }
    });
    if (nx <= 0) return;
    T out[2][NX];
#pragma unroll
    for (int n = 0; n < NX; ++n) {
        const T ph = T(0.5) * sp[c + n];
        out[0][n] = ph * T(TS(dx) * o0[n] + e0[n]);
        out[1][n] = ph * T(TS(dx) * o1[n] + e1[n]);
    }
    stn<NX>(L, 0, off, nx, out[0]);
    stn<NX>(L + g.nb, 0, off, nx, out[1]);
}

// 3D: a block takes 16 x 8 x 8 nodes, two per thread along x, with a halo of
// M nodes on every side in LDS (u and chi: 75 KB in FP32, 150 KB in FP64 at M
// = 3), which keeps eight waves on a CU in either type; the 4.6 halo loads
// per node are small beside the ~2000 vector instructions of 122 bonds.
// Measured on the 128^3 block: FP32 420 -> 97 us against the 13-field chain of
// the (y, z) pass, L2 error 6.2e-8 -> 6.0e-8 (sums by plane: short chains).
struct Tile3 {
    static constexpr int TX = 16, TY = 8, TZ = 8, NX = 2, NT = TX / NX * TY * TZ;
};
template <class T, int M>
__global__ void __launch_bounds__(Tile3::NT) k_nbb3(int b1, int b2, int b3, Radial<T, M> tp, T dx,
                                                    const uint8_t* __restrict__ chiB, const T* __restrict__ u,
                                                    T* __restrict__ L) {
    using TL = Tile3;
    using VA = typename Vec<T, TL::NX>::A;
    constexpr int NX = TL::NX, H = (M + NX - 1) / NX * NX, W = TL::TX + 2 * H, HY = TL::TY + 2 * M;
    constexpr int HZ = TL::TZ + 2 * M, FX = TL::TX + 2 * M, PL = W * HY, VOL = PL * HZ;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    lds_ptr<T> sm = as_lds(reinterpret_cast<T*>(smem_raw));
    const int x0 = blockIdx.x * TL::TX, y0 = blockIdx.y * TL::TY, z0 = blockIdx.z * TL::TZ;
    const long nb = (long)b1 * b2 * b3;
    constexpr int NE = (FX * HY * HZ + TL::NT - 1) / TL::NT;
    Node<T, 4> pre[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = threadIdx.x + TL::NT * k, cx = e % FX, t = e / FX, ry = t % HY, rz = t / HY;
        const int gx = x0 - M + cx, gy = y0 - M + ry, gz = z0 - M + rz;
        const bool in = rz < HZ && gx >= 0 && gx < b1 && gy >= 0 && gy < b2 && gz >= 0 && gz < b3;
        const long i = in ? ((long)gz * b2 + gy) * b1 + gx : 0;
        const T a0 = u[i], a1 = u[nb + i], a2 = u[2 * nb + i], ph = chiB[i] ? T(1) : T(0);
        pre[k] = Node<T, 4>{{in ? a0 : T(0), in ? a1 : T(0), in ? a2 : T(0), in ? ph : T(0)}};
    }
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int e = threadIdx.x + TL::NT * k, cx = e % FX, t = e / FX, ry = t % HY, rz = t / HY;
        const int slot = rz * PL + ry * W + cx + (H - M);
        if (rz < HZ) {
#pragma unroll
            for (int f = 0; f < 4; ++f) sm[f * VOL + slot] = pre[k].v[f];
        }
    }
    __syncthreads();
    // eight lanes cover a row of 16 nodes; the row bits are swapped so that
    // the two rows of a 16-lane group are two apart (rows of 24 values: half
    // the banks each)
    const int tx = threadIdx.x & 7, t8 = (threadIdx.x >> 3) & 7, tz = threadIdx.x >> 6;
    const int ty = ((t8 & 1) << 1) | ((t8 >> 1) & 1) | (t8 & 4);
    const int x = x0 + tx * NX, y = y0 + ty, z = z0 + tz;
    const int nx = (y < b2 && z < b3) ? min(max(b1 - x, 0), NX) : 0;
    const int c = (tz + M) * PL + (ty + M) * W + tx * NX + H;
    const T dx2 = T(2) * dx;
    T uc[3][NX], so[3][NX], se[3][NX];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            uc[d][n] = sm[d * VOL + c + n];
            so[d][n] = se[d][n] = T(0);
        }
    each<0, 2 * M + 1>([&](auto zc) {
        constexpr int cz = decltype(zc)::value - M;
        // sums over the plane (short chains round less)
        T zs[NX], ps[2][NX], pe[3][NX];
#pragma unroll
        for (int n = 0; n < NX; ++n) zs[n] = ps[0][n] = ps[1][n] = pe[0][n] = pe[1][n] = pe[2][n] = T(0);
        each<0, 2 * M + 1>([&](auto rc) {
            constexpr int b = decltype(rc)::value - M, R2 = M * M - b * b - cz * cz;
            if constexpr (R2 >= 0) {
                constexpr int R = isqrt(R2), RA = (R + NX - 1) / NX * NX, WN = NX + 2 * RA;
                pin(zs);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    if (d < 2) pin(ps[d]);
                    pin(pe[d]);
                }
                row_fence();
                T w[4][WN];
#pragma unroll
                for (int f = 0; f < 4; ++f)
#pragma unroll
                    for (int k = 0; k < WN / NX; ++k) {
                        const VA a = *(lds_ptr<VA>)(sm + f * VOL + c + cz * PL + b * W - RA + k * NX);
#pragma unroll
                        for (int n = 0; n < NX; ++n) w[f][k * NX + n] = a[n];
                    }
                T rs[NX];   // sum of s along the row
#pragma unroll
                for (int n = 0; n < NX; ++n) rs[n] = T(0);
                each<0, 2 * R + 1>([&](auto ac) {
                    constexpr int a = decltype(ac)::value - R, r2 = a * a + b * b + cz * cz;
                    if constexpr (r2 > 0) {
#pragma unroll
                        for (int n = 0; n < NX; ++n) {
                            T h[3];
#pragma unroll
                            for (int d = 0; d < 3; ++d) h[d] = w[d][RA + n + a] - uc[d][n];
                            T e = T(0);
                            if constexpr (a != 0) e += T(a) * h[0];
                            if constexpr (b != 0) e += T(b) * h[1];
                            if constexpr (cz != 0) e += T(cz) * h[2];
                            const T s = tp.k[r2] * w[3][RA + n + a] * (dx2 * e + h[0] * h[0] + h[1] * h[1] + h[2] * h[2]);
                            if constexpr (a != 0) ps[0][n] += T(a) * s;
                            rs[n] += s;
#pragma unroll
                            for (int d = 0; d < 3; ++d) pe[d][n] += s * h[d];
                        }
                    }
                });
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    if constexpr (b != 0) ps[1][n] += T(b) * rs[n];
                    zs[n] += rs[n];
                }
            }
        });
#pragma unroll
        for (int n = 0; n < NX; ++n) {
            so[0][n] += ps[0][n];
            so[1][n] += ps[1][n];
            if constexpr (cz != 0) so[2][n] += T(cz) * zs[n];
#pragma unroll
            for (int d = 0; d < 3; ++d) se[d][n] += pe[d][n];
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            pin(so[d]);
            pin(se[d]);
        }
    });
    if (nx <= 0) return;
    const uint32_t off = (uint32_t)(y * b1 + x);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T out[NX];
#pragma unroll
        for (int n = 0; n < NX; ++n) out[n] = T(0.5) * sm[3 * VOL + c + n] * (dx * so[d][n] + se[d][n]);
        stn<NX>(L + d * nb + (long)z * b1 * b2, 0, off, nx, out);
    }
}

}  // namespace pdd
