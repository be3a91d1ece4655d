// pd_direct.hpp -- direct evaluation of the horizon sums in 3D (internal).
//
// For the short horizons of the paper's runs the correlations of a chain,
//   conv_O(x) = sum_J sum_o K_OJ(o) g_J(x + o),
// cost less as sums over the horizon ball than as transforms: the x passes
// and the (y, z) pass move ~260 B per node and step through HBM (256^3 FP32
// LPS), the sums read each field once (plus tile halos from the caches) and
// need ~300 multiply-adds and adds per node, because the octant symmetry of
// the kernels (C_ij = c(r) o_i o_j, a_i = w(r) o_i: even or odd along every
// axis) folds the eight points (+-a, +-b, +-c) into one product.
//
// A block takes a tile of TX x TY columns and a chunk of planes and sweeps
// the input planes upwards.  Each plane of the NI input fields goes through
// LDS (double-buffered, one barrier per plane; the next plane's loads are in
// flight meanwhile) with MT halo nodes around the tile.  A thread owns NX
// consecutive nodes along x: it reads the rows y + b and y - b of a field
// with NX-wide LDS loads, folds them along y (sum and difference, shared by
// its NX nodes), folds along x per node, and adds each folded value times the
// kernel value of (a, b, c) to the plane sums q_c of every output that takes
// it.  The plane sums then go to the outputs at z - c and z + c, which a
// thread keeps in 2 MT + 1 accumulators per output and node that shift by
// one per plane (the shift is the destination register of the add); the
// accumulator that has received its last plane goes to the epilogue.
//
// Measured against the x transforms and the (y, z) pass (10 Verlet steps of
// the 256^3 LPS block in FP32 9.38 -> 7.65 ms, of a 201 x 150 x 97 block in
// FP64 3.89 -> 3.26 ms; FP64 force of the 128^3 cube 262 -> 176 us; four
// spacings, 150 x 125 x 100 in FP32, 364 -> 158 us).
//
// The kernel values are block-uniform: with one spacing along all axes they
// depend on r^2 and the product of the offsets only, so that a horizon of
// three spacings needs 8 + 8 + 12 distinct numbers, which stay in scalar
// registers (kernel arguments) for the whole sweep.
#pragma once

#include "pd_plan.hpp"

namespace pdd {

using namespace pdk;

// ------------------------------------------------------------ compile-time loops
template <int I0, int I1, class F>
__device__ __forceinline__ void each(F&& f) {
    if constexpr (I0 < I1) {
        f(std::integral_constant<int, I0>{});
        each<I0 + 1, I1>(f);
    }
}
// Ends a row of the straight-line code of a horizon: pinned sums are complete
// here, and later LDS reads stay behind.  Left to itself the compiler orders
// the whole horizon sum by sum and keeps every row's values in registers.
template <class T>
__device__ __forceinline__ void pin(T& x) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x)::"memory");
#endif
}
template <class T, int N>
__device__ __forceinline__ void pin(T (&x)[N]) {
#pragma unroll
    for (int n = 0; n < N; ++n) pin(x[n]);
}
__device__ __forceinline__ void row_fence() { __builtin_amdgcn_sched_barrier(0); }
__host__ __device__ constexpr int iabs(int a) { return a < 0 ? -a : a; }
// largest a >= 0 with a^2 <= n, or -1
__host__ __device__ constexpr int isqrt(int n) {
    int a = -1;
    while ((a + 1) * (a + 1) <= n) ++a;
    return a;
}

// ------------------------------------------------------------ kernel values
// Numbering of the distinct kernel values inside the ball of radius MT:
// C values by (r^2, o_i o_j) with o_i, o_j >= 1, and a values by (r^2, o_i).
__host__ __device__ constexpr bool c_exists(int MT, int r2, int pr) {
    for (int a = 1; a <= MT; ++a)
        for (int b = 0; b <= MT; ++b)
            for (int c = 0; c <= MT; ++c)
                if (a * a + b * b + c * c == r2 && r2 <= MT * MT && (a * a == pr || (b > 0 && a * b == pr))) return true;
    return false;
}
__host__ __device__ constexpr bool a_exists(int MT, int r2, int a) {
    for (int b = 0; b <= MT; ++b)
        for (int c = 0; c <= MT; ++c)
            if (a * a + b * b + c * c == r2 && r2 <= MT * MT) return true;
    return false;
}
template <int MT>
struct TapIds {
    int c[MT * MT + 1][MT * MT + 1], a[MT * MT + 1][MT + 1];   // -1: no such value
    int nc, na;
};
template <int MT>
constexpr TapIds<MT> tap_ids() {
    TapIds<MT> t{};
    for (int q = 0; q <= MT * MT; ++q) {
        for (int s = 0; s <= MT * MT; ++s) t.c[q][s] = (s > 0 && c_exists(MT, q, s)) ? t.nc++ : -1;
        for (int s = 0; s <= MT; ++s) t.a[q][s] = (s > 0 && a_exists(MT, q, s)) ? t.na++ : -1;
    }
    return t;
}
template <int MT>
constexpr TapIds<MT> kTapIds = tap_ids<MT>();
template <class T, int MT>
struct Taps {
    T c[kTapIds<MT>.nc];   // c(r) o_i o_j dV
    T a[kTapIds<MT>.na];   // w(r) o_i dV (times k_a in the force stage)
};

// ------------------------------------------------------------ operators
// A term (O, J): which coordinates multiply the radial function (i, and j for
// a C term), -1 for none.
struct Term {
    int i, j;   // i < 0: no such term; j < 0: an a value w(r) o_i
};
// dilatation sum: S = sum_J a_J (*) u_J
struct OpA {
    static constexpr int NI = 3, NO = 1;
    __host__ __device__ static constexpr Term term(int, int J) { return Term{J, -1}; }
};
// LPS force sums: conv_O = sum_J C_OJ (*) u_J + k_a a_O (*) theta
struct OpB {
    static constexpr int NI = 4, NO = 3;
    __host__ __device__ static constexpr Term term(int O, int J) { return J < 3 ? Term{O, J} : Term{O, -1}; }
};
// bond-based: conv_O = sum_J C_OJ (*) u_J
struct OpC {
    static constexpr int NI = 3, NO = 3;
    __host__ __device__ static constexpr Term term(int O, int J) { return Term{O, J}; }
};
// parity of a term along axis d, and its value at the octant point (a, b, c)
__host__ __device__ constexpr int t_par(Term t, int d) { return ((t.i == d) + (t.j == d)) & 1; }
__host__ __device__ constexpr int t_coord(int d, int a, int b, int c) { return d == 0 ? a : (d == 1 ? b : c); }
__host__ __device__ constexpr bool t_nonzero(Term t, int MT, int a, int b, int c) {
    if (t.i < 0 || a * a + b * b + c * c > MT * MT || a + b + c == 0) return false;
    if (t_coord(t.i, a, b, c) == 0) return false;
    return t.j < 0 || t_coord(t.j, a, b, c) != 0;
}
// whether output O takes any term of z-parity pz at plane offset c
template <class Op>
__host__ __device__ constexpr bool takes(int MT, int O, int pz, int c) {
    for (int J = 0; J < Op::NI; ++J) {
        const Term t = Op::term(O, J);
        if (t.i < 0 || t_par(t, 2) != pz) continue;
        for (int a = 0; a <= MT; ++a)
            for (int b = 0; b <= MT; ++b)
                if (t_nonzero(t, MT, a, b, c)) return true;
    }
    return false;
}
// whether input J has a nonzero term with x/y parities (px, py) at (a, b)
template <class Op>
__host__ __device__ constexpr bool uses(int MT, int J, int px, int py, int a, int b) {
    for (int O = 0; O < Op::NO; ++O) {
        const Term t = Op::term(O, J);
        if (t.i < 0 || t_par(t, 0) != px || t_par(t, 1) != py) continue;
        for (int c = 0; c <= MT; ++c)
            if (t_nonzero(t, MT, a, b, c)) return true;
    }
    return false;
}

// ------------------------------------------------------------ NX-wide accesses
// NX consecutive values of a field, aligned to one element (global accesses
// of this width need no more on gfx950).
template <class T, int NX>
struct Vec {
    typedef T U __attribute__((ext_vector_type(NX), aligned(sizeof(T))));   // element-aligned
    typedef T A __attribute__((ext_vector_type(NX), aligned(NX * sizeof(T))));
};
// values of p at nodes base + off .. + NX - 1, of which the first n exist
template <int NX, class T>
__device__ __forceinline__ void ldn(const T* p, long base, uint32_t off, int n, T (&out)[NX]) {
    auto b = uniform_base(p + base) + off * (uint32_t)sizeof(T);
    if (n >= NX) {
        const typename Vec<T, NX>::U w = *reinterpret_cast<const __attribute__((address_space(1))) typename Vec<T, NX>::U*>(b);
#pragma unroll
        for (int q = 0; q < NX; ++q) out[q] = w[q];
    } else {
#pragma unroll
        for (int q = 0; q < NX; ++q)
            out[q] = q < n ? reinterpret_cast<const __attribute__((address_space(1))) T*>(b)[q] : T(0);
    }
}
template <int NX, class T>
__device__ __forceinline__ void stn(T* p, long base, uint32_t off, int n, const T (&val)[NX]) {
    auto b = uniform_base(p + base) + off * (uint32_t)sizeof(T);
    if (n >= NX) {
        typename Vec<T, NX>::U w;
#pragma unroll
        for (int q = 0; q < NX; ++q) w[q] = val[q];
        *reinterpret_cast<__attribute__((address_space(1))) typename Vec<T, NX>::U*>(b) = w;
    } else {
#pragma unroll
        for (int q = 0; q < NX; ++q)
            if (q < n) reinterpret_cast<__attribute__((address_space(1))) T*>(b)[q] = val[q];
    }
}

// ------------------------------------------------------------ epilogues
// Dilatation: theta = 3 chi / m (S - g_i u_i), 0 off the body or where m = 0.
template <class T>
struct EpTheta {
    static constexpr int NOUT = 1, NRED = 0;
    NodeCtx<T> c;
    const T* u;
    T* theta;
    __host__ double nbytes() const { return 4.0 * sizeof(T) + 4.0 * sizeof(T) * c.edge_frac + 1.0; }
    template <int NX>
    struct Ld { T u[3][NX]; uint8_t cb[NX]; };
    template <int NX>
    __device__ __forceinline__ void load(long base, uint32_t off, int n, Ld<NX>& Q) const {
        ldn<NX>(c.chiB, base, off, n, Q.cb);
#pragma unroll
        for (int d = 0; d < 3; ++d) ldn<NX>(u + d * c.nb, base, off, n, Q.u[d]);
    }
    template <int NX>
    __device__ __forceinline__ void fin(long base, uint32_t off, int n, const Ld<NX>& Q, const T (&val)[1][NX],
                                        double*) const {
        T out[NX];
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            T st[4] = {c.sint[6], c.sint[7], c.sint[8], c.sint[9]};
            if (q < n) c.template st_range<6, 4>(Nd{base, off + q}, Q.cb[q], st);
            T acc = val[0][q];
#pragma unroll
            for (int d = 0; d < 3; ++d) acc -= st[d] * Q.u[d][q];
            const bool on = Q.cb[q] && st[3] != T(0);
            out[q] = on ? T(3) / (on ? st[3] : T(1)) * acc : T(0);
        }
        stn<NX>(theta, base, off, n, out);
    }
};

// Force: L_i = chi (conv_i [+ k_a theta g_i] - G_ij u_j), then by mode
// (kernel-uniform)
//   NR = 0, mode 0   L
//   NR = 0 / 4, mode 1   Verlet: F' = L + b, v <- chi_O [v + c1 (F + F')]
//       (NR = 4: with energy sums).  vh_in: v holds the half-step velocity
//       v + c1 F and F is not read; vh_out: v receives v' + c1 F' and F is
//       not written, and u_next (another buffer than u, which other blocks
//       still read) receives the next positions chi_O (u + dt vh') + (1 -
//       chi_O) w.
//   NR = 1, mode 2   -chi_O L and the partial sum of u . (-chi_O L)
//   NR = 1, mode 3   r = chi_O (L + b) and the partial sum of |r|^2
template <class T, bool LPS, int NR>
struct EpForce {
    static constexpr int NOUT = 3, NRED = NR;
    NodeCtx<T> c;
    int mode;
    T ka;
    const T* u; const T* theta;
    T* L; T* v; T* F; const T* b; const T* w;
    T c1, rho, dt;
    T* u_next;
    double* nanflag;
    int vh_in, vh_out;
    __host__ double nbytes() const {
        const double t = sizeof(T);
        double r = 3 * t + 1 + 6 * t * c.edge_frac + (LPS ? t + 3 * t * c.edge_frac : 0.0) + (b ? 3 * t : 0.0);
        if (mode == 1) return r + 3 * t * (2 + (vh_in ? 0 : 1) + 1 + (vh_out && w ? 1 : 0));
        return r + 3 * t;
    }
    template <int NX>
    struct Ld { T u[3][NX], th[NX], x[NR == 1 ? 1 : 3][NX], y[3][NX]; uint8_t cb[NX]; };
    template <int NX>
    __device__ __forceinline__ void load(long base, uint32_t off, int n, Ld<NX>& Q) const {
        ldn<NX>(c.chiB, base, off, n, Q.cb);
#pragma unroll
        for (int d = 0; d < 3; ++d) ldn<NX>(u + d * c.nb, base, off, n, Q.u[d]);
        if constexpr (LPS) ldn<NX>(theta, base, off, n, Q.th);
        if constexpr (NR != 1) {
            if (mode == 1) {
#pragma unroll
                for (int d = 0; d < 3; ++d) ldn<NX>(v + d * c.nb, base, off, n, Q.x[d]);
                if (!vh_in) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) ldn<NX>(F + d * c.nb, base, off, n, Q.y[d]);
                }
            }
        } else {
            if (mode == 3) {
#pragma unroll
                for (int d = 0; d < 3; ++d) ldn<NX>(b + d * c.nb, base, off, n, Q.y[d]);
            }
        }
    }
    template <int NX>
    __device__ __forceinline__ void fin(long base, uint32_t off, int n, const Ld<NX>& Q, const T (&val)[3][NX],
                                        double* red) const {
        T La[3][NX];
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            constexpr int NS = LPS ? 9 : 6;
            T st[NS];
#pragma unroll
            for (int k = 0; k < NS; ++k) st[k] = c.sint[k];
            if (q < n) c.template st_range<0, NS>(Nd{base, off + q}, Q.cb[q], st);
            const T chi = Q.cb[q] ? T(1) : T(0);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T acc = val[a][q];
#pragma unroll
                for (int j = 0; j < 3; ++j) acc -= st[symi(3, a, j)] * Q.u[j][q];
                if constexpr (LPS) acc += ka * Q.th[q] * st[6 + a];
                La[a][q] = chi * acc;
            }
        }
        if constexpr (NR == 1) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T out[NX];
#pragma unroll
                for (int q = 0; q < NX; ++q) {
                    const bool o = omega_bit(Q.cb[q], a) && q < n;
                    if (mode == 2) {
                        out[q] = o ? -La[a][q] : T(0);
                        red[0] += o ? double(Q.u[a][q]) * double(out[q]) : 0.0;
                    } else {
                        out[q] = o ? La[a][q] + Q.y[a][q] : T(0);
                        red[0] += double(out[q]) * double(out[q]);
                    }
                }
                stn<NX>(L + a * c.nb, base, off, n, out);
            }
        } else {
            if (mode == 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) stn<NX>(L + a * c.nb, base, off, n, La[a]);
                return;
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T bk[NX], vo[NX], fo[NX];
                if (b) ldn<NX>(b + a * c.nb, base, off, n, bk);
                else {
#pragma unroll
                    for (int q = 0; q < NX; ++q) bk[q] = T(0);
                }
#pragma unroll
                for (int q = 0; q < NX; ++q) {
                    const bool o = omega_bit(Q.cb[q], a);
                    const T Fn = La[a][q] + bk[q];
                    const T Fo = vh_in ? T(0) : Q.y[a][q];
                    const T vf = Q.x[a][q] + c1 * (Fo + Fn);
                    const T vn = o ? vf : T(0);
                    if (q < n) flag_nonfinite(nanflag, Fn, vn);
                    fo[q] = Fn;
                    vo[q] = vh_out ? (o ? vn + c1 * Fn : T(0)) : vn;
                    if constexpr (NR == 4) {
                        if (q < n) {
                            red[0] += 0.5 * double(rho) * double(vn) * double(vn);
                            red[1] += -0.5 * double(Q.u[a][q]) * double(La[a][q]);
                            red[2] += -double(bk[q]) * double(Q.u[a][q]);
                            red[3] += o ? double(Fn) * double(Fn) : 0.0;
                        }
                    }
                }
                stn<NX>(v + a * c.nb, base, off, n, vo);
                if (!vh_out) stn<NX>(F + a * c.nb, base, off, n, fo);
                else {
                    T wk[NX];
                    if (w) ldn<NX>(w + a * c.nb, base, off, n, wk);
#pragma unroll
                    for (int q = 0; q < NX; ++q)
                        wk[q] = omega_bit(Q.cb[q], a) ? Q.u[a][q] + dt * vo[q] : (w ? wk[q] : T(0));
                    stn<NX>(u_next + a * c.nb, base, off, n, wk);
                }
            }
        }
    }
};

// ------------------------------------------------------------ the sweep
struct D3Geo {
    int b1, b2, b3;
    int ntx, nty, nzc, zc;   // tiles along x and y, chunks of zc planes along z
};

template <class T>
struct D3In {
    const T* f[4];           // input fields (each one component)
    const uint8_t* chiB;     // node flags: inputs are multiplied by chi_B
};

// FP32 and FP64 tiles: TX columns along x, TY along y, NX nodes per thread.
template <class T, class Op, class Ep, int MT, int TX, int TY, int NX>
__global__ void __launch_bounds__((TX / NX) * TY) __attribute__((amdgpu_waves_per_eu(2)))
k_dir3(D3Geo g, D3In<T> in, Taps<T, MT> tp, Ep ep, double* __restrict__ partials) {
    using VA = typename Vec<T, NX>::A;
    constexpr int NI = Op::NI, NO = Op::NO, NT = (TX / NX) * TY;
    constexpr int H = (MT + NX - 1) / NX * NX;       // halo columns kept (aligned)
    constexpr int W = TX + 2 * H, HY = TY + 2 * MT;  // LDS row and rows of a plane
    constexpr int FX = TX + 2 * MT;                  // columns that are filled
    constexpr int NE = (FX * HY + NT - 1) / NT;      // nodes a thread fills
    extern __shared__ __align__(16) unsigned char smem_raw[];
    lds_ptr<T> lds = as_lds(reinterpret_cast<T*>(smem_raw));

    // consecutive blocks of a z-chunk on one XCD (the hardware deals blocks to
    // the 8 XCDs in turn), so that the tiles sharing halos share an L2
    const unsigned nblk = gridDim.x, bq = nblk >> 3, br = nblk & 7;
    const unsigned xcd = blockIdx.x & 7, bk = blockIdx.x >> 3;
    const unsigned lin = xcd < br ? xcd * (bq + 1) + bk : br * (bq + 1) + (xcd - br) * bq + bk;
    const int tx0 = (int)(lin % g.ntx) * TX, ty0 = (int)(lin / g.ntx % g.nty) * TY;
    const int z0 = (int)(lin / (g.ntx * g.nty)) * g.zc, z1 = min(g.b3, z0 + g.zc);
    const long pl = (long)g.b1 * g.b2;

    const int tid = threadIdx.x, tx = tid % (TX / NX), ty = tid / (TX / NX);
    const int x = tx0 + tx * NX, y = ty0 + ty;
    const int nx = y < g.b2 ? min(max(g.b1 - x, 0), NX) : 0;   // nodes of this thread in the body box
    const uint32_t off = nx > 0 ? (uint32_t)(y * g.b1 + x) : 0u;

    // this thread's share of the plane fill
    uint32_t go[NE];
    int lo[NE];
    uint32_t okm = 0;
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = tid + NT * i, r = e / FX, cx = e - r * FX;
        const int gx = tx0 - MT + cx, gy = ty0 - MT + r;
        const bool in_tile = e < FX * HY;
        const bool ok = in_tile && gx >= 0 && gx < g.b1 && gy >= 0 && gy < g.b2;
        go[i] = ok ? (uint32_t)(gy * g.b1 + gx) : 0u;
        lo[i] = in_tile ? r * W + cx + (H - MT) : -1;
        okm |= ok ? 1u << i : 0u;
    }
    T pre[NI][NE];
    uint8_t pcb[NE];
    auto fetch = [&](int z) {
        const long base = (long)min(max(z, 0), g.b3 - 1) * pl;
#pragma unroll
        for (int i = 0; i < NE; ++i) pcb[i] = ldf(in.chiB, Nd{base, go[i]});
#pragma unroll
        for (int J = 0; J < NI; ++J)
#pragma unroll
            for (int i = 0; i < NE; ++i) pre[J][i] = ldf(in.f[J], Nd{base, go[i]});
    };

    T acc[2 * MT][NO][NX];   // outputs at planes zi - MT .. zi + MT - 1 on entry of a plane
#pragma unroll
    for (int p = 0; p < 2 * MT; ++p)
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int n = 0; n < NX; ++n) acc[p][o][n] = T(0);
    double red[Ep::NRED > 0 ? Ep::NRED : 1];
#pragma unroll
    for (int r = 0; r < (Ep::NRED > 0 ? Ep::NRED : 1); ++r) red[r] = 0.0;

    // planes outside the body hold zeros: the sweep starts and ends inside
    const int zb = max(z0 - MT, 0), ze = z1 + MT;
    fetch(zb);
    for (int zi = zb; zi < ze; ++zi) {
        const bool act = zi < g.b3;   // block-uniform
        lds_ptr<T> buf = lds + ((zi & 1) ? NI * HY * W : 0);
        if (act) {
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                if (lo[i] >= 0) {
                    const bool ok = (okm >> i) & 1u;
                    const T chi = pcb[i] ? T(1) : T(0);
#pragma unroll
                    for (int J = 0; J < NI; ++J) buf[J * HY * W + lo[i]] = ok ? chi * pre[J][i] : T(0);
                }
            }
        }
        __syncthreads();
        if (zi + 1 < min(ze, g.b3)) fetch(zi + 1);
        // the finished plane's node fields, in flight during the arithmetic
        const int zo = zi - MT;
        const bool outp = zo >= z0;   // block-uniform (zo < z1 by the sweep)
        const long ob = (long)max(zo, 0) * pl;
        typename Ep::template Ld<NX> ld;
        if (outp) ep.template load<NX>(ob, off, nx, ld);

        // plane sums: a0 (offset 0, into the accumulator of plane zi), qe and
        // qo (offsets 1 .. MT, even and odd along z)
        T a0[NO][NX], qe[MT + 1][NO][NX], qo[MT + 1][NO][NX];
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int n = 0; n < NX; ++n) {
                a0[o][n] = acc[MT][o][n];
#pragma unroll
                for (int c = 1; c <= MT; ++c) qe[c][o][n] = qo[c][o][n] = T(0);
            }
        if (act) {
            each<0, NI>([&](auto Jc) {
                constexpr int J = decltype(Jc)::value;
                lds_ptr<T> fld = buf + J * HY * W + (ty + MT) * W + tx * NX;
                each<0, MT + 1>([&](auto bc) {
                    constexpr int b = decltype(bc)::value, R = isqrt(MT * MT - b * b);
                    constexpr int RA = (R + NX - 1) / NX * NX, WN = NX + 2 * RA;
                    each<0, NO>([&](auto Oc) {
                        constexpr int O = decltype(Oc)::value;
                        constexpr Term t = Op::term(O, J);
                        if constexpr (t.i >= 0) {
                            if constexpr (t_par(t, 2) == 0) pin(a0[O]);
                            each<1, MT + 1>([&](auto cc) {
                                constexpr int c = decltype(cc)::value;
                                if constexpr (t_par(t, 2) == 0 && takes<Op>(MT, O, 0, c)) pin(qe[c][O]);
                                if constexpr (t_par(t, 2) == 1 && takes<Op>(MT, O, 1, c)) pin(qo[c][O]);
                            });
                        }
                    });
                    row_fence();
                    // rows y + b and y - b around the thread's nodes: columns
                    // -RA .. NX - 1 + RA
                    T up[WN], dn[WN], E[WN], D[WN];
#pragma unroll
                    for (int k = 0; k < WN / NX; ++k) {
                        const VA a = *(lds_ptr<VA>)(fld + b * W + (H - RA) + k * NX);
#pragma unroll
                        for (int n = 0; n < NX; ++n) up[k * NX + n] = a[n];
                        if constexpr (b > 0) {
                            const VA d = *(lds_ptr<VA>)(fld - b * W + (H - RA) + k * NX);
#pragma unroll
                            for (int n = 0; n < NX; ++n) dn[k * NX + n] = d[n];
                        }
                    }
#pragma unroll
                    for (int k = 0; k < WN; ++k) {
                        if constexpr (b > 0) {
                            E[k] = up[k] + dn[k];
                            D[k] = up[k] - dn[k];
                        } else {
                            E[k] = up[k];
                            D[k] = T(0);
                        }
                    }
                    each<0, R + 1>([&](auto ac) {
                        constexpr int a = decltype(ac)::value;
                        each<0, 4>([&](auto pc) {
                            constexpr int px = decltype(pc)::value & 1, py = decltype(pc)::value >> 1;
                            if constexpr (uses<Op>(MT, J, px, py, a, b)) {
#pragma unroll
                                for (int n = 0; n < NX; ++n) {
                                    const T p = py ? D[RA + n + a] : E[RA + n + a];
                                    const T m = py ? D[RA + n - a] : E[RA + n - a];
                                    const T f = a == 0 ? p : (px ? p - m : p + m);
                                    each<0, NO>([&](auto Oc) {
                                        constexpr int O = decltype(Oc)::value;
                                        constexpr Term t = Op::term(O, J);
                                        if constexpr (t.i >= 0 && t_par(t, 0) == px && t_par(t, 1) == py) {
                                            each<0, MT + 1>([&](auto cc) {
                                                constexpr int c = decltype(cc)::value;
                                                if constexpr (t_nonzero(t, MT, a, b, c)) {
                                                    constexpr int r2 = a * a + b * b + c * c;
                                                    constexpr int oi = t_coord(t.i, a, b, c);
                                                    constexpr int oj = t_coord(t.j < 0 ? 0 : t.j, a, b, c);
                                                    constexpr int id = t.j >= 0 ? kTapIds<MT>.c[r2][oi * oj]
                                                                                : kTapIds<MT>.a[r2][oi];
                                                    T k;
                                                    if constexpr (t.j >= 0) k = tp.c[id];
                                                    else k = tp.a[id];
                                                    if constexpr (c == 0) a0[O][n] += k * f;
                                                    else if constexpr (t_par(t, 2) == 0) qe[c][O][n] += k * f;
                                                    else qo[c][O][n] += k * f;
                                                }
                                            });
                                        }
                                    });
                                }
                            }
                        });
                    });
                });
            });
        }
        // add the plane sums and shift by one plane
        T out[NO][NX];
        each<0, 2 * MT + 1>([&](auto pc) {
            constexpr int p = decltype(pc)::value, c = iabs(p - MT);
            each<0, NO>([&](auto Oc) {
                constexpr int O = decltype(Oc)::value;
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    T s;
                    if constexpr (p == MT) s = a0[O][n];
                    else if constexpr (p < 2 * MT) s = acc[p][O][n];
                    else s = T(0);
                    if constexpr (c > 0) {
                        if constexpr (takes<Op>(MT, O, 0, c)) s += qe[c][O][n];
                        if constexpr (takes<Op>(MT, O, 1, c)) s = p < MT ? s + qo[c][O][n] : s - qo[c][O][n];
                    }
                    if constexpr (p == 0) out[O][n] = s;
                    else acc[p - 1][O][n] = s;
                }
            });
        });
        if (outp && nx > 0) ep.template fin<NX>(ob, off, nx, ld, out, red);
    }
    if constexpr (Ep::NRED > 0) {
        __syncthreads();
        double* sm = reinterpret_cast<double*>(smem_raw);
        block_reduce_store<Ep::NRED>(red, partials + (long)blockIdx.x * Ep::NRED, sm);
    }
}

// Tile of a block and nodes per thread: 32 x 16 columns, two nodes per
// thread.
constexpr int kTX3 = 32, kTY3 = 16, kRes3 = 2;
template <class T, class Op, int MT>
struct Shape3 {
    static constexpr int TX = kTX3, TY = kTY3, NX = 2, NT = TX / NX * TY;
    static constexpr size_t lds() {
        return sizeof(T) * 2 * Op::NI * (TY + 2 * MT) * (TX + 2 * ((MT + NX - 1) / NX * NX));
    }
};

// ------------------------------------------------------------ position update
template <class T, int D>
__global__ void __launch_bounds__(256) k_drift(long n, const uint8_t* __restrict__ chiB, const T* u, T* u_out,
                                               const T* __restrict__ v, const T* __restrict__ F, const T* w, T dt,
                                               T c2, const uint8_t* lam, uint8_t* lam_out, const T* __restrict__ W,
                                               T Wc, int fail) {
    for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const uint8_t cb = chiB[i];
        T x[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const long k = i + d * n;
            const T xn = u[k] + dt * v[k] + c2 * F[k];
            x[d] = omega_bit(cb, d) ? xn : (w ? w[k] : T(0));
        }
#pragma unroll
        for (int d = 0; d < D; ++d) u_out[i + d * n] = x[d];
        if (lam) {
            const uint8_t l = lam[i];
            lam_out[i] = fail ? (uint8_t)((l != 0 && W[i] <= Wc) ? 1 : 0) : l;
        }
    }
}

}  // namespace pdd
