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
// Whether (J, b, a) is the first of the sweep's order (inputs, then rows, then
// columns) whose term goes to the plane sum of output O, z-parity pz, offset
// c > 0: it starts the sum.
template <class Op>
__host__ __device__ constexpr bool starts(int MT, int O, int pz, int c, int J, int b, int a) {
    for (int j = 0; j <= J; ++j) {
        const Term t = Op::term(O, j);
        if (t.i < 0 || t_par(t, 2) != pz) continue;
        for (int bb = 0; bb <= MT; ++bb)
            for (int aa = 0; aa <= MT; ++aa) {
                if (j == J && (bb > b || (bb == b && aa >= a))) continue;
                if (t_nonzero(t, MT, aa, bb, c)) return false;
            }
    }
    return true;
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

// ------------------------------------------------------------ plane accesses
// A field's plane as a buffer: the base and the plane's size sit in scalar
// registers, an access takes one 32-bit offset per thread, and an offset
// beyond the plane (kOut) reads zero and writes nothing, which stands for the
// nodes outside the body box without a branch or a select.
constexpr uint32_t kOut = 0x40000000u;
template <class T>
struct Plane {
#if defined(__HIP_DEVICE_COMPILE__)
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Plane(const T* p, long base, long nodes)
        : r(__builtin_amdgcn_make_buffer_rsrc((void*)(p + base), 0, (int)(nodes * (long)sizeof(T)), 0x00020000)) {}
    __device__ __forceinline__ T ld(uint32_t off) const {
        if constexpr (sizeof(T) == 1) return T(__builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0));
        else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
        else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
    }
    __device__ __forceinline__ void st(uint32_t off, T v) const {
        if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 0);
    }
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    // NX values at byte offset off; with tail the values from n on do not
    // exist (rows that NX does not divide: block-uniform)
    template <int NX>
    __device__ __forceinline__ void ldv(uint32_t off, bool tail, int n, T (&out)[NX]) const {
        constexpr int B = NX * (int)sizeof(T);
        if constexpr (NX == 1) out[0] = ld(off);
        else if constexpr (sizeof(T) == 1) {
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = ld(q < n ? off + q : kOut);
        } else if (tail) {
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = ld(q < n ? off + q * (uint32_t)sizeof(T) : kOut);
        } else if constexpr (B == 8) {
            const auto w = __builtin_bit_cast(typename Vec<T, NX>::A, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = w[q];
        } else {
            static_assert(B == 16, "8 or 16 bytes per thread");
            const auto w = __builtin_bit_cast(typename Vec<T, NX>::A, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = w[q];
        }
    }
    template <int NX>
    __device__ __forceinline__ void stv(uint32_t off, bool tail, int n, const T (&val)[NX]) const {
        constexpr int B = NX * (int)sizeof(T);
        if (NX == 1) st(off, val[0]);
        else if (tail) {
#pragma unroll
            for (int q = 0; q < NX; ++q) st(q < n ? off + q * (uint32_t)sizeof(T) : kOut, val[q]);
        } else {
            typename Vec<T, NX>::A w;
#pragma unroll
            for (int q = 0; q < NX; ++q) w[q] = val[q];
            if constexpr (B == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, w), r, off, 0, 0);
            else if constexpr (B == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), r, off, 0, 0);
        }
    }
#else   // host pass: never runs
    __device__ Plane(const T*, long, long) {}
    __device__ T ld(uint32_t) const { return T(0); }
    template <int NX>
    __device__ void ldv(uint32_t, bool, int, T (&)[NX]) const {}
    template <int NX>
    __device__ void stv(uint32_t, bool, int, const T (&)[NX]) const {}
#endif
};

// Where a thread's nodes are: plane [base, base + pl) of the box, NX nodes
// from off on, of which n exist (n is 0 or NX unless tail).
struct At {
    long base, pl;
    uint32_t off;
    int n;
    bool tail;
    template <class T>
    __device__ __forceinline__ uint32_t at() const { return n > 0 ? off * (uint32_t)sizeof(T) : kOut; }
    template <int NX, class T>
    __device__ __forceinline__ void ld(const T* p, T (&out)[NX]) const {
        Plane<T>(p, base, pl).template ldv<NX>(at<T>(), tail, n, out);
    }
    template <int NX, class T>
    __device__ __forceinline__ void st(T* p, const T (&val)[NX]) const {
        Plane<T>(p, base, pl).template stv<NX>(at<T>(), tail, n, val);
    }
};
// Static fields Q0 .. Q0 + N - 1 of the NX nodes: the interior values (scalar
// registers) in a wave without edge nodes; else edge nodes load their own.
template <int Q0, int N, int NX, class T, class F>
__device__ __forceinline__ void with_static(const NodeCtx<T>& c, const At& a, const uint8_t (&cb)[NX], F&& f) {
    bool edge = false;
#pragma unroll
    for (int q = 0; q < NX; ++q) edge = edge || (q < a.n && !(cb[q] & 2));
    T st[NX][N];
#pragma unroll
    for (int q = 0; q < NX; ++q)
#pragma unroll
        for (int k = 0; k < N; ++k) st[q][k] = c.sint[Q0 + k];
    if (__ballot(edge) == 0) {
        f(st);
        return;
    }
#pragma unroll
    for (int q = 0; q < NX; ++q)
        if (q < a.n) c.template st_range<Q0, N>(Nd{a.base, a.off + q}, cb[q], st[q]);
    f(st);
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
    __device__ __forceinline__ void load(const At& a, Ld<NX>& Q) const {
        a.ld<NX>(c.chiB, Q.cb);
#pragma unroll
        for (int d = 0; d < 3; ++d) a.ld<NX>(u + d * c.nb, Q.u[d]);
    }
    template <int NX>
    __device__ __forceinline__ void fin(const At& a, const Ld<NX>& Q, const T (&val)[1][NX], double*) const {
        with_static<6, 4, NX>(c, a, Q.cb, [&](const T (&st)[NX][4]) {
            T out[NX];
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                T acc = val[0][q];
#pragma unroll
                for (int d = 0; d < 3; ++d) acc -= st[q][d] * Q.u[d][q];
                const T m = st[q][3];
                const bool on = Q.cb[q] && m != T(0);
                out[q] = on ? T(3) / (on ? m : T(1)) * acc : T(0);
            }
            a.st<NX>(theta, out);
        });
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
    __device__ __forceinline__ void load(const At& a, Ld<NX>& Q) const {
        a.ld<NX>(c.chiB, Q.cb);
#pragma unroll
        for (int d = 0; d < 3; ++d) a.ld<NX>(u + d * c.nb, Q.u[d]);
        if constexpr (LPS) a.ld<NX>(theta, Q.th);
        if constexpr (NR != 1) {
            if (mode == 1) {
#pragma unroll
                for (int d = 0; d < 3; ++d) a.ld<NX>(v + d * c.nb, Q.x[d]);
                if (!vh_in) {
#pragma unroll
                    for (int d = 0; d < 3; ++d) a.ld<NX>(F + d * c.nb, Q.y[d]);
                }
            }
        } else {
            if (mode == 3) {
#pragma unroll
                for (int d = 0; d < 3; ++d) a.ld<NX>(b + d * c.nb, Q.y[d]);
            }
        }
    }
    template <int NX>
    __device__ __forceinline__ void fin(const At& a, const Ld<NX>& Q, const T (&val)[3][NX], double* red) const {
        constexpr int NS = LPS ? 9 : 6;
        T La[3][NX];
        with_static<0, NS, NX>(c, a, Q.cb, [&](const T (&st)[NX][NS]) {
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                const T chi = Q.cb[q] ? T(1) : T(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    T acc = val[d][q];
#pragma unroll
                    for (int j = 0; j < 3; ++j) acc -= st[q][symi(3, d, j)] * Q.u[j][q];
                    if constexpr (LPS) acc += ka * Q.th[q] * st[q][6 + d];
                    La[d][q] = chi * acc;
                }
            }
        });
        finish<NX>(a, Q, La, red);
    }
    template <int NX>
    __device__ __forceinline__ void finish(const At& at, const Ld<NX>& Q, const T (&La)[3][NX], double* red) const {
        const int n = at.n;
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
                at.st<NX>(L + a * c.nb, out);
            }
        } else {
            if (mode == 0) {
#pragma unroll
                for (int a = 0; a < 3; ++a) at.st<NX>(L + a * c.nb, La[a]);
                return;
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                T bk[NX], vo[NX], fo[NX];
                if (b) at.ld<NX>(b + a * c.nb, bk);
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
                at.st<NX>(v + a * c.nb, vo);
                if (!vh_out) at.st<NX>(F + a * c.nb, fo);
                else {
                    T wk[NX];
                    if (w) at.ld<NX>(w + a * c.nb, wk);
#pragma unroll
                    for (int q = 0; q < NX; ++q)
                        wk[q] = omega_bit(Q.cb[q], a) ? Q.u[a][q] + dt * vo[q] : (w ? wk[q] : T(0));
                    at.st<NX>(u_next + a * c.nb, wk);
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
// All arguments of a launch.  The epilogue's are read from the argument
// segment plane by plane through an address the compiler cannot follow: held
// in scalar registers over the sweep, next to the kernel values, they would
// spill.
template <class T, class Ep, int MT>
struct D3Args {
    D3Geo g;
    D3In<T> in;
    Taps<T, MT> tp;
    double* partials;
    Ep ep;
};
template <class A>
__device__ __forceinline__ const A& launch_args() {
#if defined(__HIP_DEVICE_COMPILE__)
    auto p = (const __attribute__((address_space(4))) A*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const A*)p;
#else
    return *(const A*)nullptr;
#endif
}

// FP32 and FP64 tiles: TX columns along x, TY along y, NX nodes per thread.
template <class T, class Op, class Ep, int MT, int TX, int TY, int NX>
__global__ void __launch_bounds__((TX / NX) * TY) __attribute__((amdgpu_waves_per_eu(2)))
k_dir3(D3Args<T, Ep, MT> A) {
    using VA = typename Vec<T, NX>::A;
    constexpr int NI = Op::NI, NO = Op::NO, NT = (TX / NX) * TY;
    constexpr int H = (MT + NX - 1) / NX * NX;       // halo columns kept (aligned)
    constexpr int W = TX + 2 * H, HY = TY + 2 * MT;  // LDS row and rows of a plane
    constexpr int FX = TX + 2 * MT;                  // columns that are filled
    constexpr int NE = (FX * HY + NT - 1) / NT;      // nodes a thread fills
    extern __shared__ __align__(16) unsigned char smem_raw[];
    lds_ptr<T> lds = as_lds(reinterpret_cast<T*>(smem_raw));
    const D3Geo g = A.g;
    const Taps<T, MT>& tp = A.tp;

    // consecutive blocks of a z-chunk on one XCD (the hardware deals blocks to
    // the 8 XCDs in turn), so that the tiles sharing halos share an L2
    const unsigned nblk = gridDim.x, bq = nblk >> 3, br = nblk & 7;
    const unsigned xcd = blockIdx.x & 7, bk = blockIdx.x >> 3;
    const unsigned lin = xcd < br ? xcd * (bq + 1) + bk : br * (bq + 1) + (xcd - br) * bq + bk;
    const int tx0 = (int)(lin % g.ntx) * TX, ty0 = (int)(lin / g.ntx % g.nty) * TY;
    const int z0 = (int)(lin / (g.ntx * g.nty)) * g.zc, z1 = min(g.b3, z0 + g.zc);
    const long pl = (long)g.b1 * g.b2;

    const int tid = threadIdx.x, tx = tid % (TX / NX), ty = tid / (TX / NX);
    At at;
    {
        const int x = tx0 + tx * NX, y = ty0 + ty;
        at.pl = pl;
        at.n = y < g.b2 ? min(max(g.b1 - x, 0), NX) : 0;   // nodes of this thread in the body box
        at.off = at.n > 0 ? (uint32_t)(y * g.b1 + x) : 0u;
        at.tail = g.b1 % NX != 0;
    }

    // this thread's share of the plane fill: node offsets (kOut / 8 outside the
    // box, which reads zero) and LDS slots
    uint32_t go[NE];
    int lo[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = tid + NT * i, r = e / FX, cx = e - r * FX;
        const int gx = tx0 - MT + cx, gy = ty0 - MT + r;
        const bool ok = e < FX * HY && gx >= 0 && gx < g.b1 && gy >= 0 && gy < g.b2;
        go[i] = ok ? (uint32_t)(gy * g.b1 + gx) : kOut / 8;
        lo[i] = r * W + cx + (H - MT);
    }
    T pre[NI][NE];
    uint8_t pcb[NE];
    auto fetch = [&](int z) {
        const long base = (long)z * pl, in = z < g.b3 ? pl : 0;   // planes beyond the body read zero
        const Plane<uint8_t> fc(A.in.chiB, base, in);
#pragma unroll
        for (int i = 0; i < NE; ++i) pcb[i] = fc.ld(go[i]);
#pragma unroll
        for (int J = 0; J < NI; ++J) {
            const Plane<T> f(A.in.f[J], base, in);
#pragma unroll
            for (int i = 0; i < NE; ++i) pre[J][i] = f.ld(go[i] * (uint32_t)sizeof(T));
        }
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

    // (planes below the body would only add zeros)
    const int zb = max(z0 - MT, 0), ze = z1 + MT;
    fetch(zb);
    for (int zi = zb; zi < ze; ++zi) {
        lds_ptr<T> buf = lds + ((zi & 1) ? NI * HY * W : 0);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            if (NT * (i + 1) <= FX * HY || tid + NT * i < FX * HY) {
                const T chi = pcb[i] ? T(1) : T(0);
#pragma unroll
                for (int J = 0; J < NI; ++J) buf[J * HY * W + lo[i]] = chi * pre[J][i];
            }
        }
        __syncthreads();
        if (zi + 1 < ze) fetch(zi + 1);
        // the finished plane's node fields, in flight during the arithmetic
        const int zo = zi - MT;
        const bool outp = zo >= z0;   // block-uniform (zo < z1 by the sweep)
        at.base = (long)max(zo, 0) * pl;
        typename Ep::template Ld<NX> ld;
        if (outp) launch_args<D3Args<T, Ep, MT>>().ep.template load<NX>(at, ld);

        // plane sums: a0 (offset 0, into the accumulator of plane zi), qe and
        // qo (offsets 1 .. MT, even and odd along z)
        T a0[NO][NX], qe[MT + 1][NO][NX], qo[MT + 1][NO][NX];
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int n = 0; n < NX; ++n) {
                a0[o][n] = acc[MT][o][n];
            }
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
                            constexpr int pz = t_par(t, 2);
                            if constexpr (takes<Op>(MT, O, pz, c) && !starts<Op>(MT, O, pz, c, J, b, 0))
                                pin(pz ? qo[c][O] : qe[c][O]);
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
                                                else {
                                                    constexpr int pz = t_par(t, 2);
                                                    T& q = pz ? qo[c][O][n] : qe[c][O][n];
                                                    if constexpr (starts<Op>(MT, O, pz, c, J, b, a)) q = k * f;
                                                    else q += k * f;
                                                }
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
        if (outp) launch_args<D3Args<T, Ep, MT>>().ep.template fin<NX>(at, ld, out, red);
    }
    if constexpr (Ep::NRED > 0) {
        __syncthreads();
        double* sm = reinterpret_cast<double*>(smem_raw);
        block_reduce_store<Ep::NRED>(red, A.partials + (long)blockIdx.x * Ep::NRED, sm);
    }
}

// Tile of a block and nodes per thread: 32 x 16 columns, two nodes per
// thread.  RES: blocks a CU holds at once (by their registers).
template <class T, class Op, int MT>
struct Shape3 {
    static constexpr int TX = 32, TY = 16, NX = 2, NT = TX / NX * TY;
    static constexpr int RES = sizeof(T) == 4 ? (Op::NO == 1 ? 4 : (MT <= 3 ? 3 : 2)) : (Op::NO == 1 && MT <= 3 ? 3 : 2);
    static constexpr size_t lds() {
        return sizeof(T) * 2 * Op::NI * (TY + 2 * MT) * (TX + 2 * ((MT + NX - 1) / NX * NX));
    }
};
// Planes per chunk: enough blocks for every CU to hold its resident ones, but
// chunks no shorter than that needs, since each also sweeps up to 2 MT planes
// of its neighbours: the chunk count that minimises rounds x planes swept, a
// round being the blocks that 256 CUs hold at once (a last round that is
// partly empty costs as much as a full one).
inline int chunk3(const Geo& g, int mt, int tx, int ty, int res) {
    const long tiles = (long)((g.b1 + tx - 1) / tx) * ((g.b2 + ty - 1) / ty), slots = 256L * res;
    int best_zc = g.b3;
    double best = 0;
    for (int nz = 1; nz <= g.b3; ++nz) {
        const int zc = (g.b3 + nz - 1) / nz;
        const long blocks = tiles * ((g.b3 + zc - 1) / zc);
        const double cost = (double)((blocks + slots - 1) / slots) * (zc + (nz > 1 ? 2.0 * mt : 0.0));
        if (nz == 1 || cost < 0.98 * best) {
            best = cost;
            best_zc = zc;
        }
        if (blocks > 4 * slots) break;
    }
    return best_zc;
}

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
