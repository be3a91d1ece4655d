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
// flight meanwhile) with the nodes around the tile that its discs reach.  A
// thread owns NX consecutive nodes along x: it reads the rows y + b and y - b
// of a field, folds them along y (sum and difference), folds along x, and adds
// each folded value times the kernel value of (a, b, c) to the plane sums q_c
// of every output that takes it.  The plane sums then go to the outputs at
// z - c and z + c, which a thread keeps in 2 MT + 1 accumulators per output
// and node that shift by one per plane (the shift is the destination register
// of the add); the accumulator that has received its last plane goes to the
// epilogue.  Planes beyond the chunk run code of their own that leaves out the
// offsets that do not reach the chunk (128^3 FP32 force stage 62 -> 55 us).
//
// The kernel values are block-uniform: with one spacing along all axes they
// depend on r^2 and the product of the offsets only, so that a horizon of
// three spacings needs 12 + 8 + 12 distinct numbers, which stay in scalar
// registers (kernel arguments) for the whole sweep.  The epilogue's static
// fields are the same numbers at every interior node; a wave without edge
// nodes takes them from scalar registers.
//
// Measured, 256^3 LPS body in FP32, one Verlet step: dilatation 139 us, force
// stage 295 us (0.94 ms per step for the x transforms and (y, z) passes).  The
// force stage issues 1.27e8 wave instructions (485 per node, 0.70 per CU and
// cycle; k_nbb3, which does little else, 1.2) and moves 1.25 GB (0.97 GB of
// fields), the dilatation 4.6e7 (176 per node, 0.54 per CU and cycle, its LDS
// pipe as busy) and 0.53 GB (0.31 GB of fields, the rest tile and chunk halos:
// 3.8 TB/s).  In FP64 the issue rates are lower, 0.4 and 0.24 at 128^3: too few
// blocks per CU to overlap arithmetic and LDS reads; the pair tile of the FP64
// dilatation spends 44 % of its LDS cycles in bank conflicts.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "pd_plan.hpp"

namespace pdd {

using namespace pdk;

// Position update u + dt v + c2 F, as fixed multiply-adds: the element-wise
// pass and the epilogues give the same bits.
__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <class T>
__device__ __forceinline__ T position_update(T u, T dt, T v, T c2, T F) { return mad(c2, F, mad(dt, v, u)); }

// ------------------------------------------------------------ compile-time loops
template <int I0, int... I, class F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I0 + I>{}), ...);
}
// f(integral_constant<I>) for I = I0 .. I1 - 1
template <int I0, int I1, class F>
__device__ __forceinline__ void each(F&& f) {
    if constexpr (I0 < I1) each_of<I0>(std::make_integer_sequence<int, I1 - I0>{}, f);
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
// What the sweep's straight-line code asks of an operator, tabulated once:
//   takes[O][pz][c]     output O has a term of z-parity pz at plane offset c
//   first[O][pz][c]     the first (J, b, a), as (J 8 + b) 8 + a, in the
//                       sweep's order (inputs, rows, columns) of such a term:
//                       it starts the plane sum
//   uses[J][py][px][b][a]   input J has a term of x/y parities (px, py) at (a, b)
template <class Op, int MT>
struct OpTable {
    bool takes[Op::NO][2][MT + 1], uses[Op::NI][2][2][MT + 1][MT + 1];
    int first[Op::NO][2][MT + 1];
};
template <class Op, int MT>
constexpr OpTable<Op, MT> op_table() {
    OpTable<Op, MT> t{};
    for (int J = 0; J < Op::NI; ++J)
        for (int b = 0; b <= MT; ++b)
            for (int a = 0; a <= MT; ++a)
                for (int O = 0; O < Op::NO; ++O) {
                    const Term e = Op::term(O, J);
                    for (int c = 0; c <= MT; ++c) {
                        if (!t_nonzero(e, MT, a, b, c)) continue;
                        const int pz = t_par(e, 2);
                        t.uses[J][t_par(e, 1)][t_par(e, 0)][b][a] = true;
                        if (!t.takes[O][pz][c]) t.first[O][pz][c] = (J * 8 + b) * 8 + a;
                        t.takes[O][pz][c] = true;
                    }
                }
    return t;
}
template <class Op, int MT>
constexpr OpTable<Op, MT> kOp = op_table<Op, MT>();

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
    // NT: touched once per launch, not kept in the caches (non-temporal)
    template <bool NT = false>
    __device__ __forceinline__ T ld(uint32_t off) const {
        constexpr int C = NT ? 2 : 0;
        if constexpr (sizeof(T) == 1) return T(__builtin_amdgcn_raw_buffer_load_b8(r, off, 0, C));
        else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, C));
        else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, C));
    }
    __device__ __forceinline__ void st(uint32_t off, T v) const {
        if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 2);
        else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, 2);
    }
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    // NX values at byte offset off
    template <int NX, bool NT>
    __device__ __forceinline__ void ldv(uint32_t off, T (&out)[NX]) const {
        constexpr int B = NX * (int)sizeof(T), C = NT ? 2 : 0;
        if constexpr (NX == 1 || sizeof(T) == 1) {
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = ld<NT>(off + q);
        } else {
            static_assert(B == 8 || B == 16, "8 or 16 bytes per thread");
            typename Vec<T, NX>::A w;
            if constexpr (B == 8) w = __builtin_bit_cast(typename Vec<T, NX>::A, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, C));
            else w = __builtin_bit_cast(typename Vec<T, NX>::A, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, C));
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = w[q];
        }
    }
    template <int NX>
    __device__ __forceinline__ void stv(uint32_t off, const T (&val)[NX]) const {
        if constexpr (NX == 1) st(off, val[0]);
        else {
            typename Vec<T, NX>::A w;
#pragma unroll
            for (int q = 0; q < NX; ++q) w[q] = val[q];
            if constexpr (NX * sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, w), r, off, 0, 2);
            else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), r, off, 0, 2);
        }
    }
#else   // host pass: never runs
    __device__ Plane(const T*, long, long) {}
    template <bool NT = false>
    __device__ T ld(uint32_t) const { return T(0); }
    __device__ void st(uint32_t, T) const {}
    template <int NX, bool NT>
    __device__ void ldv(uint32_t, T (&)[NX]) const {}
    template <int NX>
    __device__ void stv(uint32_t, const T (&)[NX]) const {}
#endif
};

// Where a thread's nodes are: plane [base, base + pl) of the box, from off on,
// n of them.  WIDE: n is 0 or NX (NX divides the rows), accesses are NX wide;
// else node by node.  nb: nodes of the box, the distance of a field's
// components (kept opaque per plane, so that the sweep does not hold every
// component's address in scalar registers).
template <bool WIDE>
struct At {
    long base, pl, nb;
    uint32_t off;
    int n;
    template <class T>
    __device__ __forceinline__ uint32_t at(int q) const { return q < n ? (off + q) * (uint32_t)sizeof(T) : kOut; }
    template <int NX, bool NT = false, class T>
    __device__ __forceinline__ void ld(const T* p, int d, T (&out)[NX]) const {
        const Plane<T> f(p, base + d * nb, pl);
        if constexpr (WIDE && sizeof(T) > 1) f.template ldv<NX, NT>(at<T>(0), out);
        else {
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = f.template ld<NT>(at<T>(q));
        }
    }
    template <int NX, class T>
    __device__ __forceinline__ void st(T* p, int d, const T (&val)[NX]) const {
        const Plane<T> f(p, base + d * nb, pl);
        if constexpr (WIDE) f.template stv<NX>(at<T>(0), val);
        else {
#pragma unroll
            for (int q = 0; q < NX; ++q) f.st(at<T>(q), val[q]);
        }
    }
};
// Whether a wave has a node of the body that is not interior (its static
// fields differ from the interior sums).
template <int NX, class AT>
__device__ __forceinline__ bool edge_wave(const AT& a, const uint8_t (&cb)[NX]) {
    bool edge = false;
#pragma unroll
    for (int q = 0; q < NX; ++q) edge = edge || (q < a.n && !(cb[q] & 2));
    return __ballot(edge) != 0;
}
// Static fields Q0 .. Q0 + N - 1 of the nodes in such a wave.
template <int Q0, int N, int NX, class T, class AT>
__device__ __forceinline__ void statics(const NodeCtx<T>& c, const AT& a, const uint8_t (&cb)[NX], T (&st)[NX][N]) {
#pragma unroll
    for (int q = 0; q < NX; ++q) {
#pragma unroll
        for (int k = 0; k < N; ++k) st[q][k] = c.sint[Q0 + k];
        if (q < a.n) c.template st_range<Q0, N>(Nd{a.base, a.off + q}, cb[q], st[q]);
    }
}

// ------------------------------------------------------------ arguments
struct D3Geo {
    int b1, b2, b3;
    int ntx, nty, nzc, zc;   // tiles along x and y, chunks of zc planes along z
};
template <class T>
struct D3In {
    const T* f[4];           // input fields (each one component)
    const uint8_t* chiB;     // node flags: inputs are multiplied by chi_B
};
// All arguments of a launch.  The sweep keeps the kernel values and what every
// plane needs in scalar registers; what only some waves need (the static
// fields of edge nodes, loads and prescribed values, the non-finite flag) is
// read from the argument segment where it is needed (rare_args), through an
// address the compiler cannot follow: kept over the sweep it would spill.
template <class T, class Ep, int MT>
struct D3Args {
    D3Geo g;
    D3In<T> in;
    Taps<T, MT> tp;
    double* partials;
    T g0;       // interior node: G_ij = g0 [i == j] (force), 3 / m (dilatation); g_i = 0
    Ep ep;
};
template <class A>
__device__ __forceinline__ const A& rare_args() {
#if defined(__HIP_DEVICE_COMPILE__)
    auto p = (const __attribute__((address_space(4))) A*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const A*)p;
#else
    return *(const A*)nullptr;
#endif
}

// ------------------------------------------------------------ epilogues
// Each has load (node fields, issued before the plane's arithmetic; HELD: the
// input values at the nodes, chi u and chi theta, come from the sweep through
// hold instead) and fin.
// Dilatation: theta = 3 chi / m (S - g_i u_i), 0 off the body or where m = 0.
template <class T>
struct EpTheta {
    static constexpr int NOUT = 1, NRED = 0;
    static constexpr bool HOLD = true;
    NodeCtx<T> c;
    const T* u;
    T* theta;
    __host__ double nbytes() const { return 4.0 * sizeof(T) + 4.0 * sizeof(T) * c.edge_frac + 1.0; }
    template <int NX>
    struct Ld { T u[3][NX]; uint8_t cb[NX]; };
    template <int MT, int NX, bool HELD, class AT>
    __device__ __forceinline__ void load(const AT& a, const uint8_t* chiB, Ld<NX>& Q) const {
        a.template ld<NX>(chiB, 0, Q.cb);
        if constexpr (!HELD) {
#pragma unroll
            for (int d = 0; d < 3; ++d) a.template ld<NX>(u, d, Q.u[d]);
        }
    }
    template <int NX>
    __device__ __forceinline__ static void hold(Ld<NX>& Q, const T (&in)[3][NX]) {
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int q = 0; q < NX; ++q) Q.u[d][q] = in[d][q];
    }
    template <int MT, int NX, class AT>
    __device__ __forceinline__ void fin(const AT& a, const Ld<NX>& Q, T g0, const T (&val)[1][NX], double*) const {
        T out[NX];
        if (!edge_wave(a, Q.cb)) {
#pragma unroll
            for (int q = 0; q < NX; ++q) out[q] = Q.cb[q] ? g0 * val[0][q] : T(0);
        } else {
            T st[NX][4];
            statics<6, 4, NX>(rare_args<D3Args<T, EpTheta, MT>>().ep.c, a, Q.cb, st);
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                T acc = val[0][q];
#pragma unroll
                for (int d = 0; d < 3; ++d) acc -= st[q][d] * Q.u[d][q];
                const T m = st[q][3];
                const bool on = Q.cb[q] && m != T(0);
                out[q] = on ? T(3) / (on ? m : T(1)) * acc : T(0);
            }
        }
        a.template st<NX>(theta, 0, out);
    }
};

// Force: L_i = chi (conv_i [+ k_a theta g_i] - G_ij u_j), then by kind
//   FORCE   L
//   STEP    Verlet: F' = L + b, v <- chi_O [v + c1 (F + F')], with vh_in,
//           vh_out and next (kernel-uniform) as pdd::Eval; u_next is another
//           buffer than u, which other blocks still read
//   INNER   STEP with vh_in = vh_out = next = 1: no F
//   ENERGY  STEP with the energy sums
//   SOLVER  mode 2: -chi_O L and the partial sum of u . (-chi_O L);
//           mode 3: r = chi_O (L + b) and the partial sum of |r|^2
enum { FORCE = 0, STEP = 1, INNER = 2, ENERGY = 3, SOLVER = 4 };
template <class T, bool LPS, int KIND>
struct EpForce {
    static constexpr int NOUT = 3, NRED = KIND == ENERGY ? 4 : (KIND == SOLVER ? 1 : 0);
    static constexpr bool VV = KIND == STEP || KIND == INNER || KIND == ENERGY;
    // (the energy sums take u off the body too: no held values there)
    static constexpr bool HOLD = KIND != ENERGY;
    NodeCtx<T> c;
    int mode;
    T ka;
    const T* u; const T* theta;
    T* L; T* v; T* F; const T* b; const T* w;
    T c1, c2, rho, dt;
    T* u_next;
    double* nanflag;
    int vh_in, vh_out, next;
    int has;            // bit 0: b, bit 1: w
    __host__ double nbytes() const {
        const double t = sizeof(T);
        double r = 3 * t + 1 + 6 * t * c.edge_frac + (LPS ? t + 3 * t * c.edge_frac : 0.0) + (b ? 3 * t : 0.0);
        if (VV) return r + 3 * t * (2 + (vh_in ? 0 : 1) + (vh_out ? 0 : 1) + (next ? (w ? 2 : 1) : 0));
        return r + 3 * t;
    }
    // x: v; y: F (STEP, ENERGY), else b
    template <int NX>
    struct Ld { T u[3][NX], th[NX], x[VV ? 3 : 1][NX], y[3][NX]; uint8_t cb[NX]; };
    template <int MT, int NX, bool HELD, class AT>
    __device__ __forceinline__ void load(const AT& a, const uint8_t* chiB, Ld<NX>& Q) const {
        a.template ld<NX>(chiB, 0, Q.cb);
        if constexpr (!HELD) {
#pragma unroll
            for (int d = 0; d < 3; ++d) a.template ld<NX>(u, d, Q.u[d]);
            if constexpr (LPS) a.template ld<NX>(theta, 0, Q.th);
        }
        if constexpr (VV) {
#pragma unroll
            for (int d = 0; d < 3; ++d) a.template ld<NX, true>(v, d, Q.x[d]);
        }
        if constexpr (KIND != FORCE) {
            const bool some = KIND == INNER ? (has & 1) != 0 : (KIND == SOLVER ? mode == 3 : !vh_in);
            if (some) {
                const EpForce& e = rare_args<D3Args<T, EpForce, MT>>().ep;
                const T* y = KIND == INNER || KIND == SOLVER ? e.b : e.F;
#pragma unroll
                for (int d = 0; d < 3; ++d) a.template ld<NX, true>(y, d, Q.y[d]);
            } else {
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                    for (int q = 0; q < NX; ++q) Q.y[d][q] = T(0);
            }
        }
    }
    template <int NX>
    __device__ __forceinline__ static void hold(Ld<NX>& Q, const T (&in)[LPS ? 4 : 3][NX]) {
#pragma unroll
        for (int q = 0; q < NX; ++q) {
#pragma unroll
            for (int d = 0; d < 3; ++d) Q.u[d][q] = in[d][q];
            if constexpr (LPS) Q.th[q] = in[3][q];
        }
    }
    template <int MT, int NX, class AT>
    __device__ __forceinline__ void fin(const AT& at, const Ld<NX>& Q, T g0, const T (&val)[3][NX], double* red) const {
        T La[3][NX];
        if (!edge_wave(at, Q.cb)) {
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                const T chi = Q.cb[q] ? T(1) : T(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) La[d][q] = chi * (val[d][q] - g0 * Q.u[d][q]);
            }
        } else {
            constexpr int NS = LPS ? 9 : 6;
            const EpForce& e = rare_args<D3Args<T, EpForce, MT>>().ep;
            T st[NX][NS];
            statics<0, NS, NX>(e.c, at, Q.cb, st);
#pragma unroll
            for (int q = 0; q < NX; ++q) {
                const T chi = Q.cb[q] ? T(1) : T(0);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    T acc = val[d][q];
#pragma unroll
                    for (int j = 0; j < 3; ++j) acc -= st[q][symi(3, d, j)] * Q.u[j][q];
                    if constexpr (LPS) acc += e.ka * Q.th[q] * st[q][6 + d];
                    La[d][q] = chi * acc;
                }
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if constexpr (KIND == FORCE) {
                at.template st<NX>(L, a, La[a]);
            } else if constexpr (KIND == SOLVER) {
                T out[NX];
#pragma unroll
                for (int q = 0; q < NX; ++q) {
                    const bool o = omega_bit(Q.cb[q], a);   // (false where the thread has no node)
                    if (mode == 2) {
                        out[q] = o ? -La[a][q] : T(0);
                        red[0] += o ? double(Q.u[a][q]) * double(out[q]) : 0.0;
                    } else {
                        out[q] = o ? La[a][q] + Q.y[a][q] : T(0);
                        red[0] += double(out[q]) * double(out[q]);
                    }
                }
                at.template st<NX>(L, a, out);
            } else if constexpr (KIND == INNER) {
                T vo[NX], un[NX];
                if (has & 2) at.template ld<NX, true>(rare_args<D3Args<T, EpForce, MT>>().ep.w, a, un);
                bool bad = false;
#pragma unroll
                for (int q = 0; q < NX; ++q) {
                    const bool o = omega_bit(Q.cb[q], a);
                    const T Fn = La[a][q] + Q.y[a][q], vf = Q.x[a][q] + c1 * Fn, vn = o ? vf : T(0);
                    bad = bad || (q < at.n && !(__builtin_isfinite(Fn) && __builtin_isfinite(vn)));
                    vo[q] = o ? vn + c1 * Fn : T(0);
                    un[q] = o ? mad(dt, vo[q], Q.u[a][q]) : ((has & 2) ? un[q] : T(0));
                }
                if (bad) {
                    double* flag = rare_args<D3Args<T, EpForce, MT>>().ep.nanflag;
                    if (flag) *flag = 1.0;
                }
                at.template st<NX>(v, a, vo);
                at.template st<NX>(u_next, a, un);
            } else {
                T bk[NX], vo[NX], fo[NX];
#pragma unroll
                for (int q = 0; q < NX; ++q) bk[q] = T(0);
                if (b) at.template ld<NX, true>(b, a, bk);
#pragma unroll
                for (int q = 0; q < NX; ++q) {
                    const bool o = omega_bit(Q.cb[q], a);
                    const T Fn = La[a][q] + bk[q];
                    const T vf = Q.x[a][q] + c1 * (Q.y[a][q] + Fn);
                    const T vn = o ? vf : T(0);
                    if (q < at.n) flag_nonfinite(nanflag, Fn, vn);
                    fo[q] = Fn;
                    vo[q] = vh_out ? (o ? vn + c1 * Fn : T(0)) : vn;
                    if constexpr (KIND == ENERGY) {
                        if (q < at.n) {
                            red[0] += 0.5 * double(rho) * double(vn) * double(vn);
                            red[1] += -0.5 * double(Q.u[a][q]) * double(La[a][q]);
                            red[2] += -double(bk[q]) * double(Q.u[a][q]);
                            red[3] += o ? double(Fn) * double(Fn) : 0.0;
                        }
                    }
                }
                at.template st<NX>(v, a, vo);
                if (!vh_out) at.template st<NX>(F, a, fo);
                if (next) {
                    T un[NX];
                    if (w) at.template ld<NX, true>(w, a, un);
#pragma unroll
                    for (int q = 0; q < NX; ++q) {
                        const T x = vh_out ? mad(dt, vo[q], Q.u[a][q])
                                           : position_update(Q.u[a][q], dt, vo[q], c2, fo[q]);
                        un[q] = omega_bit(Q.cb[q], a) ? x : (w ? un[q] : T(0));
                    }
                    at.template st<NX>(u_next, a, un);
                }
            }
        }
    }
};

// ------------------------------------------------------------ the sweep
// Nodes of a plane that a tile of TX x TY columns reads: row by row the
// columns within the disc's reach of the tile (fewer beyond its corners).
template <int MT, int TX, int TY>
struct Fill {
    static constexpr int HY = TY + 2 * MT;
    __host__ __device__ static constexpr int reach(int r) {
        const int d = r < MT ? MT - r : (r >= TY + MT ? r - (TY + MT) + 1 : 0);
        return isqrt(MT * MT - d * d);
    }
    __host__ __device__ static constexpr int start(int r) {   // nodes in the rows before r
        int n = 0;
        for (int k = 0; k < r; ++k) n += TX + 2 * reach(k);
        return n;
    }
    static constexpr int N = start(HY);
};

// A launch shape: tile of TX x TY columns, NX nodes per thread (all along x),
// WIDE: NX divides the rows; RING: the nodes' own inputs wait in LDS for the
// epilogue; WPE: waves per SIMD the registers are bounded for.
template <int TX_, int TY_, int NX_, bool WIDE_, bool RING_, int WPE_>
struct Shape {
    static constexpr int TX = TX_, TY = TY_, NX = NX_, NT = TX / NX * TY, WPE = WPE_;
    static constexpr bool WIDE = WIDE_, RING = RING_;
    template <class T, class Op, int MT>
    static constexpr size_t lds() {
        return sizeof(T) * Op::NI * (2 * (TY + 2 * MT) * (TX + 2 * ((MT + NX - 1) / NX * NX)) + (RING ? MT * TX * TY : 0));
    }
};

template <class T, class Op, class Ep, int MT, class SH>
__global__ void __launch_bounds__(SH::NT) __attribute__((amdgpu_waves_per_eu(SH::WPE)))
k_dir3(D3Args<T, Ep, MT> A) {
    constexpr int TX = SH::TX, TY = SH::TY, NX = SH::NX, NT = SH::NT;
    using VA = typename Vec<T, NX>::A;
    using FL = Fill<MT, TX, TY>;
    constexpr int NI = Op::NI, NO = Op::NO;
    constexpr int H = (MT + NX - 1) / NX * NX;       // halo columns kept (aligned)
    constexpr int W = TX + 2 * H, HY = TY + 2 * MT;  // LDS row and rows of a plane
    constexpr int NE = (FL::N + NT - 1) / NT;        // nodes a thread fills
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
    At<SH::WIDE> at;
    {
        const int x = tx0 + tx * NX, y = ty0 + ty;
        at.pl = pl;
        at.n = y < g.b2 ? min(max(g.b1 - x, 0), NX) : 0;   // nodes of this thread in the body box
        at.off = at.n > 0 ? (uint32_t)(y * g.b1 + x) : 0u;
        at.nb = A.ep.c.nb;
    }

    // this thread's share of the plane fill: node offsets (kOut / 8 outside the
    // box, which reads zero) and LDS slots
    uint32_t go[NE];
    int lo[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int e = tid + NT * i;
        int r = 0, cx = e + MT - FL::reach(0);   // row, and column counted from tx0 - MT
        each<1, HY>([&](auto rc) {
            constexpr int k = decltype(rc)::value;
            if (e >= FL::start(k)) {
                r = k;
                cx = e - FL::start(k) + MT - FL::reach(k);
            }
        });
        const int gx = tx0 - MT + cx, gy = ty0 - MT + r;
        const bool ok = e < FL::N && gx >= 0 && gx < g.b1 && gy >= 0 && gy < g.b2;
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

    // One input plane zi.  D: its distance beyond the chunk (0 inside), on
    // side S (-1 below, +1 above): only plane offsets c >= D reach the chunk,
    // on one side, so the planes of the neighbouring chunks cost a third of
    // an inner one on average.
    const int zb = max(z0 - MT, 0), ze = z1 + MT;   // (planes below the body would only add zeros)
    constexpr bool HELD = SH::RING && Ep::HOLD;
    lds_ptr<T> ring = lds + 2 * NI * HY * W + tid * NX;   // [MT][NI][NT * NX]
    fetch(zb);
    auto plane = [&](auto Dc, auto Sc, const int zi) {
        constexpr int D = decltype(Dc)::value, S = decltype(Sc)::value;
        lds_ptr<T> buf = lds + ((zi & 1) ? NI * HY * W : 0);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            if (NT * (i + 1) <= FL::N || tid + NT * i < FL::N) {
                const T chi = pcb[i] ? T(1) : T(0);
#pragma unroll
                for (int J = 0; J < NI; ++J) buf[J * HY * W + lo[i]] = chi * pre[J][i];
            }
        }
        __syncthreads();
        if (zi + 1 < ze) fetch(zi + 1);
        // the finished plane's node fields, in flight during the arithmetic
        const int zo = zi - MT;
        const bool outp = S >= 0 && zo >= z0;   // block-uniform (zo < z1 by the sweep)
        typename Ep::template Ld<NX> ld;
        if constexpr (S >= 0) {
            at.base = (long)max(zo, 0) * pl;
            #if defined(__HIP_DEVICE_COMPILE__)
            asm volatile("" : "+s"(at.nb));
#endif
            if (outp) A.ep.template load<MT, NX, HELD>(at, A.in.chiB, ld);
        }
        if constexpr (HELD && S >= 0) {
            // the nodes' own inputs of the finished plane, kept in LDS since
            // that plane went by (each thread its own slots, MT planes)
            lds_ptr<T> slot = ring + (zi % MT) * (NI * NT * NX);
            T own[NI][NX];
#pragma unroll
            for (int J = 0; J < NI; ++J) {
                const VA w = *(lds_ptr<VA>)(slot + J * NT * NX);
#pragma unroll
                for (int n = 0; n < NX; ++n) own[J][n] = w[n];
                if constexpr (D == 0)
                    *(lds_ptr<VA>)(slot + J * NT * NX) = *(lds_ptr<VA>)(buf + J * HY * W + (ty + MT) * W + H + tx * NX);
            }
            Ep::template hold<NX>(ld, own);
        }

        // plane sums: a0 (offset 0, into the accumulator of plane zi), qe and
        // qo (offsets 1 .. MT, even and odd along z)
        T a0[NO][NX], qe[MT + 1][NO][NX], qo[MT + 1][NO][NX];
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int n = 0; n < NX; ++n) {
                a0[o][n] = acc[MT][o][n];
            }
        constexpr int RD = D == 0 ? MT : isqrt(MT * MT - D * D);   // |(a, b)| of the terms with c >= D
        // Row pair (J, b), k = J (RD + 1) + b: the rows y + b and y - b of input
        // J around the thread's nodes, columns -RA .. NX - 1 + RA.  The reads of
        // pair k + 1 are in flight during the sums of pair k.
        auto row_read = [&](auto kc, auto& up, auto& dn) {
            constexpr int J = decltype(kc)::value / (RD + 1), b = decltype(kc)::value % (RD + 1);
            constexpr int R = isqrt(MT * MT - D * D - b * b), RA = (R + NX - 1) / NX * NX, WN = NX + 2 * RA;
            lds_ptr<T> fld = buf + J * HY * W + (ty + MT) * W + tx * NX + (H - RA);
#pragma unroll
            for (int k = 0; k < WN / NX; ++k) {
                const VA a = *(lds_ptr<VA>)(fld + b * W + k * NX);
#pragma unroll
                for (int n = 0; n < NX; ++n) up[k * NX + n] = a[n];
                if constexpr (b > 0) {
                    const VA d = *(lds_ptr<VA>)(fld - b * W + k * NX);
#pragma unroll
                    for (int n = 0; n < NX; ++n) dn[k * NX + n] = d[n];
                }
            }
        };
        auto row_sums = [&](auto kc, const auto& up, const auto& dn) {
            constexpr int J = decltype(kc)::value / (RD + 1), b = decltype(kc)::value % (RD + 1);
            constexpr int R = isqrt(MT * MT - D * D - b * b), RA = (R + NX - 1) / NX * NX, WN = NX + 2 * RA;
            T E[WN], Od[WN];
#pragma unroll
            for (int k = 0; k < WN; ++k) {
                E[k] = b > 0 ? up[k] + dn[k] : up[k];
                Od[k] = b > 0 ? up[k] - dn[k] : T(0);
            }
            each<0, R + 1>([&](auto ac) {
                constexpr int a = decltype(ac)::value;
                each<0, 4>([&](auto pc) {
                    constexpr int px = decltype(pc)::value & 1, py = decltype(pc)::value >> 1;
                    if constexpr (kOp<Op, MT>.uses[J][py][px][b][a]) {
#pragma unroll
                        for (int n = 0; n < NX; ++n) {
                            const T p = py ? Od[RA + n + a] : E[RA + n + a];
                            const T m = py ? Od[RA + n - a] : E[RA + n - a];
                            const T f = a == 0 ? p : (px ? p - m : p + m);
                            each<0, NO>([&](auto Oc) {
                                constexpr int O = decltype(Oc)::value;
                                constexpr Term t = Op::term(O, J);
                                if constexpr (t.i >= 0 && t_par(t, 0) == px && t_par(t, 1) == py) {
                                    each<D, MT + 1>([&](auto cc) {
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
                                                if constexpr (kOp<Op, MT>.first[O][pz][c] == (J * 8 + b) * 8 + a) q = k * f;
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
            // the sums this pair added to end here
            each<0, NO>([&](auto Oc) {
                constexpr int O = decltype(Oc)::value;
                constexpr Term t = Op::term(O, J);
                if constexpr (t.i >= 0) {
                    if constexpr (D == 0 && t_par(t, 2) == 0) pin(a0[O]);
                    each<(D > 0 ? D : 1), MT + 1>([&](auto cc) {
                        constexpr int c = decltype(cc)::value, pz = t_par(t, 2);
                        if constexpr (kOp<Op, MT>.takes[O][pz][c] && kOp<Op, MT>.first[O][pz][c] < (J * 8 + b + 1) * 8)
                            pin(pz ? qo[c][O] : qe[c][O]);
                    });
                }
            });
            row_fence();
        };
        constexpr int NK = NI * (RD + 1), WM = NX + 2 * H;   // row pairs; the widest row
        T ru[2][WM], rd[2][WM];
        row_read(std::integral_constant<int, 0>{}, ru[0], rd[0]);
        each<0, NK>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if constexpr (k + 1 < NK) row_read(std::integral_constant<int, k + 1>{}, ru[(k + 1) & 1], rd[(k + 1) & 1]);
            row_sums(kc, ru[k & 1], rd[k & 1]);
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
                    if constexpr (c > 0 && c >= D && (S == 0 || (S < 0) == (p > MT))) {
                        if constexpr (kOp<Op, MT>.takes[O][0][c]) s += qe[c][O][n];
                        if constexpr (kOp<Op, MT>.takes[O][1][c]) s = p < MT ? s + qo[c][O][n] : s - qo[c][O][n];
                    }
                    if constexpr (p == 0) out[O][n] = s;
                    else acc[p - 1][O][n] = s;
                }
            });
        });
        if constexpr (S >= 0) {
            if (outp) A.ep.template fin<MT, NX>(at, ld, A.g0, out, red);
        }
    };
    using std::integral_constant;
    each<0, MT>([&](auto kc) {
        constexpr int D = MT - decltype(kc)::value;
        if (z0 - D >= 0) plane(integral_constant<int, D>{}, integral_constant<int, -1>{}, z0 - D);
    });
    for (int zi = z0; zi < z1; ++zi) plane(integral_constant<int, 0>{}, integral_constant<int, 0>{}, zi);
    each<1, MT + 1>([&](auto kc) {
        constexpr int D = decltype(kc)::value;
        plane(integral_constant<int, D>{}, integral_constant<int, 1>{}, z1 - 1 + D);
    });
    if constexpr (Ep::NRED > 0) {
        __syncthreads();
        double* sm = reinterpret_cast<double*>(smem_raw);
        block_reduce_store<Ep::NRED>(red, A.partials + (long)blockIdx.x * Ep::NRED, sm);
    }
}

// Launch shapes.  Four waves cover a tile of 32 x 8 columns, one node per
// thread: the tile reads exactly 512 nodes of a plane at a horizon of three
// spacings, two per thread, and its few registers keep five (FP32) or three
// (FP64) blocks on a CU.  (256^3 FP32 force stage: 288 us, against 293 us for
// 32 x 16 columns with two nodes per thread, 366 us for 16 x 16 columns; 81 x
// 80 x 77: 23.1, 26.8 and 27 us.)  The FP64 dilatation, one output and three
// inputs, is bound by LDS reads instead and takes two nodes per thread (256^3
// 226 us against 263 us).
template <class T, class Op, int MT>
struct Shape3 {
    static constexpr bool PAIR = sizeof(T) == 8 && Op::NO == 1;
    template <bool WIDE>
    using S = std::conditional_t<PAIR, Shape<32, 16, 2, WIDE, true, 2>, Shape<32, 8, 1, true, sizeof(T) == 4 || Op::NO == 1, 2>>;
    // blocks that a CU holds at once, by their registers and LDS
    static constexpr int regs = sizeof(T) == 4 ? (Op::NO == 1 ? 7 : (MT == 2 ? 7 : (MT == 3 ? 5 : 4)))
                                               : (Op::NO == 1 ? 2 : (MT == 2 ? 4 : (MT == 3 ? 3 : 2)));
    static constexpr int RES = std::min<int>(regs, 160 * 1024 / (int)S<true>::template lds<T, Op, MT>());
    // of a plane's time, the part that does not grow with the blocks on the
    // CU (latencies) over the part each adds (its arithmetic): measured 2 in
    // FP32, 1 in FP64
    static constexpr double LAT = sizeof(T) == 4 ? 2.0 : 1.0;
};
// Planes per chunk: enough chunks to fill the CUs, but no more, since each
// also sweeps 2 MT planes of its neighbours (at a third of the cost of its
// own): the chunk that minimises the time of its rounds, a round being the
// blocks that 256 CUs hold at once.
inline int chunk3(const Geo& g, int mt, int tx, int ty, int res, double lat) {
    const long tiles = (long)((g.b1 + tx - 1) / tx) * ((g.b2 + ty - 1) / ty), slots = 256L * res;
    int best_zc = g.b3;
    double best = 0;
    for (int nz = 1; nz <= g.b3; ++nz) {
        const int zc = (g.b3 + nz - 1) / nz;
        const long blocks = tiles * ((g.b3 + zc - 1) / zc), full = blocks / slots, rest = blocks - full * slots;
        const double rounds = full * (lat + res) + (rest ? lat + (double)((rest + 255) / 256) : 0.0);
        const double cost = rounds * (zc + mt + 1);
        if (nz == 1 || cost < best) {
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
            const T xn = position_update(u[k], dt, v[k], c2, F[k]);
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
