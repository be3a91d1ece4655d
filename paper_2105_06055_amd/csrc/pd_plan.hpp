// pd_plan.hpp -- host-side plan object and chain runners (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <vector>

#include "pd_fcbm.h"
#include "pd_fcbm_testing.h"
#include "pd_passes.hpp"

// One timed kernel launch (profiling mode): events recorded on the launch
// stream right before and after the kernel, plus its algorithmic bytes.
struct ProfRec {
    char name[32];
    hipEvent_t a, b;
    double bytes;
};

struct pd_plan_s {
    // geometry
    int dim;
    int n[3], b[3];
    double dx[3];
    double delta;
    int influence;
    pd_kernel kern;
    pd_dtype dtype;
    int flags;
    hipStream_t stream0;
    int device;
    int max_lds;                 // bytes of LDS a block may use
    int lastaxis;                // PD_LASTAXIS_* (kernel choice for the last axis)
    pdk::Geo geo;
    long nb, nfft;
    // stencil and kernels
    int ns;                      // bonds per node
    int ntap;                    // taps along the last axis (max |o_last| + 1)
    int nct, ncs;                // taps components, static components
    uint32_t oddmask;            // last-axis parity of each taps component
    double alpha, m0, kappa, mu, ka, Wc, dt_max, dV;
    // spectral preconditioner of the static solve, in tap units (Ĉ/Nfft):
    // diagonal of Ĉ(0), identity shift, normalisation s0 = Ĉ(0)_xx/Nfft
    double pre_k0[3], pre_shift, pre_s0;
    int beta_comp;               // static component holding the omega_0 bond count
    // device buffers
    void* tw;                    // T twiddles: table for length N at [N, 2N)
    double* tw64;                // FP64 twiddles, same layout
    void* taps;                  // T [NP][nct][ntap], transform convention
    void* taps_d;                // T [NP][nct][ntap], direct convention
    void* taps_yz;               // T [h1][nct_yz][yz_nu]: partial x-spectra over the (y, z) quarter disc (3D)
    int yz_mt, yz_nu;            // its radius in spacings (0: no (y, z) direct pass) and tap count
    int nct_yz;                  // components in taps_yz (nct, + 3 scaled copies k_a a0_i for LPS)
    void* stat;                  // T [nb][ncs]
    void* stat_int;              // T [ncs]: the static fields at interior nodes
    double stat_int_h[10];       // the same values (rounded to T) on the host
    long n_edge;                 // body-box nodes that are not interior
    uint8_t* chiB;               // [nb] body | interior << 1 (interior: whole horizon in the body)
    uint8_t* chiO;               // [dim][nb]
    void* SA;                    // complex T workspaces (see pd_passes.hpp)
    void* SB;
    long saf_cap, sbf_cap, scf_cap;   // field capacity of each workspace
    int Pz;                      // z pitch of SB (body planes rounded up to 16)
    long sbf;                    // field stride of SB: h1*n2*Pz
    void* theta;                 // T [nb] (LPS)
    void* vtmp;                  // T [dim][nb] scratch (solver / adjoint)
    void* vtmp2;                 // T [dim][nb]
    double* partials;            // per-block reduction partials
    long partials_cap;
    double* cg_partials;         // those of the solver's vector updates [kCgBlocks]
    bool raw_sum;                // finish_reduction leaves single sums to their reader
    pdk::PartialSum sum;         // the last single sum
    double* red;                 // final reductions [8]
    double* red_host;            // pinned host copy [16]
    double* red_host_dev;        // device address of red_host (null if not mapped)
    hipEvent_t lag_ev[2];        // completion events of the solver's lagged residual reads
    int* offs_dev;               // stencil offsets [ns][3]
    void* etab;                  // T [ns][4]: xi_x, xi_y, alpha omega / |xi|^2 dV, 0 (2D bond-based energy)
    int emt;                     // largest |o_x|, |o_y| of the stencil (halo of the energy kernel)
    int energy_form;             // 0: W by direct bond sums, 1: by the convolution form (test mode)
    double* kval_dev;            // kernel values [ns][ncs]
    // direct horizon sums (pd_direct.hpp): radius of the ball of offsets in
    // spacings (0: the plan does not qualify) and, by r^2 in spacings, the
    // radial factors c and a with C_ij(o) = c[r^2] o_i o_j, a_i(o) = a[r^2] o_i
    int dir_mt;
    double dir_c[65], dir_a[65];
    bool dir_linear;             // the unweighted linear calls too (pdd::linear_on)
    long dir_blocks;             // most blocks of a launch (reduction partials)
    int dir_planes;              // planes per block in 3D (test mode; 0: chunk3)
    size_t bytes;
    std::vector<ProfRec>* prof;  // non-null while pass timing is enabled
    pd_plan_s* sub32;            // FP32 operator for the mixed solve
    pd_plan_s* parent;           // set on sub32
};

// Whether the transform chains of a plan take their default forms (the plans
// without direct sums, and PD_LASTAXIS_TRANSFORM on the others).
inline bool default_lines(pd_plan p) {
    return p->lastaxis == PD_LASTAXIS_AUTO || p->lastaxis == PD_LASTAXIS_TRANSFORM;
}

namespace pdh {

pd_status check(hipError_t e);

}  // namespace pdh

namespace pdi {

template <class T>
pdk::NodeCtx<T> ctx(pd_plan p) {
    pdk::NodeCtx<T> c;
    c.nb = p->nb;
    c.chiB = p->chiB;
    c.stat = reinterpret_cast<const T*>(p->stat);
    c.ncs = p->ncs;
    c.stat_int = reinterpret_cast<const T*>(p->stat_int);
    for (int q = 0; q < 10; ++q) c.sint[q] = T(q < p->ncs ? p->stat_int_h[q] : 0.0);
    c.edge_frac = p->nb > 0 ? (double)p->n_edge / (double)p->nb : 0.0;
    return c;
}

template <class K>
void allow_lds(K kern, size_t bytes) {
    if (bytes > 65536) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Records a pair of events around one launch when timing is enabled.
struct ProfScope {
    pd_plan p;
    hipStream_t st;
    hipEvent_t a = nullptr;
    ProfScope(pd_plan p_, hipStream_t st_) : p(p_), st(st_) {
        if (p->prof && hipEventCreate(&a) == hipSuccess) (void)hipEventRecord(a, st);
    }
    void done(const char* name, double bytes) {
        if (!p->prof || !a) return;
        hipEvent_t b;
        if (hipEventCreate(&b) != hipSuccess) return;
        (void)hipEventRecord(b, st);
        ProfRec r;
        std::snprintf(r.name, sizeof(r.name), "%s", name);
        r.a = a;
        r.b = b;
        r.bytes = bytes;
        p->prof->push_back(r);
        a = nullptr;
    }
};

constexpr int kCgBlocks = 1024;   // most blocks of a CG vector kernel

// p->red[0 .. nr) = the sums of the blocks' partials; or, for a single sum
// whose reader forms it itself (p->raw_sum), no launch.  Beyond 4096 partials
// a reader of kCgBlocks blocks would spend more on them than the launch
// takes: 32 MB from the L2s, ~4 us.
inline pd_status finish_reduction(pd_plan p, long nblk, int nr, hipStream_t st) {
    if (p->raw_sum && nr == 1 && nblk <= 4096) {
        p->sum = {p->partials, nblk};
        return PD_OK;
    }
    p->sum = {p->red, 1};
    if (nr < 1 || nr > pdk::kReduceThreads || (nr & (nr - 1)) != 0) return PD_EINVAL;
    hipLaunchKernelGGL(pdk::k_reduce_final, dim3(1), dim3(pdk::kReduceThreads), 0, st, p->partials, nblk, nr, p->red,
                       (double*)nullptr);
    return pdh::check(hipGetLastError());
}

}  // namespace pdi
