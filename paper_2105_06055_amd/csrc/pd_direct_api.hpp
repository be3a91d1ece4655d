// pd_direct_api.hpp -- what the chains and solvers call of the direct
// horizon sums (internal; the kernels are in pd_direct.hpp and compiled by
// pd_direct.hip).
#pragma once

#include "pd_plan.hpp"

namespace pdd {

// Whether the calls of a plan run the direct sums: the default kernel choice,
// and a plan that qualifies (dir_plan).
inline bool on(pd_plan p) { return p->dir_mt > 0 && p->lastaxis == PD_LASTAXIS_AUTO; }

// Whether the unweighted linear operator (force without W, Verlet, solves) runs
// them: plans whose bond sums cost less than its transforms (dir_plan).
inline bool linear_on(pd_plan p) { return on(p) && p->dir_linear; }

// Launch shapes of a qualifying plan (dir_blocks).
void dir_launch_shape(pd_plan p);

// Fields of one evaluation.  mode 0: L (and W where it is not null);
// mode 1: Verlet velocity update, F' = L + b, v <- chi_O [v + c1 (F + F')];
// vh_in: v holds the half-step velocity v + c1 F and F is not read; vh_out: v
// receives v' + c1 F' and F is not written; next: the next step's position
// update (position_update, with v' and F', or with the half-step
// velocity and no F) goes to u_next (not u: other blocks still read it), and
// the next integrity lam && W <= Wc to lam_next; mode 2: L = -chi_O L and
// red[0] = u . L; mode 3: L = chi_O (L + b) and red[0] = |L|^2.  energy:
// red[0 .. 3] = the energy sums of mode 1.
template <class T>
struct Eval {
    int mode;
    const T* u;
    const T* theta;        // LPS: chi theta (written by dir3_theta)
    const uint8_t* lam;    // 2D weights: integrity, or
    const T* s;            // micromodulus scale, or neither
    T* L; T* W;
    T* v; T* F; const T* b; const T* w;
    T c1, c2, dt, rho;
    int vh_in, vh_out, next, energy;
    T* u_next; uint8_t* lam_next;
    T Wc;
    int fail;
    double* nanflag;
};

// LPS dilatation theta of u (3D).
template <class T>
pd_status dir3_theta(pd_plan p, const T* u, T* theta, hipStream_t st);
// Force sums and epilogue, 3D (LPS or unweighted bond-based; e.theta for LPS).
template <class T>
pd_status dir3_force(pd_plan p, const Eval<T>& e, hipStream_t st);
// Force and energy sums and epilogue of the 2D bond-based plate.
template <class T>
pd_status dir2_force(pd_plan p, const Eval<T>& e, hipStream_t st);
// Nonlinear bond-based force, 2D and 3D; 3D up to three spacings.
template <class T>
pd_status dir_nbb(pd_plan p, const T* u, T* L, hipStream_t st);
inline bool nbb_on(pd_plan p) { return on(p) && (p->dim == 2 || p->dir_mt <= 3); }

// 2D adjoint: u_bar = L_phi g and w_bar = wscale * dL/ds . g (accumulated
// where acc), u the sum of u and u2 (u2 may be null); either result may be
// null.
template <class T>
pd_status dir2_adjoint(pd_plan p, const T* u, const T* u2, const T* s, const T* g, T* ubar, T* wbar, T wscale,
                       int acc, hipStream_t st);
// 2D Verlet reverse step (pd_verlet_adjoint) in two launches; ut and tmp are
// vector scratch.
template <class T>
pd_status dir2_verlet_adjoint(pd_plan p, const T* un, const T* unp1, const T* s, T* ub, T* vb, T* sb, T* bb, T c1,
                              T c2, T dt, T* ut, T* tmp, hipStream_t st);
// 2D damage index.
template <class T>
pd_status dir2_damage(pd_plan p, const uint8_t* lam, T* d, hipStream_t st);

// Position update u' = chi_O [u + dt v + c2 F] + (1 - chi_O) w and, with
// lam, lam' = lam && W <= Wc, element by element; u' may be u and lam' lam.
template <class T>
pd_status dir_drift(pd_plan p, const T* u, T* u_out, const T* v, const T* F, const T* w, T dt, T c2,
                    const uint8_t* lam, uint8_t* lam_out, const T* W, T Wc, int fail, hipStream_t st);

}  // namespace pdd
