// Pieces shared by the two organisations of the A pass: 16-byte loads widened to fp64, the choice
// of the vector A multiplies, and the objective's per-row operation.
#pragma once

#include <cstddef>

#include "common.h"

namespace lb {

template <typename T, int VEC>
struct Loader;
template <>
struct Loader<float, 4> {
    static __device__ __forceinline__ void load(const float* p, double (&o)[4]) {
        const float4 v = *reinterpret_cast<const float4*>(p);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
};
template <>
struct Loader<double, 2> {
    static __device__ __forceinline__ void load(const double* p, double (&o)[2]) {
        const double2 v = *reinterpret_cast<const double2*>(p);
        o[0] = v.x; o[1] = v.y;
    }
};
template <typename T>
struct Loader<T, 1> {
    static __device__ __forceinline__ void load(const T* p, double (&o)[1]) { o[0] = (double)*p; }
};

// Resolves the vector A multiplies: either fixed pointers, or the direction Algorithm 2 selected.
// branch: Algorithm 2's choice when the caller has made it itself (0: read it from the scalar block)
__device__ __forceinline__ void resolve_v(const APassArgs& a, const Scal* scal, int64_t cols, const double*& va,
                                          const double*& vb, int branch = 0) {
    va = a.va;
    vb = a.vb;
    if (a.select_p) {
        va = (branch ? branch : scal->branch) == 1 ? a.p1 : a.p2;
        vb = a.split ? va + cols : nullptr;
    }
}

// What a pass over A does before anything else: the status word (from the copy of the scalar block the direction kernel
// left in a.scal_next, when there is one), Algorithm 2's choice between the candidate directions from that kernel's partial
// sums (every wave of every workgroup gets the same bits; workgroup 0 records it), and, by the first wave of workgroup 0,
// the move of that copy into the scalar block.  In two parts, so that a pass may request its rows in between: loads return
// in the order they were issued, and these few come first.  At most kPassDirBlocksMax records of
// partial sums, one per lane.  (The ring
// kernel, whose registers are counted and whose rows are wider, has this in line.)
struct PassStart {
    static constexpr int kWords = (int)(sizeof(Scal) / 4), kPerLane = (kWords + 63) / 64;
    int status, fresh, branch;
    int moved[kPerLane];
    double alpha_ub;
    double rec[7];
    bool mover, own_choice;
};
// own_choice: the choice is made here (a.dir_part), not read from the scalar block
__device__ __forceinline__ void pass_request(const APassArgs& a, const Scal* scal, bool own_choice, PassStart& ps) {
    const int tid = threadIdx.x, lane = tid & 63;
    const Scal* src = a.scal_next ? a.scal_next : scal;
    ps.status = a.check_status ? src->status : LBFGSB_RUNNING;
    ps.mover = a.scal_next && blockIdx.x == 0 && tid < 64;
    ps.own_choice = own_choice;
    ps.fresh = 0;
    ps.branch = 0;
    ps.alpha_ub = 1.0;
    if (own_choice) {
        const double* r = a.dir_part + (int64_t)(lane < a.dir_blocks ? lane : 0) * kDirRed;
#pragma unroll
        for (int k = 0; k < 7; ++k) ps.rec[k] = r[k];
    }
    if (ps.mover) {
        ps.fresh = a.scal_next->fresh;
#pragma unroll
        for (int j = 0; j < PassStart::kPerLane; ++j) {
            const int idx = tid + 64 * j;
            ps.moved[j] = idx < PassStart::kWords ? reinterpret_cast<const int*>(a.scal_next)[idx] : 0;
        }
    }
}
// Returns whether the solver is running; ps.branch (0: it is to be read from the scalar block) and ps.alpha_ub are then
// the choice and its step bound.
__device__ __forceinline__ bool pass_decide(const APassArgs& a, Scal* scal, PassStart& ps) {
    const int tid = threadIdx.x;
    DirChoice ch{};
    if (ps.own_choice) ch = dir_choice_from_records((tid & 63) < a.dir_blocks, ps.rec, a.eps);
    if (ps.mover && ps.fresh) {
#pragma unroll
        for (int j = 0; j < PassStart::kPerLane; ++j) {
            const int idx = tid + 64 * j;
            int v = ps.moved[j];
            auto put_double = [&](size_t off, double val) {
                if (idx == (int)(off / 4)) v = __double2loint(val);
                if (idx == (int)(off / 4) + 1) v = __double2hiint(val);
            };
            if (ps.own_choice && ps.status == LBFGSB_RUNNING) {
                if (idx == (int)(offsetof(Scal, branch) / 4)) v = ch.branch;
                put_double(offsetof(Scal, gp), ch.gp);
                put_double(offsetof(Scal, alpha_ub), ch.alpha_ub);
                put_double(offsetof(Scal, pp), ch.pp);
                put_double(offsetof(Scal, xp), ch.xp);
            }
            if (idx == (int)(offsetof(Scal, fresh) / 4)) v = 0;
            if (idx < PassStart::kWords) reinterpret_cast<int*>(scal)[idx] = v;
        }
        if (tid == 0) a.scal_next->fresh = 0;
    }
    if (ps.status != LBFGSB_RUNNING) return false;
    if (ps.own_choice) {
        ps.branch = ch.branch;
        ps.alpha_ub = ch.alpha_ub;
        if (blockIdx.x == 0 && tid == 0 && !(a.scal_next && ps.fresh)) {
            scal->branch = ch.branch; scal->gp = ch.gp; scal->alpha_ub = ch.alpha_ub; scal->pp = ch.pp; scal->xp = ch.xp;
        }
    }
    return true;
}

// The objective's per-row operation on u = a_r . v.  Returns the row's loss contribution.
__device__ __forceinline__ double row_op(int mode, double u, int64_t r, int64_t rows, const double* __restrict__ b,
                                         const double* __restrict__ w, double* __restrict__ row,
                                         double* __restrict__ t, double* __restrict__ psi) {
    switch (mode) {
        case kRowLsqEval: {
            const double res = u - b[r];
            const double wr = w ? w[r] : 1.0;
            row[r] = res;
            psi[r] = wr * res;
            return 0.5 * wr * res * res;
        }
        case kRowDir: {
            const double wr = w ? w[r] : 1.0;
            t[r] = u;
            psi[r] = wr * u;
            return wr * u * u;
        }
        case kRowLogiEval: {
            const double y = b[r];
            const double a = -y * u;
            row[r] = u;
            psi[r] = -y * sigmoid_d(a) / (double)rows;
            return softplus_d(a) / (double)rows;
        }
        case kRowLogiDir:
            t[r] = u;
            return 0.0;
        default:
            return 0.0;   // the QP modes need the row's own entry of v: see k_gemv
    }
}

}  // namespace lb
