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
// the move of that copy into the scalar block.  Returns whether the solver is running; branch: the choice, 0 if it is to
// be read from the scalar block.  (The ring kernel, whose registers are counted, has this in line.)
__device__ __forceinline__ bool pass_start(const APassArgs& a, Scal* __restrict__ scal, int& branch) {
    const int tid = threadIdx.x;
    const int status = a.check_status ? (a.scal_next ? a.scal_next : scal)->status : LBFGSB_RUNNING;
    constexpr int kScalWords = (int)(sizeof(Scal) / 4), kPerLane = (kScalWords + 63) / 64;
    const bool mover = a.scal_next && blockIdx.x == 0 && tid < 64;
    int moved[kPerLane];
    int fresh = 0;
    if (mover) {
        fresh = a.scal_next->fresh;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const int idx = tid + 64 * j;
            moved[j] = idx < kScalWords ? reinterpret_cast<const int*>(a.scal_next)[idx] : 0;
        }
    }
    branch = 0;
    DirChoice ch{};
    const bool own_choice = a.select_p && a.dir_blocks > 0;
    if (own_choice) ch = dir_choice_from_partials(a.dir_part, a.dir_blocks, a.eps);
    if (mover && fresh) {
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const int idx = tid + 64 * j;
            int v = moved[j];
            auto put_double = [&](size_t off, double val) {
                if (idx == (int)(off / 4)) v = __double2loint(val);
                if (idx == (int)(off / 4) + 1) v = __double2hiint(val);
            };
            if (own_choice && status == LBFGSB_RUNNING) {
                if (idx == (int)(offsetof(Scal, branch) / 4)) v = ch.branch;
                put_double(offsetof(Scal, gp), ch.gp);
                put_double(offsetof(Scal, alpha_ub), ch.alpha_ub);
                put_double(offsetof(Scal, pp), ch.pp);
                put_double(offsetof(Scal, xp), ch.xp);
            }
            if (idx == (int)(offsetof(Scal, fresh) / 4)) v = 0;
            if (idx < kScalWords) reinterpret_cast<int*>(scal)[idx] = v;
        }
        if (tid == 0) a.scal_next->fresh = 0;
    }
    if (status != LBFGSB_RUNNING) return false;
    if (own_choice) {
        branch = ch.branch;
        if (blockIdx.x == 0 && tid == 0 && !(a.scal_next && fresh)) {
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
