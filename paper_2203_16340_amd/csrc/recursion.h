// Algorithm 3 (modified two-loop recursion, appendix) carried out on coefficients: shared by the Gram kernels
// (last workgroup) and the single-workgroup resident solver.
#pragma once

#include "common.h"

namespace lb {

// value of v in lane l (l uniform across the wave): a scalar-register read, not a trip through LDS
__device__ __forceinline__ double lane_value(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// ||y^i||^2 of the stored pairs for the lane that will own pair i in the recursion (lane i of wave 0).  It does not
// depend on anything the calling kernel computes, so the kernels fetch it when they start, long before it is used.
__device__ __forceinline__ double prefetch_ynorm2(const Scal* __restrict__ scal, int c, int head, int m) {
    const int tid = threadIdx.x;
    return (tid < 64 && tid < c) ? scal->ynorm2[ring_back(head, c - tid, m)] : 1.0;
}

// The recursion for at most K pairs.  Every entry of G a lane needs is fetched at once; the three loops then run on registers
// and scalar-register broadcasts only.  Row i is scaled by 1/rho_i beforehand, and is zero where it has no say (pairs that fail
// the gate; in the first loop pairs older than k, in the second newer ones), so a step of the chain is one broadcast and one
// multiply-add, and a lane's value stays what it was at its own step.  All K steps are taken whatever c is, and the lanes past
// the last pair read the last pair's rows: alpha is zero there, which makes the surplus steps add nothing, while a test per
// step or load cost a branch each (a step took 130 cycles and not 25).
template <int K>
__device__ __forceinline__ void recursion_in_registers(const double* G, int Vp, int c, int i, int ic, bool pass,
                                                       unsigned long long pm, double inv, double rho_yn, double& alpha_i,
                                                       double& coef_s, double& gamma) {
    double gsy[K], gyy[K], gys[K];
    const double *srow = G + ic * Vp, *yrow = G + (c + ic) * Vp;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int kc = k < c ? k : (c > 0 ? c - 1 : 0);       // (uniform)
        gsy[k] = srow[c + kc];                                // <s_i, y_k>
        gyy[k] = yrow[c + kc];                                // <y_i, y_k>
        gys[k] = yrow[kc];                                    // <y_i, s_k>
    }
    const double sg = srow[2 * c];                            // <s_i, g>
    double tsum = yrow[2 * c], tsum2 = 0.0;                   // <y_i, g>
#pragma unroll
    for (int k = 0; k < K; ++k) {
        gsy[k] = pass && k > i ? gsy[k] * inv : 0.0;
        gys[k] = pass && k < i ? gys[k] * inv : 0.0;
    }
    double alpha = pass ? sg * inv : 0.0;
#pragma unroll
    for (int k = K - 1; k >= 0; --k) alpha = fma(-lane_value(alpha, k), gsy[k], alpha);
    if (c > 0 && ((pm >> (c - 1)) & 1ull)) gamma = lane_value(rho_yn, c - 1);
#pragma unroll
    for (int k = 0; k < K; k += 2) {
        tsum = fma(-lane_value(alpha, k), gyy[k], tsum);
        if (k + 1 < K) tsum2 = fma(-lane_value(alpha, k + 1), gyy[k + 1], tsum2);
    }
    double coef = pass ? alpha - gamma * (tsum + tsum2) * inv : 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) coef = fma(-lane_value(coef, k), gys[k], coef);
    alpha_i = alpha;
    coef_s = coef;
}

// The same for more pairs, whose triangular solves are longer: the rows stay as they are and each step divides by rho itself, so
// that an entry is rounded once (scaled rows add a rounding to each; the sums are those of the loops in memory, bit for bit).
template <int K>
__device__ __forceinline__ void recursion_in_registers_unscaled(const double* G, int Vp, int c, int i, int ic, bool pass,
                                                                unsigned long long pm, double inv, double rho_yn, double& alpha_i,
                                                                double& coef_s, double& gamma) {
    double gsy[K], gyy[K], gys[K];
    const double *srow = G + ic * Vp, *yrow = G + (c + ic) * Vp;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int kc = k < c ? k : (c > 0 ? c - 1 : 0);       // (uniform)
        gsy[k] = srow[c + kc];                                // <s_i, y_k>
        gyy[k] = yrow[c + kc];                                // <y_i, y_k>
        gys[k] = yrow[kc];                                    // <y_i, s_k>
    }
    const double inv_p = pass ? inv : 0.0;
    double part = pass ? srow[2 * c] : 0.0;                   // <s_i, g>
    double tsum = yrow[2 * c];                                // <y_i, g>
#pragma unroll
    for (int k = 0; k < K; ++k) {
        gsy[k] = pass && k > i ? gsy[k] : 0.0;
        gys[k] = pass && k < i ? gys[k] : 0.0;
    }
#pragma unroll
    for (int k = K - 1; k >= 0; --k) part = fma(-lane_value(part * inv_p, k), gsy[k], part);
    const double alpha = part * inv_p;
    if (c > 0 && ((pm >> (c - 1)) & 1ull)) gamma = lane_value(rho_yn, c - 1);
#pragma unroll
    for (int k = 0; k < K; ++k) tsum = fma(-lane_value(alpha, k), gyy[k], tsum);
    double by = pass ? gamma * tsum : 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) by = fma(lane_value(fma(-by, inv_p, alpha), k), gys[k], by);
    alpha_i = alpha;
    coef_s = fma(-by, inv_p, alpha);
}

// The recursion of Algorithm 3 on coefficients, by one wave (threads 0..63) of the calling workgroup, and the stopping test by
// another (which reads and writes other fields of the scalar block): called by all threads, at least 128, with a barrier before
// anybody reads either's results.  G: Vp x Vp (LDS), row-major, vectors ordered s^0..s^{c-1}, y^0..y^{c-1}, g.  gg = sum g[S]^2, pginf = max KKT residual, nfixed = #fixed,
// ynew = ||y_new||^2 (full vector), yn_old = prefetch_ynorm2().
// MAXK: up to this many pairs the recursion keeps its rows of G in registers (three numbers each), beyond it reads LDS in its
// steps (20 pairs, n = 350, 50 steps of the one-workgroup kernel: 1533 -> 1418 us with the registers).
template <int MAXK>
__device__ __forceinline__ void recursion_on_coefficients(const double* G, int Vp, int c, int head, int m, const Opts& op,
                                                          Scal* __restrict__ scal, double gg, double pginf, double nfixed,
                                                          double ynew, double yn_old, double* alpha_s, int dbg_inputs,
                                                          int evaluate_stop) {
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 64) {
        const int i = lane;   // lane i owns pair i (oldest = 0)
        // (the same in every lane: from here on in a scalar register, so that the loops below are branches and not masks)
        c = __builtin_amdgcn_readfirstlane(c);
        Vp = __builtin_amdgcn_readfirstlane(Vp);
        // lanes past the last pair work on the last pair's rows and are left out by `pass`: no access is predicated
        const int ic = i < c ? i : (c > 0 ? c - 1 : 0);
        double rho = 1.0, yn = 1.0;
        if (c > 0) {
            rho = G[ic * Vp + (c + ic)];
            // the newest pair's norm was just summed (and stored for later iterations)
            yn = (i == c - 1 && !dbg_inputs) ? ynew : yn_old;
        }
        const bool pass = i < c && rho > op.eps * yn;
        const double inv = 1.0 / rho, rho_yn = rho / yn;
        const unsigned long long pm = __ballot(pass);
        double alpha_i = 0.0, coef_s = 0.0, gamma = 1.0;
        if (c <= 5) {
            recursion_in_registers<5>(G, Vp, c, i, ic, pass, pm, inv, rho_yn, alpha_i, coef_s, gamma);
        } else if (c <= 10) {
            recursion_in_registers<10>(G, Vp, c, i, ic, pass, pm, inv, rho_yn, alpha_i, coef_s, gamma);
        } else if (MAXK > 10 && c <= MAXK) {
            recursion_in_registers_unscaled<MAXK>(G, Vp, c, i, ic, pass, pm, inv, rho_yn, alpha_i, coef_s, gamma);
        } else {
            // first loop: alpha_k, newest to oldest.  Steps of pairs that fail the gate run with alpha_k = 0;
            // a lane's row is dead once its own alpha has been taken, so updating it further is harmless.
            double part_s = i < c ? G[i * Vp + 2 * c] : 0.0;   // <s_i, g>
#pragma unroll 4
            for (int k = c - 1; k >= 0; --k) {
                const double gsy = i < c ? G[i * Vp + (c + k)] : 0.0;   // <s_i, y_k>
                double ak = lane_value(part_s * inv, k);
                if (!((pm >> k) & 1ull)) ak = 0.0;
                if (i == k) alpha_i = ak;
                part_s = fma(-ak, gsy, part_s);
            }
            if (i < c) alpha_s[i] = alpha_i;
            if (c > 0 && ((pm >> (c - 1)) & 1ull)) gamma = lane_value(rho_yn, c - 1);
            // <y_i, gamma (g - sum_k alpha_k y_k)>
            double by = 0.0;
            {
                double tsum = i < c ? G[(c + i) * Vp + 2 * c] : 0.0;
#pragma unroll 4
                for (int k = 0; k < c; ++k) {
                    const double gyy = i < c ? G[(c + i) * Vp + (c + k)] : 0.0;
                    tsum = fma(-alpha_s[k], gyy, tsum);
                }
                by = gamma * tsum;
            }
            // second loop: alpha_k - beta_k, oldest to newest
#pragma unroll 4
            for (int k = 0; k < c; ++k) {
                const double gys = i < c ? G[(c + i) * Vp + k] : 0.0;   // <y_i, s_k>
                double ck = lane_value(alpha_i - by * inv, k);
                if (!((pm >> k) & 1ull)) ck = 0.0;
                if (i == k) coef_s = ck;
                if (i > k) by = fma(ck, gys, by);
            }
        }
        if (i < c) {
            scal->delta[i] = coef_s;
            scal->delta[c + i] = -gamma * alpha_i;
        }
        if (lane == 0) {
            scal->delta[2 * c] = gamma;
            scal->pairs_used = __popcll(pm);
        }
    } else if (tid == 64 && evaluate_stop) {
        // the stopping test, by the second wave meanwhile
        stopping_test(scal, op, gg, pginf, nfixed);
    }
}

}  // namespace lb
