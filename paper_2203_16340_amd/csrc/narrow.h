// Single-read A pass for narrow rows (at most 64 KC 16-byte chunks): the waves own rows, not the workgroup.
//
// The ring kernel (fused_ring.h) gives a row to a whole workgroup, 16 bytes per thread and chunk: with 100 fp32 columns
// 25 of its 128 threads have anything to do, and every few rows end in a barrier.  Here L lanes (8 to 64) share a row
// with KC chunks each, a wave holds S (8 or 4) sets of 64/L rows in registers, and no wave waits for another before its
// last row:
//   * the accumulators of w of a lane's columns stay in its registers for the whole launch; v is in LDS and read once
//     per tile of S sets;
//   * the 8 partial dot products of a lane are added over the row's lanes all at once (each exchange halves the number
//     of values a lane carries), which leaves the row sums one per lane: the row operation -- one exponential and one
//     division, or the logarithms of the line search -- is evaluated for up to 64 different rows by one wave, not for
//     a few rows by every wave of a workgroup;
//   * the rows' weights psi come back to the row's lanes through LDS (a write and four 16-byte reads of one wave, in
//     order, no barrier), w is accumulated from the same registers, and a set is refilled with the wave's next rows as
//     soon as it has been used.
// What bounds it is the bytes in flight (8 waves per compute unit x S sets x KC kilobytes) and, for the logistic kinds,
// the transcendental functions.  Rows may start on any element and have any number of columns: a lane whose chunk is
// only partly there loads the row's last 16 bytes instead, with v zero for the columns that belong to its neighbour.
#pragma once

#include "fused_ring.h"

namespace lb {
namespace narrow {

// Sums of a[0..S) over the L lanes of a row: lane i returns the total of a[i % S].  Fixed order.
template <int L, int S>
__device__ __forceinline__ double row_sums(double (&a)[S], int lane) {
    static_assert((S == 8 && L >= 8) || (S == 4 && L == 64), "the sets used by the variants");
    if constexpr (S == 8) halve<4, kDppHalfMirror>(a, lane);   // i <-> 7 - i: flips bit 2 (and two in which nothing differs yet)
    halve<2, kDppXor2>(a, lane);
    halve<1, kDppXor1>(a, lane);
    double t = a[0];
    if constexpr (S == 4) t += __shfl_xor(t, 4);
    if constexpr (L >= 16) t += dpp_move<kDppRor8>(t);
    if constexpr (L >= 32) t += __shfl_xor(t, 16);
    if constexpr (L >= 64) t += __shfl_xor(t, 32);
    return t;
}

// LOGI: the family of row operations, as for the ring kernel (0 quadratic, 1 logistic, 2 logistic direction pass).
// mode kRowPsiGiven (LOGI 0): w = A^T psi for the weights the launch is given; nothing else is computed or stored.
// OWN: Algorithm 2's choice is made here, from the direction kernel's partial sums (direction passes only); else it is read
// from the scalar block.  (A parameter and not a test: with both in one kernel a pass behind k_small_step took 0.3 us longer.)
template <typename T, int L, int KC, int S, int LOGI, bool OWN, bool CACHED>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
void k_narrow(const T* __restrict__ A, int64_t ld, int64_t rows, int64_t cols, APassArgs a, Scal* __restrict__ scal,
              double* __restrict__ row, double* __restrict__ t, const double* __restrict__ psi_given,
              double* __restrict__ wpart, double* __restrict__ losspart) {
    using RawT = typename ring::Raw<T>::type;
    using MemT = typename ring::RawMem<T, true>::type;
    constexpr int VEC = 16 / sizeof(T);
    constexpr int GR = 64 / L;                               // rows per set
    constexpr int RT = S * GR;                           // rows per tile (one tile = what a wave holds)
    constexpr int W = KC * VEC;                              // columns per lane
    __shared__ __align__(16) double psi_s[kWaves * 64];
    __shared__ double wsum[kWaves][L * W];
    __shared__ double2 v_s[L * W / 2];                       // v: column pair q of the lane's W at [q * L + j]
    __shared__ double lsum[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane % L, g = lane / L;
    const int icols = (int)cols, full = icols - icols % VEC;
    const unsigned ldb = (unsigned)(ld * (int64_t)sizeof(T));

    // byte offsets of this lane's chunks from the first row of a set; chunks past the end read the row's last 16 bytes
    unsigned off[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int c = (k * L + j) * VEC;
        off[k] = (unsigned)g * ldb + (unsigned)(c < icols - VEC ? c : icols - VEC) * (unsigned)sizeof(T);
    }
    // (row numbers are 32-bit, tiles past the last one included: the addresses of a tile's sets take half the scalar
    // instructions that 64-bit rows did)
    const int irows = (int)rows, last = irows - GR;          // (rows >= GR)
    const int ntiles = (int)((rows + RT - 1) / RT);
    const int stride = (int)gridDim.x * kWaves;
    int tile = (int)blockIdx.x * kWaves + wave;
    RawT raw[S][KC];
    // No load is predicated (a refill under a test costs a second copy of the registers): a set that runs past the last
    // row reads the last GR rows instead, and its rows that belong to the set before it get weight zero.
    // The order of a tile's sets differs from wave to wave: where a tile is a power of two of bytes, waves that ran in
    // step would otherwise all read from the same few memory channels (0.4 GB of 1024 columns: fp64 70.4 -> 63.8 us a
    // pass, fp32 72.2 -> 65.5; 1000 columns 67.1 -> 64.4).
    const int rot = (int)(blockIdx.x * kWaves + wave) % S;
    auto set_base = [&](int r) -> int { return r < last ? r : last; };
    auto fetch = [&](RawT (&dst)[KC], int tl, int s) {
        const unsigned r = (unsigned)set_base(tl * RT + ((s + rot) % S) * GR);
        const char* rp = reinterpret_cast<const char*>(A) + (uint64_t)r * ldb;   // uniform
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            unsigned o = off[k];
            asm volatile("" : "+v"(o));                      // (opaque here: scalar base + 32-bit vector offset)
            if constexpr (CACHED) dst[k] = *reinterpret_cast<const MemT*>(rp + o);
            else dst[k] = __builtin_nontemporal_load(reinterpret_cast<const MemT*>(rp + o));
        }
    };
    // what the row operation reads, for the row whose sum this lane will hold
    const int mode = a.mode;
    const bool need_b = LOGI != 0 || mode == kRowLsqEval;
    const bool need_z = LOGI == 2 || mode == kRowPsiGiven;
    const double* zsrc = LOGI == 2 ? row : psi_given;
    const int sl = (((lane % S) + rot) % S) * GR;                          // this lane's set: its first row within the tile
    auto row_inputs = [&](int tl, double& b, double& z) {
        const unsigned r = (unsigned)(set_base(tl * RT + sl) + g);
        b = need_b ? a.b[r] : 0.0;
        z = need_z ? zsrc[r] : (a.w ? a.w[r] : 1.0);
    };

    // (the small reads first: loads return in the order they were issued)
    PassStart ps;
    int spec_ok = 0;
    if constexpr (OWN) {
        pass_request(a, scal, true, ps);
    } else {
        ps.status = a.check_status ? scal->status : LBFGSB_RUNNING;
        spec_ok = a.check_status == 2 ? scal->spec_ok : 0;
        ps.branch = scal->branch;
        ps.alpha_ub = scal->alpha_ub;
    }
    double bc = 0.0, zc = 1.0;
    {
        const int t0 = tile < ntiles ? tile : 0;
        row_inputs(t0, bc, zc);
#pragma unroll
        for (int s = 0; s < S; ++s) fetch(raw[s], t0, s);
    }
    if constexpr (OWN) {
        if (!pass_decide(a, scal, ps)) return;
    } else {
        if (ps.status != LBFGSB_RUNNING || spec_ok) return;
    }
    const double *va, *vb;
    resolve_v(a, scal, cols, va, vb, ps.branch);
    double w[W];
#pragma unroll
    for (int q = 0; q < W; ++q) w[q] = 0.0;
    for (int q = tid; q < L * W; q += kBlock) {
        const int i = (q & 1) + 2 * ((q / 2 / L) % (VEC / 2)), k = q / 2 / L / (VEC / 2), jj = q / 2 % L;
        const int p = (k * L + jj) * VEC + i;                // position; from `full` on: the ragged chunk
        const int c = p < full ? p : icols - VEC + (p - full);
        double x = 0.0;
        if ((p < full || (p < full + VEC && full < icols && c >= full)) && mode != kRowPsiGiven) {
            x = va[c];
            if (vb) x -= vb[c];
        }
        reinterpret_cast<double*>(v_s)[q] = x;
    }
    __syncthreads();
    const double alpha0 = LOGI == 2 ? fmin(1.0, ps.alpha_ub) : 0.0;   // first trial step of the line search
    const double invn = 1.0 / (double)rows;
    double loss = 0.0;
    // first trial step: rows whose loss difference is still to be taken, by the new margin, whose sigmoid is at hand:
    // softplus(q') - softplus(q' - dq)
    double lq = 0.0, ls = 0.5, ldq = 0.0;
    int pending = 0;

    for (; tile < ntiles; tile += stride) {
        double acc[S];
        // (v is read again for every tile, a chunk at a time: its registers go to the row operation)
        // (A chunk's products are added for themselves first.  In one chain over a lane's up to 24 columns the row sums of
        // Gaussian rows were off by 1.90 x 2^-53 at 1500 fp32 columns and 1.72 at 1000 fp64 ones; like this by 1.61 and 1.61,
        // the ring kernel's by 1.63 and 1.55.  The time is the same.)
        int vj = j;
        asm volatile("" : "+v"(vj));
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            double v[VEC];
#pragma unroll
            for (int i = 0; i < VEC; i += 2) {
                const double2 p2 = v_s[(k * VEC + i) / 2 * L + vj];
                v[i] = p2.x; v[i + 1] = p2.y;
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                double e[VEC];
                ring::widen(raw[s][k], e);
                double c = e[0] * v[0];
#pragma unroll
                for (int i = 1; i < VEC; ++i) c = fma(e[i], v[i], c);
                acc[s] = k == 0 ? c : acc[s] + c;
            }
        }
        const double u = row_sums<L, S>(acc, lane);
        const int r = set_base(tile * RT + sl) + g;
        const bool valid = r >= tile * RT + sl;
        const bool mine = valid && (L == S || j < S);        // (rows longer than S lanes: copies of the sums in the others)
        // the wave's next tile; behind its last one the first tile of all, which every wave then reads: from cache
        const int tn = tile + stride < ntiles ? tile + stride : 0;
        double bn, zn;
        row_inputs(tn, bn, zn);
        double psi, lo, keep, qn = 0.0, sn = 0.5;
        if (LOGI == 0 && mode == kRowPsiGiven) {
            psi = zc; lo = 0.0;
        } else {
            ring::row_eval<LOGI>(mode, u, bc, zc, alpha0, invn, psi, lo, keep, qn, sn);
            if (mine) {
                if (mode == kRowDir || mode == kRowLogiSpec) t[r] = keep; else row[r] = keep;
                loss += lo;
            }
        }
        if (!valid) psi = 0.0;
        if (LOGI == 2 && a.ls_first) {
            // softplus(-y (z + alpha0 t)) - softplus(-y z) of the rows, for as many rows at a time as the wave has lanes
            if (L == S || j / S == pending) {
                lq = valid ? qn : 0.0;                    // (no step: no contribution)
                ls = valid ? sn : 0.5;
                ldq = valid ? -bc * alpha0 * u : 0.0;
            }
            if (++pending == L / S) {
                loss -= softplus_diff(lq, ls, -ldq);
                pending = 0; ldq = 0.0;
            }
        }
        bc = bn; zc = zn;
        psi_s[wave * 64 + lane] = psi;
        __builtin_amdgcn_wave_barrier();
        double ps[S];
#pragma unroll
        for (int s = 0; s < S; s += 2) {
            const double2 p2 = *reinterpret_cast<const double2*>(&psi_s[wave * 64 + (lane & ~(S - 1)) + s]);
            ps[s] = p2.x; ps[s + 1] = p2.y;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = 0; s < S; ++s) {
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                ring::forget(raw[s][k]);                     // fp32: widened again rather than kept widened
                double e[VEC];
                ring::widen(raw[s][k], e);
#pragma unroll
                for (int i = 0; i < VEC; ++i) w[k * VEC + i] = fma(e[i], ps[s], w[k * VEC + i]);
            }
            __builtin_amdgcn_sched_barrier(0);
            fetch(raw[s], tn, s);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (LOGI == 2 && a.ls_first && pending > 0) loss -= softplus_diff(lq, ls, -ldq);

    // w over the wave's groups of lanes, then over the waves in wave order
#pragma unroll
    for (int q = 0; q < W; ++q) {
        if constexpr (L <= 8) w[q] += dpp_move<kDppRor8>(w[q]);
        if constexpr (L <= 16) w[q] += __shfl_xor(w[q], 16);
        if constexpr (L <= 32) w[q] += __shfl_xor(w[q], 32);
        if (g == 0) wsum[wave][q * L + j] = w[q];
    }
    loss = wave_sum(loss);
    if (lane == 0) lsum[wave] = loss;
    __syncthreads();
    for (int q = tid; q < L * W; q += kBlock) {
        const int i = (q / L) % VEC, k = q / L / VEC, jj = q % L;
        const int p = (k * L + jj) * VEC + i;
        const int c = p < full ? p : icols - VEC + (p - full);
        if (p < full || (p < full + VEC && full < icols && c >= full)) {
            double s = wsum[0][q];
#pragma unroll
            for (int x = 1; x < kWaves; ++x) s += wsum[x][q];
            wpart[(int64_t)blockIdx.x * cols + c] = s;
        }
    }
    if (tid == 0 && mode != kRowPsiGiven) {
        double s = lsum[0];
#pragma unroll
        for (int x = 1; x < kWaves; ++x) s += lsum[x];
        losspart[blockIdx.x] = s;
    }
}

}  // namespace narrow
}  // namespace lb
