// t = K v for a symmetric matrix from its upper triangle: the row products of the quadratic-form kind.
//
// The matrix is all an iteration of that kind reads, and half of it says everything: K_rc (r <= c) contributes K_rc v_c to
// t_r and K_rc v_r to t_c.  The columns are cut into strips of 512; a wave takes tiles of 8 rows of a strip (64 lanes with
// 8 columns each, one row per set of registers, as the kernel for narrow rows with 64 lanes to a row), adds the rows'
// partial products over its lanes and keeps the columns' sums in registers.  Unlike there the rows' weights v_r are known
// beforehand, so both products are taken as a row arrives and its registers are refilled at once.  Strip J has rows
// 0 .. 512 (J + 1) - 1; its workgroups take a share of the grid in proportion.  Left behind are the strips' row sums
// (tpart[J][r], r in strip J or above) and each workgroup's 512 column sums (wpart); a second kernel adds a column's few
// dozen numbers in fixed order and forms v^T t from the finished t, whose rounding does not depend on the split.
//
// Sums are kept short on purpose -- a tile's eight rows for the columns, then the tiles, then in pairs -- where one chain per
// column over all of a wave's rows and one over the partial numbers would do.  Error of t against 80 bits in units of 2^-53
// (kernel matrices of 4608 / 10 000 points, vectors of one sign): one chain 1.08 / 1.09, now 0.68 / 0.69, the ring kernel on
// the whole matrix 0.88 / 0.84, the two-pass kernel 0.76 / 0.80.  The time is the same.
//
// Bytes: the blocks on the diagonal are read whole, n^2/2 + 256 n entries.  Per pass at n = 10 000 fp64: 131 us with the
// ring kernel reading all of K, 70 + 5 us with these two (0.42 GB: 6.0 TB/s, with k_sym_finish 5.5).
#include "common.h"
#include "narrow.h"

namespace lb {

namespace {

constexpr int kSymGridMax = 512;    // two workgroups per compute unit
constexpr int64_t kSymMinN = 4096;

// first workgroup of strip J
__host__ __device__ inline int sym_first_block(int J, int strips, int grid) {
    return (int)((int64_t)grid * J * (J + 1) / ((int64_t)strips * (strips + 1)));
}

// rows of the strip's tiles below the diagonal block use every element; DIAG: elements left of the diagonal count zero,
// and the diagonal itself only in the row's sum
template <typename T, bool DIAG, int S, int KC, int VEC>
__device__ __forceinline__ void sym_row(const typename ring::Raw<T>::type (&raw)[KC], const double (&v)[KC * VEC], double vr,
                                        const int (&col)[KC], int row, double& acc, double (&w)[KC * VEC]) {
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        double e[VEC];
        ring::widen(raw[k], e);
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            double up = e[i], off = e[i];
            if (DIAG) {
                const int c = col[k] + i;
                up = c >= row ? up : 0.0;
                off = c > row ? off : 0.0;
            }
            sum = fma(up, v[k * VEC + i], sum);
            w[k * VEC + i] = fma(off, vr, w[k * VEC + i]);
        }
    }
    acc = sum;
}

template <typename T>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
void k_sym(const T* __restrict__ A, int64_t ld, int n, APassArgs a, int strips, int grid, Scal* __restrict__ scal,
           double* __restrict__ wpart, double* __restrict__ tpart) {
    using RawT = typename ring::Raw<T>::type;
    using MemT = typename ring::RawMem<T, true>::type;
    constexpr int VEC = 16 / sizeof(T), KC = kSymStrip / 64 / VEC, S = 8, W = KC * VEC;
    __shared__ double wsum[kWaves][kSymStrip];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.x;
    int J = 0;
    while (J + 1 < strips && sym_first_block(J + 1, strips, grid) <= b) ++J;
    const int b0 = sym_first_block(J, strips, grid), nb = sym_first_block(J + 1, strips, grid) - b0;
    const int rows = (J + 1) * kSymStrip < n ? (J + 1) * kSymStrip : n;
    const int ntiles = (rows + S - 1) / S, stride = nb * kWaves;
    int tile = (b - b0) * kWaves + wave;
    const int full = n - n % VEC;
    int col[KC];                                             // first column of each of this lane's loads
    unsigned off[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const int p = J * kSymStrip + (k * 64 + lane) * VEC;
        col[k] = p < n - VEC ? p : n - VEC;                  // (past the end, or partly there: the row's last 16 bytes)
        off[k] = (unsigned)col[k] * (unsigned)sizeof(T);
    }
    RawT raw[S][KC];
    auto fetch = [&](RawT (&dst)[KC], int tl, int s) {
        const int r = tl * S + s < rows ? tl * S + s : rows - 1;
        const char* rp = reinterpret_cast<const char*>(A + (int64_t)r * ld);   // uniform
#pragma unroll
        for (int k = 0; k < KC; ++k) dst[k] = __builtin_nontemporal_load(reinterpret_cast<const MemT*>(rp + off[k]));
    };
    PassStart ps;
    pass_request(a, scal, a.select_p && a.dir_blocks > 0, ps);
    if (!pass_decide(a, scal, ps)) return;
    {
        const int t0 = tile < ntiles ? tile : 0;
#pragma unroll
        for (int s = 0; s < S; ++s) fetch(raw[s], t0, s);
    }
    const double *va, *vb;
    resolve_v(a, scal, n, va, vb, ps.branch);
    double v[W], w[W];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const int p = J * kSymStrip + (k * 64 + lane) * VEC + i;
            const int c = col[k] + i;
            const bool own = p < full || (p < full + VEC && full < n && c >= full);
            v[k * VEC + i] = own ? va[c] * (a.vs ? a.vs[c] : 1.0) : 0.0;
            w[k * VEC + i] = 0.0;
        }
    }
    // the rows' entries of v, eight lanes at a time, one tile ahead
    auto row_v = [&](int tl) -> double {
        const int r = tl * S + (lane & 7);
        const int rc = r < rows ? r : rows - 1;
        const double x = va[rc] * (a.vs ? a.vs[rc] : 1.0);
        return r < rows ? x : 0.0;                           // (a row past the end adds nothing to the columns)
    };
    double vrl = row_v(tile < ntiles ? tile : 0);
    for (; tile < ntiles; tile += stride) {
        const int tn = tile + stride < ntiles ? tile + stride : 0;
        const double vn = row_v(tn);
        double acc[S], wt[W];
        const bool diag = tile * S + S > J * kSymStrip;      // (uniform)
#pragma unroll
        for (int q = 0; q < W; ++q) wt[q] = 0.0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const double vr = lane_bcast(vrl, s);
            if (diag) sym_row<T, true, S, KC, VEC>(raw[s], v, vr, col, tile * S + s, acc[s], wt);
            else sym_row<T, false, S, KC, VEC>(raw[s], v, vr, col, tile * S + s, acc[s], wt);
            __builtin_amdgcn_sched_barrier(0);
            fetch(raw[s], tn, s);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = 0; q < W; ++q) w[q] += wt[q];
        const double u = narrow::row_sums<64, S>(acc, lane);
        if (lane < S && tile * S + lane < rows) tpart[(int64_t)J * n + tile * S + lane] = u;
        vrl = vn;
    }
#pragma unroll
    for (int q = 0; q < W; ++q) wsum[wave][q * 64 + lane] = w[q];
    __syncthreads();
    for (int q = tid; q < kSymStrip; q += kBlock) {
        const int i = (q / 64) % VEC, k = q / 64 / VEC, ln = q % 64;
        const int p = J * kSymStrip + (k * 64 + ln) * VEC + i;
        const int c = p < full ? p : n - VEC + (p - full);
        if (p < full || (p < full + VEC && full < n && c >= full)) {
            double s = wsum[0][q];
#pragma unroll
            for (int x = 1; x < kWaves; ++x) s += wsum[x][q];
            wpart[(int64_t)b * kSymStrip + (c - J * kSymStrip)] = s;
        }
    }
}

// t_c: its workgroups' column sums, then the row sums of strips J and above; out (row or t) and the partials of v^T t.
__global__ __launch_bounds__(kBlock) void k_sym_finish(int64_t n, APassArgs a, int strips, int grid, const Scal* __restrict__ scal,
                                                       const double* __restrict__ wpart, const double* __restrict__ tpart,
                                                       double* __restrict__ out, double* __restrict__ losspart) {
    __shared__ double lds[kBlock];
    if (a.check_status && scal->status != LBFGSB_RUNNING) return;
    const double *va, *vb;
    resolve_v(a, scal, n, va, vb);
    const int tid = threadIdx.x, cx = tid % kCX, gy = tid / kCX;
    const int64_t c = (int64_t)blockIdx.x * kCX + cx;
    const int64_t cc = c < n ? c : n - 1;
    const double vc = va[cc] * (a.vs ? a.vs[cc] : 1.0);
    const int J = (int)(cc / kSymStrip);                     // (the same for the kCX columns of a workgroup)
    const int b0 = sym_first_block(J, strips, grid), nw = sym_first_block(J + 1, strips, grid) - b0;
    const int count = nw + strips - J;
    double s = 0.0;
    for (int k0 = gy; k0 < count; k0 += kGY * 4) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int kk = k0 + kGY * k;
            v[k] = kk < nw ? wpart[(int64_t)(b0 + kk) * kSymStrip + cc % kSymStrip]
                           : (kk < count ? tpart[(int64_t)(J + kk - nw) * n + cc] : 0.0);
        }
        s += (v[0] + v[1]) + (v[2] + v[3]);
    }
    lds[gy * kCX + cx] = s;
    __syncthreads();
    if (tid < 64) {
        double tot = 0.0;
        if (gy == 0) {
            double p[kGY];
#pragma unroll
            for (int k = 0; k < kGY; ++k) p[k] = lds[k * kCX + cx];
#pragma unroll
            for (int h = kGY / 2; h > 0; h /= 2)
#pragma unroll
                for (int k = 0; k < h; ++k) p[k] += p[k + h];
            tot = p[0];
            if (c < n) out[c] = tot;
        }
        const double loss = wave_sum(gy == 0 && c < n ? (a.mode == kRowQpEval ? 0.5 : 1.0) * vc * tot : 0.0);
        if (tid == 0) losspart[blockIdx.x] = loss;
    }
}

}  // namespace

// From kSymMinN columns on, while every strip gets a workgroup of the grid.  Below, most of the matrix is served by the
// caches and the second launch eats the gain.  Whole iterations, ring kernel / these two, us: n = 1024 31 / 34, 2000
// 38 / 36, 3000 47 / 42, 4000 51 / 50, 5000 68 / 53, 7000 92 / 70, 10 000 154 / 100, 15 000 307 / 183 (fp64); 5000 55 / 44,
// 10 000 97 / 70 (fp32).
bool sym_shape_ok(const Dims& dm, int* strips, int* grid) {
    *strips = *grid = 0;
    if (dm.kind != LBFGSB_OBJ_QP || dm.cols < kSymMinN || dm.ld > (int64_t)1 << 28) return false;
    const int64_t nj = (dm.cols + kSymStrip - 1) / kSymStrip, least = nj * (nj + 1) / 2;
    if (least > kSymGridMax) return false;
    const int64_t tiles = least * (kSymStrip / 8), want = (tiles + kWaves - 1) / kWaves;
    *strips = (int)nj;
    *grid = (int)(want < kSymGridMax ? want : kSymGridMax);
    return true;
}

int sym_loss_parts(const Dims& dm) { return (int)((dm.cols + kCX - 1) / kCX); }

void launch_sym(const Dims& dm, const Geometry& ge, const Buffers& bf, const APassArgs& a, hipStream_t st, hipEvent_t ev0,
                hipEvent_t ev1) {
    double* tpart = bf.wpart + (size_t)ge.fused_blocks * kSymStrip;
    if (dm.dtype == LBFGSB_F32)
        hipExtLaunchKernelGGL(k_sym<float>, dim3(ge.fused_blocks), dim3(kBlock), 0, st, ev0, nullptr, 0, (const float*)a.A, dm.ld,
                              (int)dm.cols, a, ge.sym_strips, ge.fused_blocks, bf.scal, bf.wpart, tpart);
    else
        hipExtLaunchKernelGGL(k_sym<double>, dim3(ge.fused_blocks), dim3(kBlock), 0, st, ev0, nullptr, 0, (const double*)a.A, dm.ld,
                              (int)dm.cols, a, ge.sym_strips, ge.fused_blocks, bf.scal, bf.wpart, tpart);
    hipExtLaunchKernelGGL(k_sym_finish, dim3(sym_loss_parts(dm)), dim3(kBlock), 0, st, nullptr, ev1, 0, dm.cols, a, ge.sym_strips, ge.fused_blocks,
                       (const Scal*)bf.scal, (const double*)bf.wpart, (const double*)tpart,
                       a.mode == kRowQpEval ? bf.row : bf.t, bf.losspart);
}

}  // namespace lb
