// Free set (Eq. (ws)), masked Gram matrix of the stored pairs and the gradient, and the modified
// two-loop recursion (Algorithm 3) carried out on coefficients.
//
// Batched form of Algorithm 3.  Let b_0..b_{V-1} = s^0[S]..s^{c-1}[S], y^0[S]..y^{c-1}[S], g[S]
// (c stored pairs, oldest first, S the current free set) and G = B^T B.  Every vector the recursion
// forms is B*delta for some coefficient vector delta, and every dot product it needs is an entry of
// G*delta.  Written out, with rho_i = G[s_i][y_i], pass_i = rho_i > eps*||y^i||^2 (full norm):
//   first loop  (i = c-1 .. 0):  alpha_i = (G[s_i][g] - sum_{k>i} alpha_k G[s_i][y_k]) / rho_i
//   scaling:                     gamma = rho_{c-1}/||y^{c-1}||^2 if pass_{c-1}, else 1
//   second loop (i = 0 .. c-1):  beta_i = (gamma (G[y_i][g] - sum_k alpha_k G[y_i][y_k])
//                                          + sum_{k<i} (alpha_k - beta_k) G[y_i][s_k]) / rho_i
//   result:  q = gamma g - gamma sum_k alpha_k y_k + sum_k (alpha_k - beta_k) s_k,  d = -q on S
// (pairs that fail the gate have alpha = beta = 0).  Both loops are triangular solves; lane i of one
// wave owns row i, so a step is one broadcast and one multiply-add, with no cross-lane reduction.
// G must be rebuilt every iteration because S changes; it costs one pass over the 2c+1 vectors.
//
// (Steps on short vectors build it in small.hip.)
#include <cstddef>
#include <type_traits>

#include "common.h"
#include "gram_close.h"
#include "recursion.h"

namespace lb {

namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int64_t kGramLongN = 1 << 17;   // from here on one workgroup per compute unit and the two-level sum

// A kernel is made for M slots of the pair memory (m <= M).
constexpr int gram_tot_at(int M) { return (2 * M + 2) * (2 * M + 2); }    // G, then the totals
// Blocks of 16 slots (k_gram_blocks)
constexpr int gram_slots(int M) { return 2 * M + 1; }                     // y ring 0 .. M-1 | g M | s ring M+1 .. 2M
constexpr int gram_nb(int M) { return (gram_slots(M) + 15) / 16; }
// pairs of blocks (a <= b) that hold products the recursion reads: not those of two blocks of s vectors only (16 a > M)
constexpr int gram_na(int M) { return 1 + M / 16; }
constexpr int gram_np(int M) { return 2 * gram_nb(M) - 1; }
static_assert(gram_na(20) == 2 && gram_na(31) == 2, "the first two rows of blocks");
constexpr int kGramBlockWaves = 4;                                        // (LDS: 16 NB vectors of 64 elements per wave)
// A wave's 64 elements of every vector in LDS: doubles from one vector to the next, even and an odd multiple of two, so that
// 16 lanes that read 16 bytes each of 16 vectors touch every bank once
constexpr int kGramStride = 66;
// the waves' elements and a row of zeros each; then their blocks; then G (at most (2 M + 2)^2) and the totals
constexpr int gram_lds_doubles(int M, int waves) {
    const int elems = waves * (gram_slots(M) + 1) * kGramStride, blocks = waves * gram_np(M) * 256;
    return elems > blocks ? elems : blocks;
}
static_assert(gram_tot_at(20) + gram_entries(20) <= gram_lds_doubles(20, kGramBlockWaves) &&
              gram_tot_at(31) + gram_entries(31) <= gram_lds_doubles(31, kGramBlockWaves), "G and the totals fit");

// Every workgroup has written NE doubles at grampart + blockIdx.x * NE (entry 0 is a maximum, all others are
// sums).  The workgroups form at most kGramGroups groups of consecutive indices; the last workgroup of a group
// to finish adds the group's partials in index order into grampart + (gridDim.x + group) * NE, and the last
// group to finish adds the group results (HELD: those entries that `places` names), again in index order, into tot (LDS).  Returns true in that
// one workgroup (after a barrier), false everywhere else.  No workgroup reads more than kGramGroupMax partials,
// and the order of the additions does not depend on which workgroup finishes last.  Grids of at most
// kGramOneLevelMax workgroups skip the first level (each level costs an atomic and a dependent round of loads).  groups_only: the second level, and what follows it, is left to the direction kernel.
constexpr int kGramGroupMax = 16;   // workgroups per group at most: grids of up to kGramGroups * kGramGroupMax

template <int NT, bool HELD>
__device__ __forceinline__ bool reduce_partials(double* __restrict__ grampart, int NE, Scal* __restrict__ scal, int* flag,
                                                double* tot, bool groups_only, const GramPlaces& places) {
    const int tid = threadIdx.x, nwg = gridDim.x;
    if (nwg <= kGramOneLevelMax) {
        if (groups_only) return false;
        // few workgroups: one level, the last one to finish adds all partials in index order
        if (!arrive_is_last(&scal->gram_cnt[kGramGroups], flag, (unsigned)nwg)) return false;
        if constexpr (HELD) gram_sum_held<NT>(grampart, NE, nwg, tot, places);
        else gram_sum_partials_flat<NT>(grampart, NE, nwg, tot);
        __syncthreads();
        return true;
    }
    const int gs = (nwg + kGramGroups - 1) / kGramGroups;
    const int ngroups = (nwg + gs - 1) / gs;
    const int grp = blockIdx.x / gs, gfirst = grp * gs;
    const int gsize = nwg - gfirst < gs ? nwg - gfirst : gs;
    auto add = [&](int first, int count, int idx) -> double {
        double v[kGramGroupMax];
#pragma unroll
        for (int k = 0; k < kGramGroupMax; ++k) v[k] = observe(grampart + (int64_t)(first + (k < count ? k : 0)) * NE + idx);
        double t = v[0], most = v[0];
#pragma unroll
        for (int k = 1; k < kGramGroupMax; ++k) {
            t += k < count ? v[k] : 0.0;
            most = fmax(most, v[k]);
        }
        t = idx == 0 ? most : t;
        return t;
    };
    static_assert(kGramGroups <= kGramGroupMax, "one batch of loads at either level");
    if (!arrive_is_last(&scal->gram_cnt[grp], flag, (unsigned)gsize)) return false;
    for (int idx = tid; idx < NE; idx += NT) publish(grampart + (int64_t)(nwg + grp) * NE + idx, add(gfirst, gsize, idx));
    if (groups_only) return false;
    if (!arrive_is_last(&scal->gram_cnt[kGramGroups], flag, (unsigned)ngroups)) return false;
    if constexpr (HELD) {
        for (int i = tid; i < places.count(); i += NT) tot[i] = add(nwg, ngroups, places(i));
    } else {
        for (int idx = tid; idx < NE; idx += NT) tot[idx] = add(nwg, ngroups, idx);
    }
    __syncthreads();
    return true;
}

}  // namespace

// G = B^T B on the matrix cores.  B = [vectors | n x (2m+1)], masked by the free set, is a tall-skinny contraction whose
// operands stream from memory once.
//
// Up to 10 pairs: v_mfma_f64_4x4x4_4b, four products of a 4 x 4 by a 4 x 4 block side by side.  Lane l supplies A[i][k] and
// B[k][i] of block b, i = l % 4, b = l / 4 % 4, k = l / 16, and gets D[l / 16][l % 4] of block b; for a Gram matrix both
// operands are the same kind of number, vector 4 t + i at one element, so one register feeds either side, and the four blocks
// and k are sixteen elements whose order does not matter.  A lane can therefore load its operands straight into place: 16 bytes
// of vector 4 t + i, which makes four runs of 256 bytes per load, and nothing passes through LDS.  The vectors are y | g in the
// first K tiles and s in the next K; s with s is never asked for.  With 10 pairs that is 15 pairs of tiles, 960 cycles for 64
// elements, where blocks of 16 x 16 take two, 2048 cycles, half of them for rows and columns that nobody reads -- and with
// fewer pairs held it is less: K tiles hold 4 K - 1 pairs.
//
// LONG: memory bounds it.  A wave takes 64 consecutive elements per chunk, the vectors of two chunks in flight in registers,
// eight waves per compute unit.  The chain of a chunk: x, g (and l, u) three chunks ahead, one element per lane; the free set
// two chunks ahead -- fixed variables contribute nothing: a lane whose two elements are fixed reads what the first free pair's
// lane reads, and a chunk without any reads the first chunk's -- the vectors next, then the products.  The loop is made for
// K = 1, 2 and 3 tiles and the number of pairs held chooses.
// us per launch, 16 x 16 blocks by way of LDS, whatever the number of pairs held / this: n = 2 10^6 (all free) with 0 pairs 50.9 /
// 18.4, 3 51.3 / 27.6, 7 55.7 / 45, 10 76 / 71.5 (5.4 TB/s); 10^6 with 0 31 / 14.8, 3 31 / 17.1, 10 33.7 / 33.2.  (The vector
// unit, 77 sums per lane, took 47.6 and 100 with 10 pairs; loads straight into the 16 x 16 layout, 64 bytes of each vector a load, 41 and 90.)
// else: a few chunks in all, and what bounds it is latency: everything is requested at once, the ring slots whatever they
// hold, and looked at when it is there.  10 pairs, without the closing step, as above: n = 5000 5.4 / 5.0, 40 000 7.4 / 7.0.
// The sums are kept short: 16 elements by the matrix core from zero, added to the lane's running sum, the four blocks, the
// waves, then the workgroups' sums.
constexpr int kGramTileM = 10;                                            // up to this many pairs
constexpr int gram_tiles(int M) { return M / 4 + 1; }                     // of y and g; as many of s
constexpr int gram_tile_pairs(int K) { return K * (K + 1) / 2 + K * K; }

typedef f64x2 f64x2_any __attribute__((aligned(8)));

__device__ __forceinline__ double keep_if(double v, int keep) {           // keep: 0 or -1
    return __hiloint2double(__double2hiint(v) & keep, __double2loint(v) & keep);
}

// Adds the products of 64 elements: lane l holds elements 2 (l / 4), the next, and the same behind 32 of vector 4 t + l % 4.
// A0, A1: the rows of tiles that are meant (all of them at once want 4 registers a pair).
template <int K, int A0, int A1>
__device__ __forceinline__ void tile_products_rows(const f64x2 (&v)[2 * K][2], const int (&keep)[4], double (&sum)[gram_tile_pairs(K)]) {
    constexpr int kFirst = A0 * 2 * K - A0 * (A0 - 1) / 2, kCount = A1 * 2 * K - A1 * (A1 - 1) / 2 - kFirst;
    double acc[kCount];
#pragma unroll
    for (int k = 0; k < kCount; ++k) acc[k] = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double o[2 * K];
#pragma unroll
        for (int t = A0; t < 2 * K; ++t) o[t] = keep_if(q & 1 ? v[t][q / 2].y : v[t][q / 2].x, keep[q]);
        int k = 0;
#pragma unroll
        for (int a = A0; a < A1; ++a) {
#pragma unroll
            for (int b = a; b < 2 * K; ++b, ++k) acc[k] = __builtin_amdgcn_mfma_f64_4x4x4f64(o[a], o[b], acc[k], 0, 0, 0);
        }
    }
#pragma unroll
    for (int k = 0; k < kCount; ++k) sum[kFirst + k] += acc[k];
}
template <int K, bool APART = false>
__device__ __forceinline__ void tile_products(const f64x2 (&v)[2 * K][2], unsigned long long bits, double (&sum)[gram_tile_pairs(K)]) {
    const int at = ((threadIdx.x & 63) >> 2) * 2;
    int keep[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const unsigned w = (unsigned)(bits >> (32 * h)) >> at;
        keep[2 * h] = __builtin_amdgcn_sbfe(w, 0, 1);
        keep[2 * h + 1] = __builtin_amdgcn_sbfe(w, 1, 1);
    }
    if constexpr (APART && K == 3) {
        tile_products_rows<K, 0, 1>(v, keep, sum);
        __builtin_amdgcn_sched_barrier(0);
        tile_products_rows<K, 1, 3>(v, keep, sum);
    } else {
        tile_products_rows<K, 0, K>(v, keep, sum);
    }
}

// The four blocks added, and the wave's 4 x 4 results of every pair of tiles into its part of LDS: pair k, row i, column j at
// 16 k + 4 i + j.
template <int K>
__device__ __forceinline__ void tile_results(double (&sum)[gram_tile_pairs(K)], double* mine) {
    const int lane = threadIdx.x & 63;
    constexpr int kRowRor4 = 0x124, kRowRor8 = 0x128;                     // lane i of a row of 16 takes from i - 4, i - 8
#pragma unroll
    for (int k = 0; k < gram_tile_pairs(K); ++k) {
        double t = sum[k];
        t += dpp_move<kRowRor4>(t);
        t += dpp_move<kRowRor8>(t);
        if ((lane & 12) == 0) mine[16 * k + 4 * (lane >> 4) + (lane & 3)] = t;
    }
}
// Where tile_results has left the product of row a (y and g) with row b (the same) or column b (s).
__device__ __forceinline__ int tile_place(int K, int a, int b, bool b_is_s) {
    const int lo = b_is_s || a < b ? a : b, hi = (b_is_s || a < b ? b : a) + (b_is_s ? 4 * K : 0);
    const int ta = lo >> 2, tb = hi >> 2;
    return 16 * (ta * 2 * K - ta * (ta - 1) / 2 + tb - ta) + 4 * (lo & 3) + (hi & 3);
}

// A workgroup's record: the waves' results (tile_results, `wave_lds` doubles a wave) added in wave order.  BY_AGE: rows and columns
// of the tiles are pairs by age and g is row c; else ring slots and g row M.
template <int NW, int WAVE_LDS, bool BY_AGE>
__device__ __forceinline__ void gram_record(double pginf, double ynew, int nfixed, int K, int M, int m, int c, int base_slot, int slot_a,
                                            int slot_b, const double* dyn, double* red, double* __restrict__ grampart) {
    constexpr int NT = 64 * NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    pginf = wave_max(pginf);
    ynew = wave_sum(ynew);
    if (lane == 0) { red[wave] = pginf; red[NW + wave] = (double)nfixed; red[2 * NW + wave] = ynew; }
    __syncthreads();
    double* part = grampart + (int64_t)blockIdx.x * gram_entries(m);
    for (int idx = tid; idx < gram_products(m); idx += NT) {
        int a = slot_a, b = slot_b;
        if (idx != tid) gram_product_slots(idx, m, a, b);
        // row or column of a slot (past the last pair: not held, any number)
        auto place = [&](int slot) -> int {
            if (slot == m) return BY_AGE ? c : M;
            const int ring = slot < m ? slot : slot - m - 1;
            if (!BY_AGE) return ring;
            const int j = ring >= base_slot ? ring - base_slot : ring - base_slot + m;
            return j < c ? j : 0;
        };
        const int src = tile_place(K, place(a), place(b), b > m);
        double t = dyn[src];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += dyn[w * WAVE_LDS + src];
        publish(part + kGramHdr + idx, t);
    }
    if (tid < 3) {
        double t = red[tid * NW];
#pragma unroll
        for (int w = 1; w < NW; ++w) t = tid == 0 ? fmax(t, red[w]) : t + red[tid * NW + w];
        publish(part + tid, t);
    }
}

template <int M, int NW, bool LONG, bool DBG>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4)))
void k_gram(int64_t n, int m, Opts op, const double* __restrict__ x, const double* __restrict__ g, const double* __restrict__ l,
            const double* __restrict__ u, const double* __restrict__ S, const double* __restrict__ Y, uint8_t* __restrict__ mask,
            Scal* __restrict__ scal, double* __restrict__ grampart, int evaluate_stop, int no_close) {
    constexpr int NT = 64 * NW, KM = gram_tiles(M), kWaveLds = 16 * gram_tile_pairs(KM);
    constexpr int kClose = gram_tot_at(M) + gram_entries(M);
    __shared__ __align__(16) double dyn[NW * kWaveLds > kClose ? NW * kWaveLds : kClose];   // the waves' results; later G and the totals
    __shared__ double red[NW * 3];
    __shared__ double alpha_s[kMaxM + 1];
    __shared__ int flag;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // one load per wave fetches the integer header of the scalar block (status, ring position, pending
    // update); readlanes hand the fields to every lane
    static_assert(offsetof(Scal, pend_ok) < 64 && offsetof(Scal, gram_left) < 64, "header fields must sit in the first 16 ints");
    const int hdr = lane < 16 ? reinterpret_cast<const int*>(scal)[lane] : 0;

    const int64_t nchunks = (n + 63) / 64, stride = (int64_t)gridDim.x * NW;
    const int64_t ch0 = (int64_t)blockIdx.x * NW + wave;
    const int64_t bstride = op.uniform_bounds ? 0 : 1;   // same bounds everywhere: l and u are not streamed
    struct Elem { double x, g, l, u, y; uint8_t mk; };
    auto request = [&](int64_t ch, Elem& s, const double* y_new) {
        const int64_t e = ch * 64 + lane, ec = e < n ? e : n - 1;
        s.x = x[ec]; s.g = g[ec]; s.l = l[ec * bstride]; s.u = u[ec * bstride];
        s.y = LONG ? y_new[ec] : 0.0;
        if constexpr (DBG) s.mk = mask[ec];
    };
    double pginf = 0.0, ynew = 0.0;
    int nfixed = 0;
    // Eq. (ws) and the statistics of a chunk; the bits of its free elements
    auto decide = [&](int64_t ch, const Elem& s) -> unsigned long long {
        const int64_t e = ch * 64 + lane;
        const bool in = e < n;
        bool fr;
        if constexpr (DBG) {
            fr = s.mk != 0;
        } else {
            fr = !fixed_at(s.x, s.g, s.l, s.u, op.eps);
            mask[in ? e : n - 1] = (uint8_t)fr;       // (past the end: the last element's own value once more)
        }
        pginf = fmax(pginf, in ? fabs(s.x - clampd(s.x - s.g, s.l, s.u)) : 0.0);
        if (LONG) ynew = fma(in ? s.y : 0.0, s.y, ynew);
        const unsigned long long bits = __ballot(fr && in);
        nfixed += __popcll(__ballot(in)) - __popcll(bits);
        return bits;
    };
    const int i4 = lane & 3, pair_at = (lane >> 2) * 2;
    // (the second element of an odd vector's last pair is whatever follows the vector in the workspace: it counts as fixed)
    auto short_slot = [&](int t) -> const double* {      // tile t's vector of this lane, by ring slot
        const int k = 4 * (t < KM ? t : t - KM) + i4;
        if (t < KM && k >= M) return g;
        return (t < KM ? Y : S) + (int64_t)(k < m ? k : m - 1) * n;
    };
    Elem sa;
    f64x2 first[LONG ? 1 : 2 * KM][2];
    auto short_fetch = [&](int64_t ch) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t e = ch * 64 + 32 * h + pair_at, ec = e < n ? e : n - 1;
#pragma unroll
            for (int t = 0; t < (LONG ? 1 : 2 * KM); ++t) first[t][h] = *reinterpret_cast<const f64x2_any*>(short_slot(t) + ec);
        }
    };
    if constexpr (!LONG) {
        request(ch0, sa, nullptr);
        short_fetch(ch0);
    }
    int slot_a, slot_b;                                  // (entry tid of the record; here, while the loads are on their way)
    gram_product_slots(tid < gram_products(m) ? tid : 0, m, slot_a, slot_b);
    asm volatile("" : "+v"(slot_a), "+v"(slot_b));
    auto field = [&](size_t off) { return __builtin_amdgcn_readlane(hdr, (int)(off / 4)); };
    const int status = field(offsetof(Scal, status));
    if (status != LBFGSB_RUNNING) {
        // a step that finds the solver parked by the short logistic sequence is counted, so that the host can redo it
        if (evaluate_stop && !DBG && blockIdx.x == 0 && tid == 0) {
            if (status == kStatusBail) scal->bail_skipped += 1;
            note_progress(op, status);
        }
        return;
    }
    if (no_close == kGramOpenUnlessLeft && field(offsetof(Scal, gram_left))) return;
    int head = field(offsetof(Scal, head)), c = field(offsetof(Scal, count));
    if (field(offsetof(Scal, pend_valid))) {          // same rule as effective_ring()
        if (field(offsetof(Scal, pend_ok))) { head = ring_next(head, m); c = c < m ? c + 1 : m; }
        else c = 0;
    }
    const double yn_old = no_close ? 1.0 : prefetch_ynorm2(scal, c, head, m);   // (used by the last workgroup's recursion, fetched now)
    const int base_slot = c > 0 ? ring_back(head, c, m) : 0;   // ring slot of the oldest pair
    const int newest = c > 0 ? ring_back(head, 1, m) : -1;
    double* mine = dyn + wave * kWaveLds;
    int K = KM;                                          // tiles of y and g in the sums left in LDS
    if constexpr (LONG) {
        // vectors by age: y of pair j in row j, g in row c, s of pair j in column j; the rest read g, and nobody their products
        const double* y_new = newest >= 0 ? Y + (int64_t)newest * n : g;
        auto stream = [&](auto tiles) {
            constexpr int KT = decltype(tiles)::value;
            const double* from[2 * KT];
#pragma unroll
            for (int t = 0; t < 2 * KT; ++t) {
                const int j = 4 * (t < KT ? t : t - KT) + i4, slot = base_slot + j < m ? base_slot + j : base_slot + j - m;
                from[t] = j < c ? (t < KT ? Y : S) + (int64_t)slot * n : g;
            }
            auto fetch = [&](int64_t ch, unsigned long long bits, f64x2 (&v)[2 * KT][2]) {
                const unsigned head_pair = bits ? (unsigned)__builtin_ctzll(bits) & ~1u : 0u;
                const int64_t e0 = bits ? ch * 64 : 0;   // (uniform)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const unsigned w = (unsigned)(bits >> (32 * h)) >> pair_at;
                    const int64_t e = e0 + (w & 3u ? 32u * h + pair_at : head_pair);
#pragma unroll
                    for (int t = 0; t < 2 * KT; ++t) v[t][h] = *reinterpret_cast<const f64x2_any*>(from[t] + e);
                }
            };
            double sum[gram_tile_pairs(KT)];
#pragma unroll
            for (int k = 0; k < gram_tile_pairs(KT); ++k) sum[k] = 0.0;
            if (ch0 < nchunks) {
                f64x2 va[2 * KT][2], vb[2 * KT][2];
                Elem sb;
                request(ch0, sa, y_new);
                request(ch0 + stride, sb, y_new);
                unsigned long long ba = decide(ch0, sa), bb;
                fetch(ch0, ba, va);
                request(ch0 + 2 * stride, sa, y_new);
                // (two chunks a trip and one way out: a chunk past the end has no free element and adds nothing)
                for (int64_t ch = ch0; ch < nchunks; ch += 2 * stride) {
                    bb = decide(ch + stride, sb);
                    fetch(ch + stride, bb, vb);
                    request(ch + 3 * stride, sb, y_new);
                    __builtin_amdgcn_sched_barrier(0);
                    tile_products<KT>(va, ba, sum);
                    __builtin_amdgcn_sched_barrier(0);
                    ba = decide(ch + 2 * stride, sa);
                    fetch(ch + 2 * stride, ba, va);
                    request(ch + 4 * stride, sa, y_new);
                    __builtin_amdgcn_sched_barrier(0);
                    tile_products<KT>(vb, bb, sum);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            tile_results<KT>(sum, mine);
        };
        K = c / 4 + 1;
        if (K == 1) stream(std::integral_constant<int, 1>());
        else if (KM == 2 || K == 2) stream(std::integral_constant<int, 2>());
        else if constexpr (KM == 3) stream(std::integral_constant<int, 3>());
    } else {
        double sum[gram_tile_pairs(KM)];
#pragma unroll
        for (int k = 0; k < gram_tile_pairs(KM); ++k) sum[k] = 0.0;
        for (int64_t ch = ch0; ch < nchunks; ch += stride) {
            if (ch != ch0) {
                request(ch, sa, nullptr);
                short_fetch(ch);
            }
            // ||y_new||^2, over fixed variables too, by the lanes that hold it (what lies past the vector may be anything: no factor of it)
#pragma unroll
            for (int t = 0; t < KM; ++t) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int64_t e = ch * 64 + 32 * h + pair_at;
                    if (4 * t + i4 == newest) {
                        const double y0 = e < n ? first[t][h].x : 0.0, y1 = e + 1 < n ? first[t][h].y : 0.0;
                        ynew = fma(y0, y0, ynew);
                        ynew = fma(y1, y1, ynew);
                    }
                }
            }
            const unsigned long long bits = decide(ch, sa);
            tile_products<KM>(first, bits, sum);
        }
        tile_results<KM>(sum, mine);
    }

    const int NE = gram_entries(m);
    gram_record<NW, kWaveLds, LONG>(pginf, ynew, nfixed, K, M, m, c, base_slot, slot_a, slot_b, dyn, red, grampart);
    if (!LONG && no_close) return;   // the direction kernel adds the records and does the rest
    double* tot = dyn + gram_tot_at(M);
    if (!reduce_partials<NT, false>(grampart, NE, scal, &flag, tot, LONG && no_close, GramPlaces{m, c, base_slot})) return;
    gram_finish<NT, 10, false>(tot, dyn, alpha_s, scal, m, c, head, base_slot, op, yn_old, DBG, evaluate_stop, true);
    __syncthreads();
    if (tid == 0 && evaluate_stop) note_progress(op, scal->status);
}

// The Gaussian transport kind's update (k_ot_update_gauss) and the free set and Gram matrix of the next iteration in one pass: what
// the update writes -- x, g and the new pair -- the Gram kernel would read again next, and an element's products need nothing that
// other workgroups write.  The stream is k_gram's with one stage more: x, g, p and the entry's two coefficients arrive three
// chunks ahead; the new values are formed, stored and kept in LDS, from where the products take them.  A step whose line search
// fails changes nothing, and the next one starts from the gradient alone.  Rows of 64 columns at least: a chunk then crosses one row's
// end at most.
// n = 10^6, us, the update's kernel and k_gram / this: 1 pair 26 / 21.6, 4 32 / 27.7, 10 44.3 / 38.4.  (Two groups of tiles one after
// the other and 32-bit offsets from scalar bases for the registers' sake: with 11 spilled the last figure was 41.  With room for 10
// pairs all 256 are taken still and two are spilled, seven where bounds differ.)
// SAME: every variable has the same bounds.
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
template <int M, bool SAME>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_update_gram_gauss(Dims dm, Opts op, int loss_parts, const double* __restrict__ losspart, const double* __restrict__ wt,
                         const double* __restrict__ p1, const double* __restrict__ p2, const double* __restrict__ l,
                         const double* __restrict__ u, double* __restrict__ x, double* __restrict__ g, double* __restrict__ S,
                         double* __restrict__ Y, uint8_t* __restrict__ mask, Scal* __restrict__ scal, double* __restrict__ grampart) {
    constexpr int NW = 8, NT = 64 * NW, KM = gram_tiles(M), kWaveLds = 16 * gram_tile_pairs(KM);
    constexpr int kNew = 3 * 64;                         // a chunk's new g, y and s
    __shared__ __align__(16) double dyn[NW * kWaveLds];
    __shared__ __align__(16) double fresh_s[NW * 2 * kNew];
    __shared__ double red[NW * 3];
    __shared__ double ls_alpha;
    __shared__ int ls_ok, ls_bt, flag;
    if (scal->status != LBFGSB_RUNNING) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = dm.m;
    const int64_t n = dm.n, cols = dm.cols;
    const int head = scal->head, held = scal->count, branch = scal->branch;
    const double gp = scal->gp, alpha_ub = scal->alpha_ub, f_old = scal->f;
    const double tt = sum_all<NT>(losspart, loss_parts, red) + dm.lambda * scal->pp;
    if (tid == 0) {
        int ok, bt;
        ls_alpha = armijo_quadratic(gp, tt, alpha_ub, op, ok, bt);
        ls_ok = ok; ls_bt = bt;
    }
    int slot_a, slot_b;
    gram_product_slots(tid < gram_products(m) ? tid : 0, m, slot_a, slot_b);
    __syncthreads();
    const double alpha = ls_alpha;
    const bool ok = __builtin_amdgcn_readfirstlane(ls_ok) != 0;
    const int c = __builtin_amdgcn_readfirstlane(ok ? (held < m ? held + 1 : m) : 0);      // pairs held from here on; the newest in slot `head`
    const int base_slot = __builtin_amdgcn_readfirstlane(c > 0 ? ring_back(head, c - 1, m) : 0);
    const double* p = branch == 1 ? p1 : p2;
    double *Sn = S + (int64_t)head * n, *Yn = Y + (int64_t)head * n;

    const int64_t nchunks = (n + 63) / 64, stride = (int64_t)gridDim.x * NW;
    const int64_t ch0 = (int64_t)blockIdx.x * NW + wave;
    const double inv_cols = 1.0 / (double)cols;
    struct Elem { double x, g, p, wr, wc, l[SAME ? 1 : 2]; };
    auto request = [&](int64_t ch, Elem& s) {
        // (a chunk past the end: the last one's; scalar base and 32-bit offset)
        const int64_t first = (ch < nchunks ? ch : nchunks - 1) * 64;
        const unsigned at = first + 64 <= n ? (unsigned)lane : ((unsigned)lane < (unsigned)(n - first) ? (unsigned)lane : (unsigned)(n - first) - 1u);
        s.x = (x + first)[at]; s.g = (g + first)[at]; s.p = (p + first)[at];
        if constexpr (!SAME) { s.l[0] = (l + first)[at]; s.l[1] = (u + first)[at]; }
        // row and column of the chunk's first element (uniform), then of this lane's
        int64_t row = (int64_t)((double)first * inv_cols), col = first - row * cols;
        if (col < 0) { col += cols; --row; }
        if (col >= cols) { col -= cols; ++row; }
        row = uniform64(row);
        col = uniform64(col);
        const int64_t left = cols - col;                  // (of this row)
        const bool next = (int64_t)at >= left;
        s.wr = (wt + row)[next ? 1u : 0u];
        s.wc = (wt + dm.rows + (left < 64 ? 0 : col))[left < 64 ? (next ? at - (unsigned)left : (unsigned)col + at) : at];
    };
    double pginf = 0.0, ynew = 0.0;
    int nfixed = 0;
    double* fresh = fresh_s + wave * (2 * kNew);
    auto decide = [&](int64_t ch, const Elem& s, double* keep) -> unsigned long long {
        const int64_t first = ch * 64;
        const bool in = first + lane < n;
        const double y = ok ? alpha * fma(dm.lambda, s.p, s.wr + s.wc) : 0.0;
        const double lo = SAME ? op.lo : s.l[0], hi = SAME ? op.hi : s.l[SAME ? 0 : 1];
        const double xn = ok ? clampd(fma(alpha, s.p, s.x), lo, hi) : s.x;
        const double gn = s.g + y, sn = xn - s.x;
        const bool fr = !fixed_at(xn, gn, lo, hi, op.eps);
        if (in) {
            (mask + first)[(unsigned)lane] = (uint8_t)fr;
            if (ok) {
                (Sn + first)[(unsigned)lane] = sn; (Yn + first)[(unsigned)lane] = y;
                (x + first)[(unsigned)lane] = xn; (g + first)[(unsigned)lane] = gn;
            }
        }
        keep[lane] = gn; keep[64 + lane] = y; keep[128 + lane] = sn;
        pginf = fmax(pginf, in ? fabs(xn - clampd(xn - gn, lo, hi)) : 0.0);
        ynew = fma(in ? y : 0.0, y, ynew);
        const unsigned long long bits = __ballot(fr && in);
        nfixed += __popcll(__ballot(in)) - __popcll(bits);
        return bits;
    };
    const int i4 = lane & 3, pair_at = (lane >> 2) * 2;
    double* mine = dyn + wave * kWaveLds;
    auto stream = [&](auto tiles) {
        constexpr int KT = decltype(tiles)::value;
        const double* from[2 * KT];                      // (old pairs; what is new, or not there, reads g and is not looked at)
#pragma unroll
        for (int t = 0; t < 2 * KT; ++t) {
            const int j = 4 * (t < KT ? t : t - KT) + i4, slot = base_slot + j < m ? base_slot + j : base_slot + j - m;
            from[t] = j + 1 < c ? (t < KT ? Y : S) + (int64_t)slot * n : g;
        }
        // tiles that hold something new: row c is g, row and column c - 1 the new pair
        const int tile_g = c >> 2, tile_pair = (c - 1) >> 2;
        auto fetch = [&](int64_t ch, unsigned long long bits, f64x2 (&v)[2 * KT][2]) {
            const unsigned head_pair = bits ? (unsigned)__builtin_ctzll(bits) & ~1u : 0u;
            const int64_t e0 = bits ? ch * 64 : 0;       // (uniform)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned w = (unsigned)(bits >> (32 * h)) >> pair_at;
                const int64_t e = e0 + (w & 3u ? 32u * h + pair_at : head_pair);
#pragma unroll
                for (int t = 0; t < 2 * KT; ++t) v[t][h] = *reinterpret_cast<const f64x2_any*>(from[t] + e);
            }
        };
        auto insert = [&](const double* keep, f64x2 (&v)[2 * KT][2]) {
#pragma unroll
            for (int t = 0; t < 2 * KT; ++t) {
                const int tt_ = t < KT ? t : t - KT;
                if (t < KT && tt_ == tile_g) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f64x2 q = *reinterpret_cast<const f64x2*>(keep + 32 * h + pair_at);
                        v[t][h] = i4 == (c & 3) ? q : v[t][h];
                    }
                }
                if (c > 0 && tt_ == tile_pair) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f64x2 q = *reinterpret_cast<const f64x2*>(keep + (t < KT ? 64 : 128) + 32 * h + pair_at);
                        v[t][h] = i4 == ((c - 1) & 3) ? q : v[t][h];
                    }
                }
            }
        };
        double sum[gram_tile_pairs(KT)];
#pragma unroll
        for (int k = 0; k < gram_tile_pairs(KT); ++k) sum[k] = 0.0;
        if (ch0 < nchunks) {
            f64x2 va[2 * KT][2], vb[2 * KT][2];
            Elem sa, sb;
            request(ch0, sa);
            request(ch0 + stride, sb);
            unsigned long long ba = decide(ch0, sa, fresh), bb;
            fetch(ch0, ba, va);
            request(ch0 + 2 * stride, sa);
            for (int64_t ch = ch0; ch < nchunks; ch += 2 * stride) {
                bb = decide(ch + stride, sb, fresh + kNew);
                fetch(ch + stride, bb, vb);
                request(ch + 3 * stride, sb);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_wave_barrier();
                insert(fresh, va);
                tile_products<KT, true>(va, ba, sum);
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_sched_barrier(0);
                ba = decide(ch + 2 * stride, sa, fresh);
                fetch(ch + 2 * stride, ba, va);
                request(ch + 4 * stride, sa);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_wave_barrier();
                insert(fresh + kNew, vb);
                tile_products<KT, true>(vb, bb, sum);
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        tile_results<KT>(sum, mine);
    };
    const int K = c / 4 + 1;
    if (K == 1) stream(std::integral_constant<int, 1>());
    else if (KM == 2 || K == 2) stream(std::integral_constant<int, 2>());
    else if constexpr (KM == 3) stream(std::integral_constant<int, 3>());

    gram_record<NW, kWaveLds, true>(pginf, ynew, nfixed, K, M, m, c, base_slot, slot_a, slot_b, dyn, red, grampart);
    // (no workgroup of this kernel reads the pend_* fields or gram_left)
    if (blockIdx.x == 0 && tid == 0) {
        scal->pend_ok = ok;
        scal->pend_bt = ls_bt;
        scal->pend_alpha = alpha;
        scal->pend_f = f_old + alpha * (gp + 0.5 * alpha * tt);
        scal->pend_valid = 1;
        scal->gram_left = 1;
    }
    reduce_partials<NT, false>(grampart, gram_entries(m), scal, &flag, nullptr, true, GramPlaces{m, c, base_slot});
}

// The same for the quadratic form on vectors that are not long: its update is element by element as well (the change of the gradient
// is s.t, plus the folded rows' share).  As in k_gram everything is requested at once, here with what the update reads; the new
// values pass through LDS.  As many records as k_gram leaves.  (The least-squares kinds add up partial columns first, 10 MB of them
// at 20000 x 5000: few workgroups take too long over those, and the records of many keep the direction kernel, with 79 for 20
// 11.3 us for 8.4; whole calls were no faster.)
// n = 10 000, 10 pairs, us: update 5.1 and Gram kernel 5.3 / this 6.5; dual SVM, two outer iterations, with 10 000 points 1812 -> 1774.
template <int M, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4)))
void k_update_gram_form(Dims dm, Opts op, int loss_parts, const double* __restrict__ losspart, const double* __restrict__ t,
                        const double* __restrict__ sign, const double* __restrict__ p1, const double* __restrict__ p2,
                        const double* __restrict__ l, const double* __restrict__ u, double* __restrict__ x, double* __restrict__ g,
                        double* __restrict__ S, double* __restrict__ Y, uint8_t* __restrict__ mask, Scal* __restrict__ scal, int n_fold,
                        const double* __restrict__ fold_rows, const double* __restrict__ fold_weight, const double* __restrict__ dir_part,
                        int dir_blocks, double* __restrict__ grampart) {
    constexpr int NT = 64 * NW, KM = gram_tiles(M), kWaveLds = 16 * gram_tile_pairs(KM);
    __shared__ __align__(16) double dyn[NW * kWaveLds];
    __shared__ __align__(16) double fresh_s[NW * 3 * 64];
    __shared__ double red[NW * 3];
    __shared__ double fold_s[kFoldMax + 1];
    __shared__ double ls_alpha;
    __shared__ int ls_ok, ls_bt;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = dm.m;
    const int64_t n = dm.n, nchunks = (n + 63) / 64, stride = (int64_t)gridDim.x * NW, ch0 = (int64_t)blockIdx.x * NW + wave;
    const int i4 = lane & 3, pair_at = (lane >> 2) * 2;
    double xe, ge, le, ue, pe1, pe2, te, se, fe[kFoldMax];
    f64x2 v[2 * KM][2];
    auto request = [&](int64_t ch) {
        const int64_t e = ch * 64 + lane, ec = e < n ? e : n - 1;
        xe = x[ec]; ge = g[ec]; le = l[ec]; ue = u[ec]; pe1 = p1[ec]; pe2 = p2[ec]; te = t[ec];
        se = sign ? sign[ec] : 1.0;
#pragma unroll
        for (int r = 0; r < kFoldMax; ++r) fe[r] = r < n_fold ? fold_rows[(int64_t)r * n + ec] : 0.0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t e2 = ch * 64 + 32 * h + pair_at, ec2 = e2 < n ? e2 : n - 1;
#pragma unroll
            for (int k = 0; k < 2 * KM; ++k) {
                const int slot = 4 * (k < KM ? k : k - KM) + i4;
                v[k][h] = *reinterpret_cast<const f64x2_any*>((k < KM ? Y : S) + (int64_t)(slot < m ? slot : m - 1) * n + ec2);
            }
        }
    };
    request(ch0);
    const int status = scal->status, head = scal->head, branch = scal->branch;
    const double gp = scal->gp, alpha_ub = scal->alpha_ub, f_old = scal->f;
    int slot_a, slot_b;
    gram_product_slots(tid < gram_products(m) ? tid : 0, m, slot_a, slot_b);
    if (status != LBFGSB_RUNNING) return;
    if (n_fold > 0 && wave == 0) {
        // the direction kernel left only its per-workgroup sums: the folded rows' products with the chosen candidate
        double tx[2 * kFoldMax];
        dir_fold_from_partials(dir_part, dir_blocks, tx);
        if (tid == 0) fold_s[kFoldMax] = fold_coefficients(tx, branch, n_fold, fold_weight, fold_s);
    }
    double tt = sum_all<NT>(losspart, loss_parts, red);  // (a barrier inside)
    if (n_fold > 0) tt += fold_s[kFoldMax];
    if (tid == 0) {
        int ok, bt;
        ls_alpha = armijo_quadratic(gp, tt, alpha_ub, op, ok, bt);
        ls_ok = ok; ls_bt = bt;
    }
    __syncthreads();
    const double alpha = ls_alpha;
    const bool ok = ls_ok != 0;
    const int newest = ok ? head : -1;
    double *Sn = S + (int64_t)head * n, *Yn = Y + (int64_t)head * n, *keep = fresh_s + wave * (3 * 64);
    double sum[gram_tile_pairs(KM)];
#pragma unroll
    for (int k = 0; k < gram_tile_pairs(KM); ++k) sum[k] = 0.0;
    double pginf = 0.0, ynew = 0.0;
    int nfixed = 0;
    for (int64_t ch = ch0; ch < nchunks; ch += stride) {
        if (ch != ch0) request(ch);
        const int64_t e = ch * 64 + lane;
        const bool in = e < n;
        double w = se * te;
#pragma unroll
        for (int r = 0; r < kFoldMax; ++r)
            if (r < n_fold) w = fma(fold_s[r], fe[r], w);
        const double y = ok ? alpha * w : 0.0;
        const double xn = ok ? clampd(fma(alpha, branch == 1 ? pe1 : pe2, xe), le, ue) : xe;
        const double gn = ge + y, sn = xn - xe;
        const bool fr = !fixed_at(xn, gn, le, ue, op.eps);
        if (in) {
            mask[e] = (uint8_t)fr;
            if (ok) { Sn[e] = sn; Yn[e] = y; x[e] = xn; g[e] = gn; }
        }
        keep[lane] = gn; keep[64 + lane] = y; keep[128 + lane] = sn;
        pginf = fmax(pginf, in ? fabs(xn - clampd(xn - gn, le, ue)) : 0.0);
        ynew = fma(in ? y : 0.0, y, ynew);
        const unsigned long long bits = __ballot(fr && in);
        nfixed += __popcll(__ballot(in)) - __popcll(bits);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 2 * KM; ++k) {
            const int slot = 4 * (k < KM ? k : k - KM) + i4;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (k < KM && 4 * k <= M && M < 4 * k + 4) {         // (the tile that holds g)
                    const f64x2 q = *reinterpret_cast<const f64x2*>(keep + 32 * h + pair_at);
                    v[k][h] = slot == M ? q : v[k][h];
                }
                const f64x2 q = *reinterpret_cast<const f64x2*>(keep + (k < KM ? 64 : 128) + 32 * h + pair_at);
                v[k][h] = slot == newest ? q : v[k][h];
            }
        }
        tile_products<KM>(v, bits, sum);
        __builtin_amdgcn_wave_barrier();
    }
    tile_results<KM>(sum, dyn + wave * kWaveLds);
    gram_record<NW, kWaveLds, false>(pginf, ynew, nfixed, KM, M, m, 0, 0, slot_a, slot_b, dyn, red, grampart);
    // (no workgroup of this kernel reads the pend_* fields or gram_left)
    if (blockIdx.x == 0 && tid == 0) {
        scal->pend_ok = ok;
        scal->pend_bt = ls_bt;
        scal->pend_alpha = alpha;
        scal->pend_f = f_old + alpha * (gp + 0.5 * alpha * tt);
        scal->pend_valid = 1;
        scal->gram_left = 1;
    }
}

// Beyond 10 pairs: v_mfma_f64_16x16x4_f64, a 16 x 4 by a 4 x 16 block (the pairs of 4 x 4 tiles would take all registers).  A lane
// loads one element of every vector (512 contiguous bytes per load) and writes it, masked, to the wave's own part of LDS; from
// there lane (i = lane % 16, q = lane / 16) supplies vector 16 b + i at elements 8 s + 2 q and the next, for either operand.  Result
// of lane l, register r of a block: row l/16 + 4 r, column l % 16.  The rest is as above.  20 pairs, n = 10^6: 96 us a launch.
template <int M, int NW, bool LONG, bool DBG>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 4, NW / 4)))
void k_gram_blocks(int64_t n, int m, Opts op, const double* __restrict__ x, const double* __restrict__ g, const double* __restrict__ l,
            const double* __restrict__ u, const double* __restrict__ S, const double* __restrict__ Y, uint8_t* __restrict__ mask,
            Scal* __restrict__ scal, double* __restrict__ grampart, int evaluate_stop, int) {
    constexpr int NT = 64 * NW, NB = gram_nb(M), NA = gram_na(M), NP = gram_np(M), NV = gram_slots(M);
    extern __shared__ __align__(16) double dyn[];   // the waves' elements; their blocks; later G and the totals
    __shared__ double red[NW * 3];
    __shared__ double alpha_s[kMaxM + 1];
    __shared__ int flag;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // one load per wave fetches the integer header of the scalar block (status, ring position, pending
    // update); readlanes hand the fields to every lane
    static_assert(offsetof(Scal, pend_ok) < 64, "header fields must sit in the first 16 ints");
    const int hdr = lane < 16 ? reinterpret_cast<const int*>(scal)[lane] : 0;

    const int64_t nchunks = (n + 63) / 64, stride = (int64_t)gridDim.x * NW;
    const int64_t ch0 = (int64_t)blockIdx.x * NW + wave;
    const int64_t bstride = op.uniform_bounds ? 0 : 1;   // same bounds everywhere: l and u are not streamed
    struct Elem { double x, g, l, u, y; uint8_t mk; };
    auto request = [&](int64_t ch, Elem& s, const double* y_new) {
        const int64_t e = ch * 64 + lane, ec = e < n ? e : n - 1;
        s.x = x[ec]; s.g = g[ec]; s.l = l[ec * bstride]; s.u = u[ec * bstride];
        s.y = LONG ? y_new[ec] : 0.0;
        if constexpr (DBG) s.mk = mask[ec];
    };
    double pginf = 0.0, ynew = 0.0;
    int nfixed = 0;
    // Eq. (ws) and the statistics of a chunk; the bits of its free elements
    auto decide = [&](int64_t ch, const Elem& s) -> unsigned long long {
        const int64_t e = ch * 64 + lane;
        const bool in = e < n;
        bool fr;
        if constexpr (DBG) {
            fr = s.mk != 0;
        } else {
            fr = !fixed_at(s.x, s.g, s.l, s.u, op.eps);
            mask[in ? e : n - 1] = (uint8_t)fr;       // (past the end: the last element's own value once more)
        }
        pginf = fmax(pginf, in ? fabs(s.x - clampd(s.x - s.g, s.l, s.u)) : 0.0);
        ynew = fma(in ? s.y : 0.0, s.y, ynew);
        const unsigned long long bits = __ballot(fr && in);
        nfixed += __popcll(__ballot(in)) - __popcll(bits);
        return bits;
    };
    f64x4 sum[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) sum[k] = f64x4{0.0, 0.0, 0.0, 0.0};
    double* mine = dyn + wave * ((NV + 1) * kGramStride);
    const int i16 = lane & 15, q = lane >> 4;
    // (slots past the last vector: a row of zeros)
    const double* opnd_at[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) opnd_at[b] = mine + (16 * b + i16 < NV ? 16 * b + i16 : NV) * kGramStride + 2 * q;
    mine[NV * kGramStride + lane] = 0.0;
    auto multiply = [&](const double (&v)[NV], unsigned long long bits) {
        const int keep = (bits >> lane) & 1ull ? -1 : 0;
#pragma unroll
        for (int k = 0; k < NV; ++k)
            mine[k * kGramStride + lane] = __hiloint2double(__double2hiint(v[k]) & keep, __double2loint(v[k]) & keep);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            f64x4 acc[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) acc[k] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s8 = 4 * half; s8 < 4 * half + 4; ++s8) {
                f64x2 o[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) o[b] = *reinterpret_cast<const f64x2*>(opnd_at[b] + 8 * s8);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    int k = 0;
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
#pragma unroll
                        for (int b = a; b < NB; ++b, ++k)
                            acc[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(t ? o[a].y : o[a].x, t ? o[b].y : o[b].x, acc[k], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < NP; ++k) sum[k] += acc[k];
        }
        __builtin_amdgcn_wave_barrier();
    };
    // where the waves' blocks hold the product that is entry idx of a record
    auto block_place = [&](int idx) -> int {
        int a, b;
        gram_product_slots_many(idx, m, a, b);
        // (record: y, g, s of m slots each; here of M)
        a += a == m ? M - m : 0;
        b += b >= m ? M - m : 0;
        const int ab = a >> 4, bb = b >> 4, pair = ab * NB - ab * (ab - 1) / 2 + bb - ab;
        return pair * 256 + ((a & 15) >> 2) * 64 + (a & 3) * 16 + (b & 15);
    };
    auto slot_ptr = [&](int k) -> const double* {
        if (k == M) return g;
        const int ring = k < M ? k : k - M - 1;
        return (k < M ? Y : S) + (int64_t)(ring < m ? ring : m - 1) * n;
    };
    Elem sa;
    double va[NV];
    if constexpr (!LONG) {
        request(ch0, sa, nullptr);
        const int64_t e = ch0 * 64 + lane, ec = e < n ? e : n - 1;
#pragma unroll
        for (int k = 0; k < NV; ++k) va[k] = slot_ptr(k)[ec];
    }

    int place = block_place(tid < gram_products(m) ? tid : 0);   // (here, while the loads are on their way)
    asm volatile("" : "+v"(place));
    auto field = [&](size_t off) { return __builtin_amdgcn_readlane(hdr, (int)(off / 4)); };
    const int status = field(offsetof(Scal, status));
    if (status != LBFGSB_RUNNING) {
        // a step that finds the solver parked by the short logistic sequence is counted, so that the host can redo it
        if (evaluate_stop && !DBG && blockIdx.x == 0 && tid == 0) {
            if (status == kStatusBail) scal->bail_skipped += 1;
            note_progress(op, status);
        }
        return;
    }
    int head = field(offsetof(Scal, head)), c = field(offsetof(Scal, count));
    if (field(offsetof(Scal, pend_valid))) {          // same rule as effective_ring()
        if (field(offsetof(Scal, pend_ok))) { head = ring_next(head, m); c = c < m ? c + 1 : m; }
        else c = 0;
    }
    const double yn_old = prefetch_ynorm2(scal, c, head, m);   // (used by the last workgroup's recursion, fetched now)
    const int base_slot = c > 0 ? ring_back(head, c, m) : 0;   // ring slot of the oldest pair
    const int newest = c > 0 ? ring_back(head, 1, m) : -1;
    if constexpr (LONG) {
        const double* y_new = newest >= 0 ? Y + (int64_t)newest * n : g;
        unsigned long long active = 1ull << M;        // bit k: slot k holds a vector
        for (int j = 0; j < c; ++j) {
            const int sl = base_slot + j < m ? base_slot + j : base_slot + j - m;
            active |= (1ull << sl) | (1ull << (M + 1 + sl));
        }
        auto fetch = [&](int64_t ch, unsigned long long bits, double (&v)[NV]) {
            const int first = bits ? __builtin_ctzll(bits) : 0;
            const int64_t e0 = bits ? ch * 64 : 0;    // (uniform)
            const unsigned off = (unsigned)((bits >> lane) & 1ull ? lane : first);
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = (((active >> k) & 1ull ? slot_ptr(k) : g) + e0)[off];
        };
        if (ch0 < nchunks) {
            double vb[NV];
            Elem sb;
            request(ch0, sa, y_new);
            request(ch0 + stride, sb, y_new);
            unsigned long long ba = decide(ch0, sa), bb;
            fetch(ch0, ba, va);
            request(ch0 + 2 * stride, sa, y_new);
            // (two chunks a trip and one way out: a chunk past the end has no free element and adds nothing)
            for (int64_t ch = ch0; ch < nchunks; ch += 2 * stride) {
                bb = decide(ch + stride, sb);
                fetch(ch + stride, bb, vb);
                request(ch + 3 * stride, sb, y_new);
                __builtin_amdgcn_sched_barrier(0);
                multiply(va, ba);
                __builtin_amdgcn_sched_barrier(0);
                ba = decide(ch + 2 * stride, sa);
                fetch(ch + 2 * stride, ba, va);
                request(ch + 4 * stride, sa, y_new);
                __builtin_amdgcn_sched_barrier(0);
                multiply(vb, bb);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
        for (int64_t ch = ch0; ch < nchunks; ch += stride) {
            if (ch != ch0) {
                request(ch, sa, nullptr);
                const int64_t e = ch * 64 + lane, ec = e < n ? e : n - 1;
#pragma unroll
                for (int k = 0; k < NV; ++k) va[k] = slot_ptr(k)[ec];
            }
#pragma unroll
            for (int k = 0; k < M; ++k)
                if (k == newest) sa.y = va[k];
            const unsigned long long bits = decide(ch, sa);
            multiply(va, bits);
        }
    }

    // this workgroup's record: the waves' blocks added in wave order
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
#pragma unroll
        for (int r = 0; r < 4; ++r) dyn[(wave * NP + k) * 256 + r * 64 + lane] = sum[k][r];
    }
    pginf = wave_max(pginf);
    ynew = wave_sum(ynew);
    if (lane == 0) { red[wave] = pginf; red[NW + wave] = (double)nfixed; red[2 * NW + wave] = ynew; }
    __syncthreads();
    const int NE = gram_entries(m);
    double* part = grampart + (int64_t)blockIdx.x * NE;
    for (int idx = tid; idx < gram_products(m); idx += NT) {
        const int src = idx == tid ? place : block_place(idx);
        double t = dyn[src];
#pragma unroll
        for (int w = 1; w < NW; ++w) t += dyn[w * NP * 256 + src];
        publish(part + kGramHdr + idx, t);
    }
    if (tid < 3) {
        double t = red[tid * NW];
#pragma unroll
        for (int w = 1; w < NW; ++w) t = tid == 0 ? fmax(t, red[w]) : t + red[tid * NW + w];
        publish(part + tid, t);
    }
    double* tot = dyn + gram_tot_at(M);
    // (a record has more entries than the workgroup threads, so only those are added that the pairs held need)
    if (!reduce_partials<NT, true>(grampart, NE, scal, &flag, tot, false, GramPlaces{m, c, base_slot})) return;
    gram_finish<NT, M, true>(tot, dyn, alpha_s, scal, m, c, head, base_slot, op, yn_old, DBG, evaluate_stop, true);
    __syncthreads();
    if (tid == 0 && evaluate_stop) note_progress(op, scal->status);
}

namespace {
constexpr int gram_m_for(int m) { return m <= 5 ? 5 : (m <= 10 ? 10 : (m <= 20 ? 20 : 31)); }
}  // namespace

// Waves per workgroup.  A problem of few chunks has four, so that the matrix cores' work is spread; beyond 64 workgroups their
// records would take the direction kernel more than one round of loads to add.
static int gram_waves_for(int64_t n, int m) { return m > kGramTileM || n <= 64 * 4 * 64 ? 4 : 8; }

int gram_blocks_for(int64_t n, int m, bool few) {
    const int nw = gram_waves_for(n, m);
    const int64_t b = ((n + 63) / 64 + nw - 1) / nw;
    const int64_t cap = n >= kGramLongN && !few ? kGramGroups * kGramGroupMax : kGramOneLevelMax;
    return (int)(b > cap ? cap : b);
}

// (the records of the groups of workgroups, where there are any, lie behind the workgroups')
size_t gram_partial_bytes(int blocks, int m) {
    return (size_t)(blocks + (blocks > kGramOneLevelMax ? kGramGroups : 0)) * gram_entries(m) * 8;
}

bool gram_can_skip_close(const Dims& dm) { return dm.m <= kGramOpenM; }

GramRecords gram_records(const Dims& dm, const Geometry& ge, const Buffers& bf) {
    if (ge.gram_blocks <= kGramOneLevelMax) return GramRecords{bf.grampart, ge.gram_blocks};
    const int gs = (ge.gram_blocks + kGramGroups - 1) / kGramGroups;
    return GramRecords{bf.grampart + (size_t)ge.gram_blocks * gram_entries(dm.m), (ge.gram_blocks + gs - 1) / gs};
}

namespace {

typedef void (*GramKernel)(int64_t, int, Opts, const double*, const double*, const double*, const double*, const double*,
                           const double*, uint8_t*, Scal*, double*, int, int);
GramKernel gram_kernel_for(const Dims& dm, bool dbg, size_t* lds, int* threads) {
    const bool is_long = dm.n >= kGramLongN;
    const int M = gram_m_for(dm.m), nw = gram_waves_for(dm.n, dm.m);
    *lds = M > kGramTileM ? (size_t)gram_lds_doubles(M, nw) * 8 : 0;
    *threads = 64 * nw;
#define LB_GRAM(K, M, NW, LONG) (dbg ? K<M, NW, LONG, true> : K<M, NW, LONG, false>)
    switch (M) {
        case 5: return is_long ? LB_GRAM(k_gram, 5, 8, true) : (nw == 4 ? LB_GRAM(k_gram, 5, 4, false) : LB_GRAM(k_gram, 5, 8, false));
        case 10: return is_long ? LB_GRAM(k_gram, 10, 8, true) : (nw == 4 ? LB_GRAM(k_gram, 10, 4, false) : LB_GRAM(k_gram, 10, 8, false));
        case 20: return is_long ? LB_GRAM(k_gram_blocks, 20, 4, true) : LB_GRAM(k_gram_blocks, 20, 4, false);
        default: return is_long ? LB_GRAM(k_gram_blocks, 31, 4, true) : LB_GRAM(k_gram_blocks, 31, 4, false);
    }
#undef LB_GRAM
}

}  // namespace

// (the limit is a property of the kernel; the hooks' instantiation is prepared by them)
hipError_t gram_prepare(const Dims& dm, int dbg_inputs) {
    size_t lds;
    int threads;
    const GramKernel k = gram_kernel_for(dm, dbg_inputs != 0, &lds, &threads);
    if (lds <= 64 * 1024 - 1024) return hipSuccess;   // (the default, less what the kernel holds besides)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

void launch_gram(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, int dbg_inputs,
                 int evaluate_stop, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1, int no_close) {
    size_t lds;
    int threads;
    const GramKernel k = gram_kernel_for(dm, dbg_inputs != 0, &lds, &threads);
    hipExtLaunchKernelGGL(k, dim3(ge.gram_blocks), dim3(threads), lds, st, ev0, ev1, 0, dm.n, dm.m, op, (const double*)bf.x,
                          (const double*)bf.g, (const double*)bf.l, (const double*)bf.u, (const double*)bf.S, (const double*)bf.Y,
                          bf.mask, bf.scal, bf.grampart, evaluate_stop, no_close);
}

// Transport: rows of 64 columns at least (see the kernel) and long vectors; the quadratic form: vectors that are not; and a direction
// kernel that does the closing step.
bool update_gram_ok(const Dims& dm) {
    if (!gram_can_skip_close(dm)) return false;
    if (dm.kind == LBFGSB_OBJ_QP) return dm.n < kGramLongN;
    return dm.kind == LBFGSB_OBJ_OT_GAUSS && dm.n >= kGramLongN && dm.cols >= 64;
}
void launch_update_gram_form(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, const double* sign, hipStream_t st,
                             const double* fold_rows, const double* fold_weight, int dir_blocks) {
    const int n_fold = fold_rows && dir_folds_extra_rows(dm) ? dm.n_extra : 0, nw = gram_waves_for(dm.n, dm.m);
    const auto k = gram_m_for(dm.m) == 5 ? (nw == 4 ? k_update_gram_form<5, 4> : k_update_gram_form<5, 8>)
                                         : (nw == 4 ? k_update_gram_form<10, 4> : k_update_gram_form<10, 8>);
    hipLaunchKernelGGL(k, dim3(ge.gram_blocks), dim3(64 * nw), 0, st, dm, op, ge.loss_parts, (const double*)bf.losspart, (const double*)bf.t,
                       sign, (const double*)bf.p1, (const double*)bf.p2, (const double*)bf.l, (const double*)bf.u, bf.x, bf.g, bf.S, bf.Y,
                       bf.mask, bf.scal, n_fold, fold_rows, fold_weight, (const double*)bf.redpart, dir_blocks, bf.grampart);
}
void launch_update_gram_gauss(const Dims& dm, const Opts& op, const Geometry& ge, const Buffers& bf, const double* wt, int loss_parts,
                              hipStream_t st) {
    const auto k = gram_m_for(dm.m) == 5 ? (op.uniform_bounds ? k_update_gram_gauss<5, true> : k_update_gram_gauss<5, false>)
                                         : (op.uniform_bounds ? k_update_gram_gauss<10, true> : k_update_gram_gauss<10, false>);
    hipLaunchKernelGGL(k, dim3(ge.gram_blocks), dim3(512), 0, st,
                       dm, op, loss_parts, (const double*)bf.losspart, wt, (const double*)bf.p1, (const double*)bf.p2,
                       (const double*)bf.l, (const double*)bf.u, bf.x, bf.g, bf.S, bf.Y, bf.mask, bf.scal, bf.grampart);
}

// The scalar block into pinned host memory, by NT threads.
template <int NT>
__device__ __forceinline__ void copy_scal(const Scal* scal, Scal* __restrict__ host_scal) {
    constexpr int kWords = (int)(sizeof(Scal) / 8);
    static_assert(sizeof(Scal) % 8 == 0, "copied in 8-byte words");
    for (int k = threadIdx.x; k < kWords; k += NT)
        reinterpret_cast<uint64_t*>(host_scal)[k] = reinterpret_cast<const uint64_t*>(scal)[k];
}
// Applies a pending update when nothing else is about to (before an evaluation from scratch, and
// before the host reads the scalars).  host_scal: where the host reads them, in pinned memory: written by this kernel,
// one wave, instead of by a copy command behind it.
__global__ __launch_bounds__(64) void k_commit(Scal* scal, int m, Scal* __restrict__ host_scal) {
    if (scal->status >= kStatusRefused) return;
    if (threadIdx.x == 0) apply_pending(scal, m);
    if (!host_scal) return;
    __threadfence_block();           // thread 0's stores, before the wave reads the block
    __builtin_amdgcn_wave_barrier();
    copy_scal<64>(scal, host_scal);
}
void launch_commit(const Dims& dm, const Buffers& bf, hipStream_t st, Scal* host_scal) {
    hipLaunchKernelGGL(k_commit, dim3(1), dim3(64), 0, st, bf.scal, dm.m, host_scal);
}

// The same, and a run that ended in convergence is open again: the gradient it was judged by is about to be recomputed
// from x and judged once more.  One launch behind the last step, where the host used to fetch the scalar block, wait, and
// then set the status with a launch of its own.  Against fetching the block first, whole calls: NNLS 3001 x 301 400 -> 390 us,
// 28 inner solves over 8000 x 2000 with one constraint row 8.68 -> 8.30 ms.
__global__ void k_reopen(Scal* scal, int m) {
    if (threadIdx.x != 0) return;
    apply_pending(scal, m);
    if (scal->status == LBFGSB_CONVERGED) scal->status = LBFGSB_RUNNING;
}
void launch_reopen(const Dims& dm, const Buffers& bf, hipStream_t st) {
    hipLaunchKernelGGL(k_reopen, dim3(1), dim3(64), 0, st, bf.scal, dm.m);
}
// The test itself needs four vectors and none of the pair memory: where one workgroup can stream them (kRetestMax), it takes the place
// of a Gram kernel with closing step and recursion (9 us) and hands the scalar block to the host as well (a launch, 4 us);
// k_eval_finish reopens (another).  In Algorithm 4 the kernel between two inner solves makes the test.  Whole calls: NNLS 3001 x 301
// 330 -> 315 us, 28 inner solves over 8000 x 2000 6640 -> 6500.
constexpr int kRetestThreads = 1024;
__global__ __launch_bounds__(kRetestThreads) void k_retest(int64_t n, Opts op, const double* __restrict__ x, const double* __restrict__ g,
                                                           const double* __restrict__ l, const double* __restrict__ u, Scal* scal,
                                                           Scal* __restrict__ host_scal) {
    __shared__ double lds[3 * kRetestThreads / 64];
    if (scal->status == LBFGSB_RUNNING) retest_point<kRetestThreads>(n, op, x, g, l, u, scal, lds);
    if (host_scal) copy_scal<kRetestThreads>(scal, host_scal);
}
void launch_retest(const Dims& dm, const Opts& op, const Buffers& bf, hipStream_t st, Scal* host_scal) {
    hipLaunchKernelGGL(k_retest, dim3(1), dim3(kRetestThreads), 0, st, dm.n, op, (const double*)bf.x, (const double*)bf.g,
                       (const double*)bf.l, (const double*)bf.u, bf.scal, host_scal);
}

}  // namespace lb
