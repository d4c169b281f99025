// What the Gram kernel (gram.hip) and the direction kernel (vec.hip) share: the layout of a workgroup's partial sums, their
// addition in workgroup order, and the closing step -- Gram matrix in the recursion's order, pending update, Algorithm 3 on
// coefficients with the stopping test.  The closing step runs either in the Gram kernel's last workgroup on the scalar block
// itself, or in every workgroup of the direction kernel on a private copy of it.
#pragma once

#include "common.h"
#include "recursion.h"

namespace lb {

// The vectors by static slot: y ring 0 .. m-1 | g m | s ring m+1 .. 2m.  Of the products <a, b>, a <= b, the recursion reads
// those with a <= m; <s, s> is never asked for.  Kept row by row: (0,0) (0,1) .. (0,2m) (1,1) ..
constexpr int kGramHdr = 4;             // a workgroup's record: [0] max KKT residual, [1] #fixed, [2] ||y_new||^2, then the products
constexpr int kGramOneLevelMax = 128;   // grids up to this size add their partials in one level
constexpr int kGramOpenM = 10;          // up to this many pairs the direction kernel can do the closing step itself

__host__ __device__ constexpr int gram_products(int m) { return (m + 1) * (2 * m + 1) - m * (m + 1) / 2; }
__host__ __device__ constexpr int gram_entries(int m) { return kGramHdr + gram_products(m); }

__device__ __forceinline__ void gram_product_slots(int idx, int m, int& a, int& b) {
    int len = 2 * m + 1;
    a = 0;
    while (idx >= len) { idx -= len; --len; ++a; }
    b = a + idx;
}
// The same for many slots, without the walk: row a begins at entry a (4 m + 3 - a)/2, a quadratic whose root the hardware's square
// root hits to within one row.
__device__ __forceinline__ void gram_product_slots_many(int idx, int m, int& a, int& b) {
    const int q = 4 * m + 3;
    a = (int)(((float)q - __builtin_amdgcn_sqrtf((float)(q * q - 8 * idx))) * 0.5f);
    a += (a + 1) * (q - a - 1) / 2 <= idx ? 1 : 0;
    a -= a * (q - a) / 2 > idx ? 1 : 0;
    b = a + idx - a * (q - a) / 2;
}

// Where a record holds what the closing step reads, for c pairs, the oldest in ring slot base_slot: entry i < kGramHdr of the
// statistics, behind them the products of c pairs in the order a ring of c slots that starts with the oldest would have.
struct GramPlaces {
    int m, c, base_slot;
    __device__ __forceinline__ int count() const { return gram_entries(c); }
    __device__ __forceinline__ int operator()(int i) const {
        if (i < kGramHdr) return i;
        int a, b;
        gram_product_slots_many(i - kGramHdr, c, a, b);
        auto slot = [&](int k) -> int {
            if (k == c) return m;
            int ring = base_slot + (k < c ? k : k - c - 1);
            ring -= ring >= m ? m : 0;
            return k < c ? ring : m + 1 + ring;
        };
        const int sa = slot(a), sb = slot(b), lo = sa < sb ? sa : sb, hi = sa < sb ? sb : sa;
        return kGramHdr + lo * (4 * m + 3 - lo) / 2 + hi - lo;
    }
};

// Adds the records of `nwg` workgroups (NE doubles each; entry 0 is a maximum, the others are sums) in workgroup order into
// tot[0 .. NE): thread idx takes entry idx, BATCH records at a time with every load of a batch issued before the first is used and
// none of them under a test (past the last record: the last one again, not added).
// Called by all NT threads; no barrier inside.  The records are of this launch (published).
template <int NT, int BATCH>
__device__ __forceinline__ void gram_sum_batches(const double* __restrict__ grampart, int NE, int nwg, double* tot) {
    for (int idx = threadIdx.x; idx < NE; idx += NT) {
        double sum = 0.0, most = -INFINITY;
        for (int k0 = 0; k0 < nwg; k0 += BATCH) {
            double v[BATCH];
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                const double* r = grampart + (int64_t)(k0 + k < nwg ? k0 + k : nwg - 1) * NE + idx;
                v[k] = observe(r);
            }
#pragma unroll
            for (int k = 0; k < BATCH; ++k) {
                sum += k0 + k < nwg ? v[k] : 0.0;
                most = fmax(most, v[k]);
            }
        }
        tot[idx] = idx == 0 ? most : sum;
    }
}
template <int NT>
__device__ __forceinline__ void gram_sum_partials_flat(const double* __restrict__ grampart, int NE, int nwg, double* tot) {
    // (the trips of different batches to memory follow one another: a batch for all where that is not too many loads)
    if (nwg <= 16) gram_sum_batches<NT, 16>(grampart, NE, nwg, tot);
    else if (nwg <= 32) gram_sum_batches<NT, 32>(grampart, NE, nwg, tot);
    else gram_sum_batches<NT, 64>(grampart, NE, nwg, tot);
}

// For the direction kernel: records of an earlier launch with no more entries than threads, a thread an entry and no loop over them
// (0.4 us of 8.5 there); waves without an entry ask for nothing.
template <int NT, int BATCH>
__device__ __forceinline__ void gram_sum_entry_batches(const double* __restrict__ grampart, int NE, int nwg, double* tot) {
    const int idx = threadIdx.x, at = idx < NE ? idx : NE - 1;
    if (__builtin_amdgcn_readfirstlane(idx & ~63) >= NE) return;
    double sum = 0.0, most = -INFINITY;
    for (int k0 = 0; k0 < nwg; k0 += BATCH) {
        double v[BATCH];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) v[k] = grampart[(int64_t)(k0 + k < nwg ? k0 + k : nwg - 1) * NE + at];
#pragma unroll
        for (int k = 0; k < BATCH; ++k) {
            sum += k0 + k < nwg ? v[k] : 0.0;
            most = fmax(most, v[k]);
        }
    }
    if (idx < NE) tot[idx] = idx == 0 ? most : sum;
}
template <int NT>
__device__ __forceinline__ void gram_sum_entries(const double* __restrict__ grampart, int NE, int nwg, double* tot) {
    static_assert(gram_entries(kGramOpenM) <= NT, "one entry a thread");
    if (nwg <= 16) gram_sum_entry_batches<NT, 16>(grampart, NE, nwg, tot);
    else if (nwg <= 32) gram_sum_entry_batches<NT, 32>(grampart, NE, nwg, tot);
    else gram_sum_entry_batches<NT, 64>(grampart, NE, nwg, tot);
}

// The same beyond 10 pairs, where a record has more entries than the workgroup threads: only those that the pairs held need, entry
// places(i) of the records into tot[i].  Short vectors leave few records, and a thread then asks for PER of its entries at once.
// (A function of its own: one for both made the kernel for 10 pairs 0.4 us longer on short vectors.)  Gram kernel with room for 31
// pairs, 12 held at most, us: every entry of the records added one after the other and its slots found by walking the rows / this:
// n = 500 26.4 / 17.4, 20 000 51.5 / 21.2; 60 steps, 31 held, n = 500 27.7 / 20.3.
template <int NT, int BATCH, int PER>
__device__ __forceinline__ void gram_sum_held_batches(const double* __restrict__ grampart, int NE, int nwg, double* tot,
                                                      const GramPlaces& places) {
    const int count = places.count();
    for (int i0 = threadIdx.x; i0 < count; i0 += NT * PER) {
        double sum[PER], most = -INFINITY;
        int at[PER];
#pragma unroll
        for (int p = 0; p < PER; ++p) {
            sum[p] = 0.0;
            at[p] = places(i0 + p * NT < count ? i0 + p * NT : i0);
        }
        for (int k0 = 0; k0 < nwg; k0 += BATCH) {
            double v[PER][BATCH];
#pragma unroll
            for (int p = 0; p < PER; ++p) {
#pragma unroll
                for (int k = 0; k < BATCH; ++k)   // (at most kGramOneLevelMax records: 32 bits)
                    v[p][k] = observe(grampart + ((k0 + k < nwg ? k0 + k : nwg - 1) * NE + at[p]));
            }
#pragma unroll
            for (int p = 0; p < PER; ++p) {
#pragma unroll
                for (int k = 0; k < BATCH; ++k) {
                    sum[p] += k0 + k < nwg ? v[p][k] : 0.0;
                    if (p == 0) most = fmax(most, v[p][k]);
                }
            }
        }
#pragma unroll
        for (int p = 0; p < PER; ++p)
            if (i0 + p * NT < count) tot[i0 + p * NT] = i0 + p * NT == 0 ? most : sum[p];
    }
}
template <int NT>
__device__ __forceinline__ void gram_sum_held(const double* __restrict__ grampart, int NE, int nwg, double* tot, const GramPlaces& places) {
    if (nwg <= 4) gram_sum_held_batches<NT, 4, 8>(grampart, NE, nwg, tot, places);
    else if (nwg <= 8) gram_sum_held_batches<NT, 8, 4>(grampart, NE, nwg, tot, places);
    else if (nwg <= 16) gram_sum_held_batches<NT, 16, 4>(grampart, NE, nwg, tot, places);
    else if (nwg <= 32) gram_sum_held_batches<NT, 32, 2>(grampart, NE, nwg, tot, places);
    else gram_sum_held_batches<NT, 64, 1>(grampart, NE, nwg, tot, places);
}

// The closing step from the totals tot (HELD: of GramPlaces, else of whole records; LDS, complete: a barrier lies between their last write and this
// call).  c, head: the ring as it will be once the pending update is applied; base_slot: ring slot of the oldest pair.
// Gs: (2 m + 2)^2 doubles, alpha_s: kMaxM + 1 (both LDS).  sc: the scalar block this works on.  mine_a, mine_b (or -1): the
// slots of entry threadIdx.x, when the caller has worked them out while it waited for something.
// MAXK: see recursion_on_coefficients.
template <int NT, int MAXK, bool HELD>
__device__ __forceinline__ void gram_finish(const double* tot, double* Gs, double* alpha_s, Scal* sc, int m,
                                            int c, int head, int base_slot, const Opts& op, double yn_old, int dbg_inputs,
                                            int evaluate_stop, bool record, int mine_a = -1, int mine_b = 0) {
    const int tid = threadIdx.x;
    const int V = 2 * c + 1, Vp = V + 1;
    // The update the previous kernel left pending is applied by the last thread while the others put the matrix
    // together: a chain of two dozen dependent accesses that nothing below the barrier has to wait for twice.  (c and
    // head already are the ring as it will be; the recursion reads the iteration count and the status after the barrier.)
    if (tid == NT - 1) apply_pending(sc, m, record);
    // static slots -> the recursion's order (s oldest..newest, y oldest..newest, g)
    for (int idx = tid; idx < gram_products(HELD ? c : m); idx += NT) {
        int a = mine_a, b = mine_b;
        if (HELD) gram_product_slots_many(idx, c, a, b);
        else if (mine_a < 0 || idx != tid) gram_product_slots(idx, m, a, b);
        auto logical = [&](int slot) -> int {
            if (HELD) return slot == c ? 2 * c : (slot < c ? c + slot : slot - c - 1);
            if (slot == m) return 2 * c;
            const int ring = slot < m ? slot : slot - m - 1;
            const int j = ring >= base_slot ? ring - base_slot : ring - base_slot + m;
            if (j >= c) return -1;
            return slot < m ? c + j : j;
        };
        const int row = logical(a), col = logical(b);
        if (row >= 0 && col >= 0) {
            const double t = tot[kGramHdr + idx];
            Gs[row * Vp + col] = t;
            Gs[col * Vp + row] = t;
        }
    }
    __syncthreads();
    const double gg = Gs[(2 * c) * Vp + 2 * c];   // sum over the free set of g^2
    const double ynew = tot[2];                    // ||y_new||^2 over the full vector: kept for later iterations
    if (tid == 0 && c > 0 && !dbg_inputs) sc->ynorm2[ring_back(head, 1, m)] = ynew;
    recursion_on_coefficients<MAXK>(Gs, Vp, c, head, m, op, sc, gg, tot[0], tot[1], ynew, yn_old, alpha_s, dbg_inputs, evaluate_stop);
}

}  // namespace lb
