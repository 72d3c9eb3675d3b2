// sg_dense.hip -- dense hyper-Ising instances (Sec. VI eq. (5)): at most 64
// spins, couplings over any set of spins with int64 coefficients, e.g. the
// factoring hypergraphs of eqs. (6)-(8), whose terms reach four spins and whose
// coefficients outgrow the sparse kernels' int8/int32 ranges.
//
// One lane per replica, 64 replicas of one instance per wavefront (an item =
// instance, first restart, count).  A lane holds its spins as a 64-bit word
// (bit i set when s_i = -1); the product of the spins of a term t is
// (-1)^popcount(state & mask_t), so a term costs a few integer instructions
// and the term lists, the same for every lane, are read with scalar loads.
//   k_dense_init    random start (the Philox start rule of the sparse path),
//                   energy, replica state reset
//   k_dense_energy  energies of the stored spins
//   k_dense_sweep   colour-ordered sweeps, GREEDY / GREEDY_TIE, the stopping
//                   rule of the sparse path
//   k_dense_fm      the pass-based search (max-gain moves, locking,
//                   hill-climbing, best state of a pass kept); the gains live
//                   in LDS as [spin][lane] and a move updates only the gains of
//                   the spins that share a term with it: flipping s_p changes
//                   the gain of every other member j of a term t by
//                   4 coef_t prod_{k in t} s_k (the product before the flip)
//   k_dense_table_low, k_dense_table_high, k_dense_fm_table
//                   the same search on instances of at most kDenseTableMaxN
//                   spins by a table of all 2^n energies, built by each call
//                   that uses it (see below)
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "sg_device.h"
#include "sg_launch.h"
#include "sg_layout.h"

namespace sg {

constexpr int kDenseThreads = 256;
constexpr int kDenseWaves = kDenseThreads / 64;

__device__ __forceinline__ long long dense_term(uint64_t state, uint64_t m, long long c)
{
    return (__popcll(state & m) & 1) ? -c : c;
}

// f_i = sum over terms holding i of coef * (product of the other members)
__device__ __forceinline__ long long dense_field(const DenseTab& D, uint64_t state, int i)
{
    long long f = 0;
    for (int e = D.dstart[i]; e < D.dstart[i + 1]; ++e) f += dense_term(state, D.dmask[e], D.dcoef[e]);
    return f;
}

__device__ __forceinline__ uint64_t dense_load(const DenseTab& D, int r)
{
    const int8_t* s = D.spins + D.spin_stride * r;
    uint64_t state = 0;
    for (int i = 0; i < D.n; ++i)
        if (s[i] < 0) state |= 1ull << i;
    return state;
}

__device__ __forceinline__ void dense_store(const DenseTab& D, int r, uint64_t state)
{
    int8_t* s = D.spins + D.spin_stride * r;
    for (int i = 0; i < D.n; ++i) s[i] = (int8_t)(((state >> i) & 1ull) ? -1 : 1);
}

// call totals: one atomic per block
__device__ __forceinline__ void dense_totals(CallStats* cs, long long att, long long flips, long long sweeps,
                                             int unconv)
{
    __shared__ unsigned long long b[4];
    if (threadIdx.x < 4) b[threadIdx.x] = 0;
    __syncthreads();
    if (att) atomicAdd(&b[0], (unsigned long long)att);
    if (flips) atomicAdd(&b[1], (unsigned long long)flips);
    if (sweeps) atomicMax(&b[2], (unsigned long long)sweeps);
    if (unconv) atomicAdd(&b[3], 1ull);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (b[0]) atomicAdd(&cs->attempts, b[0]);
        if (b[1]) atomicAdd(&cs->flips, b[1]);
        if (b[2]) atomicMax(&cs->sweeps_max, b[2]);
        if (b[3]) atomicAdd(&cs->unconverged, b[3]);
    }
}

// Energies of 64 replicas (state: each wavefront's lane l holds replica l's)
// by the workgroup's kDenseEWaves wavefronts, each over its share of the terms;
// valid in the first wavefront.  One wavefront alone walks all terms in a
// chain of scalar loads (15000 replicas of 3135 terms: 329 us on 235
// wavefronts).
constexpr int kDenseEWaves = 8;

__device__ __forceinline__ long long dense_energy_shared(const DenseTab& D, uint64_t state)
{
    __shared__ long long part[kDenseEWaves][64];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int t0 = (int)((int64_t)D.nterms * wave / kDenseEWaves), t1 = (int)((int64_t)D.nterms * (wave + 1) / kDenseEWaves);
    long long E = 0;
#pragma unroll 4
    for (int t = t0; t < t1; ++t) E -= dense_term(state, D.tmask[t], D.tcoef[t]);
    part[wave][lane] = E;
    __syncthreads();
    E = 0;
    for (int w = 0; w < kDenseEWaves; ++w) E += part[w][lane];
    return E;
}

// Workgroup k: item k, its replicas on the lanes of every wavefront.
__global__ __launch_bounds__(64 * kDenseEWaves) void k_dense_init(const DenseTab* __restrict__ tabs,
                                                                  const BlockItem* __restrict__ items,
                                                                  RepState* __restrict__ rs, uint64_t seed)
{
    __shared__ unsigned long long first[64];
    const int lane = threadIdx.x & 63;
    const bool lead = threadIdx.x < 64;
    const BlockItem it = items[blockIdx.x];
    const DenseTab D = tabs[it.inst];
    const int r = it.r0 + lane;
    // the draws, split over the wavefronts by spin
    if (lead) first[lane] = 0;
    __syncthreads();
    unsigned long long bits = 0;
    for (int i = (int)(threadIdx.x >> 6); i < D.n; i += kDenseEWaves)
        if (rng_bit(seed, (uint32_t)i, 0xFFFFFFFFu, D.instance_id, (uint32_t)r)) bits |= 1ull << i;
    if (bits) atomicOr(&first[lane], bits);
    __syncthreads();
    const uint64_t state = first[lane];
    RepState z;
    z.E = dense_energy_shared(D, state);
    z.flips = 0;
    z.sweeps = 0;
    z.lastflip = 0;
    z.converged = 0;
    if (lead && lane < it.nr) {
        dense_store(D, r, state);
        rs[D.rep_base + r] = z;
    }
}

__global__ __launch_bounds__(64 * kDenseEWaves) void k_dense_energy(const DenseTab* __restrict__ tabs,
                                                                    const BlockItem* __restrict__ items,
                                                                    int64_t* __restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const BlockItem it = items[blockIdx.x];
    const DenseTab D = tabs[it.inst];
    const int r = it.r0 + min(lane, it.nr - 1);
    const long long E = dense_energy_shared(D, dense_load(D, r));
    if (threadIdx.x < 64 && lane < it.nr) out[D.rep_base + r] = E;
}

template <bool TIE>
__global__ __launch_bounds__(kDenseThreads) void k_dense_sweep(const DenseTab* __restrict__ tabs,
                                                               const BlockItem* __restrict__ items, int nitems,
                                                               RepState* __restrict__ rs, CallStats* __restrict__ cs,
                                                               int max_sweeps, int until_conv, uint64_t seed)
{
    const int item = blockIdx.x * kDenseWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    long long att = 0, nfl = 0, nsw = 0;
    int unconv = 0;
    if (item < nitems) {
        const BlockItem it = items[item];
        const DenseTab D = tabs[it.inst];
        const int r = it.r0 + lane;
        const bool mine = lane < it.nr;
        RepState* st = rs + D.rep_base + (mine ? r : it.r0);
        bool active = mine && !st->converged;
        uint64_t state = mine ? dense_load(D, r) : 0;
        long long E = mine ? st->E : 0;
        const long long sw0 = mine ? st->sweeps : 0;
        int done = 0;
        // every lane walks the same spins in the same order (wave-uniform loops)
        for (int t = 0; t < max_sweeps && __ballot(active); ++t) {
            const uint32_t sweep = (uint32_t)(sw0 + t);
            int F = 0;
            for (int k = 0; k < D.n; ++k) {
                const int i = D.order[k];
                const long long f = dense_field(D, state, i);
                const long long d = ((state >> i) & 1ull) ? -2 * f : 2 * f;
                bool flip = d < 0;
                if (TIE && d == 0 && active)
                    flip = rng_bit(seed, (uint32_t)i, sweep, D.instance_id, (uint32_t)r) != 0;
                if (active && flip) {
                    state ^= 1ull << i;
                    E += d;
                    ++F;
                }
            }
            if (active) {
                ++done;
                nfl += F;
                if (until_conv && F == 0) active = false;
            }
        }
        if (mine && !st->converged) {
            dense_store(D, r, state);
            st->E = E;
            st->sweeps += done;
            st->flips += nfl;
            const bool conv = until_conv && done > 0 && !active;
            if (conv) st->converged = 1;
            att = (long long)done * D.n;
            nsw = done;
            unconv = (until_conv && !conv) ? 1 : 0;
        } else {
            nfl = 0;
        }
    }
    dense_totals(cs, att, nfl, nsw, unconv);
}

__global__ __launch_bounds__(kDenseThreads) void k_dense_fm(const DenseTab* __restrict__ tabs,
                                                            const BlockItem* __restrict__ items, int nitems, int nmax,
                                                            RepState* __restrict__ rs, CallStats* __restrict__ cs,
                                                            int max_passes, int until_conv)
{
    extern __shared__ long long dgain[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int item = blockIdx.x * kDenseWaves + wave;
    long long att = 0, kept = 0, npass = 0;
    int unconv = 0;
    if (item < nitems) {
        const BlockItem it = items[item];
        const DenseTab D = tabs[it.inst];
        const int n = D.n;
        long long* G = dgain + (size_t)wave * nmax * 64;  // G[i * 64 + lane]
        const int r = it.r0 + lane;
        const bool mine = lane < it.nr;
        RepState* st = rs + D.rep_base + (mine ? r : it.r0);
        bool active = mine && !st->converged;
        uint64_t state = mine ? dense_load(D, r) : 0;
        long long E = mine ? st->E : 0;
        int done = 0;
        for (int pass = 0; pass < max_passes && __ballot(active); ++pass) {
            for (int i = 0; i < n; ++i) {
                const long long f = dense_field(D, state, i);
                G[i * 64 + lane] = ((state >> i) & 1ull) ? 2 * f : -2 * f;
            }
            // the wavefront runs the pass for all lanes; a lane that has
            // stopped gets its state back at the end of the pass
            const uint64_t start = state;
            uint64_t locked = 0, best = state;
            const long long Estart = E;
            long long Elow = E;
            int best_len = 0;
            for (int step = 0; step < n; ++step) {
                int pick = -1;
                long long pg = 0;
                for (int i = 0; i < n; ++i) {
                    if ((locked >> i) & 1ull) continue;
                    const long long g = G[i * 64 + lane];
                    if (pick < 0 || g > pg) {
                        pick = i;
                        pg = g;
                    }
                }
                const uint64_t old = state;
                const uint64_t pb = 1ull << pick;
                state ^= pb;
                locked |= pb;
                E -= pg;
                for (int e = D.dstart[pick]; e < D.dstart[pick + 1]; ++e) {
                    uint64_t m = D.dmask[e];
                    const long long delta = 4 * dense_term(old, m | pb, D.dcoef[e]);
                    while (m) {
                        const int j = __builtin_ctzll(m);
                        m &= m - 1;
                        G[j * 64 + lane] += delta;
                    }
                }
                if (E < Elow) {
                    Elow = E;
                    best = state;
                    best_len = step + 1;
                }
            }
            if (active) {
                state = best;
                E = Elow;
                ++done;
                kept += best_len;
                if (until_conv && !(Elow < Estart)) active = false;
            } else {
                state = start;
                E = Estart;
            }
        }
        if (mine && !st->converged) {
            dense_store(D, r, state);
            st->E = E;
            st->sweeps += done;
            st->flips += kept;
            const bool conv = until_conv && done > 0 && !active;
            if (conv) st->converged = 1;
            att = (long long)done * n;
            npass = done;
            unconv = (until_conv && !conv) ? 1 : 0;
        } else {
            kept = 0;
        }
    }
    dense_totals(cs, att, kept, npass, unconv);
}

// ---------------------------------------------------------------------------
// The pass-based search by a table of energies.  E(s) = -sum_t coef_t
// (-1)^popcount(s & mask_t) over all 2^n states is the Walsh-Hadamard transform
// of -coef laid out by mask: n 2^n additions instead of a term evaluation per
// (state, term).  With it the gain of moving spin i is E(s) - E(s with bit i
// flipped), so a move is one round of n independent 8-byte reads per replica
// and the choice of the smallest, instead of the picked spin's terms (560 of
// them with 10 + 10 factor bits), each updating three gains in LDS.
//
// Bound by the latency of its serial moves: 20 spins, 3135 terms, 15000
// replicas to convergence (6 passes at most): 32 us for the table (8 MB) and
// 170 us for the search, 1.4 us a step, against 30.5 ms for k_dense_fm.

constexpr int kDenseTileBits = 11;  // spins of one LDS tile of the low transform (16 KB)
constexpr int kDenseTileCols = 8;   // columns of the high transform's tile (64-byte rows)

// Spins 0 .. 10: tile x of instance inst0 + y, states with high bits x.
__global__ __launch_bounds__(256) void k_dense_table_low(const DenseTab* __restrict__ tabs, int inst0,
                                                         long long* __restrict__ table, int nmax)
{
    __shared__ long long tile[1 << kDenseTileBits];
    const DenseTab D = tabs[inst0 + blockIdx.y];
    const int low = min(D.n, kDenseTileBits), size = 1 << low;
    if (blockIdx.x >> (D.n - low)) return;
    for (int k = threadIdx.x; k < size; k += 256) tile[k] = 0;
    __syncthreads();
    for (int t = threadIdx.x; t < D.nterms; t += 256) {
        const uint64_t m = D.tmask[t];
        if ((m >> low) == blockIdx.x) tile[m & (uint64_t)(size - 1)] = -D.tcoef[t];
    }
    for (int b = 0; b < low; ++b) {
        __syncthreads();
        for (int k = threadIdx.x; k < size / 2; k += 256) {
            const int a = (k >> b << (b + 1)) | (k & ((1 << b) - 1)), c = a | 1 << b;
            const long long x = tile[a], y = tile[c];
            tile[a] = x + y;
            tile[c] = x - y;
        }
    }
    __syncthreads();
    long long* out = table + ((size_t)blockIdx.y << nmax) + ((size_t)blockIdx.x << low);
    for (int k = threadIdx.x; k < size; k += 256) out[k] = tile[k];
}

// The spins from 11 up: columns 8 x .. 8 x + 7 of the rows of 2^11 states.
// Dynamic LDS: 64 bytes per row of the largest instance.
__global__ __launch_bounds__(256) void k_dense_table_high(const DenseTab* __restrict__ tabs, int inst0,
                                                          long long* __restrict__ table, int nmax)
{
    extern __shared__ long long rows[];
    const int n = tabs[inst0 + blockIdx.y].n, hb = n - kDenseTileBits;
    if (hb <= 0) return;
    long long* T = table + ((size_t)blockIdx.y << nmax) + blockIdx.x * kDenseTileCols;
    const int size = kDenseTileCols << hb;
    for (int k = threadIdx.x; k < size; k += 256)
        rows[k] = T[((size_t)(k / kDenseTileCols) << kDenseTileBits) + k % kDenseTileCols];
    for (int b = 3; b < 3 + hb; ++b) {  // element index: row * 8 + column
        __syncthreads();
        for (int k = threadIdx.x; k < size / 2; k += 256) {
            const int a = (k >> b << (b + 1)) | (k & ((1 << b) - 1)), c = a | 1 << b;
            const long long x = rows[a], y = rows[c];
            rows[a] = x + y;
            rows[c] = x - y;
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < size; k += 256)
        T[((size_t)(k / kDenseTileCols) << kDenseTileBits) + k % kDenseTileCols] = rows[k];
}

// Workgroup (one wavefront) k: item k, a replica per lane; instance inst's
// table is number inst - inst0.
__global__ __launch_bounds__(64) void k_dense_fm_table(const DenseTab* __restrict__ tabs,
                                                       const BlockItem* __restrict__ items, int inst0,
                                                       const long long* __restrict__ table, int nmax,
                                                       RepState* __restrict__ rs, CallStats* __restrict__ cs,
                                                       int max_passes, int until_conv)
{
    static_assert(kDenseTableMaxN <= 24, "three groups of eight neighbours");
    const int lane = threadIdx.x;
    const BlockItem it = items[blockIdx.x];
    const DenseTab D = tabs[it.inst];
    const int n = D.n;
    const long long* T = table + ((size_t)(it.inst - inst0) << nmax);
    const int r = it.r0 + lane;
    const bool mine = lane < it.nr;
    RepState* st = rs + D.rep_base + (mine ? r : it.r0);
    bool active = mine && !st->converged;
    const bool ran = active;
    uint32_t state = active ? (uint32_t)dense_load(D, r) : 0u;
    long long E = active ? st->E : 0, att = 0, kept = 0;
    int done = 0;
    for (int pass = 0; pass < max_passes && __ballot(active); ++pass) {
        if (!active) continue;
        uint32_t cur = state, open = n == 32 ? ~0u : (1u << n) - 1u, best = state;
        long long Elow = E;
        int best_len = 0;
        for (int step = 0; step < n; ++step) {
            long long v[24];
#pragma unroll
            for (int c = 0; c < 24; c += 8)
                if (c < n)
#pragma unroll
                    for (int u = c; u < c + 8; ++u) v[u] = T[cur ^ (1u << min(u, n - 1))];
            // the open spin whose move leads lowest, the lowest index among equals
            int pick = 0;
            long long low = INT64_MAX;
#pragma unroll
            for (int c = 0; c < 24; c += 8)
                if (c < n)
#pragma unroll
                    for (int u = c; u < c + 8; ++u)
                        if (((open >> u) & 1u) & (uint32_t)(v[u] < low)) {
                            low = v[u];
                            pick = u;
                        }
            cur ^= 1u << pick;
            open &= ~(1u << pick);
            if (low < Elow) {
                Elow = low;
                best = cur;
                best_len = step + 1;
            }
        }
        if (until_conv && !(Elow < E)) active = false;
        state = best;
        E = Elow;
        ++done;
        kept += best_len;
    }
    int unconv = 0;
    if (ran) {
        dense_store(D, r, state);
        st->E = E;
        st->sweeps += done;
        st->flips += kept;
        const bool conv = until_conv && done > 0 && !active;
        if (conv) st->converged = 1;
        att = (long long)done * n;
        unconv = (until_conv && !conv) ? 1 : 0;
    }
    dense_totals(cs, att, kept, done, unconv);
}

// ---------------------------------------------------------------------------

hipError_t launch_dense_init(const DenseTab* tabs, const BlockItem* items, int nitems, RepState* rs, uint64_t seed,
                             hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dense_init, dim3(nitems), dim3(64 * kDenseEWaves), 0, st, tabs, items, rs, seed);
    return hipGetLastError();
}

hipError_t launch_dense_energy(const DenseTab* tabs, const BlockItem* items, int nitems, int64_t* out, hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_dense_energy, dim3(nitems), dim3(64 * kDenseEWaves), 0, st, tabs, items, out);
    return hipGetLastError();
}

hipError_t launch_dense_run(const DenseTab* tabs, const BlockItem* items, int nitems, int nmax, RepState* rs,
                            CallStats* cs, int rule, int max_sweeps, int until_conv, uint64_t seed, hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    const dim3 grid((nitems + kDenseWaves - 1) / kDenseWaves);
    if (rule == 2) {
        const size_t lds = (size_t)kDenseWaves * nmax * 64 * 8;
        hipError_t e = hipFuncSetAttribute((const void*)k_dense_fm, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_dense_fm, grid, dim3(kDenseThreads), lds, st, tabs, items, nitems, nmax, rs, cs,
                           max_sweeps, until_conv);
    } else if (rule == 1) {
        hipLaunchKernelGGL(k_dense_sweep<true>, grid, dim3(kDenseThreads), 0, st, tabs, items, nitems, rs, cs,
                           max_sweeps, until_conv, seed);
    } else {
        hipLaunchKernelGGL(k_dense_sweep<false>, grid, dim3(kDenseThreads), 0, st, tabs, items, nitems, rs, cs,
                           max_sweeps, until_conv, seed);
    }
    return hipGetLastError();
}

hipError_t launch_dense_fm_table(const DenseTab* tabs, int inst0, int ninst, const BlockItem* items, int nitems,
                                 int64_t* table, int nmax, RepState* rs, CallStats* cs, int max_passes, int until_conv,
                                 hipStream_t st)
{
    if (nitems <= 0 || ninst <= 0) return hipSuccess;
    if (nmax < 1 || nmax > kDenseTableMaxN || ninst > 65535) return hipErrorInvalidValue;
    long long* T = reinterpret_cast<long long*>(table);
    const int hb = std::max(0, nmax - kDenseTileBits);
    hipLaunchKernelGGL(k_dense_table_low, dim3(1u << hb, ninst), dim3(256), 0, st, tabs, inst0, T, nmax);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (hb > 0) {
        const int lds = (kDenseTileCols * 8) << hb;
        e = hipFuncSetAttribute((const void*)k_dense_table_high, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_dense_table_high, dim3((1 << kDenseTileBits) / kDenseTileCols, ninst), dim3(256), lds, st,
                           tabs, inst0, T, nmax);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_dense_fm_table, dim3(nitems), dim3(64), 0, st, tabs, items, inst0, T, nmax, rs, cs,
                       max_passes, until_conv);
    return hipGetLastError();
}

}  // namespace sg
