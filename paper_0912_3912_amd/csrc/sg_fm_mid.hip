// sg_fm_mid.hip -- the paper's pass-based local search with hill-climbing
// (Sec. IV, Fig. 3) on instances of more than 4096 spins whose half-gains fit
// one compute unit's LDS: one wavefront per replica.  The pass, its tie-break,
// best prefix, stopping rule and counters are those of the other pass kernels
// (sg_fm.hip); what is larger runs on k_fm_big (sg_fm_big.hip), whose term
// rows (FmbRows, external order), slots and replica counter this kernel
// shares.
//
// Per wavefront in LDS: the half-gains v_e = -s_e f_e, as int32, or as bytes
// v + 128 (0: locked) where every spin's sum of |coefficients| is at most 127,
// the spins as bits, and the maxima of the leaves of 256 spins (four per
// lane), which fmcore::run_pass moves the spins by.  The move list goes to the
// slot in device memory (stored without a wait, read when the pass ends).
//
// The kernel is bound by the latency of its serial chain of moves, of which
// the mover's row, read from device memory (the rows of an instance stay in
// the L2), is one link: about 300 of the 1600 cycles a move takes.  Four
// passes of 64 replicas on a 164 x 164 +-J lattice take 73 ms, 0.68 us a move,
// against 403 ms on k_fm_big; 2048 replicas of a 20000-spin graph with
// hyper-couplings one pass in 58 ms against 291 ms.  Asking ahead for the row
// of the best spin outside the stale leaves (76.6 ms: the next move is mostly
// in a stale leaf, and its row then waits behind that one), and touching the
// partners' rows (74.0 ms), were measured and left out.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "sg_fm_core.h"
#include "sg_launch.h"
#include "sg_layout.h"

namespace sg {

namespace {

constexpr int kLeaf = 256;

// The row table as device memory (its pointer comes from a table in memory,
// so the compiler would otherwise address it as generic memory).
typedef __attribute__((address_space(1))) const uint32_t mid_g32;

__host__ __device__ inline size_t mid_pad(int n) { return ((size_t)n + kLeaf - 1) / kLeaf * kLeaf; }

// The replica's LDS state and the rows, as fmcore::run_pass wants them.  The
// byte form's words take several lanes' changes in one addition: the bytes
// before and after a move lie in 1..255 (or stay 0), so the sum of their
// changes leaves the neighbours as they are.
template <bool BYTES, int RL, bool TRI>
struct MidPolicy {
    static constexpr int kRL = RL;
    static constexpr bool kTri = TRI, kPlaced = false;
    static constexpr int32_t kNone = BYTES ? 0 : INT32_MIN, kBias = BYTES ? 128 : 0;
    mid_g32* rows;
    uint8_t* half;
    uint32_t* bits;
    int2* lf;
    int32_t* moves;
    int dc_, tt_, stride, lane, qc;  // qc: where this lane's coupling stands in a row
    bool wide;

    static constexpr int32_t kLocked = kNone;
    __device__ __forceinline__ void tag(int e, int step)
    {
        if (lane == 0) {
            set(e, kNone);
            moves[step] = e;
        }
    }
    __device__ __forceinline__ void row(int e, int& j, int32_t& J) const
    {
        mid_g32* r = rows + (int64_t)e * stride + qc;
        const uint32_t w = r[0];
        if (!wide) {
            j = (int)(w >> 8);
            J = (int8_t)(w & 0xffu);
        } else {
            j = (int)w;
            J = (int32_t)r[1];
        }
    }

    __device__ __forceinline__ int dc() const { return dc_; }
    __device__ __forceinline__ int tt() const { return tt_; }
    __device__ __forceinline__ int spin(int e) const { return 1 - 2 * (int)((bits[e >> 5] >> (e & 31)) & 1u); }
    __device__ __forceinline__ int32_t v(int e) const
    {
        if constexpr (BYTES) return half[e];
        else return reinterpret_cast<const int32_t*>(half)[e];
    }
    __device__ __forceinline__ void set(int e, int32_t x)
    {
        if constexpr (BYTES) half[e] = (uint8_t)x;
        else reinterpret_cast<int32_t*>(half)[e] = x;
    }
    __device__ __forceinline__ void add(int e, int32_t d)
    {
        if constexpr (BYTES) atomicAdd(reinterpret_cast<uint32_t*>(half) + (e >> 2), (uint32_t)d << (8 * (e & 3)));
        else atomicAdd(reinterpret_cast<int32_t*>(half) + e, d);
    }
    __device__ __forceinline__ void lock(int e, int, int step)
    {
        set(e, kNone);
        atomicXor(bits + (e >> 5), 1u << (e & 31));
        moves[step] = e;
    }
    __device__ __forceinline__ int leaf(int e) const { return e >> 8; }
    __device__ __forceinline__ int2 leaf_max(int g) const { return lf[g]; }
    __device__ __forceinline__ void set_leaf(int g, int32_t m, int32_t a) { lf[g] = make_int2(m, a); }
    __device__ __forceinline__ void coupling(int e, int q, int& j, int32_t& J) const
    {
        mid_g32* row = rows + (int64_t)e * stride;
        const bool in = q < dc_;
        if (!wide) {
            uint32_t w = row[in ? 1 + q : 0];
            w = in ? w : 0u;
            j = (int)(w >> 8);
            J = (int8_t)(w & 0xffu);
        } else {
            const uint32_t w0 = row[in ? 1 + 2 * q : 0], w1 = row[in ? 2 + 2 * q : 0];
            j = in ? (int)w0 : 0;
            J = in ? (int32_t)w1 : 0;
        }
    }
    __device__ __forceinline__ void triple(int e, int q, int& a, int& b, int32_t& K) const
    {
        mid_g32* row = rows + (int64_t)e * stride;
        const bool in = q < tt_;
        if (!wide) {
            mid_g32* t = row + (in ? 1 + dc_ + 2 * q : 0);
            uint32_t w = t[0];
            const uint32_t w1 = t[in ? 1 : 0];
            w = in ? w : 0u;
            a = (int)(w >> 8);
            b = in ? (int)w1 : 0;
            K = (int8_t)(w & 0xffu);
        } else {
            mid_g32* t = row + (in ? 1 + 2 * dc_ + 3 * q : 0);
            const uint32_t w0 = t[0], w1 = t[in ? 1 : 0], w2 = t[in ? 2 : 0];
            a = in ? (int)w0 : 0;
            b = in ? (int)w1 : 0;
            K = in ? (int32_t)w2 : 0;
        }
    }
    // lane l's spins of a leaf are its 4 l .. 4 l + 3
    using Word = std::conditional_t<BYTES, uint32_t, int4>;
    __device__ __forceinline__ Word fetch(int g) const { return reinterpret_cast<const Word*>(half)[g * 64 + lane]; }
    __device__ __forceinline__ void part(const Word w, int32_t& x, int32_t& at) const
    {
        if constexpr (BYTES) {
            const uint32_t t0 = (w & 255u) << 2 | 3u, t1 = (w >> 8 & 255u) << 2 | 2u;
            const uint32_t t2 = (w >> 16 & 255u) << 2 | 1u, t3 = w >> 24 << 2;
            const uint32_t t = max(max(t0, t1), max(t2, t3));
            x = (int32_t)(t >> 2);
            at = (int32_t)(3u - (t & 3u));
        } else {
            x = max(max(w.x, w.y), max(w.z, w.w));
            at = w.x == x ? 0 : w.y == x ? 1 : w.z == x ? 2 : 3;
        }
    }
    __device__ __forceinline__ void load(int g, int32_t& x, int32_t& at) const { part(fetch(g), x, at); }
    __device__ __forceinline__ int index(int g, int o, int32_t at) const
    {
        return g * kLeaf + 4 * o + __builtin_amdgcn_readlane(at, o);
    }
};

}  // namespace

// Grid: one 64-thread workgroup per slot; a wavefront takes replicas from
// *counter.  Dynamic LDS: fm_mid_lds_bytes of the largest instance.
template <bool BYTES, int RL, bool TRI>
__global__ __launch_bounds__(64) void k_fm_mid(const InstTab* __restrict__ tab, const FmbRows* __restrict__ rows,
                                               const QueueItem* __restrict__ items, int nitems,
                                               uint32_t* __restrict__ counter, int32_t* __restrict__ moves_all,
                                               int64_t slot_spins, RepState* __restrict__ rs,
                                               CallStats* __restrict__ cs, uint32_t* __restrict__ err, int max_passes,
                                               int until_conv)
{
    extern __shared__ __align__(16) uint8_t mid_lds[];
    const int lane = threadIdx.x;
    long long att = 0, kept_all = 0, passes_max = 0, unconv = 0;
    for (;;) {
        int k = 0;
        if (lane == 0) k = (int)atomicAdd(counter, 1u);
        k = __builtin_amdgcn_readfirstlane(k);
        if (k >= nitems) break;
        const QueueItem it = items[k];
        const InstTab& Q = tab[it.inst];
        const FmbRows Rw = rows[it.inst];
        RepState* st = rs + Q.rep_base + it.r;
        if (st->converged) continue;
        const int n = Q.I.n;
        const int pad = (int)mid_pad(n), G = pad / kLeaf;
        int8_t* sp = Q.spins + Q.spin_stride * it.r;
        const uint32_t* ext = Q.I.ext;
        using P = MidPolicy<BYTES, RL, TRI>;
        P p;
        p.rows = (mid_g32*)Rw.rows;
        p.half = mid_lds;
        p.bits = reinterpret_cast<uint32_t*>(mid_lds + (size_t)pad * (BYTES ? 1 : 4));
        p.lf = reinterpret_cast<int2*>(p.bits + pad / 32);
        p.moves = moves_all + (int64_t)blockIdx.x * slot_spins;
        p.dc_ = Rw.dc;
        p.tt_ = Rw.tt;
        p.stride = Rw.stride;
        p.lane = lane;
        p.wide = Rw.wide != 0;
        p.qc = lane < p.dc_ ? 1 + lane * (p.wide ? 2 : 1) : 1;
        const bool pairs = !TRI && p.dc_ > 0 && p.dc_ <= 64;  // the shorter move loop
        for (int i = lane; i < pad / 32; i += 64) p.bits[i] = 0u;
        fmcore::order();
        for (int i = lane; i < n; i += 64)
            if (sp[i] < 0) {
                const uint32_t e = ext[i];
                atomicOr(p.bits + (e >> 5), 1u << (e & 31u));
            }
        fmcore::order();
        const long long E0 = st->E;  // the same in every lane: kept in scalar registers
        long long Estar = (long long)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(E0 >> 32)) << 32 |
                                      (uint32_t)__builtin_amdgcn_readfirstlane((int)E0));
        long long kept = 0;
        int passes = 0;
        bool conv = false, bad = false;
        for (int pass = 0; pass < max_passes; ++pass) {
            // half-gains from the definition, a leaf at a time (every partial
            // sum of a field is within the spin's sum of |coefficients|)
            fmcore::Leaves<RL> mx, ix;
#pragma unroll
            for (int i = 0; i < RL; ++i) {
                mx[i] = P::kNone;
                ix[i] = 0;
            }
            for (int g = 0; g < G; ++g) {
                int32_t f[4];
                mid_g32* row[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = g * kLeaf + u * 64 + lane;
                    row[u] = p.rows + (int64_t)(e < n ? e : 0) * p.stride;
                    f[u] = p.wide ? (int32_t)row[u][0] : (int32_t)(int8_t)(row[u][0] & 0xffu);
                }
                if (!p.wide)
                    for (int q = 0; q < p.dc_; ++q)
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const uint32_t w = row[u][1 + q];
                            f[u] += (int)(int8_t)(w & 0xffu) * p.spin((int)(w >> 8));
                        }
                else
                    for (int q = 0; q < p.dc_; ++q)
#pragma unroll
                        for (int u = 0; u < 4; ++u) f[u] += (int32_t)row[u][2 + 2 * q] * p.spin((int)row[u][1 + 2 * q]);
                if (TRI)
                    for (int q = 0; q < p.tt_; ++q)
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int e = g * kLeaf + u * 64 + lane;
                            int a, b;
                            int32_t K;
                            p.triple(e < n ? e : 0, q, a, b, K);
                            f[u] += K * p.spin(a) * p.spin(b);
                        }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int e = g * kLeaf + u * 64 + lane;
                    p.set(e, e < n ? P::kBias - p.spin(e) * f[u] : P::kNone);
                }
                fmcore::order();
                int32_t x[1], at, m[1];
                p.load(g, x[0], at);
                fmcore::wave_max<1>(x, m);
                const int a = p.index(g, fmcore::first_lane(x[0] == m[0]), at);
#pragma unroll
                for (int i = 0; i < RL; ++i) {
                    const bool mine = lane * RL + i == g;
                    mx[i] = mine ? m[0] : mx[i];
                    ix[i] = mine ? a : ix[i];
                }
            }
#pragma unroll
            for (int i = 0; i < RL; ++i) p.lf[lane * RL + i] = make_int2(mx[i], ix[i]);
            fmcore::order();
            long long Elow = Estar;
            int len;
            if (pairs) {
                if constexpr (!TRI) len = fmcore::run_pass_pairs(p, n, lane, Elow, mx, ix);
            } else {
                len = fmcore::run_pass(p, n, lane, Elow, mx, ix);
            }
            if (len < 0) {
                bad = true;
                break;
            }
            // the move list's stores are complete before it is read
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
            // make the moves of the best prefix, or undo those after it
            for (int t = (pairs ? 0 : len) + lane; t < (pairs ? len : n); t += 64) {
                const int e = p.moves[t];
                atomicXor(p.bits + (e >> 5), 1u << (e & 31));
            }
            fmcore::order();
            ++passes;
            kept += len;
            const bool improved = Elow < Estar;
            Estar = Elow;
            if (until_conv && !improved) {
                conv = true;
                break;
            }
        }
        if (bad) {
            if (lane == 0) atomicOr(err, 1u);
            continue;
        }
        for (int i = lane; i < n; i += 64) sp[i] = (int8_t)p.spin((int)ext[i]);
        if (lane == 0) {
            st->E = Estar;
            st->sweeps += passes;
            st->flips += kept;
            if (conv) st->converged = 1;
        }
        att += (long long)passes * n;
        kept_all += kept;
        passes_max = passes > passes_max ? passes : passes_max;
        unconv += (until_conv && !conv) ? 1 : 0;
        fmcore::order();
    }
    if (lane == 0 && (att || unconv)) {
        atomicAdd(&cs->attempts, (unsigned long long)att);
        atomicAdd(&cs->flips, (unsigned long long)kept_all);
        atomicMax(&cs->sweeps_max, (unsigned long long)passes_max);
        atomicAdd(&cs->unconverged, (unsigned long long)unconv);
    }
}

// Leaves per lane of an instance: a power of two, 64 lanes of leaves of 256 spins.
static int mid_rl(int n)
{
    int rl = 1;
    while (64 * kLeaf * rl < n) rl *= 2;
    return rl;
}

size_t fm_mid_lds_bytes(int n, bool bytes)
{
    return mid_pad(n) * (bytes ? 1 : 4) + mid_pad(n) / 8 + (size_t)mid_rl(n) * 64 * 8;
}

int fm_mid_max_n(bool bytes)
{
    // 160 KB: 8 leaves per lane of byte half-gains take 148 KB; int32 ones
    // reach 39168 spins
    return bytes ? 8 * 64 * kLeaf : 39168;
}

template <bool BYTES, int RL, bool TRI>
static hipError_t launch_mid_t(const InstTab* tab, const FmbRows* rows, const QueueItem* items, int nitems,
                               uint32_t* counter, int32_t* moves, int64_t slot_spins, int slots, size_t lds,
                               RepState* rs, CallStats* cs, uint32_t* err, int max_passes, int until_conv,
                               hipStream_t st)
{
    hipError_t e = hipFuncSetAttribute((const void*)k_fm_mid<BYTES, RL, TRI>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_fm_mid<BYTES, RL, TRI>), dim3((unsigned)std::min(slots, nitems)), dim3(64), lds, st, tab,
                       rows, items, nitems, counter, moves, slot_spins, rs, cs, err, max_passes, until_conv);
    return hipGetLastError();
}

hipError_t launch_fm_mid(const InstTab* tab, const FmbRows* rows, const QueueItem* items, int nitems, int nmax,
                         bool bytes, bool tri, uint32_t* counter, int32_t* moves, int64_t slot_spins, int slots,
                         RepState* rs, CallStats* cs, uint32_t* err, int max_passes, int until_conv, hipStream_t st)
{
    if (nitems <= 0 || slots <= 0) return hipSuccess;
    if (nmax > fm_mid_max_n(bytes)) return hipErrorInvalidValue;
    const size_t lds = fm_mid_lds_bytes(nmax, bytes);
    const int rl = mid_rl(nmax);
    auto go = [&](auto b, auto t) -> hipError_t {
        constexpr bool B = decltype(b)::value, T = decltype(t)::value;
        switch (rl) {
        case 1:
            return launch_mid_t<B, 1, T>(tab, rows, items, nitems, counter, moves, slot_spins, slots, lds, rs, cs, err,
                                         max_passes, until_conv, st);
        case 2:
            return launch_mid_t<B, 2, T>(tab, rows, items, nitems, counter, moves, slot_spins, slots, lds, rs, cs, err,
                                         max_passes, until_conv, st);
        case 4:
            return launch_mid_t<B, 4, T>(tab, rows, items, nitems, counter, moves, slot_spins, slots, lds, rs, cs, err,
                                         max_passes, until_conv, st);
        default:
            if constexpr (B)
                return launch_mid_t<B, 8, T>(tab, rows, items, nitems, counter, moves, slot_spins, slots, lds, rs, cs,
                                             err, max_passes, until_conv, st);
            else
                return hipErrorInvalidValue;
        }
    };
    if (bytes) return tri ? go(std::true_type{}, std::true_type{}) : go(std::true_type{}, std::false_type{});
    return tri ? go(std::false_type{}, std::true_type{}) : go(std::false_type{}, std::false_type{});
}

}  // namespace sg
