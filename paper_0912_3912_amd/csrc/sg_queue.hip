// sg_queue.hip -- the persistent queue schedule for many instances of uneven
// size: workgroups take (instance, restart) items from a queue sorted by
// decreasing size.  Large items run on the whole workgroup (sg_team_core.h:
// rows of the sliced layout on lanes, couplings streamed from memory a slice
// ahead, spins in LDS as bytes); small items run one per wavefront in a
// private LDS window, 16 at a time.  Items that would outlast the rest run on
// teams of workgroups first (QueueTeams).  Bound by the largest items: 96 graphs
// with triples of 100 to 100000 spins, 8 restarts each, 0.83 to 1.04 ms over
// eight seeds (0.97 to 1.23 without teams; 2.43 with loads under branches and an
// LDS wait per coupling).
// Each replica runs to its own stopping point, and the replica state and the
// call totals follow the per-phase kernels exactly: with until_converged a
// replica stops after its first sweep without a flip (that sweep counts).
// A sweep without a flip evaluates every spin on the final configuration, so
// its fields also give the replica's exact energy, which is then stored
// instead of the running sum (the start energy is not needed for it).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "sg_device.h"
#include "sg_launch.h"
#include "sg_layout.h"
#include "sg_team_core.h"

namespace sg {

__device__ __forceinline__ int bat_j(uint32_t w) { return (int)(int8_t)(w & 0xffu); }

constexpr int kBatThreads = kTeamThreads;
constexpr int kBatWaves = kBatThreads / 64;

// ---------------------------------------------------------------------------
// k_queue

// One colour phase of one replica on one wavefront: lane = row of a slice,
// couplings from memory, spins in LDS.  All coupling and hyper-coupling words
// of a slice (up to kPreW and kPreT of them, predicated on the slice's widths)
// are loaded before any is used, so a wavefront keeps a whole slice's loads in
// flight.  The slice descriptors are read with scalar loads one slice ahead
// and the instance arrays addressed as device memory.
constexpr int kPreW = 16, kPreT = 8;

struct SliceWords {
    uint32_t w[kPreW];
    uint32_t a[kPreT], b[kPreT];
    int h;
};

// Device-memory views of the instance arrays (the pointers come from the
// instance table, so the compiler would otherwise address them as generic
// memory, whose loads also hold up every LDS wait), and a read-only view of
// the slice table for loads at wavefront-uniform addresses (scalar loads).
typedef __attribute__((address_space(1))) const uint32_t q_g32;
typedef __attribute__((address_space(1))) const int8_t q_gi8;
typedef uint32_t q_v4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) const q_v4 q_kslice;

__device__ __forceinline__ q_v4 queue_slice_raw(const Slice* slices, int sl) { return *(q_kslice*)(slices + sl); }

__device__ __forceinline__ Slice queue_unpack(q_v4 v)
{
    Slice S;
    S.row0 = v.x;
    S.ebase = v.y;
    S.tbase = v.z;
    S.ew = (uint16_t)(v.w & 0xFFFFu);
    S.tw = (uint8_t)((v.w >> 16) & 0xFFu);
    S.rows = (uint8_t)(v.w >> 24);
    return S;
}

// A pointer the whole wavefront holds, in scalar registers.
template <class T>
__device__ __forceinline__ T* queue_uniform(T* p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (T*)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ void queue_load(const InstDev& I, const Slice& S, int lane, SliceWords& L)
{
    const bool row = lane < S.rows;
    q_g32* p = (q_g32*)I.nbr + S.ebase + lane;
#pragma unroll
    for (int k = 0; k < kPreW; ++k) L.w[k] = (row && k < S.ew) ? p[k * kSlice] : 0u;
    if (I.has_tri) {
        q_g32* pa = (q_g32*)I.ta + S.tbase + lane;
        q_g32* pb = (q_g32*)I.tb + S.tbase + lane;
#pragma unroll
        for (int q = 0; q < kPreT; ++q) {
            L.a[q] = (row && q < S.tw) ? pa[q * kSlice] : 0u;
            L.b[q] = (row && q < S.tw) ? pb[q * kSlice] : 0u;
        }
    }
    L.h = row ? (int)((q_gi8*)I.h)[S.row0 + lane] : 0;
}

// Energy from one sweep's fields: with f1 = h_i + (coupling part) and f the
// whole field, sum_i s_i (3 h_i + f1_i + 2 f_i) = 6 (sum h s + sum_{i<j} J s s
// + sum K s s s) = -6 E, each pair counted twice and each triple three times
// in the fields (Sec. II eq. (1), Sec. VI eq. (5)).
template <bool TIE>
__device__ __forceinline__ void queue_eval(const InstDev& I, const Slice& S, const SliceWords& L,
                                           int8_t* __restrict__ sp, int lane, uint32_t sweep, uint64_t seed,
                                           uint32_t r, long long& dE, int& my, long long& e6)
{
    if (lane >= S.rows) return;
    const int i = S.row0 + lane;
    int f = L.h;
#pragma unroll
    for (int k = 0; k < kPreW; ++k)
        if (k < S.ew) f += bat_j(L.w[k]) * sp[L.w[k] >> 8];
    if (S.ew > kPreW) {
        q_g32* p = (q_g32*)I.nbr + S.ebase + lane;
        for (int k = kPreW; k < S.ew; ++k) {
            const uint32_t w1 = p[k * kSlice];
            f += bat_j(w1) * sp[w1 >> 8];
        }
    }
    const int f1 = f;
    if (I.has_tri) {
#pragma unroll
        for (int q = 0; q < kPreT; ++q)
            if (q < S.tw) f += bat_j(L.a[q]) * sp[L.a[q] >> 8] * sp[L.b[q]];
        if (S.tw > kPreT) {
            q_g32* pa = (q_g32*)I.ta + S.tbase + lane;
            q_g32* pb = (q_g32*)I.tb + S.tbase + lane;
            for (int q = kPreT; q < S.tw; ++q) {
                const uint32_t wa = pa[q * kSlice];
                f += bat_j(wa) * sp[wa >> 8] * sp[pb[q * kSlice]];
            }
        }
    }
    const int si = sp[i];
    e6 += si * (3 * L.h + f1 + 2 * f);
    const int d = 2 * si * f;
    bool flip = d < 0;
    if (TIE && d == 0) flip = rng_bit(seed, ((q_g32*)I.ext)[i], sweep, I.instance_id, r) != 0;
    if (flip) {
        sp[i] = (int8_t)(-si);
        dE += d;
        ++my;
    }
}

template <bool TIE>
__device__ __forceinline__ void queue_phase(const InstDev& I0, const Slice* __restrict__ slices0, int s_lo, int s_hi,
                                            int8_t* __restrict__ sp, int lane, uint32_t sweep,
                                            uint64_t seed, uint32_t r, long long& dE, int& my, long long& e6)
{
    InstDev I = I0;
    I.nbr = queue_uniform(I0.nbr);
    I.ta = queue_uniform(I0.ta);
    I.tb = queue_uniform(I0.tb);
    I.h = queue_uniform(I0.h);
    I.ext = queue_uniform(I0.ext);
    const Slice* slices = queue_uniform(slices0);
    // the next slice's descriptor is read while this slice's words are in
    // flight, so a slice costs one memory latency, not two
    int sl = __builtin_amdgcn_readfirstlane(s_lo);
    q_v4 nx = {0u, 0u, 0u, 0u};
    if (sl < s_hi) nx = queue_slice_raw(slices, sl);
    for (; sl < s_hi; ++sl) {
        // the descriptor is first used here, one slice after its load was
        // issued (the empty statement keeps the compiler from unpacking, and
        // so waiting for, it right after the load)
        asm volatile("" : "+s"(nx.x), "+s"(nx.y), "+s"(nx.z), "+s"(nx.w));
        const Slice S = queue_unpack(nx);
        if (sl + 1 < s_hi) nx = queue_slice_raw(slices, sl + 1);
        SliceWords cur;
        queue_load(I, S, lane, cur);
        queue_eval<TIE>(I, S, cur, sp, lane, sweep, seed, r, dE, my, e6);
    }
}

// e6: -6 E of the last sweep's fields, exact when that sweep flipped nothing.
__device__ __forceinline__ void queue_finish(const InstTab& Q, int r, long long dE, long long e6, long long nflip,
                                             int performed, int lastflip, int T, int until_conv,
                                             RepState* __restrict__ rs, CallStats* __restrict__ cs)
{
    RepState* st = rs + Q.rep_base + r;
    if (performed > 0 && lastflip < performed) st->E = -e6 / 6;
    else st->E += dE;
    st->flips += nflip;
    st->sweeps += performed;
    st->lastflip = lastflip;
    const bool conv = until_conv && lastflip < performed;
    if (conv) st->converged = 1;
    atomicAdd(&cs->attempts, (unsigned long long)performed * (unsigned long long)Q.I.n);
    atomicAdd(&cs->flips, (unsigned long long)nflip);
    atomicMax(&cs->sweeps_max, (unsigned long long)performed);
    if (until_conv && !conv) atomicAdd(&cs->unconverged, 1ull);
}

// An instance whose arrays and sizes are in scalar registers.
__device__ __forceinline__ InstDev queue_inst(const InstDev& I)
{
    InstDev J = I;
    J.nbr = queue_uniform(I.nbr);
    J.ta = queue_uniform(I.ta);
    J.tb = queue_uniform(I.tb);
    J.h = queue_uniform(I.h);
    J.ext = queue_uniform(I.ext);
    J.slices = queue_uniform(I.slices);
    J.n = __builtin_amdgcn_readfirstlane(I.n);
    J.nslices = __builtin_amdgcn_readfirstlane(I.nslices);
    return J;
}

struct QueueLds {
    TeamLds team;
    long long pd[kBatWaves], pe[kBatWaves], pf[kBatWaves];
    int item;
};

template <bool TIE>
__global__ __launch_bounds__(kBatThreads) void k_queue(const InstTab* __restrict__ tab, const int32_t* __restrict__ ctab,
                                                       const QueueItem* __restrict__ items, int n_big, int n_items,
                                                       uint32_t* __restrict__ counters, int wave_lds,
                                                       RepState* __restrict__ rs, CallStats* __restrict__ cs, int T,
                                                       uint64_t seed, int until_conv, uint32_t fixed_off,
                                                       QueueTeams teams)
{
    // the items' spins start LDS, the fixed part stands behind them
    extern __shared__ __align__(16) int8_t lds[];
    QueueLds& F = *reinterpret_cast<QueueLds*>(lds + fixed_off);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // ---- the first items by teams of workgroups, each workgroup in one team
    if ((int)blockIdx.x < teams.nwg) {
        const QueueItem it = teams.tab[2 * blockIdx.x], mb = teams.tab[2 * blockIdx.x + 1];
        const int m = __builtin_amdgcn_readfirstlane(mb.inst & 0xFFFF), G = __builtin_amdgcn_readfirstlane(mb.inst >> 16);
        unsigned long long* w = (unsigned long long*)teams.words + (int64_t)mb.r * 4;
        const InstTab& Q = tab[it.inst];
        const RepState* st0 = rs + Q.rep_base + it.r;
        if (!st0->converged) {  // (the same for the whole team: its last member alone writes the state)
            const InstDev QI = queue_inst(Q.I);
            const TeamWait wait{(uint32_t*)(w + 4), teams.flag, (uint16_t*)(w + 8 + 4 * (int64_t)QI.nslices), teams.polls};
            const TeamArgs A{QI, queue_uniform(ctab + Q.ctab_off), __builtin_amdgcn_readfirstlane(Q.C), G, m,
                             it.r, Q.spins + (int64_t)it.r * Q.spin_stride, (uint64_t*)w + 8, wait,
                             (uint32_t)st0->sweeps, T, until_conv, seed, &F.team};
            TeamOut o;
            if (__builtin_amdgcn_readfirstlane(Q.I.has_tri)) o = team_run<false, TIE, true, true, kTeamW>(A);
            else o = team_run<false, TIE, false, true, kTeamW>(A);
            const long long wd = team_wave_sum(o.dE), we = team_wave_sum(o.e6);
            if (lane == 0) {
                atomicAdd(w, (unsigned long long)wd);
                atomicAdd(w + 1, (unsigned long long)we);
                atomicAdd(w + 2, (unsigned long long)o.nf);
                __threadfence();
            }
            __syncthreads();
            // the member that arrives last has everyone's sums (none does where
            // a wait gave up)
            if (tid == 0 && !o.dead && __hip_atomic_fetch_add(w + 3, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1 == (unsigned long long)G) {
                const long long a = (long long)__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const long long e = (long long)__hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const long long b = (long long)__hip_atomic_load(w + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                queue_finish(Q, it.r, a, e, b, o.performed, o.lastflip, T, until_conv, rs, cs);
            }
        }
        __syncthreads();
    }
    // ---- large items: the whole workgroup on one replica
    for (;;) {
        if (tid == 0) F.item = teams.n + (int)atomicAdd(&counters[0], 1u);
        __syncthreads();
        const int q = __builtin_amdgcn_readfirstlane(F.item);
        __syncthreads();
        if (q >= n_big) break;
        const QueueItem it = items[q];
        const InstTab& Q = tab[it.inst];
        const InstDev& I = Q.I;
        int8_t* gsp = Q.spins + (int64_t)it.r * Q.spin_stride;
        const RepState* st0 = rs + Q.rep_base + it.r;
        const bool frozen = st0->converged != 0;
        if (frozen) continue;
        const uint32_t base = (uint32_t)st0->sweeps;
        const TeamArgs A{queue_inst(I), queue_uniform(ctab + Q.ctab_off), __builtin_amdgcn_readfirstlane(Q.C), 1, 0,
                         it.r, gsp, nullptr, TeamWait{}, base, T, until_conv, seed, &F.team};
        TeamOut o;
        if (__builtin_amdgcn_readfirstlane(I.has_tri)) o = team_run<true, TIE, true, true, kTeamW>(A);
        else if (__builtin_amdgcn_readfirstlane(Q.max_ew) <= 4) o = team_run<true, TIE, false, true, 4>(A);
        else o = team_run<true, TIE, false, true, kTeamW>(A);
        // fold the workgroup's dE, energy sum and flips
        const long long wd = team_wave_sum(o.dE), we = team_wave_sum(o.e6);
        if (lane == 0) {
            F.pd[wave] = wd;
            F.pe[wave] = we;
            F.pf[wave] = o.nf;
        }
        __syncthreads();
        if (tid == 0) {
            long long a = 0, e = 0, b = 0;
            for (int w = 0; w < kBatWaves; ++w) {
                a += F.pd[w];
                e += F.pe[w];
                b += F.pf[w];
            }
            queue_finish(Q, it.r, a, e, b, o.performed, o.lastflip, T, until_conv, rs, cs);
        }
        __syncthreads();
    }
    // ---- small items: one wavefront per replica, 16 at a time
    int8_t* wl = lds + wave * wave_lds;
    for (;;) {
        if (tid == 0) F.item = n_big + (int)atomicAdd(&counters[1], (unsigned)kBatWaves);
        __syncthreads();
        const int q0 = __builtin_amdgcn_readfirstlane(F.item);
        __syncthreads();
        if (q0 >= n_items) break;
        const int q = __builtin_amdgcn_readfirstlane(q0 + wave);
        if (q < n_items) {
            const QueueItem it = items[q];
            const InstTab& Q = tab[it.inst];
            const InstDev& I = Q.I;
            int8_t* gsp = Q.spins + (int64_t)it.r * Q.spin_stride;
            const RepState* st0 = rs + Q.rep_base + it.r;
            if (!st0->converged) {
                const uint32_t base = (uint32_t)st0->sweeps;
                for (int k = lane; k < I.n; k += 64) wl[k] = gsp[k];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                long long dE = 0, e6 = 0, nflip = 0;  // (nflip: per lane)
                int performed = 0, lastflip = 0;
                for (int t = 0; t < T; ++t) {
                    int my = 0;
                    e6 = 0;
                    for (int c = 0; c < Q.C; ++c) {
                        queue_phase<TIE>(I, I.slices, ctab[Q.ctab_off + c], ctab[Q.ctab_off + c + 1], wl, lane,
                                         base + t, seed, (uint32_t)it.r, dE, my, e6);
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    }
                    nflip += my;
                    performed = t + 1;
                    int tot = my;
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
                    if (tot) lastflip = t + 1;
                    if (until_conv && tot == 0) break;
                }
                for (int k = lane; k < I.n; k += 64) gsp[k] = wl[k];
                long long wd = dE, we = e6, wf = nflip;
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) {
                    wd += __shfl_xor(wd, off, 64);
                    we += __shfl_xor(we, off, 64);
                    wf += __shfl_xor(wf, off, 64);
                }
                if (lane == 0) queue_finish(Q, it.r, wd, we, wf, performed, lastflip, T, until_conv, rs, cs);
            }
        }
        __syncthreads();
    }
}

// LDS of a workgroup whose items take `lds` bytes.
static size_t queue_lds(size_t lds) { return (lds + 15) / 16 * 16 + sizeof(QueueLds); }

int queue_max_blocks(size_t lds)
{
    const void* kern = (const void*)k_queue<true>;
    int per_cu = 0, dev = 0, cus = 0;
    lds = queue_lds(lds);
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kBatThreads, lds) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu * cus;
}

hipError_t launch_queue(const InstTab* tab, const int32_t* ctab, const QueueItem* items, int n_big, int n_items,
                        uint32_t* counters, int wave_lds, size_t lds, int grid, RepState* rs, CallStats* cs, int T,
                        uint64_t seed, int rule, int until_conv, hipStream_t st, const QueueTeams& teams0)
{
    const void* kern = rule == 1 ? (const void*)k_queue<true> : (const void*)k_queue<false>;
    static const bool free0 = team_lds_free((const void*)k_queue<true>) && team_lds_free((const void*)k_queue<false>);
    if (!free0) return hipErrorInvalidDeviceFunction;
    uint32_t fixed = (uint32_t)((lds + 15) / 16 * 16);
    lds = queue_lds(lds);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    QueueTeams teams = teams0;
    if (teams.nwg > grid || teams.n > n_big) return hipErrorInvalidValue;
    void* args[] = {&tab, &ctab, &items, &n_big, &n_items, &counters, &wave_lds, &rs, &cs, &T, &seed, &until_conv,
                    &fixed, &teams};
    // members wait for each other: the cooperative launch has them all resident
    if (teams.nwg) return hipLaunchCooperativeKernel(kern, dim3(grid), dim3(kBatThreads), args, (unsigned)lds, st);
    return hipLaunchKernel(kern, dim3(grid), dim3(kBatThreads), args, lds, st);
}

}  // namespace sg
