// sg_team_core.h -- the sweeps of one replica by a workgroup or a team of
// workgroups, shared by the team kernel (sg_team.hip) and the queue kernel's
// large items (sg_queue.hip).  (Internal.)
//
// Every workgroup holds the replica's whole spin configuration in LDS: one
// byte per spin (a workgroup alone, up to 150000 spins), or one bit (set when
// s = -1), so that up to 1.2 million spins fit; every partner read is an LDS
// read.  Lane = row of a slice, a wavefront takes a phase's slices in turn.
//
// Bound by what a wavefront waits for, with 16 of them on a compute unit: so a
// slice's words are loaded while the slice before is evaluated, its descriptor
// one slice earlier, and the loads are so many for every slice (buffer loads,
// team_buffer) that the wait for one slice's words leaves the next one's in
// flight; all LDS reads of a slice are issued before the first is used; a
// coupling takes two vector instructions beside its LDS read (bytes).  100000
// spins of an Erdos-Renyi graph with triples, one workgroup per replica,
// 12 sweeps of about 12 phases: 1.12 ms, against 2.33 ms with loads under
// branches and an LDS wait per coupling.
//
// A team splits a colour's slices (64 rows each) evenly; after its share of a
// phase a workgroup publishes each slice's flip mask as two words in device
// memory, reads those of the others, and flips the same bits.  A word carries
// 32 bits and the sweep's tag in one 8-byte agent-scope atomic, so a reader
// that sees the tag holds the word: no flag, no barrier across the team, no
// wait for store completion.  Two copies alternate by sweep: a workgroup writes
// a copy again two sweeps later, when it has read every other member's words
// of the sweep between, which each member publishes only after it has read the
// whole of this one (every member has a slice of the largest colour).  Each
// slice is published once a sweep.  Every member sees every flip, so all of
// them take the same decision to stop.
//
// The members of a team have to be resident together.  The cooperative launch
// sees to that, but not beside another process's grid of that kind, nor beside
// kernels that hold the compute units for seconds; so every wait is bounded
// (TeamWait), a team keeps its replica's start (one bit a spin), and the host
// runs the replicas of a team that gave up again without one.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sg_device.h"
#include "sg_layout.h"

namespace sg {

constexpr int kTeamThreads = 1024;
constexpr int kTeamWaves = kTeamThreads / 64;
constexpr int kTeamW = 12, kTeamT = 4;  // coupling and hyper-coupling words of a slice loaded at once (W: at most kTeamW)
constexpr int kTeamColours = 64;        // colours whose tables fit the static LDS

typedef __attribute__((address_space(1))) const uint32_t team_g32;
typedef __attribute__((address_space(1))) int8_t team_gw8;
typedef uint32_t team_v4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) const int32_t team_kint;

struct TeamSlice {
    uint32_t row0, ebase, tbase;
    int ew, tw, rows;
};

// A slice's descriptor, the same in every lane (sl is uniform), and its fields
// as scalars.  (Read with a vector load: scalar loads return out of order, so
// that every wait for an LDS read would wait for them too.)
__device__ __forceinline__ team_v4 team_raw(const Slice* slices, int sl, int zero)
{
    return ((__attribute__((address_space(1))) const team_v4*)slices)[sl + zero];
}
__device__ __forceinline__ TeamSlice team_unpack(team_v4 v)
{
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)v.w);
    return TeamSlice{(uint32_t)__builtin_amdgcn_readfirstlane((int)v.x), (uint32_t)__builtin_amdgcn_readfirstlane((int)v.y),
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)v.z), (int)(w & 0xFFFFu), (int)((w >> 16) & 0xFFu),
                     (int)(w >> 24)};
}

template <int W>
struct TeamWords {
    uint32_t w[W], a[kTeamT], b[kTeamT], x, h;  // (h: the dword with its byte)
};

// A slice's words of one array, as a buffer of w rows of 64: reads beyond it
// return zero without memory traffic.  So every slice takes the same number of
// loads, and the wait for a slice's words leaves the next slice's in flight
// (with loads under branches, the wait has to cover the fewest that may
// follow).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t team_buffer(const void* p, uint32_t base, int w)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const uint32_t*)p + base), 0, w * kSlice * 4, 0x00027000);
}

template <bool TIE, bool TRI, int W>
__device__ __forceinline__ void team_load(const InstDev& I, const TeamSlice& S, int lane, TeamWords<W>& L)
{
    const uint32_t l = lane < S.rows ? (uint32_t)lane : 0u;
    const __amdgpu_buffer_rsrc_t p = team_buffer(I.nbr, S.ebase, S.ew);
#pragma unroll
    for (int k = 0; k < W; ++k) L.w[k] = __builtin_amdgcn_raw_buffer_load_b32(p, (int)(l * 4 + (uint32_t)k * kSlice * 4), 0, 0);
    if (TRI) {
        const __amdgpu_buffer_rsrc_t pa = team_buffer(I.ta, S.tbase, S.tw), pb = team_buffer(I.tb, S.tbase, S.tw);
#pragma unroll
        for (int k = 0; k < kTeamT; ++k) {
            L.a[k] = __builtin_amdgcn_raw_buffer_load_b32(pa, (int)(l * 4 + (uint32_t)k * kSlice * 4), 0, 0);
            L.b[k] = __builtin_amdgcn_raw_buffer_load_b32(pb, (int)(l * 4 + (uint32_t)k * kSlice * 4), 0, 0);
        }
    }
    const uint32_t i = S.row0 + l;
    L.h = ((team_g32*)I.h)[i >> 2];  // (the array's end is padded)
    if (TIE) L.x = ((team_g32*)I.ext)[i];  // the row's index in the generator's counter
}

// The spins in LDS: bytes (+1, -1), or one bit each (set when s = -1).  A
// coupling word holds its partner's index above its coefficient's byte, and
// the four-byte dot product multiplies that byte by a value held alone in the
// low byte of the other operand: two vector instructions a coupling for bytes,
// five for bits.
// The spins begin at LDS address 0 (the kernels have no LDS but the launch's,
// team_lds_free), so that a partner's index is its address.
typedef __attribute__((address_space(3))) uint8_t team_l8;
typedef __attribute__((address_space(3))) uint16_t team_l16;
typedef __attribute__((address_space(3))) uint32_t team_l32;
typedef __attribute__((address_space(3))) team_v4 team_l128;
__device__ __forceinline__ team_l8* team_lds(uint32_t address) { return (team_l8*)(uintptr_t)address; }
struct TeamBytes {
    static constexpr bool kCheap = true;  // adding a zero word costs less than a branch
    static __device__ __forceinline__ uint32_t at(uint32_t j) { return *team_lds(j); }
    // product of two spins, from their bytes: (a ^ b) | 1
    static __device__ __forceinline__ uint32_t product(uint32_t a, uint32_t b) { return (uint32_t)__builtin_amdgcn_bitop3_b32((int)a, (int)b, 1, 0xBE); }
    static __device__ __forceinline__ int add(uint32_t w, uint32_t v, int f) { return __builtin_amdgcn_sdot4((int)w, (int)v, f, false); }
    static __device__ __forceinline__ uint32_t pick(uint32_t v, uint32_t) { return v; }
    static __device__ __forceinline__ int sign(uint32_t v, uint32_t) { return __builtin_amdgcn_sbfe((int)v, 7, 1); }  // 0 or -1
};
struct TeamBits {
    static constexpr bool kCheap = false;
    static __device__ __forceinline__ uint32_t at(uint32_t j) { return *team_lds(j >> 3); }
    static __device__ __forceinline__ uint32_t product(uint32_t a, uint32_t b) { return a ^ b; }
    static __device__ __forceinline__ int add(uint32_t w, uint32_t v, int f)
    {
        // c - 2 c v: the byte 1 or -1 from the bit
        return __builtin_amdgcn_sdot4((int)w, (int)((0u - 2u * v + 1u) & 0xFFu), f, false);
    }
    static __device__ __forceinline__ uint32_t pick(uint32_t v, uint32_t j) { return __builtin_amdgcn_ubfe(v, j & 7u, 1u); }
    static __device__ __forceinline__ int sign(uint32_t v, uint32_t j) { return __builtin_amdgcn_sbfe((int)v, j & 7u, 1u); }
};

// A row's field, the coupling part in f1 (with h).  All LDS reads are issued
// before the first is used; words beyond the slice's width are zero and add
// nothing.
template <class SP, bool TRI, int W>
__device__ __forceinline__ int team_field(const InstDev& I, const TeamSlice& S, const TeamWords<W>& L, int lane, int h,
                                          int& f1)
{
    const uint32_t l = lane < S.rows ? (uint32_t)lane : 0u;
    uint32_t v[W], ua[kTeamT], ub[kTeamT];
#pragma unroll
    for (int k = 0; k < W; ++k) v[k] = 0u;
#pragma unroll
    for (int k = 0; k < kTeamT; ++k) ua[k] = ub[k] = 0u;
#pragma unroll
    for (int k0 = 0; k0 < W; k0 += 4)
        if (k0 < S.ew) {
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) v[k] = SP::at(L.w[k] >> 8);
        }
    if (TRI) {
#pragma unroll
        for (int k0 = 0; k0 < kTeamT; k0 += 2)
            if (k0 < S.tw) {
#pragma unroll
                for (int k = k0; k < k0 + 2; ++k) {
                    ua[k] = SP::at(L.a[k] >> 8);
                    ub[k] = SP::at(L.b[k]);
                }
            }
    }
    int f = h;
#pragma unroll
    for (int k0 = 0; k0 < W; k0 += 4)
        if (SP::kCheap || k0 < S.ew) {
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) f = SP::add(L.w[k], SP::pick(v[k], L.w[k] >> 8), f);
        }
    if (W == kTeamW && S.ew > W) {  // longer rows: eight words at a time
        const __amdgpu_buffer_rsrc_t p = team_buffer(I.nbr, S.ebase, S.ew);
        for (int k = W; k < S.ew; k += 8) {
            uint32_t w[8], x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = __builtin_amdgcn_raw_buffer_load_b32(p, (int)(l * 4 + (uint32_t)(k + u) * kSlice * 4), 0, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = SP::at(w[u] >> 8);
#pragma unroll
            for (int u = 0; u < 8; ++u) f = SP::add(w[u], SP::pick(x[u], w[u] >> 8), f);
        }
    }
    f1 = f;
    if (TRI) {
#pragma unroll
        for (int k0 = 0; k0 < kTeamT; k0 += 2)
            if (SP::kCheap || k0 < S.tw) {
#pragma unroll
                for (int k = k0; k < k0 + 2; ++k)
                    f = SP::add(L.a[k], SP::product(SP::pick(ua[k], L.a[k] >> 8), SP::pick(ub[k], L.b[k])), f);
            }
        if (S.tw > kTeamT) {
            const __amdgpu_buffer_rsrc_t pa = team_buffer(I.ta, S.tbase, S.tw), pb = team_buffer(I.tb, S.tbase, S.tw);
            for (int k = kTeamT; k < S.tw; k += 4) {
                uint32_t a[4], b[4], x[4], y[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at = (int)(l * 4 + (uint32_t)(k + u) * kSlice * 4);
                    a[u] = __builtin_amdgcn_raw_buffer_load_b32(pa, at, 0, 0);
                    b[u] = __builtin_amdgcn_raw_buffer_load_b32(pb, at, 0, 0);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    x[u] = SP::at(a[u] >> 8);
                    y[u] = SP::at(b[u]);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    f = SP::add(a[u], SP::product(SP::pick(x[u], a[u] >> 8), SP::pick(y[u], b[u])), f);
            }
        }
    }
    return f;
}

// Whether a kernel has no LDS of its own.
inline bool team_lds_free(const void* kern)
{
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, kern) == hipSuccess && a.sharedSizeBytes == 0;
}

// LDS of a kernel that calls team_run, beside the spins.
struct TeamLds {
    int2 sh[kTeamColours];        // this member's slices of each colour
    int2 all[kTeamColours];       // the colour's slices
    uint32_t row[kTeamColours];   // and its first row
    int any[3], dead;  // see the end of a sweep; 1 + the sweep in which a wait gave up
};

// A member's view of its replica.  LDS from address 0 on: the replica's spins, n
// bytes (to a multiple of 16), or as bits (n + 31) / 32 + 1 words.
struct TeamArgs {
    InstDev I;
    const int32_t* ct;  // the C + 1 slice offsets of the colours
    int C, G, m, r;     // colours (at most kTeamColours if G > 1); members (1 with bytes), this one; restart
    int8_t* sp;         // the replica's spins (row padded to 256 bytes)
    uint64_t* words;    // two copies of two words per slice, tags zero on entry
    TeamWait wait;      // (G > 1)
    uint32_t base;      // sweeps before the call
    int T, until_conv;
    uint64_t seed;
    TeamLds* L;
};

// Barrier that orders LDS only: loads from memory issued before it (the next
// slice's words) stay in flight across it.
__device__ __forceinline__ void team_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What this member's rows did: energy change per lane, the sum 6 (...) of the
// last sweep's fields per lane (E6; see queue_eval), flips per wavefront.
struct TeamOut {
    long long dE, e6, nf;
    int performed, lastflip;
    bool dead;  // a wait gave up: this member's rows are not written
};

template <bool BYTES, bool TIE, bool TRI, bool E6, int W = kTeamW>
__device__ __forceinline__ TeamOut team_run(const TeamArgs& A)
{
    const InstDev& I = A.I;
    TeamLds& T = *A.L;
    const int G = A.G, m = A.m, C = A.C, n = I.n;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid < 3) T.any[tid] = 0;
    if (tid == 0) T.dead = 0;
    for (int c = tid; c < C && C <= kTeamColours; c += kTeamThreads) {
        const int s0 = A.ct[c], s1 = A.ct[c + 1];
        T.all[c] = make_int2(s0, s1);
        T.sh[c] = make_int2(s0 + (int)((int64_t)(s1 - s0) * m / G), s0 + (int)((int64_t)(s1 - s0) * (m + 1) / G));
        T.row[c] = s1 > s0 ? I.slices[s0].row0 : 0u;
    }
    using SP = typename std::conditional<BYTES, TeamBytes, TeamBits>::type;
    // the spins, or their signs, sixteen a thread
    if (BYTES) {
        for (int k = tid; k * 16 < n; k += kTeamThreads)
            *(team_l128*)team_lds((uint32_t)k * 16u) = *(const team_v4*)(A.sp + k * 16);
    } else {
        const int words16 = (n + 15) / 16;  // this member keeps its share of the start
        const int k0 = (int)((int64_t)words16 * m / G), k1 = G > 1 ? (int)((int64_t)words16 * (m + 1) / G) : 0;
        for (int k = tid; k * 16 < n; k += kTeamThreads) {
            const uint4 v = *reinterpret_cast<const uint4*>(A.sp + k * 16);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t b = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                b |= ((w[u] >> 7 & 1u) | (w[u] >> 14 & 2u) | (w[u] >> 21 & 4u) | (w[u] >> 28 & 8u)) << (4 * u);
            if (n - k * 16 < 16) b &= (1u << (n - k * 16)) - 1u;
            *(team_l16*)team_lds((uint32_t)k * 2u) = (uint16_t)b;
            if (k >= k0 && k < k1) A.wait.save[k] = (uint16_t)b;
        }
    }
    __syncthreads();
    // 32 flips from row p on
    auto flip_at = [&](uint32_t p, uint32_t f) {
        team_l32* at = (team_l32*)team_lds((p >> 5) * 4u);
        __hip_atomic_fetch_xor(at, f << (p & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const uint32_t up = (p & 31) ? f >> (32 - (p & 31)) : 0u;
        if (up) __hip_atomic_fetch_xor(at + 1, up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };

    // this member's share of colour c: slices [lo, hi) (more colours than the
    // tables hold are read from memory; G is 1 then)
    auto share = [&](int c) {
        int2 v;
        if (C <= kTeamColours) v = T.sh[c];
        else v = make_int2(((team_kint*)A.ct)[c], ((team_kint*)A.ct)[c + 1]);
        return make_int2(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y));
    };

    // A wavefront's slices of all phases form one cyclic sequence; pos is the
    // place whose descriptor was read last, raw that descriptor.
    int pc = 0, pos, phi;
    {
        const int2 v = share(0);
        pos = v.x + wave;
        phi = v.y;
    }
    auto settle = [&]() -> bool {  // pos to the first slice of this wavefront from there on
        for (int k = 0; pos >= phi; ++k) {
            if (k == C) return false;  // it has none
            pc = pc + 1 < C ? pc + 1 : 0;
            const int2 v = share(pc);
            pos = v.x + wave;
            phi = v.y;
        }
        return true;
    };
    TeamSlice SA{}, SB{};
    int zero = 0;  // kept in a vector register
    asm volatile("" : "+v"(zero));
    TeamWords<W> LA, LB;
    team_v4 raw = {0u, 0u, 0u, 0u};
    int at = 0;  // the slice whose descriptor raw holds
    auto words = [&](TeamSlice& S, TeamWords<W>& L, int& sl) {
        // the descriptor is first used here, one slice after its load was
        // issued (the empty statement keeps it from being unpacked, and so
        // waited for, right after the load)
        asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w));
        S = team_unpack(raw);
        sl = at;
        team_load<TIE, TRI, W>(I, S, lane, L);
    };
    auto advance = [&]() {
        pos += kTeamWaves;
        settle();
        at = pos;
        raw = team_raw(I.slices, pos, zero);
    };
    auto load = [&](TeamSlice& S, TeamWords<W>& L, int& sl) {
        asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w));
        S = team_unpack(raw);
        sl = at;
        advance();
        team_load<TIE, TRI, W>(I, S, lane, L);
    };
    int la = 0, lb = 0;  // the slices in A and B
    if (settle()) {
        at = pos;
        raw = team_raw(I.slices, pos, zero);
        load(SA, LA, la);
    }

    int2 mine = share(0), all = make_int2(0, 0);  // the phase's slices: this member's and all
    uint32_t row = 0;                             // the first row of them
    if (!BYTES && G > 1) {
        all = T.all[0];
        row = T.row[0];
    }
    TeamOut out{0, 0, 0, 0, 0, false};
    for (int t = 0; t < A.T; ++t) {
        uint32_t any = 0;
        uint64_t moves = 0;
        out.e6 = 0;
        uint64_t* buf = A.words + (size_t)(t & 1) * I.nslices * 2;
        const uint64_t tag = (uint64_t)(uint32_t)(t + 1) << 32;
        auto eval = [&](int sl, const TeamSlice& S, const TeamWords<W>& L) {
            const uint32_t i = S.row0 + (uint32_t)lane;
            const bool in = lane < S.rows;
            const uint32_t own = SP::at(in ? i : S.row0);
            const int h = __builtin_amdgcn_sbfe((int)L.h, (in ? i : S.row0) * 8u, 8u);
            int f1;
            const int f = team_field<SP, TRI, W>(I, S, L, lane, h, f1);
            const int mi = SP::sign(own, i);
            const int d = in ? 2 * ((f ^ mi) - mi) : 1;
            bool flip = d < 0;
            if (TIE && d == 0)
                flip = rng_bit(A.seed, L.x, A.base + (uint32_t)t, I.instance_id, (uint32_t)A.r) != 0;
            if (E6) {
                const int e = ((3 * h + f1 + 2 * f) ^ mi) - mi;
                out.e6 += in ? e : 0;
            }
            const uint64_t mask = __ballot(flip);
            out.dE += flip ? d : 0;
            if (BYTES) {
                if (flip) *team_lds(i) = (uint8_t)(0u - own);
            } else if (lane < 2) {
                const uint32_t half = (uint32_t)(lane ? mask >> 32 : mask);
                if (G > 1)
                    __hip_atomic_store(buf + 2 * (size_t)sl + lane, tag | half, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (half) flip_at(S.row0 + 32u * (uint32_t)lane, half);
            }
            moves |= mask;
            out.nf += (long long)__popcll(mask);
        };
        for (int c = 0; c < C; ++c) {
            // (its bounds were read before the barrier)
            const int lo = mine.x, hi = mine.y;
            int left = (hi - lo - wave + kTeamWaves - 1) / kTeamWaves;  // slices of this wavefront, if > 0
            // each slice's words are loaded before the slice before it is
            // evaluated, the next phase's first among them; a team's last slice
            // of a phase is published first
            bool inb = false, adv = false;
            while (left > 0) {
                if (!BYTES && G > 1 && left == 1) {
                    eval(la, SA, LA);
                    words(SA, LA, la);
                    adv = true;
                    break;
                }
                load(SB, LB, lb);
                eval(la, SA, LA);
                if (--left == 0) {
                    inb = true;
                    break;
                }
                load(SA, LA, la);
                eval(lb, SB, LB);
                --left;
            }
            if (!BYTES && G > 1) {
                // A word takes about a microsecond to reach another member, and
                // every early poll is a load of all the words by all the teams
                // that delays the words themselves: the first poll waits 1024
                // cycles, 1536 in a launch of many workgroups (500000 spins of
                // a 3-regular graph, 245 members, a sweep of 4 phases: 23 us
                // without the wait, 12.8 after 640 cycles, 10.3 after 1024, 9.8
                // after 1536, 10.3 after 2560; 20000 spins, 10 members: 12.1 us
                // after 1024, 12.9 after 1536, 14.8 after 2560)
                __builtin_amdgcn_s_sleep(16);
                if (gridDim.x >= 64) __builtin_amdgcn_s_sleep(8);
                // the other members' words: those before the share, then those after it
                const int s0 = all.x, before = 2 * (lo - s0), total = before + 2 * (all.y - hi);
                for (int x0 = tid; x0 < total; x0 += 4 * kTeamThreads) {
                    uint64_t v[4];
                    size_t w[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int x = x0 + u * kTeamThreads;
                        w[u] = 2 * (size_t)s0 + (size_t)(x < before ? x : x + 2 * (hi - lo));
                        v[u] = x < total ? __hip_atomic_load(buf + w[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tag;
                    }
                    // bounded: a wait that gives up here or in any other
                    // workgroup raises the error flag and ends them all
                    for (uint32_t polls = A.wait.polls; ((v[0] ^ tag) | (v[1] ^ tag) | (v[2] ^ tag) | (v[3] ^ tag)) >> 32;) {
                        if (--polls == 0 || ((polls & 63u) == 0 && __hip_atomic_load(A.wait.err, __ATOMIC_RELAXED,
                                                                                    __HIP_MEMORY_SCOPE_AGENT) != 0u)) {
                            __hip_atomic_store(A.wait.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            __hip_atomic_store(A.wait.flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            T.dead = t + 1;
#pragma unroll
                            for (int u = 0; u < 4; ++u) v[u] = tag;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if ((v[u] ^ tag) >> 32)
                                v[u] = __hip_atomic_load(buf + w[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t f = (uint32_t)v[u];
                        if (f) {
                            any = 1;
                            flip_at(row + 32u * (uint32_t)(w[u] - 2 * (size_t)s0), f);
                        }
                    }
                }
            }
            if (adv) advance();
            mine = share(c + 1 < C ? c + 1 : 0);
            if (!BYTES && G > 1) {
                all = T.all[c + 1 < C ? c + 1 : 0];
                row = T.row[c + 1 < C ? c + 1 : 0];
            }
            // the sweep's last barrier also tells whether it flipped anything:
            // slot t % 3 is set before the barrier and read after it; slot
            // (t + 2) % 3 is cleared for sweep t + 2, after every read of it
            // (sweep t - 1) and a barrier before any write of it
            if (c + 1 == C && (__ballot(any != 0) | moves) != 0 && lane == 0) T.any[t % 3] = 1;
            team_barrier();
            if (inb) {
                // (waited for here, past the barrier)
#pragma unroll
                for (int k = 0; k < W; ++k) asm volatile("" : "+v"(LB.w[k]));
                SA = SB;
                LA = LB;
                la = lb;
            }
        }
        const bool moved = T.any[t % 3] != 0;
        if (!BYTES && T.dead == t + 1) {  // (a thread of the next sweep may already write t + 2)
            out.dead = true;
            return out;
        }
        if (tid == 0) T.any[(t + 2) % 3] = 0;
        out.performed = t + 1;
        if (moved) out.lastflip = t + 1;
        if (A.until_conv && !moved) break;
    }
    // the words loaded ahead have no use: wait for them here, so that no wait
    // of a later item counts them
    __builtin_amdgcn_s_waitcnt(0x0F70);
    // this member's rows back
    for (int c = 0; c < C; ++c)
        for (int k = share(c).x + wave, hi = share(c).y; k < hi; k += kTeamWaves) {
            const TeamSlice Z = team_unpack(team_raw(I.slices, k, zero));
            const uint32_t i = Z.row0 + (uint32_t)lane;
            if (lane < Z.rows) ((team_gw8*)A.sp)[i] = BYTES ? (int8_t)SP::at(i) : SP::pick(SP::at(i), i) ? (int8_t)-1 : (int8_t)1;
        }
    return out;
}

__device__ __forceinline__ long long team_wave_sum(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace sg
