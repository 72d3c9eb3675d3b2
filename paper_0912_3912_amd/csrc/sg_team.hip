// sg_team.hip -- colour-ordered sweeps of one instance in one launch: a team
// of G workgroups per replica, every phase of every sweep inside the kernel.
// It runs what SG_SCHED_AUTO would give to per-phase launches: few replicas of
// an irregular graph, whose phases take a few microseconds each, so that
// launches, the gaps between them, and the host's checks of the stopping rule
// cost more than the phases.
//
// Every workgroup holds the replica's whole spin configuration in LDS, one bit
// per spin (set when s = -1), so that up to 1.1 million spins fit and every
// partner read is an LDS read.  A colour's slices (64 rows each) are split
// evenly over the team; after its share of a phase a workgroup publishes each
// slice's flip mask as two words in device memory, reads those of the others,
// and flips the same bits.  A word carries 32 bits and the sweep's tag in one
// 8-byte agent-scope atomic, so a reader that sees the tag holds the word: no
// flag, no barrier across the team, no wait for store completion.  Two copies
// alternate by sweep: a workgroup writes a copy again two sweeps later, when it
// has read every other member's words of the sweep between, which each member
// publishes only after it has read the whole of this one.  Each slice is
// published once a sweep.  Every member sees every flip, so all of them take
// the same decision to stop.
//
// The words of a wavefront's first slice of the next phase are loaded before
// the wait for the others, which hides their latency.  Bound by the latency of
// the chain of phases: LDS reads, the exchange's round trip through memory
// between compute units, the barrier.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sg_device.h"
#include "sg_launch.h"
#include "sg_layout.h"

namespace sg {

namespace {

constexpr int kTeamThreads = 1024;
constexpr int kTeamWaves = kTeamThreads / 64;
constexpr int kTeamW = 8, kTeamT = 4;   // coupling and hyper-coupling words of a slice loaded at once
constexpr int kTeamColours = 64;        // colours whose tables fit the static LDS
constexpr uint32_t kTeamSpin = 1u << 22;  // polls before a wait gives up

typedef __attribute__((address_space(1))) const uint32_t team_g32;
typedef __attribute__((address_space(1))) const int8_t team_gi8;
typedef uint32_t team_v4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(4))) const team_v4 team_kslice;

struct TeamSlice {
    uint32_t row0, ebase, tbase;
    int ew, tw, rows;
};

// A slice's descriptor, read with scalar loads (sl is uniform).
__device__ __forceinline__ TeamSlice team_slice(const Slice* slices, int sl)
{
    const team_v4 v = *(team_kslice*)(slices + sl);
    return TeamSlice{v.x, v.y, v.z, (int)(v.w & 0xFFFFu), (int)((v.w >> 16) & 0xFFu), (int)(v.w >> 24)};
}

struct TeamWords {
    uint32_t w[kTeamW], a[kTeamT], b[kTeamT];
    int h;
};

template <bool TRI>
__device__ __forceinline__ void team_load(const InstDev& I, const TeamSlice& S, int lane, TeamWords& L)
{
    const int l = lane < S.rows ? lane : 0;
    team_g32* p = (team_g32*)I.nbr + S.ebase + l;
#pragma unroll
    for (int k = 0; k < kTeamW; ++k) L.w[k] = k < S.ew ? p[k * kSlice] : 0u;
    if (TRI) {
        team_g32* pa = (team_g32*)I.ta + S.tbase + l;
        team_g32* pb = (team_g32*)I.tb + S.tbase + l;
#pragma unroll
        for (int k = 0; k < kTeamT; ++k) {
            L.a[k] = k < S.tw ? pa[k * kSlice] : 0u;
            L.b[k] = k < S.tw ? pb[k * kSlice] : 0u;
        }
    }
    L.h = (int)((team_gi8*)I.h)[S.row0 + l];
}

__device__ __forceinline__ uint32_t team_bit(const uint32_t* bits, uint32_t j) { return (bits[j >> 5] >> (j & 31)) & 1u; }

// c if the bit is 0, -c if it is 1
__device__ __forceinline__ int team_signed(uint32_t w, uint32_t bit)
{
    const int c = (int)(int8_t)(w & 0xFFu);
    return bit ? -c : c;
}

template <bool TRI>
__device__ __forceinline__ int team_field(const InstDev& I, const TeamSlice& S, const TeamWords& L, int lane,
                                          const uint32_t* bits)
{
    const int l = lane < S.rows ? lane : 0;
    int f = L.h;
#pragma unroll
    for (int k = 0; k < kTeamW; ++k)
        if (k < S.ew) f += team_signed(L.w[k], team_bit(bits, L.w[k] >> 8));
    for (int k = kTeamW; k < S.ew; ++k) {
        const uint32_t w = ((team_g32*)I.nbr + S.ebase + l)[k * kSlice];
        f += team_signed(w, team_bit(bits, w >> 8));
    }
    if (TRI) {
#pragma unroll
        for (int k = 0; k < kTeamT; ++k)
            if (k < S.tw) f += team_signed(L.a[k], team_bit(bits, L.a[k] >> 8) ^ team_bit(bits, L.b[k]));
        for (int k = kTeamT; k < S.tw; ++k) {
            const uint32_t a = ((team_g32*)I.ta + S.tbase + l)[k * kSlice], b = ((team_g32*)I.tb + S.tbase + l)[k * kSlice];
            f += team_signed(a, team_bit(bits, a >> 8) ^ team_bit(bits, b));
        }
    }
    return f;
}

__device__ __forceinline__ long long team_wave_sum(long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

}  // namespace

// Grid: R teams of G workgroups (workgroup r G + m: member m of replica r's).
// ct: the C + 1 slice offsets of the colours.  words: per replica two copies of
// two words per slice, tags zero on entry.  acc slots (nslots per replica, zero
// on entry) take the energy changes and flips, rs[r].lastflip 1 + the last
// sweep that flipped.  Dynamic LDS: (n + 31) / 32 + 1 words.
template <bool TIE, bool TRI>
__global__ __launch_bounds__(kTeamThreads) void k_team(const InstDev I, const int32_t* __restrict__ ct, int C,
                                                       int8_t* __restrict__ spins, int64_t stride,
                                                       RepState* __restrict__ rs, int G, int64_t* __restrict__ acc,
                                                       int nslots, uint64_t* __restrict__ words,
                                                       uint32_t* __restrict__ err, int T, uint64_t seed, int until_conv)
{
    extern __shared__ __align__(16) uint32_t bits[];
    __shared__ int s_ct[kTeamColours + 1];
    __shared__ uint32_t s_row[kTeamColours + 1];  // first row of each colour
    __shared__ int s_dead;
    const int r = (int)blockIdx.x / G, m = (int)blockIdx.x % G;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    RepState* st = rs + r;
    if (st->converged) return;  // the same for the whole team
    const uint32_t base = (uint32_t)st->sweeps;
    int8_t* sp = spins + stride * r;
    const int n = I.n;
    uint64_t* wr = words + (size_t)r * I.nslices * 4;
    if (tid == 0) s_dead = 0;
    for (int c = tid; c <= C; c += kTeamThreads) {
        const int s0 = ct[c];
        s_ct[c] = s0;
        s_row[c] = c < C && s0 < I.nslices ? I.slices[s0].row0 : 0u;
    }
    // the spins' signs, sixteen spins a thread (the row is padded to 256 bytes)
    for (int k = tid; k * 16 < n; k += kTeamThreads) {
        const uint4 v = *reinterpret_cast<const uint4*>(sp + k * 16);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        uint32_t b = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            b |= ((w[u] >> 7 & 1u) | (w[u] >> 14 & 2u) | (w[u] >> 21 & 4u) | (w[u] >> 28 & 8u)) << (4 * u);
        if (n - k * 16 < 16) b &= (1u << (n - k * 16)) - 1u;
        reinterpret_cast<uint16_t*>(bits)[k] = (uint16_t)b;
    }
    __syncthreads();
    // this member's share of colour c: slices [lo, hi)
    auto share_lo = [&](int c) {
        const int s0 = s_ct[c], ns = s_ct[c + 1] - s0;
        return __builtin_amdgcn_readfirstlane(s0 + (int)((int64_t)ns * m / G));
    };
    auto share_hi = [&](int c) {
        const int s0 = s_ct[c], ns = s_ct[c + 1] - s0;
        return __builtin_amdgcn_readfirstlane(s0 + (int)((int64_t)ns * (m + 1) / G));
    };
    // 32 flips from row p on
    auto flip_at = [&](uint32_t p, uint32_t f) {
        atomicXor(&bits[p >> 5], f << (p & 31));
        const uint32_t up = (p & 31) ? f >> (32 - (p & 31)) : 0u;
        if (up) atomicXor(&bits[(p >> 5) + 1], up);
    };

    long long dE = 0, nf = 0;
    int lastflip = 0;
    TeamSlice S{};
    TeamWords L;
    int sl = share_lo(0) + wave;
    if (sl < share_hi(0)) {
        S = team_slice(I.slices, sl);
        team_load<TRI>(I, S, lane, L);
    }
    for (int t = 0; t < T; ++t) {
        uint32_t any = 0;
        uint64_t* buf = wr + (size_t)(t & 1) * I.nslices * 2;
        const uint64_t tag = (uint64_t)(uint32_t)(t + 1) << 32;
        for (int c = 0; c < C; ++c) {
            const int lo = share_lo(c), hi = share_hi(c);
            for (sl = lo + wave; sl < hi;) {
                const int f = team_field<TRI>(I, S, L, lane, bits);
                const uint32_t i = S.row0 + (uint32_t)lane;
                bool flip = false;
                int d = 0;
                if (lane < S.rows) {
                    d = team_bit(bits, i) ? -2 * f : 2 * f;
                    flip = d < 0;
                    if (TIE && d == 0)
                        flip = rng_bit(seed, ((team_g32*)I.ext)[i], base + (uint32_t)t, I.instance_id, (uint32_t)r) != 0;
                }
                const uint64_t mask = __ballot(flip);
                if (flip) dE += d;
                if (lane < 2) {
                    const uint32_t half = (uint32_t)(lane ? mask >> 32 : mask);
                    if (G > 1)
                        __hip_atomic_store(buf + 2 * (size_t)sl + lane, tag | half, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    if (half) flip_at(S.row0 + 32u * (uint32_t)lane, half);
                }
                any |= mask != 0;
                nf += (long long)__popcll(mask);
                sl += kTeamWaves;
                if (sl < hi) {
                    S = team_slice(I.slices, sl);
                    team_load<TRI>(I, S, lane, L);
                }
            }
            // the next phase's first slice: its words arrive during the exchange
            const int cn = c + 1 < C ? c + 1 : 0;
            sl = share_lo(cn) + wave;
            if (sl < share_hi(cn)) {
                S = team_slice(I.slices, sl);
                team_load<TRI>(I, S, lane, L);
            }
            if (G > 1) {
                // the other members' words: those before the share, then those after it
                const int s0 = s_ct[c], before = 2 * (lo - s0), total = before + 2 * (s_ct[c + 1] - hi);
                const uint32_t row = s_row[c];
                for (int x0 = tid; x0 < total; x0 += 4 * kTeamThreads) {
                    uint64_t v[4];
                    size_t at[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int x = x0 + u * kTeamThreads;
                        at[u] = 2 * (size_t)s0 + (size_t)(x < before ? x : x + 2 * (hi - lo));
                        v[u] = x < total ? __hip_atomic_load(buf + at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tag;
                    }
                    uint32_t left = kTeamSpin;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        // bounded: a wait that gives up here or in any other
                        // workgroup raises the error flag and ends them all
                        while ((v[u] ^ tag) >> 32) {
                            if (--left == 0 || ((left & 63u) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED,
                                                                                       __HIP_MEMORY_SCOPE_AGENT) != 0u)) {
                                __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                s_dead = 1;
                                v[u] = tag;
                                left = 1;
                                break;
                            }
                            __builtin_amdgcn_s_sleep(1);
                            v[u] = __hip_atomic_load(buf + at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        }
                        const uint32_t f = (uint32_t)v[u];
                        if (f) {
                            any = 1;
                            flip_at(row + 32u * (uint32_t)(at[u] - 2 * (size_t)s0), f);
                        }
                    }
                }
            }
            if (c + 1 < C) __syncthreads();
        }
        const int moved = __syncthreads_or(any != 0);
        if (s_dead) return;
        if (moved) lastflip = t + 1;
        if (until_conv && !moved) break;
    }
    // this member's rows back
    for (int c = 0; c < C; ++c)
        for (int k = share_lo(c) + wave; k < share_hi(c); k += kTeamWaves) {
            const TeamSlice W = team_slice(I.slices, k);
            const uint32_t i = W.row0 + (uint32_t)lane;
            if (lane < W.rows) sp[i] = team_bit(bits, i) ? (int8_t)-1 : (int8_t)1;
        }
    const long long wd = team_wave_sum(dE);
    if (lane == 0) {
        int64_t* a = acc + 2 * ((int64_t)r * nslots + m % nslots);
        if (wd) atomicAdd((unsigned long long*)a, (unsigned long long)wd);
        if (nf) atomicAdd((unsigned long long*)a + 1, (unsigned long long)nf);
    }
    if (m == 0 && tid == 0) st->lastflip = lastflip;
}

static const void* team_kernel(bool tie, bool tri)
{
    if (tie) return tri ? (const void*)k_team<true, true> : (const void*)k_team<true, false>;
    return tri ? (const void*)k_team<false, true> : (const void*)k_team<false, false>;
}

static size_t team_lds(int n) { return ((size_t)(n + 31) / 32 + 1) * 4; }

bool team_fits(int n, int C) { return team_lds(n) <= 150 * 1024 && C >= 1 && C <= kTeamColours; }

int team_max_blocks(int n, bool tie, bool tri)
{
    const void* kern = team_kernel(tie, tri);
    int per_cu = 0, dev = 0, cus = 0;
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)team_lds(n)) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kTeamThreads, team_lds(n)) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu * cus;
}

hipError_t launch_team(const InstDev& I, const int32_t* ct, int C, int8_t* spins, int64_t stride, RepState* rs, int R,
                       int G, int64_t* acc, int nslots, uint64_t* words, uint32_t* err, int T, uint64_t seed, int rule,
                       int until_conv, hipStream_t st)
{
    if (R <= 0 || T <= 0) return hipSuccess;
    if (G < 1 || !team_fits(I.n, C) || (G > 1 && !words)) return hipErrorInvalidValue;
    const void* kern = team_kernel(rule == 1, I.has_tri != 0);
    const size_t lds = team_lds(I.n);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    InstDev a0 = I;
    void* args[] = {&a0, &ct, &C, &spins, &stride, &rs, &G, &acc, &nslots, &words, &err, &T, &seed, &until_conv};
    // members wait for each other: the cooperative launch has them all resident
    if (G > 1) return hipLaunchCooperativeKernel(kern, dim3((unsigned)(R * G)), dim3(kTeamThreads), args, (unsigned)lds, st);
    return hipLaunchKernel(kern, dim3((unsigned)R), dim3(kTeamThreads), args, lds, st);
}

}  // namespace sg
