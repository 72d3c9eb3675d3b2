// sg_team.hip -- colour-ordered sweeps of one instance in one launch: a team
// of G workgroups per replica, every phase of every sweep inside the kernel
// (sg_team_core.h).  It runs what SG_SCHED_AUTO would give to per-phase launches:
// few replicas of an irregular graph, whose phases take a few microseconds
// each, so that launches, the gaps between them, and the host's checks of the
// stopping rule cost more than the phases.  Bound by the latency of the chain
// of phases: LDS reads, the exchange's round trip through memory between
// compute units, the barrier (and the traffic of the exchange: every member
// reads every word of the phase).  500000 spins of a 3-regular graph to
// convergence (7 sweeps of 4 colours): the kernel 97 us, 3.5 us a phase; the
// call (sg_run_sweeps) 155 us, against 334 us with per-phase launches.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sg_launch.h"
#include "sg_layout.h"
#include "sg_team_core.h"

namespace sg {

// Grid: R teams of G workgroups (workgroup r G + m: member m of replica r's).
// ct: the C + 1 slice offsets of the colours.  words: per replica two copies of
// two words per slice, tags zero on entry.  acc slots (nslots per replica, zero
// on entry) take the energy changes (of a replica that converged, -6 times its
// energy) and flips, rs[r].lastflip 1 + the last
// sweep that flipped.  Dynamic LDS: the spins, then from word tl_off on a
// TeamLds.  save_words: the 16-bit words of a replica's start in wait.save.
// CONV: run until converged.
template <bool BYTES, bool TIE, bool TRI, int W, bool CONV>
__global__ __launch_bounds__(kTeamThreads) void k_team(const InstDev I, const int32_t* __restrict__ ct, int C,
                                                       int8_t* __restrict__ spins, int64_t stride,
                                                       RepState* __restrict__ rs, int G, int64_t* __restrict__ acc,
                                                       int nslots, uint64_t* __restrict__ words, TeamWait wait,
                                                       int64_t save_words, int T, uint64_t seed, uint32_t tl_off)
{
    extern __shared__ __align__(16) uint32_t bits[];
    // behind the spins, which start LDS
    TeamLds& tl = *reinterpret_cast<TeamLds*>(bits + tl_off);
    const int r = (int)blockIdx.x / G, m = (int)blockIdx.x % G;
    RepState* st = rs + r;
    if (st->converged) return;  // the same for the whole team
    if (G > 1) wait.save += save_words * r;
    const TeamArgs A{I,    ct, C, G,          m,    r,    spins + stride * r, words + (size_t)r * I.nslices * 4,
                     wait, (uint32_t)st->sweeps, T, CONV, seed, &tl};
    const TeamOut o = team_run<BYTES, TIE, TRI, CONV, W>(A);
    if (o.dead) return;
    // a sweep without a flip evaluates every spin on the final configuration:
    // its fields give the energy itself, which k_end takes in place of the change
    const long long wd = team_wave_sum(CONV && o.lastflip < o.performed ? o.e6 : o.dE);
    if ((threadIdx.x & 63) == 0) {
        int64_t* a = acc + 2 * ((int64_t)r * nslots + m % nslots);
        if (wd) atomicAdd((unsigned long long*)a, (unsigned long long)wd);
        if (o.nf) atomicAdd((unsigned long long*)a + 1, (unsigned long long)o.nf);
    }
    if (m == 0 && threadIdx.x == 0) st->lastflip = o.lastflip;
}

// Replicas r0 + blockIdx.y, those not frozen, back to the start that their team
// kept, sixteen spins a thread.
__global__ void k_team_restore(const uint16_t* __restrict__ save, int64_t save_words, int n, int8_t* __restrict__ spins,
                               int64_t stride, const RepState* __restrict__ rs)
{
    const int r = (int)blockIdx.y, k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (rs[r].converged || k * 16 >= n) return;
    const uint32_t b = save[save_words * r + k];
    for (int u = 0; u < 16 && k * 16 + u < n; ++u) spins[stride * r + k * 16 + u] = (b >> u & 1u) ? (int8_t)-1 : (int8_t)1;
}

// Rows of at most four couplings take a third of the loads (hyper-coupled rows
// are not that short).  A workgroup alone holds the spins as bytes where they
// fit, which takes half the instructions of bits (6000 spins of a 3-regular
// graph, 16 sweeps under TIE: 141 us as bits, 106 as bytes).
constexpr int kTeamByteN = 150000;
static bool team_bytes(int n, int G) { return G == 1 && n <= kTeamByteN; }
template <bool BYTES, bool CONV>
static const void* team_variant(bool tie, bool tri, int ew)
{
    if (tri) return tie ? (const void*)k_team<BYTES, true, true, kTeamW, CONV> : (const void*)k_team<BYTES, false, true, kTeamW, CONV>;
    if (ew <= 4) return tie ? (const void*)k_team<BYTES, true, false, 4, CONV> : (const void*)k_team<BYTES, false, false, 4, CONV>;
    return tie ? (const void*)k_team<BYTES, true, false, kTeamW, CONV> : (const void*)k_team<BYTES, false, false, kTeamW, CONV>;
}
static const void* team_kernel(bool bytes, bool conv, bool tie, bool tri, int ew)
{
    if (conv) return bytes ? team_variant<true, true>(tie, tri, ew) : team_variant<false, true>(tie, tri, ew);
    return bytes ? team_variant<true, false>(tie, tri, ew) : team_variant<false, false>(tie, tri, ew);
}

static size_t team_bits(int n) { return (((size_t)(n + 31) / 32 + 1) * 4 + 15) / 16 * 16; }
// LDS before TeamLds
static size_t team_spins(int n, int G) { return team_bytes(n, G) ? ((size_t)n + 15) / 16 * 16 : team_bits(n); }

bool team_fits(int n, int C) { return team_bits(n) <= 150 * 1024 && C >= 1 && C <= kTeamColours; }

int team_max_blocks(int n, bool tie, bool tri, int ew)
{
    const void* kern = team_kernel(false, true, tie, tri, ew);  // (the one with more registers)
    const size_t lds = team_bits(n) + sizeof(TeamLds);
    int per_cu = 0, dev = 0, cus = 0;
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kTeamThreads, lds) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu * cus;
}

hipError_t launch_team(const InstDev& I, int ew, const int32_t* ct, int C, int8_t* spins, int64_t stride, RepState* rs, int R,
                       int G, int64_t* acc, int nslots, uint64_t* words, const TeamWait& wait0, int T, uint64_t seed,
                       int rule, int until_conv, hipStream_t st)
{
    if (R <= 0 || T <= 0) return hipSuccess;
    if (G < 1 || !team_fits(I.n, C) || (G > 1 && !(words && wait0.err && wait0.flag && wait0.save)))
        return hipErrorInvalidValue;
    TeamWait wait = wait0;
    int64_t save_words = (int64_t)team_save_words(I.n);
    const void* kern = team_kernel(team_bytes(I.n, G), until_conv != 0, rule == 1, I.has_tri != 0, ew);
    const size_t lds = team_spins(I.n, G) + sizeof(TeamLds);
    static const bool free0 = [] {
        bool ok = true;
        for (int v = 0; v < 32; ++v) ok = ok && team_lds_free(team_kernel(v & 16, v & 8, v & 1, v & 4, v & 2 ? 4 : kTeamW));
        return ok;
    }();
    if (!free0) return hipErrorInvalidDeviceFunction;
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    InstDev a0 = I;
    uint32_t tl_off = (uint32_t)(team_spins(I.n, G) / 4);
    void* args[] = {&a0, &ct, &C, &spins, &stride, &rs, &G, &acc, &nslots, &words, &wait, &save_words, &T, &seed, &tl_off};
    // members wait for each other: the cooperative launch has them all resident
    if (G > 1) return hipLaunchCooperativeKernel(kern, dim3((unsigned)(R * G)), dim3(kTeamThreads), args, (unsigned)lds, st);
    return hipLaunchKernel(kern, dim3((unsigned)R), dim3(kTeamThreads), args, lds, st);
}

hipError_t launch_team_restore(const uint16_t* save, int n, int8_t* spins, int64_t stride, const RepState* rs, int R,
                               hipStream_t st)
{
    hipLaunchKernelGGL(k_team_restore, dim3((unsigned)((n + 4095) / 4096), (unsigned)R), dim3(256), 0, st, save,
                       (int64_t)team_save_words(n), n, spins, stride, rs);
    return hipGetLastError();
}

}  // namespace sg
