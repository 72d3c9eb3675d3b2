// sg_bits.hip -- the block schedule under GREEDY and GREEDY_TIE in bit-sliced
// form: one 32-bit LDS word holds spin i of 32 restarts of an instance (bit b
// set when restart b has s_i = -1), and one lane decides a row of the sliced
// layout for those 32 restarts with word operations.
//
// For spin i let W_i be the sum of |c| over its terms (field, couplings,
// hyper-couplings: Sec. II eq. (1), Sec. VI eq. (5)) and U_i the part of it
// carried by terms that s_i does not satisfy (c times the product of the
// term's spins negative).  Then s_i f_i = W_i - 2 U_i, and the local move
// lowers the energy iff 2 U_i > W_i, i.e. U_i >= floor(W_i / 2) + 1, and leaves
// it unchanged iff 2 U_i = W_i.  A term is unsatisfied in restart b iff the XOR
// of its spins' bits and of the coefficient's sign bit is 1, so U_i is a
// weighted sum of such masks, summed bit-sliced into 8 bits.  With
// k_i = 127 - floor(W_i / 2) the carry of U_i + k_i into bit 7, or bit 7 of U_i,
// is the flip mask; U_i + k_i = 127 with W_i even the mask of ties.
// Coefficients of magnitude at most 15 (4-bit weights) and W_i <= 255 keep the
// sum within 8 bits; the host routes other instances to the byte kernel.
//
// Vector instructions bound the kernel (95% of the issue slots in long runs),
// so the terms of a row are summed by columns: the field and the first three,
// four or six couplings of every weight bit through full adders (two
// v_bitop3 each), then the four columns' counts, further terms three at a
// time; and a term word holds what a lane needs in place (partner's byte
// offset, weight bits, sign).  A term costs ~11 instructions to read and mask
// and ~6 to sum, against ~16 and ~9 when each entered an 8-bit counter in
// groups of four.  50 sweeps of 1024 Chimera instances x 256 restarts (6.7e9
// attempts) take 2.09 ms under GREEDY (3.07 ms before; 228 vector instructions
// per 64 rows x 32 restarts against 363) and 2.70 ms under GREEDY_TIE (14.4 ms
// on the byte kernel, one restart per lane).
//
// Under GREEDY_TIE a wavefront queues its ties (row and restart) in LDS and
// draws them 64 at a time, the rest at the end of the colour phase: spins of one
// colour share no term, so a move may wait for the end of its phase.
//
// One wavefront per group of 32 restarts, NG groups per workgroup; each
// wavefront runs its own groups, without waiting for the others.  The 32
// restarts of a group sweep in lockstep; a restart that stops (converged, or
// out of sweeps) is masked out of its group, and a group whose restarts have
// all stopped writes its spins back and takes the next 32 restarts of the
// workgroup's range.  Flip counts per restart are kept as
// bit-sliced counters per lane and summed over lanes when a group stops.
// Energies are not tracked incrementally: a finished group computes them from
// its final spins and the instance's term list (the same integer the
// incremental sum would give).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sg_device.h"
#include "sg_launch.h"
#include "sg_layout.h"

namespace sg {

// One wavefront per group of 32 restarts: NG groups make a workgroup of 64 NG
// threads (measured on 4096 Chimera instances x 256 restarts, 8 groups:
// 3.57 ms with 512 threads, against 4.22 ms with 1024 threads, two
// wavefronts per group; smaller workgroups share a CU and hide each other's
// phase synchronisation).
template <int NG>
constexpr int bits_threads() { return 64 * NG; }

__device__ __forceinline__ int bits_coef(uint32_t w) { return (int)(int8_t)(w & 0xffu); }

__device__ __forceinline__ uint32_t bit_xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t bit_maj(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
// a + b + c of one column: its bit, and its carry.
__device__ __forceinline__ void bit_fa(uint32_t a, uint32_t b, uint32_t c, uint32_t& s, uint32_t& cy)
{
    const uint32_t t = bit_xor3(a, b, c);
    cy = bit_maj(a, b, c);
    s = t;
}
__device__ __forceinline__ void bit_ha(uint32_t a, uint32_t b, uint32_t& s, uint32_t& cy)
{
    const uint32_t t = a ^ b;
    cy = a & b;
    s = t;
}

// Term words in LDS: bits 0..15 the byte offset of the partner's spin word,
// bits 16..19 |c|, bit 31 set when c < 0.
__device__ __forceinline__ uint32_t bits_term(uint32_t off, int c)
{
    return off | (uint32_t)abs(c) << 16 | (c < 0 ? 0x80000000u : 0u);
}
__device__ __forceinline__ uint32_t bits_sign(uint32_t w) { return (uint32_t)((int32_t)w >> 31); }
__device__ __forceinline__ uint32_t bits_spin(const uint32_t* sp, uint32_t w)
{
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint8_t*>(sp) + (w & 0xFFFFu));
}
// The weight's bits where the term is unsatisfied.
__device__ __forceinline__ void bits_mask(uint32_t w, uint32_t unsat, uint32_t (&m)[4])
{
#pragma unroll
    for (int p = 0; p < 4; ++p) m[p] = unsat & (uint32_t)__builtin_amdgcn_sbfe((int)w, 16 + p, 1);
}

// U (7 bits) = the sum of N terms' weighted masks, N = 4, 5 or 7 (at most 105).
template <int N>
__device__ __forceinline__ void bits_sum(const uint32_t (&m)[N][4], uint32_t (&U)[8])
{
    static_assert(N == 4 || N == 5 || N == 7, "columns of 4, 5 or 7");
    uint32_t c[4][3];  // per weight bit the count of its masks
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        uint32_t s, a, b;
        bit_fa(m[0][p], m[1][p], m[2][p], s, a);
        if constexpr (N == 4) {
            bit_ha(s, m[3][p], c[p][0], b);
            bit_ha(a, b, c[p][1], c[p][2]);
        } else if constexpr (N == 5) {
            bit_fa(s, m[3][p], m[4][p], c[p][0], b);
            bit_ha(a, b, c[p][1], c[p][2]);
        } else {
            uint32_t s2, d;
            bit_fa(m[3][p], m[4][p], m[5][p], s2, b);
            bit_fa(s, s2, m[6][p], c[p][0], d);
            bit_fa(a, b, d, c[p][1], c[p][2]);
        }
    }
    uint32_t t[2][5];  // count 0 + 2 count 1, count 2 + 2 count 3
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t k;
        t[h][0] = c[2 * h][0];
        bit_ha(c[2 * h][1], c[2 * h + 1][0], t[h][1], k);
        bit_fa(c[2 * h][2], c[2 * h + 1][1], k, t[h][2], k);
        bit_ha(c[2 * h + 1][2], k, t[h][3], t[h][4]);
    }
    uint32_t k;
    U[0] = t[0][0];
    U[1] = t[0][1];
    bit_ha(t[0][2], t[1][0], U[2], k);
    bit_fa(t[0][3], t[1][1], k, U[3], k);
    bit_fa(t[0][4], t[1][2], k, U[4], k);
    bit_ha(t[1][3], k, U[5], k);
    U[6] = t[1][4] ^ k;
    U[7] = 0u;
}

// U += three terms' weighted masks (at most 45), on 8 bits.
__device__ __forceinline__ void bits_add3(uint32_t (&U)[8], const uint32_t (&m)[3][4])
{
    uint32_t s[4], c[4], T[6], k;
#pragma unroll
    for (int p = 0; p < 4; ++p) bit_fa(m[0][p], m[1][p], m[2][p], s[p], c[p]);
    T[0] = s[0];
    bit_ha(s[1], c[0], T[1], k);
    bit_fa(s[2], c[1], k, T[2], k);
    bit_fa(s[3], c[2], k, T[3], k);
    bit_ha(c[3], k, T[4], T[5]);
    bit_ha(U[0], T[0], U[0], k);
#pragma unroll
    for (int p = 1; p < 6; ++p) bit_fa(U[p], T[p], k, U[p], k);
    bit_ha(U[6], k, U[6], k);
    U[7] ^= k;
}

__device__ __forceinline__ uint32_t wave_or(uint32_t v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v |= __shfl_xor(v, off, 64);
    return v;
}

// The value of lane ^ 1, 2, (mirrors within 8 and 16), 16, 32, for step 0..5:
// together they reach every lane, and each step pairs lanes whose sums so far
// cover distinct lanes.
template <int STEP>
__device__ __forceinline__ uint32_t bits_other(uint32_t v)
{
    if constexpr (STEP == 0) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
    else if constexpr (STEP == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
    else if constexpr (STEP == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true);
    else if constexpr (STEP == 3) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true);
    else return (uint32_t)__shfl_xor((int)v, STEP == 4 ? 16 : 32, 64);
}

// Sum over the wavefront of bit-sliced counters of IN bits (OUT >= IN + 6, or
// any OUT that holds the sum): lane b < 32 returns the sum of bit b's counters.
template <int STEP, int IN, int OUT>
__device__ __forceinline__ void bits_fold(uint32_t (&B)[OUT])
{
    if constexpr (STEP < 6) {
        constexpr int N = IN + STEP < OUT ? IN + STEP : OUT;  // bits in use
        uint32_t k = 0;
#pragma unroll
        for (int p = 0; p < N; ++p) {
            const uint32_t o = bits_other<STEP>(B[p]);
            bit_fa(B[p], o, k, B[p], k);
        }
        if constexpr (N < OUT) B[N] = k;
        bits_fold<STEP + 1, IN, OUT>(B);
    }
}
template <int IN, int OUT>
__device__ __forceinline__ int bits_total(uint32_t (&B)[OUT], int lane)
{
    bits_fold<0, IN, OUT>(B);
    int v = 0;
#pragma unroll
    for (int p = 0; p < OUT; ++p) v |= (int)((B[p] >> (lane & 31)) & 1u) << p;
    return v;
}

constexpr int kTieCap = 128;  // queued ties of a wavefront: at most 63 kept, 64 appended at a time

template <int NG, bool TIE>
__global__ __launch_bounds__(bits_threads<NG>()) void k_block_bits(const InstTab* __restrict__ tab,
                                                             const int32_t* __restrict__ ctab,
                                                             const BlockItem* __restrict__ items,
                                                             RepState* __restrict__ rs, CallStats* __restrict__ cs,
                                                             int T, uint64_t seed, int until_conv)
{
    constexpr int kBitsThreads = bits_threads<NG>(), kBitsWaves = kBitsThreads / 64;
    constexpr int WPG = kBitsWaves / NG;  // wavefronts per group of 32 restarts
    static_assert(WPG == 1, "one wavefront per group");
    extern __shared__ uint64_t lds64[];
    const BlockItem it = items[blockIdx.x];
    const InstTab& Q = tab[it.inst];
    const InstDev& I = Q.I;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = wave % NG, wk = wave / NG;  // the wavefront's group, its index within the group
    const int n = I.n;
    const int r_end = it.r0 + it.nr;
    const int ew = Q.nbr_words, tw = Q.tri_words, nsl = I.nslices, C = Q.C;

    // LDS: slices | coupling words | triple words a | triple words b (byte offsets) | row words |
    // colour table | spin words [NG][n] (group-major: a wavefront's neighbour reads spread over the banks) |
    // per-restart state [NG][32] x 3, and under TIE the restarts' first sweeps, the external indices and
    // the tie queues
    Slice* l_sl = reinterpret_cast<Slice*>(lds64);
    uint32_t* l_nbr = reinterpret_cast<uint32_t*>(l_sl + nsl);
    uint32_t* l_ta = l_nbr + ew;
    uint32_t* l_tb = l_ta + tw;
    uint32_t* l_row = l_tb + tw;  // k_i, bit 7 set when W_i is even; |h_i| and its sign as in a term word
    int32_t* l_cs = reinterpret_cast<int32_t*>(l_row + n);
    uint32_t* l_sp = reinterpret_cast<uint32_t*>(l_cs + C + 1);
    int* r_t = reinterpret_cast<int*>(l_sp + (size_t)n * NG);  // sweeps of each restart in this call
    int* r_last = r_t + NG * 32;                                // 1 + its last sweep that flipped
    int* r_flips = r_last + NG * 32;                            // its flips in this call
    uint32_t* r_base = reinterpret_cast<uint32_t*>(r_flips + NG * 32);  // its sweeps before the call
    uint32_t* l_ext = r_base + NG * 32;
    uint32_t* l_tie = l_ext + n;                                // [NG][kTieCap]: row | restart's bit << 16
    __shared__ int g_r0[NG], g_cnt[NG];                         // restarts [g_r0, g_r0 + g_cnt) in the group's bits
    __shared__ uint32_t g_act[NG], g_part[NG];                  // sweeping; taking part in the call
    __shared__ int next_r, kflush;
    __shared__ unsigned long long b_att, b_flips, b_smax, b_unconv;

    for (int k = tid; k < ew; k += kBitsThreads) {
        const uint32_t w = I.nbr[k];
        l_nbr[k] = bits_term((w >> 8) * 4, bits_coef(w));
    }
    if (I.has_tri)
        for (int k = tid; k < tw; k += kBitsThreads) {
            const uint32_t w = I.ta[k];
            l_ta[k] = bits_term((w >> 8) * 4, bits_coef(w));
            l_tb[k] = I.tb[k] * 4;
        }
    for (int k = tid; k < nsl; k += kBitsThreads) l_sl[k] = I.slices[k];
    for (int k = tid; k <= C; k += kBitsThreads) l_cs[k] = ctab[Q.ctab_off + k];
    if (TIE)
        for (int k = tid; k < n; k += kBitsThreads) l_ext[k] = I.ext[k];
    if (tid == 0) {
        next_r = it.r0;
        b_att = b_flips = b_smax = b_unconv = 0;
    }
    if (tid < NG) {
        g_cnt[tid] = 0;
        g_act[tid] = g_part[tid] = 0u;
    }
    __syncthreads();
    // row words: the field, k_i = 127 - floor(W_i / 2) and W_i's parity
    auto weight = [](uint32_t w) { return (int)((w >> 16) & 15u); };
    for (int sl = wave; sl < nsl; sl += kBitsWaves) {
        const Slice S = l_sl[sl];
        if (lane < S.rows) {
            const int i = (int)S.row0 + lane, h = I.h[i];
            int W = abs(h);
            for (int k = 0; k < S.ew; ++k) W += weight(l_nbr[S.ebase + k * kSlice + lane]);
            for (int k = 0; k < S.tw; ++k) W += weight(l_ta[S.tbase + k * kSlice + lane]);
            l_row[i] = bits_term((uint32_t)(127 - W / 2) | (W & 1 ? 0u : 128u), h);
        }
    }
    if (tid == 0) {
        int rows = 0;
        for (int c = 0; c < C; ++c) rows += (l_cs[c + 1] - l_cs[c] + WPG - 1) / WPG;
        kflush = max(1, 255 / max(1, rows));  // sweeps between counter flushes: a lane flips a row at most once a sweep
    }

    // next group of up to 32 restarts with at least one not frozen (the group's wavefront)
    auto fetch = [&]() {
        for (;;) {
            int r = 0;
            if (lane == 0) r = atomicAdd(&next_r, 32);
            r = __shfl(r, 0, 64);
            if (r >= r_end) {
                if (lane == 0) {
                    g_cnt[g] = 0;
                    g_act[g] = g_part[g] = 0u;
                }
                return false;
            }
            const int cnt = min(32, r_end - r);
            const bool live = lane < cnt && !rs[Q.rep_base + r + lane].converged;
            const uint32_t act = (uint32_t)__ballot(live);
            if (!act) continue;
            if (lane < 32) {
                r_t[g * 32 + lane] = 0;
                r_last[g * 32 + lane] = 0;
                r_flips[g * 32 + lane] = 0;
                if (TIE) r_base[g * 32 + lane] = lane < cnt ? (uint32_t)rs[Q.rep_base + r + lane].sweeps : 0u;
            }
            if (lane == 0) {
                g_r0[g] = r;
                g_cnt[g] = cnt;
                g_act[g] = g_part[g] = act;
            }
            return true;
        }
    };
    // spins of group g between global bytes and LDS words (its WPG
    // wavefronts): lane b + 32 h moves 16 consecutive spins of restart b, rows
    // [16 (2 q + h), +16) for chunk pair q, with one 16-byte access, and 16
    // ballots turn the bytes of 64 lanes into 32 spin words.  Rows past n in a
    // chunk stay within the replica's padded spin row and are not stored.
    auto load_group = [&]() {
        const int r0 = g_r0[g], cnt = g_cnt[g];
        const int b = lane & 31, hh = lane >> 5;
        for (int q = wk; q * 32 < n; q += WPG) {
            const int i0 = q * 32 + hh * 16;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (b < cnt && i0 < n)
                v = *reinterpret_cast<const uint4*>(Q.spins + (int64_t)(r0 + b) * Q.spin_stride + i0);
            const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint64_t m = __ballot((wv[r >> 2] >> (8 * (r & 3) + 7)) & 1u);
                const int ia = q * 32 + r, ib = q * 32 + 16 + r;
                if (lane == r && ia < n) l_sp[g * n + ia] = (uint32_t)m;
                if (lane == 32 + r && ib < n) l_sp[g * n + ib] = (uint32_t)(m >> 32);
            }
        }
    };
    auto store_group = [&]() {
        const int r0 = g_r0[g], cnt = g_cnt[g];
        const int b = lane & 31, hh = lane >> 5;
        for (int q = wk; q * 32 < n; q += WPG) {
            const int i0 = q * 32 + hh * 16;
            if (b >= cnt || i0 >= n) continue;
            uint32_t wv[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int i = i0 + r;
                const uint32_t bit = i < n ? (l_sp[g * n + i] >> b) & 1u : 0u;
                wv[r >> 2] |= (bit ? 0xFFu : 0x01u) << (8 * (r & 3));
            }
            int8_t* dst = Q.spins + (int64_t)(r0 + b) * Q.spin_stride + i0;
            if (i0 + 16 <= n) {
                *reinterpret_cast<uint4*>(dst) = make_uint4(wv[0], wv[1], wv[2], wv[3]);
            } else {
                for (int r = 0; r < n - i0; ++r) dst[r] = (int8_t)((wv[r >> 2] >> (8 * (r & 3))) & 0xFFu);
            }
        }
    };

    // Energies of the group's 32 restarts from their final spins (Sec. II
    // eq. (1), Sec. VI eq. (5)): E = -sum c prod s = 2 V - W, with W = sum |c|
    // over the instance's terms and V the |c|-weighted count of unsatisfied
    // terms.  The lanes split the term list, three terms at a time, into an 8-bit
    // bit-sliced count (at most five triples of weight <= 45) that is folded into
    // a 20-bit one (sum |c| <= 2048 * 255 < 2^20 for the instances this kernel
    // takes, and a lane may hold most of it); those are summed over the lanes.
    // Lane b < 32 returns the energy of restart b.
    const uint32_t* ET = Q.eterm;
    const int n_eh = Q.n_eh, n_ee = Q.n_ee, n_et = Q.n_et;
    auto group_energy = [&]() -> long long {
        const uint32_t* spg = l_sp + g * n;
        constexpr int kBW = 20;
        uint32_t A[8] = {0, 0, 0, 0, 0, 0, 0, 0}, B[kBW];
#pragma unroll
        for (int p = 0; p < kBW; ++p) B[p] = 0u;
        int wsum = 0, pending = 0;
        auto fold = [&]() {  // B += A, A = 0
            uint32_t c = 0;
#pragma unroll
            for (int p = 0; p < kBW; ++p) {
                if (p < 8) bit_fa(B[p], A[p], c, B[p], c);
                else bit_ha(B[p], c, B[p], c);
            }
#pragma unroll
            for (int p = 0; p < 8; ++p) A[p] = 0u;
            pending = 0;
        };
        // three terms: word w (coefficient in its top ten bits), spins' bits xored
        auto terms = [&](const uint32_t (&w)[3], const uint32_t (&x)[3]) {
            uint32_t m[3][4];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const int cf = bits_coef(w[u] >> 22);
                wsum += abs(cf);
                const uint32_t t = bits_term(0, cf);
                bits_mask(t, x[u] ^ bits_sign(t), m[u]);
            }
            bits_add3(A, m);
            if (++pending == 5) fold();
        };
        for (int t = lane; t < n_eh; t += 192) {
            uint32_t w[3], x[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                w[u] = t + 64 * u < n_eh ? ET[t + 64 * u] : 0u;
                x[u] = spg[w[u] & 0x7FFu];
            }
            terms(w, x);
        }
        for (int t = lane; t < n_ee; t += 192) {
            uint32_t w[3], x[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                w[u] = t + 64 * u < n_ee ? ET[n_eh + t + 64 * u] : 0u;
                x[u] = spg[w[u] & 0x7FFu] ^ spg[(w[u] >> 11) & 0x7FFu];
            }
            terms(w, x);
        }
        for (int t = lane; t < n_et; t += 192) {
            uint32_t w[3], x[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const bool in = t + 64 * u < n_et;
                w[u] = in ? ET[n_eh + n_ee + 2 * (t + 64 * u)] : 0u;
                const uint32_t b = in ? ET[n_eh + n_ee + 2 * (t + 64 * u) + 1] : 0u;
                x[u] = spg[w[u] & 0x7FFu] ^ spg[(w[u] >> 11) & 0x7FFu] ^ spg[b];
            }
            terms(w, x);
        }
        fold();
        const long long V = bits_total<kBW, kBW>(B, lane);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) wsum += __shfl_xor(wsum, off, 64);
        return 2 * V - (long long)wsum;
    };

    // Each wavefront runs its own group (one wavefront per group): it sweeps,
    // keeps its restarts' counters, finishes the group and takes the next
    // restarts without waiting for the other groups of the workgroup.  Its
    // LDS writes and later reads by other lanes of the same wavefront are
    // ordered by wavefront fences (LDS operations of a wavefront complete in
    // order; the fences keep the compiler from moving them).
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    __syncthreads();  // flip offsets and kflush are read by every wavefront
    bool have = fetch();
    wave_sync();
    if (have) load_group();
    wave_sync();

    uint32_t cnt8[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // this lane's flips per restart of its group, bit-sliced
    int since = 0;                                 // sweeps since the counters were last flushed
    uint32_t act = have ? g_act[g] : 0u;
    uint32_t* sp = l_sp + g * n;
    uint32_t* ties = l_tie + g * kTieCap;
    while (have) {
        uint32_t any = 0;
        int queued = 0;
        // draw up to 64 queued ties, the last ones: flip where the sweep's
        // random bit is 1 (Philox counter: spin, absolute sweep, instance, restart)
        auto draw = [&]() {
            wave_sync();
            const int k = queued < 64 ? queued : 64;
            if (lane < k) {
                const uint32_t e = ties[queued - 1 - lane];
                const int i = (int)(e & 0xFFFFu), b = (int)(e >> 16);
                const uint32_t sweep = r_base[g * 32 + b] + (uint32_t)r_t[g * 32 + b];
                if (rng_bit(seed, l_ext[i], sweep, I.instance_id, (uint32_t)(g_r0[g] + b))) {
                    atomicXor(&sp[i], 1u << b);
                    atomicAdd(&r_flips[g * 32 + b], 1);
                    any |= 1u << b;
                }
            }
            queued -= k;
            wave_sync();
        };
        for (int c = 0; c < C; ++c) {
            const int s_hi = __builtin_amdgcn_readfirstlane(l_cs[c + 1]);
            for (int sl = __builtin_amdgcn_readfirstlane(l_cs[c]); sl < s_hi; ++sl) {
                // the slice's numbers are the same in every lane: scalar loop bounds
                const uint4 raw = *reinterpret_cast<const uint4*>(l_sl + sl);
                const int row0 = __builtin_amdgcn_readfirstlane((int)raw.x);
                const uint32_t widths = (uint32_t)__builtin_amdgcn_readfirstlane((int)raw.w);
                const int sew = (int)(widths & 0xFFFFu), stw = (int)(widths >> 16 & 0xFFu), rows = (int)(widths >> 24);
                uint32_t tie = 0;
                const int i = row0 + lane;
                if (lane < rows) {
                    const uint32_t* pw = l_nbr + __builtin_amdgcn_readfirstlane((int)raw.y) + lane;
                    const uint32_t rw = l_row[i], xi = sp[i];
                    uint32_t U[8];
                    // the field and the first N - 1 couplings
                    auto head = [&](auto nt) {
                        constexpr int N = decltype(nt)::value;
                        uint32_t w[N], x[N], m[N][4];
#pragma unroll
                        for (int u = 1; u < N; ++u) w[u] = u <= sew ? pw[(u - 1) * kSlice] : 0u;
#pragma unroll
                        for (int u = 1; u < N; ++u) x[u] = bits_spin(sp, w[u]);
                        bits_mask(rw, xi ^ bits_sign(rw), m[0]);
#pragma unroll
                        for (int u = 1; u < N; ++u) bits_mask(w[u], bit_xor3(xi, x[u], bits_sign(w[u])), m[u]);
                        bits_sum<N>(m, U);
                    };
                    int done;
                    if (sew == 0) {  // the field alone (300 free spins, 600 restarts, 200 sweeps: 705 -> 447 us)
                        uint32_t m[4];
                        bits_mask(rw, xi ^ bits_sign(rw), m);
#pragma unroll
                        for (int p = 0; p < 8; ++p) U[p] = p < 4 ? m[p] : 0u;
                        done = 0;
                    } else if (sew <= 3) {
                        head(std::integral_constant<int, 4>{});
                        done = 3;
                    } else if (sew == 4) {
                        head(std::integral_constant<int, 5>{});
                        done = 4;
                    } else {
                        head(std::integral_constant<int, 7>{});
                        done = 6;
                    }
                    for (; done < sew; done += 3) {
                        uint32_t w[3], x[3], m[3][4];
#pragma unroll
                        for (int u = 0; u < 3; ++u) w[u] = done + u < sew ? pw[(done + u) * kSlice] : 0u;
#pragma unroll
                        for (int u = 0; u < 3; ++u) x[u] = bits_spin(sp, w[u]);
#pragma unroll
                        for (int u = 0; u < 3; ++u) bits_mask(w[u], bit_xor3(xi, x[u], bits_sign(w[u])), m[u]);
                        bits_add3(U, m);
                    }
                    if (stw > 0) {
                        const uint32_t* pa = l_ta + __builtin_amdgcn_readfirstlane((int)raw.z) + lane;
                        const uint32_t* pb = pa + tw;
                        for (int k = 0; k < stw; k += 3) {
                            uint32_t wa[3], wb[3], x[3], m[3][4];
#pragma unroll
                            for (int u = 0; u < 3; ++u) {
                                wa[u] = k + u < stw ? pa[(k + u) * kSlice] : 0u;
                                wb[u] = k + u < stw ? pb[(k + u) * kSlice] : 0u;
                            }
#pragma unroll
                            for (int u = 0; u < 3; ++u) x[u] = bits_spin(sp, wa[u]) ^ bits_spin(sp, wb[u]);
#pragma unroll
                            for (int u = 0; u < 3; ++u) bits_mask(wa[u], bit_xor3(xi, x[u], bits_sign(wa[u])), m[u]);
                            bits_add3(U, m);
                        }
                    }
                    // U + k_i: the carry into bit 7, and where all seven bits are 1
                    uint32_t cy = 0, ones = 0;
                    if (TIE) ones = (uint32_t)__builtin_amdgcn_sbfe((int)rw, 7, 1) & ~U[7];
#pragma unroll
                    for (int p = 0; p < 7; ++p) {
                        const uint32_t kp = (uint32_t)__builtin_amdgcn_sbfe((int)rw, p, 1);
                        cy = p == 0 ? U[0] & kp : bit_maj(U[p], kp, cy);
                        if (TIE) ones = __builtin_amdgcn_bitop3_b32(ones, U[p], kp, 0x60);  // ones & (U ^ k)
                    }
                    const uint32_t F = (cy | U[7]) & act;
                    if (TIE) tie = ones & act;
                    if (F) {
                        sp[i] = xi ^ F;
                        any |= F;
                        uint32_t carry = F;
#pragma unroll
                        for (int b = 0; b < 8; ++b) {
                            const uint32_t t = cnt8[b] & carry;
                            cnt8[b] ^= carry;
                            carry = t;
                        }
                    }
                }
                if (TIE) {
                    // one tie of every lane that has one, until none is left
                    for (uint64_t has = __ballot(tie != 0u); has; has = __ballot(tie != 0u)) {
                        if (tie) {
                            const int at = __builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
                            ties[queued + at] = (uint32_t)i | (uint32_t)__builtin_ctz(tie) << 16;
                            tie &= tie - 1;
                        }
                        queued += (int)__popcll(has);
                        if (queued >= 64) draw();
                    }
                }
            }
            if (TIE && queued) draw();
            wave_sync();
        }
        any = wave_or(any);
        // per-restart bookkeeping of the sweep
        bool done = false;
        if (lane < 32 && ((act >> lane) & 1u)) {
            const int t = ++r_t[g * 32 + lane];
            const bool flipped = (any >> lane) & 1u;
            if (flipped) r_last[g * 32 + lane] = t;
            done = (until_conv && !flipped) || t >= T;
        }
        act &= ~(uint32_t)__ballot(done);
        const bool fin = act == 0u;
        if (fin || ++since >= kflush) {
            // flip counters: per restart b, the sum over the lanes
            since = 0;
            uint32_t B[14];
#pragma unroll
            for (int k = 0; k < 14; ++k) B[k] = k < 8 ? cnt8[k] : 0u;
#pragma unroll
            for (int k = 0; k < 8; ++k) cnt8[k] = 0u;
            const int mine = bits_total<8, 14>(B, lane);
            if (lane < 32) r_flips[g * 32 + lane] += mine;
        }
        if (fin) {
            store_group();
            const long long Eg = group_energy();
            if (lane < 32 && ((g_part[g] >> lane) & 1u)) {
                const int t = r_t[g * 32 + lane], last = r_last[g * 32 + lane], nf = r_flips[g * 32 + lane];
                RepState* st = rs + Q.rep_base + g_r0[g] + lane;
                st->E = Eg;
                st->flips += nf;
                st->sweeps += t;
                st->lastflip = last;
                const bool conv = until_conv && last < t;
                if (conv) st->converged = 1;
                atomicAdd(&b_att, (unsigned long long)t * (unsigned long long)n);
                atomicAdd(&b_flips, (unsigned long long)nf);
                atomicMax(&b_smax, (unsigned long long)t);
                if (until_conv && !conv) atomicAdd(&b_unconv, 1ull);
            }
            wave_sync();
            have = fetch();
            wave_sync();
            if (have) load_group();
            wave_sync();
            act = have ? g_act[g] : 0u;
        }
    }
    __syncthreads();
    if (tid == 0) {
        if (b_att) atomicAdd(&cs->attempts, b_att);
        if (b_flips) atomicAdd(&cs->flips, b_flips);
        atomicMax(&cs->sweeps_max, b_smax);
        if (b_unconv) atomicAdd(&cs->unconverged, b_unconv);
    }
}

size_t block_bits_lds_bytes(int n, int nbr_words, int tri_words, int nslices, int C, int NG, bool tie)
{
    size_t b = (size_t)nslices * sizeof(Slice) + (size_t)nbr_words * 4 + (size_t)tri_words * 8;
    b += (size_t)n * 4 + (size_t)(C + 1) * 4;
    b += (size_t)n * NG * 4;
    b += (size_t)NG * 32 * 4 * 3;
    if (tie) b += (size_t)NG * 32 * 4 + (size_t)n * 4 + (size_t)NG * kTieCap * 4;
    return (b + 15) / 16 * 16;
}

static const void* bits_kernel(int NG, bool tie)
{
    switch (NG) {
    case 2: return tie ? (const void*)k_block_bits<2, true> : (const void*)k_block_bits<2, false>;
    case 4: return tie ? (const void*)k_block_bits<4, true> : (const void*)k_block_bits<4, false>;
    case 8: return tie ? (const void*)k_block_bits<8, true> : (const void*)k_block_bits<8, false>;
    case 16: return tie ? (const void*)k_block_bits<16, true> : (const void*)k_block_bits<16, false>;
    default: return nullptr;
    }
}

template <int NG>
static hipError_t launch_bits_ng(const InstTab* tab, const int32_t* ctab, const BlockItem* items, int n_items,
                                 size_t lds, RepState* rs, CallStats* cs, int T, uint64_t seed, bool tie,
                                 int until_conv, hipStream_t st)
{
    hipError_t e = hipFuncSetAttribute(bits_kernel(NG, tie), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (tie)
        hipLaunchKernelGGL((k_block_bits<NG, true>), dim3(n_items), dim3(bits_threads<NG>()), lds, st, tab, ctab, items,
                           rs, cs, T, seed, until_conv);
    else
        hipLaunchKernelGGL((k_block_bits<NG, false>), dim3(n_items), dim3(bits_threads<NG>()), lds, st, tab, ctab,
                           items, rs, cs, T, seed, until_conv);
    return hipGetLastError();
}

hipError_t launch_block_bits(const InstTab* tab, const int32_t* ctab, const BlockItem* items, int n_items, size_t lds,
                             RepState* rs, CallStats* cs, int NG, int T, uint64_t seed, int rule, int until_conv,
                             hipStream_t st)
{
    if (n_items <= 0) return hipSuccess;
    const bool tie = rule == 1;
    switch (NG) {
    case 2: return launch_bits_ng<2>(tab, ctab, items, n_items, lds, rs, cs, T, seed, tie, until_conv, st);
    case 4: return launch_bits_ng<4>(tab, ctab, items, n_items, lds, rs, cs, T, seed, tie, until_conv, st);
    case 8: return launch_bits_ng<8>(tab, ctab, items, n_items, lds, rs, cs, T, seed, tie, until_conv, st);
    case 16: return launch_bits_ng<16>(tab, ctab, items, n_items, lds, rs, cs, T, seed, tie, until_conv, st);
    default: return hipErrorInvalidValue;
    }
}

int block_bits_max_blocks(size_t lds, int NG, bool tie)
{
    const void* kern = bits_kernel(NG, tie);
    int per_cu = 0, dev = 0, cus = 0;
    if (!kern || hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * NG, lds) != hipSuccess ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return per_cu * cus;
}

}  // namespace sg
