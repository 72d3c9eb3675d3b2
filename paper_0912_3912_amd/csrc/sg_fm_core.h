// sg_fm_core.h -- the move loop shared by the pass kernels that keep a
// replica's half-gains in LDS in external order (sg_fm_rows.hip,
// sg_fm_mid.hip): one wavefront per replica, the unlocked spin of largest
// half-gain found through one level of maxima.  (Internal.)
//
// The spins are split into leaves of consecutive external indices, at most
// 64 RL of them: lane l holds, in registers, the largest half-gain and the
// lowest spin that has it of leaves l RL .. l RL + RL - 1, and the same pairs
// sit in LDS for the lanes that update a partner.  Leaves, and the spins
// inside one, ascend with the lanes, so among equal half-gains the first lane
// that holds the maximum names the lowest spin: no index is carried through a
// maximum, and 32 bits hold any half-gain.
//
// A move is a serial chain, and its length is what a pass costs: (1) the
// mover's row, one word per lane; (2) the partners' half-gains, spins and leaf
// maxima, one partner per lane; (3) the values of the leaves whose maximum may
// have changed; (4) their maxima, two leaves at a time, and the maximum of the
// other leaves beside them, each six fused DPP steps (three chains fill each
// other's wait states), which is the next move.  A leaf is rescanned only if
// it held the mover, if a partner in it passes its maximum, or if that partner
// was its maximum.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sg {
namespace fmcore {

// A lane's leaves in registers (a vector type: an array indexed by a running
// maximum would go to scratch memory).
template <int RL>
using Leaves = int32_t __attribute__((ext_vector_type(RL)));

// Same-wavefront LDS operations complete in issue order: this only keeps the
// compiler from moving them across the point.
__device__ __forceinline__ void order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One step of a wave-wide signed maximum; lanes that receive nothing see the
// identity, so that the move and the maximum become one instruction.
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t max_step(int32_t v)
{
    const int32_t w = __builtin_amdgcn_update_dpp(INT32_MIN, v, CTRL, ROWS, 0xF, false);
    return w > v ? w : v;
}

// Maxima over the 64 lanes (all active) of NU independent values, uniform.
template <int NU>
__device__ __forceinline__ void wave_max(const int32_t (&in)[NU], int32_t (&out)[NU])
{
    int32_t v[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = max_step<0xB1, 0xF>(in[u]);  // quad_perm [1,0,3,2]
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = max_step<0x4E, 0xF>(v[u]);  // quad_perm [2,3,0,1]
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = max_step<0x141, 0xF>(v[u]);  // row_half_mirror
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = max_step<0x140, 0xF>(v[u]);  // row_mirror
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = max_step<0x142, 0xA>(v[u]);  // row_bcast:15 into rows 1 and 3
#pragma unroll
    for (int u = 0; u < NU; ++u) v[u] = max_step<0x143, 0xC>(v[u]);  // row_bcast:31 into rows 2 and 3
#pragma unroll
    for (int u = 0; u < NU; ++u) out[u] = __builtin_amdgcn_readlane(v[u], 63);
}

__device__ __forceinline__ int first_lane(bool p) { return (int)__builtin_ctzll(__ballot(p)); }

// One pass from the current spins, whose half-gains, leaf maxima (registers
// mx, ix and the leaf table) are in place: moves each of the n spins once.
// Returns the lowest energy's prefix length, or -1 on an internal error; E is
// the start's energy and becomes the lowest seen (both uniform).  The policy P
// holds the replica's LDS state and the instance's rows:
//   kRL, kTri             leaves per lane; whether the instance has hyper-couplings
//   kNone, kBias          the value of a locked spin (below all others); what a
//                         stored value exceeds its half-gain by
//   dc(), tt()            couplings and hyper-couplings per row
//   spin(e), v(e)         +-1; stored half-gain, kNone once e is locked
//   set(e, v), add(e, d)  store a half-gain; add to one (several lanes may name e)
//   lock(e, s, step)      lock e, flip its spin s, record the move
//   leaf(e)               the leaf of spin e
//   leaf_max(g), set_leaf the leaf table (value, spin), for kRL > 1
//   coupling(e, q, j, J), triple(e, q, a, b, K)   entry q of e's row, any q >= 0
//                         (coefficient 0 past the row, the spins then any of the instance's)
//   load(g, x, at)        this lane's part of leaf g: its largest value, and
//                         where in the part it stands first
//   index(g, o, at)       the spin at lane o's position at of leaf g
template <class P>
__device__ __forceinline__ int run_pass(P& p, const int n, const int lane, long long& E, Leaves<P::kRL>& mx,
                                        Leaves<P::kRL>& ix)
{
    constexpr int kPend = P::kTri ? 3 : 1;
    constexpr int RL = P::kRL;
    long long above = 0;  // current energy minus the lowest seen
    int best_len = 0;
    const int nq = P::kTri && p.tt() > p.dc() ? p.tt() : p.dc();
    // a lane's largest leaf but for the leaves g0 and g1
    auto lane_max = [&](int g0, int g1, int32_t& m, int32_t& a) {
        m = P::kNone;
        a = 0;
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const int g = lane * RL + i;
            const int32_t x = ((g == g0) | (g == g1)) ? P::kNone : mx[i];
            a = x > m ? ix[i] : a;
            m = x > m ? x : m;
        }
    };
    // the first move
    int32_t top;
    int me;
    {
        int32_t a, in[1], out[1];
        lane_max(-1, -1, in[0], a);
        wave_max<1>(in, out);
        top = out[0];
        me = __builtin_amdgcn_readlane(a, first_lane(in[0] == top));
    }
    for (int step = 0; step < n; ++step) {
        if (top == P::kNone) return -1;
        // the mover's row and spin in one round trip
        int j, a3 = 0, b3 = 0;
        int32_t J, K = 0;
        p.coupling(me, lane, j, J);
        if (P::kTri) p.triple(me, lane, a3, b3, K);
        const int s_me = p.spin(me);
        above -= 2LL * (top - P::kBias);
        if (above < 0) {
            E += above;
            above = 0;
            best_len = step + 1;
        }
        int g0 = p.leaf(me), g1;
        for (int q0 = 0;;) {
            int pend[kPend];  // leaves to take again, per lane
            // a partner's half-gain changes by 2 J s_j s_me or 2 K s_a s_b s_me,
            // modulo 2^32 on the way (the values it ends at are in range)
            auto leaf_of = [&](int e) -> int2 {
                if constexpr (RL == 1) {
                    const int l = p.leaf(e) * 4;
                    return make_int2(__builtin_amdgcn_ds_bpermute(l, mx[0]), __builtin_amdgcn_ds_bpermute(l, ix[0]));
                } else {
                    return p.leaf_max(p.leaf(e));
                }
            };
            auto stale = [&](bool live, int e, int32_t v, int2 l) {
                return (live & ((v > l.x) | (e == l.y) | ((v == l.x) & (e < l.y)))) ? p.leaf(e) : -1;
            };
            if constexpr (!P::kTri) {
                const int32_t v = p.v(j);
                const int sj = p.spin(j);
                const int2 l = leaf_of(j);
                const bool live = (J != 0) & (v != P::kNone);
                const int32_t nv = (int32_t)((uint32_t)v + (uint32_t)J * (uint32_t)(2 * sj * s_me));
                pend[0] = stale(live, j, nv, l);
                if (live) p.set(j, nv);
            } else {
                // a spin may sit in several of the row's terms: the changes
                // are added, then the sums are read
                const int sj = p.spin(j), sa = p.spin(a3), sb = p.spin(b3);
                const int32_t vj = p.v(j), va = p.v(a3), vb = p.v(b3);
                const bool lj = (J != 0) & (vj != P::kNone), la = (K != 0) & (va != P::kNone),
                           lb = (K != 0) & (vb != P::kNone);
                const int32_t dJ = (int32_t)((uint32_t)J * (uint32_t)(2 * sj * s_me));
                const int32_t dK = (int32_t)((uint32_t)K * (uint32_t)(2 * sa * sb * s_me));
                const int2 xj = leaf_of(j), xa = leaf_of(a3), xb = leaf_of(b3);
                order();
                if (lj) p.add(j, dJ);
                if (la) p.add(a3, dK);
                if (lb) p.add(b3, dK);
                order();
                pend[0] = stale(lj, j, p.v(j), xj);
                pend[kPend - 2] = stale(la, a3, p.v(a3), xa);
                pend[kPend - 1] = stale(lb, b3, p.v(b3), xb);
            }
            order();
            if (q0 == 0 && lane == 0) p.lock(me, s_me, step);
            order();
            // the stale leaves, two at a time; the mover's first
            auto next = [&]() {  // -1: none
                int g = -1;
#pragma unroll
                for (int c = kPend - 1; c >= 0; --c) {
                    const uint64_t b = __ballot(pend[c] >= 0);
                    if (b) g = __builtin_amdgcn_readlane(pend[c], (int)__builtin_ctzll(b));
                }
#pragma unroll
                for (int c = 0; c < kPend; ++c) pend[c] = pend[c] == g ? -1 : pend[c];
                return g;
            };
            auto keep = [&](int g, int32_t x, int32_t a) {
#pragma unroll
                for (int i = 0; i < RL; ++i) {
                    const bool mine = lane * RL + i == g;
                    mx[i] = mine ? x : mx[i];
                    ix[i] = mine ? a : ix[i];
                }
            };
            q0 += 64;
            const bool last = q0 >= nq;
            if (q0 != 64) g0 = next();
#pragma unroll
            for (int c = 0; c < kPend; ++c) pend[c] = pend[c] == g0 ? -1 : pend[c];
            for (;;) {
                if (g0 < 0) g0 = 0;  // nothing is stale: any leaf serves
                g1 = next();
                int any = pend[0];
#pragma unroll
                for (int c = 1; c < kPend; ++c) any &= pend[c];
                const bool more = g1 >= 0 && __ballot(any >= 0) != 0;
                if (g1 < 0) g1 = g0;
                // the two leaves' maxima and that of the others, in one go
                int32_t x[3], at[2], m[3], a;
                p.load(g0, x[0], at[0]);
                p.load(g1, x[1], at[1]);
                lane_max(g0, g1, x[2], a);
                wave_max<3>(x, m);
                const int o0 = first_lane(x[0] == m[0]), o1 = first_lane(x[1] == m[1]);
                const int i0 = p.index(g0, o0, at[0]), i1 = p.index(g1, o1, at[1]);
                keep(g0, m[0], i0);
                keep(g1, m[1], i1);
                if (RL > 1 && lane < 2) p.set_leaf(lane ? g1 : g0, lane ? m[1] : m[0], lane ? i1 : i0);
                if (more) {
                    g0 = next();
                    continue;
                }
                if (last) {  // the next move: the largest, the lowest spin among equals
                    const int i2 = __builtin_amdgcn_readlane(a, first_lane(x[2] == m[2]));
                    top = max(m[0], max(m[1], m[2]));
                    me = m[0] == top ? i0 : INT32_MAX;
                    me = m[1] == top ? min(me, i1) : me;
                    me = m[2] == top ? min(me, i2) : me;
                }
                break;
            }
            order();
            if (last) break;
            p.coupling(me, q0 + lane, j, J);
            if (P::kTri) p.triple(me, q0 + lane, a3, b3, K);
        }
    }
    return best_len;
}

// run_pass for instances without hyper-couplings whose rows have 1 to 64
// couplings (one lane per coupling).  Spins are not flipped while it runs: an
// unlocked partner has not moved and the mover moves once, so every spin that
// a move reads is the pass's first.  Beyond what run_pass asks of it, the
// policy gives
//   kLocked               the largest value of a locked spin
//   row(e, j, J)          this lane's coupling of e, for the lanes past the row
//                         any of them (the same update, stored twice); unused
//                         entries name e itself, which is locked by then
//   tag(e, step)          lane 0: lock e and record its step
//   fetch(g), part(w, x, at)  load in two halves
//   kPlaced               where the loop stands matters: its head comes to lie 4
//                         bytes past a multiple of 32 (instructions are fetched
//                         32 bytes at a time, and a wavefront is alone on its
//                         SIMD: a pass of a 50 x 50 lattice takes 0.995 ms
//                         there, 1.004 to 1.040 at the other seven places)
template <class P>
__device__ __forceinline__ int run_pass_pairs(P& p, const int n, const int lane, long long& E, Leaves<P::kRL>& mx,
                                              Leaves<P::kRL>& ix)
{
    constexpr int RL = P::kRL;
    long long above = 0, low = 0;  // half the energy over the lowest seen; half the lowest, from the start's
    int best_len = 0;
    int32_t top, worst = INT32_MAX;
    int me;
    {
        int32_t a = ix[0], in[1] = {mx[0]}, out[1];
#pragma unroll
        for (int i = 1; i < RL; ++i) {
            a = mx[i] > in[0] ? ix[i] : a;
            in[0] = mx[i] > in[0] ? mx[i] : in[0];
        }
        wave_max<1>(in, out);
        top = out[0];
        me = __builtin_amdgcn_readlane(a, first_lane(in[0] == top));
    }
    auto keep = [&](int g, int32_t x, int32_t a) {
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const bool mine = lane * RL + i == g;
            mx[i] = mine ? x : mx[i];
            ix[i] = mine ? a : ix[i];
        }
    };
    int step = 0;
    if constexpr (P::kPlaced) asm volatile(".p2align 5\n\t.rept 4\n\ts_nop 0\n\t.endr");
    do {
        worst = min(worst, top);  // a locked spin's: an internal error, seen at the end
        me = min(me, n - 1);
        int j;
        int32_t J;
        p.row(me, j, J);
        const int s_me = p.spin(me);
        p.tag(me, step);
        order();
        above -= top - P::kBias;
        if ((int32_t)(above >> 32) < 0) {
            asm volatile("");  // a branch: most moves of a pass's long tail skip it
            low += above;
            above = 0;
            best_len = step + 1;
        }
        // the partners: v_j changes by 2 J s_j s_me
        const int32_t v = p.v(j);
        const int sj = p.spin(j);
        const int lj = p.leaf(j);
        int2 l;
        if constexpr (RL == 1)
            l = make_int2(__builtin_amdgcn_ds_bpermute(lj * 4, mx[0]), __builtin_amdgcn_ds_bpermute(lj * 4, ix[0]));
        else
            l = p.leaf_max(lj);
        const int32_t nv = (int32_t)((uint32_t)v + (uint32_t)J * (uint32_t)(2 * sj * s_me));
        if (v > P::kLocked) p.set(j, nv);
        order();
        // stale leaves (one ballot per comparison: that of a combined
        // condition costs a select and another comparison)
        uint64_t st = __ballot(nv > l.x) | __ballot(j == l.y) | (__ballot(nv == l.x) & __ballot(j < l.y));
        st &= __ballot(v > P::kLocked);
        const int g0 = p.leaf(me);
        st &= ~__ballot(lj == g0);
        int g1 = g0;
        if (st) g1 = __builtin_amdgcn_readlane(lj, (int)__builtin_ctzll(st));
        st &= ~__ballot(lj == g1);
        while (st) {  // a third stale leaf and further ones
            const int g = __builtin_amdgcn_readlane(lj, (int)__builtin_ctzll(st));
            st &= ~__ballot(lj == g);
            int32_t x[1], at, m[1];
            p.load(g, x[0], at);
            wave_max<1>(x, m);
            const int i = p.index(g, first_lane(x[0] == m[0]), at);
            keep(g, m[0], i);
            if (RL > 1 && lane == 0) p.set_leaf(g, m[0], i);
        }
        // the maximum of the other leaves while the two leaves' values are read
        const auto w0 = p.fetch(g0), w1 = p.fetch(g1);
        int32_t y[1] = {INT32_MIN}, my[1], a = ix[0];
#pragma unroll
        for (int i = 0; i < RL; ++i) {
            const int g = lane * RL + i;
            const int32_t z = ((g == g0) | (g == g1)) ? INT32_MIN : mx[i];
            a = i && z > y[0] ? ix[i] : a;
            y[0] = i && y[0] > z ? y[0] : z;
        }
        wave_max<1>(y, my);
        const int i2 = __builtin_amdgcn_readlane(a, first_lane(y[0] == my[0]));
        __builtin_amdgcn_sched_barrier(0);
        int32_t x[2], at[2], m[2];
        p.part(w0, x[0], at[0]);
        p.part(w1, x[1], at[1]);
        wave_max<2>(x, m);
        const int i0 = p.index(g0, first_lane(x[0] == m[0]), at[0]);
        const int i1 = p.index(g1, first_lane(x[1] == m[1]), at[1]);
        // the next move: the largest, the lowest spin among equals
        top = max(my[0], max(m[0], m[1]));
        me = m[0] == top ? i0 : INT32_MAX;
        me = m[1] == top ? min(me, i1) : me;
        me = my[0] == top ? min(me, i2) : me;
        keep(g0, m[0], i0);
        keep(g1, m[1], i1);
        if (RL > 1 && lane < 2) p.set_leaf(lane ? g1 : g0, lane ? m[1] : m[0], lane ? i1 : i0);
        order();
    } while (++step < n);
    E += 2 * low;
    return worst > P::kLocked ? best_len : -1;
}

}  // namespace fmcore
}  // namespace sg
