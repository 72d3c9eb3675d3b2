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
// wavefront's maximum, six fused DPP steps; (2) the mover's row, one word per
// lane; (3) the partners' half-gains, spins and leaf maxima, one partner per
// lane; (4) the values of the leaves whose maximum may have changed, and their
// maxima, two leaves at a time (the two chains fill each other's wait states).
// A leaf is rescanned only if it held the mover, if a partner in it passes its
// maximum, or if that partner was its maximum.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sg {
namespace fmcore {

constexpr int32_t kNone = INT32_MIN;  // no unlocked spin; half-gains lie above

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
// the start's energy and becomes the lowest seen (both uniform).  The policy P holds the
// replica's LDS state and the instance's rows:
//   kRL, kTri             leaves per lane; whether the instance has hyper-couplings
//   dc(), tt()            couplings and hyper-couplings per row
//   spin(e), v(e)         +-1; half-gain or kNone once e is locked
//   set(e, v), add(e, d)  store a half-gain; add to one (several lanes may name e)
//   lock(e, s, step)      lock e, flip its spin s, record the move
//   leaf(e)               the leaf of spin e
//   leaf_max(g), set_leaf the leaf table (half-gain, spin)
//   coupling(e, q, j, J), triple(e, q, a, b, K)   entry q of e's row, any q >= 0
//                         (coefficient 0 past the row, the spins then any of the instance's)
//   scan(g, m, a)         maxima of the leaves g[0], g[1] and the spins holding them
template <class P>
__device__ __forceinline__ int run_pass(P& p, const int n, const int lane, long long& E, int32_t (&mx)[P::kRL],
                                        int32_t (&ix)[P::kRL])
{
    constexpr int kPend = P::kTri ? 3 : 1;
    long long above = 0;  // current energy minus the lowest seen
    int best_len = 0;
    const int nq = P::kTri && p.tt() > p.dc() ? p.tt() : p.dc();
    for (int step = 0; step < n; ++step) {
        int32_t m = mx[0], a = ix[0];
#pragma unroll
        for (int i = 1; i < P::kRL; ++i)
            if (mx[i] > m) {
                m = mx[i];
                a = ix[i];
            }
        const int32_t in[1] = {m};
        int32_t top[1];
        wave_max<1>(in, top);
        const int me = __builtin_amdgcn_readlane(a, first_lane(m == top[0]));
        if (top[0] == kNone || (uint32_t)me >= (uint32_t)n) return -1;
        // the mover's row and spin in one round trip
        int j, a3 = 0, b3 = 0;
        int32_t J, K = 0;
        p.coupling(me, lane, j, J);
        if (P::kTri) p.triple(me, lane, a3, b3, K);
        const int s_me = p.spin(me);
        above -= 2LL * top[0];
        if (above < 0) {
            E += above;
            above = 0;
            best_len = step + 1;
        }
        int g0 = p.leaf(me);
        for (int q0 = 0;;) {
            int pend[kPend];  // leaves to take again, per lane
            // a partner's half-gain changes by 2 J s_j s_me or 2 K s_a s_b s_me,
            // modulo 2^32 on the way (the values it ends at are in range)
            auto stale = [&](bool live, int e, int32_t v, int2 l) {
                return live & ((v > l.x) | (e == l.y) | ((v == l.x) & (e < l.y))) ? p.leaf(e) : -1;
            };
            if (!P::kTri) {
                const int32_t v = p.v(j);
                const int sj = p.spin(j);
                const int2 l = p.leaf_max(p.leaf(j));
                const bool live = (J != 0) & (v != kNone);
                const int32_t nv = (int32_t)((uint32_t)v + (uint32_t)J * (uint32_t)(2 * sj * s_me));
                pend[0] = stale(live, j, nv, l);
                if (live) p.set(j, nv);
            } else {
                // a spin may sit in several of the row's terms: the changes
                // are added, then the sums are read
                const int sj = p.spin(j), sa = p.spin(a3), sb = p.spin(b3);
                const int32_t vj = p.v(j), va = p.v(a3), vb = p.v(b3);
                const bool lj = (J != 0) & (vj != kNone), la = (K != 0) & (va != kNone), lb = (K != 0) & (vb != kNone);
                const int32_t dJ = (int32_t)((uint32_t)J * (uint32_t)(2 * sj * s_me));
                const int32_t dK = (int32_t)((uint32_t)K * (uint32_t)(2 * sa * sb * s_me));
                order();
                if (lj) p.add(j, dJ);
                if (la) p.add(a3, dK);
                if (lb) p.add(b3, dK);
                order();
                const int2 xj = p.leaf_max(p.leaf(j)), xa = p.leaf_max(p.leaf(a3)), xb = p.leaf_max(p.leaf(b3));
                pend[0] = stale(lj, j, p.v(j), xj);
                pend[kPend - 2] = stale(la, a3, p.v(a3), xa);
                pend[kPend - 1] = stale(lb, b3, p.v(b3), xb);
            }
            order();
            if (q0 == 0 && lane == 0) p.lock(me, s_me, step);
            order();
            // the stale leaves, two at a time; the mover's first
            auto next = [&]() {
                int g = -1;
#pragma unroll
                for (int c = kPend - 1; c >= 0; --c) {
                    const uint64_t b = __ballot(pend[c] >= 0);
                    if (b) g = __builtin_amdgcn_readlane(pend[c], (int)__builtin_ctzll(b));
                }
                return g;
            };
            auto done = [&](int g) {
#pragma unroll
                for (int c = 0; c < kPend; ++c) pend[c] = pend[c] == g ? -1 : pend[c];
            };
            if (q0 != 0) g0 = next();
            while (g0 >= 0) {
                int g[2] = {g0, g0}, gx[2], gi[2];
                done(g0);
                const int g1 = next();
                if (g1 >= 0) {
                    g[1] = g1;
                    done(g1);
                }
                p.scan(g, gx, gi);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
#pragma unroll
                    for (int i = 0; i < P::kRL; ++i)
                        if (lane * P::kRL + i == g[u]) {
                            mx[i] = gx[u];
                            ix[i] = gi[u];
                        }
                }
                if (lane < 2) p.set_leaf(lane ? g[1] : g[0], lane ? gx[1] : gx[0], lane ? gi[1] : gi[0]);
                g0 = g1 >= 0 ? next() : -1;
            }
            order();
            q0 += 64;
            if (q0 >= nq) break;
            p.coupling(me, q0 + lane, j, J);
            if (P::kTri) p.triple(me, q0 + lane, a3, b3, K);
        }
    }
    return best_len;
}

}  // namespace fmcore
}  // namespace sg
