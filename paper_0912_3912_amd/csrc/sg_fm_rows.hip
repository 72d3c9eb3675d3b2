// sg_fm_rows.hip -- the paper's pass-based local search with hill-climbing
// (Sec. IV, Fig. 3) on instances of at most 4096 spins whose term rows fit a
// workgroup's LDS: one wavefront per replica, the instance's rows shared by
// the workgroup's wavefronts.  The pass, its tie-break, best prefix, stopping
// rule and counters are those of k_fm (sg_fm.hip).
//
// Everything is in external order.  The workgroup rebuilds the instance's
// rows from the sliced layout once: per spin dc coupling words (partner << 8 |
// J & 255; in the wide form pairs partner, J) and tt hyper-couplings (a << 8 |
// K & 255 and b; in the wide form a, b, K), unused entries with coefficient
// zero, couplings among them naming the spin itself.  A wavefront
// keeps its replica's half-gains v_e = -s_e f_e (int32), spins and move list
// there, and the 64 leaf maxima (leaves of 64 spins) in registers;
// fmcore::run_pass moves the spins.
//
// The kernel is bound by the latency of its serial chain of moves (see
// fmcore::run_pass): a 50 x 50 +-J lattice with 62 restarts to convergence
// takes 10.0 ms here, 0.40 us or 965 cycles a move (119 instructions and four
// LDS round trips), against 107 ms on k_fm, whose lanes each rescan n / 64
// spins one after another and look their rows up through the sliced layout;
// with Gaussian int32 couplings 9.9 ms against 130 ms.  With the device full
// (8192 restarts, two passes) 13.7 ms against 166 ms.  Building the rows counts
// where they are many and the moves few: three passes of one replica of a
// complete graph of 200 spins (a slice per spin) take 1.8 ms, 2.3 ms on k_fm, and
// 12.5 ms if a lane copies a row's couplings one after another.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sg_fm_core.h"
#include "sg_launch.h"
#include "sg_layout.h"

namespace sg {

namespace {

constexpr int kRowsThreads = 1024;

__host__ __device__ inline size_t rows_n64(int n) { return ((size_t)n + 63) & ~(size_t)63; }

// Bytes of the shared rows, and of one wavefront's state.
__host__ __device__ inline size_t rows_stage_bytes(int n, int dc, int tt, bool wide)
{
    const size_t w = (size_t)n * ((size_t)dc * (wide ? 8 : 4) + (size_t)tt * (wide ? 12 : 8));
    return (w + 15) & ~(size_t)15;
}
__host__ __device__ inline size_t rows_wave_bytes(int n) { return 7 * rows_n64(n); }

// The replica's LDS state and the rows, as fmcore::run_pass wants them.
template <bool WIDE, bool TRI>
struct RowsPolicy {
    static constexpr int kRL = 1;
    static constexpr bool kTri = TRI, kPlaced = true;
    static constexpr int32_t kNone = INT32_MIN, kBias = 0;
    const uint32_t* cw;  // couplings
    const uint32_t* tw;  // hyper-couplings
    int32_t* half;
    uint16_t* moves;
    int8_t* sp;
    int dc_, tt_, lane, qc;  // qc: this lane's coupling of a row, or any

    static constexpr int32_t kLocked = INT32_MIN + 4095;
    __device__ __forceinline__ void tag(int e, int step)
    {
        if (lane == 0) half[e] = INT32_MIN + step;
    }
    __device__ __forceinline__ int32_t fetch(int g) const { return half[g * 64 + lane]; }
    __device__ __forceinline__ void part(int32_t w, int32_t& x, int32_t& at) const
    {
        x = w;
        at = 0;
    }
    __device__ __forceinline__ void row(int e, int& j, int32_t& J) const
    {
        if constexpr (WIDE) {
            const uint2 w = reinterpret_cast<const uint2*>(cw)[e * dc_ + qc];
            j = (int)w.x;
            J = (int32_t)w.y;
        } else {
            const uint32_t w = cw[e * dc_ + qc];
            j = (int)(w >> 8);
            J = (int8_t)(w & 0xffu);
        }
    }
    __device__ __forceinline__ int dc() const { return dc_; }
    __device__ __forceinline__ int tt() const { return tt_; }
    __device__ __forceinline__ int spin(int e) const { return sp[e]; }
    __device__ __forceinline__ int32_t v(int e) const { return half[e]; }
    __device__ __forceinline__ void set(int e, int32_t x) { half[e] = x; }
    __device__ __forceinline__ void add(int e, int32_t d) { atomicAdd(half + e, d); }
    __device__ __forceinline__ void lock(int e, int s, int step)
    {
        half[e] = kNone;
        sp[e] = (int8_t)-s;
        moves[step] = (uint16_t)e;
    }
    __device__ __forceinline__ int leaf(int e) const { return e >> 6; }
    __device__ __forceinline__ int2 leaf_max(int) const { return make_int2(0, 0); }  // one leaf per lane: registers
    __device__ __forceinline__ void set_leaf(int, int32_t, int32_t) {}
    __device__ __forceinline__ void coupling(int e, int q, int& j, int32_t& J) const
    {
        if constexpr (WIDE) {
            const bool in = q < dc_;
            const uint2 w = reinterpret_cast<const uint2*>(cw)[in ? e * dc_ + q : 0];
            j = in ? (int)w.x : 0;
            J = in ? (int32_t)w.y : 0;
        } else {
            uint32_t w = cw[q < dc_ ? e * dc_ + q : 0];
            w = q < dc_ ? w : 0u;
            j = (int)(w >> 8);
            J = (int8_t)(w & 0xffu);
        }
    }
    __device__ __forceinline__ void triple(int e, int q, int& a, int& b, int32_t& K) const
    {
        if constexpr (WIDE) {
            const bool in = q < tt_;
            const uint32_t* w = tw + (in ? (e * tt_ + q) * 3 : 0);
            a = in ? (int)w[0] : 0;
            b = in ? (int)w[1] : 0;
            K = in ? (int32_t)w[2] : 0;
        } else {
            const bool in = q < tt_;
            const uint32_t* w = tw + (in ? (e * tt_ + q) * 2 : 0);
            const uint32_t wa = in ? w[0] : 0u;
            a = (int)(wa >> 8);
            b = in ? (int)w[1] : 0;
            K = (int8_t)(wa & 0xffu);
        }
    }
    __device__ __forceinline__ void load(int g, int32_t& x, int32_t& at) const { part(fetch(g), x, at); }
    __device__ __forceinline__ int index(int g, int o, int32_t) const { return g * 64 + o; }
};

// f(l, k) for every row l below `rows` and k below `width` of a slice, on the
// lanes of a wavefront: load(l, k) of four of them before put(l, k, value).
template <class LOAD, class PUT>
__device__ __forceinline__ void slice_entries(int rows, int width, int lane, const LOAD& load, const PUT& put)
{
    const int m = rows * width;
    for (int x0 = lane; x0 < m; x0 += 256) {
        decltype(load(0, 0)) v[4];
        int l[4], k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int x = min(x0 + 64 * u, m - 1);
            k[u] = x / rows;
            l[u] = x - k[u] * rows;
            v[u] = load(l[u], k[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (x0 + 64 * u < m) put(l[u], k[u], v[u]);
    }
}

// What a workgroup runs: restarts [r0, r0 + nr) of one instance.
struct RowsInst {
    const uint32_t* ext;
    int8_t* spins;
    int64_t stride;
    RepState* rs;  // restart 0's
    int n, r0, nr;
};

template <bool WIDE, bool TRI, class ROW, class FIELD>
__device__ __forceinline__ void rows_body(const RowsInst I, const int dc, const int tt, const ROW& fill_rows,
                                          const FIELD& field, CallStats* cs, uint32_t* err, const int max_passes,
                                          const int until_conv)
{
    extern __shared__ __align__(16) uint8_t rows_lds[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int n = I.n;
    const size_t n64 = rows_n64(n);
    uint32_t* cw = reinterpret_cast<uint32_t*>(rows_lds);
    uint32_t* tw = cw + (size_t)n * dc * (WIDE ? 2 : 1);
    uint8_t* state = rows_lds + rows_stage_bytes(n, dc, tt, WIDE);
    // the rows, with the external index of every spin held meanwhile where
    // the first wavefront's half-gains go
    uint32_t* ext = reinterpret_cast<uint32_t*>(state);
    for (int i = threadIdx.x; i < n; i += blockDim.x) ext[i] = I.ext[i];
    for (int i = threadIdx.x; i < n * dc; i += blockDim.x) {
        const uint32_t e = (uint32_t)(i / dc);
        if (WIDE) {
            cw[2 * i] = e;
            cw[2 * i + 1] = 0u;
        } else {
            cw[i] = e << 8;
        }
    }
    for (int i = threadIdx.x; i < n * tt * (WIDE ? 3 : 2); i += blockDim.x) tw[i] = 0u;
    __syncthreads();
    fill_rows(cw, tw, ext, wave, lane);
    __syncthreads();

    long long att = 0, kept_all = 0, passes_done = 0;
    int unconv = 0;
    const int r = I.r0 + wave;
    if (wave < I.nr && !I.rs[r].converged) {
        RepState* st = I.rs + r;
        uint8_t* base = state + (size_t)wave * rows_wave_bytes(n);
        RowsPolicy<WIDE, TRI> p;
        p.cw = cw;
        p.tw = tw;
        p.half = reinterpret_cast<int32_t*>(base);
        p.moves = reinterpret_cast<uint16_t*>(base + 4 * n64);
        p.sp = reinterpret_cast<int8_t*>(base + 6 * n64);
        p.dc_ = dc;
        p.tt_ = tt;
        p.lane = lane;
        p.qc = lane < dc ? lane : 0;
        // rows of at most 64 couplings and no hyper-couplings: the shorter
        // move loop, in which a locked spin's value is the step it moved at
        // (every half-gain lies above: the host checks)
        const bool pairs = !TRI && dc > 0 && dc <= 64;
        int8_t* gs = I.spins + I.stride * r;
        for (int i = lane; i < n; i += 64) p.sp[I.ext[i]] = gs[i];
        const long long E0 = st->E;  // the same in every lane: kept in scalar registers
        long long Estar = (long long)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(E0 >> 32)) << 32 |
                                      (uint32_t)__builtin_amdgcn_readfirstlane((int)E0));
        long long kept = 0;
        int passes = 0;
        bool conv = false, bad = false;
        for (int pass = 0; pass < max_passes; ++pass) {
            // half-gains from the definition, the fields scattered first;
            // every partial sum of a field is within the spin's sum of
            // |coefficients|
            for (int i = lane; i < n; i += 64) p.half[I.ext[i]] = field(i);
            fmcore::order();
            fmcore::Leaves<1> mx = INT32_MIN, ix = 0;
            for (int g = 0; g * 64 < n; ++g) {
                const int e = g * 64 + lane;
                int32_t v = INT32_MIN;
                if (e < n) {
                    int32_t f = p.half[e];
                    for (int q = 0; q < dc; ++q) {
                        int j;
                        int32_t J;
                        p.coupling(e, q, j, J);
                        f += J * p.sp[j];
                    }
                    if (TRI)
                        for (int q = 0; q < tt; ++q) {
                            int a, b;
                            int32_t K;
                            p.triple(e, q, a, b, K);
                            f += K * p.sp[a] * p.sp[b];
                        }
                    v = -p.sp[e] * f;
                }
                p.half[e] = v;
                const int32_t in[1] = {v};
                int32_t m[1];
                fmcore::wave_max<1>(in, m);
                const int a = g * 64 + fmcore::first_lane(v == m[0]);
                if (lane == g) {
                    mx[0] = m[0];
                    ix[0] = a;
                }
            }
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
            fmcore::order();
            if (pairs) {  // make the moves of the best prefix
                for (int e = lane; e < n; e += 64)
                    if ((uint32_t)p.half[e] - 0x80000000u < (uint32_t)len) p.sp[e] = (int8_t)-p.sp[e];
            } else {  // undo the moves after it
                for (int t = len + lane; t < n; t += 64) {
                    const int e = p.moves[t];
                    p.sp[e] = (int8_t)-p.sp[e];
                }
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
        } else {
            for (int i = lane; i < n; i += 64) gs[i] = p.sp[I.ext[i]];
            if (lane == 0) {
                st->E = Estar;
                st->sweeps += passes;
                st->flips += kept;
                if (conv) st->converged = 1;
            }
        }
        att = (long long)passes * n;
        kept_all = kept;
        passes_done = passes;
        unconv = (until_conv && !conv) ? 1 : 0;
    }
    // call totals: one set of atomics per workgroup
    __shared__ unsigned long long b_att, b_kept, b_passes;
    __shared__ int b_unconv;
    if (threadIdx.x == 0) {
        b_att = 0;
        b_kept = 0;
        b_passes = 0;
        b_unconv = 0;
    }
    __syncthreads();
    if (lane == 0 && (att || unconv)) {
        atomicAdd(&b_att, (unsigned long long)att);
        atomicAdd(&b_kept, (unsigned long long)kept_all);
        atomicMax(&b_passes, (unsigned long long)passes_done);
        atomicAdd(&b_unconv, unconv);
    }
    __syncthreads();
    if (threadIdx.x == 0 && (b_att || b_unconv)) {
        atomicAdd(&cs->attempts, b_att);
        atomicAdd(&cs->flips, b_kept);
        atomicMax(&cs->sweeps_max, b_passes);
        atomicAdd(&cs->unconverged, (unsigned long long)b_unconv);
    }
}

}  // namespace

// Packed form: workgroup k runs the restarts of item k (QueueItem: r holds the
// first restart and, above 16 bits, their number); the row widths are those
// of the instance table.
template <bool TRI>
__global__ __launch_bounds__(kRowsThreads) void k_fm_rows(const InstTab* __restrict__ tab,
                                                          const QueueItem* __restrict__ items,
                                                          RepState* __restrict__ rs, CallStats* __restrict__ cs,
                                                          uint32_t* __restrict__ err, int max_passes, int until_conv)
{
    const QueueItem it = items[blockIdx.x];
    const InstTab& Q = tab[it.inst];
    const InstDev D = Q.I;
    const int dc = Q.fml_dc, tt = Q.fml_tt;
    const RowsInst I{D.ext, Q.spins, Q.spin_stride, rs + Q.rep_base, D.n, it.r & 0xFFFF, it.r >> 16};
    auto fill = [&](uint32_t* cw, uint32_t* tw, const uint32_t* ext, int wave, int lane) {
        for (int s = wave; s < D.nslices; s += (int)(blockDim.x >> 6)) {
            const Slice S = D.slices[s];
            if (S.ew <= dc && (!TRI || S.tw <= tt)) {
                // every entry where it stands in the slice, on all lanes (a
                // complete graph has a row per slice)
                slice_entries(S.rows, S.ew, lane, [&](int l, int k) { return D.nbr[S.ebase + k * kSlice + l]; },
                              [&](int l, int k, uint32_t w) {
                                  if (w & 0xffu) cw[(size_t)ext[S.row0 + l] * dc + k] = ext[w >> 8] << 8 | (w & 0xffu);
                              });
                if (!TRI) continue;
                slice_entries(S.rows, S.tw, lane,
                              [&](int l, int k) {
                                  const uint32_t at = S.tbase + k * kSlice + l;
                                  return make_uint2(D.ta[at], D.tb[at]);
                              },
                              [&](int l, int k, uint2 w) {
                                  if (!(w.x & 0xffu)) return;
                                  uint32_t* t = tw + ((size_t)ext[S.row0 + l] * tt + k) * 2;
                                  t[0] = ext[w.x >> 8] << 8 | (w.x & 0xffu);
                                  t[1] = ext[w.y];
                              });
                continue;
            }
            // rows narrower than the slice, whose unused entries are left out
            if (lane >= S.rows) continue;
            const uint32_t e = ext[S.row0 + lane];
            uint32_t* c = cw + (size_t)e * dc;
            for (int k = 0; k < S.ew; ++k) {
                const uint32_t w = D.nbr[S.ebase + k * kSlice + lane];
                if (w & 0xffu) *c++ = ext[w >> 8] << 8 | (w & 0xffu);
            }
            if (!TRI) continue;
            uint32_t* t = tw + (size_t)e * tt * 2;
            for (int k = 0; k < S.tw; ++k) {
                const uint32_t w = D.ta[S.tbase + k * kSlice + lane], b = D.tb[S.tbase + k * kSlice + lane];
                if (!(w & 0xffu)) continue;
                *t++ = ext[w >> 8] << 8 | (w & 0xffu);
                *t++ = ext[b];
            }
        }
    };
    auto field = [&](int i) { return (int32_t)D.h[i]; };
    rows_body<false, TRI>(I, dc, tt, fill, field, cs, err, max_passes, until_conv);
}

// Wide form, one instance: workgroup k runs restarts [k W, k W + W) on its W
// wavefronts.
template <bool TRI>
__global__ __launch_bounds__(kRowsThreads) void k_fm_rows_wide(const WideDev D, int8_t* __restrict__ spins,
                                                               int64_t stride, RepState* __restrict__ rs, int R,
                                                               int dc, int tt, CallStats* __restrict__ cs,
                                                               uint32_t* __restrict__ err, int max_passes,
                                                               int until_conv)
{
    const int W = (int)(blockDim.x >> 6), r0 = (int)blockIdx.x * W;
    const RowsInst I{D.ext, spins, stride, rs, D.n, r0, min(W, R - r0)};
    auto fill = [&](uint32_t* cw, uint32_t* tw, const uint32_t* ext, int wave, int lane) {
        for (int s = wave; s < D.nslices; s += W) {
            // (the widths are those of the widest slice)
            const WSlice S = D.slices[s];
            slice_entries((int)S.rows, (int)S.ew, lane,
                          [&](int l, int k) {
                              const uint64_t at = S.ebase + (uint64_t)k * kSlice + l;
                              return make_uint2(D.nbr[at], (uint32_t)D.J[at]);
                          },
                          [&](int l, int k, uint2 w) {
                              if (!w.y) return;
                              uint32_t* c = cw + ((size_t)ext[S.row0 + l] * dc + k) * 2;
                              c[0] = ext[w.x];
                              c[1] = w.y;
                          });
            if (!TRI) continue;
            slice_entries((int)S.rows, (int)S.tw, lane,
                          [&](int l, int k) {
                              const uint64_t at = S.tbase + (uint64_t)k * kSlice + l;
                              return make_uint3(D.ta[at], D.tb[at], (uint32_t)D.K[at]);
                          },
                          [&](int l, int k, uint3 w) {
                              if (!w.z) return;
                              uint32_t* t = tw + ((size_t)ext[S.row0 + l] * tt + k) * 3;
                              t[0] = ext[w.x];
                              t[1] = ext[w.y];
                              t[2] = w.z;
                          });
        }
    };
    auto field = [&](int i) { return D.h[i]; };
    rows_body<true, TRI>(I, dc, tt, fill, field, cs, err, max_passes, until_conv);
}

size_t fm_rows_lds_bytes(int n, int dc, int tt, bool wide, int waves)
{
    return rows_stage_bytes(n, dc, tt, wide) + (size_t)waves * rows_wave_bytes(n);
}

static const void* rows_kernel(bool wide, bool tri)
{
    if (wide) return tri ? (const void*)k_fm_rows_wide<true> : (const void*)k_fm_rows_wide<false>;
    return tri ? (const void*)k_fm_rows<true> : (const void*)k_fm_rows<false>;
}

hipError_t launch_fm_rows(const InstTab* tab, const QueueItem* items, int nitems, int waves, size_t lds, bool tri,
                          RepState* rs, CallStats* cs, uint32_t* err, int max_passes, int until_conv, hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    if (waves < 1 || waves * 64 > kRowsThreads) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(rows_kernel(false, tri), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (tri)
        hipLaunchKernelGGL(k_fm_rows<true>, dim3(nitems), dim3(waves * 64), lds, st, tab, items, rs, cs, err,
                           max_passes, until_conv);
    else
        hipLaunchKernelGGL(k_fm_rows<false>, dim3(nitems), dim3(waves * 64), lds, st, tab, items, rs, cs, err,
                           max_passes, until_conv);
    return hipGetLastError();
}

hipError_t launch_fm_rows_wide(const WideDev& I, int8_t* spins, int64_t stride, RepState* rs, int R, int dc, int tt,
                               int waves, CallStats* cs, uint32_t* err, int max_passes, int until_conv, hipStream_t st)
{
    if (R <= 0) return hipSuccess;
    if (waves < 1 || waves * 64 > kRowsThreads || I.n < 1 || I.n > 4096) return hipErrorInvalidValue;
    const bool tri = I.has_tri != 0;
    const size_t lds = fm_rows_lds_bytes(I.n, dc, tt, true, waves);
    hipError_t e = hipFuncSetAttribute(rows_kernel(true, tri), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((R + waves - 1) / waves);
    if (tri)
        hipLaunchKernelGGL(k_fm_rows_wide<true>, dim3(blocks), dim3(waves * 64), lds, st, I, spins, stride, rs, R, dc,
                           tt, cs, err, max_passes, until_conv);
    else
        hipLaunchKernelGGL(k_fm_rows_wide<false>, dim3(blocks), dim3(waves * 64), lds, st, I, spins, stride, rs, R, dc,
                           tt, cs, err, max_passes, until_conv);
    return hipGetLastError();
}

}  // namespace sg
