// transport_kernel.h -- the persistent packet-queue transport kernel.
//
// One lane holds one photon packet in registers (the packet state is a
// structure of arrays across the 64 lanes of a wave).  Waves are persistent:
// each loops until the global work queue is drained, the analogue of the
// thread pool that keeps taking the next task index with an atomic increment
// (Section 5.2, Parallel class, Fig. 6).  Work is taken in chunks of packets
// with one atomic per wave; within a wave
//   * dead lanes are refilled from the wave's chunk, ranked by mbcnt over the
//     ballot of dead lanes (compaction of live packets);
//   * the lanes advance their ray marches together, a fixed number of cells
//     per iteration (the geometric steps first, then their density loads in
//     flight together), one kind of march at a time: the propagation loop
//     carries the deposits and nothing else; once at least `threshold` lanes
//     have finished their propagation (ballot), the finished lanes process
//     their events, and the short interaction searches and peel-offs that
//     these start run to their end in a loop of their own, before the wave
//     goes back to propagating.
// One kind of march per loop: a wave whose lanes mix kinds pays for every
// kind's instructions in each iteration, and the event code, which costs as
// much as several iterations, for each few lanes that finish.  With the kinds
// apart it pays to wait for all lanes (threshold 64) on Cartesian grids and
// for 48 on octrees, whose longest rays are further from the mean: 1.6e6
// packets in a depth-7 torus 22.4 -> 16.8 ms, with copies of the table (see
// transport_body) 1e6 in a 32^3 sphere in FP64 13.8 -> 7.2 ms (mixed kinds at 16
// lanes, against 48 and 64).  FP32 launches that add direct light to their images
// packet by packet keep the mixed loop (see launch_plan.h).
// The last packets are the longest: once the queue is empty a wave leaves the
// propagation loop only when all its lanes have finished, and a launch that
// cannot fill every wave spreads its packets over all of them, `lanes` to a
// wave, so that few lanes wait for each other.
// Per-wavelength optics and the instrument frames are staged in LDS.  The
// absorbed luminosity goes to the FP64 (wavelength, cell) table through
// hardware FP64 atomic adds, the GPU form of the lock-free addition of
// Section 5.2 (issued transposed through LDS, see DevSink); peel-offs go to
// the images through hardware float atomics.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>

#define MCRT_HD __device__ __forceinline__
#include "transport_core.h"
#include "internal.h"
#include "proposal.h"

namespace mcrt {

// One addition to an image element, or (DIRECT) to a sum of direct light
// (see View).
template <bool DIRECT, typename Real, typename ImgT, int G>
__device__ __forceinline__ void add_pixel(const View<Real, ImgT, G> &v, long long idx, double val)
{
    if constexpr (DIRECT) {
        if (v.direct != nullptr && idx >= v.direct0) {
            const long long at = (idx - v.direct0) * v.direct_shards + (blockIdx.x & (v.direct_shards - 1));
            unsafeAtomicAdd(v.direct + at * v.direct_stride, val);
            return;
        }
    }
    unsafeAtomicAdd(v.images + idx, (ImgT)val);
}

// TRK > 0 (FP32 kernels): deposits go through a per-wave LDS tile of TRK
// slots per lane and are issued transposed -- one atomic instruction carries
// the slots of 64/TRK rays, a ray's slots in consecutive lanes, so the cells
// of one ray that share a line of the table travel as one L2 request (the L2
// retires FP64 atomics per 64-byte line request: ~1.8e11/s for 8 lanes on one
// line against ~2.4e10/s for 64 scattered lanes).  The deposits of a ray's
// open run -- its latest cells that share one line -- are held back while
// the propagation march goes on, so a run that spans two march iterations
// still goes out as one request (at most TRK - K slots are held: K new
// deposits per iteration always fit; TRK == K holds nothing).  Without held
// runs (HOLD false) a tile of TRK >= 2 K slots lets the wave skip the flush
// of every other iteration (see must_flush).  A slot holds the table element
// (u32; in tables of 2^32 elements and more the cell) and the FP32 absorbed
// luminosity, which converts to FP64 exactly, side by side: one LDS access
// each way, and an issued atomic's address is one shift and add from it.
template <bool LEARN, bool HIST, int TRK = 0, int K = 0, bool HOLD = true, bool DIRECT = false> struct DevSink {
    static constexpr bool kLearn = LEARN, kHist = HIST, kDirect = DIRECT;
    static constexpr int kPitch = 64 + (TRK > 0 ? 64 / TRK : 0); // slot-major rows, padded
    static constexpr bool kHold = HOLD && TRK > K;
    static_assert(TRK == 0 || (64 % TRK == 0 && TRK <= 16 && TRK >= K), "slot tile");
    uint2 *slots = nullptr; // this lane's column of the wave's slot tile
    uint32_t slab = 0;      // first table element of the lane's wavelength (0 in wide tables)
    int np = 0;             // slots in use
    int base = 0;           // ring position of the first slot in use (kHold)
    int run = 0;            // first slot (from base) of the open run
    uint32_t rl = ~0u;      // table line of the open run
    template <typename Real, typename ImgT, int G>
    __device__ __forceinline__ void begin(const View<Real, ImgT, G> &v, uint32_t lam)
    {
        if constexpr (TRK > 0) slab = v.wide ? 0u : lam * (uint32_t)v.n_store;
    }
    template <typename Real, typename ImgT, int G>
    __device__ __forceinline__ void deposit(const View<Real, ImgT, G> &v, const Lane<Real> &ln, int cell, Real a)
    {
        if constexpr (TRK > 0) {
            if (a != Real(0)) {
                const uint32_t elem = slab + (uint32_t)cell;
                int slot = np;
                if constexpr (kHold) {
                    const uint32_t line = elem >> 3; // a wavelength's elements start on a line
                    if (line != rl) {
                        rl = line;
                        run = np;
                    }
                    slot = (base + np) & (TRK - 1);
                }
                slots[slot * kPitch] = make_uint2(elem, __float_as_uint(a));
                ++np;
            }
        } else {
            if (a != Real(0)) unsafeAtomicAdd(v.table + ((long long)ln.lam * v.n_store + cell), (double)a);
        }
    }
    // True when some lane of the wave could overflow its slots in the next
    // march iteration (K more deposits), so the wave must flush now.
    __device__ __forceinline__ bool must_flush() const { return __ballot(np > TRK - K) != 0; }
    // Issues the slots of closed runs; `hold` keeps the open run for the next
    // iteration (the lane's propagation march goes on).  Every lane posts one
    // word for its ray (wavelength, ring base, slots to issue), laid out so
    // that an issuing lane reads the words of all its rays with 128-bit loads;
    // the slots are read four rays at a time, so a flush waits on a few LDS
    // round trips.  table: the wave's table (uniform).  Whole wave active.
    __device__ __forceinline__ void flush(int lane, bool hold, int lam, double *table, long long n_store, int wide,
                                          const uint2 *tile, uint32_t *wave_word)
    {
        if constexpr (TRK > 0) {
            constexpr int R = 64 / TRK;
            int keep = 0;
            if constexpr (kHold) {
                keep = hold ? np - run : 0;
                keep = keep < TRK - K ? keep : TRK - K;
            }
            const int lim = np - keep;
            // lam < 2^20 (the medium's limit), base < 16, lim <= 16
            wave_word[(lane % R) * TRK + lane / R] = ((uint32_t)lam << 9) | ((uint32_t)base << 5) | (uint32_t)lim;
            wave_lds_sync();
            const int s = lane % TRK, q = lane / TRK;
            constexpr int GW = TRK < 4 ? TRK : 4; // rays per group
            const unsigned long long any = __ballot(lim > 0); // rays with slots to issue
#pragma unroll
            for (int g = 0; g < TRK / GW; ++g) {
                if ((any >> (R * GW * g)) == 0) break; // small launches use the first lanes only
                uint32_t w[GW];
                if constexpr (GW == 4) {
                    const uint4 x = reinterpret_cast<const uint4 *>(wave_word + q * TRK)[g];
                    w[0] = x.x;
                    w[1] = x.y;
                    w[2] = x.z;
                    w[3] = x.w;
                } else {
#pragma unroll
                    for (int i = 0; i < GW; ++i) w[i] = wave_word[q * TRK + GW * g + i];
                }
                uint2 x[GW];
#pragma unroll
                for (int i = 0; i < GW; ++i) {
                    const int slot = kHold ? (int)((((w[i] >> 5) & 15u) + (uint32_t)s) & (TRK - 1)) : s;
                    x[i] = tile[slot * kPitch + R * (GW * g + i) + q];
                }
#pragma unroll
                for (int i = 0; i < GW; ++i) {
                    if ((uint32_t)s < (w[i] & 31u)) {
                        double *p = table + (size_t)x[i].x;
                        if (wide) p += (long long)(w[i] >> 9) * n_store;
                        __builtin_amdgcn_global_atomic_fadd_f64((__attribute__((address_space(1))) double *)p,
                                                                (double)__uint_as_float(x[i].y));
                    }
                }
            }
            wave_lds_sync();
            if constexpr (kHold) {
                base = (base + lim) & (TRK - 1);
                run = 0;
            }
            np = keep;
        }
    }
    // Pixel adds are held in the lane (one pending add) and combined across
    // the wave at the next uniform point (flush_pixels); a second add before
    // that goes out directly.
    template <typename Real, typename ImgT, int G>
    __device__ __forceinline__ void pixel(const View<Real, ImgT, G> &v, Lane<Real> &ln, long long idx, ImgT val)
    {
        if (ln.pix >= 0) add_pixel<DIRECT>(v, ln.pix, (double)ln.pval);
        ln.pix = idx;
        ln.pval = (Real)val;
    }
};

// Second level of the pixel accumulation: one pixel per wave whose combined
// adds are summed in FP64 across flushes and added to the image once that
// pixel stops being the wave's combined pixel, and when the wave ends (or
// leaves the model's images).  The carry lives in a per-wave LDS slot (no
// registers held across the event loop): every lane reads it, lane 0 writes
// it; one wave's LDS operations complete in order.
struct PixelCarry {
    long long key; // image element, -1 when empty
    double val;
};

__device__ __forceinline__ void carry_init(PixelCarry *c, int lane)
{
    if (lane == 0) {
        c->key = -1;
        c->val = 0.0;
    }
}

template <bool DIRECT, typename Real, typename ImgT, int G>
__device__ __forceinline__ void flush_carry(const View<Real, ImgT, G> &v, PixelCarry *c, int lane)
{
    const long long key = c->key;
    const double val = c->val;
    if (key >= 0 && lane == 0) add_pixel<DIRECT>(v, key, val);
    carry_init(c, lane);
}

// Wave-level combine of the pending pixel adds: the lanes whose pixel equals
// the first pending lane's pixel are summed across the wave (a point
// source's emission peel-offs all land in one pixel per wavelength) and
// join the wave's carry; the other lanes add their own.  Whole wave active.
template <bool DIRECT, typename Real, typename ImgT, int G>
__device__ __forceinline__ void flush_pixels(const View<Real, ImgT, G> &v, Lane<Real> &ln, int lane, PixelCarry *c)
{
    const unsigned long long m = __ballot(ln.pix >= 0);
    if (m == 0) return;
    const int leader = __ffsll((long long)m) - 1;
    const long long key = __shfl(ln.pix, leader, 64);
    const bool same = ln.pix == key;
    ImgT s = same ? (ImgT)ln.pval : (ImgT)0;
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    const long long ckey = c->key;
    const double cval = c->val;
    if (ckey >= 0 && ckey != key && lane == leader) add_pixel<DIRECT>(v, ckey, cval);
    if (lane == leader) {
        c->key = key;
        c->val = (ckey == key ? cval : 0.0) + (double)s;
    }
    if (ln.pix >= 0 && !same) add_pixel<DIRECT>(v, ln.pix, (double)ln.pval);
    ln.pix = -1;
}

__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ double wave_sum(double x)
{
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x)
{
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

// Lane `src`'s value, in scalar registers.
__device__ __forceinline__ int lane_value(int x, int src) { return __builtin_amdgcn_readlane(x, src); }
__device__ __forceinline__ float lane_value(float x, int src)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), src));
}
__device__ __forceinline__ double lane_value(double x, int src)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), src),
                            __builtin_amdgcn_readlane(__double2loint(x), src));
}

// x to lane `to` (each lane that matters to another one).
__device__ __forceinline__ int push_value(int x, int to) { return __builtin_amdgcn_ds_permute(to << 2, x); }
__device__ __forceinline__ float push_value(float x, int to)
{
    return __int_as_float(__builtin_amdgcn_ds_permute(to << 2, __float_as_int(x)));
}
__device__ __forceinline__ double push_value(double x, int to)
{
    return __hiloint2double(__builtin_amdgcn_ds_permute(to << 2, __double2hiint(x)),
                            __builtin_amdgcn_ds_permute(to << 2, __double2loint(x)));
}

// Lane 0's march on a Cartesian grid, to its end, by the whole wave, for
// launches of one packet to a wave: an iteration of the march loops costs as much
// for one lane as for 64 (about 130 vector instructions per cell, of which a wave
// alone on its SIMD issues one in four cycles).  The wave takes 21 to 61 cells
// at a time instead:
//   * lane 21 a + m takes crossing m of axis a (the ray parameter of a plane
//     follows from the plane's number alone) and finds its rank among all
//     three axes' crossings: an estimate from the position, made exact by
//     comparing the planes next to it, ties in axis order as geo_step takes
//     them;
//   * the crossings move to the lanes of their ranks, which load their cells'
//     densities together and take their optical depths and exponentials;
//   * what is a chain -- the running luminosity, the running optical depth -- is
//     multiplied or summed through lane by lane, in the order of the cells.
// Every value is computed by the operations of march_batch, so deposits,
// interaction points and depths are bit for bit the same.  Kernel of 500 packets
// in a 32^3 sphere 285 -> 222 us, of 220 on a 61 x 45 x 27 disk 830 -> 620 us (what
// remains is the events, about 2500 vector instructions each); with more than one
// packet to a wave, marched one after another, nothing is gained (4000 in the
// sphere, two to a wave: 316 and 327 us), and 1e5 there lose 5 % to the registers.
// Nor on grids of a few cells (see launch_plan.h).
// PROP: a propagation, else a search or a peel-off.  Whole wave active.
// A march that cannot go on this way (no finite crossing) stays with lane 0.
template <bool PROP, typename Real, typename ImgT, int G>
__device__ __forceinline__ void lone_march(const View<Real, ImgT, G> &v, Lane<Real> &ln, Tally &ty, int lane)
{
    constexpr int src = 0;
    if (!__builtin_amdgcn_readfirstlane(ln.marching ? 1 : 0)) return;
    constexpr int M = 21; // crossings per axis
    Real r[3], d[3], id[3];
    int c[3], u[3], s[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        r[b] = lane_value(ln.r[b], src);
        d[b] = lane_value(ln.d[b], src);
        id[b] = lane_value(ln.id3[b], src);
        c[b] = lane_value(cidx(ln, b), src);
        u[b] = d[b] > Real(0) ? 1 : 0;
        s[b] = 2 * u[b] - 1;
    }
    Real t = lane_value(ln.t, src);
    const Real kappa = lane_value(ln.opt.kappa, src), wabs = lane_value(ln.wabs, src);
    const bool loc = !PROP && lane_value(ln.mode, src) == kLocate;
    const Real limit = loc ? lane_value(ln.tau_int, src) : v.tau_peel_max;
    Real E = lane_value(ln.E, src), tau = lane_value(ln.tau, src);
    const long long slab = (long long)lane_value((int)ln.lam, src) * v.n_store;
    const int ax = lane >= 2 * M ? 2 : (lane >= M ? 1 : 0), m = lane - M * ax;
    auto crossing = [&](int b, int k) -> Real { // of plane k along the ray on axis b
        const Real x = Prec<Real>::over_k(v.lo[b] + (Real)(c[b] + u[b] + s[b] * k) * v.cs[b] - r[b], d[b], id[b]);
        return d[b] != Real(0) ? x : Prec<Real>::inf();
    };
    bool done = false;
    while (!done) {
        Real T = crossing(0, m);
        T = ax == 1 ? crossing(1, m) : T;
        T = ax == 2 ? crossing(2, m) : T;
        bool valid = m < M && T < Prec<Real>::inf();
        int n[3]; // crossings of each axis before this one
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            auto before = [&](int k) {
                const Real x = crossing(b, k);
                return x < T || (x == T && b < ax);
            };
            int k = s[b] * ((int)((r[b] + T * d[b] - v.lo[b]) * v.ics[b]) - c[b]);
            k = k < 0 ? 0 : (k > M ? M : k);
            const bool look = valid && ax != b && d[b] != Real(0);
            while (look && k > 0 && !before(k - 1)) --k;
            while (look && k < M && before(k)) ++k;
            n[b] = ax == b ? m : (look ? k : 0);
            valid = valid && n[b] < M;
        }
        const unsigned long long all = __ballot(valid);
        int count = __popcll(all);
        if (count == 0) break;
        const int rank = valid ? n[0] + n[1] + n[2] : 63; // ranks stay below 61
        const int x0 = c[0] + s[0] * n[0], x1 = c[1] + s[1] * n[1], x2 = c[2] + s[2] * n[2];
        const int next = ax == 0 ? x0 + s[0] : (ax == 1 ? x1 + s[1] : x2 + s[2]);
        const int size = ax == 0 ? v.n[0] : (ax == 1 ? v.n[1] : v.n[2]);
        const int to = push_value(store_index(v, x0, x1, x2) | ((unsigned)next >= (unsigned)size ? INT_MIN : 0), rank);
        const Real te = rmax(push_value(T, rank), t);
        Real ts = __shfl_up(te, 1, 64);
        ts = lane == 0 ? t : ts;
        const unsigned long long ex = __ballot(lane < count && to < 0);
        done = ex != 0;
        t = lane_value(te, count - 1);
        count = done ? __ffsll((long long)ex) : count;
        bool ok = lane < count;
        const Real ds = ok ? te - ts : Real(0);
        const float rho = gload(v.density, ok ? to & 0x7fffffff : 0);
        const Real kr = ok ? kappa * (Real)rho : Real(0);
        const Real dtau = ok ? kr * ds : Real(0);
        if constexpr (PROP) {
            const Real x = -Math<Real>::e_expm1(-fabs(dtau));
            const Real f = Real(1) - x; // 1 where not ok
            Real El = E;
            for (int k = 0; k < count; k += 8) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    El = lane == k + i ? E : El;
                    E = E * lane_value(f, k + i);
                }
            }
            const Real A = ok ? wabs * El * x : Real(0);
            if (A != Real(0))
                __builtin_amdgcn_global_atomic_fadd_f64(
                    (__attribute__((address_space(1))) double *)(v.table + (slab + (to & 0x7fffffff))), (double)A);
            ty.absorbed += (double)A;
            ty.prop_cells += ok ? 1u : 0u;
            const unsigned long long some = __ballot(dtau > Real(0));
            if (some) tau = rmax(lane_value(dtau, __ffsll((long long)some) - 1), tau); // asked only whether it is 0
        } else {
            Real tl = tau;
            int k = 0;
            for (; k < count; k += 8) {
                if (k > 0 && __builtin_amdgcn_readfirstlane(tau >= limit ? 1 : 0)) break; // the cells after a hit do not matter
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    tl = lane == k + i ? tau : tl;
                    tau = Prec<Real>::mac(lane_value(ds, k + i), lane_value(kr, k + i), tau);
                }
            }
            count = k < count ? k : count;
            const Real ta = Prec<Real>::mac(ds, kr, tl);
            const unsigned long long hits = __ballot(lane < count && ta >= limit);
            if (hits) count = __ffsll((long long)hits);
            tau = lane_value(ta, count - 1);
            ok = lane < count;
            const unsigned long long deep = __ballot(ok && dtau > Real(0));
            if (loc && deep) { // last segment with positive depth
                const int l = 63 - __clzll((long long)deep);
                const Real a0 = lane_value(ts, l), a1 = lane_value(tl, l), a2 = lane_value(kr, l),
                           a3 = lane_value(ds, l), a4 = (Real)lane_value(rho, l);
                if (lane == src) {
                    ln.a_t0 = a0;
                    ln.a_tau = a1;
                    ln.a_kr = a2;
                    ln.a_ds = a3;
                    ln.rho_star = a4;
                }
            }
            ty.locate_cells += ok && loc ? 1u : 0u;
            ty.peel_cells += ok && !loc ? 1u : 0u;
            if (hits) {
                done = true;
                if (lane == src) {
                    ln.found = ln.found || loc;
                    ln.dropped = ln.dropped || !loc;
                }
            }
        }
#pragma unroll
        for (int b = 0; b < 3; ++b) c[b] += s[b] * (int)__popcll(all >> (M * b) & ((1ull << M) - 1));
    }
    if (lane == src) {
        ln.E = E;
        ln.tau = tau;
        ln.t = t;
        ln.c0 = c[0];
        ln.c1 = c[1];
        ln.c2 = c[2];
        ln.marching = !done;
        if (!done) {
            ln.tn0 = next_plane_t(v, ln, 0);
            ln.tn1 = next_plane_t(v, ln, 1);
            ln.tn2 = next_plane_t(v, ln, 2);
        }
    }
}

// Adds the wave's tally to a shard of the result's (see kTallyShards) and
// clears it: the words side by side in lanes, so that all energy sums and all
// counters are one request each.  Whole wave active.
__device__ __forceinline__ void add_tally(Tally &ty, unsigned long long *tally, int lane)
{
    const double e0 = wave_sum(ty.emitted), e1 = wave_sum(ty.absorbed);
    const double e2 = wave_sum(ty.escaped), e3 = wave_sum(ty.truncated);
    const uint32_t s[kNumStats] = {ty.packets, ty.events, ty.prop_cells, ty.locate_cells, ty.peel_cells,
                                   ty.peel_adds, ty.peel_dropped, ty.capped, ty.guard, ty.nonfinite};
    unsigned long long n = 0;
#pragma unroll
    for (int i = 0; i < kNumStats; ++i) {
        const unsigned long long x = wave_sum_u64(s[i]);
        n = lane == 4 + i ? x : n;
    }
    const double e = lane == 0 ? e0 : (lane == 1 ? e1 : (lane == 2 ? e2 : e3));
    unsigned long long *p = tally + (size_t)(blockIdx.x % kTallyShards) * kTallyWords + lane;
    if (lane < 4) unsafeAtomicAdd((double *)p, e);
    else if (n) atomicAdd(p, n);
    ty = Tally{};
}

// Learned proposal, FP32: the lanes waiting for a direction are ranked
// (mbcnt over the ballot) and evaluated 16 at a time on the matrix cores;
// their features go through a per-wave LDS tile into the B operand, the 40
// outputs per sample come back through a second tile.  Must be called with
// the whole wave active.
template <typename ImgT, int G>
__device__ __forceinline__ void resolve_wave(const View<float, ImgT, G> &v, Lane<float> &ln, Tally &ty,
                                             const bf16x4 *Wf, const float *bias, uint16_t *feat, float *stage,
                                             int lane)
{
    const unsigned long long need = __ballot(ln.parked);
    const int n = __popcll(need);
    const bool mine = ln.parked;
    const int rank = (int)lanes_below(need);
    float f[9];
    if (mine) event_features(v, ln, !ln.emis_dir, f);
    for (int sb = 0; 16 * sb < n; ++sb) {
        const bool in_block = mine && (rank >> 4) == sb;
        if (in_block) {
            uint16_t *row = feat + 16 * (rank & 15);
#pragma unroll
            for (int i = 0; i < 16; ++i) row[i] = i < 9 ? bf16_bits(f[i]) : (uint16_t)0;
        }
        wave_lds_sync();
        bf16x4 x = *reinterpret_cast<const bf16x4 *>(feat + 16 * (lane & 15) + 4 * (lane >> 4));
        f32x4 o[3];
        mlp_forward16<false>(Wf, bias, x, lane, o);
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                int row = 16 * t + 4 * (lane >> 4) + i;
                if (row < 40) stage[(lane & 15) * 41 + row] = o[t][i];
            }
        wave_lds_sync();
        if (in_block) apply_proposal<DevSink<true, false>>(v, ln, ty, stage + (rank & 15) * 41);
        wave_lds_sync();
    }
}

// LEARN: learned proposal; HIST: plain run recording histories.  A variant
// carries only the code (and registers) of its own features.
template <typename Real, typename ImgT, int G, bool LEARN, bool HIST, bool MIX, bool LONE>
__device__ __forceinline__ void transport_body()
{
    // The kernel's only argument, read where it is used: through a pointer
    // whose origin is hidden at every call, so that the compiler loads the
    // fields a phase needs with scalar loads instead of holding all of them
    // (more than the scalar registers) across the event loop, spilled to
    // vector registers and read back lane by lane (with slots of one LDS access
    // and one-instruction atomic addresses, the propagation loop of 8 cells
    // went from about 1400 to 970 VALU instructions: learned depth-7 torus 8.7 ->
    // 8.1 ms, depth-9 torus -2 %, 1e5 packets in a 32^3 sphere -3 %).
    typedef TransportArgs<Real, ImgT, G> Args;
    auto A = []() -> const Args & {
        auto p = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return *(const Args *)p;
    };
    __shared__ Optics<Real> s_opt[kMaxLdsLambda];
    __shared__ InsDesc<Real> s_ins[kMaxIns];
    const Args &a = A();
    // Copies, for the memory side adds to one line at a time: of the table
    // for point sources (every packet crosses the few cells around the
    // source), of small images for extended ones (all packets share the
    // pixels).  Workgroups are placed round-robin over the XCDs, so eight
    // copies give each XCD its own.  1.6e6 packets in a depth-7 torus, 8
    // wavelengths: 17.3 ms with one table, 12.8 with eight; disks gain nothing
    // from copies of their tables.
    // 2.2e6 packets of a 61 x 45 x 27 disk, 11 wavelengths, three 33^2 images:
    // 18.5 ms in chunks of 64 with one set of images, 8.6 with eight.
    double *table = a.view.table;
    ImgT *images = a.view.images;
    if (const int c = blockIdx.x & (a.table_copies - 1))
        table = a.more_tables + (c - 1) * a.view.n_store * a.view.n_lambda;
    if (const int c = blockIdx.x & (a.image_copies - 1)) images = a.more_images + (c - 1) * a.image_elems;
    const Optics<Real> *optics = a.optics;
    if (a.view.n_lambda <= kMaxLdsLambda) {
        for (int i = threadIdx.x; i < a.view.n_lambda; i += blockDim.x) s_opt[i] = optics[i];
        optics = s_opt;
    }
    for (int i = threadIdx.x; i < a.view.n_ins; i += blockDim.x) s_ins[i] = a.ins[i];
    auto view = [&]() {
        View<Real, ImgT, G> v = A().view;
        v.table = table;
        v.images = images;
        v.optics = optics;
        v.ins = s_ins;
        return v;
    };
    // learned proposal (FP32): network fragments and biases in LDS, plus a
    // feature tile [16][16] bf16 and an output tile [16][41] FP32 per wave
    constexpr bool kMfma = LEARN && sizeof(Real) == 4;
    __shared__ bf16x4 s_wf[kMfma ? kFragFwd * 64 : 1];
    __shared__ float s_bias[kMfma ? kBiasFloats : 1];
    __shared__ __attribute__((aligned(16))) uint16_t s_feat[kMfma ? (kBlock / 64) * 256 : 1];
    __shared__ float s_stage[kMfma ? (kBlock / 64) * 16 * 41 : 1];
    if constexpr (kMfma) {
        const bf16x4 *wf = reinterpret_cast<const bf16x4 *>(a.mlp_frags);
        for (int i = threadIdx.x; i < kFragFwd * 64; i += blockDim.x) s_wf[i] = wf[i];
        for (int i = threadIdx.x; i < kBiasFloats; i += blockDim.x) s_bias[i] = a.mlp_bias[i];
    }
    __syncthreads();

    // Segments per march iteration: FP32 8 (4 with the learned proposal,
    // whose network needs the registers), FP64 as the host simulator.  FP32 deposits are issued transposed through LDS:
    // Cartesian runs hold their open run (16 slots per lane); octree runs and
    // the learned proposal (registers, LDS) take one slot per segment -- on
    // the octree's smaller tables the extra issue costs more than the held
    // runs save.
    //
    // A flush's atomics stay in the wave's count of outstanding vector memory
    // operations, which retire in order: the next load the wave waits for
    // (on the octree, the first walk load of the next iteration) also waits
    // until every atomic of the flush has been acknowledged by the memory
    // side.  Octree runs therefore hold no runs but take 2 kK slots, and the
    // wave flushes only when a lane could overflow in the next iteration or
    // when it leaves the march loop: every other iteration.
    constexpr int kK = sizeof(Real) != 4 ? BatchOf<G>::value
                                         : (G == kCartesian ? (LEARN ? 4 : 8) : (LEARN ? 4 : 8));
    constexpr bool kLazy = sizeof(Real) == 4 && G == kOctree;
    constexpr int kTR = sizeof(Real) == 4 ? (kLazy ? 2 * kK : (G == kCartesian && !LEARN ? 16 : kK)) : 0;
    typedef DevSink<LEARN, HIST, kTR, kK, !kLazy, sizeof(ImgT) == 4 && !MIX> SinkT;
    constexpr int kTile = kTR ? kTR * SinkT::kPitch : 1;
    __shared__ uint2 s_tile[kTR ? (kBlock / 64) * kTile : 1];
    __shared__ __attribute__((aligned(16))) uint32_t s_word[kTR ? kBlock : 4];
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
    SinkT sink;
    if constexpr (kTR > 0) {
        sink.slots = s_tile + wave * kTile + lane;
    }
    Lane<Real> ln;
    ln.mode = kDead;
    ln.marching = false;
    ln.parked = false;
    ln.pix = -1;
    Tally ty = {};
    __shared__ PixelCarry s_carry[kBlock / 64];
    PixelCarry *carry = s_carry + wave;
    carry_init(carry, lane);
    uint64_t cur = 0, end = 0; // the wave's chunk: ids [cur, end) of wavelength lam
    int lam = 0;
    bool exhausted = false, took = false;
    const bool slot = lane < a.lanes;

    for (;;) {
        // refill dead lanes from the wave's chunk (one atomic per chunk); a
        // refilled lane only launches here, its events run below
        bool launched = false;
        for (;;) {
            const bool free = slot && ln.mode == kDead && !ln.parked && !launched;
            unsigned long long dead = __ballot(free);
            if (dead == 0 || exhausted) break;
            if (cur >= end) {
                const Args &a = A();
                unsigned long long c = (uint64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x;
                if (a.own_chunks) {
                    if (took) c = a.n_chunks;
                } else {
                    if (lane == 0) c = atomicAdd(a.counter, 1ull);
                    c = __shfl(c, 0, 64);
                }
                took = true;
                if (c >= a.n_chunks) {
                    exhausted = true;
                    break;
                }
                lam = __builtin_amdgcn_readfirstlane((int)(c / a.lam_chunks));
                cur = c % a.lam_chunks * a.chunk;
                end = cur + a.chunk < a.count ? cur + a.chunk : a.count;
                continue;
            }
            const uint64_t avail = end - cur;
            const uint32_t rank = lanes_below(dead);
            if (free && (uint64_t)rank < avail) {
                const uint64_t i = cur + rank;
                const auto v = view();
                const Args &a = A();
                launch<decltype(sink)>(v, ln, ty, (uint32_t)lam, (uint32_t)(a.first_id + i),
                                       (uint32_t)(lam * a.count + i));
                sink.begin(v, (uint32_t)lam);
                launched = true;
            }
            const uint64_t ndead = (uint64_t)__popcll(dead);
            cur += ndead < avail ? ndead : avail;
        }
        // events, and the interaction searches and peel-offs they start, until
        // every live lane has a propagation to march; with the learned
        // proposal, the lanes parked for a direction get it here
        for (;;) {
            const auto v = view();
            if (!ln.marching && ln.mode != kDead) settle(v, ln, ty, sink);
            flush_pixels<SinkT::kDirect>(v, ln, lane, carry);
            bool again = false;
            if constexpr (LEARN) {
                if (__ballot(ln.parked) != 0) {
                    again = true;
                    if constexpr (kMfma)
                        resolve_wave(v, ln, ty, s_wf, s_bias, s_feat + wave * 256, s_stage + wave * 16 * 41, lane);
                    else if (ln.parked)
                        resolve_direction_scalar<decltype(sink)>(v, ln, ty);
                }
            }
            if constexpr (!MIX) {
                while (__ballot(ln.marching && ln.mode != kProp) != 0) {
                    again = true;
                    if constexpr (LONE) lone_march<false>(v, ln, ty, lane);
                    if (ln.marching && ln.mode != kProp) march_batch<kScans, kK>(v, ln, ty, sink);
                }
            }
            if (!again) break;
        }
        if (__ballot(ln.mode != kDead) == 0) {
            if (exhausted) break;
            continue;
        }

        // propagation: every marching lane advances kK cells per iteration;
        // the iteration's deposits go out after it
        const auto v = view();
        const int threshold = A().threshold;
        for (;;) {
            if constexpr (LONE) lone_march<true>(v, ln, ty, lane);
            if (ln.marching) march_batch<MIX ? kMixed : kProps, kK>(v, ln, ty, sink);
            unsigned long long waiting = __ballot(!ln.marching && (ln.mode != kDead || (slot && !exhausted)));
            unsigned long long active = __ballot(ln.marching);
            const bool leave = active == 0 || ((MIX || !exhausted) && __popcll(waiting) >= threshold);
            // a lane's wavelength changes only after the loop: the slots may
            // wait across iterations, never across a relaunch
            if (!kLazy || leave || sink.must_flush())
                sink.flush(lane, ln.marching && ln.mode == kProp, (int)ln.lam, v.table, v.n_store, v.wide,
                           s_tile + wave * kTile, s_word + wave * 64);
            if (leave) break;
        }
    }

    flush_carry<SinkT::kDirect>(view(), carry, lane);
    add_tally(ty, A().tally, lane);
}

// FP32 production kernels: at most 168 VGPRs, three waves per SIMD; the
// plain octree kernel, bound by the latency of its walk's dependent loads,
// four waves per SIMD (128 VGPRs, a few registers spilled).
template <int G, bool LEARN, bool HIST, bool MIX, bool LONE = false>
__global__ void __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(G == kOctree && !LEARN && !HIST ? 4 : (LONE ? 2 : 3))))
transport_kernel_f32(TransportArgs<float, float, G>)
{
    transport_body<float, float, G, LEARN, HIST, MIX, LONE>();
}

// FP64 validation kernels (the scalar FP64 network needs more registers).
template <int G, bool LEARN, bool HIST, bool LONE = false>
__global__ void __launch_bounds__(kBlock) transport_kernel_f64(TransportArgs<double, double, G>)
{
    transport_body<double, double, G, LEARN, HIST, false, LONE>();
}

// Batched launch over many Cartesian models (the many-small-models use case
// of Section 3.1 run as one persistent launch).  The queue is a list of chunks
// that never straddle models; a wave works on one model at a time, so the
// model's parameters are wave-uniform, and drains its lanes before it
// switches to a chunk of another model (tallies are flushed at the switch).
// The model index is the fourth word of every packet's Philox counter.
//
// DRAIN: a batch of few chunks is bound by its longest ones (48 models of
// 942 000 packets: vector units busy 22 % of the time, one wave to a SIMD on
// average).  Its waves take 256 registers, so that nothing is spilled on the
// way, and once nothing more is launched into a wave it goes over to one kind of
// march per loop (see above).  Before that, and in batches that fill the chip, a
// wave mixes the kinds: its launches then keep the sizes, and the images the
// rounding, that they always had, and at four waves per SIMD it is faster
// (942 000 packets of 48 models 34.6 -> 29.7 ms; 16.5e6 of 64 models 385 mixed,
// 395 to 420 so).  Models of at most 3072 packets per wavelength, whose images
// differ by less than 1e-5 between any two orders of their additions, march apart
// from the start, in chunks that spread the batch over the chip, as far as waves
// take them in turn (126 000 packets of 48 models 20.4 -> 12.8 ms).  These chunks,
// 64 packets at most, pay as well where the batch has too many for this kernel
// (256 models of 3000 packets 19.0 -> 11.0 ms, 1000 of them 37.4 -> 31.0).
template <typename Real, typename ImgT, int SLOTS, bool DRAIN>
__device__ __forceinline__ void batch_body(const BatchArgs<Real, ImgT> &a,
                                           const ModelDesc<Real, ImgT> *__restrict__ models)
{
    // one deposit slot per segment (the batch's small tables stay in the L2,
    // where holding runs does not pay for its extra issue).  SLOTS (FP32) is
    // the tile per lane, a tuning choice: kK slots, issued after every march
    // iteration, or 2 kK, issued only when a lane could overflow or the wave
    // leaves the march loop (as in the octree kernels: a flush's atomics
    // delay the next loads the wave waits for)
    constexpr int kK = sizeof(Real) == 4 ? 8 : BatchOf<0>::value;
    constexpr int kTR = sizeof(Real) == 4 ? SLOTS : 0;
    static_assert(sizeof(Real) != 4 || SLOTS == kK || SLOTS == 2 * kK, "deposit tile");
    constexpr bool kLazyB = kTR == 2 * kK;
    typedef DevSink<false, false, kTR, kK, false> SinkT;
    constexpr int kTile = kTR ? kTR * SinkT::kPitch : 1;
    __shared__ uint2 s_tile[kTR ? (kBlock / 64) * kTile : 1];
    __shared__ __attribute__((aligned(16))) uint32_t s_word[kTR ? kBlock : 4];
    const int wave = threadIdx.x >> 6;
    const int lane = __lane_id();
    SinkT sink;
    if constexpr (kTR > 0) {
        sink.slots = s_tile + wave * kTile + lane;
    }
    Lane<Real> ln;
    ln.mode = kDead;
    ln.marching = false;
    ln.pix = -1;
    Tally ty = {};
    __shared__ PixelCarry s_carry[kBlock / 64];
    PixelCarry *carry = s_carry + wave;
    carry_init(carry, lane);
    int cur_model = -1, pend_model = -1;
    // The current model's view is read through a constant-address-space
    // pointer formed from a wave-uniform model index at every use: its fields
    // become scalar loads the compiler may repeat instead of holding ~60
    // values in registers across the event loop (a pointer carried across
    // the queue loop is not provably uniform, and its loads go to the vector
    // memory path).
    auto V = [&]() -> const View<Real, ImgT, 0> & {
        const int m = __builtin_amdgcn_readfirstlane(cur_model < 0 ? 0 : cur_model);
        return models[m].view;
    };
    uint64_t count = 1, first_id = 0;
    uint64_t cur = 0, end = 0, pend_cur = 0, pend_end = 0;
    bool exhausted = false, apart = false;

    for (;;) {
        bool launched = false;
        for (;;) {
            unsigned long long dead = __ballot(ln.mode == kDead && !launched);
            if (dead == 0 || exhausted) break;
            if (cur >= end) {
                if (pend_model < 0) {
                    unsigned long long c = 0;
                    if (lane == 0) c = atomicAdd(a.counter, 1ull);
                    c = __shfl(c, 0, 64);
                    if (c >= a.total_chunks) {
                        exhausted = true;
                        break;
                    }
                    int lo = 0, hi = a.n_models - 1; // last model with chunk0 <= c
                    while (lo < hi) {
                        int mid = (lo + hi + 1) >> 1;
                        if (a.models[mid].chunk0 <= c) lo = mid;
                        else hi = mid - 1;
                    }
                    pend_model = __builtin_amdgcn_readfirstlane(lo);
                    const ModelDesc<Real, ImgT> &m = a.models[pend_model];
                    pend_cur = (c - m.chunk0) * m.chunk;
                    pend_end = pend_cur + m.chunk < m.total ? pend_cur + m.chunk : m.total;
                }
                if (pend_model != cur_model) {
                    if (__ballot(ln.mode != kDead) != 0) break; // drain before switching
                    if (cur_model >= 0) {
                        flush_carry<false>(V(), carry, lane);
                        add_tally(ty, a.models[cur_model].tally, lane);
                    }
                    cur_model = pend_model;
                    const ModelDesc<Real, ImgT> &m = a.models[cur_model];
                    count = m.count;
                    first_id = m.first_id;
                    if constexpr (DRAIN) apart = __builtin_amdgcn_readfirstlane(m.apart) != 0;
                }
                cur = pend_cur;
                end = pend_end;
                pend_model = -1;
                continue;
            }
            uint64_t avail = end - cur;
            uint32_t rank = lanes_below(dead);
            if (ln.mode == kDead && !launched && (uint64_t)rank < avail) {
                uint64_t P = cur + rank;
                launch<decltype(sink)>(V(), ln, ty, (uint32_t)(P / count), (uint32_t)(first_id + P % count), (uint32_t)P);
                sink.begin(V(), ln.lam);
                launched = true;
            }
            uint64_t ndead = (uint64_t)__popcll(dead);
            cur += ndead < avail ? ndead : avail;
        }
        bool drain = false;
        if (!ln.marching && ln.mode != kDead) settle(V(), ln, ty, sink);
        flush_pixels<false>(V(), ln, lane, carry);
        if constexpr (DRAIN) {
            drain = apart || (cur >= end && (exhausted || pend_model >= 0));
            while (drain && __ballot(ln.marching && ln.mode != kProp) != 0) {
                do {
                    if (ln.marching && ln.mode != kProp) march_batch<kScans, kK>(V(), ln, ty, sink);
                } while (__ballot(ln.marching && ln.mode != kProp) != 0);
                if (!ln.marching && ln.mode != kDead) settle(V(), ln, ty, sink);
                flush_pixels<false>(V(), ln, lane, carry);
            }
        }
        if (__ballot(ln.mode != kDead) == 0) {
            if (exhausted) break;
            continue;
        }
        for (;;) {
            if constexpr (DRAIN) {
                if (drain) {
                    if (ln.marching) march_batch<kProps, kK>(V(), ln, ty, sink);
                } else {
                    if (ln.marching) march_batch<kMixed, kK>(V(), ln, ty, sink);
                }
            } else {
                if (ln.marching) march_batch<kMixed, kK>(V(), ln, ty, sink);
            }
            unsigned long long waiting = __ballot(!ln.marching && (ln.mode != kDead || !exhausted));
            unsigned long long active = __ballot(ln.marching);
            const bool leave = active == 0 || ((!DRAIN || !drain) && __popcll(waiting) >= a.threshold);
            if (!kLazyB || leave || sink.must_flush())
                sink.flush(lane, ln.marching && ln.mode == kProp, (int)ln.lam, V().table, V().n_store, V().wide,
                           s_tile + wave * kTile, s_word + wave * 64);
            if (leave) break;
        }
    }
    if (cur_model >= 0) {
        flush_carry<false>(V(), carry, lane);
        add_tally(ty, a.models[cur_model].tally, lane);
    }
}

// FP32: four waves per SIMD (128 VGPRs, a few registers spilled): the
// event-heavy batch gains more from the extra wave than the spills cost; two
// where the waves are few (see DRAIN).
template <typename ImgT, int SLOTS, bool DRAIN>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(DRAIN ? 2 : 4)))
batch_transport_kernel_f32(BatchArgs<float, ImgT> a, const ModelDesc<float, ImgT> *__restrict__ models)
{
    batch_body<float, ImgT, SLOTS, DRAIN>(a, models);
}

template <typename ImgT>
__global__ void __launch_bounds__(kBlock) batch_transport_kernel_f64(BatchArgs<double, ImgT> a, const ModelDesc<double, ImgT> *__restrict__ models)
{
    batch_body<double, ImgT, 0, false>(a, models);
}

// After an FP32 launch: its sums of direct light join their pixels and are
// cleared for the next launch.  A wave's share is a tree of FP32 additions over
// its lanes (six roundings at most), the pixel one more, where thousands of FP32
// additions of equal size to one pixel all round the same way (32^3 sphere: up
// to 2.5e-5 of the pixel in launches of 6e4 packets, 1e-3 in 2e5).
template <typename ImgT> __global__ void __launch_bounds__(64) direct_kernel(View<float, ImgT, 0> v)
{
    const int slots = v.n_ins * v.n_lambda;
    for (int s = blockIdx.x * 64 + threadIdx.x; s < slots; s += gridDim.x * 64) {
        double sum = 0.0;
        for (int k = 0; k < v.direct_shards; ++k) {
            double *p = v.direct + ((long long)s * v.direct_shards + k) * v.direct_stride;
            sum += *p;
            *p = 0.0;
        }
        if (sum != 0.0) v.images[v.direct_pix[s]] += (ImgT)sum;
    }
}

template <typename Real, typename ImgT, int SLOTS, bool DRAIN>
hipError_t launch_batch_impl(const BatchArgs<Real, ImgT> &a, int grid, hipStream_t stream)
{
    if constexpr (sizeof(Real) == 4)
        hipLaunchKernelGGL((batch_transport_kernel_f32<ImgT, SLOTS, DRAIN>), dim3(grid), dim3(kBlock), 0, stream, a,
                           a.models);
    else
        hipLaunchKernelGGL(batch_transport_kernel_f64<ImgT>, dim3(grid), dim3(kBlock), 0, stream, a, a.models);
    return hipGetLastError();
}

template <typename Real, typename ImgT, int G>
hipError_t launch_transport_impl(const TransportArgs<Real, ImgT, G> &a, int grid, hipStream_t stream)
{
    if constexpr (sizeof(Real) == 4) {
        if (a.view.learned)
            hipLaunchKernelGGL((transport_kernel_f32<G, true, false, false>), dim3(grid), dim3(kBlock), 0, stream, a);
        else if (a.view.hist)
            hipLaunchKernelGGL((transport_kernel_f32<G, false, true, false>), dim3(grid), dim3(kBlock), 0, stream, a);
        else if (a.mixed)
            hipLaunchKernelGGL((transport_kernel_f32<G, false, false, true>), dim3(grid), dim3(kBlock), 0, stream, a);
        else if (G == kCartesian && a.lone)
            hipLaunchKernelGGL((transport_kernel_f32<G, false, false, false, G == kCartesian>), dim3(grid), dim3(kBlock), 0, stream, a);
        else
            hipLaunchKernelGGL((transport_kernel_f32<G, false, false, false>), dim3(grid), dim3(kBlock), 0, stream, a);
        if (a.view.direct) {
            View<float, ImgT, 0> v{};
            v.n_ins = a.view.n_ins;
            v.n_lambda = a.view.n_lambda;
            v.images = a.view.images;
            v.direct = a.view.direct;
            v.direct_pix = a.view.direct_pix;
            v.direct_shards = a.view.direct_shards;
            v.direct_stride = a.view.direct_stride;
            const int blocks = (int)((long long)v.n_ins * v.n_lambda / 64) + 1;
            hipLaunchKernelGGL(direct_kernel<ImgT>, dim3(blocks < 1024 ? blocks : 1024), dim3(64), 0, stream, v);
        }
    } else {
        if (a.view.learned)
            hipLaunchKernelGGL((transport_kernel_f64<G, true, false>), dim3(grid), dim3(kBlock), 0, stream, a);
        else if (a.view.hist)
            hipLaunchKernelGGL((transport_kernel_f64<G, false, true>), dim3(grid), dim3(kBlock), 0, stream, a);
        else if (G == kCartesian && a.lone)
            hipLaunchKernelGGL((transport_kernel_f64<G, false, false, G == kCartesian>), dim3(grid), dim3(kBlock), 0, stream, a);
        else
            hipLaunchKernelGGL((transport_kernel_f64<G, false, false>), dim3(grid), dim3(kBlock), 0, stream, a);
    }
    return hipGetLastError();
}

} // namespace mcrt
