// launch_plan.h -- how a single launch spreads its packets over waves, chunks
// and lanes.  Whole numbers only, no device code: the CPU tests call it as it is.
#pragma once

#include <algorithm>
#include <cstdint>

namespace mcrt {

// What the rules look at.
struct LaunchIn {
    uint64_t n_cu;     // compute units
    uint64_t count;    // packets per wavelength
    uint64_t n_lambda;
    uint64_t cells;    // along the three axes together
    bool octree;
    bool point;        // the packets start in one place
    bool direct;       // FP32 packets of a point source that emits towards an instrument
    bool plain;        // no learned proposal, no histories
    int chunk, chunk_shift, waves_per_cu, threshold; // the caller's (mcrt_options), 0: automatic
};

struct LaunchPlan {
    uint64_t waves;
    int waves_per_cu;            // at most
    uint32_t chunk;              // packets per chunk
    uint64_t lam_chunks, n_chunks;
    int lanes;                   // lanes of a wave that take packets
    bool lone;                   // one, which the whole wave marches
    int threshold;
    bool mixed;                  // all kinds of march in one loop
    bool sums;                   // direct light in FP64 sums
    bool own_chunks;             // a wave takes the chunk of its number
    bool copies;                 // further copies of the table or the images, if they pay
};

// The automatic chunk times 2^shift (at least 1, at most 2^24 packets).
inline uint64_t shifted_chunk(uint64_t c, int shift)
{
    c = shift >= 0 ? c << shift : c >> (-shift);
    return c < 1 ? 1 : (c > (uint64_t(1) << 24) ? (uint64_t(1) << 24) : c);
}

// Lanes of a wave that must finish their propagation before its events run
// (see transport_kernel.h).
inline int default_threshold(bool octree) { return octree ? 48 : 64; }

inline LaunchPlan plan_launch(const LaunchIn &in)
{
    LaunchPlan p{};
    const uint64_t total = in.count * in.n_lambda;
    const int full_per_cu = in.waves_per_cu > 0 ? in.waves_per_cu : 16;
    const uint64_t full = in.n_cu * (uint64_t)full_per_cu;
    p.waves_per_cu = full_per_cu;
    // The queue's chunks: whole waves, eight or more chunks to a wave (the
    // tail: 1.6e6 packets of a depth-9 torus take 20.1 ms in chunks of 64, 25.9
    // in chunks of 192), at most 512 packets (1.6e7 packets of a 256^3 disk:
    // 217 ms in chunks of 64, 210 in chunks of 512).
    uint64_t auto_chunk = total / (8 * full) / 64 * 64;
    auto_chunk = auto_chunk < 64 ? 64 : (auto_chunk > 512 ? 512 : auto_chunk);
    p.threshold = in.threshold > 0 ? in.threshold : default_threshold(in.octree);
    // A launch of fewer packets than lanes: every wave takes one chunk of
    // total / waves packets (55 000 packets on a 61 x 45 x 27 disk with 11
    // wavelengths: 1.3 ms with 14 lanes to a wave, 1.4-1.5 ms with 32 or 64).
    // On Cartesian grids as many waves as are resident (12 per compute unit),
    // for a wave that has to wait for another one to end starts its only chunk
    // then; point sources, whose packets all begin in the same cells, two to a
    // SIMD while that gives a wave 32 packets at most (packets in a 32^3
    // sphere with 16, 12 and 8 waves: 8000 540, 398 and 361 us, 32 000 654, 488
    // and 421; on the disk, 22 000 packets 1198, 1170 and 1202, in FP64 4000 for
    // each of 6 wavelengths 2076, 1890 and 2052).
    if (!in.octree && in.waves_per_cu <= 0) {
        const int few = in.point && total <= in.n_cu * 8 * 32 ? 8 : 12;
        if (total < 64 * in.n_cu * few) p.waves_per_cu = few;
    }
    p.waves = in.n_cu * (uint64_t)p.waves_per_cu;
    uint64_t lanes = (total + p.waves - 1) / p.waves;
    // A point source's direct light towards an instrument lands in one pixel,
    // in FP32 additions of one wave's share each, whose rounding follows their
    // sizes.  Up to 32768 packets per wavelength the waves' shares are summed in
    // FP64 instead, so that their number does not matter (500 packets in a 32^3
    // sphere: 0.27 ms with a lane to a wave, 0.44 with 32).
    // Larger launches make the additions that this library has always made: full
    // waves, chunks of 32 to 256 packets from the queue, in plain runs the mixed
    // loop, and where a wave refills its lanes (chunks of more than 32) one table,
    // for copies of it change which lanes are free together.  Any other shape
    // rounds otherwise, and to more: image against 64 bits in that sphere, mean of
    // 12 seeds, 60 000 packets 1.2e-5 so, 1.4e-5 in chunks that waves own, marching
    // apart (0.73 and 0.52 ms); 1e5 packets 1.5e-5 in any shape on average, but 0.8
    // and 1.1e-5 at one seed (0.97 and 0.78 ms); 2e5 packets 3.6 to 4.7e-4 so, 5.8e-4
    // with copies (1.97 and 1.65 ms).  FP64 sums would be exact to 1e-6 at every
    // size, but move images by the whole of these errors, which is more than a
    // change of the launch may move them.  (Learned runs and histories have no mixed
    // loop: 1.5e-5 of 1e5 packets, 2.4e-5 of 2e5, where full waves refill at once.)
    p.sums = in.direct && in.count <= 32768;
    p.copies = true;
    const bool queue = in.direct && !p.sums;
    if (queue) {
        lanes = 64;
        p.waves_per_cu = full_per_cu;
        p.waves = full;
        auto_chunk = std::min<uint64_t>(256, std::max<uint64_t>(32, total / full));
        if (in.plain) {
            p.mixed = true;
            if (in.threshold <= 0) p.threshold = 16;
            p.copies = auto_chunk <= 32;
        }
    }
    p.lanes = lanes < 64 ? (int)lanes : 64;
    if (p.lanes < 64) auto_chunk = (uint64_t)p.lanes;
    p.chunk = (uint32_t)(in.chunk > 0 ? (uint64_t)in.chunk : shifted_chunk(auto_chunk, in.chunk_shift));
    // A chunk that the caller made larger is not marched by fewer lanes than it has
    // packets (500 packets of a 32^3 sphere in chunks of 256: 34 ms in two waves of
    // one lane, 1.4 ms in two of 64).
    if (in.chunk > 0 || in.chunk_shift > 0) p.lanes = std::max(p.lanes, (int)std::min<uint32_t>(64, p.chunk));
    // One packet to a wave: the whole wave marches it, but on small grids, where the
    // usual loop's 8 cells at a time reach a ray's end as soon (kernels of 10 to 2000
    // packets, usual loop against the wave's, FP32: 4^3 sphere 0.75 to 1.03 of its
    // time, 8^3 0.81 to 1.10, 10^3 0.87 to 1.12, 24^3 1.07 to 1.52; disk of 8 x 8 x 4
    // cells 0.76 to 1.0, 32 x 32 x 16 0.98 to 1.13).
    p.lone = p.lanes == 1 && !in.octree && in.plain && in.cells >= 30;
    p.lam_chunks = (in.count + p.chunk - 1) / p.chunk;
    p.n_chunks = p.lam_chunks * in.n_lambda;
    // (a wavelength's last chunk is a part, so there may be a few more of them
    // than the waves they were made for)
    p.own_chunks = !in.octree && !queue && p.n_chunks <= in.n_cu * 12 && (in.waves_per_cu <= 0 || p.n_chunks <= p.waves);
    if (p.waves > p.n_chunks || p.own_chunks) p.waves = p.n_chunks;
    return p;
}

} // namespace mcrt
