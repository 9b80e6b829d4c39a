// aux_kernels.hip -- fills and readback conversions around the transport
// kernel: zeroing of tallies (a kernel rather than a memset, so the sequence
// stays valid under stream capture), the (wavelength, cell) -> (cell,
// wavelength) table transpose of the readback, and image scaling to flux.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace mcrt {

__global__ void fill_zero_kernel(uint4 *p, size_t n16, unsigned char *tail, size_t ntail)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) p[i] = make_uint4(0u, 0u, 0u, 0u);
    if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t stream)
{
    if (bytes == 0) return hipSuccess;
    size_t n16 = bytes / 16;
    size_t ntail = bytes - n16 * 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (uint4 *)p, n16,
                       (unsigned char *)p + n16 * 16, ntail);
    return hipGetLastError();
}

// The parts of a result in one launch (three launches of small areas: 5 us more).
struct Areas {
    Area a[3];
};
__global__ void __launch_bounds__(256) clear_kernel(Areas areas)
{
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const size_t n16 = areas.a[k].bytes / 16, tail = areas.a[k].bytes % 16;
        uint4 *p = (uint4 *)areas.a[k].p;
        for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256)
            p[i] = make_uint4(0, 0, 0, 0);
        if (blockIdx.x == 0 && threadIdx.x < tail) ((unsigned char *)(p + n16))[threadIdx.x] = 0;
    }
}

hipError_t launch_clear(const Area (&areas)[3], hipStream_t stream)
{
    Areas a;
    size_t most = 1;
    for (int k = 0; k < 3; ++k) {
        a.a[k] = areas[k];
        most = areas[k].bytes > most ? areas[k].bytes : most;
    }
    size_t blocks = (most / 16 + 255) / 256;
    blocks = blocks < 1 ? 1 : (blocks > 8192 ? 8192 : blocks);
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// Readback of the table: dst[(c - c0) * n_lambda + l] = src[l * n_store +
// store(c)] for the natural cells c in [c0, c1).  A tile is a run of bricks
// along x (consecutive in storage) for some wavelengths: read coalesced along
// storage, turned in LDS, written coalesced along (x, wavelength).  A grid
// without bricks is one row of 32-cell bricks.  Bound by memory: 2.1 GB of a
// 256^3 table of 16 wavelengths take 1.6 ms (gathered by wavelength: 3.8 ms).
struct Readback {
    int n[3], bs[3], nb[3], sh[3];
    int b0[3], nt[3];  // first brick (x: first run of bricks) and tiles per axis
    int run;           // bricks along x per tile
    int lam_tile, lam_tiles;
    int n_lambda;
    int64_t n_store, c0, c1;
};
constexpr int kTileElems = 4096; // doubles of a tile

__global__ void __launch_bounds__(256) table_readback_kernel(const double *src, double *dst, Readback r)
{
    // rows of one stored cell's wavelengths, padded to an odd length
    __shared__ double tile[kTileElems + kTileElems / 2];
    int64_t t = blockIdx.x;
    const int lt = (int)(t % r.lam_tiles);
    t /= r.lam_tiles;
    const int bx0 = (r.b0[0] + (int)(t % r.nt[0])) * r.run;
    t /= r.nt[0];
    const int by = r.b0[1] + (int)(t % r.nt[1]), bz = r.b0[2] + (int)(t / r.nt[1]);
    const int l0 = lt * r.lam_tile, nl = min(r.lam_tile, r.n_lambda - l0);
    const int pitch = nl | 1;
    const int64_t s0 = (bx0 + (int64_t)r.nb[0] * (by + (int64_t)r.nb[1] * bz)) * 32;
    const int bricks = min(r.run, r.nb[0] - bx0);
    const int cells = bricks * 32;
    for (int e = threadIdx.x; e < cells * nl; e += 256) {
        const int l = e / cells, s = e - l * cells;
        if (s0 + s < r.n_store) tile[s * pitch + l] = src[(int64_t)(l0 + l) * r.n_store + s0 + s];
    }
    __syncthreads();
    const int row = bricks << r.bs[0]; // cells of the tile along x
    for (int e = threadIdx.x; e < cells * nl; e += 256) {
        const int q = e / nl, l = e - q * nl; // cell of the tile, x fastest
        const int yz = q / row, x = q - yz * row;
        const int y = yz & ((1 << r.bs[1]) - 1), z = yz >> r.bs[1];
        const int ix = (bx0 << r.bs[0]) + x, iy = (by << r.bs[1]) + y, iz = (bz << r.bs[2]) + z;
        if (ix >= r.n[0] || iy >= r.n[1] || iz >= r.n[2]) continue;
        const int64_t c = ix + (int64_t)r.n[0] * (iy + (int64_t)r.n[1] * iz);
        if (c < r.c0 || c >= r.c1) continue;
        const int s = (x >> r.bs[0]) * 32 + ((x & ((1 << r.bs[0]) - 1)) << r.sh[0]) + (y << r.sh[1]) + (z << r.sh[2]);
        dst[(c - r.c0) * r.n_lambda + l0 + l] = tile[s * pitch + l];
    }
}

hipError_t launch_table_readback(const double *src, double *dst, int64_t n_store, int n_lambda, const int *n,
                                 const int *bs, const int *sh, const int *nb, int64_t c0, int64_t n_cells,
                                 int64_t grid_cells, hipStream_t stream)
{
    Readback r{};
    r.n_lambda = n_lambda;
    r.n_store = n_store;
    r.c0 = c0;
    r.c1 = c0 + n_cells;
    for (int a = 0; a < 3; ++a) {
        r.n[a] = bs ? n[a] : (a == 0 ? (int)grid_cells : 1);
        r.bs[a] = bs ? bs[a] : (a == 0 ? 5 : 0);
        r.sh[a] = bs ? sh[a] : 0;
        r.nb[a] = bs ? nb[a] : (a == 0 ? (int)((grid_cells + 31) / 32) : 1);
    }
    // wavelengths per tile: all of them up to 64, so that a row of cells is one run of the output
    r.lam_tile = n_lambda < 64 ? n_lambda : 64;
    r.lam_tiles = (n_lambda + r.lam_tile - 1) / r.lam_tile;
    r.run = kTileElems / (32 * r.lam_tile);
    // the box of bricks that holds cells [c0, c1)
    const int64_t nxy = (int64_t)r.n[0] * r.n[1], last = r.c1 - 1;
    int lo[3] = {0, 0, (int)(c0 / nxy)}, hi[3] = {r.n[0] - 1, r.n[1] - 1, (int)(last / nxy)};
    if (lo[2] == hi[2]) {
        lo[1] = (int)(c0 % nxy / r.n[0]);
        hi[1] = (int)(last % nxy / r.n[0]);
        if (lo[1] == hi[1]) {
            lo[0] = (int)(c0 % r.n[0]);
            hi[0] = (int)(last % r.n[0]);
        }
    }
    int64_t tiles = 0;
    for (;; r.run /= 2) {
        tiles = r.lam_tiles;
        for (int a = 0; a < 3; ++a) {
            int b0 = lo[a] >> r.bs[a], b1 = hi[a] >> r.bs[a];
            if (a == 0) {
                b0 /= r.run;
                b1 /= r.run;
            }
            r.b0[a] = b0;
            r.nt[a] = b1 - b0 + 1;
            tiles *= r.nt[a];
        }
        // small tables: shorter runs, up to 1024 workgroups (whole calls for 20^3 cells of 4
        // wavelengths 17.1 -> 13.5 us, 40^3 20.3 -> 16.1, a depth-7 octree 20.2 -> 13.5)
        if (tiles >= 1024 || r.run == 1) break;
    }
    if (n_cells <= 0) return hipSuccess;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(table_readback_kernel, dim3((unsigned)tiles), dim3(256), 0, stream, src, dst, r);
    return hipGetLastError();
}

// The copies are summed in copy order, in FP64; entries that no copy holds
// (most of a large grid's, in a short launch) cost their reads only.  Bound
// by those: 49 MB of copies of a 7 MB table take 18 us.
template <typename T>
__global__ void __launch_bounds__(256) merge_copies_kernel(T *dst, T *copies, int n, size_t elems)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < elems; i += stride) {
        double sum = 0.0;
        bool any = false;
        for (int k = 0; k < n; ++k) {
            const T x = copies[(size_t)k * elems + i];
            any = any || x != T(0);
            sum += (double)x;
        }
        if (!any) continue;
        for (int k = 0; k < n; ++k) copies[(size_t)k * elems + i] = T(0);
        dst[i] = (T)((double)dst[i] + sum);
    }
}

template <typename T>
hipError_t launch_merge_copies(T *dst, T *copies, int n, size_t elems, hipStream_t stream)
{
    size_t blocks = (elems + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(merge_copies_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, stream, dst, copies, n, elems);
    return hipGetLastError();
}

template hipError_t launch_merge_copies<float>(float *, float *, int, size_t, hipStream_t);
template hipError_t launch_merge_copies<double>(double *, double *, int, size_t, hipStream_t);

// A result's energy sums and counters from its shards, in order (shard 0 first).
__global__ void __launch_bounds__(64) sum_tally_kernel(const unsigned long long *tally, unsigned long long *dst)
{
    const int i = threadIdx.x;
    if (i >= kTallyWords) return;
    unsigned long long n = 0;
    double e = 0.0;
#pragma unroll
    for (int k = 0; k < kTallyShards; ++k) {
        const unsigned long long x = tally[k * kTallyWords + i];
        n += x;
        e += __longlong_as_double((long long)x);
    }
    dst[i] = i < 4 ? (unsigned long long)__double_as_longlong(e) : n;
}

hipError_t launch_sum_tally(const unsigned long long *tally, unsigned long long *dst, hipStream_t stream)
{
    hipLaunchKernelGGL(sum_tally_kernel, dim3(1), dim3(64), 0, stream, tally, dst);
    return hipGetLastError();
}

// A few words into pinned memory: one launch instead of a copy that the host
// waits for by itself (8 us against 15).
__global__ void copy_words_kernel(const unsigned long long *src, unsigned long long *dst, unsigned n)
{
    for (unsigned i = threadIdx.x; i < n; i += blockDim.x) dst[i] = src[i];
}

hipError_t launch_copy_words(const void *src, void *dst, size_t n, hipStream_t stream)
{
    hipLaunchKernelGGL(copy_words_kernel, dim3(1), dim3(64), 0, stream, (const unsigned long long *)src,
                       (unsigned long long *)dst, (unsigned)n);
    return hipGetLastError();
}

template <typename ImgT>
__global__ void image_scale_kernel(const ImgT *src, double *dst, int64_t n, double scale)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) dst[i] = (double)src[i] * scale;
}

template <typename ImgT>
hipError_t launch_image_scale(const ImgT *src, double *dst, int64_t n, double scale, hipStream_t stream)
{
    int64_t blocks = (n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(image_scale_kernel<ImgT>, dim3((unsigned)blocks), dim3(256), 0, stream, src, dst, n, scale);
    return hipGetLastError();
}

template hipError_t launch_image_scale<float>(const float *, double *, int64_t, double, hipStream_t);
template hipError_t launch_image_scale<double>(const double *, double *, int64_t, double, hipStream_t);

// SED of an instrument: sed[l] = scale * sum over the pixels of wavelength
// slice l, in FP64.  A workgroup sums a part of a slice (a fixed stride of
// pixels per thread, then a fixed-shape tree in LDS), a second kernel a
// slice's parts in order, so the result does not depend on timing.  Bound by
// the reads: 34 MB of a 1024^2 image of 8 wavelengths take 13 us (a slice to one
// workgroup: 1100 us).
constexpr int64_t kSedPart = 1 << 14; // pixels of a part

template <typename ImgT>
__global__ void __launch_bounds__(256) sed_parts_kernel(const ImgT *img, double *parts, int64_t npix)
{
    __shared__ double part[256];
    const ImgT *row = img + (int64_t)blockIdx.y * npix;
    const int64_t p0 = (int64_t)blockIdx.x * kSedPart, p1 = p0 + kSedPart < npix ? p0 + kSedPart : npix;
    double acc = 0.0;
#pragma unroll 8
    for (int64_t i = p0 + threadIdx.x; i < p1; i += 256) acc += (double)row[i];
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) parts[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = part[0];
}

__global__ void __launch_bounds__(64) sed_sum_kernel(const double *parts, int n_parts, double *sed, int n_lambda,
                                                     double scale)
{
    const int l = blockIdx.x * 64 + threadIdx.x;
    if (l >= n_lambda) return;
    double acc = 0.0;
#pragma unroll 16
    for (int k = 0; k < n_parts; ++k) acc += parts[(int64_t)l * n_parts + k];
    sed[l] = acc * scale;
}

int64_t sed_parts(int64_t npix) { return (npix + kSedPart - 1) / kSedPart; }

template <typename ImgT>
hipError_t launch_sed(const ImgT *img, double *parts, double *sed, int n_lambda, int64_t npix, double scale,
                      hipStream_t stream)
{
    const unsigned n = (unsigned)sed_parts(npix);
    // the grid's y is limited to 65535 slices
    for (int l0 = 0; l0 < n_lambda; l0 += 65535) {
        const int nl = n_lambda - l0 < 65535 ? n_lambda - l0 : 65535;
        hipLaunchKernelGGL(sed_parts_kernel<ImgT>, dim3(n, (unsigned)nl), dim3(256), 0, stream, img + l0 * npix,
                           parts + (int64_t)l0 * n, npix);
    }
    if (n_lambda > 0)
        hipLaunchKernelGGL(sed_sum_kernel, dim3((unsigned)((n_lambda + 63) / 64)), dim3(64), 0, stream, parts, (int)n,
                           sed, n_lambda, scale);
    return hipGetLastError();
}

template hipError_t launch_sed<float>(const float *, double *, double *, int, int64_t, double, hipStream_t);
template hipError_t launch_sed<double>(const double *, double *, double *, int, int64_t, double, hipStream_t);

} // namespace mcrt
