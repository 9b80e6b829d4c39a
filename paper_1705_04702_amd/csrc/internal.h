// internal.h -- declarations shared by the library's translation units (not
// part of the public C-ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mcrt {

constexpr int kBlock = 256;    // threads per workgroup (4 waves)
constexpr int kNumStats = 10;  // packets, events, prop, locate, peel cells, adds, dropped, capped, guard, nonfinite
// A result's energy sums (4, FP64) and counters (kNumStats): kTallyShards shards
// of 16 words, each on a line of its own.  Every wave adds its tally when it
// ends, and additions to one line take turns at the memory side (7.7 ns each):
// with one line and an instruction per word, a launch of 4096 waves spent 340 us
// on them.
constexpr int kTallyShards = 32, kTallyWords = 16;

template <typename Real, typename ImgT, int G> struct View;
template <typename Real> struct Optics;
template <typename Real> struct InsDesc;

template <typename Real, typename ImgT, int G> struct TransportArgs {
    View<Real, ImgT, G> view;
    const Optics<Real> *optics;   // global copies, staged into LDS by the kernel
    const InsDesc<Real> *ins;
    uint64_t count;               // packets per wavelength in this launch
    uint64_t first_id;            // first packet id
    uint64_t n_chunks;            // chunks in the work queue: n_lambda * lam_chunks
    uint64_t lam_chunks;          // chunks of each wavelength
    uint32_t chunk;               // packets per chunk (all of one wavelength)
    int threshold;                // lanes that must finish their propagation before events run
    int lanes;                    // lanes of a wave that take packets (64 but in small launches)
    int lone;                     // one lane, whose packets the whole wave marches (see lone_march)
    // no more chunks than waves, all resident: a wave takes the chunk of its
    // number (neighbouring chunks, of like cost, on different compute units),
    // and not from the queue, whose counter is one line for all waves (8000
    // packets in a 32^3 sphere: 567 -> 527 us)
    int own_chunks;
    int mixed;                    // march all kinds in one loop (see launch_plan.h)
    unsigned long long *counter;  // queue position (chunks handed out)
    // further copies of the table, [table_copies - 1][n_lambda][n_store], and
    // of the images; workgroup b adds to copy b mod their (power-of-two) number
    double *more_tables;
    ImgT *more_images;
    int table_copies, image_copies;
    long long image_elems;
    unsigned long long *tally;    // [kTallyShards][kTallyWords]
    const void *mlp_frags;        // learned FP32: forward fragments (bf16, fragment order)
    const float *mlp_bias;        // learned FP32: biases [176]
};

// G = 0 Cartesian, 1 octree
hipError_t launch_transport_f32c(const TransportArgs<float, float, 0> &a, int grid, hipStream_t stream);
hipError_t launch_transport_f32o(const TransportArgs<float, float, 1> &a, int grid, hipStream_t stream);
hipError_t launch_transport_f64c(const TransportArgs<double, double, 0> &a, int grid, hipStream_t stream);
hipError_t launch_transport_f64o(const TransportArgs<double, double, 1> &a, int grid, hipStream_t stream);

// Allocation-free runs (noalloc.hip): a file-scope device array per GPU
// holds the queue counter (first kNoAllocHeader bytes) and the launch's
// per-wavelength optics (at most kNoAllocMaxLambda).  setup takes the
// array's device address for `device` (that device current) once; scratch
// returns it (NULL before setup).  launch_noalloc_setup zeroes the counter and
// writes the optics from the sim's device copies with L0 = lum / n_per_lambda.
constexpr size_t kNoAllocHeader = 256;
constexpr int kNoAllocMaxLambda = 4096;
size_t noalloc_scratch_bytes();
hipError_t noalloc_scratch_setup(int device);
void *noalloc_scratch(int device);
template <typename Real>
hipError_t launch_noalloc_setup(void *scratch_dev, const Optics<Real> *optics_base, const double *lum, int n_lambda,
                                uint64_t n_per_lambda, hipStream_t stream);

// auxiliary kernels (aux_kernels.hip)
hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t stream);
// The sums of a result's shards, kTallyWords words, to memory that a kernel can write.
hipError_t launch_sum_tally(const unsigned long long *tally, unsigned long long *dst, hipStream_t stream);
hipError_t launch_copy_words(const void *src, void *dst, size_t n, hipStream_t stream);
// Clears three areas, each of whole 16-byte pieces but for its end.
struct Area {
    void *p;
    size_t bytes;
};
hipError_t launch_clear(const Area (&areas)[3], hipStream_t stream);
// dst[(c - c0) * n_lambda + l] = src[l * n_store + store(c)] for the n_cells
// cells c from c0; store() is the bricked layout (bs, sh, nb) of a Cartesian
// grid with n cells per axis, or the identity over grid_cells when bs == NULL.
hipError_t launch_table_readback(const double *src, double *dst, int64_t n_store, int n_lambda,
                                 const int *n, const int *bs, const int *sh, const int *nb, int64_t c0,
                                 int64_t n_cells, int64_t grid_cells, hipStream_t stream);
// dst[i] += the n copies' elements i (copies[n][elems]), which are cleared
template <typename T>
hipError_t launch_merge_copies(T *dst, T *copies, int n, size_t elems, hipStream_t stream);
template <typename ImgT>
hipError_t launch_image_scale(const ImgT *src, double *dst, int64_t n, double scale, hipStream_t stream);
// Dust emission (dust.hip).  Cartesian cells in natural order
// m = ix + nx (iy + ny iz), tables and density in the bricked storage order;
// octree leaves in leaf order (storage order too).
struct DustGrid {
    long long n_cells, n_store;
    int n_lambda;
    int n[3], bs[3], sh[3], nb[3];
    const int *leaf; // octree: per leaf (origin x, y, z, level); NULL for Cartesian
};
struct DustTables {
    const double *t[4]; // absorption tables [n_lambda][n_store], summed
    int n;
};
int dust_blocks(long long n);          // blocks of the per-cell kernels over n cells (partial sums)
int dust_scan_tiles(long long n);       // tiles per row of the scan
// absorbed[s] = sum over wavelengths of the summed tables, s in storage
// order (n_store entries); part_* per block of dust_blocks(n_store)
hipError_t launch_dust_absorbed(const DustGrid &g, const DustTables &tabs, const float *density, double *absorbed,
                                double *part_abs, double *part_mass, hipStream_t st);
// T[m] and emis[l][m] (see dust.hip)
hipError_t launch_dust_emission(const DustGrid &g, const double *absorbed, const float *density,
                                const double *lambda_um, const double *kw, double u0, double T0, double beta,
                                double *T, double *emis, hipStream_t st);
// x[rows][n] := inclusive running sums of each row; tile_sums[rows][tiles]
hipError_t launch_dust_scan(double *x, long long n, int rows, double *tile_sums, hipStream_t st);
// total[rows]: the last running sum of each row
hipError_t launch_dust_totals(const double *cdf, long long n, int rows, double *total, hipStream_t st);
// guide[rows][K]: first index whose running sum exceeds k (row total / K)
hipError_t launch_dust_guide(const double *cdf, long long n, int K, int rows, int *guide, hipStream_t st);

// sed[l] = scale * sum of the npix pixels of slice l (n_lambda slices);
// parts: [n_lambda][sed_parts(npix)] scratch
int64_t sed_parts(int64_t npix);
template <typename ImgT>
hipError_t launch_sed(const ImgT *img, double *parts, double *sed, int n_lambda, int64_t npix, double scale,
                      hipStream_t stream);

} // namespace mcrt

namespace mcrt {

// One model of a batched launch: its scene view (pointers to global optics and
// instrument arrays), its packet range and its own tally accumulators.
template <typename Real, typename ImgT> struct ModelDesc {
    View<Real, ImgT, 0> view;
    const Optics<Real> *optics;
    const InsDesc<Real> *ins;
    uint64_t count;       // packets per wavelength in this launch
    uint64_t first_id;
    uint64_t total;       // count * n_lambda
    uint64_t chunk0;      // index of the model's first chunk in the batch queue
    uint32_t chunk;       // packets per chunk
    int apart;            // one kind of march per loop from the start (see the batch kernel)
    unsigned long long *tally; // [kTallyShards][kTallyWords]
};

template <typename Real, typename ImgT> struct BatchArgs {
    const ModelDesc<Real, ImgT> *models;
    int n_models;
    uint64_t total_chunks;
    int drain;            // the kernel for few chunks
    int threshold;
    unsigned long long *counter;
};

// slots: the deposit tile per lane, 8 or 16
hipError_t launch_batch_f32(const BatchArgs<float, float> &a, int grid, hipStream_t stream, int slots);

// learned proposal (proposal.hip)
struct GradArgs {
    const uint16_t *frags;    // all 60 fragments
    const float *bias;        // [176]
    const float *X, *KP, *C;  // samples: features [n][9], direction [n][3], weight [n]
    int64_t n;                // samples available
    int64_t m;                // samples in this pass
    int random;               // 0: samples 0 .. m-1; 1: m uniform draws (with replacement) from [0, n)
    uint32_t key0, key1, step;
    float scale;              // multiplies every weight (1 / sum of the weights of the pass)
    float *partial;           // [workgroups][kGradStride]
    double *loss_partial;     // [workgroups]
};
struct AdamArgs {
    float *theta, *m, *v;     // FP32 master parameters and moments [7400]
    uint16_t *frags;          // packed copies of the parameters: fragments,
    float *bias;              // biases,
    double *theta64;          // FP64 copy
    float lr, b1, b2, eps;
    int step;                 // Adam time step (>= 1)
    int update;               // 0: only sum the gradient
    float *grad_out;          // optional [7400]: the summed gradient
    double *loss_out;         // optional: the summed loss
};
constexpr int kGradStrideFloats = 7424;
constexpr int kFragAllElems = 60 * 64 * 4; // bf16 values of all fragments
hipError_t launch_sum_f32(const float *x, int64_t n, double *cols, double *out, hipStream_t stream); // cols [1024]
// Tiles of records that the compaction counts and scans.
int64_t hist_tiles(int64_t n_slots, int E);
hipError_t launch_proposal_pack(const float *theta, uint16_t *frags, float *bias, double *theta64,
                                hipStream_t stream);
hipError_t launch_proposal_forward(const uint16_t *frags, const float *bias, const float *X, int64_t n, float *out,
                                   hipStream_t stream);
hipError_t launch_proposal_grad(const GradArgs &g, int groups, hipStream_t stream); // workgroups
hipError_t launch_proposal_adam(const float *partial, int n, const double *loss_partial, const AdamArgs &a,
                                hipStream_t stream);
hipError_t launch_hist_count(const void *h, const void *tot, bool fp64, int64_t n_slots, int E, uint32_t *count,
                             uint64_t *offset, uint64_t *block_sums, uint64_t *total, hipStream_t st);
hipError_t launch_hist_write(const void *h, const void *tot, bool fp64, int64_t n_slots, int E,
                             const uint64_t *offset, float *X, float *KP, float *C, hipStream_t st);
hipError_t launch_batch_f64(const BatchArgs<double, double> &a, int grid, hipStream_t stream);

} // namespace mcrt
