// pm_kernels.hip -- launchers of the particle step's kernels (all but the
// fused and advance kernels, whose variants live in pm_step_f64.hip and
// pm_step_f32.hip).
#include "pm_device.h"

namespace pm {
bool stage_shape_supported(Shape sh)
{
#define PM_ONE(W, I) if (sh.wg == W && sh.items == I) return true;
    PM_STAGE_SHAPES(PM_ONE)
#undef PM_ONE
    return false;
}

bool shape_supported(Shape sh)
{
#define PM_ONE(W, I) if (sh.wg == W && sh.items == I) return true;
    PM_SHAPES(PM_ONE)
#undef PM_ONE
    return false;
}

hipError_t launch_prep(const KArgs &a, int mode, hipStream_t st)
{
    int64_t work = 1;
    if (mode & kPrepZeroLb)  // four times the status words: workgroup 0 is busy with the tables
        work = (int64_t)a.ws.pool_extent / a.tile + a.sub_count + 2;
    if (mode & (kPrepZeroCounts | kPrepCheckSend))
        work = work > (int64_t)a.dc.nsub * 27 ? work : (int64_t)a.dc.nsub * 27;
    if (mode & kPrepZeroCounts)
        work = work > (int64_t)a.sub_count * 27 ? work : (int64_t)a.sub_count * 27;
    int64_t g = (work + 1023) / 1024;
    const int grid = (int)(g < 1 ? 1 : (g > 1024 ? 1024 : g));
    hipLaunchKernelGGL(k_prep, dim3(grid), dim3(256), 0, st, a, mode);
    return hipGetLastError();
}

// The plain path's kernels in every launch shape.
#define PM_PLAIN(K, W, I)                                                               \
    if (sh.wg == W && sh.items == I) {                                                  \
        if (mixed)                                                                      \
            hipLaunchKernelGGL((K<W, I, float>), dim3(grid), dim3(W), 0, st, a);        \
        else                                                                            \
            hipLaunchKernelGGL((K<W, I, double>), dim3(grid), dim3(W), 0, st, a);       \
        return hipGetLastError();                                                       \
    }
#define PM_CLS_CASE(W, I) PM_PLAIN(k_classify, W, I)
#define PM_CMP_CASE(W, I) PM_PLAIN(k_compact, W, I)

hipError_t launch_classify(const KArgs &a, Shape sh, bool mixed, int grid, hipStream_t st)
{
    PM_SHAPES(PM_CLS_CASE)
    return hipErrorInvalidValue;
}

hipError_t launch_compact(const KArgs &a, Shape sh, bool mixed, int grid, hipStream_t st)
{
    PM_SHAPES(PM_CMP_CASE)
    return hipErrorInvalidValue;
}

hipError_t launch_append(const KArgs &a, bool mixed, int grid, hipStream_t st)
{
    if (mixed)
        hipLaunchKernelGGL((k_append<float>), dim3(grid), dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((k_append<double>), dim3(grid), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_route(const KArgs &a, bool mixed, bool append, hipStream_t st, bool ext)
{
    const int64_t jobs = (int64_t)a.sub_count * 27;
    const int grid = (int)(jobs < 4096 ? jobs : 4096);
    if (ext) {  // mid-step records of per-stage migration (always appended)
        if (mixed)
            hipLaunchKernelGGL((k_route<float, true, true>), dim3(grid), dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_route<double, true, true>), dim3(grid), dim3(256), 0, st, a);
        return hipGetLastError();
    }
    if (mixed) {
        if (append)
            hipLaunchKernelGGL((k_route<float, true, false>), dim3(grid), dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_route<float, false, false>), dim3(grid), dim3(256), 0, st, a);
    } else {
        if (append)
            hipLaunchKernelGGL((k_route<double, true, false>), dim3(grid), dim3(256), 0, st, a);
        else
            hipLaunchKernelGGL((k_route<double, false, false>), dim3(grid), dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

// Workgroups of 256 points that an XCD takes in a row.  Points in blobs need
// small chunks: an eighth of them a chunk leaves the XCDs with the dense regions
// idle (10^6 points of 256^3 in blobs, split float64: 68 us with consecutive
// workgroups on different XCDs, 71 in chunks of 16, 78 in eighths; 4 x 10^6
// interleaved float32 82, 85, 95), and uniform points lose little by them (7 x
// 10^6 of 400^3, float32: 347, 338, 349).  Eighths where so few points a cell
// share lines that a chunk's neighbours matter, and so many points that every
// eighth has its share of blobs (split float64 of 512^3, uniform: 5 x 10^6 744,
// 741, 704; 8.4 x 10^6 933, 924, 838; 9 x 10^6 in blobs 628, 632, 640).
// Interleaved fields show nothing for eighths.
template <int FA>
uint32_t interp_chunk(int64_t n, int64_t cells)
{
    const int64_t blocks = (n + 255) / 256;
    return FA != kFieldIlv && n >= (1 << 22) && n < cells / 12 ? (uint32_t)((blocks + 7) / 8) : 16;
}

template <typename FT, bool H, int FA>
hipError_t interp_t(const KArgs &a, int64_t n, const double *x, const double *y,
                    const double *z, void *ux, void *uy, void *uz, hipStream_t st)
{
    // Where points are fewer than cells, more workgroups on a compute unit push
    // each other's lines out of its L1: dynamic LDS that nothing uses leaves
    // room for four (8 million points of a split 256^3 field in float32: 0.193
    // ms with eight, 0.180 with four).  Points in blobs share lines whatever
    // their mean, but lose little by it (4 million: 0.110 and 0.113).  Not on
    // interleaved fields, which ask for a third of the lines (8 million points:
    // 0.126 with eight, 0.128 with four; 10 million in blobs: 0.146 and 0.161).
    const int64_t cells = (int64_t)a.f.n[0] * a.f.n[1] * a.f.n[2];
    const size_t lds = FA != kFieldIlv && n < cells ? 40 * 1024 : 0;
    const uint32_t chunk = interp_chunk<FA>(n, cells);
    const int64_t round = 8 * (int64_t)chunk;
    const int64_t g = ((n + 255) / 256 + round - 1) / round * round;
    const int grid = (int)(g > 65536 ? 65536 : g);
    hipLaunchKernelGGL((k_interp<FT, H, FA>), dim3(grid), dim3(256), lds, st, a, n, x, y, z,
                       (FT *)ux, (FT *)uy, (FT *)uz, chunk);
    return hipGetLastError();
}

template <typename FT, bool H>
hipError_t interp_h(const KArgs &a, int64_t n, const double *x, const double *y,
                    const double *z, void *ux, void *uy, void *uz, hipStream_t st)
{
    switch (field_arr(a.f)) {
    case kFieldMac:
        return interp_t<FT, H, kFieldMac>(a, n, x, y, z, ux, uy, uz, st);
    case kFieldIlv:
        return interp_t<FT, H, kFieldIlv>(a, n, x, y, z, ux, uy, uz, st);
    default:
        return interp_t<FT, H, kFieldSplit>(a, n, x, y, z, ux, uy, uz, st);
    }
}

template <typename FT>
hipError_t interp_ft(const KArgs &a, int64_t n, const double *x, const double *y,
                     const double *z, void *ux, void *uy, void *uz, hipStream_t st)
{
    return a.f.halo != 0 ? interp_h<FT, true>(a, n, x, y, z, ux, uy, uz, st)
                         : interp_h<FT, false>(a, n, x, y, z, ux, uy, uz, st);
}

hipError_t launch_interp(const KArgs &a, bool mixed, int64_t n, const double *x,
                         const double *y, const double *z, void *ux, void *uy, void *uz,
                         hipStream_t st)
{
    return mixed ? interp_ft<float>(a, n, x, y, z, ux, uy, uz, st)
                 : interp_ft<double>(a, n, x, y, z, ux, uy, uz, st);
}

hipError_t launch_touch(const KArgs &a, bool mixed, uint64_t *bits, hipStream_t st)
{
    const int grid = 4096;
    if (mixed) {
        if (a.f.halo)
            hipLaunchKernelGGL((k_touch<float, true>), dim3(grid), dim3(256), 0, st, a, bits);
        else
            hipLaunchKernelGGL((k_touch<float, false>), dim3(grid), dim3(256), 0, st, a, bits);
    } else {
        if (a.f.halo)
            hipLaunchKernelGGL((k_touch<double, true>), dim3(grid), dim3(256), 0, st, a, bits);
        else
            hipLaunchKernelGGL((k_touch<double, false>), dim3(grid), dim3(256), 0, st, a, bits);
    }
    return hipGetLastError();
}

hipError_t launch_popcount(const uint64_t *bits, int64_t words, unsigned long long *out,
                           hipStream_t st)
{
    hipLaunchKernelGGL(k_popcount, dim3(2048), dim3(256), 0, st, bits, words, out);
    return hipGetLastError();
}

hipError_t launch_fill(uint64_t *p, int64_t words, hipStream_t st)
{
    int64_t g = (words + 255) / 256;
    const int grid = (int)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
    hipLaunchKernelGGL(k_fill, dim3(grid), dim3(256), 0, st, p, words);
    return hipGetLastError();
}

hipError_t launch_flags_move(uint32_t *hdr, uint32_t *dst, hipStream_t st)
{
    hipLaunchKernelGGL(k_flags_move, dim3(1), dim3(64), 0, st, hdr, dst);
    return hipGetLastError();
}

hipError_t launch_step(const KArgs &a, Shape sh, bool mixed, int grid, hipStream_t st)
{
    return mixed ? launch_step_f32(a, sh, grid, st) : launch_step_f64(a, sh, grid, st);
}

hipError_t launch_advance(const KArgs &a, Shape sh, bool mixed, int grid, hipStream_t st)
{
    return mixed ? launch_advance_f32(a, sh, grid, st) : launch_advance_f64(a, sh, grid, st);
}

hipError_t launch_stage(const KArgs &a, Shape sh, bool mixed, int stage, int grid,
                        hipStream_t st)
{
    return mixed ? launch_stage_f32(a, sh, stage, grid, st)
                 : launch_stage_f64(a, sh, stage, grid, st);
}

int stage_occupancy(Shape sh, bool mixed, bool halo, bool nonlinear, int stage, bool ilv)
{
    const int nb = mixed ? stage_occupancy_f32(sh, halo, nonlinear, stage, ilv)
                         : stage_occupancy_f64(sh, halo, nonlinear, stage, ilv);
    return nb < 1 ? 1 : nb;
}

int step_occupancy(Shape sh, bool mixed, bool halo, bool nonlinear, int arr)
{
    const int nb = mixed ? step_occupancy_f32(sh, halo, nonlinear, arr)
                         : step_occupancy_f64(sh, halo, nonlinear, arr);
    return nb < 1 ? 1 : nb;
}

}  // namespace pm
