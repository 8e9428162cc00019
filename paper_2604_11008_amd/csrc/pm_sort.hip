// pm_sort.hip -- cell re-sort of the particle segments (gfx950).
//
// Not a step of the particle method: particles disperse from any order as
// they move, and the fused step's stencil gathers share cache lines only when
// neighbouring records are neighbours in space.  A caller re-sorts every few
// tens of steps.  Order within each segment: by the cell key (Z-order over
// pairs of cells along x, then the parity of the cell's x index), ties by
// input position -- a stable least-significant-digit radix sort of
// (key, position) pairs over tiles that never straddle a segment, followed by
// one gather of the records.  Keys are 32 bits up to 1024 cells an axis; a
// pass takes 9 bits where that saves a pass (25-bit keys of 256^3: three
// instead of four), else 8.  One sort of 4.2 million records in 64 segments of
// 256^3 cells, 25 steps after the last: 0.31 ms against 0.61 ms with 64-bit
// keys and tiles of 8192 records in rounds of 256 (keys 35 us, three passes of
// counts 6, scan 5 and scatter 27, gather 143; the records alone, read and
// written once, are 107 us at the 5 TB/s of a plain copy).  Every scatter and gather
// index is checked against its segment's range; a violation sets PM_F_LAYOUT
// instead of writing.
#include "pm_device.h"

namespace pm {
namespace {

constexpr int kSortWG = 512;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortWG * kSortItems;
constexpr int kSortWaves = kSortWG / 64;
constexpr int kScanBatch = 32;  // tiles whose counts a scan thread loads at once
constexpr int kScanParts = 8;   // threads that share a digit's tiles in the scan

// The 10 (21) low bits of v moved to bits 0, 3, 6, ... (the magic-mask bit
// spreading of Morton encoding: shift-or-mask steps).
__device__ __forceinline__ uint32_t spread3(uint32_t v, uint32_t)
{
    uint32_t x = v & 0x3ffu;
    x = (x | x << 16) & 0x30000ffu;
    x = (x | x << 8) & 0x300f00fu;
    x = (x | x << 4) & 0x30c30c3u;
    x = (x | x << 2) & 0x9249249u;
    return x;
}

__device__ __forceinline__ uint64_t spread3(uint32_t v, uint64_t)
{
    uint64_t x = v & 0x1fffffu;
    x = (x | x << 32) & 0x1f00000000ffffull;
    x = (x | x << 16) & 0x1f0000ff0000ffull;
    x = (x | x << 8) & 0x100f00f00f00f00full;
    x = (x | x << 4) & 0x10c30c30c30c30c3ull;
    x = (x | x << 2) & 0x1249249249249249ull;
    return x;
}

// Z-order code of (i >> 1, j, k) (bit b of each at 3b, 3b+1, 3b+2), times
// two, plus the parity of i.
template <typename KT>
__device__ __forceinline__ KT cell_key(int i, int j, int k)
{
    const KT code = spread3((uint32_t)i >> 1, KT()) | spread3((uint32_t)j, KT()) << 1 |
                    spread3((uint32_t)k, KT()) << 2;
    return code * 2 + ((uint32_t)i & 1u);
}

// Cell index of x along an axis of n cells (r = n / L): floor(x r) clamped to
// [0, n-1]; a NaN lands in cell 0.
__device__ __forceinline__ int cell_of(double x, double r, int n)
{
    const double s = x * r;
    if (!(s >= 0.0))
        return 0;
    if (!(s < (double)n))
        return n - 1;
    return (int)floor(s);
}

// The range's tile count, or -1 (PM_F_LAYOUT raised) when the layout is
// inconsistent or there are more tiles than the sort's tables hold.
__device__ __forceinline__ int64_t sort_tiles(const KArgs &a, const DSort &s)
{
    uint32_t *hdr = a.ws.hdr;
    if (flags_now(hdr) & PM_F_LAYOUT)
        return -1;
    const int64_t total = hdr[kHdrTiles];
    if (total > s.tiles) {
        if (blockIdx.x == 0 && threadIdx.x == 0)
            flag_or(hdr, PM_F_LAYOUT);
        return -1;
    }
    return total;
}

// One record of each active lane into the digit counts.  The high digits of a
// segment's keys, and the keys of a dense cell, are often the same in a whole
// wave: one addition then, instead of one after the other to one address.
__device__ __forceinline__ void count_digit(uint32_t *cnt, uint32_t d)
{
    const uint32_t d0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)d);
    const uint64_t active = __ballot(true);
    if (__ballot(d == d0) != active)
        atomicAdd(&cnt[d], 1u);
    else if ((int)__lane_id() == __ffsll((unsigned long long)active) - 1)
        atomicAdd(&cnt[d], (uint32_t)__popcll(active));
}

// Keys and positions of every record of the range, at the record's own pool
// position; per tile its place in the pool (the later kernels read it instead
// of searching the tile table again) and the counts of the first digit.
template <typename KT, int ND>
__global__ __launch_bounds__(kSortWG) void k_sort_keys(const KArgs a, DSort s)
{
    __shared__ uint32_t cnt[ND];
    __shared__ TileHead H;
    const int64_t total = sort_tiles(a, s);
    if (total < 0)
        return;
    const int tid = threadIdx.x;
    KT *keys = (KT *)s.keys[0];
    for (int64_t q = blockIdx.x; q < total; q += gridDim.x) {
        for (int d = tid; d < ND; d += kSortWG)
            cnt[d] = 0;
        if (tid == 0) {
            locate(a, kSortTile, q, H, a.ws.tile_start);
            s.place[q] = SortTile{(uint32_t)H.first, H.nitems, H.s, H.sl};
        }
        __syncthreads();
        const int64_t first = H.first;
        const int nitems = H.nitems;
        for (int i = tid; i < nitems; i += kSortWG) {
            const int64_t p = first + i;
            const int ci = cell_of(a.in.x[0][p], a.f.r[0], a.f.n[0]);
            const int cj = cell_of(a.in.x[1][p], a.f.r[1], a.f.n[1]);
            const int ck = cell_of(a.in.x[2][p], a.f.r[2], a.f.n[2]);
            const KT key = cell_key<KT>(ci, cj, ck);
            keys[p] = key;
            s.vals[0][p] = (uint32_t)p;
            count_digit(cnt, (uint32_t)key & (ND - 1));
        }
        __syncthreads();
        for (int d = tid; d < ND; d += kSortWG)
            s.hist[q * ND + d] = cnt[d];
        __syncthreads();
    }
}

// Per tile: the counts of the pass's digit.
template <typename KT, int ND>
__global__ __launch_bounds__(kSortWG) void k_sort_hist(const KArgs a, DSort s, int src,
                                                        int shift)
{
    __shared__ uint32_t cnt[ND];
    const int64_t total = sort_tiles(a, s);
    if (total < 0)
        return;
    const int tid = threadIdx.x;
    const KT *keys = (const KT *)s.keys[src];
    for (int64_t q = blockIdx.x; q < total; q += gridDim.x) {
        const SortTile t = s.place[q];
        for (int d = tid; d < ND; d += kSortWG)
            cnt[d] = 0;
        KT key[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int i = k * kSortWG + tid;
            key[k] = keys[t.first + (i < t.nitems ? i : t.nitems - 1)];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortItems; ++k)
            if (k * kSortWG + tid < t.nitems)
                count_digit(cnt, (uint32_t)(key[k] >> shift) & (ND - 1));
        __syncthreads();
        for (int d = tid; d < ND; d += kSortWG)
            s.hist[q * ND + d] = cnt[d];
        __syncthreads();
    }
}

// Per (segment, 64 digits): a tile's count of a digit becomes the records of
// that digit in the segment's earlier tiles, in place; the segment's totals
// beside.  Lane = digit, so every load is one run; each wave takes one of
// kScanParts equal shares of the tiles.
template <int ND>
__global__ __launch_bounds__(64 * kScanParts) void k_sort_scan(const KArgs a, DSort s)
{
    __shared__ uint32_t part_sum[kScanParts][64];
    if (sort_tiles(a, s) < 0)
        return;
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int64_t jobs = (int64_t)a.sub_count * (ND / 64);
    for (int64_t job = blockIdx.x; job < jobs; job += gridDim.x) {
        const int64_t sl = job / (ND / 64);
        const int d = (int)(job % (ND / 64)) * 64 + lane;
        const int64_t t0 = a.ws.tile_start[sl], t1 = a.ws.tile_start[sl + 1];
        const int64_t len = (t1 - t0 + kScanParts - 1) / kScanParts;
        const int64_t p0 = t0 + part * len, p1 = p0 + len < t1 ? p0 + len : t1;
        uint32_t tot = 0;
        int64_t t = p0;
        for (; t + kScanBatch <= p1; t += kScanBatch) {
            uint32_t c[kScanBatch];
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                c[u] = s.hist[(t + u) * ND + d];
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                tot += c[u];
        }
        for (; t < p1; ++t)
            tot += s.hist[t * ND + d];
        part_sum[part][lane] = tot;
        __syncthreads();
        uint32_t run = 0, all = 0;
#pragma unroll
        for (int q = 0; q < kScanParts; ++q) {
            const uint32_t c = part_sum[q][lane];
            run += q < part ? c : 0u;
            all += c;
        }
        if (part == 0)
            s.tot[sl * ND + d] = all;
        t = p0;
        for (; t + kScanBatch <= p1; t += kScanBatch) {
            uint32_t c[kScanBatch];
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                c[u] = s.hist[(t + u) * ND + d];
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u) {
                s.hist[(t + u) * ND + d] = run;
                run += c[u];
            }
        }
        for (; t < p1; ++t) {
            const uint32_t c = s.hist[t * ND + d];
            s.hist[t * ND + d] = run;
            run += c;
        }
        __syncthreads();  // part_sum is reused by the next job
    }
}

// Per tile: every record to its place for this digit, in tile order among
// the records of equal digit (so each pass is stable).  The tile's 4096 keys
// are read at once, each wave's 512 in order; a record's rank among its
// wave's earlier records of the same digit comes from ballots over the digit's
// bits and the wave's own counters in LDS (no barrier), the waves' counts and
// the digits are scanned once, and the tile leaves through LDS in digit order,
// so that the stores of a digit are runs.  Bound by the latency of a tile's
// few dependent steps: 4.2 million records (256^3 cells, 64 segments) pass in
// 26-29 us; rounds of 256 records, three barriers and a dependent load each,
// took 42-79 us.  8 items on 512 threads rather than 16 on 256: 128 registers
// instead of 190.
template <typename KT, int BITS>
__global__ __launch_bounds__(kSortWG) void k_sort_scatter(const KArgs a, DSort s, int src,
                                                           int shift)
{
    constexpr int ND = 1 << BITS;
    static_assert(ND <= kSortWG, "one digit a thread");
    __shared__ uint32_t cnt[kSortWaves][ND];
    __shared__ uint32_t place[ND];  // pool position of a digit's run, less its start in the tile
    __shared__ KT box[kSortTile];
    __shared__ uint64_t wave_tot[kSortWaves];
    const int64_t total = sort_tiles(a, s);
    if (total < 0)
        return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int dst = src ^ 1;
    const KT *kin = (const KT *)s.keys[src];
    KT *kout = (KT *)s.keys[dst];
    uint32_t fl = 0;
    for (int64_t q = blockIdx.x; q < total; q += gridDim.x) {
        const SortTile t = s.place[q];
        const uint32_t lo = (uint32_t)a.in.base[t.seg], n = (uint32_t)a.in.count[t.seg];
        KT key[kSortItems];
        uint32_t val[kSortItems], rank[kSortItems];
        const int i0 = w * (64 * kSortItems) + lane;  // item k: record i0 + 64 k
        const KT *kp = kin + t.first + i0;
        const uint32_t *vp = s.vals[src] + t.first + i0;
        if (t.nitems == kSortTile) {
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) {
                key[k] = kp[64 * k];
                val[k] = vp[64 * k];
            }
        } else {
#pragma unroll
            for (int k = 0; k < kSortItems; ++k) {
                key[k] = 0;
                val[k] = 0;
                if (i0 + 64 * k < t.nitems) {
                    key[k] = kp[64 * k];
                    val[k] = vp[64 * k];
                }
            }
        }
        uint32_t off = 0, seg_tot = 0;  // of digit tid
        if (tid < ND) {
            off = s.hist[q * ND + tid];
            seg_tot = s.tot[(int64_t)t.sl * ND + tid];
#pragma unroll
            for (int v = 0; v < kSortWaves; ++v)
                cnt[v][tid] = 0;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const bool valid = i0 + 64 * k < t.nitems;
            const uint32_t d = (uint32_t)(key[k] >> shift) & (ND - 1);
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int b = 0; b < BITS; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bb = __ballot(bit);
                m &= bit ? bb : ~bb;
            }
            const uint64_t below = m & ((1ull << lane) - 1ull);
            // one wave's LDS operations run in order; the barriers only keep
            // the compiler from moving them across each other
            __builtin_amdgcn_wave_barrier();
            const uint32_t before = cnt[w][d];
            __builtin_amdgcn_wave_barrier();
            if (valid && below == 0)
                cnt[w][d] = before + (uint32_t)__popcll(m);
            rank[k] = before + (uint32_t)__popcll(below);
            __builtin_amdgcn_sched_barrier(0);  // or all 16 masks are kept at once
        }
        __syncthreads();
        // starts of the digits in the tile and (high half) in the segment
        uint32_t wc[kSortWaves], mine = 0;
        if (tid < ND) {
#pragma unroll
            for (int v = 0; v < kSortWaves; ++v) {
                wc[v] = mine;
                mine += cnt[v][tid];
            }
        }
        const uint64_t sum = (uint64_t)seg_tot << 32 | mine;
        uint64_t incl = sum;
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) {
            const uint32_t l = (uint32_t)__shfl_up((int)(uint32_t)incl, sh, 64);
            const uint32_t h = (uint32_t)__shfl_up((int)(uint32_t)(incl >> 32), sh, 64);
            if (lane >= sh)
                incl += (uint64_t)h << 32 | l;
        }
        if (lane == 63)
            wave_tot[w] = incl;
        __syncthreads();
        uint64_t run = incl - sum;
#pragma unroll
        for (int v = 0; v < kSortWaves; ++v)
            run += v < w ? wave_tot[v] : 0;
        if (tid < ND) {
            const uint32_t start = (uint32_t)run;
            place[tid] = lo + (uint32_t)(run >> 32) + off - start;
#pragma unroll
            for (int v = 0; v < kSortWaves; ++v)
                cnt[v][tid] = start + wc[v];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            rank[k] += cnt[w][(uint32_t)(key[k] >> shift) & (ND - 1)];
            if (i0 + 64 * k < t.nitems)
                box[rank[k]] = key[k];
        }
        __syncthreads();
        uint32_t to[kSortItems];
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int i = k * kSortWG + tid;
            if (i < t.nitems) {
                const KT kk = box[i];
                to[k] = place[(uint32_t)(kk >> shift) & (ND - 1)] + i;
                if (to[k] - lo < n) {
                    kout[to[k]] = kk;
                } else {
                    to[k] = ~0u;
                    fl |= PM_F_LAYOUT;
                }
            }
        }
        __syncthreads();
        uint32_t *vbox = (uint32_t *)box;
#pragma unroll
        for (int k = 0; k < kSortItems; ++k)
            if (i0 + 64 * k < t.nitems)
                vbox[rank[k]] = val[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kSortItems; ++k) {
            const int i = k * kSortWG + tid;
            if (i < t.nitems && to[k] != ~0u)
                s.vals[dst][to[k]] = vbox[i];
        }
        __syncthreads();
    }
    if (fl)
        flag_or(a.ws.hdr, fl);
}

// The records in sorted order: out[out.base[s] + r] = in[vals[in.base[s] + r]].
// A workgroup takes half a tile, four records a thread, whose loads (8 arrays
// each) are all in flight at once: 143 us on 4.2 million records, against 203
// with a tile of 8192 a workgroup, one record after the other.
template <typename FT>
__global__ __launch_bounds__(kSortWG) void k_sort_gather(const KArgs a, DSort s, int src)
{
    constexpr int U = 4, Q = kSortItems / U;
    const int64_t total = sort_tiles(a, s);
    if (total < 0)
        return;
    uint32_t fl = 0;
    for (int64_t job = blockIdx.x; job < total * Q; job += gridDim.x) {
        const SortTile t = s.place[job / Q];
        const uint32_t lo = (uint32_t)a.in.base[t.seg], n = (uint32_t)a.in.count[t.seg];
        const int64_t obase = a.out.base[t.seg], ocap = a.out.cap[t.seg];
        uint32_t from[U];
        int64_t to[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = (int)(job % Q) * (U * kSortWG) + u * kSortWG + threadIdx.x;
            ok[u] = i < t.nitems;
            const uint32_t p = t.first + (ok[u] ? i : 0);
            from[u] = s.vals[src][p];
            to[u] = p - lo;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (ok[u] && from[u] - lo >= n) {
                fl |= PM_F_LAYOUT;
                ok[u] = false;
            }
            if (ok[u] && to[u] >= ocap) {
                fl |= PM_F_DEST_OVERFLOW;
                ok[u] = false;
            }
            from[u] = ok[u] ? from[u] : lo;  // a record of the segment: never written
            to[u] += obase;
        }
        double x[U][3];
        FT v[U][3], tau[U];
        uint64_t id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[u][c] = a.in.x[c][from[u]];
                v[u][c] = ((const FT *)a.in.v[c])[from[u]];
            }
            tau[u] = ((const FT *)a.in.tau)[from[u]];
            id[u] = a.in.id[from[u]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (ok[u])
                put_record<FT>(a.out, to[u], x[u], v[u], tau[u], id[u]);
    }
    for (int64_t sl = (int64_t)blockIdx.x * kSortWG + threadIdx.x; sl < a.sub_count;
         sl += (int64_t)gridDim.x * kSortWG) {
        const int sg = a.sub_first + (int)sl;
        a.out.count[sg] = a.in.count[sg];
        if (a.in.count[sg] > a.out.cap[sg])
            fl |= PM_F_DEST_OVERFLOW;
    }
    if (fl)
        flag_or(a.ws.hdr, fl);
}

// The workgroups of a launch over `work` jobs: one each up to eight a compute
// unit (of 512 threads, twice what it holds at a time), the rest in strides.
int sort_grid(int64_t work, int cus)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>(work, (int64_t)cus * 8));
}

template <typename KT, int BITS>
hipError_t sort_passes(const KArgs &a, const DSort &s, int passes, int64_t tiles, int cus,
                       hipStream_t st, int *last)
{
    const int grid = sort_grid(tiles, cus);
    hipLaunchKernelGGL((k_sort_keys<KT, 1 << BITS>), dim3(grid), dim3(kSortWG), 0, st, a, s);
    int src = 0;
    for (int p = 0; p < passes; ++p) {
        if (p)
            hipLaunchKernelGGL((k_sort_hist<KT, 1 << BITS>), dim3(grid), dim3(kSortWG), 0, st,
                               a, s, src, BITS * p);
        hipLaunchKernelGGL((k_sort_scan<1 << BITS>),
                           dim3(sort_grid((int64_t)a.sub_count << (BITS - 6), cus)),
                           dim3(64 * kScanParts), 0, st, a, s);
        hipLaunchKernelGGL((k_sort_scatter<KT, BITS>), dim3(grid), dim3(kSortWG), 0, st, a, s,
                           src, BITS * p);
        src ^= 1;
    }
    *last = src;
    return hipGetLastError();
}

}  // namespace

int sort_tile() { return kSortTile; }

hipError_t launch_sort(const KArgs &a, const DSort &s, int passes, bool mixed, int64_t tiles,
                       int cus, hipStream_t st)
{
    int src = 0;
    hipError_t e;
    if (s.wide)
        e = sort_passes<uint64_t, 8>(a, s, passes, tiles, cus, st, &src);
    else if (s.bits == 9)
        e = sort_passes<uint32_t, 9>(a, s, passes, tiles, cus, st, &src);
    else
        e = sort_passes<uint32_t, 8>(a, s, passes, tiles, cus, st, &src);
    if (e != hipSuccess)
        return e;
    const int grid = sort_grid(tiles * 2, cus);
    if (mixed)
        hipLaunchKernelGGL(k_sort_gather<float>, dim3(grid), dim3(kSortWG), 0, st, a, s, src);
    else
        hipLaunchKernelGGL(k_sort_gather<double>, dim3(grid), dim3(kSortWG), 0, st, a, s, src);
    return hipGetLastError();
}

}  // namespace pm
