// Symmetric-heap tile copy: the pointer-based put and get of Section 3.3.2
// applied to every tile of a matrix, every emulated rank r taking part in one
// launch.  Put: rank r copies its own buffer into rank (r + shift) mod w's.
// Get: rank r copies rank (r - shift) mod w's buffer into its own.  Either
// way one release-published counter per tile lands in the destination slot,
// and the post-state is the same; what differs is which side's addresses are
// translated (the remote read of a get, the remote write of a put).
//
// Data path: HBM-bound.  A workgroup owns a run of adjacent tiles of one tile
// row, copied as one rectangle, row by row, so the memory sees long row
// segments instead of many short ones; every thread moves 16-byte chunks,
// issuing a batch of loads before the matching stores so many requests are
// in flight per wave.  Stores are written through to memory (cold copies
// measured fastest that way), so their acknowledgement is the release and the
// run's counters follow it.  Loads carry the streaming hint (kLoadStream) when
// source and destination together fill the 256 MiB memory-side cache, so that
// the next call could not find its source there anyway (see kStreamBytes).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "symtile.h"
#include "symtile_device.h"
#include "symtile_internal.h"

namespace {

using symtile::u32x4;
using symtile_host::Div;
using symtile_host::make_div;

// Workgroup shape: 16 waves of one wide workgroup keep enough loads in flight
// per CU to cover HBM latency.
#ifndef SYMTILE_COPY_THREADS
#define SYMTILE_COPY_THREADS 1024
#endif
#ifndef SYMTILE_COPY_BATCH
#define SYMTILE_COPY_BATCH 8
#endif
constexpr int kThreads = SYMTILE_COPY_THREADS;
constexpr int kBatch = SYMTILE_COPY_BATCH;   // chunks in flight per thread

// (What the rectangle kernel needs lies in the first 108 bytes, two 64-byte
// lines: kernel arguments are in host memory, and a workgroup waits for every
// line of them that it touches.)
struct CopyParams {
    const uint64_t* bases;
    uint64_t src_off, dst_off;
    int rows;                // matrix rows
    int row_chunks;          // 16-byte chunks per matrix row
    int ld_bytes;            // row stride in bytes
    int tile_r;              // tile rows
    int tile_chunks;         // 16-byte chunks per tile row
    int tiles_r;             // tile rows of the matrix
    // Rectangle runs (segs > 0): each tile row is cut into segs runs of
    // seg_tiles tiles, the first seg_more of them one more.
    int segs, seg_tiles, seg_more;
    uint32_t who;            // world, shift (in [0, world)), only_rank + 1, mode: 4 bits each
    Div by_segs, by_tiles_r;
    // A pass of the workgroup covers kThreads chunks of rectangles up to width
    // chunks wide: lg_w >= 0, 1 << lg_w chunk columns; else row-major through
    // the rectangle.
    int width, lg_w;
    Div by_width;
    uint64_t flag_off;
    int tiles_c;             // tiles per matrix row of tiles
    // Otherwise workgroup g takes the (rank, tile) items [g * per_wg, ...).
    int nitems, per_wg, ntiles;
    Div by_ntiles, by_tiles_c;

    __device__ __forceinline__ int world() const { return who & 15; }
    __device__ __forceinline__ int shift() const { return who >> 4 & 15; }
    __device__ __forceinline__ int only_rank() const { return (int)(who >> 8 & 15) - 1; }
    __device__ __forceinline__ int mode() const { return who >> 12 & 15; }
};

// Source and destination ranks of executing rank r.
__device__ __forceinline__ void copy_ranks(const CopyParams& p, int r, int& src, int& dst) {
    const int up = symtile::wrap_rank(r + p.shift(), p.world());
    const int down = symtile::wrap_rank(r - p.shift() + p.world(), p.world());
    src = (p.mode() == SYMTILE_GET) ? down : r;
    dst = (p.mode() == SYMTILE_GET) ? r : up;
}

// Copy the nrows x nchunks block at (row0, chunk0) of the matrix from rank
// src_rank to rank dst: both buffers are symmetric objects named by their
// address in rank r's heap and translated from there.  lg_w >= 0 is the tile
// verb `copy`.  Rectangles whose width is no power of two are numbered
// row-major, p.width chunks a row, so that no lane idles on a padded column;
// loads of the next batch (LB chunks a thread) are issued before the stores of
// this one (see symtile::move_tile).
template <int POLICY, int LB, int LOAD>
__device__ __forceinline__ void copy_block(const CopyParams& p, int r, int src_rank, int dst,
                                           int row0, int chunk0, int nrows, int nchunks,
                                           bool pow2) {
    const uint8_t* src = reinterpret_cast<const uint8_t*>(p.bases[r] + p.src_off) +
                         (size_t)row0 * p.ld_bytes + (size_t)chunk0 * 16;
    uint8_t* dst_local = reinterpret_cast<uint8_t*>(p.bases[r] + p.dst_off) +
                         (size_t)row0 * p.ld_bytes + (size_t)chunk0 * 16;
    symtile::TileGeom g;
    g.rows = nrows;
    g.chunks = nchunks;
    g.ld_bytes = (uint32_t)p.ld_bytes;
    g.lg_w = p.lg_w;
    if (pow2) {
        symtile::copy<POLICY, kBatch, LOAD>(src, dst_local, g, src_rank, dst, r, p.bases,
                                            threadIdx.x, kThreads);
        return;
    }
    const symtile::rsrc_t rs = symtile::tile_rsrc(src, g, r, src_rank, p.bases);
    const symtile::rsrc_t rd = symtile::tile_rsrc(dst_local, g, r, dst, p.bases);
    const int total = nrows * p.width;
    const int nb = (total + kThreads * LB - 1) / (kThreads * LB);
    u32x4 x[LB], y[LB];
    uint32_t ox[LB], oy[LB];
    auto load = [&](u32x4 (&v)[LB], uint32_t (&off)[LB], int batch) {
#pragma unroll
        for (int u = 0; u < LB; ++u) {
            const int q = (batch * LB + u) * kThreads + (int)threadIdx.x;
            const int row = p.by_width(q), c = q - row * p.width;
            off[u] = (q < total && c < nchunks) ? (uint32_t)(row * p.ld_bytes + c * 16)
                                                : symtile::kOOB;
            v[u] = symtile::buf_ld16p<LOAD>(rs, off[u], 0);
        }
    };
    auto store = [&](const u32x4 (&v)[LB], const uint32_t (&off)[LB]) {
#pragma unroll
        for (int u = 0; u < LB; ++u) symtile::buf_st16p<POLICY>(v[u], rd, off[u], 0);
    };
    load(x, ox, 0);
    int i = 0;
    for (; i + 2 < nb; i += 2) {
        load(y, oy, i + 1);
        store(x, ox);
        load(x, ox, i + 2);
        store(y, oy);
    }
    if (i + 1 < nb) {
        load(y, oy, i + 1);
        store(x, ox);
        store(y, oy);
    } else {
        store(x, ox);
    }
}

// Every tile of the run is in its destination heap before any of its
// counters moves: the stores' acknowledgement is the release.  Wave 0's lanes
// then increment the counters together (one tile per lane), rather than one
// thread issuing them one after another into the same cache lines.
template <typename F>
__device__ __forceinline__ void publish_run(const CopyParams& p, int first, int last, F&& flag_of) {
    symtile::wg_stores_done();
    if (threadIdx.x < 64) {
        symtile::release_written_through();
        for (int it = first + (int)threadIdx.x; it < last; it += 64) {
            int r, tile;
            flag_of(it, r, tile);
            int src, dst;
            copy_ranks(p, r, src, dst);
            uint32_t* flag_local = reinterpret_cast<uint32_t*>(p.bases[r] + p.flag_off) + tile;
            symtile::flag_signal(symtile::translate(flag_local, r, dst, p.bases));
        }
    }
}

// One rectangle per workgroup: run `seg` of tile row tr of rank r.  SMALL: it has
// fewer chunks than the workgroup threads, and the waves without any stay out of
// the copy (their loads outside the rectangle cost as much as others: bf16
// 65536x64, 2 ranks, 64x64 tiles 23.8 -> 18.5 us).  A kernel of its own, since the
// test costs the others 0.07 us of 4.
template <int LOAD, bool SMALL>
__global__ __launch_bounds__(kThreads) void tile_copy_kernel(const CopyParams p) {
    const int band = p.by_segs(blockIdx.x), seg = (int)blockIdx.x - band * p.segs;
    const int rr = p.by_tiles_r(band), tr = band - rr * p.tiles_r;
    const int r = p.only_rank() >= 0 ? p.only_rank() : rr;
    const int t0 = seg * p.seg_tiles + min(seg, p.seg_more);
    const int t1 = t0 + p.seg_tiles + (seg < p.seg_more ? 1 : 0);
    int src, dst;
    copy_ranks(p, r, src, dst);
    const int row0 = tr * p.tile_r, chunk0 = t0 * p.tile_chunks;
    const int nrows = min(p.tile_r, p.rows - row0);
    if (!SMALL || (int)threadIdx.x < nrows * p.width)
        copy_block<symtile::kStoreWriteThrough, kBatch, LOAD>(
            p, r, src, dst, row0, chunk0, nrows,
            min((t1 - t0) * p.tile_chunks, p.row_chunks - chunk0), p.lg_w >= 0);
    publish_run(p, t0, t1, [&](int it, int& rank, int& tile) {
        rank = r;
        tile = tr * p.tiles_c + it;
    });
}

// A run of consecutive (rank, tile) items, tile by tile: the caller's
// tiles_per_wg where it gives no rectangle.  POW2: the tile's width (lg_w >= 0).
// A kernel for each: with both copies in one loop the compiler waits for a
// tile's stores before it loads the next one (fp32 2048x2048, 8 ranks, 64x64
// tiles, 3 per workgroup: 120 -> 89 us; bf16 1500x1160, 4 ranks, 4 per
// workgroup: 20.8 -> 10.8).
template <bool POW2>
__global__ __launch_bounds__(kThreads) void tile_list_copy_kernel(const CopyParams p) {
    const int first = blockIdx.x * p.per_wg;
    const int last = min(first + p.per_wg, p.nitems);
    auto item = [&](int it, int& r, int& tile) {
        const int rr = p.by_ntiles(it);
        r = p.only_rank() >= 0 ? p.only_rank() : rr;
        tile = it - rr * p.ntiles;
    };
    for (int it = first; it < last; ++it) {
        int r, tile, src, dst;
        item(it, r, tile);
        copy_ranks(p, r, src, dst);
        const int tr = p.by_tiles_c(tile), tc = tile - tr * p.tiles_c;
        const int row0 = tr * p.tile_r, chunk0 = tc * p.tile_chunks;
        const int nrows = min(p.tile_r, p.rows - row0);
        if ((int)threadIdx.x >= nrows * p.width) continue;    // small tile: nothing for this thread
        copy_block<symtile::kStoreWriteThrough, kBatch / 2, symtile::kLoadDefault>(
            p, r, src, dst, row0, chunk0, nrows, min(p.tile_chunks, p.row_chunks - chunk0), POW2);
    }
    publish_run(p, first, last, item);
}

// Bytes read and written by a call from which its loads are streaming ones.
// fp32, 8 ranks, us a call without / with the hint, the same buffers again and
// again: 128 MiB 20.0 / 21.2, 224 MiB 38.2 / 38.5, 244 MiB 39.9 / 41.8, 256 MiB
// 44.6 / 39.9; three sets of buffers in turn: 256 MiB 48.1 / 47.0.  (On the
// stores too it costs more than it gives: 11.8 -> 15.6 on 1442x684.)
constexpr size_t kStreamBytes = size_t(256) << 20;

// Runs per tile row when the caller leaves it open.  A CU moves some 25 GB/s
// each way whatever its workgroups do, so the busiest CU sets the time: the
// count that gives it the fewest bytes, each run charged a fixed kRunBytes
// for its latency (launch, first loads, acknowledgement), the smaller count
// on a tie; one or two runs per CU are looked at, at most kThreads chunks
// wide.  Runs need not be equal (19 tiles a row used to mean one tile per
// workgroup: bf16 1500x1160, 4 ranks, 64x64 tiles 23.4 -> 6.5 us a call;
// fp32 1442x684, 8 ranks, 128x128 tiles 14.9 -> 12.0).
//
// From kHugeBytes read and written on, memory alone sets the time, and runs of 1
// KiB a row are best: the workgroups that are active together then cover whole
// rows of a few tile rows (us with the rule above -> so: fp32 8192x8192, 8 ranks,
// 128x128 tiles 715 -> 677, 64x64 767 -> 687; 16384x8192, 2 ranks, 256x256 389 ->
// 346; bf16 8192x8192, 8 ranks, 128x128 429 -> 347; at half of it some calls lose:
// fp32 8192x8192, 2 ranks, 128x128 170 -> 184).
constexpr size_t kHugeBytes = size_t(2) << 30;
constexpr int kHugeWidth = 1024 / 16;      // chunks
int choose_segs(size_t bands, int tiles_c, size_t tile_bytes, int tile_chunks, size_t cus,
                size_t call_bytes) {
    constexpr size_t kRunBytes = 32 << 10;
    if (call_bytes >= kHugeBytes) {
        const int per = std::max(1, kHugeWidth / tile_chunks);
        return (tiles_c + per - 1) / per;
    }
    const size_t widest = std::max<size_t>(1, (size_t)kThreads / tile_chunks);
    size_t best = 0, best_cost = SIZE_MAX;
    for (size_t r = 1; r <= 2; ++r) {      // runs per CU (where the tile rows are fewer)
        const size_t want = std::min<size_t>(std::max<size_t>(r * cus / bands, 1), tiles_c);
        const size_t per = std::min((tiles_c + want - 1) / want, widest);
        const size_t segs = (tiles_c + per - 1) / per;
        const size_t cost = (bands * segs + cus - 1) / cus * (per * tile_bytes + kRunBytes);
        if (cost < best_cost) {
            best_cost = cost;
            best = segs;
        }
    }
    return (int)best;
}

}  // namespace

// The checks and launch of symtile_tile_copy; with t0 and t1 set the kernel
// is launched with hipExtLaunchKernel, which records the two events as part
// of the kernel's dispatch.
static symtile_status tile_copy_launch(symtile_heap* h, size_t src_off, size_t dst_off, int rows,
                                       int cols, int ld, int dtype, int tile_r, int tile_c,
                                       int shift, int only_rank, size_t flag_off,
                                       int tiles_per_wg, int mode, symtile_stream s,
                                       hipEvent_t t0, hipEvent_t t1) {

    using symtile_host::fail;
    if (!h) return fail(SYMTILE_EINVAL, "heap is NULL");
    int esize = 0;
    if (dtype == SYMTILE_F16 || dtype == SYMTILE_BF16) esize = 2;
    else if (dtype == SYMTILE_F32) esize = 4;
    else return fail(SYMTILE_EINVAL, "unknown dtype");
    if (rows < 0 || cols < 0 || tile_r <= 0 || tile_c <= 0 || ld < cols)
        return fail(SYMTILE_EINVAL, "bad matrix or tile extents");
    if ((size_t)cols * esize % 16 || (size_t)tile_c * esize % 16 || (size_t)ld * esize % 16)
        return fail(SYMTILE_EINVAL, "cols, tile_c and ld must span multiples of 16 bytes");
    if (src_off % 16 || dst_off % 16 || flag_off % 4)
        return fail(SYMTILE_EINVAL, "offsets misaligned (16 bytes for data, 4 for flags)");
    if (only_rank >= h->world) return fail(SYMTILE_EINVAL, "only_rank out of range");
    if (tiles_per_wg < 0) return fail(SYMTILE_EINVAL, "tiles_per_wg < 0");
    if (mode != SYMTILE_PUT && mode != SYMTILE_GET)
        return fail(SYMTILE_EINVAL, "mode must be SYMTILE_PUT or SYMTILE_GET");
    if (rows == 0 || cols == 0) return SYMTILE_OK;
    const size_t ld_bytes = (size_t)ld * esize;
    const size_t span = (size_t)(rows - 1) * ld_bytes + (size_t)cols * esize;
    const int tiles_r = (rows + tile_r - 1) / tile_r;
    const int tiles_c = (cols + tile_c - 1) / tile_c;
    const size_t ntiles = (size_t)tiles_r * tiles_c;
    if (ld_bytes * (size_t)tile_r >= (size_t(1) << 31) || ntiles > INT32_MAX)
        return fail(SYMTILE_EINVAL, "a tile row band exceeds 2 GiB or too many tiles");
    if (src_off > h->slot_stride || span > h->slot_stride - src_off ||
        dst_off > h->slot_stride || span > h->slot_stride - dst_off ||
        flag_off > h->slot_stride || ntiles * 4 > h->slot_stride - flag_off)
        return fail(SYMTILE_EINVAL, "source, destination or flags exceed the slot");
    if (src_off < dst_off + span && dst_off < src_off + span)
        return fail(SYMTILE_EINVAL, "source and destination regions overlap");
    if ((flag_off < src_off + span && src_off < flag_off + ntiles * 4) ||
        (flag_off < dst_off + span && dst_off < flag_off + ntiles * 4))
        return fail(SYMTILE_EINVAL, "flags overlap the data");

    CopyParams p{};
    p.bases = h->dev_bases;
    const int up = (shift % h->world + h->world) % h->world;
    p.who = (uint32_t)h->world | (uint32_t)up << 4 | (uint32_t)(std::max(only_rank, -1) + 1) << 8 |
            (uint32_t)mode << 12;
    p.src_off = src_off;
    p.dst_off = dst_off;
    p.flag_off = flag_off;
    p.rows = rows;
    p.row_chunks = (int)((size_t)cols * esize / 16);
    p.ld_bytes = (int)ld_bytes;
    p.tile_r = tile_r;
    p.tile_chunks = (int)((size_t)std::min(tile_c, cols) * esize / 16);
    p.tiles_c = tiles_c;
    p.ntiles = (int)ntiles;
    const size_t nitems = ntiles * (only_rank >= 0 ? 1 : (size_t)h->world);
    if (nitems > INT32_MAX) return fail(SYMTILE_EINVAL, "too many tiles");
    p.nitems = (int)nitems;
    const bool automatic = tiles_per_wg == 0;
    if (automatic) {
        // the equal power-of-two runs that the stride check below is stated for
        const size_t target = (size_t)std::max(1, symtile_host::cu_count(h->device));
        size_t per = std::max<size_t>(1, (nitems + target - 1) / target);
        size_t pow2 = 1;
        while (pow2 * 2 <= per && tiles_c % (pow2 * 2) == 0) pow2 *= 2;
        tiles_per_wg = (int)pow2;
    }
    p.per_wg = tiles_per_wg;
    // Rectangle mode: runs never straddle a tile row and the run width
    // (rounded up to a power of two) fits the workgroup.
    int band_lg_w = -1;
    if (tiles_c % tiles_per_wg == 0) {
        const size_t width = (size_t)tiles_per_wg * p.tile_chunks;
        int lg = 0;
        while (((size_t)1 << lg) < width) ++lg;
        if (((size_t)1 << lg) <= (size_t)kThreads) band_lg_w = lg;
    }
    // Buffer offsets are 32-bit: a tile's rows plus the out-of-range passes
    // that complete its last batch must stay below 2 GiB (the out-of-range
    // offset marker), or an offset could wrap back into the tile.
    auto passes_fit = [&](size_t rows_per_pass) {
        return ((size_t)tile_r + rows_per_pass * kBatch) * ld_bytes < (size_t(1) << 31);
    };
    {
        size_t rows_per_pass = 0;
        if (band_lg_w >= 0)
            rows_per_pass = (size_t)kThreads >> band_lg_w;
        else if (p.tile_chunks == 16 || p.tile_chunks == 32 || p.tile_chunks == 64)
            rows_per_pass = (size_t)kThreads / p.tile_chunks;
        if (rows_per_pass && !passes_fit(rows_per_pass))
            return fail(SYMTILE_EINVAL, "row stride too large for this tile shape");
    }
    p.tiles_r = tiles_r;
    const size_t bands = (size_t)tiles_r * (only_rank >= 0 ? 1 : (size_t)h->world);
    const size_t call_bytes = 2 * (size_t)rows * cols * esize * (bands / tiles_r);
    p.segs = automatic ? choose_segs(bands, tiles_c, (size_t)tile_r * tile_c * esize, p.tile_chunks,
                                     (size_t)std::max(1, symtile_host::cu_count(h->device)),
                                     call_bytes)
             : band_lg_w >= 0 ? tiles_c / tiles_per_wg
                              : 0;
    const int run_tiles = p.segs ? (tiles_c + p.segs - 1) / p.segs : 1;
    p.seg_tiles = p.segs ? tiles_c / p.segs : 0;
    p.seg_more = p.segs ? tiles_c % p.segs : 0;
    p.width = run_tiles * p.tile_chunks;
    p.lg_w = -1;
    if ((p.width & (p.width - 1)) == 0 && p.width <= kThreads) {
        const int lg = __builtin_ctz(p.width);
        if (passes_fit((size_t)kThreads >> lg)) p.lg_w = lg;
    }
    if (p.segs) {
        p.by_segs = make_div(p.segs);
        p.by_tiles_r = make_div(tiles_r);
    } else {
        p.by_ntiles = make_div(p.ntiles);
        p.by_tiles_c = make_div(tiles_c);
    }
    if (p.lg_w < 0) p.by_width = make_div(p.width);

    int prev = -1;
    if (symtile_status st = symtile_host::set_device(h, &prev)) return st;
    const dim3 grid((unsigned)(p.segs ? bands * p.segs : (nitems + p.per_wg - 1) / p.per_wg));
    hipStream_t stream = static_cast<hipStream_t>(s);
    const bool stream_loads = call_bytes >= kStreamBytes;
    const bool small = (size_t)tile_r * p.width <= kThreads - 64;
    const void* kernel =
        !p.segs        ? p.lg_w >= 0 ? reinterpret_cast<const void*>(&tile_list_copy_kernel<true>)
                                     : reinterpret_cast<const void*>(&tile_list_copy_kernel<false>)
        : small        ? stream_loads ? reinterpret_cast<const void*>(&tile_copy_kernel<symtile::kLoadStream, true>)
                                      : reinterpret_cast<const void*>(&tile_copy_kernel<symtile::kLoadDefault, true>)
        : stream_loads ? reinterpret_cast<const void*>(&tile_copy_kernel<symtile::kLoadStream, false>)
                       : reinterpret_cast<const void*>(&tile_copy_kernel<symtile::kLoadDefault, false>);
    void* args[] = {&p};
    hipError_t e = t0 ? hipExtLaunchKernel(kernel, grid, dim3(kThreads), args, 0, stream, t0, t1, 0)
                      : hipLaunchKernel(kernel, grid, dim3(kThreads), args, 0, stream);
    if (e == hipSuccess) e = hipGetLastError();
    if (prev >= 0) (void)hipSetDevice(prev);
    if (e != hipSuccess) return symtile_host::hip_fail(e, "tile_copy_kernel launch");
    return SYMTILE_OK;
}

extern "C" symtile_status symtile_tile_copy(symtile_heap* h, size_t src_off, size_t dst_off,
                                            int rows, int cols, int ld, int dtype, int tile_r,
                                            int tile_c, int shift, int only_rank,
                                            size_t flag_off, int tiles_per_wg, int mode,
                                            symtile_stream s) {
    return tile_copy_launch(h, src_off, dst_off, rows, cols, ld, dtype, tile_r, tile_c, shift,
                            only_rank, flag_off, tiles_per_wg, mode, s, nullptr, nullptr);
}

extern "C" symtile_status symtile_tile_copy_timed(symtile_heap* h, size_t src_off,
                                                  size_t dst_off, int rows, int cols, int ld,
                                                  int dtype, int tile_r, int tile_c, int shift,
                                                  int only_rank, size_t flag_off,
                                                  int tiles_per_wg, int mode, symtile_stream s,
                                                  float* kernel_ms) {
    using symtile_host::fail;
    if (!h) return fail(SYMTILE_EINVAL, "heap is NULL");
    if (!kernel_ms) return fail(SYMTILE_EINVAL, "kernel_ms is NULL");
    *kernel_ms = 0.0f;
    int prev = -1;
    if (symtile_status st = symtile_host::set_device(h, &prev)) return st;
    struct Restore {
        int d;
        ~Restore() {
            if (d >= 0) (void)hipSetDevice(d);
        }
    } restore{prev};
    if (!h->ev_t0) SYMTILE_HIP(hipEventCreate(&h->ev_t0));
    if (!h->ev_t1) SYMTILE_HIP(hipEventCreate(&h->ev_t1));
    if (symtile_status st = tile_copy_launch(h, src_off, dst_off, rows, cols, ld, dtype, tile_r,
                                             tile_c, shift, only_rank, flag_off, tiles_per_wg,
                                             mode, s, h->ev_t0, h->ev_t1))
        return st;
    if (rows == 0 || cols == 0) return SYMTILE_OK;   // nothing launched
    SYMTILE_HIP(hipEventSynchronize(h->ev_t1));
    SYMTILE_HIP(hipEventElapsedTime(kernel_ms, h->ev_t0, h->ev_t1));
    return SYMTILE_OK;
}
