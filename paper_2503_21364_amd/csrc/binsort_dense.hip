// Stage 2 for frames of many pairs per primitive (splats of tens to hundreds of pixels: early training
// steps, fly-throughs, the 4K stress frame).  There a primitive is sorted with every one of its many
// tiles although its place in the depth order is the same in all of them.  Here the primitives are put
// in order once, and every tile's list is then written front to back, in its final form:
//
//   order    the primitives by (depth bits, index): chunks of 4096 sorted in LDS, then pairwise merges
//            of 2048 outputs a workgroup.  The last of these launches also lays rectangles and the tile
//            test's operands out in that order; what was not binned comes last, with an empty rectangle.
//   count    a workgroup takes a bin of 4 x 4 tiles, each of its wavefronts a share ("unit") of the
//            ordered primitives.  64 rectangles at a time are tested against the bin; those that
//            meet it queue up in order, and 256 of them at a time (lane = primitive) get a mask of the 16
//            tiles they keep: all or none where a look at the whole bin decides (an inner or an outer
//            part of a large splat), else from the tile test.  Per tile the number kept is the
//            population count of a ballot.
//   scan     per tile over the units of its bin; then tile_scan_kernel as for every frame.
//   emit     the count walk again.  The ballots give every kept primitive its place in the tile's list:
//            a tile's share of the 256 is put together in LDS and leaves as
//            one run of consecutive keys and values, sorted, with no atomics and nothing left for the
//            per-tile sorts to do.
//
// Bound by the vector instructions of the tile tests (twice per candidate) and by writing 12 bytes a
// pair.  400 000 primitives at 3840 x 2160, 615 M pairs: order 0.1 ms, count 1.2 ms, emit 3.3 ms (2.2 TB/s),
// where counting, emitting and sorting pairs took 8.5 + 10.4 + 15.7 ms.  Tried there: bins of 8 x 8 tiles
// (a third of the tested tiles kept instead of 44 %; count 1.9 ms), testing every tile of every candidate
// (count 1.8 ms), storing each ballot's pairs as they come (emit 3.7 ms), one tile at a time through LDS
// (3.5 ms), cached instead of streaming stores (+ 0.3 ms).  The workspace is the alternate key buffer, which only the merges of the per-tile sort use.
#include "lds_sort.h"
#include "lmk_gs_internal.h"
#include "tile_test.h"

namespace lmk {

namespace {

constexpr u32 kSortThreads = 512, kSortItems = 8, kSortChunk = kSortThreads * kSortItems;    // 4096
constexpr u32 kMergeThreads = 256, kMergeItems = 8, kMergeOut = kMergeThreads * kMergeItems; // 2048
constexpr u32 kBinEdge = 4, kBinTiles = kBinEdge * kBinEdge;
constexpr u32 kDenseThreads = 256, kDenseWaves = kDenseThreads / kWave;
constexpr u32 kSets = 4, kBatch = kSets * kWave;            // primitives of an emit batch
static_assert(kBinTiles <= 16, "masks are 16 bits wide");
// units: enough wavefronts to even out bins of very different weight, but not so few pairs each that the
// last, partly filled batch of a unit is most of its work
constexpr u32 kMaxBinUnits = 65536, kMaxUnits = 64, kUnitMin = 512, kUnitPairs = 2048, kMinWaves = 12288;

// Carving of the workspace (all offsets multiples of 256 bytes).
struct DenseLayout {
    size_t ops;         // float4 [n][2]  operands of the tile test in depth order: u, v, A, B | C, rx, ry, tau
    size_t pairs0, pairs1;   // u64 [n]   depth bits << 32 | index: ping and pong of the merges
    size_t rects;       // ushort4 [n]    rectangles in depth order
    size_t counts;      // u32 [bins][units][kBinTiles]
    size_t total;
    u32 bins_x, bins, units;
    u32 rounds;         // merge rounds: the order ends in pairs0 if even, else in pairs1
};

DenseLayout dense_layout(u32 n, u32 tiles_x, u32 tiles_y)
{
    DenseLayout L;
    L.bins_x = (tiles_x + kBinEdge - 1) / kBinEdge;
    L.bins = L.bins_x * ((tiles_y + kBinEdge - 1) / kBinEdge);
    u32 units = kMaxBinUnits / (L.bins ? L.bins : 1u);
    units = units < kMaxUnits ? units : kMaxUnits;
    units = units < n / kUnitMin ? units : n / kUnitMin;
    L.units = units < kDenseWaves ? kDenseWaves : units / kDenseWaves * kDenseWaves;     // whole workgroups
    L.rounds = 0;
    for (u64 run = kSortChunk; run < n; run <<= 1) ++L.rounds;
    size_t o = 0;
    L.ops = o;    o += align256((size_t)n * 2 * sizeof(float4));
    L.pairs0 = o; o += align256((size_t)n * sizeof(u64));
    L.pairs1 = o; o += align256((size_t)n * sizeof(u64));
    L.rects = o;  o += align256((size_t)n * sizeof(ushort4));
    L.counts = o; o += align256((size_t)L.bins * L.units * kBinTiles * sizeof(u32));
    L.total = o;
    return L;
}

__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ u32 lanes_below(u64 m)
{
    return __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
}

// ---------------------------------------------------------------- order
// where the sorted order goes: the composites, and from the last launch the rectangles and operands
struct OrderOut {
    u64 *pairs;
    const u32 *tiles_touched; const ushort4 *rect; const float4 *feat;
    ushort4 *rects; float4 *ops;
};

template <bool LAST, bool TIGHT>
__device__ __forceinline__ void put_ordered(const OrderOut &out, const ProjParams &pp, u32 pos, u64 v, u32 n)
{
    out.pairs[pos] = v;
    if (!LAST) return;
    const u32 i = (u32)v;
    ushort4 r = make_ushort4(0, 0, 0, 0);
    if (i < n) {                                            // what was not binned carries no index
        r = out.rect[i];
        if (TIGHT) {
            const float4 *f = out.feat + (size_t)i * (LMK_GS_FEAT_STRIDE / 4);
            const float4 f0 = f[0], f1 = f[1];
            const TileTest t = make_tile_test(f0.x, f0.y, f0.z, f0.w, f1.x, opacity_tau(pp, f1.y));
            out.ops[2 * (size_t)pos] = make_float4(t.u, t.v, t.A, t.B);
            out.ops[2 * (size_t)pos + 1] = make_float4(t.C, t.rx, t.ry, t.tau);
        }
    }
    out.rects[pos] = r;
}

template <bool LAST, bool TIGHT>
__global__ __launch_bounds__(kSortThreads) void depth_sort_kernel(
    const float *__restrict__ depth, u32 n, ProjParams pp, OrderOut out,
    const ScratchHeader *__restrict__ header, u64 dense_min)
{
    __shared__ u64 s[kSortChunk + kSortChunk / 16];
    if (header->dup_count < dense_min) return;
    const u32 beg = blockIdx.x * kSortChunk;
    const u32 count = n - beg < kSortChunk ? n - beg : kSortChunk;
    sort_in_lds<kSortThreads, kSortItems>(count, s, [&](u32 k) {
        const u32 i = beg + k;
        return out.tiles_touched[i] ? ((u64)__float_as_uint(depth[i]) << 32) | (u64)i : ~0ull;
    });
    for (u32 k = threadIdx.x; k < count; k += kSortThreads) put_ordered<LAST, TIGHT>(out, pp, beg + k, s[ts_slot(k)], n);
}

// number of elements of A = src[a0, a1) among the first `diag` of its merge with B = src[a1, b1), by one
// wavefront: every round the lanes probe 64 evenly spaced candidates
__device__ __forceinline__ u32 wave_split(const u64 *__restrict__ src, u32 a0, u32 a1, u32 b1, u32 diag, u32 lane)
{
    const u32 lenA = a1 - a0, lenB = b1 - a1;
    u32 lo = diag > lenB ? diag - lenB : 0, hi = diag < lenA ? diag : lenA;
    while (lo < hi) {                                       // wave-uniform
        const u32 step = (hi - lo + 63) / 64;
        const u32 m = lo + (lane + 1) * step - 1;
        const bool p = m < hi && src[a0 + m] < src[a1 + (diag - 1 - m)];
        const u32 c = (u32)__builtin_popcountll(__builtin_amdgcn_ballot_w64(p));
        const u32 nhi = lo + (c + 1) * step - 1;
        hi = nhi < hi ? nhi : hi;
        lo += c * step;
    }
    return lo;
}

// one merge round over sorted runs of length `run`; workgroup = kMergeOut consecutive outputs
template <bool LAST, bool TIGHT>
__global__ __launch_bounds__(kMergeThreads) void depth_merge_kernel(
    const u64 *__restrict__ src, u32 n, u32 run, ProjParams pp, OrderOut out,
    const ScratchHeader *__restrict__ header, u64 dense_min)
{
    __shared__ u64 s[kMergeOut + kMergeOut / 16];
    __shared__ u32 s_split[2];
    if (header->dup_count < dense_min) return;
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 o = blockIdx.x * kMergeOut;
    const u64 a0w = (u64)o / (2ull * run) * (2ull * run);
    const u32 a0 = (u32)a0w;
    const u32 a1 = a0w + run < n ? (u32)(a0w + run) : n;
    const u32 b1 = a0w + 2ull * run < n ? (u32)(a0w + 2ull * run) : n;
    const u32 oe = b1 - o < kMergeOut ? b1 : o + kMergeOut;             // run is a multiple of kMergeOut
    if (wv < 2) {
        const u32 v = wave_split(src, a0, a1, b1, (wv == 0 ? o : oe) - a0, lane);
        if (lane == 0) s_split[wv] = v;
    }
    __syncthreads();
    const u32 i0 = s_split[0], la = s_split[1] - i0, total = oe - o;
    const u32 j0 = (o - a0) - i0;                           // elements of B before the segment
    for (u32 k = tid; k < total; k += kMergeThreads) s[ts_slot(k)] = src[k < la ? a0 + i0 + k : a1 + j0 + (k - la)];
    __syncthreads();
    const u32 o0 = tid * kMergeItems;
    u64 e[kMergeItems];
    if (o0 < total) merge_from_lds<kMergeItems>(s, 0u, la, total, o0, e);
    __syncthreads();
    if (o0 < total) {
#pragma unroll
        for (u32 k = 0; k < kMergeItems; ++k)
            if (o0 + k < total) s[ts_slot(o0 + k)] = e[k];
    }
    __syncthreads();
    for (u32 k = tid; k < total; k += kMergeThreads) put_ordered<LAST, TIGHT>(out, pp, o + k, s[ts_slot(k)], n);
}

// ---------------------------------------------------------------- count / emit
// What a wavefront works on: bin and unit from the grid position, the unit's share of the order.
struct UnitWork { u32 bin, unit, bx, by, beg, end; };

// of the `units` that the workspace and the grid have room for, those that this frame's pairs are worth
__device__ __forceinline__ u32 units_in_use(const ScratchHeader *__restrict__ header, u32 bins, u32 units)
{
    u64 worth = header->dup_count / ((u64)bins * kUnitPairs);
    if (worth < kMinWaves / bins) worth = kMinWaves / bins;     // fill the chip
    if (worth >= units) return units;
    return worth < kDenseWaves ? kDenseWaves : (u32)worth / kDenseWaves * kDenseWaves;
}

// The nearest primitives have the most tiles, and workgroups are dealt to the eight dies in turn.  Up to
// kByShare primitives the grid goes through all bins with one share before the next, heaviest first, and
// every die gets all shares alike (4K frame of 400 000: 3.9 ms of emitting when this was chosen; with a bin's shares next to
// each other a die has the same share of every bin and waits for the one with the nearest, 4.5 ms).  Where
// the order is larger than the dies' L2 that loses more than it gives (2 M: 1.9 instead of 1.5 ms): there a
// bin's shares follow one another.
constexpr u32 kByShare = 1u << 20;

__device__ __forceinline__ UnitWork unit_work(u32 n, u32 bins_x, u32 bins, u32 units, u32 wv)
{   // units: those in use; a workgroup beyond them gets a bin beyond `bins`
    UnitWork w;
    const u32 per_bin = units / kDenseWaves;
    const bool by_share = n <= kByShare;
    w.bin = by_share ? (blockIdx.x < bins * per_bin ? blockIdx.x % bins : bins) : blockIdx.x / per_bin;
    w.unit = (by_share ? blockIdx.x / bins : blockIdx.x % per_bin) * kDenseWaves + wv;
    w.bx = (w.bin % bins_x) * kBinEdge;
    w.by = (w.bin / bins_x) * kBinEdge;
    const u32 rounds = (n + kWave - 1) / kWave, per = (rounds + units - 1) / units * kWave;
    const u64 b = (u64)w.unit * per, e = b + per;
    w.beg = b < n ? (u32)b : n;
    w.end = e < n ? (u32)e : n;
    return w;
}

// The ordered primitives of the unit that meet its bin, BATCH at a time: g(queued, count), where
// queued[0 .. count) are their positions and count < BATCH for the last batch only.  `queue` holds
// BATCH + kWave positions.
template <u32 BATCH, class G>
__device__ __forceinline__ void bin_candidates(const ushort4 *__restrict__ rects, const UnitWork &w, u32 lane,
                                               u32 *queue, G &&g)
{
    // kAhead rounds of 64 rectangles in flight: most rounds find little, and the walk is then bound by the
    // latency of these loads (one round ahead: 0.27 ms for 300 000 primitives and the 510 bins of 1080p)
    constexpr u32 kAhead = 4;
    const u64 *r64 = reinterpret_cast<const u64 *>(rects);
    u32 queued = 0;
    u64 next[kAhead];                                       // x0 | y0 | x1 | y1, 16 bits each
#pragma unroll
    for (u32 q = 0; q < kAhead; ++q) {
        const u32 i = w.beg + q * kWave + lane;
        next[q] = i < w.end ? r64[i] : 0ull;
    }
    for (u32 i0 = w.beg; i0 < w.end; i0 += kAhead * kWave) {
        u64 r[kAhead];
#pragma unroll
        for (u32 q = 0; q < kAhead; ++q) {
            r[q] = next[q];
            const u32 i = i0 + (kAhead + q) * kWave + lane;
            next[q] = i < w.end ? r64[i] : 0ull;
        }
#pragma unroll
        for (u32 q = 0; q < kAhead; ++q) {
            const u32 lo = (u32)r[q], hi = (u32)(r[q] >> 32);
            // an empty rectangle (all zero) meets nothing
            const bool meets = (lo & 0xffffu) < w.bx + kBinEdge && (hi & 0xffffu) > w.bx &&
                               (lo >> 16) < w.by + kBinEdge && (hi >> 16) > w.by;
            const u64 m = __builtin_amdgcn_ballot_w64(meets);
            if (meets) queue[queued + lanes_below(m)] = i0 + q * kWave + lane;
            queued += (u32)__builtin_popcountll(m);         // at most BATCH - 1 + 64
            if (queued >= BATCH) {
                wave_fence();
                g(queue, BATCH);
                const u32 rest = queue[BATCH + lane];
                wave_fence();
                queue[lane] = rest;
                queued -= BATCH;
            }
        }
    }
    wave_fence();
    if (queued) g(queue, queued);
}

// What a primitive does in the whole bin, where that can be told without its tiles: bit t = tile t is
// kept.  tile_kept compares q - 4e-6 m at (a rounding of) the minimum of q over the tile's square of pixel
// centres with tau, q = A x^2 + 2 B x y + C y^2 and m = A x^2 + C y^2 about the splat's centre; its value is
// within 1e-6 m of exact.  M below bounds m over the bin, so with 2e-5 M to spare
//  - no tile is kept if the minimum over the square of the whole bin is beyond tau;
//  - every tile is kept if q at the centres of the bin's corner tiles is within tau: q is convex, so it is
//    at the centres of all others, and a tile's minimum is no larger than at its centre.
// Returns false where neither holds (and for NaN): the tiles have to be asked.
struct Ops { TileTest t; u32 x0, y0, x1, y1; };

__device__ __forceinline__ bool bin_decided(const Ops &p, u32 bx, u32 by, u32 &mask)
{
    const float kHalf = 0.5f * (float)(kBinEdge * LMK_GS_TILE) - 0.5f;              // of the bin's pixel centres
    const float kCorner = 0.5f * (float)((kBinEdge - 1) * LMK_GS_TILE);             // centres of the corner tiles
    const TileTest &t = p.t;
    const float xs = t.u - ((float)(bx * LMK_GS_TILE) + 0.5f * (float)(kBinEdge * LMK_GS_TILE));
    const float ys = t.v - ((float)(by * LMK_GS_TILE) + 0.5f * (float)(kBinEdge * LMK_GS_TILE));
    const float fx = fabsf(xs) + kHalf, fy = fabsf(ys) + kHalf;
    const float slack = 2e-5f * (t.A * fx * fx + t.C * fy * fy);
    const float ex1 = clampf3(xs, -kHalf, kHalf) - xs;
    const float ey1 = clampf3(ys + t.ry * ex1, -kHalf, kHalf) - ys;
    const float ey2 = clampf3(ys, -kHalf, kHalf) - ys;
    const float ex2 = clampf3(xs + t.rx * ey2, -kHalf, kHalf) - xs;
    const float B2 = 2.0f * t.B;
    const float q1 = t.A * ex1 * ex1 + t.C * ey1 * ey1 + B2 * ex1 * ey1;
    const float q2 = t.A * ex2 * ex2 + t.C * ey2 * ey2 + B2 * ex2 * ey2;
    const float xl = -kCorner - xs, xr = kCorner - xs, yl = -kCorner - ys, yr = kCorner - ys;
    const float al = t.A * xl * xl, ar = t.A * xr * xr, cl = t.C * yl * yl, cr = t.C * yr * yr;
    const float bl = B2 * xl, br = B2 * xr;
    const float qc = fmaxf(fmaxf(al + cl + bl * yl, ar + cl + br * yl), fmaxf(al + cr + bl * yr, ar + cr + br * yr));
    const bool none = fminf(q1, q2) - slack > t.tau;
    const bool all = qc + slack <= t.tau && p.x0 <= bx && p.x1 >= bx + kBinEdge && p.y0 <= by && p.y1 >= by + kBinEdge;
    mask = all ? (1u << kBinTiles) - 1u : 0u;
    return none || all;
}

template <bool TIGHT>
__device__ __forceinline__ Ops load_ops(u32 pos, const ushort4 *__restrict__ rects, const float4 *__restrict__ ops)
{
    Ops p;
    const u64 r = reinterpret_cast<const u64 *>(rects)[pos];
    p.x0 = (u32)r & 0xffffu; p.y0 = (u32)r >> 16; p.x1 = (u32)(r >> 32) & 0xffffu; p.y1 = (u32)(r >> 48);
    if (TIGHT) {
        const float4 a = ops[2 * (size_t)pos], b = ops[2 * (size_t)pos + 1];
        p.t.u = a.x; p.t.v = a.y; p.t.A = a.z; p.t.B = a.w; p.t.C = b.x; p.t.rx = b.y; p.t.ry = b.z; p.t.tau = b.w;
    }
    return p;
}

// the tiles of the bin that a primitive keeps, tile by tile
template <bool TIGHT>
__device__ __forceinline__ u32 bin_mask(const Ops &p, u32 bx, u32 by)
{
    u32 mask = 0;
#pragma unroll
    for (u32 j = 0; j < kBinEdge; ++j) {
        const u32 ty = by + j;
#pragma unroll
        for (u32 i = 0; i < kBinEdge; ++i) {
            const u32 tx = bx + i;
            bool keep = ty >= p.y0 && ty < p.y1 && tx >= p.x0 && tx < p.x1;
            if (TIGHT) keep = keep & tile_kept(p.t, tx, ty);
            mask |= keep ? 1u << (j * kBinEdge + i) : 0u;
        }
    }
    return mask;
}

// Masks of the queued primitives 0 .. count (count <= BATCH) to masks[0 .. BATCH): those that a look at the
// whole bin decides first, then the others, put together so that the tile tests run on full wavefronts.
// `undecided` is room for BATCH numbers.
template <bool TIGHT, u32 BATCH>
__device__ __forceinline__ void bin_masks(const u32 *queued, u32 count, const ushort4 *__restrict__ rects,
                                          const float4 *__restrict__ ops, u32 bx, u32 by, u32 lane,
                                          unsigned short *masks, unsigned short *undecided)
{
    u32 open = 0;
#pragma unroll 1
    for (u32 k0 = 0; k0 < BATCH; k0 += kWave) {
        const u32 k = k0 + lane;
        u32 mask = 0;
        bool ask = false;
        if (k < count) {
            const Ops p = load_ops<TIGHT>(queued[k], rects, ops);
            if (TIGHT) ask = !bin_decided(p, bx, by, mask);
            else mask = bin_mask<false>(p, bx, by);
        }
        masks[k] = (unsigned short)mask;
        if (TIGHT) {
            const u64 m = __builtin_amdgcn_ballot_w64(ask);
            if (ask) undecided[open + lanes_below(m)] = (unsigned short)k;
            open += (u32)__builtin_popcountll(m);
        }
    }
    wave_fence();
    if (TIGHT) {
#pragma unroll 1
        for (u32 j0 = 0; j0 < open; j0 += kWave) {
            if (j0 + lane < open) {
                const u32 k = undecided[j0 + lane];
                masks[k] = (unsigned short)bin_mask<true>(load_ops<true>(queued[k], rects, ops), bx, by);
            }
        }
        wave_fence();
    }
}

template <bool TIGHT>
__global__ __launch_bounds__(kDenseThreads) void dense_count_kernel(
    const ushort4 *__restrict__ rects, const float4 *__restrict__ ops, u32 n,
    u32 bins_x, u32 bins, u32 units, u32 *__restrict__ counts, const ScratchHeader *__restrict__ header, u64 dense_min)
{
    __shared__ u32 s_queue[kDenseWaves][kBatch + kWave];
    __shared__ unsigned short s_mask[kDenseWaves][kBatch], s_open[kDenseWaves][kBatch];
    if (header->dup_count < dense_min) return;
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 used = units_in_use(header, bins, units);
    const UnitWork w = unit_work(n, bins_x, bins, used, wv);
    if (w.bin >= bins) return;
    u32 mine = 0;                                           // kept by tile `lane` of the bin
    bin_candidates<kBatch>(rects, w, lane, s_queue[wv], [&](const u32 *queued, u32 count) {
        bin_masks<TIGHT, kBatch>(queued, count, rects, ops, w.bx, w.by, lane, s_mask[wv], s_open[wv]);
        u32 m[kSets];
#pragma unroll
        for (u32 set = 0; set < kSets; ++set) m[set] = s_mask[wv][set * kWave + lane];
#pragma unroll
        for (u32 tile = 0; tile < kBinTiles; ++tile) {
            u32 kept = 0;
#pragma unroll
            for (u32 set = 0; set < kSets; ++set)
                kept += (u32)__builtin_popcountll(__builtin_amdgcn_ballot_w64((m[set] >> tile) & 1u));
            mine += lane == tile ? kept : 0u;
        }
        wave_fence();
    });
    if (lane < kBinTiles) counts[((size_t)w.bin * units + w.unit) * kBinTiles + lane] = mine;
}

// 16 lanes per bin, lane = tile: the counts of the units become the offsets of their runs
__global__ __launch_bounds__(kWave) void dense_scan_kernel(
    u32 *__restrict__ counts, u32 bins, u32 bins_x, u32 units, u32 tiles_x, u32 tiles_y, u32 *__restrict__ tile_count,
    const ScratchHeader *__restrict__ header, u64 dense_min)
{
    if (header->dup_count < dense_min) return;
    const u32 used = units_in_use(header, bins, units);
    const u32 bin = blockIdx.x * (kWave / kBinTiles) + threadIdx.x / kBinTiles, tile = threadIdx.x % kBinTiles;
    if (bin >= bins) return;
    const u32 tx = (bin % bins_x) * kBinEdge + tile % kBinEdge, ty = (bin / bins_x) * kBinEdge + tile / kBinEdge;
    u32 *c = counts + (size_t)bin * units * kBinTiles + tile;
    u32 run = 0;
    for (u32 k0 = 0; k0 < used; k0 += kDenseWaves) {        // a multiple of kDenseWaves
        u32 v[kDenseWaves];
#pragma unroll
        for (u32 k = 0; k < kDenseWaves; ++k) v[k] = c[(size_t)(k0 + k) * kBinTiles];
#pragma unroll
        for (u32 k = 0; k < kDenseWaves; ++k) { c[(size_t)(k0 + k) * kBinTiles] = run; run += v[k]; }
    }
    if (tx < tiles_x && ty < tiles_y) tile_count[ty * tiles_x + tx] = run;
}

template <bool TIGHT>
__global__ __launch_bounds__(kDenseThreads) void dense_emit_kernel(
    const ushort4 *__restrict__ rects, const float4 *__restrict__ ops, const u64 *__restrict__ ordered,
    u32 n, u32 bins_x, u32 bins, u32 units, u32 tiles_x, u32 tiles_y,
    const u32 *__restrict__ counts, const u64 *__restrict__ tile_offsets, u64 capacity,
    u64 *__restrict__ keys, u32 *__restrict__ vals, const ScratchHeader *__restrict__ header,
    const u32 *__restrict__ classes)
{
    __shared__ u32 s_queue[kDenseWaves][kBatch + kWave];
    __shared__ unsigned short s_mask[kDenseWaves][kBatch], s_open[kDenseWaves][kBatch];
    __shared__ u64 s_run[kDenseWaves][2 * kBatch];
    if (!classes[kDenseClass] || header->status != LMK_GS_OK) return;
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 used = units_in_use(header, bins, units);
    const UnitWork w = unit_work(n, bins_x, bins, used, wv);
    if (w.bin >= bins) return;
    u64 *run = s_run[wv];
    // running position of tile `lane` of the bin (the first kBinTiles lanes)
    u64 first = capacity;
    {
        const u32 tx = w.bx + lane % kBinEdge, ty = w.by + lane / kBinEdge;
        if (lane < kBinTiles && tx < tiles_x && ty < tiles_y)
            first = tile_offsets[ty * tiles_x + tx] + counts[((size_t)w.bin * units + w.unit) * kBinTiles + lane];
    }
    u32 next_lo = (u32)first, next_hi = (u32)(first >> 32);
    bin_candidates<kBatch>(rects, w, lane, s_queue[wv], [&](const u32 *queued, u32 count) {
        bin_masks<TIGHT, kBatch>(queued, count, rects, ops, w.bx, w.by, lane, s_mask[wv], s_open[wv]);
        u32 m[kSets];
        u64 pair[kSets];
#pragma unroll
        for (u32 set = 0; set < kSets; ++set) {
            const u32 k = set * kWave + lane;
            m[set] = s_mask[wv][k];
            pair[set] = k < count ? ordered[queued[k]] : 0ull;
        }
#pragma unroll 1
        for (u32 tile0 = 0; tile0 < kBinTiles; tile0 += 2) {
            u32 total[2];
#pragma unroll
            for (u32 q = 0; q < 2; ++q) {
                total[q] = 0;
#pragma unroll
                for (u32 set = 0; set < kSets; ++set) {
                    const bool keep = ((m[set] >> (tile0 + q)) & 1u) != 0u;
                    const u64 b = __builtin_amdgcn_ballot_w64(keep);
                    if (keep) run[q * kBatch + total[q] + lanes_below(b)] = pair[set];
                    total[q] += (u32)__builtin_popcountll(b);
                }
            }
            wave_fence();
#pragma unroll
            for (u32 q = 0; q < 2; ++q) {
                const u32 tile = tile0 + q;
                const u64 at = ((u64)(u32)__builtin_amdgcn_readlane((int)next_hi, (int)tile) << 32) |
                               (u64)(u32)__builtin_amdgcn_readlane((int)next_lo, (int)tile);
                const u64 after = at + total[q];
                next_lo = lane == tile ? (u32)after : next_lo;
                next_hi = lane == tile ? (u32)(after >> 32) : next_hi;
                const u64 id = (u64)((w.by + tile / kBinEdge) * tiles_x + w.bx + tile % kBinEdge) << 32;
                u64 v[kSets];
#pragma unroll
                for (u32 r = 0; r < kSets; ++r) v[r] = run[q * kBatch + r * kWave + lane];
#pragma unroll
                for (u32 r = 0; r < kSets; ++r) {
                    const u32 k = r * kWave + lane;
                    if (k < total[q] && at + k < capacity) {
                        __builtin_nontemporal_store(id | (v[r] >> 32), keys + at + k);
                        __builtin_nontemporal_store((u32)v[r], vals + at + k);
                    }
                }
            }
            wave_fence();
        }
    });
}

}  // namespace

// ---------------------------------------------------------------- launchers
u64 dense_min_pairs(u32 n, const lmk_gs_binned &out, u32 tiles_x, u32 tiles_y)
{
    constexpr u64 kNever = ~0ull;
    if (n == 0 || out.capacity < kDenseMinCapacity) return kNever;
    if (reinterpret_cast<uintptr_t>(out.keys_alt) & 15u) return kNever;     // the workspace holds 16-byte vectors
    const DenseLayout L = dense_layout(n, tiles_x, tiles_y);
    const u32 ratio = kDenseRatio + L.bins / kDenseBins;
    const u64 least = (u64)(ratio > kDenseRatioMin ? ratio : kDenseRatioMin) * n;
    return L.bins <= kMaxBinUnits / kDenseWaves && least <= out.capacity && L.total <= out.capacity * sizeof(u64) ? least : kNever;
}

hipError_t launch_dense_count(const lmk_gs_projected &proj, u32 n, const ProjParams &pp, const lmk_gs_binned &out,
                              u32 *tile_count, const ScratchHeader *header, u64 dense_min, hipStream_t stream)
{
    const DenseLayout L = dense_layout(n, pp.tiles_x, pp.tiles_y);
    char *w = reinterpret_cast<char *>(out.keys_alt);
    u64 *pairs[2] = { reinterpret_cast<u64 *>(w + L.pairs0), reinterpret_cast<u64 *>(w + L.pairs1) };
    u32 *counts = reinterpret_cast<u32 *>(w + L.counts);
    OrderOut order = { pairs[0], proj.tiles_touched, reinterpret_cast<const ushort4 *>(proj.rect),
                       reinterpret_cast<const float4 *>(proj.feat),
                       reinterpret_cast<ushort4 *>(w + L.rects), reinterpret_cast<float4 *>(w + L.ops) };
    const bool tight = pp.cam.binning == 1u;
    auto sort = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((n + kSortChunk - 1) / kSortChunk), dim3(kSortThreads), 0, stream,
                           proj.depth, n, pp, order, header, dense_min);
    };
    if (L.rounds) sort(depth_sort_kernel<false, false>);
    else if (tight) sort(depth_sort_kernel<true, true>);
    else sort(depth_sort_kernel<true, false>);
    u32 run = kSortChunk;
    for (u32 round = 0; round < L.rounds; ++round, run <<= 1) {
        order.pairs = pairs[(round & 1u) ^ 1u];
        auto merge = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((n + kMergeOut - 1) / kMergeOut), dim3(kMergeThreads), 0, stream,
                               pairs[round & 1u], n, run, pp, order, header, dense_min);
        };
        if (round + 1 < L.rounds) merge(depth_merge_kernel<false, false>);
        else if (tight) merge(depth_merge_kernel<true, true>);
        else merge(depth_merge_kernel<true, false>);
    }
    auto count = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(L.bins * (L.units / kDenseWaves)), dim3(kDenseThreads), 0, stream,
                           order.rects, order.ops, n, L.bins_x, L.bins, L.units, counts, header, dense_min);
    };
    if (tight) count(dense_count_kernel<true>);
    else count(dense_count_kernel<false>);
    const u32 bins_per_wave = kWave / kBinTiles;
    hipLaunchKernelGGL(dense_scan_kernel, dim3((L.bins + bins_per_wave - 1) / bins_per_wave), dim3(kWave), 0, stream,
                       counts, L.bins, L.bins_x, L.units, pp.tiles_x, pp.tiles_y, tile_count, header, dense_min);
    return hipGetLastError();
}

hipError_t launch_dense_emit(u32 n, const ProjParams &pp, const lmk_gs_binned &out,
                             const ScratchHeader *header, const u32 *classes, hipStream_t stream)
{
    const DenseLayout L = dense_layout(n, pp.tiles_x, pp.tiles_y);
    const char *w = reinterpret_cast<const char *>(out.keys_alt);
    const u64 *ordered = reinterpret_cast<const u64 *>(w + (L.rounds & 1u ? L.pairs1 : L.pairs0));
    auto emit = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(L.bins * (L.units / kDenseWaves)), dim3(kDenseThreads), 0, stream,
                           reinterpret_cast<const ushort4 *>(w + L.rects), reinterpret_cast<const float4 *>(w + L.ops),
                           ordered, n, L.bins_x, L.bins, L.units, pp.tiles_x, pp.tiles_y,
                           reinterpret_cast<const u32 *>(w + L.counts), out.tile_offsets,
                           out.capacity, out.keys, out.vals, header, classes);
    };
    if (pp.cam.binning == 1u) emit(dense_emit_kernel<true>);
    else emit(dense_emit_kernel<false>);
    return hipGetLastError();
}

}  // namespace lmk
