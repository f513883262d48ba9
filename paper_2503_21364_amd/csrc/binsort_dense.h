// Stage 2 for frames of many pairs per primitive (splats of tens to hundreds of pixels: early training
// steps, fly-throughs, the 4K stress frame).  There a primitive is sorted with every one of its many
// tiles although its place in the depth order is the same in all of them.  Here the primitives are put
// in order once, and every tile's list is then written front to back, in its final form:
//
//   order    the primitives by (depth bits, index): chunks of 4096 sorted in LDS, then merged some at a time by
//            rank (one round up to 131 000 primitives).  The last of these launches also lays rectangles and the
//            tile test's operands out in that order; what was not binned comes last, with an empty rectangle.
//   count    a workgroup takes a bin of 4 x 4 tiles, each of its wavefronts a share ("unit") of the
//            ordered primitives.  64 rectangles at a time are tested against the bin; those that
//            meet it queue up in order, and 256 of them at a time (lane = primitive) get a mask of the 16
//            tiles they keep: all or none where a look at the whole bin decides (an inner or an outer
//            part of a large splat), else from where its ellipse crosses the rows of tiles, and the tile test at its ends.  Per tile the number kept is the
//            population count of a ballot; one atomic per wavefront and tile adds it up.  Where the workspace has the room
//            the primitives that keep a tile are left with their masks for the emit ("records").
//   scan     tile_scan_kernel, as for every frame.
//   emit     the records again, or the count's walk.  The ballots give every kept primitive its place in the tile's list,
//            behind what the units before keep there: a tile's share of the 256 is put together in LDS and
//            leaves as one run of consecutive keys and values, sorted, with no atomics and nothing left for
//            the per-tile sorts to do.  From records, runs leave in whole lines: what does not fill one waits in LDS for the next 256.
//
// Whether a frame goes this way is known on the device only, so buffers with room for such a frame pay for
// both ways.  The chunk sort and the count are therefore bodies that share the launches of the other way, count_kernel and
// count_large_kernel; only the merge rounds and the emit are launches of their own, 2 us each where they leave at once.
//
// Bound by the vector instructions of the tile tests (count) and by writing 12 bytes a
// pair (emit).  What writing costs is the lines that are not written whole: runs of 150 pairs from anywhere reach 2.4 to 3 TB/s, from
// multiples of 32 pairs on 5.4.  400 000 primitives at 3840 x 2160, 615 M pairs, 48 M records: order 0.1 ms, count 1.05, emit
// 1.87 ms (4.0 TB/s); with all 16 tiles of an undecided primitive tested count 1.26, rectangles compared a word at a time 1.09; with records but runs as they come 2.9; with the walk instead of records 3.3 (count then 0.1 less);
// counting, emitting and sorting pairs took 8.5 + 10.4 + 15.7 ms.  Tried there: bins of 8 x 8 tiles
// (a third of the tested tiles kept instead of 44 %; count 1.9 ms), testing every tile of every candidate
// (count 1.8 ms), storing each ballot's pairs as they come (emit 3.7 ms); from records one tile at a time through LDS (1.90 ms), multiples
// of 64 pairs (1.86, and half of the wavefronts), a quarter of the units (2.04, count 1.72) or twice (1.93, 1.39), cached instead of
// streaming stores (2.16; only for a unit's first and last lines, which two of them write, is cached the better one: 1.88 and 2.00).
// Lines held back on the walk: slower (3 M pairs to 110 M, 20 %), its LDS leaves three wavefronts per SIMD.
// The workspace is the alternate key buffer, which only the longest lists of the per-tile sort use.  Records take 4 bytes per
// primitive and bin of it, so buffers with room for bins / 2 pairs per primitive have them (1080p 255, 2160p 1020); bin_sort in buffers that
// have, and with the walk: 100 000 of 52 tiles at 1080p 210 us, 275; 300 000 of 62 441, 637; 400 000 of 104 at 1440p 660, 993; 200 000 of
// 558 at 2160p 945, 1244.
#ifndef LMK_GS_BINSORT_DENSE_H
#define LMK_GS_BINSORT_DENSE_H
#include "lds_sort.h"
#include "lmk_gs_internal.h"
#include "tile_test.h"

namespace lmk {

namespace {

// A frame goes this way if its pair count D is at least dense_min: the device knows D and decides.  This way
// looks at every primitive in every bin of 4 x 4 tiles, the other way at every pair, so that the line in pairs per
// primitive rises with the bins.  Even by measurement (bin_sort of one frame; splats of one size, and one in
// twenty forty times as large as the rest): 510 bins (1080p) 20 (100 000 primitives) to 36 (300 000), 900 (1440p)
// 52, 2040 (4K) 40 to 82, 8160 (8K) 110 to 280.  kDenseRatio + bins / kDenseBins is above all of these, and no
// frame gets slower; at twice the line the gain is 1.5 to 2.5x.
// Below 2^18 pairs of room a frame is too short to carry a launch that it may not need.
constexpr u32 kDenseRatio = 22, kDenseBins = 30, kDenseRatioMin = 32;
constexpr u64 kDenseMinCapacity = 1ull << 18;
constexpr u32 kDenseClass = 5;                      // entry of ScratchLayout::classes: 1 = the frame went this way

constexpr u32 kSortChunk = 4096;                            // primitives sorted in LDS by one workgroup
constexpr u32 kRankThreads = 256;
constexpr u32 kDenseThreads = 256, kDenseWaves = kDenseThreads / kWave;
constexpr u32 kSets = 4, kBatch = kSets * kWave;            // primitives of an emit batch
static_assert(kBinTiles <= 16, "masks are 16 bits wide");
// units: enough wavefronts to even out bins of very different weight, but not so few pairs each that the
// last, partly filled batch of a unit is most of its work
constexpr u32 kMaxBinUnits = 65536, kMaxUnits = 64, kUnitMin = 512, kUnitPairs = 2048, kMinWaves = 12288;

// Of one round up to kOneRound runs are merged at a time, of several up to kWays, so that a million primitives
// take two; beyond that a launch is little beside the searches, whose sum is least for few ways.
constexpr u32 kOneRound = 32, kWays = 16, kWaysMany = 8, kMany = 1u << 20;

// the units per bin that a frame of D pairs is worth
__host__ __device__ inline u64 units_worth(u64 D, u32 bins)
{
    const u64 worth = D / ((u64)bins * kUnitPairs), fill = kMinWaves / bins;     // fill the chip
    return worth < fill ? fill : worth;
}

inline u64 power(u32 base, u32 exponent)
{
    u64 p = 1;
    for (u32 k = 0; k < exponent; ++k) p *= base;
    return p;
}

// room for the records of a bin: units, which start at whole wavefronts, start at whole lines
__host__ __device__ inline size_t record_row(u32 n) { return ((size_t)n + kWave - 1) / kWave * kWave; }

// Carving of the workspace (all offsets multiples of 256 bytes).
struct DenseLayout {
    size_t ops;         // float4 [n][2]  operands of the tile test in depth order: u, v, A, B | C, rx, ry, tau
    size_t pairs0, pairs1;   // u64 [n]   depth bits << 32 | index: ping and pong of the merge rounds
    size_t rects;       // ushort4 [n]    rectangles in depth order
    size_t counts;      // u32 [bins][units][kBinTiles]
    size_t kept;        // u32 [bins][units]    number of records of a unit
    size_t records;     // u32 [bins][record_row(n)]        a unit's from its first primitive on; behind `total`, if the workspace has the room
    size_t total, with_records;
    u32 bins_x, bins, units;
    u32 chunk, chunks;  // primitives sorted in LDS at a time (the last may be fewer), and how many of them
    u32 ways, rounds;   // runs merged at a time, merge rounds: the order ends in pairs0 if even, else in pairs1
};

DenseLayout dense_layout(u32 n, u64 capacity, u32 tiles_x, u32 tiles_y)
{
    DenseLayout L;
    L.bins_x = (tiles_x + kBinEdge - 1) / kBinEdge;
    L.bins = L.bins_x * ((tiles_y + kBinEdge - 1) / kBinEdge);
    u32 units = kMaxBinUnits / (L.bins ? L.bins : 1u);
    units = units < kMaxUnits ? units : kMaxUnits;
    units = units < n / kUnitMin ? units : n / kUnitMin;
    const u64 worth = units_worth(capacity, L.bins ? L.bins : 1u);      // no frame that fits is worth more
    units = worth < units ? (u32)worth : units;
    L.units = units < kDenseWaves ? kDenseWaves : units / kDenseWaves * kDenseWaves;     // whole workgroups
    // A round costs a launch and reads and writes the composites once; what it does per run it merges is a search
    // by every primitive, in windows that are short only if the runs are of one length: ways^rounds chunks.
    L.chunks = (n + kSortChunk - 1) / kSortChunk;
    L.rounds = 0; L.ways = 1;
    if (L.chunks > 1) { L.rounds = 1; L.ways = L.chunks; }
    while (L.ways > (L.rounds == 1 ? kOneRound : n <= kMany ? kWays : kWaysMany)) {
        ++L.rounds;
        for (L.ways = 2; power(L.ways, L.rounds) < L.chunks; ++L.ways) {}
    }
    if (L.chunks > 1) L.chunks = (u32)power(L.ways, L.rounds);
    L.chunk = L.chunks ? (n + L.chunks - 1) / L.chunks : 0u;
    size_t o = 0;
    L.ops = o;    o += align256((size_t)n * 2 * sizeof(float4));
    L.pairs0 = o; o += align256((size_t)n * sizeof(u64));
    L.pairs1 = o; o += align256((size_t)n * sizeof(u64));
    L.rects = o;  o += align256((size_t)n * sizeof(ushort4));
    L.counts = o; o += align256((size_t)L.bins * L.units * kBinTiles * sizeof(u32));
    L.kept = o;   o += align256((size_t)L.bins * L.units * sizeof(u32));
    L.total = o;
    L.records = o; o += (size_t)L.bins * record_row(n) * sizeof(u32);
    L.with_records = o;
    return L;
}

__device__ __forceinline__ u32 lanes_below(u64 m)
{
    return __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u));
}

// What the kernels that carry these bodies get (by value); OneWay stands for it where the host has ruled this way out.
struct OneWay { static constexpr bool kDense = false; };
struct DenseArgs {
    static constexpr bool kDense = true;
    u64 dense_min;
    ProjParams pp;
    u32 n, bins_x, bins, units;
    u32 chunk;
    bool sorted;                // the chunk sort's order is the final one (no merge rounds)
    u64 *pairs;                 // of the chunk sort
    const u64 *ordered;         // of the last round
    ushort4 *rects; float4 *ops; u32 *counts;
    u32 *kept, *records;        // records: null if the workspace has no room for them
    const float *depth; const u32 *tiles_touched; const ushort4 *rect; const float4 *feat;
};

// ---------------------------------------------------------------- order
// Primitive v (depth bits << 32 | index; what was not binned has ~0 for depth bits and comes last) is at `pos` of
// its run; from the last launch of the order its rectangle and operands go there too.
template <bool TIGHT>
__device__ __forceinline__ void put_ordered(const DenseArgs &d, u64 *pairs, bool last, u64 pos, u64 v)
{
    pairs[pos] = v;
    if (!last) return;
    const u32 i = (u32)v;
    ushort4 r = make_ushort4(0, 0, 0, 0);
    if ((u32)(v >> 32) != ~0u) {
        r = d.rect[i];
        if (TIGHT) {
            const float4 *f = d.feat + (size_t)i * (LMK_GS_FEAT_STRIDE / 4);
            const float4 f0 = f[0], f1 = f[1];
            const TileTest t = make_tile_test(f0.x, f0.y, f0.z, f0.w, f1.x, opacity_tau(d.pp, f1.y));
            d.ops[2 * pos] = make_float4(t.u, t.v, t.A, t.B);
            d.ops[2 * pos + 1] = make_float4(t.C, t.rx, t.ry, t.tau);
        }
    }
    d.rects[pos] = r;
}

// chunk blockIdx.x, by a workgroup of THREADS; s: kSortChunk + kSortChunk / 16 composites
template <u32 THREADS, bool TIGHT>
__device__ __forceinline__ void sort_chunk(const DenseArgs &d, u64 *s)
{
    const u64 beg = (u64)blockIdx.x * d.chunk;
    if (beg >= d.n) return;
    const u32 count = d.n - beg < d.chunk ? (u32)(d.n - beg) : d.chunk;
    sort_in_lds<THREADS, kSortChunk / THREADS>(count, s, [&](u32 k) {
        const u32 i = (u32)beg + k;
        return ((u64)(d.tiles_touched[i] ? __float_as_uint(d.depth[i]) : ~0u) << 32) | (u64)i;
    });
    for (u32 k = threadIdx.x; k < count; k += THREADS) put_ordered<TIGHT>(d, d.pairs, d.sorted, beg + k, s[ts_slot(k)]);
}

// The number of elements below v among src[0 .. len), which are in order; by eight neighbouring lanes, each with a
// probe of its own per step (one lane alone needs three times the steps, a trip to memory each).
__device__ __forceinline__ u32 count_below(const u64 *src, u32 len, u64 v, u32 lane)
{
    u32 lo = 0, hi = len;
    while (__builtin_amdgcn_ballot_w64(lo < hi)) {
        const u32 step = (hi - lo + 8u) / 9u, m = lo + ((lane & 7u) + 1u) * step - 1u;
        const u64 less = __builtin_amdgcn_ballot_w64(m < hi && src[m] < v);
        const u32 c = (u32)__builtin_popcount((u32)(less >> (lane & 56u)) & 0xffu);
        const u32 next = lo + (c + 1u) * step - 1u;         // the first probe that is not below v, if one is not
        if (lo < hi) { hi = c < 8u && next < hi ? next : hi; lo += c * step; }
    }
    return lo;
}

// One merge round: sorted runs of length `run`, `ways` at a time.  An element's place is its own index plus, for
// every other run of its group, the number of smaller elements there (no two are equal).  The workgroup
// finds the window of each other run that its 256 consecutive elements fall into, and searches in windows
// staged in LDS, kAtOnce runs at a time.  All rounds, against merges of two runs at a time: 20 000 primitives
// 10 us (30), 100 000 28 (45), 300 000 48 (68), 1 M 152 (135), 3 M 451 (318): there the fewer launches make up for it
// in frames that go the other way.  Searches in memory by every lane: 100 000 50 us.
template <bool TIGHT>
__global__ __launch_bounds__(kRankThreads) void depth_rank_kernel(
    const u64 *__restrict__ src, u64 *__restrict__ dst, u64 run, u32 run_blocks, u32 ways, u32 all_runs, bool last,
    DenseArgs d, const ScratchHeader *__restrict__ header)
{
    constexpr u32 kAtOnce = 4, kWindow = 512;
    static_assert(kWays <= kOneRound && kWaysMany <= kOneRound, "s_end has room");
    __shared__ u64 s_win[kAtOnce][kWindow];
    __shared__ u32 s_end[kOneRound][2];
    if (header->dup_count < d.dense_min) return;
    const u32 tid = threadIdx.x;
    const u64 n = d.n;
    const u32 mine = blockIdx.x / run_blocks, first = mine / ways * ways;   // run_blocks workgroups per run
    const u32 runs = all_runs - first < ways ? all_runs - first : ways;     // of the group
    const u64 own = (u64)mine * run, b0 = own + (u64)(blockIdx.x % run_blocks) * kRankThreads, i = b0 + tid;
    const u64 end = own + run < n ? own + run : n;
    if (b0 >= end) return;                                                  // the same for the workgroup
    const u64 v = i < end ? src[i] : ~0ull;
    for (u32 e0 = 0; e0 < 2 * runs; e0 += kRankThreads / 8) {               // both ends of every window
        const u32 e = e0 + tid / 8;
        const u64 beg = (u64)(first + e / 2) * run, at = e & 1u ? (b0 + kRankThreads < end ? b0 + kRankThreads : end) - 1 : b0;
        const u32 len = e < 2 * runs ? (u32)(n - beg < run ? n - beg : run) : 0u;
        const u32 less = count_below(src + beg, len, src[at], tid & (kWave - 1));
        if (e < 2 * runs && (tid & 7u) == 0u) s_end[e / 2][e & 1u] = less;
    }
    __syncthreads();
    u64 pos = (u64)first * run + (i - own);
    for (u32 q0 = 0; q0 < runs; q0 += kAtOnce) {
        const u64 *win[kAtOnce];
        u32 len[kAtOnce], longest = 0;
#pragma unroll
        for (u32 j = 0; j < kAtOnce; ++j) {                         // all of this is the same for the workgroup
            const u32 q = q0 + j;
            const bool other = q < runs && first + q != mine;
            const u32 lo = other ? s_end[q][0] : 0u;
            len[j] = other ? s_end[q][1] - lo : 0u;
            longest = len[j] > longest ? len[j] : longest;
            pos += lo;
            win[j] = src + (u64)(first + q) * run + lo;
        }
        for (u32 w0 = 0; w0 < longest; w0 += kWindow) {             // once, unless the runs are very unlike
            u32 part[kAtOnce], less[kAtOnce];
#pragma unroll
            for (u32 j = 0; j < kAtOnce; ++j) {
                less[j] = 0;
                part[j] = len[j] > w0 ? (len[j] - w0 < kWindow ? len[j] - w0 : kWindow) : 0u;
                for (u32 k = tid; k < part[j]; k += kRankThreads) s_win[j][k] = win[j][w0 + k];
            }
            __syncthreads();
            const u32 most = longest - w0 < kWindow ? longest - w0 : kWindow;
            for (u32 half = 1u << (31 - __builtin_clz(most)); half > 0; half >>= 1) {
                u64 c[kAtOnce];
#pragma unroll
                for (u32 j = 0; j < kAtOnce; ++j) c[j] = s_win[j][(less[j] + half - 1) % kWindow];   // read whether it counts or not
#pragma unroll
                for (u32 j = 0; j < kAtOnce; ++j) less[j] += less[j] + half <= part[j] && c[j] < v ? half : 0u;
            }
#pragma unroll
            for (u32 j = 0; j < kAtOnce; ++j) pos += less[j];
            __syncthreads();
        }
    }
    if (i < end) put_ordered<TIGHT>(d, dst, last, pos, v);
}

// ---------------------------------------------------------------- count / emit
// What a wavefront works on: bin and unit from the grid position, the unit's share of the order.
struct UnitWork { u32 bin, unit, bx, by, beg, end; };
// ordered primitives of a unit: whole wavefronts
__host__ __device__ __forceinline__ u32 unit_share(u32 n, u32 units)
{
    const u32 rounds = (n + kWave - 1) / kWave;
    return (rounds + units - 1) / units * kWave;
}

// of the `units` that the workspace and the grid have room for, those that a frame of D pairs is worth
__host__ __device__ __forceinline__ u32 units_in_use(u64 D, u32 bins, u32 units)
{
    const u64 worth = units_worth(D, bins);
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
    const u32 per = unit_share(n, units);
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
    typedef short tiles_t __attribute__((ext_vector_type(2)));
    const tiles_t bin_beg = __builtin_bit_cast(tiles_t, w.bx | (w.by << 16)), bin_end = __builtin_bit_cast(tiles_t, (w.bx + kBinEdge) | ((w.by + kBinEdge) << 16));
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
            // x0 < bx + kBinEdge, y0 < by + kBinEdge, bx < x1, by < y1, two 16-bit differences at a time (a grid has at most 4096
            // tiles along an axis); an empty rectangle (all zero) meets nothing
            const u32 ahead = __builtin_bit_cast(u32, __builtin_bit_cast(tiles_t, (u32)r[q]) - bin_end);
            const u32 behind = __builtin_bit_cast(u32, bin_beg - __builtin_bit_cast(tiles_t, (u32)(r[q] >> 32)));
            const bool meets = (ahead & behind & 0x80008000u) == 0x80008000u;
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

// the tiles of the bin that a primitive keeps: those of its rectangle, of which only those near its ellipse are asked
template <bool TIGHT>
__device__ __forceinline__ u32 bin_mask(const Ops &p, u32 bx, u32 by)
{
    auto within = [](u32 first, u32 end, u32 from) -> uint2 {                  // of kBinEdge tiles from `from` on
        const u32 a = first > from ? first - from : 0u, b = end > from ? end - from : 0u;
        return make_uint2(a < kBinEdge ? a : kBinEdge, b < kBinEdge ? b : kBinEdge);
    };
    const uint2 cols = within(p.x0, p.x1, bx), rows = within(p.y0, p.y1, by);
    if (cols.x >= cols.y || rows.x >= rows.y) return 0u;
    const u32 rect = ((1u << cols.y) - (1u << cols.x)) * 0x1111u & ((1u << (kBinEdge * rows.y)) - (1u << (kBinEdge * rows.x)));
    if (!TIGHT) return rect;
    u32 mask, open;
    bin_tiles(p.t, bx, by, mask, open);
    mask &= rect;
    open &= rect;
    while (open) {
        const u32 tile = (u32)__builtin_ctz(open);
        open &= open - 1u;
        if (tile_kept(p.t, bx + tile % kBinEdge, by + tile / kBinEdge)) mask |= 1u << tile;
    }
    return mask;
}
static_assert(kBinEdge == 4, "rows of four bits");

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

// LDS of a wavefront: `queue` BATCH + kWave positions, masks and undecided BATCH numbers each
struct WaveSpace {
    u32 queue[kBatch + kWave];
    unsigned short mask[kBatch], open[kBatch];
};
struct CountSpace : WaveSpace { u32 records[kBatch + 2 * kWave]; };
// of the emit: a batch's pairs of two tiles; from records, also what does not fill a line of values (and two of keys) of every tile yet
constexpr u32 kLine = 32;
struct EmitSpace { WaveSpace w; u64 run[2 * kBatch]; };
struct EmitRuns { u64 run[2 * kBatch], carry[kBinTiles * kLine]; };

// A record of the count for the emit: a primitive that keeps a tile of the bin, its position in the unit's share and the mask of the
// tiles.
constexpr u32 kRecordBits = 16;
static_assert(kBinTiles <= 32 - kRecordBits, "a record is a word");

// workgroup blockIdx.x of the count: kDenseThreads threads
template <bool TIGHT>
__device__ __forceinline__ void dense_count(const DenseArgs &d, const ScratchHeader *__restrict__ header,
                                            u32 *__restrict__ tile_count, CountSpace *space)
{
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 used = units_in_use(header->dup_count, d.bins, d.units);
    const UnitWork w = unit_work(d.n, d.bins_x, d.bins, used, wv);
    if (w.bin >= d.bins) return;
    CountSpace &my = space[wv];
    u32 mine = 0;                                           // kept by tile `lane` of the bin
    const bool saved = d.records != nullptr;
    u32 *rec = saved ? d.records + (size_t)w.bin * record_row(d.n) + w.beg : nullptr;
    u32 kept_prims = 0, waiting = 0;                        // records written, and in LDS
    bin_candidates<kBatch>(d.rects, w, lane, my.queue, [&](const u32 *queued, u32 count) {
        bin_masks<TIGHT, kBatch>(queued, count, d.rects, d.ops, w.bx, w.by, lane, my.mask, my.open);
        u32 m[kSets];
#pragma unroll
        for (u32 set = 0; set < kSets; ++set) m[set] = my.mask[set * kWave + lane];
        if (saved) {
#pragma unroll
            for (u32 set = 0; set < kSets; ++set) {         // (beyond `count` the masks are zero)
                const u64 some = __builtin_amdgcn_ballot_w64(m[set] != 0u);
                if (m[set]) my.records[waiting + lanes_below(some)] = (queued[set * kWave + lane] - w.beg) | (m[set] << 16);
                waiting += (u32)__builtin_popcountll(some);
            }
            wave_fence();
            u32 out = 0;                                    // whole wavefronts of them, so that whole lines are written
            for (; out + kWave <= waiting; out += kWave) rec[kept_prims + out + lane] = my.records[out + lane];
            if (out) {
                const u32 rest = my.records[out + lane];
                wave_fence();
                my.records[lane] = rest;
                kept_prims += out;
                waiting -= out;
            }
        }
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
    if (saved) {
        if (lane < waiting) rec[kept_prims + lane] = my.records[lane];
        if (lane == 0) d.kept[(size_t)w.bin * d.units + w.unit] = kept_prims + waiting;
    }
    if (lane < kBinTiles) {
        d.counts[((size_t)w.bin * d.units + w.unit) * kBinTiles + lane] = mine;
        const u32 tx = w.bx + lane % kBinEdge, ty = w.by + lane / kBinEdge;
        if (mine && tx < d.pp.tiles_x && ty < d.pp.tiles_y) atomicAdd(&tile_count[ty * d.pp.tiles_x + tx], mine);
    }
}

// workgroup blockIdx.x of the emit: kDenseThreads threads; RECORDS: from what the count has left
template <bool TIGHT, bool RECORDS>
__device__ __forceinline__ void dense_emit(const DenseArgs &d, const ScratchHeader *__restrict__ header,
                                           const u64 *__restrict__ tile_offsets, u64 capacity,
                                           u64 *__restrict__ keys, u32 *__restrict__ vals, u64 *space)
{
    if (header->status != LMK_GS_OK) return;                // more pairs than the buffers hold: nothing is emitted
    const u32 tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const u32 used = units_in_use(header->counted, d.bins, d.units);           // those that the count had, whatever the lists add up to
    const UnitWork w = unit_work(d.n, d.bins_x, d.bins, used, wv);
    if (w.bin >= d.bins) return;
    EmitRuns &lines = reinterpret_cast<EmitRuns *>(space)[RECORDS ? wv : 0u];
    EmitSpace &walk = reinterpret_cast<EmitSpace *>(space)[RECORDS ? 0u : wv];
    WaveSpace &my = walk.w;
    u64 *const run = RECORDS ? lines.run : walk.run, *const carry = lines.carry;
    const u64 *ordered = d.ordered;
    const u32 tiles_x = d.pp.tiles_x;
    // what the units before this one keep: lane = (a quarter of them, tile), then added up
    u32 before = 0;
    const u32 *c = d.counts + (size_t)w.bin * d.units * kBinTiles + lane % kBinTiles;
#pragma unroll 4
    for (u32 k = lane / kBinTiles; k < w.unit; k += kWave / kBinTiles) before += c[(size_t)k * kBinTiles];
#pragma unroll
    for (u32 o = kBinTiles; o < kWave; o <<= 1) before += __shfl_xor(before, (int)o, 64);
    // running position of tile `lane` of the bin (the first kBinTiles lanes)
    u64 first = capacity;
    {
        const u32 tx = w.bx + lane % kBinEdge, ty = w.by + lane / kBinEdge;
        if (lane < kBinTiles && tx < tiles_x && ty < d.pp.tiles_y) first = tile_offsets[ty * tiles_x + tx] + before;
    }
    u32 next_lo = (u32)first, next_hi = (u32)(first >> 32), left = 0;
    auto position = [&](u32 tile) -> u64 {
        return ((u64)(u32)__builtin_amdgcn_readlane((int)next_hi, (int)tile) << 32) | (u64)(u32)__builtin_amdgcn_readlane((int)next_lo, (int)tile);
    };
    auto tile_id = [&](u32 tile) -> u64 { return (u64)((w.by + tile / kBinEdge) * tiles_x + w.bx + tile % kBinEdge) << 32; };
    // kBatch primitives, kSets per lane: masks of their tiles, and composites
    auto put = [&](const u32 (&m)[kSets], const u64 (&pair)[kSets]) {
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
                const u64 at = position(tile);
                const u32 old = RECORDS ? (u32)__builtin_amdgcn_readlane((int)left, (int)tile) : 0u, have = old + total[q];
                const u64 line = (at + have) & ~(u64)(kLine - 1u);
                const u32 out = !RECORDS ? have : (line > at ? (u32)(line - at) : 0u);   // then all that was left before is among them
                const u64 *const found = run + q * kBatch;
                const u64 id = tile_id(tile);
#pragma unroll
                for (u32 r = 0; r < kSets + (RECORDS ? 1u : 0u); ++r) {
                    const u32 k = r * kWave + lane;
                    if (k < out && at + k < capacity) {
                        const u64 v = RECORDS && k < old ? carry[tile * kLine + k] : found[k - old];
                        if (RECORDS && ((u32)at & (kLine - 1u))) {      // the unit's first; the same for the wavefront
                            keys[at + k] = id | (v >> 32);
                            vals[at + k] = (u32)v;
                        } else {
                            __builtin_nontemporal_store(id | (v >> 32), keys + at + k);
                            __builtin_nontemporal_store((u32)v, vals + at + k);
                        }
                    }
                }
                if constexpr (RECORDS) {
                    const u32 from = out ? out - old : 0u, to = out ? 0u : old;
                    if (from + lane < total[q] && to + lane < kLine) carry[tile * kLine + to + lane] = found[from + lane];
                }
                const u64 after = at + out;
                next_lo = lane == tile ? (u32)after : next_lo;
                next_hi = lane == tile ? (u32)(after >> 32) : next_hi;
                left = lane == tile ? have - out : left;
            }
            wave_fence();
        }
    };
    // what is left of every tile, less than a line
    auto finish = [&] {
#pragma unroll 1
        for (u32 tile = 0; tile < kBinTiles; ++tile) {
            const u64 at = position(tile) + lane;
            if (lane < (u32)__builtin_amdgcn_readlane((int)left, (int)tile) && at < capacity) {
                const u64 v = carry[tile * kLine + lane];
                keys[at] = tile_id(tile) | (v >> 32);
                vals[at] = (u32)v;
            }
        }
    };
    if constexpr (RECORDS) {
        // (the records are read two batches ahead and the composites one; beyond the end a record of no tiles)
        const u32 *rec = d.records + (size_t)w.bin * record_row(d.n) + w.beg;
        u32 count = d.kept[(size_t)w.bin * d.units + w.unit];
        count = count < w.end - w.beg ? count : w.end - w.beg;          // cannot happen: one per primitive at most
        if (count == 0u) return;
        u32 r0[kSets], r1[kSets];
        u64 c0[kSets];
        auto load = [&](u32 k0, u32 (&r)[kSets]) {
#pragma unroll
            for (u32 set = 0; set < kSets; ++set) {
                const u32 k = k0 + set * kWave + lane;
                r[set] = k < count ? rec[k] : 0u;
            }
        };
        auto fetch = [&](const u32 (&r)[kSets], u64 (&c)[kSets]) {
#pragma unroll
            for (u32 set = 0; set < kSets; ++set) c[set] = ordered[w.beg + (r[set] & ((1u << kRecordBits) - 1u))];
        };
        load(0, r0);
        load(kBatch, r1);
        fetch(r0, c0);
        for (u32 k0 = 0; k0 < count; k0 += kBatch) {
            u32 m[kSets];
            u64 pair[kSets];
#pragma unroll
            for (u32 set = 0; set < kSets; ++set) { m[set] = r0[set] >> kRecordBits; pair[set] = c0[set]; r0[set] = r1[set]; }
            fetch(r0, c0);
            load(k0 + 2u * kBatch, r1);
            put(m, pair);
        }
        finish();
    } else {
        bin_candidates<kBatch>(d.rects, w, lane, my.queue, [&](const u32 *queued, u32 count) {
            bin_masks<TIGHT, kBatch>(queued, count, d.rects, d.ops, w.bx, w.by, lane, my.mask, my.open);
            u32 m[kSets];
            u64 pair[kSets];
#pragma unroll
            for (u32 set = 0; set < kSets; ++set) {
                const u32 k = set * kWave + lane;
                m[set] = my.mask[k];
                pair[set] = k < count ? ordered[queued[k]] : 0ull;
            }
            put(m, pair);
        });
    }
}

// ---------------------------------------------------------------- host side
// The least pair count with which a frame goes this way; ~0: these buffers hold no such frame.
inline u64 dense_min_pairs(u32 n, const lmk_gs_binned &out, u32 tiles_x, u32 tiles_y)
{
    constexpr u64 kNever = ~0ull;
    if (n == 0 || out.capacity < kDenseMinCapacity) return kNever;
    if (reinterpret_cast<uintptr_t>(out.keys_alt) & 15u) return kNever;     // the workspace holds 16-byte vectors
    const DenseLayout L = dense_layout(n, out.capacity, tiles_x, tiles_y);
    const u32 ratio = kDenseRatio + L.bins / kDenseBins;
    const u64 least = (u64)(ratio > kDenseRatioMin ? ratio : kDenseRatioMin) * n;
    return L.bins <= kMaxBinUnits / kDenseWaves && least <= out.capacity && L.total <= out.capacity * sizeof(u64) ? least : kNever;
}

inline DenseArgs dense_args(const lmk_gs_projected &proj, u32 n, const ProjParams &pp, const lmk_gs_binned &out,
                            const DenseLayout &L, u64 dense_min)
{
    char *w = reinterpret_cast<char *>(out.keys_alt);
    DenseArgs d = {};
    d.dense_min = dense_min;
    d.pp = pp;
    d.n = n; d.bins_x = L.bins_x; d.bins = L.bins; d.units = L.units;
    d.chunk = L.chunk; d.sorted = L.rounds == 0;
    d.pairs = reinterpret_cast<u64 *>(w + L.pairs0);
    d.ordered = reinterpret_cast<const u64 *>(w + (L.rounds & 1u ? L.pairs1 : L.pairs0));
    d.rects = reinterpret_cast<ushort4 *>(w + L.rects);
    d.ops = reinterpret_cast<float4 *>(w + L.ops);
    d.counts = reinterpret_cast<u32 *>(w + L.counts);
    d.kept = reinterpret_cast<u32 *>(w + L.kept);
    // a frame that goes this way has dense_min pairs at least, so no unit's share is larger than that many are worth
    const bool fit = unit_share(n, units_in_use(dense_min, L.bins, L.units)) <= (1u << kRecordBits);
    d.records = fit && L.with_records <= out.capacity * sizeof(u64) ? reinterpret_cast<u32 *>(w + L.records) : nullptr;
    d.depth = proj.depth; d.tiles_touched = proj.tiles_touched;
    d.rect = reinterpret_cast<const ushort4 *>(proj.rect);
    d.feat = reinterpret_cast<const float4 *>(proj.feat);
    return d;
}

// workgroups of the count and of the emit
inline u32 dense_blocks(const DenseLayout &L) { return L.bins * (L.units / kDenseWaves); }

// the merge rounds between the launch that sorts the chunks and the one that counts
inline void launch_depth_rank(const lmk_gs_binned &out, const DenseLayout &L, const DenseArgs &d,
                              const ScratchHeader *header, hipStream_t stream)
{
    char *w = reinterpret_cast<char *>(out.keys_alt);
    u64 *pairs[2] = { reinterpret_cast<u64 *>(w + L.pairs0), reinterpret_cast<u64 *>(w + L.pairs1) };
    u64 run = L.chunk;
    for (u32 round = 0; round < L.rounds; ++round, run *= L.ways) {
        const u32 run_blocks = (u32)((run + kRankThreads - 1) / kRankThreads), runs = (u32)((d.n + run - 1) / run);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(runs * run_blocks), dim3(kRankThreads), 0, stream,
                               pairs[round & 1u], pairs[(round & 1u) ^ 1u], run, run_blocks, L.ways, runs,
                               round + 1 == L.rounds, d, header);
        };
        if (d.pp.cam.binning == 1u) go(depth_rank_kernel<true>);
        else go(depth_rank_kernel<false>);
    }
}

}  // namespace

}  // namespace lmk
#endif
