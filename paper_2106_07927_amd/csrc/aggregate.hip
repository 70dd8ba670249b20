// aggregate.hip -- the sum over paths of Eq. (sgm_path_aggr) (Sec. 2.1.2)
// from the pair slices the path pass writes (paths.hip), the choice of the
// path pass's lane layout, and its launch, gfx950.
//
// A pair slice holds, per volume element, A_r + A_-r (uint8, P2 <= 127) or
// L_r + L_-r (uint16) for one pair of opposite directions; merge_kernel forms
// S_bar = R C + sum of the uint8 slices, or the sum of the uint16 ones, for
// the four-call form.  The streamlined form sums the slices inside the
// selection pass instead (wta_lrc.hip).
#include "sgm_internal.h"

#include <algorithm>
#include <vector>

namespace sgm {
namespace {

// S_bar of the kMergeChunk elements of block lb from the pair slices: uint8
// slices hold A_r + A_-r, so S_bar = R C + sum of the R/2 slices; uint16
// slices hold L_r + L_-r, so S_bar = their sum.  Each thread sums 16 elements.
template <int NS>
__device__ __forceinline__ void merge_u8_block(const Frame& f, int lb) {
    const size_t n = (size_t)f.width * f.height * f.ndisp;
    const size_t e0 = (size_t)lb * kMergeChunk + (size_t)threadIdx.x * 16;
    const uint8_t* cost = f.cost;
    const uint8_t* slices = f.slices;
    uint16_t* agg = f.agg;
    if (e0 + 16 <= n) {
        const size_t i = e0 / 16;
        const uint4 c = reinterpret_cast<const uint4*>(cost)[i];
        uint4 a[NS];
#pragma unroll
        for (int r = 0; r < NS; ++r) a[r] = load_once16(slices + (size_t)r * f.slice_stride + 16 * i);
        uint32_t s[8];
        merge16<NS, 2 * NS>(c, a, s);
        reinterpret_cast<uint4*>(agg)[2 * i] = make_uint4(s[0], s[1], s[2], s[3]);
        reinterpret_cast<uint4*>(agg)[2 * i + 1] = make_uint4(s[4], s[5], s[6], s[7]);
    } else {
        for (size_t e = e0; e < n && e < e0 + 16; ++e) {
            uint32_t s = (uint32_t)cost[e] * (2 * NS);
            for (int r = 0; r < NS; ++r) s += slices[(size_t)r * f.slice_stride + e];
            agg[e] = (uint16_t)s;
        }
    }
}

// uint16 slices: two blocks of 8 elements a thread, so that the lanes of a load
// or store lie on end (32 consecutive bytes a lane in two accesses:
// 101 us at 1242x375, D = 128, now 82).
template <int NS>
__device__ __forceinline__ void merge_u16_block(const Frame& f, int lb) {
    const size_t n = (size_t)f.width * f.height * f.ndisp;
    const uint16_t* slices = reinterpret_cast<const uint16_t*>(f.slices);
    uint16_t* agg = f.agg;
    const size_t e0 = (size_t)lb * kMergeChunk + (size_t)threadIdx.x * 8;
    constexpr int kHalf = kMergeChunk / 2;
    if ((size_t)(lb + 1) * kMergeChunk <= n) {     // the whole chunk
        uint4 a[NS][2];
#pragma unroll
        for (int r = 0; r < NS; ++r) {
            a[r][0] = load_once16(slices + (size_t)r * f.slice_stride + e0);
            a[r][1] = load_once16(slices + (size_t)r * f.slice_stride + e0 + kHalf);
        }
        uint32_t s[8];
        wide_sum16<NS>(a, s);
        *reinterpret_cast<uint4*>(agg + e0) = make_uint4(s[0], s[1], s[2], s[3]);
        *reinterpret_cast<uint4*>(agg + e0 + kHalf) = make_uint4(s[4], s[5], s[6], s[7]);
    } else {
        for (size_t e = (size_t)lb * kMergeChunk + threadIdx.x; e < n; e += blockDim.x) {
            uint32_t s = 0;
            for (int r = 0; r < NS; ++r) s += slices[(size_t)r * f.slice_stride + e];
            agg[e] = (uint16_t)s;
        }
    }
}

// MODE: 0 / 1 = uint16 slices of 4 / 8 paths, 2 / 3 = uint8 slices of 4 / 8
template <int MODE>
__device__ __forceinline__ void merge_block(const Frame& f, int lb) {
    if constexpr (MODE == 0) merge_u16_block<2>(f, lb);
    else if constexpr (MODE == 1) merge_u16_block<4>(f, lb);
    else if constexpr (MODE == 2) merge_u8_block<2>(f, lb);
    else merge_u8_block<4>(f, lb);
}

template <int MODE>
__global__ __launch_bounds__(256) void merge_kernel(Frame f) {
    merge_block<MODE>(f, blockIdx.x);
}

int merge_mode(int npaths, int p2) { return (slices_u8(p2) ? 2 : 0) + (npaths == 8 ? 1 : 0); }

// Lane layouts (indices into kPathLayouts) of the ranges up to max_d, all with
// identical results: the variants trade waves, the length of a line's chain
// and total work.
struct LayoutClass {
    int max_d, n;
    int8_t id[6];
};
constexpr LayoutClass kLayoutClasses[] = {
    {2, 1, {0}},
    {4, 1, {1}},
    {8, 1, {2}},
    {16, 4, {3, 13, 14, 15}},
    {32, 5, {4, 16, 17, 18, 19}},
    {64, 5, {5, 6, 20, 21, 22}},
    {128, 6, {7, 8, 9, 23, 24, 25}},
    {256, 3, {10, 11, 12}},
};

const LayoutClass& layout_class(int ndisp) {
    const LayoutClass* c = kLayoutClasses;
    while (c->max_d < ndisp) ++c;
    return *c;
}

// The kernels with 16 disparities per lane do not fit two waves on a SIMD when
// D cuts a lane's disparities, so such a D has the layouts of 8 or fewer only
// (803x397, D = 100, path pass alone: 111 us against 186).
bool layout_takes(int id, int ndisp) { return kPathLayouts[id].nreg_o < 8 || ndisp % 16 == 0; }

int path_layout_id(int ndisp, int variant) {
    const LayoutClass& c = layout_class(ndisp);
    const int id = c.id[variant >= 0 && variant < c.n ? variant : 0];
    if (layout_takes(id, ndisp)) return id;
    int v = 0;
    while (!layout_takes(c.id[v], ndisp)) ++v;      // every range has one
    return c.id[v];
}

// Blocks that take `us` each, in launch order.
struct Run {
    int blocks;
    float us;
};

// How long the blocks of `runs` take: block b goes to compute unit b % 256, and
// blocks that share one cost the longest's time plus half of the others'.
// Against timed passes of 16 .. 256 disparities, 4 and 8 paths, 160x120 ..
// 1920x1080: off by 5% in the mean while memory does not bound the pass.
constexpr int kUnits = 256;
float shared_time(float sum, float longest) { return longest + 0.5f * (sum - longest); }

// Of a few runs (a frame's, on every call): what a unit holds changes only where
// a run begins, so each of these is reckoned.
float run_time_few(const Run* runs, int n) {
    float worst = 0.0f;
    for (int k = 0, first = 0; k < n; first += runs[k++].blocks) {
        float sum = 0.0f, longest = 0.0f;
        int b = first % kUnits;                        // the unit's next block
        for (int at = 0, end = 0; at < n; ++at) {
            end += runs[at].blocks;
            for (; b < end; b += kUnits) {
                sum += runs[at].us;
                longest = std::max(longest, runs[at].us);
            }
        }
        worst = std::max(worst, shared_time(sum, longest));
    }
    return worst;
}

// Of many (a batch plan may have thousands): each is dealt once, its whole rounds
// over the units as one sum, the rest block by block (4,000 pairs of one size:
// 1 ms, all of different sizes: 10 ms; reckoned as above 660 ms and more).  Not
// for a few: the 256 units cost a call 1 us.
float run_time_many(const Run* runs, int n) {
    float sum[kUnits] = {}, longest[kUnits] = {};
    float every_sum = 0.0f, every_longest = 0.0f;      // of the whole rounds, on every unit
    int unit = 0;
    for (int k = 0; k < n; ++k) {
        const int rounds = runs[k].blocks / kUnits;
        if (rounds > 0) {
            every_sum += (float)rounds * runs[k].us;
            every_longest = std::max(every_longest, runs[k].us);
        }
        for (int b = runs[k].blocks % kUnits; b > 0; --b) {
            sum[unit] += runs[k].us;
            longest[unit] = std::max(longest[unit], runs[k].us);
            unit = (unit + 1) % kUnits;
        }
    }
    float worst = 0.0f;
    for (int u = 0; u < kUnits; ++u)
        worst = std::max(worst, shared_time(sum[u] + every_sum, std::max(longest[u], every_longest)));
    return worst;
}

float run_time(const Run* runs, int n) { return n <= 4 ? run_time_few(runs, n) : run_time_many(runs, n); }

// `count` frames of one size.
struct Frames {
    int width, height, count;
};

// Microseconds of the horizontal lines of a frame, which are one chain each.
float chain_time(int width, const PathLayout& l) { return 1e-3f * (float)(width * l.ns_h); }

// How long the pass over these frames takes in a layout; `runs` has room for
// npaths / 2 of them per size.
float pass_time(const Frames* sizes, int n, int npaths, const PathLayout& l, Run* runs) {
    int m = 0;
    for (int i = 0; i < n; ++i) {
        const int w = sizes[i].width, h = sizes[i].height;
        for (int q = 0; q < npaths / 2; ++q)
            runs[m++] = {sizes[i].count * pair_blocks(q, w, h, l),
                         q == 0 ? chain_time(w, l) : 1e-3f * (float)(h * (q == 1 ? l.ns_v : l.ns_d))};
    }
    // The blocks that take longest first.  A work list starts with the blocks of
    // most steps, which is not quite the same (a diagonal step takes up to three
    // times a horizontal one): over 480 batches of small frames, reckoning in that
    // order chooses as well (-23 .. +18%, 0.1% less in the geometric mean), and
    // lists in this order run slower (0.4%; 64 pairs of 320x240, P2 = 880, 5 .. 8%)
    if (n > 1 || sizes[0].count > 1) std::sort(runs, runs + m, [](const Run& a, const Run& b) { return a.us > b.us; });
    return run_time(runs, m);
}

// The variant that pass_time puts first.
int fastest_variant(const Frames* sizes, int n, int ndisp, int npaths, Run* runs) {
    const LayoutClass& c = layout_class(ndisp);
    if (c.n == 1) return 0;
    int best = -1;
    float best_us = 0.0f;
    for (int v = 0; v < c.n; ++v) {
        if (!layout_takes(c.id[v], ndisp)) continue;
        const float us = pass_time(sizes, n, npaths, kPathLayouts[c.id[v]], runs);
        // up to D = 128 the first variant stays unless another is clearly
        // ahead: in wide frames it does better than reckoned (1242x375,
        // D = 128, 4 paths: 107, the next 117).  Mean loss against the best
        // layout over 15 sizes, byte and 16-bit slices: D = 65 .. 128 0.5 and
        // 1.0%, without this 1.2 and 2.1; 33 .. 64 0.1 and 0.4, without 0.3 and
        // 1.0; 9 .. 32 the same with and without
        if (best < 0 || us < best_us * (best == 0 && ndisp <= 128 ? 0.92f : 1.0f)) {
            best = v;
            best_us = us;
        }
    }
    return best;
}

}  // namespace

int path_variants(int ndisp) { return layout_class(ndisp).n; }

PathLayout path_layout(int ndisp, int variant) { return kPathLayouts[path_layout_id(ndisp, variant)]; }

// Variant used when none is asked for (variant < 0): the one that run_time
// puts first.  Microseconds of the pass, the former choice by pixels and
// blocks against this one: 320x240, D = 16, 4 paths 28 -> 19; 640x480, D = 32,
// 8 paths 67 -> 54; 1242x375, D = 64, 8 paths 121 -> 86; 640x480, D = 128,
// 4 paths 91 -> 67; 1024x768, D = 128, 8 paths 270 -> 227; 320x240, D = 256,
// 4 paths 49 -> 39; over 86 such sizes 13% less in the geometric mean.
int default_variant(const FrameSize* sizes, int n, int ndisp, int npaths) {
    // a batch has many frames of few sizes
    std::vector<FrameSize> sorted(sizes, sizes + n);
    std::sort(sorted.begin(), sorted.end(), [](const FrameSize& a, const FrameSize& b) {
        return a.width != b.width ? a.width < b.width : a.height < b.height;
    });
    std::vector<Frames> frames;
    for (const FrameSize& s : sorted) {
        if (!frames.empty() && frames.back().width == s.width && frames.back().height == s.height) ++frames.back().count;
        else frames.push_back({s.width, s.height, 1});
    }
    std::vector<Run> runs(frames.size() * (size_t)(npaths / 2));
    return fastest_variant(frames.data(), (int)frames.size(), ndisp, npaths, runs.data());
}

int default_variant(int width, int height, int ndisp, int npaths, int p2) {
    const long px = (long)width * height;
    const Frames size = {width, height, 1};
    Run runs[4];
    // 8 paths of the widest ranges are bound by memory
    if (ndisp > 128 && ndisp % 16 == 0 && npaths == 8) {
        // uint16 slices of large volumes and the widest ranges: eight disparities
        // per lane, one 16-byte store each, streamed to memory without
        // half-written pieces.  Whole frames against the better of the other two,
        // P2 = 880, a dozen sizes from 1200x1200 up: D = 256 2 .. 11% less, 240
        // 0 .. 9% less, 224 4% less .. 4% more, 208 1% less .. 6% more, 192 3 .. 14%
        // more; D = 256 below 300 M elements, thirty sizes: 4% less .. 8% more
        if (!slices_u8(p2) && ndisp > 208 && px * ndisp >= 300000000L) return 2;
        // In wide frames helpers, which read the cost bytes of the horizontal lines
        // once more, cost more than reckoned; without them the pass is as long as
        // the longer chain of such a line at least.  Whole frames, layout 1 against
        // 0, chain of 1 by reckoned pass of 0: 1242x375 0.84, 3 .. 9% less (P2 =
        // 880: 6% less .. 4% more); 1392x400 0.86, 9 .. 16% less (6% less .. 2%
        // more); 2048x400 0.86, even; 3000x300 0.96, 5 .. 11% more; 1600x300 0.98,
        // 5% less .. 9% more; 2048x200 1.04, 27% more; 4000x130 1.12, 36% more
        if (width > 2 * height && px >= 400000) {
            const PathLayout helped = path_layout(ndisp, 0), plain = path_layout(ndisp, 1);
            if (chain_time(width, plain) < 0.9f * pass_time(&size, 1, npaths, helped, runs)) return 1;
        }
    }
    return fastest_variant(&size, 1, ndisp, npaths, runs);
}

// Launch of the path pass for the layout `l`: the layout's kernels live in
// their own object (paths.hip, compiled per layout).
hipError_t launch_paths_any(const Frame* one, const WorkList* wl, int ndisp, int variant, int p2,
                            int nblocks, hipStream_t stream) {
    const int id = path_layout_id(ndisp, variant);
#define SGM_CASE(K)                                                                                  \
    if (id == K)                                                                                     \
        return one ? launch_paths_layout_id<K>(*one, ndisp, p2, nblocks, stream)                     \
                   : launch_paths_batch_layout_id<K>(*wl, ndisp, p2, nblocks, stream);
    SGM_PATH_LAYOUT_IDS(SGM_CASE)
#undef SGM_CASE
    return hipErrorInvalidValue;
}

int path_horizontal_blocks(int width, int height, int ndisp, int variant) {
    const PathLayout l = path_layout(ndisp, variant);
    return pair_blocks(0, width, height, l);
}

int path_blocks(int width, int height, int ndisp, int npaths, int variant) {
    const PathLayout l = path_layout(ndisp, variant);
    int nb = 0;
    for (int q = 0; q < npaths / 2; ++q) nb += pair_blocks(q, width, height, l);
    return nb;
}

// Slices start on 256-element boundaries so every vector access is aligned.
size_t aggregate_slice_elems(int width, int height, int ndisp) {
    const size_t n = (size_t)width * height * ndisp;
    return (n + 255) / 256 * 256;
}

size_t aggregate_work_bytes(int width, int height, int ndisp, int npaths, int p2) {
    return (size_t)(npaths / 2) * aggregate_slice_elems(width, height, ndisp) * (slices_u8(p2) ? 1 : 2);
}

hipError_t launch_paths(const Frame& f, hipStream_t stream) {
    const int variant = (f.variant >= 0 && f.variant < path_variants(f.ndisp))
                            ? f.variant
                            : default_variant(f.width, f.height, f.ndisp, f.npaths, f.p2);
    const int nb = path_blocks(f.width, f.height, f.ndisp, f.npaths, variant);
    return launch_paths_any(&f, nullptr, f.ndisp, variant, f.p2, nb, stream);
}

hipError_t launch_aggregate(const Frame& f, hipStream_t stream) {
    hipError_t e = launch_paths(f, stream);
    if (e != hipSuccess) return e;
    const int mb = merge_blocks((size_t)f.width * f.height * f.ndisp);
    switch (merge_mode(f.npaths, f.p2)) {
        case 0: merge_kernel<0><<<mb, 256, 0, stream>>>(f); break;
        case 1: merge_kernel<1><<<mb, 256, 0, stream>>>(f); break;
        case 2: merge_kernel<2><<<mb, 256, 0, stream>>>(f); break;
        default: merge_kernel<3><<<mb, 256, 0, stream>>>(f); break;
    }
    return hipGetLastError();
}

hipError_t launch_paths_batch(const WorkList& wl, int ndisp, int npaths, int p2, int variant,
                              hipStream_t stream) {
    (void)npaths;
    if (variant < 0 || variant >= path_variants(ndisp)) variant = 0;
    return launch_paths_any(nullptr, &wl, ndisp, variant, p2, wl.total, stream);
}

}  // namespace sgm
