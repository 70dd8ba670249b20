// cost.hip -- Hamming matching-cost volume, Eq. (image_matching) of Ruf et
// al. 2021 with the census Hamming distance (Sec. 2.1.1) and the 0xFF value
// for matches left of the image (Sec. 2.3.1), gfx950.
//
// A workgroup owns a run of kCostPix pixels of one row.  It stages the left
// descriptors of the run and the right descriptors of [x0 - D + 1, x0 + kCostPix)
// in LDS, so every right descriptor is read from HBM once per run.  Each thread
// produces 4 consecutive disparities for a run of PPG pixels (XOR + two v_bcnt
// each, packed into one dword), keeping the PPG + 3 right descriptors it needs
// in registers; consecutive threads write consecutive dwords, so the uint8
// volume is written fully coalesced.  Bound by that write in large frames:
// 1920x1080, D = 256: 531 MB in 120 us.  A D that is no multiple of 4 goes the
// same way with dwords at any byte (1242x375, D = 101: 18 us, a byte per thread
// took 47).  In an image narrower than a run, shorter ones: 16x4000, D = 250 with
// 32 pixels a thread 22 us, with 4 pixels 11 (a byte per thread 16).
#include "sgm_internal.h"

#include <algorithm>
#include <type_traits>

namespace sgm {
namespace {

constexpr int kMaxD = 256;

// Right descriptors in LDS: four planes, plane j % 4 holding every fourth one
// at j / 4.  The lanes of a wave read descriptors four apart (one per dword of
// costs), which are neighbours in a plane; in one row they would meet in a
// quarter of the banks (1242x375, D = 128: 19.0 us, now 17.0; 640x512 15.8,
// now 13.9).  At most 96 to a plane; 104 sets the four on banks of their own
// when a row is staged.
constexpr int kPlane = (kCostPix + kMaxD) / 4 + 8;
__device__ __forceinline__ int right_at(int j) { return (j & 3) * kPlane + (j >> 2); }

// Columns before x0 whose right descriptors a run holds: at least the D - 1 it
// needs, a multiple of 4, so that it is known which plane a thread's k-th one
// lies in.
__host__ __device__ inline int right_back(int ndisp) { return (ndisp + 3) & ~3; }

struct CostTile {
    uint64_t sl[kCostPix];
    uint64_t sr[4 * kPlane];
};

__device__ __forceinline__ int stage_row(CostTile& t, const uint64_t* __restrict__ cl,
                                         const uint64_t* __restrict__ cr, int width, int ndisp,
                                         int x0, int y) {
    const int npix = min(kCostPix, width - x0);
    const uint64_t* rowl = cl + (size_t)y * width;
    const uint64_t* rowr = cr + (size_t)y * width;
    const int back = right_back(ndisp);
    // entries [0, npix) of the left row, then [0, npix + back) of the right
    // one; all loads are issued before the first LDS write (one round trip)
    const int nl = npix, n = npix + npix + back;
    constexpr int kIt = (kCostPix + kCostPix + kMaxD + 127) / 128;   // blocks of >= 128 threads
    uint64_t v[kIt];
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int i = (int)threadIdx.x + it * (int)blockDim.x;
        v[it] = 0ull;
        if (i < nl) {
            v[it] = rowl[x0 + i];
        } else if (i < n) {
            const int x = x0 - back + (i - nl);
            if (x >= 0) v[it] = rowr[x];
        }
    }
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int i = (int)threadIdx.x + it * (int)blockDim.x;
        if (i < nl) t.sl[i] = v[it];
        else if (i < n) t.sr[right_at(i - nl)] = v[it];
    }
    __syncthreads();
    return npix;
}

// Thread (q, g) produces disparities 4q .. 4q+3 for the PPG consecutive pixels
// of group g; the right descriptors it needs, CR(x - d) for those pixels and
// disparities, are PPG + 3 consecutive ones, read once into registers and
// reused across the run.  FULL: the run holds kCostPix pixels and starts at
// x0 >= D - 1, so no pixel lies past the row's end and no disparity reaches
// left of the image (no checks).  RAGGED: D is no multiple of 4; the dwords
// start at any byte, and the last one of a pixel holds D % 4 costs.
template <int PPG, bool FULL, bool RAGGED>
__device__ __forceinline__ void cost_tile_vec4(const CostTile& t, int npix, int ndisp,
                                               uint8_t* __restrict__ out, int x0) {
    const int dwords = RAGGED ? (ndisp + 3) >> 2 : ndisp >> 2;       // dwords per pixel
    const int q = threadIdx.x % dwords;
    const int g = threadIdx.x / dwords;
    const int d0 = q * 4;
    const int p0 = g * PPG;
    if (!FULL && p0 >= npix) return;
    // CR(x - d) for pixel p is number p + back - d; the first one wanted, 1 mod 4
    // where PPG is a multiple of 4
    const int back = right_back(ndisp);
    const int rb = p0 + back - d0 - 3;
    uint64_t r[PPG + 3];
#pragma unroll
    for (int k = 0; k < PPG + 3; ++k) {
        const int at = PPG >= 4 ? ((k + 1) & 3) * kPlane + (rb >> 2) + ((k + 1) >> 2) : right_at(rb + k);
        r[k] = (FULL || rb + k < npix + back) ? t.sr[at] : 0ull;
    }
    uint8_t* o = out + p0 * ndisp + d0;
#pragma unroll
    for (int i = 0; i < PPG; ++i) {
        const int p = p0 + i;
        if (FULL || p < npix) {
            const uint64_t l = t.sl[p];
            uint32_t c0 = __popcll(l ^ r[i + 3]);
            uint32_t c1 = __popcll(l ^ r[i + 2]);
            uint32_t c2 = __popcll(l ^ r[i + 1]);
            uint32_t c3 = __popcll(l ^ r[i]);
            if (!FULL) {
                const int x = x0 + p;
                if (x < d0 + 3) {                       // some of d0..d0+3 exceed x
                    c0 = (x - d0 >= 0) ? c0 : 255u;
                    c1 = (x - d0 - 1 >= 0) ? c1 : 255u;
                    c2 = (x - d0 - 2 >= 0) ? c2 : 255u;
                    c3 = (x - d0 - 3 >= 0) ? c3 : 255u;
                }
            }
            // bytes c0..c3 (each <= 255): two shift-ors and one byte permute
            const uint32_t v = __builtin_amdgcn_perm(c2 | (c3 << 8), c0 | (c1 << 8), 0x05040100u);
            uint8_t* at = o + i * ndisp;
            if (!RAGGED) {
                *reinterpret_cast<uint32_t*>(at) = v;
            } else if (d0 + 4 <= ndisp) {
                __builtin_memcpy(at, &v, 4);
            } else {
                if (ndisp & 2) {
                    const uint16_t two = (uint16_t)v;
                    __builtin_memcpy(at, &two, 2);
                }
                if (ndisp & 1) at[ndisp & 2] = (uint8_t)(ndisp & 2 ? v >> 16 : v);
            }
        }
    }
}

template <int PPG, bool RAGGED>
__device__ __forceinline__ void cost_run_vec4(CostTile& t, const uint64_t* __restrict__ cl,
                                              const uint64_t* __restrict__ cr, int width,
                                              int ndisp, uint8_t* __restrict__ cost, int bx, int y) {
    const int x0 = bx * kCostPix;
    const int npix = stage_row(t, cl, cr, width, ndisp, x0, y);
    uint8_t* out = cost + ((size_t)y * width + x0) * ndisp;
    if (npix == kCostPix && x0 >= ndisp - 1) cost_tile_vec4<PPG, true, RAGGED>(t, npix, ndisp, out, x0);
    else cost_tile_vec4<PPG, false, RAGGED>(t, npix, ndisp, out, x0);
    __syncthreads();   // the tile is reused by the next work item
}

template <int PPG, bool RAGGED>
__global__ __launch_bounds__(256) void cost_kernel_vec4(const uint64_t* __restrict__ cl,
                                                        const uint64_t* __restrict__ cr, int width,
                                                        int ndisp, uint8_t* __restrict__ cost) {
    __shared__ CostTile t;
    cost_run_vec4<PPG, RAGGED>(t, cl, cr, width, ndisp, cost, blockIdx.x, blockIdx.y);
}

template <int PPG, bool RAGGED>
__global__ __launch_bounds__(256) void cost_batch_vec4(WorkList wl) {
    __shared__ CostTile t;
    for (int b = blockIdx.x; b < wl.total; b += gridDim.x) {
        const int fi = find_frame(wl, b);
        const Frame& f = wl.frames[fi];
        const int lb = b - wl.starts[fi];
        const int bxs = cost_blocks_x(f.width);
        cost_run_vec4<PPG, RAGGED>(t, f.census_left, f.census_right, f.width, f.ndisp, f.cost, lb % bxs,
                                   lb / bxs);
    }
}

// pixels per thread group and threads per block, for runs of `pix` pixels
// (staging a row needs 128 threads)
void vec4_shape(int ndisp, int pix, int* ppg, int* threads) {
    const int dwords = (ndisp + 3) / 4;
    *ppg = 1;
    while (dwords * ((pix + *ppg - 1) / *ppg) > 256) *ppg *= 2;        // 32 at most
    *threads = std::max(128, dwords * ((pix + *ppg - 1) / *ppg));
}

// launch(PPG, RAGGED) with the run length of D as constants; `pix` is kCostPix, or
// the width of a narrower image
template <typename Launch>
void with_shape(int ndisp, int pix, const Launch& launch) {
    int ppg, threads;
    vec4_shape(ndisp, pix, &ppg, &threads);
    auto go = [&](auto p) {
        if (ndisp & 3) launch(p, std::true_type{}, threads);
        else launch(p, std::false_type{}, threads);
    };
    if (ppg == 1) go(std::integral_constant<int, 1>{});
    else if (ppg == 2) go(std::integral_constant<int, 2>{});
    else if (ppg == 4) go(std::integral_constant<int, 4>{});
    else if (ppg == 8) go(std::integral_constant<int, 8>{});
    else if (ppg == 16) go(std::integral_constant<int, 16>{});
    else go(std::integral_constant<int, 32>{});
}

}  // namespace

hipError_t launch_cost(const Frame& f, hipStream_t stream) {
    const dim3 grid(cost_blocks_x(f.width), f.height);
    with_shape(f.ndisp, std::min(kCostPix, f.width), [&](auto ppg, auto ragged, int threads) {
        cost_kernel_vec4<ppg.value, ragged.value>
            <<<grid, threads, 0, stream>>>(f.census_left, f.census_right, f.width, f.ndisp, f.cost);
    });
    return hipGetLastError();
}

hipError_t launch_cost_batch(const WorkList& wl, int ndisp, hipStream_t stream) {
    const int grid = persistent_grid(wl.total);
    with_shape(ndisp, kCostPix, [&](auto ppg, auto ragged, int threads) {
        cost_batch_vec4<ppg.value, ragged.value><<<grid, threads, 0, stream>>>(wl);
    });
    return hipGetLastError();
}

}  // namespace sgm
