// wta_lrc.hip -- disparity selection and post-processing of Ruf et al. 2021:
// WTA (Eq. wta), the approximate right disparity map (Eq. right_disparity),
// the left-right consistency check (Eq. LR_check) and the 3x3 median
// (Sec. 2.1.3, Sec. 2.2.4), gfx950.
//
// Pass 1 (select_tile_kernel, below): a tile of one row's S_bar in LDS, formed
// there from the pair slices or read from the S_bar volume; every value
// becomes a 32-bit key (S_bar << 8) | d, so a plain minimum yields the
// smallest cost and, among equal costs, the smallest d.
// Pass 2 (check_median_kernel): per 64x4 tile plus a one-pixel halo, applies
// the LR check into LDS, then the median over the 3x3 window with 0xFFFF for
// pixels outside the image and for invalid pixels.
#include "sgm_internal.h"

namespace sgm {
namespace {

constexpr uint32_t kInf = 0xFFFFFFFFu;
constexpr uint16_t kInvalid = 0xFFFFu;

// Subpixel refinement (Sec. 2.1.3): d plus the vertex offset of the parabola
// through S_bar at d - 1, d, d + 1; no offset at either end of the range or
// when the three costs are equal.
__device__ __forceinline__ float refine(int d, uint32_t s_prev, uint32_t s_min, uint32_t s_next) {
    const float den = (float)s_prev - 2.0f * (float)s_min + (float)s_next;
    const float off = den > 0.0f ? ((float)s_prev - (float)s_next) / (2.0f * den) : 0.0f;
    return (float)d + off;
}

// ---- the tile pass -----------------------------------------------------------
// A block owns a tile of one row: 64 pixels, or 32 when D > 128, so that the
// tile holds at most 8192 volume elements.
//  (1) Its 256 threads read blocks of 16 bytes from every pair slice (and,
//      for uint8 slices, from the cost volume) -- all loads issued before any
//      is used -- and sum them into an LDS copy of S_bar, so that in the
//      streamlined form S_bar never goes to HBM.  Without FLAT (D % 16 == 0)
//      a block lies inside one pixel's vector; LDS rows are padded by 16
//      bytes, which spreads the rows over the banks.  FLAT takes any other D:
//      the volume's aligned blocks that cover the tile, laid out as they are;
//      a row of D values then starts anywhere, and D no multiple of 16
//      spreads the rows by itself.
//  (2) D^L: 256 / tile threads per pixel take the minimum key over their share
//      of the disparities, then a DPP reduction; with FINE also the refined
//      value, from the winner's two neighbours in LDS.
//  (3) D^R(q) = min_d key(q + d, d): a wave walks a quarter of the tile's
//      pixels, lane l holding the running minima T_d for q = x - d of its EPL
//      disparities.  Each pixel every T moves on by one disparity (one lane
//      shift) and takes in the pixel's key; what leaves at d = D - 1 is the
//      segment's minimum for q = x - D + 1.  The segments meet in LDS, then
//      one atomicMin per q merges the tile into the D^R key map.  Up to 32
//      disparities a wave walks two or four segments at once, GL lanes each
//      (selection from S_bar, 640x480, D = 16: 8.4 us with a thread per q,
//      10.9 with one segment a wave, now 6.8).
// Keys are built with one byte permute per value (the disparity bytes of a
// lane are constants).  The fused form is bound by the bytes it reads (NS + 1
// per element: 46 us at 1242x375, D = 128, 6.5 TB/s); the pass over S_bar was
// bound by its instructions (17 per element, D^R folded by one thread per q:
// 33 us) before (2) and (3) took this form, 24 us since.
// NS pair slices: uint8 (S_bar = 2 NS C + sum) or uint16 (S_bar = sum).
struct TileShape {
    int rs, tpx, width, ndisp, x0, npx;
    size_t row;
    __device__ __forceinline__ TileShape(const Frame& f, int bx, int y, bool flat) {
        width = f.width;
        ndisp = f.ndisp;
        tpx = fused_tile_px(ndisp);
        rs = flat ? ndisp : ndisp + 8;             // LDS row stride (uint16)
        x0 = bx * tpx;
        npx = min(tpx, width - x0);
        row = (size_t)y * width;
    }
};

// LDS of the tile pass: S_bar (rows, or the aligned blocks of a FLAT tile), 32
// spare values a FLAT tile may end in, EPL * 64 that the lanes past D read.
__host__ __device__ inline int tile_values(int ndisp) {
    return fused_tile_px(ndisp) * (ndisp + 8) + 32 + 256;
}
__host__ __device__ inline size_t tile_lds_bytes(int ndisp) {
    return (size_t)tile_values(ndisp) * sizeof(uint16_t) +
           (size_t)(fused_tile_px(ndisp) + ndisp) * sizeof(uint32_t);
}

// 16 bytes of a volume of n bytes, byte by byte where they reach past its end
__device__ __forceinline__ uint4 load16_checked(const uint8_t* __restrict__ p, size_t at, size_t n) {
    if (at + 16 <= n) return *reinterpret_cast<const uint4*>(p + at);
    uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (at + i < n) w[i >> 2] |= (uint32_t)p[at + i] << (8 * (i & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// (1): returns the LDS index of the tile's first value.  A thread's blocks are
// 16 bytes of a slice, so the lanes of a load read on end: 16 elements of uint8
// slices, 8 of uint16 ones (two loads of 32 bytes a lane: 97 us at 1242x375,
// D = 128, P2 = 880; now 77).
template <bool FLAT, int NS, bool U8>
__device__ __forceinline__ int tile_sum(uint16_t* __restrict__ sb, const Frame& f, const TileShape& t) {
    constexpr int B = U8 ? 16 : 8;                 // elements of a block
    const int ndisp = t.ndisp;
    const uint32_t e_tile = (uint32_t)(t.row + t.x0) * (uint32_t)ndisp;
    const uint32_t e_end = (uint32_t)(t.row + t.x0 + t.npx) * (uint32_t)ndisp;
    const size_t n = (size_t)f.width * f.height * ndisp;
    const uint32_t e0 = FLAT ? e_tile & ~(uint32_t)(B - 1) : e_tile;
    const int nblk = FLAT ? (int)((e_end - e0 + (uint32_t)(B - 1)) / B) : t.tpx * ndisp / B;
    // blocks past the tile's end re-read its last block and land in LDS that is
    // never read
    const uint32_t e_last = FLAT ? (e_end - 1u) & ~(uint32_t)(B - 1) : e_end - (uint32_t)B;
    // b / (blocks per row) by a product: exact for b < 1024 and at most 32 of them
    const uint32_t bpr = (uint32_t)ndisp / B;
    const uint32_t magic = FLAT ? 0u : (65536u + bpr - 1u) / bpr;
    constexpr int kPasses = (U8 ? 2 : 4) + (FLAT ? 1 : 0);     // a FLAT tile has up to two blocks more
    uint32_t sum[kPasses][B / 2];
    if constexpr (U8) {
        uint4 c[kPasses];
        uint4 a[kPasses][NS];
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            if (256 * i >= nblk) break;            // uniform
            const uint32_t e = min(e0 + 16u * (uint32_t)(threadIdx.x + 256 * i), e_last);
            c[i] = FLAT ? load16_checked(f.cost, e, n) : *reinterpret_cast<const uint4*>(f.cost + e);
#pragma unroll
            for (int r = 0; r < NS; ++r) a[i][r] = load_once16(f.slices + (size_t)r * f.slice_stride + e);
        }
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            if (256 * i >= nblk) break;
            merge16<NS, 2 * NS>(c[i], a[i], sum[i]);
        }
    } else {
        const uint16_t* slices = reinterpret_cast<const uint16_t*>(f.slices);
        uint4 a[kPasses][NS];
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            if (256 * i >= nblk) break;
            const uint32_t e = min(e0 + 8u * (uint32_t)(threadIdx.x + 256 * i), e_last);
#pragma unroll
            for (int r = 0; r < NS; ++r) {
                // NS == 1: the caller's S_bar, which ends with its last value
                if (FLAT && NS == 1 && e + 8u > n)
                    a[i][r] = load16_checked(reinterpret_cast<const uint8_t*>(slices), 2 * (size_t)e, 2 * n);
                else a[i][r] = load_once16(slices + (size_t)r * f.slice_stride + e);
            }
        }
#pragma unroll
        for (int i = 0; i < kPasses; ++i) {
            if (256 * i >= nblk) break;
#pragma unroll
            for (int k = 0; k < 4; ++k) sum[i][k] = 0;
#pragma unroll
            for (int r = 0; r < NS; ++r) {         // S_bar fits 16 bits: no carry crosses the halves
                sum[i][0] += a[i][r].x;
                sum[i][1] += a[i][r].y;
                sum[i][2] += a[i][r].z;
                sum[i][3] += a[i][r].w;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kPasses; ++i) {
        const int b = threadIdx.x + 256 * i;
        if (b < nblk) {
            int at = B * b;
            if constexpr (!FLAT) {
                const int p = (int)(((uint32_t)b * magic) >> 16);
                at = p * t.rs + B * (b - p * (int)bpr);
            }
            uint4* dst = reinterpret_cast<uint4*>(sb + at);
            dst[0] = make_uint4(sum[i][0], sum[i][1], sum[i][2], sum[i][3]);
            if constexpr (U8) dst[1] = make_uint4(sum[i][4], sum[i][5], sum[i][6], sum[i][7]);
        }
    }
    return (int)(e_tile - e0);
}

// key of the low / high half of w with the disparity in byte e of `ds`
__device__ __forceinline__ uint32_t key_lo(uint32_t w, uint32_t ds, int e) {
    return __builtin_amdgcn_perm(w, ds, 0x0c050400u | (uint32_t)e);
}
__device__ __forceinline__ uint32_t key_hi(uint32_t w, uint32_t ds, int e) {
    return __builtin_amdgcn_perm(w, ds, 0x0c070600u | (uint32_t)e);
}

template <int EPL, int GL, bool FLAT, int NS, bool U8, bool FINE>
__device__ __forceinline__ void select_tile_block(uint16_t* __restrict__ sb, const Frame& f, int bx,
                                                  int y) {
    const TileShape t(f, bx, y, FLAT);
    const int ndisp = t.ndisp, npx = t.npx;
    uint32_t* rk = reinterpret_cast<uint32_t*>(sb + tile_values(ndisp));   // key of q = x0 - D + 1 + i
    const int nq = npx + ndisp - 1;
    for (int i = threadIdx.x; i < nq; i += 256) rk[i] = kInf;
    const int first = tile_sum<FLAT, NS, U8>(sb, f, t);
    __syncthreads();

    // (2) D^L
    {
        constexpr int tpp = EPL == 4 ? 8 : 4;      // threads per pixel
        const int p = threadIdx.x / tpp, part = threadIdx.x % tpp;
        const uint16_t* src = sb + first + p * t.rs;
        uint32_t best = kInf;
        if (p < npx) {
            if constexpr (FLAT) {
                for (int d = part; d < ndisp; d += tpp) best = min(best, ((uint32_t)src[d] << 8) | (uint32_t)d);
            } else {
                // eight values a time: d = 8 c .. 8 c + 7 for c = part, part + tpp, ..
                uint32_t ds = 0x03020100u + (uint32_t)(8 * part) * 0x01010101u;
                for (int c = part; c < (ndisp >> 3); c += tpp) {
                    const uint4 w = *reinterpret_cast<const uint4*>(src + 8 * c);
                    const uint32_t dt = ds + 0x04040404u;
                    uint32_t k = min(min(key_lo(w.x, ds, 0), key_hi(w.x, ds, 1)),
                                     min(key_lo(w.y, ds, 2), key_hi(w.y, ds, 3)));
                    k = min(k, min(key_lo(w.z, dt, 0), key_hi(w.z, dt, 1)));
                    best = min(best, min(k, min(key_lo(w.w, dt, 2), key_hi(w.w, dt, 3))));
                    ds += (uint32_t)(8 * tpp) * 0x01010101u;
                }
            }
        }
        best = min(best, dpp<kDppQuadSwap1>(kInf, best));
        best = min(best, dpp<kDppQuadSwap2>(kInf, best));
        if constexpr (tpp == 8) best = min(best, dpp<kDppRowHalfMirror>(kInf, best));
        if (part == 0 && p < npx) {
            const int d = (int)(best & 0xFFu);
            f.disp_left[t.row + t.x0 + p] = (uint16_t)d;
            if constexpr (FINE) {
                float v = (float)d;
                if (d > 0 && d < ndisp - 1) v = refine(d, src[d - 1], best >> 8, src[d + 1]);
                f.fine_left[t.row + t.x0 + p] = v;
            }
        }
    }

    if (!f.right_keys) {                           // D^L alone is asked for
        __syncthreads();
        return;
    }

    // (3) D^R
    if constexpr (GL < 64) {
        constexpr int kSeg = kFusedTile / (4 * (64 / GL));       // pixels per group of lanes
        const int d = threadIdx.x % GL;
        const int s0 = (int)threadIdx.x / GL * kSeg, s1 = min(npx, s0 + kSeg);
        const uint32_t off = d < ndisp ? 0u : kInf;
        const uint16_t* src = sb + first + s0 * t.rs + d;
        uint32_t T = kInf, exits[kSeg];                          // exits: of the lane d = D - 1
#pragma unroll
        for (int i = 0; i < kSeg; ++i) {
            const uint32_t key = ((uint32_t)src[i * t.rs] << 8) | (uint32_t)d | off;
            uint32_t carry;
            if constexpr (GL == 16) {
                carry = dpp<kDppRowShr1>(kInf, T);
            } else {
                carry = (uint32_t)__builtin_amdgcn_update_dpp((int)kInf, (int)T, 0x138, 0xF, 0xF, false);
                carry = d == 0 ? kInf : carry;
            }
            T = s0 + i < s1 ? min(carry, key) : T;
            exits[i] = T;
        }
        if (s0 < s1) {
            if (d == ndisp - 1) {
#pragma unroll
                for (int i = 0; i < kSeg; ++i)
                    if (s0 + i < s1) atomicMin(&rk[s0 + i], exits[i]);
            } else if (d < ndisp) {
                atomicMin(&rk[s1 - 1 - d + ndisp - 1], T);
            }
        }
    } else {
        const int lane = threadIdx.x & 63;
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        constexpr int kSeg = EPL == 4 ? 8 : 16;    // pixels per wave
        const int s0 = wave * kSeg, s1 = min(npx, s0 + kSeg);
        if (s0 < s1) {
            const int d0 = lane * EPL;
            const uint32_t ds = (uint32_t)d0 * 0x01010101u + 0x03020100u;
            uint32_t off_d[EPL];                   // all ones for the disparities past D
#pragma unroll
            for (int e = 0; e < EPL; ++e) off_d[e] = d0 + e < ndisp ? 0u : kInf;
            const int last_lane = (ndisp - 1) / EPL, last_e = (ndisp - 1) % EPL;
            uint32_t T[EPL];
#pragma unroll
            for (int e = 0; e < EPL; ++e) T[e] = kInf;
            uint32_t done = kInf;                  // lane i: what left at pixel s0 + i
            const uint16_t* src = sb + first + s0 * t.rs + d0;
#pragma unroll 4
            for (int i = 0; i < s1 - s0; ++i, src += t.rs) {
                uint32_t w[(EPL + 1) / 2];
                if constexpr (FLAT || EPL == 1) {
#pragma unroll
                    for (int k = 0; k < (EPL + 1) / 2; ++k)
                        w[k] = (uint32_t)src[2 * k] | (EPL > 1 ? (uint32_t)src[EPL > 1 ? 2 * k + 1 : 0] << 16 : 0u);
                } else if constexpr (EPL == 2) {
                    w[0] = *reinterpret_cast<const uint32_t*>(src);
                } else {
                    const uint2 v = *reinterpret_cast<const uint2*>(src);
                    w[0] = v.x;
                    w[1] = v.y;
                }
                uint32_t key[EPL];
#pragma unroll
                for (int e = 0; e < EPL; ++e)
                    key[e] = ((e & 1) ? key_hi(w[e >> 1], ds, e) : key_lo(w[e >> 1], ds, e)) | off_d[e];
                const uint32_t carry =
                    (uint32_t)__builtin_amdgcn_update_dpp((int)kInf, (int)T[EPL - 1], 0x138, 0xF, 0xF, false);
#pragma unroll
                for (int e = EPL - 1; e >= 1; --e) T[e] = min(T[e - 1], key[e]);
                T[0] = min(carry, key[0]);
                uint32_t out = T[0];
                if constexpr (EPL >= 2) out = last_e == 1 ? T[1] : out;
                if constexpr (EPL == 4) out = last_e == 2 ? T[2] : last_e == 3 ? T[3] : out;
                const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)out, last_lane);
                done = lane == i ? v : done;
            }
            // q index of pixel s0 + i's exit: s0 + i; of T_d at the segment's
            // end: (s1 - 1 - d) + D - 1
            if (lane < s1 - s0) atomicMin(&rk[s0 + lane], done);
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                if (d0 + e < ndisp - 1) atomicMin(&rk[s1 - 1 - (d0 + e) + ndisp - 1], T[e]);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nq; i += 256) {
        const int q = t.x0 - ndisp + 1 + i;
        const uint32_t k = rk[i];
        if (q >= 0 && k != kInf) atomicMin(&f.right_keys[t.row + q], k);
    }
    __syncthreads();   // the LDS tile is reused by the next work item
}

template <int EPL, int GL, bool FLAT, int NS, bool U8, bool FINE>
__global__ __launch_bounds__(256) void select_tile_kernel(Frame f) {
    extern __shared__ __align__(16) uint16_t sb[];
    select_tile_block<EPL, GL, FLAT, NS, U8, FINE>(sb, f, blockIdx.x, blockIdx.y);
}

template <int EPL, int GL, bool FLAT, int NS, bool U8>
__global__ __launch_bounds__(256) void select_tile_batch_kernel(WorkList wl) {
    extern __shared__ __align__(16) uint16_t sb[];
    for (int b = blockIdx.x; b < wl.total; b += gridDim.x) {
        const int fi = find_frame(wl, b);
        const Frame& f = wl.frames[fi];
        const int lb = b - wl.starts[fi];
        const int bxs = fused_blocks_x(f.width, f.ndisp);
        select_tile_block<EPL, GL, FLAT, NS, U8, false>(sb, f, lb % bxs, lb / bxs);
    }
}

// D^R keys start at "no candidate" (all ones).
__device__ __forceinline__ void fill_keys_block(const Frame& f, int lb) {
    const size_t n = (size_t)f.width * f.height;
    const size_t e0 = (size_t)lb * kFillChunk;
    for (size_t e = e0 + threadIdx.x; e < n && e < e0 + kFillChunk; e += blockDim.x) f.right_keys[e] = kInf;
}

__global__ __launch_bounds__(256) void fill_keys_kernel(Frame f) { fill_keys_block(f, blockIdx.x); }

__global__ __launch_bounds__(256) void fill_keys_batch_kernel(WorkList wl) {
    for (int b = blockIdx.x; b < wl.total; b += gridDim.x) {
        const int fi = find_frame(wl, b);
        fill_keys_block(wl.frames[fi], b - wl.starts[fi]);
    }
}

// Median of nine by the first five passes of a bubble-sort network (App. F).
__device__ __forceinline__ uint32_t median9(uint32_t v[9]) {
#pragma unroll
    for (int pass = 0; pass < 5; ++pass) {
#pragma unroll
        for (int i = 0; i < 8 - pass; ++i) {
            const uint32_t lo = min(v[i], v[i + 1]);
            const uint32_t hi = max(v[i], v[i + 1]);
            v[i] = lo;
            v[i + 1] = hi;
        }
    }
    return v[4];
}

constexpr int kTW = kMedianTileW, kTH = kMedianTileH;

struct MedianTile {
    uint16_t v[(kTH + 2) * (kTW + 2)];
};

// D^R of pixel (xr, row): from the key map of the approximate D^R, or, for the
// exact check, from the disparity map of the swapped, flipped pair.
struct RightSource {
    const uint32_t* keys;            // approximate: key & 0xFF
    const uint16_t* flipped;         // exact: flipped[row][width - 1 - xr]
    __device__ __forceinline__ int at(size_t row, int xr, int width) const {
        if (flipped) return flipped[row + (width - 1 - xr)];
        return (int)(keys[row + xr] & 0xFFu);
    }
};

__device__ __forceinline__ void check_median_block(MedianTile& mt, const uint16_t* __restrict__ disp_left,
                                                   RightSource rs, int width, int height,
                                                   int tolerance, int median,
                                                   uint16_t* __restrict__ disp,
                                                   uint16_t* __restrict__ disp_right, int bx, int by) {
    uint16_t* tile = mt.v;
    const int x0 = bx * kTW, y0 = by * kTH;
    for (int i = threadIdx.x; i < (kTH + 2) * (kTW + 2); i += 256) {
        const int ly = i / (kTW + 2), lx = i - ly * (kTW + 2);
        const int gx = x0 + lx - 1, gy = y0 + ly - 1;
        uint16_t v = kInvalid;
        if (gx >= 0 && gx < width && gy >= 0 && gy < height) {
            const size_t row = (size_t)gy * width;
            const int dl = disp_left[row + gx];
            v = (uint16_t)dl;
            if (tolerance >= 0) {
                const int xr = gx - dl;
                v = kInvalid;
                if (xr >= 0) {
                    const int dr = rs.at(row, xr, width);
                    const int diff = dl > dr ? dl - dr : dr - dl;
                    if (diff <= tolerance) v = (uint16_t)dl;
                }
            }
        }
        tile[i] = v;
    }
    __syncthreads();
    const int tx = threadIdx.x & (kTW - 1), ty = threadIdx.x / kTW;
    const int gx = x0 + tx, gy = y0 + ty;
    if (gx < width && gy < height) {
        const uint16_t* c = &tile[(ty + 1) * (kTW + 2) + tx + 1];
        uint16_t out = *c;
        if (median && out != kInvalid) {
            uint32_t v[9];
            int k = 0;
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
                for (int dx = -1; dx <= 1; ++dx) v[k++] = c[dy * (kTW + 2) + dx];
            out = (uint16_t)median9(v);
        }
        const size_t row = (size_t)gy * width;
        disp[row + gx] = out;
        if (disp_right) disp_right[row + gx] = (uint16_t)rs.at(row, gx, width);
    }
    __syncthreads();   // the tile is reused by the next work item
}

__global__ __launch_bounds__(256) void check_median_kernel(Frame f) {
    __shared__ MedianTile mt;
    check_median_block(mt, f.disp_left, RightSource{f.right_keys, nullptr}, f.width, f.height,
                       f.lr_tolerance, f.median3x3, f.disp, f.disp_right, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(256) void check_median_batch_kernel(WorkList wl) {
    __shared__ MedianTile mt;
    for (int b = blockIdx.x; b < wl.total; b += gridDim.x) {
        const int fi = find_frame(wl, b);
        const Frame& f = wl.frames[fi];
        const int lb = b - wl.starts[fi];
        const int bxs = median_blocks_x(f.width);
        check_median_block(mt, f.disp_left, RightSource{f.right_keys, nullptr}, f.width, f.height,
                           f.lr_tolerance, f.median3x3, f.disp, f.disp_right, lb % bxs, lb / bxs);
    }
}

// Exact consistency check: disp_left = D^L of the pair, flipped = the WTA map
// of the swapped, horizontally flipped pair (so D^R(xr) = flipped[W-1-xr]).
__global__ __launch_bounds__(256) void check_median_exact_kernel(const uint16_t* __restrict__ disp_left,
                                                                  const uint16_t* __restrict__ flipped,
                                                                  int width, int height, int tolerance,
                                                                  int median, uint16_t* __restrict__ disp,
                                                                  uint16_t* __restrict__ disp_right) {
    __shared__ MedianTile mt;
    check_median_block(mt, disp_left, RightSource{nullptr, flipped}, width, height, tolerance, median,
                       disp, disp_right, blockIdx.x, blockIdx.y);
}

// The swapped, horizontally flipped pair: ref[y][x] = right[y][W-1-x] (the
// new reference image), mat[y][x] = left[y][W-1-x].  Outputs have pitch W.
__global__ __launch_bounds__(256) void flip_pair_kernel(const uint8_t* __restrict__ left,
                                                        const uint8_t* __restrict__ right, int width,
                                                        int height, int pitch,
                                                        uint8_t* __restrict__ ref,
                                                        uint8_t* __restrict__ mat) {
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= width) return;
    const size_t src = (size_t)y * pitch + (width - 1 - x);
    const size_t dst = (size_t)y * width + x;
    ref[dst] = right[src];
    mat[dst] = left[src];
}

template <int EPL, int GL, bool FLAT, int NS, bool U8, bool FINE>
void launch_tile_kernel(const Frame* one, const WorkList* wl, int ndisp, hipStream_t stream) {
    const size_t lds = tile_lds_bytes(ndisp);
    if (one) {
        const dim3 g(fused_blocks_x(one->width, ndisp), one->height);
        select_tile_kernel<EPL, GL, FLAT, NS, U8, FINE><<<g, 256, lds, stream>>>(*one);
    } else if constexpr (NS > 1 && !FINE) {
        select_tile_batch_kernel<EPL, GL, FLAT, NS, U8><<<persistent_grid(wl->total), 256, lds, stream>>>(*wl);
    }
}

// frames of one launch share D
template <int NS, bool U8, bool FINE>
void launch_tile(const Frame* one, const WorkList* wl, int ndisp, hipStream_t stream) {
#define SGM_TILE(E, G)                                                                         \
    (ndisp % 16 == 0 ? launch_tile_kernel<E, G, false, NS, U8, FINE>(one, wl, ndisp, stream)   \
                     : launch_tile_kernel<E, G, true, NS, U8, FINE>(one, wl, ndisp, stream))
    if (ndisp <= 16) SGM_TILE(1, 16);
    else if (ndisp <= 32) SGM_TILE(1, 32);
    else if (ndisp <= 64) SGM_TILE(1, 64);
    else if (ndisp <= 128) SGM_TILE(2, 64);
    else SGM_TILE(4, 64);
#undef SGM_TILE
}

template <bool FINE>
void launch_fused_any(const Frame* one, const WorkList* wl, int ndisp, int npaths, int p2,
                      hipStream_t stream) {
    const bool u8 = slices_u8(p2);
    if (npaths == 4) {
        if (u8) launch_tile<2, true, FINE>(one, wl, ndisp, stream);
        else launch_tile<2, false, FINE>(one, wl, ndisp, stream);
    } else {
        if (u8) launch_tile<4, true, FINE>(one, wl, ndisp, stream);
        else launch_tile<4, false, FINE>(one, wl, ndisp, stream);
    }
}

// ---- subpixel output: LR check on the integer maps, then the median over
// the refined values (pixels outside the image and invalid pixels count as
// +inf; a median of +inf is invalid).  Invalid pixels are -1.0f.
constexpr float kInvalidF = -1.0f;

struct MedianTileF {
    float v[(kTH + 2) * (kTW + 2)];
};

__device__ __forceinline__ float median9f(float v[9]) {
#pragma unroll
    for (int pass = 0; pass < 5; ++pass) {
#pragma unroll
        for (int i = 0; i < 8 - pass; ++i) {
            const float lo = fminf(v[i], v[i + 1]);
            const float hi = fmaxf(v[i], v[i + 1]);
            v[i] = lo;
            v[i + 1] = hi;
        }
    }
    return v[4];
}

__global__ __launch_bounds__(256) void check_median_fine_kernel(Frame f) {
    __shared__ MedianTileF mt;
    float* tile = mt.v;
    const int width = f.width, height = f.height, tolerance = f.lr_tolerance;
    const int x0 = blockIdx.x * kTW, y0 = blockIdx.y * kTH;
    for (int i = threadIdx.x; i < (kTH + 2) * (kTW + 2); i += 256) {
        const int ly = i / (kTW + 2), lx = i - ly * (kTW + 2);
        const int gx = x0 + lx - 1, gy = y0 + ly - 1;
        float v = INFINITY;
        if (gx >= 0 && gx < width && gy >= 0 && gy < height) {
            const size_t row = (size_t)gy * width;
            const int dl = f.disp_left[row + gx];
            bool ok = true;
            if (tolerance >= 0) {
                const int xr = gx - dl;
                ok = false;
                if (xr >= 0) {
                    const int dr = (int)(f.right_keys[row + xr] & 0xFFu);
                    const int diff = dl > dr ? dl - dr : dr - dl;
                    ok = diff <= tolerance;
                }
            }
            if (ok) v = f.fine_left[row + gx];
        }
        tile[i] = v;
    }
    __syncthreads();
    const int tx = threadIdx.x & (kTW - 1), ty = threadIdx.x / kTW;
    const int gx = x0 + tx, gy = y0 + ty;
    if (gx < width && gy < height) {
        const float* c = &tile[(ty + 1) * (kTW + 2) + tx + 1];
        float out = *c;
        if (f.median3x3 && out != INFINITY) {
            float v[9];
            int k = 0;
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
                for (int dx = -1; dx <= 1; ++dx) v[k++] = c[dy * (kTW + 2) + dx];
            out = median9f(v);
        }
        const size_t idx = (size_t)gy * width + gx;
        f.disp_fine[idx] = out == INFINITY ? kInvalidF : out;
        if (f.disp_right) f.disp_right[idx] = (uint16_t)(f.right_keys[idx] & 0xFFu);
    }
}

}  // namespace

hipError_t launch_aggregate_select(const Frame& f, hipStream_t stream, bool fine) {
    Frame g = f;
    g.paths_fill_keys = 1;                     // the path kernel clears the D^R keys
    hipError_t e = launch_paths(g, stream);
    if (e != hipSuccess) return e;
    if (fine) launch_fused_any<true>(&f, nullptr, f.ndisp, f.npaths, f.p2, stream);
    else launch_fused_any<false>(&f, nullptr, f.ndisp, f.npaths, f.p2, stream);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 g2(median_blocks_x(f.width), (f.height + kTH - 1) / kTH);
    if (fine) check_median_fine_kernel<<<g2, 256, 0, stream>>>(f);
    else check_median_kernel<<<g2, 256, 0, stream>>>(f);
    return hipGetLastError();
}

// D^L alone, into f.disp_left: no D^R keys, no check, no median.
hipError_t launch_aggregate_wta(const Frame& f, hipStream_t stream) {
    Frame g = f;
    g.right_keys = nullptr;
    g.paths_fill_keys = 0;
    const hipError_t e = launch_paths(g, stream);
    if (e != hipSuccess) return e;
    launch_fused_any<false>(&g, nullptr, g.ndisp, g.npaths, g.p2, stream);
    return hipGetLastError();
}

hipError_t launch_select_fused_batch(const WorkList& wl, int ndisp, int npaths, int p2,
                                     hipStream_t stream) {
    launch_fused_any<false>(nullptr, &wl, ndisp, npaths, p2, stream);
    return hipGetLastError();
}

hipError_t launch_wta_lrc(const Frame& f, hipStream_t stream) {
    const size_t n = (size_t)f.width * f.height;
    fill_keys_kernel<<<fill_blocks(n), 256, 0, stream>>>(f);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // the tile pass, fed S_bar itself as its one uint16 slice (the sum of one
    // slice is the slice)
    Frame g = f;
    g.slices = reinterpret_cast<uint8_t*>(f.agg);
    g.slice_stride = 0;
    launch_tile<1, false, false>(&g, nullptr, f.ndisp, stream);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 g2(median_blocks_x(f.width), (f.height + kTH - 1) / kTH);
    check_median_kernel<<<g2, 256, 0, stream>>>(f);
    return hipGetLastError();
}

hipError_t launch_flip_pair(const uint8_t* left, const uint8_t* right, int width, int height,
                            int pitch, uint8_t* ref, uint8_t* mat, hipStream_t stream) {
    const dim3 g((width + 255) / 256, height);
    flip_pair_kernel<<<g, 256, 0, stream>>>(left, right, width, height, pitch, ref, mat);
    return hipGetLastError();
}

hipError_t launch_check_exact(const uint16_t* disp_left, const uint16_t* flipped, int width,
                              int height, int tolerance, int median, uint16_t* disp,
                              uint16_t* disp_right, hipStream_t stream) {
    const dim3 g(median_blocks_x(width), (height + kTH - 1) / kTH);
    check_median_exact_kernel<<<g, 256, 0, stream>>>(disp_left, flipped, width, height, tolerance,
                                                      median, disp, disp_right);
    return hipGetLastError();
}

hipError_t launch_fill_keys_batch(const WorkList& wl, hipStream_t stream) {
    fill_keys_batch_kernel<<<persistent_grid(wl.total), 256, 0, stream>>>(wl);
    return hipGetLastError();
}

hipError_t launch_median_batch(const WorkList& wl, hipStream_t stream) {
    check_median_batch_kernel<<<persistent_grid(wl.total), 256, 0, stream>>>(wl);
    return hipGetLastError();
}

}  // namespace sgm
