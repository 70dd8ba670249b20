// census.hip -- census transform (Sec. 2.2.1 of Ruf et al. 2021; centre
// omitted as in Sec. 2.3.1), gfx950.
//
// A 256-thread workgroup owns a 64 x 16 output tile.  The tile plus its
// (RX, RY) halo is staged once through LDS, a dword per load, with the zero
// margin applied at the image border; every thread then computes four
// consecutive pixels of one row, four comparisons per instruction.
// Output: one uint64 per pixel, two per store.
// Bound by its instructions: per window offset and four pixels a byte
// alignment, one v_lerp_u8 as the comparison, and a shift and a select that
// file the results.  9x7, both images of 1920x1080: 20 -> 14 us
// (the write alone 8), of 1242x375: 7.4 -> 6.7 us.
#include "sgm_internal.h"

namespace sgm {
namespace {

constexpr int kThreads = 256;

template <int RX, int RY>
struct CensusTile {
    static constexpr int LW = kCensusTileW + 2 * RX;
    static constexpr int LH = kCensusTileH + 2 * RY;
    static constexpr int LWP = (LW + 3) & ~3;
    alignas(16) uint8_t px[LH * LWP];          // rows start on dword boundaries
};

// Bit 7 of every byte: a > b, for four byte pairs at once, with b given
// inverted.  v_lerp_u8 halves a + (255 - b) per byte: 128 or more iff a > b.
__device__ __forceinline__ uint32_t bytes_greater(uint32_t a, uint32_t not_b) {
    return __builtin_amdgcn_lerp(a, not_b, 0u);
}

// (mask & a) | (~mask & b); the table is f(0xF0, 0xCC, 0xAA)
__device__ __forceinline__ uint32_t select_bits(uint32_t mask, uint32_t a, uint32_t b) {
    return __builtin_amdgcn_bitop3_b32(mask, a, b, 0xCA);
}

// Bit 7 of every byte of t[0] .. t[7] as bits 7 .. 0 of the result's bytes.
// What the other bits of t hold, and what a shift carries over a byte's
// border, never gets through the masks.
__device__ __forceinline__ uint32_t file_bits(const uint32_t (&t)[8]) {
    uint32_t two[4], four[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) two[k] = select_bits(0x80808080u, t[2 * k], t[2 * k + 1] >> 1);
#pragma unroll
    for (int k = 0; k < 2; ++k) four[k] = select_bits(0xC0C0C0C0u, two[2 * k], two[2 * k + 1] >> 2);
    return select_bits(0xF0F0F0F0u, four[0], four[1] >> 4);
}

// Word j: byte j of w[0] .. w[3], w[0]'s on top.
__device__ __forceinline__ void transpose_bytes(const uint32_t (&w)[4], uint32_t (&o)[4]) {
    // the selector's values 0 .. 3 name the second operand's bytes
    const uint32_t a01 = __builtin_amdgcn_perm(w[0], w[1], 0x05010400u), b01 = __builtin_amdgcn_perm(w[0], w[1], 0x07030602u);
    const uint32_t a23 = __builtin_amdgcn_perm(w[2], w[3], 0x05010400u), b23 = __builtin_amdgcn_perm(w[2], w[3], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(a01, a23, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(a01, a23, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(b01, b23, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(b01, b23, 0x07060302u);
}

// Tile (bx, by) of one image.  Every thread passes the same barriers.  A
// thread owns four consecutive pixels of one tile row: for every window
// offset it compares the four centres against the four neighbour bytes at
// once; eight offsets' results make one word whose byte j holds eight bits of
// pixel j's descriptor (the first offset's on top; a descriptor's unused bits
// lead and are zero), and a byte transpose then gives each pixel its uint64.
template <int RX, int RY>
__device__ __forceinline__ void census_tile(CensusTile<RX, RY>& t, const uint8_t* __restrict__ img,
                                            int width, int height, int pitch,
                                            uint64_t* __restrict__ out, int bx, int by) {
    using T = CensusTile<RX, RY>;
    const int x0 = bx * kCensusTileW;
    const int y0 = by * kCensusTileH;
    // Every load of the tile is issued before the first LDS write, so staging
    // costs one memory round trip.  A tile inside the image takes whole
    // dwords (at any alignment); one that reaches past the border takes bytes
    // at clamped positions, zero where clamped.
    constexpr int kRowWords = T::LW / 4;
    static_assert(T::LW % 4 == 0 && T::LWP == T::LW, "a tile row is whole dwords");
    constexpr int kN = kRowWords * T::LH;
    constexpr int kIt = (kN + kThreads - 1) / kThreads;
    uint32_t v[kIt];
    const bool inside = x0 >= RX && y0 >= RY && x0 + T::LW - RX <= width && y0 + T::LH - RY <= height;
    if (inside) {
        const uint8_t* corner = img + (size_t)(y0 - RY) * pitch + (x0 - RX);
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int i = min((int)threadIdx.x + it * kThreads, kN - 1);
            const int ly = i / kRowWords, lw = i - ly * kRowWords;
            __builtin_memcpy(&v[it], corner + (size_t)ly * pitch + 4 * lw, 4);
        }
    } else {
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int i = min((int)threadIdx.x + it * kThreads, kN - 1);
            const int ly = i / kRowWords, lw = i - ly * kRowWords;
            const int gy = y0 + ly - RY, cy = min(max(gy, 0), height - 1);
            const uint8_t* row = img + (size_t)cy * pitch;
            v[it] = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int gx = x0 + 4 * lw + b - RX, cx = min(max(gx, 0), width - 1);
                const uint32_t p = row[cx];
                v[it] |= (gx == cx && gy == cy ? p : 0u) << (8 * b);
            }
        }
    }
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const int i = min((int)threadIdx.x + it * kThreads, kN - 1);   // equal values where clamped
        reinterpret_cast<uint32_t*>(t.px)[i] = v[it];
    }
    __syncthreads();

    constexpr int kBits = (2 * RX + 1) * (2 * RY + 1) - 1;
    constexpr int kLead = 64 - kBits;                  // unused top bits of the uint64
    constexpr int kWords = (4 + 2 * RX + 3) / 4;       // dwords covering a quad's window row
    const int q = threadIdx.x & 15;                    // quad of the tile row
    const int ty = threadIdx.x >> 4;                   // tile row
    const int gy = y0 + ty;
    const int gx = x0 + 4 * q;
    uint32_t acc[8];                                   // acc[0] is the top byte
    // the centres: columns 4q + RX .. 4q + RX + 3 of LDS row ty + RY
    const uint32_t* crow = reinterpret_cast<const uint32_t*>(&t.px[(ty + RY) * T::LWP + 4 * q]);
    const uint32_t centre = __builtin_amdgcn_alignbyte(crow[RX / 4 + 1], crow[RX / 4], RX % 4);
    uint32_t bits[8] = {};
#pragma unroll
    for (int g = 0; g < kLead / 8; ++g) acc[g] = 0;
    int pos = kLead;                                   // bit index from the top
#pragma unroll
    for (int dy = -RY; dy <= RY; ++dy) {
        const uint32_t* row = reinterpret_cast<const uint32_t*>(&t.px[(ty + RY + dy) * T::LWP + 4 * q]);
        uint32_t w[kWords + 1];
#pragma unroll
        for (int k = 0; k < kWords; ++k) w[k] = ~row[k];
        w[kWords] = 0;
#pragma unroll
        for (int dx = -RX; dx <= RX; ++dx) {
            if (dx == 0 && dy == 0) continue;
            const int c = RX + dx;                     // first column of the four neighbours
            const uint32_t nb = c % 4 ? __builtin_amdgcn_alignbyte(w[c / 4 + 1], w[c / 4], c % 4) : w[c / 4];
            bits[pos & 7] = bytes_greater(centre, nb);
            if ((pos & 7) == 7) acc[pos >> 3] = file_bits(bits);
            ++pos;
        }
    }
    const uint32_t top[4] = {acc[0], acc[1], acc[2], acc[3]}, low[4] = {acc[4], acc[5], acc[6], acc[7]};
    uint32_t hi[4], lo[4];
    transpose_bytes(top, hi);
    transpose_bytes(low, lo);
    if (gy < height && gx < width) {
        uint64_t* o = out + (size_t)gy * width + gx;
        if (gx + 3 < width) {
            const uint32_t d01[4] = {lo[0], hi[0], lo[1], hi[1]}, d23[4] = {lo[2], hi[2], lo[3], hi[3]};
            __builtin_memcpy(__builtin_assume_aligned(o, 8), d01, 16);
            __builtin_memcpy(__builtin_assume_aligned(o + 2, 8), d23, 16);
        } else {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (gx + j < width) o[j] = ((uint64_t)hi[j] << 32) | lo[j];
        }
    }
    __syncthreads();   // the tile is reused by the next work item
}

template <int RX, int RY>
__global__ __launch_bounds__(kThreads) void census_kernel(const uint8_t* __restrict__ img, int width,
                                                          int height, int pitch,
                                                          uint64_t* __restrict__ out) {
    __shared__ CensusTile<RX, RY> tile;
    census_tile<RX, RY>(tile, img, width, height, pitch, out, blockIdx.x, blockIdx.y);
}

// Both images of every frame of the work list: block b of a frame is tile b
// of the left image, tile b - census_blocks(w, h) of the right one.
template <int RX, int RY>
__global__ __launch_bounds__(kThreads) void census_batch_kernel(WorkList wl) {
    __shared__ CensusTile<RX, RY> tile;
    for (int b = blockIdx.x; b < wl.total; b += gridDim.x) {
        const int fi = find_frame(wl, b);
        const Frame& f = wl.frames[fi];
        int lb = b - wl.starts[fi];
        const int nb = census_blocks(f.width, f.height);
        const bool right = lb >= nb;
        lb -= right ? nb : 0;
        const int bxs = census_blocks_x(f.width);
        census_tile<RX, RY>(tile, right ? f.right : f.left, f.width, f.height, f.pitch,
                            right ? f.census_right : f.census_left, lb % bxs, lb / bxs);
    }
}

// Both images of one frame in one launch: blockIdx.z selects the image.
template <int RX, int RY>
__global__ __launch_bounds__(kThreads) void census_pair_kernel(Frame f) {
    __shared__ CensusTile<RX, RY> tile;
    const bool right = blockIdx.z != 0;
    census_tile<RX, RY>(tile, right ? f.right : f.left, f.width, f.height, f.pitch,
                        right ? f.census_right : f.census_left, blockIdx.x, blockIdx.y);
}

}  // namespace

hipError_t launch_census_pair(const Frame& f, hipStream_t stream) {
    const dim3 grid(census_blocks_x(f.width), (f.height + kCensusTileH - 1) / kCensusTileH, 2);
    if (f.win_w == 5 && f.win_h == 5) census_pair_kernel<2, 2><<<grid, kThreads, 0, stream>>>(f);
    else census_pair_kernel<4, 3><<<grid, kThreads, 0, stream>>>(f);
    return hipGetLastError();
}

hipError_t launch_census(const Frame& f, bool right, hipStream_t stream) {
    const dim3 grid(census_blocks_x(f.width), (f.height + kCensusTileH - 1) / kCensusTileH);
    const uint8_t* img = right ? f.right : f.left;
    uint64_t* out = right ? f.census_right : f.census_left;
    if (f.win_w == 5 && f.win_h == 5) {
        census_kernel<2, 2><<<grid, kThreads, 0, stream>>>(img, f.width, f.height, f.pitch, out);
    } else {
        census_kernel<4, 3><<<grid, kThreads, 0, stream>>>(img, f.width, f.height, f.pitch, out);
    }
    return hipGetLastError();
}

hipError_t launch_census_batch(const WorkList& wl, int win_w, int win_h, hipStream_t stream) {
    const int grid = persistent_grid(wl.total);
    if (win_w == 5 && win_h == 5) census_batch_kernel<2, 2><<<grid, kThreads, 0, stream>>>(wl);
    else census_batch_kernel<4, 3><<<grid, kThreads, 0, stream>>>(wl);
    return hipGetLastError();
}

}  // namespace sgm
