// ncc.hip -- inverted, truncated normalised cross-correlation matching cost
// (Sec. 2.1.1, Sec. 2.2.1 of Ruf et al. 2021), gfx950.
//
//   s = 1 - max(0, Phi),  Phi = (n S_LR - S_L S_R) / (sqrt(n S_LL - S_L^2) sqrt(n S_RR - S_R^2))
//
// over win x win patches (n = win^2), stored as the uint8 cost round(255 s).
// Pixels outside the image read as zero (the zero margin of the census
// window); a patch without variance has no correlation (cost 255); x - d < 0
// costs 255.  The window sums are exact integers; the float part runs in
// float32 with IEEE square root and division in a fixed order, so the
// quantised cost is reproducible bit for bit.
//
// A 256-thread block owns 128 pixels of one row and every disparity.  It
// stages the window columns of both images in LDS -- each column's win bytes
// packed into dwords so that one v_dot4_u32_u8 multiplies four rows -- plus
// each column's sum and sum of squares.  Per-pixel patch sums (the mean and
// variance terms of the paper's per-pixel struct) follow from sums over the
// columns.  A thread then takes four consecutive disparities and a run of
// consecutive pixels: it slides the four cross sums S_LR along x (one new left
// and one new right column per pixel serve all four) and stores four costs at
// a time.
// Bound by its instructions.  An IEEE division per element is most of them, so
// the cost is first taken from the product with the two deviations'
// reciprocals; where that lies so near a rounding tie that the defined
// arithmetic could round to the other side (5 elements in 10,000), the lane
// evaluates the definition.  1242x375, D = 128, 5x5: 68.7 -> 41.0 us (100
// vector instructions per pixel and four disparities), 9x9: 78.1 -> 50.6 us;
// 1920x1080, D = 256, 5x5: 504 -> 270 us.
#include "sgm_internal.h"

namespace sgm {
namespace {

constexpr int kNccTile = 128;                  // pixels of a row per block
constexpr int kMaxD = 256;

// Entry i of an array that lanes read four entries apart: one entry of gap after
// every 32 puts the lanes of a half wave on banks of their own (entries of 8
// bytes; without the gaps they meet four at a time: 44.9 us at 1242x375, D = 128).
constexpr __host__ __device__ int spread(int i) { return i + (i >> 5); }

// The patch sum and the reciprocal deviation of a pixel (0 for a patch without
// variance and for a right pixel outside the image: such a cost is 255); on the
// left side times -255.
struct PatchTerms {
    int32_t sum;
    float inv;
};

template <int WIN>
struct NccTile {
    static constexpr int R = (WIN - 1) / 2;
    static constexpr int CW = (WIN + 3) / 4;   // dwords per packed column
    static constexpr int LCOLS = kNccTile + 2 * R;
    static constexpr int RCOLS = kNccTile + kMaxD - 1 + 2 * R;
    static constexpr int RPIX = kNccTile + kMaxD - 1;
    alignas(8) uint32_t lcol[LCOLS][CW];
    alignas(8) uint32_t rcol[spread(RCOLS)][CW];
    int32_t lsum[LCOLS], lsq[LCOLS];
    int32_t rsum[RCOLS], rsq[RCOLS];
    // per tile pixel / right pixel x0 - D + 1 + i, and the deviations
    // sqrt(n SS - S^2)
    alignas(8) PatchTerms lp[kNccTile];
    alignas(8) PatchTerms rp[spread(RPIX)];
    float lsig[kNccTile], rsig[RPIX];
};

// Column c of a staged image: rows y - R .. y + R at image column gx.
template <int WIN>
__device__ __forceinline__ void stage_column(const uint8_t* __restrict__ img, int width, int height,
                                             int pitch, int gx, int y, uint32_t (&col)[NccTile<WIN>::CW],
                                             int32_t& sum, int32_t& sq) {
    constexpr int R = NccTile<WIN>::R;
#pragma unroll
    for (int k = 0; k < NccTile<WIN>::CW; ++k) col[k] = 0;
    int s = 0, q = 0;
#pragma unroll
    for (int i = 0; i < WIN; ++i) {
        const int gy = y - R + i;
        uint32_t v = 0;
        if (gx >= 0 && gx < width && gy >= 0 && gy < height) v = img[(size_t)gy * pitch + gx];
        col[i >> 2] |= v << (8 * (i & 3));
        s += (int)v;
        q += (int)(v * v);
    }
    sum = s;
    sq = q;
}

template <int WIN>
__device__ __forceinline__ uint32_t column_dot(const uint32_t (&a)[NccTile<WIN>::CW],
                                               const uint32_t (&b)[NccTile<WIN>::CW]) {
    uint32_t acc = 0;
#pragma unroll
    for (int k = 0; k < NccTile<WIN>::CW; ++k) acc = __builtin_amdgcn_udot4(a[k], b[k], acc, false);
    return acc;
}

// sqrt(n SS - S^2) as float32 (IEEE square root), 0 for a patch without
// variance.
__device__ __forceinline__ float patch_sigma(int n, int32_t s, int32_t ss) {
    const int32_t v = n * ss - s * s;
    return v > 0 ? sqrtf((float)v) : 0.0f;
}

#pragma clang fp contract(off)
__device__ __forceinline__ uint8_t ncc_cost_value(int n, int32_t slr, int32_t sl, int32_t sr,
                                                  float sigl, float sigr) {
    if (sigl == 0.0f || sigr == 0.0f) return 255;
    const int32_t num = n * slr - sl * sr;
    const float den = sigl * sigr;
    const float phi = (float)num / den;
    const float s = 1.0f - (phi > 0.0f ? phi : 0.0f);
    float v = rintf(255.0f * s);
    v = v < 0.0f ? 0.0f : (v > 255.0f ? 255.0f : v);
    return (uint8_t)v;
}

// WHOLE: D is a multiple of 4.
template <int WIN, bool WHOLE>
__global__ __launch_bounds__(256) void ncc_cost_kernel(const uint8_t* __restrict__ left,
                                                       const uint8_t* __restrict__ right, int width,
                                                       int height, int pitch, int ndisp,
                                                       uint8_t* __restrict__ cost) {
    using T = NccTile<WIN>;
    constexpr int R = T::R;
    constexpr int N = WIN * WIN;
    constexpr int CW = T::CW;
    __shared__ T t;
    const int x0 = blockIdx.x * kNccTile;
    const int y = blockIdx.y;
    const int npx = min(kNccTile, width - x0);
    const int rbase = x0 - ndisp + 1 - R;      // image column of rcol[0]
    const int nr = npx + ndisp - 1 + 2 * R;

    // stage the window columns
    for (int c = threadIdx.x; c < npx + 2 * R; c += blockDim.x)
        stage_column<WIN>(left, width, height, pitch, x0 - R + c, y, t.lcol[c], t.lsum[c], t.lsq[c]);
    for (int c = threadIdx.x; c < nr; c += blockDim.x)
        stage_column<WIN>(right, width, height, pitch, rbase + c, y, t.rcol[spread(c)], t.rsum[c], t.rsq[c]);
    __syncthreads();

    // patch sums and deviations
    for (int p = threadIdx.x; p < npx; p += blockDim.x) {
        int32_t s = 0, q = 0;
#pragma unroll
        for (int k = 0; k < WIN; ++k) {
            s += t.lsum[p + k];
            q += t.lsq[p + k];
        }
        const float sig = patch_sigma(N, s, q);
        t.lp[p] = PatchTerms{s, sig > 0.0f ? -255.0f * (1.0f / sig) : 0.0f};
        t.lsig[p] = sig;
    }
    for (int p = threadIdx.x; p < npx + ndisp - 1; p += blockDim.x) {
        int32_t s = 0, q = 0;
#pragma unroll
        for (int k = 0; k < WIN; ++k) {
            s += t.rsum[p + k];
            q += t.rsq[p + k];
        }
        const float sig = patch_sigma(N, s, q);
        t.rp[spread(p)] = PatchTerms{s, sig > 0.0f && x0 - ndisp + 1 + p >= 0 ? 1.0f / sig : 0.0f};
        t.rsig[p] = sig;
    }
    __syncthreads();

    // costs: item = (run of pixels, four disparities d0 .. d0 + 3); right pixel
    // x - d is index p + D - 1 - d
    const int groups = (ndisp + 3) / 4;
    const int nruns = max(1, 256 / groups);
    const int run = (npx + nruns - 1) / nruns;
    uint8_t* out = cost + ((size_t)y * width + x0) * ndisp;
    for (int item = threadIdx.x; item < nruns * groups; item += blockDim.x) {
        const int d0 = 4 * (item % groups);
        const int p0 = (item / groups) * run;
        const int p1 = min(npx, p0 + run);
        // index of disparity d0 + 3 at pixel 0; below 0 only for disparities past D
        const int base = ndisp - 1 - d0 - 3;
        auto at = [&](int i) { return spread(WHOLE ? i : max(i, 0)); };
        // right columns and right pixels of the four disparities, the largest first
        uint32_t rc[4][CW];
        PatchTerms rp[4];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
#pragma unroll
            for (int c = 0; c < CW; ++c) rc[j][c] = t.rcol[at(p0 + base + j)][c];
            rp[j] = t.rp[at(p0 + base + j)];
        }
        uint32_t ring[WIN][4];                  // column products of the window, by column mod WIN
        uint32_t slr[4] = {0, 0, 0, 0};
        auto column = [&](int c, uint32_t (&slot)[4]) {
            const int i = at(c + base + 3);
#pragma unroll
            for (int k = 0; k < CW; ++k) rc[3][k] = t.rcol[i][k];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                slot[j] = column_dot<WIN>(t.lcol[c], rc[j]);
                slr[j] += slot[j];
            }
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int k = 0; k < CW; ++k) rc[j][k] = rc[j + 1][k];
        };
        if (p0 < p1) {
#pragma unroll
            for (int k = 0; k < WIN - 1; ++k) column(p0 + k, ring[k]);
        }
        for (int pb = p0; pb < p1; pb += WIN) {
#pragma unroll
            for (int u = 0; u < WIN; ++u) {
                const int p = pb + u;
                if (p < p1) {
                    column(p + WIN - 1, ring[(u + WIN - 1) % WIN]);
                    rp[3] = t.rp[at(p + base + 3)];
                    const PatchTerms lp = t.lp[p];
                    uint32_t b[4];
                    float tie[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        // all factors fit 24 bits
                        const int32_t num = __mul24((int)slr[j], N) - __mul24(lp.sum, rp[j].sum);
                        const float v = __builtin_amdgcn_fmed3f(
                            __builtin_fmaf((float)num * lp.inv, rp[j].inv, 255.0f), 0.0f, 255.0f);
                        const float r = v + 12582912.0f;         // 1.5 * 2^23: the integer part, ties to even
                        b[j] = __float_as_uint(r);
                        tie[j] = fabsf(v - (r - 12582912.0f));
                    }
                    // The product differs from the defined quotient by at most
                    // 6 * 2^-24 of phi <= 1 (the definition rounds the product of
                    // the deviations and the quotient, this the two reciprocals
                    // and two products), the rounding of s, of 255 s and of v by
                    // 2^-25 and twice 2^-17: together below 2^-13 in v
                    constexpr float kTie = 0.5f - 0x1p-12f;
                    if (fmaxf(fmaxf(tie[0], tie[1]), fmaxf(tie[2], tie[3])) > kTie) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (tie[j] > kTie)
                                b[j] = ncc_cost_value(N, (int32_t)slr[j], lp.sum, rp[j].sum, t.lsig[p],
                                                      t.rsig[max(p + base + j, 0)]);
                    }
                    // j = 3 is disparity d0, j = 0 is d0 + 3
                    uint8_t* o = out + (size_t)p * ndisp + d0;
                    const uint32_t lo = __builtin_amdgcn_perm(b[2], b[3], 0x0c0c0400u);
                    const uint32_t hi = __builtin_amdgcn_perm(b[0], b[1], 0x0c0c0400u);
                    const uint32_t w = lo | (hi << 16);
                    if (WHOLE) {
                        *reinterpret_cast<uint32_t*>(o) = w;
                    } else if (d0 + 4 <= ndisp) {
                        __builtin_memcpy(o, &w, 4);
                    } else {
#pragma unroll
                        for (int j = 0; j < 3; ++j)
                            if (d0 + j < ndisp) o[j] = (uint8_t)b[3 - j];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) slr[j] -= ring[u][j];
#pragma unroll
                    for (int j = 0; j < 3; ++j) rp[j] = rp[j + 1];
                }
            }
        }
    }
}

}  // namespace

hipError_t launch_ncc_cost(const uint8_t* left, const uint8_t* right, int width, int height,
                           int pitch, int win, int ndisp, uint8_t* cost, hipStream_t stream) {
    const dim3 grid((width + kNccTile - 1) / kNccTile, height);
#define SGM_NCC(W, F) ncc_cost_kernel<W, F><<<grid, 256, 0, stream>>>(left, right, width, height, pitch, ndisp, cost)
    if (win == 5) {
        if (ndisp % 4 == 0) SGM_NCC(5, true);
        else SGM_NCC(5, false);
    } else {
        if (ndisp % 4 == 0) SGM_NCC(9, true);
        else SGM_NCC(9, false);
    }
#undef SGM_NCC
    return hipGetLastError();
}

}  // namespace sgm
