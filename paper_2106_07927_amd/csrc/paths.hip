// paths.hip -- the path pass of the SGM aggregation, Eq. (sgm_path) and Eq. (sgm_path_aggr)
// of Ruf et al. 2021 (Sec. 2.1.2), gfx950.
//
// This file is compiled once per lane layout (-DSGM_PATH_LAYOUT=<index into
// kPathLayouts>) and per form (-DSGM_PATH_PART=0: the single-frame kernel,
// 1: the work-list kernel), so the kernels build in parallel; aggregate.hip
// holds the pass that sums the slices and picks the layout.
//
// Lines.  Every path direction r splits the image into independent lines:
// rows for the horizontal paths, columns for the vertical ones, and for the
// diagonals W "wrapped" lines that take one pixel per row and restart when
// they cross the left/right border -- the paper's CUDA scheme (Sec. 2.2.2) --
// so every diagonal line is H pixels long.  The path set is taken as pairs of
// opposite directions (r, -r): (LR, RL), (TB, BT), (TLBR, BRTL), (TRBL, BLTR).
// Both directions of a pair cover the same lines, in opposite orders (for a
// diagonal, the same wrapped pixel sequence backwards).
//
// Pairs.  A forward wave walks r along a group of lines and a reverse wave
// walks -r along the same lines; both belong to one block.  The pass writes
// one slice per pair: with P2 <= 127 the penalty parts A = L - C of both
// directions lie in [0, P2] and their sum fits a byte; otherwise the slice is
// uint16 and holds L_r + L_-r.  Either is exact.  The two directions visit a
// pixel at different times, so one of the two values has to be kept until the
// other one is there:
//   first half   each wave walks the first half of its lines and stores only
//                the first step of every chunk of K steps (a checkpoint, in
//                the place of the slice that its pixel has anyway);
//   barrier      of the block;
//   second half  each wave goes on along the half its partner came from.  For
//                every chunk it reads the partner's checkpoint, walks the
//                partner's steps of that chunk again from the cost bytes it
//                needs itself, and stores the sum of both.
// So a slice is written once (plus 2 / K of it as checkpoints) and the cost
// volume is read once per direction.  The pass is bound by that traffic on
// all but small frames (per volume element 8 + 4 + 1 bytes for 8 paths, where
// storing the first half's values instead took 8 + 8 + 4); the steps walked
// twice cost less than the bytes they save: 1920x1080, D = 256: 1910 -> 1102
// us (6.2 TB/s), 1242x375, D = 128: 182 -> 134 us, with P2 = 880: 320 -> 192 us.
// In small frames a line is a chain that nothing else hides.  There two more
// waves per line group (PathLayout::help_*) walk the partner's steps and hand
// them over through LDS, a chunk ahead: 320x240, D = 64, 4 paths: 30 -> 24 us
// (67 ns a step: some 32 instructions, which one wave issues at best every two
// nanoseconds).
// Where lines are many the same waves do better on lines of their own.
//
// Both waves run the same number of steps T = n + delta (a multiple of K):
// the forward wave's extra steps come after its line's end, the reverse
// wave's before its start, so chunks of both cover the same pixels.  Extra
// steps read zeros (which leave a fresh state as it is) and never store.
//
// Lanes.  A line is owned by LPL consecutive lanes; each lane keeps 2*NREG
// consecutive disparities as packed uint16 pairs, register k holding
// (d0 + k, d0 + NREG + k): the neighbours d +- 1 of a register are then the
// registers beside it, and only the first and the last one need the lanes
// beside (one DPP lane shift and one alignbit each way per step).  The state
// is the path vector up to an offset common to the line, taken off once per
// chunk; with m its minimum, one step is
//     V(d) = min(L(d), min(L(d-1), L(d+1)) + P1, m + P2),
//     A(d) = V(d) - m,  L'(d) = V(d) + C(d).
// Per register: a minimum, an add, a three-way minimum (v_pk_minimum3_f16 on
// the integers' bit patterns), a byte permute and an add.  That minimum asks
// for states below 0x7C00: in the 16 steps between two offsets taken off m
// grows to 16 * 255 at most, a real state to m + P2 + 255, padding to twice P2
// (below), and with P1 <= P2 added that is 0x7C00 only where P2 > 7936
// (kNarrowP2); a larger one, which 4 paths may have, takes two minima
// (1242x375, D = 128, 4 paths: 126 us with two at P2 = 7937, 116 with one at
// 7936).  m is a tree over the registers and an all-reduce over the line's lanes
// that runs beside the neighbour terms.  Disparities beyond D (padding) are
// lifted by 255 + P2 in every step: as neighbours they never come below m + P2,
// and m never is one.
//
// Where D cuts a lane's disparities (RAGGED) the accesses stay whole vectors,
// at any byte alignment; only the lane that holds d = D - 1 stores its values
// in parts, and only the chunk with the line's last pixel is loaded byte by
// byte, since there a vector may reach past the volume (803x397, D = 100:
// 594 us with byte accesses in the first design, 310 in this one, now 111).
//
// Memory.  Loads run a chunk ahead.  Cost and checkpoint loads and the slice
// stores go through raw buffer resources: offsets past the volume read as
// zero and stores there are dropped, so positions beyond a line need no
// clamping; a lane or step that must not write carries kNoWrite in its offset.
#include "sgm_internal.h"

#include <type_traits>

#ifndef SGM_PATH_LAYOUT
#error "paths.hip is compiled once per lane layout: -DSGM_PATH_LAYOUT=<index>"
#endif
#if !defined(SGM_PATH_PART) || (SGM_PATH_PART != 0 && SGM_PATH_PART != 1)
#error "paths.hip is compiled in two parts: -DSGM_PATH_PART=0 (single frame) or 1 (work list)"
#endif

namespace sgm {
namespace {

// A block is four waves: one per SIMD of a compute unit (two-wave blocks let
// the dispatcher stack waves of the long horizontal lines on the same SIMD).
constexpr int kThreads = 256;

enum Kind : int { kHorizontal = 0, kVertical = 1, kDiagonal = 2 };

// Steps per chunk of the path loop.  Half as many for the vertical and
// diagonal lines: with 16 their kernels pass 256 registers and only one wave
// fits a SIMD (1242x375, D = 128, 8 registers per lane: 239 us against 148).
constexpr int kStepsH = 16, kStepsO = 8;

// Cache policy of the slice stores: 2 = nontemporal.
constexpr int kStorePolicy = kPathLayouts[SGM_PATH_LAYOUT].stream ? 2 : 0;

// ---- packed pairs ----------------------------------------------------------
// Minimum of three per half.  NARROW: every half is below 0x7C00, where the
// bit patterns of non-negative half floats order like the integers
// (denormals are kept), so one v_pk_minimum3_f16 takes it.
template <bool NARROW>
__device__ __forceinline__ uint32_t pk_min3(uint32_t a, uint32_t b, uint32_t c) {
    if constexpr (NARROW) {
        typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
        const f16x2 x = __builtin_bit_cast(f16x2, a), y = __builtin_bit_cast(f16x2, b),
                    z = __builtin_bit_cast(f16x2, c);
        return __builtin_bit_cast(uint32_t,
                                  __builtin_elementwise_minimum(__builtin_elementwise_minimum(x, y), z));
    } else {
        return pk_min(pk_min(a, b), c);
    }
}

// The smaller half of v in both halves (one instruction: the swap is an operand
// modifier).
__device__ __forceinline__ uint32_t pk_min_swapped(uint32_t v) {
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    const u16x2 x = __builtin_bit_cast(u16x2, v);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(x, __builtin_shufflevector(x, x, 1, 0)));
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp0(uint32_t v) {      // lanes without a source read 0
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true);
}

// ---- cross-lane helpers for lines of up to 64 lanes -----------------------
// Minimum of the packed state over a line, as the same value in both halves
// of every lane of the line (LPL == 64: of a scalar register).
template <int NREG, int LPL, bool NARROW>
__device__ __forceinline__ uint32_t line_min2(const uint32_t (&L)[NREG]) {
    uint32_t v = L[0];
    if constexpr (NREG >= 8) {
        uint32_t w = pk_min3<NARROW>(L[1], L[2], L[3]);
        v = pk_min3<NARROW>(v, L[4], L[5]);
        if constexpr (NREG == 16) {
            w = pk_min3<NARROW>(w, L[8], L[9]);
            v = pk_min3<NARROW>(v, L[10], L[11]);
            w = pk_min3<NARROW>(w, L[12], L[13]);
            v = pk_min3<NARROW>(v, L[14], L[15]);
        }
        w = pk_min3<NARROW>(w, L[6], L[7]);
        v = pk_min(v, w);
    } else if constexpr (NREG == 4) {
        v = pk_min3<NARROW>(v, L[1], pk_min(L[2], L[3]));
    } else if constexpr (NREG == 2) {
        v = pk_min(v, L[1]);
    }
    v = pk_min_swapped(v);
    if constexpr (LPL >= 2) v = min(v, dpp0<kDppQuadSwap1>(v));
    if constexpr (LPL >= 4) v = min(v, dpp0<kDppQuadSwap2>(v));
    if constexpr (LPL >= 8) v = min(v, dpp0<kDppRowHalfMirror>(v));
    if constexpr (LPL >= 16) v = min(v, dpp0<kDppRowMirror>(v));
    if constexpr (LPL == 32) {
        auto s16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = min((uint32_t)s16[0], (uint32_t)s16[1]);
    }
    if constexpr (LPL == 64) {
        // row_bcast:15 / row_bcast:31 carry the minimum to lane 63; from there
        // it travels as a scalar, off the vector chain of the step
        v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0xFFFFFFFF, (int)v, 0x142, 0xA, 0xF, false));
        v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0xFFFFFFFF, (int)v, 0x143, 0xC, 0xF, false));
        v = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
    }
    return v;
}

// Value of the next / previous lane (rows of 16 up to LPL == 16, else the
// whole wave); the caller overrides what crosses a line's edge.
template <int LPL>
__device__ __forceinline__ uint32_t lane_next(uint32_t v) {
    if constexpr (LPL == 1) return 0;
    else if constexpr (LPL <= 16) return dpp0<kDppRowShl1>(v);
    else return dpp0<0x130>(v);
}
template <int LPL>
__device__ __forceinline__ uint32_t lane_prev(uint32_t v) {
    if constexpr (LPL == 1) return 0;
    else if constexpr (LPL <= 16) return dpp0<kDppRowShr1>(v);
    else return dpp0<0x138>(v);
}

// Where a line is a row of 16 lanes or the whole wave, its edge lanes have no
// source: registers that a lane shift leaves alone there and that are kept from
// step to step need their edge value only once.  (Not with 8 registers per
// lane, where no more fit.)
template <int NREG, int LPL>
struct Beside {
    static constexpr bool kKeeps = (LPL == 16 || LPL == 64) && NREG < 8;
    uint32_t next, prev;
    __device__ __forceinline__ void shift(uint32_t lowest, uint32_t highest) {
        constexpr int kNext = LPL <= 16 ? kDppRowShl1 : 0x130, kPrev = LPL <= 16 ? kDppRowShr1 : 0x138;
        next = (uint32_t)__builtin_amdgcn_update_dpp((int)next, (int)lowest, kNext, 0xF, 0xF, false);
        prev = (uint32_t)__builtin_amdgcn_update_dpp((int)prev, (int)highest, kPrev, 0xF, 0xF, false);
    }
};

// ---- bytes of one lane for one pixel: 2*NREG bytes --------------------------
template <int NREG>
struct ByteVec {
    static constexpr int kWords = (NREG + 1) / 2;
    uint32_t w[kWords];
};

// uint16 values of one lane for one pixel: 2*NREG values
template <int NREG>
struct WideVec {
    uint32_t w[NREG];
};

typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr uint32_t kNoWrite = 0x80000000u;
constexpr int kRawBufferWord3 = 0x00020000;     // 32-bit data format, no swizzle

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                             kRawBufferWord3);
}

// 2*NREG bytes at byte offset `off` (out of range: zero).  Any alignment: the
// hardware takes unaligned buffer accesses.
template <int NREG>
__device__ __forceinline__ ByteVec<NREG> load_bytes(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    ByteVec<NREG> c;
    if constexpr (NREG == 1) {
        c.w[0] = __builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
    } else if constexpr (NREG == 2) {
        c.w[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
    } else if constexpr (NREG == 4) {
        const v2u v = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
        c.w[0] = v.x;
        c.w[1] = v.y;
    } else {
        const v4u v = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
        c.w[0] = v.x;
        c.w[1] = v.y;
        c.w[2] = v.z;
        c.w[3] = v.w;
    }
    return c;
}

// the same byte by byte, each checked by itself: where the 2*NREG bytes may
// reach past the volume's end
template <int NREG>
__device__ __forceinline__ ByteVec<NREG> load_bytes_each(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    ByteVec<NREG> c{};
#pragma unroll
    for (int e = 0; e < 2 * NREG; ++e)
        c.w[e >> 2] |= (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, off + e, 0, 0) << (8 * (e & 3));
    return c;
}

// 2*NREG uint16 values at byte offset `off` (out of range: zero)
template <int NREG>
__device__ __forceinline__ WideVec<NREG> load_wide(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    WideVec<NREG> v;
    if constexpr (NREG == 1) {
        v.w[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
    } else if constexpr (NREG == 2) {
        const v2u a = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
        v.w[0] = a.x;
        v.w[1] = a.y;
    } else {
#pragma unroll
        for (int q = 0; q < NREG / 4; ++q) {
            const v4u a = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16 * q, 0, 0);
            v.w[4 * q] = a.x;
            v.w[4 * q + 1] = a.y;
            v.w[4 * q + 2] = a.z;
            v.w[4 * q + 3] = a.w;
        }
    }
    return v;
}

template <int NREG>
__device__ __forceinline__ WideVec<NREG> load_wide_each(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
    WideVec<NREG> v;
#pragma unroll
    for (int k = 0; k < NREG; ++k)
        v.w[k] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off + 4 * k, 0, 0) |
                 ((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off + 4 * k + 2, 0, 0) << 16);
    return v;
}

// State registers hold the lane's disparities split in halves: register k is
// the pair (d0 + k, d0 + NREG + k), so that the neighbours d +- 1 of a whole
// register are the registers beside it and only the first and the last one
// need a shift.  These convert from and to memory order.

// register k of 2*NREG bytes in memory order, zero-extended
template <int NREG>
__device__ __forceinline__ uint32_t byte_pair(const ByteVec<NREG>& c, int k) {
    if constexpr (NREG == 1) return __builtin_amdgcn_perm(0u, c.w[0], 0x0c010c00u);
    const int lo = k, hi = NREG + k;                     // byte indices
    return __builtin_amdgcn_perm(c.w[hi >> 2], c.w[lo >> 2],
                                 0x0c000c00u | (uint32_t)(lo & 3) | ((uint32_t)(4 + (hi & 3)) << 16));
}

// Bytes of a lane in state order: word j = bytes (d0 + 2j, d0 + 2j + 1,
// d0 + NREG + 2j, d0 + NREG + 2j + 1); NREG == 1: the one pair itself, two
// 16-bit halves.
template <int NREG>
struct StateBytes {
    static constexpr int kWords = NREG == 1 ? 1 : NREG / 2;
    uint32_t w[kWords];
};

// Low bytes of V[k] - m for every half, as state-order bytes; m2 holds m in
// both halves.  Exact as plain 32-bit arithmetic: V[2j] + 256 V[2j+1] - 257 m2
// is, modulo 2^32, the sum of the four byte values (each 0..255) at their
// places.
template <int NREG>
__device__ __forceinline__ uint32_t neg257(uint32_t m2) {
    const uint32_t n = 0u - m2;
    return NREG == 1 ? n : n + (n << 8);
}
template <int NREG>
__device__ __forceinline__ uint32_t state_word(const uint32_t (&V)[NREG], int j) {
    return NREG == 1 ? V[0] : V[2 * j] + (V[2 * j + 1 < NREG ? 2 * j + 1 : 0] << 8);
}

// state order -> memory order
template <int NREG>
__device__ __forceinline__ ByteVec<NREG> to_memory(const StateBytes<NREG>& a) {
    ByteVec<NREG> o;
    if constexpr (NREG == 1) {
        o.w[0] = __builtin_amdgcn_perm(0u, a.w[0], 0x0c0c0200u);
    } else if constexpr (NREG == 2) {
        o.w[0] = a.w[0];
    } else {
#pragma unroll
        for (int i = 0; i < NREG / 4; ++i) {
            o.w[i] = __builtin_amdgcn_perm(a.w[2 * i + 1], a.w[2 * i], 0x05040100u);
            o.w[NREG / 4 + i] = __builtin_amdgcn_perm(a.w[2 * i + 1], a.w[2 * i], 0x07060302u);
        }
    }
    return o;
}

// memory order -> state order
template <int NREG>
__device__ __forceinline__ StateBytes<NREG> to_state(const ByteVec<NREG>& o) {
    StateBytes<NREG> a;
    if constexpr (NREG == 1) {
        a.w[0] = __builtin_amdgcn_perm(0u, o.w[0], 0x0c010c00u);
    } else if constexpr (NREG == 2) {
        a.w[0] = o.w[0];
    } else {
#pragma unroll
        for (int i = 0; i < NREG / 4; ++i) {
            a.w[2 * i] = __builtin_amdgcn_perm(o.w[NREG / 4 + i], o.w[i], 0x05040100u);
            a.w[2 * i + 1] = __builtin_amdgcn_perm(o.w[NREG / 4 + i], o.w[i], 0x07060302u);
        }
    }
    return a;
}

// the same for uint16 values: register k of 2*NREG values in memory order
template <int NREG>
__device__ __forceinline__ uint32_t wide_pair(const WideVec<NREG>& c, int k) {
    if constexpr (NREG == 1) return c.w[0];
    const int lo = k, hi = NREG + k;
    return __builtin_amdgcn_perm(c.w[hi >> 1], c.w[lo >> 1],
                                 (k & 1) ? 0x07060302u : 0x05040100u);
}
template <int NREG>
__device__ __forceinline__ WideVec<NREG> to_memory_wide(const uint32_t (&S)[NREG]) {
    WideVec<NREG> o;
    if constexpr (NREG == 1) {
        o.w[0] = S[0];
    } else {
#pragma unroll
        for (int i = 0; i < NREG / 2; ++i) {
            o.w[i] = __builtin_amdgcn_perm(S[2 * i + 1], S[2 * i], 0x05040100u);
            o.w[NREG / 2 + i] = __builtin_amdgcn_perm(S[2 * i + 1], S[2 * i], 0x07060302u);
        }
    }
    return o;
}

// What a lane stores of its 2*NREG slice values: all of them (`full` is 0), or
// with RAGGED (D no multiple of 2*NREG) the lane that holds d = D - 1 stores
// its first D % (2*NREG) = r values, in parts of 8, 4, 2 and 1 values
// (part[k] is 0 where the lane stores the part of 8 >> k).  Any other of these
// is kNoWrite, and OR-ed onto the offset.
struct StoreLanes {
    uint32_t full, part[4];
    int r;
};

// One word of `w` by an index that is the same for the whole wave: bitwise,
// since a choice by comparisons becomes an indexed load from scratch memory.
template <int N>
__device__ __forceinline__ uint32_t pick(const uint32_t (&w)[N], int i) {
    if constexpr (N == 1) {
        return w[0];
    } else {
        const uint32_t up = (i & (N / 2)) ? 0xFFFFFFFFu : 0u;
        uint32_t h[N / 2];
#pragma unroll
        for (int k = 0; k < N / 2; ++k) h[k] = (w[k + N / 2] & up) | (w[k] & ~up);
        return pick(h, i);
    }
}

// Stores one lane's slice bytes at element offset `off` (kNoWrite outside the
// line).
template <int NREG, bool RAGGED>
__device__ __forceinline__ void store_bytes(__amdgpu_buffer_rsrc_t rs, uint32_t off, const StoreLanes& sl,
                                            const ByteVec<NREG>& v) {
    const uint32_t o = off | sl.full;
    if constexpr (NREG == 1) {
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)v.w[0], rs, o, 0, kStorePolicy);
    } else if constexpr (NREG == 2) {
        __builtin_amdgcn_raw_buffer_store_b32(v.w[0], rs, o, 0, kStorePolicy);
    } else if constexpr (NREG == 4) {
        __builtin_amdgcn_raw_buffer_store_b64(v2u{v.w[0], v.w[1]}, rs, o, 0, kStorePolicy);
    } else {
        __builtin_amdgcn_raw_buffer_store_b128(v4u{v.w[0], v.w[1], v.w[2], v.w[3]}, rs, o, 0, kStorePolicy);
    }
    if constexpr (RAGGED) {
        constexpr int W = ByteVec<NREG>::kWords;
        const int r = sl.r;
        if constexpr (NREG == 8)
            __builtin_amdgcn_raw_buffer_store_b64(v2u{v.w[0], v.w[W > 1 ? 1 : 0]}, rs, off | sl.part[0], 0, 0);
        if constexpr (NREG >= 4)
            __builtin_amdgcn_raw_buffer_store_b32(pick(v.w, (r & 8) >> 2), rs, (off | sl.part[1]) + (r & 8), 0, 0);
        if (r & 3) {
            const uint32_t last = pick(v.w, r >> 2);
            if constexpr (NREG >= 2)
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)last, rs, (off | sl.part[2]) + (r & 12), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(last >> (8 * (r & 2))), rs,
                                                 (off | sl.part[3]) + (r & 14), 0, 0);
        }
    }
}

// The same for uint16 values; their byte offsets use all 32 bits, so a value
// that must not be stored gets an offset past any slice (a slice holds at
// most 2^31 - 2 values).
template <int NREG, bool RAGGED>
__device__ __forceinline__ void store_wide(__amdgpu_buffer_rsrc_t rs, uint32_t off, const StoreLanes& sl,
                                           const WideVec<NREG>& v) {
    auto at = [&](uint32_t bias, uint32_t add) { return (off | bias) < kNoWrite ? 2u * off + add : 0xFFFFFFFCu; };
    if constexpr (NREG == 1) {
        __builtin_amdgcn_raw_buffer_store_b32(v.w[0], rs, at(sl.full, 0), 0, kStorePolicy);
    } else if constexpr (NREG == 2) {
        __builtin_amdgcn_raw_buffer_store_b64(v2u{v.w[0], v.w[1]}, rs, at(sl.full, 0), 0, kStorePolicy);
    } else {
#pragma unroll
        for (int q = 0; q < NREG / 4; ++q)
            __builtin_amdgcn_raw_buffer_store_b128(
                v4u{v.w[4 * q], v.w[4 * q + 1], v.w[4 * q + 2], v.w[4 * q + 3]}, rs, at(sl.full, 16 * q), 0,
                kStorePolicy);
    }
    if constexpr (RAGGED) {
        const int r = sl.r;
        if constexpr (NREG == 8)
            __builtin_amdgcn_raw_buffer_store_b128(v4u{v.w[0], v.w[1], v.w[2], v.w[3]}, rs, at(sl.part[0], 0), 0, 0);
        if constexpr (NREG >= 4) {
            __builtin_amdgcn_raw_buffer_store_b64(v2u{pick(v.w, (r & 8) >> 1), pick(v.w, ((r & 8) >> 1) + 1)}, rs,
                                                  at(sl.part[1], 2 * (r & 8)), 0, 0);
        }
        if (r & 3) {
            const uint32_t last = pick(v.w, r >> 1);          // holds value r & ~1, ...
            if constexpr (NREG >= 2)
                __builtin_amdgcn_raw_buffer_store_b32(pick(v.w, (r & 12) >> 1), rs, at(sl.part[2], 2 * (r & 12)),
                                                      0, 0);
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)last, rs, at(sl.part[3], 2 * (r & 14)), 0, 0);
        }
    }
}

// Lane constants of the recursion.  Unless RAGGED, a lane is padding as a whole
// or not at all.
template <int NREG, bool RAGGED>
struct LaneConst {
    uint32_t p1x2, p2x2;
    uint32_t edge_next, edge_prev;     // OR-ed onto what the neighbour lanes give at a line's edges
    uint32_t pad[RAGGED ? NREG : 1];   // 0, or what lifts a padding disparity above m + P2
    __device__ __forceinline__ uint32_t lift(int k) const { return pad[RAGGED ? k : 0]; }
};

// V(d) = min(L(d), min(L(d-1), L(d+1)) + P1, m + P2) for every disparity of
// the lane, from the state L and its line minimum m (m2: in both halves).
template <int NREG, int LPL, bool NARROW, bool RAGGED>
__device__ __forceinline__ void relax(const uint32_t (&L)[NREG], uint32_t m2, const LaneConst<NREG, RAGGED>& lc,
                                      Beside<NREG, LPL>& beside, uint32_t (&V)[NREG]) {
    const uint32_t cap = m2 + lc.p2x2;           // no carry crosses the halves
    uint32_t nx, pv;
    if constexpr (Beside<NREG, LPL>::kKeeps) {
        beside.shift(L[0], L[NREG - 1]);
        nx = beside.next;
        pv = beside.prev;
    } else {
        nx = lane_next<LPL>(L[0]) | lc.edge_next;
        pv = lane_prev<LPL>(L[NREG - 1]) | lc.edge_prev;
    }
    const uint32_t below = __builtin_amdgcn_alignbit(L[NREG - 1], pv, 16);    // of register 0
    const uint32_t above = __builtin_amdgcn_alignbit(nx, L[0], 16);           // of register NREG - 1
#pragma unroll
    for (int k = 0; k < NREG; ++k) {
        const uint32_t nb = pk_min(k == 0 ? below : L[k - 1], k == NREG - 1 ? above : L[k + 1]);
        V[k] = pk_min3<NARROW>(nb + lc.p1x2, L[k], cap);
    }
}

// the next state: V + C (and the padding lift)
template <int NREG, bool PADDED, bool RAGGED>
__device__ __forceinline__ void advance(const uint32_t (&V)[NREG], const ByteVec<NREG>& c,
                                        const LaneConst<NREG, RAGGED>& lc, uint32_t (&L)[NREG]) {
#pragma unroll
    for (int k = 0; k < NREG; ++k) {
        L[k] = V[k] + byte_pair<NREG>(c, k);
        if constexpr (PADDED) L[k] += lc.lift(k);
    }
}

// Chunk schedule of one line pair of n pixels: both waves run T = n + delta
// steps (T a multiple of K).  The forward wave's step s is its pixel s; the
// reverse wave's step s is its pixel s - delta.  The forward wave writes its
// own values for steps [0, split_fwd), the reverse wave for steps
// [0, split_rev) -- together every pixel of the line exactly once, with each
// split on a chunk boundary -- and then each completes the pixels the other
// wrote.
struct Schedule {
    int T, delta, split_fwd, split_rev;
    __host__ __device__ Schedule(int n, int K) {
        delta = (K - n % K) % K;
        T = n + delta;
        split_fwd = K * (T / (2 * K));
        split_rev = T - split_fwd;
    }
};

__device__ __forceinline__ void pair_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Orders LDS accesses of the block's waves only: global loads and stores stay
// in flight across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Values of one direction at the K steps of a chunk, as the sum with the other
// one takes them: penalty bytes in state order, or path values as packed
// pairs.  put / get carry them through LDS, one row of 64 lanes per step.
template <int NREG, int K, bool U8>
struct StepValues {
    static constexpr int kWords = U8 ? StateBytes<NREG>::kWords : NREG;
    StateBytes<NREG> a[U8 ? K : 1];
    uint32_t l[U8 ? 1 : K][NREG];
    __device__ __forceinline__ void put(uint32_t* row, int lane) const {
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
            for (int i = 0; i < kWords; ++i) row[(j * 64 + lane) * kWords + i] = U8 ? a[U8 ? j : 0].w[U8 ? i : 0] : l[U8 ? 0 : j][U8 ? 0 : i];
    }
    __device__ __forceinline__ void get(const uint32_t* row, int lane) {
#pragma unroll
        for (int j = 0; j < K; ++j)
#pragma unroll
            for (int i = 0; i < kWords; ++i) {
                if constexpr (U8) a[j].w[i] = row[(j * 64 + lane) * kWords + i];
                else l[j][i] = row[(j * 64 + lane) * kWords + i];
            }
    }
};

// Position of one lane along its line, laid out a chunk of K steps at a time.
// A diagonal's line wraps at the left / right border: the recursion restarts
// there, `left` steps from now.  Most chunks hold no such step in any line of
// the wave and advance by one stride like the other kinds.
template <int KIND, int K>
struct Walker {
    uint32_t e;            // element offset of the next step
    int left;              // diagonal: steps before the next restart (0: the next step is one)
    int32_t stride, wrap;  // wrap: added to e at a restart
    int width;

    // offsets of the next K steps and their restart flags; true if some line
    // of the wave restarts among them
    __device__ __forceinline__ bool next(uint32_t (&offs)[K], bool (&restart)[K]) {
        if (KIND == kDiagonal && __builtin_amdgcn_ballot_w64(left < K) != 0) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                restart[j] = left == 0;
                e += restart[j] ? (uint32_t)wrap : 0u;
                left = (restart[j] ? width : left) - 1;
                offs[j] = e;
                e += (uint32_t)stride;
            }
            return true;
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            offs[j] = e + (uint32_t)(j * stride);
            restart[j] = false;
        }
        e += (uint32_t)(K * stride);
        left -= K;
        return false;
    }
};

// One wave of a line pair, the whole way along.  The offsets of the steps of
// the next chunk are laid out one chunk ahead and serve its cost loads,
// its checkpoint and its stores.
template <int KIND, int NREG, int LPL, int K, bool RAGGED, bool PADDED, bool U8, bool NARROW, bool HELP>
__device__ __forceinline__ void run_wave(const Frame& f, uint8_t* __restrict__ slice, int q, bool fwd,
                                         bool helper, int group, uint32_t* __restrict__ lds) {
    constexpr int DPL = 2 * NREG;
    constexpr int LPW = 64 / LPL;
    constexpr int SW = StateBytes<NREG>::kWords;
    const int width = f.width, height = f.height, ndisp = f.ndisp;
    const int lane = threadIdx.x & 63;
    const int sub = lane % LPL;
    const int nlines = pair_lines(q, width, height);
    const int line = group * LPW + lane / LPL;
    const bool line_ok = line < nlines;
    const int lc = line_ok ? line : nlines - 1;
    const bool d_ok = sub * DPL < ndisp;
    const int d0 = d_ok ? sub * DPL : 0;             // padding lanes read d = 0
    const bool write = line_ok && d_ok;
    const int n = KIND == kHorizontal ? width : height;
    const Schedule sch(n, K);
    const int dlt = fwd ? 0 : sch.delta;             // pixel of step s = s - dlt
    const int nchunks = sch.T / K;
    const int c_split = (fwd ? sch.split_fwd : sch.split_rev) / K;
    // chunks of the longer second half of the two directions
    const int rounds = nchunks - sch.split_fwd / K;
    // The chunk that holds the forward line's last pixel.  If that is the
    // volume's last one, the bytes of its last lane may end before the vector.
    const int c_edge = RAGGED ? (fwd ? nchunks - 1 : 0) : -1;
    // the forward wave's last chunk holds steps past its line's end
    const int c_last_checked = (fwd && sch.delta > 0) ? nchunks - 1 : -1;

    const uint32_t vol = (uint32_t)((size_t)width * height * ndisp);
    const __amdgpu_buffer_rsrc_t rc = buffer_rsrc(f.cost, vol);
    const __amdgpu_buffer_rsrc_t rs = buffer_rsrc(slice, U8 ? vol : 2u * vol);

    LaneConst<NREG, RAGGED> cst;
    cst.p1x2 = pk_splat((uint32_t)f.p1);
    cst.p2x2 = pk_splat((uint32_t)f.p2);
    constexpr uint32_t kEdge = NARROW ? 0x4000u : 0x8000u;
    cst.edge_next = sub == LPL - 1 ? kEdge : 0u;
    cst.edge_prev = sub == 0 ? kEdge << 16 : 0u;
    Beside<NREG, LPL> beside = {cst.edge_next, cst.edge_prev};
    const uint32_t lift = 255u + (uint32_t)f.p2;
#pragma unroll
    for (int k = 0; k < (RAGGED ? NREG : 1); ++k) {
        const uint32_t lo = (sub * DPL + k < ndisp) ? 0u : lift;
        const uint32_t hi = (sub * DPL + (RAGGED ? NREG + k : 0) < ndisp) ? 0u : lift;
        cst.pad[k] = PADDED ? lo | (hi << 16) : 0u;
    }
    StoreLanes sl;
    sl.r = ndisp % DPL;
    const bool whole = write && d0 + DPL <= ndisp;
    sl.full = whole ? 0u : kNoWrite;
#pragma unroll
    for (int i = 0; i < 4; ++i) sl.part[i] = RAGGED && write && !whole && (sl.r & (8 >> i)) ? 0u : kNoWrite;

    // the wave's own direction and first pixel; the reverse wave starts where
    // the forward line ends
    int dx, dy;
    pair_dir(q, &dx, &dy);
    const int sdx = fwd ? dx : -dx, sdy = fwd ? dy : -dy;
    int x0, y0;
    if constexpr (KIND == kHorizontal) {
        y0 = lc;
        x0 = sdx > 0 ? 0 : width - 1;
    } else if constexpr (KIND == kVertical) {
        x0 = lc;
        y0 = sdy > 0 ? 0 : height - 1;
    } else {
        y0 = sdy > 0 ? 0 : height - 1;
        const int e = fwd ? lc : (lc + dx * (height - 1)) % width;
        x0 = e < 0 ? e + width : e;
    }
    // position of step s of the wave: pixel s - dlt of its line
    Walker<KIND, K> wk;
    auto walk_from = [&](int step) {
        const int t = step - dlt;
        int xs = x0, ys = y0;
        if constexpr (KIND == kHorizontal) xs += t * sdx;
        else ys += t * sdy;
        if constexpr (KIND == kDiagonal) {
            xs = (x0 + t * sdx) % width;
            xs = xs < 0 ? xs + width : xs;
        }
        wk.e = ((uint32_t)ys * (uint32_t)width + (uint32_t)xs) * (uint32_t)ndisp + (uint32_t)d0;
        wk.left = sdx > 0 ? width - xs : xs + 1;
        wk.stride = (sdy * width + sdx) * ndisp;
        wk.wrap = -sdx * width * ndisp;
        wk.width = width;
    };

    // The next chunk: step offsets, restart flags (wrap_n: some line of the
    // wave restarts in it), cost bytes.  Positions outside the line read as
    // zero, which keeps a fresh state fresh, so the reverse wave needs no
    // restart at its first pixel.
    uint32_t offs_n[K];
    bool rst_n[K];
    ByteVec<NREG> cn[K];
    bool wrap_n;
    auto load_next = [&](int c) {
        if (RAGGED && c == c_edge) {
#pragma unroll
            for (int j = 0; j < K; ++j) cn[j] = load_bytes_each<NREG>(rc, offs_n[j]);
        } else {
#pragma unroll
            for (int j = 0; j < K; ++j) cn[j] = load_bytes<NREG>(rc, offs_n[j]);
        }
    };
    // of the last chunk, the forward wave's steps past its line's end
    auto drop_tail = [&](int c) {
        if (c == c_last_checked) {
#pragma unroll
            for (int j = 0; j < K; ++j) offs_n[j] = j >= K - sch.delta ? kNoWrite : offs_n[j];
        }
    };
    // state of the own recursion, up to an offset common to the line
    uint32_t L[NREG];
#pragma unroll
    for (int k = 0; k < NREG; ++k) L[k] = cst.lift(k);
    auto restart = [&](uint32_t (&s)[NREG], bool r) {
#pragma unroll
        for (int k = 0; k < NREG; ++k) s[k] = r ? cst.lift(k) : s[k];
    };
    // one own step: V and the new state; returns m as a pair.  Once per chunk
    // the offset is taken off.
    auto own_step = [&](int j, const ByteVec<NREG>& cost, uint32_t (&V)[NREG]) {
        uint32_t m2 = line_min2<NREG, LPL, NARROW>(L);
        if (j == 0) {
#pragma unroll
            for (int k = 0; k < NREG; ++k) L[k] -= m2;
            m2 = 0;
        }
        relax<NREG, LPL, NARROW>(L, m2, cst, beside, V);
        advance<NREG, PADDED>(V, cost, cst, L);
        return m2;
    };

    // The partner's recursion over a chunk starts from the step it stored, at
    // the chunk's last pixel, and runs back to the chunk's first.
    using PartnerSteps = StepValues<NREG, K, U8>;
    uint32_t P[NREG];
    ByteVec<NREG> kb;
    WideVec<NREG> kw;
    auto load_checkpoint = [&](int c) {
        const uint32_t off = offs_n[K - 1];
        if constexpr (U8) {
            if (RAGGED && c == c_edge) kb = load_bytes_each<NREG>(rs, off);
            else kb = load_bytes<NREG>(rs, off);
        } else {
            if (RAGGED && c == c_edge) kw = load_wide_each<NREG>(rs, 2u * off);
            else kw = load_wide<NREG>(rs, 2u * off);
            // twice a no-write offset is inside the slice again
#pragma unroll
            for (int k = 0; k < NREG; ++k) kw.w[k] = off >= kNoWrite ? 0u : kw.w[k];
        }
    };
    auto partner_first = [&](PartnerSteps& out, const ByteVec<NREG>& cost, const ByteVec<NREG>& kb,
                             const WideVec<NREG>& kw) {
        if constexpr (U8) {
            uint32_t V[NREG];
            out.a[K - 1] = to_state<NREG>(kb);
#pragma unroll
            for (int k = 0; k < NREG; ++k) V[k] = byte_pair<NREG>(kb, k);
            advance<NREG, PADDED>(V, cost, cst, P);
        } else {
#pragma unroll
            for (int k = 0; k < NREG; ++k) {
                P[k] = wide_pair<NREG>(kw, k);
                out.l[K - 1][k] = P[k];
                // padding may hold anything: bounded (a real value is at most
                // 255 + P2), so that the lift cannot overflow
                if constexpr (PADDED) P[k] = pk_min(P[k], NARROW ? 0x1FFF1FFFu : 0x7FFF7FFFu) + cst.lift(k);
            }
        }
    };
    auto partner_step = [&](int j, PartnerSteps& out, const ByteVec<NREG>& cost) {
        uint32_t V[NREG];
        const uint32_t m2 = line_min2<NREG, LPL, NARROW>(P);
        relax<NREG, LPL, NARROW>(P, m2, cst, beside, V);
        advance<NREG, PADDED>(V, cost, cst, P);
        if constexpr (U8) {
            const uint32_t nm = neg257<NREG>(m2);
#pragma unroll
            for (int i = 0; i < SW; ++i) out.a[j].w[i] = state_word<NREG>(V, i) + nm;
        } else {
#pragma unroll
            for (int k = 0; k < NREG; ++k) out.l[j][k] = P[k] - m2;
        }
    };
    if constexpr (HELP) {
        if (helper) {
            // the partner's steps of every chunk of the second half, through
            // LDS to the wave that walks it
            walk_from(c_split * K);
            pair_barrier();
            if (c_split < nchunks) {
                wrap_n = wk.next(offs_n, rst_n);
                drop_tail(c_split);
                load_next(c_split);
                load_checkpoint(c_split);
            }
            for (int i = 0; i < rounds; ++i) {
                const int c = c_split + i;
                if (c < nchunks) {
                    ByteVec<NREG> cur[K];
                    bool rst[K];
                    const bool w = wrap_n;
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        cur[j] = cn[j];
                        rst[j] = rst_n[j];
                    }
                    const ByteVec<NREG> kb0 = kb;
                    const WideVec<NREG> kw0 = kw;
                    if (c + 1 < nchunks) {
                        wrap_n = wk.next(offs_n, rst_n);
                        drop_tail(c + 1);
                        load_next(c + 1);
                        load_checkpoint(c + 1);
                    }
                    auto steps = [&](auto wraps) {
                        constexpr bool WRAPS = decltype(wraps)::value;
                        PartnerSteps out;
                        partner_first(out, cur[K - 1], kb0, kw0);
#pragma unroll
                        for (int j = K - 2; j >= 0; --j) {
                            if constexpr (WRAPS) restart(P, rst[j + 1]);
                            partner_step(j, out, cur[j]);
                        }
                        out.put(lds + (i & 1) * (K * 64 * PartnerSteps::kWords), lane);
                    };
                    if (KIND == kDiagonal && w) steps(std::true_type{});
                    else steps(std::false_type{});
                }
                lds_barrier();
            }
            return;
        }
    }

    walk_from(0);
    wrap_n = wk.next(offs_n, rst_n);
#pragma unroll
    for (int j = 0; j < K; ++j) offs_n[j] = j < dlt ? kNoWrite : offs_n[j];
    drop_tail(0);
    load_next(0);

    // ---- first half: only the first step of every chunk is stored.  The
    // next chunk's loads are issued as this chunk's bytes are used up.
    auto first_half = [&](auto wraps) {
        constexpr bool WRAPS = decltype(wraps)::value;
        const uint32_t off0 = offs_n[0];
        bool rst[K];
#pragma unroll
        for (int j = 0; j < K; ++j) rst[j] = rst_n[j];
        wrap_n = wk.next(offs_n, rst_n);
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if constexpr (WRAPS) restart(L, rst[j]);
            uint32_t V[NREG];
            own_step(j, cn[j], V);
            cn[j] = load_bytes<NREG>(rc, offs_n[j]);
            if (j == 0) {
                if constexpr (U8) {
                    StateBytes<NREG> a;
#pragma unroll
                    for (int i = 0; i < SW; ++i) a.w[i] = state_word<NREG>(V, i);
                    store_bytes<NREG, RAGGED>(rs, off0, sl, to_memory<NREG>(a));
                } else {
                    store_wide<NREG, RAGGED>(rs, off0, sl, to_memory_wide<NREG>(L));
                }
            }
        }
    };
    for (int c = 0; c < c_split; ++c) {
        if (KIND == kDiagonal && wrap_n) first_half(std::true_type{});
        else first_half(std::false_type{});
    }
    if (c_split > 0 && c_split < nchunks && (c_split == c_last_checked || c_split == c_edge)) {
        // of a chunk that was laid out as any other: again, with its checks
        drop_tail(c_split);
        load_next(c_split);
    }
    pair_barrier();
    if (!HELP && c_split == nchunks) return;

    // ---- second half -----------------------------------------------------------
    // one own step; the sum of both directions goes out
    auto own_out = [&](int j, const ByteVec<NREG>& cost, const PartnerSteps& p, uint32_t off) {
        uint32_t V[NREG];
        const uint32_t m2 = own_step(j, cost, V);
        if constexpr (U8) {
            const uint32_t nm = neg257<NREG>(m2);
            StateBytes<NREG> a;
#pragma unroll
            for (int i = 0; i < SW; ++i) a.w[i] = state_word<NREG>(V, i) + (p.a[j].w[i] + nm);
            store_bytes<NREG, RAGGED>(rs, off, sl, to_memory<NREG>(a));
        } else {
            uint32_t S[NREG];
#pragma unroll
            for (int k = 0; k < NREG; ++k) S[k] = L[k] + (p.l[j][k] - m2);
            store_wide<NREG, RAGGED>(rs, off, sl, to_memory_wide<NREG>(S));
        }
    };

    if constexpr (!HELP) load_checkpoint(c_split);
    uint32_t offs[K];
    bool rst[K];
    ByteVec<NREG> cur[K];
    PartnerSteps pa;
    auto second_half = [&](int c, auto wraps) {
        constexpr bool WRAPS = decltype(wraps)::value;
        if constexpr (HELP) {
            pa.get(lds + ((c - c_split) & 1) * (K * 64 * PartnerSteps::kWords), lane);
        } else {
            partner_first(pa, cur[K - 1], kb, kw);
            if (c + 1 < nchunks) load_checkpoint(c + 1);
#pragma unroll
            for (int j = K - 2; j >= 0; --j) {
                if constexpr (WRAPS) restart(P, rst[j + 1]);
                partner_step(j, pa, cur[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if constexpr (WRAPS) restart(L, rst[j]);
            own_out(j, cur[j], pa, offs[j]);
        }
    };
    // Loads and stores share one in-order counter, and the wait at the loop's
    // top has to hold on its first round too: without a chunk's worth of
    // stores behind the first loads it would wait for the last round's stores
    // on every round.  The range check of an empty buffer drops these.
    const __amdgpu_buffer_rsrc_t nowhere = buffer_rsrc(slice, 0);
#pragma unroll
    for (int j = 0; j < K; ++j) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)0, nowhere, 4 * j, 0, 0);
    for (int c = c_split; c < nchunks; ++c) {
        const bool w = wrap_n;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            offs[j] = offs_n[j];
            rst[j] = rst_n[j];
            cur[j] = cn[j];
        }
        if (c + 1 < nchunks) {
            wrap_n = wk.next(offs_n, rst_n);
            drop_tail(c + 1);
            load_next(c + 1);
        }
        if constexpr (HELP) lds_barrier();
        if (KIND == kDiagonal && w) second_half(c, std::true_type{});
        else second_half(c, std::false_type{});
    }
    if constexpr (HELP) {
        for (int i = nchunks - c_split; i < rounds; ++i) lds_barrier();
    }
}

// Block lb of the path pass of one frame: pair q, line groups 2g and 2g + 1;
// waves 0, 1 walk the forward direction along them, waves 2, 3 the reverse
// one.
template <int NH, int LH, int NO, int LO, bool RGH, bool PDH, bool RGO, bool PDO, bool U8, bool NARROW>
__device__ __forceinline__ void paths_block(const Frame& f, int lb) {
    constexpr int KH = kStepsH, KO = kStepsO;
    constexpr PathLayout kLayout = kPathLayouts[SGM_PATH_LAYOUT];
    constexpr bool HELPH = kLayout.help_h, HELPO = kLayout.help_o;
    const int npairs = f.npaths / 2;
    if (f.paths_fill_keys) {
        // the D^R key map of the selection that follows starts at "no
        // candidate"; every block clears an equal share of it
        int nb = 0;
        for (int q = 0; q < npairs; ++q) nb += pair_blocks(q, f.width, f.height, kLayout);
        const size_t n = (size_t)f.width * f.height;
        const size_t per = (n + nb - 1) / nb;
        const size_t e1 = min(n, (size_t)(lb + 1) * per);
        for (size_t e = (size_t)lb * per + threadIdx.x; e < e1; e += blockDim.x) f.right_keys[e] = 0xFFFFFFFFu;
    }
    int q = 0, start = 0;
    for (; q < npairs - 1; ++q) {
        const int nb = pair_blocks(q, f.width, f.height, kLayout);
        if (lb < start + nb) break;
        start += nb;
    }
    // the same for all lanes of a wave, and known to be: the loops and branches
    // below stay scalar
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lb0 = lb - start;
    uint8_t* slice = f.slices + (size_t)q * f.slice_stride * (U8 ? 1 : 2);
    constexpr int kLdsH = HELPH ? 2 * KH * 64 * StepValues<NH, KH, U8>::kWords : 0;
    constexpr int kLdsO = HELPO ? 2 * KO * 64 * StepValues<NO, KO, U8>::kWords : 0;
    constexpr int kLds = kLdsH > kLdsO ? kLdsH : kLdsO;
    __shared__ __align__(16) uint32_t lds[kLds > 0 ? 2 * kLds : 1];
    const bool help = q == 0 ? HELPH : HELPO;
    const bool fwd = help ? (wave & 1) == 0 : wave < 2;
    const int group = help ? lb0 : 2 * lb0 + (wave & 1);
    uint32_t* mine = lds + (fwd ? 0 : kLds);
    if (q == 0) {
        __builtin_amdgcn_s_setprio(2);
        run_wave<kHorizontal, NH, LH, KH, RGH, PDH, U8, NARROW, HELPH>(f, slice, q, fwd, wave >= 2, group, mine);
        __builtin_amdgcn_s_setprio(0);
    } else if (q == 1) {
        run_wave<kVertical, NO, LO, KO, RGO, PDO, U8, NARROW, HELPO>(f, slice, q, fwd, wave >= 2, group, mine);
    } else {
        run_wave<kDiagonal, NO, LO, KO, RGO, PDO, U8, NARROW, HELPO>(f, slice, q, fwd, wave >= 2, group, mine);
    }
}

template <int NH, int LH, int NO, int LO, bool RGH, bool PDH, bool RGO, bool PDO, bool U8, bool NARROW>
__global__ __launch_bounds__(kThreads, 2) void paths_kernel(Frame f) {
    paths_block<NH, LH, NO, LO, RGH, PDH, RGO, PDO, U8, NARROW>(f, blockIdx.x);
}

template <int NH, int LH, int NO, int LO, bool RGH, bool PDH, bool RGO, bool PDO, bool U8, bool NARROW>
__global__ __launch_bounds__(kThreads, 2) void paths_batch_kernel(WorkList wl) {
    // one block per item, the longest lines first (a loop over items here costs
    // the registers that let two waves share a SIMD)
    const int b = blockIdx.x;
    paths_block<NH, LH, NO, LO, RGH, PDH, RGO, PDO, U8, NARROW>(wl.frames[wl.items[2 * b]], wl.items[2 * b + 1]);
}

// Path-kernel launches for one lane layout: the single-frame kernel, or the
// work-list form.  The two are compiled in separate objects
// (SGM_PATH_PART 0 and 1), so the library's longest compile splits in two.
struct LayoutFlags {
    bool ragged, padded;   // D cuts a lane's disparities; some lane holds padding
};

__host__ inline LayoutFlags layout_flags(int nh, int lh, int no, int lo, int ndisp) {
    return {ndisp % (2 * nh) != 0 || ndisp % (2 * no) != 0, lh * 2 * nh > ndisp || lo * 2 * no > ndisp};
}

#if SGM_PATH_PART == 0
template <int NH, int LH, int NO, int LO>
hipError_t launch_paths_single(const Frame& one, int ndisp, int p2, int nblocks, hipStream_t stream) {
    const LayoutFlags fl = layout_flags(NH, LH, NO, LO, ndisp);
#define SGM_PATHS(A, B)                                                                                    \
    do {                                                                                                   \
        if (slices_u8(p2)) paths_kernel<NH, LH, NO, LO, A, B, A, B, true, true><<<nblocks, kThreads, 0, stream>>>(one);   \
        else if (p2 <= kNarrowP2)                                                                          \
            paths_kernel<NH, LH, NO, LO, A, B, A, B, false, true><<<nblocks, kThreads, 0, stream>>>(one);            \
        else                                                                                               \
            paths_kernel<NH, LH, NO, LO, A, B, A, B, false, false><<<nblocks, kThreads, 0, stream>>>(one);           \
    } while (0)
    if (fl.ragged) {
        if constexpr (NO <= 4) SGM_PATHS(true, true);
        else return hipErrorInvalidValue;                // path_layout_id gives no other layout such a D
    } else if (fl.padded) {
        SGM_PATHS(false, true);
    } else {
        SGM_PATHS(false, false);
    }
#undef SGM_PATHS
    return hipGetLastError();
}
#else
template <int NH, int LH, int NO, int LO>
hipError_t launch_paths_worklist(const WorkList& wl, int ndisp, int p2, int nblocks, hipStream_t stream) {
    const LayoutFlags fl = layout_flags(NH, LH, NO, LO, ndisp);
#define SGM_PATHS(A, B)                                                                                    \
    do {                                                                                                   \
        if (slices_u8(p2)) paths_batch_kernel<NH, LH, NO, LO, A, B, A, B, true, true><<<nblocks, kThreads, 0, stream>>>(wl);   \
        else if (p2 <= kNarrowP2)                                                                          \
            paths_batch_kernel<NH, LH, NO, LO, A, B, A, B, false, true><<<nblocks, kThreads, 0, stream>>>(wl);            \
        else                                                                                               \
            paths_batch_kernel<NH, LH, NO, LO, A, B, A, B, false, false><<<nblocks, kThreads, 0, stream>>>(wl);           \
    } while (0)
    if (fl.ragged) {
        if constexpr (NO <= 4) SGM_PATHS(true, true);
        else return hipErrorInvalidValue;                // path_layout_id gives no other layout such a D
    } else if (fl.padded) {
        SGM_PATHS(false, true);
    } else {
        SGM_PATHS(false, false);
    }
#undef SGM_PATHS
    return hipGetLastError();
}
#endif

}  // namespace

#if SGM_PATH_PART == 0
template <>
hipError_t launch_paths_layout_id<SGM_PATH_LAYOUT>(const Frame& one, int ndisp, int p2, int nblocks,
                                                   hipStream_t stream) {
    constexpr PathLayout L = kPathLayouts[SGM_PATH_LAYOUT];
    return launch_paths_single<L.nreg_h, L.lpl_h, L.nreg_o, L.lpl_o>(one, ndisp, p2, nblocks, stream);
}
#else
template <>
hipError_t launch_paths_batch_layout_id<SGM_PATH_LAYOUT>(const WorkList& wl, int ndisp, int p2,
                                                         int nblocks, hipStream_t stream) {
    constexpr PathLayout L = kPathLayouts[SGM_PATH_LAYOUT];
    return launch_paths_worklist<L.nreg_h, L.lpl_h, L.nreg_o, L.lpl_o>(wl, ndisp, p2, nblocks, stream);
}
#endif

}  // namespace sgm
