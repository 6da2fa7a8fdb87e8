// Device helpers shared by the particle passes of the forward step and of its
// adjoint: global-pointer casts, fixed-point window accumulators, small
// integer division, wave reductions and window geometry.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace sipf {

#define GLOBAL __attribute__((address_space(1)))
template <typename T> __device__ __forceinline__ GLOBAL T* gp(T* p) { return (GLOBAL T*)p; }
template <typename T> __device__ __forceinline__ const GLOBAL T* gp(const T* p) { return (const GLOBAL T*)p; }

// Complex values through global-address-space pointers (a pointer read from a
// descriptor in memory is generic to the compiler, its accesses flat).
template <typename V> struct PairOf;
template <> struct PairOf<float2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct PairOf<double2> { typedef double type __attribute__((ext_vector_type(2))); };
template <typename V> __device__ __forceinline__ V ldg(const V* p) {
    const typename PairOf<V>::type v = *(const GLOBAL typename PairOf<V>::type*)p;
    V r;
    r.x = v.x;
    r.y = v.y;
    return r;
}
template <typename V> __device__ __forceinline__ void stg(V* p, const V& v) {
    typename PairOf<V>::type r;
    r.x = v.x;
    r.y = v.y;
    *(GLOBAL typename PairOf<V>::type*)p = r;
}

__device__ __forceinline__ void gatomic_add(float* p, float v) { __builtin_amdgcn_global_atomic_fadd_f32(gp(p), v); }
__device__ __forceinline__ void gatomic_add(double* p, double v) { __builtin_amdgcn_global_atomic_fadd_f64(gp(p), v); }

template <typename T> __device__ __forceinline__ int ifloor(T v) { return (int)floor(v); }

// Fixed-point accumulator of the LDS deposit window.  Float atomic adds on
// LDS run ~25x slower than integer ones on gfx950, so weights are rounded to
// integers at a power-of-two scale 2^S chosen per work item so that no node
// sum can overflow, summed exactly with integer LDS atomics, and converted
// back once when the window is added to the grid.  A sum of magnitude at most m
// takes S = SUM_BITS - bitlength(m): m 2^S <= 2^SUM_BITS - 2^S, and 2^S is more
// than the weights' rounding, half a unit each, adds up to.
template <typename T> struct Fixed;
template <> struct Fixed<float> {
    using I = int32_t;
    using U = uint32_t;
    static constexpr int BITS = 30, SUM_BITS = 31;
    __device__ static I quant(float v) { return (I)rintf(v); }
};
template <> struct Fixed<double> {
    using I = long long;
    using U = unsigned long long;
    static constexpr int BITS = 62, SUM_BITS = 63;
    __device__ static I quant(double v) { return (I)rint(v); }
};

// Exact round-to-nearest integer of |v| < 2^22 (float) or 2^51 (double): in
// v + 1.5 2^23 (resp. 1.5 2^52) the unit in the last place is 1, so the low
// mantissa bits of the sum hold round(v) offset by the magic constant.
template <typename T> struct Magic;
template <> struct Magic<float> {
    static constexpr float M = 12582912.0f;
    static constexpr int MAXS = 21;
    __device__ static int32_t take(float v) { return __float_as_int(v) - 0x4B400000; }
};
template <> struct Magic<double> {
    static constexpr double M = 6755399441055744.0;
    static constexpr int MAXS = 50;
    __device__ static long long take(double v) { return __double_as_longlong(v) - 0x4338000000000000LL; }
};

// floor(v + 1/2) as an integer in one instruction (|v| < 2^31).
__device__ __forceinline__ int round_half_up(float v) {
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// a * b + c for 0 <= a, b < 2^24 (24-bit multiply, full rate)
__device__ __forceinline__ int mad24(int a, int b, int c) { return (int)__umul24((unsigned)a, (unsigned)b) + c; }

// q = e / d, r = e % d for 0 <= e < 2^20, 0 < d < 2^10: float reciprocal
// estimate, corrected by one step.
__device__ __forceinline__ void divmod_small(int e, int d, float inv_d, int& q, int& r) {
    q = (int)((float)e * inv_d);
    r = e - q * d;
    if (r < 0) {
        --q;
        r += d;
    } else if (r >= d) {
        ++q;
        r -= d;
    }
}
// (i, j, k) of flat index e in a box of sizes (., ey, ez), row-major
__device__ __forceinline__ void unflatten3(int e, int ey, int ez, float inv_ez, float inv_ey, int& i, int& j, int& k) {
    int r;
    divmod_small(e, ez, inv_ez, r, k);
    divmod_small(r, ey, inv_ey, i, j);
}

template <typename T> __device__ __forceinline__ T wrap_box(T v, T L, T halfL, T invL) {
    return v - L * floor((v + halfL) * invL);
}

__device__ __forceinline__ int wave_min(int v) {
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ __forceinline__ int wave_max(int v) {
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// Bounds of up to three small signed values over a workgroup of NW waves, in
// one barrier.  Each value c travels as the 16-bit pair (c, -c), whose
// pairwise minimum gives the lower bound and minus the upper one, through the
// lanes of a wave by DPP moves (a lane-shuffle reduction of six separate
// values goes through LDS 36 times); one 16-byte LDS word per wave then
// combines the waves.  sh: NW int4, read until the caller's next barrier.
typedef short short2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int pk_bounds(int c) { return (c & 0xFFFF) | (int)((unsigned)(-c) << 16); }
__device__ __forceinline__ int pk_min(int a, int b) {
    return __builtin_bit_cast(int, __builtin_elementwise_min(__builtin_bit_cast(short2v, a), __builtin_bit_cast(short2v, b)));
}
__device__ __forceinline__ int pk_lo(int v) { return (int)(short)(v & 0xFFFF); }
__device__ __forceinline__ int pk_hi(int v) { return -(v >> 16); }
// lane 63 receives the minimum over the wave
__device__ __forceinline__ int wave_pk_min(int v) {
    v = pk_min(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));  // row_shr 1, 2, 4, 8
    v = pk_min(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = pk_min(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = pk_min(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = pk_min(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));  // row_bcast 15, 31
    v = pk_min(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return v;
}
constexpr int BOUNDS_NONE = 0x7FFF7FFF;  // of no value: the pairwise minimum's identity
// lane 63 receives the maximum of non-negative v over the wave
__device__ __forceinline__ int wave_max_dpp(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x143, 0xc, 0xf, false));
    return v;
}
// The bounds of three values (as block_bounds3) and the maximum of m >= 0
template <int NW> __device__ __forceinline__ int block_bounds3_max(int& x, int& y, int& z, int m, int4* sh) {
    const int bx = wave_pk_min(x), by = wave_pk_min(y), bz = wave_pk_min(z), bm = wave_max_dpp(m);
    if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = make_int4(bx, by, bz, bm);
    __syncthreads();
    int4 r = sh[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        const int4 v = sh[w];
        r.x = pk_min(r.x, v.x);
        r.y = pk_min(r.y, v.y);
        r.z = pk_min(r.z, v.z);
        r.w = max(r.w, v.w);
    }
    x = __builtin_amdgcn_readfirstlane(r.x);
    y = __builtin_amdgcn_readfirstlane(r.y);
    z = __builtin_amdgcn_readfirstlane(r.z);
    return __builtin_amdgcn_readfirstlane(r.w);
}
template <int NW> __device__ __forceinline__ void block_bounds3(int& x, int& y, int& z, int4* sh) {
    const int bx = wave_pk_min(x), by = wave_pk_min(y), bz = wave_pk_min(z);
    if ((threadIdx.x & 63) == 63) sh[threadIdx.x >> 6] = make_int4(bx, by, bz, 0);
    __syncthreads();
    int4 r = sh[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
        const int4 v = sh[w];
        r.x = pk_min(r.x, v.x);
        r.y = pk_min(r.y, v.y);
        r.z = pk_min(r.z, v.z);
    }
    x = __builtin_amdgcn_readfirstlane(r.x);
    y = __builtin_amdgcn_readfirstlane(r.y);
    z = __builtin_amdgcn_readfirstlane(r.z);
}

// Window along one axis covering relative cells [lo, hi] of a chunk whose
// reference cell is r: origin and width, or the whole axis when it would wrap.
__device__ __forceinline__ void axis_window(int r, int lo, int hi, int H, int& o, int& W) {
    const int w = hi - lo + 1;
    if (w >= H) {
        o = 0;
        W = H;
    } else {
        o = (r + lo) & (H - 1);
        W = w;
    }
}

// Periodic grid index onto [0, H), for any int argument: a mask when H is a
// power of two, else one conditional step each way (arguments of the passes lie
// within a period or two of the grid) and, past that, the quotient in FP64
// (exact for every int up to the step that follows).  An integer remainder is
// some 40 instructions and a particle takes about a dozen wraps.
template <bool P2> struct Wrap {
    int H, m;  // m = H - 1
    __device__ __forceinline__ int operator()(int v) const {
        if constexpr (P2) {
            return v & m;
        } else {
            int r = v < 0 ? v + H : v;
            r = r >= H ? r - H : r;
            if ((unsigned)r >= (unsigned)H) {
                r = v - H * (int)floor((double)v * (1.0 / (double)H));
                r = r < 0 ? r + H : r;
                r = r >= H ? r - H : r;
            }
            return r;
        }
    }
};

// Window cells along one axis: n cells from relative cell o for an item whose
// cells span [lo, hi] (mean: about `mean`), wanted with m cells of margin on
// both sides, on a grid of H cells with at most `most` cells in the window.
// Cells that find no room are the item's outermost ones.
__device__ __forceinline__ void window_axis(int lo, int hi, int m, int mean, int most, int H, int& o, int& n) {
    const int nb = hi - lo + 1;
    n = min(min(nb + 2 * m, most), H);
    o = lo - (n - nb) / 2;  // spare cells on both sides
    if (nb > n) o = max(lo, min(hi - n + 1, mean - n / 2));
}

// Work queue of the persistent item passes.  The item list's header holds the
// item count n (hdr[0], written by the sort) and a ticket counter (hdr[1],
// zero between launches).  Workgroup b takes item b first; with more items
// than workgroups it then draws tickets t for item grid + t, in list order,
// until a draw is past the end, so items of uneven cost spread over the
// workgroups that free up first.  Each workgroup's last draw is that failing
// one, hence a launch draws exactly n tickets and the draw that returns n - 1
// is its last: it puts the counter back to zero.  Launches that share a
// header must not overlap (they run on one stream).  Call with the whole
// workgroup after an item; returns the next item (>= n: none).
__device__ __forceinline__ int next_item(int* hdr, int n, int* slot) {
    const int grid = (int)gridDim.x;
    if (n <= grid) return n;
    __syncthreads();  // the item's use of LDS has ended
    if (threadIdx.x == 0) {
        const int t = atomicAdd(hdr + 1, 1);
        if (t == n - 1) atomicExch(hdr + 1, 0);
        *slot = grid + t;
    }
    __syncthreads();
    return *slot;
}

// The same queue with the draw ahead of time: draw() once per item, by the
// whole workgroup and after a barrier of that item (other waves may still be
// reading the last draw; the box's reduction has one), wherever its round trip
// is covered by work that waits for no other memory; next() after the item.
struct Ticket {
    int* hdr;
    int n;
    int* slot;
    __device__ __forceinline__ void draw() const {
        if (n > (int)gridDim.x && threadIdx.x == 0) {
            const int t = atomicAdd(hdr + 1, 1);
            if (t == n - 1) atomicExch(hdr + 1, 0);
            *slot = (int)gridDim.x + t;
        }
    }
    __device__ __forceinline__ int next() const {
        if (n <= (int)gridDim.x) return n;
        __syncthreads();  // the item's use of LDS has ended, the slot is written
        return *slot;
    }
};

}  // namespace sipf
