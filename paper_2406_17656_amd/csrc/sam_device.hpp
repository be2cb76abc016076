// sam_device.hpp -- device helpers shared by the gfx950 kernels of the SAM
// library: wave64 group reductions built on DPP row/quad permutations, the
// per-context status word, and small integer utilities.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace samk {

constexpr int kWave = 64;

// Status codes (same numeric values as sam_status in include/sam.h).
constexpr int kStRank = 5;
constexpr int kStNonfinite = 6;
constexpr int kStIndex = 3;
constexpr int kStUnsupported = 8;

// The status word keeps the earliest failing column: (col << 8) | code,
// reduced with atomicMin.  0x7fff... means "no failure".
__device__ inline void report(unsigned long long* status, int col, int code) {
    unsigned long long v = ((unsigned long long)(unsigned)col << 8) | (unsigned)code;
    atomicMin(status, v);
}

// ---------------------------------------------------------------------------
// DPP lane exchanges inside a wave64.  Controls (GCN/CDNA DPP encoding):
//   quad_perm [1,0,3,2] = 0xB1   (xor 1)
//   quad_perm [2,3,0,1] = 0x4E   (xor 2)
//   row_half_mirror     = 0x141  (lane i <-> 7-i inside each 8-lane half row)
//   row_mirror          = 0x140  (lane i <-> 15-i inside each 16-lane row)
// After the quad stages every lane of a quad holds the quad value, so a
// mirror stage pairs each lane with one holding the other half's value; the
// resulting sums are identical in every lane of the group (a + b == b + a).
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ inline int dpp_i32(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}

template <int CTRL>
__device__ inline float dpp(float v) {
    return __int_as_float(dpp_i32<CTRL>(__float_as_int(v)));
}

template <int CTRL>
__device__ inline double dpp(double v) {
    int2 p = *reinterpret_cast<int2*>(&v);
    int2 q;
    q.x = dpp_i32<CTRL>(p.x);
    q.y = dpp_i32<CTRL>(p.y);
    return *reinterpret_cast<double*>(&q);
}

// xor-8 exchange inside 32-lane halves (ds_swizzle bitmask mode:
// and_mask = 0x1F, or_mask = 0, xor_mask = 0x08): the LDS pipe's form of the
// last exchange of a 16-lane sum.
__device__ inline float xor8(float v) {
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x201F));
}
// xor-16 exchange inside 32-lane halves (ds_swizzle bitmask mode:
// and_mask = 0x1F, or_mask = 0, xor_mask = 0x10).
__device__ inline float xor16(float v) {
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 0x401F));
}
__device__ inline double xor16(double v) {
    int2 p = *reinterpret_cast<int2*>(&v);
    int2 q;
    q.x = __builtin_amdgcn_ds_swizzle(p.x, 0x401F);
    q.y = __builtin_amdgcn_ds_swizzle(p.y, 0x401F);
    return *reinterpret_cast<double*>(&q);
}
__device__ inline float xor32(float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute((int)((threadIdx.x ^ 32) << 2), __float_as_int(v)));
}
__device__ inline double xor32(double v) {
    int2 p = *reinterpret_cast<int2*>(&v);
    int2 q;
    int a = (int)((threadIdx.x ^ 32) << 2);
    q.x = __builtin_amdgcn_ds_bpermute(a, p.x);
    q.y = __builtin_amdgcn_ds_bpermute(a, p.y);
    return *reinterpret_cast<double*>(&q);
}

// Sum over the G consecutive lanes of a group (G in 1,2,4,...,64); every
// lane of the group receives the same value.
template <int G, typename T>
__device__ inline T group_sum(T v) {
    if constexpr (G >= 2) v += dpp<0xB1>(v);
    if constexpr (G >= 4) v += dpp<0x4E>(v);
    if constexpr (G >= 8) v += dpp<0x141>(v);
    if constexpr (G >= 16) v += dpp<0x140>(v);
    if constexpr (G >= 32) v += xor16(v);
    if constexpr (G >= 64) v += xor32(v);
    return v;
}

// group_sum for FP32 with the exchange between the two 8-lane halves of a
// 16-lane group taken through the LDS pipe (ds_swizzle) instead of a DPP move
// and an add on the VALU: for kernels whose VALU is saturated and whose sums
// are not on the critical path.  The result equals group_sum's (each lane
// adds the same two half sums).
template <int G>
__device__ inline float group_sum_x(float v) {
    if constexpr (G == 16) {
        v += dpp<0xB1>(v);
        v += dpp<0x4E>(v);
        v += dpp<0x141>(v);
        return v + xor8(v);
    } else {
        return group_sum<G>(v);
    }
}

template <int G, typename T>
__device__ inline T group_max(T v) {
    if constexpr (G >= 2) v = fmax(v, dpp<0xB1>(v));
    if constexpr (G >= 4) v = fmax(v, dpp<0x4E>(v));
    if constexpr (G >= 8) v = fmax(v, dpp<0x141>(v));
    if constexpr (G >= 16) v = fmax(v, dpp<0x140>(v));
    if constexpr (G >= 32) v = fmax(v, xor16(v));
    if constexpr (G >= 64) v = fmax(v, xor32(v));
    return v;
}

// Value of lane `src` (0 <= src < G) of the caller's group, in every lane of
// the group: the other lanes contribute an exact zero to a group sum.
template <int G, typename T>
__device__ inline T group_bcast(T v, int g, int src) {
    // groups of 2 or 4 lanes: one quad_perm move; src is a constant once the
    // caller's loop is unrolled, so the switch folds away
    if constexpr (G == 1) {
        return v;
    } else if constexpr (G == 2) {
        return (src & 1) ? dpp<0xF5>(v) : dpp<0xA0>(v);  // [1,1,3,3] / [0,0,2,2]
    } else if constexpr (G == 4) {
        switch (src & 3) {
            case 0: return dpp<0x00>(v);  // [0,0,0,0]
            case 1: return dpp<0x55>(v);  // [1,1,1,1]
            case 2: return dpp<0xAA>(v);  // [2,2,2,2]
            default: return dpp<0xFF>(v); // [3,3,3,3]
        }
    } else {
        return group_sum<G>(g == src ? v : T(0));
    }
}

template <int CTRL>
__device__ inline int dppi(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false); }
template <int CTRL>
__device__ inline int dppb(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }

// Integer sums / minima / maxima over the GS = 8 or 16 lanes of a group (all
// lanes get the result): quad exchanges, then the half-row mirror, then (GS = 16) the row
// mirror
template <int GS>
__device__ inline int grp_sum(int v) {
    v += dppb<0xB1>(v);
    v += dppb<0x4E>(v);
    v += dppb<0x141>(v);
    if (GS == 16) v += dppb<0x140>(v);
    return v;
}
template <int GS>
__device__ inline int grp_min(int v) {
    v = min(v, dppb<0xB1>(v));
    v = min(v, dppb<0x4E>(v));
    v = min(v, dppb<0x141>(v));
    if (GS == 16) v = min(v, dppb<0x140>(v));
    return v;
}
template <int GS>
__device__ inline int grp_max(int v) {
    v = max(v, dppb<0xB1>(v));
    v = max(v, dppb<0x4E>(v));
    v = max(v, dppb<0x141>(v));
    if (GS == 16) v = max(v, dppb<0x140>(v));
    return v;
}
// exclusive prefix sum inside the group (Kogge-Stone with row_shr; a lane
// whose source lies before its group's first lane adds 0)
template <int GS>
__device__ inline int grp_excl_scan(int v) {
    const int p = (int)(threadIdx.x & (GS - 1));
    int x = v, y;
    y = dppi<0x111>(x);
    x += (GS == 16 || p >= 1) ? y : 0;
    y = dppi<0x112>(x);
    x += (GS == 16 || p >= 2) ? y : 0;
    y = dppi<0x114>(x);
    x += (GS == 16 || p >= 4) ? y : 0;
    if (GS == 16) x += dppi<0x118>(x);
    return x - v;
}

// The number of this block in a launch over flat_grid (sam_kernels.hpp).
__device__ inline int64_t flat_block() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

__device__ inline int wave_lane() { return (int)(threadIdx.x & 63); }

// Wave-level barrier for LDS traffic that stays inside one wavefront.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Row i of M x over the row view, by the kSpmvLanes consecutive lanes of the
// row, so that the lanes of a wave read each row's column indices (and values)
// as one contiguous run instead of one entry of 64 different rows.  Lane g
// sums entries g, g + 4, ... of the row in ascending order; the four partials
// are added by the quad exchanges of group_sum (the same order on every call).
// Each lane issues the loads of kSpmvUnroll of its entries (indices and
// values, then the x values they select) before it adds them, so a row of up
// to 16 entries costs two dependent round trips instead of two per entry;
// slots past the row's end load a valid entry of the row with a zero value,
// which adds an exact zero.  Every lane takes part; rows with live = false
// give 0.
// PERM: the values are read through the row view's permutation (else they
// are in the row view's order).  SCALE: x is scale .* x.  DIV: x is x / div
// (before the scale).
constexpr int kSpmvLanes = 4;
constexpr int kSpmvUnroll = 4;
template <bool F32, bool PERM, bool SCALE, bool DIV = false>
__device__ inline double row_product(bool live, int i, const int* rowptr, const int* colind, const int* perm,
                                     const void* val, const double* x, const double* scale, double div = 1.0) {
    const int g = threadIdx.x % kSpmvLanes;
    double s = 0.0;
    if (live) {
        const unsigned b = (unsigned)rowptr[i + 1];   // unsigned: steps past 2^31 - 1 entries stay in range
        for (unsigned e = (unsigned)rowptr[i] + g; e < b; e += kSpmvLanes * kSpmvUnroll) {
            int c[kSpmvUnroll];
            double v[kSpmvUnroll], xv[kSpmvUnroll];
#pragma unroll
            for (int u = 0; u < kSpmvUnroll; ++u) {
                const unsigned eu = e + u * kSpmvLanes < b ? e + u * kSpmvLanes : e;   // e < b: in the row
                c[u] = colind[eu];
                const unsigned ev = PERM ? (unsigned)perm[eu] : eu;
                v[u] = F32 ? (double)static_cast<const float*>(val)[ev] : static_cast<const double*>(val)[ev];
            }
#pragma unroll
            for (int u = 0; u < kSpmvUnroll; ++u) {
                xv[u] = DIV ? x[c[u]] / div : x[c[u]];
                if (SCALE) xv[u] = scale[c[u]] * xv[u];
            }
#pragma unroll
            for (int u = 0; u < kSpmvUnroll; ++u) s = fma(e + u * kSpmvLanes < b ? v[u] : 0.0, xv[u], s);
        }
    }
    return group_sum<kSpmvLanes>(s);
}

template <typename T>
__device__ inline bool finite_val(T x) { return isfinite(x); }

}  // namespace samk
