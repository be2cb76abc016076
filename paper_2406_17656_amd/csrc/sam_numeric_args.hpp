// sam_numeric_args.hpp -- the interface of the numeric least-squares kernels
// (internal to the library): their arguments, the kernel variants and the
// compiled menu.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace samk {

struct NumericArgs {
    int n;
    // extents of the arrays the kernels read through 32-bit buffer offsets
    // (the plan guarantees nnz(A_k) * 8, nnz(A_0) * 8 and E below 2^32)
    uint32_t nnzA, nnzA0, E;
    const int* Ak_cp;
    const double* Ak_v;
    const int* A0_cp;
    const double* A0_v;
    const int* S_cp;
    const int* S_ri;
    const int* nI;
    const int64_t* eoff;
    const unsigned char* posA;
    const unsigned char* posB;
    const int* queue;     // all buckets' columns
    const int* bstart;    // device, bucket offsets
    int bucket;           // which bucket this launch serves
    void* M;
    double* col_res2;     // n or nullptr
    // per-block partial sums of the column residuals (the launch's blocks
    // write part[part_base + block]); nullptr: none
    double* part;
    int part_base;
    unsigned long long* status;
    // soft weights (nullptr for the plain map)
    const double* w;
    double mu;
    // adjoint outputs (backward launches only)
    double dL;
    const double* dL_dev; // the scale on the device instead (may be null)
    double* contrib;      // per gathered entry, at eoff[j] + offset in the block
    int64_t* segoff;      // per S entry: where its column's contributions start
    double* gA0;          // nnz(A_0)
    double* gw;           // nnz(S) or nullptr
};

// One kernel variant of the menu: solves every column of one bucket whose
// block fits max_rows x max_cols.
struct NumericVariant {
    int prec;        // 0 = FP64, 1 = FP32 + refinement
    int G;           // lanes per column problem
    int R;           // rows per lane
    int NC;          // max columns
    int weighted;    // 1: stacked penalty rows
    int TC;          // columns staged per LDS tile pass
    int LPL;         // entries per lane and column moved with static indices
    hipError_t (*launch)(const NumericArgs&, int grid, hipStream_t);
    hipError_t (*launch_backward)(const NumericArgs&, int grid, hipStream_t);  // weighted only
    int (*blocks_per_cu)();  // resident one-wave blocks per CU of the forward kernel (0: unknown)
    // the plain launch for matrices most of whose columns are longer than
    // G * LPL entries (one more entry per lane in registers; null: the same)
    hipError_t (*launch_long)(const NumericArgs&, int grid, hipStream_t);
    int (*blocks_per_cu_long)();
    // measured cost of a plain launch (0: not measured): one round of blocks
    // (us), and a column once the GPU is full (ns); then the same on such
    // matrices
    float round_us, col_ns, round_us_long, col_ns_long;
    // the plain form for few columns: more lanes a problem, the same blocks or
    // larger (null: none), and the waves a SIMD up to which it is the faster
    const NumericVariant* few;
    int few_waves;
    int max_rows() const { return G * R; }
    int per_wave() const { return 64 / G; }
    int64_t few_columns(int CUs) const { return few ? (int64_t)4 * few_waves * CUs * few->per_wave() : 0; }
    // Columns longer than the lanes hold take a memory loop, a load at a time.
    // A few of them (boundary rows, one dense column) are cheaper left to it
    // than an entry more per lane for all: most columns have to be that long.
    bool long_columns(int64_t n, int64_t nnzA, int longest) const {
        return longest > G * LPL && nnzA >= (int64_t)(G * LPL - 1) * n;
    }
};
// The compiled menu, ordered from the cheapest per column to the most
// general for each precision.
const NumericVariant* numeric_menu(int* count);

// Blocks of a launch over `groups` groups, at most `cap` (a multiple of 8):
// from 64 on a multiple of 8, as the XCD-aware block order wants, rounded up
// (a block without a group ends at once).  Rounded down, a launch of 125
// groups ran 120 blocks, five of them for two rounds: 1000 columns took 23.5
// us where 1024 took 13.1.
inline int launch_grid(int64_t groups, int cap) {
    const int64_t up = groups >= 64 ? (groups + 7) / 8 * 8 : groups;
    return (int)(up < cap ? up : cap);
}

}  // namespace samk
