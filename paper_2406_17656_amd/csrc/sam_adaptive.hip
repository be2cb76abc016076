// sam_adaptive.hip -- adjoint-guided pattern adaptation, the direction the
// paper leaves for future work (adaptive patterns in parallel environments,
// end of Section 2; more refined sparsification, Section 6): the entries
// of a candidate pattern S (a higher level) that are not in the base pattern
// B carry soft weights w < 1; the gradient of the loss with respect to w
// ranks them, and each column keeps its base entries plus the k candidates
// whose admission lowers the loss fastest (most negative dL/dw).
//
// Columns hold tens of entries, so the rank of a candidate is counted directly
// over its column (no sort).
#include "sam_device.hpp"
#include "sam_kernels.hpp"

#include <climits>
#include <cmath>

namespace samk {

namespace {

// w[e] = w_base where row S_ri[e] of column j is in B(:, j), else w_cand
// (both columns ascending: one merge).
__global__ void k_candidate_weights(int n, const int* S_cp, const int* S_ri, const int* B_cp, const int* B_ri,
                                    double w_base, double w_cand, double* w) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    int f = B_cp[j];
    const int fb = B_cp[j + 1];
    for (int e = S_cp[j]; e < S_cp[j + 1]; ++e) {
        const int r = S_ri[e];
        while (f < fb && B_ri[f] < r) ++f;
        w[e] = (f < fb && B_ri[f] == r) ? w_base : w_cand;
    }
}

// Order of candidates: smaller gradient first (NaN counts as +inf), ties to
// the smaller row.
__device__ inline bool ahead(double ga, int ra, double gb, int rb) {
    ga = isnan(ga) ? INFINITY : ga;
    gb = isnan(gb) ? INFINITY : gb;
    return ga < gb || (ga == gb && ra < rb);
}

// A group of lanes per column, a lane per entry: its rank among the
// candidates comes from one pass over the column, staged in LDS (columns
// longer than kTopkStage are read from memory).  A thread per column read its
// entries once per candidate, each read waiting for the one before: 49 us for
// the 65536 columns of 13 entries of a 256^2 five-point level-2 pattern, now
// 11 us.
constexpr int kTopkThreads = 256;
constexpr int kTopkLanes = 16;
constexpr int kTopkStage = 64;

template <bool FILL>
__global__ void __launch_bounds__(kTopkThreads)
k_topk(int n, const int* S_cp, const int* S_ri, const double* w, const double* grad, int k,
       int* counts, const int* out_cp, int* out_ri) {
    constexpr int kGroups = kTopkThreads / kTopkLanes;
    __shared__ double grad_sh[kGroups][kTopkStage];
    __shared__ int row_sh[kGroups][kTopkStage];   // INT_MIN: not a candidate
    const int grp = threadIdx.x / kTopkLanes, g = threadIdx.x % kTopkLanes;
    const int64_t j = flat_block() * kGroups + grp;
    if (j >= n) return;   // whole groups; no block barrier below
    const int a = S_cp[j], b = S_cp[j + 1], len = b - a;
    const bool staged = len <= kTopkStage;
    if (staged) {
        for (int x = g; x < len; x += kTopkLanes) {
            grad_sh[grp][x] = grad[a + x];
            row_sh[grp][x] = w[a + x] < 1.0 ? S_ri[a + x] : INT_MIN;
        }
        wave_sync();
    }
    int o = FILL ? out_cp[j] : 0;
    int kept = 0;
    for (int x0 = 0; x0 < len; x0 += kTopkLanes) {   // the same for all lanes of a group
        const int x = x0 + g;
        bool keep = false;
        if (x < len) {
            keep = w[a + x] >= 1.0;
            if (!keep) {
                int rank = 0;
                const double ge = grad[a + x];
                const int re = S_ri[a + x];
                if (staged) {
                    for (int f = 0; f < len; ++f)
                        rank += f != x && row_sh[grp][f] != INT_MIN && ahead(grad_sh[grp][f], row_sh[grp][f], ge, re);
                } else {
                    for (int f = 0; f < len && rank < k; ++f)
                        rank += f != x && w[a + f] < 1.0 && ahead(grad[a + f], S_ri[a + f], ge, re);
                }
                keep = rank < k;
            }
        }
        const unsigned long long m = __ballot(keep) >> (wave_lane() / kTopkLanes * kTopkLanes);
        const unsigned mine = (unsigned)(m & ((1u << kTopkLanes) - 1u));
        if (FILL && keep) out_ri[o + kept + __popc(mine & ((1u << g) - 1u))] = S_ri[a + x];
        kept += __popc(mine);
    }
    if (!FILL && g == 0) counts[j] = kept;
}

dim3 topk_grid(int n) {
    constexpr int kGroups = kTopkThreads / kTopkLanes;
    return flat_grid((n - 1) / kGroups + 1);
}

}  // namespace

hipError_t candidate_weights(int n, const int* S_cp, const int* S_ri, const int* B_cp, const int* B_ri,
                             double w_base, double w_cand, double* w, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_candidate_weights, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, S_cp, S_ri,
                       B_cp, B_ri, w_base, w_cand, w);
    return hipGetLastError();
}

hipError_t topk_count(int n, const int* S_cp, const int* S_ri, const double* w, const double* grad, int k,
                      int* counts, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_topk<false>, topk_grid(n), dim3(kTopkThreads), 0, s, n, S_cp, S_ri, w, grad,
                       k, counts, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t topk_fill(int n, const int* S_cp, const int* S_ri, const double* w, const double* grad, int k,
                     const int* out_cp, int* out_ri, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_topk<true>, topk_grid(n), dim3(kTopkThreads), 0, s, n, S_cp, S_ri, w, grad,
                       k, nullptr, out_cp, out_ri);
    return hipGetLastError();
}

}  // namespace samk
