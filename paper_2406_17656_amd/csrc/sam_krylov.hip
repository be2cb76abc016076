// sam_krylov.hip -- gfx950 kernels of one Arnoldi step of right-preconditioned
// GMRES on A_k with the map (Section 1: the map updates a preconditioner):
//     z = N (d .* v_k),  w = A z,  orthogonalise w against v_0 .. v_k,
//     v_{k+1} = w / ||w||,  and the Givens rotation of the new column of H.
//
// The orthogonalisation is classical Gram-Schmidt taken twice: all dot
// products of a pass in one kernel, all updates in the next, so a step is four
// launches whatever k is, six beyond kInlineChunks chunks (modified Gram-Schmidt
// needs a reduction over the whole vector per earlier vector), and the basis is
// orthogonal to rounding.
//
// A chunk of rows per block of 16 waves: the block that forms w (or subtracts a
// pass) goes straight on to its chunk's share of the next dot products.  The
// kernels are bound by the latency of their dependent loads, so a row has
// four threads: four lanes of its product with A, then a quarter of the basis
// vectors each: 25 us per step of a 128 x 128 system with a level-2 FP64 map
// (mean over a cycle of 50; 36 us with one thread per row, and 900 us with one
// host-synchronised dot product per earlier vector).  Every sum
// has a fixed order (lanes, waves, chunks), so runs are bitwise repeatable.
//
// The residual test runs on the device: once it holds, `done` is set and the
// launches already enqueued return at once, so the host looks only now and
// then.  state: [0] steps done, [1] done, [2 + i] |residual| after step i,
// [2 + restart + i] the rotated right side g.
#include "sam_device.hpp"
#include "sam_kernels.hpp"

#include <algorithm>

namespace samk {

namespace {

constexpr int kRows = 256;          // rows of a chunk in flight
constexpr int kParts = 4;           // threads per row
constexpr int kThreads = kRows * kParts;
static_assert(kParts == kSpmvLanes, "k_gm_apply_dots gives a row of its product the threads of a row");
constexpr int kRowWaves = kRows / 64;
constexpr int kFlat = 256;          // threads per block of the kernels without chunks
constexpr int kTile = 8;            // basis vectors whose loads are in flight together
// Up to here every block sums the chunks' partials itself, one load per lane
// and product; beyond it a launch does, twice a step.  Microseconds per step of a
// cycle of 50, every block against a launch: 33.0 / 35.8 at 64 chunks (n = 16384),
// 34.1 / 36.4 at 67, 35.5 / 37.3 at 128, 38.5 / 38.7 at 256 and 55.4 / 53.0 at 512
// (the blocks' reads grow with the square of the chunks).
constexpr int kInlineChunks = 64;
constexpr int kMaxChunks = 1024;

// Rows [r0, r1) of this block's chunk (unsigned: a step past the last row stays
// in range up to n = 2^31 - 1).
__device__ inline void chunk_range(int n, unsigned& r0, unsigned& r1) {
    const int64_t c = gridDim.x, b = blockIdx.x;
    r0 = (unsigned)(n * b / c);
    r1 = (unsigned)(n * (b + 1) / c);
}

// part[j * chunks + block] = sum over the chunk of v_j w, j in [0, count).
// Thread part p takes the tiles p, p + 4, ... of kTile vectors.  sh:
// kRowWaves * count doubles.
__device__ inline void chunk_dots(int n, unsigned r0, unsigned r1, int count, const double* V, const double* w, double* part,
                                  double* sh) {
    const int row = threadIdx.x % kRows, wv = row >> 6;
    for (int j0 = threadIdx.x / kRows * kTile; j0 < count; j0 += kParts * kTile) {
        double acc[kTile];
#pragma unroll
        for (int u = 0; u < kTile; ++u) acc[u] = 0.0;
        for (unsigned r = r0 + row; r < r1; r += kRows) {
            const double x = w[r];
#pragma unroll
            for (int u = 0; u < kTile; ++u)   // past the last vector: v_0 again, not stored
                acc[u] += V[(int64_t)(j0 + u < count ? j0 + u : 0) * n + r] * x;
        }
#pragma unroll
        for (int u = 0; u < kTile; ++u) {
            const double s = group_sum<64>(acc[u]);
            if (wave_lane() == 0 && j0 + u < count) sh[wv * count + j0 + u] = s;
        }
    }
    __syncthreads();
    for (int j = threadIdx.x; j < count; j += kThreads) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < kRowWaves; ++q) s += sh[q * count + j];
        part[(int64_t)j * gridDim.x + blockIdx.x] = s;
    }
}

// The sum over one wave of chunks values, the same in every lane.
__device__ inline double wave_sum_of(const double* p, int chunks) {
    double s = 0.0;
    for (int c = wave_lane(); c < chunks; c += 64) s += p[c];
    return group_sum<64>(s);
}

// h[j] for j in [0, count) into LDS: from the chunks' partials, or already
// summed (chunks = 0).
__device__ inline void load_coefficients(int count, int chunks, const double* src, double* h) {
    if (chunks == 0) {
        for (int j = threadIdx.x; j < count; j += kThreads) h[j] = src[j];
    } else {
        for (int j = threadIdx.x >> 6; j < count; j += kThreads / 64) {
            const double s = wave_sum_of(src + (int64_t)j * chunks, chunks);
            if (wave_lane() == 0) h[j] = s;
        }
    }
    __syncthreads();
}

// w -= sum_j h_j v_j on the chunk: a quarter of the vectors per thread of a
// row, the four sums added in order.  visit(w) sees every new entry, in the
// threads of part 0.  ps: kThreads doubles.
template <typename F>
__device__ inline void chunk_subtract(int n, unsigned r0, unsigned r1, int count, const double* V, const double* h, double* w,
                                      double* ps, F visit) {
    const int row = threadIdx.x % kRows, p = threadIdx.x / kRows;
    const int ja = count * p / kParts, jb = count * (p + 1) / kParts;
    for (unsigned b = r0; b < r1; b += kRows) {   // the same trips for every thread
        const unsigned r = b + row;
        double x = 0.0;
        if (r < r1) {
            int j = ja;
            for (; j + kTile <= jb; j += kTile) {
                double v[kTile];
#pragma unroll
                for (int u = 0; u < kTile; ++u) v[u] = V[(int64_t)(j + u) * n + r];
#pragma unroll
                for (int u = 0; u < kTile; ++u) x += h[j + u] * v[u];
            }
            if (j < jb) {   // the rest, loads together
                double v[kTile];
#pragma unroll
                for (int u = 0; u < kTile; ++u) v[u] = V[(int64_t)(j + u < jb ? j + u : j) * n + r];
#pragma unroll
                for (int u = 0; u < kTile; ++u) x += j + u < jb ? h[j + u] * v[u] : 0.0;
            }
        }
        ps[threadIdx.x] = x;
        __syncthreads();
        if (p == 0 && r < r1) {
            double s = ps[row];
#pragma unroll
            for (int q = 1; q < kParts; ++q) s += ps[q * kRows + row];
            const double y = w[r] - s;
            w[r] = y;
            visit(y);
        }
        __syncthreads();
    }
}

__global__ void k_gm_init(int restart, double beta, double* state) {
    for (int i = threadIdx.x; i < 2 + 2 * restart + 1; i += blockDim.x) state[i] = i == 2 + restart ? beta : 0.0;
}

// z = N (d .* v), or d .* v without a map.
template <bool MAP, bool F32>
__global__ void __launch_bounds__(kFlat)
k_gm_precond(int n, const int* rowptr, const int* colind, const void* val, const double* d, const double* v,
             double* z, const double* state) {
    if (state[1] != 0.0) return;
    const int64_t t = flat_block() * kFlat + threadIdx.x;
    if constexpr (MAP) {
        const int64_t i = t / kSpmvLanes;
        const double s = row_product<F32, false, true>(i < n, (int)i, rowptr, colind, nullptr, val, v, d);
        if (i < n && t % kSpmvLanes == 0) z[i] = s;
    } else if (t < n) {
        z[t] = d[t] * v[t];
    }
}

// w = A z on the chunk, then its dot products with v_0 .. v_{count-1}.
__global__ void __launch_bounds__(kThreads)
k_gm_apply_dots(int n, const int* rowptr, const int* colind, const double* val, const double* z, double* w, int count,
                const double* V, double* part, const double* state) {
    if (state[1] != 0.0) return;
    extern __shared__ double sh[];
    unsigned r0, r1;
    chunk_range(n, r0, r1);
    for (unsigned t = threadIdx.x; t < (r1 - r0 + kRows - 1) / kRows * kThreads; t += kThreads) {   // whole blocks
        const unsigned i = r0 + t / kSpmvLanes;
        const double s = row_product<false, false, false>(i < r1, (int)i, rowptr, colind, nullptr, val, z, nullptr);
        if (i < r1 && t % kSpmvLanes == 0) w[i] = s;
    }
    __syncthreads();
    chunk_dots(n, r0, r1, count, V, w, part, sh);
}

// h[j] = sum over the chunks (more than kInlineChunks of them).
__global__ void __launch_bounds__(64)
k_gm_reduce(int chunks, const double* part, double* h, const double* state) {
    if (state[1] != 0.0) return;
    const double s = wave_sum_of(part + (int64_t)blockIdx.x * chunks, chunks);
    if (threadIdx.x == 0) h[blockIdx.x] = s;
}

// First pass subtracted, then the second pass's dot products.
__global__ void __launch_bounds__(kThreads)
k_gm_update_dots(int n, int count, int chunks, const double* src, const double* V, double* w, double* h1,
                 double* part, const double* state) {
    if (state[1] != 0.0) return;
    extern __shared__ double sh[];
    __shared__ double ps[kThreads];
    double* h = sh + kRowWaves * count;
    load_coefficients(count, chunks, src, h);
    if (blockIdx.x == 0)
        for (int j = threadIdx.x; j < count; j += kThreads) h1[j] = h[j];
    unsigned r0, r1;
    chunk_range(n, r0, r1);
    chunk_subtract(n, r0, r1, count, V, h, w, ps, [](double) {});
    chunk_dots(n, r0, r1, count, V, w, part, sh);
}

// Second pass subtracted, the chunk's share of ||w||^2, and H's raw column.
__global__ void __launch_bounds__(kThreads)
k_gm_update_norm(int n, int count, int chunks, const double* src, const double* V, double* w, const double* h1,
                 double* Hcol, double* nrm, const double* state) {
    if (state[1] != 0.0) return;
    extern __shared__ double h[];
    __shared__ double ps[kThreads];
    __shared__ double ws[kRowWaves];
    load_coefficients(count, chunks, src, h);
    if (blockIdx.x == 0)
        for (int j = threadIdx.x; j < count; j += kThreads) Hcol[j] = h1[j] + h[j];
    unsigned r0, r1;
    chunk_range(n, r0, r1);
    double s = 0.0;
    chunk_subtract(n, r0, r1, count, V, h, w, ps, [&](double y) { s += y * y; });
    if (threadIdx.x < kRows) {
        s = group_sum<64>(s);
        if (wave_lane() == 0) ws[threadIdx.x >> 6] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int q = 0; q < kRowWaves; ++q) t += ws[q];
        nrm[blockIdx.x] = t;
    }
}

// Givens rotation of H's column k (its first k + 1 entries; hn = ||w|| below
// them) and of the right side; one block, sh: 3 (k + 1) doubles.
__device__ inline void rotate_column(int k, int restart, double hn, double* Hcol, double* cs, double* sn, double tol,
                                     double* state, double* sh) {
    double *hc = sh, *c = sh + k + 1, *d = c + k + 1;
    for (int i = threadIdx.x; i <= k; i += kFlat) {
        hc[i] = Hcol[i];
        c[i] = i < k ? cs[i] : 0.0;
        d[i] = i < k ? sn[i] : 0.0;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double* g = state + 2 + restart;
    double a = hc[0];
    for (int i = 0; i < k; ++i) {     // earlier rotations
        const double b = hc[i + 1];
        Hcol[i] = c[i] * a + d[i] * b;
        a = -d[i] * a + c[i] * b;
    }
    const double den = hypot(a, hn);
    const double ck = den == 0.0 ? 1.0 : a / den, sk = den == 0.0 ? 0.0 : hn / den;
    cs[k] = ck;
    sn[k] = sk;
    Hcol[k] = ck * a + sk * hn;
    Hcol[k + 1] = 0.0;
    const double gk = g[k];
    g[k + 1] = -sk * gk;
    g[k] = ck * gk;
    state[2 + k] = fabs(sk * gk);
    state[0] = k + 1;
    if (fabs(sk * gk) <= tol || hn == 0.0) state[1] = 1.0;
}

// ||w|| from the chunks' shares, the same in every thread; negative once the
// cycle is done (block 0 of the same launch may be setting that: a block looks
// once).
__device__ inline double step_norm(const double* nrm, int chunks, const double* state, double* hn_sh) {
    if (threadIdx.x < 64) {
        const double s = wave_sum_of(nrm, chunks);
        if (threadIdx.x == 0)
            *hn_sh = __hip_atomic_load(state + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0.0 ? -1.0 : sqrt(s);
    }
    __syncthreads();
    return *hn_sh;
}

// The last step of a batch: v_{k+1} = w / ||w||, block 0 the rotation.
__global__ void __launch_bounds__(kFlat)
k_gm_next(int n, int k, int restart, int chunks, const double* nrm, const double* w, double* vnext, double* Hcol,
          double* cs, double* sn, double tol, double* state) {
    extern __shared__ double sh[];     // H column, cs, sn: 3 (k + 1)
    __shared__ double hn_sh;
    const double hn = step_norm(nrm, chunks, state, &hn_sh);
    if (hn < 0.0) return;
    unsigned r0, r1;
    chunk_range(n, r0, r1);
    if (hn != 0.0)
        for (unsigned r = r0 + threadIdx.x; r < r1; r += kFlat) vnext[r] = w[r] / hn;
    if (blockIdx.x == 0) rotate_column(k, restart, hn, Hcol, cs, sn, tol, state, sh);
}

// Between two steps of a batch: the rotation of column k in block 0, in the
// others v_{k+1} = w / ||w|| and the next step's z = N (d .* v_{k+1}), which
// divides the entries of w that it gathers itself (the same quotients) instead
// of waiting for a launch that writes them: 3.8 us at n = 16384 with a level-2
// FP64 map, 3.4 + 3.2 us as two launches, and one gap between launches less.
template <bool MAP, bool F32>
__global__ void __launch_bounds__(kFlat)
k_gm_next_precond(int n, int k, int restart, int chunks, const double* nrm, const double* w, double* vnext,
                  double* Hcol, double* cs, double* sn, double tol, double* state, const int* rowptr,
                  const int* colind, const void* val, const double* d, double* z) {
    extern __shared__ double sh[];     // H column, cs, sn: 3 (k + 1)
    __shared__ double hn_sh;
    const double hn = step_norm(nrm, chunks, state, &hn_sh);
    if (hn < 0.0) return;
    const int64_t block = flat_block();
    if (block == 0) {
        rotate_column(k, restart, hn, Hcol, cs, sn, tol, state, sh);
        return;
    }
    if (hn == 0.0) return;
    const int64_t t = (block - 1) * kFlat + threadIdx.x;
    if constexpr (MAP) {
        const int i = (int)(t / kSpmvLanes);
        const double s = row_product<F32, false, true, true>(i < n, i, rowptr, colind, nullptr, val, w, d, hn);
        if (i < n && t % kSpmvLanes == 0) {
            z[i] = s;
            vnext[i] = w[i] / hn;
        }
    } else if (t < n) {
        const double v = w[t] / hn;
        z[t] = d[t] * v;
        vnext[t] = v;
    }
}

// x += sum_i y_i z_i, i ascending.
__global__ void __launch_bounds__(kFlat)
k_gm_solution(int n, int used, const double* y, const double* Z, double* x) {
    const int64_t r = flat_block() * kFlat + threadIdx.x;
    if (r >= n) return;
    double s = x[r];
    int i = 0;
    for (; i + kTile <= used; i += kTile) {
        double z[kTile];
#pragma unroll
        for (int u = 0; u < kTile; ++u) z[u] = Z[(int64_t)(i + u) * n + r];
#pragma unroll
        for (int u = 0; u < kTile; ++u) s += y[i + u] * z[u];
    }
    for (; i < used; ++i) s += y[i] * Z[(int64_t)i * n + r];
    x[r] = s;
}

int64_t blocks_for(int64_t threads) { return (threads + kFlat - 1) / kFlat; }

}  // namespace

// Chunks of kRows rows, longer ones beyond kMaxChunks of them.
int gmres_chunks(int n) { return std::max(1, std::min((n + kRows - 1) / kRows, kMaxChunks)); }

hipError_t gmres_init(int restart, double beta, double* state, hipStream_t s) {
    hipLaunchKernelGGL(k_gm_init, dim3(1), dim3(kFlat), 0, s, restart, beta, state);
    return hipGetLastError();
}

namespace {

// A step up to the chunks' shares of ||w||; z is there already.
void enqueue_step(const GmresArgs& a, int k, hipStream_t s) {
    const int n = a.n, count = k + 1;
    const int chunks = gmres_chunks(n);
    const dim3 block(kThreads), cg((unsigned)chunks);
    const double* z = a.Z + (int64_t)k * n;
    double* Hcol = a.H + (int64_t)k * (a.restart + 1);
    const size_t wave_sums = sizeof(double) * kRowWaves * (size_t)count, coef = sizeof(double) * (size_t)count;
    hipLaunchKernelGGL(k_gm_apply_dots, cg, block, wave_sums, s, n, a.A_rowptr, a.A_colind, a.A_val, z, a.w, count,
                       a.V, a.part, a.state);
    // up to kInlineChunks partials per product, every block of the next kernel
    // sums them itself; beyond that (the reads would grow with the square of
    // the chunks) one small launch does
    const bool own = chunks <= kInlineChunks;
    auto reduced = [&]() -> const double* {
        if (own) return a.part;
        hipLaunchKernelGGL(k_gm_reduce, dim3((unsigned)count), dim3(64), 0, s, chunks, a.part, a.h2, a.state);
        return a.h2;
    };
    const double* src = reduced();
    hipLaunchKernelGGL(k_gm_update_dots, cg, block, wave_sums + coef, s, n, count, own ? chunks : 0, src, a.V, a.w,
                       a.h1, a.part2, a.state);
    if (!own)
        hipLaunchKernelGGL(k_gm_reduce, dim3((unsigned)count), dim3(64), 0, s, chunks, a.part2, a.h2, a.state);
    hipLaunchKernelGGL(k_gm_update_norm, cg, block, coef, s, n, count, own ? chunks : 0, own ? a.part2 : a.h2, a.V,
                       a.w, a.h1, Hcol, a.nrm, a.state);
}

}  // namespace

hipError_t gmres_steps(const GmresArgs& a, int first, int count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int n = a.n, chunks = gmres_chunks(n);
    const dim3 flat(kFlat);
    const int64_t rows = blocks_for(a.N_rowptr ? (int64_t)n * kSpmvLanes : n);
    for (int k = first; k < first + count; ++k) {
        double *v = a.V + (int64_t)k * n, *z = a.Z + (int64_t)k * n;
        if (k == first) {
            auto run = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, flat_grid(rows), flat, 0, s, n, a.N_rowptr, a.N_colind, a.N_val, a.d, v, z,
                                   a.state);
            };
            if (!a.N_rowptr) run(k_gm_precond<false, false>);
            else if (a.N_f32) run(k_gm_precond<true, true>);
            else run(k_gm_precond<true, false>);
        } else {
            auto run = [&](auto kernel) {
                hipLaunchKernelGGL(kernel, flat_grid(rows + 1), flat, 3 * sizeof(double) * (size_t)k, s, n, k - 1,
                                   a.restart, chunks, a.nrm, a.w, v, a.H + (int64_t)(k - 1) * (a.restart + 1), a.cs,
                                   a.sn, a.tol, a.state, a.N_rowptr, a.N_colind, a.N_val, a.d, z);
            };
            if (!a.N_rowptr) run(k_gm_next_precond<false, false>);
            else if (a.N_f32) run(k_gm_next_precond<true, true>);
            else run(k_gm_next_precond<true, false>);
        }
        enqueue_step(a, k, s);
    }
    const int k = first + count - 1;
    hipLaunchKernelGGL(k_gm_next, dim3((unsigned)chunks), flat, 3 * sizeof(double) * (size_t)(k + 1), s, n, k,
                       a.restart, chunks, a.nrm, a.w, a.V + (int64_t)(k + 1) * n,
                       a.H + (int64_t)k * (a.restart + 1), a.cs, a.sn, a.tol, a.state);
    return hipGetLastError();
}

hipError_t gmres_solution(int n, int used, const double* y, const double* Z, double* x, hipStream_t s) {
    if (used <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gm_solution, flat_grid(blocks_for(n)), dim3(kFlat), 0, s, n, used, y, Z, x);
    return hipGetLastError();
}

}  // namespace samk
