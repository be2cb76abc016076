// sam_aux.hip -- gfx950 kernels for the explicit residual of a stored map
// (Section 2, eq. res: R = A_k M - A_0, recomputed column by column from M's
// values, independently of the build's own residuals) and for y = M x.
#include "sam_device.hpp"
#include "sam_kernels.hpp"

#include <algorithm>
#include <climits>

namespace samk {

namespace {

__device__ inline double mval(const void* M, int e, int f32) {
    return f32 ? (double)static_cast<const float*>(M)[e] : static_cast<const double*>(M)[e];
}

// Eight (or 16) lanes per column j.  The rows of column j of
// A_k M - A_0 are the union U of rows(A_k(:, l)) for l in M(:, j) and
// rows(A_0(:, j)); every row of U has an LDS accumulator, and contributions
// are added column by column of M, the lanes taking the entries of one A_k
// column at a time: rows are distinct inside it, so the lanes of one
// instruction never share a slot and every row's sum keeps the order of M's
// entries (A_0 last).
//
// U is built as a bitmap over a window of kResRows rows (the sweep jumps to
// the next occupied window), and the rank of a row inside U picks its
// accumulator.  The TABLE forms find it in a small hash table keyed by the row
// instead (columns whose entries fit the registers, fetched once, all loads
// independent): its cost does not depend on where the rows lie.  More rows
// than slots: the bitmap again.
//
// Bound: VALU and LDS instructions per entry, and the latency of the
// dependent loads (column of M, its extents in A_k, the entries).  One wave
// per column took 2.76 ms for the 512 x 512 level-2 map, eight problems per
// wave 0.18 ms, with the entries held in registers 0.11 ms.  Windows -> table,
// us: 64^3 seven-point level 1 238 -> 157, level 2 1070 -> 388; 512^2 level 3
// 495 -> 388.
constexpr int kResWPL = 16;               // bitmap words per lane
constexpr int kResAcc = 64;               // accumulators per column and pass (bitmap form)
constexpr int kResWords = kResWPL * 64;   // bitmap words of a block
// Entries beyond which a column takes a whole wave: on groups of lanes the work
// is a column's entries times its ranges of 64 rows.  Groups / wave, us:
// 512^2 nine-point level 3 (441 entries) 3390 / 3546, 40^3 27-point level 1
// (729) 817 / 587, with the level-2 pattern (3375) 8370 / 1499; one dense
// column of A_0 in 20000 short ones 87000 / 300.
constexpr int kResWide = 512;

struct alignas(16) ResList {  // one column of M's pattern: its run in A_k and its value
    int start, len;
    double m;
};

struct ResArgs {
    int n;
    const int *Ak_cp, *Ak_ri;
    const double* Ak_v;
    const int *A0_cp, *A0_ri;
    const double* A0_v;
    const int *M_cp, *M_ri;
    const void* M_v;
    int f32;
    double* col_out;
    unsigned long long* status;
};

__device__ inline int wave_min(int v) {
    v = grp_min<16>(v);
#pragma unroll
    for (int d = 16; d < 64; d <<= 1) v = min(v, __shfl_xor(v, d));
    return v;
}
__device__ inline int wave_sum(int v) {
    v = grp_sum<16>(v);
#pragma unroll
    for (int d = 16; d < 64; d <<= 1) v += __shfl_xor(v, d);
    return v;
}
__device__ inline double readlane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The first of the ascending rows ri[a, b) that is at least `row` (b: none),
// by the wave: 64 probes a round.
__device__ inline int first_row(const int* ri, int a, int b, int row) {
    const int lane = wave_lane();
    while (b - a > 64) {
        const int step = (b - a) / 64 + 1;
        const int p = a + min(step * (lane + 1), b - a) - 1;   // the last of lane's share
        a += step * __popcll(__ballot(p < b - 1 && ri[p] < row));
        b = a + min(step, b - a);
    }
    return a + __popcll(__ballot(lane < b - a && ri[a + lane] < row));
}

// Column j by the whole wave, for columns of many entries: a window of 32768
// rows as a bitmap, whose words are taken in ranges of at most kAcc rows.  The
// runs of A_k and A_0 ascend, so a range reads of a long run what lies in it,
// and of 64 runs of M's column those that reach it: the work grows with the
// entries, not with their product with the ranges.  Bound by the latency of the
// runs' loads (kAhead of them in flight) and of the LDS reads that place a row.
// bm, pre: kResWords; acc: kAcc.
template <int kAcc>
__device__ double wave_column(const ResArgs& a, int j, unsigned* bm, unsigned short* pre, double* acc) {
    constexpr int kShort = 64;   // entries of a run taken at once
    constexpr int kAhead = 8;    // short runs whose loads are in flight together
    const int lane = wave_lane();
    const int ma = a.M_cp[j], mb = a.M_cp[j + 1], aa = a.A0_cp[j], ab = a.A0_cp[j + 1];
    int start = 0, len = 0;      // lane's run of the 64 at hand
    auto runs = [&](unsigned t) {
        start = len = 0;
        if (t >= (unsigned)mb) return;
        const int l = a.M_ri[t];
        if (l < 0 || l >= a.n) {
            report(a.status, j, kStIndex);
            return;
        }
        start = a.Ak_cp[l];
        len = a.Ak_cp[l + 1] - start;
    };
    int lo = lane == 0 && ab > aa ? a.A0_ri[aa] : INT_MAX;
    for (unsigned t = ma; t < (unsigned)mb; t += 64) {
        runs(t + lane);
        if (len > 0) lo = min(lo, a.Ak_ri[start]);
    }
    double colsum = 0.0;
    for (int base = wave_min(lo); base != INT_MAX;) {
#pragma unroll
        for (int w = 0; w < kResWPL; ++w) bm[w * 64 + lane] = 0u;
        wave_sync();
        int next = INT_MAX;   // the first row past the window
        auto mark = [&](int r) {
            const int d = r - base;
            if (d < kResWords * 32) atomicOr(&bm[d >> 5], 1u << (d & 31));
            else next = min(next, r);
            return d < kResWords * 32;
        };
        auto mark_run = [&](const int* ri, int e, int end) {   // by the wave
            for (e = first_row(ri, e, end, base);; e += 64) {
                bool in = lane < end - e;
                if (in) in = mark(ri[e + lane]);
                if (__ballot(!in)) break;
            }
        };
        for (unsigned t = ma; t < (unsigned)mb; t += 64) {
            runs(t + lane);
            if (len <= kShort)
                for (int e = start; e < start + len; ++e) {
                    const int r = a.Ak_ri[e];
                    if (r >= base && !mark(r)) break;
                }
            for (unsigned long long left = __ballot(len > kShort); left; left &= left - 1) {
                const int b = __ffsll(left) - 1, s = __builtin_amdgcn_readlane(start, b);
                mark_run(a.Ak_ri, s, s + __builtin_amdgcn_readlane(len, b));
            }
        }
        mark_run(a.A0_ri, aa, ab);
        wave_sync();
        // pre[w]: the window's rows before word w
        int mine = 0;
#pragma unroll
        for (int w = 0; w < kResWPL; ++w) mine += __popc(bm[lane * kResWPL + w]);
        int run = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(run, d);
            if (lane >= d) run += y;
        }
        const int cnt = __builtin_amdgcn_readlane(run, 63);
        run -= mine;
#pragma unroll
        for (int w = 0; w < kResWPL; ++w) {
            pre[lane * kResWPL + w] = (unsigned short)run;
            run += __popc(bm[lane * kResWPL + w]);
        }
        wave_sync();
        for (int w0 = 0, r0 = 0; r0 < cnt;) {
            // the words from w0 on whose rows fit the accumulators
            int w1 = kResWords, r1 = cnt;
            if (cnt - r0 > kAcc) {
                int more = 0;
#pragma unroll
                for (int w = 0; w < kResWPL; ++w) {
                    const int x = lane * kResWPL + w;
                    more += x > w0 && pre[x] - r0 <= kAcc;
                }
                w1 = w0 + wave_sum(more);
                r1 = pre[w1];
            }
            const int d0 = w0 * 32, d1 = w1 * 32;
#pragma unroll
            for (int i = 0; i < kAcc / 64; ++i) acc[i * 64 + lane] = 0.0;
            wave_sync();
            auto add = [&](int r, double v) {
                const int d = r - base;
                if (d < d0 || d >= d1) return;
                const int w = d >> 5, rank = pre[w] + __popc(bm[w] & ((1u << (d & 31)) - 1u)) - r0;
                __hip_atomic_fetch_add(&acc[rank], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            };
            auto add_run = [&](const int* ri, const double* val, int e, int end, double m) {
                for (e = first_row(ri, e, end, base + d0);; e += 64) {
                    bool in = lane < end - e;
                    if (in) {
                        const int r = ri[e + lane];
                        add(r, val[e + lane] * m);
                        in = r - base < d1;
                    }
                    if (__ballot(!in)) break;
                }
            };
            for (unsigned t = ma; t < (unsigned)mb; t += 64) {
                runs(t + lane);
                double m = 0.0;
                bool touches = false;
                if (len > 0) {
                    m = mval(a.M_v, (int)(t + lane), a.f32);
                    touches = a.Ak_ri[start] - base < d1 && a.Ak_ri[start + len - 1] - base >= d0;
                }
                for (unsigned long long left = __ballot(touches); left;) {   // in M's order
                    int s[kAhead], l[kAhead], row[kAhead];
                    double v[kAhead], c[kAhead];
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        s[u] = l[u] = 0;
                        c[u] = 0.0;
                        if (!left) continue;
                        const int b = __ffsll(left) - 1;
                        left &= left - 1;
                        s[u] = __builtin_amdgcn_readlane(start, b);
                        l[u] = __builtin_amdgcn_readlane(len, b);
                        c[u] = readlane(m, b);
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        const bool in = l[u] <= kShort && lane < l[u];
                        row[u] = in ? a.Ak_ri[s[u] + lane] : -1;
                        v[u] = in ? a.Ak_v[s[u] + lane] : 0.0;
                    }
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) {
                        if (l[u] > kShort) add_run(a.Ak_ri, a.Ak_v, s[u], s[u] + l[u], c[u]);
                        else if (row[u] >= 0) add(row[u], v[u] * c[u]);
                    }
                }
            }
            add_run(a.A0_ri, a.A0_v, aa, ab, -1.0);
            wave_sync();
            double s = 0.0;
#pragma unroll
            for (int i = 0; i < kAcc / 64; ++i) {
                const double x = acc[i * 64 + lane];
                s += x * x;
            }
            colsum += group_sum<64>(s);
            wave_sync();
            w0 = w1;
            r0 = r1;
        }
        base = wave_min(next);
    }
    return colsum;
}

// Every column by a wave.
constexpr int kWideAcc = 1024;
__global__ void __launch_bounds__(64)
k_residual_wide(ResArgs a) {
    __shared__ unsigned bm[kResWords];
    __shared__ unsigned short pre[kResWords];
    __shared__ double acc[kWideAcc];
    for (int64_t j = blockIdx.x; j < a.n; j += gridDim.x) {
        const double s = wave_column<kWideAcc>(a, (int)j, bm, pre, acc);
        if (wave_lane() == 0) a.col_out[j] = s;
    }
}

// kResLanes lanes per column, kResBatch columns of M per problem held in
// registers: 8 and 16, or 16 and 32.
template <int kResLanes, int kResBatch, bool TABLE>
__global__ void __launch_bounds__(64, kResLanes == 8 ? 3 : 2)
k_residual_columns(ResArgs a) {
    const int n = a.n, f32 = a.f32;
    const int *Ak_cp = a.Ak_cp, *Ak_ri = a.Ak_ri, *A0_cp = a.A0_cp, *A0_ri = a.A0_ri, *M_cp = a.M_cp, *M_ri = a.M_ri;
    const double *Ak_v = a.Ak_v, *A0_v = a.A0_v;
    const void* M_v = a.M_v;
    double* col_out = a.col_out;
    unsigned long long* status = a.status;
    constexpr int kResCols = 64 / kResLanes;              // columns per wave
    constexpr int kResRows = kResWPL * kResLanes * 32;    // rows per window
    // word w of a lane sits at w * 64 + lane: the passes over a lane's own
    // words touch 64 consecutive words
    __shared__ unsigned bm[kResWords];
    __shared__ unsigned short pre[kResWords];
    // table slots per column: twice the rows of a level-2 column and more
    // (25 of a five-point, 63 of a seven-point stencil)
    constexpr int kHashBits = kResLanes == 8 ? 6 : 7;
    constexpr int kHash = 1 << kHashBits;
    constexpr int kResAccStride = (TABLE ? kHash : kResAcc) + 4;   // 8 banks apart: eight columns cover the 64 banks
    static_assert(kHash >= kResAcc, "the bitmap form uses the same accumulators");
    struct Groups {
        double accs[kResCols * kResAccStride];
        int keys[TABLE ? kResCols * kHash : 4];
        ResList lists[kResCols][kResBatch];
    };
    constexpr int kWaveAcc = (int)(sizeof(Groups) / sizeof(double)) / 64 * 64;
    __shared__ union {
        Groups groups;
        double wave[kWaveAcc];   // a column that takes the whole wave
    } sh;
    auto& lists = sh.groups.lists;
    auto& keys = sh.groups.keys;
    double* accs = sh.groups.accs;
    const int lane = wave_lane();
    const int g = lane % kResLanes, q = lane / kResLanes;
    double* acc = accs + q * kResAccStride;
    const int own = q * kResLanes;        // this group's first lane
    auto slot = [&](int wi) { return (wi % kResWPL) * 64 + own + wi / kResWPL; };
    // contiguous ranges of columns per block, neighbouring ranges on one XCD
    const int nb = gridDim.x;
    const int lb = (nb & 7) ? (int)blockIdx.x : ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    const int64_t ngroups = ((int64_t)n + kResCols - 1) / kResCols;
    const int grp_lo = (int)(lb * ngroups / nb), grp_hi = (int)((lb + 1) * ngroups / nb);
    for (int grp = grp_lo; grp < grp_hi; ++grp) {
        const int64_t jj = (int64_t)grp * kResCols + q;
        const bool valid = jj < n;
        const int j = valid ? (int)jj : 0;
        int ma = 0, mb = 0, aa = 0, ab = 0;
        if (valid) {
            ma = M_cp[j];
            mb = M_cp[j + 1];
            aa = A0_cp[j];
            ab = A0_cp[j + 1];
        }
        // the first kResBatch columns of M: their runs in A_k and their values
#pragma unroll
        for (int h = 0; h < kResBatch / kResLanes; ++h) {
            ResList x{0, 0, 0.0};
            const int t = ma + g + h * kResLanes;
            if (t < mb) {
                const int l = M_ri[t];
                if (l < 0 || l >= n) {
                    report(status, j, kStIndex);
                } else {
                    x.start = Ak_cp[l];
                    x.len = Ak_cp[l + 1] - x.start;
                    x.m = mval(M_v, t, f32);
                }
            }
            lists[q][g + h * kResLanes] = x;
        }
        wave_sync();
        // wave-uniform: every column problem of the wave fits the registers
        // (kResBatch columns of M, eight entries each and eight of A_0)
        bool fits = mb - ma <= kResBatch && ab - aa <= kResLanes;
#pragma unroll
        for (int h = 0; h < kResBatch / kResLanes; ++h) fits &= lists[q][g + h * kResLanes].len <= kResLanes;
        const bool fast = __ballot(!fits) == 0ull;
        int rows[kResBatch + 1];              // -1: no entry
        double vals[kResBatch + 1];           // entry times coefficient
        int lo = INT_MAX;
        unsigned long long wides = 0;         // columns that the whole wave has summed: their first lanes
        if (fast) {
#pragma unroll
            for (int u = 0; u < kResBatch; ++u) {
                const ResList y = lists[q][u];
                rows[u] = -1;
                vals[u] = 0.0;
                if (g < y.len) {
                    rows[u] = Ak_ri[y.start + g];
                    vals[u] = Ak_v[y.start + g];
                }
            }
            rows[kResBatch] = -1;
            vals[kResBatch] = 0.0;
            if (aa + g < ab) {
                rows[kResBatch] = A0_ri[aa + g];
                vals[kResBatch] = -A0_v[aa + g];
            }
#pragma unroll
            for (int u = 0; u < kResBatch; ++u) vals[u] *= lists[q][u].m;
#pragma unroll
            for (int u = 0; u <= kResBatch; ++u) lo = rows[u] >= 0 ? min(lo, rows[u]) : lo;
            if constexpr (TABLE) {
                int* key = keys + q * kHash;
#pragma unroll
                for (int i = 0; i < kHash / kResLanes; ++i) {
                    key[i * kResLanes + g] = -1;
                    acc[i * kResLanes + g] = 0.0;
                }
                wave_sync();
                bool full = false;
                constexpr int kTries = 11;   // first tries in flight together: 17 = 11 + 6, 33 = 3 * 11
#pragma unroll
                for (int u0 = 0; u0 <= kResBatch; u0 += kTries) {
                    int at[kTries], seen[kTries];
#pragma unroll
                    for (int i = 0; i < kTries; ++i) {
                        const int u = u0 + i;
                        seen[i] = -1;
                        if (u > kResBatch) continue;
                        at[i] = (int)(((unsigned)rows[u] * 0x9E3779B1u) >> (32 - kHashBits));
                        if (rows[u] >= 0) seen[i] = atomicCAS(&key[at[i]], -1, rows[u]);
                    }
                    // taken slots: the next ones, again all together
                    bool more = true;
                    for (int tries = 1; more; ++tries) {
                        more = false;
#pragma unroll
                        for (int i = 0; i < kTries; ++i) {
                            const int u = u0 + i;
                            if (u > kResBatch) continue;
                            if (seen[i] != -1 && seen[i] != rows[u]) {
                                at[i] = (at[i] + 1) & (kHash - 1);
                                seen[i] = atomicCAS(&key[at[i]], -1, rows[u]);
                            }
                        }
#pragma unroll
                        for (int i = 0; i < kTries; ++i)
                            if (u0 + i <= kResBatch) more |= seen[i] != -1 && seen[i] != rows[u0 + i];
                        if (tries == kHash) {
                            full |= more;
                            break;
                        }
                    }
#pragma unroll
                    for (int i = 0; i < kTries; ++i) {
                        const int u = u0 + i;
                        if (u <= kResBatch && rows[u] >= 0)
                            __hip_atomic_fetch_add(&acc[at[i]], vals[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                    }
                }
                wave_sync();
                if (__ballot(full) == 0ull) {   // wave-uniform
                    double s = 0.0;   // empty slots hold zeros
#pragma unroll
                    for (int i = 0; i < kHash / kResLanes; ++i) {
                        const double x = acc[i * kResLanes + g];
                        s += x * x;
                    }
                    s = group_sum<kResLanes>(s);
                    if (valid && g == 0) col_out[j] = s;
                    wave_sync();
                    continue;
                }
            }
        } else {   // the columns are ascending, so the smallest row heads one of them
            int entries = g == 0 ? min(ab - aa, kResWide + 1) : 0;   // counted no further than needed
            for (int t = ma + g; t < mb && entries <= kResWide; t += kResLanes) {
                const int l = M_ri[t];
                if (l < 0 || l >= n) {
                    report(status, j, kStIndex);
                    continue;
                }
                const int qa = Ak_cp[l], len = Ak_cp[l + 1] - qa;
                entries += min(len, kResWide + 1);
                if (len > 0) lo = min(lo, Ak_ri[qa]);
            }
            if (ab > aa) lo = min(lo, A0_ri[aa]);
            const bool wide = grp_sum<kResLanes>(entries) > kResWide;
            wides = __ballot(wide && g == 0);
            for (unsigned long long left = wides; left; left &= left - 1) {
                const int qw = (__ffsll(left) - 1) / kResLanes;
                const int jw = (int)((int64_t)grp * kResCols + qw);
                const double s = wave_column<kWaveAcc>(a, jw, bm, pre, sh.wave);
                if (lane == 0) col_out[jw] = s;
            }
            if (wide) lo = INT_MAX;   // no window follows
        }
        int base = grp_min<kResLanes>(lo);
        double colsum = 0.0;
        while (base != INT_MAX) {
#pragma unroll
            for (int w = 0; w < kResWPL; ++w) bm[w * 64 + lane] = 0u;
            wave_sync();
            // every entry of column j's problem in order: entry(row, product)
            auto sweep = [&](bool values, auto entry) {
                if (fast) {
#pragma unroll
                    for (int u = 0; u <= kResBatch; ++u)
                        if (rows[u] >= 0) entry(rows[u], vals[u]);
                    wave_sync();
                    return;
                }
                for (int t = ma; t < mb; ++t) {
                    const int l = M_ri[t];
                    if (l < 0 || l >= n) continue;
                    const double m = values ? mval(M_v, t, f32) : 0.0;
                    const int fb = Ak_cp[l + 1];
                    for (int f = Ak_cp[l] + g; f < fb; f += kResLanes) entry(Ak_ri[f], values ? Ak_v[f] * m : 0.0);
                }
                for (int e = aa + g; e < ab; e += kResLanes) entry(A0_ri[e], values ? -A0_v[e] : 0.0);
                wave_sync();
            };
            int next = INT_MAX;
            sweep(false, [&](int r, double) {
                const int d = r - base;
                if (d >= kResRows) next = min(next, r);
                else if (d >= 0) atomicOr(&bm[slot(d >> 5)], 1u << (d & 31));
            });
            int c = 0;
#pragma unroll
            for (int w = 0; w < kResWPL; ++w) c += __popc(bm[w * 64 + lane]);
            int run = grp_excl_scan<kResLanes>(c);
            const int cnt = grp_sum<kResLanes>(c);
#pragma unroll
            for (int w = 0; w < kResWPL; ++w) {
                pre[w * 64 + lane] = (unsigned short)run;
                run += __popc(bm[w * 64 + lane]);
            }
            wave_sync();
            for (int r0 = 0; r0 < cnt; r0 += kResAcc) {   // rank ranges of kResAcc rows
#pragma unroll
                for (int i = 0; i < kResAcc / kResLanes; ++i) acc[i * kResLanes + g] = 0.0;
                wave_sync();
                sweep(true, [&](int r, double v) {
                    const int d = r - base;
                    if (d < 0 || d >= kResRows) return;
                    const int p = slot(d >> 5);
                    const int rank = pre[p] + __popc(bm[p] & ((1u << (d & 31)) - 1u)) - r0;
                    if (rank >= 0 && rank < kResAcc)
                        __hip_atomic_fetch_add(&acc[rank], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                });
                double s = 0.0;   // slots past the last rank hold zeros
#pragma unroll
                for (int i = 0; i < kResAcc / kResLanes; ++i) {
                    const double x = acc[i * kResLanes + g];
                    s += x * x;
                }
                colsum += group_sum<kResLanes>(s);
                wave_sync();
            }
            base = grp_min<kResLanes>(next);
        }
        if (valid && g == 0 && !(wides >> lane & 1)) col_out[j] = colsum;
    }
}

}  // namespace

hipError_t residual_columns(int n, int64_t nnzA, int64_t nnzM, const int* Ak_cp, const int* Ak_ri, const double* Ak_v,
                            const int* A0_cp, const int* A0_ri, const double* A0_v, const int* M_cp,
                            const int* M_ri, const void* M_v, int m_is_f32, double* col_out,
                            unsigned long long* status, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    // Eight lanes per column where most columns of A_k and A_0 have at most
    // eight entries and those of M at most 16 (means of 7 and 14: stencil
    // columns are the same length but for the boundary), else 16 lanes, which
    // hold columns of 16 entries and 32 columns of M.  The table pays off in
    // the 16-lane form, and in the other for columns of more than six entries
    // (three-dimensional stencils, whose rows span planes); shorter ones have
    // their rows in a window or two and keep the registers and LDS that it
    // takes for more waves.  Bitmap / table, us: eight lanes 512^2 level 1
    // 91 / 115, level 2 113 / 133, 64^3 level 1 238 / 155; sixteen lanes 512^2
    // level 3 495 / 388, 64^3 level 2 1070 / 388, 1024^2 nine-point level 2
    // 1955 / 1540, level 1 1418 / 1252.
    const ResArgs a{n, Ak_cp, Ak_ri, Ak_v, A0_cp, A0_ri, A0_v, M_cp, M_ri, M_v, m_is_f32, col_out, status};
    if ((double)nnzA * (double)nnzM > (double)kResWide * n * n) {   // entries of a column's problem, in the mean
        hipLaunchKernelGGL(k_residual_wide, dim3((unsigned)std::min(n, 256 * 32)), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    const bool narrow = nnzA <= (int64_t)7 * n && nnzM <= (int64_t)14 * n;
    const int cols = narrow ? 8 : 4;
    // up to 12 one-wave blocks per CU are resident
    const int grid = launch_grid(((int64_t)n + cols - 1) / cols, 256 * 12);
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), 0, s, a); };
    if (!narrow) run(k_residual_columns<16, 32, true>);
    else if (nnzA > (int64_t)6 * n) run(k_residual_columns<8, 16, true>);
    else run(k_residual_columns<8, 16, false>);
    return hipGetLastError();
}

// ----------------------------------------------------------------- apply

namespace {

__global__ void k_tcount(int64_t nnz, const int* ri, int n, int* rowcount) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nnz) {
        const int r = ri[e];
        if (r >= 0 && r < n) atomicAdd(&rowcount[r], 1);
    }
}

// Eight lanes per column: a thread per column took its entries one atomic
// round trip after the other (128^2 five-point level-2 map 10 -> 6 us, 48^3
// seven-point level 2 80 -> 67; at 256^2 the atomics' rate shows, 17 -> 22).
constexpr int kTfillLanes = 8;

__global__ void k_tfill(int n, const int* cp, const int* ri, const int* rowptr, int* cursor, int* colind,
                        int* perm) {
    const int64_t t = flat_block() * blockDim.x + threadIdx.x;
    const int64_t j = t / kTfillLanes;
    if (j >= n) return;
    const int end = cp[j + 1];
    for (int64_t e = cp[j] + (int64_t)(t % kTfillLanes); e < end; e += kTfillLanes) {
        const int r = ri[e];
        if (r < 0 || r >= n) continue;
        const int slot = rowptr[r] + atomicAdd(&cursor[r], 1);
        colind[slot] = (int)j;
        perm[slot] = (int)e;
    }
}

// Each row's (col, perm) by column (entries of one column by slot): makes the
// row view independent of the atomic slot order.  Sixteen lanes per row hold
// up to kTsortStage entries and write each to its rank, counted over the row's
// columns in LDS; longer rows are sorted by insertion in memory.  That sort,
// a thread per row, moved entry by entry through dependent loads: 687 us for
// the 110592 rows of a 48^3 seven-point level-2 pattern (25 entries), now
// 31 us.
constexpr int kTsortThreads = 256;
constexpr int kTsortLanes = 16;
constexpr int kTsortStage = 64;

__global__ void __launch_bounds__(kTsortThreads)
k_tsort(int n, const int* rowptr, int* colind, int* perm) {
    constexpr int kGroups = kTsortThreads / kTsortLanes;
    constexpr int kHeld = kTsortStage / kTsortLanes;
    __shared__ int col_sh[kGroups][kTsortStage];
    const int grp = threadIdx.x / kTsortLanes, g = threadIdx.x % kTsortLanes;
    const int64_t i = flat_block() * kGroups + grp;
    if (i >= n) return;   // whole groups; no block barrier below
    const int a = rowptr[i], b = rowptr[i + 1], len = b - a;
    if (len > kTsortStage) {
        if (g) return;
        for (int x = a + 1; x < b; ++x) {
            const int c = colind[x], p = perm[x];
            int y = x - 1;
            while (y >= a && colind[y] > c) {
                colind[y + 1] = colind[y];
                perm[y + 1] = perm[y];
                --y;
            }
            colind[y + 1] = c;
            perm[y + 1] = p;
        }
        return;
    }
    int c[kHeld], p[kHeld], rank[kHeld];
#pragma unroll
    for (int u = 0; u < kHeld; ++u) {
        const int x = g + u * kTsortLanes;
        c[u] = x < len ? colind[a + x] : INT_MAX;
        p[u] = x < len ? perm[a + x] : 0;
        rank[u] = 0;
        if (x < len) col_sh[grp][x] = c[u];
    }
    wave_sync();   // all lanes hold their entries: the stores below may replace them
    for (int f = 0; f < len; ++f) {
        const int cf = col_sh[grp][f];
#pragma unroll
        for (int u = 0; u < kHeld; ++u) rank[u] += cf < c[u] || (cf == c[u] && f < g + u * kTsortLanes);
    }
#pragma unroll
    for (int u = 0; u < kHeld; ++u)
        if (g + u * kTsortLanes < len) {
            colind[a + rank[u]] = c[u];
            perm[a + rank[u]] = p[u];
        }
}

// y = M x over the row view (see row_product).
template <bool F32, bool PERM>
__global__ void __launch_bounds__(256)
k_spmv_rows(int n, const int* rowptr, const int* colind, const int* perm, const void* val, const double* x,
            double* y) {
    const int64_t t = flat_block() * blockDim.x + threadIdx.x;
    const int64_t i = t / kSpmvLanes;
    const double s = row_product<F32, PERM, false>(i < n, (int)i, rowptr, colind, perm, val, x, nullptr);
    if (i < n && t % kSpmvLanes == 0) y[i] = s;
}

__global__ void k_permute_vals(int64_t nnz, const int* perm, const void* val, int f32, void* out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    if (f32) static_cast<float*>(out)[e] = static_cast<const float*>(val)[perm[e]];
    else static_cast<double*>(out)[e] = static_cast<const double*>(val)[perm[e]];
}

}  // namespace

__global__ void k_identity_queue(int n, int* queue, int* bstart) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (queue && i < n) queue[i] = i;
    if (i == 0) {
        bstart[0] = 0;
        bstart[1] = n;
    }
}

hipError_t identity_queue(int n, int* queue, int* bstart, hipStream_t s) {
    const int blocks = queue ? (std::max(n, 1) + 255) / 256 : 1;
    hipLaunchKernelGGL(k_identity_queue, dim3((unsigned)blocks), dim3(256), 0, s, n, queue, bstart);
    return hipGetLastError();
}

__global__ void k_set4(int* p, int4 v) { *reinterpret_cast<int4*>(p) = v; }

hipError_t set4_i32(int* p, int a, int b, int c, int d, hipStream_t s) {
    hipLaunchKernelGGL(k_set4, dim3(1), dim3(1), 0, s, p, make_int4(a, b, c, d));
    return hipGetLastError();
}

__global__ void k_fill_i32(int* p, int64_t count, int v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

hipError_t fill_i32(int* p, int64_t count, int v, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count, v);
    return hipGetLastError();
}

hipError_t transpose_count(int n, const int* cp, const int* ri, int64_t nnz, int* rowcount,
                           hipStream_t s) {
    (void)cp;
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tcount, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, s, nnz, ri, n, rowcount);
    return hipGetLastError();
}

hipError_t transpose_fill(int n, const int* cp, const int* ri, const int* rowptr, int* cursor,
                          int* colind, int* perm, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t threads = (int64_t)n * kTfillLanes;
    hipLaunchKernelGGL(k_tfill, flat_grid((threads + 255) / 256), dim3(256), 0, s, n, cp, ri, rowptr, cursor,
                       colind, perm);
    return hipGetLastError();
}

hipError_t transpose_sort_rows(int n, const int* rowptr, int* colind, int* perm, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    constexpr int kRows = kTsortThreads / kTsortLanes;
    hipLaunchKernelGGL(k_tsort, flat_grid((n - 1) / kRows + 1), dim3(kTsortThreads), 0, s, n, rowptr, colind,
                       perm);
    return hipGetLastError();
}

hipError_t spmv_rows(int n, const int* rowptr, const int* colind, const int* perm, const void* val,
                     int val_f32, const double* x, double* y, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t threads = (int64_t)n * kSpmvLanes;
    const dim3 grid = flat_grid((threads + 255) / 256), block(256);
    if (val_f32 && perm) hipLaunchKernelGGL((k_spmv_rows<true, true>), grid, block, 0, s, n, rowptr, colind, perm, val, x, y);
    else if (val_f32) hipLaunchKernelGGL((k_spmv_rows<true, false>), grid, block, 0, s, n, rowptr, colind, perm, val, x, y);
    else if (perm) hipLaunchKernelGGL((k_spmv_rows<false, true>), grid, block, 0, s, n, rowptr, colind, perm, val, x, y);
    else hipLaunchKernelGGL((k_spmv_rows<false, false>), grid, block, 0, s, n, rowptr, colind, perm, val, x, y);
    return hipGetLastError();
}

hipError_t permute_vals(int64_t nnz, const int* perm, const void* val, int val_f32, void* out, hipStream_t s) {
    if (nnz <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_permute_vals, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, s, nnz, perm, val,
                       val_f32, out);
    return hipGetLastError();
}

}  // namespace samk
