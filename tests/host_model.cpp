// A model of the HIP runtime and of the kernels for the library's host code
// (sam_capi.cpp, sam_sequence.cpp), without a GPU.  Work enqueued on a stream
// runs only when that stream (or the device) is waited for, which is the
// latest that asynchronous work may run: host code that relies on work it has
// not waited for reads poisoned memory here.  The numeric kernels are modelled
// by their reads of the bucket table and queue: each column has to be served
// once, by a class it fits.  Prints what is wrong and ends with status 1.
#include "sam_host.hpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <random>
#include <set>

namespace {

using Op = std::function<void()>;
int g_errors = 0;
int g_graph_launches = 0;

void wrong(const char* what, long a = 0, long b = 0) {
    if (++g_errors <= 10) printf("WRONG: %s (%ld, %ld)\n", what, a, b);
}

struct Stream {
    std::deque<Op> ops;
    int captures = 0;
};
struct Graph {
    std::vector<Op> ops;
};
struct Exec {
    std::vector<Op> ops;
    int in_flight = 0;
};
struct Event {
    Stream* on = nullptr;
    int recorded = 0, reached = 0, captures = 0;
};
std::set<Stream*> g_streams;
Stream g_null;
Graph* g_capture = nullptr;

Stream* of(hipStream_t s) { return s ? (Stream*)s : &g_null; }
hipError_t enqueue(hipStream_t s, Op op) {
    if (g_capture) g_capture->ops.push_back(std::move(op));
    else of(s)->ops.push_back(std::move(op));
    return hipSuccess;
}
// Streams and events are captured with once in the library.
hipError_t note_capture(int* captures) {
    if (++*captures > 1) wrong("captured with twice");
    return hipSuccess;
}
void drain(Stream* s) {
    while (!s->ops.empty()) {
        Op op = std::move(s->ops.front());
        s->ops.pop_front();
        op();
    }
}

}  // namespace

// ------------------------------------------------------------ HIP runtime
extern "C" {

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    *p = hipDeviceProp_tR0600{};
    p->multiProcessorCount = 256;
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "model"; }
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t st) {
    if (kind == hipMemcpyHostToDevice) {   // pageable memory is read at the call
        std::vector<char> copy((const char*)s, (const char*)s + n);
        return enqueue(st, [=] { memcpy(d, copy.data(), n); });
    }
    return enqueue(st, [=] { memcpy(d, s, n); });
}
hipError_t hipStreamSynchronize(hipStream_t s) { drain(of(s)); return hipSuccess; }
hipError_t hipDeviceSynchronize() {
    drain(&g_null);
    for (Stream* s : g_streams) drain(s);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    auto* x = new Stream;
    g_streams.insert(x);
    *s = (hipStream_t)x;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    drain(of(s));
    g_streams.erase((Stream*)s);
    delete (Stream*)s;
    return hipSuccess;
}
// Inside a capture, events add nothing: the order of the calls is an order of
// the graph.  Elsewhere a wait is for the last record before it: whoever runs it
// runs the recorded stream up to there first.
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t) new Event;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    auto* x = (Event*)e;
    if (x->reached != x->recorded) wrong("event destroyed before it is reached");
    else delete x;
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    auto* x = (Event*)e;
    if (g_capture) return note_capture(&x->captures);
    x->on = of(s);
    const int at = ++x->recorded;
    return enqueue(s, [x, at] { x->reached = at; });
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    auto* x = (Event*)e;
    if (g_capture) return hipSuccess;
    const int at = x->recorded;
    Stream* on = x->on;
    return enqueue(s, [x, at, on] {
        while (x->reached < at) {
            Op op = std::move(on->ops.front());
            on->ops.pop_front();
            op();
        }
    });
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
    *st = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    g_capture = new Graph;
    return note_capture(&of(s)->captures);
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = (hipGraph_t)g_capture;
    g_capture = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    auto* x = new Exec;
    x->ops = ((Graph*)g)->ops;
    *e = (hipGraphExec_t)x;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
    auto* x = (Exec*)e;
    ++g_graph_launches;
    for (const Op& op : x->ops) (void)enqueue(s, op);
    ++x->in_flight;
    return enqueue(s, [x] { --x->in_flight; });
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete (Graph*)g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
    auto* x = (Exec*)e;
    if (x->in_flight) wrong("graph destroyed while it runs", x->in_flight);   // and kept: its end is still to come
    else delete x;
    return hipSuccess;
}

}  // extern "C"

// ---------------------------------------------------------------- kernels
namespace samh {
hipError_t scratch_setup(int) { return hipSuccess; }
}  // namespace samh

namespace samk {

namespace {

std::vector<int> g_visits;   // per column, of the launches since the last clear

template <int I>
hipError_t model_launch(const NumericArgs& a, int, hipStream_t s) {
    return enqueue(s, [a] {
        int cnt = 0;
        const NumericVariant& v = numeric_menu(&cnt)[I];
        const int b0 = a.bstart[a.bucket], b1 = a.bstart[a.bucket + 1];
        if (b0 < 0 || b1 < b0 || b1 > a.n) return wrong("bucket offsets", b0, b1);
        for (int i = b0; i < b1; ++i) {
            const int j = b1 - b0 == a.n ? i : a.queue[i];
            if (j < 0 || j >= a.n) return wrong("queue entry", i, j);
            if (a.nI[j] > v.max_rows() || a.S_cp[j + 1] - a.S_cp[j] > v.NC) wrong("class too small", j, I);
            ++g_visits[(size_t)j];
        }
    });
}
int model_blocks() { return 8; }

#define V(i, prec, G, R, NC, w) \
    NumericVariant{prec, G, R, NC, w, 1, 2, &model_launch<i>, nullptr, &model_blocks, nullptr, nullptr, \
                   1.f * R, .01f * R * NC, 1.f * R, .01f * R * NC}
const NumericVariant kMenu[] = {V(0, 1, 2, 8, 5, 0),  V(1, 1, 4, 7, 13, 0), V(2, 1, 8, 8, 25, 0), V(3, 1, 32, 4, 32, 0),
                                V(4, 1, 1, 13, 5, 0), V(5, 1, 4, 7, 9, 0),  V(6, 0, 2, 8, 5, 0),  V(7, 0, 8, 4, 16, 0),
                                V(8, 0, 64, 2, 32, 0), V(9, 1, 64, 2, 32, 1), V(10, 0, 64, 2, 32, 1)};
constexpr int kF32 = 6;   // of them FP32, unweighted
#undef V

// B = S(A~) with the diagonal; any rule keeps the entries of at least 1/2
std::vector<int> kept(const int* cp, const int* ri, const double* v, const SparsifySpec& sp, int j) {
    std::set<int> r{j};
    for (int e = cp[j]; e < cp[j + 1]; ++e)
        if (sp.kind == SAM_SPARSIFY_NONE || std::abs(v[e]) >= 0.5) r.insert(ri[e]);
    return {r.begin(), r.end()};
}
std::vector<int> united(const int* P_cp, const int* P_cnt, const int* P_ri, const int* Q_cp, const int* Q_cnt,
                        const int* Q_ri, int j) {
    std::set<int> r;
    const int pn = P_cnt ? P_cnt[j] : P_cp[j + 1] - P_cp[j];
    for (int x = 0; x < pn; ++x) {
        const int l = P_ri[P_cp[j] + x];
        const int qn = Q_cnt ? Q_cnt[l] : Q_cp[l + 1] - Q_cp[l];
        r.insert(Q_ri + Q_cp[l], Q_ri + Q_cp[l] + qn);
    }
    return {r.begin(), r.end()};
}

}  // namespace

const NumericVariant* numeric_menu(int* count) {
    *count = (int)(sizeof kMenu / sizeof kMenu[0]);
    return kMenu;
}

size_t scan_temp_bytes(int64_t) { return 256; }
hipError_t scan_counts(const int* counts, int64_t n, int64_t* off, int* off32, int*, void*, hipStream_t s,
                       int* maxcount, int64_t* total) {
    return enqueue(s, [=] {
        int64_t run = 0;
        for (int64_t i = 0; i <= n; ++i) {
            off[i] = run;
            if (off32) off32[i] = (int)run;
            if (i == n) break;
            if (maxcount) *maxcount = std::max(*maxcount, counts[i]);
            run += counts[i];
        }
        if (total) *total = run;
    });
}
hipError_t check_structures(const CheckArgs& a, hipStream_t s) {
    return enqueue(s, [a] {
        *a.total = 0;
        for (int i = 0; i < a.count; ++i) {
            const CscRef& m = a.m[i];
            CscFacts f{a.n, a.n, 0, 0};
            for (int j = 0; j < a.n; ++j) {
                bool diag = false;
                int got = 0;
                f.longest = std::max(f.longest, m.cp[j + 1] - m.cp[j]);
                for (int e = m.cp[j]; m.ri && e < m.cp[j + 1]; ++e) {
                    diag |= m.ri[e] == j;
                    if (m.gather_cp) got += m.gather_cp[m.ri[e] + 1] - m.gather_cp[m.ri[e]];
                }
                f.missing += !diag;
                if (m.gather_counts) m.gather_counts[j] = got;
                if (m.gather_cp) *a.total += (unsigned long long)got;
            }
            a.facts[i] = f;
        }
    });
}
hipError_t sparsify_count(int n, const int* cp, const int* ri, const double* v, SparsifySpec sp, double*, int* counts,
                          hipStream_t s) {
    return enqueue(s, [=] {
        for (int j = 0; j < n; ++j) counts[j] = (int)kept(cp, ri, v, sp, j).size();
    });
}
hipError_t sparsify_fill(int n, const int* cp, const int* ri, const double* v, SparsifySpec sp, const double*,
                         const int* out_cp, int* out_ri, hipStream_t s) {
    return enqueue(s, [=] {
        for (int j = 0; j < n; ++j) {
            const auto r = kept(cp, ri, v, sp, j);
            std::copy(r.begin(), r.end(), out_ri + out_cp[j]);
        }
    });
}
hipError_t sparsify_slots(int n, const int* cp, const int* ri, const double* v, SparsifySpec sp, double* d,
                          const int* slot_cp, int* slot_ri, int* counts, hipStream_t s) {
    (void)sparsify_count(n, cp, ri, v, sp, d, counts, s);
    return sparsify_fill(n, cp, ri, v, sp, d, slot_cp, slot_ri, s);
}
hipError_t expand_slots(int n, const int* P_cp, const int* P_cnt, const int* P_ri, const int* Q_cp, const int* Q_cnt,
                        const int* Q_ri, const int* slot_cp, int* slot_ri, int* counts, int, int, hipStream_t s) {
    return enqueue(s, [=] {
        for (int j = 0; j < n; ++j) {
            const auto r = united(P_cp, P_cnt, P_ri, Q_cp, Q_cnt, Q_ri, j);
            if (slot_ri) std::copy(r.begin(), r.end(), slot_ri + slot_cp[j]);
            if (counts) counts[j] = (int)r.size();
        }
    });
}
hipError_t expand_count(int n, const int* P_cp, const int* P_ri, const int* Q_cp, const int* Q_ri, int* counts, int*,
                        int, hipStream_t s) {
    return expand_slots(n, P_cp, nullptr, P_ri, Q_cp, nullptr, Q_ri, nullptr, nullptr, counts, 0, 0, s);
}
hipError_t expand_fill(int n, const int* P_cp, const int* P_ri, const int* Q_cp, const int* Q_ri, const int* out_cp,
                       int* out_ri, int, int, hipStream_t s) {
    return expand_slots(n, P_cp, nullptr, P_ri, Q_cp, nullptr, Q_ri, out_cp, out_ri, nullptr, 0, 0, s);
}
hipError_t plan_positions_slots(int n, const int* S_cp, const int* S_cnt, const int* S_ri, const int* cS_cp, int* cS_ri,
                                const int* Ak_cp, const int* Ak_ri, const int*, const int*, const int64_t*, int* nI,
                                unsigned char*, unsigned char*, int, int, hipStream_t s) {
    return enqueue(s, [=] {
        for (int j = 0; j < n; ++j) {
            nI[j] = (int)united(S_cp, S_cnt, S_ri, Ak_cp, nullptr, Ak_ri, j).size();
            if (cS_ri) std::copy(S_ri + S_cp[j], S_ri + S_cp[j] + S_cnt[j], cS_ri + cS_cp[j]);
        }
    });
}
hipError_t plan_positions(int n, const int* S_cp, const int* S_ri, const int* Ak_cp, const int* Ak_ri, const int*,
                          const int*, const int64_t*, int* nI, unsigned char*, unsigned char*, int, int, hipStream_t s) {
    return plan_positions_slots(n, S_cp, nullptr, S_ri, nullptr, nullptr, Ak_cp, Ak_ri, nullptr, nullptr, nullptr, nI,
                                nullptr, nullptr, 0, 0, s);
}
hipError_t shape_histogram(int n, const int* S_cp, const int* nI, int* hist, hipStream_t s) {
    return enqueue(s, [=] {
        std::fill(hist, hist + kShapeCells, 0);
        for (int j = 0; j < n; ++j) {
            const int r = nI[j], c = S_cp[j + 1] - S_cp[j];
            ++hist[r <= kShapeRows && c <= kShapeCols ? r * (kShapeCols + 1) + c : kShapeCells - 1];
        }
    });
}
size_t bucket_temp_bytes(int jobs) { return 256 * (size_t)jobs; }
hipError_t bucket_sort(int n, const int* S_cp, const int* nI, const BucketJobs& jobs, unsigned long long*, void*,
                       hipStream_t s) {
    return enqueue(s, [=] {
        for (int k = 0; k < jobs.count; ++k) {
            const BucketJob& job = jobs.job[k];
            int at = 0;
            std::vector<int> first((size_t)n);
            for (int j = 0; j < n; ++j) {
                const int c = S_cp[j + 1] - S_cp[j], r = job.tab.penalty_rows ? std::max(nI[j], 2 * c) : nI[j];
                int b = 0;
                while (b < job.tab.nb && (r > job.tab.max_rows[b] || c > job.tab.max_cols[b])) ++b;
                first[(size_t)j] = b;
            }
            for (int b = 0; b < job.tab.nb; ++b) {
                job.bstart[b] = at;
                for (int j = 0; j < n; ++j)
                    if (first[(size_t)j] == b) job.queue[at++] = j;
            }
            job.bstart[job.tab.nb] = at;
        }
    });
}
size_t reduce_temp_bytes(int64_t) { return 256; }
hipError_t reduce_sum(const double*, int64_t, double*, void*, hipStream_t) { return hipSuccess; }
hipError_t reduce_sumsq(const double*, int64_t, double*, void*, hipStream_t) { return hipSuccess; }
hipError_t residual_columns(int, int64_t, int64_t, const int*, const int*, const double*, const int*, const int*,
                            const double*, const int*, const int*, const void*, int, double*, unsigned long long*,
                            hipStream_t) { return hipSuccess; }
hipError_t fill_i32(int* p, int64_t count, int v, hipStream_t s) {
    return enqueue(s, [=] { std::fill(p, p + count, v); });
}
hipError_t set4_i32(int* p, int a, int b, int c, int d, hipStream_t s) {
    return enqueue(s, [=] { p[0] = a, p[1] = b, p[2] = c, p[3] = d; });
}
hipError_t identity_queue(int n, int* queue, int* bstart, hipStream_t s) {
    return enqueue(s, [=] {
        for (int i = 0; queue && i < n; ++i) queue[i] = i;
        bstart[0] = 0;
        bstart[1] = n;
    });
}
hipError_t transpose_count(int, const int*, const int*, int64_t, int*, hipStream_t) { return hipSuccess; }
hipError_t transpose_fill(int, const int*, const int*, const int*, int*, int*, int*, hipStream_t) { return hipSuccess; }
hipError_t transpose_sort_rows(int, const int*, int*, int*, hipStream_t) { return hipSuccess; }
hipError_t spmv_rows(int, const int*, const int*, const int*, const void*, int, const double*, double*, hipStream_t) {
    return hipSuccess;
}
hipError_t permute_vals(int64_t, const int*, const void*, int, void*, hipStream_t) { return hipSuccess; }

}  // namespace samk

// ------------------------------------------------------------------ tests
namespace {

struct Buf {
    void* p;
    size_t bytes;
    explicit Buf(size_t n) : p(aligned_alloc(256, samh::align256(n))), bytes(samh::align256(n)) { memset(p, 0xA5, bytes); }
    Buf(const Buf&) = delete;
    ~Buf() { free(p); }
};

void ok(sam_status st, sam_ctx* ctx, const char* what) {
    if (st == SAM_OK) return;
    printf("WRONG: %s: %s\n", what, sam_last_error(ctx));
    exit(1);
}

// A five-point stencil on an m x m grid; `shift` makes the entries that a rule
// drops differ between sources.
struct Matrix {
    int n;
    std::vector<int> cp, ri;
    std::vector<double> v;
    explicit Matrix(int m, int shift = 0) : n(m * m), cp{0} {
        for (int j = 0; j < n; ++j) {
            const int x = j % m, y = j / m;
            auto put = [&](int r, bool in) {
                if (!in) return;
                ri.push_back(r);
                v.push_back(r == j ? 4.0 : (r * 7 + j * 3 + shift) % 5 ? -1.0 : -0.25);
            };
            put(j - m, y > 0);
            put(j - 1, x > 0);
            put(j, true);
            put(j + 1, x + 1 < m);
            put(j + m, y + 1 < m);
            cp.push_back((int)ri.size());
        }
    }
    sam_csc csc() const { return sam_csc{n, (int32_t)ri.size(), cp.data(), ri.data(), v.data()}; }
};

void served(int times, const char* what) {
    for (size_t j = 0; j < samk::g_visits.size(); ++j)
        if (samk::g_visits[j] != times) return wrong(what, (long)j, samk::g_visits[j]);
}
void clear(int n) { samk::g_visits.assign((size_t)n, 0); }

hipStream_t stream() {
    hipStream_t s;
    (void)hipStreamCreateWithFlags(&s, 0);
    return s;
}

struct Plan {
    sam_ctx* ctx;
    Matrix A;
    sam_csc a;
    std::vector<int> S_cp, S_ri;
    std::vector<char> mem;
    Buf* buf = nullptr;
    sam_plan* plan = nullptr;
    Plan(sam_ctx* c, int m, hipStream_t s) : ctx(c), A(m), a(A.csc()) {
        sam_pattern_spec spec{};
        spec.power = 2;
        size_t nb = 0;
        int64_t nnz = 0;
        ok(sam_pattern_workspace_size(ctx, &a, &spec, &nb, s), ctx, "pattern size");
        Buf ws(nb);
        ok(sam_pattern_count(ctx, &a, &spec, ws.p, nb, &nnz, s), ctx, "pattern count");
        S_cp.resize((size_t)A.n + 1);
        S_ri.resize((size_t)nnz);
        ok(sam_pattern_fill(ctx, &a, &spec, ws.p, nb, S_cp.data(), S_ri.data(), s), ctx, "pattern fill");
        (void)hipStreamSynchronize(s);
        ok(sam_plan_size(ctx, &a, &a, S_cp.data(), S_ri.data(), nnz, &nb, s), ctx, "plan size");
        buf = new Buf(nb);
        ok(sam_plan_create(ctx, &a, &a, S_cp.data(), S_ri.data(), nnz, buf->p, nb, &plan, s), ctx, "plan");
    }
    ~Plan() {
        ok(sam_plan_destroy(plan), ctx, "plan destroy");
        delete buf;
    }
    void build(int prec, hipStream_t s) {
        std::vector<double> M(S_ri.size());
        clear(A.n);
        ok(sam_build_planned(plan, a.val, a.val, prec, M.data(), nullptr, nullptr, s), ctx, "build");
        (void)hipStreamSynchronize(s);
        served(1, "columns of a build");
    }
};

struct Seq {
    sam_ctx* ctx;
    int N;
    Matrix A;
    std::vector<Matrix> As;
    sam_csc a;
    Buf* buf = nullptr;
    sam_seq* seq = nullptr;
    std::vector<double> M, res2;
    Seq(sam_ctx* c, int m, int n_src, int kind, int power, int replan, hipStream_t s)
        : ctx(c), N(n_src), A(m), a(A.csc()), res2((size_t)n_src) {
        for (int k = 0; k < N; ++k) As.emplace_back(m, k);
        sam_pattern_spec spec{};
        spec.kind = kind;
        spec.power = power;
        spec.tau = 0.5;
        size_t nb = 0, total = 0;
        ok(sam_pattern_workspace_size(ctx, &a, &spec, &nb, s), ctx, "pattern size");
        Buf ws(nb);
        ok(sam_sequence_size(ctx, &a, &a, &spec, N, 1, replan, ws.p, nb, &total, s), ctx, "sequence size");
        buf = new Buf(total);
        ok(sam_sequence_create(ctx, &a, &a, &spec, N, 1, replan, buf->p, total, &seq, s), ctx, "sequence");
        int64_t bound = 0;
        ok(sam_sequence_info(seq, &bound), ctx, "info");
        M.resize((size_t)bound * 2);
    }
    ~Seq() {
        ok(sam_sequence_destroy(seq), ctx, "sequence destroy");
        delete buf;
    }
    // which = 0 or 1: two sets of outputs
    void run(int which, hipStream_t s) {
        std::vector<const double*> v;
        std::vector<void*> m;
        for (int k = 0; k < N; ++k) {
            v.push_back(As[(size_t)k].v.data());
            m.push_back(M.data() + which * (M.size() / 2));
        }
        ok(sam_sequence_run(seq, v.data(), m.data(), res2.data(), s), ctx, "run");
    }
};

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    sam_ctx* ctx = nullptr;
    if (sam_create(&ctx, 0) != SAM_OK) return 1;
    const hipStream_t s = stream(), other = stream();
    int done = 0;
    if (what == "plan") {   // a plan made on one stream serves builds on another at once
        for (int m : {3, 7})
            for (int prec : {1, 0}) {
                Plan p(ctx, m, s);
                p.build(prec, other);
                ++done;
            }
    } else if (what == "sequence") {   // the same for a sequence
        for (int replan : {0, 1})
            for (int kind : {SAM_SPARSIFY_NONE, SAM_SPARSIFY_COLUMN}) {
                Seq q(ctx, 7, 4, kind, 2, replan, s);
                clear(q.A.n);
                q.run(0, other);
                (void)hipStreamSynchronize(other);
                served(q.N, "columns of a run");
                ++done;
            }
    } else if (what == "outputs") {   // other outputs while the last runs are still on their way
        for (hipStream_t second : {s, other}) {
            Seq q(ctx, 6, 4, SAM_SPARSIFY_COLUMN, 2, 1, s);
            clear(q.A.n);
            for (int k = 0; k < 7; ++k) q.run(0, s);   // some of them a graph's
            const bool waited = of(s)->ops.empty();
            if (second != s) (void)hipStreamSynchronize(s);   // runs of one sequence do not overlap
            q.run(1, second);
            if (second == s && (waited || of(s)->ops.empty())) wrong("a run waited for another on its stream");
            for (int k = 0; k < 9; ++k) q.run(k & 1, second);
            (void)hipDeviceSynchronize();
            served(17 * q.N, "columns of the runs");
            ++done;
        }
    } else if (what == "graphs") {   // which runs a graph takes
        for (int replan : {0, 1}) {
            Seq q(ctx, 5, 3, SAM_SPARSIFY_NONE, 2, replan, s);
            const int32_t wide[] = {3};
            auto runs = [&](int which, int k, int graph, const char* what) {
                const int before = g_graph_launches;
                clear(q.A.n);
                for (int i = 0; i < k; ++i) q.run(which, s);
                (void)hipStreamSynchronize(s);
                served(k * q.N, "columns of the runs");
                if (g_graph_launches - before != graph) wrong(what, g_graph_launches - before, graph);
            };
            runs(0, 7, 3, "the fifth run is captured");
            runs(1, 2, 0, "other outputs are not, at first");
            for (int i = 0; i < 2; ++i) {   // alternating outputs
                runs(0, 1, 1, "the first come back to their graph");
                runs(1, 1, 0, "outputs that came fewer than five times");
            }
            runs(1, 3, 3, "the fifth time");
            ok(sam_sequence_select(q.seq, wide, 1, s), ctx, "select");
            runs(0, 4, 0, "a graph of other classes is not launched");
            runs(0, 2, 2, "the new classes get one of their own");
            for (int i = 0; i < 5; ++i) {
                ok(sam_sequence_select(q.seq, wide, 1, s), ctx, "select");
                runs(0, 6, i == 0 ? 2 : 0, "four graphs at most");
            }
            ++done;
        }
    } else if (what == "select") {   // other classes while the last run is still on its way on another stream
        for (int replan : {0, 1})
            for (int before : {1, 6}) {   // runs, the last by a graph or not
                Seq q(ctx, 6, 4, SAM_SPARSIFY_NONE, 2, replan, s);
                const int32_t wide[] = {3}, many[] = {0, 1, 2, 3};
                ok(sam_sequence_select(q.seq, many, 4, s), ctx, "select");
                clear(q.A.n);
                for (int k = 0; k < before; ++k) q.run(0, s);
                ok(sam_sequence_select(q.seq, wide, 1, other), ctx, "select");
                q.run(0, other);
                (void)hipDeviceSynchronize();
                served((before + 1) * q.N, "columns of the runs");
                ++done;
            }
    } else if (what == "orders") {   // every kind of order, good and refused, runs between them
        std::mt19937 rng(argc > 2 ? (unsigned)atoi(argv[2]) : 0);
        auto pick = [&](int k) { return (int)(rng() % (unsigned)k); };
        for (int round = 0; round < 12; ++round) {
            const int replan = pick(2), kind = pick(2) ? SAM_SPARSIFY_COLUMN : SAM_SPARSIFY_NONE;
            Seq q(ctx, 2 + pick(6), 1 + pick(5), kind, 1 + pick(3), replan, s);
            for (int i = 0; i < 40; ++i) {
                std::vector<int32_t> order;
                for (int k = pick(8); k > 0; --k) order.push_back(pick(samk::kF32 + 1) - (pick(20) == 0));
                const sam_status st = sam_sequence_select(q.seq, order.data(), (int32_t)order.size(), pick(2) ? s : other);
                bool valid = !order.empty();
                for (int32_t x : order) valid &= x >= 0 && x < samk::kF32;
                if (!valid && st != SAM_ERR_ARG) wrong("a bad order was not refused", st);
                if (valid && st != SAM_OK && st != SAM_ERR_UNSUPPORTED) wrong("status of an order", st);
                if (pick(3) == 0) continue;
                (void)hipDeviceSynchronize();
                clear(q.A.n);
                const int runs = 1 + pick(8);
                const hipStream_t on = pick(2) ? s : other;
                for (int k = 0, which = pick(2); k < runs; ++k) q.run(pick(4) ? which : 1 - which, on);
                (void)hipDeviceSynchronize();
                served(runs * q.N, "columns of a selected run");
            }
            ++done;
        }
    } else {
        return 2;
    }
    (void)hipDeviceSynchronize();
    sam_destroy(ctx);
    for (hipStream_t x : {s, other}) (void)hipStreamDestroy(x);
    printf("%d cases, %d wrong\n", done, g_errors);
    return g_errors ? 1 : 0;
}
