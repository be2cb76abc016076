// sam_krylov_api.cpp -- C ABI of the GMRES steps (kernels: sam_krylov.hip).
#include "sam_host.hpp"

#include <climits>

using namespace samh;

namespace {

size_t gmres_layout(Carve& cv, int n, int restart, samk::GmresArgs* a) {
    const size_t chunks = (size_t)samk::gmres_chunks(n), m = (size_t)restart + 1;
    samk::GmresArgs x{};
    x.w = cv.take<double>((size_t)n);
    x.part = cv.take<double>(m * chunks);
    x.part2 = cv.take<double>(m * chunks);
    x.nrm = cv.take<double>(chunks);
    x.h1 = cv.take<double>(m);
    x.h2 = cv.take<double>(m);
    x.cs = cv.take<double>(m);
    x.sn = cv.take<double>(m);
    if (a) *a = x;
    return cv.off;
}

bool sizes_ok(int32_t n, int32_t restart) { return n >= 1 && restart >= 1 && restart <= SAM_GMRES_MAX_RESTART; }

}  // namespace

extern "C" {

sam_status sam_gmres_workspace_size(int32_t n, int32_t restart, size_t* bytes) {
    if (!sizes_ok(n, restart) || !bytes) return SAM_ERR_ARG;
    Carve cv(nullptr);
    *bytes = gmres_layout(cv, n, restart, nullptr);
    return SAM_OK;
}

sam_status sam_gmres_steps(sam_ctx* ctx, int32_t n, const int32_t* A_rowptr, const int32_t* A_colind,
                           const double* A_val, const int32_t* N_rowptr, const int32_t* N_colind, const void* N_val,
                           int32_t N_prec, const double* d, int32_t restart, int32_t first, int32_t count, double beta,
                           double tol, double* V, double* Z, double* H, double* state, void* ws, size_t ws_bytes,
                           sam_stream_t stream) {
    if (check_ctx(ctx)) return SAM_ERR_ARG;
    if (!sizes_ok(n, restart)) return fail(ctx, SAM_ERR_ARG, "n = %d, restart = %d out of range", n, restart);
    if (first < 0 || count < 0 || first > restart || count > restart - first)
        return fail(ctx, SAM_ERR_ARG, "steps %d .. +%d outside the cycle of %d", first, count, restart);
    if (!prec_ok(N_prec)) return fail(ctx, SAM_ERR_ARG, "unknown precision %d", (int)N_prec);
    if (!A_rowptr || !A_colind || !A_val || !d || !V || !Z || !H || !state ||
        (N_rowptr && (!N_colind || !N_val)))
        return fail(ctx, SAM_ERR_ARG, "NULL argument");
    Carve cv(ws);
    samk::GmresArgs a;
    sam_status st;
    if ((st = check_ws(ctx, ws, ws_bytes, gmres_layout(cv, n, restart, &a), "GMRES workspace"))) return st;
    if ((st = need_device(ctx))) return st;
    hipStream_t s = S(stream);
    a.n = n;
    a.restart = restart;
    a.A_rowptr = A_rowptr;
    a.A_colind = A_colind;
    a.A_val = A_val;
    a.N_rowptr = N_rowptr;
    a.N_colind = N_colind;
    a.N_val = N_val;
    a.N_f32 = N_prec == SAM_PREC_F32_REFINE;
    a.d = d;
    a.V = V;
    a.Z = Z;
    a.H = H;
    a.state = state;
    a.tol = tol;
    if (first == 0) HIP_TRY(ctx, samk::gmres_init(restart, beta, state, s));
    HIP_TRY(ctx, samk::gmres_steps(a, first, count, s));
    return SAM_OK;
}

sam_status sam_gmres_solution(sam_ctx* ctx, int32_t n, int32_t used, const double* y, const double* Z, double* x,
                              sam_stream_t stream) {
    if (check_ctx(ctx)) return SAM_ERR_ARG;
    if (n < 1 || used < 0) return fail(ctx, SAM_ERR_ARG, "n = %d, used = %d out of range", n, used);
    if (used > 0 && (!y || !Z || !x)) return fail(ctx, SAM_ERR_ARG, "NULL argument");
    sam_status st = need_device(ctx);
    if (st) return st;
    HIP_TRY(ctx, samk::gmres_solution(n, used, y, Z, x, S(stream)));
    return SAM_OK;
}

}  // extern "C"
