// Factor (Algorithm 1 and the boundary-to-boundary maps), apply (Algorithm 2),
// the stencil, the single-operator hook and per-kernel timing of the C ABI.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "asp_internal.h"

namespace {

size_t elem_bytes(const asp_plan* P) { return P->prec != ASP_PREC_FP64 ? sizeof(zf) : sizeof(zd); }

template <typename T>
asp_status dev_alloc(asp_plan* P, T** p, size_t count) {
    if (devmem_alloc(reinterpret_cast<void**>(p), count * sizeof(T)) != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return plan_fail(P, ASP_ERR_OOM, "device allocation failed");
    }
    return ASP_OK;
}

void dev_free(void* p) {
    devmem_free(p);
}

// elements of one slot-fastest vector of an apply over nrhs right-hand sides
size_t vec2_elems(const asp_plan* P, int nrhs) { return (size_t)nrhs * P->N; }

// the vectors of an apply over nact right-hand sides in the plan's workspace
Apply2 apply2_of(const asp_plan* P, int nact) {
    Apply2 v;
    char* b = reinterpret_cast<char*>(P->d_U);
    const size_t len = vec2_elems(P, P->ws_rhs) * elem_bytes(P);
    v.R = v.A = b;
    v.U = b + len;
    v.C = b + 2 * len;
    v.W = P->d_W;
    v.nact = nact;
    return v;
}

// algorithmic bytes and flops of a batch of layer solves: each factor entry
// read once per launch, each right-hand side's data and results (io bytes) once
void solve_cost(const asp_plan* P, int sub0, int nsub, int nact, double io, double* bytes, double* flops) {
    double fb = 0, fl = 0;
    for (int s = sub0; s < sub0 + nsub; ++s) {
        fb += factor_bytes_of(P, P->subs[s]);
        const double L = P->subs[s].L;
        fl += 2.0 * P->n * L * L * 8.0;   // forward + backward, L^2 complex MACs per block
    }
    *bytes = fb + io * nact;
    *flops = fl * nact;
}

// bytes of an R or L problem's boundary row (double) and of its results on X_p
double rl_io(const asp_plan* P, int sub) {
    const SubDesc& d = P->subs[sub];
    return (double)P->n * sizeof(zd) + (double)P->n * (d.xe - d.xs + 1) * elem_bytes(P);
}

}  // namespace

size_t solve_scratch_bytes(const asp_plan* P) {
    return P->dim == 2 ? (size_t)P->y_elems * elem_bytes(P) : 0;
}

BufSizes factor_work_sizes(const asp_plan* P) {
    if (P->dim == 3)
        return P->rec ? rec_factor_work_sizes(P) : P->nd ? nd_factor_work_sizes(P) : factor3d_work_sizes(P);
    return BufSizes{};   // 2D: the factorization and the boundary maps use no work buffers
}

double factor_bytes_of(const asp_plan* P, const SubDesc& d) {
    const double B = (P->dim == 2) ? d.L : (double)P->n * d.L;
    return (double)P->n * B * B * elem_bytes(P);
}

// ---------------------------------------------------------------------------
// timing
// ---------------------------------------------------------------------------
KTimer::KTimer(asp_plan* p, int c, double bytes, double flops, int launches)
    : P(p), cls(c), on(p->timing) {
    if (!on) return;
    if (P->tpool_used + 2 > P->tpool.size()) {
        for (int k = 0; k < 64; ++k) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) {
                on = false;
                return;
            }
            P->tpool.push_back(e);
        }
    }
    hipEvent_t a = P->tpool[P->tpool_used++], b = P->tpool[P->tpool_used++];
    P->tev[cls].push_back({a, b, launches});
    P->tbytes[cls] += bytes;
    P->tflops[cls] += flops;
    (void)hipEventRecord(a, P->stream);
}

void KTimer::end() {
    if (on) (void)hipEventRecord(P->tev[cls].back().b, P->stream);
    on = false;
}

extern "C" asp_status asp_timing_enable(asp_plan* P, int enable) {
    if (!P) return ASP_ERR_ARG;
    if (enable) {
        ASP_HIP(P, hipStreamSynchronize(P->stream));
        for (int c = 0; c < ASP_K_COUNT; ++c) {
            P->tev[c].clear();
            P->tbytes[c] = P->tflops[c] = 0;
        }
        P->tpool_used = 0;
    }
    P->timing = enable != 0;
    return ASP_OK;
}

extern "C" asp_status asp_timing_read(asp_plan* P, int cls, int* launches, double* ms,
                                      double* bytes, double* flops) {
    if (!P || cls < 0 || cls >= ASP_K_COUNT) return ASP_ERR_ARG;
    ASP_HIP(P, hipStreamSynchronize(P->stream));
    double tot = 0;
    int nl = 0;
    for (auto& sp : P->tev[cls]) {
        float t = 0;
        ASP_HIP(P, hipEventElapsedTime(&t, sp.a, sp.b));
        tot += t;
        nl += sp.launches;
    }
    if (launches) *launches = nl;
    if (ms) *ms = tot;
    if (bytes) *bytes = P->tbytes[cls];
    if (flops) *flops = P->tflops[cls];
    return ASP_OK;
}

// ---------------------------------------------------------------------------
// workspaces
// ---------------------------------------------------------------------------
asp_status ensure_apply_ws(asp_plan* P, int nrhs) {
    if (P->dim == 3)
        return P->rec ? rec_ensure_ws(P, nrhs) : P->nd ? nd_ensure_ws(P, nrhs) : ensure_apply_ws3(P, nrhs);
    nrhs = std::min(nrhs, apply_max_rhs(P));   // an apply runs in passes of at most that many
    if (nrhs <= P->ws_rhs) return ASP_OK;
    ASP_HIP(P, hipStreamSynchronize(P->stream));
    dev_free(P->d_U);
    dev_free(P->d_W);
    dev_free(P->d_wt);
    dev_free(P->d_y);
    P->d_U = P->d_W = nullptr;
    P->d_wt = P->d_y = nullptr;
    P->wt_elems = P->y_elems = 0;
    P->ws_rhs = 0;
    P->ws_bytes = 0;
    const size_t esz = elem_bytes(P);
    const size_t vec = 3 * vec2_elems(P, nrhs) * esz;
    const size_t wlen = (size_t)std::max(2 * P->m - 2, 1) * nrhs * P->n;
    const long long we = sweep_wt_len(P, nrhs), ye = solve_scratch_elems(P, nrhs);
    char* bufs[3] = {nullptr, nullptr, nullptr};
    const size_t bytes[3] = {vec, (size_t)we * esz, (size_t)ye * esz};
    for (int i = 0; i < 3; ++i)
        if (dev_alloc(P, &bufs[i], bytes[i]) != ASP_OK) {
            for (char* b : bufs) dev_free(b);
            return ASP_ERR_OOM;
        }
    P->d_U = reinterpret_cast<zd*>(bufs[0]);
    P->d_wt = bufs[1];
    P->wt_elems = we;
    P->d_y = bufs[2];
    P->y_elems = ye;
    if (dev_alloc(P, &P->d_W, wlen) != ASP_OK) return ASP_ERR_OOM;
    P->ws_rhs = nrhs;
    P->ws_bytes = vec + wlen * sizeof(zd) + (size_t)we * esz;
    return ASP_OK;
}

// whether the apply's third vector over nrhs right-hand sides holds a Krylov vector
static bool shares_vector(const asp_plan* P, int nrhs) {
    return P->dim == 2 && P->prec == ASP_PREC_FP64 && nrhs <= apply_max_rhs(P);
}

zd* shared_vector(const asp_plan* P, int nrhs) {
    return shares_vector(P, nrhs) ? static_cast<zd*>(apply2_of(P, nrhs).C) : nullptr;
}

int krylov_vectors(const asp_plan* P, int nrhs, int restart) {
    return 2 * restart + (shares_vector(P, nrhs) ? 1 : 2);
}

// ---------------------------------------------------------------------------
// apply (Algorithm 2)
// ---------------------------------------------------------------------------
// One pass of a 2D apply over the right-hand sides act[0..nact) (NULL: id0 ..).
static asp_status apply_pass2d(asp_plan* P, const zd* r, zd* z, const int* act, int id0, int nact) {
    hipStream_t st = P->stream;
    const int m = P->m;
    const Apply2 v = apply2_of(P, nact);
    const double esz = elem_bytes(P);
    const double row = (double)nact * P->n;   // entries of one grid line
    double by, fl;
    // u~_{q,q} = G~^M_q f_q for q = 1..m, all at once
    {
        SolveLaunch L;
        L.job0 = 0;
        L.njobs = m;
        L.nact = nact;
        L.in_mode = IN_GRID;
        L.r = v.R;
        L.out = v.U;
        // the caller's vectors into the packed ones, those read, u~ written
        solve_cost(P, 0, m, nact, (double)P->N * (sizeof(zd) + 3 * esz), &by, &fl);
        KTimer t(P, ASP_K_SOLVE_M, by, fl, 1 + solve_launches(P, L));
        ASP_HIP(P, launch_pack2d(P, v, r, P->N, 1, P->n, 0, act, id0, st));
        ASP_HIP(P, launch_solve2d(P, L, st));
        t.end();
    }
    if (m > 1 && P->sweep_seq) {
        // Algorithm 2 as stated: R_{t+1} and L_{m-t} solved in step t (one launch),
        // each handing its outgoing boundary line (plus u~) to the next problem of
        // its sweep; R outputs a_p in A, L outputs c_p in C
        const double line = row * esz, wline = row * sizeof(zd);
        double sb = 2 * (line + wline) + 2.0 * sweep_wt_line(P, nact) * esz;   // the seed
        double sf = 0;
        for (int t = 1; t <= m - 1; ++t) {
            const int pair[2] = {P->idx_R(t + 1), P->idx_L(m - t)};
            for (int s : pair) {
                solve_cost(P, s, 1, nact, rl_io(P, s), &by, &fl);
                sb += by;
                sf += fl;
            }
            if (t < m - 1) sb += 2 * (2 * line + wline);   // the handed lines
        }
        KTimer t(P, ASP_K_SWEEP, sb, sf, 1 + 2 * (m - 1) + (m - 2));
        ASP_HIP(P, launch_sweep_seed(P, v, P->wrow(P->idx_R(2)), P->wrow(P->idx_L(m - 1)), st));
        const int nsub = (int)P->subs.size();
        for (int s = 1; s <= m - 1; ++s) {
            SolveLaunch L;
            L.job0 = nsub + 2 * (s - 1);
            L.njobs = 2;
            L.rl = true;
            L.nact = nact;
            L.in_mode = IN_BOUNDARY;
            L.out = v.A;
            L.out_L = v.C;
            L.W = v.W;
            ASP_HIP(P, launch_solve2d(P, L, st));
            if (s < m - 1)
                ASP_HIP(P, launch_sweep_hand(P, v, P->wrow(P->idx_R(s + 2)), P->X[s][1],
                                             P->wrow(P->idx_L(m - s - 1)), P->X[m - s - 1][0], st));
        }
        t.end();
    } else if (m > 1) {
        // the two sweeps: the boundary values u~^R_{p,1:p} and u~^L_{p,p:m}
        // accumulated layer by layer (W rows hold the data entering R_p / L_p); the
        // seed and the m-2 steps are timed as one span of m-1 launches
        {
            const double line = row * esz, wline = row * sizeof(zd);
            const double nn = (double)P->n * P->n;
            const double steps = m - 2;
            // the seed; a step and side: the map, W in, u~, W out in both precisions
            KTimer t(P, ASP_K_SWEEP,
                     2 * (line + wline) + 2.0 * sweep_wt_line(P, nact) * esz +
                         steps * 2 * (nn * esz + 3 * line + wline),
                     steps * 2.0 * nn * nact * 8.0, m - 1);
            ASP_HIP(P, launch_sweep_seed(P, v, P->wrow(P->idx_R(2)), P->wrow(P->idx_L(m - 1)), st));
            for (int s = 1; s <= m - 2; ++s) ASP_HIP(P, launch_sweep_step(P, v, s, st));
            t.end();
        }
        // one launch of every R_p (a on X_p, p > 1) and L_p (c, p < m)
        SolveLaunch L;
        L.job0 = P->idx_R(2);
        L.njobs = 2 * m - 2;
        L.rl = true;
        L.nact = nact;
        L.in_mode = IN_BOUNDARY;
        L.out = v.A;
        L.out_L = v.C;
        L.W = v.W;
        double io = 0;
        for (int s = L.job0; s < L.job0 + L.njobs; ++s) io += rl_io(P, s);
        solve_cost(P, L.job0, L.njobs, nact, io, &by, &fl);
        KTimer t(P, ASP_K_SOLVE_RL, by, fl, solve_launches(P, L));
        ASP_HIP(P, launch_solve2d(P, L, st));
        t.end();
    }
    // u~_p = u~_{p,1:p-1} + u~_{p,p} + u~_{p,p+1:m}
    {
        // u~ on every line, a from line a0, c up to line c1, the caller's vectors
        const int a0 = P->X[0][1] + 1, c1 = m > 1 ? P->X[m - 2][1] : 0;
        KTimer t(P, ASP_K_COMBINE, row * ((P->n + (P->n - a0 + 1) + c1) * esz + P->n * (double)sizeof(zd)), 0.0);
        ASP_HIP(P, launch_unpack2d(P, v, v.U, m > 1 ? v.A : nullptr, m > 1 ? v.C : nullptr, a0, c1, z, P->N, 1,
                                   P->n, 0, act, id0, st));
        t.end();
    }
    return ASP_OK;
}

// z = M^-1 r for the right-hand-side ids act[0..nact) (device list, NULL for
// 0..nact-1) of batches laid out with stride N.
asp_status apply_internal(asp_plan* P, const zd* r, zd* z, const int* act, int nact) {
    if (P->dim == 3)
        return P->rec ? rec_apply(P, r, z, act, nact)
                      : P->nd ? nd_apply(P, r, z, act, nact) : apply3d_internal(P, r, z, act, nact);
    // passes of as many right-hand sides as the workspace holds
    for (int s0 = 0; s0 < nact; s0 += P->ws_rhs) {
        const asp_status s = apply_pass2d(P, r, z, act ? act + s0 : nullptr, s0, std::min(nact - s0, P->ws_rhs));
        if (s != ASP_OK) return s;
    }
    return ASP_OK;
}

// The boundary maps T^R_p, T^L_p (1 < p < m): column c of a map is the outgoing
// line of G~ (the last line of X_p for R, the first for L) for unit data at
// i1 = c + 1.  With the diagonal blocks G_k of H^-1 (launch_rgf2d), the solution
// at the data's block is the coupling times column grow of G_{c+1}, and from
// there towards the end of its half x_k = -S_k^-1 E_k x_{k+1}: the entries on one
// side of the diagonal; the other side comes from unit data on the outgoing line
// (column jout of G), read on the data line, since H is complex symmetric
// (IN_TWIST kind 0: both).  Entries between the halves are products of two rows
// of the propagators from the middle block (kind 2, then launch_map_cross).
static asp_status compute_transfer(asp_plan* P) {
    const int m = P->m;
    if (m < 3) return ASP_OK;
    const double esz = elem_bytes(P);
    const int nj = m - 2;
    // the diagonal blocks of H^-1 of both sweeps' map problems in one launch
    {
        double fb = 0, fl = 0;
        for (int side = 0; side < 2; ++side) {
            const int first = side == 0 ? P->idx_R(2) : P->idx_L(2);
            for (int s = first; s < first + nj; ++s) {
                const SubDesc& d = P->subs[s];
                fb += factor_bytes_of(P, d);
                fl += (double)P->n * 2.0 * d.L * d.L * d.L * 8.0;   // two L^3 complex products per block
            }
        }
        KTimer t(P, ASP_K_TRANSFER, fb + 2.0 * nj * P->n * 2 * P->LR_RL * esz, fl);
        ASP_HIP(P, launch_rgf2d(P, P->idx_R(2), P->idx_L(2), nj, P->stream));
        t.end();
    }
    double fb = 0, L2 = 0;
    int maxL = 0;
    for (int side = 0; side < 2; ++side) {
        const int first = side == 0 ? P->idx_R(2) : P->idx_L(2);
        for (int s = first; s < first + nj; ++s) {
            const SubDesc& d = P->subs[s];
            fb += factor_bytes_of(P, d);
            L2 += (double)d.L * d.L;
            maxL = std::max(maxL, d.L);
        }
    }
    SolveLaunch L;
    L.job0 = P->idx_R(2);
    L.job1 = P->idx_L(2);
    L.njobs0 = nj;
    L.njobs = 2 * nj;
    L.rl = true;
    L.nact = P->n;
    L.in_mode = IN_TWIST;
    const double nn = (double)P->n * P->n;
    {
        // n^2 / 2 block steps of L^2 complex MACs per problem in all; the factor
        // read once per chunk of columns and triangle over half of a half's blocks
        KTimer t(P, ASP_K_TRANSFER, 0.5 * (P->n / 32.0 + 1) * fb + 0.5 * 2 * nj * nn * esz, 0.5 * nn * L2 * 8.0);
        ASP_HIP(P, launch_solve2d(P, L, P->stream));
        t.end();
    }
    {
        L.twist_kind = 2;
        L.nact = maxL;
        KTimer t(P, ASP_K_TRANSFER, fb, (double)P->n * maxL * L2 * 8.0);
        ASP_HIP(P, launch_solve2d(P, L, P->stream));
        t.end();
    }
    {
        KTimer t(P, ASP_K_TRANSFER, 0.5 * 2 * nj * nn * esz, 0.5 * 2 * nj * nn * maxL * 8.0);
        ASP_HIP(P, launch_map_cross(P, L, P->stream));
        t.end();
    }
    return ASP_OK;
}

extern "C" asp_status asp_factor(asp_plan* P) {
    if (!P) return ASP_ERR_ARG;
    if (P->host_only) return plan_fail(P, ASP_ERR_STATE, "host-only plan");
    P->factored = false;
    if (!P->d_fac) {
        char* f = nullptr;
        if (dev_alloc(P, &f, P->fac_bytes) != ASP_OK) return ASP_ERR_OOM;
        P->d_fac = f;
    }
    if (P->dim == 3) {
        ASP_HIP(P, hipMemsetAsync(P->d_flag, 0, sizeof(int), P->stream));
        asp_status s3 = P->rec ? rec_factor(P) : P->nd ? nd_factor(P) : factor3d(P);
        if (s3 != ASP_OK) return s3;
        int flag3 = 0;
        ASP_HIP(P, hipMemcpyAsync(&flag3, P->d_flag, sizeof(int), hipMemcpyDeviceToHost, P->stream));
        ASP_HIP(P, hipStreamSynchronize(P->stream));
        if (flag3)
            return plan_fail(P, ASP_ERR_BREAKDOWN, "zero or non-finite pivot in a layer factorization");
        P->factored = true;
        return ASP_OK;
    }
    if (!P->d_T && P->t_bytes > 0) {
        char* t = nullptr;
        if (dev_alloc(P, &t, P->t_bytes) != ASP_OK) return ASP_ERR_OOM;
        P->d_T = t;
    }
    asp_status s = ASP_OK;
    ASP_HIP(P, hipMemsetAsync(P->d_flag, 0, sizeof(int), P->stream));
    {
        double fb = 0, fl = 0;
        for (const auto& d : P->subs) {
            fb += factor_bytes_of(P, d);
            fl += (double)P->n * ((double)d.L * d.L * d.L + 2.0 * d.L * d.L) * 8.0;
        }
        KTimer t(P, ASP_K_FACTOR, fb + P->N * sizeof(double), fl);
        ASP_HIP(P, launch_factor2d(P, P->stream));
        t.end();
    }
    int flag = 0;
    ASP_HIP(P, hipMemcpyAsync(&flag, P->d_flag, sizeof(int), hipMemcpyDeviceToHost, P->stream));
    ASP_HIP(P, hipStreamSynchronize(P->stream));
    if (flag) return plan_fail(P, ASP_ERR_BREAKDOWN, "zero or non-finite pivot in a layer factorization");
    if (!P->sweep_seq && (s = compute_transfer(P)) != ASP_OK) return s;
    ASP_HIP(P, hipStreamSynchronize(P->stream));
    P->factored = true;
    return ASP_OK;
}

extern "C" asp_status asp_apply(asp_plan* P, const void* r, void* z, int nrhs) {
    if (!P) return ASP_ERR_ARG;
    if (!r || !z || nrhs < 1) return plan_fail(P, ASP_ERR_ARG, "asp_apply: bad arguments");
    if (r == z) return plan_fail(P, ASP_ERR_ARG, "asp_apply: r and z must not alias");
    if (!P->factored) return plan_fail(P, ASP_ERR_STATE, "asp_apply before asp_factor");
    asp_status s = ensure_apply_ws(P, nrhs);
    if (s != ASP_OK) return s;
    return apply_internal(P, static_cast<const zd*>(r), static_cast<zd*>(z), nullptr, nrhs);
}

extern "C" asp_status asp_matvec(asp_plan* P, const void* x, void* y, int nrhs) {
    if (!P) return ASP_ERR_ARG;
    if (!x || !y || nrhs < 1 || x == y) return plan_fail(P, ASP_ERR_ARG, "asp_matvec: bad arguments");
    if (P->host_only) return plan_fail(P, ASP_ERR_STATE, "host-only plan");
    KTimer t(P, ASP_K_STENCIL, (double)nrhs * P->N * 32.0 + P->N * 8.0, 40.0 * nrhs * P->N);
    ASP_HIP(P, launch_stencil(P, static_cast<const zd*>(x), static_cast<zd*>(y), nullptr, nrhs,
                              P->stream));
    t.end();
    return ASP_OK;
}

extern "C" asp_status asp_subsolve(asp_plan* P, int kind, int p, const void* in, void* out,
                                   int nrhs) {
    if (!P) return ASP_ERR_ARG;
    if (!in || !out || nrhs < 1) return plan_fail(P, ASP_ERR_ARG, "asp_subsolve: bad arguments");
    const int m = P->m;
    int idx;
    if (kind == ASP_SUB_M && p >= 1 && p <= m) idx = P->idx_M(p);
    else if (kind == ASP_SUB_R && p >= 2 && p <= m) idx = P->idx_R(p);
    else if (kind == ASP_SUB_L && p >= 1 && p <= m - 1) idx = P->idx_L(p);
    else return plan_fail(P, ASP_ERR_ARG, "asp_subsolve: no such auxiliary problem");
    if (!P->factored) return plan_fail(P, ASP_ERR_STATE, "asp_subsolve before asp_factor");
    asp_status s = ensure_apply_ws(P, nrhs);
    if (s != ASP_OK) return s;
    if (P->dim == 3)
        return P->rec ? rec_subsolve(P, idx, in, out, nrhs)
                      : P->nd ? nd_subsolve(P, idx, in, out, nrhs) : subsolve3d(P, idx, in, out, nrhs);
    const SubDesc& d = P->subs[idx];
    hipStream_t st = P->stream;
    const int lines = d.xe - d.xs + 1;
    const long long Np = P->S * lines;
    for (int s0 = 0; s0 < nrhs; s0 += P->ws_rhs) {
        const int na = std::min(nrhs - s0, P->ws_rhs);
        Apply2 v = apply2_of(P, na);
        SolveLaunch L;
        L.job0 = idx;
        L.njobs = 1;
        L.rl = kind != ASP_SUB_M;
        L.nact = na;
        L.out = v.U;
        if (kind == ASP_SUB_M) {
            ASP_HIP(P, launch_pack2d(P, v, static_cast<const zd*>(in), Np, d.xs, d.xe, d.xs - 1, nullptr, s0, st));
            L.in_mode = IN_GRID;
            L.r = v.R;
        } else {
            ASP_HIP(P, launch_boundary2d(P, v, static_cast<const zd*>(in) + (long long)s0 * P->n, d.wrow, st));
            L.in_mode = IN_BOUNDARY;
            L.W = v.W;
        }
        ASP_HIP(P, launch_solve2d(P, L, st));
        ASP_HIP(P, launch_unpack2d(P, v, v.U, nullptr, nullptr, 0, 0, static_cast<zd*>(out), Np, d.xs, d.xe,
                                   d.xs - 1, nullptr, s0, st));
    }
    return ASP_OK;
}

// ---------------------------------------------------------------------------
// workspace accounting
// ---------------------------------------------------------------------------
static BufSizes workspace_sizes2(const asp_plan* P, int nrhs) {
    const size_t esz = elem_bytes(P);
    const int pass = std::min(nrhs, apply_max_rhs(P));
    BufSizes b;
    b.add(3 * vec2_elems(P, pass) * esz);
    b.add((size_t)std::max(2 * P->m - 2, 1) * pass * P->n * sizeof(zd));
    b.add((size_t)sweep_wt_len(P, pass) * esz);
    b.add((size_t)solve_scratch_elems(P, pass) * esz);
    return b;
}

static BufSizes workspace_sizes(const asp_plan* P, int nrhs, int restart) {
    BufSizes b = P->dim == 2 ? workspace_sizes2(P, nrhs)
                 : P->rec    ? rec_workspace_sizes(P, nrhs)
                 : P->nd     ? nd_workspace_sizes(P, nrhs)
                             : workspace_sizes3(P, nrhs);
    const size_t vec = (size_t)nrhs * P->N * sizeof(zd);
    b.add(vec * (krylov_vectors(P, nrhs, restart) - restart - 1));
    b.add(vec * restart);
    b.add(vec);
    const size_t red = krylov_red_bytes(P->N, nrhs);
    b.add(red);
    b.add((size_t)krylov_small_bytes(P->N, nrhs) - red);
    b.blocks += devmem_block_bytes(nrhs * sizeof(int));   // the list of running right-hand sides
    return b;
}

extern "C" asp_status asp_workspace_estimate(const asp_plan* P, int nrhs, int restart,
                                             size_t* bytes) {
    if (!P || !bytes || nrhs < 1 || restart < 1) return ASP_ERR_ARG;
    *bytes = workspace_sizes(P, nrhs, restart).bytes;
    return ASP_OK;
}

extern "C" asp_status asp_device_bytes(const asp_plan* P, int nrhs, int restart, size_t* factors,
                                       size_t* factor_work, size_t* workspace) {
    if (!P || nrhs < 1 || restart < 1) return ASP_ERR_ARG;
    if (factors) *factors = devmem_block_bytes(P->fac_bytes) + (P->t_bytes ? devmem_block_bytes(P->t_bytes) : 0);
    if (factor_work) *factor_work = factor_work_sizes(P).blocks;
    if (workspace) *workspace = workspace_sizes(P, nrhs, restart).blocks;
    return ASP_OK;
}

extern "C" asp_status asp_release_workspace(asp_plan* P) {
    if (!P) return ASP_ERR_ARG;
    if (P->host_only) return ASP_OK;
    ASP_HIP(P, hipStreamSynchronize(P->stream));
    void* bufs[] = {P->d_U, P->d_W, P->d_stage, P->d_wt, P->d_V, P->d_Z, P->d_b, P->d_red,
                    P->d_small, P->d_act, P->d_y3, P->d_g3, P->d_w3, P->d_nd_v, P->d_nd_x,
                    P->d_nd_lb[0], P->d_nd_lb[1], P->d_nd_rb, P->d_nd_db};
    for (void* b : bufs) dev_free(b);
    P->d_nd_v = P->d_nd_x = nullptr;
    rec_free_ws(P);
    P->d_nd_lb[0] = P->d_nd_lb[1] = nullptr;
    P->d_nd_rb = P->d_nd_db = nullptr;
    P->nd_work_bytes = 0;
    P->d_y3 = P->d_g3 = nullptr;
    P->d_w3 = nullptr;
    P->y3_elems = P->w3_elems = 0;
    P->d_U = P->d_W = P->d_stage = nullptr;
    P->d_wt = nullptr;
    P->d_V = P->d_Z = P->d_b = P->d_red = P->d_small = nullptr;
    P->d_act = nullptr;
    P->ws_rhs = 0;
    P->ws_bytes = 0;
    P->wt_elems = 0;
    P->kr_rhs = P->kr_restart = 0;
    P->kr_bytes = 0;
    // the layer solves' forward results
    dev_free(P->d_y);
    P->d_y = nullptr;
    P->y_elems = 0;
    return ASP_OK;
}
