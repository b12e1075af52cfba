// densify.cpp -- host side of the depth densification (Sec. 6, Eq. 13-20):
// buffers, the captured iteration graph and the convergence loop.
#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "dco_internal.h"

// Longest wait of a one-launch solve's workgroups for each other, in 10 ns: 20 ms.
// An exchange takes 3 to 6 us, so a word that is not there then is that of a
// workgroup which does not run.
constexpr unsigned long long kSolveWait = 2000000;

// Solves that run as launches after a given-up one before the next is tried as one
// launch again: where the CUs stay taken (another process, a masked stream), a try
// costs its wait, and twice as many launches pass before each further one.
constexpr int kFirstPause = 16, kLongestPause = 1024;

// The wait that the environment variable DCO_DENSIFY_WAIT asks for, which lets a test
// force a solve to be given up: a whole number below kSolveWait; else kSolveWait.
static unsigned long long solve_wait() {
    const char* w = getenv("DCO_DENSIFY_WAIT");
    if (!w || *w < '0' || *w > '9') return kSolveWait;
    char* end = nullptr;
    const unsigned long long v = strtoull(w, &end, 10);
    return *end == '\0' && v < kSolveWait ? v : kSolveWait;
}

struct dco_densify {
    int W = 0, H = 0, nblk = 0;
    dco_densify_params p{};
    hipStream_t stream = nullptr;
    DensifyBufs b{};
    hipGraphExec_t exec = nullptr;
    int* flags_host = nullptr;  // pinned copy of b.flags
    int launches = 0;           // graph launches of the last run (0: one launch)
    int device = 0;
    int solve_k = 0;            // pixels per thread of the one-launch solve (0: not possible)
    // longest wait of its workgroups for each other, in 10 ns
    unsigned long long ticks = kSolveWait;
    int given_up = 0;           // one-launch solves given up so far
    int pause = 0, rest = 0;    // solves as launches after the last of them, and left of these
};

// One-launch solves of a process take turns on a device: two of them at once
// could each hold CUs that the other's workgroups wait for.  A turn lasts until the
// solve has ended, with all that its stream holds before it, so a solve that has
// waited longer than solves take (0.3 to 1 ms) goes as launches instead.
static std::timed_mutex g_solve_turn[64];
constexpr std::chrono::milliseconds kTurnWait{2};

extern "C" dco_status dco_densify_default_params(dco_densify_params* out) {
    if (!out) {
        dco_set_error("dco_densify_default_params: out is NULL");
        return DCO_ERR_ARG;
    }
    out->lambda_d = 0.8f;   // Sec. 7.2
    out->lambda_s = 1.2f;
    out->lambda_s2 = 0.02f;
    out->tol = 1e-9;
    out->max_iters = 4000;
    out->iters_per_launch = 16;
    return DCO_OK;
}

static void free_densify(dco_densify* h) {
    DensifyBufs& b = h->b;
    void* ptrs[] = {b.cr, b.cd, b.diag, b.invdiag, b.x,  b.r,     b.q,  b.p[0],
                    b.p[1], b.rz[0], b.rz[1], b.rr[0], b.rr[1], b.pq, b.bb, b.flags,
                    b.words, b.res};
    for (void* q : ptrs) dev_free(q);
    if (h->exec) (void)hipGraphExecDestroy(h->exec);
    pinned_free(h->flags_host);
}

extern "C" void dco_densify_destroy(dco_densify* h) {
    if (!h) return;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    free_densify(h);
    delete h;
}

extern "C" dco_status dco_densify_create(dco_densify** out, int W, int H,
                                         const dco_densify_params* p, void* stream) {
    if (!out) {
        dco_set_error("dco_densify_create: out is NULL");
        return DCO_ERR_ARG;
    }
    *out = nullptr;
    dco_densify_params prm;
    if (p)
        prm = *p;
    else
        dco_densify_default_params(&prm);
    // every block sums all blocks' partials in a fixed order, a cost that grows
    // with the square of the grid: 2^23 pixels (a 3840 x 2160 frame) at most
    if (W < 1 || H < 1 || (long long)W * H > (1LL << 23)) {
        dco_set_error("densify grid %d x %d: need 1 <= W, H and W*H <= 2^23", W, H);
        return DCO_ERR_SHAPE;
    }
    if (!(std::isfinite(prm.lambda_d) && prm.lambda_d >= 0.0f) ||
        !(std::isfinite(prm.lambda_s) && prm.lambda_s >= 0.0f) ||
        !(std::isfinite(prm.lambda_s2) && prm.lambda_s2 >= 0.0f) ||
        !(std::isfinite(prm.tol) && prm.tol >= 0.0) || prm.max_iters < 0 ||
        prm.iters_per_launch < 2 || prm.iters_per_launch > 1024 || (prm.iters_per_launch & 1)) {
        dco_set_error("densify parameters: need finite lambdas and tol >= 0, max_iters >= 0 and "
                      "an even iters_per_launch in [2, 1024]");
        return DCO_ERR_ARG;
    }
    dco_densify* h = new (std::nothrow) dco_densify();
    if (!h) {
        dco_set_error("host allocation failed");
        return DCO_ERR_OOM;
    }
    h->W = W;
    h->H = H;
    h->p = prm;
    h->stream = (hipStream_t)stream;
    const size_t P = (size_t)W * H;
    DensifyBufs& b = h->b;
    auto fail = [&](dco_status s) {
        free_densify(h);
        delete h;
        return s;
    };
    dco_status st;
    int cus = 0;
    if (hipGetDevice(&h->device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, h->device) !=
            hipSuccess) {
        (void)hipGetLastError();
        dco_set_error("hipGetDevice failed: no usable GPU");
        return fail(DCO_ERR_HIP);
    }
    h->ticks = solve_wait();
    h->solve_k = h->device < 64 ? densify_solve_k(W, H, cus) : 0;
    const size_t nb = densify_parts(W, H, h->solve_k);
    h->nblk = (int)nb;
    double** vecs[] = {&b.cr, &b.cd, &b.diag, &b.invdiag, &b.x, &b.r, &b.q, &b.p[0], &b.p[1]};
    for (double** v : vecs)
        if ((st = dev_alloc(v, P)) != DCO_OK) return fail(st);
    double** parts[] = {&b.rz[0], &b.rz[1], &b.rr[0], &b.rr[1], &b.pq, &b.bb};
    for (double** v : parts)
        if ((st = dev_alloc(v, nb)) != DCO_OK) return fail(st);
    if ((st = dev_alloc(&b.flags, 3)) != DCO_OK) return fail(st);
    if ((st = pinned_alloc((void**)&h->flags_host, 3 * sizeof(int))) != DCO_OK) return fail(st);
    if (h->solve_k) {
        if ((st = dev_alloc(&b.words, densify_solve_words(W, H, h->solve_k))) != DCO_OK)
            return fail(st);
        if ((st = dev_alloc(&b.res, 2)) != DCO_OK) return fail(st);
    }
    // one launch = iters_per_launch iterations (two kernels each), captured
    // once on a private stream of default priority; no memset nodes
    hipStream_t cap;
    if (hipStreamCreateWithFlags(&cap, hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        dco_set_error("hipStreamCreate failed");
        return fail(DCO_ERR_HIP);
    }
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        const hipError_t e1 = launch_densify_iters(b, h->solve_k, W, H, prm.tol,
                                                   prm.iters_per_launch, cap);
        e = hipStreamEndCapture(cap, &g);
        if (e == hipSuccess) e = e1;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&h->exec, g, nullptr, nullptr, 0);
    if (g) (void)hipGraphDestroy(g);
    (void)hipStreamDestroy(cap);
    if (e != hipSuccess) {
        dco_set_error("densify graph capture failed: %s", hipGetErrorString(e));
        (void)hipGetLastError();
        return fail(DCO_ERR_HIP);
    }
    *out = h;
    return DCO_OK;
}

extern "C" dco_status dco_densify_run(dco_densify* h, const float* Ds, const float* Dpre,
                                      const uint8_t* Bdp, const float* Mfuse, const float* MI,
                                      float* D) {
    DCO_TRY(need(h, "handle"));
    DCO_TRY(need(Ds, "Ds"));
    DCO_TRY(need(Bdp, "Bdp"));
    DCO_TRY(need(Mfuse, "Mfuse"));
    DCO_TRY(need(MI, "MI"));
    DCO_TRY(need(D, "D"));
    const dco_densify_params& p = h->p;
    h->launches = 0;
    std::unique_lock<std::timed_mutex> turn;
    if (h->rest > 0)
        --h->rest;
    else if (h->solve_k)
        turn = std::unique_lock<std::timed_mutex>(g_solve_turn[h->device], kTurnWait);
    if (turn.owns_lock()) {
        // whole groups of iters_per_launch iterations, as the launches below run
        const long long groups = ((long long)p.max_iters + p.iters_per_launch - 1) /
                                 p.iters_per_launch;
        const long long limit = groups * p.iters_per_launch;
        // D that lies on an input is written only once the solve is known to have
        // ended: a solve given up at its last exchange may have written parts of it
        const size_t P = (size_t)h->W * h->H, F = P * sizeof(float);
        const bool aside = overlap(D, F, Ds, F) || overlap(D, F, Dpre, F) ||
                           overlap(D, F, Bdp, P) || overlap(D, F, Mfuse, F) || overlap(D, F, MI, F);
        DCO_HIP_CHECK(launch_densify_solve(h->b, h->solve_k, Ds, Dpre, Bdp, Mfuse, MI, h->W, h->H,
                                           p.lambda_d, p.lambda_s, p.lambda_s2, p.tol,
                                           (int)(limit < INT_MAX ? limit : INT_MAX), h->ticks,
                                           aside ? (float*)h->b.q : D, h->stream));
        DCO_HIP_CHECK(hipMemcpyAsync(h->flags_host, h->b.flags, 3 * sizeof(int),
                                     hipMemcpyDeviceToHost, h->stream));
        DCO_HIP_CHECK(hipStreamSynchronize(h->stream));
        if (h->flags_host[2] == 0) {
            h->pause = 0;
            if (aside)
                DCO_HIP_CHECK(hipMemcpyAsync(D, h->b.q, F, hipMemcpyDeviceToDevice, h->stream));
            return DCO_OK;
        }
        // given up: its workgroups could not all run (another process held the
        // CUs); the launches below need nothing to run at the same time, and give
        // the same bits
        ++h->given_up;
        h->rest = h->pause = std::min(std::max(kFirstPause, 2 * h->pause), kLongestPause);
        turn.unlock();
    }
    DCO_HIP_CHECK(launch_densify_setup(h->b, h->solve_k, Ds, Dpre, Bdp, Mfuse, MI, h->W, h->H,
                                       p.lambda_d, p.lambda_s, p.lambda_s2, h->stream));
    for (int done = 0; done < p.max_iters; done += p.iters_per_launch) {
        DCO_HIP_CHECK(hipGraphLaunch(h->exec, h->stream));
        ++h->launches;
        DCO_HIP_CHECK(hipMemcpyAsync(h->flags_host, h->b.flags, 2 * sizeof(int),
                                     hipMemcpyDeviceToHost, h->stream));
        DCO_HIP_CHECK(hipStreamSynchronize(h->stream));
        if (h->flags_host[0]) break;
    }
    DCO_HIP_CHECK(launch_densify_out(h->b, h->solve_k, h->W, h->H, D, h->stream));
    return DCO_OK;
}

extern "C" dco_status dco_densify_stats(dco_densify* h, int* iters, double* rel_residual) {
    DCO_TRY(need(h, "handle"));
    DCO_HIP_CHECK(hipStreamSynchronize(h->stream));
    int f[2];
    DCO_HIP_CHECK(hipMemcpy(f, h->b.flags, sizeof(f), hipMemcpyDeviceToHost));
    if (iters) *iters = f[1];
    if (rel_residual && h->solve_k) {
        double res[2];
        DCO_HIP_CHECK(hipMemcpy(res, h->b.res, sizeof(res), hipMemcpyDeviceToHost));
        *rel_residual = res[1] > 0.0 ? std::sqrt(res[0] / res[1]) : 0.0;
    } else if (rel_residual) {
        // the newest r.r block sums: iteration k writes parity k & 1; setup parity 1
        const double* rr = f[1] > 0 ? h->b.rr[(f[1] - 1) & 1] : h->b.rr[1];
        std::vector<double> a((size_t)h->nblk), c((size_t)h->nblk);
        DCO_HIP_CHECK(hipMemcpy(a.data(), rr, a.size() * sizeof(double), hipMemcpyDeviceToHost));
        DCO_HIP_CHECK(
            hipMemcpy(c.data(), h->b.bb, c.size() * sizeof(double), hipMemcpyDeviceToHost));
        double sr = 0.0, sb = 0.0;
        for (size_t i = 0; i < a.size(); ++i) {
            sr += a[i];
            sb += c[i];
        }
        *rel_residual = sb > 0.0 ? std::sqrt(sr / sb) : 0.0;
    }
    return DCO_OK;
}

extern "C" dco_status dco_densify_launches(dco_densify* h, int* launches) {
    DCO_TRY(need(h, "handle"));
    DCO_TRY(need(launches, "launches"));
    *launches = h->launches;
    return DCO_OK;
}

extern "C" dco_status dco_densify_given_up(dco_densify* h, int* solves) {
    DCO_TRY(need(h, "handle"));
    DCO_TRY(need(solves, "solves"));
    *solves = h->given_up;
    return DCO_OK;
}
