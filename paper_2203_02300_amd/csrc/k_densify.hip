// k_densify.hip -- depth densification by quadratic optimisation (Sec. 6,
// Eq. 13-20), solved with Jacobi-preconditioned conjugate gradients.
//
// The normal equations of Eq. 20 at pixel p (q over the 4-neighbours):
//   (lambda_d w_sparse + lambda_s2 w_stable + sum_q c_pq) D(p) - sum_q c_pq D(q)
//     = lambda_d w_sparse D_sparse + lambda_s2 w_stable D_pre,
//   c_pq = 2 lambda_s w_pq  (the double sum of Eq. 20 visits each pair twice)
// with w_pq of Eq. 16-17.  The operator is a 5-point stencil with per-edge
// coefficients c_right (p, p + x) and c_down (p, p + y), 0 off the grid.
//
// Solver state is FP64 (x, r, p; z = r / diag is formed on the fly).  One
// iteration is two launches:
//   dir:    beta = rz_new / rz_old; p' = z + beta p; q = A p'; block sums of p'.q
//   update: alpha = rz_new / (p'.q); x += alpha p'; r -= alpha q; block sums
//           of r.z and r.r
// Every block forms alpha and beta itself from the previous launch's block
// sums, added in one fixed order, so every block gets the same bits and the
// whole solve is deterministic without grid-wide synchronisation.  When
// r.r <= tol^2 b.b the update launch sets a flag and every later launch
// returns at once (no pixel is touched).
//
// Grids of up to about a million pixels run the whole solve in one launch
// instead (k_dz_solve, below), and as launches on that kernel's tiles when its
// workgroups could not all run at once; the launches above serve larger grids.
#include <climits>
#include <type_traits>

#include "dco_internal.h"

namespace {

constexpr int kDzThreads = 256;
constexpr int kDzPix = 4;  // pixels per thread: a block covers 1024 consecutive pixels

constexpr int kDzWaves = kDzThreads / 64;

// Block sums of N values per thread, in one fixed order: an xor-butterfly
// across each wavefront (every lane ends with the same bits: each step adds
// the same two values in either order), then the wavefront totals in a fixed
// tree.  Every thread returns the N sums.  Two barriers whatever N is.
template <int N>
__device__ inline void block_sums(double (&v)[N], double* red /* N x kDzWaves */) {
#pragma unroll
    for (int j = 0; j < N; ++j)
        for (int o = 32; o > 0; o >>= 1) v[j] += __shfl_xor(v[j], o, 64);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) red[j * kDzWaves + w] = v[j];
    }
    __syncthreads();
    static_assert(kDzWaves == 4, "fixed tree of four wavefront totals");
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double* t = red + j * kDzWaves;
        v[j] = (t[0] + t[1]) + (t[2] + t[3]);
    }
    __syncthreads();  // red may be reused
}

// Sums of N arrays of n block partials, the same bits in every block: thread
// t adds entries t, t + 256, ... in turn, then block_sums.
template <int N>
__device__ inline void partial_sums(const double* const (&part)[N], int n, double (&out)[N],
                                    double* red) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double s = 0.0;
        for (int i = threadIdx.x; i < n; i += kDzThreads) s += part[j][i];
        out[j] = s;
    }
    block_sums<N>(out, red);
}

// The inputs of a solve, and the edge coefficients, diagonal and right-hand side of
// a pixel.  Eq. 16: w_pq = 0 when exactly one of p, q is on the depth contour, else
// max(1 - min(s_p, s_q), 0) with s = Mfuse MI.
struct DzIn {
    const float *Ds, *Dpre;
    const uint8_t* Bdp;
    const float *Mfuse, *MI;
    int W, H;
    double lam_d, lam_s, lam_s2;
};
struct DzPixel {
    double cr, cd, cl, cu, diag, b, id;  // id = 1 / diag (0 where diag is 0)
};
template <typename In>
__device__ inline DzPixel dz_pixel(const In& A, int x, int y) {
    const int W = A.W, i = y * W + x;
    const double s = (double)A.Mfuse[i] * (double)A.MI[i];
    const int b = A.Bdp[i] != 0;
    const auto w = [&](int j) {
        const int bj = A.Bdp[j] != 0;
        if (b + bj == 1) return 0.0;
        const double sj = (double)A.Mfuse[j] * (double)A.MI[j];
        return fmax(1.0 - fmin(s, sj), 0.0);
    };
    DzPixel c;
    c.cr = x + 1 < W ? 2.0 * A.lam_s * w(i + 1) : 0.0;
    c.cd = y + 1 < A.H ? 2.0 * A.lam_s * w(i + W) : 0.0;
    c.cl = x > 0 ? 2.0 * A.lam_s * w(i - 1) : 0.0;
    c.cu = y > 0 ? 2.0 * A.lam_s * w(i - W) : 0.0;
    const double ds = A.Ds[i], dp = A.Dpre ? (double)A.Dpre[i] : 0.0;
    const double wsp = ds > 0.0 ? 1.0 : 0.0, wst = dp > 0.0 ? 1.0 : 0.0;
    c.diag = A.lam_d * wsp + A.lam_s2 * wst + c.cr + c.cd + c.cl + c.cu;
    c.b = A.lam_d * wsp * ds + A.lam_s2 * wst * dp;
    c.id = c.diag > 0.0 ? 1.0 / c.diag : 0.0;
    return c;
}

// Where a solve keeps its state between launches.
struct DzMem {
    double *cr, *cd, *diag, *invdiag, *x, *r, *p0, *p1;
    double *rz, *rr, *bb, *rz_init;  // block sums
    int* flags;                      // [0] converged, [1] iterations done
    __device__ void put(int i, const DzPixel& c) const {
        cr[i] = c.cr;
        cd[i] = c.cd;
        diag[i] = c.diag;
        invdiag[i] = c.id;
        x[i] = 0.0;
        r[i] = c.b;
        p0[i] = 0.0;
        p1[i] = 0.0;
    }
    __device__ void put_sums(int k, double rz_k, double rr_k) const {
        rz[k] = rz_k;
        rr[k] = rr_k;
        bb[k] = rr_k;
        rz_init[k] = 1.0;  // any nonzero "old" r.z: p starts at 0
    }
};

// The initial state x = 0, r = b, p = 0, block sums of r.z, r.r and b.b.
__global__ __launch_bounds__(kDzThreads) void k_dz_setup(DzIn A, DzMem m) {
    __shared__ double red[2 * kDzWaves];
    const int P = A.W * A.H;
    double rz = 0.0, rr = 0.0;
    for (int k = 0; k < kDzPix; ++k) {
        const int i = (blockIdx.x * kDzPix + k) * kDzThreads + threadIdx.x;
        if (i >= P) break;
        const int y = i / A.W;
        const DzPixel c = dz_pixel(A, i - y * A.W, y);
        m.put(i, c);
        rz += c.b * c.b * c.id;
        rr += c.b * c.b;
    }
    double sums[2] = {rz, rr};
    block_sums<2>(sums, red);
    if (threadIdx.x == 0) m.put_sums(blockIdx.x, sums[0], sums[1]);
    if (blockIdx.x == 0 && threadIdx.x < 2) m.flags[threadIdx.x] = 0;
}

struct DzState {
    const double* cr;
    const double* cd;
    const double* diag;
    const double* invdiag;
    double* x;
    double* r;
    double* q;
    const double* bb_part;
    int* flags;  // [0] converged, [1] iterations done
    int W, H, nblk;
    double tol2;
};

// The convergence flag as one value for the whole block.
__device__ inline bool solve_done(const int* flags) {
    __shared__ int done;
    if (threadIdx.x == 0) done = *(const volatile int*)&flags[0];
    __syncthreads();
    return done != 0;
}

// p_out = r / diag + beta p_in (4-neighbours recomputed from r and p_in);
// q = A p_out; block sums of p_out . q.
__global__ __launch_bounds__(kDzThreads) void k_dz_dir(DzState s, const double* __restrict__ rz_new,
                                                       const double* __restrict__ rz_old,
                                                       const double* __restrict__ p_in,
                                                       double* __restrict__ p_out,
                                                       double* __restrict__ pq_part) {
    __shared__ double red[2 * kDzWaves];
    if (solve_done(s.flags)) return;
    const double* const parts[2] = {rz_new, rz_old};
    double rz[2];
    partial_sums<2>(parts, s.nblk, rz, red);
    const double beta = rz[0] / rz[1];
    const int W = s.W, P = W * s.H;
    double pq = 0.0;
    for (int k = 0; k < kDzPix; ++k) {
        const int i = (blockIdx.x * kDzPix + k) * kDzThreads + threadIdx.x;
        if (i >= P) break;
        const int y = i / W, xx = i - y * W;
        auto pn = [&](int j) { return s.r[j] * s.invdiag[j] + beta * p_in[j]; };
        const double pc = pn(i);
        double off = 0.0;  // sum over the 4-neighbours of c_pq p(q), in a fixed order
        if (xx + 1 < W) off += s.cr[i] * pn(i + 1);
        if (xx > 0) off += s.cr[i - 1] * pn(i - 1);
        if (y + 1 < s.H) off += s.cd[i] * pn(i + W);
        if (y > 0) off += s.cd[i - W] * pn(i - W);
        const double qi = s.diag[i] * pc - off;
        p_out[i] = pc;
        s.q[i] = qi;
        pq += pc * qi;
    }
    double sum[1] = {pq};
    block_sums<1>(sum, red);
    if (threadIdx.x == 0) pq_part[blockIdx.x] = sum[0];
}

// alpha = rz / pq; x += alpha p; r -= alpha q; block sums of r.z and r.r of
// the new residual.  Convergence (r.r <= tol^2 b.b, from the previous
// update's sums) stops the solve before any pixel changes.
__global__ __launch_bounds__(kDzThreads) void k_dz_update(DzState s,
                                                          const double* __restrict__ rz_in,
                                                          const double* __restrict__ rr_in,
                                                          const double* __restrict__ pq_part,
                                                          const double* __restrict__ p,
                                                          double* __restrict__ rz_out,
                                                          double* __restrict__ rr_out) {
    __shared__ double red[4 * kDzWaves];
    if (solve_done(s.flags)) return;
    const double* const parts[4] = {rr_in, s.bb_part, pq_part, rz_in};
    double sums[4];
    partial_sums<4>(parts, s.nblk, sums, red);
    const double rr = sums[0], bb = sums[1], pq = sums[2];
    if (rr <= s.tol2 * bb) {  // converged before this step: the same decision in every block
        if (blockIdx.x == 0 && threadIdx.x == 0) s.flags[0] = 1;
        return;
    }
    const double alpha = pq > 0.0 ? sums[3] / pq : 0.0;
    const int P = s.W * s.H;
    double rz = 0.0, rrn = 0.0;
    for (int k = 0; k < kDzPix; ++k) {
        const int i = (blockIdx.x * kDzPix + k) * kDzThreads + threadIdx.x;
        if (i >= P) break;
        s.x[i] += alpha * p[i];
        const double ri = s.r[i] - alpha * s.q[i];
        s.r[i] = ri;
        rz += ri * ri * s.invdiag[i];
        rrn += ri * ri;
    }
    double out[2] = {rz, rrn};
    block_sums<2>(out, red);
    if (threadIdx.x == 0) {
        rz_out[blockIdx.x] = out[0];
        rr_out[blockIdx.x] = out[1];
        if (blockIdx.x == 0) s.flags[1] += 1;
    }
}

__global__ __launch_bounds__(kDzThreads) void k_dz_out(const double* __restrict__ x, int P,
                                                       float* __restrict__ D) {
    const int i = blockIdx.x * kDzThreads + threadIdx.x;
    if (i < P) D[i] = (float)x[i];
}

// ---------------------------------------------------------------------------
// The whole solve in one launch
// ---------------------------------------------------------------------------
//
// One workgroup of 1024 threads per tile of 32 x 32 K pixels, at most one per
// CU, so that all of them run at once.  A pixel's state (x, r, p, its
// coefficients) stays in its thread's registers for the whole solve and p
// passes to the neighbours through an LDS tile; the arithmetic per pixel is
// that of the launches above.  Per iteration the workgroups exchange two
// things through memory, and wait for nothing else:
//   after the update: the partial sums of r.z and r.r, and z along the tile's
//       edges, from which the neighbours keep p on their halo themselves;
//   after q = A p: the partial sum of p.q.
// A double travels as two 64-bit words that each carry 32 of its bits and the
// iteration's number, written and read as single (relaxed, device-scope)
// atomics: a reader takes a word as soon as it bears the number it waits for,
// so no fence, counter or barrier is needed.  Words of one iteration are
// written over in the next: a workgroup writes its sums of p.q for iteration
// k + 1 only after it has read everybody's update of iteration k, which
// everybody writes after reading the sums of p.q of iteration k, and so on in
// turn.  Every workgroup adds all partial sums itself in the same order, so
// all hold the same alpha and beta bits.
//
// A wait ends after `ticks` (20 ms) without the awaited word (workgroups that do
// not run: another process holds the CUs): the workgroup raises an abort flag
// that every wait looks at, all leave, and the host repeats the solve as a
// sequence of launches on the same tiles (k_dz_tile_*), which form every value and
// every sum as this kernel does: the same bits either way.
//
// What bounds it: the two exchanges of an iteration (a store to memory and
// loads from it across the XCDs, 1.3 us each, more with the tiles polled) and
// the sums within a workgroup.  640 x 360: 0.42 ms (62 iterations) where the
// launches above took 1.42; 1280 x 720: 0.77 ms (67) instead of 2.88.

constexpr int kSolveThreads = 1024, kSolveWaves = kSolveThreads / 64;
constexpr int kTileW = 32, kTileRows = 32;           // a tile is 32 x 32 K pixels
constexpr int kLineWords = 32;                       // a tile's sums, 256 bytes apart: every
                                                     // workgroup polls them

struct SolveArgs {
    const float *Ds, *Dpre;
    const uint8_t* Bdp;
    const float *Mfuse, *MI;
    float* D;
    int W, H, tx, ntiles, limit;  // tiles per row, tiles, iterations at most
    double lam_d, lam_s, lam_s2, tol2;
    uint64_t ticks;  // longest wait, in ticks of the 100 MHz clock
    uint64_t* pq;    // ntiles lines: p.q (two words)
    uint64_t* rzr;   // ntiles lines: r.z, r.r (two words each)
    uint64_t* edge;  // ntiles x (64 + 64 K) x 2 words: top, bottom, left, right
    int* flags;      // [0] converged, [1] iterations done, [2] abort
    double* res;     // [0] r.r, [1] b.b
};

__device__ inline void put_word(uint64_t* p, uint32_t v, uint32_t epoch) {
    __hip_atomic_store(p, (uint64_t)epoch << 32 | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void put_double(uint64_t* p, double v, uint32_t epoch) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    put_word(p, (uint32_t)b, epoch);
    put_word(p + 1, (uint32_t)(b >> 32), epoch);
}

// The N doubles at p once all their words bear the epoch; false if the wait
// was given up (the abort flag is then set).
template <int N>
__device__ inline bool get_doubles(const uint64_t* p, uint32_t epoch, uint64_t ticks,
                                   int* abort_flag, double (&v)[N]) {
    uint64_t w[2 * N];
    uint64_t t0 = 0;
    for (uint32_t n = 0;; ++n) {
        bool all = true;
#pragma unroll
        for (int k = 0; k < 2 * N; ++k)
            w[k] = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int k = 0; k < 2 * N; ++k) all = all && (uint32_t)(w[k] >> 32) == epoch;
        if (all) break;
        if ((n & 63) == 63 || !ticks) {  // now and then: is it time to give up, has somebody?
            const uint64_t t = __builtin_amdgcn_s_memrealtime();
            if (!t0) t0 = t;
            const bool late = t - t0 >= ticks;
            if (late) __hip_atomic_store(abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (late ||
                __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                return false;
        }
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
        v[k] = __builtin_bit_cast(double, (uint64_t)(uint32_t)w[2 * k] | w[2 * k + 1] << 32);
    return true;
}

// Sum of a double over the wavefront's lanes 16 r .. 16 r + 15 in lane 15 of
// each such row (kAll: over the whole wavefront, in lane 63), in a fixed
// order: DPP row shifts 1, 2, 4, 8, then the row broadcasts 15 and 31.  Lanes
// without a source add nothing.
template <unsigned Ctrl, unsigned RowMask>
__device__ inline double dpp_f64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, Ctrl, RowMask,
                                                              0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), Ctrl,
                                                              RowMask, 0xf, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <bool kAll>
__device__ inline double lane_sum(double v) {
    v += dpp_f64<0x111, 0xf>(v);
    v += dpp_f64<0x112, 0xf>(v);
    v += dpp_f64<0x114, 0xf>(v);
    v += dpp_f64<0x118, 0xf>(v);
    if constexpr (kAll) {
        v += dpp_f64<0x142, 0xa>(v);
        v += dpp_f64<0x143, 0xc>(v);
    }
    return v;
}

// The sum of N values per thread of a tile's workgroup, in a fixed order: across each
// wavefront, then over the wavefronts' totals.  put(j, total) in one thread.
template <int N, typename Put>
__device__ inline void tile_sums(double (&v)[N], double (*red)[kSolveWaves], Put put) {
    const int t = threadIdx.x;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        v[j] = lane_sum<true>(v[j]);
        if ((t & 63) == 63) red[j][t >> 6] = v[j];
    }
    __syncthreads();
    static_assert(kSolveWaves == 16, "one wavefront total per lane of a DPP row");
    if (t < kSolveWaves) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const double u = lane_sum<false>(red[j][t]);
            if (t == kSolveWaves - 1) put(j, u);
        }
    }
}

// The sum over the tiles, in a fixed order, of what threads 0 .. 255 hold of tiles t,
// t + 256, ...; in every thread.
template <int N>
__device__ inline void over_tiles(double (&v)[N], double (*all)[4]) {
    const int t = threadIdx.x;
    if (t < 256) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            v[j] = lane_sum<true>(v[j]);
            if ((t & 63) == 63) all[j][t >> 6] = v[j];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = (all[j][0] + all[j][1]) + (all[j][2] + all[j][3]);
}

// Clears what k_dz_solve waits on (words of an earlier solve bear the same
// iteration numbers) and the flags.
__global__ __launch_bounds__(256) void k_dz_clear(uint64_t* __restrict__ words, size_t n,
                                                  int* __restrict__ flags) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) words[i] = 0;
    if (i < 3) flags[i] = 0;
}

template <int K>
__global__ __launch_bounds__(kSolveThreads) void k_dz_solve(SolveArgs A) {
    constexpr int TH = kTileRows * K, E = 2 * kTileW + 2 * TH;
    __shared__ double P[TH + 2][kTileW + 2];
    __shared__ double red[2][kSolveWaves];  // wavefront sums of this tile
    __shared__ double all[2][4];            // wavefront sums over the tiles
    __shared__ int gave_up;
    const int t = threadIdx.x, lx = t & 31, ly = t >> 5;
    const int tile = blockIdx.x, ty0 = tile / A.tx, tx0 = tile - ty0 * A.tx;
    const int x0 = tx0 * kTileW, y0 = ty0 * TH, W = A.W, H = A.H;
    if (t == 0) gave_up = 0;

    // own pixels: rows ly + 32 k of the tile; outside the image all is zero
    double x[K], r[K], p[K], id[K], dg[K], cr[K], cd[K], cl[K], cu[K];
    double rz = 0.0, rr = 0.0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int xx = x0 + lx, y = y0 + ly + kTileRows * k;
        x[k] = r[k] = p[k] = id[k] = dg[k] = cr[k] = cd[k] = cl[k] = cu[k] = 0.0;
        if (xx >= W || y >= H) continue;
        const DzPixel c = dz_pixel(A, xx, y);
        cr[k] = c.cr;
        cd[k] = c.cd;
        cl[k] = c.cl;
        cu[k] = c.cu;
        dg[k] = c.diag;
        r[k] = c.b;
        id[k] = c.id;
        rz += r[k] * r[k] * id[k];
        rr += r[k] * r[k];
    }
    // halo cell of threads 256 .. 256 + E - 1: whose edge entry it is and
    // where its p goes (corners are never read)
    uint64_t* const my_edge = A.edge + (size_t)tile * E * 2;
    const int e = t - 256;
    const uint64_t* src = nullptr;
    double* dst = nullptr;
    if (e >= 0 && e < E) {
        int nb = -1, idx = 0;  // neighbour tile, its edge entry
        if (e < kTileW) {  // row above: the upper tile's bottom row
            nb = ty0 > 0 ? tile - A.tx : -1;
            idx = kTileW + e;
            dst = &P[0][e + 1];
        } else if (e < 2 * kTileW) {  // row below: the lower tile's top row
            nb = y0 + TH < H ? tile + A.tx : -1;
            idx = e - kTileW;
            dst = &P[TH + 1][e - kTileW + 1];
        } else if (e < 2 * kTileW + TH) {  // column left: the left tile's right column
            nb = tx0 > 0 ? tile - 1 : -1;
            idx = e + TH;
            dst = &P[e - 2 * kTileW + 1][0];
        } else {  // column right: the right tile's left column
            nb = tx0 + 1 < A.tx ? tile + 1 : -1;
            idx = e - TH;
            dst = &P[e - 2 * kTileW - TH + 1][kTileW + 1];
        }
        if (nb >= 0) src = A.edge + ((size_t)nb * E + idx) * 2;
        *dst = 0.0;
    }
    double ph = 0.0;

    // Block sum of N values per thread in a fixed order, then published by one
    // thread as this tile's words at `at`.
    const auto publish = [&](auto& v, uint64_t* at, uint32_t epoch) {
        tile_sums(v, red, [&](int j, double u) { put_double(at + 2 * j, u, epoch); });
    };
    // All tiles' sums (N doubles of every tile), added in a
    // fixed order, in every thread's v; with halo, also z of the thread's halo
    // cell.  False, in the whole workgroup, when a wait was given up.
    const auto collect = [&](auto& v, const uint64_t* words, uint32_t epoch, bool halo,
                             double& zh) {
        constexpr int N = sizeof(v) / sizeof(double);
        bool ok = true;
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = 0.0;
        for (int i = t; i < A.ntiles && t < 256; i += 256) {
            double u[N];
            ok = ok && get_doubles<N>(words + (size_t)i * kLineWords, epoch, A.ticks, A.flags + 2,
                                       u);
            if (!ok) break;
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] += u[j];
        }
        if (halo && src) {
            double u[1];
            ok = get_doubles<1>(src, epoch, A.ticks, A.flags + 2, u);
            zh = u[0];
        }
        if (!ok) gave_up = 1;
        // over_tiles, written out: with a call here the wait above compiles to 28
        // instructions more
        if (t < 256) {
#pragma unroll
            for (int j = 0; j < N; ++j) {
                v[j] = lane_sum<true>(v[j]);
                if ((t & 63) == 63) all[j][t >> 6] = v[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = (all[j][0] + all[j][1]) + (all[j][2] + all[j][3]);
        const bool stop = gave_up != 0;
        __syncthreads();  // all[] may be reused
        return !stop;
    };
    const auto publish_update = [&](uint32_t epoch) {
        // z along the edges, then the sums
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int row = ly + kTileRows * k;
            const double z = r[k] * id[k];
            if (row == 0) put_double(my_edge + 2 * lx, z, epoch);
            if (row == TH - 1) put_double(my_edge + 2 * (kTileW + lx), z, epoch);
            if (lx == 0) put_double(my_edge + 2 * (2 * kTileW + row), z, epoch);
            if (lx == kTileW - 1) put_double(my_edge + 2 * (2 * kTileW + TH + row), z, epoch);
        }
        double v[2] = {rz, rr};
        publish(v, A.rzr + (size_t)tile * kLineWords, epoch);
    };

    uint32_t epoch = 1;
    publish_update(epoch);
    double bb = 0.0, rz_old = 1.0, rr_all = 0.0;
    int it = 0, converged = 0;
    bool ok = true;
    for (;; ++it) {
        double s2[2], zh = 0.0;
        ok = collect(s2, A.rzr, epoch, true, zh);
        if (!ok) break;
        const double rz_all = s2[0];
        rr_all = s2[1];
        if (it == 0) bb = rr_all;
        if (rr_all <= A.tol2 * bb) {  // the same decision in every workgroup
            converged = 1;
            break;
        }
        if (it >= A.limit) break;
        const double beta = it ? rz_all / rz_old : 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            p[k] = r[k] * id[k] + beta * p[k];
            P[ly + kTileRows * k + 1][lx + 1] = p[k];
        }
        if (src) {
            ph = zh + beta * ph;
            *dst = ph;
        }
        __syncthreads();
        double q[K], pq = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int py = ly + kTileRows * k + 1, px = lx + 1;
            double off = 0.0;  // right, left, below, above, as in k_dz_dir
            off += cr[k] * P[py][px + 1];
            off += cl[k] * P[py][px - 1];
            off += cd[k] * P[py + 1][px];
            off += cu[k] * P[py - 1][px];
            q[k] = dg[k] * p[k] - off;
            pq += p[k] * q[k];
        }
        double s1[1] = {pq};
        publish(s1, A.pq + (size_t)tile * kLineWords, epoch);
        ok = collect(s1, A.pq, epoch, false, zh);
        if (!ok) break;
        const double alpha = s1[0] > 0.0 ? rz_all / s1[0] : 0.0;
        rz = rr = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[k] += alpha * p[k];
            r[k] = r[k] - alpha * q[k];
            rz += r[k] * r[k] * id[k];
            rr += r[k] * r[k];
        }
        rz_old = rz_all;
        publish_update(++epoch);
    }
    if (!ok) return;  // uniform
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int xx = x0 + lx, y = y0 + ly + kTileRows * k;
        if (xx < W && y < H) A.D[(size_t)y * W + xx] = (float)x[k];
    }
    if (tile == 0 && t == 0) {
        A.flags[0] = converged;
        A.flags[1] = it;
        A.res[0] = rr_all;
        A.res[1] = bb;
    }
}

// The same solve as a sequence of launches, a tile per workgroup as above: the state
// between them in memory, a tile's sums in plain arrays.  dir and update are one
// iteration; out makes D and the residual.
struct DzTiles {
    DzMem m;
    double *q, *pq;
    int W, H, tx, ntiles;
    double tol2;
};

// body(i, x, y) for the thread's own pixels inside the image
template <int K, typename Body>
__device__ inline void tile_pixels(int W, int H, int tx, Body body) {
    const int t = threadIdx.x, ty0 = blockIdx.x / tx, tx0 = blockIdx.x - ty0 * tx;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int x = tx0 * kTileW + (t & 31), y = (ty0 * K + k) * kTileRows + (t >> 5);
        if (x < W && y < H) body(y * W + x, x, y);
    }
}

// The sums over all tiles of N arrays of tile sums, in every thread.
template <int N>
__device__ inline void tiles_total(const double* const (&part)[N], int ntiles, double (&v)[N],
                                   double (*all)[4]) {
    const int t = threadIdx.x;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        v[j] = 0.0;
        for (int i = t; i < ntiles && t < 256; i += 256) v[j] += part[j][i];
    }
    over_tiles(v, all);
    __syncthreads();  // all[] may be reused
}

template <int K>
__global__ __launch_bounds__(kSolveThreads) void k_dz_tile_setup(DzIn A, DzTiles s) {
    __shared__ double red[2][kSolveWaves];
    double v[2] = {0.0, 0.0};
    tile_pixels<K>(A.W, A.H, s.tx, [&](int i, int x, int y) {
        const DzPixel c = dz_pixel(A, x, y);
        s.m.put(i, c);
        v[0] += c.b * c.b * c.id;
        v[1] += c.b * c.b;
    });
    double rz = 0.0;
    tile_sums(v, red, [&](int j, double u) {
        if (j == 0)
            rz = u;
        else
            s.m.put_sums(blockIdx.x, rz, u);
    });
    if (blockIdx.x == 0 && threadIdx.x < 2) s.m.flags[threadIdx.x] = 0;
}

template <int K>
__global__ __launch_bounds__(kSolveThreads) void k_dz_tile_dir(DzTiles s, const double* rz_new,
                                                               const double* rz_old,
                                                               const double* p_in, double* p_out) {
    __shared__ double red[1][kSolveWaves];
    __shared__ double all[2][4];
    if (solve_done(s.m.flags)) return;
    const double* const parts[2] = {rz_new, rz_old};
    double rz[2], v[1] = {0.0};
    tiles_total(parts, s.ntiles, rz, all);
    const double beta = rz[0] / rz[1];
    const DzMem& m = s.m;
    const int W = s.W;
    tile_pixels<K>(W, s.H, s.tx, [&](int i, int x, int y) {
        const auto pn = [&](int j) { return m.r[j] * m.invdiag[j] + beta * p_in[j]; };
        const double pc = pn(i);
        double off = 0.0;
        if (x + 1 < W) off += m.cr[i] * pn(i + 1);
        if (x > 0) off += m.cr[i - 1] * pn(i - 1);
        if (y + 1 < s.H) off += m.cd[i] * pn(i + W);
        if (y > 0) off += m.cd[i - W] * pn(i - W);
        const double qi = m.diag[i] * pc - off;
        p_out[i] = pc;
        s.q[i] = qi;
        v[0] += pc * qi;
    });
    tile_sums(v, red, [&](int, double u) { s.pq[blockIdx.x] = u; });
}

template <int K>
__global__ __launch_bounds__(kSolveThreads) void k_dz_tile_update(DzTiles s, const double* rz_in,
                                                                  const double* rr_in,
                                                                  const double* p, double* rz_out,
                                                                  double* rr_out) {
    __shared__ double red[2][kSolveWaves];
    __shared__ double all[4][4];
    if (solve_done(s.m.flags)) return;
    const double* const parts[4] = {rr_in, s.m.bb, s.pq, rz_in};
    double sums[4], v[2] = {0.0, 0.0};
    tiles_total(parts, s.ntiles, sums, all);
    if (sums[0] <= s.tol2 * sums[1]) {
        if (blockIdx.x == 0 && threadIdx.x == 0) s.m.flags[0] = 1;
        return;
    }
    const double alpha = sums[2] > 0.0 ? sums[3] / sums[2] : 0.0;
    const DzMem& m = s.m;
    tile_pixels<K>(s.W, s.H, s.tx, [&](int i, int, int) {
        m.x[i] += alpha * p[i];
        const double ri = m.r[i] - alpha * s.q[i];
        m.r[i] = ri;
        v[0] += ri * ri * m.invdiag[i];
        v[1] += ri * ri;
    });
    tile_sums(v, red, [&](int j, double u) { (j ? rr_out : rz_out)[blockIdx.x] = u; });
    if (blockIdx.x == 0 && threadIdx.x == 0) m.flags[1] += 1;
}

template <int K>
__global__ __launch_bounds__(kSolveThreads) void k_dz_tile_out(DzTiles s, const double* rr_even,
                                                               const double* rr_odd, float* D,
                                                               double* res) {
    __shared__ double all[2][4];
    tile_pixels<K>(s.W, s.H, s.tx, [&](int i, int, int) { D[i] = (float)s.m.x[i]; });
    if (blockIdx.x != 0) return;
    const int it = s.m.flags[1];  // iteration k writes parity k & 1; setup parity 1
    const double* const parts[2] = {it > 0 && ((it - 1) & 1) == 0 ? rr_even : rr_odd, s.m.bb};
    double v[2];
    tiles_total(parts, s.ntiles, v, all);
    if (threadIdx.x < 2) res[threadIdx.x] = v[threadIdx.x];
}

}  // namespace

int densify_blocks(int W, int H) {
    return (W * H + kDzThreads * kDzPix - 1) / (kDzThreads * kDzPix);
}

static int solve_tiles(int W, int H, int k) {
    const long long n = (long long)((W + kTileW - 1) / kTileW) *
                        ((H + kTileRows * k - 1) / (kTileRows * k));
    return n < INT_MAX ? (int)n : INT_MAX;
}

// Pixels per thread of the one-launch solve on a device with `cus` CUs, or 0
// when the grid does not fit: its tiles must all run at once, one per CU.
// An iteration takes about 3.3 us, 0.55 us per pixel of a thread and 23.5 ns
// per tile that every workgroup polls (measured per iteration: 240 tiles of
// one pixel 9.7 us, 120 of two 6.9, 80 of three 6.3, 60 of four 6.6 at
// 640 x 360; 35 of one 4.5, 21 of two 4.8, 14 of three 5.3 at 200 x 150), so
// the k with the least 23 k + tiles is taken.
int densify_solve_k(int W, int H, int cus) {
    int best = 0;
    for (int k = 1; k <= kDensifyMaxK; ++k)
        if (solve_tiles(W, H, k) <= cus &&
            (!best || 23 * k + solve_tiles(W, H, k) < 23 * best + solve_tiles(W, H, best)))
            best = k;
    return best;
}

size_t densify_solve_words(int W, int H, int k) {
    const size_t tiles = solve_tiles(W, H, k);
    return tiles * (2 * kLineWords + 2 * (size_t)(2 * kTileW + 2 * kTileRows * k));
}

// go(K) with the pixels per thread as a constant
template <typename Go>
static void with_tile_k(int k, Go go) {
    switch (k) {
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        default: go(std::integral_constant<int, 4>{}); break;
    }
}

static DzMem dz_mem(const DensifyBufs& b) {
    return DzMem{b.cr, b.cd,    b.diag,  b.invdiag, b.x,     b.r,    b.p[0],
                 b.p[1], b.rz[1], b.rr[1], b.bb,      b.rz[0], b.flags};
}

static DzTiles dz_tiles(const DensifyBufs& b, int k, int W, int H, double tol) {
    return DzTiles{dz_mem(b), b.q, b.pq, W, H, (W + kTileW - 1) / kTileW, solve_tiles(W, H, k),
                   tol * tol};
}

size_t densify_parts(int W, int H, int k) {
    return k ? solve_tiles(W, H, k) : densify_blocks(W, H);
}

hipError_t launch_densify_setup(const DensifyBufs& b, int k, const float* Ds, const float* Dpre,
                                const uint8_t* Bdp, const float* Mfuse, const float* MI, int W,
                                int H, double lam_d, double lam_s, double lam_s2, hipStream_t st) {
    const DzIn in{Ds, Dpre, Bdp, Mfuse, MI, W, H, lam_d, lam_s, lam_s2};
    if (k) {
        const DzTiles s = dz_tiles(b, k, W, H, 0.0);
        with_tile_k(k, [&](auto K) {
            hipLaunchKernelGGL(k_dz_tile_setup<decltype(K)::value>, dim3(s.ntiles),
                               dim3(kSolveThreads), 0, st, in, s);
        });
    } else {
        hipLaunchKernelGGL(k_dz_setup, dim3(densify_blocks(W, H)), dim3(kDzThreads), 0, st, in,
                           dz_mem(b));
    }
    return hipGetLastError();
}

// Iterations [0, n) of one launch sequence; n even, so parities repeat.
hipError_t launch_densify_iters(const DensifyBufs& b, int k, int W, int H, double tol, int n,
                                hipStream_t st) {
    const int nb = densify_blocks(W, H);
    DzState s{b.cr, b.cd, b.diag, b.invdiag, b.x, b.r, b.q, b.bb, b.flags, W, H, nb, tol * tol};
    const DzTiles t = k ? dz_tiles(b, k, W, H, tol) : DzTiles{};
    for (int it = 0; it < n; ++it) {
        const int a = it & 1;  // rz[1 - a] is the newest r.z, rz[a] the one before
        if (k) {
            with_tile_k(k, [&](auto K) {
                hipLaunchKernelGGL(k_dz_tile_dir<decltype(K)::value>, dim3(t.ntiles),
                                   dim3(kSolveThreads), 0, st, t, b.rz[1 - a], b.rz[a], b.p[a],
                                   b.p[1 - a]);
                hipLaunchKernelGGL(k_dz_tile_update<decltype(K)::value>, dim3(t.ntiles),
                                   dim3(kSolveThreads), 0, st, t, b.rz[1 - a], b.rr[1 - a],
                                   b.p[1 - a], b.rz[a], b.rr[a]);
            });
            continue;
        }
        hipLaunchKernelGGL(k_dz_dir, dim3(nb), dim3(kDzThreads), 0, st, s, b.rz[1 - a], b.rz[a],
                           b.p[a], b.p[1 - a], b.pq);
        hipLaunchKernelGGL(k_dz_update, dim3(nb), dim3(kDzThreads), 0, st, s, b.rz[1 - a],
                           b.rr[1 - a], b.pq, b.p[1 - a], b.rz[a], b.rr[a]);
    }
    return hipGetLastError();
}

hipError_t launch_densify_out(const DensifyBufs& b, int k, int W, int H, float* D,
                              hipStream_t st) {
    const int P = W * H;
    if (k) {
        const DzTiles t = dz_tiles(b, k, W, H, 0.0);
        with_tile_k(k, [&](auto K) {
            hipLaunchKernelGGL(k_dz_tile_out<decltype(K)::value>, dim3(t.ntiles),
                               dim3(kSolveThreads), 0, st, t, b.rr[0], b.rr[1], D, b.res);
        });
    } else {
        hipLaunchKernelGGL(k_dz_out, dim3((P + kDzThreads - 1) / kDzThreads), dim3(kDzThreads), 0,
                           st, b.x, P, D);
    }
    return hipGetLastError();
}

hipError_t launch_densify_solve(const DensifyBufs& b, int k, const float* Ds, const float* Dpre,
                                const uint8_t* Bdp, const float* Mfuse, const float* MI, int W,
                                int H, double lam_d, double lam_s, double lam_s2, double tol,
                                int limit, uint64_t ticks, float* D, hipStream_t st) {
    const int tx = (W + kTileW - 1) / kTileW, tiles = solve_tiles(W, H, k);
    SolveArgs A{Ds, Dpre, Bdp, Mfuse, MI, D, W, H, tx, tiles, limit, lam_d, lam_s, lam_s2,
                tol * tol, ticks, b.words, b.words + (size_t)tiles * kLineWords,
                b.words + 2 * (size_t)tiles * kLineWords, b.flags, b.res};
    const size_t n = densify_solve_words(W, H, k);
    hipLaunchKernelGGL(k_dz_clear, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, b.words, n,
                       b.flags);
    with_tile_k(k, [&](auto K) {
        hipLaunchKernelGGL(k_dz_solve<decltype(K)::value>, dim3(tiles), dim3(kSolveThreads), 0, st,
                           A);
    });
    return hipGetLastError();
}
