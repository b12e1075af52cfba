// k_wta.hip -- winner-take-all over the aggregated volumes (Eq. 3) with
// parabola sub-pixel refinement, and the left-right consistency check, in one
// launch (two where rows suit workgroups badly).  On volumes in the paired layout (dco::paired_at)
// only the even slices are read; for the sub-pixel step the winner's pair partner
// is gathered and, when it is not the adjacent pair's minimum kept from the scan,
// its other neighbour.  A thread takes four consecutive pixels with 16-byte loads and
// walks d = 0 .. D-1; loads of one slice are coalesced across the row, so each
// volume is read exactly once.  The stage bodies live in dco_device.h.
#include <algorithm>

#include "dco_device.h"

namespace {

constexpr int kWtaThreads = 1024;          // most threads of a row
constexpr int kRowCols = 2 * kWtaThreads;  // longest row that k_wta_row takes

// One workgroup per image row: its second half takes the right view's quads of
// four pixels, the first half the left view's; the right disparities go to LDS
// for the left-right check, which the left view's threads make on their own
// quads: a row has no more of them than half a workgroup has threads (kRowCols).
// The last quad of a row is moved back to end with it (rows of less than four
// pixels: kNarrow), so quads may start at any pixel.
//
// Bound by the volumes' bytes at large frames (1280 x 720, D = 128: 472 MB read
// in 0.09 ms) and by the latency of about D / 42 batches of loads at small ones.
// As a launch per step, with quads only where W H was a multiple of four (else
// one pixel and one load in flight per thread): frames of 437 x 93, D = 40 took
// 61.4 us, now 57.0; 64 x 48, D = 16 43.2, now 40.0; 640 x 480, D = 64 168.8,
// now 167.2; 1280 x 720 the same.  Workgroups of at most 128, 256, 512 and 640
// threads: 437 x 93 63.0, 57.0, 57.0, 57.2; staged 640 x 480 256, 254, 239, 239
// (243 before).  Rows of more than 1024 columns want more than 512: with them a
// row's last quads went in a second turn, staged 1280 x 720, D = 128 192 us
// instead of 153 with up to 1024 threads (157 as two launches), the one-call
// launch 87.2 instead of 85.0.
template <bool kPaired, bool kNarrow>
__global__ __launch_bounds__(kWtaThreads) void k_wta_row(
    const float* __restrict__ aggL, const float* __restrict__ aggR, int pitch, int P, int W, int D,
    int subpixel, int maxdiff, int16_t* __restrict__ dL, int16_t* __restrict__ dR,
    float* __restrict__ disp, uint8_t* __restrict__ valid, HalfOut half) {
    extern __shared__ int16_t right[];  // W entries
    const int t = threadIdx.x, nt = blockDim.x / 2, nq = (W + 3) / 4;
    const int row = blockIdx.x * W, vrow = blockIdx.x * pitch;  // P: a plane of the volumes
    const auto start = [&](int q) { return kNarrow ? 0 : min(4 * q, W - 4); };
    const auto left = [&](int q) {
        return dco::wta_any<kPaired, true, kNarrow>(aggL, P, D, vrow + start(q), W, subpixel);
    };
    const auto check = [&](int q, const dco::WtaQuad& l) {
        const int x = start(q), i = row + x;
        float dv[4];
        uint8_t ok[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int xr = x + k - l.bd[k];
            const bool in = xr >= 0 && xr < W && abs(l.bd[k] - (int)right[xr]) <= maxdiff;
            ok[k] = in ? 1 : 0;
            dv[k] = in ? (float)l.bd[k] + l.del[k] : 0.0f;
            if (half.on) dv[k] *= 2.0f;
        }
        if (half.depth) {
            float z[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) z[k] = dv[k] > 0.0f ? half.fB / dv[k] : 0.0f;
            dco::wta_store<kNarrow, dco::f32x4u>(half.depth + i, z[0], z[1], z[2], z[3], W);
        }
        dco::put_bd<kNarrow>(dL + i, l, W);
        dco::wta_store<kNarrow, dco::f32x4u>(disp + i, dv[0], dv[1], dv[2], dv[3], W);
        dco::wta_store<kNarrow, dco::u8x4u>(valid + i, ok[0], ok[1], ok[2], ok[3], W);
    };
    dco::WtaQuad l{};
    if (t >= nt) {
        if (t - nt < nq) {
            const int x = start(t - nt);
            const dco::WtaQuad r =
                dco::wta_any<kPaired, false, kNarrow>(aggR, P, D, vrow + x, W, subpixel);
            dco::put_bd<kNarrow>(right + x, r, W);
            dco::put_bd<kNarrow>(dR + row + x, r, W);
        }
    } else if (t < nq) {
        l = left(t);
    }
    __syncthreads();
    if (t < nt && t < nq) check(t, l);
}

// Rows that suit workgroups badly (by_quads): WTA as a launch of a quad per thread,
// whatever row it is in, the left view (blockIdx.y = 0) with disp = its disparity
// before the check, and the check as a launch after it, which costs 2 to 5 us.
template <bool kPaired>
__global__ __launch_bounds__(256) void k_wta_quads(const float* __restrict__ aggL,
                                                   const float* __restrict__ aggR, int pitch,
                                                   int P, int W, int H, int D, int subpixel,
                                                   int16_t* __restrict__ dL,
                                                   int16_t* __restrict__ dR,
                                                   float* __restrict__ disp) {
    const int nq = (W + 3) / 4, k = blockIdx.x * 256 + threadIdx.x, y = k / nq;
    if (y >= H) return;
    const int x = min(4 * (k - y * nq), W - 4), i = y * W + x, v = y * pitch + x;
    if (blockIdx.y == 0) {
        const dco::WtaQuad l = dco::wta_any<kPaired, true, false>(aggL, P, D, v, W, subpixel);
        dco::put_bd<false>(dL + i, l, W);
        dco::wta_store<false, dco::f32x4u>(disp + i, (float)l.bd[0] + l.del[0],
                                           (float)l.bd[1] + l.del[1], (float)l.bd[2] + l.del[2],
                                           (float)l.bd[3] + l.del[3], W);
    } else {
        dco::put_bd<false>(dR + i, dco::wta_any<kPaired, false, false>(aggR, P, D, v, W, subpixel),
                           W);
    }
}

__global__ __launch_bounds__(256) void k_lrcheck(const int16_t* __restrict__ dL,
                                                 const int16_t* __restrict__ dR, int W,
                                                 int P, int maxdiff, float* __restrict__ disp,
                                                 uint8_t* __restrict__ valid, HalfOut half) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= P) return;
    const int x = i % W, d = dL[i], xr = x - d;
    const bool ok = xr >= 0 && abs(d - (int)dR[i - d]) <= maxdiff;
    float v = ok ? disp[i] : 0.0f;
    if (half.on) v *= 2.0f;
    if (half.depth) half.depth[i] = v > 0.0f ? half.fB / v : 0.0f;
    disp[i] = v;
    valid[i] = ok ? 1 : 0;
}

// Where k_wta_quads and k_lrcheck are faster than k_wta_row.  Times of the row kernel,
// then of the two launches, for paired volumes (whole ones in brackets):
//   - rows past kRowCols, which k_wta_row would take in turns: 8192 x 16, D = 64 68.1 us
//     (78.2), 17.6 (20.2); 2100 x 400 67.2 (93.2), 56.5 (77.8); 2560 x 600 110.5
//     (153.1), 92.1 (142.6); 3840 x 1080 257.0 (389.9), 243.0 (386.1);
//   - many short rows, whose idle lanes (of both views) would make more than 1536
//     threads on each CU: 33 x 4000, D = 32 14.2 (20.7), 13.4 (12.2); 33 x 16000 42.8
//     (64.8), 25.2 (28.8); 65 x 8000 25.8 (37.4), 22.5 (28.6); but 33 x 2384 10.9
//     (13.6), 11.7 (11.0), 17 x 2300, D = 12 8.0 (7.1), 10.1 (7.5);
//   - few long rows of many disparities, whose volumes are more than half of the CUs or
//     fewer can read in that time: 2048 x 8, D = 128 20.1 (29.4), 12.7 (27.5); 2048 x
//     100 24.2 (51.2), 22.8 (38.6); 1600 x 64 20.4 (35.4), 15.6 (30.4); but 2048 x 200
//     34.3 (62.9), 43.9 (73.6), 1280 x 48 15.5 (27.3), 14.2 (28.6), 2048 x 32, D = 32
//     9.6 (8.0), 9.7 (10.0).
// Else the launch that the row kernel saves is worth more: 320 x 240, D = 32 5.9 (8.6),
// 10.0 (11.0).
constexpr int kCus = 256;
bool by_quads(int W, int H, int D, int nt) {
    const int idle = nt - (W + 3) / 4;  // of a view's threads in a row's workgroup
    return W >= 4 && (W > kRowCols || 2LL * H * idle > kCus * 1536 ||
                      (2 * H <= kCus && (long long)W * D > 192 * 1024));
}

// Slices d0 .. d0 + n - 1 of a paired-layout volume, decoded to n x P.
__global__ __launch_bounds__(256) void k_unpair(const float* __restrict__ vol, int pitch, int W,
                                                int H, int D, int d0, int n,
                                                float* __restrict__ out) {
    const size_t k = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int P = W * H;
    if (k >= (size_t)n * P) return;
    const int s = (int)(k / P), i = (int)(k - (size_t)s * P), y = i / W;
    out[k] = dco::paired_at(vol, pitch * H, D, d0 + s, i + y * (pitch - W));
}

}  // namespace

hipError_t launch_wta_lr(const float* aggL, const float* aggR, bool paired, int pitch, int W,
                         int H, int D, int subpixel, int maxdiff, int16_t* dL, int16_t* dR,
                         float* disp, uint8_t* valid, const HalfOut& half, hipStream_t st) {
    const int nt = std::min(kWtaThreads / 2, ((W + 3) / 4 + 63) / 64 * 64);
    if (by_quads(W, H, D, nt)) {
        const auto quads = paired ? k_wta_quads<true> : k_wta_quads<false>;
        const unsigned n = (unsigned)H * ((W + 3) / 4);
        hipLaunchKernelGGL(quads, dim3((n + 255) / 256, 2), dim3(256), 0, st, aggL, aggR, pitch,
                           pitch * H, W, H, D, subpixel, dL, dR, disp);
        hipLaunchKernelGGL(k_lrcheck, dim3((unsigned)(W * H + 255) / 256), dim3(256), 0, st, dL, dR,
                           W, W * H, maxdiff, disp, valid, half);
        return hipGetLastError();
    }
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(H), dim3(2 * nt), (size_t)W * sizeof(int16_t), st, aggL,
                           aggR, pitch, pitch * H, W, D, subpixel, maxdiff, dL, dR, disp, valid,
                           half);
    };
    if (W < 4)
        paired ? go(k_wta_row<true, true>) : go(k_wta_row<false, true>);
    else
        paired ? go(k_wta_row<true, false>) : go(k_wta_row<false, false>);
    return hipGetLastError();
}

hipError_t launch_unpair(const float* vol, int pitch, int W, int H, int D, int d0, int n,
                         float* out, hipStream_t st) {
    const size_t total = (size_t)n * W * H;
    hipLaunchKernelGGL(k_unpair, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, vol,
                       pitch, W, H, D, d0, n, out);
    return hipGetLastError();
}
