// k_contour.hip -- depth contour extraction given the two optical flow
// fields (Sec. 5): gradient amplitude of each flow (Eq. 6-8), bidirectional
// fusion (Eq. 9-12), box filter and normalisation (Sec. 5.2), and Canny on
// the grey image with the depth gate (Sec. 5.3).
//
// Every floating-point value that decides a pixel (the fusion choice, the
// gate) is formed with the same IEEE operations, in the same order, as the
// definition; square roots are correctly rounded (sqrt_rn), so the maps are
// exact functions of the inputs.  The Sobel gradients are exact integers.
// Hysteresis grows strong pixels into 8-connected weak ones on bit planes (one
// 64-bit word per 64 pixels of a row): each launch iterates inside 64 x 16 tiles
// in registers until nothing changes, from one plane into the other, and the
// host repeats launches until a launch changes nothing.  The fixed point is the
// set of weak pixels connected to a strong one, whatever the order of the
// growth.
//
// A frame is a chain of short launches: three for the maps, then a group of
// kHystGroup hysteresis launches, of which the one after the first that changed
// nothing writes the contour and the rest do nothing, and one host check.
// 1280 x 720: the maps 27 us (49 as six launches, the Sobel tiles 64 x 4 with a
// load per byte: 21 us of them), a hysteresis launch 4 us (9.5 on bytes in
// LDS), the whole call 81 us (180 with groups of four launches, a check after
// each, and the contour as a launch after the last).  It is bound by its
// eleven launches and the check, not by its 30 MB.
#include "dco_device.h"

namespace {

// Correctly rounded single-precision square root: the hardware root is
// within one ulp, and the exact double squares of the two half-ulp
// boundaries around it pick the rounded value (a float's square root is
// never exactly at a boundary).
__device__ inline float sqrt_rn(float x) {
    if (!(x > 0.0f)) return x == 0.0f ? 0.0f : __builtin_nanf("");
    float y = __builtin_sqrtf(x);
    const double xd = x;
    const float up = __uint_as_float(__float_as_uint(y) + 1u);  // y > 0: the next floats
    const float dn = __uint_as_float(__float_as_uint(y) - 1u);
    const double hi = ((double)y + (double)up) * 0.5, lo = ((double)y + (double)dn) * 0.5;
    if (hi * hi < xd) y = up;
    else if (lo * lo > xd) y = dn;
    return y;
}

__device__ inline float flow_r(const float2* F, int i) {
    const float2 f = F[i];
    return sqrt_rn(f.x * f.x + f.y * f.y);
}

// Eq. 6-8: max(|r(p_right) - r(p)|, |r(p_bottom) - r(p)|), 0 for a missing neighbour.
__device__ inline float flow_amp(const float2* F, int w, int h, int x, int y) {
    const int i = y * w + x;
    const float r = flow_r(F, i);
    const float gu = x + 1 < w ? fabsf(flow_r(F, i + 1) - r) : 0.0f;
    const float gv = y + 1 < h ? fabsf(flow_r(F, i + w) - r) : 0.0f;
    return gu > gv ? gu : gv;
}

// Eq. 9-11: f1 - f0, the flow at p +- rint(e) projected on e = I(p) / |I(p)|.
__device__ inline float flow_score(const float2* F, int w, int h, int x, int y) {
    const int i = y * w + x;
    const float r = flow_r(F, i);
    if (r == 0.0f) return 0.0f;
    const float2 f = F[i];
    const float ex = f.x / r, ey = f.y / r;
    const int sx = (int)rintf(ex), sy = (int)rintf(ey);
    const int x1 = dco::clampi(x + sx, 0, w - 1), y1 = dco::clampi(y + sy, 0, h - 1);
    const int x0 = dco::clampi(x - sx, 0, w - 1), y0 = dco::clampi(y - sy, 0, h - 1);
    const float2 a = F[y1 * w + x1], b = F[y0 * w + x0];
    const float f1 = a.x * ex + a.y * ey;
    const float f0 = b.x * ex + b.y * ey;
    return f1 - f0;
}

// Largest v over the 256-thread block, then one atomic maximum per block
// into one of kContourMaxSlots slots (spread so that thousands of blocks do
// not queue on one address); the maximum does not depend on the order.
template <typename T>
__device__ inline void block_max_to(T v, T* slots) {
    __shared__ T red[4];
    for (int o = 32; o > 0; o >>= 1) {
        const T u = __shfl_xor(v, o, 64);
        v = u > v ? u : v;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        T m = red[0];
        for (int k = 1; k < 4; ++k) m = red[k] > m ? red[k] : m;
        atomicMax(slots + ((blockIdx.x + blockIdx.y * gridDim.x) & (kContourMaxSlots - 1)), m);
    }
}

// The maximum over the slots, for every thread of the block (all threads
// must call it).
template <typename T>
__device__ inline T slots_max(const T* slots) {
    static_assert(kContourMaxSlots == 64, "one slot per lane of the first wavefront");
    __shared__ T m;
    if (threadIdx.x < 64) {
        T v = slots[threadIdx.x];
        for (int o = 32; o > 0; o >>= 1) {
            const T u = __shfl_xor(v, o, 64);
            v = u > v ? u : v;
        }
        if (threadIdx.x == 0) m = v;
    }
    __syncthreads();
    return m;
}

// Eq. 12 per pixel of the flow grid (equal scores keep the larger amplitude).
// The first block clears the frame's maxima and the first group's flags.
__global__ __launch_bounds__(256) void k_fuse(const float2* __restrict__ past,
                                              const float2* __restrict__ future, int w, int h,
                                              float* __restrict__ fused,
                                              unsigned* __restrict__ box_max,
                                              int* __restrict__ g2_max,
                                              int* __restrict__ changed) {
    if (blockIdx.x == 0 && threadIdx.x < kContourMaxSlots) {
        box_max[threadIdx.x] = 0u;
        g2_max[threadIdx.x] = 0;
        if (threadIdx.x < kHystGroup) changed[threadIdx.x] = 0;
    }
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= w * h) return;
    const int y = i / w, x = i - y * w;
    const float mp = flow_amp(past, w, h, x, y), mf = flow_amp(future, w, h, x, y);
    const float sp = flow_score(past, w, h, x, y), sf = flow_score(future, w, h, x, y);
    fused[i] = sp > sf ? mp : (sf > sp ? mf : (mp > mf ? mp : mf));
}

// Mean over the (2R + 1)^2 window clipped to the grid, summed row by row,
// left to right; the largest mean goes to *mx (non-negative floats order
// like their bit patterns, so an integer maximum is exact).  kR >= 0: the
// window size at compile time, so its loads are issued together; a place
// outside the grid adds zero, which changes no bit of the sum.
template <int kR>
__device__ inline unsigned box_pixel(const float* __restrict__ fused, int w, int h, int R, int i,
                                     float* __restrict__ box) {
    const int y = i / w, x = i - y * w;
    float s = 0.0f;
    if constexpr (kR >= 0) {
        float v[(2 * kR + 1) * (2 * kR + 1)];
        int k = 0;
#pragma unroll
        for (int dy = -kR; dy <= kR; ++dy)
#pragma unroll
            for (int dx = -kR; dx <= kR; ++dx)
                v[k++] = fused[dco::clampi(y + dy, 0, h - 1) * w + dco::clampi(x + dx, 0, w - 1)];
        k = 0;
#pragma unroll
        for (int dy = -kR; dy <= kR; ++dy)
#pragma unroll
            for (int dx = -kR; dx <= kR; ++dx) {
                const bool in = y + dy >= 0 && y + dy < h && x + dx >= 0 && x + dx < w;
                s += in ? v[k] : 0.0f;
                ++k;
            }
    } else {
        for (int yy = max(y - R, 0); yy <= min(y + R, h - 1); ++yy)
            for (int xx = max(x - R, 0); xx <= min(x + R, w - 1); ++xx) s += fused[yy * w + xx];
    }
    const int n = (min(y + R, h - 1) - max(y - R, 0) + 1) * (min(x + R, w - 1) - max(x - R, 0) + 1);
    const float v = s / (float)n;
    box[i] = v;
    return __float_as_uint(v);
}

// Sobel of the census grey (replicated borders): gx and gy, exact integers; the
// largest G2 = gx^2 + gy^2 of the block is returned to each thread's share.
// One block per 64 x 16 tile: the grey of the tile and a one-pixel ring is
// computed once into LDS, four pixels (12 bytes) per load where the tile lies
// inside the image (else pixel by pixel, clamped, which replicates the
// borders); a thread then takes four rows of one column.
constexpr int kSobTW = 64, kSobTH = 16;
constexpr int kSobRW = kSobTW + 4, kSobRH = kSobTH + 2;  // columns x0 - 2 .. x0 + 65
struct SobelLds {
    int Y[kSobRH][kSobRW];
};

__device__ inline int sobel_tile(const uint8_t* __restrict__ rgb, int W, int H, int x0, int y0,
                                 short2* __restrict__ g, SobelLds& S) {
    typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
    typedef u32x3 u32x3u __attribute__((aligned(1)));
    const int t = threadIdx.x;
    if (x0 >= 2 && y0 >= 1 && x0 + kSobTW + 2 <= W && y0 + kSobTH + 1 <= H) {
        for (int k = t; k < kSobRH * (kSobRW / 4); k += 256) {
            const int ry = k / (kSobRW / 4), c = 4 * (k - ry * (kSobRW / 4));
            const u32x3 v = *reinterpret_cast<const u32x3u*>(
                rgb + 3 * ((size_t)(y0 + ry - 1) * W + (x0 + c - 2)));
            S.Y[ry][c] = (int)dco::grey_of(v.x);
            S.Y[ry][c + 1] = (int)dco::grey_of(__builtin_amdgcn_alignbyte(v.y, v.x, 3));
            S.Y[ry][c + 2] = (int)dco::grey_of(__builtin_amdgcn_alignbyte(v.z, v.y, 2));
            S.Y[ry][c + 3] = (int)dco::grey_of(v.z >> 8);
        }
    } else {
        for (int k = t; k < kSobRH * kSobRW; k += 256) {
            const int ry = k / kSobRW, c = k - ry * kSobRW;
            const int xx = dco::clampi(x0 + c - 2, 0, W - 1);
            const int yy = dco::clampi(y0 + ry - 1, 0, H - 1);
            const size_t q = 3 * ((size_t)yy * W + xx);
            S.Y[ry][c] = (int)dco::grey_of((uint32_t)rgb[q] | (uint32_t)rgb[q + 1] << 8 |
                                           (uint32_t)rgb[q + 2] << 16);
        }
    }
    __syncthreads();
    const int tx = t & (kSobTW - 1), ty = t / kSobTW * 4, x = x0 + tx;
    int best = 0;
    int l[3], m[3], r[3];  // S.Y[row][tx + 2 + dx] is the grey at x + dx
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        l[k] = S.Y[ty + k][tx + 1];
        m[k] = S.Y[ty + k][tx + 2];
        r[k] = S.Y[ty + k][tx + 3];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i0 = k % 3, i1 = (k + 1) % 3, i2 = (k + 2) % 3;  // rows above, of, below
        l[i2] = S.Y[ty + k + 2][tx + 1];
        m[i2] = S.Y[ty + k + 2][tx + 2];
        r[i2] = S.Y[ty + k + 2][tx + 3];
        const int y = y0 + ty + k;
        if (x < W && y < H) {
            const int a = r[i0] + 2 * r[i1] + r[i2] - l[i0] - 2 * l[i1] - l[i2];
            const int b = l[i2] + 2 * m[i2] + r[i2] - l[i0] - 2 * m[i0] - r[i0];
            g[(size_t)y * W + x] = make_short2((short)a, (short)b);
            best = max(best, a * a + b * b);
        }
    }
    return best;
}

// The Sobel tiles of the frame (blocks 0 .. nsob - 1) and the box means of the
// flow grid (the others) in one launch.
__global__ __launch_bounds__(256) void k_sobel_box(const uint8_t* __restrict__ rgb, int W, int H,
                                                   short2* __restrict__ g,
                                                   int* __restrict__ g2_max, int nsob,
                                                   const float* __restrict__ fused, int w, int h,
                                                   int R, float* __restrict__ box,
                                                   unsigned* __restrict__ box_max) {
    __shared__ SobelLds S;
    if ((int)blockIdx.x < nsob) {
        const int nx = (W + kSobTW - 1) / kSobTW;
        const int by = blockIdx.x / nx, bx = blockIdx.x - by * nx;
        block_max_to(sobel_tile(rgb, W, H, bx * kSobTW, by * kSobTH, g, S), g2_max);
    } else {
        const int i = (blockIdx.x - nsob) * 256 + threadIdx.x;
        unsigned bits = 0u;
        if (i < w * h)
            bits = R == 2 ? box_pixel<2>(fused, w, h, R, i, box)
                          : box_pixel<-1>(fused, w, h, R, i, box);
        block_max_to(bits, box_max);
    }
}

__device__ inline int mag2(short2 v) { return (int)v.x * (int)v.x + (int)v.y * (int)v.y; }

// Words of a bit plane's row.
__host__ __device__ inline int plane_words(int W) { return (W + 63) / 64; }

// Suppression along the gradient's sector, the depth gate on the flow grid,
// and the double threshold, as bit planes: strong, and weak (above the low
// threshold only).  MI = the normalised magnitude sqrt(G2 / max G2), Mn = the
// box means over their maximum (pixel (2 x, 2 y) writes that of (x, y)).  A
// wavefront takes 64 pixels of a row, a block four rows.
__global__ __launch_bounds__(256) void k_nms(const short2* __restrict__ g, int W, int H,
                                             const float* __restrict__ box, int w, int h,
                                             const unsigned* __restrict__ box_max,
                                             const int* __restrict__ g2_max, float Thigh,
                                             float Tlow, float Tdepth,
                                             unsigned long long* __restrict__ strong,
                                             unsigned long long* __restrict__ weak,
                                             float* __restrict__ MI, float* __restrict__ Mn) {
    const int mx = slots_max(g2_max);
    const float bm = __uint_as_float(slots_max(box_max));
    const int x = blockIdx.x * 64 + (threadIdx.x & 63), y = blockIdx.y * 4 + (threadIdx.x >> 6);
    if (y >= H) return;  // whole wavefronts
    int s = 0;
    if (x < W) {
        const int i = y * W + x;
        const short2 gi = g[i];
        const int v = mag2(gi);
        if (MI) MI[i] = mx > 0 ? sqrt_rn((float)((double)v / (double)mx)) : 0.0f;
        const int fx = min(x / 2, w - 1), fy = min(y / 2, h - 1);
        const float bv = box[fy * w + fx];
        const float gate = bm > 0.0f ? bv / bm : 0.0f;
        if (Mn && x == 2 * fx && y == 2 * fy) Mn[fy * w + fx] = gate;
        const int ax = abs((int)gi.x), ay = abs((int)gi.y);
        int dx, dy;
        if (128 * ay < 53 * ax) {
            dx = 1;
            dy = 0;
        } else if (128 * ax < 53 * ay) {
            dx = 0;
            dy = 1;
        } else if ((gi.x > 0) == (gi.y > 0)) {
            dx = 1;
            dy = 1;
        } else {
            dx = 1;
            dy = -1;
        }
        const int xa = x - dx, ya = y - dy, xb = x + dx, yb = y + dy;
        const int ga = xa >= 0 && xa < W && ya >= 0 && ya < H ? mag2(g[ya * W + xa]) : 0;
        const int gb = xb >= 0 && xb < W && yb >= 0 && yb < H ? mag2(g[yb * W + xb]) : 0;
        if (v > ga && v >= gb && !(gate < Tdepth)) {
            const double th = (double)Thigh * (double)Thigh * (double)mx;
            const double tl = (double)Tlow * (double)Tlow * (double)mx;
            const double dv = (double)v;
            s = dv > th ? 2 : (dv > tl ? 1 : 0);
        }
    }
    const unsigned long long ms = __ballot(s == 2), mw = __ballot(s == 1);
    if ((threadIdx.x & 63) == 0) {
        const size_t q = (size_t)y * plane_words(W) + blockIdx.x;
        strong[q] = ms;
        weak[q] = mw;
    }
}

// 64 pixels of the contour from their word.
__device__ inline void put_edges(unsigned long long m, int W, int x0, uint8_t* __restrict__ row) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef u32x4 u32x4u __attribute__((aligned(1)));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t b = (uint32_t)(m >> (16 * k)) & 0xffffu;
        const int x = x0 + 16 * k;
        if (x + 16 <= W) {
            u32x4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = (b >> (4 * j) & 15u) * 0x00204081u & 0x01010101u;
            *reinterpret_cast<u32x4u*>(row + x) = o;
        } else {
            for (int j = 0; j < 16 && x + j < W; ++j) row[x + j] = (uint8_t)(b >> j & 1u);
        }
    }
}

// v of the lane before / after in its 16 lanes (a tile's rows); 0 past its ends.
template <unsigned Ctrl>
__device__ inline unsigned long long row_shift(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, Ctrl, 0xf, 0xf,
                                                              true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), Ctrl,
                                                              0xf, 0xf, true);
    return (unsigned long long)hi << 32 | lo;
}

// The bits of `s` and everything that candidates `c` connect to them along the
// word, both ways (s within s | c).
__device__ inline unsigned long long fill_row(unsigned long long s, unsigned long long c) {
    unsigned long long u = c, d = c, a = s, b = s;
#pragma unroll
    for (int k = 1; k < 64; k *= 2) {
        a |= u & (a << k);
        u &= u << k;
        b |= d & (b >> k);
        d &= d >> k;
    }
    return a | b;
}

// One hysteresis launch.  A lane holds one row of a 64 x 16 tile (a wavefront
// four tiles, one above the other) and grows its strong bits into the weak ones
// around them until its tiles are stable; strong bits outside the tile count as
// `in` has them.  *changed is set if any pixel changed.  prev: the flag of the
// launch before (none for a group's first): if it changed nothing, the state is
// final, and the first launch to see that writes the contour.
constexpr int kHystRows = 64;  // rows of a block's four wavefronts, one word each

__global__ __launch_bounds__(256) void k_hyst(const unsigned long long* __restrict__ in,
                                              const unsigned long long* __restrict__ weak, int W,
                                              int H, unsigned long long* __restrict__ out,
                                              const int* __restrict__ prev,
                                              const int* __restrict__ prev2,
                                              int* __restrict__ changed,
                                              uint8_t* __restrict__ B) {
    const int nw = plane_words(W);
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int y = blockIdx.y * kHystRows + (threadIdx.x & 63);
    // the same values for every thread of every block
    const bool final_state = prev && *prev == 0;
    if (final_state) {
        if (!(prev2 && *prev2 == 0) && q < nw && y < H)
            put_edges(in[(size_t)y * nw + q], W, 64 * q, B + (size_t)y * W);
        return;
    }
    if (q >= nw) return;  // whole wavefronts
    const auto word = [&](int yy, int qq) {
        return yy >= 0 && yy < H && qq >= 0 && qq < nw ? in[(size_t)yy * nw + qq] : 0ull;
    };
    // a row's strong bits and their neighbours along the row, as `in` has them
    const auto halo = [&](int yy) { return word(yy, q - 1) >> 63 | word(yy, q + 1) << 63; };
    const auto spread = [](unsigned long long s) { return s | s << 1 | s >> 1; };
    const unsigned long long c = y < H ? weak[(size_t)y * nw + q] : 0ull;
    const unsigned long long s0 = word(y, q), side = halo(y);
    unsigned long long fixed = side;  // neighbours outside the tile
    if ((y & 15) == 0) fixed |= spread(word(y - 1, q)) | halo(y - 1);
    if ((y & 15) == 15) fixed |= spread(word(y + 1, q)) | halo(y + 1);
    unsigned long long s = s0;
    for (;;) {
        const unsigned long long n = spread(s) | side;
        const unsigned long long around = n | row_shift<0x111>(n) | row_shift<0x101>(n) | fixed;
        const unsigned long long grown = fill_row(s | (c & around), c);
        const bool grew = grown != s;
        s = grown;
        if (!__any(grew)) break;
    }
    if (y < H) out[(size_t)y * nw + q] = s;
    if (__any(s != s0) && (threadIdx.x & 63) == 0) *changed = 1;
}

__global__ __launch_bounds__(256) void k_edges(const unsigned long long* __restrict__ st, int W,
                                               int H, uint8_t* __restrict__ B) {
    const int nw = plane_words(W);
    const size_t k = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= (size_t)nw * H) return;
    const int y = (int)(k / nw), q = (int)(k - (size_t)y * nw);
    put_edges(st[k], W, 64 * q, B + (size_t)y * W);
}

__global__ void k_zero1(int* a, int n) {
    if ((int)threadIdx.x < n) a[threadIdx.x] = 0;
}

inline dim3 grid1(int n) { return dim3((n + 255) / 256); }

}  // namespace

hipError_t launch_contour_maps(const float* past, const float* future, int w, int h, int R,
                               const uint8_t* rgb, int W, int H, float Thigh, float Tlow,
                               float Tdepth, const ContourBufs& b, float* Mn, float* MI,
                               hipStream_t st) {
    static_assert(kHystGroup <= kContourMaxSlots, "the clearing block covers the flags");
    hipLaunchKernelGGL(k_fuse, grid1(w * h), dim3(256), 0, st,
                       reinterpret_cast<const float2*>(past),
                       reinterpret_cast<const float2*>(future), w, h, b.fused, b.box_max, b.g2_max,
                       b.changed);
    const int nsob = (W + kSobTW - 1) / kSobTW * ((H + kSobTH - 1) / kSobTH);
    hipLaunchKernelGGL(k_sobel_box, dim3(nsob + (w * h + 255) / 256), dim3(256), 0, st, rgb, W, H,
                       b.g, b.g2_max, nsob, b.fused, w, h, R, b.box, b.box_max);
    hipLaunchKernelGGL(k_nms, dim3(plane_words(W), (H + 3) / 4), dim3(256), 0, st, b.g, W, H,
                       b.box, w, h, b.box_max, b.g2_max, Thigh, Tlow, Tdepth, b.strong[0], b.weak,
                       MI, Mn);
    return hipGetLastError();
}

size_t contour_plane_words(int W, int H) { return (size_t)plane_words(W) * H; }

// Launch k of the group reads strong[parity ^ (k & 1)] and writes the other
// plane; kHystGroup is even, so the group's last output is strong[parity].
hipError_t launch_contour_hyst_group(const ContourBufs& b, int W, int H, int parity, bool first,
                                     uint8_t* B, hipStream_t st) {
    static_assert(kHystGroup % 2 == 0 && kHystGroup <= 64, "even group, one flag per lane");
    if (!first)  // the first group's flags are cleared with the maps
        hipLaunchKernelGGL(k_zero1, dim3(1), dim3(64), 0, st, b.changed, kHystGroup);
    const dim3 grid((plane_words(W) + 3) / 4, (H + kHystRows - 1) / kHystRows);
    for (int k = 0; k < kHystGroup; ++k) {
        const int p = parity ^ (k & 1);
        const int* none = nullptr;
        hipLaunchKernelGGL(k_hyst, grid, dim3(256), 0, st, b.strong[p], b.weak, W, H,
                           b.strong[1 - p], k > 0 ? (const int*)(b.changed + k - 1) : none,
                           k > 1 ? (const int*)(b.changed + k - 2) : none, b.changed + k, B);
    }
    return hipGetLastError();
}

hipError_t launch_contour_edges(const ContourBufs& b, int W, int H, int parity, uint8_t* B,
                                hipStream_t st) {
    hipLaunchKernelGGL(k_edges, dim3((unsigned)((contour_plane_words(W, H) + 255) / 256)),
                       dim3(256), 0, st, b.strong[parity], W, H, B);
    return hipGetLastError();
}
