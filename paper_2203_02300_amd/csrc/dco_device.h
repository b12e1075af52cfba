// dco_device.h -- device-side bodies of every stage of the plain matcher.
//
// The one-call kernels (k_census.hip, k_aggregate.hip, k_wta.hip) and the
// batched work-list kernels (k_batch.hip) run exactly these functions, so a
// pair matched alone and the same pair matched in a batch give the same bits.
// Each function takes its LDS as an explicit struct.
#pragma once

#include "dco_internal.h"

namespace dco {

// ===========================================================================
// Census codes and cross-support arms (Sec. 4.1; C_census of Eq. 1)
// ===========================================================================

constexpr int kCenTW = 64, kCenTH = 16;     // pixel tile (one of TH rows in small frames)
constexpr int kCenRW = kCenTW + 2 * kLMax;  // staged RGB region
constexpr int kCenHW = 4, kCenHH = 4;       // census half-window limits
constexpr int kCenGW = kCenTW + 2 * kCenHW;

template <int TH>
struct CensusLdsOf {
    uint32_t rgb[TH + 2 * kLMax][kCenRW];  // channels in 10-bit fields
    uint32_t grey[TH + 2 * kCenHH][kCenGW];
};
using CensusLds = CensusLdsOf<kCenTH>;

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// DPP move of v (lanes without a source read 0): row shifts 0x111..0x118,
// row broadcasts 0x142 (lane 15 of each row to the next row) and 0x143
// (lane 31 to rows 2 and 3).
template <unsigned Ctrl, unsigned RowMask>
__device__ inline uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, Ctrl, RowMask, 0xf, false);
}

__device__ inline uint32_t grey_of(uint32_t c) {
    uint32_t r = c & 0xffu, g = (c >> 8) & 0xffu, b = (c >> 16) & 0xffu;
    return (77u * r + 150u * g + 29u * b + 128u) >> 8;
}

// The three channels in 10-bit fields (8 bits and two guard bits each).
__device__ inline uint32_t rgb_fields(uint32_t r, uint32_t g, uint32_t b) {
    return r | g << 10 | b << 20;
}
__device__ inline uint32_t rgb_of_fields(uint32_t f) {
    return (f & 0xffu) | (f >> 2 & 0xff00u) | (f >> 4 & 0xff0000u);
}
__device__ inline uint32_t grey_of_fields(uint32_t f) {
    return (77u * (f & 0xffu) + 150u * (f >> 10 & 0xffu) + 29u * (f >> 20) + 128u) >> 8;
}

// Largest per-channel absolute difference below tau (1 <= tau <= 256), for the
// three channels of centre a and neighbour b at once: with every field of `lo`
// a + tau + 511 and of `hi` tau + 511 - a, bit 9 of a field of lo - b says b - a <
// tau and that of hi + b says a - b < tau (both stay within ten bits, so no field
// borrows from the next).  Bit 31 of the result is set when all six bits are.
// Five instructions per step with the shift into the mask; a byte at a time
// seven (census and arms of both views of 1280 x 720 in 47 us, were 52: bound by
// vector issue).
struct Centre {
    uint32_t lo, hi;
};
constexpr uint32_t kField9 = 512u * (1u | 1u << 10 | 1u << 20);
__device__ inline Centre centre_of(uint32_t a, int tau) {
    const uint32_t k = (511u + (uint32_t)tau) * (1u | 1u << 10 | 1u << 20);
    return Centre{k + a, k - a};
}
__device__ inline uint32_t close_rgb(const Centre& c, uint32_t b) {
    return ((c.lo - b) & (c.hi + b) & kField9) + (0x80000000u - kField9);
}

// Census code of tile pixel (tx, ty) from the grey levels in LDS: bit k is
// set when neighbour k (row-major over the window, centre skipped) is darker
// than the centre.  The fixed-size form unrolls, so its LDS reads pipeline.
// Grey levels are below 256, so n - c is negative exactly when n < c: each
// bit enters as the sign of n - c with one funnel shift (alignbit), from the
// last neighbour back to the first, the upper bits in one word and the lower
// in another.
template <int HW, int HH, typename Lds>
__device__ inline uint64_t census_code(const Lds& S, int tx, int ty) {
    constexpr int kBits = (2 * HW + 1) * (2 * HH + 1) - 1;
    static_assert(kBits <= 64, "one 64-bit code");
    const uint32_t c = S.grey[ty + kCenHH][tx + kCenHW];
    uint32_t hi = 0, lo = 0;
#pragma unroll
    for (int k = kBits - 1; k >= 0; --k) {
        constexpr int kCentre = HH * (2 * HW + 1) + HW;
        const int n = k < kCentre ? k : k + 1;  // window index, centre skipped
        const int dy = n / (2 * HW + 1) - HH, dx = n % (2 * HW + 1) - HW;
        const uint32_t d = S.grey[ty + kCenHH + dy][tx + kCenHW + dx] - c;
        if (k >= 32)
            hi = __builtin_amdgcn_alignbit(hi, d, 31);
        else
            lo = __builtin_amdgcn_alignbit(lo, d, 31);
    }
    return (uint64_t)hi << 32 | lo;
}

template <typename Lds>
__device__ inline uint64_t census_code_any(const Lds& S, int tx, int ty, int hw, int hh) {
    const uint32_t c = S.grey[ty + kCenHH][tx + kCenHW];
    uint64_t code = 0;
    int bit = 0;
    for (int dy = -hh; dy <= hh; ++dy)
        for (int dx = -hw; dx <= hw; ++dx) {
            if (dy == 0 && dx == 0) continue;
            code |= (uint64_t)(S.grey[ty + kCenHH + dy][tx + kCenHW + dx] < c) << bit;
            ++bit;
        }
    return code;
}

// One 64 x TH tile at (x0, y0), NT threads, each 64 TH / NT pixels.  The tile plus
// a kLMax apron (edge-clamped) is staged in LDS as RGB fields; grey levels of the
// tile plus the census apron go to a second array.
//   grey:   Y = (77 R + 150 G + 29 B + 128) >> 8
//   census: bit k = Y(q_k) < Y(p), neighbours row-major without the centre
//   arms:   steps j = 1.. while inside, j <= L1 and max channel |diff| < tau1
template <int NT, int TH = kCenTH>
__device__ inline __attribute__((always_inline)) void census_tile(
    const uint8_t* __restrict__ rgb, int W, int H, int cw, int ch, int L1, int tau1,
    uint64_t* __restrict__ census, uint32_t* __restrict__ arms, uint32_t* __restrict__ rgb_packed,
    uint4* __restrict__ pix, bool planes, int x0, int y0, CensusLdsOf<TH>& S) {
    constexpr int kRH = TH + 2 * kLMax, kGH = TH + 2 * kCenHH;
    static_assert(NT % 64 == 0 && (kCenTW * TH) % NT == 0, "whole rows per pass");
    const int t = threadIdx.x;
    {   // stage the region: every load issued before any is stored
        constexpr int kN = (kCenRW * kRH + NT - 1) / NT;
        uint32_t v[kN];
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int i = min(t + NT * k, kCenRW * kRH - 1);
            const int ry = i / kCenRW, rx = i - ry * kCenRW;
            const int gx = clampi(x0 - kLMax + rx, 0, W - 1);
            const int gy = clampi(y0 - kLMax + ry, 0, H - 1);
            const uint8_t* p = rgb + 3 * ((size_t)gy * W + gx);
            v[k] = rgb_fields(p[0], p[1], p[2]);
        }
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int i = t + NT * k;
            if (i < kCenRW * kRH) {
                const int ry = i / kCenRW;
                S.rgb[ry][i - ry * kCenRW] = v[k];
            }
        }
    }
    __syncthreads();
    for (int i = t; i < kCenGW * kGH; i += NT) {
        int gy = i / kCenGW, gx = i - gy * kCenGW;
        S.grey[gy][gx] = grey_of_fields(S.rgb[gy + kLMax - kCenHH][gx + kLMax - kCenHW]);
    }
    __syncthreads();

    const int hw = cw >> 1, hh = ch >> 1;
    const int tx = t & 63;
    for (int k = 0; k < TH / (NT / 64); ++k) {
        const int ty = (t >> 6) + (NT / 64) * k;
        const int x = x0 + tx, y = y0 + ty;
        if (x >= W || y >= H) continue;
        const uint64_t code = cw == 9 && ch == 7
                                  ? census_code<4, 3>(S, tx, ty)
                                  : census_code_any(S, tx, ty, hw, hh);
        if (census) census[(size_t)y * W + x] = code;

        const int rx = tx + kLMax, ry = ty + kLMax;
        const uint32_t cf = S.rgb[ry][rx], cp = rgb_of_fields(cf);
        // each arm: the closeness of all kLMax steps as a bit mask (the reads
        // are independent, so they pipeline), then the run of ones from
        // step 1, capped by L1 and the border
        const Centre cc = centre_of(cf, tau1);
        uint32_t ml = 0, mr = 0, mu = 0, md = 0;
#pragma unroll
        for (int j = kLMax; j >= 1; --j) {  // step j's bit ends at j - 1
            ml = __builtin_amdgcn_alignbit(ml, close_rgb(cc, S.rgb[ry][rx - j]), 31);
            mr = __builtin_amdgcn_alignbit(mr, close_rgb(cc, S.rgb[ry][rx + j]), 31);
            mu = __builtin_amdgcn_alignbit(mu, close_rgb(cc, S.rgb[ry - j][rx]), 31);
            md = __builtin_amdgcn_alignbit(md, close_rgb(cc, S.rgb[ry + j][rx]), 31);
        }
        const int al = min(min(L1, x), __builtin_ctz(~ml));
        const int ar = min(min(L1, W - 1 - x), __builtin_ctz(~mr));
        const int au = min(min(L1, y), __builtin_ctz(~mu));
        const int ad = min(min(L1, H - 1 - y), __builtin_ctz(~md));
        arms[(size_t)y * W + x] =
            (uint32_t)al | ((uint32_t)ar << 8) | ((uint32_t)au << 16) | ((uint32_t)ad << 24);
        if (rgb_packed) rgb_packed[(size_t)y * W + x] = cp;
        // everything the fused raw cost needs of a pixel: census code, packed
        // RGB and 8 L_min (the byte offset of the pixel's (alpha, beta) pair),
        // in planes for the two-slice kernel or in one 16-byte word
        const uint32_t lmin8 = (uint32_t)(8 * min(min(al, ar), min(au, ad)));
        if (pix && planes) {
            const PixPlanes px(W, H);
            uint32_t* p = reinterpret_cast<uint32_t*>(pix);
            const size_t i = (size_t)y * px.Wq + x;
            p[kPixPad + i] = (uint32_t)code;
            p[px.plane + kPixPad + i] = (uint32_t)(code >> 32);
            p[2 * px.plane + kPixPad + i] = cp;
            reinterpret_cast<uint8_t*>(p + 3 * px.plane)[i] = (uint8_t)lmin8;
        } else if (pix) {
            pix[(size_t)y * W + x] =
                make_uint4((uint32_t)code, (uint32_t)(code >> 32), cp, lmin8);
        }
    }
}

// ===========================================================================
// Region counts and packed aggregation records of one pixel
// ===========================================================================
//   N1 = sum over y' in [y-u, y+dn] of (l(x,y') + r(x,y') + 1)
//   N2 = sum over x' in [x-l, x+r] of (u(x',y) + dn(x',y) + 1)
// A final division by N uses N' = N * 2^20 and y' = RN(1/N) * 2^-20 (both
// exact scalings), so that it also removes the Q20 scale (div_q20 below).
//
// The streaming kernels keep row r of a column-prefix ring in slot r mod R,
// so the byte offsets of the two prefix rows of a vertical range are fixed
// per pixel and are stored here (16 bits each).

constexpr int kAggK = kStripThreads / 64;             // rows per chunk = wavefronts (4)
constexpr int kSeg = kStripThreads / 64;              // 64-column segments of a strip row
constexpr int kRing1 = 2 * kLMax + 1 + kAggK;         // prefix rows per column (one stage)
constexpr int kRingCols = kStripThreads - 2 * kLMax;  // columns with a ring: 222
constexpr int kRingStride = 224;                      // a multiple of the 32 LDS banks
constexpr uint32_t kSlotBytes = kRingStride * 4;
constexpr int kPStride = 280;                         // prefix row: P(-1) at 0, P(i) at i + 1
constexpr uint32_t kOOB = 0x7fffffffu;                // buffer offset that reads as 0
static_assert(kRing1 * kSlotBytes < 65536, "ring offsets are stored in 16 bits");
static_assert(kStripThreads == 256 && kAggK == 4, "one row per wavefront per chunk");

__device__ inline uint32_t ring_slot(int row, int ring) {
    int s = row % ring;
    if (s < 0) s += ring;
    return (uint32_t)s;
}
__device__ inline uint32_t ring_slot_bytes(int row, int ring) {
    return ring_slot(row, ring) * kSlotBytes;
}

// Layout of the two-slice kernel (agg_stream_ws) that its records address.
constexpr int kWsThreads = 3 * kStripThreads;
constexpr int kWsSlices = 2;
constexpr int kWsRing = 2 * kLMax + 2;
constexpr int kWsCols = 224;                          // columns with a ring, from kWsI0 on
constexpr uint32_t kWsSlotBytes = kWsCols * 8;        // one ring row of both slices
constexpr int kWsLanes = kWsCols / 4;                 // output lanes with columns
constexpr int kWsPlane = kWsLanes + 1;                // entries of a plane of an output row's
                                                      // prefixes (with the sum of all columns)
constexpr uint32_t kWsPlaneBytes = kWsPlane * 8;
constexpr uint32_t kWsOffBias = 64;                   // keeps the left offsets non-negative
static_assert(kWsRing % kAggK == 0, "a chunk's slots are consecutive");
static_assert(kWsApron % 4 == 0 && kWsOut % 4 == 0 && kWsI0 % 4 == 0 && kWsCols % 4 == 0,
              "quads are aligned");
static_assert(kWsI0 <= kWsApron - kLMax && kWsI0 + kWsCols >= kWsApron + kWsOut + kLMax &&
                  kWsApron >= 2 * kLMax && kWsApron + kWsOut + 2 * kLMax <= kStripThreads &&
                  kWsI0 + kWsCols >= kWsApron + kWsOut + kWsEdge,
              "the strip's aprons");
static_assert((4 * kWsPlane) % 2 == 0, "16-byte rows");
static_assert((kWsRing - 1) * kWsSlotBytes < 65536, "ring offsets are stored in 16 bits");
static_assert(8 * (kLMax + 1) < 256, "arm offsets are stored in 8 bits");

// RN(1 / n) for whole 1 <= n <= (2 kLMax + 1)^2: one Newton step on the hardware
// reciprocal (one ulp) rounds to nearest for each of them.
__device__ inline float recip_count(uint32_t n) {
    const float f = (float)n, y = __builtin_amdgcn_rcpf(f);
    return __builtin_fmaf(__builtin_fmaf(-f, y, 1.0f), y, y);
}

// Arms of a pixel, each at most kLMax (census_tile's never exceed it; the clamp
// only keeps an arbitrary caller-supplied arms map from indexing outside the
// tile).
struct Arms {
    int l, r, u, dn;
};
__device__ inline Arms arms_of(uint32_t a) {
    return Arms{min((int)(a & 0xff), kLMax), min((int)(a >> 8 & 0xff), kLMax),
                min((int)(a >> 16 & 0xff), kLMax), min((int)(a >> 24), kLMax)};
}

// Region counts and records (layouts: AggRecords) of 64 columns and 16 record rows
// from (x0, r0) on, 1024 threads.  A record of row r holds N2 of row r, N1
// of row r - kLMax and range ends of row r - 2 kLMax, so the arms of rows r0 - 2
// kLMax .. r0 + 15 (the rows that N1's regions reach) go to LDS as h = l + r + 1
// and v = u + dn + 1; prefix sums of h down each tile column and of v along each
// of the last 16 rows then give every N1 and N2 with two reads.  Apron cells
// outside the image hold 0 and never fall inside a region (arms stop at the
// border).  Each record is one 16-byte store: written in pieces by the pixels it
// takes from, its lines went to memory up to three times (85 MB written for both
// views of 1280 x 720 in 29 us, now 24 us).
constexpr int kGeoTW = 64, kGeoTH = 16;
constexpr int kGeoRW = kGeoTW + 2 * kLMax, kGeoRH = kGeoTH + 2 * kLMax;
__host__ __device__ constexpr int geo_rows(int H) { return H + kWsRecRows; }  // record rows

struct GeomLds {
    uint32_t hv[kGeoRH][kGeoRW];       // h | v << 16
    uint32_t cp[kGeoRH + 1][kGeoTW];   // column prefixes of h (row 0 = 0)
    uint32_t rp[kGeoTH][kGeoRW + 1];   // row prefixes of v (column 0 = 0)
};

// The prefixes are DPP scans (16 lanes per column, one wavefront per row), then
// each thread takes one record.
__device__ inline __attribute__((always_inline)) void geometry_tile(
    const uint32_t* __restrict__ arms, int W, int H, int iters, const AggRecords& rec, int x0,
    int r0, GeomLds& S) {
    constexpr int NT = 1024;
    static_assert(kGeoTW * kGeoTH == NT, "a record per thread");
    const int t = threadIdx.x;
    const int tx = t & 63, ty = t >> 6, x = x0 + tx, r = r0 + ty;
    const int y1 = r - kLMax, y2 = r - 2 * kLMax;
    const bool in0 = r < H, in1 = y1 >= 0 && y1 < H, in2 = y2 >= 0 && y2 < H;
    const int xc = min(x, W - 1);
    const uint32_t w0 = arms[(size_t)min(r, H - 1) * W + xc];
    const uint32_t w1 = arms[(size_t)clampi(y1, 0, H - 1) * W + xc];
    const uint32_t w2 = arms[(size_t)clampi(y2, 0, H - 1) * W + xc];
    {   // stage the arms: every load issued before any is used (clamped addresses)
        constexpr int kN = (kGeoRW * kGeoRH + NT - 1) / NT;
        uint32_t v[kN];
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int i = min(t + NT * k, kGeoRW * kGeoRH - 1);
            const int ry = i / kGeoRW, rx = i - ry * kGeoRW;
            const int x = clampi(x0 - kLMax + rx, 0, W - 1);
            const int y = clampi(r0 - 2 * kLMax + ry, 0, H - 1);
            v[k] = arms[(size_t)y * W + x];
        }
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const int i = t + NT * k;
            if (i < kGeoRW * kGeoRH) {
                const int ry = i / kGeoRW, rx = i - ry * kGeoRW;
                const int x = x0 - kLMax + rx, y = r0 - 2 * kLMax + ry;
                const uint32_t a = v[k];
                S.hv[ry][rx] = x >= 0 && x < W && y >= 0 && y < H
                                   ? ((a & 0xff) + ((a >> 8) & 0xff) + 1) |
                                         ((a >> 16 & 0xff) + (a >> 24) + 1) << 16
                                   : 0u;
            }
        }
    }
    __syncthreads();
    {   // column prefixes of h: column c = t / 16, rows 4 s .. 4 s + 3 with
        // s = t % 16 (16 lanes = one DPP row per column)
        const int c = t >> 4, sg = t & 15;
        uint32_t a[4], tot = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ry = 4 * sg + i;
            tot += ry < kGeoRH ? S.hv[ry][c + kLMax] & 0xffff : 0u;
            a[i] = tot;
        }
        uint32_t inc = tot;
        inc += dpp<0x111, 0xf>(inc);
        inc += dpp<0x112, 0xf>(inc);
        inc += dpp<0x114, 0xf>(inc);
        inc += dpp<0x118, 0xf>(inc);
        const uint32_t before = inc - tot;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ry = 4 * sg + i;
            if (ry < kGeoRH) S.cp[ry + 1][c] = before + a[i];
        }
        if (sg == 0) S.cp[0][c] = 0;
    }
    {   // row prefixes of v: wavefront w takes row w, lane l columns 2 l, 2 l + 1
        const int l = tx;
        const uint32_t v0 = 2 * l < kGeoRW ? S.hv[ty + 2 * kLMax][2 * l] >> 16 : 0u;
        const uint32_t v1 = 2 * l + 1 < kGeoRW ? S.hv[ty + 2 * kLMax][2 * l + 1] >> 16 : 0u;
        const uint32_t tot = v0 + v1;
        uint32_t inc = tot;
        inc += dpp<0x111, 0xf>(inc);
        inc += dpp<0x112, 0xf>(inc);
        inc += dpp<0x114, 0xf>(inc);
        inc += dpp<0x118, 0xf>(inc);
        inc += dpp<0x142, 0xa>(inc);
        inc += dpp<0x143, 0xc>(inc);
        const uint32_t before = inc - tot;
        if (2 * l < kGeoRW) S.rp[ty][2 * l + 1] = before + v0;
        if (2 * l + 1 < kGeoRW) S.rp[ty][2 * l + 2] = before + tot;
        if (l == 0) S.rp[ty][0] = 0;
    }
    __syncthreads();
    if (x >= W || r >= geo_rows(H)) return;
    const Arms a0 = arms_of(in0 ? w0 : 0u), a1 = arms_of(in1 ? w1 : 0u),
               a2 = arms_of(in2 ? w2 : 0u);
    const uint32_t n1 = S.cp[ty + kLMax + a1.dn + 1][tx] - S.cp[ty + kLMax - a1.u][tx];
    const uint32_t n2 = S.rp[ty][tx + kLMax + a0.r + 1] - S.rp[ty][tx + kLMax - a0.l];
    const size_t col = (size_t)x + kRecApronL;
    uint4 w = make_uint4(0u, 0u, 0u, 0u);
    if (iters == 2) {
        constexpr int R = kWsRing;
        if (in1) {
            w.x = __float_as_uint(recip_count(n1));
            w.y = ring_slot(y1 + a1.dn, R) * kWsSlotBytes |
                  ring_slot(y1 - a1.u - 1, R) * kWsSlotBytes << 16;
            w.w = (uint32_t)(uint16_t)(0 - (int)n1) << 16;
        }
        if (in2)
            w.z = ring_slot(y2 + a2.dn + kLMax, R) * kWsSlotBytes |
                  ring_slot(y2 - a2.u - 1 + kLMax, R) * kWsSlotBytes << 16;
        if (in0) {
            w.w |= (uint32_t)(8 * (a0.r + 1) | (8 * a0.l) << 8);
            // byte offsets, from the lane's own entry, of columns x + r + 1 and
            // x - l in a row of prefixes kept in four planes
            const auto plane_off = [&](int k) {
                return (uint32_t)(k & 3) * kWsPlaneBytes + (uint32_t)(8 * (k >> 2)) +
                       kWsOffBias;
            };
            const int j = x & 3;
            uint32_t* c = rec.c + (size_t)r * rec.Wp + col;
            const size_t plane = (size_t)rec.Wp * H;
            c[0] = plane_off(j + a0.r + 1) | plane_off(j - a0.l) << 16;
            c[plane] = __float_as_uint(recip_count(n2) * 0x1p-20f);
            c[2 * plane] = __float_as_uint((float)n2 * 0x1p20f);
        }
    } else {
        if (in1) {
            w.x = __float_as_uint(recip_count(n1) * 0x1p-20f);
            w.y = ring_slot_bytes(y1 + a1.dn, kRing1) |
                  ring_slot_bytes(y1 - a1.u - 1, kRing1) << 16;
            w.z = n1 << 16;
        }
        if (in0) w.z |= (uint32_t)(4 * (a0.r + 1) | (4 * a0.l) << 8);
    }
    *reinterpret_cast<uint4*>(rec.b + 4 * ((size_t)r * rec.Wp + col)) = w;
}

// ===========================================================================
// Streaming one-stage aggregation (Eq. 2 once), one slice x one column strip
// ===========================================================================
//
// A strip is 256 consecutive columns: 2 kLMax apron columns on each side and
// kStripOut output columns in the middle.  The workgroup streams down the
// rows in chunks of kAggK = 4 rows, in two steps per chunk:
//   1 (wavefront w, row yc + w, all 256 columns as 4 segments of 64):
//       raw cost q (fused: Eq. 1 from the images; staged: read), inclusive
//       row prefix P1 by a wavefront scan per segment plus segment carries
//   2 (thread t owns column t, rows yc .. yc + 3 in order):
//       H1: E1 = P1(t + r) - P1(t - l - 1); push the column prefix of E1
//       V1: S1 of row y - kLMax from two prefix rows of the ring
//           out = RN(S1 / N1) * 2^-20
// Two barriers per chunk: after step 1 (P1 rows) and after step 2 (the end of
// its reads of P1).  The ring holds kAggK - 1 rows more than a vertical range
// spans so that a chunk's four pushes can precede its four range reads.
//
// Every sum is an integer and differences of prefix sums are taken mod 2^32
// (every true range sum is below 2^31), so the result does not depend on the
// summation order, and a band of output rows [y0, y1) can start from zero
// prefixes kLMax rows above y0: the rows before the start then shift every
// prefix by the same constant.
//
// Per-pixel data comes from padded records (zero apron) through buffer loads
// with a per-lane column offset and a uniform row offset, so the chunk body
// has no bounds branches.

// Every member starts below 64 KB, so LDS addresses fold into the 16-bit
// instruction offsets.  Reads of a prefix row reach up to kLMax words before
// it (apron lanes, results unused): `guard` and the tables keep them inside
// the allocation.
template <bool kFused>
struct AggLds {
    float tabA[kFused ? 768 : 1];
    float tabC[kFused ? 68 : 1];
    float2 ab[kFused ? kLMax + 1 : 1];
    uint32_t guard[32];
    uint32_t prow[kAggK][kPStride];
    uint32_t ring1[kRing1 * kRingStride];
};

typedef __amdgpu_buffer_rsrc_t rsrc_t;

__device__ inline rsrc_t make_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                             0x00020000);
}
__device__ inline uint32_t ld32(rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0);
}
__device__ inline uint4 ld128(rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
// Stores of the aggregated volume are non-temporal (the volume is streamed to
// HBM and read once by WTA), so they do not evict reused inputs from L2.
__device__ inline void st32(float v, rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, 2);
}

// Inclusive prefix sums of the kSeg segments across the wavefront: DPP row
// shifts 1, 2, 4, 8 and the gfx9 row broadcasts 15 and 31, step-major so the
// segments interleave; then each segment adds the totals of the ones before.
__device__ inline void wave_scan_segments(uint32_t (&v)[kSeg]) {
#pragma unroll
    for (int j = 0; j < kSeg; ++j) v[j] += dpp<0x111, 0xf>(v[j]);
#pragma unroll
    for (int j = 0; j < kSeg; ++j) v[j] += dpp<0x112, 0xf>(v[j]);
#pragma unroll
    for (int j = 0; j < kSeg; ++j) v[j] += dpp<0x114, 0xf>(v[j]);
#pragma unroll
    for (int j = 0; j < kSeg; ++j) v[j] += dpp<0x118, 0xf>(v[j]);
#pragma unroll
    for (int j = 0; j < kSeg; ++j) v[j] += dpp<0x142, 0xa>(v[j]);
#pragma unroll
    for (int j = 0; j < kSeg; ++j) v[j] += dpp<0x143, 0xc>(v[j]);
    uint32_t carry = 0;
#pragma unroll
    for (int j = 0; j < kSeg; ++j) {
        const uint32_t tot = __builtin_amdgcn_readlane(v[j], 63);
        v[j] += carry;
        carry += tot;
    }
}

// Wavefront index inside the workgroup, known to the compiler as uniform.
__device__ inline int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6); }

__device__ inline uint32_t lds_ld(const uint32_t* base, uint32_t byte_off) {
    return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(base) + byte_off);
}
__device__ inline void lds_st(uint32_t* base, uint32_t byte_off, uint32_t v) {
    *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(base) + byte_off) = v;
}

// One Q20 term of Eq. 1, rint(a t) rounded once from the exact product of
// the float factors (a carries the 2^20 scale), for 0 <= a t < 2^22: the
// fused a t + 2^23 rounds to 2^23 + rint(a t), whose float bits are
// 0x4B000000 + rint(a t).
__device__ inline uint32_t q20_term(float a, float t) {
    return __builtin_bit_cast(uint32_t, __builtin_fmaf(a, t, 0x1p23f)) - 0x4B000000u;
}

// RN((float)s / N) * 2^-20 given N' = N * 2^20 and y' = RN(1/N) * 2^-20.
// With y = RN(1/N): q0 = RN(s * y) is within two ulps of s/N, r = s - q0 * N
// is then exact, and s/N is never a float midpoint for integer N, so
// RN(q0 + r * y) = RN(s / N).  Scaling y and q0 by 2^-20 and N by 2^20 is
// exact and commutes with the roundings (no result is subnormal).
__device__ inline float div_q20(uint32_t s, float n_scaled, float rcp_scaled) {
    const float a = (float)s;
    const float q0 = a * rcp_scaled;
    const float r = __builtin_fmaf(-q0, n_scaled, a);
    return __builtin_fmaf(r, rcp_scaled, q0);
}

struct AggArgs {
    const float* cost;         // staged: D x H x W raw costs
    const uint4* pixL;         // fused: packed pixels of both views: census lo,
    const uint4* pixR;         //   census hi, RGB, 8 L_min (one stage: 16-byte words,
                               //   H x W; two: planes, see PixPlanes)
    const float* tabA;         // fused: Eq. 1 tables
    const float* tabC;
    const float* alpha;
    const float* beta;
    AggRecords rec;            // padded per-pixel records of the reference view
    float* out;                // D x H rows of `pitch` columns (one stage: W)
    // two-slice kernel: store `out` in the paired layout (see paired_at)
    bool paired;
    int W, H, D, nstrips, ref, L1;
    int pitch;  // two-slice kernel: columns past W may hold anything
};

// Paired layout of a D-slice cost volume: for each pixel and pair of slices
// (2g, 2g + 1), slice 2g holds the bits of the smaller cost (the first on a
// tie; costs are >= 0, so bit 31 is free) with bit 31 set when that is slice
// 2g + 1's, and slice 2g + 1 holds the other cost.  A last slice without a
// partner (odd D) holds its cost as it is.  Winner-take-all then reads only
// the even slices.  paired_at returns the cost of slice s at pixel i.
__device__ inline float paired_at(const float* __restrict__ vol, int P, int D, int s, int i) {
    const int e = s & ~1;
    const uint32_t w = __builtin_bit_cast(uint32_t, vol[(size_t)e * P + i]);
    if (e + 1 >= D || (s & 1) == (int)(w >> 31))
        return __builtin_bit_cast(float, w & 0x7fffffffu);
    return vol[(size_t)(e + 1) * P + i];
}

// Loads of one chunk.  Step 1 loads are for this lane's four segment columns
// of its wavefront's row; step 2 loads are for the owned column and the
// chunk's four rows.
template <bool kFused>
struct ChunkIn {
    uint4 ref[kSeg];            // fused: reference pixel; staged: .x = raw cost bits
    uint4 par[kSeg];            // fused: partner pixel
    uint4 b2[kAggK];            // step 2: records b of rows yc + k
};

// Per-lane constants of a strip.
struct AggLane {
    uint32_t img[kSeg];   // byte offset of each segment column in an H x W row (packed
                          // pixels: x16; cost slice: x4), or kOOB
    uint32_t par[kSeg];   // fused: the partner column's byte offset, or kOOB
    uint32_t inval[kSeg]; // fused: raw cost when the partner is outside (2^20; 0 off-image)
    uint32_t reco;        // record column index x4 of the owned column
    uint32_t cb1;         // ring byte offset of the owned column
    uint32_t vout_o;      // output byte offset of the owned column, or kOOB
    bool pok[kSeg];       // fused: partner inside the image
};

struct AggRes {
    rsrc_t rB, rq, rIr, rIp, rOut;
};

template <bool kFused>
__device__ inline void load_chunk(const AggArgs& A, int yc, const AggLane& ln, const AggRes& R,
                                  ChunkIn<kFused>& in) {
    const int H = A.H;
    const uint32_t Wp = (uint32_t)A.rec.Wp, W = (uint32_t)A.W;
    const int w = wave_id();
    {   // step 1: row yc + w
        const int y = yc + w;
        const uint32_t yq = (uint32_t)min(y, H - 1);
#pragma unroll
        for (int j = 0; j < kSeg; ++j) {
            if (kFused) {
                in.ref[j] = ld128(R.rIr, ln.img[j], yq * W * 16);
                in.par[j] = ld128(R.rIp, ln.par[j], yq * W * 16);
            } else {
                in.ref[j].x = ld32(R.rq, ln.img[j], yq * W * 4);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {  // step 2: b row yc + k (rows past the last read zeros)
        const int y = yc + k;
        const uint32_t rb = (uint32_t)min(y, H + kLMax);
        in.b2[k] = ld128(R.rB, ln.reco * 4, rb * Wp * 16);
    }
}

template <bool kFused>
__device__ inline void process_chunk(const AggArgs& A, int yc, int y0, int y1, const AggLane& ln,
                                     const AggRes& R, const ChunkIn<kFused>& in,
                                     uint32_t& cp1, uint32_t& s1off, AggLds<kFused>& S) {
    const int t = threadIdx.x, w = wave_id(), lane = t & 63;
    const int H = A.H, W = A.W;
    uint32_t* prow_w = S.prow[w];
    // ---- step 1: raw costs and row prefixes of row yc + w ----
    {
        const int y = yc + w;
        uint32_t v[kSeg];
        if (y < H) {  // uniform: rows below the image contribute nothing
#pragma unroll
            for (int j = 0; j < kSeg; ++j) {
                if (kFused) {
                    const uint32_t s = __builtin_amdgcn_sad_u8(in.ref[j].z, in.par[j].z, 0u);
                    const uint64_t x = ((uint64_t)in.ref[j].y << 32 | in.ref[j].x) ^
                                       ((uint64_t)in.par[j].y << 32 | in.par[j].x);
                    const uint32_t h = (uint32_t)__popcll(x);
                    const float2 ab = *reinterpret_cast<const float2*>(
                        reinterpret_cast<const char*>(S.ab) + in.ref[j].w);
                    uint32_t q = q20_term(ab.x, S.tabA[s]) + q20_term(ab.y, S.tabC[h]);
                    // keep the lookups unconditional (interleaved across
                    // segments); the select is then one lane-mask cndmask
                    asm volatile("" : "+v"(q));
                    v[j] = ln.pok[j] ? q : ln.inval[j];
                } else {
                    v[j] = (uint32_t)(__builtin_bit_cast(float, in.ref[j].x) * 1048576.0f);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < kSeg; ++j) v[j] = 0u;
        }
        wave_scan_segments(v);
#pragma unroll
        for (int j = 0; j < kSeg; ++j) prow_w[64 * j + lane + 1] = v[j];
    }
    __syncthreads();
    // ---- step 2: column prefixes, means of rows yc + k - kLMax ----
    // Ring 1 keeps kAggK - 1 rows more than a range needs, so the chunk's
    // four pushes can all go before its four range reads.
    uint32_t e1[kAggK], s1[kAggK];
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        const uint32_t a = in.b2[k].z;
        const uint32_t pb = (uint32_t)(k * kPStride + t) * 4;
        e1[k] = lds_ld(S.prow[0], pb + (a & 0xff)) - lds_ld(S.prow[0], pb - ((a >> 8) & 0xff));
    }
    uint32_t off = s1off;
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        cp1 += e1[k];
        lds_st(S.ring1, ln.cb1 + off, cp1);
        off = off + kSlotBytes == kRing1 * kSlotBytes ? 0u : off + kSlotBytes;
    }
    s1off = off;
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        const uint32_t o = in.b2[k].y;
        s1[k] = lds_ld(S.ring1, ln.cb1 + (o & 0xffff)) - lds_ld(S.ring1, ln.cb1 + (o >> 16));
    }
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        const uint4 b = in.b2[k];
        const int yv = yc + k - kLMax;
        const float a1 = div_q20(s1[k], (float)(b.z >> 16) * 0x1p20f,
                                 __builtin_bit_cast(float, b.x));
        if (yv >= y0 && yv < y1) st32(a1, R.rOut, ln.vout_o, (uint32_t)(yv * W) * 4);
    }
    __syncthreads();
}

// Output rows [y0, y1) of slice d and column strip `strip` (256 threads).
template <bool kFused>
__device__ inline void agg_stream(const AggArgs& A, int d, int strip, int y0, int y1,
                                  AggLds<kFused>& S) {
    const int W = A.W, H = A.H;
    const int t = threadIdx.x, lane = t & 63;
    const int x0 = strip * kStripOut;
    const size_t slice = (size_t)W * H;

    if (kFused) {
        for (int i = t; i < 766; i += kStripThreads) S.tabA[i] = A.tabA[i];
        if (t < 65) S.tabC[t] = A.tabC[t];
        if (t <= kLMax) {
            const int L = min(t, A.L1);
            S.ab[t] = make_float2(A.alpha[L], A.beta[L]);
        }
    }
    if (t < kAggK) S.prow[t][0] = 0;  // P(-1) of every prefix row
    // zero column prefixes: rows before the start contribute nothing
    for (int i = t; i < kRing1 * kRingStride; i += kStripThreads) S.ring1[i] = 0;

    AggLane ln;
#pragma unroll
    for (int j = 0; j < kSeg; ++j) {
        const int i = 64 * j + lane;            // strip column of segment j
        const int c = x0 - 2 * kLMax + i;       // image column
        const bool in_img = c >= 0 && c < W;
        const int cp = A.ref == 0 ? c - d : c + d;
        const bool pok = in_img && cp >= 0 && cp < W;
        ln.img[j] = in_img ? (uint32_t)c * (kFused ? 16 : 4) : kOOB;
        ln.par[j] = pok ? (uint32_t)cp * 16 : kOOB;
        ln.pok[j] = pok;
        ln.inval[j] = in_img ? (1u << 20) : 0u;
    }
    {
        const int c = x0 - 2 * kLMax + t;
        const int jj = t - kLMax;
        const bool ring = jj >= 0 && jj < kRingCols;
        // owners without a ring column share one scratch column
        ln.cb1 = (uint32_t)(ring ? jj : kRingCols) * 4;
        ln.reco = (uint32_t)(c + kRecApronL) * 4;
        ln.vout_o = t >= 2 * kLMax && t < 2 * kLMax + kStripOut && c < W ? (uint32_t)c * 4 : kOOB;
    }
    const uint32_t P4 = (uint32_t)(slice * 4);
    const uint4* Iref = A.ref == 0 ? A.pixL : A.pixR;
    const uint4* Ipar = A.ref == 0 ? A.pixR : A.pixL;
    AggRes R;
    R.rB = make_rsrc(A.rec.b, (uint32_t)(A.rec.Wp * (H + kLMax + 1)) * 16);
    R.rq = make_rsrc(kFused ? (const void*)A.rec.b : (const void*)(A.cost + (size_t)d * slice),
                     kFused ? 0u : P4);
    R.rIr = make_rsrc(kFused ? (const void*)Iref : (const void*)A.rec.b, kFused ? 4 * P4 : 0u);
    R.rIp = make_rsrc(kFused ? (const void*)Ipar : (const void*)A.rec.b, kFused ? 4 * P4 : 0u);
    R.rOut = make_rsrc(A.out + (size_t)d * slice, P4);
    __syncthreads();

    // warm-up rows so that the first output row sees complete ranges
    const int warm = kLMax;
    const int ys = max(0, y0 - warm);
    const int yend = y1 + warm;
    uint32_t cp1 = 0;
    uint32_t s1off = ring_slot_bytes(ys, kRing1);
    ChunkIn<kFused> ca, cb;
    load_chunk<kFused>(A, ys, ln, R, ca);
    for (int yc = ys; yc < yend; yc += 2 * kAggK) {
        // the next chunk's loads are in flight while this chunk is processed
        load_chunk<kFused>(A, yc + kAggK, ln, R, cb);
        process_chunk<kFused>(A, yc, y0, y1, ln, R, ca, cp1, s1off, S);
        if (yc + kAggK >= yend) break;
        load_chunk<kFused>(A, yc + 2 * kAggK, ln, R, ca);
        process_chunk<kFused>(A, yc + kAggK, y0, y1, ln, R, cb, cp1, s1off, S);
    }
}

// ===========================================================================
// Two-slice streaming aggregation with specialised wavefronts (two stages)
// ===========================================================================
//
// One workgroup of 768 threads streams two adjacent disparity slices of one
// column strip down the rows, in chunks of kAggK rows, with each step done by
// a fixed set of wavefronts and three consecutive chunks in flight.  Phase p:
//   cost wavefronts 0-3 (wavefront w: row w of chunk p): the raw costs of
//       Eq. 1 of both slices and their row prefixes;
//   column wavefronts 4-7 (thread 256 + t owns ring column t), chunk p - 1,
//       row by row: stage-1 horizontal range sums from the prefix rows, the
//       vertical ones through ring 1, the stage-1 mean, the stage-2 vertical
//       range sums through ring 2;
//   output wavefronts 8-11 (wavefront w: row w of chunk p - 2): row prefixes
//       of those sums, the horizontal range sums, the final division, stores.
// One barrier ends a phase; a SIMD holds one wavefront of each kind.
//
// A strip is 256 input columns, kWsApron of them left of its kWsOut output
// columns.  A cost or output lane owns four consecutive columns, so a row
// prefix is three adds per lane and one wavefront scan of the lane totals,
// every per-pixel input is a 16-byte load of four columns from a plane, and a
// store is one 16-byte word; in a row of any length only the quad that the
// border cuts is stored as what is left of it (stored and, in the staged call,
// read as single words wherever W % 4 != 0, a frame of 1279 x 720, D = 128 took
// 0.865 ms, now 0.764, a staged one of 295 x 717, D = 41 0.312 and 0.255).  The
// apron is 36 rather than 2 kLMax = 34, and the strip 184 rather than 188, so that
// those quads are aligned to the image's.  The first and last strip have no apron
// at the image's border and take 20 columns more, so that narrower strips do not
// mean more of them (960 columns are five strips, not six: 960 x 540 with D = 96
// and two vote passes takes 0.445 ms instead of 0.491).  Every LDS word holds the
// two slices' values of one column (one 64-bit access serves both).
//  * Prefix rows are exclusive (entry i is the sum of the columns before i),
//    so a range sum over [x - l, x + r] is entry x + r + 1 minus entry x - l
//    and no entry is needed before the first column.
//  * Both rings are private to the column thread, which pushes a row and
//    reads that row's range before the next push, so 2 kLMax + 2 rows do.
//    Stream row r lies in slot r mod 36 of ring 1, and so does the a1 row
//    pushed with it, r - kLMax, in ring 2.
//  * The output wavefront works in place on its row of the stage-2 sums: it
//    takes four columns per lane as 16-byte words and writes the prefixes
//    back in four planes (column mod 4), in which the lanes' range reads are
//    consecutive.
//
// What bounds it: between two barriers a SIMD's three wavefronts share VALU
// and LDS (busy 65 % and 53 %), and the rings fill a CU's LDS, so there is no
// fourth.  Two kinds of wavefront on 512 threads, a column per lane and
// segment, took 0.829 ms for both views at 1280 x 720, D = 128; this form
// takes 0.579 ms (row prefixes without a pass through LDS, a third wavefront
// per SIMD, no 64-bit multiply in the mean, 16-byte stores).
struct AggLdsWs {
    float tabA[768];
    float tabC[68];
    float2 ab[kLMax + 1];
    alignas(16) uint2 x1[2][kAggK][kStripThreads];  // stage-1 row prefixes, by chunk parity
    alignas(16) uint2 e2[2][kAggK][4 * kWsPlane];   // stage-2 vertical sums, by chunk parity
    uint2 ring1[kWsRing * kWsCols];                 // [slot][column]
    uint2 ring2[kWsRing * kWsCols];
};
static_assert(sizeof(AggLdsWs) <= 160 * 1024, "one workgroup per CU");

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline uint2 lds_ld2(const void* base, uint32_t byte_off) {
    return *reinterpret_cast<const uint2*>(static_cast<const char*>(base) + byte_off);
}
__device__ inline void lds_st2(void* base, uint32_t byte_off, uint2 v) {
    *reinterpret_cast<uint2*>(static_cast<char*>(base) + byte_off) = v;
}
// A 16-byte buffer store reads its data registers late: a vector instruction
// right behind it that writes one of them changed the stored words on gfx950
// (the compiler expects this only of stores without a register offset).  The
// wait state that names the data keeps the registers until it has passed.
__device__ inline void st128(u32x4 v, rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, soff, 2);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 0" : : "v"(v));
    __builtin_amdgcn_sched_barrier(0);
}

__device__ inline void st96(u32x3 v, rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b96(v, r, voff, soff, 2);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 0" : : "v"(v));
    __builtin_amdgcn_sched_barrier(0);
}
__device__ inline void st64(u32x2 v, rsrc_t r, uint32_t voff, uint32_t soff) {
    __builtin_amdgcn_raw_buffer_store_b64(v, r, voff, soff, 2);
}

// What the wavefronts of a workgroup share: the item and its buffers.
struct WsItem {
    rsrc_t rB, rC, rRef, rPar, rCost, rOut;
    uint32_t Wq4, plane4, lm;      // pixel planes: bytes of a row and of a plane, L_min plane
    uint32_t slice_bytes;          // distance between the output slices
    uint32_t in_slice_bytes;       // ... and the cost volume's (0 when one slice is left)
    int nout;                      // slices that exist (the others are not stored)
    bool paired;                   // paired layout (see paired_at)
    bool quads;                    // W >= 4: a row of the volumes holds a quad
    bool cut;                      // W % 4 != 0, and the image's right border cuts a quad of
                                   // the strip's columns
    int tail;                      // columns that the strip stores of a quad the rows' end cuts
    int base, o0, o1;              // image columns of the strip's first, of its output range
    int ys, y0, y1, nch;           // first stream row (a multiple of 4), band, chunks
};

// Loads of a cost wavefront for one chunk.  Fused: the lane's four reference
// pixels and the five partner pixels of its columns in both slices; staged:
// the two slices' raw costs in ref[0] and ref[1].
struct WsCostIn {
    uint4 ref[3], par[3];   // census lo, census hi, RGB
    uint32_t lmin, par4[3];
};
struct WsColIn {
    uint4 b[kAggK];
};
struct WsOutIn {
    uint4 off, rcp, n;
};

struct WsCostLane {
    uint32_t vref, vlm, vpar;      // byte offsets of the lane's columns in a plane row
    uint32_t vq[4];                // staged: byte offsets in a cost row, or kOOB
    int shift;                     // staged: columns the lane's quad is read further left
    bool ok[kWsSlices][4];         // fused: partner inside the image
};

template <bool kFused>
__device__ inline void ws_cost_load(const WsItem& I, int H, int W, int p, int w,
                                    const WsCostLane& ln, WsCostIn& in) {
    const uint32_t y = (uint32_t)min(I.ys + kAggK * p + w, H - 1);
    if constexpr (kFused) {
        const uint32_t row = y * I.Wq4;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            in.ref[k] = ld128(I.rRef, ln.vref, row + k * I.plane4);
            in.par[k] = ld128(I.rPar, ln.vpar, row + k * I.plane4);
            in.par4[k] = ld32(I.rPar, ln.vpar + 16, row + k * I.plane4);
        }
        in.lmin = ld32(I.rRef, ln.vlm, I.lm + (row >> 2));
    } else {
        const uint32_t row = y * (uint32_t)W * 4;
#pragma unroll
        for (int s = 0; s < kWsSlices; ++s) {
            const uint32_t o = row + s * I.in_slice_bytes;
            if (I.quads)  // uniform
                in.ref[s] = ld128(I.rCost, ln.vq[0], o);
            else
                in.ref[s] = make_uint4(ld32(I.rCost, ln.vq[0], o), ld32(I.rCost, ln.vq[1], o),
                                       ld32(I.rCost, ln.vq[2], o), ld32(I.rCost, ln.vq[3], o));
        }
    }
}

// Exclusive prefixes across the wavefront of four columns per lane: v[s][i]
// becomes the sum of slice s over all columns before the lane's column i
// (mod 2^32; only differences are used).  One DPP scan of the lane totals:
// row shifts 1, 2, 4, 8 and row broadcasts 15 and 31.
__device__ inline void ws_scan(uint32_t (&v)[kWsSlices][4]) {
    uint32_t tot[kWsSlices], inc[kWsSlices];
#pragma unroll
    for (int s = 0; s < kWsSlices; ++s) {
        v[s][1] += v[s][0];
        v[s][2] += v[s][1];
        tot[s] = inc[s] = v[s][2] + v[s][3];
    }
#define DCO_WS_SCAN(CTRL, MASK) \
    _Pragma("unroll") for (int s = 0; s < kWsSlices; ++s) inc[s] += dpp<CTRL, MASK>(inc[s]);
    DCO_WS_SCAN(0x111, 0xf)
    DCO_WS_SCAN(0x112, 0xf)
    DCO_WS_SCAN(0x114, 0xf)
    DCO_WS_SCAN(0x118, 0xf)
    DCO_WS_SCAN(0x142, 0xa)
    DCO_WS_SCAN(0x143, 0xc)
#undef DCO_WS_SCAN
#pragma unroll
    for (int s = 0; s < kWsSlices; ++s) {
        const uint32_t before = inc[s] - tot[s];
        v[s][3] = before + v[s][2];
        v[s][2] = before + v[s][1];
        v[s][1] = before + v[s][0];
        v[s][0] = before;
    }
}

// Cost wavefront: raw costs and row prefixes of one row.  Rows below the
// image load row H - 1 and columns outside it whatever their address holds:
// prefixes are modular and every range of a stored output ends inside the
// image (arms stop at the border), so neither reaches a stored output.
template <bool kFused>
__device__ inline void ws_cost_phase(const WsItem& I, const WsCostLane& ln, const WsCostIn& in,
                                     uint2* row, AggLdsWs& S) {
    uint32_t q[kWsSlices][4];
    if constexpr (kFused) {
        const uint32_t rlo[4] = {in.ref[0].x, in.ref[0].y, in.ref[0].z, in.ref[0].w};
        const uint32_t rhi[4] = {in.ref[1].x, in.ref[1].y, in.ref[1].z, in.ref[1].w};
        const uint32_t rc[4] = {in.ref[2].x, in.ref[2].y, in.ref[2].z, in.ref[2].w};
        const uint32_t plo[5] = {in.par[0].x, in.par[0].y, in.par[0].z, in.par[0].w, in.par4[0]};
        const uint32_t phi[5] = {in.par[1].x, in.par[1].y, in.par[1].z, in.par[1].w, in.par4[1]};
        const uint32_t pc[5] = {in.par[2].x, in.par[2].y, in.par[2].z, in.par[2].w, in.par4[2]};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 ab = *reinterpret_cast<const float2*>(
                reinterpret_cast<const char*>(S.ab) + ((in.lmin >> 8 * j) & 0xff));
#pragma unroll
            for (int s = 0; s < kWsSlices; ++s) {
                const uint32_t sad = __builtin_amdgcn_sad_u8(rc[j], pc[j + s], 0u);
                const uint32_t h = (uint32_t)__popc(rlo[j] ^ plo[j + s]) +
                                   (uint32_t)__popc(rhi[j] ^ phi[j + s]);
                q[s][j] = q20_term(ab.x, S.tabA[sad]) + q20_term(ab.y, S.tabC[h]);
            }
        }
        // every lookup stays unconditional; the selects are lane-mask cndmasks
        asm volatile(""
                     : "+v"(q[0][0]), "+v"(q[0][1]), "+v"(q[0][2]), "+v"(q[0][3]), "+v"(q[1][0]),
                       "+v"(q[1][1]), "+v"(q[1][2]), "+v"(q[1][3]));
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < kWsSlices; ++s) q[s][j] = ln.ok[s][j] ? q[s][j] : 1u << 20;
    } else {
        // the volume holds q 2^-20 exactly (1.0 where the partner is outside)
#pragma unroll
        for (int s = 0; s < kWsSlices; ++s) {
            uint32_t c[4] = {in.ref[s].x, in.ref[s].y, in.ref[s].z, in.ref[s].w};
            if (I.cut && I.quads) {  // uniform
                const bool one = ln.shift & 1, two = ln.shift & 2;
                c[0] = one ? c[1] : c[0];
                c[1] = one ? c[2] : c[1];
                c[2] = one ? c[3] : c[2];
                c[0] = two ? c[2] : c[0];
                c[1] = two ? c[3] : c[1];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                q[s][j] = (uint32_t)(__builtin_bit_cast(float, c[j]) * 0x1p20f);
        }
    }
    ws_scan(q);
    const uint4 lo = make_uint4(q[0][0], q[1][0], q[0][1], q[1][1]);
    const uint4 hi = make_uint4(q[0][2], q[1][2], q[0][3], q[1][3]);
    uint2* dst = row + 4 * (threadIdx.x & 63);
    __builtin_memcpy(__builtin_assume_aligned(dst, 16), &lo, 16);
    __builtin_memcpy(__builtin_assume_aligned(dst + 2, 16), &hi, 16);
}

// Column thread: the b records of chunk q.
__device__ inline void ws_col_load(const WsItem& I, int H, uint32_t Wp16, int q, uint32_t vcol,
                                   WsColIn& in) {
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        const uint32_t r = (uint32_t)min(I.ys + kAggK * q + k, H + kWsRecRows - 1);
        in.b[k] = ld128(I.rB, vcol, r * Wp16);
    }
}

// floor((s + floor(n / 2)) / n) for 0 <= s <= n 2^20, 1 <= n <= 1225, given
// rcp = RN(1 / n) and neg_n = -n.  (float)s, rcp and the fused multiply-add
// round, together by less than 0.19 of a quotient of at most 2^20, so
// q = trunc(s / n + 0.25 -+ 0.19) is the result or one less; the remainder
// s - q n (24-bit multiply, 32-bit sum) decides: one more when it is at
// least ceil(n / 2).
__device__ inline uint32_t mean_q20(uint32_t s, float rcp, int neg_n, int half_up) {
    const uint32_t q = (uint32_t)__builtin_fmaf((float)s, rcp, 0.25f);
    const int r = (int)s + __mul24((int)q, neg_n);
    return q + (r >= half_up ? 1u : 0u);
}

// Column thread of ring column ct (byte offset cb in a ring row), one chunk:
// x = its entry of the chunk's first prefix row, e = its entry of the first
// output row, slot = the ring byte offset of the chunk's first row.
__device__ inline void ws_col_phase(const uint2* x, uint2* e, uint32_t cb, uint32_t slot,
                                    const WsColIn& in, uint32_t (&cp1)[kWsSlices],
                                    uint32_t (&cp2)[kWsSlices], AggLdsWs& S) {
    uint32_t e1[kWsSlices][kAggK], s1[kWsSlices][kAggK];
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        const uint32_t a = in.b[k].w;
        const uint2* xk = x + k * kStripThreads;
        const uint2 hi = lds_ld2(xk, a & 0xff);
        const uint2 lo = lds_ld2(xk, 0u - ((a >> 8) & 0xff));
        e1[0][k] = hi.x - lo.x;
        e1[1][k] = hi.y - lo.y;
    }
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {  // push a row, then read its range
        cp1[0] += e1[0][k];
        cp1[1] += e1[1][k];
        lds_st2(S.ring1, cb + slot + k * kWsSlotBytes, make_uint2(cp1[0], cp1[1]));
        const uint32_t o = in.b[k].y;
        const uint2 hi = lds_ld2(S.ring1, cb + (o & 0xffff));
        const uint2 lo = lds_ld2(S.ring1, cb + (o >> 16));
        s1[0][k] = hi.x - lo.x;
        s1[1][k] = hi.y - lo.y;
    }
#pragma unroll
    for (int k = 0; k < kAggK; ++k) {
        const float rcp = __builtin_bit_cast(float, in.b[k].x);
        const int neg_n = (int)in.b[k].w >> 16, half_up = (1 - neg_n) >> 1;
#pragma unroll
        for (int s = 0; s < kWsSlices; ++s) cp2[s] += mean_q20(s1[s][k], rcp, neg_n, half_up);
        lds_st2(S.ring2, cb + slot + k * kWsSlotBytes, make_uint2(cp2[0], cp2[1]));
        const uint32_t o = in.b[k].z;
        const uint2 hi = lds_ld2(S.ring2, cb + (o & 0xffff));
        const uint2 lo = lds_ld2(S.ring2, cb + (o >> 16));
        e[k * 4 * kWsPlane] = make_uint2(hi.x - lo.x, hi.y - lo.y);
    }
}

// Output wavefront: the c records of its row of chunk q.
__device__ inline int ws_out_row(const WsItem& I, int q, int w) {
    return I.ys + kAggK * q + w - 2 * kLMax;
}
__device__ inline void ws_out_load(const WsItem& I, int H, uint32_t Wp4, uint32_t cplane4, int q,
                                   int w, uint32_t vcol, WsOutIn& in) {
    const uint32_t row = (uint32_t)min(max(ws_out_row(I, q, w), 0), H - 1) * Wp4;
    in.off = ld128(I.rC, vcol, row);
    in.rcp = ld128(I.rC, vcol, row + cplane4);
    in.n = ld128(I.rC, vcol, row + 2 * cplane4);
}

// Output wavefront: its row's prefixes, horizontal range sums, division and
// stores.  Slot s of a lane's values is slice s for the right view and slice
// 1 - s for the left (kRef = 0), whose partners lie the other way.  Every call
// issues the same number of stores (the hardware drops those out of range):
// loads and stores complete in order, so with a fixed count the next chunk's
// records are waited for without waiting for this chunk's stores.
template <int kRef, bool kTail>
__device__ inline void ws_out_phase(const WsItem& I, int pitch, int y2, uint2* row,
                                    const uint32_t (&vout)[2], const WsOutIn& in) {
    const int lane = threadIdx.x & 63;
    uint32_t v[kWsSlices][4];
    {
        uint4 lo, hi;
        const uint2* src = row + 4 * min(lane, kWsLanes - 1);
        __builtin_memcpy(&lo, __builtin_assume_aligned(src, 16), 16);
        __builtin_memcpy(&hi, __builtin_assume_aligned(src + 2, 16), 16);
        v[0][0] = lo.x, v[1][0] = lo.y, v[0][1] = lo.z, v[1][1] = lo.w;
        v[0][2] = hi.x, v[1][2] = hi.y, v[0][3] = hi.z, v[1][3] = hi.w;
    }
    ws_scan(v);
    __builtin_amdgcn_wave_barrier();  // the row is this wavefront's own
    if (lane < kWsPlane) {  // the lane past the last: its first prefix is the sum of all
#pragma unroll
        for (int j = 0; j < 4; ++j) row[j * kWsPlane + lane] = make_uint2(v[0][j], v[1][j]);
    }
    __builtin_amdgcn_wave_barrier();
    const uint32_t off[4] = {in.off.x, in.off.y, in.off.z, in.off.w};
    const uint32_t rcp[4] = {in.rcp.x, in.rcp.y, in.rcp.z, in.rcp.w};
    const uint32_t n[4] = {in.n.x, in.n.y, in.n.z, in.n.w};
    uint32_t out[kWsSlices][4];
    const char* base = reinterpret_cast<const char*>(row) + 8 * lane - kWsOffBias;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint2 a = lds_ld2(base, off[j] & 0xffff), b = lds_ld2(base, off[j] >> 16);
        const float nf = __builtin_bit_cast(float, n[j]), rf = __builtin_bit_cast(float, rcp[j]);
        out[0][j] = __builtin_bit_cast(uint32_t, div_q20(a.x - b.x, nf, rf));
        out[1][j] = __builtin_bit_cast(uint32_t, div_q20(a.y - b.y, nf, rf));
    }
    constexpr int kLo = kRef == 0 ? 1 : 0, kHi = 1 - kLo;  // slots of slices d and d + 1
    if (I.paired && I.nout == kWsSlices) {                 // uniform: the pair's minimum first
        // div_q20 of an unsigned sum is never negative nor -0, so the bits
        // order like the values, and bit 31 of b1 - b0 is set exactly when
        // b1 < b0 (the second slice strictly smaller)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t b0 = out[kLo][j], b1 = out[kHi][j];
            out[kLo][j] = ((b1 - b0) & 0x80000000u) | min(b0, b1);
            out[kHi][j] = max(b0, b1);
        }
    }
    const bool live = y2 >= I.y0 && y2 < I.y1;  // uniform
    const uint32_t row4 = live ? (uint32_t)(y2 * pitch) * 4 : 0u;
#pragma unroll
    for (int k = 0; k < kWsSlices; ++k) {
        const uint32_t(&o)[4] = out[k ? kHi : kLo];
        const bool keep = live && k < I.nout;
        const uint32_t so = keep ? row4 + k * I.slice_bytes : 0u;
        st128(u32x4{o[0], o[1], o[2], o[3]}, I.rOut, keep ? vout[0] : kOOB, so);
        if constexpr (kTail) {
            if (I.tail == 1)  // uniform
                st32(__builtin_bit_cast(float, o[0]), I.rOut, keep ? vout[1] : kOOB, so);
            else if (I.tail == 2)
                st64(u32x2{o[0], o[1]}, I.rOut, keep ? vout[1] : kOOB, so);
            else
                st96(u32x3{o[0], o[1], o[2]}, I.rOut, keep ? vout[1] : kOOB, so);
        }
    }
}

// kTail: the output rows' end cuts the strip's last quad.
template <int kRef, bool kTail>
__device__ inline void ws_out_loop(const AggArgs& A, const WsItem& I, int w, AggLdsWs& S) {
    const int lane = threadIdx.x & 63, H = A.H;
    const uint32_t Wp4 = (uint32_t)A.rec.Wp * 4, cplane4 = Wp4 * (uint32_t)H;
    const int c = I.base + kWsI0 + 4 * lane;  // image column of the lane's first
    const uint32_t vcol = (uint32_t)(c + kRecApronL) * 4;
    // whole quads are stored as 16 bytes (rows of the volumes keep words aligned,
    // which is all a buffer store needs); the one that the rows' end cuts, as its
    // columns inside
    const bool out = c >= I.o0 && c < I.o1 && lane < kWsLanes, whole = c + 3 < I.o1;
    const uint32_t vout[2] = {out && whole ? (uint32_t)c * 4 : kOOB,
                              out && !whole ? (uint32_t)c * 4 : kOOB};
    // the first chunk, even, with an output row of the band: before it there
    // is nothing to do but keep the phases
    const int q0 = max(0, I.y0 + 2 * kLMax - I.ys) / kAggK & ~1;
    WsOutIn ia, ib;
    ws_out_load(I, H, Wp4, cplane4, q0, w, vcol, ia);
    for (int p = 0; p < q0 + 2; ++p) __syncthreads();  // phases without a chunk to finish
    for (int q = q0;; q += 2) {
        ws_out_load(I, H, Wp4, cplane4, q + 1, w, vcol, ib);
        ws_out_phase<kRef, kTail>(I, A.pitch, ws_out_row(I, q, w), S.e2[0][w], vout, ia);
        __syncthreads();
        if (q + 1 >= I.nch) break;
        ws_out_load(I, H, Wp4, cplane4, q + 2, w, vcol, ia);
        ws_out_phase<kRef, kTail>(I, A.pitch, ws_out_row(I, q + 1, w), S.e2[1][w], vout, ib);
        __syncthreads();
        if (q + 2 >= I.nch) break;
    }
}

// Output rows [y0, y1) of slices d and d + 1 and column strip `strip`
// (768 threads; two stages); slices at or past dend are computed but not
// stored.  kFused: the raw cost computed from the packed pixels; else read
// from the cost volume A.cost.
template <bool kFused = true>
__device__ inline void agg_stream_ws(const AggArgs& A, int d, int dend, int strip, int y0, int y1,
                                     AggLdsWs& S) {
    const int W = A.W, H = A.H;
    const int t = threadIdx.x, lane = t & 63;
    const int kind = __builtin_amdgcn_readfirstlane(t >> 8);  // 0 cost, 1 column, 2 output
    const int w = __builtin_amdgcn_readfirstlane((t >> 6) & 3);
    const size_t slice = (size_t)W * H;
    const uint32_t P4 = (uint32_t)(slice * 4);

    WsItem I;
    I.base = strip * kWsOut - kWsI0;
    I.o0 = strip == 0 ? 0 : I.base + kWsApron;
    I.o1 = strip == A.nstrips - 1 ? A.pitch : I.base + kWsApron + kWsOut;
    I.y0 = y0;
    I.y1 = y1;
    I.ys = max(0, y0 - 2 * kLMax) & ~3;  // warm-up rows so that every range is complete
    I.nch = (y1 + 2 * kLMax - I.ys + kAggK - 1) / kAggK;
    I.nout = min(kWsSlices, min(A.D, dend) - d);
    I.paired = A.paired;
    I.quads = W >= 4;
    I.cut = W % 4 != 0 && I.base + kStripThreads > W;
    I.tail = strip == A.nstrips - 1 ? A.pitch % 4 : 0;
    const PixPlanes px(W, H);
    const uint32_t pixbytes = px.bytes();
    I.Wq4 = px.Wq * 4;
    I.plane4 = px.plane * 4;
    I.lm = 3 * I.plane4;
    I.rB = make_rsrc(A.rec.b, (uint32_t)(A.rec.Wp * (H + kWsRecRows)) * 16);
    I.rC = make_rsrc(A.rec.c, (uint32_t)(A.rec.Wp * H) * 12);
    I.rRef = kFused ? make_rsrc(A.ref == 0 ? A.pixL : A.pixR, pixbytes) : I.rB;
    I.rPar = kFused ? make_rsrc(A.ref == 0 ? A.pixR : A.pixL, pixbytes) : I.rB;
    // raw costs of slices d and d + 1; past the last slice, slice d again
    I.rCost = kFused ? I.rB
                     : make_rsrc(A.cost + (size_t)d * slice,
                                 (uint32_t)min(kWsSlices, A.D - d) * P4);
    I.in_slice_bytes = A.D - d >= 2 ? P4 : 0u;
    I.slice_bytes = (uint32_t)A.pitch * H * 4;
    I.rOut = make_rsrc(A.out + (size_t)d * A.pitch * H, (uint32_t)I.nout * I.slice_bytes);

    if constexpr (kFused) {
        for (int i = t; i < 766; i += kWsThreads) S.tabA[i] = A.tabA[i];
        if (t < 65) S.tabC[t] = A.tabC[t];
        if (t <= kLMax) {
            const int L = min(t, A.L1);
            S.ab[t] = make_float2(A.alpha[L], A.beta[L]);
        }
    }
    // the prefix before the first stream row is zero; rings hold nothing else
    // that a stored output reads before it is written
    const uint32_t slot0 = (uint32_t)(I.ys % kWsRing);
    if (t < kWsCols) S.ring1[(slot0 + kWsRing - 1) % kWsRing * kWsCols + t] = make_uint2(0u, 0u);
    __syncthreads();

    if (kind == 0) {
        WsCostLane ln;
        const int c = I.base + 4 * lane;  // image column of the lane's first
        if constexpr (kFused) {
            const bool in_img = c >= 0 && c < px.Wq;
            ln.vref = (uint32_t)(kPixPad + (in_img ? c : 0)) * 4;
            ln.vlm = (uint32_t)(in_img ? c : 0);
            // partner columns b .. b + 4: slot s of column j takes b + j + s
            const int b = A.ref == 0 ? c - d - 1 : c + d;
            ln.vpar = (uint32_t)(b > -5 && b < W ? b + kPixPad : 0) * 4;
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int s = 0; s < kWsSlices; ++s)
                    ln.ok[s][j] = b + j + s >= 0 && b + j + s < W;
        } else {
            // the quad that the border cuts is read as the row's last four
            // columns and shifted (columns outside the image may hold anything:
            // they only shift prefixes whose differences nothing takes)
            ln.shift = I.cut && c < W && c + 4 > W ? c + 4 - W : 0;
            ln.vq[0] = c >= 0 && c < W ? (uint32_t)(I.quads ? c - ln.shift : c) * 4 : kOOB;
#pragma unroll
            for (int j = 1; j < 4; ++j)
                ln.vq[j] = c + j >= 0 && c + j < W ? (uint32_t)(c + j) * 4 : kOOB;
        }
        const int last = I.nch + 1;  // phases 0 .. nch + 1
        if constexpr (kFused) {
            WsCostIn ia, ib;
            ws_cost_load<kFused>(I, H, W, 0, w, ln, ia);
            for (int p = 0;; p += 2) {
                ws_cost_load<kFused>(I, H, W, p + 1, w, ln, ib);
                ws_cost_phase<kFused>(I, ln, ia, S.x1[0][w], S);
                __syncthreads();
                if (p + 1 > last) break;
                ws_cost_load<kFused>(I, H, W, p + 2, w, ln, ia);
                ws_cost_phase<kFused>(I, ln, ib, S.x1[1][w], S);
                __syncthreads();
                if (p + 2 > last) break;
            }
        } else {
            // the volume's rows come from memory, not from L2: three phases ahead
            // (1280 x 720, D = 128, one view: 0.451 ms with one, 0.427 with
            // three, 0.421 with five, which small frames lose again)
            constexpr int kAhead = 3;  // odd: a buffer keeps its phases' parity
            WsCostIn in[kAhead + 1];
#pragma unroll
            for (int k = 0; k < kAhead; ++k) ws_cost_load<kFused>(I, H, W, k, w, ln, in[k]);
            for (int p = 0;;) {
#pragma unroll
                for (int k = 0; k <= kAhead; ++k, ++p) {
                    ws_cost_load<kFused>(I, H, W, p + kAhead, w, ln,
                                         in[(k + kAhead) % (kAhead + 1)]);
                    ws_cost_phase<kFused>(I, ln, in[k], S.x1[k & 1][w], S);
                    __syncthreads();
                    if (p + 1 > last) return;
                }
            }
        }
    } else if (kind == 1) {
        __builtin_amdgcn_s_setprio(1);
        const int ct = t - kStripThreads;
        const bool owns = ct < kWsCols;
        const uint32_t cb = (uint32_t)ct * 8;
        const uint32_t vcol = (uint32_t)(I.base + kWsI0 + ct + kRecApronL) * 16;
        const uint32_t Wp16 = (uint32_t)A.rec.Wp * 16;
        uint32_t cp1[kWsSlices] = {0, 0}, cp2[kWsSlices] = {0, 0};
        uint32_t slot = slot0 * kWsSlotBytes;
        constexpr uint32_t kStep = kAggK * kWsSlotBytes, kTurn = kWsRing * kWsSlotBytes;
        WsColIn ja, jb;
        ws_col_load(I, H, Wp16, 0, vcol, ja);
        __syncthreads();  // phase 0: no chunk yet
        for (int q = 0;; q += 2) {
            ws_col_load(I, H, Wp16, q + 1, vcol, jb);
            if (owns)
                ws_col_phase(&S.x1[0][0][kWsI0 + ct], &S.e2[0][0][ct], cb, slot, ja, cp1, cp2, S);
            slot = slot + kStep == kTurn ? 0u : slot + kStep;
            __syncthreads();
            if (q + 1 >= I.nch) break;
            ws_col_load(I, H, Wp16, q + 2, vcol, ja);
            if (owns)
                ws_col_phase(&S.x1[1][0][kWsI0 + ct], &S.e2[1][0][ct], cb, slot, jb, cp1, cp2, S);
            slot = slot + kStep == kTurn ? 0u : slot + kStep;
            __syncthreads();
            if (q + 2 >= I.nch) break;
        }
        __syncthreads();  // the last phase: output wavefronts only
    } else {
        const bool right = !kFused || A.ref != 0;
        if (right && I.tail == 0)
            ws_out_loop<1, false>(A, I, w, S);
        else if (right)
            ws_out_loop<1, true>(A, I, w, S);
        else if (I.tail == 0)
            ws_out_loop<0, false>(A, I, w, S);
        else
            ws_out_loop<0, true>(A, I, w, S);
    }
}

// Work item of block b of n, remapped so that the blocks one XCD runs
// (round-robin block -> XCD dispatch) get consecutive items, which then
// share their inputs in that XCD's L2.
__device__ inline int xcd_work_item(int b, int n) {
    const int xcd = b & 7, i = b >> 3;
    const int per = n >> 3, rem = n & 7;
    return xcd < rem ? xcd * (per + 1) + i : rem * (per + 1) + (xcd - rem) * per + i;
}

// ===========================================================================
// Winner-take-all (Eq. 3) with parabola sub-pixel refinement; LR check
// ===========================================================================

// Parabola vertex offset through (d-1, m), (d, c), (d+1, pl), in this FP32
// order, clamped to [-0.5, 0.5]; 0 at the range ends or for den <= 0.
__device__ inline float subpixel_delta(float m, float c, float pl, int bd, int D) {
    float del = 0.f;
    if (bd > 0 && bd < D - 1) {
        const float num = m - pl;
        const float den = (m - c) + (pl - c);
        if (den > 0.f) {
            del = num / (2.0f * den);
            del = fminf(fmaxf(del, -0.5f), 0.5f);
        }
    }
    return del;
}


typedef float f32x4 __attribute__((ext_vector_type(4)));
// Four words at any 4-byte address, four int16 at any 2-byte address, four
// bytes at any: the hardware's vector accesses need no more.
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef int16_t i16x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint8_t u8x4u __attribute__((ext_vector_type(4), aligned(1)));

// WTA result of four consecutive pixels (del: the parabola's offset).
struct WtaQuad {
    int bd[4];
    float del[4];
};

// Words of pixels i .. i + 3 of the slice at p.  kNarrow: of pixels i .. i + n - 1,
// the last repeated (rows of n < 4 pixels).
template <bool kNarrow>
__device__ inline u32x4 wta_load(const uint32_t* p, int n) {
    if constexpr (kNarrow)
        return u32x4{p[0], p[min(1, n - 1)], p[min(2, n - 1)], p[n - 1]};
    else
        return __builtin_nontemporal_load(reinterpret_cast<const u32x4u*>(p));
}

// Stores of a quad's values (kNarrow: the first n of them).
template <bool kNarrow, typename V, typename T>
__device__ inline void wta_store(T* p, T a, T b, T c, T d, int n) {
    if constexpr (kNarrow) {
        p[0] = a;
        if (n > 1) p[1] = b;
        if (n > 2) p[2] = c;
    } else {
        *reinterpret_cast<V*>(p) = V{a, b, c, d};
    }
}

// Smallest d minimising agg, per pixel of the quad, with the values at d - 1 and
// d + 1 tracked on the fly (ties keep the smallest d).
__device__ inline void wta_quad_step(float v, int d, float& best, int& bd, float& m, float& pl,
                                     float& prev) {
    if (d == bd + 1) pl = v;
    if (v < best) {
        best = v;
        bd = d;
        m = prev;
    }
    prev = v;
}

// Four consecutive pixels from i on of a D-slice volume, with one 16-byte load
// per slice and eight slices in flight.
template <bool kSub, bool kNarrow>
__device__ inline __attribute__((always_inline)) WtaQuad wta_quad(
    const float* __restrict__ agg, int P, int D, int i, int n, int subpixel) {
    // each volume is read once: non-temporal loads keep it from evicting
    // reused data from the caches
    const uint32_t* __restrict__ a = reinterpret_cast<const uint32_t*>(agg) + i;
    const auto load = [&](int d) {
        return __builtin_bit_cast(f32x4, wta_load<kNarrow>(a + (size_t)d * P, n));
    };
    const f32x4 v0 = load(0);
    float best[4] = {v0.x, v0.y, v0.z, v0.w}, prev[4] = {v0.x, v0.y, v0.z, v0.w};
    float m[4] = {0.f, 0.f, 0.f, 0.f}, pl[4] = {0.f, 0.f, 0.f, 0.f};
    WtaQuad r{};
    const auto step = [&](const f32x4& v, int d) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            wta_quad_step(v[q], d, best[q], r.bd[q], m[q], pl[q], prev[q]);
    };
    constexpr int U = 8;
    int d = 1;
    for (; d + U <= D; d += U) {
        f32x4 v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = load(d + k);
#pragma unroll
        for (int k = 0; k < U; ++k) step(v[k], d + k);
    }
    if (d < D) {  // the last slices as one batch (640 x 480, D = 64: 29 -> 27 us)
        f32x4 v[U - 1];
#pragma unroll
        for (int k = 0; k < U - 1; ++k) v[k] = load(min(d + k, D - 1));
#pragma unroll
        for (int k = 0; k < U - 1; ++k)
            if (d + k < D) step(v[k], d + k);
    }
    if (kSub && subpixel) {
#pragma unroll
        for (int q = 0; q < 4; ++q) r.del[q] = subpixel_delta(m[q], best[q], pl[q], r.bd[q], D);
    }
    return r;
}

// Winner-take-all on a volume in the paired layout: the same rule and the
// same result as wta_quad, since each even slice holds the smaller cost of its
// pair (the first on a tie) and the pairs are visited in order with a strict
// comparison; only the G = ceil(D / 2) even slices are read.  The sub-pixel step
// needs the costs at d - 1 and d + 1, which is exactly where wta_quad's m and pl
// come from when 0 < d < D - 1 (the only
// case in which subpixel_delta uses them).
__device__ inline void wta_pair_step(uint32_t s, int g, float& best, int& bd) {
    const float v = __builtin_bit_cast(float, s & 0x7fffffffu);
    if (v < best) {
        best = v;
        bd = 2 * g + (int)(s >> 31);
    }
}

// Pair step that also keeps, for the left view's parabola, the word of the
// pair before the best one (prevw) and of the pair after it (nextw): the
// neighbour of the winner in an adjacent pair is then often that pair's
// minimum, already loaded.
__device__ inline void wta_pair_step_tr(uint32_t s, int g, float& best, int& bd, uint32_t& lastw,
                                        uint32_t& prevw, uint32_t& nextw, bool& pend) {
    const float v = __builtin_bit_cast(float, s & 0x7fffffffu);
    if (pend) {
        nextw = s;
        pend = false;
    }
    if (v < best) {
        best = v;
        bd = 2 * g + (int)(s >> 31);
        prevw = lastw;
        pend = true;
    }
    lastw = s;
}

// Parabola's offset, with the adjacent pairs' words from the scan: the winner's
// pair partner is that pair's maximum (the odd slice), and the neighbour in
// the adjacent pair is read only when it is not that pair's minimum.  The
// values are the same ones paired_at decodes.
__device__ inline float wta_pair_delta_tr(const float* __restrict__ vol, int P, int D, int i,
                                          float best, int bd, uint32_t prevw, uint32_t nextw) {
    if (bd <= 0 || bd >= D - 1) return 0.f;
    const int g = bd >> 1;
    const float partner = vol[(size_t)(2 * g + 1) * P + i];
    float m, pl;
    if ((bd & 1) == 0) {
        m = (prevw >> 31) ? __builtin_bit_cast(float, prevw & 0x7fffffffu)
                          : vol[(size_t)(2 * g - 1) * P + i];
        pl = partner;
    } else {
        m = partner;
        pl = (nextw >> 31) == 0u || 2 * g + 3 >= D ? __builtin_bit_cast(float, nextw & 0x7fffffffu)
                                                   : vol[(size_t)(2 * g + 3) * P + i];
    }
    return subpixel_delta(m, best, pl, bd, D);
}

// Four consecutive pixels from i on: one 16-byte load per even slice, 21 slices
// in flight.  kSub: the left view, with the parabola's offset.
template <bool kSub, bool kNarrow>
__device__ inline __attribute__((always_inline)) WtaQuad wta_pairs_quad(
    const float* __restrict__ vol, int P, int D, int i, int n, int subpixel) {
    const int G = (D + 1) / 2;
    const uint32_t* __restrict__ s = reinterpret_cast<const uint32_t*>(vol) + i;
    const size_t st = (size_t)P * 2;  // two slices
    const u32x4 w0 = wta_load<kNarrow>(s, n);
    WtaQuad r{};
    float best[4];
    uint32_t lastw[4], prevw[4] = {0u, 0u, 0u, 0u}, nextw[4] = {0u, 0u, 0u, 0u};
    bool pend[4] = {true, true, true, true};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        best[q] = __builtin_bit_cast(float, w0[q] & 0x7fffffffu);
        r.bd[q] = (int)(w0[q] >> 31);
        lastw[q] = w0[q];
    }
    const auto step = [&](const u32x4& v, int g) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (kSub)
                wta_pair_step_tr(v[q], g, best[q], r.bd[q], lastw[q], prevw[q], nextw[q], pend[q]);
            else
                wta_pair_step(v[q], g, best[q], r.bd[q]);
        }
    };
    constexpr int U = 21;  // 21 loads in flight per thread (three batches for D = 128)
    int g = 1;
    for (; g + U <= G; g += U) {
        u32x4 v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) v[k] = wta_load<kNarrow>(s + (size_t)(g + k) * st, n);
#pragma unroll
        for (int k = 0; k < U; ++k) step(v[k], g + k);
    }
    if (g < G) {  // the last groups as one batch (loads clamped to the last group)
        u32x4 v[U];
#pragma unroll
        for (int k = 0; k < U; ++k)
            v[k] = wta_load<kNarrow>(s + (size_t)min(g + k, G - 1) * st, n);
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (g + k < G) step(v[k], g + k);
    }
    if (kSub && subpixel) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            r.del[q] = wta_pair_delta_tr(vol, P, D, i + (kNarrow ? min(q, n - 1) : q), best[q],
                                         r.bd[q], prevw[q], nextw[q]);
    }
    return r;
}

// Either layout.  Inlined always: as a call its loads were flat ones and its registers
// spilled (1280 x 720, D = 128: 119 us instead of 85).
template <bool kPaired, bool kSub, bool kNarrow>
__device__ inline __attribute__((always_inline)) WtaQuad wta_any(
    const float* __restrict__ vol, int P, int D, int i, int n, int subpixel) {
    if constexpr (kPaired)
        return wta_pairs_quad<kSub, kNarrow>(vol, P, D, i, n, subpixel);
    else
        return wta_quad<kSub, kNarrow>(vol, P, D, i, n, subpixel);
}

template <bool kNarrow>
__device__ inline void put_bd(int16_t* p, const WtaQuad& r, int n) {
    wta_store<kNarrow, i16x4u>(p, (int16_t)r.bd[0], (int16_t)r.bd[1], (int16_t)r.bd[2],
                               (int16_t)r.bd[3], n);
}

// WTA of both views for a list of pixels: quad i of an image of P pixels (the
// last one moved back to end with the image; an image of less than four pixels
// is one narrow quad).
template <bool kPaired>
__device__ inline void wta_quad_both(const float* __restrict__ aggL,
                                     const float* __restrict__ aggR, int P, int D, int i4,
                                     int subpixel, int16_t* __restrict__ dL,
                                     float* __restrict__ deltaL, int16_t* __restrict__ dR) {
    const auto both = [&](auto narrow) {
        constexpr bool kN = decltype(narrow)::value;
        const int i = kN ? 0 : min(i4, P - 4);
        const WtaQuad l = wta_any<kPaired, true, kN>(aggL, P, D, i, P, subpixel);
        put_bd<kN>(dL + i, l, P);
        wta_store<kN, f32x4u>(deltaL + i, l.del[0], l.del[1], l.del[2], l.del[3], P);
        put_bd<kN>(dR + i, wta_any<kPaired, false, kN>(aggR, P, D, i, P, subpixel), P);
    };
    if (P >= 4)
        both(std::false_type{});
    else
        both(std::true_type{});
}

__device__ inline void lr_pixel(const int16_t* __restrict__ dL, const float* __restrict__ deltaL,
                                const int16_t* __restrict__ dR, int W, int x, int y, int maxdiff,
                                float* __restrict__ disp, uint8_t* __restrict__ valid) {
    const size_t i = (size_t)y * W + x;
    const int dl = dL[i];
    const int xr = x - dl;
    const bool ok = xr >= 0 && abs(dl - (int)dR[(size_t)y * W + xr]) <= maxdiff;
    valid[i] = ok ? 1 : 0;
    disp[i] = ok ? (float)dl + deltaL[i] : 0.0f;
}

}  // namespace dco
