// k_soft.hip -- differentiable soft-argmin form of the matcher (left view).
//
// Forward, per pair b, disparity d, pixel p (all float):
//   c(p,d)  = alpha_p (1 - exp(-(s/3)/lambda_AD)) + (1 - alpha_p)(1 - exp(-h/lambda_census))
//             (Eq. 1; c = 1 where the partner pixel x - d is outside the image)
//   E1 = row range sum of c       a1 = (column range sum of E1) / N1     (Eq. 2, stage 1)
//   E2 = column range sum of a1   A2 = (row range sum of E2) / N2         (Eq. 2, stage 2)
//   dhat = sum_d d softmax_d(-A2 / T),  lse = log sum_d exp(-A2 / T)
// The row sums are exact sums of fixed-point values on the matrix cores (a term is
// held to 2^-46 of the largest one that its wavefront has met in the row), the
// column sums differences of two FP64 prefix sums running down the column; each
// sum is then rounded once to FP32.  Every sum runs in a fixed order, so results
// are bit-reproducible.
//
// Backward, given g = dLoss/d dhat:
//   G_A2  = g w (dhat - d) / T,   dLoss/dT = sum g w (d - dhat) A2 / T^2
// then the adjoint of each range sum: an output that summed a range hands its
// adjoint back to every pixel of that range.  The row adjoints are exact products of
// fixed-point G with the transposed band (k_soft_wide); column adjoints are FP64
// difference arrays streamed down each column by one thread.  The last row adjoint is
// not stored: with E1 = H c, its values go in FP64 into
//   dLoss/dlambda_AD     = sum H^T G_E1 . alpha d(1 - exp(-(s/3)/lambda_AD))/dlambda_AD
//   dLoss/dlambda_census = sum H^T G_E1 . (1 - alpha) d(1 - exp(-h/lambda_census))/dlambda_census
// with fixed-order two-level reductions.  The only atomics are LDS adds that one
// thread makes to its own column in program order.
//
// Layout: volumes are B x D x H x pitch float in handle scratch; arms and the
// packed pixels (census, RGB, L_min) are per pair B x H x W.  The cost and row
// passes run one wavefront per image row and 16 disparities (k_soft_mrow,
// k_soft_wide); the column pass runs one thread per column, streaming down the
// rows with two rings of FP64 sums in LDS (k_soft_vv).
#include <algorithm>
#include <type_traits>

#include "dco_internal.h"

namespace {

struct SoftGeom {
    const uint32_t* arms;  // B x H x W packed arms of the left view
    const uint2* vrec;     // B x H x W column records (col_record, 1 / stage-1 region count)
    const float* n2;       // B x H x W stage-2 region counts
    int B, W, H, D;
    int pitch;             // columns of a volume's row
    __host__ __device__ size_t plane() const { return (size_t)pitch * H; }
};

__device__ inline int arm(uint32_t a, int k) { return (a >> (8 * k)) & 0xff; }

// Tables of Eq. 1 for the current theta, and their lambda derivatives:
// tab[0..765] = 1 - exp(-(s/3)/lambda_AD),   tab[768..1533] = d/dlambda_AD
// tab[1536..1600] = 1 - exp(-h/lambda_c),    tab[1664..1728] = d/dlambda_c
constexpr int kTabThreads = 1024;  // entry i of them, 0 <= i < kTabThreads

__device__ inline void table_entry(int i, const float* __restrict__ theta,
                                   float* __restrict__ tab) {
    const float la = theta[0], lc = theta[1];
    if (i < 766) {
        const float x = (float)i / 3.0f;
        const float e = expf(-x / la);
        tab[i] = -expm1f(-x / la);
        tab[768 + i] = -e * x / (la * la);
    } else if (i >= 768 && i < 768 + 65) {
        const int h = i - 768;
        const float e = expf(-(float)h / lc);
        tab[1536 + h] = -expm1f(-(float)h / lc);
        tab[1664 + h] = -e * (float)h / (lc * lc);
    }
}

// Column record of a pixel: dn in bits 9 .. 13 and kLMax - u in bits 4 .. 8
// (so that one mask and or give the LDS offset of a ring row, 512 bytes each),
// -N1 as a 16-bit float (exact: N1 <= (2 kLMax + 1)^2) in the high half.
__device__ inline uint32_t col_record(uint32_t a, int n1) {
    const _Float16 n = (_Float16)(-n1);
    return (uint32_t)arm(a, 3) << 9 | (uint32_t)(kLMax - arm(a, 2)) << 4 |
           (uint32_t)__builtin_bit_cast(uint16_t, n) << 16;
}

// Region pixel counts of the left view (as floats) for every pair: one
// block per 64 x 4 tile; the first blocks also make the tables (as a launch of
// its own 3 us of a 320 x 240 forward of 74).  The row lengths l + r + 1 of the
// tile's columns over kLMax rows above and below, and the column lengths u + dn
// + 1 of the tile's rows over kLMax columns left and right, go to LDS (0 outside
// the image, where no arm reaches); each count is then a sum of LDS entries.
constexpr int kCntTW = 64, kCntTH = 4;
__global__ __launch_bounds__(256) void k_soft_counts(SoftGeom g, const float* __restrict__ theta,
                                                     float* __restrict__ tab,
                                                     uint2* __restrict__ vrec,
                                                     float* __restrict__ n2) {
    constexpr int CH = kCntTH + 2 * kLMax, RW = kCntTW + 2 * kLMax;
    __shared__ uint8_t hl[CH][kCntTW];  // l + r + 1 down each tile column
    __shared__ uint8_t vl[kCntTH][RW];  // u + dn + 1 along each tile row
    const int t = threadIdx.x, b = blockIdx.z;
    const int x0 = blockIdx.x * kCntTW, y0 = blockIdx.y * kCntTH;
    {   // the tables, which only the later passes need: the first blocks' threads
        const unsigned n = gridDim.x * gridDim.y * gridDim.z;
        unsigned i = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        for (; i < kTabThreads / 256; i += n) table_entry((int)i * 256 + t, theta, tab);
    }
    const uint32_t* A = g.arms + (size_t)b * g.W * g.H;
    for (int k = t; k < CH * kCntTW; k += 256) {
        const int r = k / kCntTW, c = k - r * kCntTW;
        const int x = x0 + c, y = y0 - kLMax + r;
        const bool in = x < g.W && y >= 0 && y < g.H;
        const uint32_t q = in ? A[(size_t)y * g.W + x] : 0u;
        hl[r][c] = in ? (uint8_t)(arm(q, 0) + arm(q, 1) + 1) : 0;
    }
    for (int k = t; k < kCntTH * RW; k += 256) {
        const int r = k / RW, c = k - r * RW;
        const int x = x0 - kLMax + c, y = y0 + r;
        const bool in = x >= 0 && x < g.W && y < g.H;
        const uint32_t q = in ? A[(size_t)y * g.W + x] : 0u;
        vl[r][c] = in ? (uint8_t)(arm(q, 2) + arm(q, 3) + 1) : 0;
    }
    __syncthreads();
    const int tx = t & (kCntTW - 1), ty = t / kCntTW;
    const int x = x0 + tx, y = y0 + ty;
    if (x >= g.W || y >= g.H) return;
    const uint32_t a = A[(size_t)y * g.W + x];
    int s1 = 0, s2 = 0;
    for (int k = -arm(a, 2); k <= arm(a, 3); ++k) s1 += hl[ty + kLMax + k][tx];
    for (int k = -arm(a, 0); k <= arm(a, 1); ++k) s2 += vl[ty][tx + kLMax + k];
    const size_t i = (size_t)b * g.W * g.H + (size_t)y * g.W + x;
    vrec[i] = make_uint2(col_record(a, s1), __float_as_uint(1.0f / (float)s1));
    n2[i] = (float)s2;
}

struct SoftImg {
    const uint4* pixL;   // B x H x W packed pixels: census lo, census hi,
    const uint4* pixR;   //   RGB, 8 L_min
    const float* alpha;  // alpha_L, L = 0..kLMax
    const float* tab;    // table_entry's
};

// Workgroup index in the row order of workgroup b of n: the workgroups one
// XCD runs (round-robin dispatch, b mod 8) take a contiguous run, so the
// workgroups that share an image row share that XCD's L2.
__device__ inline int xcd_block(int b, int n) {
    const int xcd = b & 7, i = b >> 3;
    const int per = n >> 3, rem = n & 7;
    return xcd < rem ? xcd * (per + 1) + i : rem * (per + 1) + (xcd - rem) * per + i;
}

// Row sums of the costs on the matrix cores.
// Along one image row E1(x, d) = sum_p [x - l <= p <= x + r] c(p, d): a product
// of a banded 0/1 matrix, which the disparities share, with the costs.  The
// costs go in as fixed point q = c 2^k in two 24-bit halves, each of three signed
// bytes (balanced digits: q = sum_i 256^i b_i), so six i8 products with 32-bit
// accumulation give the exact sum of the q.  2^k puts the largest |c| that the
// wavefront has met in its row at 2^45: a cost is exact down to 2^-21 of that and
// within 2^-46 of it below.  (FP64 prefix sums along the row, 2^-53 of a sum of
// hundreds of them, keep as much; 30 bits of the largest cost that theta allows
// lost up to 5e-3 of costs far below it.)  Where a block raises the scale, its
// outputs add the block before in the old one: two products apart.  Costs of
// partners outside the image are 1 by definition: they enter as 0 and are counted.
// A cost that is not finite makes the outputs from its block on NaN.
//
// A workgroup takes one image row (or one of `segs` parts of it), a wavefront
// 16 of its disparities (those past 64 are other workgroups'), and they walk
// the row together in blocks of 64 columns:
//   - bands: the 0/1 operand of the block, which all the row's wavefronts use,
//     each building its share: a lane's 16 columns are the bits of one
//     interval, spread to bytes;
//   - costs: lane = column, 16 disparities in turn, so a reference pixel is
//     read once per block, and the partners are 80 consecutive pixels, in LDS;
//   - the lanes' q go through LDS (16 x 68 words, conflict-free both ways), a half
//     at a time, into the operand layout: lane = (disparity lane & 15, columns 16
//     (lane >> 4) .. + 15), a byte per column;
//   - after block [X, X + 64) the 16-column outputs at X - 32, X - 16, X and
//     X + 16 have all their columns (x - 17 .. x + 32) in this block and the one
//     before, whose digits stay in registers: two products per digit and output;
//   - E1 goes back through LDS to be stored as 256 contiguous bytes per
//     disparity (64-byte pieces of 16 planes: 0.35 ms instead of 0.30 then).
//
// Measured at 8 pairs of 640 x 480, D = 64: 0.28 ms (writes 0.63 GB, past the caches;
// bound by vector issue).  As FP64 prefix sums per row and disparity, two table
// passes, four LDS scans and eight gathers per 256 columns, 0.35.  In 32-bit fixed
// point (four digits) 0.22.  Steps there: 32 or 64 disparities per wavefront 0.35 and
// 0.44 ms (too few wavefronts), 16 with its own bands 0.32, rows stored whole 0.30,
// partners in LDS and a block ahead 0.25.  The lower half taken to digits before the
// barrier, the halves' products one after the other and the last partners of a block
// kept in LDS: 124 registers; without, 0.30 and more to spilling.
constexpr int kMxWaves = 4;          // most wavefronts per workgroup
constexpr int kMxSimds = 4 * 256;    // SIMDs of the device
constexpr int kMxStride = 68;        // words per disparity of the stage
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4), may_alias));
typedef uint32_t v4u __attribute__((ext_vector_type(4), may_alias));

// Bytes 0 / 1 of the columns pb .. pb + 15 that lie in [lo, hi).
__device__ inline v4i band_bytes(int lo, int hi, int pb) {
    const int a = min(max(lo - pb, 0), 16), e = min(max(hi - pb, 0), 16);
    const uint32_t bits = (1u << e) - (1u << a);
    v4i r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        r[i] = (int)((bits >> (4 * i) & 15u) * 0x00204081u & 0x01010101u);
    return r;
}

// Tables of the colour and census terms in LDS.
constexpr int kCenTab = 766;
__device__ inline void put_tables(const float* colour, const float* census, float* tab) {
    for (int i = threadIdx.x; i < kCenTab; i += blockDim.x) tab[i] = colour[i];
    for (int i = threadIdx.x; i < 65; i += blockDim.x) tab[kCenTab + i] = census[i];
    __syncthreads();
}

// The lane's 16 columns of disparity lane & 15, as digit planes.
__device__ inline void digit_planes3(const uint32_t* stage, v4i (&b)[3]) {
    const int lane = threadIdx.x & 63;
    const uint32_t* s = stage + (lane & 15) * kMxStride + 16 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const v4u w = *reinterpret_cast<const v4u*>(s + 4 * i);
        const uint32_t t0 = __builtin_amdgcn_perm(w.y, w.x, 0x05010400u);
        const uint32_t t1 = __builtin_amdgcn_perm(w.w, w.z, 0x05010400u);
        const uint32_t t2 = __builtin_amdgcn_perm(w.y, w.x, 0x0c0c0602u);
        const uint32_t t3 = __builtin_amdgcn_perm(w.w, w.z, 0x06020c0cu);
        b[0][i] = (int)__builtin_amdgcn_perm(t1, t0, 0x05040100u);
        b[1][i] = (int)__builtin_amdgcn_perm(t1, t0, 0x07060302u);
        b[2][i] = (int)(t2 | t3);
    }
}

// A wavefront's fixed point: |v| <= 2^ex for every value it has met in its row.
struct WideScale {
    int ex = -100;
    bool bad = false;  // a value was not finite
};

// Largest of the wavefront's values (DPP row shifts, then the row broadcasts).
template <unsigned Ctrl, unsigned RowMask>
__device__ inline uint32_t dpp_max(uint32_t m) {
    return max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, Ctrl, RowMask, 0xf, false));
}
__device__ inline uint32_t wave_max(uint32_t m) {
    m = dpp_max<0x111, 0xf>(m);
    m = dpp_max<0x112, 0xf>(m);
    m = dpp_max<0x114, 0xf>(m);
    m = dpp_max<0x118, 0xf>(m);
    m = dpp_max<0x142, 0xa>(m);
    m = dpp_max<0x143, 0xc>(m);
    return (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
}

// A lane's values of 16 disparities as q = v 2^(45 - ex) in two halves of three
// balanced digits, with ex raised to the largest of the wavefront's values: the
// upper halves go to the stage, the lower ones to `lo`.
__device__ inline void put_wide(const float (&v)[16], uint32_t* stage, uint32_t (&lo)[16],
                                WideScale& s) {
    const int lane = threadIdx.x & 63;
    uint32_t m = 0;  // bits of the largest |v| (a NaN's are larger still)
#pragma unroll
    for (int j = 0; j < 16; ++j) m = max(m, __float_as_uint(v[j]) & 0x7fffffffu);
    m = wave_max(m);
    s.bad = s.bad || m >= 0x7f800000u;
    s.ex = max(s.ex, (int)(m >> 23) - 126);
    const float up = ldexpf(1.0f, 22 - s.ex);
    // x + kMagic rounds |x| <= 2^22 to a whole number, the sum's low bits
    constexpr float kMagic = 0x1.8p23f;
    constexpr uint32_t kDigits = 0x8080u - 0x4b400000u;  // kMagic's bits, and balanced digits
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const float h = __builtin_fmaf(v[j], up, kMagic);
        const float r = __builtin_fmaf(v[j], up, kMagic - h);  // exact
        stage[j * kMxStride + lane] = (__float_as_uint(h) + kDigits) ^ 0x8080u;
        lo[j] = (__float_as_uint(__builtin_fmaf(r, 0x1p23f, kMagic)) + kDigits) ^ 0x8080u;
    }
    __builtin_amdgcn_wave_barrier();
}

// The digits of both halves as operands.
__device__ inline void wide_planes(uint32_t* stage, const uint32_t (&lo)[16], v4i (&b)[2][3]) {
    const int lane = threadIdx.x & 63;
    digit_planes3(stage, b[0]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 16; ++j) stage[j * kMxStride + lane] = lo[j];
    __builtin_amdgcn_wave_barrier();
    digit_planes3(stage, b[1]);
    __builtin_amdgcn_wave_barrier();
}

// The four 16-column outputs of block X over the block before (digits bp, scale
// 2^ex_old) and this one (bc): sink(i, xb, v) gets the lane's four sums of output
// i, columns xb + 4 (lane >> 4) .. + 3 of disparity lane & 15.  band(c): operand c
// of the block's eight.  Where the block raised the scale, the two products are
// taken apart.
template <typename Band, typename Sink>
__device__ inline void wide_outputs(int X, int W, const v4i (&bp)[2][3], const v4i (&bc)[2][3],
                                    int ex_old, const WideScale& sc, Band band, Sink sink) {
    const double inv = sc.bad ? __builtin_nan("") : ldexp(1.0, sc.ex - 45);
    // a half's sums from its digits'
    const auto whole = [](const v4i (&s)[3], int r) {
        return s[0][r] + ((s[1][r] + (s[2][r] << 8)) << 8);
    };
    const auto outputs = [&](auto rescaled) {
        constexpr bool kTwo = decltype(rescaled)::value;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int xb = X - 32 + 16 * i;
            if (xb < 0 || xb >= W) continue;
            const v4i b0 = band(2 * i), b1 = band(2 * i + 1);
            int q[2][4], old[2][4];  // of both blocks together, or of each
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                v4i s[3];
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    s[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b0, bp[h][k], v4i{0, 0, 0, 0}, 0,
                                                                 0, 0);
                if (kTwo) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) old[h][r] = whole(s, r);
#pragma unroll
                    for (int k = 0; k < 3; ++k) s[k] = v4i{0, 0, 0, 0};
                }
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    s[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b1, bc[h][k], s[k], 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) q[h][r] = whole(s, r);
            }
            double v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = __builtin_fma((double)q[0][r], 0x1p23, (double)q[1][r]) * inv;
                if (kTwo)
                    v[r] = __builtin_fma(
                        __builtin_fma((double)old[0][r], 0x1p23, (double)old[1][r]),
                        ldexp(1.0, ex_old - 45), v[r]);
            }
            sink(i, xb, v);
        }
    };
    if (sc.ex == ex_old)
        outputs(std::false_type{});
    else
        outputs(std::true_type{});
}

// What a wavefront of a row pass works on.  kShare: the workgroup's wavefronts take
// one row and its groups of 16 disparities in turns, and share the bands.  Else
// (one or two groups, where the shared buffers would leave a CU few wavefronts):
// the workgroup takes as many rows as it has wavefronts for, and each builds its
// own.  A forward and backward of two pairs of 600 x 400, D = 16 takes 259 us so
// and 404 shared, of eight of 400 x 300, D = 17 538 and 680; at three groups
// shared is as fast (five pairs of 90 x 300, D = 40: 264).
struct RowTask {
    int row, grp;
    bool on;
};
template <bool kShare>
__device__ inline RowTask row_task(int block, int rows, int ng, int w, int nw) {
    if constexpr (kShare) return RowTask{block, w, true};
    const int row = block * (nw / ng) + w / ng;
    return RowTask{min(row, rows - 1), w % ng, row < rows};
}

// How a volume's rows are stored.  Rows are whole 64-byte pieces (soft_pitch) and
// their columns past the image's hold nothing; kPast: past the caches, which a large
// volume only passes through (soft_stream).  kCut: rows of W columns, for volumes that
// do not fit the card with more: the quad that a row's end cuts is stored as words.
enum Rows { kWhole, kPast, kCut };

// Stores the stage's 16 x 64 outputs: disparities d0 .. d0 + 15, columns x0 ..
// x0 + 63, those inside the volume (rows of W columns) only; `out` is row y of
// disparity 0, P a plane.  256 contiguous bytes per disparity, and four disparities
// per store.
template <Rows kRows>
__device__ inline void put_rows(const uint32_t* stage, float* __restrict__ out, size_t P, int d0,
                                int D, int x0, int W) {
    typedef float v4fu __attribute__((ext_vector_type(4), aligned(4), may_alias));
    const int lane = threadIdx.x & 63;
    const int c = 4 * (lane & 15), x = x0 + c;
    asm volatile("" : "+s"(P));  // the row addresses are made here, not kept over the row
    v4f o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        o[j] = *reinterpret_cast<const v4f*>(stage + (4 * j + (lane >> 4)) * kMxStride + c);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int d = d0 + 4 * j + (lane >> 4);
        if (x < 0 || x >= W || d >= D) continue;
        float* const q = out + d * P + x;
        if constexpr (kRows == kPast) {
            __builtin_nontemporal_store(o[j], reinterpret_cast<v4f*>(q));
        } else if constexpr (kRows == kWhole) {
            *reinterpret_cast<v4f*>(q) = o[j];
        } else if (x + 4 <= W) {
            *reinterpret_cast<v4fu*>(q) = o[j];
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (x + k < W) q[k] = o[j][k];
        }
    }
}

template <bool kShare, Rows kRows>
__global__ __launch_bounds__(64 * kMxWaves, 4) void k_soft_mrow(SoftGeom g, SoftImg im,
                                                                float* __restrict__ out,
                                                                int seg_its) {
    __shared__ v4i bands[kShare ? 2 : 1][kShare ? 8 : 1][64];
    __shared__ __align__(16) uint32_t stages[kMxWaves][16 * kMxStride];
    __shared__ uint2 cen[kMxWaves][80];
    __shared__ uint32_t rgb[kMxWaves][80];
    __shared__ float tab[kCenTab + 65];
    const int nt = blockDim.x, nw = nt >> 6;
    put_tables(im.tab, im.tab + 1536, tab);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 15, kg = lane >> 4;
    const int W = g.W, D = g.D, ng = (D + 15) >> 4;
    // the workgroups of one image row on one XCD: its pixels are the shared input
    const RowTask rt = row_task<kShare>(xcd_block(blockIdx.x, gridDim.x), g.B * g.H, ng, w, nw);
    const int row = rt.row, y = row % g.H, b = row / g.H;
    const int it0 = blockIdx.y * seg_its, it1 = min(it0 + seg_its, (W + 95) >> 6);
    const size_t P = (size_t)W * g.H, pix = (size_t)b * P + (size_t)y * W;
    const uint4* pl = im.pixL + pix;
    const uint4* pr = im.pixR + pix;
    const uint32_t* ar = g.arms + pix;
    const size_t Q = g.plane(), vol = (size_t)b * D * Q + (size_t)y * g.pitch;
    uint32_t* stage = stages[w];
    int par = 0;
    const int grp = (kShare ? (int)blockIdx.z * nw : 0) + rt.grp, d0 = 16 * grp, d = d0 + n;
    const bool active = rt.on && grp < ng;
    v4i bp[2][3];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 3; ++k) bp[h][k] = v4i{0, 0, 0, 0};
    WideScale sc;
    // Partners of a block's 16 disparities: the 64 pixels from column X - d0 on
    // and the last 16 of the 64 before, through LDS (entry 16 + lane - j holds
    // column X + lane - (d0 + j)).  They and the reference pixels are loaded a
    // block ahead.
    const auto pixel = [&](int x) {
        const uint4* q = pr + min(max(x - d0, 0), W - 1);
        return uint3{q->x, q->y, q->z};
    };
    uint3 rc{};
    uint4 pn{};
    if (active) {
        const int X = 64 * max(it0 - 1, 0);
        if (lane < 16) {
            const uint3 r = pixel(X - 16 + lane);
            cen[w][64 + lane] = uint2{r.x, r.y};
            rgb[w][64 + lane] = r.z;
        }
        rc = pixel(X + lane);
        pn = pl[min(X + lane, W - 1)];
    }
    // the block before a segment's first only gives its digits
    for (int it = max(it0 - 1, 0); it < it1; ++it, par ^= 1) {
        const int X = it << 6;
        // bands of the four 16-column outputs over the block before and this one
        const auto band = [&](int c) {
            const int x = X - 32 + 16 * (c >> 1) + n;
            const uint32_t a = ar[min(max(x, 0), W - 1)];
            return band_bytes(x - arm(a, 0), x + arm(a, 1) + 1,
                              X - 64 + 64 * (c & 1) + 16 * kg);
        };
        if constexpr (kShare)
            for (int c = w; c < 8; c += nw) bands[par][c][lane] = band(c);
        v4i bc[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < 3; ++k) bc[h][k] = v4i{0, 0, 0, 0};
        const int ex_old = sc.ex;
        if (active && X < W) {
            if (lane < 16) {  // the last 16 of the block before
                cen[w][lane] = cen[w][64 + lane];
                rgb[w][lane] = rgb[w][64 + lane];
            }
            __builtin_amdgcn_wave_barrier();
            cen[w][16 + lane] = uint2{rc.x, rc.y};
            rgb[w][16 + lane] = rc.z;
            const uint4 pa = pn;
            rc = pixel(X + 64 + lane);
            pn = pl[min(X + 64 + lane, W - 1)];
            __builtin_amdgcn_wave_barrier();
            const float al = im.alpha[pa.w >> 3], be = 1.0f - al;
            const bool in_row = X + lane < W;
            float v[16];
            const auto costs = [&](auto all_in) {
                constexpr bool kIn = decltype(all_in)::value;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const uint2 cb = cen[w][16 + lane - j];
                    const uint32_t s = __builtin_amdgcn_sad_u8(pa.z, rgb[w][16 + lane - j], 0u);
                    const int hm = __popc(pa.x ^ cb.x) + __popc(pa.y ^ cb.y);
                    const float c = al * tab[s] + be * tab[kCenTab + hm];
                    v[j] = kIn || (in_row && X + lane - d0 - j >= 0) ? c : 0.0f;
                }
            };
            if (X >= d0 + 15 && X + 64 <= W)  // every column and partner is in the image
                costs(std::true_type{});
            else
                costs(std::false_type{});
            uint32_t lo[16];
            put_wide(v, stage, lo, sc);
            wide_planes(stage, lo, bc);
        }
        // the bands; the buffer's next writers pass the next one first
        if (kShare) __syncthreads();
        if (!active) continue;
        if (it >= it0) {
            const auto bands_of = [&](int c) { return kShare ? bands[par][c][lane] : band(c); };
            wide_outputs(X, W, bp, bc, ex_old, sc, bands_of, [&](int i, int xb, double(&v)[4]) {
                if (xb - kLMax < d0 + 15) {  // ranges may hold columns left of d: c = 1
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int x = xb + 4 * kg + r;
                        const uint32_t a = ar[min(x, W - 1)];
                        const int len = arm(a, 0) + arm(a, 1) + 1;
                        v[r] += (double)min(max(d - (x - arm(a, 0)), 0), len);
                    }
                }
                // to the stage (free since the digits), one row per d
                *reinterpret_cast<v4f*>(stage + n * kMxStride + 16 * i + 4 * kg) =
                    v4f{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
            });
            __builtin_amdgcn_wave_barrier();
            put_rows<kRows>(stage, out + vol, Q, d0, D, X - 32, g.pitch);
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < 3; ++k) bp[h][k] = bc[h][k];
    }
}

// e^x as 2^(x log2 e) on the hardware base-2 exponential (about 1 ulp); the
// rounding of the product adds a relative error of about |x| 2^-24.
__device__ inline float exp_e(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }

// Row sums of a volume, as k_soft_mrow makes those of the costs: on the same blocks,
// in the same fixed point of the value G.
//
// kMean: A2(x, d) = (sum of E2 over [x - l, x + r]) / N2(x), and, where the
// workgroup's wavefronts hold all disparities (dhat given, D <= 64), the soft
// argmin: each wavefront's 16 disparities give a maximum and two sums per column,
// merged one block later.
//
// kSeed: the seed and the transposed sums.  Per pixel and disparity, with
// w = softmax weight and g = dLoss/d dhat:
//   G(x, d) = G_A2 / N2 = g w (dhat - d) / (T N2),
//   dLoss/dT term = g w (d - dhat) A2 / T^2;
// out(p, d) = sum_x [x - l(x) <= p <= x + r(x)] G(x, d), the adjoint of A2's row
// range sums (G_E2): the transposed band.  The band's bytes of a lane's 16 pixels x
// come four at a time: with e = x - p, l - e and r + e are not negative, tested in
// bit 7 of biased bytes.  The temperature terms of the wavefront's row and
// disparities are summed into one FP64 value.
//
// kDot: the same adjoint of E1's row range sums, of G = G_E1, whose outputs are not
// stored: each goes in FP64 into the sums of its product with the two FP32
// derivatives of Eq. 1, looked up for the output's pixels and partners, which lie on
// the stage once the digits have left it.  (The other way round, row sums of the two
// derivatives dotted with G, takes two fixed points instead of one: 0.63 ms with
// these digits, 0.35 with 30 bits of the derivatives' bound, which left nothing of
// those far below it; 0.58 as FP64 prefix sums.)
//
// 8 pairs of 640 x 480, D = 64: 0.35, 0.33 and 0.37 ms, bound by vector issue (0.63
// GB read by each, and written by the first two).
// A G that is not finite makes the outputs from its block on NaN.
__device__ inline v4i band_bytes_t(const uint32_t* lp, const uint32_t* r, int e) {
    const v4u l4 = *reinterpret_cast<const v4u*>(lp), r4 = *reinterpret_cast<const v4u*>(r);
    uint32_t e4 = (uint32_t)(e + 128) * 0x01010101u + 0x03020100u;  // e + 128 + byte
    v4i o;
#pragma unroll
    for (int i = 0; i < 4; ++i, e4 += 0x04040404u) {
        const uint32_t a = l4[i] + ~e4;  // (l + 1) + 255 - (e + 128) = l - e + 128
        const uint32_t b = r4[i] + e4;   // r + e + 128
        o[i] = (int)((a & b & 0x80808080u) >> 7);
    }
    return o;
}

enum WideKind { kMean, kSeed, kDot };

template <WideKind kKind, bool kShare, Rows kRows>
__global__ __launch_bounds__(64 * kMxWaves, 4) void k_soft_wide(
    SoftGeom g, SoftImg im, const float* __restrict__ in, const float* __restrict__ theta,
    float* __restrict__ dhat, float* __restrict__ lse, const float* __restrict__ gdhat,
    float* __restrict__ out, double* __restrict__ part, int seg_its) {
    constexpr bool kAdj = kKind != kMean;  // transposed bands
    __shared__ v4i bands[kShare ? 2 : 1][kShare ? 8 : 1][64];
    __shared__ __align__(16) uint32_t stages[kMxWaves][16 * kMxStride];
    // adjoint: l + 1 and r of the columns of this block and the one before, a byte each
    __shared__ __align__(16) uint32_t arml[kAdj ? kMxWaves : 1][2][16],
        armr[kAdj ? kMxWaves : 1][2][16];
    // kMean: the wavefronts' softmax sums of a block's columns
    __shared__ float soft[2][kAdj ? 1 : kMxWaves][3][64];
    // kDot: the derivatives' tables
    __shared__ float tab[kKind == kDot ? kCenTab + 65 : 1];
    if constexpr (kKind == kDot) put_tables(im.tab + 768, im.tab + 1664, tab);
    const int nt = blockDim.x, nw = nt >> 6;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = lane & 15, kg = lane >> 4;
    const int W = g.W, D = g.D, ng = (D + 15) >> 4;
    const RowTask rt = row_task<kShare>(blockIdx.x, g.B * g.H, ng, w, nw);
    const int row = rt.row, y = row % g.H, b = row / g.H;
    const int it0 = blockIdx.y * seg_its, it1 = min(it0 + seg_its, (W + 95) >> 6);
    const size_t P = (size_t)W * g.H, pix = (size_t)b * P + (size_t)y * W;
    const size_t Q = g.plane(), vol = (size_t)b * D * Q + (size_t)y * g.pitch;
    const float T = theta[2], invT = 1.0f / T;
    uint32_t* stage = stages[w];
    int par = 0;
    const int grp = (kShare ? (int)blockIdx.z * nw : 0) + rt.grp, d0 = 16 * grp;
    const bool active = rt.on && grp < ng;
    v4i bp[2][3];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 3; ++k) bp[h][k] = v4i{0, 0, 0, 0};
    double acc = 0.0, acc2 = 0.0;
    WideScale sc;
    // the block before a segment's first only gives its digits
    const auto merge = [&](int it, int buf) {
        // dhat and lse of block it's columns from the wavefronts' sums
        const int x = (it << 6) - 32 + lane;
        float m = -INFINITY, z = 0.0f, zd = 0.0f;
        const auto* r = soft[buf] + (w - rt.grp);  // the row's wavefronts
        for (int k = 0; k < ng; ++k) m = fmaxf(m, r[k][0][lane]);
        for (int k = 0; k < ng; ++k) {
            const float sc = exp_e(r[k][0][lane] - m);
            z += sc * r[k][1][lane];
            zd += sc * r[k][2][lane];
        }
        if (rt.on && x >= 0 && x < W) {
            dhat[pix + x] = zd / z;
            lse[pix + x] = m + logf(z);
        }
    };
    for (int it = max(it0 - 1, 0), first = it; it < it1; ++it, par ^= 1) {
        const int X = it << 6;
        const int xc = min(X + lane, W - 1);
        const bool in_row = X + lane < W;
        if constexpr (kAdj) {
            const uint32_t a = X < W ? g.arms[pix + xc] : 0u;
            reinterpret_cast<uint8_t*>(arml[w][it & 1])[lane] = (uint8_t)(arm(a, 0) + 1);
            reinterpret_cast<uint8_t*>(armr[w][it & 1])[lane] = (uint8_t)arm(a, 1);
            if (it == first) {  // no block before (its digits are zero)
                reinterpret_cast<uint8_t*>(arml[w][~it & 1])[lane] = 1;
                reinterpret_cast<uint8_t*>(armr[w][~it & 1])[lane] = 0;
            }
            __builtin_amdgcn_wave_barrier();
        }
        const auto band = [&](int c) {
            const int k = c & 1;  // 0: the block before, 1: this one
            const int x = X - 32 + 16 * (c >> 1) + n;
            if constexpr (kAdj) {
                return band_bytes_t(arml[w][(it + 1 + k) & 1] + 4 * kg,
                                    armr[w][(it + 1 + k) & 1] + 4 * kg,
                                    X - 64 + 64 * k + 16 * kg - x);
            } else {
                const uint32_t a = g.arms[pix + min(max(x, 0), W - 1)];
                return band_bytes(x - arm(a, 0), x + arm(a, 1) + 1, X - 64 + 64 * k + 16 * kg);
            }
        };
        if constexpr (kShare)
            for (int c = w; c < 8; c += nw) bands[par][c][lane] = band(c);
        v4i bc[2][3];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < 3; ++k) bc[h][k] = v4i{0, 0, 0, 0};
        const int ex_old = sc.ex;
        if (active && X < W) {
            const float gp = kKind == kSeed && in_row ? gdhat[pix + xc] : 0.0f;
            const float dh = kKind == kSeed ? dhat[pix + xc] : 0.0f;
            const float ls = kKind == kSeed ? lse[pix + xc] : 0.0f;
            const float g1 =
                kKind == kSeed ? gp * invT * __builtin_amdgcn_rcpf(g.n2[pix + xc]) : 0.0f;
            const float dh0 = dh - (float)d0;
            float G[16];
            double t = 0.0;
            size_t Pv = Q;
            asm volatile("" : "+s"(Pv));  // else 16 row addresses live in registers
            const float* a2 = in + vol + (size_t)d0 * Pv + xc;
            const auto seed = [&](auto full) {
                constexpr bool kFull = decltype(full)::value;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    G[j] = *a2;
                    if (kFull || d0 + j + 1 < D) a2 += Pv;
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const bool on = kFull || d0 + j < D;
                    if constexpr (kKind == kSeed) {
                        const float u = exp_e(-G[j] * invT - ls) * (dh0 - (float)j);
                        t += (double)(on ? gp * u * G[j] : 0.0f);
                        G[j] = on ? g1 * u : 0.0f;
                    } else {
                        G[j] = in_row && on ? G[j] : 0.0f;
                    }
                }
            };
            if (d0 + 16 <= D)
                seed(std::true_type{});
            else
                seed(std::false_type{});
            if (kKind == kSeed && it >= it0) acc -= t;
            uint32_t lo[16];
            put_wide(G, stage, lo, sc);
            wide_planes(stage, lo, bc);
        }
        // the bands and the softmax sums; the buffers' next writers pass the next
        // one first
        if (kShare || (!kAdj && dhat)) __syncthreads();
        if (!kAdj && dhat && it > it0 && rt.grp == it % ng) merge(it - 1, par ^ 1);
        if (!active) continue;
        const auto bands_of = [&](int c) { return kShare ? bands[par][c][lane] : band(c); };
        if (kKind == kDot && it >= it0) {
            // the outputs' pixels and their partners, on the stage: reference
            // columns X - 32 .. X + 31, partner columns X - 47 - d0 .. X + 31 - d0
            uint32_t* const rx = stage;            // census of the reference pixels
            uint32_t* const ry = stage + 64;
            uint32_t* const rz = stage + 128;      // their colours
            float* const ra = reinterpret_cast<float*>(stage + 192);  // their alphas
            uint2* const px = reinterpret_cast<uint2*>(stage + 256);  // partners: census
            uint32_t* const pz = stage + 416;                         // colours
            // 0 <= x - d < span: the disparity is one, column and partner in the image
            const int xd = X - 32 - (d0 + n);
            const uint32_t span = d0 + n < D ? (uint32_t)(W - (d0 + n)) : 0u;
            const auto at = [&](const uint4* p, int x) {
                return p[pix + min(max(x, 0), W - 1)];
            };
            const uint4 r = at(im.pixL, X - 32 + lane);
            const uint4 q0 = at(im.pixR, X - 47 - d0 + lane);
            const uint4 q1 = at(im.pixR, X + 17 - d0 + (lane & 15));
            rx[lane] = r.x;
            ry[lane] = r.y;
            rz[lane] = r.z;
            ra[lane] = im.alpha[r.w >> 3];
            px[lane] = uint2{q0.x, q0.y};
            pz[lane] = q0.z;
            if (lane < 16) {
                px[64 + lane] = uint2{q1.x, q1.y};
                pz[64 + lane] = q1.z;
            }
            __builtin_amdgcn_wave_barrier();
            wide_outputs(X, W, bp, bc, ex_old, sc, bands_of, [&](int i, int, double(&v)[4]) {
                int c = 16 * i + 4 * kg;
                asm volatile("" : "+v"(c));  // the addresses are made here, not kept
                const v4u cx = *reinterpret_cast<const v4u*>(rx + c);
                const v4u cy = *reinterpret_cast<const v4u*>(ry + c);
                const v4u cz = *reinterpret_cast<const v4u*>(rz + c);
                const v4f al = *reinterpret_cast<const v4f*>(ra + c);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int e = c + k + 15 - n;
                    const uint2 q = px[e];
                    const uint32_t s = __builtin_amdgcn_sad_u8(cz[k], pz[e], 0u);
                    const int hm = __popc(cx[k] ^ q.x) + __popc(cy[k] ^ q.y);
                    const float da = al[k] * tab[s], dc = (1.0f - al[k]) * tab[kCenTab + hm];
                    const bool on = (uint32_t)(xd + c + k) < span;
                    acc = __builtin_fma(v[k], (double)(on ? da : 0.0f), acc);
                    acc2 = __builtin_fma(v[k], (double)(on ? dc : 0.0f), acc2);
                }
            });
            __builtin_amdgcn_wave_barrier();
        } else if (it >= it0) {
            wide_outputs(X, W, bp, bc, ex_old, sc, bands_of,
                         [&](int i, int, double(&v)[4]) {
                             *reinterpret_cast<v4f*>(stage + n * kMxStride + 16 * i + 4 * kg) =
                                 v4f{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
                         });
            __builtin_amdgcn_wave_barrier();
            if constexpr (!kAdj) {
                // A2 = sum / N2, and the softmax sums of the wavefront's 16
                // disparities for each column
                const float rn = __builtin_amdgcn_rcpf(
                    g.n2[pix + min(max(X - 32 + lane, 0), W - 1)]);
                float v[16], m = -INFINITY, z = 0.0f, zd = 0.0f;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    uint32_t* q = stage + j * kMxStride + lane;
                    const float a = __builtin_bit_cast(float, *q) * rn;
                    *q = __builtin_bit_cast(uint32_t, a);
                    v[j] = -a * invT;
                }
                if (dhat) {
#pragma unroll
                    for (int j = 0; j < 16; ++j) m = d0 + j < D ? fmaxf(m, v[j]) : m;
#pragma unroll
                    for (int j = 0; j < 16; ++j) {
                        const float e = d0 + j < D ? exp_e(v[j] - m) : 0.0f;
                        z += e;
                        zd += (float)j * e;
                    }
                    soft[par][w][0][lane] = m;
                    soft[par][w][1][lane] = z;
                    soft[par][w][2][lane] = zd + (float)d0 * z;
                }
                __builtin_amdgcn_wave_barrier();
            }
            put_rows<kRows>(stage, out + vol, Q, d0, D, X - 32, g.pitch);
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < 3; ++k) bp[h][k] = bc[h][k];
    }
    if (!kAdj && dhat) {
        __syncthreads();
        if (rt.grp == 0) merge(it1 - 1, par ^ 1);
    }
    if (kAdj && active) {
        for (int off = 32; off > 0; off >>= 1) {  // fixed-order wavefront reduction
            acc += __shfl_down(acc, off, 64);
            if (kKind == kDot) acc2 += __shfl_down(acc2, off, 64);
        }
        const size_t k = ((size_t)row * gridDim.y + blockIdx.y) * ng + grp;
        if (lane == 0 && kKind == kSeed) part[k] = acc * (double)(invT * invT);
        if (lane == 0 && kKind == kDot) {
            part[2 * k] = acc;
            part[2 * k + 1] = acc2;
        }
    }
}

// Column passes: both column sums of the forward (a1 = (column sum of E1) / N1,
// E2 = column sum of a1), or both of their adjoints, in one pass over the
// volume.  One thread per column, kSoftCols columns and one plane (or one of
// S row segments of it) per wavefront, rows in batches of kSoftPre.  Each of
// the two sums keeps FP64 running sums in an LDS ring of kSoftRing rows per
// column, so every range sum is exact to FP32 rounding of the final value,
// and each thread touches only its own column, so the result does not depend
// on scheduling; the first sum's rows go to the second in registers, rounded
// to FP32.
//
// The two rings (40 KB) leave a CU four wavefronts, one per SIMD, so the
// instruction stream of one wavefront has to cover every latency by itself:
//   - inputs are loaded kSoftLead batches ahead of their use;
//   - the LDS reads of one batch are issued in one step and used in the next
//     (a step works on batch j of the first sum's reads, on batch j - 1's
//     result, and on the second sum's reads, whose rows are stored one step
//     later);
//   - the row loop is unrolled over one turn of the ring (kSoftTurn batches),
//     so every ring slot and buffer index is a compile-time constant: slots
//     are immediate LDS offsets, and the wrap of a range end around the ring
//     is tested only in the batches where it can happen;
//   - no row is clamped or branched on: buffer loads outside the plane return
//     zero and stores outside the segment are dropped by the buffer's bounds.
// A plane's rows below 0 and past H then hold v = 0 and a record of N = 0,
// 1/N = 0: they add zero to both sums.
//
// Measured at 8 x 64 planes of 640 x 480 (1.26 GB in and out; a copy of that
// size takes about 0.25 ms): 0.33 ms forward and 0.38 to 0.41 ms adjoint, bound by the
// issue of the four wavefronts (33 instructions per row) and, in the adjoint,
// the LDS adds; as two passes over the volume, each near the copy's rate, 0.58
// ms each.  Record and 1 / N in one 8-byte load instead of two loads: forward
// 0.36 -> 0.34, adjoint 0.37 -> 0.38, 320 x 240 forward 74.0 -> 72.7 us.  Loading 2, 5 or 7
// batches ahead instead of 3: 0.37, 0.35, 0.35 ms.  At 32 planes of 320 x 240
// (160 wavefronts, six segments each) 19 us, was 53 us.
constexpr int kSoftCols = 64;
constexpr int kSoftPre = 5;                       // rows per batch
constexpr int kSoftRing = 2 * kLMax + 1 + kSoftPre;  // 40 rows
constexpr int kSoftTurn = kSoftRing / kSoftPre;   // batches per turn of the ring
constexpr int kSoftLead = 3;                      // batches loaded ahead
constexpr int kSoftBufs = kSoftLead < 4 ? 4 : 8;  // batches held per thread
constexpr int kSoftLag = 2 * kLMax + 2 * kSoftPre;  // rows from a row's input to its output
constexpr int kSoftSlots = 4 * 256;               // wavefronts the device holds at once
constexpr uint32_t kSoftDrop = 0x80000000u;       // buffer offset past any plane (W H <= 2^27)
static_assert(kSoftRing % kSoftPre == 0 && kSoftTurn % kSoftBufs == 0 && kSoftLead < kSoftBufs,
              "a turn of the ring is a whole number of batches and of buffer rotations");

// r / N1 from the record and 1/N1 (correctly rounded): the quotient's
// remainder is exact, so its correction rounds correctly (Markstein).
__device__ inline float col_div(float r, uint32_t rec, float rn) {
    const float n = (float)__builtin_bit_cast(_Float16, (uint16_t)(rec >> 16));
    const float q = r * rn;
    return __builtin_fmaf(__builtin_fmaf(n, q, r), rn, q);
}

constexpr int ring_mod(int s) { return ((s % kSoftRing) + kSoftRing) % kSoftRing; }

// LDS byte offset of ring row base + v (mod kSoftRing) of this thread's column,
// for a compile-time base in [0, kSoftRing), from o = 512 v + 8 t with
// 0 <= v <= span: the wrap folds away where it cannot happen (min picks the
// wrapped offset only where it does not go below zero).
__device__ inline uint32_t ring_at(int base, uint32_t o, int span) {
    const uint32_t r = (uint32_t)(base * (kSoftCols * 8)) + o;
    return base + span < kSoftRing ? r : min(r, r - (uint32_t)(kSoftRing * kSoftCols * 8));
}

// LDS add that returns nothing (a thread's adds to its own column stay in
// program order).
__device__ inline void lds_add(double* p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <bool kAdj>
__global__ __launch_bounds__(kSoftCols) void k_soft_vv(SoftGeom g, const float* __restrict__ in,
                                                       float* __restrict__ out, int seg_rows) {
    __shared__ __align__(16) double rings[2][kSoftRing][kSoftCols];
    const int t = threadIdx.x, x = blockIdx.x * kSoftCols + t;
    const int bd = blockIdx.y, b = bd / g.D;
    const size_t P = (size_t)g.W * g.H, Q = g.plane();
    const int r0 = blockIdx.z * seg_rows, r1 = min(r0 + seg_rows, g.H);
    const uint32_t W4 = 4u * (uint32_t)g.pitch, W8 = 8u * (uint32_t)g.W;
    const auto src = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(in + (size_t)bd * Q),
                                                       (short)0, (int)(Q * 4), 0x00020000);
    const auto rec = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint2*>(g.vrec + (size_t)b * P), (short)0, (int)(P * 8), 0x00020000);
    const auto dst = __builtin_amdgcn_make_buffer_rsrc(
        out + (size_t)bd * Q + (size_t)r0 * g.pitch, (short)0,
        (int)((uint32_t)(r1 - r0) * W4), 0x00020000);
    const uint32_t x4 = x < g.W ? 4u * (uint32_t)x : kSoftDrop;
    const uint32_t t8 = 8u * t;
    char* const R1 = reinterpret_cast<char*>(&rings[0][0][0]);
    char* const R2 = reinterpret_cast<char*>(&rings[1][0][0]);
    for (int i = 0; i < kSoftRing; ++i) rings[0][i][t] = rings[1][i][t] = 0.0;
    // first input row that the segment's outputs need; the stream starts
    // kSoftLead batches before it on zeroed buffers
    const int first = max(r0 - 2 * kLMax, 0);
    const int last = r1 + kSoftLag;
    uint32_t v_off = x4 + (uint32_t)first * W4;                     // row y + lead
    // records of row y + lead (adjoint) or y - kLMax + lead (forward)
    uint32_t n_off = x < g.W ? 2 * x4 + (uint32_t)(first - (kAdj ? 0 : kLMax)) * W8 : kSoftDrop;
    uint32_t d_off = x4 + (uint32_t)(first - r0 - kSoftLead * kSoftPre - kSoftLag) * W4;
    float v[kSoftBufs][kSoftPre], rn[kSoftTurn][kSoftPre];
    uint32_t p[kSoftBufs][kSoftPre], p2[kSoftTurn][kSoftPre];
    float rl[kSoftBufs][kSoftPre];
    double h1[kSoftPre], l1[kSoftPre], h2[kSoftPre], l2[kSoftPre];
#pragma unroll
    for (int k = 0; k < kSoftPre; ++k) {
#pragma unroll
        for (int j = 0; j < kSoftBufs; ++j) v[j][k] = rl[j][k] = 0.0f, p[j][k] = 0u;
#pragma unroll
        for (int j = 0; j < kSoftTurn; ++j) p2[j][k] = 0u, rn[j][k] = 0.0f;
        h1[k] = l1[k] = h2[k] = l2[k] = 0.0;
    }
    double acc1 = 0.0, acc2 = 0.0;
    const auto up = [&](uint32_t q) { return (q & 0x3e00u) | t8; };       // 512 dn + 8 t
    const auto dn = [&](uint32_t q) { return (q << 5 & 0x3e00u) | t8; };  // 512 (kLMax - u) + 8 t
    const auto at = [](char* r, uint32_t o) { return reinterpret_cast<double*>(r + o); };
    for (int y0 = first - kSoftLead * kSoftPre; y0 < last; y0 += kSoftRing) {
#pragma unroll
        for (int j = 0; j < kSoftTurn; ++j) {
            const int s1 = ring_mod((j - kSoftLead) * kSoftPre);       // slot of row y0 + 5 j
            const int s2 = ring_mod((j - kSoftLead - 1) * kSoftPre);   // and of the batch before
            float (&cv)[kSoftPre] = v[j % kSoftBufs];
            uint32_t (&cp)[kSoftPre] = p[j % kSoftBufs];
            float (&crn)[kSoftPre] = rl[j % kSoftBufs];
            // The batch's values are used from here on: without this pin the
            // compiler starts converting a later batch early, which waits for
            // loads that should still be in flight.
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k)
                asm volatile("" : "+v"(cv[k]), "+v"(cp[k]), "+v"(crn[k]));
            // the second sum's finished rows, read in the step before
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                float o;
                if (kAdj) {
                    acc2 += h2[k];
                    o = (float)acc2;
                } else {
                    o = (float)(h2[k] - l2[k]);
                }
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, o), dst, d_off,
                                                      0, 0);
                d_off += W4;
            }
            // the first sum's rows, read in the step before, into the second
            // (row record q of stream row y0 - kSoftPre + k - kLMax)
            float a1[kSoftPre];
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                const uint32_t q = kAdj ? (k < 2 ? p2[(j + 3) % kSoftTurn][k + 3]
                                                 : p2[(j + 4) % kSoftTurn][k - 2])
                                        : p2[(j + kSoftTurn - 1) % kSoftTurn][k];
                float r;
                if (kAdj) {
                    acc1 += h1[k];
                    r = (float)acc1;
                } else {
                    r = (float)(h1[k] - l1[k]);
                }
                const float rq = kAdj ? (k < 2 ? rn[(j + 3) % kSoftTurn][k + 3]
                                               : rn[(j + 4) % kSoftTurn][k - 2])
                                      : rn[(j + kSoftTurn - 1) % kSoftTurn][k];
                a1[k] = col_div(r, q, rq);
            }
            // first sum, batch j
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                if (kAdj) {
                    const double e = (double)cv[k];
                    lds_add(at(R1, ring_at(ring_mod(s1 + k - kLMax), dn(cp[k]), kLMax)), e);
                    lds_add(at(R1, ring_at(ring_mod(s1 + k + 1), up(cp[k]), kLMax)), -e);
                } else {
                    acc1 += (double)cv[k];
                    *at(R1, (uint32_t)(ring_mod(s1 + k) * kSoftCols * 8) + t8) = acc1;
                }
            }
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                if (kAdj) {
                    h1[k] = __hip_atomic_exchange(
                        at(R1, (uint32_t)(ring_mod(s1 + k - kLMax) * kSoftCols * 8) + t8), 0.0,
                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                } else {
                    h1[k] = *at(R1, ring_at(ring_mod(s1 + k - kLMax), up(cp[k]), kLMax));
                    l1[k] = *at(R1, ring_at(ring_mod(s1 + k - 2 * kLMax - 1), dn(cp[k]), kLMax));
                }
            }
            // second sum, batch j - 1
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                if (kAdj) {
                    const uint32_t q = k < 2 ? p2[(j + 3) % kSoftTurn][k + 3]
                                             : p2[(j + 4) % kSoftTurn][k - 2];
                    const double e = (double)a1[k];
                    lds_add(at(R2, ring_at(ring_mod(s2 + k - kLMax), dn(q), kLMax)), e);
                    lds_add(at(R2, ring_at(ring_mod(s2 + k + 1), up(q), kLMax)), -e);
                } else {
                    acc2 += (double)a1[k];
                    *at(R2, (uint32_t)(ring_mod(s2 + k) * kSoftCols * 8) + t8) = acc2;
                }
            }
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                if (kAdj) {
                    h2[k] = __hip_atomic_exchange(
                        at(R2, (uint32_t)(ring_mod(s2 + k - kLMax) * kSoftCols * 8) + t8), 0.0,
                        __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                } else {
                    const uint32_t q = k < 2 ? p2[(j + 3) % kSoftTurn][k + 3]
                                             : p2[(j + 4) % kSoftTurn][k - 2];
                    h2[k] = *at(R2, ring_at(ring_mod(s2 + k - kLMax), up(q), kLMax));
                    l2[k] = *at(R2, ring_at(ring_mod(s2 + k - 2 * kLMax - 1), dn(q), kLMax));
                }
            }
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                p2[j][k] = cp[k];
                rn[j][k] = crn[k];
            }
            // the batch kSoftLead ahead
#pragma unroll
            for (int k = 0; k < kSoftPre; ++k) {
                const int f = (j + kSoftLead) % kSoftBufs;
                v[f][k] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(src, v_off, 0, 0));
                const auto r = __builtin_amdgcn_raw_buffer_load_b64(rec, n_off, 0, 0);
                p[f][k] = r[0];
                rl[f][k] = __builtin_bit_cast(float, (uint32_t)r[1]);
                v_off += W4;
                n_off += W8;
            }
        }
    }
}


// Soft-argmin over d per pixel: dhat and lse (log-sum-exp of -A2/T), in one
// pass over the slices: kArgBatch slices are loaded at a time and the running
// sums are rescaled whenever the running maximum grows.
constexpr int kArgBatch = 16;

__global__ __launch_bounds__(256) void k_soft_argmin(SoftGeom g, const float* __restrict__ A2,
                                                     const float* __restrict__ theta,
                                                     float* __restrict__ dhat,
                                                     float* __restrict__ lse) {
    const size_t P = (size_t)g.W * g.H;
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    const int b = blockIdx.y;
    if (i >= P) return;
    const float invT = 1.0f / theta[2];
    const size_t Q = g.plane();
    const float* a = A2 + (size_t)b * g.D * Q + i +
                     (uint32_t)i / (uint32_t)g.W * (uint32_t)(g.pitch - g.W);
    float m = -INFINITY, z = 0.0f, zd = 0.0f;
    for (int d0 = 0; d0 < g.D; d0 += kArgBatch) {
        float v[kArgBatch];
#pragma unroll
        for (int j = 0; j < kArgBatch; ++j) v[j] = -a[(size_t)min(d0 + j, g.D - 1) * Q] * invT;
        float mb = m;
#pragma unroll
        for (int j = 0; j < kArgBatch; ++j) mb = d0 + j < g.D ? fmaxf(mb, v[j]) : mb;
        const float sc = exp_e(m - mb);  // 0 on the first batch (m = -inf)
        z *= sc;
        zd *= sc;
#pragma unroll
        for (int j = 0; j < kArgBatch; ++j) {
            if (d0 + j < g.D) {
                const float e = exp_e(v[j] - mb);
                z += e;
                zd += (float)(d0 + j) * e;
            }
        }
        m = mb;
    }
    dhat[(size_t)b * P + i] = zd / z;
    lse[(size_t)b * P + i] = m + logf(z);
}

// Two-level fixed-order reduction of the gradient partial sums: block k of
// kRedBlocks sums a contiguous chunk of the per-row lambda partials and of
// the per-block temperature partials; then one block sums the block totals.
constexpr int kRedBlocks = 256;

__device__ inline void tree3(double (*red)[256], double a, double c, double t) {
    red[0][threadIdx.x] = a;
    red[1][threadIdx.x] = c;
    red[2][threadIdx.x] = t;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int k = 0; k < 3; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_soft_reduce1(const double* __restrict__ partAC,
                                                      size_t nAC,
                                                      const double* __restrict__ partT, size_t nT,
                                                      double* __restrict__ blk) {
    __shared__ double red[3][256];
    const size_t ca = (nAC + kRedBlocks - 1) / kRedBlocks, ct = (nT + kRedBlocks - 1) / kRedBlocks;
    const size_t a0 = blockIdx.x * ca, a1 = a0 + ca < nAC ? a0 + ca : nAC;
    const size_t t0 = blockIdx.x * ct, t1 = t0 + ct < nT ? t0 + ct : nT;
    double a = 0.0, c = 0.0, t = 0.0;
    for (size_t i = a0 + threadIdx.x; i < a1; i += 256) {
        a += partAC[2 * i];
        c += partAC[2 * i + 1];
    }
    for (size_t i = t0 + threadIdx.x; i < t1; i += 256) t += partT[i];
    tree3(red, a, c, t);
    if (threadIdx.x == 0)
        for (int k = 0; k < 3; ++k) blk[3 * blockIdx.x + k] = red[k][0];
}

__global__ __launch_bounds__(256) void k_soft_reduce2(const double* __restrict__ blk,
                                                      float* __restrict__ grad) {
    __shared__ double red[3][256];
    const int t = threadIdx.x;
    tree3(red, blk[3 * t], blk[3 * t + 1], blk[3 * t + 2]);
    if (t == 0)
        for (int k = 0; k < 3; ++k) grad[k] = (float)red[k][0];
}

}  // namespace

// ---- launchers -------------------------------------------------------------

// Row segments of the column passes.  A wavefront streams its segment's rows,
// the 2 kLMax rows above and kSoftLag below that its outputs reach, and the
// lead-in, in whole turns; a CU holds four of them.  The split that needs the
// fewest turns one after the other is taken (the fewest segments on a tie):
// one segment where the planes alone fill the device, several where they do
// not.
static int soft_segments(int W, int H, int planes) {
    const long long wgs = (long long)((W + kSoftCols - 1) / kSoftCols) * planes;
    int best = 1;
    long long least = -1;
    for (int s = 1; s <= 8; ++s) {
        const int rows = (H + s - 1) / s;
        const int head = s > 1 ? 2 * kLMax : 0;
        const int walked = kSoftLead * kSoftPre + head + rows + kSoftLag;
        const int turns = (walked + kSoftRing - 1) / kSoftRing;
        const long long cost = (wgs * s + kSoftSlots - 1) / kSoftSlots * turns;
        if (least < 0 || cost < least) least = cost, best = s;
    }
    return best;
}

template <bool kAdj>
static void launch_vv(const SoftGeom& g, const float* in, float* out, hipStream_t st) {
    const int n = soft_segments(g.W, g.H, g.B * g.D), seg = (g.H + n - 1) / n;
    hipLaunchKernelGGL(k_soft_vv<kAdj>,
                       dim3((g.W + kSoftCols - 1) / kSoftCols, g.B * g.D, (g.H + seg - 1) / seg),
                       dim3(kSoftCols), 0, st, g, in, out, seg);
}

// Launch shape of the matrix-core row passes (RowTask): the groups that a workgroup
// has no wavefronts for go to further workgroups (grid z), and rows are split in parts
// (each computes one more block).  A block takes a SIMD's lone wavefront about as long
// as four wavefronts issue in, so the split with the least blocks times wavefronts per
// SIMD (four at least) is taken; the partial sums have room for D values per row.
// Forwards, with the groups in rounds of one workgroup and parts of two blocks at
// least: 1 x 128 x 100, D = 80 75 us, 57 so; 4 x 200 x 150, D = 128 172 and 157; 4 x
// 154 x 61, D = 23 57 and 48.  With a lone wavefront's block counted as two instead of
// four 1 x 320 x 240, D = 32 takes 63, 60 so.
struct RowGrid {
    bool share;
    int seg, parts;  // blocks per part of a row, values in all
    dim3 grid, block;
};

static RowGrid row_grid(const SoftGeom& g) {
    const int ng = (g.D + 15) / 16, rows = g.B * g.H, its = (g.W + 95) / 64;
    const bool share = ng > 2;
    // shared: wavefronts for the groups in as few workgroups as possible, evenly
    const int turns = (ng + kMxWaves - 1) / kMxWaves, zs = share ? turns : 1;
    const int nw = share ? (ng + turns - 1) / turns : kMxWaves;
    const int blocks = share ? rows : (rows + kMxWaves / ng - 1) / (kMxWaves / ng);
    int seg = its;
    long long least = -1;
    for (int n = 1; n <= std::min(its, g.D / ng); ++n) {
        const int len = (its + n - 1) / n, parts = (its + len - 1) / len;
        const long long waves = (long long)blocks * nw * zs * parts;
        const long long cost =
            (parts > 1 ? len + 1 : len) * std::max(4LL, (waves + kMxSimds - 1) / kMxSimds);
        if (least < 0 || cost < least) least = cost, seg = len;
    }
    const int segs = (its + seg - 1) / seg;
    return RowGrid{share, seg, rows * segs * ng, dim3(blocks, segs, zs), dim3(64 * nw)};
}

// Large volumes are written past the caches.  8 pairs of 640 x 480, D = 64: forward
// and backward 2147 us, 2050 so, the forward alone 1063 and 977; 8 of 400 x 300,
// D = 32 (31 M entries) 677 and 658; 1 of 640 x 480, D = 63 (19 M) 393 and 385; but 4
// of 328 x 240, D = 40 (13 M) 333 and 342.
static bool soft_stream(const SoftGeom& g) {
    return (long long)g.B * g.D * g.H * g.W > 16LL << 20;
}

// go(share, rows): the values as types
template <typename Go>
static void with_row_kind(const RowGrid& rg, const SoftGeom& g, Go go) {
    const auto second = [&](auto share) {
        if (g.pitch != soft_pitch(g.W))
            go(share, std::integral_constant<Rows, kCut>{});
        else if (soft_stream(g))
            go(share, std::integral_constant<Rows, kPast>{});
        else
            go(share, std::integral_constant<Rows, kWhole>{});
    };
    if (rg.share)
        second(std::true_type{});
    else
        second(std::false_type{});
}

static void launch_mrow(const RowGrid& rg, const SoftGeom& g, const SoftImg& im, float* out,
                        hipStream_t st) {
    with_row_kind(rg, g, [&](auto share, auto rows) {
        hipLaunchKernelGGL((k_soft_mrow<decltype(share)::value, decltype(rows)::value>), rg.grid,
                           rg.block, 0, st, g, im, out, rg.seg);
    });
}

template <WideKind kKind>
static void launch_wide(const RowGrid& rg, const SoftGeom& g, const SoftImg& im, const float* in,
                        const float* theta, float* dhat, float* lse, const float* gdhat, float* out,
                        double* part, hipStream_t st) {
    with_row_kind(rg, g, [&](auto share, auto rows) {
        // the dot products write no volume
        constexpr Rows kRows = kKind == kDot ? kWhole : decltype(rows)::value;
        hipLaunchKernelGGL((k_soft_wide<kKind, decltype(share)::value, kRows>), rg.grid, rg.block,
                           0, st, g, im, in, theta, dhat, lse, gdhat, out, part, rg.seg);
    });
}

hipError_t soft_prepare(const float* theta, float* tab, const uint32_t* arms, int B, int W, int H,
                        int D, uint2* vrec, float* n2, hipStream_t st) {
    SoftGeom g{arms, nullptr, nullptr, B, W, H, D, 0};
    hipLaunchKernelGGL(k_soft_counts, dim3((W + kCntTW - 1) / kCntTW, (H + kCntTH - 1) / kCntTH, B),
                       dim3(256), 0, st, g, theta, tab, vrec, n2);
    return hipGetLastError();
}

// Forward aggregation into A2 (B x D x H x W), and the soft argmin where dhat
// (and lse) are given; t1, t2 are volume-sized scratch.
hipError_t soft_aggregate(const SoftBuffers& s, int B, int W, int H, int D, float* A2, float* t1,
                          float* t2, const float* theta, float* dhat, float* lse,
                          hipStream_t st) {
    SoftGeom g{s.arms, s.vrec, s.n2, B, W, H, D, s.pitch};
    SoftImg im{s.pixL, s.pixR, s.alpha, s.tab};
    const RowGrid rg = row_grid(g);
    launch_mrow(rg, g, im, t1, st);                                 // E1
    launch_vv<false>(g, t1, t2, st);                                                         // E2
    const bool soft = dhat && D <= 16 * kMxWaves;
    launch_wide<kMean>(rg, g, im, t2, theta, soft ? dhat : nullptr, lse, nullptr, A2, nullptr,
                       st);                                                                  // A2
    if (dhat && !soft) {
        const size_t P = (size_t)W * H;
        hipLaunchKernelGGL(k_soft_argmin, dim3((unsigned)((P + 255) / 256), B), dim3(256), 0, st,
                           g, A2, theta, dhat, lse);
    }
    return hipGetLastError();
}

// Backward: A2 recomputed by the caller into `A2`; t1, t2 volume scratch.
hipError_t soft_backward(const SoftBuffers& s, int B, int W, int H, int D, const float* A2,
                         const float* theta, const float* dhat, const float* lse,
                         const float* gdhat, float* t1, float* t2, double* partAC,
                         double* partT, float* grad, hipStream_t st) {
    SoftGeom g{s.arms, s.vrec, s.n2, B, W, H, D, s.pitch};
    SoftImg im{s.pixL, s.pixR, s.alpha, s.tab};
    const int nrows = B * D * H;
    const RowGrid rg = row_grid(g);
    launch_wide<kSeed>(rg, g, im, A2, theta, const_cast<float*>(dhat), const_cast<float*>(lse),
                       gdhat, t2, partT, st);                         // G_E2, T-gradient terms
    launch_vv<true>(g, t2, t1, st);                                   // G_E1
    launch_wide<kDot>(rg, g, im, t1, theta, nullptr, nullptr, nullptr, nullptr, partAC,
                      st);                                            // H^T G_E1 . dc/dlambda
    double* blk = partT + (size_t)nrows;  // kRedBlocks x 3 after the row partials
    hipLaunchKernelGGL(k_soft_reduce1, dim3(kRedBlocks), dim3(256), 0, st, partAC,
                       (size_t)rg.parts, partT, (size_t)rg.parts, blk);
    hipLaunchKernelGGL(k_soft_reduce2, dim3(1), dim3(256), 0, st, blk, grad);
    return hipGetLastError();
}
