// k_vote.hip -- disparity refinement by region vote (Eq. 4, Sec. 4.3).
//
// One pass: every valid pixel p takes the disparity with the most votes in
// its stage-1 cross region N_p (for each y' on p's vertical arm, the pixels
// of (x, y')'s horizontal segment); equal counts go to the smallest
// disparity.  Invalid pixels (-1) neither vote nor change.  Passes read only
// the previous pass's map.
//
// Layout: one workgroup of eight wavefronts per 16 x 30 pixel tile (16
// columns, 30 rows), one thread per pixel.  The tile's votes plus a kLMax
// apron on every side (64 rows x 50 columns) are run-length coded as they are
// read, a wavefront per row and a lane per column (a ballot of the run starts
// gives every column its run), and the runs and the horizontal arms of the tile
// columns over the apron rows go to LDS.  A pixel's region is the union of the
// horizontal segments of the rows on its vertical arm, and the segment of
// (column, row) is the same for every pixel whose arm covers that row; so the
// votes are counted once per segment: for a window of kVBins disparities at a
// time, each of the 64 x 16 segments adds, for every run it meets, the overlap
// length to its own counters; the counters are then prefix-summed down each
// tile column, and a pixel reads its counts as the difference of two prefix
// rows (the ends of its vertical arm).  Counters are 16-bit, two per 32-bit
// word (a count is at most 64 rows x 35 columns, so packed sums and
// differences never carry between the halves).
// Disparities are counted by rank among those that occur in the tile's staged
// votes, in increasing order, so the windows step over what occurs and not over
// the range it spans (960 x 540: 1.05 windows per tile instead of 2.2); a strict
// running maximum keeps the smallest disparity among equal counts.  All counts
// are integers, so the result does not depend on the order of the additions.
//
// Bound by the chain of loads and LDS steps of a tile, not by issue or memory, and
// longer with more runs in the tile's rows.  Pairs of a slanted background and six
// boxes, noise of two grey levels: a pass over 640 x 360 (480 tiles, one round) takes
// 12.4 us, over 960 x 540, D = 96 (1080 tiles, three per CU) 23.7.  With the rows coded
// by a thread each, the prefixes by a quarter of the threads, windows of 16 over the
// range and two tiles per CU they took 19.4 and 50.  (Ten slanted planes and two boxes
// at 1280 x 720, reduced to 640 x 360: 23.6 us.)  The last pass makes the outputs
// itself (2.8 to 3.5 us more; as a launch 5.2 to 5.9, and 5 for the depth of the
// quarter-size front end).
#include "dco_device.h"

namespace {

constexpr int kVTW = 16, kVTH = 30;         // tile width and height
constexpr int kVThreads = 512;              // a segment each, twice; kVTW kVTH have a pixel
constexpr int kVWaves = kVThreads / 64;
constexpr int kVRW = kVTW + 2 * kLMax;      // staged width
constexpr int kVRH = kVTH + 2 * kLMax;      // staged height
constexpr int kVRows = kVRH / kVWaves;      // staged rows per wavefront

constexpr int kVBins = 14;               // disparities per counter window: three tiles per CU
constexpr int kVWords = kVBins / 2;      // two 16-bit counters per word
constexpr int kVWordStride = kVWords;    // per tile column (odd: no bank conflicts)
constexpr int kVRowStride = kVTW * kVWordStride + 1;  // 16 rows apart: 16 banks apart
constexpr int kVSegs = kVRH * kVTW;      // segments: staged rows x tile columns
constexpr int kVMaxD = 16384;            // D < W <= 16384
constexpr int kVParts = 4;               // threads per column word of the prefixes
static_assert(kVBins % 2 == 0 && (kVRH + 1) * 35 < 65536, "packed 16-bit counters");
static_assert(kVRW <= 64 && kVRH % kVWaves == 0 && kVSegs % kVThreads == 0 &&
                  kVTW * kVTH <= kVThreads && kVParts * kVTW * kVWords <= kVThreads &&
                  kVRH % kVParts == 0 && kVWordStride % 2 == 1,
              "rows per wavefront, segments and prefix parts per thread");

struct VoteLds {
    // cnt: entry (r, c, k), r kVRowStride + c kVWordStride + k: for tile column c
    // and the window's bins 2k, 2k + 1, the votes over the segments of staged
    // rows 0 .. r - 1 (row 0: none)
    uint32_t cnt[(kVRH + 1) * kVRowStride];
    uint32_t bits[kVMaxD / 32];       // disparities that occur
    uint16_t pre[kVMaxD / 32];        // ... in the words before
    // rank of run k of each staged row; run of each column; start column of run
    // k, st[nruns] = kVRW (rows padded: runs are read in fours)
    int16_t rv[kVRH][kVRW + 4];
    uint8_t rs[kVRH][kVRW + 2], st[kVRH][kVRW + 4];
    uint8_t l[kVRH][kVTW], r[kVRH][kVTW];  // horizontal arms of the tile columns
};

// Output of a voted map at pixel i: disp = d + the parabola offset at d (Eq. 3's
// sub-pixel step on the aggregated costs) and valid = 1 where d is in [0, D);
// else disp = 0, valid = 0.  dv (optional) gets d, or -1 where invalid.
struct VoteOut {
    const float* agg;
    float* disp;
    uint8_t* valid;
    int16_t* dv;
    HalfOut half;
    int pitch, W, H, D, subpixel, paired;  // volume rows of `pitch` columns
};

__device__ inline void vote_output(const VoteOut& o, int d, int x, int y) {
    const size_t i = (size_t)y * o.W + x;
    const int v = y * o.pitch + x, P = o.pitch * o.H;  // in the volume
    const bool ok = d >= 0 && d < o.D;
    float out = 0.0f;
    if (ok) {
        float del = 0.0f;
        if (o.subpixel && d > 0 && d < o.D - 1) {
            if (o.paired)
                del = dco::subpixel_delta(dco::paired_at(o.agg, P, o.D, d - 1, v),
                                          dco::paired_at(o.agg, P, o.D, d, v),
                                          dco::paired_at(o.agg, P, o.D, d + 1, v), d, o.D);
            else
                del = dco::subpixel_delta(o.agg[(size_t)(d - 1) * P + v], o.agg[(size_t)d * P + v],
                                          o.agg[(size_t)(d + 1) * P + v], d, o.D);
        }
        out = (float)d + del;
    }
    if (o.half.on) {
        out *= 2.0f;
        if (o.half.depth) o.half.depth[i] = out > 0.0f ? o.half.fB / out : 0.0f;
    }
    o.disp[i] = out;
    o.valid[i] = (uint8_t)ok;
    if (o.dv) o.dv[i] = (int16_t)(ok ? d : -1);
}

// din: H x W int16; valid (first pass only, else null): H x W uint8; a vote
// outside [0, D) counts as invalid.  dout: H x W int16, -1 where invalid; or, for
// the last pass (kOut), the outputs.
template <bool kOut>
__global__ __launch_bounds__(kVThreads) void k_vote(const int16_t* __restrict__ din,
                                                    const uint8_t* __restrict__ valid,
                                                    const uint32_t* __restrict__ arms, int W,
                                                    int H, int D, int16_t* __restrict__ dout,
                                                    VoteOut o) {
    __shared__ __align__(16) VoteLds S;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int tx = tid & (kVTW - 1), ty = tid / kVTW;
    const int x0 = blockIdx.x * kVTW, y0 = blockIdx.y * kVTH;
    const int nwords = (D + 31) >> 5;
    for (int i = tid; i < nwords; i += kVThreads) S.bits[i] = 0u;

    // every load issued before any is used (clamped addresses): the votes of row
    // w + 8 k, column `lane` of the staged region, the horizontal arms of two
    // segments, and this pixel's own
    int dv[kVRows], ok[kVRows];
#pragma unroll
    for (int k = 0; k < kVRows; ++k) {
        const int x = x0 - kLMax + lane, y = y0 - kLMax + w + kVWaves * k;
        const size_t q = (size_t)min(max(y, 0), H - 1) * W + min(max(x, 0), W - 1);
        dv[k] = din[q];
        ok[k] = valid ? valid[q] : 1;
        if (!(x >= 0 && x < W && y >= 0 && y < H)) ok[k] = 0;
    }
    uint32_t av[kVSegs / kVThreads];
#pragma unroll
    for (int t = 0; t < kVSegs / kVThreads; ++t) {
        const int i = tid + kVThreads * t, ry = i / kVTW, cx = i - ry * kVTW;
        const int x = x0 + cx, y = y0 - kLMax + ry;
        av[t] = arms[(size_t)min(max(y, 0), H - 1) * W + min(x, W - 1)];
        if (!(x < W && y >= 0 && y < H)) av[t] = 0u;
    }
    const int x = x0 + tx, y = y0 + ty;
    const bool in = x < W && y < H && ty < kVTH;
    const size_t pq = (size_t)min(y, H - 1) * W + min(x, W - 1);
    const uint32_t a = arms[pq];
    int mine = din[pq];
    if (!in || mine < 0 || mine >= D || (valid && valid[pq] == 0)) mine = -1;
    __syncthreads();  // the cleared bits

    // run-length code the staged rows
    int id[kVRows];  // run that starts at this lane's column, or -1
#pragma unroll
    for (int k = 0; k < kVRows; ++k) {
        const int row = w + kVWaves * k;
        dv[k] = ok[k] && dv[k] >= 0 && dv[k] < D ? dv[k] : -1;
        const int v = dv[k];
        const int prev = __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, false);  // lane - 1
        const bool start = lane < kVRW && (lane == 0 || v != prev);
        const unsigned long long m = __ballot(start);
        const int before = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        id[k] = start ? before : -1;
        if (lane < kVRW) S.rs[row][lane] = (uint8_t)(before - (start ? 0 : 1));
        if (start) {
            S.st[row][before] = (uint8_t)lane;
            if (v >= 0) atomicOr(&S.bits[v >> 5], 1u << (v & 31));
        }
        if (lane == 0) S.st[row][__popcll(m)] = (uint8_t)kVRW;
    }
#pragma unroll
    for (int t = 0; t < kVSegs / kVThreads; ++t) {
        const int i = tid + kVThreads * t, ry = i / kVTW, cx = i - ry * kVTW;
        S.l[ry][cx] = (uint8_t)min(av[t] & 0xff, (uint32_t)kLMax);
        S.r[ry][cx] = (uint8_t)min((av[t] >> 8) & 0xff, (uint32_t)kLMax);
    }
    __syncthreads();
    // ranks: disparities that occur below each.  Up to 64 words, every wavefront
    // scans them in registers (lane = word); more, they are scanned once into LDS
    const int per = (nwords + 63) >> 6;  // words per lane
    uint32_t word = 0, n = 0;
    for (int i = 0; i < per; ++i) {
        const int q = lane * per + i;
        word = q < nwords ? S.bits[q] : 0u;
        n += __popc(word);
    }
    uint32_t inc = n;
    inc += dco::dpp<0x111, 0xf>(inc);
    inc += dco::dpp<0x112, 0xf>(inc);
    inc += dco::dpp<0x114, 0xf>(inc);
    inc += dco::dpp<0x118, 0xf>(inc);
    inc += dco::dpp<0x142, 0xa>(inc);
    inc += dco::dpp<0x143, 0xc>(inc);
    const int nd = __builtin_amdgcn_readlane((int)inc, 63);
    uint32_t below = inc - n;
    const auto put_ranks = [&](auto rank) {
#pragma unroll
        for (int k = 0; k < kVRows; ++k) {
            const int r = rank(max(dv[k], 0));
            if (id[k] >= 0) S.rv[w + kVWaves * k][id[k]] = (int16_t)(dv[k] >= 0 ? r : -1);
        }
    };
    if (per == 1) {
        put_ranks([&](int v) {  // all lanes are here
            return __shfl((int)below, v >> 5, 64) +
                   __popc((uint32_t)__shfl((int)word, v >> 5, 64) & ((1u << (v & 31)) - 1u));
        });
        if (w == 0 && lane < nwords) S.pre[lane] = (uint16_t)below;
    } else {
        if (w == 0)
            for (int i = 0; i < per; ++i) {
                const int q = lane * per + i;
                if (q < nwords) {
                    S.pre[q] = (uint16_t)below;
                    below += __popc(S.bits[q]);
                }
            }
        __syncthreads();
        put_ranks([&](int v) {
            return (int)S.pre[v >> 5] + __popc(S.bits[v >> 5] & ((1u << (v & 31)) - 1u));
        });
    }
    if (tid < kVTW * kVWords)
        S.cnt[(tid / kVWords) * kVWordStride + tid % kVWords] = 0u;  // row 0
    __syncthreads();

    const int u = min((int)((a >> 16) & 0xff), kLMax), dn = min((int)(a >> 24), kLMax);
    // this pixel's vertical arm in staged rows: prefix rows r0 (before it)
    // and r1 (through its last row)
    const int r0 = min(ty, kVTH - 1) + kLMax - u, r1 = min(ty, kVTH - 1) + kLMax + dn + 1;
    int best = 0, bc = -1;
    for (int base = 0; base < nd; base += kVBins) {  // uniform
        const int nb = min(kVBins, nd - base);       // bins past nd get no votes
        // 1. each segment's counts (one thread per segment, in two turns)
        for (int sg = tid; sg < kVSegs; sg += kVThreads) {
            const int ry = sg / kVTW, cx = sg - ry * kVTW;
            uint32_t* c = S.cnt + (ry + 1) * kVRowStride + cx * kVWordStride;
#pragma unroll
            for (int k = 0; k < kVWords; ++k) c[k] = 0u;
            const int lo = cx + kLMax - S.l[ry][cx], hi = cx + kLMax + S.r[ry][cx];
            const int k1 = S.rs[ry][hi];
            int from = lo;  // first column of the segment in run j
            // four runs' reads together, and adds that return nothing: the chain
            // is one LDS round trip per four runs
            for (int j = S.rs[ry][lo]; j <= k1; j += 4) {
                int b[4], next[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    b[i] = S.rv[ry][j + i] - base;
                    next[i] = S.st[ry][j + i + 1];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (j + i <= k1 && b[i] >= 0 && b[i] < nb)
                        __hip_atomic_fetch_add(
                            c + (b[i] >> 1),
                            (uint32_t)(min(next[i], hi + 1) - from) << (16 * (b[i] & 1)),
                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    from = next[i];
                }
            }
        }
        __syncthreads();
        {   // 2. prefix sums down each tile column: four threads per column word,
            // sixteen rows each
            const int part = tid & (kVParts - 1), q = min(tid / kVParts, kVTW * kVWords - 1);
            constexpr int kRows = kVRH / kVParts;
            uint32_t* c = S.cnt + (1 + part * kRows) * kVRowStride +
                          (q / kVWords) * kVWordStride + q % kVWords;
            uint32_t v[kRows];
#pragma unroll
            for (int i = 0; i < kRows; ++i) v[i] = c[i * kVRowStride];
#pragma unroll
            for (int i = 1; i < kRows; ++i) v[i] += v[i - 1];
            const uint32_t t = v[kRows - 1];
            const uint32_t b1 = dco::dpp<0x111, 0xf>(t), b2 = dco::dpp<0x112, 0xf>(t),
                           b3 = dco::dpp<0x113, 0xf>(t);  // totals of the parts before
            const uint32_t before =
                (part > 0 ? b1 : 0u) + (part > 1 ? b2 : 0u) + (part > 2 ? b3 : 0u);
#pragma unroll
            for (int i = 0; i < kRows; ++i)
                if (tid < kVParts * kVTW * kVWords) c[i * kVRowStride] = v[i] + before;
        }
        __syncthreads();
        // 3. this pixel's counts: two prefix rows per word (bins past nd count 0
        // or what an earlier window left, and are not looked at)
        if (mine >= 0) {
            const uint32_t* c0 = S.cnt + r0 * kVRowStride + tx * kVWordStride;
            const uint32_t* c1 = S.cnt + r1 * kVRowStride + tx * kVWordStride;
            uint32_t d[kVWords];
#pragma unroll
            for (int k = 0; k < kVWords; ++k) d[k] = c1[k] - c0[k];
#pragma unroll
            for (int k = 0; k < kVBins; ++k) {
                const int n = (int)(k & 1 ? d[k / 2] >> 16 : d[k / 2] & 0xffffu);
                if (k < nb && n > bc) {
                    bc = n;
                    best = base + k;
                }
            }
        }
        __syncthreads();
    }
    if (in) {
        int d = -1;
        if (mine >= 0) {  // the disparity of rank `best`
            int q = 0;
            while (q + 1 < nwords && (int)S.pre[q + 1] <= best) ++q;
            uint32_t m = S.bits[q];
            for (int k = best - S.pre[q]; k > 0; --k) m &= m - 1;
            d = 32 * q + __builtin_ctz(m);
        }
        if constexpr (kOut)
            vote_output(o, d, x, y);
        else
            dout[(size_t)y * W + x] = (int16_t)d;
    }
}

// The output step of a map in memory.
__global__ __launch_bounds__(256) void k_vote_finish(const int16_t* dv, const uint8_t* valid_in,
                                                     VoteOut o) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= o.W * o.H) return;
    const int y = i / o.W;
    vote_output(o, valid_in && !valid_in[i] ? -1 : dv[i], i - y * o.W, y);
}

}  // namespace

hipError_t launch_vote(const int16_t* dL, const uint8_t* valid, const uint32_t* arms,
                       const float* agg, bool paired, int pitch, int W, int H, int D, int iters,
                       int subpixel, int16_t* buf0, int16_t* buf1, float* disp, uint8_t* valid_out,
                       int16_t* dv_out, const HalfOut& half, hipStream_t st) {
    const VoteOut o{agg, disp, valid_out, dv_out, half, pitch, W, H, D, subpixel, (int)paired};
    const dim3 grid((W + kVTW - 1) / kVTW, (H + kVTH - 1) / kVTH);
    // the last pass makes the outputs, unless it is also the first (other tiles then
    // still read the mask that valid_out may be) or an output lies on the arms
    const size_t P = (size_t)W * H;
    const bool fused = iters > 1 && !overlap(disp, 4 * P, arms, 4 * P) &&
                       !overlap(valid_out, P, arms, 4 * P) && !overlap(dv_out, 2 * P, arms, 4 * P);
    const int16_t* src = dL;
    const uint8_t* mask = valid;
    int16_t* bufs[2] = {buf0, buf1};
    for (int it = 0; it < iters - (fused ? 1 : 0); ++it) {
        int16_t* dst = bufs[it & 1];
        hipLaunchKernelGGL(k_vote<false>, grid, dim3(kVThreads), 0, st, src, mask, arms, W, H, D,
                           dst, VoteOut{});
        src = dst;
        mask = nullptr;
    }
    if (fused)
        hipLaunchKernelGGL(k_vote<true>, grid, dim3(kVThreads), 0, st, src, mask, arms, W, H, D,
                           (int16_t*)nullptr, o);
    else
        hipLaunchKernelGGL(k_vote_finish, dim3((W * H + 255) / 256), dim3(256), 0, st, src, mask,
                           o);
    return hipGetLastError();
}
