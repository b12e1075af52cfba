// k_cost.hip -- raw AD-census cost volume of one reference view (Eq. 1) in
// fixed point: q = rint(alpha_L * TA[s] * 2^20) + rint(beta_L * TC[h] * 2^20),
// each term rounded once from the exact product of its float factors, stored
// as q * 2^-20.
//
// One workgroup = one image row, kTX consecutive reference pixels and a chunk
// of kDC disparities: the reference pixels, the partner pixels they can reach
// and the two lookup tables are staged in LDS.  A thread owns four consecutive
// columns and kDT disparities, taken four at a time: the seven partners of a
// 4 x 4 block are two quads of each staged plane, and the second is the next
// block's first, so a value costs a fifth of a 16-byte read besides its two
// table lookups, and its store is a quarter of a 16-byte store (at any row
// length: buffers keep words aligned, which is all that store needs).
//
// Bound by the volume's bytes, or by launch latency below about 10 MB.  With one
// column per thread and 32 disparities in turn: 640 x 480, D = 64 21.9 us per
// view (3.6 TB/s), now 18.5; 295 x 717, D = 41 15.6, now 13.4.  Four disparities
// per thread instead of eight 17.8 and 13.5, sixteen 19.0 and 15.0.
#include <type_traits>

#include "dco_device.h"

namespace {

constexpr int kDT = 8;  // disparities of a thread
// disparities of a workgroup of kTX columns
template <int kTX>
constexpr int kDCOf = kDT * (256 / (kTX / 4));

template <int kRef, int kTX, bool kStream>
__global__ __launch_bounds__(256) void k_cost(const uint8_t* __restrict__ rgb_ref,
                                              const uint8_t* __restrict__ rgb_par,
                                              const uint64_t* __restrict__ cen_ref,
                                              const uint64_t* __restrict__ cen_par,
                                              const uint32_t* __restrict__ arms, int W, int H,
                                              int D, const float* __restrict__ tabA,
                                              const float* __restrict__ tabC,
                                              const float* __restrict__ alpha,
                                              const float* __restrict__ beta,
                                              float* __restrict__ cost) {
    constexpr int kQuads = kTX / 4;            // threads across
    constexpr int kDC = kDCOf<kTX>;
    constexpr int kPar = kTX + kDC;            // partner pixels staged
    __shared__ float s_tabA[768];
    __shared__ float s_tabC[65];
    __shared__ __align__(16) uint32_t s_par[3][kPar];  // rgb, census low and high word
    __shared__ __align__(16) uint32_t s_ref[3][kTX];
    __shared__ __align__(16) float s_ab[2][kTX];       // alpha and beta, without the 2^20

    const int t = threadIdx.x;
    const int x0 = blockIdx.x * kTX, y = blockIdx.y, d0 = blockIdx.z * kDC;
    const size_t row = (size_t)y * W;

    for (int i = t; i < 766; i += 256) s_tabA[i] = tabA[i];
    if (t < 65) s_tabC[t] = tabC[t];
    // partner columns base .. base + kPar - 1
    const int base = kRef == 0 ? x0 - d0 - kDC : x0 + d0;
    for (int i = t; i < kPar; i += 256) {
        const int xp = base + i;
        uint32_t c = 0;
        uint64_t cc = 0;
        if (xp >= 0 && xp < W) {
            const uint8_t* p = rgb_par + 3 * (row + xp);
            c = (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16);
            cc = cen_par[row + xp];
        }
        s_par[0][i] = c;
        s_par[1][i] = (uint32_t)cc;
        s_par[2][i] = (uint32_t)(cc >> 32);
    }
    // the upper half of the threads, which has fewer partners to stage
    if (t >= 256 - kTX) {
        const int i = t - (256 - kTX), x = min(x0 + i, W - 1);
        const uint8_t* p = rgb_ref + 3 * (row + x);
        s_ref[0][i] = (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16);
        const uint64_t cc = cen_ref[row + x];
        s_ref[1][i] = (uint32_t)cc;
        s_ref[2][i] = (uint32_t)(cc >> 32);
        const uint32_t a = arms[row + x];
        const int lmin = min(min(min((int)(a & 0xff), (int)((a >> 8) & 0xff)),
                                 min((int)((a >> 16) & 0xff), (int)(a >> 24))), kLMax);
        s_ab[0][i] = alpha[lmin] * 0x1p-20f;
        s_ab[1][i] = beta[lmin] * 0x1p-20f;
    }
    __syncthreads();

    const int c = 4 * (t % kQuads), x = x0 + c;
    const int dt = kDT * (t / kQuads);  // first disparity of the thread within the chunk
    if (x >= W || d0 + dt >= D) return;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
    const auto quad = [](const uint32_t* p) { return *reinterpret_cast<const u32x4*>(p); };
    u32x4 ref[3], nr[3], fr[3];  // nr, fr: the block's nearer and farther partner quads
#pragma unroll
    for (int k = 0; k < 3; ++k) ref[k] = quad(s_ref[k] + c);
    const f32x4 al = *reinterpret_cast<const f32x4*>(s_ab[0] + c);
    const f32x4 be = *reinterpret_cast<const f32x4*>(s_ab[1] + c);
    // partner of the thread's first column at its first disparity
    const int i0 = kRef == 0 ? c + kDC - dt : c + dt;
#pragma unroll
    for (int k = 0; k < 3; ++k) nr[k] = quad(s_par[k] + i0);
    const size_t slice = (size_t)W * H;
    float* out = cost + (size_t)(d0 + dt) * slice + row + x;
#pragma unroll
    for (int b = 0; b < kDT; b += 4) {
        const int d = d0 + dt + b;
        if (d >= D) break;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            fr[k] = quad(s_par[k] + (kRef == 0 ? i0 - b - 4 : i0 + b + 4));
        // partner of column j at disparity d + e: place m = j - e (left
        // reference) or j + e from the nearer quad's first
        f32x4 v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int m = kRef == 0 ? j - e : j + e;
                const bool n = m >= 0 && m < 4;
                const int f = kRef == 0 ? m + 4 : m - 4;
                const uint32_t pc = n ? nr[0][m & 3] : fr[0][f & 3];
                const uint32_t pl = n ? nr[1][m & 3] : fr[1][f & 3];
                const uint32_t ph = n ? nr[2][m & 3] : fr[2][f & 3];
                const uint32_t s = __builtin_amdgcn_sad_u8(ref[0][j], pc, 0u);
                const uint32_t h = (uint32_t)__popc(ref[1][j] ^ pl) +
                                   (uint32_t)__popc(ref[2][j] ^ ph);
                // 8 + q1 2^-20 and 8 + q2 2^-20, each rounded once (a unit in
                // the last place of [8, 16) is 2^-20); the sums are exact
                const float q1 = __builtin_fmaf(al[j], s_tabA[s], 8.0f);
                const float q2 = __builtin_fmaf(be[j], s_tabC[h], 8.0f);
                const float q = q1 + (q2 - 16.0f);
                const bool in = kRef == 0 ? x - d + m >= 0 : x + d + m < W;
                v[e][j] = in ? q : 1.0f;
            }
#pragma unroll
        for (int e = 0; e < 4; ++e, out += slice) {
            if (d + e >= D) break;
            if (x + 4 <= W) {
                if (kStream)
                    __builtin_nontemporal_store(v[e], reinterpret_cast<f32x4u*>(out));
                else
                    *reinterpret_cast<f32x4u*>(out) = v[e];
            } else {  // the quad that the right border cuts
                out[0] = v[e][0];
                if (x + 1 < W) out[1] = v[e][1];
                if (x + 2 < W) out[2] = v[e][2];
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) nr[k] = fr[k];
    }
}

// A volume that the 256 MB memory-side cache holds is read from there by the
// aggregation that follows; a larger one is written past it, and in longer runs
// of a row.  All staged calls, 1280 x 720 with D = 128: 1304 us as the smaller
// volumes, 1198 so (256 columns without the streaming stores 1251, 128 with them
// 1215); D = 64 (236 MB) 672 and 647; 960 x 540, D = 128 (265 MB) 706 and 679.
// Below the line it is the other way: 960 x 540, D = 96 (199 MB) 433 and 493;
// 1280 x 720, D = 48 (177 MB) 533 and 576.
constexpr long long kKeepVolume = 54LL << 20;

}  // namespace

hipError_t launch_cost(int ref, const uint8_t* rgbL, const uint8_t* rgbR, const uint64_t* cenL,
                       const uint64_t* cenR, const uint32_t* arms_ref, int W, int H, int D,
                       const float* tabA, const float* tabC, const float* alpha,
                       const float* beta, int L1, float* cost, hipStream_t st) {
    (void)L1;
    const auto go = [&](auto columns, auto kernel0, auto kernel1) {
        constexpr int kTX = decltype(columns)::value, kDC = kDCOf<kTX>;
        const dim3 grid((W + kTX - 1) / kTX, H, (D + kDC - 1) / kDC);
        if (ref == 0)
            hipLaunchKernelGGL(kernel0, grid, dim3(256), 0, st, rgbL, rgbR, cenL, cenR, arms_ref,
                               W, H, D, tabA, tabC, alpha, beta, cost);
        else
            hipLaunchKernelGGL(kernel1, grid, dim3(256), 0, st, rgbR, rgbL, cenR, cenL, arms_ref,
                               W, H, D, tabA, tabC, alpha, beta, cost);
    };
    if ((long long)W * H * D <= kKeepVolume)
        go(std::integral_constant<int, 128>{}, k_cost<0, 128, false>, k_cost<1, 128, false>);
    else
        go(std::integral_constant<int, 256>{}, k_cost<0, 256, true>, k_cost<1, 256, true>);
    return hipGetLastError();
}
