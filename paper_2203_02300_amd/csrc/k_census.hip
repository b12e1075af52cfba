// k_census.hip -- census codes and cross-support arms of one image
// (Sec. 4.1; the C_census term of Eq. 1), and the per-pixel region counts and
// aggregation records.  The stage bodies live in dco_device.h.
#include <type_traits>

#include "dco_device.h"

namespace {

// One thread per pixel of a tile (16 rows: 1024 threads, at most 64 VGPRs so that
// two workgroups share a CU).
template <int TH>
__global__ __launch_bounds__(64 * TH) __attribute__((amdgpu_waves_per_eu(8))) void k_census_arms(
    const uint8_t* __restrict__ rgb, int W, int H, int cw, int ch, int L1, int tau1,
    uint64_t* __restrict__ census, uint32_t* __restrict__ arms, uint32_t* __restrict__ rgb_packed,
    uint4* __restrict__ pix) {
    __shared__ dco::CensusLdsOf<TH> S;
    dco::census_tile<64 * TH, TH>(rgb, W, H, cw, ch, L1, tau1, census, arms, rgb_packed, pix, false,
                           blockIdx.x * dco::kCenTW, blockIdx.y * TH, S);
}

__global__ __launch_bounds__(1024) void k_geometry(const uint32_t* __restrict__ arms, int W, int H,
                                                   int iters, AggRecords rec) {
    __shared__ dco::GeomLds S;
    dco::geometry_tile(arms, W, H, iters, rec, blockIdx.x * dco::kGeoTW,
                       blockIdx.y * dco::kGeoTH, S);
}

// Both views of the one-call path in one launch each (blockIdx.z = view);
// one thread per pixel of a tile.
template <int TH>
__global__ __launch_bounds__(64 * TH) __attribute__((amdgpu_waves_per_eu(8))) void k_census_arms2(
    const uint8_t* __restrict__ rgbL, const uint8_t* __restrict__ rgbR, int W, int H, int cw,
    int ch, int L1, int tau1, uint32_t* __restrict__ armsL, uint32_t* __restrict__ armsR,
    uint4* __restrict__ pixL, uint4* __restrict__ pixR, bool planes) {
    __shared__ dco::CensusLdsOf<TH> S;
    const bool r = blockIdx.z != 0;
    dco::census_tile<64 * TH, TH>(r ? rgbR : rgbL, W, H, cw, ch, L1, tau1, nullptr,
                                  r ? armsR : armsL, nullptr, r ? pixR : pixL, planes,
                                  blockIdx.x * dco::kCenTW, blockIdx.y * TH, S);
}

__global__ __launch_bounds__(1024) void k_geometry2(const uint32_t* __restrict__ armsL,
                                                   const uint32_t* __restrict__ armsR, int W,
                                                   int H, int iters, AggRecords recL,
                                                   AggRecords recR) {
    __shared__ dco::GeomLds S;
    const bool r = blockIdx.z != 0;
    dco::geometry_tile(r ? armsR : armsL, W, H, iters, r ? recR : recL, blockIdx.x * dco::kGeoTW,
                       blockIdx.y * dco::kGeoTH, S);
}

// Every view of a batch of pairs in one launch (blockIdx.z = 2 * pair + view),
// for the soft path: arms and packed pixels; one thread per pixel of a tile.
template <int TH>
__global__ __launch_bounds__(64 * TH) __attribute__((amdgpu_waves_per_eu(8))) void k_census_pairs(
    const uint8_t* __restrict__ rgbL, const uint8_t* __restrict__ rgbR, int W, int H, int cw,
    int ch, int L1, int tau1, uint32_t* __restrict__ armsL, uint32_t* __restrict__ armsR,
    uint4* __restrict__ pixL, uint4* __restrict__ pixR) {
    __shared__ dco::CensusLdsOf<TH> S;
    const bool r = (blockIdx.z & 1) != 0;
    const size_t P = (size_t)W * H, o = P * (blockIdx.z >> 1);
    dco::census_tile<64 * TH, TH>((r ? rgbR : rgbL) + 3 * o, W, H, cw, ch, L1, tau1, nullptr,
                                  (r ? armsR : armsL) + o, nullptr, (r ? pixR : pixL) + o, false,
                                  blockIdx.x * dco::kCenTW, blockIdx.y * TH, S);
}

// Rows of a census tile.  A tile of 16 rows is least work per pixel (its apron is
// shared by more rows), but a workgroup runs its pixels on one CU: where such
// tiles leave CUs idle, tiles of 8 rows finish sooner.  Both views of 64 x 48 in
// 6.1 us with 8 rows, 8.1 with 16; of 437 x 93 7.0 and 9.1 (4 rows: 5.7, 8.0).
constexpr int kSmallTiles = 256, kSmallRows = 8;

template <typename Go>
void with_tile_rows(int W, int H, int views, Go go) {
    const long long tiles = (long long)((W + dco::kCenTW - 1) / dco::kCenTW) * views;
    if (tiles * ((H + 15) / 16) > kSmallTiles)
        go(std::integral_constant<int, 16>{});
    else
        go(std::integral_constant<int, kSmallRows>{});
}

}  // namespace

hipError_t launch_census_pairs(const uint8_t* rgbL, const uint8_t* rgbR, int B, int W, int H,
                               int cw, int ch, int L1, int tau1, uint32_t* armsL, uint32_t* armsR,
                               uint4* pixL, uint4* pixR, hipStream_t st) {
    const size_t P = (size_t)W * H;
    constexpr int kMaxPairs = 16384;  // keeps gridDim.z = 2 * pairs within the launch limit
    for (int b0 = 0; b0 < B; b0 += kMaxPairs) {
        const int nb = B - b0 < kMaxPairs ? B - b0 : kMaxPairs;
        const size_t o = P * b0;
        with_tile_rows(W, H, 2 * nb, [&](auto rows) {
            constexpr int TH = decltype(rows)::value;
            const dim3 g((W + dco::kCenTW - 1) / dco::kCenTW, (H + TH - 1) / TH, 2 * nb);
            hipLaunchKernelGGL(k_census_pairs<TH>, g, dim3(64 * TH), 0, st, rgbL + 3 * o,
                               rgbR + 3 * o, W, H, cw, ch, L1, tau1, armsL + o, armsR + o,
                               pixL + o, pixR + o);
        });
    }
    return hipGetLastError();
}

hipError_t launch_front2(const uint8_t* rgbL, const uint8_t* rgbR, int W, int H, int cw, int ch,
                         int L1, int tau1, int iters, uint32_t* armsL, uint32_t* armsR,
                         uint4* pixL, uint4* pixR, const AggRecords& recL, const AggRecords& recR,
                         hipStream_t st) {
    with_tile_rows(W, H, 2, [&](auto rows) {
        constexpr int TH = decltype(rows)::value;
        const dim3 g((W + dco::kCenTW - 1) / dco::kCenTW, (H + TH - 1) / TH, 2);
        hipLaunchKernelGGL(k_census_arms2<TH>, g, dim3(64 * TH), 0, st, rgbL, rgbR, W, H, cw, ch,
                           L1, tau1, armsL, armsR, pixL, pixR, iters == 2);
    });
    dim3 g2((W + dco::kGeoTW - 1) / dco::kGeoTW,
            (dco::geo_rows(H) + dco::kGeoTH - 1) / dco::kGeoTH, 2);
    hipLaunchKernelGGL(k_geometry2, g2, dim3(1024), 0, st, armsL, armsR, W, H, iters, recL, recR);
    return hipGetLastError();
}

hipError_t launch_census_arms(const uint8_t* rgb, int W, int H, int cw, int ch, int L1, int tau1,
                              uint64_t* census, uint32_t* arms, uint32_t* rgb_packed, uint4* pix,
                              hipStream_t st) {
    with_tile_rows(W, H, 1, [&](auto rows) {
        constexpr int TH = decltype(rows)::value;
        const dim3 g((W + dco::kCenTW - 1) / dco::kCenTW, (H + TH - 1) / TH);
        hipLaunchKernelGGL(k_census_arms<TH>, g, dim3(64 * TH), 0, st, rgb, W, H, cw, ch, L1, tau1,
                           census, arms, rgb_packed, pix);
    });
    return hipGetLastError();
}

hipError_t launch_geometry(const uint32_t* arms, int W, int H, int iters, const AggRecords& rec,
                           hipStream_t st) {
    dim3 grid((W + dco::kGeoTW - 1) / dco::kGeoTW,
              (dco::geo_rows(H) + dco::kGeoTH - 1) / dco::kGeoTH);
    hipLaunchKernelGGL(k_geometry, grid, dim3(1024), 0, st, arms, W, H, iters, rec);
    return hipGetLastError();
}
