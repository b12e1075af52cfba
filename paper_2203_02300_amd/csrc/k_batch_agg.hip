// k_batch_agg.hip -- the batched matcher's cost + two-stage aggregation (stage
// 2 of k_batch.hip), in a file of its own so that it is compiled with the
// machine scheduler that the aggregation body needs (build.py): eight mixed
// pairs of 320x240 to 1280x720 take 3.71 ms with it and 4.16 ms with the default
// one, which suits the other stages better.
#include "dco_batch.h"
#include "dco_device.h"

namespace {

// Stage 2 with two aggregation stages: slices a .. a + dchunk - 1 of strip b,
// row band c, two adjacent disparities per pass of dco::agg_stream_ws (768
// threads, one workgroup per CU).  The workgroups of XCD x take that XCD's
// contiguous part of the list, one item each.
__global__ __launch_bounds__(dco::kWsThreads, 1) void k_batch_agg_ws(BatchArgs B, int first) {
    __shared__ dco::AggLdsWs S;
    const int x = blockIdx.x % kXcds;
    const int k = B.xsplit[x] - first + blockIdx.x / kXcds;
    if (k >= B.xsplit[x + 1] - first) return;  // uniform
    const BatchItem I = B.items[first + k];
    const BatchPair& pr = B.pairs[I.pair];
    dco::AggArgs A{};
    A.pixL = pr.pix[0];
    A.pixR = pr.pix[1];
    A.tabA = B.tabA;
    A.tabC = B.tabC;
    A.alpha = B.alpha;
    A.beta = B.beta;
    A.rec = pr.rec[I.view];
    A.out = pr.agg[I.view];
    A.W = pr.W;
    A.pitch = pr.W;
    A.H = pr.H;
    A.D = pr.D;
    A.nstrips = pr.nstrips;
    A.ref = I.view;
    A.L1 = B.L1;
    // with an even chunk every pass starts at an even slice, so the passes'
    // slice pairs are the layout's pairs; stage 3 reads the even slices
    A.paired = pr.dchunk % 2 == 0;
    const int y0 = I.c * pr.band, y1 = min(pr.H, y0 + pr.band);
    const int dend = min(pr.D, I.a + pr.dchunk);
    for (int d = I.a; d < dend; d += dco::kWsSlices) {
        dco::agg_stream_ws(A, d, dend, I.b, y0, y1, S);
        __syncthreads();
    }
}

}  // namespace

void launch_batch_agg_ws(const BatchArgs& a, int first, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_batch_agg_ws, dim3(grid), dim3(dco::kWsThreads), 0, st, a, first);
}

int batch_agg_ws_per_cu() {
    int nb = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_batch_agg_ws,
                                                                      dco::kWsThreads, 0);
    return e == hipSuccess && nb > 0 ? nb : 1;
}
