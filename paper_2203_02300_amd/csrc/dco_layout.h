// dco_layout.h -- sizes and per-pixel record layout that the aggregation
// kernels are built for (shared by host code and kernels; not part of the
// ABI).
#pragma once

#include <stddef.h>
#include <stdint.h>

// Largest arm length the kernels are built for.  The aggregation halo is
// 2 * kLMax columns/rows on each side of an output pixel.
constexpr int kLMax = 17;
// Threads of a streaming-aggregation workgroup = input columns of a strip.
constexpr int kStripThreads = 256;
// Output columns of one strip of the one-stage kernels.
constexpr int kStripOut = kStripThreads - 4 * kLMax;
// The two-stage kernel: a strip's 256 input columns start kWsI0 columns before
// image column kWsOut * s.  An inner strip has kWsOut output columns after an
// apron of kWsApron; the first and the last need no apron at the image's
// border and take kWsEdge more.  (All multiples of four: the kernel's lanes
// own aligned quads.)
constexpr int kWsI0 = 16;
constexpr int kWsApron = 36;
constexpr int kWsOut = 184;
constexpr int kWsEdge = kWsApron - kWsI0;
// Strips of an image W columns wide.  With the wider ones at the borders there
// are never more than the 188-column strips of the one-stage kernels give, up
// to W = 2064.
constexpr int agg_strips(int W, int iters) {
    if (iters != 2) return (W + kStripOut - 1) / kStripOut;
    const int n = (W - 2 * kWsEdge + kWsOut - 1) / kWsOut;
    return n > 0 && W > kWsOut + 2 * kWsEdge ? n : 1;
}

// Packed per-pixel records of one view for the aggregation kernels, written
// by k_geometry.  Entries of rows and columns outside the image are zero
// (zeroed once; only the image's are written).  Wp entries per row (a
// multiple of four); column x sits at x + kRecApronL.
// Two stages, with slot(r) = r mod 36 times the bytes of a ring row:
//   b row r (H + 2 kLMax rows of 16-byte entries), read at stream row r:
//     RN(1/N1), slots of rows y + dn and y - u - 1 (16 bits each)  of y = r - kLMax
//     the same slots + kLMax rows                                  of y = r - 2 kLMax
//     8 (r + 1) | 8 l << 8 (low half)                              of y = r
//     -N1 (high half)                                              of y = r - kLMax
//   c (three planes of H rows of words), read at output row y:
//     offsets of columns x + r + 1 and x - l in a row of prefixes (16 bits
//     each), RN(1/N2) 2^-20, N2 2^20 (floats)
// One stage, with hw = 4 (r + 1) | 4 l << 8 and rb the ring's byte offsets:
//   b row r: RN(1/N1) 2^-20, rb, hw | N1 << 16 (the fourth word is unused:
//     one 16-byte load per pixel is cheaper than a 12-byte one); hw of y = r,
//     the rest of y = r - kLMax
struct AggRecords {
    uint32_t* b;
    uint32_t* c;
    int Wp;
};
constexpr int kRecApronL = kWsApron;         // left apron of the records (2 kLMax at least)
constexpr int kRecApronR = kStripThreads;    // right apron (covers a strip's overhang)
constexpr int kWsRecRows = 2 * kLMax;        // rows of b past the image's
constexpr int rec_wp(int W) { return (W + kRecApronL + kRecApronR + 3) & ~3; }
constexpr size_t rec_b_words(int W, int H) { return 4 * (size_t)rec_wp(W) * (H + kWsRecRows); }
constexpr size_t rec_c_words(int W, int H) { return 3 * (size_t)rec_wp(W) * H; }

// Packed pixels of one view in planes, for the two-stage kernel: census lo,
// census hi and RGB words, then a plane of bytes holding 8 L_min.  Rows hold
// Wq = W rounded up to a multiple of four entries; kPixPad words before and
// after each word plane keep a quad that starts up to four columns before the
// image, or ends after it, inside the buffer (the values there are not used).
constexpr int kPixPad = 4;
struct PixPlanes {
    int Wq;
    uint32_t plane, H;  // words from one plane to the next, rows
    constexpr PixPlanes(int W, int rows)
        : Wq((W + 3) & ~3), plane((uint32_t)rows * ((W + 3) & ~3) + 2 * kPixPad),
          H((uint32_t)rows) {}
    constexpr uint32_t bytes() const { return 12 * plane + H * (uint32_t)Wq; }
};
// 16-byte entries of a view's packed pixels: the planes, or one word a pixel.
constexpr size_t pix_entries(int W, int H) {
    const size_t a = (size_t)W * H, b = (PixPlanes(W, H).bytes() + 15) / 16;
    return a > b ? a : b;
}
