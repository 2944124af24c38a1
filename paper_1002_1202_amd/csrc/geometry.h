// Launch geometry of the product kernels: whole numbers only, so that the rules
// can be checked without a device.
#pragma once

#ifdef __HIPCC__
#define GSC_HOST_DEVICE __host__ __device__
#else
#define GSC_HOST_DEVICE
#endif

namespace gsc {

// Place (column chunk cx, row group gy) of workgroup l of a launch over gx
// chunks and G row groups (a multiple of 8); workgroups go to the 8 XCDs in turn
// (l mod 8).  Every XCD walks chunks one after the other, each over consecutive
// row groups: the x rows that a chunk needs (its rows and the neighbour halo) then
// come into one L2 instead of eight, and one window of one chunk is what that L2
// has to hold.  As many whole chunks as go to all XCDs alike; the gx mod 8 left
// over are one sequence of (chunk, group) cut into eight equal slices.
// Against all chunks of a row window side by side, at counts that neither divide
// 8 nor are its multiples (FP64 charges of 256 H2O, 16 shifts, ms a solve): 22
// chunks 380 -> 215, 19 chunks 311 -> 192, 12 chunks 169 -> 136; 4,096 Si x 7
// chunks 279 -> 274; 1, 2, 4, 8, 16 and 24 chunks the same within the runs' spread.
GSC_HOST_DEVICE inline void chunk_order(int l, int gx, int G, int &cx, int &gy) {
    const int x = l & 7, whole = gx / 8 * G;
    int k = l >> 3;
    if (k < whole) {
        cx = x + 8 * (k / G);
        gy = k % G;
        return;
    }
    k += x * (gx % 8) * (G / 8) - whole;
    cx = gx / 8 * 8 + k / G;
    gy = k % G;
}

}  // namespace gsc
