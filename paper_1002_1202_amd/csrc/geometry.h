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
//
// ragged: the last chunk is far from full (ragged_end).  Its workgroups cost little
// beside the others, so each XCD takes an eighth of its rows, a run of 32 (one for
// each of an XCD's CUs) after every 32 (gx - 1) of an equal share of the full chunks.
// With that chunk as a full one, its XCDs wait for the others (3 chunks, the last of
// 2 columns: 4,096 Si 116 -> 103 ms, 256 H2O 76 -> 53, 3,000 H2O 372 -> 328; 4
// chunks 148 -> 137, 89 -> 62, 475 -> 438).
constexpr int kRaggedRun = 32;
GSC_HOST_DEVICE inline void chunk_order(int l, int gx, int G, bool ragged, int &cx, int &gy) {
    const int x = l & 7, full = ragged ? gx - 1 : gx;
    int k = l >> 3;
    if (ragged) {
        const int w = k / (gx * kRaggedRun), left = G / 8 - w * kRaggedRun;
        const int run = left < kRaggedRun ? left : kRaggedRun, pos = k - w * gx * kRaggedRun;
        if (pos >= full * run) {
            cx = full;
            gy = x * (G / 8) + w * kRaggedRun + pos - full * run;
            return;
        }
        k -= w * kRaggedRun;
    }
    const int whole = full / 8 * G;
    if (k < whole) {
        cx = x + 8 * (k / G);
        gy = k % G;
        return;
    }
    k += x * (full % 8) * (G / 8) - whole;
    cx = full / 8 * 8 + k / G;
    gy = k % G;
}

// Whether the last chunk (`width` columns) of a launch whose columns end at `end` is
// ragged, of R columns in all: at least a quarter is empty.  Beyond that the rows of
// several chunks in one L2 cost more than the waiting (4 chunks, the last of 56
// columns, as a ragged and as a full one: 256 H2O 64.4 | 63.1 ms, 3,000 H2O 489 |
// 484; of 48: 63.7 | 63.4, 483 | 486; of 32: 62.6 | 62.4, 463 | 474).
GSC_HOST_DEVICE inline bool ragged_end(int end, int R, int width) { return 4 * (end - R) >= width; }

}  // namespace gsc
