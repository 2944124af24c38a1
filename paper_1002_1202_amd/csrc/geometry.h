// Launch geometry of the product kernels: whole numbers only, so that the rules
// can be checked without a device.
#pragma once

#include <algorithm>
#include <cstdint>

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

// ------------------------------------------------------------------ row groups
inline int up8(int64_t g) { return static_cast<int>((std::min<int64_t>(g, 65528) + 7) / 8 * 8); }

// Groups of four block rows (one wave each): one row a wave while a launch
// stays within 16384 workgroups, else about 4096 workgroups with equal rows
// per wave, at least 256 groups when there are more than 8 column chunks (an
// XCD would otherwise run the groups of several chunks at once).
inline int one_wave_groups(int64_t nb, int chunks) {
    const int64_t slots = std::max<int64_t>(1, (nb + 3) / 4);
    int64_t g = slots;
    if (chunks * slots > 16384) {
        int64_t g0 = std::max(1, 4096 / chunks);
        if (chunks > 8) g0 = std::max<int64_t>(g0, 256);
        g0 = std::min(g0, slots);
        const int64_t passes = (slots + g0 - 1) / g0;
        g = (slots + passes - 1) / passes;
    }
    return up8(g);
}

// Row groups (multiples of 8) of the product launches: a group is one workgroup a
// column chunk and takes a block row (four with one wave a row) in turn, every Gth.
struct RowGroups {
    int Gs;       // launches with one matrix that leave partial sums per group and column
    int Gw;       // launches that leave none and share a row
    int G1;       // launches that leave none, one wave a row
    int G2;       // whole products with partial sums (of the seed, of Lanczos, of the inner CG)
    int waves2;   // waves they give a row, four or one
};

// Whether block rows are long: a wave gathers row_orbitals (stored blocks times B)
// orbital rows of x for one.  Measured at 68 (Si, 17 blocks of 4) and 162 (water, 27
// of 6); the line lies between.
inline bool long_rows(int64_t row_orbitals) { return row_orbitals >= 112; }

// Waves that the whole products with partial sums (S and H: the seed product, the
// Lanczos product; S: the inner CG) give a block row. Their groups take up to four rows
// in turn, and the two sums a lane of S and H leave 5 waves on a SIMD against 8, so
// with short rows and enough of them to fill the card one wave a row is ahead; the
// chain of loads of a long row is worth sharing at every size. Runs of 30 iterations,
// ms, one wave / four. Short: 512 rows x 512 columns 11.1 / 11.3, 1,024 x 320 13.5 /
// 13.7, 2,048 x 128 11.4 / 11.5, 4,096 x 64 11.8 / 11.9, 4,096 x 256 29.5 / 29.8, 8,192
// x 64 19.5 / 19.8, 18,432 x 64 80.2 / 80.7; below the line 512 x 64 5.5 / 4.5, 1,024 x
// 64 6.0 / 5.7, 2,048 x 64 7.6 / 7.4. Long: 3,000 H2O x 128 30.9 / 30.6, x 192 43.6 /
// 42.9, x 256 53.3 / 52.5, x 512 110 / 109; mixed x 192 39.2 / 38.1, x 256 42.7 / 41.9.
// Inner CG, 10 iterations, short rows: 18,432 x 190 columns 185 / 191, 18,432 x 64 59.0
// / 60.6, 4,096 x 64 9.6 / 9.8, 4,096 x 256 22.3 / 23.1.
inline int product_waves(int64_t nb, int chunks, int64_t row_orbitals) {
    return !long_rows(row_orbitals) && nb * chunks >= 4096 ? 1 : 4;
}

// Waves that a launch of Chebyshev steps (or of their residuals) gives a block row;
// narrow: complex64 with one column a lane. Four, except for short rows in launches of
// one chunk with enough rows: the waves of one chunk then fill the card without
// sharing, whose LDS pass and barriers are left as cost. Runs of 30 iterations with 64
// columns, ms, four / one: FP64 8,192 rows 19.5 / 20.2, 12,288 30.1 / 29.3, 18,432 83.1
// / 80.2, 32,768 74.7 / 72.8; mixed 2,048 rows 7.7 / 7.9, 4,096 12.0 / 12.0 (8 columns
// 10.3 / 10.0), 8,192 19.3 / 19.0, 12,288 26.0 / 25.0, 18,432 70.3 / 66.4, 32,768 63.1
// / 60.4. Two chunks and more, or two columns a lane, mixed: 8,192 rows x 128 columns
// 27.0 / 29.2. Long rows (with the seed product), 12,000 H2O x 64 columns: FP64 60.6 /
// 62.8, mixed 49.0 / 53.7.
inline int step_waves(int64_t nb, int chunks, int64_t row_orbitals, bool narrow) {
    return !long_rows(row_orbitals) && chunks == 1 && nb >= (narrow ? 4096 : 12288) ? 1 : 4;
}

// For a tile of `chunks` column chunks, `width` of them in a Chebyshev launch;
// one_wave: every launch gives a row one wave.  Launches that leave no partial sums
// give every block row its own workgroup (1, 2, 4 and 8 rows a workgroup on the
// Chebyshev step: 4,096 Si x 128 columns 35.8 / 38.2 / 40.8 / 35.6 us, 2,668 Si x
// 128 25.2 / 27.7 / 29.5 / 31.8, 64 H2O x 384 9.5 / 11.9 / 18.7 / 35.5).  Those that
// leave them take up to four rows a group, as many as bring the groups to about 1024
// and the workgroups of the tile's chunks to about 1024 (the reductions read every
// group's value of every column), and never more: with 1024 groups whatever the rows,
// a launch of one chunk is too small for the card (N 131,072, 60 seed products of 8
// chunks 115 ms, now 73).  Fewer rows a group than that, 4 / 2 / 1 at 8,192 rows x
// 128 columns 30.7 / 32.5 / 36.9 ms a run; at 512 rows x 512 columns 19.5 / 20.0 /
// 20.4, 256 x 1024 21.1 / 21.5 / 22.4, 1,024 x 1024 55.4 / - / 57.1, 256 H2O x 1024
// 39.4 / 39.9 / 40.7.  One wave a row never takes more groups than that needs: the
// groups beyond the last row would be whole XCDs' share (2,048 Si x 256 columns, seed
// product 65 -> 42 us).
inline RowGroups row_groups(int64_t nb, int chunks, int width, int64_t row_orbitals, bool one_wave) {
    RowGroups g;
    g.G1 = one_wave_groups(nb, width);
    g.Gw = up8(nb);
    const int64_t rows = std::min<int64_t>(4, std::max((nb + 1023) / 1024, nb * chunks / 1024));
    g.Gs = one_wave || rows == 4 ? g.G1 : up8((nb + rows - 1) / rows);
    g.waves2 = one_wave ? 1 : product_waves(nb, chunks, row_orbitals);
    g.G2 = g.waves2 == 1 ? g.G1 : g.Gs;
    return g;
}

// The same with a caller's number of groups (gsc_opts.row_groups), each of four block
// rows as in the automatic rule beyond 3,072 rows: launches that share rows without
// partial sums take four workgroups for one group, so that as many rows are in flight.
inline void set_groups(RowGroups &g, int64_t nb, int asked) {
    const int64_t slots = (nb + 3) / 4;
    g.Gs = g.G1 = g.G2 = up8(std::min<int64_t>(asked, slots));
    g.Gw = up8(std::min<int64_t>(4 * static_cast<int64_t>(asked), nb));
}

// ------------------------------------------------------------------ small systems
// Whether one workgroup a column (small.hip) also carries the full x^k and p^k of K
// shifts of N orbitals: their update is one CU's traffic there and the card's on the
// tiles.  (The projected carries are ahead at every K measured, up to 4096.)  One
// workgroup | tiles, ms, 8 columns, shifts over the whole spectrum: N 512 K 1024 33 |
// 41, K 2048 53 | 48, K 4096 92 | 64; N 384 K 2048 38 | 46, K 4096 70 | 60; N 144 K
// 2048 43 | 57, K 4096 76 | 69.  All shifts inside a band (none finishes early): N
// 512 K 512 35 | 43, K 1024 56 | 52; N 384 K 1024 39 | 48, K 2048 71 | 61; N 256 K
// 1024 29 | 47, K 2048 55 | 59; N 144 K 1024 65 | 70, K 2048 124 | 93.  The line
// lies between the two kinds of grids.
inline bool small_full_carry(int64_t N, int64_t K) { return K <= 2048 && N * K <= 5 << 17; }

}  // namespace gsc
