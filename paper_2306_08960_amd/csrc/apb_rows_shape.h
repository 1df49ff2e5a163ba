// Launch shapes of the matrix-core forward kernel (apb_rows.hip): arithmetic on sizes only, kept apart from the device
// code so that a host compiler can walk it over the sizes the entry points accept.
#pragma once

#include <algorithm>
#include <cmath>

namespace apb {

constexpr int kComputeUnits = 256;                             // of the MI355X
constexpr int kMaxLdsBytes = 160 * 1024;
constexpr int kFloatRows = 128;                                // rows a workgroup of the one-kernel step holds at most

// What the choice depends on.
struct RowsProblem {
    int N, M;
    int ksteps;                                                // K in steps of 128, rounded up
    int bits;                                                  // of the input
    bool general;                                              // see rows_item
    bool packed_out;
    bool from_float;                                           // the one-kernel step
};

struct RowsShape {
    int groups;                                                // column groups of 16 per workgroup (1, 2 or 4)
    int nt, ncw;                                               // an item: nt tiles of 16 rows x ncw column groups
    int waves;                                                 // per workgroup
    int chunk;                                                 // tiles per workgroup, a multiple of nt
};

// Tiles of 16 rows: an even number, so that two of them make a word of a packed output.
inline int rows_tiles(int N) { return 2 * (N / 32 + (N % 32 != 0)); }

// Where the columns-in-lanes kernel (apb_sparse.hip) is the faster one: few residuals per row and many outputs.  There a
// residual costs four instructions for 64 columns; here a pair of rows takes at least one digit step, of which a layer of 6
// residuals per row fills a tenth, and the epilogue of a short K weighs more than its products.  Residuals per row up
// to which it wins, fitted to both kernels over K 96 .. 1152, N 32 .. 512, M 8192 .. 131072 and 1 .. 24 residuals per
// row (N = 64, K = 288, M = 131072, 6 per row: the step 48 us here, 39 there, packed output 22 and 18; K = 576, 12
// per row: 72 and 64; N = 64, K = 1152, M = 50176, 6 per row: 53 and 54, 16 and 18).  A packed output of more than 128
// rows takes it atomics.  The rule looks at nothing but sizes and the kind of output: a step gives the same bits as
// its two calls.
inline double columns_kernel_residuals(int N, int K, int M, bool packed_out) {
    if (packed_out) return N <= 128 && M >= 40000 ? 12.0 - K / 96.0 : -1.0;
    if (N <= 32 || (N <= 64 && M < 90000)) return M >= 60000 ? 12.0 - K / 64.0 : -1.0;
    if ((long long)N * M < 4000000) return -1.0;
    return N <= 128 ? 20.0 - K / 96.0 : 8.0 - K / 200.0;
}
inline bool columns_kernel_better(int N, int K, long long nnz, int M, bool packed_out) {
    return (double)nnz <= columns_kernel_residuals(N, K, M, packed_out) * N;
}
inline bool columns_kernel_possible(int N, int K, long long nnz) {     // for some M
    const int most = 0x7fffffff;
    return columns_kernel_better(N, K, nnz, most, false) || columns_kernel_better(N, K, nnz, most, true);
}

// Quantize + forward in one kernel: where one workgroup holds every row of the layer, so that no column of X is
// quantized twice, and the columns fill the chip (a narrow tail of them would read X with too few waves; 24000 columns:
// 128 x 1152 26 us against 34 as two kernels, 128 x 2304 48 and 62, 64 x 2304 42 and 59; the line is a careful one: at
// 16384 columns 128 x 1152 takes 21 and 29); and where X is so small (a quarter of a MB: every workgroup's share comes
// from the L2) or K so short (K <= 512, 65 to 128 rows, up to 23000 columns: 11.0 .. 12.5 us against 13.9 .. 15.8 as two
// kernels) that the launch saved is worth more.
inline bool rows_from_float(int N, int K, int M) {
    if ((long long)K * M <= 65536) return true;
    if (N > kFloatRows || (K + 127) / 128 > 38) return false;
    return N <= kFloatRows / 2 || M >= 64 * 375 || K <= 512;
}

// LDS of a workgroup: the tables, one step that the binary part reads past them, the code sums of the columns, and per
// row the affine map of a packed output and the sums that 1-bit inputs need.
inline long long rows_lds_bytes(const RowsProblem& q, int groups, int chunk) {
    return (long long)groups * (q.ksteps * 1024 + 128) + 1024 +
           16LL * chunk * ((q.packed_out ? 8 : 0) + (q.bits == 1 ? 12 : 0));
}

// How many tiles a workgroup takes (of all, shared evenly) and how many waves work on them.  The time of a launch,
// in units of a fifth of an item (an item alone on its SIMD takes five): rounds of workgroups on the chip, times the
// items a wave takes one after another (two waves on a SIMD take 1.5 times as long, four 2.5 times: the matrix cores,
// the LDS and the L1 fill are shared, latencies overlap) and the table build (three items' time for one wave, shared).  From
// four rounds on the last one's emptiness no longer counts, and a split has to gain 3 %.  Next
// to large tables the rows' own sums may leave room for a share of the tiles only.
inline void rows_spread(const RowsProblem& q, RowsShape& h, long long cts, int max_waves, int waves_per_cu) {
    const int tiles = rows_tiles(q.N), shares = h.groups / h.ncw;
    double best = 1e300;
    int chunk = (tiles + h.nt - 1) / h.nt * h.nt;
    while (chunk > h.nt && rows_lds_bytes(q, h.groups, chunk) > kMaxLdsBytes) chunk = (chunk / 2 + h.nt - 1) / h.nt * h.nt;
    for (;;) {
        const int lds = (int)rows_lds_bytes(q, h.groups, chunk) + 896 * h.groups;   // (in kilobytes per column group)
        const long long items = (long long)chunk / h.nt * shares, parts = ((long long)tiles + chunk - 1) / chunk;
        int waves = shares;
        while (waves < max_waves && waves < items) waves *= 2;
        const long long wgs = cts * parts;
        const int fit = std::max(1, std::min(kMaxLdsBytes / lds, waves_per_cu / waves));
        const long long per_cu = std::min<long long>(fit, (wgs + kComputeUnits - 1) / kComputeUnits);
        const double rounds = wgs <= (long long)kComputeUnits * per_cu ? 1.0 : (double)wgs / (kComputeUnits * per_cu);
        const int active = (int)std::min<long long>(waves, items);
        const double crowd = 0.5 + 0.5 * (double)((per_cu * active + 3) / 4);
        const double cost = (rounds > 1.0 && rounds < 4.0 ? std::ceil(rounds) : rounds) * (5.0 * ((items + waves - 1) / waves) * crowd + 16.0 / waves);
        if (cost < best * 0.97) {                                // (fewer workgroups where it makes no difference)
            best = cost;
            h.chunk = chunk;
            h.waves = waves;
        }
        if (chunk <= h.nt) break;
        chunk = (chunk / 2 + h.nt - 1) / h.nt * h.nt;
    }
}

inline RowsShape pick_rows_shape(const RowsProblem& q) {
    RowsShape h{};
    const int tiles = rows_tiles(q.N), ksteps = q.ksteps;
    const long long ct16 = ((long long)q.M + 15) / 16, ct64 = ((long long)q.M + 63) / 64;
    if (q.general) {
        h.groups = ksteps <= 72 ? 2 : 1;
        h.nt = h.ncw = 1;
        rows_spread(q, h, ((long long)q.M + 16 * h.groups - 1) / (16 * h.groups), 8, 16);
        return h;
    }
    if (q.from_float && q.N <= kFloatRows && ct16 >= 4 * kComputeUnits) {
        // Rows of X are read 64 or 32 columns (two or one lines of memory) at a time, by a workgroup that has all rows of the layer.
        h = RowsShape{tiles <= 4 ? 4 : 2, 2, 2, 4, tiles};
        return h;
    }
    if ((ct16 + 1) / 2 * (tiles / 2) < 4 * kComputeUnits && (ksteps <= 19 || ct64 * tiles < 2 * kComputeUnits || ksteps > 38)) {
        // Few items: single tiles of one column group, in as many workgroups as give every SIMD of the chip a wave.
        // (A column group alone may have more workgroups than that: the doubling ends at all tiles.)
        h = RowsShape{1, 1, 1, 2, 2};
        while (h.chunk < tiles && ct16 * ((tiles + h.chunk - 1) / h.chunk) > 4 * kComputeUnits) h.chunk *= 2;
        // A packed output whose rows sit in several workgroups needs a launch that clears the column sums first (2 us);
        // up to 256 rows of not too long a K are done sooner by one (192 x 4608, 256 columns: 12.1 us and 11.5; 256 x 4608:
        // 12.1 and 13.1; 256 x 2304 and less: 12.1 and 10.0).
        if (q.packed_out && tiles <= 16 && tiles * ksteps <= 450) h.chunk = tiles;
        h.waves = std::min(8, h.chunk);
        // Where that leaves compute units to spare, more waves build the tables of a long K (2115 x 2574 in skewed rows, 39
        // columns: step 17.4 us with two waves, 17.0 with eight; 4096 x 4096, 16 columns: 21.5 and 12.7).
        while (2 * h.waves <= std::min(8, ksteps) && ct16 * ((tiles + h.chunk - 1) / h.chunk) * 2 * h.waves <= 8 * kComputeUnits) h.waves *= 2;
        return h;
    }
    if (ksteps > 19 && ksteps <= 38) {
        // Long K, one workgroup per CU whatever the shape: 64 columns per item, so that a digit step fetched through the
        // L1 (64 bytes a clock: 22 clocks) serves four matrix instructions.
        h = RowsShape{4, 1, 4, 8, tiles};
        rows_spread(q, h, ct64, 8, 8);
        h.waves = 8;                                             // (at least two waves per SIMD to build 150 KB of tables)
        return h;
    }
    h.groups = ksteps <= 19 && tiles <= 4 ? 4 : 2;
    h.nt = h.ncw = 2;
    rows_spread(q, h, ((long long)q.M + 16 * h.groups - 1) / (16 * h.groups), 8, 16);
    return h;
}

}  // namespace apb
