// The shapes of the blocked row-walk kernel (blocked_rows.hip) and what they are expected to take; which plans take it:
// staged_rows.h.  Host code only.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "plan.h"

namespace sparsert {

constexpr int kBlockedRows = 84;      // rows of A per wave, at most
constexpr int kBlockedColumns = 16;   // columns of A whose rows of B a wave holds at a time
constexpr int kBlockedRecord = 20;    // words of a record of the stream

struct BlockedRows {
    int rows = 0, blocks = 0;         // rows per block; 0: the plan does not take this kernel
    int parts = 0;                    // waves of a workgroup, which split a block's columns: four or eight
    int lanes = 0, tiles = 0;         // columns of C per tile: twice the lanes
    int per_part = 0;                 // blocks that stand together in the order of the tasks
    double microseconds = 0;          // what it is expected to take
};

// Fitted to the products of the rule, each timed in up to twelve shapes (8 % root mean square): a start, a wave's
// nonzeros and columns (alone, or as many of them as share a SIMD), the exchange of the partial sums per workgroup of the busiest
// compute unit, eight waves at a time, and the results.  The shape it chooses is 1.007 times slower than the best one.
inline double blocked_rows_microseconds(const HostPlan &h, const BlockedRows &s) {
    const double density = (double)h.nnz / ((double)h.M * h.K);
    const double nonzeros = (double)h.nnz / s.blocks / s.parts, columns = h.K * (1.0 - std::pow(1.0 - density, s.rows)) / s.parts;
    const int64_t workgroups = (int64_t)s.blocks * s.tiles * h.batch;
    const double each = workgroups > 2048 ? workgroups / 256.0 : (double)((workgroups + 255) / 256), simd = each * s.parts / 4;
    return 2.91 + std::max(0.0088 * nonzeros + 0.00888 * columns, simd * (0.00346 * nonzeros + 0.0223 * columns))
         + 0.0237 * s.rows * simd + 2.66 * std::max(1.0, std::ceil(each * s.parts / 8)) + 0.21e-6 * h.M * (double)h.N * h.batch * 4;
}

// Blocks that stand together: the number for which the eight L2s, each of which has an eighth of the tasks, pull the least of the
// stream and of B.
inline int blocked_rows_per_part(const HostPlan &h, const BlockedRows &s) {
    const int64_t tasks = (int64_t)s.blocks * s.tiles, share = (tasks + 7) / 8;
    if (tasks > 16384) return s.blocks;   // (rounds enough to even it out, and the count below is not free)
    const double block = 5.5 * h.nnz / s.blocks, tile = 8.0 * h.K * s.lanes;
    int best = s.blocks;
    double least = 0;
    std::vector<int32_t> block_of((size_t)s.blocks), tile_of((size_t)s.tiles);   // the XCD that touched it last, counted from 1
    for (int parts = 1; parts <= 16 && parts <= s.blocks; ++parts) {
        const int per = (s.blocks + parts - 1) / parts;
        double bytes = 0;
        std::fill(block_of.begin(), block_of.end(), 0);
        std::fill(tile_of.begin(), tile_of.end(), 0);
        for (int64_t t = 0; t < tasks; ++t) {
            const int xcd = (int)(t / share) + 1, part = (int)(t / ((int64_t)per * s.tiles)), in = (int)(t - (int64_t)part * per * s.tiles);
            const int here = std::min(per, s.blocks - part * per), b = part * per + in % here, n = in / here;
            if (block_of[b] != xcd) { block_of[b] = xcd; bytes += block; }
            if (tile_of[n] != xcd) { tile_of[n] = xcd; bytes += tile; }
        }
        if (parts == 1 || bytes < least) { least = bytes; best = per; }
    }
    return best;
}

// The shape that is expected to take the least, its per_part still open.  fp32, no more than a fifth of A kept, at least 64 rows and 49
// columns: what the products that the estimate was fitted to are like.  Below, the choice would not hold: of eleven products of 1 to 20 rows four
// were slower blocked (1 x 12870 x 229, batch 64, at 82 % 57.3 -> 73.7 us), of sixteen of 1 to 48 columns two, 1.9 times (136 x 10639 x 8, batch
// 64, at 89 % 88.7 -> 165.8 us).  Beyond 4096 rows or columns of A, or a batch of 4, it does: fourteen of 372 to 3218 rows, K from 4996 to
// 14174, batches of up to 64, 0.75 times the time on average and 1.02 at most.
inline BlockedRows blocked_rows_candidate(const HostPlan &h) {
    BlockedRows best;
    if (h.dtype != SPARSERT_F32 || h.M < 64 || h.N < 49 || (int64_t)h.nnz * 5 > (int64_t)h.M * h.K || (int64_t)h.nnz >= 1 << 28) return best;
    BlockedRows s;
    s.tiles = (h.N + 2 * kWave - 1) / (2 * kWave);
    s.lanes = ((h.N + s.tiles - 1) / s.tiles + 1) / 2;
    for (int rows = std::min<int>(kBlockedRows, h.M), last = 0; rows >= 16; --rows) {
        s.blocks = (h.M + rows - 1) / rows;
        if (s.blocks == last) continue;
        last = s.blocks;
        s.rows = (h.M + s.blocks - 1) / s.blocks;
        if ((int64_t)s.blocks * s.tiles > (1 << 24)) break;
        for (s.parts = 4; s.parts <= 8; s.parts += 4) {
            s.microseconds = blocked_rows_microseconds(h, s);
            if (best.rows == 0 || s.microseconds < best.microseconds) best = s;
        }
    }
    return best;
}

}  // namespace sparsert
