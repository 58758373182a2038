// Which plans take the staged row-walk kernel (staged_rows.hip) or the blocked one (blocked_rows.hip), and the shape of the staged one.
// Host code only.
#pragma once
#include <algorithm>
#include <cstdint>

#include "blocked_rows.h"
#include "plan.h"

namespace sparsert {

constexpr int kStagedWaves = 16;            // waves per workgroup
constexpr int kStagedLdsBytes = 160 * 1024;
constexpr int kStagedTouchBytes = 256;      // corner of LDS that the stream's cache-line touches land in

struct StagedRows {
    int V = 0;             // columns per lane; 0: the plan does not take this kernel
    int rows_per_wave = 0; // 4 or 8
    int lanes = 0, tiles = 0, groups = 0;   // lanes that own columns, column tiles, row groups
    int pitch = 0;         // bytes of a row of the tile in LDS
    int chunk = 0, chunks = 0;   // rows of B per LDS buffer
    double microseconds = 0;     // what it is expected to take
    bool short_shares = false;   // pairs in steps of four at most
};

// The estimates below are fits to 230 products drawn from M, K <= 4096, N from 49 to 4096 and 80 % to 98 %
// zeros (126 fp32, the rest half and int8; a quarter of them with skewed rows), timed with steps of four pairs and a v_dot4
// per row and column.  Microseconds.  Against the kernels as they are (700 products drawn from the same ranges whose first two estimates
// are within 0.35 to 1.5 of each other, each timed with both kernels), root mean square: staged fp32 12 % to 20 %, half 10 %,
// int8 30 % (1.24 times too long), plain 22 % to 25 %.

// Staged: a start, then per round of workgroups a fixed cost per chunk (barrier, first loads), the copied
// bytes and the operands read from LDS; the longest row as one wave's serial
// chain, whatever else runs; and the results.
inline double staged_rows_microseconds(const HostPlan &h, const StagedRows &s, int32_t longest, const double (*fit)[6]) {
    const double *f = fit[h.dtype == SPARSERT_I8 ? 4 : h.dtype == SPARSERT_F16 ? 3 : s.V == 4 ? 2 : s.rows_per_wave / 8];
    const int esz = h.elem_size(), slots = s.groups * kStagedWaves * s.rows_per_wave;
    const double wgs = (double)s.groups * s.tiles * h.batch;
    const double rounds = wgs > 1024 ? wgs / 256 : (double)(((int64_t)wgs + 255) / 256);
    const double pairs = (double)h.nnz / s.groups + 0.5 * s.chunks * kStagedWaves * s.rows_per_wave * std::min(1.0, (double)h.M / slots);
    return f[0] + rounds * (f[1] * s.chunks + 1e-6 * f[2] * h.K * s.pitch + 1e-6 * f[3] * pairs * kWave * s.V * esz)
         + 1e-3 * f[4] * longest + 1e-6 * f[5] * h.M * h.N * (double)h.batch * h.out_elem_size();
}
inline double staged_rows_microseconds(const HostPlan &h, const StagedRows &s, int32_t longest) {
    static const double fit[5][6] = {{1.83, 0.913, 0.43, 4.13, 15.9, 0.335},   // fp32, V = 2, four rows
                                     {2.18, 0.873, 2.38, 4.05, 15.6, 0.260},   // fp32, V = 2, eight rows
                                     {2.14, 0.481, 5.69, 2.48, 18.9, 0.259},   // fp32, V = 4
                                     {2.26, 0.941, 0.00, 4.47, 18.8, 0.367},   // half
                                     {2.44, 0.326, 3.85, 12.7, 22.9, 0.231}};  // int8
    return staged_rows_microseconds(h, s, longest, fit);
}

// Plain: the wave loads of B (one per nonzero and column tile; part of the cost is per load, part per byte),
// the longest chain of one wave, and the results.
inline double plain_rows_microseconds(const HostPlan &h, int32_t longest) {
    static const double fit[3][5] = {{2.42, 0.58, 0.69, 2.23, 0.44}, {2.78, 0.69, 0.79, 2.11, 0.50}, {2.53, 0.82, 1.11, 2.44, 0.34}};
    const double *f = fit[h.dtype == SPARSERT_F32 ? 0 : h.dtype == SPARSERT_F16 ? 1 : 2];
    const double chain = longest < h.split_threshold ? longest : longest / (double)kGy;
    return f[0] + 1e-5 * (double)h.nnz * h.n_tiles * h.batch * (f[1] + f[2] * h.vec * h.elem_size() / 4.0)
         + 1e-2 * f[3] * chain + 1e-6 * f[4] * h.M * h.N * (double)h.batch * h.out_elem_size();
}

// Second estimates of both, fitted to 5303 products of the same ranges that the first ones give to the staged kernel, each
// timed with both kernels, also before the steps of eight: 6 % and 13 % root mean square then; over the 700 above staged fp32 7 % to 15 %,
// half 11 %, int8 32 % (1.27 times too long), plain 13 % to 15 %.  (fp32 at V = 4 is of the kernel whose values reached the multiply-adds in scalar
// registers: over 60 products that take it the estimate is 1.11 times too long for the present one, 12 % root mean square, so that some that staging would
// gain stay plain; of the 60 one is slower for being staged, 1.1 times, 0.49 times the plain kernel's time on average.)  The plain kernel's loads cost by columns per lane, and more where
// rows of B do not begin on 64 bytes; every wave costs something of its own.
inline double staged_rows_microseconds_again(const HostPlan &h, const StagedRows &s, int32_t longest) {
    static const double fit[5][6] = {{2.26, 0.81, 5.68, 3.64, 14.1, 0.219}, {2.41, 1.40, 2.92, 3.88, 7.12, 0.183}, {2.57, 0.847, 3.68, 2.82, 4.91, 0.176},
                                     {2.23, 0.984, 1.70, 5.78, 11.0, 0.275}, {2.54, 0.803, 4.89, 14.9, 10.9, 0.170}};
    return staged_rows_microseconds(h, s, longest, fit);
}
inline double plain_rows_microseconds_again(const HostPlan &h, int32_t longest) {
    static const double plain[3][9] = {{1.84, 0.856, 2.71, 3.09, 0.00, 0.167, 2.77, 16.1, 0.0412},    // fp32: launch, loads at 1, 2, 4, 8 columns per lane,
                                       {1.69, 0.760, 0.887, 2.67, 3.28, 0.176, 2.81, 17.8, 0.0},      // half  off 64 bytes, the longest chain, waves, results
                                       {2.04, 0.754, 0.00, 1.39, 0.00, 0.138, 2.33, 17.9, 0.062}};    // int8
    const double *f = plain[h.dtype == SPARSERT_F32 ? 0 : h.dtype == SPARSERT_F16 ? 1 : 2];
    const double chain = longest < h.split_threshold ? longest : longest / (double)kGy, loads = 1e-5 * (double)h.nnz * h.n_tiles * h.batch;
    const int v = h.vec == 1 ? 1 : h.vec == 2 ? 2 : h.vec == 4 ? 3 : 4;
    return f[0] + loads * (f[v] + ((int64_t)h.ldb * h.elem_size() % 64 ? f[5] : 0.0)) + 1e-2 * f[6] * chain
         + 1e-5 * f[7] * h.M * h.n_tiles * (double)h.batch + 1e-6 * f[8] * h.M * h.N * (double)h.batch * h.out_elem_size();
}
inline bool staged_rows_confirmed(const HostPlan &h, const StagedRows &s, int32_t longest) {
    return staged_rows_microseconds_again(h, s, longest) < plain_rows_microseconds_again(h, longest) + 1.4;   // (what the two are off by at 10 to 20 us)
}

// What the kernel's addressing holds: the pair stream, with at most one filler per row and chunk and the padding
// at its end, under 2 GiB (its touches go through a descriptor with 32-bit offsets), and a launch of less than
// 2^32 threads.  Larger plans stay with the plain kernel, which counts pairs and not bytes.
inline bool staged_rows_fits(const HostPlan &h, const StagedRows &s) {
    const int64_t pairs = (int64_t)h.nnz + (int64_t)h.M * s.chunks + 16, tasks = (int64_t)s.tiles * s.groups;
    return pairs * 8 < (1ll << 31) && (tasks + 7) / 8 * 8 * kStagedWaves * kWave < (1ll << 32);
}

// The staged kernel pays where many nonzeros share a workgroup's copy of B; few columns, few rows, a long K
// with few nonzeros per chunk, or one row much longer than the rest leave it behind (1/2 to 2 times the plain
// kernel's time over the products above), so it is taken where it is estimated to need less than 0.8 of the
// plain kernel's time and the second estimates do not contradict that.  Of 5303 drawn products that pass the first test
// 5138 pass the second; they gain 1.51 times on average, 133 lose more than 5 % (0.80 times the plain kernel's speed
// at worst; 263 and 0.62 with the first test alone), and 8 that gained more than 5 % are given up.  (With the kernel of that time.
// The present one loses less: of the 700, 252 are taken, two of them 11 % slower at most; and of the rest 152 would gain more
// than 5 %, 74 of them int8, 31 half, 1.31 times on average and 3.4 times at most, fp32 with skewed rows.)
inline StagedRows staged_rows_candidate(const HostPlan &h, int32_t longest) {
    StagedRows best;
    const int esz = h.elem_size();
    // 4-byte accesses past the operand's end are dropped whole: the copies need rows that end on 4 bytes.
    if ((int64_t)h.ldb * esz % 4 || (int64_t)h.N * esz % 4 || (int64_t)h.K * h.ldb * esz >= (1ll << 31)) return best;
    static const int shapes[3][2] = {{4, 4}, {2, 4}, {2, 8}};   // V, rows per wave; the last two: fp32 only
    for (int i = 0; i < (esz == 4 ? 3 : 1); ++i) {
        StagedRows s;
        s.V = shapes[i][0]; s.rows_per_wave = shapes[i][1];
        const int nvc = (h.N + s.V - 1) / s.V;
        s.tiles = (nvc + kWave - 1) / kWave;
        s.lanes = (nvc + s.tiles - 1) / s.tiles;
        const int64_t per_round = 256 / std::min<int64_t>(256, (int64_t)s.tiles * h.batch);   // row groups that fit one round of workgroups
        s.groups = (h.M + kStagedWaves * s.rows_per_wave - 1) / (kStagedWaves * s.rows_per_wave);
        if (s.groups < per_round) s.groups = (int)std::min<int64_t>(per_round, (h.M + kStagedWaves - 1) / kStagedWaves);
        s.pitch = (s.lanes * s.V * esz + 15) / 16 * 16;
        // two buffers of a chunk and one row of zeros each; a row's count of pairs of a chunk, in twos, fits a byte
        s.chunk = std::min(510, (kStagedLdsBytes - 2048) / 2 / s.pitch - 1);
        s.chunk = std::min(s.chunk, h.K);
        s.chunks = (h.K + s.chunk - 1) / s.chunk;
        if (!staged_rows_fits(h, s)) continue;
        s.microseconds = staged_rows_microseconds(h, s, longest);
        if (best.V == 0 || s.microseconds < best.microseconds) best = s;
    }
    if (best.V && (best.microseconds > 0.8 * plain_rows_microseconds(h, longest) || !staged_rows_confirmed(h, best, longest))) best.V = 0;
    // A step of eight loads 64 bytes of pairs ahead whatever is left of a row's share.  In fp32 that pays from about eight
    // pairs to a share on, in us, steps of four and of eight: eight rows to a wave 2049 x 256 x 784 at 95.4 % (7.2 pairs) 7.86 and 8.24,
    // 2049 x 4096 x 196, batch 4, at 92.8 % (14.5) 77.5 and 75.3; four rows 4096 x 3072 x 2048 at 93.6 % (5.0) 184.2 and 189.5,
    // 4096 x 3072 x 516 at 92.4 % (8.8) 73.7 and 72.1.  Half and int8 lose nothing with as few as 5.4 (0.5 % within the noise).
    best.short_shares = best.V && esz == 4 && (int64_t)h.nnz < 8 * (int64_t)h.M * best.chunks;
    return best;
}

// ---- the kernel of a row-walk plan: blocked, staged, or neither.
struct RowsChoice { StagedRows staged; BlockedRows blocked; };

// The blocked kernel is held against the one of the other two that the rules above choose, both by estimates.  60 fp32 products, most drawn from
// M, K <= 4096, N from 49 to 4096, 80 % to 98 % zeros, a third with skewed rows: it takes 17 of them, all faster for it
// than without the blocked kernel (1.62 times on average, 1.25 at least; 2816 x 630 x 128 at 84 %, skewed, 32.9 -> 10.4 us), and leaves
// ten where some number of rows and waves would have been 11 to 38 % faster than what runs.  Of 33 others drawn alike that it takes two
// are slower for it, both skewed (1342 x 2956 x 77 at 92.5 % 24.8 -> 26.4 us, the other 1.3 %); 0.71 times the time on average.  (The staged estimate leaves its longest
// row out here: a single long one, which it counts in full, would make up for what is missing to 0.77.)  The plain kernel's estimate is further off, but where it
// is above 15 us what it leaves out makes that kernel slower.
inline RowsChoice rows_choice(const HostPlan &h) {
    RowsChoice c;
    if (h.kernel != SPARSERT_KERNEL_ROWS || h.conv || h.plain_rows) return c;
    int32_t longest = 0;
    for (int32_t i = 0; i < h.M; ++i) longest = std::max(longest, h.p_row_ptr[i + 1] - h.p_row_ptr[i]);
    c.staged = staged_rows_candidate(h, longest);
    c.blocked = blocked_rows_candidate(h);
    if (c.blocked.rows == 0) return c;
    const double limit = c.staged.V ? 0.77 * staged_rows_microseconds_again(h, c.staged, 0) : 0.9 * plain_rows_microseconds_again(h, longest);
    if (c.blocked.microseconds < limit) c.staged.V = 0;
    else c.blocked.rows = 0;
    return c;
}
inline StagedRows staged_rows_shape(const HostPlan &h) { return rows_choice(h).staged; }
inline BlockedRows blocked_rows_shape(const HostPlan &h) {
    BlockedRows s = rows_choice(h).blocked;
    if (s.rows) s.per_part = blocked_rows_per_part(h, s);
    return s;
}

}  // namespace sparsert
