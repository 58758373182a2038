// The autotuner's list of executor configurations for one problem (Section 3.7 of the paper: a short,
// hand-picked list).  Host code only.
#include <algorithm>
#include <cstdint>
#include <utility>
#include <vector>

#include "mfma.h"
#include "plan.h"

namespace sparsert {

// What an untuned plan would run is in the race for every problem: the row-walk family's choice is timed before
// this list (tune.cpp), the generated kernel's and the matrix cores' are entries of it with nothing else set.
std::vector<sparsert_options> tune_candidates(int32_t M, int32_t K, int32_t N, int64_t nnz, const sparsert_options &b) {
    const bool conv = b.conv != 0, f16 = b.dtype == SPARSERT_F16, i8 = b.dtype == SPARSERT_I8;
    const int family = b.kernel;   // AUTO: both executor families; else only that one
    std::vector<sparsert_options> cands;
    if (!conv) {
        for (int v = 1; v <= (f16 ? 8 : 4); v *= 2) {
            if (N % v || (i8 && v == 2)) continue;
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_ROWS; o.vec = v;
            cands.push_back(o);
            o.split_threshold = 64;
            cands.push_back(o);
        }
    } else {
        for (int thr : {32, 64, 1 << 30}) {
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_ROWS; o.split_threshold = thr;
            cands.push_back(o);
        }
    }
    if (family == SPARSERT_KERNEL_SPEC) cands.clear();
    // Zero-filled tiles on the matrix cores - small, middle, large and the one the inspector takes - for any number of
    // nonzeros: nothing is assembled for them.
    if (!conv && (f16 || i8) && N >= 16 && !b.natural_order && family != SPARSERT_KERNEL_ROWS) {
        for (int tile : {5, 4, 3, 2, 0}) {
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_MFMA;
            o.spec_rows = kMfmaConfigs[tile].tm; o.spec_tiles = kMfmaConfigs[tile].tn / 16;
            cands.push_back(o);
        }
        sparsert_options o = b;
        o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_MFMA;
        cands.push_back(o);
    }
    if (nnz <= (4 << 20) && family != SPARSERT_KERNEL_ROWS) {
        const int64_t images = std::max(1, b.batch);   // every problem of a batch brings its own waves
        const int64_t tiles = (N + 63) / 64 * images;
        // DIRECT and K-split candidates at V columns per lane (V > 1: the halves / int8 packed in one dword)
        auto add_direct = [&](int V) {
            const int64_t vtiles = (N / V + 63) / 64 * images;
            const int max_rows = 192 / V;   // accumulator registers
            // Matrices of some size get a thinner list (a candidate costs 1-2.5 s of assembling per
            // 100 000 nonzeros): blocks of one or two rows - the largest code, and winners only on
            // small problems - and the two-tile twins of the four-tile workgroups are left out.
            const bool sizeable = nnz > (64 << 10);
            for (int r : {1, 2, 4, 8, 16, 24, 48, 96}) {
                if (r > M || r > max_rows || (r == 96 && images == 1)) continue;
                if (sizeable && r < 4 && M >= 1024) continue;
                const int64_t groups = (M + r - 1) / r;
                if (r > 1 && groups * vtiles < 256) continue;   // too few waves to be worth assembling
                if (groups > 8192) continue;
                for (int t : {2, 4}) {
                    if ((V > 1 || sizeable) && t == 2) continue;
                    sparsert_options o = b;
                    o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_DIRECT;
                    // (a few more rows where that spares a last round of workgroups on a few compute units)
                    o.spec_rows = rows_without_thin_round(M, r, 1, (vtiles / images + t - 1) / t * images, max_rows);
                    o.spec_tiles = t; o.spec_vec = V;
                    cands.push_back(o);
                }
            }
            if (K >= 512) {   // long reduction axis: split it over the waves of a workgroup
                const int rk[][2] = {{1, 8}, {2, 8}, {4, 8}, {8, 8}, {16, 8}, {24, 8}, {32, 8}, {48, 8}, {64, 8}, {96, 8}, {128, 8},
                                     {1, 4}, {2, 4}, {4, 4}, {8, 4}, {16, 4}, {32, 4}, {48, 4}, {64, 4}, {96, 4},
                                     {64, 2}, {96, 2}};
                std::vector<std::pair<int, int>> listed;
                auto add = [&](int r, int ks) {
                    if (std::find(listed.begin(), listed.end(), std::make_pair(r, ks)) != listed.end()) return;
                    listed.push_back({r, ks});
                    sparsert_options o = b;
                    o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_DIRECT;
                    o.spec_rows = r; o.spec_ksplit = ks; o.spec_vec = V;
                    cands.push_back(o);
                };
                for (auto &c : rk) {
                    // worth timing with at least two waves for every SIMD of the chip, but not with
                    // more than sixteen (the blocks are then too small to reuse a fetched row)
                    const int64_t waves = (int64_t)((M + c[0] - 1) / c[0]) * vtiles * c[1];
                    if (c[0] > M || c[0] > max_rows || waves < 2048 || waves > 16384) continue;
                    // never a last round of workgroups that only a few compute units take part in
                    add(rows_without_thin_round(M, c[0], 1, vtiles, max_rows), c[1]);
                }
                // ... and the row counts that make the launch exactly one, two or four workgroups
                // per compute unit with two or four waves per SIMD: the fewest fetches of B a
                // launch that still fills the chip can have (1024 x 4096 at 95 %, 784 columns:
                // 54 rows x 8 parts = 247 workgroups, 21.3 us; the listed 48 rows = 286: 43.7 us)
                const int whole[][2] = {{8, 1}, {8, 2}, {4, 2}, {4, 4}, {2, 4}};   // parts, workgroups per compute unit
                for (auto &c : whole) {
                    // (eight parts are two waves per SIMD, which leaves each 256 registers: blocks of up to 224 rows;
                    // 1024 x 4096 x 3136 at 95 %: 205 rows, one workgroup per compute unit, 45 us; 103 rows, two: 61 us)
                    const int r = rows_for_rounds(M, 1, vtiles, c[1], c[0] == 8 && c[1] == 1 ? 224 / V : max_rows);
                    if (r < 4) continue;
                    const int64_t wgs = (int64_t)((M + r - 1) / r) * vtiles;
                    if (wgs * 4 < (int64_t)256 * c[1] * 3) continue;   // under three quarters of the chip
                    add(r, c[0]);
                }
            }
        };
        {   // what the inspector picks when nothing is set is always in the race
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_SPEC;
            cands.push_back(o);
        }
        add_direct(1);
        if (!conv && f16 && N % 2 == 0) add_direct(2);
        if (!conv && i8 && N % 4 == 0) add_direct(4);
        if (!conv && !f16 && !i8 && K >= 256 && (int64_t)M * tiles >= 1024) {
            for (int r : {12, 24, 48, 96})
                for (int w : {4, 8}) {
                    if (((int64_t)M + r - 1) / r < w) continue;
                    sparsert_options o = b;
                    o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_LDS;
                    o.spec_rows = rows_without_thin_round(M, r, w, tiles, 128);
                    o.spec_tiles = w;
                    cands.push_back(o);
                }
        }
    }

    // Assembling a candidate costs about 12 s per million nonzeros, so large matrices get a
    // short list of generated kernels: one per family, each at the row count that fills whole
    // rounds of workgroups over the chip's compute units (rows_for_whole_rounds; measured on
    // 4096 x 4096 x 3136 at 95 %: 103 rows per block 127 us, 96 rows 180 us).  The LDS-staged
    // variant leads the list where the reduction axis is long: it is what wins there.
    if (nnz > (256 << 10) && family != SPARSERT_KERNEL_ROWS) {
        const size_t budget = nnz > (1 << 20) ? 3 : 6;
        const int64_t vt = (N + 63) / 64 * std::max(1, b.batch);
        std::vector<sparsert_options> rows_family, spec_family;
        for (const sparsert_options &o : cands)
            if (o.kernel != SPARSERT_KERNEL_SPEC || o.spec_mode == SPARSERT_SPEC_MFMA) rows_family.push_back(o);   // nothing to assemble
        auto direct = [&](int ks, int t) {
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_DIRECT;
            o.spec_ksplit = ks; o.spec_tiles = t;
            o.spec_rows = rows_for_whole_rounds(M, 1, ks > 1 ? vt : (vt + t - 1) / t, 32, 128);
            spec_family.push_back(o);
        };
        auto staged = [&](int w) {
            if (conv || K < 256 || ((int64_t)M + 31) / 32 < w) return;
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_LDS; o.spec_tiles = w;
            o.spec_rows = rows_for_whole_rounds(M, w, vt, 32, 128);
            spec_family.push_back(o);
        };
        {   // the inspector's own choice for the generated kernel (no option set) is always in the race
            sparsert_options o = b;
            o.kernel = SPARSERT_KERNEL_SPEC;
            spec_family.push_back(o);
        }
        if (K >= 2048) { staged(8); direct(1, 4); direct(2, 2); staged(4); direct(4, 4); direct(8, 8); }
        else if (K >= 512) { direct(2, 2); direct(1, 4); direct(4, 4); staged(8); direct(8, 8); staged(4); }
        else { direct(1, 4); direct(1, 2); staged(8); staged(4); }
        if (spec_family.size() > budget + 1) spec_family.resize(budget + 1);
        cands = rows_family;
        cands.insert(cands.end(), spec_family.begin(), spec_family.end());
    }
    return cands;
}

sparsert_options options_again(const HostPlan &h, const sparsert_options &b) {
    const SpecPlan &w = h.spec;
    sparsert_options o = b;
    o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = w.mode; o.spec_rows = w.rows_per_group;
    o.spec_tiles = w.tiles_per_wg; o.spec_ksplit = w.ksplit; o.spec_vec = w.vec; o.spec_swizzle = w.swizzle;
    o.spec_prefetch = w.prefetch_lines > 0 ? 1 : -1;   // (a plan with nothing set may have the touches)
    return o;
}

}  // namespace sparsert
