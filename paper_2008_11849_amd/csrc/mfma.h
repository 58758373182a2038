// Tile shapes of the matrix-core executor (mfma.hip): what the inspector chooses from and the
// launch looks up.  Host code only.
#pragma once
#include <algorithm>
#include <cstdint>

namespace sparsert {

struct MfmaConfig {
    int tm, tn;          // rows and columns of C per workgroup
    int wm, wn, mf, nf;  // waves along M and N; 16-row and 16-column fragments per wave
    int steps;           // matrix-instruction steps of K per slab
    int stages;          // slabs in LDS
    // Measured time in microseconds: launch and ends, a slab of a workgroup that has its compute unit to
    // itself, a slab for every workgroup of the busiest compute unit, a megabyte of C (mfma_microseconds).
    double fixed, slab_alone, slab_shared, store;
    constexpr int waves() const { return wm * wn; }
    constexpr int lds_bytes() const { return (tm + tn) * 64 * steps * stages; }
};

// One instruction contracts 64 bytes of every column: 32 halves or 64 int8.
constexpr int mfma_step(int elem_size) { return 64 / elem_size; }

#define SPARSERT_MFMA_CONFIGS(X)                                  \
    X(0, 128, 128, 2, 4, 4, 2, 2, 4, 3.74, 0.197, 0.376, 0.27) \
    X(1, 64, 128, 2, 4, 2, 2, 2, 3, 3.00, 0.222, 0.324, 0.21)  \
    X(2, 128, 64, 4, 2, 2, 2, 2, 3, 2.97, 0.155, 0.318, 0.22)  \
    X(3, 64, 64, 2, 2, 2, 2, 2, 4, 2.58, 0.210, 0.206, 0.27)   \
    X(4, 32, 64, 2, 2, 1, 2, 2, 4, 2.35, 0.178, 0.154, 0.29)   \
    X(5, 32, 32, 2, 2, 1, 1, 2, 4, 2.23, 0.129, 0.126, 0.34)   \
    X(6, 16, 64, 1, 4, 1, 1, 4, 4, 2.50, 0.203, 0.285, 0.62)   \
    X(7, 48, 64, 1, 4, 3, 1, 4, 4, 2.59, 0.391, 0.397, 0.69)   \
    X(8, 96, 128, 2, 2, 3, 4, 2, 4, 3.56, 0.080, 0.355, 0.33)

constexpr MfmaConfig kMfmaConfigs[] = {
#define X(id, tm, tn, wm, wn, mf, nf, steps, stages, f, a, s, o) {tm, tn, wm, wn, mf, nf, steps, stages, f, a, s, o},
    SPARSERT_MFMA_CONFIGS(X)
#undef X
};
constexpr int kMfmaConfigCount = (int)(sizeof(kMfmaConfigs) / sizeof(kMfmaConfigs[0]));

// The zero-filled copy of A for a tile: rows in whole tiles, columns in whole slabs.  It is addressed with 31 bits.
inline int64_t mfma_weight_bytes(const MfmaConfig &c, int64_t M, int64_t K, int elem_size) {
    const int64_t slab = (int64_t)c.steps * 64;
    return (M + c.tm - 1) / c.tm * c.tm * ((K * elem_size + slab - 1) / slab * slab);
}
inline bool mfma_fits(const MfmaConfig &c, int64_t M, int64_t K, int elem_size) { return mfma_weight_bytes(c, M, K, elem_size) < (1ll << 31); }

// Index of the configuration with this tile; 0 for a field means any.  -1: none.
inline int mfma_find(int tm, int tn) {
    for (int i = 0; i < kMfmaConfigCount; ++i)
        if ((!tm || kMfmaConfigs[i].tm == tm) && (!tn || kMfmaConfigs[i].tn == tn)) return i;
    return -1;
}

// Each XCD takes an eighth of the tiles: along M if that leaves its L2 less of A and B to hold, else along N.
inline bool mfma_m_fast(const MfmaConfig &c, int64_t M, int64_t K, int64_t N, int elem_size) {
    const double wb = (double)((M + c.tm - 1) / c.tm) * c.tm * K * elem_size, bb = (double)K * N * elem_size;
    return wb + bb / 8 < wb / 8 + bb;
}

// Tiles along M that stand together in the order of the tasks, of which every XCD takes an eighth: the number for which
// the eight L2s together pull the least of A and B (768 x 3072 x 1024 int8 in tiles of 64 x 64, a column of all twelve:
// 22 MB; six: 15.8 MB), a row of B in whole lines of 128 bytes.  (As if it came in the bytes of its tiles 272 x 3592 x 196
// int8 in tiles of 32 x 32 was given five of nine: 7.6 us, 5.1 with one.)  Over 164 drawn products, each timed in up to twelve
// parts, the choice is 1.005 times faster than the better of the two simple orders, the best by measuring 1.014.
inline int mfma_rows_per_part(const MfmaConfig &c, int64_t M, int64_t K, int64_t N, int64_t ldb, int elem_size) {
    const int64_t m_tiles = (M + c.tm - 1) / c.tm, n_tiles = (N + c.tn - 1) / c.tn, tasks = m_tiles * n_tiles, share = (tasks + 7) / 8;
    int64_t best = mfma_m_fast(c, M, K, N, elem_size) ? m_tiles : 1;
    double least = 0;
    struct Place { int64_t part, n, m; };
    auto place = [&](int64_t per, int64_t t) {
        const int64_t part = t / (per * n_tiles), in = t - part * per * n_tiles, here = std::min(per, m_tiles - part * per);
        return Place{part, in / here, in % here};
    };
    for (int64_t parts = 0; parts <= 16 && parts <= m_tiles && tasks <= 65536; ++parts) {
        const int64_t per = parts ? (m_tiles + parts - 1) / parts : best;   // first the better one of the two that end at 1
        double bytes = 0;
        for (int64_t x = 0; x * share < tasks; ++x) {
            const int64_t last = std::min(tasks, (x + 1) * share) - 1;
            const Place from = place(per, x * share), to = place(per, last);
            // A range over the end of a part has the last columns of the one and the first of the other.
            const bool over = from.part != to.part;
            const int64_t n_lo = over ? 0 : from.n, n_hi = over ? n_tiles - 1 : to.n;
            const int64_t m_lo = from.part * per + (from.n == (over ? n_tiles - 1 : to.n) ? from.m : 0);
            const int64_t m_hi = to.part * per + (to.n == (over ? 0 : from.n) ? to.m : std::min(per, m_tiles - to.part * per) - 1);
            // Of a row of B: its lines, with rows that begin anywhere on one, by the average, 127 bytes more.
            const int64_t first = n_lo * c.tn * elem_size, wide = std::min((n_hi + 1) * c.tn, N) * elem_size - first, pitch = ldb * elem_size;
            const int64_t pulled = pitch % 128 ? std::min(wide + 127, pitch) : (first % 128 + wide + 127) / 128 * 128;
            bytes += ((double)((m_hi - m_lo + 1) * c.tm * elem_size) + (double)pulled) * (double)K;
        }
        if (parts == 0 || bytes < 0.95 * least) { least = bytes; best = per; }
    }
    return (int)best;
}

// Time of an M x K x N product with this tile, from the constants above: they reproduce 122 measured shapes
// (M 64 ... 4000, K 64 ... 3867, N 49 ... 4096, both storage types) to about 9 %, and the tile they choose is
// within 1 % of the best one on average, 10 % at most.  That was before results left through LDS and tiles were dealt in
// blocks; the kernel as it is: 10 % root mean square over 700 drawn products for which this and the generated kernel's first estimate are within
// 0.45 to 1.5 of each other.
inline double mfma_microseconds(const MfmaConfig &c, int64_t M, int64_t K, int64_t N, int64_t batch, int elem_size, int out_size) {
    const int64_t slab = (int64_t)c.steps * mfma_step(elem_size), slabs = (K + slab - 1) / slab;
    const int64_t wgs = (M + c.tm - 1) / c.tm * ((N + c.tn - 1) / c.tn) * batch;
    const double rounds = wgs > 1024 ? wgs / 256.0 : (double)((wgs + 255) / 256);
    const double slab_us = c.slab_shared * rounds > c.slab_alone ? c.slab_shared * rounds : c.slab_alone;
    return c.fixed + slabs * slab_us + c.store * 1e-6 * (double)(M * N * batch) * out_size;
}

}  // namespace sparsert
