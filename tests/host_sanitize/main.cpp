// Drives the host half of the library (inspector, code generator, serialisation, boundary)
// through a grid of problems and options in one native process, built with
// -fsanitize=address,undefined.  Any out-of-bounds access, use after free, signed overflow or
// misaligned access in that code ends the process with a report; the test expects exit code 0.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/sparsert.h"
#include "../../paper_2008_11849_amd/csrc/mfma.h"
#include "../../paper_2008_11849_amd/csrc/staged_rows.h"

namespace {

struct Rng {
    uint64_t s;
    uint32_t next() { s = s * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(s >> 33); }
    double unit() { return next() / 2147483648.0; }
};

struct Csr { std::vector<int32_t> row_ptr, col; std::vector<uint8_t> vals; };

// `width` bytes per value; the bytes are arbitrary (the host code only moves them), except that
// half values avoid the NaN / infinity exponent so the generator's widening sees ordinary numbers too
Csr make(int M, int K, double density, int width, Rng &r, bool skew) {
    Csr c;
    c.row_ptr.push_back(0);
    for (int m = 0; m < M; ++m) {
        const double d = skew ? density * 4.0 / (1.0 + (m % 7) * (m % 7)) : density;
        for (int k = 0; k < K; ++k)
            if (r.unit() < d) {
                c.col.push_back(k);
                for (int b = 0; b < width; ++b) c.vals.push_back((uint8_t)(r.next() & (width == 2 && b == 1 ? 0x3b : 0xff)));
            }
        c.row_ptr.push_back((int32_t)c.col.size());
    }
    return c;
}

int failures = 0;
#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) { std::fprintf(stderr, "line %d: %s (%s)\n", __LINE__, #cond, sparsert_last_error()); ++failures; } \
    } while (0)

void exercise(const Csr &c, int M, int K, int N, sparsert_options o, bool may_refuse) {
    o.host_only = 1;
    sparsert_plan *p = nullptr;
    const int rc = sparsert_inspect(c.row_ptr.data(), c.col.data(), c.vals.data(), M, K, N, &o, &p);
    if (rc != SPARSERT_OK) {
        EXPECT(may_refuse && p == nullptr && (rc == SPARSERT_EINVAL || rc == SPARSERT_EUNSUPPORTED));
        return;
    }
    for (int f = SPARSERT_FIELD_INFO; f <= SPARSERT_FIELD_KERNEL_NAME; ++f) {
        size_t need = 0;
        EXPECT(sparsert_plan_export(p, f, nullptr, 0, &need) == SPARSERT_OK);
        std::vector<uint8_t> buf(need + 1);
        EXPECT(sparsert_plan_export(p, f, buf.data(), need, nullptr) == SPARSERT_OK);
        if (need) EXPECT(sparsert_plan_export(p, f, buf.data(), need - 1, nullptr) == SPARSERT_EINVAL);
    }
    size_t need = 0;
    EXPECT(sparsert_plan_save(p, nullptr, 0, &need) == SPARSERT_OK && need > 24);
    std::vector<uint8_t> blob(need), again(need);
    EXPECT(sparsert_plan_save(p, blob.data(), need, nullptr) == SPARSERT_OK);
    sparsert_plan *q = nullptr;
    EXPECT(sparsert_plan_load(blob.data(), need, 1, &q) == SPARSERT_OK && q);
    if (q) {
        size_t need2 = 0;
        EXPECT(sparsert_plan_save(q, again.data(), need, &need2) == SPARSERT_OK && need2 == need);
        EXPECT(std::memcmp(blob.data(), again.data(), need) == 0);
        sparsert_plan_destroy(q);
    }
    // damaged blobs are refused, never dereferenced: a flipped byte, a truncation
    if (need > 64) {
        std::vector<uint8_t> bad(blob);
        bad[need / 2] ^= 0x5a;
        q = nullptr;
        EXPECT(sparsert_plan_load(bad.data(), need, 1, &q) != SPARSERT_OK && !q);
        EXPECT(sparsert_plan_load(blob.data(), need - 9, 1, &q) != SPARSERT_OK && !q);
    }
    // executing a host-only plan is an error, not a crash
    EXPECT(sparsert_spmm(p, blob.data(), again.data(), nullptr) == SPARSERT_EINVAL);
    sparsert_plan_destroy(p);
}

// A row-walk plan of M rows of `row` nonzeros as far as the rule of the staged kernel looks at it.
sparsert::HostPlan rows_plan(int M, int K, int N, int row, int dtype = SPARSERT_F32) {
    sparsert::HostPlan h;
    h.M = M; h.K = K; h.N = h.ldb = h.ldc = N; h.nnz = M * row; h.dtype = dtype; h.kernel = SPARSERT_KERNEL_ROWS;
    h.vec = 4; h.n_tiles = (N / 4 + 63) / 64; h.lanes_per_tile = 64; h.split_threshold = 512;
    for (int64_t i = 0; i <= M; ++i) h.p_row_ptr.push_back((int32_t)(i * row));
    return h;
}

// What the rule hands to the staged kernel, the kernel's launch accepts: its pair stream is addressed with
// 31 bits, a launch holds less than 2^32 threads.
void staged_rule_stays_inside_the_limits() {
    EXPECT(sparsert::staged_rows_shape(rows_plan(6000, 6000, 784, 3000)).V);          // 144 MB of pairs
    EXPECT(sparsert::staged_rows_shape(rows_plan(16000, 24000, 784, 16000)).V);       // 2.05 GB
    EXPECT(!sparsert::staged_rows_shape(rows_plan(24000, 24000, 784, 12000)).V);      // 2.3 GB
    EXPECT(!sparsert::staged_rows_shape(rows_plan(16700, 30000, 784, 16000)).V);      // 2.138 GB, more with the fill
}

// The tuner's list holds what an untuned plan would run, for any number of nonzeros: the generated kernel and, for
// half and int8 products, the matrix cores with nothing else set; other families' plans only where they may win.
void tuner_candidates_hold_the_defaults() {
    for (int dtype = SPARSERT_F32; dtype <= SPARSERT_I8; ++dtype)
        for (int64_t nnz : {(int64_t)5000, (int64_t)300000, (int64_t)2000000, (int64_t)5035156, (int64_t)100000000})
            for (int family : {SPARSERT_KERNEL_AUTO, SPARSERT_KERNEL_ROWS, SPARSERT_KERNEL_SPEC})
                for (int natural : {0, 1}) {
                    sparsert_options b;
                    std::memset(&b, 0, sizeof(b));
                    b.dtype = dtype; b.kernel = family; b.natural_order = natural;
                    int rows = 0, generated = 0, mfma = 0, generated_default = 0, mfma_default = 0;
                    for (const sparsert_options &o : sparsert::tune_candidates(12288, 12288, 1024, nnz, b)) {
                        const bool tiles = o.spec_rows || o.spec_tiles || o.spec_ksplit;
                        if (o.kernel == SPARSERT_KERNEL_ROWS) { ++rows; continue; }
                        ++(o.spec_mode == SPARSERT_SPEC_MFMA ? mfma : generated);
                        if (!tiles) ++(o.spec_mode == SPARSERT_SPEC_MFMA ? mfma_default : generated_default);
                        EXPECT(o.natural_order == natural && o.dtype == dtype);
                    }
                    const bool wants_mfma = dtype != SPARSERT_F32 && family != SPARSERT_KERNEL_ROWS && !natural;
                    EXPECT((rows > 0) == (family != SPARSERT_KERNEL_SPEC));
                    EXPECT(mfma_default == (wants_mfma ? 1 : 0) && mfma == (wants_mfma ? 6 : 0));
                    EXPECT((generated > 0) == (family != SPARSERT_KERNEL_ROWS) && generated_default == (generated ? 1 : 0));
                }
}

sparsert::HostPlan host_plan(const Csr &c, int M, int K, int N, sparsert_options o) {
    sparsert::HostPlan h;
    std::string err;
    o.host_only = 1;
    EXPECT(sparsert::build_host_plan(c.row_ptr.data(), c.col.data(), c.vals.data(), M, K, N, o, h, err) == SPARSERT_OK);
    if (h.kernel == SPARSERT_KERNEL_SPEC) EXPECT(sparsert::build_spec_plan(h, o, err) == SPARSERT_OK);
    return h;
}

// What the tuner builds to try its winner with and without the touches differs from the winner in nothing else, also where
// the winner is the plan with nothing set, which may have them.
void winners_are_tried_both_ways(Rng &r) {
    const struct { int M, K, N; double density; bool touches; } shapes[] = {{2314, 520, 688, 0.144, true}, {300, 300, 196, 0.1, false}};
    for (const auto &s : shapes) {
        const Csr c = make(s.M, s.K, s.density, 4, r, false);
        sparsert_options b;
        std::memset(&b, 0, sizeof(b));
        const sparsert::HostPlan h = host_plan(c, s.M, s.K, s.N, b);
        EXPECT(h.kernel == SPARSERT_KERNEL_SPEC && (h.spec.prefetch_lines > 0) == s.touches);
        sparsert_options o = sparsert::options_again(h, b);
        const sparsert::HostPlan same = host_plan(c, s.M, s.K, s.N, o);
        EXPECT(same.spec.code == h.spec.code && same.spec.prefetch_lines == h.spec.prefetch_lines);
        o.spec_prefetch = -o.spec_prefetch;
        const sparsert::HostPlan other = host_plan(c, s.M, s.K, s.N, o);
        EXPECT((other.spec.prefetch_lines > 0) == !s.touches && other.spec.group_of_slot == h.spec.group_of_slot);
        EXPECT(other.spec.mode == h.spec.mode && other.spec.rows_per_group == h.spec.rows_per_group && other.spec.ksplit == h.spec.ksplit &&
               other.spec.tiles_per_wg == h.spec.tiles_per_wg && other.spec.vec == h.spec.vec && other.spec.lanes_per_tile == h.spec.lanes_per_tile);
    }
}

// Fragments of every matrix-core tile: each weight once, at the place its row, step and lane give, zeros elsewhere.
int mfma_layout_holds_every_weight_once(Rng &r) {
    int plans = 0;
    const int shapes[][2] = {{1, 1}, {15, 31}, {17, 65}, {97, 129}, {130, 700}};
    for (const auto &s : shapes)
        for (int dtype : {(int)SPARSERT_F16, (int)SPARSERT_I8})
            for (const sparsert::MfmaConfig &cfg : sparsert::kMfmaConfigs) {
                const int M = s[0], K = s[1], esz = dtype == SPARSERT_F16 ? 2 : 1;
                Csr c = make(M, K, 0.4, esz, r, (M & 1) != 0);
                for (uint8_t &v : c.vals) v |= 1;   // no zeros among them
                sparsert_options o;
                std::memset(&o, 0, sizeof(o));
                o.dtype = dtype; o.kernel = SPARSERT_KERNEL_SPEC; o.spec_mode = SPARSERT_SPEC_MFMA;
                o.spec_rows = cfg.tm; o.spec_tiles = cfg.tn / 16;
                const sparsert::HostPlan h = host_plan(c, M, K, 33, o);
                std::vector<uint8_t> f;
                sparsert::mfma_pack(h, f);
                EXPECT((int64_t)f.size() == sparsert::mfma_weight_bytes(cfg, M, K, esz));
                // lane 16 g + i of a fragment holds row i; its 16 bytes are the g-th eighth of K's first half of a
                // step (4 halves, 8 int8), then of the second half
                const int step = 64 / esz, piece = 8 / esz, steps = (int)(f.size() / 1024 / ((M + cfg.tm - 1) / cfg.tm * (cfg.tm / 16)));
                size_t nonzero = 0;
                for (uint8_t v : f) nonzero += v != 0;
                EXPECT(nonzero == c.vals.size());
                for (int m = 0; m < M; ++m)
                    for (int p = c.row_ptr[m]; p < c.row_ptr[m + 1]; ++p) {
                        const int k = c.col[p], second = k % step / (step / 2), g = k % (step / 2) / piece;
                        const size_t at = ((size_t)(m / 16) * steps + k / step) * 1024 + (size_t)(16 * g + m % 16) * 16 + (size_t)second * 8 + (size_t)(k % piece) * esz;
                        EXPECT(at + esz <= f.size() && std::memcmp(&f[at], &c.vals[(size_t)p * esz], esz) == 0);
                    }
                ++plans;
            }
    return plans;
}

// The staged stream walked as a wave does: every row of C belongs to one place, its pairs name its columns in order,
// operands lie inside the chunk and fillers on the row of zeros behind it.
int staged_layout_walks_every_row(Rng &r) {
    int plans = 0;
    const struct { int M, K, N, batch; double density; } shapes[] = {{2049, 200, 196, 4, 0.3}, {2100, 333, 516, 1, 0.2}, {4000, 90, 2000, 1, 0.1}, {4096, 1500, 788, 1, 0.1}};
    for (const auto &s : shapes)
        for (int dtype = SPARSERT_F32; dtype <= SPARSERT_I8; ++dtype) {
            const Csr c = make(s.M, s.K, s.density, dtype == SPARSERT_F16 ? 2 : dtype == SPARSERT_I8 ? 1 : 4, r, false);
            sparsert_options o;
            std::memset(&o, 0, sizeof(o));
            o.dtype = dtype; o.kernel = SPARSERT_KERNEL_ROWS; o.batch = s.batch;
            const sparsert::HostPlan h = host_plan(c, s.M, s.K, s.N, o);
            const sparsert::StagedRows g = sparsert::staged_rows_shape(h);
            if (!g.V) { EXPECT(dtype != SPARSERT_F32); continue; }
            sparsert::StagedPack pack;
            sparsert::staged_rows_pack(h, pack);
            const int rw = g.rows_per_wave, owners = g.groups * sparsert::kStagedWaves;
            EXPECT((int)pack.starts.size() == owners && (int)pack.rows.size() == owners * rw && (int64_t)pack.counts.size() == (int64_t)owners * g.chunks * rw);
            EXPECT((int64_t)pack.stream.size() <= 2 * ((int64_t)h.nnz + (int64_t)h.M * g.chunks + 16));   // what the rule allows for
            std::vector<int> seen(s.M, 0);
            for (int owner = 0; owner < owners; ++owner) {
                size_t p = (size_t)pack.starts[owner] * 2;
                std::vector<int> at(rw);
                for (int i = 0; i < rw; ++i)
                    if (pack.rows[owner * rw + i] >= 0) { ++seen[pack.rows[owner * rw + i]]; at[i] = c.row_ptr[pack.rows[owner * rw + i]]; }
                for (int chunk = 0; chunk < g.chunks; ++chunk)
                    for (int i = 0; i < rw; ++i) {
                        const int n = 2 * pack.counts[((size_t)owner * g.chunks + chunk) * rw + i], row = pack.rows[owner * rw + i];
                        if (row < 0) { EXPECT(n == 0); continue; }
                        for (int q = 0; q < n; ++q, p += 2) {
                            const uint32_t off = pack.stream[p], k = (uint32_t)chunk * g.chunk + off / g.pitch;
                            EXPECT(off % g.pitch == 0 && off <= (uint32_t)(g.chunk * g.pitch));
                            if (off == (uint32_t)(g.chunk * g.pitch)) { EXPECT(q == n - 1 && pack.stream[p + 1] == 0); continue; }
                            EXPECT(at[i] < c.row_ptr[row + 1] && (uint32_t)c.col[at[i]] == k);
                            ++at[i];
                        }
                    }
                for (int i = 0; i < rw; ++i)
                    if (pack.rows[owner * rw + i] >= 0) EXPECT(at[i] == c.row_ptr[pack.rows[owner * rw + i] + 1]);
            }
            for (int v : seen) EXPECT(v == 1);
            ++plans;
        }
    return plans;
}

// The blocked kernel's records walked as a wave does: every nonzero once, in its row's place and its column's group, fillers with the
// value zero and the row that nobody reads, headers that name the columns of a group and its layers, and nothing the wave
// reads ahead of its place lies behind the stream.
int blocked_records_hold_every_nonzero_once(Rng &r) {
    int plans = 0;
    const struct { int M, K, N, ldb, rows, parts; double density; bool skew; } shapes[] = {
        {300, 300, 640, 640, 75, 4, 0.0, false},  {300, 300, 640, 640, 75, 4, 0.004, false},  {64, 1500, 130, 133, 22, 8, 0.12, false},
        {200, 90, 49, 49, 84, 4, 0.2, true},      {1000, 700, 200, 200, 84, 8, 0.19, false},  {1, 40, 64, 64, 1, 4, 0.2, false},
        {85, 3, 64, 64, 43, 4, 0.2, false},       {2048, 1024, 784, 784, 57, 4, 0.15, false}, {997, 1500, 300, 317, 16, 4, 0.05, true}};
    for (const auto &t : shapes) {
        const Csr c = make(t.M, t.K, t.density, 4, r, t.skew);
        sparsert_options o;
        std::memset(&o, 0, sizeof(o));
        o.kernel = SPARSERT_KERNEL_ROWS; o.ldb = o.ldc = t.ldb;
        const sparsert::HostPlan h = host_plan(c, t.M, t.K, t.N, o);
        sparsert::BlockedRows s;
        s.blocks = (t.M + t.rows - 1) / t.rows; s.rows = (t.M + s.blocks - 1) / s.blocks; s.parts = t.parts;
        sparsert::BlockedPack pack;
        sparsert::blocked_rows_pack(h, s, pack);
        const int R = sparsert::kBlockedRows, W = sparsert::kBlockedRecord, G = sparsert::kBlockedColumns;
        EXPECT((int)pack.starts.size() == s.blocks * s.parts && (int)pack.rows.size() == s.blocks * R && pack.stream.size() % W == 0);
        const size_t records = pack.stream.size() / W;
        std::vector<int> seen_row(t.M, 0), seen(h.nnz, 0);
        for (int b = 0; b < s.blocks; ++b) {
            for (int i = 0; i < R; ++i)
                if (pack.rows[b * R + i] >= 0) { EXPECT(i < s.rows); ++seen_row[pack.rows[b * R + i]]; }
            for (int part = 0; part < s.parts; ++part) {
                size_t at = pack.starts[b * s.parts + part];
                const uint32_t *header = &pack.stream[at * W], *next = &pack.stream[(at + 1) * W];
                for (at += 2; (int32_t)header[G] >= 0;) {
                    for (int layer = 0; layer <= (int32_t)header[G]; ++layer, ++at) {
                        EXPECT(at + 1 < records);   // (the record behind is fetched while this one is worked on)
                        for (int i = 0; i < G; ++i) {
                            const uint32_t value = pack.stream[at * W + i], place = pack.stream[at * W + G + i / 4] >> (8 * (i % 4)) & 255;
                            if (place == (uint32_t)R) { EXPECT(value == 0); continue; }
                            EXPECT((int)place < s.rows && header[i] % (4 * t.ldb) == 0);
                            const int row = pack.rows[b * R + place], column = (int)(header[i] / (4 * t.ldb));
                            EXPECT(row >= 0);
                            int p = c.row_ptr[row];
                            while (p < c.row_ptr[row + 1] && c.col[p] != column) ++p;
                            EXPECT(p < c.row_ptr[row + 1] && std::memcmp(&value, &c.vals[(size_t)p * 4], 4) == 0);
                            if (p < c.row_ptr[row + 1]) ++seen[p];
                        }
                    }
                    for (int i = 0; i < G; ++i) EXPECT(header[i] / 4 <= (uint32_t)((t.K - 1) * t.ldb));
                    header = next;
                    next = &pack.stream[at++ * W];
                }
                // the wave ends on a group that is not there; it has fetched that one's header, the next one's and a record more
                EXPECT(at < records);
            }
        }
        for (int v : seen_row) EXPECT(v == 1);
        for (int v : seen) EXPECT(v == 1);
        ++plans;
    }
    return plans;
}

}  // namespace

int main() {
    tuner_candidates_hold_the_defaults();
    staged_rule_stays_inside_the_limits();
    Rng r{20081184ull};
    const int shapes[][3] = {{1, 1, 1}, {7, 5, 3}, {64, 48, 100}, {70, 150, 196}, {33, 260, 65}};
    int plans = 0;
    winners_are_tried_both_ways(r);
    plans += mfma_layout_holds_every_weight_once(r);
    plans += staged_layout_walks_every_row(r);
    plans += blocked_records_hold_every_nonzero_once(r);
    for (const auto &s : shapes) {
        const int M = s[0], K = s[1], N = s[2];
        for (int dtype = SPARSERT_F32; dtype <= SPARSERT_I8; ++dtype) {
            const int width = dtype == SPARSERT_F16 ? 2 : dtype == SPARSERT_I8 ? 1 : 4;
            for (double density : {0.08, 1.0}) {
                const Csr c = make(M, K, density, width, r, density == 0.08);
                sparsert_options base;
                std::memset(&base, 0, sizeof(base));
                base.dtype = dtype;
                {   // row-walk plans
                    sparsert_options o = base;
                    o.kernel = SPARSERT_KERNEL_ROWS;
                    exercise(c, M, K, N, o, false); ++plans;
                    o.split_threshold = 3; o.natural_order = (M & 1);
                    exercise(c, M, K, N, o, false); ++plans;
                    o.ldb = N + 8; o.ldc = N + 24; o.batch = 3;
                    exercise(c, M, K, N, o, false); ++plans;
                }
                // generated kernels: defaults, then rows x split x variant x packing
                { sparsert_options o = base; exercise(c, M, K, N, o, false); ++plans; }
                // six of the 24 (rows, split, variant) combinations per case, rotating, so that the
                // whole run meets every combination with every storage type
                const int rows_of[] = {1, 5, 200}, ks_of[] = {1, 8};
                for (int j = 0; j < 6; ++j) {
                    const int combo = (plans * 7 + j * 5) % 24;
                    const int rows = rows_of[combo % 3], ks = ks_of[(combo / 3) % 2], variant = combo / 6;
                    sparsert_options o = base;
                    o.kernel = SPARSERT_KERNEL_SPEC; o.spec_rows = rows; o.spec_ksplit = ks;
                    o.spec_swizzle = variant & 1;
                    if (variant == 1) { o.spec_depth = 2; o.spec_lanes = 32; }
                    if (variant == 2) { o.spec_vec = dtype == SPARSERT_F16 ? 2 : dtype == SPARSERT_I8 ? 4 : 1; o.ldb = N + 12; o.ldc = N + 4; }
                    if (variant == 3) { o.spec_mode = SPARSERT_SPEC_LDS; o.spec_ksplit = 0; o.spec_tiles = ks; o.batch = 2; }
                    exercise(c, M, K, N, o, true); ++plans;
                }
            }
        }
    }
    {   // the empty matrix
        const Csr c = make(9, 12, 0.0, 4, r, false);
        sparsert_options o;
        std::memset(&o, 0, sizeof(o));
        exercise(c, 9, 12, 70, o, false); ++plans;
        o.kernel = SPARSERT_KERNEL_ROWS;
        exercise(c, 9, 12, 70, o, false); ++plans;
    }
    // convolution plans: filter banks [Cout, Cin*9] on H x W images
    const int convs[][4] = {{3, 5, 1, 1}, {4, 6, 2, 3}, {6, 10, 9, 13}, {16, 24, 14, 14}};
    for (const auto &g : convs) {
        const int Cin = g[0], Cout = g[1], H = g[2], W = g[3];
        for (int dtype = SPARSERT_F32; dtype <= SPARSERT_I8; ++dtype) {
            const Csr c = make(Cout, 9 * Cin, 0.3, dtype == SPARSERT_F16 ? 2 : dtype == SPARSERT_I8 ? 1 : 4, r, false);
            sparsert_options o;
            std::memset(&o, 0, sizeof(o));
            o.dtype = dtype; o.conv = 1; o.Cin = Cin; o.H = H; o.W = W;
            for (int kernel : {SPARSERT_KERNEL_ROWS, SPARSERT_KERNEL_AUTO, SPARSERT_KERNEL_SPEC}) {
                o.kernel = kernel;
                for (int batch : {kernel == SPARSERT_KERNEL_AUTO ? 5 : 0}) {
                    o.batch = batch;
                    o.spec_rows = kernel == SPARSERT_KERNEL_SPEC ? 4 : 0;
                    o.spec_ksplit = kernel == SPARSERT_KERNEL_SPEC ? 4 : 0;
                    exercise(c, Cout, 9 * Cin, H * W, o, false); ++plans;
                }
            }
        }
    }
    // malformed input is refused before anything is read past its end
    {
        const int32_t rp_bad[] = {0, 2, 1}, cols[] = {0, 5}, rp_ok[] = {0, 1, 2}, cols_dup[] = {1, 1}, rp2[] = {0, 2, 2};
        const float v[] = {1.0f, 2.0f};
        sparsert_plan *p = nullptr;
        sparsert_options o;
        std::memset(&o, 0, sizeof(o));
        o.host_only = 1;
        EXPECT(sparsert_inspect(rp_bad, cols, v, 2, 8, 4, &o, &p) == SPARSERT_EINVAL && !p);
        EXPECT(sparsert_inspect(rp_ok, cols, v, 2, 4, 4, &o, &p) == SPARSERT_EINVAL && !p);        /* column 5 >= K */
        EXPECT(sparsert_inspect(rp2, cols_dup, v, 2, 4, 4, &o, &p) == SPARSERT_EINVAL && !p);      /* duplicate column */
        EXPECT(sparsert_inspect(nullptr, cols, v, 2, 4, 4, &o, &p) == SPARSERT_EINVAL && !p);
        EXPECT(sparsert_plan_load("SPRT", 4, 1, &p) == SPARSERT_EINVAL && !p);
    }
    std::printf("host sanitize run: %d plans built, exported, saved and reloaded; %d failed expectations\n", plans, failures);
    return failures ? 1 : 0;
}
