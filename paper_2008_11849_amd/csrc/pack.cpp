// Weights in the layouts of the fixed executors: fragments of zero-filled A for the matrix cores (mfma.hip), the
// pair stream of the LDS-staged row-walk kernel (staged_rows.hip), the
// records of the blocked one (blocked_rows.hip).  Host code only.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <exception>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

#include "blocked_rows.h"
#include "mfma.h"
#include "plan.h"
#include "staged_rows.h"

namespace sparsert {

// A as fragments, zero-filled to whole workgroup tiles and slabs.
void mfma_pack(const HostPlan &h, std::vector<uint8_t> &out) {
    const MfmaConfig &c = kMfmaConfigs[h.spec.mfma_config];
    const int esz = h.elem_size(), step = mfma_step(esz);
    const int64_t m_tiles = (h.M + c.tm - 1) / c.tm * (c.tm / 16), k_steps = (h.K + c.steps * step - 1) / (c.steps * step) * c.steps;
    out.assign((size_t)(m_tiles * k_steps) * 1024, 0);
    for (int32_t slot = 0; slot < h.M; ++slot) {
        const int32_t m = h.perm[slot];
        for (int32_t p = h.p_row_ptr[slot]; p < h.p_row_ptr[slot + 1]; ++p) {
            const int32_t k = h.p_col_idx[p];
            const int kk = k % step, half_step = step / 2, rows = step / 8;
            const int lane = kk % half_step / rows * 16 + m % 16, elem = kk / half_step * rows + kk % rows;
            std::memcpy(&out[(size_t)(((m / 16) * k_steps + k / step) * 64 + lane) * 16 + (size_t)elem * esz],
                        &h.p_vals[(size_t)p * esz], (size_t)esz);
        }
    }
}

// The nonzeros in the order the waves meet them, and what goes with it.
void staged_rows_pack(const HostPlan &h, StagedPack &out) {
    const StagedRows s = staged_rows_shape(h);
    const int rw = s.rows_per_wave, owners = s.groups * kStagedWaves;
    out.stream.reserve((size_t)h.nnz * 2 + (size_t)owners * s.chunks * rw * 3 + 32);
    out.counts.assign((size_t)owners * s.chunks * rw, 0);
    out.starts.assign(owners, 0);
    out.rows.assign((size_t)owners * rw, -1);
    std::vector<int32_t> slot_of((size_t)owners * rw, -1);
    for (int32_t i = 0; i < h.M; ++i) {   // serpentine over the groups, then over the waves of a group
        const int round = i / s.groups, pos = i % s.groups, g = round & 1 ? s.groups - 1 - pos : pos;
        const int r = round / kStagedWaves, w = round % kStagedWaves, wave = r & 1 ? kStagedWaves - 1 - w : w;
        const size_t at = ((size_t)g * kStagedWaves + wave) * rw + r;
        slot_of[at] = i;
        out.rows[at] = h.perm[i];
    }
    std::vector<int32_t> next((size_t)rw);
    for (int o = 0; o < owners; ++o) {
        out.starts[o] = (int32_t)(out.stream.size() / 2);
        for (int r = 0; r < rw; ++r) next[r] = slot_of[(size_t)o * rw + r] < 0 ? 0 : h.p_row_ptr[slot_of[(size_t)o * rw + r]];
        for (int c = 0; c < s.chunks; ++c)
            for (int r = 0; r < rw; ++r) {
                const int32_t slot = slot_of[(size_t)o * rw + r];
                if (slot < 0) continue;
                const int32_t limit = std::min<int64_t>(h.K, (int64_t)(c + 1) * s.chunk), end = h.p_row_ptr[slot + 1];
                int n = 0;
                const uint32_t zero_row = (uint32_t)(s.chunk * s.pitch);
                for (; next[r] < end && h.p_col_idx[next[r]] < limit; ++next[r], ++n) {
                    out.stream.push_back((uint32_t)(h.p_col_idx[next[r]] - c * s.chunk) * (uint32_t)s.pitch);
                    const uint32_t value = h.stream[2 * (size_t)next[r] + 1];
                    out.stream.push_back(h.dtype == SPARSERT_I8 ? (value & 0xffu) << (n % 2 * 8) : value);   // (int8: where the kernel wants it)
                }
                if (n % 2) { ++n; out.stream.push_back(zero_row); out.stream.push_back(0); }
                out.counts[((size_t)o * s.chunks + c) * rw + r] = (uint8_t)(n / 2);
            }
    }
    out.stream.resize(out.stream.size() + 32, 0);
}

// Blocks first ... last - 1: for every part of their columns the groups of columns as records.  Starts count from stream's own begin.
static void pack_blocks(const HostPlan &h, const BlockedRows &s, int first, int last, std::vector<uint32_t> &stream, BlockedPack &out) {
    stream.reserve(((size_t)((int64_t)h.nnz * (last - first) / s.blocks) / kBlockedColumns * 5 / 4 + (size_t)(last - first) * s.parts * 8) * kBlockedRecord);
    struct Entry { uint32_t row, value; };
    struct Column { int32_t column; uint32_t first, count; };
    std::vector<Entry> entries;                                  // of one block, by column
    std::vector<Column> all, columns, sorted;                    // the block's, and those of one part
    std::vector<uint32_t> position((size_t)h.K + 1);             // of a column's next entry
    std::vector<int32_t> touched;
    std::vector<uint32_t> of_count(kBlockedRows + 2);
    for (int b = first; b < last; ++b) {
        all.clear();
        touched.clear();
        auto each_slot = [&](auto f) {   // serpentine over the blocks
            for (int r = 0; r < s.rows; ++r) {
                const int64_t slot = (int64_t)r * s.blocks + (r & 1 ? s.blocks - 1 - b : b);
                if (slot < h.M) f(r, (int32_t)slot);
            }
        };
        each_slot([&](int r, int32_t slot) {
            out.rows[(size_t)b * kBlockedRows + r] = h.perm[slot];
            for (int32_t p = h.p_row_ptr[slot]; p < h.p_row_ptr[slot + 1]; ++p)
                if (position[h.p_col_idx[p]]++ == 0) touched.push_back(h.p_col_idx[p]);
        });
        // (few columns of a long K are sorted, many are met in order)
        if ((int64_t)touched.size() * 16 < h.K) std::sort(touched.begin(), touched.end());
        else for (int32_t k = 0, n = 0; k < h.K; ++k) if (position[k]) touched[n++] = k;
        uint32_t total = 0;
        for (int32_t k : touched) {
            all.push_back({k, total, position[k]});
            position[k] = total;
            total += all.back().count;
        }
        entries.resize(total);
        each_slot([&](int r, int32_t slot) {
            for (int32_t p = h.p_row_ptr[slot]; p < h.p_row_ptr[slot + 1]; ++p)
                entries[position[h.p_col_idx[p]]++] = {(uint32_t)r, h.stream[2 * (size_t)p + 1]};
        });
        for (int32_t k : touched) position[k] = 0;
        size_t next = 0;
        uint64_t seen = 0;
        for (int part = 0; part < s.parts; ++part) {   // an equal share of the nonzeros each
            columns.clear();
            for (; next < all.size() && (part == s.parts - 1 || seen * s.parts < (uint64_t)(part + 1) * total); ++next) {
                seen += all[next].count;
                columns.push_back(all[next]);
            }
            // most nonzeros first, columns of as many in order
            std::fill(of_count.begin(), of_count.end(), 0u);
            for (const Column &c : columns) ++of_count[c.count];
            for (uint32_t n = kBlockedRows + 1, at = 0; n-- > 0;) { const uint32_t here = of_count[n]; of_count[n] = at; at += here; }
            sorted.resize(columns.size());
            for (const Column &c : columns) sorted[of_count[c.count]++] = c;
            const size_t groups = (sorted.size() + kBlockedColumns - 1) / kBlockedColumns;
            auto layers = [&](size_t g) { return sorted[g * kBlockedColumns].count; };
            auto records = [&](size_t n) {
                stream.resize(stream.size() + n * kBlockedRecord, 0);
                return &stream[stream.size() - n * kBlockedRecord];
            };
            auto header = [&](size_t g) {
                uint32_t *w = records(1);
                for (size_t i = 0; i < kBlockedColumns && g * kBlockedColumns + i < sorted.size(); ++i)
                    w[i] = (uint32_t)sorted[g * kBlockedColumns + i].column * (uint32_t)h.ldb * (uint32_t)h.elem_size();
                w[kBlockedColumns] = g < groups ? layers(g) - 1 : ~0u;
            };
            out.starts[(size_t)b * s.parts + part] = (int32_t)(stream.size() / kBlockedRecord);
            header(0);
            header(1);
            for (size_t g = 0; g < groups; ++g) {
                const uint32_t depth = layers(g);
                uint32_t *w = records(depth);
                for (size_t i = 0; i < kBlockedColumns; ++i) {
                    const size_t c = g * kBlockedColumns + i;
                    const uint32_t count = c < sorted.size() ? sorted[c].count : 0, shift = 8 * (i % 4);
                    const Entry *e = count ? &entries[sorted[c].first] : nullptr;
                    for (uint32_t l = 0; l < count; ++l) {
                        w[l * kBlockedRecord + i] = e[l].value;
                        w[l * kBlockedRecord + kBlockedColumns + i / 4] |= e[l].row << shift;
                    }
                    for (uint32_t l = count; l < depth; ++l) w[l * kBlockedRecord + kBlockedColumns + i / 4] |= (uint32_t)kBlockedRows << shift;
                }
                header(g + 2);
            }
        }
    }
}

void blocked_rows_pack(const HostPlan &h, const BlockedRows &s, BlockedPack &out) {
    out.starts.assign((size_t)s.blocks * s.parts, 0);
    out.rows.assign((size_t)s.blocks * kBlockedRows, -1);
    // 15 ns per nonzero: a host thread for every 128 Ki nonzeros, up to eight (4096 x 4096 at 90 %: 24 -> 14 ms)
    const int shares = std::max(1, (int)std::min<int64_t>({8, s.blocks, h.nnz >> 17, (int64_t)std::thread::hardware_concurrency()}));
    std::vector<std::vector<uint32_t>> streams(shares);
    auto first = [&](int i) { return (int)((int64_t)s.blocks * i / shares); };
    std::vector<std::exception_ptr> failed(shares);
    auto share = [&](int i) {
        try {
            pack_blocks(h, s, first(i), first(i + 1), streams[i], out);
        } catch (...) {
            failed[i] = std::current_exception();
        }
    };
    std::vector<std::thread> threads;
    threads.reserve(shares);
    int started = 1;
    try {
        for (; started < shares; ++started) threads.emplace_back(share, started);
    } catch (const std::system_error &) {   // no more threads, or no memory for one: the rest is done here, and those that run are joined
    } catch (const std::bad_alloc &) {
    }
    share(0);
    for (int i = started; i < shares; ++i) share(i);
    for (auto &t : threads) t.join();
    for (auto &f : failed)
        if (f) std::rethrow_exception(f);
    size_t words = 2 * kBlockedRecord;   // a wave reads a record ahead
    for (auto &w : streams) words += w.size();
    out.stream.reserve(words);
    for (int i = 0; i < shares; ++i) {
        const int32_t before = (int32_t)(out.stream.size() / kBlockedRecord);
        for (int64_t at = (int64_t)first(i) * s.parts; at < (int64_t)first(i + 1) * s.parts; ++at) out.starts[at] += before;
        out.stream.insert(out.stream.end(), streams[i].begin(), streams[i].end());
    }
    out.stream.resize(words, 0);
}

}  // namespace sparsert
