// Weights in the layouts of the fixed executors: fragments of zero-filled A for the matrix cores (mfma.hip), the
// pair stream of the LDS-staged row-walk kernel (staged_rows.hip).  Host code only.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

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

}  // namespace sparsert
