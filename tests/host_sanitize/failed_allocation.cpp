// Packs a plan for the blocked row-walk kernel with every allocation of the calling thread failing in turn, packing threads
// already running or not: it leaves as std::bad_alloc, which the C boundary turns into a status, or costs a thread, and the process
// goes on.  A program of its own: it replaces operator new, which the sanitizers' runtime also does.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "../../paper_2008_11849_amd/csrc/blocked_rows.h"

static thread_local int allocations_left = -1;   // until one of this thread fails; -1: none does
void *operator new(std::size_t bytes) {
    if (allocations_left > 0) --allocations_left;
    void *p = allocations_left == 0 ? nullptr : std::malloc(bytes ? bytes : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main() {
    sparsert::HostPlan h;   // as far as the packer reads it: nonzeros enough for four threads
    h.M = 2048; h.K = 1024; h.N = h.ldb = h.ldc = 784; h.nnz = h.M * 256;
    h.p_row_ptr.push_back(0);
    for (int m = 0; m < h.M; ++m) {
        h.perm.push_back(m);
        for (int i = 0; i < 256; ++i) {
            h.p_col_idx.push_back(4 * i + m % 4);
            h.stream.push_back(0);
            h.stream.push_back((unsigned)(m * 256 + i));
        }
        h.p_row_ptr.push_back((int)h.p_col_idx.size());
    }
    sparsert::BlockedRows s;
    s.rows = 64; s.blocks = 32; s.parts = 4;
    sparsert::BlockedPack whole;
    sparsert::blocked_rows_pack(h, s, whole);
    int failed = 0, refused = 0;
    for (int n = 1; n < 1000; ++n) {
        sparsert::BlockedPack pack;
        bool threw = false;
        allocations_left = n;
        try {
            sparsert::blocked_rows_pack(h, s, pack);
        } catch (const std::bad_alloc &) {
            threw = true;
        }
        const bool none = allocations_left > 0;
        allocations_left = -1;
        if (threw ? none : pack.stream != whole.stream || pack.starts != whole.starts || pack.rows != whole.rows) ++failed;
        refused += threw;
        if (none) {
            std::printf("%d allocations, %d of them refuse the plan; %d failed expectations\n", n - 1, refused, failed);
            return failed ? 1 : 0;
        }
    }
    return 2;
}
