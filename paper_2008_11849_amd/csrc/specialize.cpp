// Per-matrix specialised executor (Section 3.5 of the paper, re-derived for gfx950).
//
// The paper unrolls the nonzero loop of Algorithm 3 into straight-line code with the
// values of A as instruction constants, so that (i) every accumulator has a fixed
// register, (ii) a row of B is loaded once and reused by every nonzero of that column
// inside the tile, (iii) A costs no data-cache traffic at all.  It emits PTX directly
// instead of going through the high-level compiler (Section 3.7).  The same is done here
// for CDNA4: the inspector emits gfx950 assembly and has the code object manager assemble
// it; going through the HIP compiler took ~50 s for the c3 matrix and serialised every
// load behind its use.
//
// Shape of the generated kernel `sparsert_spec`
//   wave  = one row group g (<= R rows, dealt by the inspector for nonzero balance,
//           Section 3.4) x one column tile (lanes own one column of C each)
//   code  = one straight-line block per group: for each column k that has a nonzero in
//           the group, ascending: fetch b <- B[k, tile columns] (several columns ahead),
//           then  v_fmac_f32 acc[row] += literal(A[row,k]) * b  for every nonzero (row,k);
//           finally one store per row.  No loops, no index loads.
//   DIRECT: workgroup = T waves running the same block on T adjacent tiles; b comes
//           straight from L2/L1 with buffer loads.
//   DIRECT with K split: workgroup = KS waves sharing one block and one tile, each walking
//           a contiguous range of the block's columns with an equal share of its nonzeros
//           (Section 3.4); the partial sums meet in LDS after the walk (Section 3.3).
//   LDS   : workgroup = W waves running W adjacent blocks on the same tile (SpMM; fp32, and half
//           and int8 widened to 32 bits on their way into LDS).  The tile's
//           B rows are staged once per workgroup through LDS in chunks of up to 128 rows
//           (double buffered, one barrier per chunk; each wave fetches a 1/W share) and
//           every wave reads its b values from LDS with compile-time offsets.  Measured
//           on MI355X the vector-memory path delivers ~37 B/clk per CU, the LDS path
//           several times that, and each FMA needs 4 B of b: DIRECT is load bound.
// All global addresses are "descriptor base + row offset literal + lane column offset"
// with the column clamped to the tile, so every access is in bounds by construction.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <dlfcn.h>
#include <map>
#include <mutex>
#include <stdexcept>
#include <string>

#include "mfma.h"
#include "plan.h"

namespace sparsert {

namespace {

// ---------------------------------------------------------------- code object manager
// Loaded at run time so the library itself has no link-time dependency on it.  The entry points
// and the enumerator values below are those of interface version 3 of the code object manager
// (amd_comgr.h); a library that reports another major version is not used.
constexpr size_t kComgrMajor = 3;
typedef struct { uint64_t handle; } comgr_handle;
enum { COMGR_SUCCESS = 0, COMGR_KIND_SOURCE = 1, COMGR_KIND_RELOCATABLE = 7, COMGR_KIND_EXECUTABLE = 8,
       COMGR_KIND_LOG = 5, COMGR_ACTION_LINK_RELOC_TO_EXE = 7, COMGR_ACTION_ASSEMBLE = 8 };

struct Comgr {
    void *lib = nullptr;
    int (*create_data)(int, comgr_handle *) = nullptr;
    int (*release_data)(comgr_handle) = nullptr;
    int (*set_data)(comgr_handle, size_t, const char *) = nullptr;
    int (*set_data_name)(comgr_handle, const char *) = nullptr;
    int (*get_data)(comgr_handle, size_t *, char *) = nullptr;
    int (*create_data_set)(comgr_handle *) = nullptr;
    int (*destroy_data_set)(comgr_handle) = nullptr;
    int (*data_set_add)(comgr_handle, comgr_handle) = nullptr;
    int (*action_data_count)(comgr_handle, int, size_t *) = nullptr;
    int (*action_data_get_data)(comgr_handle, int, size_t, comgr_handle *) = nullptr;
    int (*create_action_info)(comgr_handle *) = nullptr;
    int (*destroy_action_info)(comgr_handle) = nullptr;
    int (*set_isa_name)(comgr_handle, const char *) = nullptr;
    int (*set_logging)(comgr_handle, bool) = nullptr;
    int (*do_action)(int, comgr_handle, comgr_handle, comgr_handle) = nullptr;
    void (*get_version)(size_t *, size_t *) = nullptr;
    size_t major = 0, minor = 0;
    bool ok = false;
};

Comgr &comgr() {
    static Comgr c;
    static std::once_flag once;
    std::call_once(once, [] {
        const char *names[] = {"libamd_comgr.so.3", "libamd_comgr.so", "/opt/rocm/lib/libamd_comgr.so.3",
                               "/opt/rocm/lib/libamd_comgr.so"};
        for (const char *n : names)
            if ((c.lib = dlopen(n, RTLD_NOW | RTLD_LOCAL))) break;
        if (!c.lib) return;
        bool all = true;
        auto sym = [&](const char *n) { void *p = dlsym(c.lib, n); all = all && p; return p; };
#define COMGR_SYM(field, name) c.field = reinterpret_cast<decltype(c.field)>(sym(name))
        COMGR_SYM(create_data, "amd_comgr_create_data");
        COMGR_SYM(release_data, "amd_comgr_release_data");
        COMGR_SYM(set_data, "amd_comgr_set_data");
        COMGR_SYM(set_data_name, "amd_comgr_set_data_name");
        COMGR_SYM(get_data, "amd_comgr_get_data");
        COMGR_SYM(create_data_set, "amd_comgr_create_data_set");
        COMGR_SYM(destroy_data_set, "amd_comgr_destroy_data_set");
        COMGR_SYM(data_set_add, "amd_comgr_data_set_add");
        COMGR_SYM(action_data_count, "amd_comgr_action_data_count");
        COMGR_SYM(action_data_get_data, "amd_comgr_action_data_get_data");
        COMGR_SYM(create_action_info, "amd_comgr_create_action_info");
        COMGR_SYM(destroy_action_info, "amd_comgr_destroy_action_info");
        COMGR_SYM(set_isa_name, "amd_comgr_action_info_set_isa_name");
        COMGR_SYM(set_logging, "amd_comgr_action_info_set_logging");
        COMGR_SYM(do_action, "amd_comgr_do_action");
        COMGR_SYM(get_version, "amd_comgr_get_version");
#undef COMGR_SYM
        if (all) c.get_version(&c.major, &c.minor);
        c.ok = all && c.major == kComgrMajor;
    });
    return c;
}

std::string fetch_log(Comgr &c, comgr_handle set) {
    size_t n = 0;
    std::string out;
    if (c.action_data_count(set, COMGR_KIND_LOG, &n) != COMGR_SUCCESS) return out;
    for (size_t i = 0; i < n; ++i) {
        comgr_handle d;
        if (c.action_data_get_data(set, COMGR_KIND_LOG, i, &d) != COMGR_SUCCESS) continue;
        size_t sz = 0;
        if (c.get_data(d, &sz, nullptr) == COMGR_SUCCESS && sz) {
            std::string s(sz, '\0');
            c.get_data(d, &sz, &s[0]);
            out += s.substr(0, 2000);
        }
        c.release_data(d);
    }
    return out;
}

int assemble(const std::string &text, std::vector<char> &code, std::string &err) {
    Comgr &c = comgr();
    if (!c.ok) {
        err = c.lib && c.major != kComgrMajor
                  ? "code object manager (libamd_comgr) has interface version " + std::to_string(c.major) + "." +
                        std::to_string(c.minor) + ", this library was written against version 3"
                  : std::string("code object manager (libamd_comgr) is not available");
        return SPARSERT_ECOMPILE;
    }
    comgr_handle src{0}, in{0}, rel{0}, exe{0}, info{0}, out{0};
    int rc = SPARSERT_ECOMPILE;
    bool have_src = false, have_in = false, have_rel = false, have_exe = false, have_info = false;
    do {
        if (c.create_data(COMGR_KIND_SOURCE, &src)) { err = "comgr create_data"; break; }
        have_src = true;
        if (c.set_data(src, text.size(), text.data()) || c.set_data_name(src, "sparsert_spec.s")) { err = "comgr set_data"; break; }
        if (c.create_data_set(&in)) { err = "comgr create_data_set"; break; }
        have_in = true;
        if (c.data_set_add(in, src)) { err = "comgr data_set_add"; break; }
        if (c.create_data_set(&rel)) { err = "comgr create_data_set"; break; }
        have_rel = true;
        if (c.create_data_set(&exe)) { err = "comgr create_data_set"; break; }
        have_exe = true;
        if (c.create_action_info(&info)) { err = "comgr create_action_info"; break; }
        have_info = true;
        if (c.set_isa_name(info, "amdgcn-amd-amdhsa--gfx950")) { err = "comgr does not know gfx950"; break; }
        c.set_logging(info, true);
        if (c.do_action(COMGR_ACTION_ASSEMBLE, info, in, rel)) { err = "assembling the generated kernel failed: " + fetch_log(c, rel); break; }
        if (c.do_action(COMGR_ACTION_LINK_RELOC_TO_EXE, info, rel, exe)) { err = "linking the generated kernel failed: " + fetch_log(c, exe); break; }
        size_t n = 0;
        if (c.action_data_count(exe, COMGR_KIND_EXECUTABLE, &n) || n != 1) { err = "comgr produced no executable"; break; }
        if (c.action_data_get_data(exe, COMGR_KIND_EXECUTABLE, 0, &out)) { err = "comgr get executable"; break; }
        size_t sz = 0;
        if (c.get_data(out, &sz, nullptr) == COMGR_SUCCESS && sz) {
            code.resize(sz);
            if (c.get_data(out, &sz, code.data()) == COMGR_SUCCESS) rc = SPARSERT_OK;
        }
        c.release_data(out);
        if (rc != SPARSERT_OK) err = "comgr get executable bytes";
    } while (false);
    if (have_info) c.destroy_action_info(info);
    if (have_exe) c.destroy_data_set(exe);
    if (have_rel) c.destroy_data_set(rel);
    if (have_in) c.destroy_data_set(in);
    if (have_src) c.release_data(src);
    return rc;
}

// ---------------------------------------------------------------- assembly text
struct Emitter {
    std::string s;
    int64_t lines = 0, bytes = 0;   // text lines; code bytes, as if every constant that may be one were a literal
    char buf[256];
    void line(const char *fmt, ...) __attribute__((format(printf, 2, 3))) {
        va_list ap;
        va_start(ap, fmt);
        int n = vsnprintf(buf, sizeof(buf), fmt, ap);
        va_end(ap);
        s.append(buf, (size_t)n);
        s.push_back('\n');
        ++lines;
        bytes += code_bytes(fmt);
    }
    static int code_bytes(const char *fmt) {
        static const char *const kShort[] = {"s_waitcnt", "s_mov_b64", "s_movk", "s_barrier", "s_endpgm", "s_nop", "v_mov", "v_cvt_f32_f16_e32", "v_cvt_f16_f32_e32", "%s v%d, v%d, v%d"};
        if (fmt[0] != '\t' || fmt[1] == '.') return 0;   // labels and directives
        for (const char *k : kShort)
            if (!std::strncmp(fmt + 1, k, std::strlen(k))) return 4;
        return 8;
    }
};

// Fixed register plan of the generated kernel.
constexpr int kSgprB = 4, kSgprC = 6;          // kernarg pointers
constexpr int kRsrcB = 8, kRsrcC = 12;         // buffer descriptors (4 SGPRs each)
constexpr int kSgprTile = 16, kSgprBlock = 17, kSgprPc = 18, kSgprTmp = 20, kSgprTmp2 = 21;
constexpr int kSgprOwns = 22;                  // s[22:23] lanes that own a column
constexpr int kSgprOffRing = 24, kOffRing = 8; // s[24:31] row-offset literals in flight
constexpr int kSgprTap0 = 32;                  // conv: s[32:49] = lane masks of the 9 filter taps
constexpr int kSgprFull = 50;                  // conv: s[50:51] = all lanes
constexpr int kSgprImage = 52;                 // batch > 1: workgroup id z = image / matrix of the batch
constexpr int kSgprJump = 53;                  // byte offset of the block's entry in the table
constexpr int kSgprEntry = 54;                 // prologue only, s[54:55]: the block's table entry and the next one's (offsets of their code from the table)
constexpr int kSgprValRing = 54, kValRing = 8; // half / int8 plans: s[54:61] values of A on their way into the multiply-add
constexpr int kSgprTab = 62, kTab = 32;        // DIRECT: s[62:93] = i * (bytes between consecutive operand rows), i < 32
constexpr int kNextFreeSgpr = 94;
constexpr int kVgprOff = 0;                    // byte offset of the lane's column inside a row
constexpr int kVgprLds = 1;                    // LDS byte address of the lane's 16-byte slot
constexpr int kVgprT1 = 2, kVgprT2 = 3, kVgprAcc0 = 4;
constexpr int kVgprOut = kVgprT2;               // byte offset of the lane's column inside a row of C (after the prologue)
constexpr uint32_t kRsrcWord3 = 0x00020000u;   // raw 32-bit buffer, gfx9 family
constexpr int kMaxChunkRows = 128;             // B rows per LDS buffer (32 KiB), two buffers
constexpr int kMaxLdsBytes = 160 * 1024;        // LDS of one gfx950 compute unit, all of it usable by one workgroup
constexpr int kMaxLgkm = 15;                   // lgkmcnt is a 4-bit counter

struct Term { int acc; uint32_t bits; };

struct Gen {
    Emitter e;
    const HostPlan &h;
    SpecPlan &sp;
    int N, K, D;
    int64_t ldb, ldc;    // elements between consecutive rows of B and of C
    bool half = false;   // B, C and the values of A are IEEE half; sums stay fp32
    bool int8 = false;   // B and the values of A are int8, C is int32, sums are exact integers
    int esz = 4;         // bytes of an element of B / X
    int osz = 4;         // bytes of an element of C / Y
    int val_pos = 0;     // half / int8 plans: next slot of the value ring
    int V = 1;           // columns per lane: 2 halves or 4 int8 packed in the dword a lane loads
    int vgpr_unpack0 = 0;  // int8, V = 4: four registers holding the sign-extended bytes of the current operand;
                           // half, V = 2: one register holding the widened high half
    int vgpr_stage0 = 0, vgpr_ring0 = 0, n_vgpr = 0, lds_bytes = 0;
    int ring_size = 0;               // DIRECT: registers of the operand ring (>= D)
    int slot_bytes = 256;            // K split: bytes of one row's partial sums in the exchange area
    int xchg_rows = 0;               // K split: rows exchanged per phase (all of them if they fit the LDS)
    bool stream_stores = false;      // every wave store of C covers whole 128-byte lines
    bool staged = false;             // LDS variant: operands reach the multiply-adds through LDS, already widened to 32 bits
    int chunk_rows = kMaxChunkRows;  // LDS mode: 32 rows per wave of the workgroup, at most 128
    Gen(const HostPlan &hp, SpecPlan &s)
        : h(hp), sp(s), N(hp.N), K(hp.K), D(s.depth), ldb(hp.ldb), ldc(hp.ldc), half(hp.dtype == SPARSERT_F16), int8(hp.dtype == SPARSERT_I8),
          esz(half ? 2 : int8 ? 1 : 4), osz(half ? 2 : 4) {}

    void zero_accs(size_t n) {
        for (size_t i = 0; i < n * (size_t)V; ++i) e.line("\tv_mov_b32_e32 v%d, 0", kVgprAcc0 + (int)i);
    }
    // The value of A is a literal of the multiply-add.  Half storage: the operand just fetched is
    // widened to fp32 in place, once per fetched row of B (exact), and the value - widened to fp32
    // at generation time, exact as well - is the literal, so a nonzero costs one instruction as in
    // fp32 and the sums are the same fp32 multiply-adds.
    int acc_reg(int row, int j = 0) const { return kVgprAcc0 + row * V + j; }
    void fmas(const std::vector<Term> &terms, int vb) {
        if (terms.empty()) return;
        if (int8 && V == 4)   // the four packed operands, sign-extended once per fetched row of B
            for (int j = 0; j < 4; ++j) e.line("\tv_bfe_i32 v%d, v%d, %d, 8", vgpr_unpack0 + j, vb, 8 * j);
        if (half && !staged) {
            if (V == 2)   // the high half of the dword is the next column
                e.line("\tv_cvt_f32_f16_sdwa v%d, v%d dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1", vgpr_unpack0, vb);
            e.line("\tv_cvt_f32_f16_e32 v%d, v%d", vb, vb);
        }
        for (const Term &t : terms) {
            if (int8) {
                // exact: both factors fit 24 bits; values in -16..64 are inline constants
                const int32_t a = (int32_t)t.bits;
                char src[16];
                if (a >= -16 && a <= 64) {
                    snprintf(src, sizeof(src), "%d", a);
                } else {
                    const int sv = kSgprValRing + (val_pos++ % kValRing);
                    e.line("\ts_movk_i32 s%d, %d", sv, a);
                    snprintf(src, sizeof(src), "s%d", sv);
                }
                for (int j = 0; j < V; ++j)
                    e.line("\tv_mad_i32_i24 v%d, %s, v%d, v%d", acc_reg(t.acc, j), src, V == 4 ? vgpr_unpack0 + j : vb,
                           acc_reg(t.acc, j));
            } else {
                e.line("\tv_fmac_f32_e32 v%d, 0x%08x, v%d", acc_reg(t.acc), t.bits, vb);
                if (V == 2) e.line("\tv_fmac_f32_e32 v%d, 0x%08x, v%d", acc_reg(t.acc, 1), t.bits, vgpr_unpack0);
            }
        }
    }
    const char *load_op() const {
        return V > 1 ? "buffer_load_dword" : half ? "buffer_load_short_d16" : int8 ? "buffer_load_sbyte" : "buffer_load_dword";
    }
    void load_b_row(int k, int vdst, int ring_pos) {
        const int sreg = kSgprOffRing + (ring_pos % kOffRing);
        e.line("\ts_mov_b32 s%d, 0x%llx", sreg, (unsigned long long)((int64_t)k * ldb * esz));
        e.line("\t%s v%d, v%d, s[%d:%d], s%d offen", load_op(), vdst, kVgprOff, kRsrcB, kRsrcB + 3, sreg);
    }
    // (slot of the permuted CSR, first accumulator register of the row) pairs: one row of C each
    void stores(const std::vector<std::pair<int32_t, int>> &rows) {
        if (rows.empty()) return;
        e.line("\ts_mov_b64 exec, s[%d:%d]", kSgprOwns, kSgprOwns + 1);
        for (size_t i = 0; i < rows.size(); ++i) {
            const int sreg = kSgprOffRing + ((int)i % kOffRing), r = rows[i].second;
            e.line("\ts_mov_b32 s%d, 0x%llx", sreg, (unsigned long long)((int64_t)h.perm[rows[i].first] * ldc * osz));
            const char *op = "buffer_store_dword";
            if (half) {   // one rounding to nearest even, at the store
                for (int j = 0; j < V; ++j) e.line("\tv_cvt_f16_f32_e32 v%d, v%d", r + j, r + j);
                if (V == 2) e.line("\tv_pack_b32_f16 v%d, v%d, v%d", r, r, r + 1);
                else op = "buffer_store_short";
            }
            // C is written once and not read again by this kernel: where a wave's store covers whole
            // 128-byte lines the non-temporal hint keeps C from displacing the code and the rows of B
            // in the L2 (measured: c3 11.5 -> 10.5 us); on partial lines (N = 49, 196, 784) the same
            // hint costs 0.35 us, so it is left off there
            const char *hint = stream_stores ? " nt" : "";
            if (int8 && V == 4)
                e.line("\tbuffer_store_dwordx4 v[%d:%d], v%d, s[%d:%d], s%d offen%s", r, r + 3, kVgprOut, kRsrcC, kRsrcC + 3, sreg, hint);
            else
                e.line("\t%s v%d, v%d, s[%d:%d], s%d offen%s", op, r, kVgprOut, kRsrcC, kRsrcC + 3, sreg, hint);
        }
    }

    // column -> nonzeros of the group, ascending columns
    std::map<int32_t, std::vector<Term>> columns_of(const std::vector<int32_t> &rows) const {
        std::map<int32_t, std::vector<Term>> cols;
        for (size_t i = 0; i < rows.size(); ++i) {
            const int32_t slot = rows[i];
            for (int32_t p = h.p_row_ptr[slot]; p < h.p_row_ptr[slot + 1]; ++p) {
                uint32_t bits;  // the value as stored (the conv stream is reordered, p_vals is not), as fp32
                if (half) {
                    uint16_t hb;
                    std::memcpy(&hb, &h.p_vals[(size_t)p * 2], 2);
                    bits = half_bits_to_float_bits(hb);
                } else if (int8) {
                    bits = (uint32_t)(int32_t)(int8_t)h.p_vals[(size_t)p];   // the integer value itself
                } else {
                    std::memcpy(&bits, &h.p_vals[(size_t)p * 4], 4);
                }
                cols[h.p_col_idx[p]].push_back({(int)i, bits});
            }
        }
        return cols;
    }

    // Convolution (Section 3.6): operand row k = c*9 + tap is the input plane c displaced by the
    // tap; relative to the descriptor base X - (W+1) elements that is c*H*W + r*W + s elements.
    void load_x_row(int k, int vdst, int ring_pos) {
        const int c = k / 9, tap = k % 9, r = tap / 3, t = tap % 3;
        const int sreg = kSgprOffRing + (ring_pos % kOffRing);
        e.line("\ts_mov_b32 s%d, 0x%llx", sreg, (unsigned long long)(((int64_t)c * h.H * h.W + r * h.W + t) * esz));
        e.line("\t%s v%d, v%d, s[%d:%d], s%d offen", load_op(), vdst, kVgprOff, kRsrcB, kRsrcB + 3, sreg);
    }
    int cur_mask = -1;  // conv: tap whose lane mask is in exec; -1 = all lanes
    void want_mask(int tap) {
        if (tap == cur_mask) return;
        if (tap < 0) e.line("\ts_mov_b64 exec, s[%d:%d]", kSgprFull, kSgprFull + 1);
        else e.line("\ts_mov_b64 exec, s[%d:%d]", kSgprTap0 + 2 * tap, kSgprTap0 + 2 * tap + 1);
        cur_mask = tap;
    }

    // DIRECT: b values come straight from global memory, D columns in flight.  For a
    // convolution the columns are walked tap by tap and every load and multiply-add of a tap
    // runs under that tap's lane mask: lanes whose tap falls into the padding neither read
    // nor accumulate, which is the zero contribution of the padding.
    // With `parts` > 1 the waves of a workgroup share the block's rows and tile and split its
    // columns (Section 3.4, thread-group balance: contiguous ranges with equal nonzero counts,
    // the last one takes the remainder); partial accumulators meet in LDS (Section 3.3).
    int block_direct(const std::vector<int32_t> &rows, int part = 0, int parts = 1) {
        auto cols = columns_of(rows);
        std::vector<int32_t> order;
        for (auto &kv : cols) order.push_back(kv.first);
        if (h.conv)
            std::stable_sort(order.begin(), order.end(), [](int32_t a, int32_t b) { return a % 9 < b % 9; });
        if (parts > 1) {
            int64_t total = 0;
            for (int32_t k : order) total += (int64_t)cols[k].size();
            const int64_t share = (total + parts - 1) / parts;
            std::vector<int32_t> mine;
            int64_t seen = 0;
            for (int32_t k : order) {   // a column belongs to the part its first nonzero falls into
                const int p = share ? (int)std::min<int64_t>(parts - 1, seen / share) : 0;
                if (p == part) mine.push_back(k);
                seen += (int64_t)cols[k].size();
            }
            order.swap(mine);
        }
        const int nc = (int)order.size();
        cur_mask = -1;
        // Byte offset of operand row k from the descriptor base (convolution: Section 3.6, operand row
        // k = c*9 + tap is the input plane c displaced by the tap).
        auto offset_of = [&](int32_t k) -> int64_t {
            if (!h.conv) return (int64_t)k * ldb * esz;
            const int c = k / 9, tap = k % 9;
            return ((int64_t)c * h.H * h.W + (tap / 3) * h.W + tap % 3) * esz;
        };
        // Where the rows a block fetches lie close together, their offsets come from a table of
        // multiples of the row pitch kept in scalar registers, and the lane's address register is
        // advanced when a row falls outside the table's reach: no scalar move per fetch.  Blocks
        // whose rows are far apart would advance at every fetch and keep the move instead.
        const int64_t unit = h.conv ? (int64_t)h.H * h.W * esz : ldb * esz;
        bool use_tab = false;
        {
            int64_t base = 0;
            int bumps = 0;
            for (int j = 0; j < nc; ++j) {
                const int64_t d = offset_of(order[j]) - base;
                if (d < 0 || d % unit || d / unit >= kTab) { ++bumps; base += d; }
            }
            use_tab = nc >= 16 && (int64_t)bumps * (h.conv ? 12 : 4) <= nc;
        }
        bool tab_ready[kTab] = {false};   // an entry is written right before its first use, so no fetch waits for the whole table
        int64_t cur_base = 0;             // bytes the address register has been advanced by so far
        auto issue = [&](int j) {
            const int vdst = vgpr_ring0 + (j % D);
            if (!use_tab) {
                if (h.conv) { want_mask(order[j] % 9); load_x_row(order[j], vdst, j); }
                else load_b_row(order[j], vdst, j);
                return;
            }
            int64_t d = offset_of(order[j]) - cur_base;
            if (d < 0 || d % unit || d / unit >= kTab) {
                if (h.conv) want_mask(-1);   // every lane's address moves, whatever tap mask is current
                e.line("\tv_add_u32_e32 v%d, 0x%x, v%d", kVgprOff, (uint32_t)(int32_t)d, kVgprOff);
                cur_base += d;
                d = 0;
            }
            if (h.conv) want_mask(order[j] % 9);
            const int slot = (int)(d / unit);
            if (!tab_ready[slot]) {
                e.line("\ts_mov_b32 s%d, 0x%llx", kSgprTab + slot, (unsigned long long)(slot * unit));
                tab_ready[slot] = true;
            }
            e.line("\t%s v%d, v%d, s[%d:%d], s%d offen", load_op(), vdst, kVgprOff, kRsrcB, kRsrcB + 3, kSgprTab + slot);
        };
        for (int j = 0; j < std::min(D, nc); ++j) issue(j);
        // the accumulators are cleared while the first fetches are on their way
        if (h.conv) want_mask(-1);
        zero_accs(rows.size());
        for (int j = 0; j < nc; ++j) {
            // loads issued so far: columns [0, min(nc, j + D)); those after column j may stay in
            // flight.  (Waiting once per batch of columns was measured slower than once per column.)
            e.line("\ts_waitcnt vmcnt(%d)", std::min(nc, j + D) - 1 - j);
            if (h.conv) want_mask(order[j] % 9);
            fmas(cols[order[j]], vgpr_ring0 + (j % D));
            if (j + D < nc) issue(j + D);
        }
        if (parts > 1) {
            if (h.conv) want_mask(-1);
            // The rows of the block are dealt to the waves in contiguous runs of ceil(rows / parts).
            // Every wave leaves its partial sums of the rows it does not own in LDS, and after
            // one barrier adds the other waves' partials to its own rows in ascending wave order,
            // then stores those rows.  The accumulators of a run are consecutive registers, so
            // they travel four (two, one) at a time: a piece of n registers from one wave is an
            // LDS region [lane][n dwords], written and read with one 16- (8-, 4-) byte access per
            // lane.  Blocks whose partial sums do not fit the LDS at once exchange them in phases
            // of xchg_rows rows, with a second barrier before the area is overwritten.
            const int nr = (int)rows.size();
            const int chunk = (nr + parts - 1) / parts;
            auto own_lo = [&](int q) { return std::min(nr, q * chunk); };
            auto own_hi = [&](int q) { return std::min(nr, (q + 1) * chunk); };
            const int rb = slot_bytes / V;                        // bytes of one register's partials over the lanes of a tile
            const int cq = nr <= xchg_rows ? std::max(1, chunk) : std::max(1, xchg_rows / parts);   // rows per owner and phase
            const int n_phases = (chunk + cq - 1) / cq;
            struct Piece { int reg, len, off; };                  // first register, registers, byte offset of the region
            // address registers: lane * 4n for the three piece sizes, one set per 64 KiB window of
            // the area (ds offsets are 16 bits wide); they and the temporaries borrow the operand ring
            const int n_win = (lds_bytes + 65535) / 65536;
            const int base0 = vgpr_ring0;
            auto addr_reg = [&](int len, int off) {
                const int m = len == 4 ? 2 : len == 2 ? 1 : 0, w = off >> 16;
                return m == 0 && w == 0 ? kVgprLds : base0 + m * n_win + w - 1;
            };
            for (int m = 0; m < 3; ++m)
                for (int w = 0; w < n_win; ++w) {
                    if (m == 0 && w == 0) continue;
                    const int r = addr_reg(1 << m, w << 16);
                    if (m == 0) e.line("\tv_add_u32_e32 v%d, 0x%x, v%d", r, w * 65536, kVgprLds);
                    else if (w == 0) e.line("\tv_lshlrev_b32_e32 v%d, %d, v%d", r, m, kVgprLds);
                    else e.line("\tv_add_u32_e32 v%d, 0x%x, v%d", r, w * 65536, addr_reg(1 << m, 0));
                }
            const int tmp0 = (base0 + 3 * n_win - 1 + 1) / 2 * 2;   // even: 64-bit and wider operands need aligned registers
            const int n_tmp = vgpr_ring0 + ring_size - tmp0;
            if (n_tmp < 4) throw std::runtime_error("operand ring too small for the partial-sum exchange");
            static const char *const kWidth[5] = {"", "b32", "b64", "", "b128"};
            auto vregs = [](int r, int len, char *buf, size_t cap) {
                if (len == 1) snprintf(buf, cap, "v%d", r); else snprintf(buf, cap, "v[%d:%d]", r, r + len - 1);
            };
            std::vector<std::pair<int32_t, int>> mine;
            for (int i = own_lo(part); i < own_hi(part); ++i) mine.push_back({rows[i], acc_reg(i)});
            for (int ph = 0; ph < n_phases; ++ph) {
                // layout of the phase: for every owner q and every other wave s, the pieces of
                // q's rows of this phase as s left them
                std::vector<std::vector<std::vector<Piece>>> lay(parts, std::vector<std::vector<Piece>>(parts));
                int area = 0;
                for (int q = 0; q < parts; ++q) {
                    const int lo = std::min(own_hi(q), own_lo(q) + ph * cq), hi = std::min(own_hi(q), lo + cq);
                    for (int sw = 0; sw < parts; ++sw) {
                        if (sw == q) continue;
                        for (int f = lo * V; f < hi * V;) {
                            const int reg = kVgprAcc0 + f;
                            const int len = (reg & 1) ? 1 : f + 4 <= hi * V ? 4 : f + 2 <= hi * V ? 2 : 1;
                            lay[q][sw].push_back({reg, len, area});
                            area += len * rb;
                            f += len;
                        }
                    }
                }
                if (area > lds_bytes) throw std::runtime_error("partial-sum exchange exceeds its LDS area");
                if (ph > 0) e.line("\ts_barrier");   // every wave has read the previous phase
                char regs[32];
                for (int q = 0; q < parts; ++q)
                    for (const Piece &pc : lay[q][part]) {
                        vregs(pc.reg, pc.len, regs, sizeof(regs));
                        e.line("\tds_write_%s v%d, %s offset:%d", kWidth[pc.len], addr_reg(pc.len, pc.off), regs, pc.off & 65535);
                    }
                e.line("\ts_waitcnt lgkmcnt(0)");
                e.line("\ts_barrier");
                std::vector<Piece> items;   // ascending source wave: the order the partials are added in
                for (int sw = 0; sw < parts; ++sw) items.insert(items.end(), lay[part][sw].begin(), lay[part][sw].end());
                for (size_t b0 = 0; b0 < items.size();) {
                    std::vector<int> at;   // temporary of each piece of the batch
                    int cur = 0;
                    size_t b1 = b0;
                    for (; b1 < items.size() && (int)at.size() < kMaxLgkm; ++b1) {
                        const int len = items[b1].len;
                        const int start = len > 1 ? (cur + 1) / 2 * 2 : cur;
                        if (start + len > n_tmp) break;
                        at.push_back(tmp0 + start);
                        cur = start + len;
                    }
                    for (size_t t = b0; t < b1; ++t) {
                        vregs(at[t - b0], items[t].len, regs, sizeof(regs));
                        e.line("\tds_read_%s %s, v%d offset:%d", kWidth[items[t].len], regs, addr_reg(items[t].len, items[t].off),
                               items[t].off & 65535);
                    }
                    for (size_t t = b0; t < b1; ++t) {
                        e.line("\ts_waitcnt lgkmcnt(%d)", (int)(b1 - 1 - t));
                        for (int j = 0; j < items[t].len; ++j)
                            e.line("\t%s v%d, v%d, v%d", int8 ? "v_add_u32_e32" : "v_add_f32_e32", items[t].reg + j, items[t].reg + j,
                                   at[t - b0] + j);
                    }
                    b0 = b1;
                }
            }
            stores(mine);
            e.line("\ts_endpgm");
            return nc;
        }
        std::vector<std::pair<int32_t, int>> all;
        for (size_t i = 0; i < rows.size(); ++i) all.push_back({rows[i], acc_reg((int)i)});
        stores(all);
        e.line("\ts_endpgm");
        return nc;
    }

    // LDS: wave `w` of W stages quads q == w (mod W) of every chunk; all waves read what
    // they need.  LDS layout per buffer: [quad of 4 consecutive B rows][lane][4 floats].
    int block_lds(const std::vector<int32_t> &rows, int w, int W) {
        auto cols = columns_of(rows);
        const int kChunkRows = chunk_rows;
        const int n_chunks = (K + kChunkRows - 1) / kChunkRows;
        const int quads_per_chunk = kChunkRows / 4;
        const int buf_bytes = kChunkRows * 256;
        int ring_pos = 0;
        zero_accs(rows.size());
        // Staging runs ahead of the compute: chunk c travels through register set c % 2, so a fetch
        // has the time of two chunks to arrive before it is copied into LDS.
        const int quads_per_wave = (quads_per_chunk + W - 1) / W;
        auto stage_rows = [&](int c) {   // (row of B, register) of every fetch of this wave for chunk c
            std::vector<std::pair<int, int>> rows;
            if (c >= n_chunks) return rows;
            int t = 0;
            for (int q = w; q < quads_per_chunk; q += W, ++t)
                for (int j = 0; j < 4; ++j)
                    if (c * kChunkRows + 4 * q + j < K) rows.push_back({c * kChunkRows + 4 * q + j, vgpr_stage0 + (c & 1) * 4 * quads_per_wave + 4 * t + j});
            return rows;
        };
        auto stage_loads = [&](int c) {
            for (auto &r : stage_rows(c)) load_b_row(r.first, r.second, ring_pos++);
        };
        auto stage_write = [&](int c) {
            // fetches return in order: chunk c has arrived once only chunk c+1's are outstanding
            e.line("\ts_waitcnt vmcnt(%d)", (int)stage_rows(c + 1).size());
            int t = 0, n = 0;
            for (int q = w; q < quads_per_chunk; q += W, ++t) {
                if (c * kChunkRows + 4 * q >= K) break;
                const int v = vgpr_stage0 + (c & 1) * 4 * quads_per_wave + 4 * t;
                // half storage: widened once here (exact), so the staged tile and everything after
                // it is the fp32 code; int8 arrives sign-extended by the load itself
                if (half)
                    for (int j = 0; j < 4 && c * kChunkRows + 4 * q + j < K; ++j) e.line("\tv_cvt_f32_f16_e32 v%d, v%d", v + j, v + j);
                e.line("\tds_write_b128 v%d, v[%d:%d] offset:%d", kVgprLds, v, v + 3, (c & 1) * buf_bytes + q * 1024);
                ++n;
            }
            return n;
        };
        // The quads that hold a nonzero column of the group, over all chunks.
        struct Quad { int chunk, q; std::vector<Term> terms[4]; bool need[4] = {false, false, false, false}; int last_read = -1; };
        std::vector<Quad> quads;
        for (auto &col : cols) {
            const int c = col.first / kChunkRows, q = col.first % kChunkRows / 4, j = col.first % 4;
            if (quads.empty() || quads.back().chunk != c || quads.back().q != q) { quads.push_back(Quad()); quads.back().chunk = c; quads.back().q = q; }
            quads.back().need[j] = true;
            quads.back().terms[j] = std::move(col.second);
        }
        const int nq = (int)quads.size();
        int issued = 0;   // LDS instructions
        auto issue_reads = [&](int i) {
            Quad &Q = quads[i];
            const int v0 = vgpr_ring0 + 4 * (i % D), off = (Q.chunk & 1) * buf_bytes + Q.q * 1024;
            const int cnt = Q.need[0] + Q.need[1] + Q.need[2] + Q.need[3];
            if (cnt >= 3) {
                e.line("\tds_read_b128 v[%d:%d], v%d offset:%d", v0, v0 + 3, kVgprLds, off);
                ++issued;
            } else {
                for (int j = 0; j < 4; j += 2) {
                    if (Q.need[j] && Q.need[j + 1]) {
                        e.line("\tds_read_b64 v[%d:%d], v%d offset:%d", v0 + j, v0 + j + 1, kVgprLds, off + 4 * j);
                        ++issued;
                    } else if (Q.need[j] || Q.need[j + 1]) {
                        const int jj = Q.need[j] ? j : j + 1;
                        e.line("\tds_read_b32 v%d, v%d offset:%d", v0 + jj, kVgprLds, off + 4 * jj);
                        ++issued;
                    }
                }
            }
            Q.last_read = issued - 1;
        };
        // The reads run D quads ahead of the multiply-adds, over the ends of chunks as well: what a wave still has in
        // registers of a chunk is multiplied while the first reads of the next one are on their way.  A wave enters a
        // chunk (with its reads, that is) once its reads of the one before have returned and its share of this one is
        // written; behind the barrier every wave has, so the other buffer is free for the share of the chunk after it.
        // That is written a quarter of the way through the chunk, and the fetches that take its place in the registers
        // go out one between two quads: sixteen in a row hold every wave of the workgroup up at the same time.
        // Reads that ended with their chunk, shares written at its end and fetched in a row, against this, in us
        // (fp32, uniform masks): 4096^3 at 98 % 76.0, 72.6; 2048 x 4096 x 12544 at 98 % 149.5, 145.1; 3072 x 3000 x 2900
        // at 96 % 73.6, 72.1; 2048 x 1024 x 4096 at 97 % 19.1, 18.6; 4096 x 1024 x 784, batch 4, at 95 % 43.6, 43.1.
        // Shares written at the start of the chunk or half way: 74.3 and 74.4 for the first of them.
        // What is left there: launch and stores alone 10.5, with the staging 30.6 without any multiply-adds, which are 35
        // at full rate; two waves per SIMD issue some 54 % of that rate.  Code is not it: half as long (values that need
        // no literal) 71.7 -> 68.5.
        int chunk = 0;            // the one that is read
        bool staged_next = false; // this wave's share of the one after it is written
        int fetch_behind = -1;    // LDS instruction behind which that share has left its registers, for the chunk after the next
        std::vector<std::pair<int, int>> to_fetch;   // (row of B, register), of that chunk
        size_t fetched = 0;
        auto fetch = [&](size_t upto) {
            for (; fetched < std::min(upto, to_fetch.size()); ++fetched) load_b_row(to_fetch[fetched].first, to_fetch[fetched].second, ring_pos++);
        };
        auto fetch_open = [&]() {
            if (fetch_behind < 0) return;
            e.line("\ts_waitcnt lgkmcnt(%d)", std::min(kMaxLgkm, issued - 1 - fetch_behind));
            to_fetch = stage_rows(chunk + 3);
            fetched = 0;
            fetch_behind = -1;
        };
        auto stage_next = [&]() {
            if (staged_next || chunk + 1 >= n_chunks) return;
            issued += stage_write(chunk + 1);
            fetch_behind = issued - 1;
            staged_next = true;
        };
        auto enter_next_chunk = [&]() {
            stage_next();
            fetch_open();
            fetch(to_fetch.size());
            e.line("\ts_waitcnt lgkmcnt(0)");
            e.line("\ts_barrier");
            ++chunk;
            staged_next = false;
        };
        stage_loads(0);
        stage_loads(1);
        stage_write(0);
        e.line("\ts_waitcnt lgkmcnt(0)");
        stage_loads(2);
        e.line("\ts_barrier");
        int next = 0;             // quad to be read
        auto read_next = [&]() {
            if (next >= nq) return;
            while (chunk < quads[next].chunk) enter_next_chunk();
            issue_reads(next);
            if (quads[next++].q >= quads_per_chunk / 4) stage_next();
        };
        while (next < std::min(D, nq)) read_next();
        for (int i = 0; i < nq; ++i) {
            // LDS instructions complete in order: quad i has arrived once at most
            // (issued - 1 - last_read) later ones are outstanding
            e.line("\ts_waitcnt lgkmcnt(%d)", std::min(kMaxLgkm, issued - 1 - quads[i].last_read));
            if (fetch_behind >= 0 && fetch_behind < quads[i].last_read) fetch_open();
            fetch(fetched + 1);
            for (int j = 0; j < 4; ++j)
                if (quads[i].need[j]) fmas(quads[i].terms[j], vgpr_ring0 + 4 * (i % D) + j);
            read_next();
        }
        while (chunk + 1 < n_chunks) enter_next_chunk();   // no quads left: the other waves still need this one's share
        const int total_cols = (int)cols.size();
        std::vector<std::pair<int32_t, int>> all;
        for (size_t i = 0; i < rows.size(); ++i) all.push_back({rows[i], kVgprAcc0 + (int)i});
        stores(all);
        e.line("\ts_endpgm");
        return total_cols;
    }
};

}  // namespace

bool spec_available() { return comgr().ok; }

int rows_for_whole_rounds(int32_t M, int groups_per_wg, int64_t wg_columns, int lo, int hi) {
    constexpr int64_t kComputeUnits = 256;
    lo = std::max(1, std::min<int>(lo, M));
    hi = std::max(lo, std::min<int>(hi, M));
    int best = -1;
    int64_t best_cost = INT64_MAX;
    for (int r = lo; r <= hi; ++r) {
        const int64_t groups = ((int64_t)M + r - 1) / r;
        const int64_t wgs = (groups + groups_per_wg - 1) / groups_per_wg * wg_columns;
        if (wgs < kComputeUnits) continue;   // the model holds while every compute unit has a workgroup
        const int64_t cost = (wgs + kComputeUnits - 1) / kComputeUnits * r;
        if (cost < best_cost || (cost == best_cost && r > best)) { best = r; best_cost = cost; }
    }
    return best > 0 ? best : lo;   // too small a launch for any count in range: the most workgroups
}

static int64_t workgroups_for(int32_t M, int r, int groups_per_wg, int64_t wg_columns) {
    const int64_t groups = ((int64_t)M + r - 1) / r;
    return (groups + groups_per_wg - 1) / groups_per_wg * wg_columns;
}

int rows_for_rounds(int32_t M, int groups_per_wg, int64_t wg_columns, int rounds, int hi) {
    constexpr int64_t kComputeUnits = 256;
    for (int r = 1; r <= std::min<int>(hi, M); ++r)
        if (workgroups_for(M, r, groups_per_wg, wg_columns) <= kComputeUnits * rounds) return r;
    return 0;
}

int rows_without_thin_round(int32_t M, int R, int groups_per_wg, int64_t wg_columns, int hi) {
    constexpr int64_t kComputeUnits = 256;
    const int64_t wgs = workgroups_for(M, R, groups_per_wg, wg_columns);
    const int64_t rounds = (wgs + kComputeUnits - 1) / kComputeUnits;
    // (blocks of a few rows make small workgroups, several of which share a compute unit: no rounds there)
    if (R < 8 || rounds < 2 || rounds > 16 || wgs - kComputeUnits * (rounds - 1) > kComputeUnits / 4) return R;
    const int top = std::min<int>(std::min<int>(hi, M), R + (R * 15 + 99) / 100);
    for (int r = R + 1; r <= top; ++r)
        if (workgroups_for(M, r, groups_per_wg, wg_columns) <= kComputeUnits * (rounds - 1))
            return (rounds - 1) * r < rounds * R ? r : R;
    return R;
}

// A launch of 257 to 512 workgroups gives some compute units two and the others one, and takes as long as the
// two.  If the fewest rows per block that make it 256 workgroups are at most 7/4 of R, one larger workgroup each is
// faster: blocks of 64 rows instead of 52 on 104 column tiles (half convolution of 128 x 1152, 28 x 28, batch 8),
// 312 -> 208 workgroups, 11.3 -> 7.9 us; 504 x 1664 x 691, batch 4, fp32: 86 -> 101 rows, 264 -> 220, 37.2 -> 21.0 us.
// Over 52 drawn products and convolutions that it changes: 1.04 to 2.1 times faster, 1.36 on average.  Twice the rows lose
// what the second workgroup hides (2048 x 376 x 67, batch 4, 16 -> 32 rows: 8.4 -> 10.2 us), and so may blocks of
// more than 96 rows without a K split (1096 x 308 x 1600, batch 4, 96 -> 122: 18.8 -> 20.4 us).
static int rows_for_one_round(int32_t M, int R, int64_t wg_columns, int hi) {
    const int64_t wgs = workgroups_for(M, R, 1, wg_columns);
    if (R < 8 || wgs <= 256 || wgs > 512) return R;
    const int r = rows_for_rounds(M, 1, wg_columns, 1, std::min(hi, R * 7 / 4));
    return r > R ? r : R;
}

// What the stages below hand to each other besides the SpecPlan itself.
struct Shape {
    bool lds = false;   // LDS-staged variant
    int max_lanes = kWave, V = 1, nvc = 0, KS = 1, W = 4, wshift = 2;
};

// Stage 1, launch policy: variant, column tiling, columns per lane, rows per block, K split,
// waves per workgroup, fetch depth, number of code blocks.
static int choose_launch_shape(const HostPlan &h, const sparsert_options &opt, SpecPlan &sp, Shape &sh, std::string &err) {
    if (h.conv && opt.spec_mode == SPARSERT_SPEC_LDS) {
        err = "convolution plans use the DIRECT variant of the generated kernel";
        return SPARSERT_EUNSUPPORTED;
    }
    const bool half = h.dtype == SPARSERT_F16, int8 = h.dtype == SPARSERT_I8;
    const int32_t M = h.M, N = h.N;
    sp.mode = opt.spec_mode ? opt.spec_mode : SPARSERT_SPEC_DIRECT;
    // With nothing set, large and very sparse products take the LDS-staged variant with eight waves:
    // every wave fetches a row of B for few multiply-adds there, and staging lets eight blocks share
    // each fetch.  Over the shape sweep it is what the tuner picks from 95 % sparsity on once a
    // compute unit has 512 rows x tiles of C to itself (4096 x 4096 x 4096 at 98 %: 73 us against
    // 156 us for the DIRECT default; 2048 x 2048 x 3136, 392 per compute unit, is better off with
    // DIRECT); below 95 % the multiply-adds dominate and DIRECT is as fast.  M >= 2048 keeps the rule
    // to what was measured: eight waves with blocks of at least 32 rows and several workgroups per tile.
    bool auto_staged = false;
    if (!opt.spec_mode && !opt.spec_rows && !opt.spec_ksplit && !opt.spec_tiles && !opt.spec_lanes && opt.spec_vec <= 1 &&
        h.dtype == SPARSERT_F32 && !h.conv && M >= 2048 && h.K >= 1024 && (int64_t)h.nnz * 18 <= (int64_t)M * h.K &&
        (int64_t)M * ((N + kWave - 1) / kWave) * std::max(1, h.batch) >= 131072) {
        sp.mode = SPARSERT_SPEC_LDS;
        auto_staged = true;
    }
    const bool lds = sp.mode == SPARSERT_SPEC_LDS;
    // Column tiling with one column per lane, balanced tails (same rule as the row-walk plan at V = 1).
    const int max_lanes = opt.spec_lanes ? opt.spec_lanes : kWave;
    if (lds && max_lanes != kWave) { err = "spec_lanes applies to the DIRECT variant"; return SPARSERT_EINVAL; }
    // Columns per lane: 1, or the 2 halves / 4 int8 that share the dword a lane loads (SpMM only).
    const int V = opt.spec_vec ? opt.spec_vec : 1;
    if (!(V == 1 || (V == 2 && half) || (V == 4 && int8))) { err = "spec_vec must be 0/1, 2 for half plans or 4 for int8 plans"; return SPARSERT_EINVAL; }
    if (V > 1 && (h.conv || lds)) { err = "spec_vec > 1 applies to SpMM plans of the DIRECT variant"; return SPARSERT_EINVAL; }
    if (N % V || h.ldb % V || h.ldc % V) { err = "N, ldb and ldc must be multiples of spec_vec"; return SPARSERT_EINVAL; }
    sp.vec = V;
    const int32_t nvc = N / V;   // vector columns
    sp.n_tiles = (nvc + max_lanes - 1) / max_lanes;
    sp.lanes_per_tile = (nvc + sp.n_tiles - 1) / sp.n_tiles;
    sp.tiles_per_wg = opt.spec_tiles ? opt.spec_tiles : auto_staged ? 8 : 4;
    // Rows per block and K split.  Left at 0 they follow what the tuner's winners have in common
    // on this chip: a launch of about two waves per SIMD (2048 waves), with as many rows per
    // block as that allows, because rows per block is what saves fetches of B, and with the
    // reduction axis split over the waves of a workgroup where it is long enough to supply them.
    int R = opt.spec_rows;
    int KS = opt.spec_ksplit;
    if (KS == 0) KS = (!lds && R == 0 && h.K >= 512) ? 8 : 1;
    if (auto_staged) {
        R = rows_for_whole_rounds(M, 8, (int64_t)sp.n_tiles * std::max(1, h.batch), 32, 128);
    } else if (R == 0 && lds) {
        // LDS variant: R1 fills 1024 SIMDs with one wave each, R2 gives a wave about 400 multiply-adds
        const int64_t r1 = (int64_t)M * sp.n_tiles / 1024;
        const int64_t avg = std::max<int64_t>(1, h.nnz / M);
        const int64_t r2 = (400 + avg - 1) / avg;
        R = (int)std::min<int64_t>(96, std::max<int64_t>(4, std::max(r1, r2)));
    } else if (R == 0) {
        const int64_t tiles_all = (int64_t)sp.n_tiles * std::max(1, h.batch);
        const int64_t target = KS > 1 ? 2048 : 1024;
        R = (int)std::max<int64_t>(1, std::min<int64_t>(96 / V, (int64_t)M * tiles_all * KS / target));
        if (opt.spec_ksplit == 0)   // fewer parts where the rows alone already supply the waves
            while (KS > 1 && ((int64_t)M + R - 1) / R * tiles_all * (KS / 2) >= 2048) KS /= 2;
        // 1024 rows in blocks of 52 on 13 column tiles are 260 workgroups, four more than compute
        // units: 34.8 us; in blocks of 54 they are 247: 21.3 us (4096 columns of A at 95 %)
        const int T = opt.spec_tiles ? opt.spec_tiles : 4;
        const int64_t wg_columns = KS > 1 ? tiles_all : (sp.n_tiles + T - 1) / T * std::max(1, h.batch);
        R = rows_for_one_round(M, R, wg_columns, (KS > 1 ? 128 : 96) / V);
        R = rows_without_thin_round(M, R, 1, wg_columns, 128 / V);
    }
    sp.ksplit = KS;
    if (sp.ksplit != 1 && sp.ksplit != 2 && sp.ksplit != 4 && sp.ksplit != 8) { err = "spec_ksplit must be 0,1,2,4,8"; return SPARSERT_EINVAL; }
    if (sp.ksplit > 1 && lds) { err = "spec_ksplit applies to the DIRECT variant"; return SPARSERT_EINVAL; }
    if (sp.ksplit > 1) sp.tiles_per_wg = sp.ksplit;   // the waves of a workgroup are the K parts
    const int W = sp.tiles_per_wg;
    int wshift = 0;
    while ((1 << wshift) < W) ++wshift;
    if (R < 1 || R > 232) { err = "spec_rows must be in 1..232"; return SPARSERT_EINVAL; }
    R = std::min(R, M);
    sp.rows_per_group = R;
    sp.n_groups = (M + R - 1) / R;
    sp.depth = opt.spec_depth ? opt.spec_depth : (lds ? 6 : 16);
    if (lds && sp.depth > 12) sp.depth = 12;
    const int G = sp.n_groups;
    // LDS mode: a workgroup runs W consecutive blocks and every one of them takes part in the
    // staging and the barriers, so the block list is padded with empty blocks.
    sp.n_blocks = lds ? (G + W - 1) / W * W : G * sp.ksplit;
    sh.lds = lds; sh.max_lanes = max_lanes; sh.V = V; sh.nvc = nvc; sh.KS = sp.ksplit; sh.W = W; sh.wshift = wshift;
    return SPARSERT_OK;
}

// Stage 2, block formation: which slots (rows of the permuted CSR) share a code block.
static void form_blocks(const HostPlan &h, const sparsert_options &opt, SpecPlan &sp,
                        std::vector<std::vector<int32_t>> &members) {
    const int32_t M = h.M;
    const int R = sp.rows_per_group, G = sp.n_groups;
    // Block-level balance (Section 3.4, strategy b): slots are in descending-nnz order; deal
    // them to the groups in serpentine order so every group gets nearly the same nonzero count.
    members.assign(sp.n_blocks, {});
    sp.group_of_slot.resize(M);
    sp.swizzle = opt.spec_swizzle && !h.natural_order;
    if (!sp.swizzle) {
        for (int32_t i = 0; i < M; ++i) {
            const int32_t round = i / G, pos = i % G;
            // natural order (ablation): block g is the contiguous row range [g*R, (g+1)*R)
            const int32_t g = h.natural_order ? i / R : ((round & 1) ? G - 1 - pos : pos);
            sp.group_of_slot[i] = g;
            members[g].push_back(i);
        }
    } else {
        // Row swizzle (Section 5, named there as a preprocessing step that would help): rows that share columns go to the
        // same block, so the block fetches fewer rows of B.  The nnz-descending slots are
        // handed out in rounds of G, one row per block and round, which keeps the nonzero
        // counts of the blocks within one row's worth of each other as the serpentine deal
        // does; inside a round each block, in serpentine direction, takes the candidate that
        // shares the most columns with what the block already fetches (ties: lowest slot).
        const int words = (h.K + 63) / 64;
        std::vector<uint64_t> pattern((size_t)M * words, 0), fetched((size_t)G * words, 0);
        for (int32_t i = 0; i < M; ++i)
            for (int32_t p = h.p_row_ptr[i]; p < h.p_row_ptr[i + 1]; ++p)
                pattern[(size_t)i * words + h.p_col_idx[p] / 64] |= 1ull << (h.p_col_idx[p] % 64);
        std::vector<char> taken(M, 0);
        for (int32_t first = 0, round = 0; first < M; first += G, ++round) {
            const int32_t last = std::min<int32_t>(M, first + G);
            for (int32_t step = 0; step < last - first; ++step) {
                const int32_t g = (round & 1) ? G - 1 - step : step;
                int32_t best = -1;
                int64_t best_shared = -1;
                for (int32_t c = first; c < last; ++c) {
                    if (taken[c]) continue;
                    int64_t shared = 0;
                    if (round > 0)
                        for (int w = 0; w < words; ++w)
                            shared += __builtin_popcountll(pattern[(size_t)c * words + w] & fetched[(size_t)g * words + w]);
                    if (shared > best_shared) { best_shared = shared; best = c; }
                    if (round == 0) break;   // seeding: slot first+step goes to block step
                }
                taken[best] = 1;
                sp.group_of_slot[best] = g;
                members[g].push_back(best);
                for (int w = 0; w < words; ++w) fetched[(size_t)g * words + w] |= pattern[(size_t)best * words + w];
            }
        }
    }

}

// Stage 3, register and LDS plan: where accumulators, the operand ring, staging registers and the
// exchange area sit; the descriptor extents; the convolution's pixel-index constant.
struct Extents { int64_t b_bytes = 0, c_bytes = 0; uint32_t magic = 0; };

static int plan_registers(const HostPlan &h, SpecPlan &sp, const Shape &sh, const std::vector<std::vector<int32_t>> &members,
                          Gen &gen, Extents &ex, std::string &err) {
    const bool half = gen.half, int8 = gen.int8, lds = sh.lds;
    const int esz = gen.esz, osz = gen.osz, V = sh.V, KS = sh.KS, W = sh.W, max_lanes = sh.max_lanes;
    const int32_t M = h.M, N = h.N;
    gen.stream_stores = ((int64_t)h.ldc * osz) % 128 == 0 && ((int64_t)sp.lanes_per_tile * V * osz) % 128 == 0;
    // descriptor extents: the last row of a matrix ends after its N columns, whatever the pitch
    ex.b_bytes = h.conv ? ((int64_t)h.Cin * N + 2 * (h.W + 1)) * esz : ((int64_t)(h.K - 1) * h.ldb + N) * esz;
    ex.c_bytes = ((int64_t)(M - 1) * h.ldc + N) * osz;
    // conv: pixel -> (oh, ow) by multiplication with ceil(2^32 / W); verified here for every pixel
    uint32_t &magic = ex.magic;
    if (h.conv && h.W > 1) {
        magic = (uint32_t)(((1ull << 32) + h.W - 1) / h.W);
        for (int64_t p = 0; p < N; ++p)
            if ((int64_t)(((uint64_t)p * magic) >> 32) != p / h.W) {
                err = "image too large for the generated kernel's pixel index arithmetic";
                return SPARSERT_EUNSUPPORTED;
            }
    }
    int max_rows = 0;
    for (auto &m : members) max_rows = std::max<int>(max_rows, (int)m.size());
    const int D = sp.depth;
    if (lds) {
        gen.staged = true;
        gen.chunk_rows = std::min(kMaxChunkRows, 32 * W);
        const int kChunkRows = gen.chunk_rows;
        const int quads_per_wave = (kChunkRows / 4 + W - 1) / W;
        gen.vgpr_stage0 = (kVgprAcc0 + max_rows + 3) / 4 * 4;
        gen.vgpr_ring0 = gen.vgpr_stage0 + 2 * 4 * quads_per_wave;
        gen.n_vgpr = gen.vgpr_ring0 + 4 * D;
        const int n_chunks = (h.K + kChunkRows - 1) / kChunkRows;
        gen.lds_bytes = (n_chunks > 1 ? 2 : 1) * kChunkRows * 256;
    } else {
        gen.V = V;
        gen.vgpr_ring0 = kVgprAcc0 + max_rows * V;
        gen.ring_size = KS > 1 ? std::max(D, 20) : D;   // the K-split exchange borrows the ring: address registers and temporaries
        gen.vgpr_unpack0 = gen.vgpr_ring0 + gen.ring_size;
        gen.n_vgpr = gen.vgpr_unpack0 + (int8 && V == 4 ? 4 : half && V == 2 ? 1 : 0);
        if (KS > 1) {
            gen.slot_bytes = V * ((4 * max_lanes + 15) / 16 * 16);   // a row's partial sums: V registers over the lanes of a tile, 16-byte granules
            gen.xchg_rows = std::min(max_rows, kMaxLdsBytes / ((KS - 1) * gen.slot_bytes));
            gen.lds_bytes = (KS - 1) * gen.xchg_rows * gen.slot_bytes;
            if (gen.lds_bytes == 0) gen.lds_bytes = 256;
        }
    }
    if (gen.n_vgpr > 256) { err = "spec_rows too large for the register file"; return SPARSERT_EINVAL; }
    // A workgroup must fit a compute unit at once: its waves are spread over the four SIMDs, and a
    // SIMD has 512 registers per lane, handed out in granules of eight.  (A dispatch that does not
    // fit is rejected by the hardware queue, which aborts the process.)
    if ((W + 3) / 4 * ((gen.n_vgpr + 7) / 8 * 8) > 512) {
        err = "spec_rows too large for this many waves per workgroup: the workgroup's registers do not fit a compute unit";
        return SPARSERT_EINVAL;
    }
    // The symbol carries the problem shape so that kernel traces tell the plans of a model apart.
    char sym[96];
    snprintf(sym, sizeof(sym), "sparsert_spec_%s%dx%dx%d%s", h.conv ? "conv_" : "", (int)M, (int)h.K, (int)N,
             half ? (V == 2 ? "_f16x2" : "_f16") : int8 ? (V == 4 ? "_i8x4" : "_i8") : "");
    sp.symbol = sym;
    sp.lds_bytes = gen.lds_bytes;

    return SPARSERT_OK;
}

// Which workgroups share an L2.  Workgroup i of a launch runs on XCD i mod 8, and every XCD has an L2 of its own, which
// pulls the code blocks and the column tiles of B that its workgroups touch.  In launch order (column tile, then code
// block, then problem of the batch) that is an eighth of the tiles and all of the code if the tile count is a multiple of
// 8, and everything otherwise: 1024 x 1024 at 90 % fetched 23 MB on 13 column tiles and 11 MB on 16, and took 11.4 and
// 6.7 us.  So the prologue deals the workgroups anew: they stand in a row - part of the code blocks, column tile, block -
// and every XCD takes an eighth of that row.
struct Deal {
    int64_t tiles = 0, blocks = 0, batch = 1;   // of the launch, in workgroups
    int parts = 0, per_part = 0;                // 0: launch order
    int64_t workgroups() const { return tiles * blocks * batch; }
    // The workgroup in place `at` of the row: column tile (counted over the batch) and code block.
    void work(int64_t at, int64_t &tile, int64_t &block) const {
        const int64_t part = at / (tiles * batch * per_part), in = at - part * tiles * batch * per_part;
        const int64_t here = std::min<int64_t>(per_part, blocks - part * per_part);
        tile = in / here;
        block = part * per_part + in % here;
    }
};

// What a deal costs: the bytes that all L2s together pull, a tile (of one problem) and a code block counted once for every
// XCD that touches them, and the most code that one XCD and one compute unit run: an XCD has 32, its workgroups come to them in turn.
// A byte of code weighs three times: its misses come one after the other, B's overlap.  (Over 75 products and convolutions,
// each timed in launch order and in 1, 2, 4 and 8 parts, a factor of 3 to 5 chose best, 1 or 8 half a percent worse.)
struct DealCost { double bytes = 0, weighed = 0, busiest_xcd = 0, busiest_unit = 0; };
constexpr double kCodeByte = 3;

static DealCost deal_cost(const Deal &d, double tile_bytes, const std::vector<int64_t> &block_bytes) {
    const int64_t all = d.workgroups(), share = all / 8, more = all % 8, tiles = d.tiles * d.batch;
    std::vector<uint8_t> has_tile(8 * (size_t)tiles, 0), has_block(8 * (size_t)d.blocks, 0);
    double run[8] = {0}, unit[8 * 32] = {0};
    for (int64_t i = 0; i < all; ++i) {
        const int64_t x = i & 7;
        int64_t tile, block;
        if (d.parts) {
            d.work(x * share + std::min(x, more) + (i >> 3), tile, block);
        } else {
            tile = i / (d.tiles * d.blocks) * d.tiles + i % d.tiles;
            block = i / d.tiles % d.blocks;
        }
        has_tile[(size_t)(x * tiles + tile)] = has_block[(size_t)(x * d.blocks + block)] = 1;
        run[x] += (double)block_bytes[(size_t)block];
        unit[x * 32 + (i >> 3) % 32] += (double)block_bytes[(size_t)block];
    }
    DealCost c;
    for (uint8_t v : has_tile) c.bytes += v * tile_bytes;
    c.weighed = c.bytes;
    for (size_t i = 0; i < has_block.size(); ++i) {
        const double code = has_block[i] * (double)block_bytes[i % (size_t)d.blocks];
        c.bytes += code;
        c.weighed += kCodeByte * code;
    }
    c.busiest_xcd = *std::max_element(run, run + 8);
    c.busiest_unit = *std::max_element(unit, unit + 8 * 32);
    return c;
}

// The row that costs least and does not push an XCD's share towards the size of its L2 (4 MiB; 768 x 3072, 1024 columns, 95 %: 3.2 MB
// in launch order, 4.0 MB in two parts, 13.5 and 13.6 us).  Launch order stays where the best row saves less than a tenth; where the code,
// which every column tile of a part runs again, would not stay in an L2; where an XCD would get a tenth more code, or a compute unit any
// more and the L2s do not pull 5000 bytes less for each byte of that; and where blocks are so unequal (rows of very different lengths,
// few to a block) that the long ones, which come first in launch order, should start first and on different XCDs: half convolution of 64 x 1152, 18 x 18, skewed
// rows, one to a block: 4.9 us in launch order, 7.7 us in parts.
// The compute unit: with 33 to 64 workgroups to an XCD some run two, in launch order a long block and a short one, in parts whatever comes
// together: int8 convolution 47 x 891, 46 x 46, skewed rows, 34 to an XCD: 1.54 times the code, 3.6 and 4.7 us; half 64 x 576, 41 x 41:
// 1.2 to 1.3 times, 3.4 and 3.9 us; half 64 x 1152, 43 x 43, blocks of six and seven rows: 1.04 times, 7.7 MB less for 2 KB more, 7.5 and
// 7.7 us; but 80 x 4320, 23 x 23, batch 2: 1.04 times, 24 MB less for 3.5 KB more, 14.8 and 13.6 us.  (A compute unit runs some 7 KB in a
// microsecond; 4000 and 7000 choose as well.)
// Over 292 drawn products and convolutions (56 with skewed rows, several plans taking turns) the choice is 1.062 times faster than launch order,
// the best of the five 1.075; 6 % slower at worst where C is large (1216 x 512 x 2880 and 1856 x 120 x 3416, batch 4: 33.6 and 35.6, 29.7 and
// 31.6 us, the second 24.6 and 21.8 us while C stays in the cache behind the L2s), 3 % and less otherwise.
static Deal choose_deal(const HostPlan &h, const SpecPlan &sp, const std::vector<int64_t> &code_block_bytes) {
    Deal d;
    const bool lds = sp.mode == SPARSERT_SPEC_LDS;
    d.tiles = lds || sp.ksplit > 1 ? sp.n_tiles : (sp.n_tiles + sp.tiles_per_wg - 1) / sp.tiles_per_wg;
    d.blocks = lds ? sp.n_blocks / sp.tiles_per_wg : sp.n_groups;
    d.batch = h.batch;
    std::vector<int64_t> block_bytes((size_t)d.blocks, 0);   // the code of a workgroup
    int64_t code_bytes = 0;
    for (size_t i = 0; i < code_block_bytes.size(); ++i) {
        block_bytes[i * (size_t)d.blocks / code_block_bytes.size()] += code_block_bytes[i];
        code_bytes += code_block_bytes[i];
    }
    if (d.workgroups() > (1 << 20) || code_bytes > (3 << 20)) return d;
    if (*std::max_element(block_bytes.begin(), block_bytes.end()) * d.blocks > 2 * code_bytes) return d;
    const int64_t columns = (h.N + d.tiles - 1) / d.tiles;   // of a workgroup
    const double tile_bytes = (h.conv ? (double)h.Cin * (columns + 2 * (h.W + 1)) : (double)h.K * columns) * h.elem_size();
    Deal best = d;
    const DealCost now = deal_cost(d, tile_bytes, block_bytes);
    double least = 0.9 * now.weighed;
    for (d.parts = 1; d.parts <= 8; d.parts *= 2) {
        d.per_part = (int)((d.blocks + d.parts - 1) / d.parts);
        if (d.per_part * (d.parts - 1) >= d.blocks) continue;                                                   // a part without blocks
        if (d.workgroups() * std::max<int64_t>(d.tiles * d.batch * d.per_part, d.tiles) >= (1ll << 32)) continue;   // (the prologue's divisions)
        const DealCost c = deal_cost(d, tile_bytes, block_bytes);
        if (c.bytes > now.bytes && c.bytes > 8 * 3.5e6) continue;
        const double more = c.busiest_unit - 1.01 * now.busiest_unit;   // (1 %: equal blocks differ by as much)
        if (more > 0 && now.bytes - c.bytes < 5000 * more) continue;
        if (c.weighed < least && c.busiest_xcd < 1.1 * now.busiest_xcd) { least = c.weighed; best = d; }
    }
    return best;
}

// s[q] = s[x] / divisor by multiplication with ceil(2^32 / divisor): exact while x * divisor < 2^32.
static void emit_quotient(Emitter &e, int q, int x, int64_t divisor) {
    if (divisor > 1) e.line("\ts_mul_hi_u32 s%d, s%d, 0x%x", q, x, (unsigned)(((1ull << 32) + divisor - 1) / divisor));
    else e.line("\ts_mov_b32 s%d, s%d", q, x);
}

// Workgroup id (s2, s3, s[kSgprImage]) -> the column tile, code block and problem that Deal::work gives this workgroup.
static void emit_deal(Emitter &e, const Deal &d) {
    const int at = kSgprOffRing, tmp = kSgprOffRing + 1, part = kSgprOffRing + 2, here = kSgprOffRing + 3;
    const int64_t share = d.workgroups() / 8, more = d.workgroups() % 8, part_size = d.tiles * d.batch * d.per_part;
    const int last = (int)(d.blocks - (int64_t)d.per_part * (d.parts - 1));   // blocks of the last part
    if (d.batch > 1) {
        e.line("\ts_mul_i32 s%d, s%d, 0x%x", tmp, kSgprImage, (unsigned)d.blocks);
        e.line("\ts_add_u32 s3, s3, s%d", tmp);
    }
    e.line("\ts_mul_i32 s%d, s3, 0x%x", at, (unsigned)d.tiles);
    e.line("\ts_add_u32 s%d, s%d, s2", at, at);                       // i
    e.line("\ts_and_b32 s%d, s%d, 7", tmp, at);                       // XCD
    e.line("\ts_lshr_b32 s%d, s%d, 3", at, at);
    e.line("\ts_mul_i32 s%d, s%d, 0x%x", part, tmp, (unsigned)share);
    e.line("\ts_min_u32 s%d, s%d, %d", tmp, tmp, (int)more);
    e.line("\ts_add_u32 s%d, s%d, s%d", at, at, part);
    e.line("\ts_add_u32 s%d, s%d, s%d", at, at, tmp);                 // place in the row
    if (d.parts > 1) {
        emit_quotient(e, part, at, part_size);
        e.line("\ts_mul_i32 s%d, s%d, 0x%x", tmp, part, (unsigned)part_size);
        e.line("\ts_sub_u32 s%d, s%d, s%d", at, at, tmp);
    }
    emit_quotient(e, 2, at, d.per_part);
    e.line("\ts_mul_i32 s%d, s2, 0x%x", tmp, (unsigned)d.per_part);
    if (d.parts > 1 && last != d.per_part) {
        e.line("\ts_cmp_eq_u32 s%d, %d", part, d.parts - 1);
        emit_quotient(e, here, at, last);
        e.line("\ts_cselect_b32 s2, s%d, s2", here);
        e.line("\ts_mul_i32 s%d, s2, 0x%x", here, (unsigned)last);
        e.line("\ts_cselect_b32 s%d, s%d, s%d", tmp, here, tmp);
    }
    e.line("\ts_sub_u32 s3, s%d, s%d", at, tmp);
    if (d.parts > 1) {
        e.line("\ts_mul_i32 s%d, s%d, 0x%x", part, part, (unsigned)d.per_part);
        e.line("\ts_add_u32 s3, s3, s%d", part);
    }
    if (d.batch > 1) {
        emit_quotient(e, kSgprImage, 2, d.tiles);
        e.line("\ts_mul_i32 s%d, s%d, 0x%x", tmp, kSgprImage, (unsigned)d.tiles);
        e.line("\ts_sub_u32 s2, s2, s%d", tmp);
    }
}

// Bytes between code blocks.  The waves of a launch run through their blocks side by side, and blocks that lie a
// multiple of 8 KiB apart are then all at once on the same few channels of the memory behind the L2s: 1024 x 1024 at 90 %
// on 832 columns has 8131 bytes from one block to the next and took 12.7 us; 8.8 us with any distance from 8.7 to 15.5 KB,
// 12.1 us again at 16.4 KB.  Such blocks are moved to 2 KiB behind the multiple.  How near counts: of 260 drawn products and
// convolutions, each with its blocks moved and not, several plans taking turns, those 256 bytes before to 640 behind a multiple are
// 1.05 times faster moved, 1024 before to 1280 behind one of 16 KiB 1.07 times; further off, up to 2 KiB, 0.997 times (0.97 at worst:
// 6591 bytes apart 9.35 us, moved 9.63), and with 128 KiB of code and less, much of which the instruction caches hold, 0.99 times
// (8 blocks of 7658 bytes 9.07 us, moved 9.34).
static int gap_between_blocks(int64_t code_bytes, int64_t blocks) {
    constexpr int64_t kPeriod = 8192, kBehind = 2048;
    const int64_t distance = code_bytes / std::max<int64_t>(1, blocks), multiple = (distance + kPeriod / 2) / kPeriod, off = distance - multiple * kPeriod;
    const bool wide = multiple % 2 == 0;
    if (multiple == 0 || code_bytes <= 128 << 10 || off < (wide ? -1024 : -256) || off >= (wide ? 1280 : 640)) return 0;
    return (int)(kBehind - off + 3) / 4 * 4;
}

// Does a plan with nothing set touch its code ahead (emit_prologue)?  It pays where the plans that run in between have displaced the
// code from the L2s and a block is long: 1021 x 1027 x 771, skewed, at 90 %, four plans taking turns, 8.83 us without and 7.86 with;
// 3072 x 768 x 1024 at 95 % 9.99 and 9.72; 2314 x 520 x 688 at 86 % 10.8 and 9.0.  It costs where one plan runs alone and the
// code is still there: 6.75 us without and 7.14 with, 8.81 and 9.19, 8.10 and 8.55 (spec_prefetch = -1 leaves it out).  75 products that the
// rule takes and that did not set it, three plans each taking turns: 0.927 times the time on average, five slower by more than 1 % (3520 x 658 x
// 2344 at 91 % 1.039); one plan alone 1.021 and 1.086 at most.  What each limit leaves out (the limits set on 192 others):
// - blocks of 21 to 50 rows: 0.93 over 11, but three of them slower, 1.041 at most; code of 500 to 720 kB: 0.95 over nine, two slower, 1.078
//   at most; both: 1.00 over nine, five slower.
// - convolutions: fp32 0.96 over 25, but eight slower, 1.070 at most, and 1.09 alone; half 0.98 over 12, six slower, 1.093 at most; int8 1.06 over
//   12, eleven slower.
// - half and int8 in fewer than four parts: 1.02 over seven, four slower (2173 x 560 x 3968, half, 20.9 us without and 23.2 with).
// - a batch shares the code among its images but each image's waves touch it again (3229 x 256 x 1987, batch 4, 44.6 and 48.1); a wave
//   with many rows of B to fetch has its loads queue behind the touches (744 x 4076 x 3587 48.6 and 52.0); few nonzeros to a row
//   of B leave the time in the fetches (1664 x 2112 x 1405 at 97.6 % 21.0 and 21.9).
static bool prefetch_pays(const HostPlan &h, const sparsert_options &opt, const SpecPlan &sp, int64_t code_bytes) {
    if (sp.mode != SPARSERT_SPEC_DIRECT || opt.spec_mode || opt.spec_rows || opt.spec_ksplit || opt.spec_tiles || opt.spec_lanes || opt.spec_depth ||
        opt.spec_vec || opt.spec_swizzle || opt.natural_order)
        return false;
    if (h.conv || (h.dtype != SPARSERT_F32 && sp.ksplit < 4)) return false;
    return h.batch == 1 && sp.rows_per_group > 50 && code_bytes > 720000 && h.K <= 350 * sp.ksplit && (int64_t)h.nnz * sp.rows_per_group >= 3ll * h.M * h.K;
}

// Stage 4a, emission of everything before the blocks: directives, the prologue that turns the
// workgroup and lane ids into a block, a column and two buffer descriptors, and the jump table.
static void emit_prologue(Gen &gen, Emitter &e, const Shape &sh, const Extents &ex, const Deal &deal, int prefetch_lines, int gap) {
    const HostPlan &h = gen.h;
    SpecPlan &sp = gen.sp;
    const bool lds = sh.lds;
    const int esz = gen.esz, osz = gen.osz, V = sh.V, KS = sh.KS, wshift = sh.wshift, nvc = sh.nvc, n_blocks = sp.n_blocks;
    const int32_t M = h.M, N = h.N;
    const int64_t b_bytes = ex.b_bytes, c_bytes = ex.c_bytes;
    const uint32_t magic = ex.magic;
    e.line("\t.amdgcn_target \"amdgcn-amd-amdhsa--gfx950\"");
    e.line("\t.amdhsa_code_object_version 6");
    e.line("\t.text");
    const char *sym = sp.symbol.c_str();
    e.line("\t.protected\t%s", sym);
    e.line("\t.globl\t%s", sym);
    e.line("\t.p2align\t8");
    e.line("\t.type\t%s,@function", sym);
    e.line("%s:", sym);
    // s[0:1] kernarg, s2 = workgroup id x, s3 = workgroup id y, (s4 = workgroup id z), v0 = thread id
    const bool images = h.batch > 1;
    if (images) e.line("\ts_mov_b32 s%d, s4", kSgprImage);   // s4 is about to receive a kernel argument
    e.line("\ts_load_dwordx4 s[%d:%d], s[0:1], 0x0", kSgprB, kSgprC + 1);
    if (deal.parts) emit_deal(e, deal);
    e.line("\tv_lshrrev_b32_e32 v%d, 6, v0", kVgprT1);
    e.line("\tv_and_b32_e32 v%d, 63, v0", kVgprOff);
    e.line("\ts_nop 1");
    e.line("\tv_readfirstlane_b32 s%d, v%d", kSgprTile, kVgprT1);  // wave index inside the workgroup
    e.line("\ts_nop 4");
    if (!lds && KS > 1) {
        // grid (tiles, groups): the waves of a workgroup run the K parts of one group on one tile
        e.line("\ts_lshl_b32 s%d, s3, %d", kSgprTmp, wshift);
        e.line("\ts_add_u32 s%d, s%d, s%d", kSgprBlock, kSgprTmp, kSgprTile);
        e.line("\ts_mov_b32 s%d, s2", kSgprTile);
        e.line("\tv_lshlrev_b32_e32 v%d, 2, v%d", kVgprLds, kVgprOff);  // lane * 4
    } else if (!lds) {
        // grid (ceil(tiles/W), groups): the waves of a workgroup run one block on adjacent tiles
        e.line("\ts_lshl_b32 s%d, s2, %d", kSgprTmp, wshift);
        e.line("\ts_add_u32 s%d, s%d, s%d", kSgprTile, kSgprTmp, kSgprTile);
        e.line("\ts_mov_b32 s%d, s3", kSgprBlock);
        e.line("\ts_cmp_ge_u32 s%d, %d", kSgprTile, sp.n_tiles);
        e.line("\ts_cbranch_scc1 .Lend");
    } else {
        // grid (tiles, blocks/W): the waves of a workgroup run adjacent blocks on one tile;
        // the block list is padded, so every wave of every workgroup has a block
        e.line("\ts_lshl_b32 s%d, s3, %d", kSgprTmp, wshift);
        e.line("\ts_add_u32 s%d, s%d, s%d", kSgprBlock, kSgprTmp, kSgprTile);
        e.line("\ts_mov_b32 s%d, s2", kSgprTile);
        e.line("\tv_lshlrev_b32_e32 v%d, 4, v%d", kVgprLds, kVgprOff);  // lane * 16
    }
    // offset of this block's code, from a table kept in the text section: fetched now, needed
    // at the end of the prologue, so its latency overlaps the kernel arguments' and the lane set-up
    e.line("\ts_getpc_b64 s[%d:%d]", kSgprPc, kSgprPc + 1);
    e.line(".Lpc:");
    e.line("\ts_add_u32 s%d, s%d, .Ltable-.Lpc", kSgprPc, kSgprPc);
    e.line("\ts_addc_u32 s%d, s%d, 0", kSgprPc + 1, kSgprPc + 1);
    e.line("\ts_lshl_b32 s%d, s%d, 2", kSgprJump, kSgprBlock);
    // this block's entry and the next one's: where the code starts and how long it is
    e.line("\ts_load_dwordx2 s[%d:%d], s[%d:%d], s%d", kSgprEntry, kSgprEntry + 1, kSgprPc, kSgprPc + 1, kSgprJump);
    e.line("\ts_mul_i32 s%d, s%d, %d", kSgprTmp, kSgprTile, sp.lanes_per_tile);  // first column of the tile
    e.line("\tv_add_u32_e32 v%d, s%d, v%d", kVgprT1, kSgprTmp, kVgprOff);        // this lane's column
    e.line("\ts_mov_b32 s%d, %d", kSgprTmp2, nvc);
    e.line("\tv_cmp_gt_u32_e32 vcc, %d, v%d", sp.lanes_per_tile, kVgprOff);     // lane < lanes_per_tile
    e.line("\tv_cmp_gt_u32_e64 s[%d:%d], s%d, v%d", kSgprOwns, kSgprOwns + 1, kSgprTmp2, kVgprT1);  // column < N
    e.line("\ts_nop 4");
    e.line("\ts_and_b64 s[%d:%d], s[%d:%d], vcc", kSgprOwns, kSgprOwns + 1, kSgprOwns, kSgprOwns + 1);
    e.line("\tv_mov_b32_e32 v%d, s%d", kVgprT2, kSgprTmp);
    e.line("\ts_nop 4");
    // lanes without a column redo the tile's first column: loads stay in bounds, nothing is stored
    e.line("\tv_cndmask_b32_e64 v%d, v%d, v%d, s[%d:%d]", kVgprT1, kVgprT2, kVgprT1, kSgprOwns, kSgprOwns + 1);
    auto log2i = [](int x) { int l = 0; while ((1 << l) < x) ++l; return l; };
    e.line("\tv_lshlrev_b32_e32 v%d, %d, v%d", kVgprOut, log2i(V * osz), kVgprT1);   // byte offset of the lane's column(s) in a row of C
    e.line("\tv_lshlrev_b32_e32 v%d, %d, v%d", kVgprOff, log2i(V * esz), kVgprT1);   // ... and in a row of B / X
    // from here on only lanes that own a column are active: idle lanes fetch nothing
    e.line("\ts_mov_b64 exec, s[%d:%d]", kSgprOwns, kSgprOwns + 1);
    if (h.conv) {
        // oh = pixel / W, ow = pixel % W; then one lane mask per filter tap (r, s):
        // 0 <= oh + r - 1 < H and 0 <= ow + s - 1 < W  (Section 3.6: the padding test, made once)
        const int voh = kVgprAcc0, vow = kVgprAcc0 + 1;   // accumulators are not live yet
        const int sa0 = kSgprOffRing, sa2 = kSgprOffRing + 2, sb0 = kSgprOffRing + 4, sb2 = kSgprOffRing + 6;
        if (h.W > 1) {
            e.line("\ts_mov_b32 s%d, 0x%x", kSgprTmp, magic);
            e.line("\tv_mul_hi_u32 v%d, v%d, s%d", voh, kVgprT1, kSgprTmp);
            e.line("\ts_mov_b32 s%d, %d", kSgprTmp, h.W);
            e.line("\tv_mul_lo_u32 v%d, v%d, s%d", vow, voh, kSgprTmp);
            e.line("\tv_sub_u32_e32 v%d, v%d, v%d", vow, kVgprT1, vow);
        } else {  // one pixel per image row
            e.line("\tv_mov_b32_e32 v%d, v%d", voh, kVgprT1);
            e.line("\tv_mov_b32_e32 v%d, 0", vow);
        }
        e.line("\ts_nop 1");
        e.line("\ts_mov_b32 s%d, %d", kSgprTmp, h.H - 2);
        e.line("\ts_mov_b32 s%d, %d", kSgprTmp2, h.W - 2);
        e.line("\tv_cmp_le_i32_e64 s[%d:%d], 1, v%d", sa0, sa0 + 1, voh);             // r = 0 needs oh >= 1
        e.line("\tv_cmp_ge_i32_e64 s[%d:%d], s%d, v%d", sa2, sa2 + 1, kSgprTmp, voh);  // r = 2 needs oh <= H-2
        e.line("\tv_cmp_le_i32_e64 s[%d:%d], 1, v%d", sb0, sb0 + 1, vow);             // s = 0 needs ow >= 1
        e.line("\tv_cmp_ge_i32_e64 s[%d:%d], s%d, v%d", sb2, sb2 + 1, kSgprTmp2, vow); // s = 2 needs ow <= W-2
        e.line("\ts_nop 4");
        e.line("\ts_mov_b64 s[%d:%d], exec", kSgprFull, kSgprFull + 1);
        for (int r = 0; r < 3; ++r)
            for (int t = 0; t < 3; ++t) {
                const int m = kSgprTap0 + 2 * (r * 3 + t);
                e.line("\ts_mov_b64 s[%d:%d], exec", m, m + 1);
                if (r != 1) e.line("\ts_and_b64 s[%d:%d], s[%d:%d], s[%d:%d]", m, m + 1, m, m + 1, r == 0 ? sa0 : sa2, (r == 0 ? sa0 : sa2) + 1);
                if (t != 1) e.line("\ts_and_b64 s[%d:%d], s[%d:%d], s[%d:%d]", m, m + 1, m, m + 1, t == 0 ? sb0 : sb2, (t == 0 ? sb0 : sb2) + 1);
            }
    }
    e.line("\ts_waitcnt lgkmcnt(0)");
    if (h.conv) {
        // operand descriptor starts W+1 elements before X so that every tap displacement is
        // non-negative; lanes that would read before X are always masked off for that tap
        e.line("\ts_sub_u32 s%d, s%d, %d", kSgprB, kSgprB, (h.W + 1) * esz);
        e.line("\ts_subb_u32 s%d, s%d, 0", kSgprB + 1, kSgprB + 1);
    }
    if (images) {
        // problem z of the batch: the operand and the result advance by one image / matrix each
        const int64_t strides[2] = {(h.conv ? (int64_t)h.Cin * N : (int64_t)h.K * h.ldb) * esz, (int64_t)M * h.ldc * osz};
        const int bases[2] = {kSgprB, kSgprC};
        for (int i = 0; i < 2; ++i) {
            e.line("\ts_mov_b32 s%d, 0x%llx", kSgprTmp2, (unsigned long long)strides[i]);
            e.line("\ts_mul_hi_u32 s%d, s%d, s%d", kSgprTmp, kSgprImage, kSgprTmp2);
            e.line("\ts_mul_i32 s%d, s%d, s%d", kSgprTmp2, kSgprImage, kSgprTmp2);
            e.line("\ts_add_u32 s%d, s%d, s%d", bases[i], bases[i], kSgprTmp2);
            e.line("\ts_addc_u32 s%d, s%d, s%d", bases[i] + 1, bases[i] + 1, kSgprTmp);
        }
    }
    e.line("\ts_mov_b32 s%d, s%d", kRsrcB, kSgprB);
    e.line("\ts_and_b32 s%d, s%d, 0xffff", kRsrcB + 1, kSgprB + 1);
    e.line("\ts_mov_b32 s%d, 0x%llx", kRsrcB + 2, (unsigned long long)b_bytes);
    e.line("\ts_mov_b32 s%d, 0x%x", kRsrcB + 3, kRsrcWord3);
    e.line("\ts_mov_b32 s%d, s%d", kRsrcC, kSgprC);
    e.line("\ts_and_b32 s%d, s%d, 0xffff", kRsrcC + 1, kSgprC + 1);
    e.line("\ts_mov_b32 s%d, 0x%llx", kRsrcC + 2, (unsigned long long)c_bytes);
    e.line("\ts_mov_b32 s%d, 0x%x", kRsrcC + 3, kRsrcWord3);
    // jump to the code of this block (the table entry arrived with the kernel arguments)
    e.line("\ts_add_u32 s%d, s%d, s%d", kSgprPc, kSgprPc, kSgprEntry);
    e.line("\ts_addc_u32 s%d, s%d, 0", kSgprPc + 1, kSgprPc + 1);
    if (prefetch_lines > 0) {
        // The block's code is straight-line and read once, so inside a model, where other layers
        // have displaced it from the L2 cache, the wave would take one L2 miss after the other
        // while it runs.  Instead every lane touches `prefetch_lines` 128-byte lines of the block
        // right now, with ordinary loads whose result is never used (lanes past the end of the
        // block are masked off, so nothing outside this block's code is read): the misses overlap
        // each other and the first fetches of B.  The destination register is one no block uses.
        const int stride = 128 * prefetch_lines;
        e.line("\ts_sub_u32 s%d, s%d, s%d", kSgprEntry + 1, kSgprEntry + 1, kSgprEntry);   // from this block to the next
        if (gap) e.line("\ts_sub_u32 s%d, s%d, 0x%x", kSgprEntry + 1, kSgprEntry + 1, (unsigned)gap);   // bytes of code in this block
        e.line("\ts_mov_b64 exec, -1");
        e.line("\tv_mbcnt_lo_u32_b32 v%d, -1, 0", kVgprAcc0);
        e.line("\tv_mbcnt_hi_u32_b32 v%d, -1, v%d", kVgprAcc0, kVgprAcc0);              // lane id
        e.line("\tv_mul_u32_u24_e32 v%d, 0x%x, v%d", kVgprAcc0, stride, kVgprAcc0);    // first byte this lane touches
        for (int j = 0; j < prefetch_lines; ++j) {
            // lanes whose line starts inside the block stay active (the set only shrinks with j)
            e.line("\tv_cmpx_gt_i32_e32 vcc, s%d, v%d", kSgprEntry + 1, kVgprAcc0);
            e.line("\tglobal_load_dword v%d, v%d, s[%d:%d] offset:%d", kVgprT1, kVgprAcc0, kSgprPc, kSgprPc + 1, 128 * j);
            if (j + 1 < prefetch_lines) e.line("\ts_sub_u32 s%d, s%d, 128", kSgprEntry + 1, kSgprEntry + 1);
        }
        e.line("\ts_mov_b64 exec, s[%d:%d]", kSgprOwns, kSgprOwns + 1);
    }
    e.line("\ts_setpc_b64 s[%d:%d]", kSgprPc, kSgprPc + 1);
    e.line(".Lend:");
    e.line("\ts_endpgm");
    e.line("\t.p2align 2");
    e.line(".Ltable:");
    for (int g = 0; g < n_blocks; ++g) e.line("\t.long .Lg%d-.Ltable", g);
    e.line("\t.long .Lfunc_end-.Ltable+%d", gap);   // where a block behind the last one would be

}

// Stage 4b, emission of what follows the blocks: the kernel descriptor and the code object metadata.
static void emit_kernel_descriptor(Gen &gen, const Shape &sh) {
    const HostPlan &h = gen.h;
    SpecPlan &sp = gen.sp;
    Emitter &e = gen.e;
    const char *sym = sp.symbol.c_str();
    const bool images = h.batch > 1;
    const int n_vgpr = gen.n_vgpr, W = sh.W;
    e.line(".Lfunc_end:");
    e.line("\t.size\t%s, .Lfunc_end-%s", sym, sym);
    e.line("\t.section\t.rodata,\"a\",@progbits");
    e.line("\t.p2align\t6, 0x0");
    e.line("\t.amdhsa_kernel %s", sym);
    e.line("\t\t.amdhsa_group_segment_fixed_size %d", gen.lds_bytes);
    e.line("\t\t.amdhsa_private_segment_fixed_size 0");
    e.line("\t\t.amdhsa_kernarg_size 16");
    e.line("\t\t.amdhsa_user_sgpr_count 2");
    e.line("\t\t.amdhsa_user_sgpr_dispatch_ptr 0");
    e.line("\t\t.amdhsa_user_sgpr_queue_ptr 0");
    e.line("\t\t.amdhsa_user_sgpr_kernarg_segment_ptr 1");
    e.line("\t\t.amdhsa_user_sgpr_dispatch_id 0");
    e.line("\t\t.amdhsa_user_sgpr_kernarg_preload_length 0");
    e.line("\t\t.amdhsa_user_sgpr_kernarg_preload_offset 0");
    e.line("\t\t.amdhsa_user_sgpr_private_segment_size 0");
    e.line("\t\t.amdhsa_uses_dynamic_stack 0");
    e.line("\t\t.amdhsa_enable_private_segment 0");
    e.line("\t\t.amdhsa_system_sgpr_workgroup_id_x 1");
    e.line("\t\t.amdhsa_system_sgpr_workgroup_id_y 1");
    e.line("\t\t.amdhsa_system_sgpr_workgroup_id_z %d", images ? 1 : 0);
    e.line("\t\t.amdhsa_system_sgpr_workgroup_info 0");
    e.line("\t\t.amdhsa_system_vgpr_workitem_id 0");
    e.line("\t\t.amdhsa_next_free_vgpr %d", n_vgpr);
    e.line("\t\t.amdhsa_next_free_sgpr %d", kNextFreeSgpr);
    e.line("\t\t.amdhsa_accum_offset %d", (n_vgpr + 3) / 4 * 4);
    e.line("\t\t.amdhsa_reserve_vcc 1");
    e.line("\t\t.amdhsa_float_round_mode_32 0");
    e.line("\t\t.amdhsa_float_round_mode_16_64 0");
    e.line("\t\t.amdhsa_float_denorm_mode_32 3");
    e.line("\t\t.amdhsa_float_denorm_mode_16_64 3");
    e.line("\t\t.amdhsa_dx10_clamp 1");
    e.line("\t\t.amdhsa_ieee_mode 1");
    e.line("\t\t.amdhsa_fp16_overflow 0");
    e.line("\t\t.amdhsa_tg_split 0");
    e.line("\t.end_amdhsa_kernel");
    e.line("\t.text");
    e.line("\t.amdgpu_metadata");
    e.line("---");
    e.line("amdhsa.kernels:");
    e.line("  - .agpr_count:     0");
    e.line("    .args:");
    e.line("      - .actual_access:  read_only");
    e.line("        .address_space:  global");
    e.line("        .offset:         0");
    e.line("        .size:           8");
    e.line("        .value_kind:     global_buffer");
    e.line("      - .actual_access:  write_only");
    e.line("        .address_space:  global");
    e.line("        .offset:         8");
    e.line("        .size:           8");
    e.line("        .value_kind:     global_buffer");
    e.line("    .group_segment_fixed_size: %d", gen.lds_bytes);
    e.line("    .kernarg_segment_align: 8");
    e.line("    .kernarg_segment_size: 16");
    e.line("    .max_flat_workgroup_size: %d", W * kWave);
    e.line("    .name:           %s", sym);
    e.line("    .private_segment_fixed_size: 0");
    e.line("    .sgpr_count:     %d", kNextFreeSgpr + 6);
    e.line("    .sgpr_spill_count: 0");
    e.line("    .symbol:         %s.kd", sym);
    e.line("    .uniform_work_group_size: 1");
    e.line("    .uses_dynamic_stack: false");
    e.line("    .vgpr_count:     %d", n_vgpr);
    e.line("    .vgpr_spill_count: 0");
    e.line("    .wavefront_size: 64");
    e.line("amdhsa.target:   amdgcn-amd-amdhsa--gfx950");
    e.line("amdhsa.version:");
    e.line("  - 1");
    e.line("  - 2");
    e.line("...");
    e.line("");
    e.line("\t.end_amdgpu_metadata");

}

// The tile with the least expected time of those that hold the zero-filled A; -1: none does.
static int mfma_best_tile(const HostPlan &h, double *microseconds) {
    int best = -1;
    for (int i = 0; i < kMfmaConfigCount; ++i) {
        if (!mfma_fits(kMfmaConfigs[i], h.M, h.K, h.elem_size())) continue;
        const double t = mfma_microseconds(kMfmaConfigs[i], h.M, h.K, h.N, h.batch, h.elem_size(), h.out_elem_size());
        if (best < 0 || t < *microseconds) { *microseconds = t; best = i; }
    }
    return best;
}

// The generated kernel's time for the same problem: the fetches of B of a compute unit (one per code block, column
// tile and touched row of B) and the multiply-adds of a SIMD take 3.45 and 2.69 ns each on top of a launch of 2.33 us.
// The rows per block are those of the default shape before they are fitted to rounds of workgroups
// (rows_for_one_round, rows_without_thin_round).  Over 80 products drawn from M, K and N up to 4096, 80 % to 98 %
// zeros, 50 of them with fitted rows: 15 % root mean square, and the kernel that this estimate and mfma_microseconds
// choose takes 0.9 % more than the faster of the two on average (8 times the slower one, 1.33 times at most).  The
// fitted rows in the formula: 15 % as well, but 2.2 % (12 times, 1.47), because the products whose choice changes
// take longer than either figure says.  Those products were timed in launch order.  As workgroups are dealt now: 18 % (int8) and 20 %
// (half) over 700 drawn products near the line (this and mfma_microseconds within 0.45 to 1.5 of each other).
static double generated_microseconds(const HostPlan &h) {
    const double tiles = (double)((h.N + kWave - 1) / kWave) * h.batch, density = (double)h.nnz / ((double)h.M * h.K);
    const int ks = h.K >= 512 ? 8 : 1;
    const double rows = std::max(1.0, std::min(96.0, std::floor(h.M * tiles * ks / (ks > 1 ? 2048 : 1024))));
    const double touched = 1.0 - std::pow(1.0 - density, rows);
    return 2.33 + 3.45e-3 * std::ceil(h.M / rows) * h.K * touched * tiles / 256 + 2.69e-3 * (double)h.nnz * tiles / 1024;
}

// Second estimates of both, which look at more than the two above: a product that they put clearly on the generated
// kernel's side stays there.  Fitted, 9 % and 15 % root mean square, to 840 half and int8 products (M, K and N up to 4096,
// 80 % to 98 % zeros, uniform and skewed rows, odd sizes, batches), each timed with both kernels; with the kernels as they are now 9 %
// and 14 % (int8) to 16 % (half) over those 700.
// The matrix-core plan's time: the L2s fill up slower than the slabs are multiplied where the tiles that an XCD has in
// hand share little (in the better one of the two simple orders of tiles; the order the kernel takes, mfma_rows_per_part, shares
// as much or more); rows of C that do not begin on 8 bytes are stored in pieces, rows of B that do not begin on 4 bytes
// are copied in pieces; and a large C leaves the caches.
static double matrix_core_microseconds(const HostPlan &h, int tile, double first_estimate) {
    static const double fit[2][5] = {{0.946, 0.326, 0.179, 0.0267, 0.223}, {0.952, 0.356, 0.0306, 0.0557, 0.0228}};   // half, int8
    const double *f = fit[h.dtype == SPARSERT_I8];
    const MfmaConfig &c = kMfmaConfigs[tile];
    const int esz = h.elem_size(), osz = h.out_elem_size();
    const int64_t m_tiles = ((int64_t)h.M + c.tm - 1) / c.tm, n_tiles = ((int64_t)h.N + c.tn - 1) / c.tn, wgs = m_tiles * n_tiles * h.batch;
    const int64_t slab = (int64_t)c.steps * mfma_step(esz), slabs = (h.K + slab - 1) / slab;
    const double rounds = wgs > 1024 ? wgs / 256.0 : (double)((wgs + 255) / 256), out_mb = 1e-6 * h.M * h.N * (double)h.batch * osz;
    const bool m_fast = mfma_m_fast(c, h.M, h.K, h.N, esz);
    const double at_once = (double)std::min<int64_t>(32, (m_tiles * n_tiles + 7) / 8);   // tiles of an XCD
    const double fast = std::min((double)(m_fast ? m_tiles : n_tiles), at_once), slow = std::max(1.0, at_once / fast);
    const double bytes = 64.0 * c.steps * (m_fast ? fast * c.tm + slow * c.tn : fast * c.tn + slow * c.tm);   // of a slab
    const double fill = 8 * bytes / 4e6 - std::max(c.slab_shared * rounds, c.slab_alone) / rounds;            // all XCDs, 4 TB/s
    double t = f[0] * first_estimate + f[1] * std::max(0.0, fill) * rounds * slabs + f[4] * std::max(0.0, out_mb - 16);
    if ((int64_t)h.ldc * osz % 8) t += f[2] * out_mb;
    if ((int64_t)h.ldb * esz % 4) t += f[3] * rounds * slabs;
    return t;
}

// The generated kernel's time in its default shape: the fetches of B and the multiply-adds of the busiest compute unit, C,
// one wave's chain of fetches, the longest row (one compute unit works it off), and the code a compute unit runs, which
// the waves of a K split do not share.
static double generated_shape_microseconds(const HostPlan &h, const sparsert_options &opt) {
    static const double fit[2][7] = {{2.04, 0.696, 0.411, 0.293, 9.37, 1.74, 0.449}, {2.14, 0.459, 1.50, 0.157, 9.07, 1.99, 0.345}};   // half, int8
    const double *f = fit[h.dtype == SPARSERT_I8];
    SpecPlan sp;
    Shape sh;
    std::string err;
    if (choose_launch_shape(h, opt, sp, sh, err)) return HUGE_VAL;   // no generated kernel
    const double nonzeros = (double)h.nnz / sp.n_groups;   // of a block
    const double touched = h.K * (1.0 - std::pow(1.0 - (double)h.nnz / ((double)h.M * h.K), (double)h.M / sp.n_groups));
    const int tiles = sp.ksplit > 1 ? 1 : sp.tiles_per_wg;   // of a workgroup
    const double wgs = (double)sp.n_groups * ((sp.n_tiles + tiles - 1) / tiles) * h.batch, rounds = wgs > 1024 ? wgs / 256 : std::ceil(wgs / 256);
    const double longest = *std::max_element(h.row_nnz.begin(), h.row_nnz.end());
    return f[0] + f[3] * 1e-6 * h.M * h.N * (double)h.batch * h.out_elem_size() +
           1e-3 * (rounds * (f[1] * touched * tiles + f[2] * nonzeros * tiles / 4 + f[6] * (nonzeros + 1.5 * touched)) + f[4] * touched / sp.ksplit + f[5] * longest);
}

static bool mfma_applies(const HostPlan &h) {
    return h.dtype != SPARSERT_F32 && !h.conv && h.N >= 16;
}

// An infinite or undefined weight makes every sum of its row non-finite, and the kernel would redo that row's columns
// on every call.
static bool all_finite(const HostPlan &h, const void *vals) {
    if (h.dtype != SPARSERT_F16) return true;   // int8
    for (int32_t p = 0; p < h.nnz; ++p) {
        uint16_t v;
        std::memcpy(&v, static_cast<const char *>(vals) + 2 * (size_t)p, 2);
        if ((v & 0x7c00u) == 0x7c00u) return false;
    }
    return true;
}

int mfma_preferred(const HostPlan &h, const sparsert_options &opt, const void *vals) {
    if (opt.kernel != SPARSERT_KERNEL_AUTO || opt.vec || opt.split_threshold || opt.spec_mode || opt.spec_rows || opt.spec_depth || opt.spec_tiles ||
        opt.spec_ksplit || opt.spec_lanes || opt.spec_swizzle || opt.spec_vec || opt.spec_prefetch > 0 || opt.natural_order || !mfma_applies(h))
        return -1;
    double t = 0;
    const int tile = mfma_best_tile(h, &t);
    if (tile < 0 || t >= generated_microseconds(h)) return -1;
    // 1.1: of the 562 of those products that the first estimates give to the matrix cores, those more than 5 % slower there than generated
    // fall from 19 (1.57 times at most: half 1384 x 128 x 3489, batch 4, at 85 %, 30.0 against 19.1 us) to 8 (1.25), and
    // two that were faster there by 7 % and 8 % are given up; a factor of 1 gives up ten, 1.32 times faster at most.
    // (With the kernels of that time.  Now, of the 700 near the line both tests give 448 to the matrix cores, 57 of them more than 5 % slower there, 1.32
    // times at most; of the rest 49 would be more than 5 % faster there, 2.2 times at most; all in all 3.1 % over the faster of the two each.)
    // (Where no code is generated the row-walk kernel would take over, which is further behind.)
    if (h.nnz <= kAutoSpecNnz && spec_available() && matrix_core_microseconds(h, tile, t) > 1.1 * generated_shape_microseconds(h, opt)) return -1;
    return all_finite(h, vals) ? tile : -1;
}

// Matrix-core plan: which tile, and the name a kernel trace shows.
static int build_mfma_plan(HostPlan &h, const sparsert_options &opt, std::string &err) {
    SpecPlan &sp = h.spec;
    double t = 0;
    const int best = mfma_best_tile(h, &t);
    const int found = opt.spec_ksplit > 1 ? -1 : opt.spec_rows || opt.spec_tiles ? mfma_find(opt.spec_rows, 16 * opt.spec_tiles) : best;
    if (!mfma_applies(h) || best < 0 || (found >= 0 && !mfma_fits(kMfmaConfigs[found], h.M, h.K, h.elem_size()))) {
        err = "the matrix-core variant is for half and int8 SpMM plans of at least 16 columns whose zero-filled A stays under 2 GiB";
        return SPARSERT_EUNSUPPORTED;
    }
    if (found < 0) { err = "no matrix-core kernel with these spec_rows and spec_tiles"; return SPARSERT_EINVAL; }
    const MfmaConfig &c = kMfmaConfigs[found];
    sp.mode = SPARSERT_SPEC_MFMA;
    sp.mfma_config = found;
    sp.rows_per_group = c.tm; sp.tiles_per_wg = c.tn / 16; sp.ksplit = 1;
    sp.lds_bytes = c.lds_bytes();
    sp.n_groups = sp.n_blocks = (h.M + c.tm - 1) / c.tm;
    sp.n_tiles = (h.N + c.tn - 1) / c.tn;
    sp.lanes_per_tile = 16;
    char sym[160];
    snprintf(sym, sizeof(sym), "void sparsert::mfma_kernel<%d, %d, %d, %d, %d, %d, %d>(sparsert::MfmaArgs)", h.dtype == SPARSERT_I8 ? 1 : 0,
             c.wm, c.wn, c.mf, c.nf, c.steps, c.stages);
    sp.symbol = sym;
    return SPARSERT_OK;
}

int build_spec_plan(HostPlan &h, const sparsert_options &opt, std::string &err) {
    SpecPlan &sp = h.spec;
    if (opt.spec_mode == SPARSERT_SPEC_MFMA || mfma_preferred(h, opt, h.p_vals.data()) >= 0) return build_mfma_plan(h, opt, err);
    Shape sh;
    if (int rc = choose_launch_shape(h, opt, sp, sh, err)) return rc;
    std::vector<std::vector<int32_t>> members;
    form_blocks(h, opt, sp, members);
    Gen gen(h, sp);
    Extents ex;
    if (int rc = plan_registers(h, sp, sh, members, gen, ex, err)) return rc;
    // The blocks are emitted first: the prologue wants to know how long the longest one is.
    Emitter &e = gen.e;
    sp.group_columns.assign(sp.n_blocks, 0);
    int64_t longest = 0;   // instructions of the longest block
    std::vector<size_t> gaps;            // where the text says how far apart the blocks are
    std::vector<int64_t> block_bytes;
    for (int g = 0; g < sp.n_blocks; ++g) {
        const int64_t before = e.lines, bytes_before = e.bytes;
        gaps.push_back(e.s.size());
        e.line("\t.space %8d", 0);   // (filled in below)
        e.line("\t.p2align 2");
        e.line(".Lg%d:", g);
        sp.group_columns[g] = sh.lds ? gen.block_lds(members[g], g % sh.W, sh.W)
                                     : gen.block_direct(members[g / sh.KS], g % sh.KS, sh.KS);
        longest = std::max(longest, e.lines - before);
        block_bytes.push_back(e.bytes - bytes_before);
    }
    const int gap = gap_between_blocks(e.bytes, sp.n_blocks);
    if (gap) {
        char text[24];
        const int n = snprintf(text, sizeof(text), "\t.space %8d", gap);
        for (size_t at : gaps) e.s.replace(at, (size_t)n, text);
    }
    const Deal deal = choose_deal(h, sp, block_bytes);
    emit_kernel_descriptor(gen, sh);
    // an instruction is at most 8 bytes; 64 lanes touch one 128-byte line each per prefetch
    // instruction, at most 32 of them (their offsets must fit the load's immediate field)
    const bool prefetch = opt.spec_prefetch > 0 || (opt.spec_prefetch == 0 && prefetch_pays(h, opt, sp, e.bytes));
    const int prefetch_lines = !prefetch ? 0 : (int)std::min<int64_t>(32, (longest * 8 + 64 * 128 - 1) / (64 * 128));
    sp.prefetch_lines = prefetch_lines;
    Emitter head;
    emit_prologue(gen, head, sh, ex, deal, prefetch_lines, gap);
    e.s.insert(0, head.s);

    if (const char *dump = getenv("SPARSERT_DUMP_ASM")) {
        if (FILE *f = fopen(dump, "w")) { fwrite(e.s.data(), 1, e.s.size(), f); fclose(f); }
    }
    sp.asm_bytes = (int64_t)e.s.size();
    if (int rc = assemble(e.s, sp.code, err)) return rc;
    return SPARSERT_OK;
}

}  // namespace sparsert
