// Row-walk SpMM that keeps a block of rows in registers, for fp32 products with many nonzeros.
//
// The plain and the staged row-walk kernels (kernels.hip, staged_rows.hip) fetch an operand for every nonzero.  Here a
// wave owns up to 84 rows and two columns of C per lane, 168 sums, and fetches a row of B once for all of the block's nonzeros in
// that column of A, as the generated kernel does - but from data, not from code: the sum that a multiply-add adds to
// is picked by the row number of the nonzero (s_set_gpr_idx_idx, vector registers indexed by a scalar register).  The waves of
// a workgroup split a block's columns and their sums meet in LDS, in wave order.
//
// The columns of a wave's part are sorted by how many nonzeros they have in the block and taken in groups of sixteen, so that the
// group's nonzeros come in layers of one per column, of which hardly any is a filler (2 % at 90 % zeros and 57 rows): the
// operand registers are then the same in every layer.  The wave's stream holds, in the order it is walked, the group's layers as
// records of 80 bytes (sixteen values, sixteen row numbers in bytes) and, behind a group's last one, the header of the group after
// the next (sixteen byte offsets into B, and the number of layers less one; -1 behind the last group).  A filler multiplies zero by
// whatever the operand is, into a sum of its own that nobody reads.
//
// 4096 x 4096 x 784 at 90 %: 124.3 us staged, 90 us here (57 rows, four waves).  What bounds it: 18 clocks per nonzero and SIMD, of which
// the two multiply-adds take 8 (an indexed or scalar operand costs four clocks, not two) and setting the row 4 of another unit; without
// the fetches of B (17 k wave loads per compute unit) 75 us are left, without the multiply-adds 102, with the stream always in
// the scalar cache 92: three parts of 60 to 75 us each that two waves per SIMD do not hide well behind each other.  Measured slower: one
// column per lane with four waves per SIMD (117 us; the stream is read twice as often), groups of eight columns with three
// waves (101), the next header asked for ahead of its place (100), fetches one by one between the last layer's multiply-adds (105).
// Error against sums in 64 bits: 0.63 times the plain kernel's over 43 products, 1.007 times at most (the sums of four or eight waves meet last).
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>
#include <string>

#include "blocked_rows.h"
#include "lds_copy.h"

namespace sparsert {

struct BlockedArgs {
    const uint32_t *stream;
    const uint32_t *starts;      // [block][wave]: first record
    const int32_t *rows;         // [block][kBlockedRows]: row of C, -1 for none
    const float *in;
    float *out;
    uint32_t records;            // of the stream
    int32_t M, K, N, ldb, ldc;
    int32_t lanes, tiles, blocks, per_part, rows_per_block;
};

// Scalar registers: a record in s[36:55] and the one after it in s[56:75] (which is which changes with every record), s76 a row number, s77 the
// M0 to put back.
// Vector registers: operands of every other group in v[8:23] (first column of the lane) and v[24:39] (second), of those between in
// v[40:55] and v[56:71]; sums of the first column in v[72:156], of the second in v[158:242], the last of each for fillers.
#define SP_X "36"
#define SP_Y "56"
#define SP_EACH(...) ".set sparsert_i, 0\n\t.rept 16\n\t" __VA_ARGS__ ".set sparsert_i, sparsert_i+1\n\t.endr\n\t"
#define SP_FETCH(R) "s_load_dwordx16 s[" R ":" R "+15], %[base], %[at]\n\ts_load_dwordx4 s[" R "+16:" R "+19], %[base], %[at] offset:64\n\ts_add_u32 %[at], %[at], 80\n\t"
// The stream's next four KiB, into the L2 cache: a scalar load that has to go beyond it takes 1 us.
#define SP_TOUCH "buffer_load_dword v243, %[touch], %[rstream], %[at] offen\n\t"
#define SP_ROW(R) ".if sparsert_i & 3\n\ts_lshr_b32 s76, s[" R "+16+sparsert_i/4], 8*(sparsert_i & 3)\n\ts_set_gpr_idx_idx s76\n\t.else\n\ts_set_gpr_idx_idx s[" R "+16+sparsert_i/4]\n\t.endif\n\t"
#define SP_MAD(R, B, SUM) "v_fma_f32 v[" SUM "], s[" R "+sparsert_i], v[" B "+sparsert_i], v[" SUM "]\n\t"
#define SP_LAYER(R, B, B1) SP_EACH(SP_ROW(R) SP_MAD(R, B, "72") SP_MAD(R, B1, "158"))
#define SP_OPERANDS(R, B, OFF) SP_EACH("buffer_load_dword v[" B "+sparsert_i], " OFF ", %[rsrc], s[" R "+sparsert_i] offen\n\t")
// The layers of a group whose operands are in B and B1, the first one in record R while T arrives.  Behind the last layer T is the
// header of the group after the next, which gets this one's operand registers; the next group's operands, fetched before this group's
// layers, are there once no more than the first half of the fetches and the touch in front of it are on their way.
#define SP_GROUP(B, B1, R, T, HERE, SAME_T, OTHER_R)                                                                   \
    "Lsp_" HERE "_%=:\n\ts_waitcnt lgkmcnt(0)\n\t" SP_FETCH(T) SP_LAYER(R, B, B1)                                       \
    "s_sub_u32 %[left], %[left], 1\n\ts_cbranch_scc0 Lsp_" SAME_T "_%=\n\t"                                            \
    "s_waitcnt lgkmcnt(0)\n\t" SP_FETCH(R)                                                                              \
    "s_mov_b32 %[left], %[next]\n\ts_mov_b32 %[next], s[" T "+16]\n\t" SP_TOUCH SP_OPERANDS(T, B, "%[off0]")           \
    "s_waitcnt vmcnt(17)\n\t" SP_OPERANDS(T, B1, "%[off1]")                                                            \
    "s_cmp_lt_i32 %[left], 0\n\ts_cbranch_scc0 Lsp_" OTHER_R "_%=\n\ts_branch Lsp_end_%=\n\t"
#define SP_CLOBBERS \
    "v8", "v9", "v10", "v11", "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", "v21", "v22", "v23", "v24", "v25", "v26", "v27", "v28", \
    "v29", "v30", "v31", "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", "v48", \
    "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", \
    "v69", "v70", "v71", "v156", "v157", "v242", "v243", "s36", "s37", "s38", "s39", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", \
    "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", \
    "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "scc", "memory"

template <int PARTS>
__global__ __launch_bounds__(PARTS *kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void blocked_rows_kernel(const BlockedArgs a) {
    typedef float float32 __attribute__((ext_vector_type(32)));
    typedef float float16 __attribute__((ext_vector_type(16)));
    typedef float float4v __attribute__((ext_vector_type(4)));
    typedef const uint32_t __attribute__((address_space(4))) *words_t;
    typedef const int32_t __attribute__((address_space(4))) *ints_t;
    constexpr int PAIRS = 8;   // of rows, per phase of the exchange
    __shared__ __align__(1024) float4v lds[PARTS * PAIRS * kWave];
    // Parts of per_part blocks one after the other, in a part column tile by column tile; every XCD takes an eighth of that order.
    const int tasks = a.tiles * a.blocks;
    const int task = (int)(blockIdx.x & 7) * ((tasks + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (task >= tasks) return;
    const int part = task / (a.per_part * a.tiles), in_part = task - part * (a.per_part * a.tiles), here = min(a.per_part, a.blocks - part * a.per_part);
    const int tile = in_part / here, block = part * a.per_part + in_part - tile * here;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *in = a.in + (int64_t)blockIdx.y * ((int64_t)a.K * a.ldb);
    float *out = a.out + (int64_t)blockIdx.y * ((int64_t)a.M * a.ldc);
    // A lane's two columns are a.lanes apart, so that a wave load is a run of consecutive bytes.  Lanes without a column fetch one
    // that exists; what they sum is dropped.
    const int col0 = tile * 2 * a.lanes + lane, col1 = col0 + a.lanes;
    const bool owns0 = lane < a.lanes && col0 < a.N, owns1 = lane < a.lanes && col1 < a.N;
    const int off0 = min(col0, a.N - 1) * 4, off1 = min(col1, a.N - 1) * 4, touch = lane * 64;
    const uint32_t first = ((words_t)a.starts)[block * PARTS + wave];
    const uint64_t base = (uint64_t)a.stream + (uint64_t)first * (kBlockedRecord * 4);
    const int4v rsrc = descriptor(in, ((a.K - 1) * a.ldb + a.N) * 4);
    const int4v rstream = descriptor((const void *)base, (int)min((uint64_t)0x7fffffff, (uint64_t)(a.records - first) * (kBlockedRecord * 4)));

    float32 a0, a1, b0, b1;
    float16 a2, b2;
    float4v a3, b3;
    int left, next;
    uint32_t at = 0;
    // (s_set_gpr_idx_* write M0, which the compiler may use for an index of its own and does not take as clobbered: it is put back)
    asm volatile(
        "s_mov_b32 s77, m0\n\t" SP_FETCH(SP_X) SP_FETCH(SP_Y) ".set sparsert_i, 0\n\t.rept 171\n\tv_mov_b32 v[72+sparsert_i], 0\n\t.set sparsert_i, sparsert_i+1\n\t.endr\n\t"
        "s_waitcnt lgkmcnt(0)\n\ts_mov_b32 %[left], s[" SP_X "+16]\n\ts_mov_b32 %[next], s[" SP_Y "+16]\n\t"
        SP_OPERANDS(SP_X, "8", "%[off0]") SP_OPERANDS(SP_X, "24", "%[off1]") SP_TOUCH SP_OPERANDS(SP_Y, "40", "%[off0]")
        "s_waitcnt vmcnt(17)\n\t" SP_OPERANDS(SP_Y, "56", "%[off1]") SP_FETCH(SP_X)
        "s_set_gpr_idx_on %[left], gpr_idx(SRC2,DST)\n\ts_cmp_lt_i32 %[left], 0\n\ts_cbranch_scc1 Lsp_end_%=\n\t"
        SP_GROUP("8", "24", SP_X, SP_Y, "px", "py", "qx")
        SP_GROUP("8", "24", SP_Y, SP_X, "py", "px", "qy")
        SP_GROUP("40", "56", SP_X, SP_Y, "qx", "qy", "px")
        SP_GROUP("40", "56", SP_Y, SP_X, "qy", "qx", "py")
        "Lsp_end_%=:\n\ts_set_gpr_idx_off\n\ts_mov_b32 m0, s77\n\ts_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 4\n\t"
        : "=&{v[72:103]}"(a0), "=&{v[104:135]}"(a1), "=&{v[136:151]}"(a2), "=&{v[152:155]}"(a3),
          "=&{v[158:189]}"(b0), "=&{v[190:221]}"(b1), "=&{v[222:237]}"(b2), "=&{v[238:241]}"(b3),
          [left] "=&s"(left), [next] "=&s"(next), [at] "+&s"(at)
        : [off0] "v"(off0), [off1] "v"(off1), [touch] "v"(touch), [rsrc] "s"(rsrc), [rstream] "s"(rstream), [base] "s"(base)
        : SP_CLOBBERS);

    // ---- the waves' sums meet in LDS, sixteen rows at a time; each wave adds and stores some of them.
    const ints_t rows = (ints_t)a.rows + block * kBlockedRows;
    auto sum0 = [&](int r) { return r < 32 ? a0[r & 31] : r < 64 ? a1[r & 31] : r < 80 ? a2[r & 15] : a3[r & 3]; };   // (r is a constant)
    auto sum1 = [&](int r) { return r < 32 ? b0[r & 31] : r < 64 ? b1[r & 31] : r < 80 ? b2[r & 15] : b3[r & 3]; };
    auto store = [&](int r, float v0, float v1) {
        const int row = rows[r];
        if (row < 0) return;
        float *to = out + (size_t)row * a.ldc;
        if (owns0) to[col0] = v0;
        if (owns1) to[col1] = v1;
    };
    static_assert(kBlockedRows % 2 == 0, "rows in pairs");
#pragma unroll
    for (int r0 = 0; r0 < kBlockedRows; r0 += 2 * PAIRS) {
        if (r0 >= a.rows_per_block) return;
        if (r0) __syncthreads();
#pragma unroll
        for (int q = 0; q < PAIRS; ++q) {
            const int r = r0 + 2 * q;
            if (r < kBlockedRows && r < a.rows_per_block) lds[(wave * PAIRS + q) * kWave + lane] = float4v{sum0(r), sum1(r), sum0(r + 1), sum1(r + 1)};
        }
        __syncthreads();
        for (int q = wave; q < PAIRS && r0 + 2 * q < a.rows_per_block; q += PARTS) {
            float4v s = lds[q * kWave + lane];
#pragma unroll
            for (int p = 1; p < PARTS; ++p) s += lds[(p * PAIRS + q) * kWave + lane];
            store(r0 + 2 * q, s[0], s[1]);
            store(r0 + 2 * q + 1, s[2], s[3]);
        }
    }
}

int prepare_blocked_rows(const HostPlan &h, const BlockedRows &s, DevicePlan &d, std::string &err) {
    BlockedArgs a;
    a.stream = d.stream; a.starts = reinterpret_cast<const uint32_t *>(d.staged_starts); a.rows = d.staged_rows;
    a.in = nullptr; a.out = nullptr;   // of the call
    a.records = (uint32_t)(d.staged_stream_bytes / (kBlockedRecord * 4));
    a.M = h.M; a.K = h.K; a.N = h.N; a.ldb = h.ldb; a.ldc = h.ldc;
    a.lanes = s.lanes; a.tiles = s.tiles; a.blocks = s.blocks; a.per_part = s.per_part; a.rows_per_block = s.rows;
    const int64_t tasks = (int64_t)s.tiles * s.blocks;
    if (h.dtype != SPARSERT_F32 || h.conv || s.rows < 1 || s.rows > kBlockedRows || (s.parts != 4 && s.parts != 8) || (int64_t)s.blocks * s.rows < h.M ||
        s.lanes < 1 || s.lanes > kWave || (int64_t)s.tiles * 2 * s.lanes < h.N || s.per_part < 1 || tasks > (1ll << 24) || h.batch < 1 || h.batch > 65535 ||
        ((int64_t)(h.K - 1) * h.ldb + h.N) * 4 >= (1ll << 31) || (int64_t)d.staged_stream_bytes >= (int64_t)kBlockedRecord * 4 << 31) {
        err = "plan geometry is inconsistent";
        return SPARSERT_EINVAL;
    }
    hipFunction_t fn = nullptr;
    const hipError_t e = hipGetFuncBySymbol(&fn, s.parts == 8 ? (const void *)blocked_rows_kernel<8> : (const void *)blocked_rows_kernel<4>);
    if (e != hipSuccess) { err = std::string("blocked row-walk kernel: ") + hipGetErrorString(e); return SPARSERT_EHIP; }
    static_assert(sizeof(BlockedArgs) <= sizeof(d.launch.args), "room for the arguments");
    d.launch.function = fn;
    d.launch.grid[0] = (uint32_t)((tasks + 7) / 8) * 8u; d.launch.grid[1] = (uint32_t)h.batch; d.launch.grid[2] = 1;
    d.launch.threads = (uint32_t)(s.parts * kWave);
    d.launch.arg_bytes = sizeof(a); d.launch.in_at = offsetof(BlockedArgs, in); d.launch.out_at = offsetof(BlockedArgs, out);
    std::memcpy(d.launch.args, &a, sizeof(a));
    return SPARSERT_OK;
}

}  // namespace sparsert
