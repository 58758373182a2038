// Matrix-core executor for half and int8 SpMM plans.
//
// The generated kernel runs half and int8 products at the vector unit's fp32 rate, one multiply-add
// per kept weight and column.  The matrix cores contract a zero-filled tile of A some thirty times
// faster per element, so from a few percent of kept weights on it is cheaper to hand them the
// zeros than to skip them: products of two halves are exact in fp32 and the sums are fp32 either
// way, int8 sums are exact integers, so nothing about the result's precision changes.
//
// Layout: the plan keeps A as fragments of 16 rows x one instruction step of K (32 halves or 64
// int8), 1 KiB each in the order the lanes hold them.  Fragments and rows of B travel to LDS with
// the memory path's direct copies (buffer_load ... lds, 1 KiB per wave instruction, no registers),
// several slabs ahead: every launch finds the L2 caches empty, so a slab is 1 us away.  B lies in LDS
// as in memory and is read back transposed (ds_read_b64_tr), which leaves four (eight) consecutive
// rows of K of one column in a lane; the order of K inside a fragment follows from that and is the
// same in A's fragments.
//
// The activations are the first operand of the instruction and the weights the second, so a lane
// ends up with four consecutive columns of one row of C and stores them with one instruction.
//
// Zeros of A meet every element of B here, and zero times infinity is not zero.  A non-finite
// element of B (or weight of A) leaves a non-finite sum in every row of its column, so sums that are
// all finite prove that nothing of the kind was involved; a wave that finds one that is not redoes
// the columns that hold one from the nonzero stream alone, as the row-walk kernel would.
// 1024 x 1024 x 4096 half at 80 %, 10 us: with one infinity in B 38 us, with 64 of them scattered 64 us, with a
// whole row of B not a number 406 us (1.84, 1.96 and 2.29 ms when the wave redid all of its part, one lane one element
// at a time); latency of the fetches is what it spends the time on.
// What bounds it, from builds with one ingredient left out (128 x 128 tile, K = 2048, one tile per compute unit):
// LDS reads alone need 0.27 us per slab, matrix instructions alone 0.21 us, both 0.36 us, and 0.5 us with
// the copies, which also write LDS.  Eight waves instead of four were worth 1.1x (a wave issues an instruction
// every four clocks at best, and a slab is a hundred of them), addresses kept in the descriptor's scalar
// offset instead of vector adds 1.15x.  1024 x 1024 x 4096 half at 80 %: 45.2 us generated, 10.2 us here (operands and plans taking
// turns, as in the next two); 3072 x 768 x 1024 half at 95 %: 11.3 and 8.1 us; 768 x 3072 x 1024 int8 at 95 %: 13.9 and 9.4 us.  Measured slower: a ring of
// eight slabs, or K split over two or four groups of waves with a ring each (before a wave multiplies it issues its part of
// the ring: 128 KiB take a compute unit 1 us; 768 x 1574 x 172 int8: 3.9 -> 4.9 us), and two slabs before the first turn with the
// rest of the ring issued in the first two (0.2 us faster on repeated operands, 0.1 to 0.3 us slower on new ones).
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>
#include <string>
#include <type_traits>
#include <utility>

#include "lds_copy.h"
#include "mfma.h"
#include "plan.h"

namespace sparsert {

namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef int32_t int2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v *lds_short4;
typedef __attribute__((address_space(3))) int2v *lds_int2;

}  // namespace

struct MfmaArgs {
    const void *weights;                 // fragments of A: [row tile of 16][step of K][lane][16 bytes]
    const void *in;                      // B [K, ldb]
    void *out;                           // C [M, ldc]
    const int32_t *p_row_ptr, *inv_perm; // the nonzero stream, for tiles with non-finite sums
    const uint2 *stream;
    int32_t M, K, N, ldb, ldc;
    int32_t per_part;                    // tiles along M of a part (mfma_rows_per_part)
    uint32_t part_magic, here_magic, last_magic;   // for the divisions by a part's tiles, by per_part and by what is left for the last part
};

// x / d for d whose magic is ceil(2^32 / d), exact while x * d < 2^32; 0: d is 1 or the product too large.
__device__ __forceinline__ uint32_t quotient(uint32_t x, uint32_t d, uint32_t magic) { return magic ? __umulhi(x, magic) : x / d; }

template <int DT> struct Kind;           // 0: half, 1: int8
template <> struct Kind<0> {
    typedef _Float16 in_t; typedef _Float16 out_t; typedef float4v acc_t; typedef half8 frag_t;
    static constexpr int esz = 2;
    static __device__ __forceinline__ acc_t mma(const frag_t &a, const frag_t &b, const acc_t &c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};
template <> struct Kind<1> {
    typedef int8_t in_t; typedef int32_t out_t; typedef int4v acc_t; typedef int4v frag_t;
    static constexpr int esz = 1;
    static __device__ __forceinline__ acc_t mma(const frag_t &a, const frag_t &b, const acc_t &c) {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
    }
};

// Element (row, n) of the product from the nonzero stream: the path for non-finite operands.  Eight nonzeros at a
// time, their pairs fetched a turn ahead; what a turn reads behind the row belongs to the next one or to the 16
// pairs of padding behind the stream, and is not used.
__device__ __forceinline__ float exact_element(const MfmaArgs &a, const _Float16 *in, int row, int n) {
    constexpr int U = 8;
    const int slot = a.inv_perm[row], p1 = a.p_row_ptr[slot + 1];
    int p = a.p_row_ptr[slot];
    float s = 0.0f;
    uint2 e[U];
#pragma unroll
    for (int i = 0; i < U; ++i) e[i] = a.stream[p + i];
#pragma unroll 1
    for (; p < p1; p += U) {
        uint2 next[U];
        _Float16 b[U];
#pragma unroll
        for (int i = 0; i < U; ++i) b[i] = in[(int)e[i].x / 2 + n];
#pragma unroll
        for (int i = 0; i < U; ++i) next[i] = a.stream[p + U + i];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const float t = __builtin_fmaf(__uint_as_float(e[i].y), (float)b[i], s);
            s = p + i < p1 ? t : s;
            e[i] = next[i];
        }
    }
    return s;
}

template <typename F, int... I> __device__ __forceinline__ void each_constant(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}

// Waves per SIMD the registers are to leave room for: two, or one where the slabs in LDS keep a second workgroup of
// four waves from the compute unit (160 KiB).
constexpr int mfma_waves_per_simd(int tm, int tn, int waves, int steps, int stages) {
    return waves >= 8 || 2 * (tm + tn) * 64 * steps * stages <= 160 * 1024 ? 2 : 1;
}

template <int DT, int WM, int WN, int MF, int NF, int STEPS, int STAGES>
__global__ __launch_bounds__(WM *WN *kWave, mfma_waves_per_simd(WM *MF * 16, WN *NF * 16, WM *WN, STEPS, STAGES)) void mfma_kernel(const MfmaArgs a) {
    typedef Kind<DT> Q;
    typedef typename Q::acc_t acc_t;
    typedef typename Q::frag_t frag_t;
    typedef typename Q::in_t in_t;
    typedef typename Q::out_t out_t;
    constexpr int ESZ = Q::esz, STEP = 64 / ESZ, EPC = 16 / ESZ, WAVES = WM * WN;
    constexpr int TM = WM * MF * 16, TN = WN * NF * 16;
    constexpr int SLAB = STEPS * STEP;                   // rows of K per slab
    constexpr int A_BYTES = TM * STEPS * 64, STAGE = A_BYTES + TN * STEPS * 64;
    constexpr int IA = A_BYTES / 1024 / WAVES, IB = TN * STEPS * 64 / 1024 / WAVES;   // 1 KiB copies per wave and slab
    static_assert(IA * WAVES * 1024 == A_BYTES && (IA + IB) * WAVES * 1024 == STAGE, "the copies of a slab are dealt evenly");
    static_assert((IA + IB) * (STAGES - 1) < 64, "vmcnt is a 6-bit counter");
    constexpr int CPR = TN * ESZ / 16, RPC = 64 / CPR;   // 16-byte chunks per row of the tile, rows per copy
    constexpr int ROWS256 = 256 / (TN * ESZ) > 0 ? 256 / (TN * ESZ) : 1;
    __shared__ __align__(1024) char lds[STAGES * STAGE];

    // All arguments in one go: left alone they arrive in four batches, each waited for.
    asm volatile("" ::"s"(a.weights), "s"(a.in), "s"(a.out), "s"(a.M), "s"(a.K), "s"(a.N), "s"(a.ldb), "s"(a.ldc), "s"(a.per_part), "s"(a.part_magic), "s"(a.here_magic), "s"(a.last_magic));
    const int m_tiles = (a.M + TM - 1) / TM, n_tiles = (a.N + TN - 1) / TN, tasks = m_tiles * n_tiles;
    const int n_slabs = (a.K + SLAB - 1) / SLAB, k_steps = n_slabs * STEPS;
    const int task = (int)(blockIdx.x & 7) * ((tasks + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (task >= tasks) return;
    // Parts of per_part tiles along M one after the other, in a part column tile by column tile: an XCD's eighth of the
    // tasks is then a block of tiles in both directions.
    const uint32_t part = quotient(task, (uint32_t)(a.per_part * n_tiles), a.part_magic), in_part = (uint32_t)task - part * (uint32_t)(a.per_part * n_tiles);
    const uint32_t left = (uint32_t)m_tiles - part * (uint32_t)a.per_part;
    const uint32_t here = left < (uint32_t)a.per_part ? left : (uint32_t)a.per_part;
    const int tile_n = (int)quotient(in_part, here, here == (uint32_t)a.per_part ? a.here_magic : a.last_magic);
    const int tile_m = (int)(part * (uint32_t)a.per_part + in_part - (uint32_t)tile_n * here);
    // of one problem: reads and writes stay inside
    const int in_bytes = ((a.K - 1) * a.ldb + a.N) * ESZ, weight_bytes = m_tiles * (TM / 16) * k_steps * 1024;
    const int out_bytes = (int)(((uint32_t)(a.M - 1) * (uint32_t)a.ldc + (uint32_t)a.N) * (uint32_t)sizeof(out_t));
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int m0 = tile_m * TM + wm * MF * 16, n_tile0 = tile_n * TN, n0 = n_tile0 + wn * NF * 16;
    const in_t *in = static_cast<const in_t *>(a.in) + (int64_t)blockIdx.y * ((int64_t)a.K * a.ldb);
    out_t *out = static_cast<out_t *>(a.out) + (int64_t)blockIdx.y * ((int64_t)a.M * a.ldc);
    // Where N is no multiple of EPC the last 16-byte chunk of a row begins at N - EPC: it holds some
    // columns twice, every one of them real, so neither the loads nor the stores know ragged ends.
    auto column = [&](int n) { return n - max(0, (n & -EPC) + EPC - a.N); };   // column of C behind column n of the tiling
    // Chunk c of row r lies at position c ^ swizzle(r) of the row in LDS: the rows that half a wave reads
    // together (8 x 32 bytes of halves, 16 x 16 bytes of int8) then cover all banks once.
    auto swizzle = [](int r) { return DT == 0 ? r / ROWS256 % (CPR / 2) * 2 : r / ROWS256 % CPR; };

    // ---- copies: this lane's chunk of every copy of a slab.  What leaves the operand (rows past K in the last
    // slab, an offset of kRefused) the descriptor answers with zeros and no memory access; so it does for every
    // copy of a slab past the last one, whose descriptors have no bytes.
    const int4v rin = descriptor(in, in_bytes), rw = descriptor(a.weights, weight_bytes);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    constexpr int kRefused = (int)0x80000000;
    int b_off[IB];
#pragma unroll
    for (int i = 0; i < IB; ++i) {
        const int row = (wave * IB + i) * RPC + lane / CPR, n = n_tile0 + (lane % CPR ^ swizzle(row)) * EPC;
        b_off[i] = n < a.N && row < a.K ? (int)(((uint32_t)row * (uint32_t)a.ldb + (uint32_t)column(n)) * ESZ) : kRefused;
    }
    constexpr bool PAIRS = IA % STEPS == 0;   // a wave copies whole runs of steps of a row tile: one offset per run
    int a_off[IA];
#pragma unroll
    for (int i = 0; i < IA; ++i) {
        const int q = wave * IA + i;
        a_off[i] = ((tile_m * (TM / 16) + q / STEPS) * k_steps + q % STEPS) * 1024 + lane * 16;
    }
    struct Source { int4v rin, rw; int sin, sw; uint32_t base; };
    auto source = [&](int s) {   // what the copies of slab s have in common
        const bool live = s < n_slabs;
        Source c{rin, rw, live ? (int)((uint32_t)s * (uint32_t)(SLAB * ESZ) * (uint32_t)a.ldb) : 0, live ? s * (STEPS * 1024) : 0,
                 lds0 + (uint32_t)(s % STAGES) * STAGE};
        c.rin[2] = live ? in_bytes : 0;
        c.rw[2] = live ? weight_bytes : 0;
        return c;
    };
    // Copy i of this wave's IA + IB copies of a slab.
    auto issue = [&](const Source &c, auto which) {
        constexpr int i = which;
        if constexpr (i < IA) {
            constexpr int first = PAIRS ? i / STEPS * STEPS : i;
            copy_to_lds<(i - first) * 1024>(c.rw, a_off[first], c.sw, c.base + (uint32_t)(wave * IA + first) * 1024);
        } else {
            constexpr int b = i - IA;
            copy_to_lds<0>(c.rin, b_off[b], c.sin, c.base + A_BYTES + (uint32_t)(wave * IB + b) * 1024);
        }
    };
    acc_t acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) acc[i][j] = acc_t{0, 0, 0, 0};
    const int g = lane >> 4, lg = lane & 15;
    // Where the transposing reads of a lane begin: row 4g + lg/4 (8g + lg/2) of a step, and the piece of 8 bytes inside 16 columns.
    const int rd_row = DT == 0 ? 4 * g + (lg >> 2) : 8 * g + (lg >> 1), rd_swz = swizzle(rd_row);
    int rd[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int c = DT == 0 ? (wn * NF + j) * 2 + (lg >> 1 & 1) : wn * NF + j;
        rd[j] = A_BYTES + rd_row * (TN * ESZ) + (c ^ rd_swz) * 16 + (lg & 1) * 8;
    }
    const int rd_a = wm * MF * STEPS * 1024 + lane * 16;

    // ---- slabs.  While slab s is multiplied out of registers, the fragments of slab s + 1 are read from LDS and
    // the copies of slab s + STAGES go out, a few of each behind every group of matrix instructions: LDS, the
    // memory path and the matrix cores each need about as long as the others, so they have to run at the same time.
    constexpr int GROUPS = STEPS * NF, UNITS = STEPS * (MF + NF);
    struct Fragments { frag_t w[STEPS][MF], x[STEPS][NF]; };
    auto each_copy = [&](auto f) { each_constant(f, std::make_integer_sequence<int, IA + IB>()); };
    auto read = [&](char *base, int u, Fragments &f) {
        const int t = u / (MF + NF), r = u % (MF + NF);
        if (r < MF) {
            f.w[t][r] = *reinterpret_cast<const frag_t *>(base + rd_a + (r * STEPS + t) * 1024);
            return;
        }
        char *p = base + rd[r - MF] + t * STEP * TN * ESZ;
        int2v v[2];
        if constexpr (DT == 0) {
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)p);
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p + STEP / 2 * TN * ESZ));
            __builtin_memcpy(&v[0], &lo, 8);
            __builtin_memcpy(&v[1], &hi, 8);
        } else {
            v[0] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_int2)p);
            v[1] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_int2)(p + STEP / 2 * TN * ESZ));
        }
        __builtin_memcpy(&f.x[t][r - MF], v, 16);
    };
    auto meet = [&]() {   // every wave's copies of the slab waited for have arrived, and every read issued so far is complete
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto turn = [&](int s, Fragments &now, Fragments &next, auto last) {
        if constexpr (!last) {
            wait_loads<(IA + IB) * (STAGES - 2)>();      // this wave's copies of slab s + 1
            meet();
        }
        char *base = lds + (s + 1) % STAGES * STAGE;
        const Source from = source(s + STAGES);
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
#pragma unroll
            for (int j = 0; j < NF; ++j) {
#pragma unroll
                for (int i = 0; i < MF; ++i) acc[i][j] = Q::mma(now.x[t][j], now.w[t][i], acc[i][j]);
                if constexpr (last) continue;
                const int q = t * NF + j;   // (a constant: the loops are unrolled)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = q * UNITS / GROUPS; u < (q + 1) * UNITS / GROUPS; ++u) read(base, u, next);
                each_copy([&](auto i) {
                    if (i >= q * (IA + IB) / GROUPS && i < (q + 1) * (IA + IB) / GROUPS) issue(from, i);
                });
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    Fragments even, odd;
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
        const Source from = source(s);
        each_copy([&](auto i) { issue(from, i); });
    }
    wait_loads<(IA + IB) * (STAGES - 1)>();
    meet();
#pragma unroll
    for (int u = 0; u < UNITS; ++u) read(lds, u, even);
    int s = 0;
    for (; s + 1 < n_slabs; s += 2) {
        turn(s, even, odd, std::false_type());
        turn(s + 1, odd, even, std::false_type());
    }
    if (s < n_slabs) turn(s, even, odd, std::true_type());
    wait_loads<0>();

    // ---- results.  Stores outside C (rows past M, chunks past N) are refused by the descriptor.
    const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(out, 0, out_bytes, 0x00020000);
    const uint32_t row_bytes = (uint32_t)a.ldc * (uint32_t)sizeof(out_t);
    const bool lines = row_bytes % 128 == 0 && TN * sizeof(out_t) % 128 == 0;   // whole ones are written
    // Through LDS, so that a wave stores whole rows of the tile: straight from the accumulators it would be 16 rows of 32
    // (int8: 64) bytes each.  Without whole lines int8 stays with that (3784 x 182 x 200, batch 4: 6.4 against 6.6 us), and so do half
    // tiles of 32 x 32, whose rows never are whole lines (83 products of 3 to 5 us: 1.2 % faster).  Half tiles of 32 x 64: 0.98 times as fast
    // through LDS where rows of C begin on 8 bytes, 1.03 times with whole lines or many rows that do not; asking at run time costs 2 %.
    // 3072 x 768 x 1024 half, repeated, with plain stores: 9.2 -> 8.6 us; 1472 x 168 x 2592 int8 7.8 -> 6.3 us (stored as below).
    bool finite = true;   // all sums of the workgroup
    if (DT == 0 ? TM > 32 || TN > 32 : lines) {
        constexpr int PITCH = TN * (int)sizeof(out_t) + 16;   // rows 16 bytes further apart: fewer bank conflicts
        constexpr int FLAGS = TM * PITCH;
        static_assert(FLAGS + WAVES * 4 <= STAGES * STAGE, "the tile's results fit the slabs");
        float probe = 0.0f;   // becomes NaN with the first sum that is not finite
        meet();   // every wave has read the last slab, and no copy is on its way
        char *mine = lds + (wm * MF * 16 + lg) * PITCH + (wn * NF * 16 + 4 * g) * (int)sizeof(out_t);
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const acc_t v = acc[i][j];
                char *to = mine + i * 16 * PITCH + j * 16 * (int)sizeof(out_t);
                if constexpr (DT == 0) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) probe = __builtin_fmaf(v[r], 0.0f, probe);
                    *reinterpret_cast<half4 *>(to) = half4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};   // one rounding to nearest even
                } else {
                    *reinterpret_cast<acc_t *>(to) = v;
                }
            }
        if constexpr (DT == 0) *reinterpret_cast<int *>(lds + FLAGS + wave * 4) = __any(probe != probe);
        __syncthreads();
        if constexpr (DT == 0) {
            int flags = 0;
#pragma unroll
            for (int w = 0; w < WM * WN; ++w) flags |= *reinterpret_cast<const int *>(lds + FLAGS + w * 4);
            finite = __builtin_amdgcn_readfirstlane(flags) == 0;
        }
        if (__builtin_expect(finite, 1)) {
            constexpr int CHUNKS = TN * (int)sizeof(out_t) / 16, ROWS = WAVES * kWave / CHUNKS;   // 16-byte pieces of a row; rows per pass
            static_assert((TM + ROWS - 1) / ROWS * ROWS * PITCH <= STAGES * STAGE, "the last pass reads inside the slabs");
            const int n = n_tile0 + tid % CHUNKS * (16 / (int)sizeof(out_t)), r0 = tid / CHUNKS;
            uint32_t off = (uint32_t)(tile_m * TM + r0) * row_bytes + (uint32_t)column(n) * (uint32_t)sizeof(out_t);
            const bool columns = (n & -EPC) < a.N;
            const char *from = lds + r0 * PITCH + tid % CHUNKS * 16;
            auto store = [&](auto policy) {
#pragma unroll
                for (int r = 0; r < TM; r += ROWS, off += ROWS * row_bytes) {
                    const int4v v = *reinterpret_cast<const int4v *>(from + r * PITCH);
                    const bool stored = columns & (tile_m * TM + r + r0 < a.M) & (TM % ROWS == 0 || r + r0 < TM);
                    __builtin_amdgcn_raw_buffer_store_b128(v, rout, stored ? (int)off : kRefused, 0, policy);
                }
            };
            // Whole lines of half results go through the L2 on their way (sc1), so that the launch's end has nothing left to write back, and
            // the caches behind it keep them for the layer that reads them next.  3072 x 768 x 1024, operands taking turns: plain 8.36 us, sc1
            // 7.83, not to be kept (nt) 8.07; with 768 x 3072 x 1024 behind it 20.7, 20.1 and 25.8, two square layers 1024 x 1024 x 4096
            // 23.4, 22.2 and 23.5.  39 drawn products: 1.03 times faster than plain; 26 whose lines are not whole up to 0.87 times, so those stay plain.
            // Int32 results are nt: an element-wise kernel reads them first, which takes as long behind it as behind plain stores
            // (35 products, to 0.5 %); alone they are 1.03 times faster for it, 1.1 with operands that no cache holds.
            if (lines) store(std::integral_constant<int, DT == 0 ? 16 : 2>());
            else store(std::integral_constant<int, 0>());
            return;
        }
    }
    float probe = 0.0f;
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const acc_t v = acc[i][j];
            const int row = m0 + i * 16 + lg, n = n0 + j * 16 + 4 * g;
            const bool mine = (row < a.M) & ((n & -EPC) < a.N);
            const int off = mine ? (int)((uint32_t)row * row_bytes + (uint32_t)column(n) * (uint32_t)sizeof(out_t)) : kRefused;
            if constexpr (DT == 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) probe = __builtin_fmaf(v[r], 0.0f, probe);
                const half4 h = {(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
                int2v b;
                __builtin_memcpy(&b, &h, 8);
                __builtin_amdgcn_raw_buffer_store_b64(b, rout, off, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128(v, rout, off, 0, 0);
            }
        }
    // A sum that is not finite: columns to redo.
    if constexpr (DT == 0) {
        if (__any(probe != probe)) {
            wait_loads<0>();   // the sums are out before what replaces them
            // The columns to redo, as bits: those of this wave in which any row's sum is not finite.  A column that two
            // waves store is in both or in neither, and with it every result is a function of its own operands alone.
            uint64_t bad = 0;
#pragma unroll
            for (int j = 0; j < NF; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float t = 0.0f;
#pragma unroll
                    for (int i = 0; i < MF; ++i) t = __builtin_fmaf(acc[i][j][r], 0.0f, t);
                    const uint64_t lanes = __ballot(t != t);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if ((lanes >> (16 * q) & 0xffffu) && ((n0 + j * 16 + 4 * q) & -EPC) < a.N) bad |= 1ull << (j * 16 + 4 * q + r);
                }
            // Lane i gets the i-th of them.  (The lanes without one go behind: the permutation reads no undefined lane.)
            const uint64_t below = (1ull << lane) - 1;
            const int count = __popcll(bad), to = bad >> lane & 1 ? __popcll(bad & below) : count + __popcll(~bad & below);
            const int nth = __builtin_amdgcn_ds_permute(to * 4, lane);
            // Elements column by column over the lanes: neighbouring lanes share a row where several columns are redone.
#pragma unroll 1
            for (int first = 0; first < count * MF * 16; first += kWave) {
                const int e = first + lane, i = e / count, row = m0 + i;
                const int n = column(n0 + __builtin_amdgcn_ds_bpermute((e - i * count) * 4, nth));
                if (i < MF * 16 && row < a.M) out[(size_t)row * a.ldc + n] = (_Float16)exact_element(a, in, row, n);
            }
        }
    }
}

int prepare_mfma(const HostPlan &h, DevicePlan &d, std::string &err) {
    const SpecPlan &sp = h.spec;
    if (!d.mfma_weights || sp.mfma_config < 0 || sp.mfma_config >= kMfmaConfigCount || h.N < 16 || h.batch < 1 || h.batch > 65535) {
        err = "plan geometry is inconsistent";
        return SPARSERT_EINVAL;
    }
    const MfmaConfig &c = kMfmaConfigs[sp.mfma_config];
    const int esz = h.elem_size();
    MfmaArgs a;
    a.weights = d.mfma_weights; a.in = nullptr; a.out = nullptr;   // of the call
    a.p_row_ptr = d.p_row_ptr; a.inv_perm = d.inv_perm; a.stream = reinterpret_cast<const uint2 *>(d.stream);
    a.M = h.M; a.K = h.K; a.N = h.N; a.ldb = h.ldb; a.ldc = h.ldc;
    const int64_t m_tiles = (h.M + c.tm - 1) / c.tm, tasks = m_tiles * ((h.N + c.tn - 1) / c.tn);
    if (tasks > (1ll << 30)) { err = "too many workgroups"; return SPARSERT_EUNSUPPORTED; }
    const int64_t n_tiles = (h.N + c.tn - 1) / c.tn;
    a.per_part = mfma_rows_per_part(c, h.M, h.K, h.N, h.ldb, esz);
    auto magic = [&](int64_t d) { return d > 1 && tasks * d < (1ll << 32) ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u; };
    a.part_magic = magic(a.per_part * n_tiles); a.here_magic = magic(a.per_part); a.last_magic = magic(m_tiles % a.per_part);
    if (!mfma_fits(c, h.M, h.K, esz) || ((int64_t)(h.K - 1) * h.ldb + h.N) * esz >= (1ll << 31)) { err = "plan geometry is inconsistent"; return SPARSERT_EINVAL; }
    const void *kernel = nullptr;
    switch (sp.mfma_config * 2 + (h.dtype == SPARSERT_I8 ? 1 : 0)) {
#define X(id, tm, tn, wm, wn, mf, nf, steps, stages, ...)                                              \
    case id * 2 + 0: kernel = (const void *)mfma_kernel<0, wm, wn, mf, nf, steps, stages>; break; \
    case id * 2 + 1: kernel = (const void *)mfma_kernel<1, wm, wn, mf, nf, steps, stages>; break;
        SPARSERT_MFMA_CONFIGS(X)
#undef X
    }
    hipFunction_t fn = nullptr;
    const hipError_t e = hipGetFuncBySymbol(&fn, kernel);
    if (e != hipSuccess) { err = std::string("matrix-core kernel: ") + hipGetErrorString(e); return SPARSERT_EHIP; }
    static_assert(sizeof(MfmaArgs) <= sizeof(d.launch.args), "room for the arguments");
    d.launch.function = fn;
    d.launch.grid[0] = (uint32_t)((tasks + 7) / 8) * 8u; d.launch.grid[1] = (uint32_t)h.batch; d.launch.grid[2] = 1;
    d.launch.threads = (uint32_t)(c.waves() * kWave);
    d.launch.arg_bytes = sizeof(a); d.launch.in_at = offsetof(MfmaArgs, in); d.launch.out_at = offsetof(MfmaArgs, out);
    std::memcpy(d.launch.args, &a, sizeof(a));
    return SPARSERT_OK;
}

}  // namespace sparsert
