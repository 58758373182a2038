// Row-walk SpMM with B staged through LDS, for products that are long enough to fill the chip with it.
//
// The plain row-walk kernel (kernels.hip) fetches a row segment of B through the vector-memory path for
// every nonzero and column tile, and that path delivers about 30 bytes per clock and compute unit: on
// 4096 x 4096 at 90 % with 784 columns it was all of the 287 us.  Here a workgroup copies the column tile's
// rows of B into LDS once, chunk by chunk (two buffers, the next chunk travels while one is worked on), for
// all of its 64 or 128 rows of A, and every nonzero reads its operand there.  A read of 8 or
// 16 bytes per lane takes LDS 2.2 or 4.1 clocks (250 bytes per clock; one of 4 bytes 2.3), so for the same product (49 of 64
// lanes own columns, 5 % of pairs only fill up) operand reads are 46 us, multiply-adds and addresses 50 us of every SIMD, and copies,
// 3.2 MB per compute unit, 18 us as writes to LDS and 25 us on the vector-memory path.  No one of them is the bound: without
// multiply-adds, reads or copies 106 to 118 us are left of 124, because the parts of a wave's step follow each other and
// the waves meet at every chunk's end.  Half and int8 move fewer bytes per nonzero and
// are bound by the instructions per nonzero and by the waits between them (2048 x 2048 at 95 %, 784 columns: half
// 39.2 us in the plain kernel, 25.9 us here in fours; int8 41.0 us, 24.7 us in fours with a v_dot4 per row and column).
//
// A wave owns up to RW rows, whose accumulators stay in registers over all chunks.  The nonzeros are laid
// out in the order the waves meet them - row group, wave, chunk, row - so a wave walks one contiguous
// stream of {LDS offset of the operand row, value} pairs with scalar loads, eight pairs at a time and four and
// two at the end of a row's share; how many twos belong to each of its rows comes packed in bytes, one word or two
// per chunk.  A share of odd length is filled up with a zero value times a row of zeros behind the chunk,
// never with elements of B.  A wave waits once per step, for its operands and the next step's words, some 400
// clocks with sixteen waves at the LDS; in steps of four at most it waited nearly twice as often (the product
// above 140.5 us; half 4096 x 1000 x 784 with skewed rows at 93.5 % 38.4 -> 31.2 us, int8 2048 x 3072 x 516, batch 4,
// at 82 % 304.8 -> 262.8 us).  A fourth size, six, cost 2 to 7 % of it all in fp32.  Row groups and waves are dealt in serpentine
// order over the rows by descending length.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>
#include <string>
#include <type_traits>

#include "lds_copy.h"
#include "staged_rows.h"

namespace sparsert {

struct StagedArgs {
    const uint2 *stream;          // {LDS byte offset, value bits}
    const uint32_t *counts;       // [group][wave][chunk][RW bytes]
    const int32_t *starts;        // [group][wave]: first stream position
    const int32_t *rows;          // [group][wave][RW]: row of C, -1 for none
    const void *in;
    void *out;
    int32_t M, K, N, ldb, ldc;
    int32_t lanes, tiles, groups;
    int32_t stream_bytes, pitch, chunk, chunks;
};

struct StagedShortArgs : StagedArgs {};   // of plans whose rows have few pairs in a chunk

// Bytes of one of the two LDS buffers: a chunk's rows and one row of zeros, in whole copies.
__host__ __device__ constexpr int staged_buffer_bytes(int chunk, int pitch) { return ((chunk + 1) * pitch + 1023) & ~1023; }

// A value of the stream in a vector register.  A v_fma_f32 with a scalar operand keeps its SIMD for four clocks, one with vector
// registers only (or a literal) for two where a second wave takes turns with it (4.2 and 2.2 measured with two to eight waves), so a
// move of four clocks pays from three multiply-adds on, so with four columns per lane: 4096 x 4096 x 784 at 90 % 135.9 -> 124.3 us, 3000 x
// 2048 x 784, batch 4, at 84.7 % 260 -> 232 us; at 98 % (4096 x 4096 x 784, 63.4 us) nothing changes, and of 16 others with four columns one, skewed, loses
// (4096 x 484 x 2036 at 91 % 40.0 -> 40.6); of 60 more, at 50 % to 95 %, 48 gain over 3 %, 0.935 times the time on average, and two lose, with
// skewed rows again (602 x 2898 x 1983 at 69 % 99.3 -> 104.2, 920 x 1308 x 1136 at 61 % 45.3 -> 46.5): there a wave with a row far longer than
// the others' has its SIMD to itself, which takes five clocks for either form, and the move comes on top.  With two columns it is not done: 1928 x 320 x 840 at 88 %, skewed, 11.4 us without, 12.4 with.  Half stays with the scalar operand: its products widen
// the operand as they go (v_fma_mix_f32), four clocks in any case.  (Assembly: the compiler would fold the move away.)
__device__ __forceinline__ float in_vector(uint32_t bits) {
    float f;
    asm("v_mov_b32 %0, %1" : "=v"(f) : "s"(bits));
    return f;
}

// Operands, multiply-adds and results of one storage type at V columns per lane.
template <typename T, int V> struct StagedOps {
    typedef float acc_t;
    typedef T out_t;
    typedef T opd_t __attribute__((ext_vector_type(V)));
    static __device__ __forceinline__ void mad2(float (&acc)[V], uint32_t w0, uint32_t w1, const opd_t &b0, const opd_t &b1) {
        float f0 = __uint_as_float(w0), f1 = __uint_as_float(w1);
        if constexpr (std::is_same<T, float>::value && V > 2) { f0 = in_vector(w0); f1 = in_vector(w1); }
#pragma unroll
        for (int j = 0; j < V; ++j) acc[j] = __builtin_fmaf(f0, (float)b0[j], acc[j]);
#pragma unroll
        for (int j = 0; j < V; ++j) acc[j] = __builtin_fmaf(f1, (float)b1[j], acc[j]);
    }
};
// The four packed columns stay in their dword.  Two operand rows are interleaved, so that one v_dot4 does a column of both;
// the stream has the values where they meet: in byte 0 of the first pair, in byte 1 of the second.
// (A v_dot4 per row and column, the value shifted into place by the scalar unit, took 1.07 to 1.29 times as long over 17 products:
// 3000 x 2048 x 784, batch 4, at 84.7 % 237 -> 183 us.)
template <> struct StagedOps<int8_t, 4> {
    typedef int32_t acc_t;
    typedef int32_t out_t;
    typedef int32_t opd_t;
    static __device__ __forceinline__ void mad2(int32_t (&acc)[4], uint32_t w0, uint32_t w1, const opd_t &b0, const opd_t &b1) {
        const int32_t lo = (int32_t)(w0 | w1), hi = (int32_t)((w0 | w1) << 16);
        const int32_t b01 = (int32_t)__builtin_amdgcn_perm((uint32_t)b1, (uint32_t)b0, 0x05010400u);   // columns 0 and 1
        const int32_t b23 = (int32_t)__builtin_amdgcn_perm((uint32_t)b1, (uint32_t)b0, 0x07030602u);
        acc[0] = __builtin_amdgcn_sdot4(b01, lo, acc[0], false);
        acc[1] = __builtin_amdgcn_sdot4(b01, hi, acc[1], false);
        acc[2] = __builtin_amdgcn_sdot4(b23, lo, acc[2], false);
        acc[3] = __builtin_amdgcn_sdot4(b23, hi, acc[3], false);
    }
};

template <typename T, int V, int RW, int MOST>   // MOST: pairs at a time, four or eight
__device__ __forceinline__ void staged_rows(const StagedArgs &a) {
    typedef StagedOps<T, V> Q;
    typedef typename Q::opd_t opd_t;
    typedef typename Q::out_t out_t;
    typedef typename Q::acc_t acc_t;
    constexpr int COPIES = kStagedLdsBytes / 2 / 1024 / kStagedWaves;   // 1 KiB copies per wave and chunk, at most
    __shared__ __align__(1024) char lds[kStagedLdsBytes];
    const int task = (int)(blockIdx.x & 7) * ((a.tiles * a.groups + 7) >> 3) + (int)(blockIdx.x >> 3);
    if (task >= a.tiles * a.groups) return;
    const int tile = task / a.groups, group = task - tile * a.groups;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T *in = static_cast<const T *>(a.in) + (int64_t)blockIdx.y * ((int64_t)a.K * a.ldb);
    const int col0 = tile * a.lanes * V;

    // this lane's 16 bytes of every copy of a chunk; what lies past the operand arrives as zeros
    const int4v rin = descriptor(in, ((a.K - 1) * a.ldb + a.N) * (int)sizeof(T)), rstream = descriptor(a.stream, a.stream_bytes);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;
    const int per_row = a.pitch >> 4, buffer = staged_buffer_bytes(a.chunk, a.pitch);
    int off[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
        const int unit = (i * kStagedWaves + wave) * 64 + lane, row = unit / per_row;
        // (rows past the chunk: zeros; the first of them is what the pairs that fill a group up refer to)
        off[i] = row < a.chunk ? row * a.ldb * (int)sizeof(T) + col0 * (int)sizeof(T) + (unit - row * per_row) * 16 : (int)0x80000000;
    }
    auto issue = [&](int c) {
        const int from = c * a.chunk * a.ldb * (int)sizeof(T);
        const uint32_t to = lds0 + (uint32_t)(c & 1) * (uint32_t)buffer;
#pragma unroll
        for (int i = 0; i < COPIES; ++i)
            if ((i * kStagedWaves + wave) * 1024 < buffer) copy_to_lds<0>(rin, off[i], from, to + (uint32_t)(i * kStagedWaves + wave) * 1024);
    };

    acc_t acc[RW][V];
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int j = 0; j < V; ++j) acc[r][j] = 0;
    const int owner = group * kStagedWaves + wave;
    // (constant address space: scalar loads, whatever the copies' assembly may touch)
    typedef uint32_t group_t __attribute__((ext_vector_type(2 * MOST), aligned(4)));
    typedef const uint2 __attribute__((address_space(4))) *pairs_t;
    typedef const uint32_t __attribute__((address_space(4))) *words_t;
    typedef const int32_t __attribute__((address_space(4))) *ints_t;
    pairs_t p = (pairs_t)a.stream + ((ints_t)a.starts)[owner];
    const words_t counts = (words_t)a.counts + (size_t)owner * a.chunks * (RW / 4);
    group_t next = *reinterpret_cast<const group_t __attribute__((address_space(4))) *>(p);
    // The next PAIRS pairs of the stream, of one row.
    auto step = [&](acc_t (&sum)[V], const char *base, auto pairs) {
        constexpr int PAIRS = decltype(pairs)::value;
        const group_t g = next;
        p += PAIRS;
        next = *reinterpret_cast<const group_t __attribute__((address_space(4))) *>(p);   // (the stream is padded by two groups of eight)
        opd_t b[PAIRS];
#pragma unroll
        for (int i = 0; i < PAIRS; ++i) b[i] = *reinterpret_cast<const opd_t *>(base + g[2 * i]);
#pragma unroll
        for (int i = 0; i < PAIRS; i += 2) Q::mad2(sum, g[2 * i + 1], g[2 * i + 3], b[i], b[i + 1]);
    };

    issue(0);
    for (int c = 0; c < a.chunks; ++c) {
        wait_loads<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();   // the chunk is there, and nobody reads the other buffer any more
        asm volatile("" ::: "memory");
        // The stream's cache lines of the next four KiB, into the L2 cache: a scalar load that has to go beyond it
        // takes 1 us, and waiting for LDS waits for scalar loads as well.  (The words themselves go to a corner of LDS.)
        touch_to_lds(rstream, (int)((const char __attribute__((address_space(4))) *)p - (const char __attribute__((address_space(4))) *)a.stream) + lane * 64, lds0 + kStagedLdsBytes - kStagedTouchBytes);
        if (c + 1 < a.chunks) issue(c + 1);
        const char *base = lds + (c & 1) * buffer + lane * (int)(V * sizeof(T));
        uint32_t cnt[RW / 4];
#pragma unroll
        for (int i = 0; i < RW / 4; ++i) cnt[i] = counts[c * (RW / 4) + i];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            int n = (int)(cnt[r / 4] >> (8 * (r % 4)) & 0xffu);   // twos
#pragma unroll 1
            for (; n >= MOST / 2; n -= MOST / 2) step(acc[r], base, std::integral_constant<int, MOST>());
            if (MOST == 8 && n > 1) { step(acc[r], base, std::integral_constant<int, 4>()); n -= 2; }
            if (n) step(acc[r], base, std::integral_constant<int, 2>());
        }
    }

    typedef out_t out_v __attribute__((ext_vector_type(V), aligned(sizeof(out_t))));
    const int col = col0 + lane * V;
    if (lane >= a.lanes || col >= a.N) return;
    out_t *out = static_cast<out_t *>(a.out) + (int64_t)blockIdx.y * ((int64_t)a.M * a.ldc);
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int row = ((ints_t)a.rows)[owner * RW + r];
        if (row < 0) continue;
        out_t *dst = out + (size_t)row * a.ldc + col;
        if (col + V <= a.N) {
            out_v v;
#pragma unroll
            for (int j = 0; j < V; ++j) v[j] = (out_t)acc[r][j];   // half: one rounding to nearest even
            *reinterpret_cast<out_v *>(dst) = v;
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j)
                if (col + j < a.N) dst[j] = (out_t)acc[r][j];
        }
    }
}

template <typename T, int V, int RW>
__global__ __launch_bounds__(kStagedWaves *kWave, 4) void staged_rows_kernel(const StagedArgs a) { staged_rows<T, V, RW, 8>(a); }
template <typename T, int V, int RW>
__global__ __launch_bounds__(kStagedWaves *kWave, 4) void staged_rows_kernel(const StagedShortArgs a) { staged_rows<T, V, RW, 4>(a); }

int prepare_staged_rows(const HostPlan &h, DevicePlan &d, std::string &err) {
    const StagedRows s = staged_rows_shape(h);
    StagedArgs a;
    const int esz = h.elem_size();
    a.stream = reinterpret_cast<const uint2 *>(d.stream);
    a.counts = reinterpret_cast<const uint32_t *>(d.staged_counts);
    a.starts = d.staged_starts; a.rows = d.staged_rows;
    a.in = nullptr; a.out = nullptr;   // of the call
    a.M = h.M; a.K = h.K; a.N = h.N; a.ldb = h.ldb; a.ldc = h.ldc;
    a.lanes = s.lanes; a.tiles = s.tiles; a.groups = s.groups;
    const int64_t tasks = (int64_t)s.tiles * s.groups;
    a.stream_bytes = (int32_t)d.staged_stream_bytes;
    a.pitch = s.pitch; a.chunk = s.chunk; a.chunks = s.chunks;
    // (the rule of staged_rows.h hands over nothing that does not fit)
    if (s.V == 0 || !staged_rows_fits(h, s) || 2 * staged_buffer_bytes(s.chunk, s.pitch) > kStagedLdsBytes - kStagedTouchBytes || d.staged_stream_bytes >= (1ull << 31) || s.chunk > 510 || s.lanes > kWave || s.pitch < s.lanes * s.V * esz ||
        (int64_t)s.groups * kStagedWaves * s.rows_per_wave < h.M || (int64_t)s.tiles * s.lanes * s.V < h.N) {
        err = "plan geometry is inconsistent";
        return SPARSERT_EINVAL;
    }
    typedef void (*plain_t)(StagedArgs);
    const void *kernel = nullptr;
    if (h.dtype == SPARSERT_I8) kernel = (const void *)static_cast<plain_t>(staged_rows_kernel<int8_t, 4, 4>);
    else if (h.dtype == SPARSERT_F16) kernel = (const void *)static_cast<plain_t>(staged_rows_kernel<_Float16, 4, 4>);
    else if (s.short_shares) {
        typedef void (*short_t)(StagedShortArgs);
        kernel = (const void *)(s.V == 4 ? static_cast<short_t>(staged_rows_kernel<float, 4, 4>) : s.rows_per_wave == 8 ? static_cast<short_t>(staged_rows_kernel<float, 2, 8>) : static_cast<short_t>(staged_rows_kernel<float, 2, 4>));
    } else {
        kernel = (const void *)(s.V == 4 ? static_cast<plain_t>(staged_rows_kernel<float, 4, 4>) : s.rows_per_wave == 8 ? static_cast<plain_t>(staged_rows_kernel<float, 2, 8>) : static_cast<plain_t>(staged_rows_kernel<float, 2, 4>));
    }
    hipFunction_t fn = nullptr;
    const hipError_t e = hipGetFuncBySymbol(&fn, kernel);
    if (e != hipSuccess) { err = std::string("staged row-walk kernel: ") + hipGetErrorString(e); return SPARSERT_EHIP; }
    static_assert(sizeof(StagedArgs) <= sizeof(d.launch.args), "room for the arguments");
    d.launch.function = fn;
    d.launch.grid[0] = (uint32_t)((tasks + 7) / 8) * 8u; d.launch.grid[1] = (uint32_t)h.batch; d.launch.grid[2] = 1;
    d.launch.threads = kStagedWaves * kWave;
    d.launch.arg_bytes = sizeof(a); d.launch.in_at = offsetof(StagedArgs, in); d.launch.out_at = offsetof(StagedArgs, out);
    std::memcpy(d.launch.args, &a, sizeof(a));
    return SPARSERT_OK;
}

}  // namespace sparsert
