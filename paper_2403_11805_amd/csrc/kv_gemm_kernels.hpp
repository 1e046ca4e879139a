// gfx950 GEMMs for the dense projections of the recompute path (Sec. 3.3): C[M][N] = A[M][K] * B[K][N] (+ Cin),
// fp16 operands, binary32 accumulation on MFMA, result in binary32 or rounded once to fp16.  The weights B keep
// their row-major [in][out] layout; the activations A come in fragment order (below), which the kernels that
// produce them write.  Up to three weight matrices that share A (q | k | v, gate | up) go through one launch.
// All extents are guarded: M any, N and K multiples of 8.
//
// Neither kernel passes the weights through LDS.  v_mfma_f32_32x32x16_f16 wants eight consecutive k of one
// column in a lane, the memory holds consecutive columns of one k: a lane loads two (four) adjacent columns of
// eight rows, and one v_perm_b32 per pair of rows and column turns them into the operands of two (four) column
// blocks - a register operation in the shadow of the MFMAs, where a transpose through LDS costs a write, a read
// and a barrier.  The lane's columns are adjacent, so results leave as 8- or 16-byte pieces.
//
// With few rows K is divided among workgroups (`splits`): each writes a binary32 partial product, and the kernel
// that reads the product next adds them in split order as it loads them (rotary encoding, the second norm, the
// gate activation: kv_recompute_kernels.hpp); gemm_reduce_kernel does it where no such kernel follows.
// (Measured: a workgroup that counts itself in on a tile counter and, as the last to arrive, adds the partial
// products itself needs device-scope fences around the counter, which more than double the time of a layer.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace kvs {

typedef _Float16 gv8h_t __attribute__((ext_vector_type(8)));
typedef _Float16 gv4h_t __attribute__((ext_vector_type(4)));
typedef _Float16 gv2h_t __attribute__((ext_vector_type(2)));
typedef float gv16f_t __attribute__((ext_vector_type(16)));
typedef float gv4f_t __attribute__((ext_vector_type(4)));
typedef float gv2f_t __attribute__((ext_vector_type(2)));
typedef unsigned int gu4_t __attribute__((ext_vector_type(4)));
typedef unsigned int gu2_t __attribute__((ext_vector_type(2)));

constexpr int kGemmMaxSplits = 16;
constexpr int kGemmMaxMats = 3;
constexpr int kGemmStep = 16;            // contraction length of one MFMA
constexpr int kGemmStage = 4;            // steps whose activations gemm_tile_kernel stages at a time
constexpr int kStreamCols = 128;         // columns of a workgroup of gemm_stream_kernel
constexpr int kTileCols = 256;           // columns of a workgroup of gemm_tile_kernel

// Fragment order of an activation matrix [M][K]: blocks of 32 rows (the last one may be shorter), inside a block
// the 16-byte pieces (eight consecutive k of one row) by (k / 8, row).  The MFMA operand of 32 rows x 16 k - rows
// across the lanes, the second eight k in the upper half of the wavefront - is then 1 KiB in one piece.  The
// matrix takes M * K halves, as it does row-major.
__host__ __device__ __forceinline__ int64_t fragment_at(int m, int k, int M, int K) {
    const int b = m >> 5;
    const int rows = M - 32 * b < 32 ? M - 32 * b : 32;
    return static_cast<int64_t>(b) * 32 * K + (static_cast<int64_t>(k >> 3) * rows + (m & 31)) * 8 + (k & 7);
}

struct GemmArgs {
    const _Float16* A;                  // [M][K] in fragment order
    const _Float16* B[kGemmMaxMats];    // [K][N[j]]
    void* C[kGemmMaxMats];              // [M][N[j]] fp16 or binary32, row-major or (fp16, gemm_stream_kernel) in fragment order
    const _Float16* Cin;                // [M][N[0]] fp16 or NULL (added before the result is rounded; one matrix only)
    float* part;                        // matrix j: part + part_at[j], [splits][M][N[j]] binary32 (splits > 1)
    uint64_t part_at[kGemmMaxMats];
    int32_t N[kGemmMaxMats];
    int32_t tile_end[kGemmMaxMats];     // column tiles of matrices 0..j together; unused entries: the total
    int32_t M, K;
    int32_t steps;                      // steps of one split
    int32_t splits;
    int32_t out_f32, out_fragments;
};

// Which rows of a weight matrix step `st` reads: the last step of a K that is no multiple of 16 reads the last 16
// rows, of which only the upper half of the wavefront is used (gemm_half_step: the lower half is zeroed there).
__device__ __forceinline__ int gemm_step_row(int st, int K) { return max(min(st * kGemmStep, K - kGemmStep), 0); }

// Buffer descriptor of a weight matrix from a row on: loads take the lane's offset from a register and the row
// from a scalar, so that a load costs no address arithmetic.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gemm_rows(const _Float16* B, int row, uint32_t row_bytes) {
    const char* at = reinterpret_cast<const char*>(B) + static_cast<size_t>(row) * row_bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(at), static_cast<short>(0), 0xffffffffu, 0x00027000);
}

// Results of row m, columns n .. n + 7: into the partial product of this split, or the result.
__device__ __forceinline__ void gemm_store8(const GemmArgs& g, int mat, int split, int m, int n, gv4f_t lo, gv4f_t hi) {
    const int N = g.N[mat];
    const size_t at = static_cast<size_t>(m) * N + n;
    if (g.splits > 1 || g.out_f32) {
        float* dst = g.splits > 1 ? g.part + g.part_at[mat] + split * (static_cast<size_t>(g.M) * N) : static_cast<float*>(g.C[mat]);
        *reinterpret_cast<gv4f_t*>(dst + at) = lo;
        *reinterpret_cast<gv4f_t*>(dst + at + 4) = hi;
        return;
    }
    gv8h_t r;
    if (g.Cin) {
        const gv8h_t c = *reinterpret_cast<const gv8h_t*>(g.Cin + at);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            lo[k] += static_cast<float>(c[k]);
            hi[k] += static_cast<float>(c[k + 4]);
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        r[k] = static_cast<_Float16>(lo[k]);
        r[k + 4] = static_cast<_Float16>(hi[k]);
    }
    *reinterpret_cast<gv8h_t*>(static_cast<_Float16*>(g.C[mat]) + (g.out_fragments ? fragment_at(m, n, g.M, N) : at)) = r;
}

// Up to 64 rows: bound by streaming the weights.  A workgroup owns all rows x 128 columns; its four wavefronts take
// the 16-row steps of K in turn, each holding the whole tile, with no barrier until their sums meet in LDS at the
// end.  A wavefront keeps its loads kDepth steps ahead (8 x 512 bytes of weights and MB KiB of activations each);
// the scheduling barriers keep the compiler from pulling the operand permutes of later steps, and with them the
// waits for their loads, in front.  Weights are read once and marked non-temporal (8 % of a loop over the four
// launches of a layer).
// Measured in a kernel trace, the four launches of a Llama-2-7B layer (404 MB of weights) at 16 rows: 80 us (5.05 TB/s;
// 82 with two workgroups on a third of the CUs in gate | up, 86 with the last few in a second round, the LDS-tiled kernel
// before it 107).
// Grid (column tiles of all matrices, splits), 256 threads; at most MB * 32 rows.
template <int MB>
__global__ __launch_bounds__(256, 2) void gemm_stream_kernel(GemmArgs g) {
    constexpr int kWaves = 4, kDepth = MB == 1 ? 4 : 3, kCols = kStreamCols;
    __shared__ gv4f_t sums[kWaves * 32 * kCols / 4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, j = lane & 31;
    const int tile = blockIdx.x;
    const int mat = (tile >= g.tile_end[0]) + (tile >= g.tile_end[1]);
    const int n0 = (tile - (mat ? g.tile_end[mat - 1] : 0)) * kCols;
    const int N = g.N[mat], K = g.K, K8 = K / 8;
    const int s_all = (K + kGemmStep - 1) / kGemmStep;
    const int sb = blockIdx.y * g.steps, se = min(s_all, sb + g.steps);
    const int n = (se - sb - wave + kWaves - 1) / kWaves;          // this wavefront: steps sb + wave + 4 i
    const uint32_t row_bytes = static_cast<uint32_t>(N) * 2u;
    const int col = min(n0 + 4 * j, N - 4);                        // columns beyond N repeat the last four, unstored
    const uint32_t voff = ((K >= kGemmStep ? half * 8u * static_cast<uint32_t>(N) : 0u) + static_cast<uint32_t>(col)) * 2u;
    const _Float16* a_base[MB];
    uint32_t a_rows[MB], a_lane[MB];                               // rows of the block, this lane's row in it
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const int rb = min(b * 32, (g.M - 1) / 32 * 32);
        a_rows[b] = static_cast<uint32_t>(min(32, g.M - rb));
        a_base[b] = g.A + static_cast<size_t>(rb) * K;
        a_lane[b] = min(static_cast<uint32_t>(j), a_rows[b] - 1);
    }
    gu2_t w[kDepth][8];
    gu4_t a[kDepth][MB];
    auto load = [&](int set, int i) __attribute__((always_inline)) {
        const int st = sb + wave + kWaves * min(i, n - 1);
        const __amdgpu_buffer_rsrc_t rows = gemm_rows(g.B[mat], gemm_step_row(st, K), row_bytes);
#pragma unroll
        for (int k = 0; k < 8; ++k)
            w[set][k] = __builtin_bit_cast(gu2_t, __builtin_amdgcn_raw_buffer_load_b64(rows, voff, k * row_bytes, 2));
        const uint32_t k8 = static_cast<uint32_t>(min(2 * st + half, K8 - 1));
#pragma unroll
        for (int b = 0; b < MB; ++b)
            a[set][b] = *reinterpret_cast<const gu4_t*>(a_base[b] + (k8 * a_rows[b] + a_lane[b]) * 8u);
    };
    gv16f_t acc[4][MB];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[c][b] = gv16f_t{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    auto multiply = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            gu4_t lo, hi;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                lo[p] = __builtin_amdgcn_perm(w[set][2 * p + 1][i], w[set][2 * p][i], 0x05040100u);
                hi[p] = __builtin_amdgcn_perm(w[set][2 * p + 1][i], w[set][2 * p][i], 0x07060302u);
            }
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                const gv8h_t af = __builtin_bit_cast(gv8h_t, a[set][b]);
                acc[2 * i][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, __builtin_bit_cast(gv8h_t, lo), acc[2 * i][b], 0, 0, 0);
                acc[2 * i + 1][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af, __builtin_bit_cast(gv8h_t, hi), acc[2 * i + 1][b], 0, 0, 0);
            }
        }
    };
    if (n > 0) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            load(d, d);
            __builtin_amdgcn_sched_barrier(0);
        }
        int s = 0;
        for (; s + kDepth < n; s += kDepth) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                multiply(d);
                load(d, s + d + kDepth);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const bool half_step = (K & 8) && se == s_all;
#pragma unroll
        for (int d = 0; d < kDepth; ++d)
            if (s + d < n) {
                if (half_step && sb + wave + kWaves * (s + d) == s_all - 1 && !half) {
#pragma unroll
                    for (int k = 0; k < 8; ++k) w[d][k] = gu2_t{0u, 0u};
#pragma unroll
                    for (int b = 0; b < MB; ++b) a[d][b] = gu4_t{0u, 0u, 0u, 0u};
                }
                multiply(d);
                __builtin_amdgcn_sched_barrier(0);
            }
    }
    // acc[c][b][v]: row b*32 + 8*(v/4) + 4*half + v%4, column n0 + 4*j + c; the wavefronts' sums are added in order
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        if (b) __syncthreads();
        gv4f_t* mine = sums + wave * (32 * kCols / 4);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            mine[(8 * (v / 4) + 4 * half + v % 4) * (kCols / 4) + j] = gv4f_t{acc[0][b][v], acc[1][b][v], acc[2][b][v], acc[3][b][v]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 32 * kCols / 8 / 256; ++i) {
            // eight columns of a row per thread; rows side by side where the result is in fragment order
            const int q = i * 256 + tid;
            const int r = g.out_fragments ? q % 32 : q / (kCols / 8), c8 = g.out_fragments ? q / 32 : q % (kCols / 8);
            gv4f_t lo = sums[r * (kCols / 4) + 2 * c8], hi = sums[r * (kCols / 4) + 2 * c8 + 1];
#pragma unroll
            for (int k = 1; k < kWaves; ++k) {
                lo += sums[(k * 32 + r) * (kCols / 4) + 2 * c8];
                hi += sums[(k * 32 + r) * (kCols / 4) + 2 * c8 + 1];
            }
            const int m = b * 32 + r, nn = n0 + 8 * c8;
            if (m < g.M && nn < N) gemm_store8(g, mat, blockIdx.y, m, nn, lo, hi);
        }
    }
}

// More than 64 rows.  A workgroup owns MB * 32 rows x 256 columns; each of its four wavefronts holds all the rows
// of 64 columns, so that a weight is loaded by one wavefront only, straight into registers, and only the
// activations go through LDS: 64 of K at a time, three buffers, loaded a stage ahead in registers, one barrier per
// stage and that in its middle, so that the first operands of the next stage are read without a wait.  One
// wavefront per SIMD (up to 256 accumulators; two at MB <= 4): nothing else hides an instruction that is not an
// MFMA, so the operand reads, permutes and loads of the next step are dealt out behind the MFMAs of this one, two
// and two (the scheduling barriers fix that order; left alone the compiler clusters them: 179 against 229 us for
// the four launches at 304 rows, 1509 against 1851 us at 4096).
// Measured, the four launches of a Llama-2-7B layer in a kernel trace: 304 rows 210 us (the LDS-tiled kernel before
// it 312), 512 rows 301 (348), 2048 rows 832 us = 1.00 PFLOP/s (the GEMM library's standard choice 1042).
// Loading eight columns of two rows per lane and exchanging them between lanes changes nothing (269 and 267 us a
// layer at 304 rows, 990 and 998 at 2048): the width of the weight loads is not what a step waits for.
// At few rows a step is bound by what the CU takes in: some 55 bytes per ns as soon as some loads miss L2, 52 KB for 64 of
// K at five row blocks (no MFMAs at all: 81 of 92 us for gate | up at 304 rows); at many by the chip's power and by the
// last round of workgroups.
// Grid 8 * ceil(column tiles * splits / 8) * row tiles, 256 threads; kGemmStage divides g.steps.
// (MB 8, GATED spills three registers, the others none.)
// GATED: two matrices of one width, splits == 1, and the result is C[0] = fp16(silu(A B[0]) * (A B[1])) in fragment
// order, both products rounded to fp16 first; a column tile is 128 columns of each.
template <int MB, bool GATED>
__global__ __launch_bounds__(256, MB <= 4 ? 2 : 1) void gemm_tile_kernel(GemmArgs g) {
    constexpr int kSets = MB <= 4 ? 4 : 8;           // steps of weights in registers
    constexpr int kUnroll = kSets / kGemmStage;      // stages per trip, so that the sets are named statically
    constexpr int kBuf = kGemmStage * MB * 64;       // 16-byte pieces of a stage
    __shared__ gu4_t stage_lds[3 * kBuf];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, j = lane & 31;
    // workgroups are dealt to the eight XCDs in turn: the row tiles of one column tile and split follow each other
    // on one XCD, whose L2 then serves these weights to all of them.  Splits and column tiles are dealt together:
    // each split by itself left XCDs short where the column tiles are no multiple of eight (20 of them, six splits,
    // 512 rows: 36 workgroups for the 32 CUs of four XCDs, 24 for those of the others)
    const int row_tiles = (g.M + MB * 32 - 1) / (MB * 32);
    const int grp = blockIdx.x / (8 * row_tiles), local = blockIdx.x - grp * 8 * row_tiles;
    const int unit = grp * 8 + (local & 7), m0 = (local >> 3) * MB * 32;
    const int tiles = g.tile_end[kGemmMaxMats - 1];
    if (unit >= tiles * g.splits) return;
    const int split = unit / tiles, tile = unit - split * tiles;
    // GATED: wavefronts 0 and 1 hold 128 columns of matrix 0, 2 and 3 the same columns of matrix 1
    const int mat = GATED ? wave >> 1 : (tile >= g.tile_end[0]) + (tile >= g.tile_end[1]);
    const int n0 = GATED ? tile * (kTileCols / 2) + (wave & 1) * 64
                           : (tile - (mat ? g.tile_end[mat - 1] : 0)) * kTileCols + wave * 64;
    const int N = g.N[mat], K = g.K, K8 = K / 8;
    const int s_all = (K + kGemmStep - 1) / kGemmStep;
    const int sb = split * g.steps, se = min(s_all, sb + g.steps);
    const int ns = se - sb, n_stages = (ns + kGemmStage - 1) / kGemmStage;
    const bool half_step = (K & 8) && se == s_all;
    const int full = (ns - (half_step ? 1 : 0)) / kGemmStage;      // stages of whole steps only
    const uint32_t row_bytes = static_cast<uint32_t>(N) * 2u;
    const int col = min(n0 + 2 * j, N - 2);                        // columns beyond N repeat the last two, unstored
    const uint32_t voff = ((K >= kGemmStep ? half * 8u * static_cast<uint32_t>(N) : 0u) + static_cast<uint32_t>(col)) * 2u;
    uint32_t w[kSets][8];
    gu4_t a_next[MB], af[2][MB], op[2][2];

    auto rows_of = [&](int step) __attribute__((always_inline)) {  // step of this split; beyond the last: the last
        return gemm_rows(g.B[mat], gemm_step_row(sb + min(step, ns - 1), K), row_bytes);
    };
    auto load_w = [&](int set, const __amdgpu_buffer_rsrc_t& rows, int k) __attribute__((always_inline)) {
        w[set][k] = __builtin_amdgcn_raw_buffer_load_b32(rows, voff, k * row_bytes, 0);
    };
    // activations: piece i * 256 + tid of a stage, i.e. fragment i * 4 + wave = (step, row block); byte offsets from
    // the first row block of the workgroup, so that the loads take a scalar base and a 32-bit offset
    const char* a_base = reinterpret_cast<const char*>(g.A + static_cast<size_t>(m0) * K);
    uint32_t a_at[MB], a_stage[MB], a_last[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int f = i * 4 + wave, st = f / MB, b = f % MB;
        const int rb = min(m0 + b * 32, (g.M - 1) / 32 * 32);
        const uint32_t rows = static_cast<uint32_t>(min(32, g.M - rb));
        const uint32_t at = static_cast<uint32_t>(rb - m0) * static_cast<uint32_t>(K) * 2u + min(static_cast<uint32_t>(j), rows - 1) * 16u;
        a_at[i] = at + static_cast<uint32_t>(2 * (sb + st) + half) * rows * 16u;
        a_stage[i] = 2 * kGemmStage * rows * 16u;
        a_last[i] = at + static_cast<uint32_t>(K8 - 1) * rows * 16u;       // pieces beyond K repeat the last one
    }
    auto load_a = [&](int i, int stage) __attribute__((always_inline)) {
        return *reinterpret_cast<const gu4_t*>(a_base + min(a_at[i] + static_cast<uint32_t>(stage) * a_stage[i], a_last[i]));
    };
    auto read_a = [&](int set, int buf, int st, int b) __attribute__((always_inline)) {
        af[set][b] = stage_lds[buf * kBuf + (st * MB + b) * 64 + lane];
    };
    auto permute = [&](int to, int set, int p) __attribute__((always_inline)) {
        op[to][0][p] = __builtin_amdgcn_perm(w[set][2 * p + 1], w[set][2 * p], 0x05040100u);
        op[to][1][p] = __builtin_amdgcn_perm(w[set][2 * p + 1], w[set][2 * p], 0x07060302u);
    };
    gv16f_t acc[2][MB];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < MB; ++b) acc[c][b] = gv16f_t{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    auto multiply = [&](int set, int b) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
            acc[c][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(gv8h_t, af[set][b]),
                                                               __builtin_bit_cast(gv8h_t, op[set][c]), acc[c][b], 0, 0, 0);
    };

    // Stages 0 and 1 of the activations, then the weights of the first kSets steps, in the order of the loop: a wait
    // for a stage's activations then leaves the weights behind them in flight.
    {
        gu4_t a_first[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) a_first[i] = load_a(i, 0);
#pragma unroll
        for (int i = 0; i < MB; ++i) a_next[i] = load_a(i, 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < kSets; ++d) {
            const __amdgpu_buffer_rsrc_t rows = rows_of(d);
#pragma unroll
            for (int k = 0; k < 8; ++k) load_w(d, rows, k);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) stage_lds[i * 256 + tid] = a_first[i];
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < MB; ++b) read_a(0, 0, 0, b);
    {
        const __amdgpu_buffer_rsrc_t rows = rows_of(kSets);
#pragma unroll
        for (int p = 0; p < 4; ++p) permute(0, 0, p);
#pragma unroll
        for (int k = 0; k < 8; ++k) load_w(0, rows, k);
    }
    int rd = 0;                                      // LDS buffer of the stage at hand
    // Stage s; its step t is weight set u * 4 + t.  Buffer rd + 1 receives stage s + 1: it was last read in stage
    // s - 2, which every wavefront has left when the barrier of stage s - 1 opens; what is written to it in step 0
    // is read behind this stage's barrier.  CHECKED: some step of the stage is missing or half.
    auto run_stage = [&](int s, int u, auto checked) __attribute__((always_inline)) {
        constexpr bool CHECKED = decltype(checked)::value;
        const int nx = rd == 2 ? 0 : rd + 1;
#pragma unroll
        for (int t = 0; t < kGemmStage; ++t) {
            const int cur = t & 1, step = kGemmStage * s + t, set = (u * kGemmStage + t + 1) % kSets;
            const int buf = t + 1 < kGemmStage ? rd : nx, st = t + 1 < kGemmStage ? t + 1 : 0;
            if (t == kGemmStage / 2) __syncthreads();
            const __amdgpu_buffer_rsrc_t rows = rows_of(step + 1 + kSets);
            if constexpr (CHECKED) {
                if (half_step && step == ns - 1 && !half) {
                    op[cur][0] = op[cur][1] = gu4_t{0u, 0u, 0u, 0u};
#pragma unroll
                    for (int b = 0; b < MB; ++b) af[cur][b] = gu4_t{0u, 0u, 0u, 0u};
                }
                if (step < ns) {
#pragma unroll
                    for (int b = 0; b < MB; ++b) multiply(cur, b);
                }
            }
#pragma unroll
            for (int b = 0; b < MB; ++b) {
                if constexpr (!CHECKED) multiply(cur, b);
                read_a(cur ^ 1, buf, st, b);
                if (b < 4) permute(cur ^ 1, set, b);
                if (MB < 4 && b == MB - 1) permute(cur ^ 1, set, 3);
                if (t == 0) {
                    stage_lds[nx * kBuf + b * 256 + tid] = a_next[b];
                    a_next[b] = load_a(b, s + 2);
                }
                // rows 2 p and 2 p + 1 are free once permute p has read them
                if (b >= 1 && b <= 4) {
                    load_w(set, rows, 2 * b - 2);
                    load_w(set, rows, 2 * b - 1);
                }
                if (b == MB - 1 && MB <= 4) {
#pragma unroll
                    for (int k = 2 * MB - 2; k < 8; ++k) load_w(set, rows, k);
                }
                if constexpr (!CHECKED) __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        rd = nx;
    };
    int s = 0;
    for (; s + kUnroll <= full; s += kUnroll) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) run_stage(s + u, u, std::false_type{});
    }
    // what is left: at most kUnroll - 1 whole stages and one that is not
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
        if (s + u < n_stages) run_stage(s + u, u, std::true_type{});
    // acc[c][b][v]: row m0 + b*32 + 8*(v/4) + 4*half + v%4, column n0 + 2*j + c.  Through LDS, block by block and
    // each wavefront for itself, so that the results leave in 16-byte pieces (rows padded by four floats)
    constexpr int kPitch = 64 + 4;
    static_assert(4 * 32 * kPitch * 4 <= 3 * kBuf * 16, "the staging buffers hold a block per wavefront");
    __syncthreads();
    float* tile_lds = reinterpret_cast<float*>(stage_lds) + wave * 32 * kPitch;
    if constexpr (GATED) {
        // Two row blocks at a time: the wavefront of matrix 0 finishes the first, its partner with the same columns
        // of matrix 1 the second; each hands the other the block it needs, lane by lane.
        const bool second = wave >= 2;
        const float* theirs = reinterpret_cast<float*>(stage_lds) + (wave ^ 2) * 32 * kPitch;
        _Float16* act_lds = reinterpret_cast<_Float16*>(tile_lds);
        constexpr int kActPitch = 64 + 8;            // halves
#pragma unroll
        for (int b = 0; b < MB; b += 2) {
            const int b2 = b + 1 < MB ? b + 1 : b;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                *reinterpret_cast<gv2f_t*>(tile_lds + (v * 64 + lane) * 2) =
                    second ? gv2f_t{acc[0][b][v], acc[1][b][v]} : gv2f_t{acc[0][b2][v], acc[1][b2][v]};
            __syncthreads();
            gv2f_t other[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) other[v] = *reinterpret_cast<const gv2f_t*>(theirs + (v * 64 + lane) * 2);
            __syncthreads();
            const int mb = m0 + (second ? b2 : b) * 32;
            if (second && b2 == b) continue;         // (uniform; nothing is left of an odd number of blocks)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                gv2h_t o;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float own = second ? acc[c][b2][v] : acc[c][b][v];
                    const float x = static_cast<float>(static_cast<_Float16>(second ? other[v][c] : own));
                    const float u = static_cast<float>(static_cast<_Float16>(second ? own : other[v][c]));
                    o[c] = static_cast<_Float16>(x / (1.0f + __expf(-x)) * u);
                }
                *reinterpret_cast<gv2h_t*>(act_lds + (8 * (v / 4) + 4 * half + v % 4) * kActPitch + 2 * j) = o;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c8 = 2 * i + half, m = mb + j, n = n0 + 8 * c8;
                const gv8h_t r = *reinterpret_cast<const gv8h_t*>(act_lds + j * kActPitch + 8 * c8);
                if (m < g.M && n < N) *reinterpret_cast<gv8h_t*>(static_cast<_Float16*>(g.C[0]) + fragment_at(m, n, g.M, N)) = r;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    } else {
#pragma unroll
        for (int b = 0; b < MB; ++b) {
#pragma unroll
            for (int v = 0; v < 16; ++v)
                *reinterpret_cast<gv2f_t*>(tile_lds + (8 * (v / 4) + 4 * half + v % 4) * kPitch + 2 * j) = gv2f_t{acc[0][b][v], acc[1][b][v]};
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 8 * i + (lane >> 3), c8 = lane & 7;
                const gv4f_t* src = reinterpret_cast<const gv4f_t*>(tile_lds + r * kPitch + 8 * c8);
                const int m = m0 + b * 32 + r, n = n0 + 8 * c8;
                if (m < g.M && n < N) gemm_store8(g, mat, split, m, n, src[0], src[1]);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    }
}

// C[0] = fp16(sum of matrix 0's partial products in split order + Cin); four adjacent columns per thread.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmArgs g) {
    const size_t n4 = static_cast<size_t>(g.M) * g.N[0] / 4;
    const size_t i = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n4) return;
    const gv4f_t* part = reinterpret_cast<const gv4f_t*>(g.part);
    gv4f_t a = part[i];
#pragma unroll 4
    for (int s = 1; s < g.splits; ++s) a += part[static_cast<size_t>(s) * n4 + i];
    if (g.Cin) {
        const gv4h_t c = reinterpret_cast<const gv4h_t*>(g.Cin)[i];
        a += gv4f_t{static_cast<float>(c[0]), static_cast<float>(c[1]), static_cast<float>(c[2]), static_cast<float>(c[3])};
    }
    const gv4h_t h = {static_cast<_Float16>(a[0]), static_cast<_Float16>(a[1]), static_cast<_Float16>(a[2]),
                      static_cast<_Float16>(a[3])};
    reinterpret_cast<gv4h_t*>(g.C[0])[i] = h;
}

}  // namespace kvs
