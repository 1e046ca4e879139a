// libkvswitch: recompute of interleaved chunks through one Llama-style block
// (Sec. 3.3, "Making interleaved chunks recomputable").  Host side: argument
// checks, the workspace plan, the dense projections and the launches of the
// kernels in kv_recompute_kernels.hpp.  The projections of up to kOwnGemmRows
// recomputed tokens - what a plan of Eq. 4 recomputes beside a Load - run on the
// library's own MFMA GEMM (kv_gemm_kernels.hpp); larger ones go to rocBLAS, which
// is loaded at run time if it is there (the rest of the library does not depend
// on it, and without it every size runs on the library's own kernel).

#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "kv_gemm_kernels.hpp"
#include "kv_internal.h"
#include "kv_launch_rules.hpp"
#include "kv_recompute_kernels.hpp"

using namespace kvs;

namespace {

// The few rocBLAS entry points used, with the library's published C signatures and enum values.
typedef void* rb_handle;
typedef int (*rb_create_fn)(rb_handle*);
typedef int (*rb_destroy_fn)(rb_handle);
typedef int (*rb_set_stream_fn)(rb_handle, hipStream_t);
typedef int (*rb_gemm_ex_fn)(rb_handle, int, int, int, int, int, const void*, const void*, int, int,
                             const void*, int, int, const void*, const void*, int, int, void*, int, int,
                             int, int, int32_t, uint32_t);
constexpr int kRbOpNone = 111;        // rocblas_operation_none
constexpr int kRbF16 = 150;           // rocblas_datatype_f16_r
constexpr int kRbF32 = 151;           // rocblas_datatype_f32_r
constexpr int kRbAlgoStandard = 0;    // rocblas_gemm_algo_standard
constexpr int kRbAlgoSolution = 1;    // rocblas_gemm_algo_solution_index
// Lists the library's kernels ("solutions") that can run a given gemm_ex call (same arguments,
// then flags, list, list size; a NULL list returns the count).
typedef int (*rb_get_solutions_fn)(rb_handle, int, int, int, int, int, const void*, const void*, int, int,
                                   const void*, int, int, const void*, const void*, int, int, void*, int, int,
                                   int, int, uint32_t, int*, int*);

// Measured on MI355X, a whole layer in us: own kernels / the GEMM library's standard choice
//   d_model 4096, 32 kv heads, d_ff 11008:  1536 rows 808 / 852   2048 rows 982 / 1208   2560 rows 1203 / 1167
//                                           3072 rows 1403 / 1476   4096 rows 1844 / 1839
//   d_model 4096,  8 kv heads, d_ff 14336:  2048 rows 1024 / 1070
//   d_model 2048, 16 kv heads, d_ff 5632:   1024 rows 236 / 302   2048 rows 413 / 432
// Up to 2048 rows the own kernels are no slower at any width from 1024 to 8192 (table in kvswitch.h); of the
// library's tuned kernels one is faster there (d_model 5120, 2048 rows: 1457 against 1520 us).
constexpr int64_t kOwnGemmRows = KV_RECOMPUTE_OWN_GEMM_ROWS;

uint64_t align256(uint64_t v) { return (v + 255) & ~static_cast<uint64_t>(255); }

struct Plan {
    uint64_t xn, q32, k32, v32, q16, attn, x1, gate, up, part_o, total;
};

// Up to three weight matrices [K][N[j]] applied to the same activations in one launch.
struct GemmGroup {
    int n;
    int64_t N[kGemmMaxMats];
    const void* B[kGemmMaxMats];
    void* C[kGemmMaxMats];
};

// Launch shape of the library's own GEMM: row blocks of 32 per workgroup, streamed or tiled, steps of K per
// split, number of splits.
struct OwnGemm {
    int mb, steps, splits;
    bool stream;
    uint32_t col_tiles, row_tiles;      // (row tiles: tiled only; a streamed workgroup holds all rows)
};

// Up to 64 rows the weights are streamed: one row block with stream_splits, two with as many splits (at most 8) as keep
// one workgroup on a CU: for a Llama-2-7B layer q | k | v 2 and 2, o and down 8 and 8, gate | up 1 and 1.
// Above, the row blocks per workgroup (3..8) and the splits that minimise
//     rounds of 256 workgroups * steps * (0.184 + 0.0453 * row blocks) us
//     + writing and reading the partial products at 3.25 TB/s each;
// up to four row blocks a CU holds two workgroups, and two full rounds together cost 1.72 of one.  Fitted to all
// row blocks and splits of the four launches of layers of width 1024, 4096 and 5120 at 80 .. 2048 rows (28 layers):
// the choice costs a launch 0.3 % of its layer's time on average over the fastest one (a rule without the discount,
// with 5 TB/s and a floor for the weights' bytes: 0.5 %; down, 4096 wide, d_ff 14336, 512 rows, a layer in all: 4
// splits of 4 row blocks 340 us, that rule's 8 splits of 8 row blocks 348).
// `room` bytes are there for partial products.  A handle may fix the row blocks and the splits of the tiled launches
// (`fixed`; as many splits as room and K allow).
struct FixedTile {
    int row_blocks = 0, splits = 0;     // 0: chosen
};
OwnGemm own_gemm_plan(int64_t M, const int64_t* N, int n_mats, int64_t K, uint64_t room, FixedTile fixed) {
    OwnGemm best{};
    int64_t n_sum = 0;
    for (int j = 0; j < n_mats; ++j) n_sum += N[j];
    const int64_t steps = (K + kGemmStep - 1) / kGemmStep;
    const int64_t part = M * n_sum * 4;                                  // bytes of one split's partial product
    const int64_t room_splits = std::min<int64_t>(kGemmMaxSplits, static_cast<int64_t>(room / static_cast<uint64_t>(part)));
    auto tiles = [&](int64_t cols) {
        int64_t t = 0;
        for (int j = 0; j < n_mats; ++j) t += (N[j] + cols - 1) / cols;
        return t;
    };
    if (M <= 64) {
        best.stream = true;
        best.mb = M <= 32 ? 1 : 2;
        best.col_tiles = static_cast<uint32_t>(tiles(kStreamCols));
        int64_t s = std::max<int64_t>(1, std::min<int64_t>({256 / best.col_tiles, 8, room_splits, steps / 16}));
        if (best.mb == 1) s = stream_splits(best.col_tiles, steps, room_splits);
        best.steps = static_cast<int>((steps + s - 1) / s);
        best.splits = static_cast<int>((steps + best.steps - 1) / best.steps);
        return best;
    }
    double least = 0.0;
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>(room_splits, steps / (2 * kGemmStage)));
    const int64_t s_from = fixed.splits ? std::min<int64_t>(fixed.splits, most) : 1, s_to = fixed.splits ? s_from : most;
    for (int mb = 3; mb <= 8; ++mb) {
        if (fixed.row_blocks && mb != fixed.row_blocks) continue;
        const int64_t row_tiles = (M + 32 * mb - 1) / (32 * mb);
        for (int64_t s = s_from; s <= s_to; ++s) {
            const int64_t each = ((steps + s - 1) / s + kGemmStage - 1) / kGemmStage * kGemmStage;
            const int64_t splits = (steps + each - 1) / each;
            const int64_t groups = (tiles(kTileCols) * splits + 7) / 8 * 8 * row_tiles;
            double rounds = static_cast<double>((groups + 255) / 256);
            if (mb <= 4) rounds -= 0.28 * static_cast<double>(groups / 512);
            double us = rounds * static_cast<double>(each) * (0.184 + 0.0453 * mb);
            if (splits > 1) us += 2.0 * static_cast<double>(splits * part) / 3.25e6;
            if (best.mb == 0 || us < least) {
                least = us;
                best.mb = mb;
                best.steps = static_cast<int>(each);
                best.splits = static_cast<int>(splits);
                best.col_tiles = static_cast<uint32_t>(tiles(kTileCols));
                best.row_tiles = static_cast<uint32_t>(row_tiles);
            }
        }
    }
    return best;
}

// Bytes set aside for partial products at the end of the workspace.  Part of what kv_recompute_workspace_bytes has
// always promised, whatever the launches make of it: tiles of up to 128 x 128, K divided until some 256 (up to 128
// rows) or 512 workgroups exist, at least 256 of K per split, the largest of a layer's four groups of projections.
uint64_t partials_reserve(int64_t M, const int64_t* N, int n_mats, int64_t K) {
    const int64_t rows = M <= 32 ? 32 : (M <= 64 ? 64 : 128);
    int64_t tiles_n = 0, n_sum = 0;
    for (int j = 0; j < n_mats; ++j) {
        tiles_n += (N[j] + 127) / 128;
        n_sum += N[j];
    }
    const int64_t tiles = tiles_n * ((M + rows - 1) / rows);
    const int64_t groups = M <= 128 ? 256 : 512;
    int64_t want = (groups + tiles - 1) / tiles;
    want = std::min<int64_t>(want, std::min<int64_t>(kGemmMaxSplits, std::max<int64_t>(1, K / 256)));
    const int64_t slice = ((K + want - 1) / want + 31) / 32 * 32;
    const int64_t splits = (K + slice - 1) / slice;
    return splits > 1 ? static_cast<uint64_t>(splits) * M * n_sum * 4u : 0u;
}

uint64_t attention_share_bytes(const kv_shape_t& s, int64_t M) {
    return static_cast<uint64_t>(M) * s.n_q_heads * (s.head_dim + 2) * 4;
}

int attention_splits(const kv_shape_t& s, int64_t M, uint64_t room) {
    const int64_t pairs = static_cast<int64_t>(s.n_q_heads / s.n_kv_heads) * ((M + 31) / 32);
    return static_cast<int>(attention_shares(pairs, s.n_kv_heads, (s.n_tokens + 31) / 32,
                                             static_cast<int64_t>(room / attention_share_bytes(s, M)), kAttnWaves, kMaxSplits));
}

// Shares that the workspace has a place of their own for.  Part of what kv_recompute_workspace_bytes has always
// promised, whatever the launch makes of it (eight pairs per workgroup, 256 workgroups, at most 64 MiB).
int attention_reserve(const kv_shape_t& s, int64_t M) {
    const int64_t pairs = static_cast<int64_t>(s.n_q_heads / s.n_kv_heads) * ((M + 31) / 32);
    const int64_t base = (pairs + 7) / 8 * s.n_kv_heads;
    int64_t splits = 256 / base;
    splits = std::min<int64_t>(splits, (s.n_tokens + 31) / 32 / 4);
    splits = std::min<int64_t>(splits, 16);
    splits = std::min<int64_t>(splits, (64ll << 20) / static_cast<int64_t>(attention_share_bytes(s, M)));
    return static_cast<int>(std::max<int64_t>(splits, 1));
}

Plan plan_workspace(const kv_shape_t& s, const kv_layer_dims_t& d, int64_t M) {
    const uint64_t dq = static_cast<uint64_t>(s.n_q_heads) * s.head_dim;
    const uint64_t dkv = static_cast<uint64_t>(s.n_kv_heads) * s.head_dim;
    Plan p;
    uint64_t o = 0;
    p.xn = o;   o += align256(M * d.d_model * 2u);
    p.q32 = o;  o += align256(M * dq * 4u);
    p.k32 = o;  o += align256(M * dkv * 4u);
    p.v32 = o;  o += align256(M * dkv * 4u);
    p.q16 = o;  o += align256(M * dq * 2u);
    p.attn = o; o += align256(M * dq * 2u);
    p.x1 = o;   o += align256(M * d.d_model * 2u);
    p.gate = o; o += align256(M * static_cast<uint64_t>(d.d_ff) * 2u);
    p.up = o;   o += align256(M * static_cast<uint64_t>(d.d_ff) * 2u);
    p.part_o = o;
    const int reserved = attention_reserve(s, M);
    if (reserved > 1) {
        o += align256(static_cast<uint64_t>(reserved) * M * dq * 4u);
        o += align256(static_cast<uint64_t>(reserved) * M * s.n_q_heads * 8u);
    }
    // the library's own GEMM: partial products
    const int64_t n_qkv[3] = {static_cast<int64_t>(dq), static_cast<int64_t>(dkv), static_cast<int64_t>(dkv)};
    const int64_t n_o[1] = {d.d_model}, n_ff[2] = {d.d_ff, d.d_ff};
    const uint64_t part = std::max(
        std::max(partials_reserve(M, n_qkv, 3, d.d_model), partials_reserve(M, n_o, 1, static_cast<int64_t>(dq))),
        std::max(partials_reserve(M, n_ff, 2, d.d_model), partials_reserve(M, n_o, 1, d.d_ff)));
    o += align256(part);
    p.total = o;
    return p;
}

int check_layer(const kv_shape_t* shape, const kv_layer_dims_t* dims, int32_t n_missing) {
    if (int rc = check_shape(shape)) return rc;
    if (!dims) return fail(KV_EINVAL, "dims is NULL");
    if (!is_f16(*shape)) return fail(KV_ESHAPE, "recompute needs an fp16 cache format");
    if (shape->head_dim != 64 && shape->head_dim != 128)
        return fail(KV_ESHAPE, "recompute needs head_dim 64 or 128, got %d", shape->head_dim);
    if (dims->d_model <= 0 || dims->d_model % 8 || dims->d_ff <= 0 || dims->d_ff % 8)
        return fail(KV_ESHAPE, "d_model %d and d_ff %d must be positive multiples of 8", dims->d_model, dims->d_ff);
    if (!(dims->rope_base > 1.0f) || !(dims->rms_eps >= 0.0f))
        return fail(KV_EINVAL, "rope_base must exceed 1 and rms_eps must not be negative");
    const int32_t n_chunks = shape->n_tokens / shape->chunk_tokens;
    if (n_missing < 1 || n_missing > n_chunks)
        return fail(KV_EINVAL, "n_missing %d outside [1,%d]", n_missing, n_chunks);
    return KV_OK;
}

}  // namespace

// One projection of the block: row-major C[M][N] = A[M][K] * B[K][N] (+ Cin), fp16 operands.
struct GemmShape {
    int64_t M, N, K;
    bool out_f32, add;
    bool operator==(const GemmShape& o) const {
        return M == o.M && N == o.N && K == o.K && out_f32 == o.out_f32 && add == o.add;
    }
};

struct kv_recompute {
    void* lib = nullptr;
    rb_handle handle = nullptr;
    rb_destroy_fn destroy = nullptr;
    rb_set_stream_fn set_stream = nullptr;
    rb_gemm_ex_fn gemm_ex = nullptr;
    rb_get_solutions_fn get_solutions = nullptr;     // optional
    std::vector<std::pair<GemmShape, int>> tuned;    // shapes kv_recompute_tune examined: kernel, or -1 = standard
    FixedTile fixed;                                 // KVSWITCH_GEMM_TILE
};

namespace {

// The GEMM library's status for C[M][N] = A * B (+ Cin) with the standard choice of kernel
// (solution < 0) or a given one.  Column-major view: Cout^T [N][M] = B^T [N][K] * A^T [K][M].
int gemm_status(kv_recompute* rc, const GemmShape& g, const void* A, const void* B, const void* Cin, void* Cout,
                int solution) {
    const float alpha = 1.0f, beta = g.add ? 1.0f : 0.0f;
    const int ct = g.out_f32 ? kRbF32 : kRbF16;
    return rc->gemm_ex(rc->handle, kRbOpNone, kRbOpNone, static_cast<int>(g.N), static_cast<int>(g.M),
                       static_cast<int>(g.K), &alpha, B, kRbF16, static_cast<int>(g.N), A, kRbF16,
                       static_cast<int>(g.K), &beta, g.add ? Cin : Cout, ct, static_cast<int>(g.N), Cout, ct,
                       static_cast<int>(g.N), kRbF32, solution < 0 ? kRbAlgoStandard : kRbAlgoSolution,
                       solution < 0 ? 0 : solution, 0);
}

// Where a group's product may leave partial products: bytes [begin, end) of the workspace, free at that time.
struct Room {
    uint8_t* at;
    uint64_t bytes;
};
Room larger(Room a, Room b) { return a.bytes >= b.bytes ? a : b; }

// What became of a group's product: complete in the C matrices (splits == 1), or `splits` partial products per
// matrix, matrix after matrix ([splits][M][N[j]] binary32), from `part` on, for the caller's next kernel to add.
// gated: C[0] already holds silu(first) * second.
struct Product {
    int splits;
    const float* part;
    bool gated;
};

// kGate: two matrices of one width for a gated activation, in fragment order; where the kernel at hand can, it
// applies the activation itself (a layer of 2048 rows: 23 us of silu_mul_kernel and the way through memory).
enum class Out { kF32, kF16, kGate };

// The library's own GEMM (kv_gemm_kernels.hpp) over a group of weight matrices; A in fragment order.  Without
// `left` (one matrix only) a divided product is added here.
int own_gemm(hipStream_t st, FixedTile fixed, int64_t M, int64_t K, const void* A, const GemmGroup& grp, const void* Cin,
             Out out, Room room, Product* left, const char* what) {
    if (!left && (grp.n != 1 || out != Out::kF16)) return fail(KV_EINVAL, "GEMM (%s): added by its reader only", what);
    if (K % 8 || K < 8 || M < 1 || grp.n < 1 || grp.n > kGemmMaxMats || (Cin && grp.n != 1))
        return fail(KV_ESHAPE, "GEMM (%s): unsupported shape", what);
    for (int j = 0; j < grp.n; ++j)
        if (grp.N[j] % 8 || grp.N[j] < 8) return fail(KV_ESHAPE, "GEMM (%s) needs N a multiple of 8", what);
    OwnGemm h = own_gemm_plan(M, grp.N, grp.n, K, room.bytes, fixed);
    const bool gated = out == Out::kGate && !h.stream && h.splits == 1;
    if (gated) h.col_tiles = static_cast<uint32_t>((grp.N[0] + kTileCols / 2 - 1) / (kTileCols / 2));
    const int64_t cols = h.stream ? kStreamCols : kTileCols;
    GemmArgs g;
    g.A = static_cast<const _Float16*>(A);
    g.Cin = static_cast<const _Float16*>(Cin);
    g.part = reinterpret_cast<float*>(room.at);
    int32_t tiles = 0;
    uint64_t at = 0;
    for (int j = 0; j < kGemmMaxMats; ++j) {
        const int k = std::min(j, grp.n - 1);                 // unused entries repeat the last matrix and get no tile
        g.B[j] = static_cast<const _Float16*>(grp.B[k]);
        g.C[j] = grp.C[k];
        g.N[j] = static_cast<int32_t>(grp.N[k]);
        g.part_at[j] = at;
        if (j < grp.n) {
            tiles += static_cast<int32_t>((grp.N[j] + cols - 1) / cols);
            at += static_cast<uint64_t>(h.splits) * M * grp.N[j];
        }
        g.tile_end[j] = tiles;
    }
    if (gated) g.tile_end[0] = g.tile_end[1] = g.tile_end[2] = static_cast<int32_t>(h.col_tiles);
    g.M = static_cast<int32_t>(M);
    g.K = static_cast<int32_t>(K);
    g.steps = h.steps;
    g.splits = h.splits;
    g.out_f32 = out == Out::kF32 ? 1 : 0;
    g.out_fragments = out == Out::kGate && h.splits == 1 ? 1 : 0;
    if (h.stream) {
        const dim3 grid(h.col_tiles, static_cast<uint32_t>(h.splits));
        if (h.mb == 1) hipLaunchKernelGGL(gemm_stream_kernel<1>, grid, dim3(256), 0, st, g);
        else hipLaunchKernelGGL(gemm_stream_kernel<2>, grid, dim3(256), 0, st, g);
    } else {
        const int64_t blocks = (static_cast<int64_t>(h.col_tiles) * h.splits + 7) / 8 * 8 * h.row_tiles;
        if (blocks > 0x7fffffffLL) return fail(KV_ESHAPE, "GEMM (%s): grid exceeds 2^31 workgroups", what);
        const dim3 grid(static_cast<uint32_t>(blocks));
#define KV_TILE(MB)                                                                                       \
    do {                                                                                                  \
        if (gated) hipLaunchKernelGGL((gemm_tile_kernel<MB, true>), grid, dim3(256), 0, st, g);           \
        else hipLaunchKernelGGL((gemm_tile_kernel<MB, false>), grid, dim3(256), 0, st, g);                \
    } while (0)
        switch (h.mb) {
            case 3: KV_TILE(3); break;
            case 4: KV_TILE(4); break;
            case 5: KV_TILE(5); break;
            case 6: KV_TILE(6); break;
            case 7: KV_TILE(7); break;
            default: KV_TILE(8); break;
        }
#undef KV_TILE
    }
    if (left) *left = {h.splits, reinterpret_cast<const float*>(room.at), gated};
    else if (h.splits > 1)
        hipLaunchKernelGGL(gemm_reduce_kernel, dim3(static_cast<uint32_t>((M * grp.N[0] / 4 + 255) / 256)), dim3(256), 0, st, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(KV_EHIP, "GEMM launch (%s): %s", what, hipGetErrorString(e));
    return KV_OK;
}

// Whether the projections of M rows run on the library's own kernels.
bool own_projections(const kv_recompute* rc, int64_t M) { return M <= kOwnGemmRows || !rc->gemm_ex; }

// The projections of a group: one launch of the library's own kernel (A in fragment order), or one GEMM of the
// library per matrix (A and the results row-major).
int gemm(kv_recompute* rc, hipStream_t stream, int64_t M, int64_t K, const void* A, const GemmGroup& grp, const void* Cin,
         Out out, Room room, Product* left, const char* what) {
    if (own_projections(rc, M)) return own_gemm(stream, rc->fixed, M, K, A, grp, Cin, out, room, left, what);
    if (left) *left = {1, nullptr, false};
    for (int j = 0; j < grp.n; ++j) {
        const GemmShape g = {M, grp.N[j], K, out == Out::kF32, Cin != nullptr};
        int solution = -1;
        for (const auto& t : rc->tuned)
            if (t.first == g) solution = t.second;
        const int st = gemm_status(rc, g, A, grp.B[j], Cin, grp.C[j], solution);
        if (st != 0) return fail(KV_EHIP, "rocblas_gemm_ex (%s, matrix %d) failed with status %d", what, j, st);
    }
    return KV_OK;
}

// One projection of a block with its operands.
struct GemmJob {
    GemmShape g;
    const void* A;
    const void* B;
    const void* Cin;
    void* Cout;
};

// Picks the kernel of jobs[which] in two passes.  Pass 1 times every kernel the library lists
// back to back, which ranks them with the weights sitting in the last-level cache; pass 2 times
// the standard choice and the best few of pass 1 with cold weights, as a layer meets them: the
// other projections of the block (several hundred MB of weights) run in between.  The fastest of
// pass 2 is remembered if it beats the standard choice by more than 5 %.  Synchronises `st`.
int tune_gemm(kv_recompute* rc, const GemmJob* jobs, int n_jobs, int which, hipStream_t st, hipEvent_t e0,
              hipEvent_t e1, int* improved) {
    const GemmJob& job = jobs[which];
    const GemmShape& g = job.g;
    for (const auto& t : rc->tuned)
        if (t.first == g) return KV_OK;                       // already tuned
    const float alpha = 1.0f, beta = g.add ? 1.0f : 0.0f;
    const int ct = g.out_f32 ? kRbF32 : kRbF16;
    int n = 0;
    auto list = [&](int* out, int* count) {
        return rc->get_solutions(rc->handle, kRbOpNone, kRbOpNone, static_cast<int>(g.N), static_cast<int>(g.M),
                                 static_cast<int>(g.K), &alpha, job.B, kRbF16, static_cast<int>(g.N), job.A, kRbF16,
                                 static_cast<int>(g.K), &beta, g.add ? job.Cin : job.Cout, ct, static_cast<int>(g.N),
                                 job.Cout, ct, static_cast<int>(g.N), kRbF32, kRbAlgoSolution, 0, out, count);
    };
    if (list(nullptr, &n) != 0 || n <= 0) return KV_OK;      // nothing to choose from
    std::vector<int> sols(static_cast<size_t>(n));
    if (list(sols.data(), &n) != 0) return KV_OK;
    auto run = [&](int solution) { return gemm_status(rc, g, job.A, job.B, job.Cin, job.Cout, solution); };
    // elapsed time of `reps` runs; 1: this kernel cannot run the problem; -1: the runtime failed
    auto time_ms = [&](int solution, int reps, float* ms) -> int {
        hipError_t e = hipEventRecord(e0, st);
        for (int r = 0; r < reps && e == hipSuccess; ++r)
            if (run(solution) != 0) return 1;
        if (e == hipSuccess) e = hipEventRecord(e1, st);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(ms, e0, e1);
        return e == hipSuccess ? 0 : -1;
    };
    constexpr int kKeep = 6;
    int keep[kKeep];
    float keep_ms[kKeep];
    int n_keep = 0;
    for (int i = 0; i < n; ++i) {
        const int sol = sols[static_cast<size_t>(i)];
        float t = 0.0f;
        if (run(sol) != 0) continue;                          // warm-up, and "can it run"
        const int rc_t = time_ms(sol, 3, &t);
        if (rc_t < 0) return fail(KV_EHIP, "timing a GEMM kernel failed");
        if (rc_t != 0) continue;
        int at;                                               // insertion into the sorted short list
        if (n_keep < kKeep) at = n_keep++;
        else if (t < keep_ms[kKeep - 1]) at = kKeep - 1;
        else continue;
        while (at > 0 && keep_ms[at - 1] > t) {
            keep[at] = keep[at - 1];
            keep_ms[at] = keep_ms[at - 1];
            --at;
        }
        keep[at] = sol;
        keep_ms[at] = t;
    }
    auto cold_ms = [&](int solution, float* ms) -> int {
        *ms = 1e30f;
        for (int rep = 0; rep < 3; ++rep) {
            for (int k = 0; k < n_jobs; ++k)                  // push this job's weights out of the cache
                if (jobs[k].B != job.B) {
                    const GemmJob& o = jobs[k];
                    if (gemm_status(rc, o.g, o.A, o.B, o.Cin, o.Cout, -1) != 0) return -1;
                }
            float t = 0.0f;
            const int rc_t = time_ms(solution, 1, &t);
            if (rc_t != 0) return rc_t;
            if (t < *ms) *ms = t;
        }
        return 0;
    };
    float t_std = 0.0f;
    if (cold_ms(-1, &t_std) != 0) return fail(KV_EHIP, "timing the standard GEMM kernel failed");
    float t_best = t_std;
    int best = -1;
    for (int i = 0; i < n_keep; ++i) {
        float t = 0.0f;
        const int rc_t = cold_ms(keep[i], &t);
        if (rc_t < 0) return fail(KV_EHIP, "timing a GEMM kernel failed");
        if (rc_t == 0 && t < t_best) {
            t_best = t;
            best = keep[i];
        }
    }
    const bool better = best >= 0 && t_best < 0.95f * t_std;
    rc->tuned.emplace_back(g, better ? best : -1);            // examined: not timed again
    if (better) ++*improved;
    return KV_OK;
}

}  // namespace

extern "C" {

kv_recompute_t* kv_recompute_create(void) {
    clear_error();
    kv_recompute* rc = new (std::nothrow) kv_recompute();
    if (!rc) {
        fail(KV_ENOMEM, "out of host memory");
        return nullptr;
    }
    // KVSWITCH_GEMM_TILE=<row blocks>,<splits> fixes the launch shape of the library's own kernel above 64 rows
    if (const char* tile = getenv("KVSWITCH_GEMM_TILE")) {
        int blocks = 0, splits = 0, end = 0;
        if (sscanf(tile, "%d,%d%n", &blocks, &splits, &end) != 2 || tile[end] || blocks < 3 || blocks > 8 || splits < 1 ||
            splits > kGemmMaxSplits) {
            fail(KV_EINVAL, "KVSWITCH_GEMM_TILE=%s: want <row blocks 3..8>,<splits 1..%d>", tile, kGemmMaxSplits);
            delete rc;
            return nullptr;
        }
        rc->fixed = {blocks, splits};
    }
    // KVSWITCH_OWN_GEMM=1 in the environment keeps the GEMM library out: every projection then runs
    // on the library's own kernel, as it does where rocBLAS is not installed
    const char* own = getenv("KVSWITCH_OWN_GEMM");
    if (own && own[0] == '1') return rc;
    rc->lib = dlopen("librocblas.so.5", RTLD_NOW | RTLD_LOCAL);
    if (!rc->lib) rc->lib = dlopen("librocblas.so", RTLD_NOW | RTLD_LOCAL);
    if (!rc->lib) return rc;
    rb_create_fn create = reinterpret_cast<rb_create_fn>(dlsym(rc->lib, "rocblas_create_handle"));
    rc->destroy = reinterpret_cast<rb_destroy_fn>(dlsym(rc->lib, "rocblas_destroy_handle"));
    rc->set_stream = reinterpret_cast<rb_set_stream_fn>(dlsym(rc->lib, "rocblas_set_stream"));
    rc->gemm_ex = reinterpret_cast<rb_gemm_ex_fn>(dlsym(rc->lib, "rocblas_gemm_ex"));
    rc->get_solutions = reinterpret_cast<rb_get_solutions_fn>(dlsym(rc->lib, "rocblas_gemm_ex_get_solutions"));
    if (!create || !rc->destroy || !rc->set_stream || !rc->gemm_ex) {
        fail(KV_EHIP, "rocBLAS lacks a required entry point");
        dlclose(rc->lib);
        delete rc;
        return nullptr;
    }
    const int st = create(&rc->handle);
    if (st != 0 || !rc->handle) {
        fail(KV_EHIP, "rocblas_create_handle failed with status %d", st);
        dlclose(rc->lib);
        delete rc;
        return nullptr;
    }
    return rc;
}

void kv_recompute_destroy(kv_recompute_t* rc) {
    if (!rc) return;
    if (rc->handle && rc->destroy) rc->destroy(rc->handle);
    // the library stays loaded: other users in the process may share it
    delete rc;
}

uint64_t kv_recompute_workspace_bytes(const kv_shape_t* shape, const kv_layer_dims_t* dims, int32_t n_missing) {
    if (check_layer(shape, dims, n_missing) != KV_OK) return 0;
    return plan_workspace(*shape, *dims, static_cast<int64_t>(n_missing) * shape->chunk_tokens).total;
}

int32_t kv_recompute_tune(kv_recompute_t* rc, const kv_shape_t* shape, const kv_layer_dims_t* dims,
                          const kv_layer_weights_t* w, int32_t n_missing, void* workspace,
                          uint64_t workspace_bytes, void* stream, int32_t* n_improved) {
    if (n_improved) *n_improved = 0;
    if (!rc) return fail(KV_EINVAL, "handle is NULL");
    if (int st = check_layer(shape, dims, n_missing)) return st;
    if (!w || !w->wq || !w->wk || !w->wv || !w->wo || !w->w_gate || !w->w_up || !w->w_down)
        return fail(KV_EINVAL, "a weight pointer is NULL");
    if (!workspace || !aligned(workspace, 256)) return fail(KV_EINVAL, "workspace must be a 256-byte aligned device pointer");
    const kv_shape_t& s = *shape;
    const int64_t M = static_cast<int64_t>(n_missing) * s.chunk_tokens;
    const Plan p = plan_workspace(s, *dims, M);
    if (workspace_bytes < p.total)
        return fail(KV_ENOMEM, "workspace %llu bytes, %llu needed", static_cast<unsigned long long>(workspace_bytes),
                    static_cast<unsigned long long>(p.total));
    // projections of few rows run on the library's own kernel; nothing to choose there, nor without a GEMM library
    if (own_projections(rc, M) || !rc->get_solutions) return KV_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (rc->set_stream(rc->handle, st) != 0) return fail(KV_EHIP, "rocblas_set_stream failed");
    // operands of ordinary magnitude and varied bits in every buffer a GEMM reads
    const int64_t n_words = static_cast<int64_t>(p.total / 4);
    hipLaunchKernelGGL(fill_noise_kernel, dim3(static_cast<uint32_t>((n_words + 255) / 256)), dim3(256), 0, st,
                       static_cast<uint32_t*>(workspace), n_words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(KV_EHIP, "fill_noise_kernel launch: %s", hipGetErrorString(e));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    e = hipEventCreate(&e0);
    if (e == hipSuccess) e = hipEventCreate(&e1);
    if (e != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return fail(KV_EHIP, "hipEventCreate: %s", hipGetErrorString(e));
    }
    uint8_t* base = static_cast<uint8_t*>(workspace);
    void *xn = base + p.xn, *q32 = base + p.q32, *k32 = base + p.k32, *attn = base + p.attn, *x1 = base + p.x1,
         *gate = base + p.gate;
    const int64_t dq = static_cast<int64_t>(s.n_q_heads) * s.head_dim;
    const int64_t dkv = static_cast<int64_t>(s.n_kv_heads) * s.head_dim;
    void* up = base + p.up;
    void* v32 = base + p.v32;
    const GemmShape gq = {M, dq, dims->d_model, true, false}, gk = {M, dkv, dims->d_model, true, false};
    const GemmShape go = {M, dims->d_model, dq, false, true}, gg = {M, dims->d_ff, dims->d_model, false, false};
    const GemmShape gd = {M, dims->d_model, dims->d_ff, false, true};
    const GemmJob jobs[7] = {{gq, xn, w->wq, nullptr, q32}, {gk, xn, w->wk, nullptr, k32}, {gk, xn, w->wv, nullptr, v32},
                             {go, attn, w->wo, xn, x1},     {gg, xn, w->w_gate, nullptr, gate},
                             {gg, xn, w->w_up, nullptr, up}, {gd, gate, w->w_down, x1, xn}};
    int improved = 0;
    int rcode = KV_OK;
    for (int which : {0, 1, 3, 4, 6})
        if (!rcode) rcode = tune_gemm(rc, jobs, 7, which, st, e0, e1, &improved);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (n_improved) *n_improved = improved;
    return rcode;
}

int32_t kv_recompute_layer(kv_recompute_t* rc, const kv_shape_t* shape, const kv_layer_dims_t* dims,
                           const kv_layer_weights_t* w, int32_t layer, const int32_t* chunk_idx_dev,
                           int32_t n_missing, const void* x_in, void* kv, void* x_out, void* workspace,
                           uint64_t workspace_bytes, void* stream) {
    if (!rc) return fail(KV_EINVAL, "handle is NULL");
    if (int st = check_layer(shape, dims, n_missing)) return st;
    if (layer < 0 || layer >= shape->n_layers) return fail(KV_EINVAL, "layer %d outside [0,%d)", layer, shape->n_layers);
    if (!w || !w->w_norm1 || !w->wq || !w->wk || !w->wv || !w->wo || !w->w_norm2 || !w->w_gate || !w->w_up ||
        !w->w_down)
        return fail(KV_EINVAL, "a weight pointer is NULL");
    if (!chunk_idx_dev || !x_in || !kv || !x_out || !workspace) return fail(KV_EINVAL, "NULL device pointer");
    if (!aligned(x_in, 16) || !aligned(x_out, 16) || !aligned(kv, 16) || !aligned(workspace, 256) ||
        !aligned(chunk_idx_dev, 4))
        return fail(KV_EINVAL, "x_in/x_out/kv must be 16-byte aligned, workspace 256-byte aligned");
    const void* ws_ptrs[] = {w->w_norm1, w->wq, w->wk, w->wv, w->wo, w->w_norm2, w->w_gate, w->w_up, w->w_down};
    for (const void* p : ws_ptrs)
        if (!aligned(p, 16)) return fail(KV_EINVAL, "weights must be 16-byte aligned");
    const kv_shape_t& s = *shape;
    const int64_t M = static_cast<int64_t>(n_missing) * s.chunk_tokens;
    const Plan p = plan_workspace(s, *dims, M);
    if (workspace_bytes < p.total)
        return fail(KV_ENOMEM, "workspace %llu bytes, %llu needed", static_cast<unsigned long long>(workspace_bytes),
                    static_cast<unsigned long long>(p.total));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool own = own_projections(rc, M);
    if (!own && rc->set_stream(rc->handle, st) != 0)
        return fail(KV_EHIP, "rocblas_set_stream failed");

    uint8_t* base = static_cast<uint8_t*>(workspace);
    _Float16* xn = reinterpret_cast<_Float16*>(base + p.xn);
    float* q32 = reinterpret_cast<float*>(base + p.q32);
    float* k32 = reinterpret_cast<float*>(base + p.k32);
    float* v32 = reinterpret_cast<float*>(base + p.v32);
    _Float16* q16 = reinterpret_cast<_Float16*>(base + p.q16);
    _Float16* attn = reinterpret_cast<_Float16*>(base + p.attn);
    _Float16* x1 = reinterpret_cast<_Float16*>(base + p.x1);
    _Float16* gate = reinterpret_cast<_Float16*>(base + p.gate);
    _Float16* up = reinterpret_cast<_Float16*>(base + p.up);
    const _Float16* xin = static_cast<const _Float16*>(x_in);
    const int D = s.head_dim, Hq = s.n_q_heads, Hkv = s.n_kv_heads;
    const int64_t dq = static_cast<int64_t>(Hq) * D, dkv = static_cast<int64_t>(Hkv) * D;
    _Float16* k_plane = static_cast<_Float16*>(kv) + (static_cast<int64_t>(layer) * 2 + 0) * Hkv * s.n_tokens * D;
    _Float16* v_plane = k_plane + static_cast<int64_t>(Hkv) * s.n_tokens * D;
    const dim3 rows(static_cast<uint32_t>(M));
    const int32_t m32 = static_cast<int32_t>(M);
    auto room = [&](uint64_t begin, uint64_t end) { return Room{base + begin, end - begin}; };
    const _Float16 *norm1 = static_cast<const _Float16*>(w->w_norm1), *norm2 = static_cast<const _Float16*>(w->w_norm2);

    // 1. norm, q/k/v projections (binary32 results, rounded once after the rotation)
    if (own) hipLaunchKernelGGL((rmsnorm_kernel<false, true>), rows, dim3(256), 0, st, nullptr, 1, xin, nullptr, norm1, xn, m32, dims->d_model, dims->rms_eps);
    else hipLaunchKernelGGL((rmsnorm_kernel<false, false>), rows, dim3(256), 0, st, nullptr, 1, xin, nullptr, norm1, xn, m32, dims->d_model, dims->rms_eps);
    Product pr;
    const GemmGroup qkv = {3, {dq, dkv, dkv}, {w->wq, w->wk, w->wv}, {q32, k32, v32}};
    // (partial products behind q16, which the rotary kernel writes while it adds them)
    if (int e = gemm(rc, st, M, dims->d_model, xn, qkv, nullptr, Out::kF32, room(p.attn, p.total), &pr, "q | k | v")) return e;
    const float* q_src = pr.splits > 1 ? pr.part : q32;
    const float* k_src = pr.splits > 1 ? pr.part + pr.splits * M * dq : k32;
    const float* v_src = pr.splits > 1 ? pr.part + pr.splits * M * (dq + dkv) : v32;
    // 2. global position encoding; the recomputed K/V go to their places in the cache
    RopeTable tab;
    for (int i = 0; i < D / 2; ++i) tab.theta[i] = std::pow(static_cast<double>(dims->rope_base), -2.0 * i / D);
    hipLaunchKernelGGL(rope_scatter_kernel, dim3(static_cast<uint32_t>(M), 4), dim3(256), 0, st, q_src, k_src, v_src,
                       chunk_idx_dev, q16, k_plane, v_plane, tab, s.chunk_tokens, s.n_tokens, Hq, Hkv, D, pr.splits);
    // 3. causal attention over the recovered K/V
    AttnGeom g;
    g.M = static_cast<int32_t>(M);
    g.T = s.chunk_tokens;
    g.N = s.n_tokens;
    g.Hq = Hq;
    g.Hkv = Hkv;
    g.n_rb = static_cast<int32_t>((M + 31) / 32);
    g.pairs = (Hq / Hkv) * g.n_rb;
    g.fragments = own ? 1 : 0;
    g.scale_log2e = static_cast<float>(1.4426950408889634 / std::sqrt(static_cast<double>(D)));
    const bool few = few_pairs(g.pairs);
    // (the shares of a divided attention lie behind its output)
    const Room shares = room(p.x1, p.total);
    const int splits = attention_splits(s, M, shares.bytes);
    const int64_t pairs_all = M * Hq;
    float* part_o = splits > 1 ? reinterpret_cast<float*>(shares.at) : nullptr;
    float* part_ml = splits > 1 ? part_o + static_cast<int64_t>(splits) * pairs_all * D : nullptr;
    const dim3 agrid(static_cast<uint32_t>(few ? g.pairs : (g.pairs + kAttnWaves - 1) / kAttnWaves), static_cast<uint32_t>(Hkv),
                     static_cast<uint32_t>(splits));
#define KV_ATTENTION(KERNEL, DD, SPLIT)                                                                          \
    hipLaunchKernelGGL((KERNEL<DD, SPLIT>), agrid, dim3(64 * kAttnWaves), 0, st, q16, k_plane, v_plane, chunk_idx_dev, \
                       attn, g, part_o, part_ml)
#define KV_ATTENTION_D(DD)                                                                                       \
    do {                                                                                                         \
        if (few && splits > 1) KV_ATTENTION(recompute_attention_few_kernel, DD, true);                           \
        else if (few) KV_ATTENTION(recompute_attention_few_kernel, DD, false);                                   \
        else if (splits > 1) KV_ATTENTION(recompute_attention_kernel, DD, true);                                 \
        else KV_ATTENTION(recompute_attention_kernel, DD, false);                                                \
        if (splits > 1)                                                                                          \
            hipLaunchKernelGGL(attention_combine_kernel<DD>, dim3(static_cast<uint32_t>((pairs_all * (DD / 4) + 255) / 256)), \
                               dim3(256), 0, st, part_o, part_ml, attn, pairs_all, splits, Hq, g.fragments);     \
    } while (0)
    if (D == 64) KV_ATTENTION_D(64);
    else KV_ATTENTION_D(128);
#undef KV_ATTENTION_D
#undef KV_ATTENTION
    // 4. output projection + residual, feed-forward + residual
    const GemmGroup og = {1, {dims->d_model}, {w->wo}, {x1}};
    // (free but for xn and x1, which the norm writes while it adds the partial products)
    if (int e = gemm(rc, st, M, dq, attn, og, xin, Out::kF16, larger(room(p.q32, p.attn), room(p.gate, p.total)), &pr, "o")) return e;
    if (pr.splits > 1)
        hipLaunchKernelGGL((rmsnorm_kernel<true, true>), rows, dim3(256), 0, st, pr.part, pr.splits, xin, x1, norm2, xn, m32, dims->d_model, dims->rms_eps);
    else if (own)
        hipLaunchKernelGGL((rmsnorm_kernel<false, true>), rows, dim3(256), 0, st, nullptr, 1, x1, nullptr, norm2, xn, m32, dims->d_model, dims->rms_eps);
    else
        hipLaunchKernelGGL((rmsnorm_kernel<false, false>), rows, dim3(256), 0, st, nullptr, 1, x1, nullptr, norm2, xn, m32, dims->d_model, dims->rms_eps);
    const GemmGroup ff = {2, {dims->d_ff, dims->d_ff}, {w->w_gate, w->w_up}, {gate, up}};
    // (the activation goes to `gate`)
    if (int e = gemm(rc, st, M, dims->d_model, xn, ff, nullptr, own ? Out::kGate : Out::kF16,
                     larger(room(p.q32, p.x1), room(p.part_o, p.total)), &pr, "gate | up")) return e;
    const int64_t n8 = M * (dims->d_ff / 8);
    const float* no_part = nullptr;
    if (!pr.gated) hipLaunchKernelGGL(silu_mul_kernel, dim3(static_cast<uint32_t>((n8 + 255) / 256)), dim3(256), 0, st, gate, up,
                       gate, m32, dims->d_ff, pr.splits > 1 ? pr.part : no_part,
                       pr.splits > 1 ? pr.part + pr.splits * M * dims->d_ff : no_part, pr.splits, own ? 1 : 0);
    const GemmGroup down = {1, {dims->d_model}, {w->w_down}, {x_out}};
    if (int e = gemm(rc, st, M, dims->d_ff, gate, down, x1, Out::kF16, larger(room(p.xn, p.x1), room(p.up, p.total)), nullptr, "down")) return e;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(KV_EHIP, "recompute launch: %s", hipGetErrorString(e));
    return KV_OK;
}

}  // extern "C"
