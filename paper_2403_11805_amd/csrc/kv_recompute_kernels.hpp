// gfx950 kernels for the recompute of interleaved chunks (Sec. 3.3, "Making
// interleaved chunks recomputable"): the tokens of the missing chunks go through
// one Llama-style block; q and k are encoded with the tokens' GLOBAL positions,
// the recomputed K/V are inserted between the resident K/V of the cache, and the
// recomputed queries attend to the recovered K/V under a causal mask by global
// position.  The dense projections are in kv_gemm_kernels.hpp; everything else is here.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kv_gemm_kernels.hpp"
#include "kv_lane_ops.hpp"

namespace kvs {

typedef _Float16 rv8h_t __attribute__((ext_vector_type(8)));
typedef _Float16 rv4h_t __attribute__((ext_vector_type(4)));
typedef short rv4s_t __attribute__((ext_vector_type(4)));
typedef float rv16f_t __attribute__((ext_vector_type(16)));
typedef float rv4f_t __attribute__((ext_vector_type(4)));
typedef unsigned int ru4_t __attribute__((ext_vector_type(4)));

// Global position of recomputed token m: chunks of T tokens, chunk_idx ascending.
__device__ __forceinline__ int global_position(const int32_t* __restrict__ chunk_idx, int T, int m) {
    return chunk_idx[m / T] * T + m % T;
}

// xn[m][:] = x[m][:] / sqrt(mean(x[m][:]^2) + eps) * w[:]      (fp16 in/out, binary32 inside)
// FRAGMENTS: xn is written in the GEMM kernels' fragment order, otherwise row-major.  SUM: the row is first made
// from what a projection left as `splits` binary32 partial products [splits][M][d_model]:
// x[m][:] = fp16(part[0][m][:] + part[1][m][:] + ... + resid[m][:])  (split order, rounded once) is stored - it is
// the next residual - and normed; otherwise resid is the row and x is not written.  One workgroup per row: with a
// wavefront per row its loads come in eight dependent trips (16 rows of 4096: 9.3 us).  d_model % 8 == 0; up to
// kNormPieces * 2048 elements of a row stay in registers, a longer row is read (SUM: from x) a second time.
constexpr int kNormPieces = 2;
// Row of a workgroup that writes one row in fragment order: its pieces share 128-byte lines with those of the rows
// beside it, so the 32 rows of a block go to workgroups of one XCD (ids are dealt to the eight in turn), in whose
// L2 the lines fill up.  (2048 rows of 4096: 11.0 us, 18.3 with row = id.)
__device__ __forceinline__ int fragment_row(int id, int M) {
    if (id >= M / 256 * 256) return id;
    const int in = id & 255;
    return (id - in) + (in & 7) * 32 + (in >> 3);
}
template <bool SUM, bool FRAGMENTS>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ part, int32_t splits,
                                                      const _Float16* __restrict__ resid, _Float16* __restrict__ x,
                                                      const _Float16* __restrict__ w, _Float16* __restrict__ xn,
                                                      int32_t M, int32_t d_model, float eps) {
    __shared__ float wave_ss[4];
    const int m = FRAGMENTS ? fragment_row(blockIdx.x, M) : static_cast<int>(blockIdx.x);
    const int pieces = d_model / 8;
    const rv8h_t* res = reinterpret_cast<const rv8h_t*>(resid + static_cast<int64_t>(m) * d_model);
    rv8h_t* row = SUM ? reinterpret_cast<rv8h_t*>(x + static_cast<int64_t>(m) * d_model) : nullptr;
    auto piece = [&](int p) __attribute__((always_inline)) {
        rv8h_t v = res[p];
        if constexpr (SUM) {
            const int64_t plane4 = static_cast<int64_t>(M) * d_model / 4;
            const rv4f_t* src = reinterpret_cast<const rv4f_t*>(part) + static_cast<int64_t>(m) * d_model / 4 + 2 * p;
            rv4f_t lo = src[0], hi = src[1];
#pragma unroll 4
            for (int sp = 1; sp < splits; ++sp) {
                lo += src[sp * plane4];
                hi += src[sp * plane4 + 1];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = static_cast<_Float16>(lo[k] + static_cast<float>(v[k]));
                v[k + 4] = static_cast<_Float16>(hi[k] + static_cast<float>(v[k + 4]));
            }
            row[p] = v;                              // read again below, if at all, by this same thread
        }
        return v;
    };
    float ss = 0.0f;
    auto square = [&](const rv8h_t& v) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 8; ++k) ss += static_cast<float>(v[k]) * static_cast<float>(v[k]);
    };
    rv8h_t held[kNormPieces];
#pragma unroll
    for (int i = 0; i < kNormPieces; ++i) {
        const int p = i * 256 + static_cast<int>(threadIdx.x);
        if (p < pieces) {
            held[i] = piece(p);
            square(held[i]);
        }
    }
    for (int p = kNormPieces * 256 + threadIdx.x; p < pieces; p += 256) square(piece(p));
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
    ss = xhalf_sum(ss);
    if ((threadIdx.x & 63) == 0) wave_ss[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = (wave_ss[0] + wave_ss[1]) + (wave_ss[2] + wave_ss[3]);
    const float r = 1.0f / sqrtf(ss / static_cast<float>(d_model) + eps);
    const rv8h_t* wp = reinterpret_cast<const rv8h_t*>(w);
    auto scaled = [&](int p, const rv8h_t& v) __attribute__((always_inline)) {
        const rv8h_t g = wp[p];
        rv8h_t o;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            o[k] = static_cast<_Float16>(static_cast<float>(v[k]) * r * static_cast<float>(g[k]));
        const int64_t at = FRAGMENTS ? fragment_at(m, 8 * p, M, d_model) : static_cast<int64_t>(m) * d_model + 8 * p;
        *reinterpret_cast<rv8h_t*>(xn + at) = o;
    };
#pragma unroll
    for (int i = 0; i < kNormPieces; ++i) {
        const int p = i * 256 + static_cast<int>(threadIdx.x);
        if (p < pieces) scaled(p, held[i]);
    }
    for (int p = kNormPieces * 256 + threadIdx.x; p < pieces; p += 256) scaled(p, SUM ? row[p] : res[p]);
}

// Rotary angles: theta[i] = base^(-2i/D) in double, computed on the host.
struct RopeTable {
    double theta[128];      // head_dim / 2 <= 128
};

// Four workgroups per recomputed token m at global position p (grid (M, 4): q, k and the two halves of v;
// with some hundred tokens a workgroup per token leaves half the CUs idle and walks its row in eight
// dependent trips to memory):
//   q16[m][h][:]            = rope(q32[m][h][:], p)                       (fp16)
//   K plane [g][p][:]       = rope(k32[m][g][:], p)   V plane [g][p][:] = v32[m][g][:]   (fp16 cache)
// The pair (i, i + D/2) is rotated by p * theta[i]; sine and cosine are taken in
// double (positions reach tens of thousands of radians).  q32, k32 and v32 may be `splits` partial
// products each ([splits][M][heads * D], M = the grid size), which are added in split order as they
// are read.
__global__ __launch_bounds__(256) void rope_scatter_kernel(const float* __restrict__ q32,
                                                           const float* __restrict__ k32,
                                                           const float* __restrict__ v32,
                                                           const int32_t* __restrict__ chunk_idx,
                                                           _Float16* __restrict__ q16,
                                                           _Float16* __restrict__ k_plane,
                                                           _Float16* __restrict__ v_plane,
                                                           RopeTable tab, int32_t T, int32_t N,
                                                           int32_t Hq, int32_t Hkv, int32_t D, int32_t splits) {
    __shared__ __attribute__((aligned(16))) float cs[2][128];
    const int64_t plane_q = static_cast<int64_t>(gridDim.x) * Hq * D, plane_kv = static_cast<int64_t>(gridDim.x) * Hkv * D;
    // four adjacent elements, the partial products added in split order
    auto sum4 = [&](const float* at, int64_t plane) {
        rv4f_t a = *reinterpret_cast<const rv4f_t*>(at);
#pragma unroll 4
        for (int sp = 1; sp < splits; ++sp) a += *reinterpret_cast<const rv4f_t*>(at + sp * plane);
        return a;
    };
    auto to_half4 = [](rv4f_t a) {
        return rv4h_t{static_cast<_Float16>(a[0]), static_cast<_Float16>(a[1]), static_cast<_Float16>(a[2]),
                      static_cast<_Float16>(a[3])};
    };
    const int m = blockIdx.x;
    const int part = blockIdx.y;            // 0: q, 1: k, 2 and 3: the halves of v (uniform per workgroup)
    const int p = global_position(chunk_idx, T, m);
    const int half = D / 2, half4 = D / 8;
    if (part >= 2) {
        const float* vrow = v32 + static_cast<int64_t>(m) * Hkv * D;
        const int n4 = Hkv * D / 4, mid = n4 / 2;
        for (int e = (part == 2 ? 0 : mid) + threadIdx.x; e < (part == 2 ? mid : n4); e += blockDim.x) {
            const int g = e / (D / 4), d = (e % (D / 4)) * 4;
            *reinterpret_cast<rv4h_t*>(v_plane + (static_cast<int64_t>(g) * N + p) * D + d) = to_half4(sum4(vrow + e * 4, plane_kv));
        }
        return;
    }
    for (int i = threadIdx.x; i < half; i += blockDim.x) {
        double s, c;
        sincos(static_cast<double>(p) * tab.theta[i], &s, &c);
        cs[0][i] = static_cast<float>(c);
        cs[1][i] = static_cast<float>(s);
    }
    __syncthreads();
    if (part == 0) {
        const float* qrow = q32 + static_cast<int64_t>(m) * Hq * D;
        _Float16* qout = q16 + static_cast<int64_t>(m) * Hq * D;
        for (int e = threadIdx.x; e < Hq * half4; e += blockDim.x) {
            const int h = e / half4, i = (e % half4) * 4;
            const rv4f_t a = sum4(qrow + h * D + i, plane_q), b = sum4(qrow + h * D + i + half, plane_q);
            const rv4f_t c = *reinterpret_cast<const rv4f_t*>(&cs[0][i]), s = *reinterpret_cast<const rv4f_t*>(&cs[1][i]);
            *reinterpret_cast<rv4h_t*>(qout + h * D + i) = to_half4(a * c - b * s);
            *reinterpret_cast<rv4h_t*>(qout + h * D + i + half) = to_half4(b * c + a * s);
        }
        return;
    }
    const float* krow = k32 + static_cast<int64_t>(m) * Hkv * D;
    for (int e = threadIdx.x; e < Hkv * half4; e += blockDim.x) {
        const int g = e / half4, i = (e % half4) * 4;
        const rv4f_t a = sum4(krow + g * D + i, plane_kv), b = sum4(krow + g * D + i + half, plane_kv);
        const rv4f_t c = *reinterpret_cast<const rv4f_t*>(&cs[0][i]), s = *reinterpret_cast<const rv4f_t*>(&cs[1][i]);
        _Float16* dst = k_plane + (static_cast<int64_t>(g) * N + p) * D;
        *reinterpret_cast<rv4h_t*>(dst + i) = to_half4(a * c - b * s);
        *reinterpret_cast<rv4h_t*>(dst + i + half) = to_half4(b * c + a * s);
    }
}

// act[M][d_ff] = silu(gate) * up, 8 elements per thread (d_ff % 8 == 0); the three have one layout, row-major or
// fragment order, and act may be gate (each thread reads its elements before it writes them).
// With `part_gate` the two operands are instead made from projections left as `splits` binary32 partial products
// [splits][M][d_ff]: gate = fp16(sum in split order), up likewise; with `fragments` act is then written in fragment
// order, the threads following it (32 rows side by side: a workgroup writes consecutive pieces, and the eight pieces
// it reads of a row fill a 256-byte line).
__global__ __launch_bounds__(256) void silu_mul_kernel(const _Float16* gate, const _Float16* up, _Float16* act, int32_t M,
                                                       int32_t d_ff, const float* __restrict__ part_gate,
                                                       const float* __restrict__ part_up, int32_t splits, int32_t fragments) {
    const int64_t id = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t n8 = static_cast<int64_t>(M) * (d_ff / 8);
    if (id >= n8) return;
    int64_t i = id;
    if (part_gate && fragments) {                    // the row-major piece that belongs to piece `id` of the result
        const int per_row = d_ff / 8;
        const int b = static_cast<int>(id / (32 * per_row));
        const int in = static_cast<int>(id - static_cast<int64_t>(b) * 32 * per_row);
        const int rows = min(32, M - 32 * b);
        const int k8 = in / rows;
        i = static_cast<int64_t>(32 * b + in - k8 * rows) * per_row + k8;
    }
    rv8h_t g, u;
    if (part_gate) {
        const rv4f_t* pg = reinterpret_cast<const rv4f_t*>(part_gate);
        const rv4f_t* pu = reinterpret_cast<const rv4f_t*>(part_up);
        rv4f_t g0 = pg[2 * i], g1 = pg[2 * i + 1], u0 = pu[2 * i], u1 = pu[2 * i + 1];
        for (int sp = 1; sp < splits; ++sp) {
            const int64_t at = (sp * n8 + i) * 2;
            g0 += pg[at]; g1 += pg[at + 1];
            u0 += pu[at]; u1 += pu[at + 1];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            g[k] = static_cast<_Float16>(g0[k]); g[k + 4] = static_cast<_Float16>(g1[k]);
            u[k] = static_cast<_Float16>(u0[k]); u[k + 4] = static_cast<_Float16>(u1[k]);
        }
    } else {
        g = reinterpret_cast<const rv8h_t*>(gate)[i];
        u = reinterpret_cast<const rv8h_t*>(up)[i];
    }
    rv8h_t o;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const float x = static_cast<float>(g[k]);
        o[k] = static_cast<_Float16>(x / (1.0f + __expf(-x)) * static_cast<float>(u[k]));
    }
    reinterpret_cast<rv8h_t*>(act)[id] = o;
}

// Stand-in operands for timing GEMM kernels: every 16-bit half is a binary16 of magnitude
// [0.5, 1) with a hashed mantissa and sign (timings with constant operands mislead: they draw
// less power, and the clock, hence the ranking of kernels, follows the power).
__global__ __launch_bounds__(256) void fill_noise_kernel(uint32_t* __restrict__ words, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t h = static_cast<uint32_t>(i) * 2654435761u + 0x9e3779b9u;
    h ^= h >> 15; h *= 0x85ebca6bu; h ^= h >> 13; h *= 0xc2b2ae35u; h ^= h >> 16;
    words[i] = (h & 0x83ff83ffu) | 0x38003800u;
}

struct AttnGeom {
    int32_t M;        // recomputed tokens
    int32_t T;        // chunk tokens
    int32_t N;        // cache tokens
    int32_t Hq, Hkv;
    int32_t n_rb;     // ceil(M / 32): blocks of 32 query rows
    int32_t pairs;    // (Hq / Hkv) * n_rb: (row block, query head) pairs per kv head
    int32_t fragments; // 1: the output is written in the GEMM kernels' fragment order
    float scale_log2e;
};

constexpr float kRefSlack = 8.0f;
// Piece c of row r of a K tile in LDS sits at c ^ attn_swz(r); a token row of a V tile there takes attn_v_pitch halves.
template <int D>
__device__ __forceinline__ int attn_swz(int r) { return D == 64 ? (r >> 1) & 7 : r & 15; }
constexpr int attn_v_pitch(int D) { return D + 16; }

// One tile of 32 tokens from `t * 32` on, in LDS, against a wavefront's 32 query rows: folds it into the outputs o_acc,
// the references m_run and the denominators l_run.
template <int D>
__device__ __forceinline__ void attention_tile(const ru4_t* ktile, const _Float16* vt, const rv8h_t (&qreg)[D / 16],
                                               rv16f_t (&o_acc)[D / 32], float& m_run, float& l_run, int t, int min_pos,
                                               int pos, float scale_log2e, int lane) {
    constexpr int KS = D / 16, DB = D / 32, kRowPieces = D / 8, kVPitch = attn_v_pitch(D);
    const int lrow = lane & 31, half = lane >> 5;
    rv8h_t kreg[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        kreg[ks] = __builtin_bit_cast(rv8h_t, ktile[lrow * kRowPieces + ((2 * ks + half) ^ attn_swz<D>(lrow))]);
    rv16f_t acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kreg[ks], qreg[ks], acc, 0, 0, 0);
    // acc[v]: token t*32 + 8*(v/4) + 4*half + v%4 against this lane's query row
    // maxima on the raw logits (the scale is positive), the scale folded into the exponent
    const bool masked = t * 32 + 31 > min_pos;     // wave-uniform
    float mloc = -INFINITY;
    if (masked) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int tk = t * 32 + 8 * (v / 4) + 4 * half + (v % 4);
            if (tk > pos) acc[v] = -INFINITY;
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) mloc = fmaxf(mloc, acc[v]);
    // The reference of a row moves only when some row of the wavefront has left it by more than 2^8: until
    // then its probabilities are up to 2^8 instead of 1, which costs fp16 no precision, and the 64
    // accumulators are not touched.
    const float m_tile = xhalf_max(mloc) * scale_log2e;
    if (__any(m_tile > m_run + kRefSlack)) {        // wave-uniform
        const float m_new = fmaxf(m_run, m_tile);
        const float alpha = __builtin_amdgcn_exp2f(m_run - (m_new == -INFINITY ? 0.0f : m_new));
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) o_acc[b][v] *= alpha;
    }
    const float m_safe = (m_run == -INFINITY) ? 0.0f : m_run;
    float psum = 0.0f;
    rv8h_t pb[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v], scale_log2e, -m_safe));
        psum += pv;
        pb[v / 8][v % 8] = static_cast<_Float16>(pv);
    }
    l_run += xhalf_sum(psum);
    // contraction slot (half, e) of step st holds token 16*st + 4*half + e (e < 4) or
    // 16*st + 8 + 4*half + e - 4: the order of acc[8*st .. 8*st+7] on the P side
#pragma unroll
    for (int b = 0; b < DB; ++b) {
        // this lane's piece of the block of its 16-lane group: token row (lane % 16) / 4, channels
        // 32 b + 16 (group % 2) + 4 (lane % 4) ..; the read returns channel 32 b + lane % 32
        const _Float16* vblk = &vt[((lane & 15) >> 2) * kVPitch + 32 * b + 16 * ((lane >> 4) & 1) + 4 * (lane & 3)];
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const rv4s_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) rv4s_t*)(vblk + (16 * st + 4 * half) * kVPitch));
            const rv4s_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) rv4s_t*)(vblk + (16 * st + 8 + 4 * half) * kVPitch));
            const rv4h_t lo_h = __builtin_bit_cast(rv4h_t, lo), hi_h = __builtin_bit_cast(rv4h_t, hi);
            const rv8h_t a = {lo_h[0], lo_h[1], lo_h[2], lo_h[3], hi_h[0], hi_h[1], hi_h[2], hi_h[3]};
            o_acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, pb[st], o_acc[b], 0, 0, 0);
        }
    }
}

// Causal attention of the recomputed queries over the recovered K/V of one layer.
// A wavefront owns one (block of 32 query rows, query head) pair: S^T = K_tile Q^T
// with mfma_f32_32x32x16_f16 (a lane owns one query row and 16 of the tile's 32
// tokens), online softmax per row, O^T += V_tile^T P^T with the probabilities
// rounded to fp16 as the B operand straight from the registers (the contraction
// index is permuted the same way on both operands).  The four wavefronts of a
// workgroup take four consecutive pairs of ONE kv head, so K and V tiles are
// fetched once per workgroup (coalesced 16-byte loads, two tiles ahead) and shared
// through LDS: K with its row pieces permuted by the row number, V in cache order and
// read through the LDS transpose read.  Tokens after a row's global position
// are masked; a wavefront skips the tiles that lie entirely behind its last row,
// and the output accumulators are rescaled only when some row's maximum has moved by more than 2^kRefSlack.
constexpr int kAttnWaves = 4;
constexpr int kMaxSplits = 16;     // workgroups that may share the key range of a row block
// Measured, 32 heads of 128 over 4096 tokens (kernel alone): 2048 rows anywhere in the cache 123 us, 304 rows 45 us,
// 16 rows 7.8 to 13.5 by where they lie (at token 2928 13.5; 12.6 in recompute_attention_few_kernel, which takes them).  Eight
// wavefronts per workgroup, loads behind branches - the compiler then waits for every load in flight before it parks a
// tile, so that the second tile ahead never is -, accumulators in AGPRs and rescaled whenever a maximum moved: 160, 57 and
// 13.5 us.  The unequal key ranges of a causal mask leave the chip waiting
// for the longest workgroup: two or three small workgroups per CU, a long one beside a short one, and shares of
// each workgroup's own range even them out.  A tile costs a wavefront some 1100 cycles of MFMA and VALU work and 16
// KiB of LDS reads.  (second __launch_bounds__ argument: accumulators stay in VGPRs)
//
// SPLIT: with few recomputed rows there are too few workgroups to fill the chip and each walks
// the whole key range alone.  The key tiles that a workgroup's last row sees are then divided evenly among
// gridDim.z workgroups; each writes the unnormalised output, running maximum and denominator of its
// share (part_o [split][row][head][D], part_ml [split][row][head][2], binary32) and
// attention_combine_kernel merges the shares in a fixed order.
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kAttnWaves, 2) void recompute_attention_kernel(
    const _Float16* __restrict__ q16, const _Float16* __restrict__ k_plane,
    const _Float16* __restrict__ v_plane, const int32_t* __restrict__ chunk_idx,
    _Float16* __restrict__ out, AttnGeom g, float* __restrict__ part_o, float* __restrict__ part_ml) {
    constexpr int KS = D / 16;
    constexpr int DB = D / 32;                      // 32-wide blocks of the head dimension
    constexpr int kRowPieces = D / 8;
    constexpr int kThreads = 64 * kAttnWaves;
    constexpr int kTilePieces = 32 * kRowPieces;    // 16-byte pieces of a K (or V) tile
    constexpr int kPer = (kTilePieces + kThreads - 1) / kThreads;
    __shared__ ru4_t ktile[2][32 * kRowPieces];
    // V stays in cache order, [token][channel] with 32 bytes of padding per token row; the
    // operand of O^T += V^T P^T (a channel per lane, tokens along the contraction) is taken with
    // the LDS transpose read (ds_read_b64_tr_b16): the 16 lanes of a group hand in the sixteen
    // 8-byte pieces of a 4-token x 16-channel block, row by row, and lane i receives the four
    // tokens of channel i.  The padding puts the four token rows of a block on different banks.
    constexpr int kVPitch = attn_v_pitch(D);
    __shared__ __align__(16) _Float16 vt[2][32 * kVPitch];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lrow = lane & 31, half = lane >> 5;
    // Workgroups are handed to the 8 XCDs in turn (linear id modulo 8), each with an L2 of its
    // own: the workgroups of one kv head are placed on one XCD, so that its K/V planes are
    // fetched into one L2 only.  Needs n_kv_heads % 8 == 0, otherwise the plain order is kept.
    const int gx = static_cast<int>(gridDim.x), nz = SPLIT ? static_cast<int>(gridDim.z) : 1;
    int kvh = blockIdx.y, bxi = blockIdx.x, share = SPLIT ? static_cast<int>(blockIdx.z) : 0;
    bool ascending = false;
    if (g.Hkv % 8 == 0) {
        const int lin = (static_cast<int>(SPLIT ? blockIdx.z : 0) * g.Hkv + static_cast<int>(blockIdx.y)) * gx + static_cast<int>(blockIdx.x);
        const int per_xcd = lin >> 3;                       // position among this XCD's workgroups
        const int nth = per_xcd / (gx * nz), in = per_xcd - nth * (gx * nz);
        kvh = (lin & 7) + 8 * nth;
        share = in / gx;
        bxi = in - share * gx;
        // Workgroups with the longest key ranges are dispatched first; where an XCD's 32 CUs take a second round of
        // them beside the first, the other way round, so that a CU holds a long and a short one.
        ascending = (nth * gx * nz / 32) & 1;
    }
    const int per = g.Hq / g.Hkv;
    const int bx = ascending ? bxi : gx - 1 - bxi;
    const int pair = bx * kAttnWaves + wave;
    const bool valid = pair < g.pairs;
    const int head = kvh * per + (valid ? pair % per : 0);
    const int rb = valid ? pair / per : 0;
    const int m = rb * 32 + lrow;
    const bool ok = valid && m < g.M;
    const int pos = ok ? global_position(chunk_idx, g.T, m) : -1;
    // rows ascend in position: first and last row of this wavefront, last row of the workgroup
    const int min_pos = valid ? global_position(chunk_idx, g.T, rb * 32) : -1;
    const int max_pos = valid ? global_position(chunk_idx, g.T, min(rb * 32 + 31, g.M - 1)) : -1;
    const int rb_hi = min(bx * kAttnWaves + kAttnWaves - 1, g.pairs - 1) / per;
    const int wg_max_pos = global_position(chunk_idx, g.T, min(rb_hi * 32 + 31, g.M - 1));
    // key tiles [t_first, n_tiles) of this workgroup
    const int all_tiles = wg_max_pos / 32 + 1, per_share = (all_tiles + nz - 1) / nz;
    const int t_first = share * per_share;
    const int n_tiles = min(all_tiles, t_first + per_share);

    rv8h_t qreg[KS];
    {
        const _Float16* qp = q16 + (static_cast<int64_t>(ok ? m : 0) * g.Hq + head) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            rv8h_t v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (ok) v = *reinterpret_cast<const rv8h_t*>(qp + ks * 16);
            qreg[ks] = v;
        }
    }
    const ru4_t* kbase = reinterpret_cast<const ru4_t*>(k_plane + static_cast<int64_t>(kvh) * g.N * D);
    const ru4_t* vbase = reinterpret_cast<const ru4_t*>(v_plane + static_cast<int64_t>(kvh) * g.N * D);
    // tiles in flight: set 0 holds even tiles, set 1 odd ones (loads are issued two tiles ahead)
    ru4_t kst[2][kPer], vst[2][kPer];
    auto fetch = [&](int set, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = min(i * kThreads + tid, kTilePieces - 1);       // surplus threads repeat the last piece
            // tokens behind the workgroup's last row are masked, but their V is still multiplied, by a probability of
            // 0, and the cache may hold anything there (NaN too): the last row's token takes their place
            const int token = min(t * 32 + p / kRowPieces, wg_max_pos);
            const int64_t src = static_cast<int64_t>(token) * kRowPieces + p % kRowPieces;
            kst[set][i] = kbase[src];
            vst[set][i] = vbase[src];
        }
    };
    auto park = [&](int set, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = min(i * kThreads + tid, kTilePieces - 1);
            const int r = p / kRowPieces, c = p % kRowPieces;
            ktile[buf][r * kRowPieces + (c ^ attn_swz<D>(r))] = kst[set][i];
            *reinterpret_cast<ru4_t*>(&vt[buf][r * kVPitch + c * 8]) = vst[set][i];
        }
    };

    rv16f_t o_acc[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) o_acc[b] = rv16f_t{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    float m_run = -INFINITY, l_run = 0.0f;

    // one tile: the arithmetic on LDS buffer `buf` (tile t), then tile t + 1 (fetched two steps ago
    // into the other register set) goes to the other buffer and its set fetches tile t + 3
    auto step = [&](int t, int buf) __attribute__((always_inline)) {
        if (t < n_tiles && t * 32 <= max_pos) {     // wave-uniform
            attention_tile<D>(ktile[buf], vt[buf], qreg, o_acc, m_run, l_run, t, min_pos, pos, g.scale_log2e, lane);
        }
        // (both unconditional, beyond the last tile with that tile again: behind a branch the compiler waits for every
        // load in flight before it parks)
        park(buf ^ 1, buf ^ 1);
        fetch(buf ^ 1, min(t + 3, n_tiles - 1));
        __syncthreads();
    };
    if (t_first < n_tiles) {            // uniform per workgroup
        fetch(0, t_first);
        park(0, 0);
        fetch(1, min(t_first + 1, n_tiles - 1));
        fetch(0, min(t_first + 2, n_tiles - 1));
        __syncthreads();
        for (int t = t_first; t < n_tiles; t += 2) {
            step(t, 0);
            step(t + 1, 1);                 // beyond the last tile: nothing but the barrier (see above)
        }
    }
    if constexpr (SPLIT) {
        if (ok) {
            // the share of this workgroup: an empty one has m = -inf, l = 0 and zeros
            const int64_t row = (static_cast<int64_t>(share) * g.M + m) * g.Hq + head;
            if (half == 0) {
                part_ml[row * 2] = m_run;
                part_ml[row * 2 + 1] = l_run;
            }
            float* dst = part_o + row * D;
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const rv4f_t o4 = {o_acc[b][4 * j], o_acc[b][4 * j + 1], o_acc[b][4 * j + 2], o_acc[b][4 * j + 3]};
                    *reinterpret_cast<rv4f_t*>(dst + 32 * b + 8 * j + 4 * half) = o4;
                }
        }
        return;
    }
    if (ok) {
        // o_acc[b][v]: head dimension 32*b + 8*(v/4) + 4*half + v%4 of this lane's query row
        const float inv = 1.0f / l_run;         // a row sees at least its own token
        // row-major, or in fragment order: rows side by side, eight head dimensions per piece
        const int piece = g.fragments ? min(32, g.M - rb * 32) * 8 : 8;
        _Float16* dst = out + (g.fragments ? fragment_at(m, head * D, g.M, g.Hq * D) : (static_cast<int64_t>(m) * g.Hq + head) * D);
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                rv4h_t o4;
#pragma unroll
                for (int k = 0; k < 4; ++k) o4[k] = static_cast<_Float16>(o_acc[b][4 * j + k] * inv);
                *reinterpret_cast<rv4h_t*>(dst + (4 * b + j) * piece + 4 * half) = o4;
            }
    }
}

// The same with few (row block, query head) pairs per kv head, where most wavefronts of the kernel above would have no
// pair of their own: the four wavefronts of a workgroup share ONE pair and take the key tiles of the workgroup's share in
// turn, each through a tile of LDS of its own and with no barrier before their outputs meet at the end.  A tile of a lone
// wavefront is a serial chain of LDS reads, MFMAs and exponentials, some 3000 cycles, and four chains run side by side.  The
// kernel alone in a trace, 32 heads of 128 over 4096 tokens, the other kernel / this one: 16 rows 13.5 / 12.6 us (48 MB of
// keys and values at 3.8 TB/s), 32 rows 14.9 / 13.4, 48 rows 16.0 / 15.9, 64 rows 19.0 / 18.7; longer contexts gain more (the rule and
// layers: few_pairs).
// Grid (pairs, kv heads, shares).
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * kAttnWaves, 2) void recompute_attention_few_kernel(
    const _Float16* __restrict__ q16, const _Float16* __restrict__ k_plane,
    const _Float16* __restrict__ v_plane, const int32_t* __restrict__ chunk_idx,
    _Float16* __restrict__ out, AttnGeom g, float* __restrict__ part_o, float* __restrict__ part_ml) {
    constexpr int KS = D / 16;
    constexpr int DB = D / 32;
    constexpr int kRowPieces = D / 8;
    constexpr int kVPitch = attn_v_pitch(D);
    constexpr int kPer = 32 * kRowPieces / 64;      // 16-byte pieces of a K (or V) tile per lane
    constexpr int kVPieces = kVPitch / 8;
    static_assert(32 * (kRowPieces + kVPieces) >= 8 * D, "a wavefront's tile holds its outputs");
    __shared__ ru4_t tile_lds[kAttnWaves][32 * (kRowPieces + kVPieces)];
    __shared__ float ml_lds[kAttnWaves][2][32];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int lrow = lane & 31, half = lane >> 5;
    // (the workgroups of a kv head on one XCD, the longest key ranges first: as above)
    const int gx = static_cast<int>(gridDim.x), nz = SPLIT ? static_cast<int>(gridDim.z) : 1;
    int kvh = blockIdx.y, bxi = blockIdx.x, share = SPLIT ? static_cast<int>(blockIdx.z) : 0;
    if (g.Hkv % 8 == 0) {
        const int lin = (share * g.Hkv + static_cast<int>(blockIdx.y)) * gx + static_cast<int>(blockIdx.x);
        const int per_xcd = lin >> 3, nth = per_xcd / (gx * nz), in = per_xcd - nth * (gx * nz);
        kvh = (lin & 7) + 8 * nth;
        share = in / gx;
        bxi = in - share * gx;
    }
    const int per = g.Hq / g.Hkv;
    const int pair = gx - 1 - bxi;
    const int head = kvh * per + pair % per, rb = pair / per;
    const int m = rb * 32 + lrow;
    const bool ok = m < g.M;
    const int pos = ok ? global_position(chunk_idx, g.T, m) : -1;
    const int min_pos = global_position(chunk_idx, g.T, rb * 32);
    const int max_pos = global_position(chunk_idx, g.T, min(rb * 32 + 31, g.M - 1));
    const int all_tiles = max_pos / 32 + 1, per_share = (all_tiles + nz - 1) / nz;
    const int t_first = share * per_share, n_tiles = min(all_tiles, t_first + per_share);

    const ru4_t* kbase = reinterpret_cast<const ru4_t*>(k_plane + static_cast<int64_t>(kvh) * g.N * D);
    const ru4_t* vbase = reinterpret_cast<const ru4_t*>(v_plane + static_cast<int64_t>(kvh) * g.N * D);
    ru4_t kst[kPer], vst[kPer];
    auto fetch = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = i * 64 + lane;
            const int token = min(t * 32 + p / kRowPieces, max_pos);     // (what lies behind the last row may be anything)
            const int64_t src = static_cast<int64_t>(token) * kRowPieces + p % kRowPieces;
            kst[i] = kbase[src];
            vst[i] = vbase[src];
        }
    };
    ru4_t* ktile = tile_lds[wave];
    _Float16* vt = reinterpret_cast<_Float16*>(ktile + 32 * kRowPieces);
    auto park = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int p = i * 64 + lane, r = p / kRowPieces, c = p % kRowPieces;
            ktile[r * kRowPieces + (c ^ attn_swz<D>(r))] = kst[i];
            *reinterpret_cast<ru4_t*>(vt + r * kVPitch + c * 8) = vst[i];
        }
    };
    auto in_order = [] {                            // LDS accesses of this wavefront on either side stay there
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    fetch(min(t_first + wave, all_tiles - 1));
    rv8h_t qreg[KS];
    {
        const _Float16* qp = q16 + (static_cast<int64_t>(ok ? m : 0) * g.Hq + head) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            rv8h_t v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (ok) v = *reinterpret_cast<const rv8h_t*>(qp + ks * 16);
            qreg[ks] = v;
        }
    }
    rv16f_t o_acc[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b) o_acc[b] = rv16f_t{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    float m_run = -INFINITY, l_run = 0.0f;
    for (int t = t_first + wave; t < n_tiles; t += kAttnWaves) {
        park();
        fetch(min(t + kAttnWaves, n_tiles - 1));
        in_order();
        attention_tile<D>(ktile, vt, qreg, o_acc, m_run, l_run, t, min_pos, pos, g.scale_log2e, lane);
        in_order();
    }
    // the four outputs against one reference per row, added in the order of the wavefronts
    if (half == 0) {
        ml_lds[wave][0][lrow] = m_run;
        ml_lds[wave][1][lrow] = l_run;
    }
    __syncthreads();
    float m_all = -INFINITY, l_all = 0.0f;
#pragma unroll
    for (int k = 0; k < kAttnWaves; ++k) m_all = fmaxf(m_all, ml_lds[k][0][lrow]);
#pragma unroll
    for (int k = 0; k < kAttnWaves; ++k) {
        const float mk = ml_lds[k][0][lrow];
        l_all += mk == -INFINITY ? 0.0f : ml_lds[k][1][lrow] * __builtin_amdgcn_exp2f(mk - m_all);
    }
    const float f = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_run - m_all);
    rv4f_t* mine = reinterpret_cast<rv4f_t*>(ktile);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            mine[(b * 4 + j) * 64 + lane] = rv4f_t{o_acc[b][4 * j], o_acc[b][4 * j + 1], o_acc[b][4 * j + 2], o_acc[b][4 * j + 3]} * f;
    __syncthreads();
    // wavefront b finishes channels 32 b ..: 32 b + 8 j + 4 half .. of this lane's row
    if (wave >= DB || !ok) return;
    rv4f_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        o[j] = reinterpret_cast<const rv4f_t*>(tile_lds[0])[(wave * 4 + j) * 64 + lane];
#pragma unroll
        for (int k = 1; k < kAttnWaves; ++k) o[j] += reinterpret_cast<const rv4f_t*>(tile_lds[k])[(wave * 4 + j) * 64 + lane];
    }
    if constexpr (SPLIT) {
        const int64_t row = (static_cast<int64_t>(share) * g.M + m) * g.Hq + head;
        if (wave == 0 && half == 0) {
            part_ml[row * 2] = m_all;
            part_ml[row * 2 + 1] = l_all;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<rv4f_t*>(part_o + row * D + 32 * wave + 8 * j + 4 * half) = o[j];
    } else {
        const float inv = 1.0f / l_all;             // a row sees at least its own token
        const int piece = g.fragments ? min(32, g.M - rb * 32) * 8 : 8;
        _Float16* dst = out + (g.fragments ? fragment_at(m, head * D, g.M, g.Hq * D) : (static_cast<int64_t>(m) * g.Hq + head) * D);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            rv4h_t o4;
#pragma unroll
            for (int k = 0; k < 4; ++k) o4[k] = static_cast<_Float16>(o[j][k] * inv);
            *reinterpret_cast<rv4h_t*>(dst + (4 * wave + j) * piece + 4 * half) = o4;
        }
    }
}

// Merges the shares of a split attention: out[row][head][:] = sum_s w_s o_s / sum_s w_s l_s with
// w_s = 2^(m_s - max_s m_s), shares taken in ascending order.  One thread per 4 channels.
template <int D>
__global__ __launch_bounds__(256) void attention_combine_kernel(const float* __restrict__ part_o,
                                                                const float* __restrict__ part_ml,
                                                                _Float16* __restrict__ out, int64_t rows,
                                                                int n_splits, int Hq, int fragments) {
    constexpr int kQuads = D / 4;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= rows * kQuads) return;
    const int64_t row = i / kQuads;
    const int quad = static_cast<int>(i % kQuads);
    // all loads of a pass are issued before its arithmetic: up to kMaxSplits shares, a clamped
    // index for the surplus slots (their weight is forced to zero)
    float m_s[kMaxSplits], l_s[kMaxSplits];
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {
        const int sc = s < n_splits ? s : n_splits - 1;
        const float2 ml = *reinterpret_cast<const float2*>(part_ml + (sc * rows + row) * 2);
        m_s[s] = s < n_splits ? ml.x : -INFINITY;
        l_s[s] = ml.y;
    }
    float m_all = -INFINITY;
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) m_all = fmaxf(m_all, m_s[s]);
    float l_all = 0.0f;
    rv4f_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s0 = 0; s0 < kMaxSplits; s0 += 4) {
        if (s0 >= n_splits) break;
        rv4f_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int sc = s0 + k < n_splits ? s0 + k : n_splits - 1;
            o[k] = *reinterpret_cast<const rv4f_t*>(part_o + (sc * rows + row) * D + quad * 4);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // an empty share (m = -inf) and a surplus slot weigh nothing
            const float w = m_s[s0 + k] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m_s[s0 + k] - m_all);
            l_all += w * l_s[s0 + k];
            acc += o[k] * w;
        }
    }
    const float inv = 1.0f / l_all;                     // a row sees at least its own token
    rv4h_t o4;
#pragma unroll
    for (int k = 0; k < 4; ++k) o4[k] = static_cast<_Float16>(acc[k] * inv);
    int64_t at = row * D + quad * 4;
    if (fragments) {
        const int m = static_cast<int>(row / Hq), head = static_cast<int>(row - static_cast<int64_t>(m) * Hq);
        at = fragment_at(m, head * D + quad * 4, static_cast<int>(rows / Hq), Hq * D);
    }
    *reinterpret_cast<rv4h_t*>(out + at) = o4;
}

}  // namespace kvs
