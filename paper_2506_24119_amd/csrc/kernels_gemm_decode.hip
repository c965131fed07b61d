// Projections of at most 128 rows (a decode step, small prefills, the last rows of a prefill):
// out[m][n] = sum_k A[m][k] * W[n][k], K % 128 == 0.
//
// Bound by the stream over W, on the small shapes by what comes before and after it (a launch is 3 to 10 us), and from about 100
// rows on by the power limit: matrix instructions and operand loads overlap in time but not in energy (a loop of 12
// instructions and 7 KB of loads from L2 takes 556 cycles with zeros for operands, as long as the longer of the two alone, and
// 810 with random ones, their sum).  So every operand is moved once.  The four waves of a workgroup share its 32 * NT weight
// rows and split K: every wave multiplies all rows of the batch with all weight rows of the workgroup over every fourth k step.  A
// fragment of either operand is then used by one wave only: both go from memory straight to operand registers, P k steps ahead, without
// LDS and without a barrier until the end, when the waves' partial tiles meet in LDS, in wave order.  Waves that own weight rows
// and share the activations through LDS (gemm_stream_kernel) read every activation fragment four times from LDS, wait for each other
// every 128 k, and need up to four times the split of K over workgroups (blockIdx.y) to fill the chip with a narrow projection, whose
// partial sums the next kernel reads.  The activations come in the order of the operand (act_frag()): in rows a load touches 32
// half-used lines (128 rows, gate/up of the 4B shape 52 us against 27).
// Loads past a wave's last k step and of weight tiles past the last one carry an offset beyond the buffer's size: the memory
// pipeline drops them, and no branch stands between the loads.
// One launch by itself, us, gemm_stream_kernel / this, at 3, 32 and 128 rows (4B and 7B shapes at 128: bound by power; inside a step,
// between events, q/k/v, O and down of the 4B shape at 128 rows 15.7 / 16.8, 13.5 / 13.7 and 20.4 / 21.6, which fewer partial sums make up for):
//   0.6B  q/k/v 4.3 / 4.1, 4.8 / 4.5, 7.7 / 6.2; O 4.0 / 3.2, 4.5 / 3.5, 6.9 / 4.8; gate/up 7.2 / 5.3, 7.7 / 5.9, 13.4 / 8.5;
//         down 4.2 / 3.5, 4.7 / 4.0, 7.3 / 5.7; LM head 59 / 48, 71 / 56 (5.5 to 6.4 TB/s)
//   4B    q/k/v 8.5 / 7.1, 9.8 / 7.8, 12.7 / 12.1; O 5.7 / 5.5, 6.4 / 6.1, 10.0 / 9.4;
//         down 9.8 / 9.8, 10.6 / 10.6, 17.0 / 16.1; LM head 124 / 116, 149 / 141
//   7B    q/k/v 8.5 / 7.5, 9.6 / 8.4, 12.8 / 12.8; O 7.3 / 6.3, 8.4 / 7.1, 12.2 / 10.8
#include <algorithm>

#include "spiral_internal.h"
#include "mfma_ops.h"

namespace spiral {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr uint32_t kDropped = 0x80000000u;       // an offset no buffer below holds
constexpr int kBufferBytes = 0x7FFFFFFF;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kBufferBytes, 0x00027000);
}

// M32: batch tiles of 32 rows; NT: 32-row weight tiles of a workgroup; P: k steps of 16 whose operands a wave holds or waits for;
// WAVES: waves per SIMD that the registers are bounded for.  FRAG: weights in fragment order (already halves), else rows as given.
template <int M32, int NT, int EPI, bool FRAG, int P, int WAVES>
__global__ __launch_bounds__(256, WAVES) void gemm_decode_kernel(GemmArgs g) {
    constexpr int TROW = 144;                        // bytes of a staged row: 32 floats + 16 pad
    constexpr int TILE = 32 * TROW;
    constexpr int UNITS = M32 * NT;                  // 32 x 32 tiles of the product
    constexpr int GROUP = UNITS < 4 ? UNITS : 4;     // tiles that meet in LDS at a time
    constexpr int PASSES = (UNITS + 3) / 4;
    constexpr int BUF = 4 * GROUP * TILE;
    __shared__ __attribute__((aligned(16))) char lds[(PASSES > 1 ? 2 : 1) * BUF];
    __shared__ float s_val[EPI == EPI_SAMPLE ? NT * M32 * 32 : 1];
    __shared__ int s_idx[EPI == EPI_SAMPLE ? NT * M32 * 32 : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int K = g.K, tile0 = blockIdx.x * NT, split = blockIdx.y;
    const int tiles = EPI == EPI_SWIGLU ? (g.N + 15) >> 4 : (g.N + 31) >> 5;

    // ---- this wave's k steps: kb, kb + 4, ... (at least two: a split has 128 k)
    const int steps = K >> 4;
    const int first = (int)((long long)steps * split / g.splits), end = (int)((long long)steps * (split + 1) / g.splits);
    const int kb = first + wave, n = (end - kb + 3) >> 2;

    __amdgpu_buffer_rsrc_t wbuf;
    uint32_t woff[NT];
    const uint16_t* wrow[NT];
    if (FRAG) {
        wbuf = buffer_of((const uint16_t*)g.wf + frag_block(tile0, kb, K));
#pragma unroll
        for (int j = 0; j < NT; ++j) woff[j] = tile0 + j < tiles ? (uint32_t)j * (uint32_t)K * 64u + (uint32_t)lane * 16u : kDropped;
    } else {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const uint16_t* base;
            int row;
            if (EPI == EPI_SWIGLU) {
                row = min((tile0 + j) * 16 + (l32 & 15), g.N - 1);
                base = (const uint16_t*)(l32 < 16 ? g.w[0] : g.w[1]);
            } else {
                const int c = min((tile0 + j) * 32 + l32, g.N - 1);
                if (c < g.rows[0]) { base = (const uint16_t*)g.w[0]; row = c; }
                else if (c < g.rows[0] + g.rows[1]) { base = (const uint16_t*)g.w[1]; row = c - g.rows[0]; }
                else { base = (const uint16_t*)g.w[2]; row = c - g.rows[0] - g.rows[1]; }
            }
            wrow[j] = base + (size_t)row * K + (size_t)kb * 16 + lh * 8;
        }
    }
    // activations in rows or in fragment order; lanes of rows past the last read the last row, row tiles past the last the last tile
    const __amdgpu_buffer_rsrc_t abuf = buffer_of(g.A);
    uint32_t aoff[M32], astep[M32];
#pragma unroll
    for (int t = 0; t < M32; ++t) {
        const int m0 = min(t * 32, (g.M - 1) & ~31), rows = min(32, g.M - m0), r = min(l32, rows - 1);
        aoff[t] = g.a_frag ? (uint32_t)m0 * K * 2u + (uint32_t)(lh * rows + r) * 16u : (uint32_t)(m0 + r) * K * 2u + (uint32_t)lh * 16u;
        astep[t] = g.a_frag ? (uint32_t)rows * 32u : 32u;
    }

    f32x16 acc[M32][NT];
#pragma unroll
    for (int t = 0; t < M32; ++t)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[t][j][q] = 0.f;

    constexpr int LOADS = M32 + NT;
    u32x4 wf[P][NT], af[P][M32];
    auto load = [&](int slot, int i, int x) {        // operand x (the weight tiles, then the activations) of k step kb + 4 i
        const uint32_t dropped = i < n ? 0u : kDropped;
        if (x >= NT) af[slot][x - NT] = __builtin_amdgcn_raw_buffer_load_b128(abuf, aoff[x - NT] | dropped, (kb + 4 * i) * astep[x - NT], 0);
        else if (FRAG) wf[slot][x] = __builtin_amdgcn_raw_buffer_load_b128(wbuf, woff[x] | dropped, i * 4096, 2);      // non-temporal
        else wf[slot][x] = *(const u32x4*)(wrow[x] + (size_t)(i < n ? i : n - 1) * 64);
    };
    // one k step; the slot before it, which the step before has used up, is refilled between the matrix instructions
    auto step = [&](int slot, int i, bool loads) {
        const int prev = (slot + P - 1) % P;
        u32x4 w[NT];
        int l = 0;
#pragma unroll
        for (int x = 0; x < UNITS; ++x) {
            if (loads)
#pragma unroll
                for (; l < LOADS && l * UNITS <= x * LOADS; ++l) load(prev, i, l);
            if (x < NT) w[x] = FRAG ? wf[slot][x] : prep_w(wf[slot][x]);
            acc[x / NT][x % NT] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w[x % NT]), __builtin_bit_cast(f16x8, af[slot][x / NT]),
                                                                         acc[x / NT][x % NT], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (loads)
#pragma unroll
            for (; l < LOADS; ++l) load(prev, i, l);
    };
#pragma unroll
    for (int i = 0; i < P - 1; ++i)
#pragma unroll
        for (int x = 0; x < LOADS; ++x) load(i, i, x);
    int i0 = 0;
    for (; i0 + P <= n; i0 += P) {
#pragma unroll
        for (int i = 0; i < P; ++i) step(i, i0 + i + P - 1, true);
    }
#pragma unroll
    for (int i = 0; i < P - 1; ++i)
        if (i0 + i < n) step(i, 0, false);

    // ---- the waves' partial tiles.  A lane holds batch row l32 and, in registers 4b .. 4b+3, the weight rows 8b + 4*lh .. +3; the
    //      staged rows are batch rows.  Up to four tiles at a time, each added and written by one wave (two tiles by two waves
    //      each, a single one by all four), in the order of the waves that made the parts.
    bool bad = false;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        char* buf = lds + (ps & 1) * BUF;
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            if (ps * 4 + u >= UNITS) continue;
            char* dst = buf + (wave * GROUP + u) * TILE + l32 * TROW + lh * 16;
            const f32x16& c = acc[(ps * 4 + u) / NT][(ps * 4 + u) % NT];
#pragma unroll
            for (int b = 0; b < 4; ++b) *(float4*)(dst + b * 32) = make_float4(c[4 * b], c[4 * b + 1], c[4 * b + 2], c[4 * b + 3]);
        }
        __syncthreads();
        if (EPI == EPI_SWIGLU) {
            // columns 0..15 of a staged row are gate, 16..31 the same ffn columns' up values: a lane has 8 of one row
            const int u = ps * 4 + wave, m = u / NT * 32 + l32, f = (tile0 + u % NT) * 16 + lh * 8;
            if (u >= UNITS || m >= g.M || f >= g.N) continue;
            const char* p = buf + wave * TILE + l32 * TROW + lh * 32;
            float gate[8], up[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float4 a = *(const float4*)(p + h * 16), b = *(const float4*)(p + 64 + h * 16);
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float4 oa = *(const float4*)(p + w * GROUP * TILE + h * 16), ob = *(const float4*)(p + w * GROUP * TILE + 64 + h * 16);
                    a.x += oa.x; a.y += oa.y; a.z += oa.z; a.w += oa.w;
                    b.x += ob.x; b.y += ob.y; b.z += ob.z; b.w += ob.w;
                }
                gate[4 * h] = a.x; gate[4 * h + 1] = a.y; gate[4 * h + 2] = a.z; gate[4 * h + 3] = a.w;
                up[4 * h] = b.x; up[4 * h + 1] = b.y; up[4 * h + 2] = b.z; up[4 * h + 3] = b.w;
            }
            uint32_t o[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                o[q] = (uint32_t)f32_to_act16_noting(silu_f(gate[2 * q]) * up[2 * q], bad) |
                       ((uint32_t)f32_to_act16_noting(silu_f(gate[2 * q + 1]) * up[2 * q + 1], bad) << 16);
            *(u32x4*)((uint16_t*)g.out + (g.out_frag ? act_frag(m, f, g.M, g.N) : (size_t)m * g.N + f)) = u32x4{o[0], o[1], o[2], o[3]};
        } else {
            constexpr int SHARE = UNITS == 1 ? 4 : UNITS == 2 ? 2 : 1;      // waves to a tile
            const int lu = wave / SHARE, u = ps * 4 + lu, j = u % NT, m0 = u / NT * 32;
            if (u >= UNITS) continue;
            const int rr = lane >> 3, cg = lane & 7;
            const int c = (tile0 + j) * 32 + cg * 4;
#pragma unroll
            for (int q0 = 0; q0 < 4 / SHARE; ++q0) {
                const int q = SHARE == 1 ? q0 : q0 * SHARE + wave % SHARE;        // rows 8 q .. 8 q + 7, 8 lanes of 16 bytes to a row
                if (m0 + 8 * q >= g.M) continue;
                const int m = m0 + rr + 8 * q;
                const char* p = buf + lu * TILE + (rr + 8 * q) * TROW + cg * 16;
                float4 v = *(const float4*)p;
#pragma unroll
                for (int w = 1; w < 4; ++w) {
                    const float4 o = *(const float4*)(p + w * GROUP * TILE);
                    v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w;
                }
                if (EPI == EPI_STORE_F32) {
                    if (m < g.M && c < g.N) *(float4*)((float*)g.out + ((size_t)split * g.M + m) * g.N + c) = v;
                } else {
                    // score = logit / T + noise (the sampler's own expression); the best of the tile's columns per batch row
                    const float T = g.s_temperature;
                    const uint64_t key = (T > 0.f && m < g.M) ? g.s_keys[m] : 0ull;
                    const float x[4] = {v.x, v.y, v.z, v.w};
                    const uint64_t at = noise_at(key, c);
                    float bv = -INFINITY;
                    int bi = 0x7FFFFFFF;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float sc = T > 0.f ? x[e] / T + gumbel_noise(at + (uint64_t)e * kNoiseStep) : x[e];
                        if (c + e < g.N && better(sc, c + e, bv, bi)) { bv = sc; bi = c + e; }
                    }
#pragma unroll
                    for (int s = 1; s < 8; s <<= 1) {
                        const float ov = __shfl_xor(bv, s, 64);
                        const int oi = __shfl_xor(bi, s, 64);
                        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
                    }
                    if (cg == 0) { s_val[j * M32 * 32 + m] = bv; s_idx[j * M32 * 32 + m] = bi; }
                }
            }
        }
    }
    if (EPI == EPI_SWIGLU) report_saturation(g.sat_count, bad);
    if (EPI == EPI_SAMPLE) {                         // the workgroup's best per batch row; a second kernel picks among workgroups
        __syncthreads();
        const int m = threadIdx.x;
        if (m < g.M) {
            float bv = s_val[m];
            int bi = s_idx[m];
#pragma unroll
            for (int j = 1; j < NT; ++j)
                if (better(s_val[j * M32 * 32 + m], s_idx[j * M32 * 32 + m], bv, bi)) { bv = s_val[j * M32 * 32 + m]; bi = s_idx[j * M32 * 32 + m]; }
            g.s_part[(size_t)m * g.s_tiles + blockIdx.x] = make_float2(bv, __int_as_float(bi));
        }
    }
}

template <int M32, int NT, int EPI, int P, int WAVES>
static hipError_t launch_one(const GemmArgs& a, hipStream_t s) {
    const int tiles = EPI == EPI_SWIGLU ? (a.N + 15) / 16 : (a.N + 31) / 32, wgs = (tiles + NT - 1) / NT;
    if (EPI == EPI_SAMPLE && (!a.wf || !a.s_part || a.splits != 1 || a.s_tiles != wgs)) return hipErrorInvalidValue;
    if (a.wf) hipLaunchKernelGGL((gemm_decode_kernel<M32, NT, EPI, true, P, WAVES>), dim3(wgs, a.splits), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((gemm_decode_kernel<M32, NT, EPI, EPI == EPI_SAMPLE, P, WAVES>), dim3(wgs, a.splits), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Steps in flight: as far as the registers of two waves per SIMD go up to 64 rows.  Beyond, where the activations, which come from
// L2, are more than the weights, which come from memory, more loads of both kinds in flight make them slower (loads alone, 3 KB of
// weights and 4 KB of activations a step, 203 x 4 waves x 40 steps: 26 us with three steps in flight, 34 with seven): gate/up of
// the 4B shape, 128 rows, 2 / 3 / 4 / 8 slots 32.9 / 29.3 / 29.7 / 30.9 us.  More than four accumulator tiles take the registers of
// one wave per SIMD, and their staging the LDS of one workgroup.
template <int EPI, int M32>
static hipError_t launch_tiles(const GemmArgs& a, int nt, hipStream_t s) {
    if (nt == 1) return launch_one<M32, 1, EPI, M32 <= 2 ? 8 : 4, 2>(a, s);
    if (nt == 2) return launch_one<M32, 2, EPI, M32 <= 2 ? 6 : 3, M32 <= 2 ? 2 : 1>(a, s);
    return launch_one<M32, 3, EPI, M32 == 1 ? 6 : M32 == 2 ? 4 : 3, M32 == 1 ? 2 : 1>(a, s);
}

// Which projections launch_gemm_decode takes (A in act_frag() order or in rows).  All row counts up to 128 take the same kernel and
// the same K splits, so that a sequence's sums do not follow from how many others are in the call; repacked and row-major weights too, so
// that they give the same bits.  Row-major weights draw the lines for large projections, which is where they are slow here: a load has 32
// bytes of each of 32 rows, the four waves share every line of 128 bytes, and the lines in flight leave the L1 before the last of them has come.
// Gate/up of more than 512 tiles (two to a compute unit) stays on the streaming kernel.  Streaming kernel -> this, us between events at
// 1, 32 and 128 rows, d 2,048: 512 tiles row-major 23.6 -> 23.7, 25.7 -> 23.6, 32.4 -> 30.8, repacked 17.1 -> 16.8, 18.9 -> 17.1,
// 26.4 -> 24.1; 688 tiles row-major 24.7 -> 31.6, 25.7 -> 32.3, 34.0 -> 37.8, repacked 20.4 -> 20.6, 21.0 -> 20.5, 28.3 -> 28.6; the 4B
// shape's 608 tiles row-major 31.8 -> 39.2, 34.8 -> 41.6, 41.7 -> 51.8, repacked 21.4 -> 21.9, 23.1 -> 22.3, 32.5 -> 33.9.
// The others stay there from 64 MB of weights on: the 7B shape's down (136 MB) row-major 31.8 -> 47.4, 35.1 -> 49.8, 44.0 -> 58.0, repacked 27.0
// -> 26.2, 28.8 -> 28, 37.0 -> 37; 2,560 x 12,288 (63 MB) row-major 19.8 -> 20.9, 21.0 -> 21.9, 26.4 -> 30.8, repacked 16.1 -> 14.9,
// 18.6 -> 16.2, 23.4 -> 24.7.
// The LM head does up to 32 rows, a small one (2^25 weights) up to 128, with logits and with the sampler's winners alike, as both have to
// come from the same sums: they are rounded by nothing that follows.  Its limit is the second round of workgroups: above 64 rows they have one wave
// a SIMD, whose noise runs under nothing else, so 256 of 64 columns (16,384) are one round.  One layer and head, sampled, streaming kernel -> this, 128 rows:
// 8,192 x 1024 72 -> 63, x 2560 100 -> 84, x 3584 120 -> 101, 40 rows x 2560 68 -> 62, but 32,768 x 1024 76 -> 83, 65,536 x 128 60 -> 90.  The line at
// eight columns to a k is short of that: heads of 10,240 to 16,384 columns at K = 1024, 8,192 and 16,384 at 512, which stay on the streaming kernel,
// would gain as well (winners of 128 rows 31 -> 22 and 26 -> 19 us, logits 18 -> 13..15 and 12..13 -> 8..11; 24,576 at 1024 32 -> 40 and 20 -> 18).  Streaming kernel
// -> this, us, 8,192 columns at 33, 64 and 128 rows: K = 1024 8.7 -> 5.2, 9.0 -> 5.6, 13.5 -> 7.9; 2560 17 -> 9.6, 19 -> 10.2, 30.5 -> 15.1; 3584 23 -> 12.4,
// 25 -> 14.3, 41 -> 21.4.  One layer and a row-major head of 151,936, 1, 16 and 32 rows: 0.6B 119 -> 107, 129 -> 115, 136 -> 122; 4B 252 -> 229,
// 267 -> 264, 283 -> 287; 7B 337 -> 333, 364 -> 370, 382 -> 402.
bool gemm_decode_takes(int M, int N, int K, int epilogue, bool head) {
    if (M < 1 || M > 128 || (K & 127) || (N & 15)) return false;
    if (epilogue == EPI_SWIGLU) return (N + 15) / 16 <= 512;
    if (head) return M <= 32 || (N <= 8LL * K && (long long)N * K <= 1 << 25);
    return (long long)N * K <= 1 << 25;
}

// Whether the down projection reads act_frag() order: whenever it comes here, as gate/up (d columns in, ffn out) writes that order from
// either kernel.  (In rows the 7B shape's down took, at 32, 64 and 128 rows, 34, 45 and 64 us for 29, 30 and 37 on the streaming kernel.)
bool gemm_mlp_in_frag(int M, int d, int ffn) {
    return gemm_decode_takes(M, d, ffn, EPI_STORE_F32, false) && (d & 127) == 0;
}

// K splits of a projection, by its shape alone: the least sum of rounds over the 256 compute units x k steps of a wave x operand blocks
// of a step at 32 rows, and of the partial sums (in the same unit, 0.1 us, N / 640 each), over 1 to 3 weight tiles a workgroup.  Against
// a sweep of 1 to 4 tiles x 1 to 16 splits on the q/k/v, O and down projections of three shapes at 3, 32, 64 and 128 rows the
// choice is within 4 % of the fastest launch.
int gemm_decode_splits(int N, int K, int most) {
    const int tiles = (N + 31) / 32, steps = K / 16;
    most = std::max(1, std::min(most, K / 128));
    float best = 1e30f;
    int splits = 1;
    for (int t = 1; t <= 3; ++t)
        for (int s = 1; s <= most; ++s) {
            const int rounds = ((tiles + t - 1) / t * s + 255) / 256;
            const float cost = (float)(rounds * ((steps + 4 * s - 1) / (4 * s)) * (t + 1)) + (float)s * N / 640.f;
            if (cost < best) { best = cost; splits = s; }
        }
    return splits;
}

// Weight tiles of a workgroup: the least of the same at the call's rows.
int gemm_decode_tiles(int M, int N, int K, int epilogue, int splits) {
    const int tiles = epilogue == EPI_SWIGLU ? (N + 15) / 16 : (N + 31) / 32;
    float best = 1e30f;
    int nt = 1;
    for (int t = 1; t <= 3; ++t) {
        const int rounds = ((tiles + t - 1) / t * splits + 255) / 256;
        const float cost = (float)rounds * (t + (M + 31) / 32);
        if (cost < best) { best = cost; nt = t; }
    }
    return nt;
}

hipError_t launch_gemm_decode(const GemmArgs& a, int epilogue, int nt, hipStream_t s) {
    if (!gemm_decode_takes(a.M, a.N, a.K, epilogue, a.head != 0) || a.splits < 1 || a.splits > (a.K >> 7)) return hipErrorInvalidValue;
    // a large head: two tiles a workgroup (the winners' array has room for 64 columns each), one for logits of a few rows and a long K (151,936
    // columns, 1 / 2 / 3 tiles, us, K = 2560: 3 rows 110 / 116 / 119, 16 123 / 125 / 129, 24 140 / 132 / 135; K = 1024: 3 rows 48 / 47 / 47, 16 56 / 51 / 52; row-major weights, of whose lines a load has 32 bytes, lose 10 % of the step)
    if (epilogue == EPI_SAMPLE)
        return a.M <= 32 ? launch_one<1, 2, EPI_SAMPLE, 6, 2>(a, s) : a.M <= 64 ? launch_one<2, 2, EPI_SAMPLE, 6, 2>(a, s)
             : a.M <= 96 ? launch_one<3, 2, EPI_SAMPLE, 3, 1>(a, s) : launch_one<4, 2, EPI_SAMPLE, 3, 1>(a, s);
    if (epilogue == EPI_SWIGLU && a.splits != 1) return hipErrorInvalidValue;
    if (nt == 0) nt = a.head && (long long)a.N * a.K > 1 << 25 ? (a.wf && a.M <= 16 && a.K >= 2048 ? 1 : 2) : gemm_decode_tiles(a.M, a.N, a.K, epilogue, a.splits);
    if (epilogue == EPI_SWIGLU)
        return a.M <= 32 ? launch_tiles<EPI_SWIGLU, 1>(a, nt, s) : a.M <= 64 ? launch_tiles<EPI_SWIGLU, 2>(a, nt, s)
             : a.M <= 96 ? launch_tiles<EPI_SWIGLU, 3>(a, nt, s) : launch_tiles<EPI_SWIGLU, 4>(a, nt, s);
    return a.M <= 32 ? launch_tiles<EPI_STORE_F32, 1>(a, nt, s) : a.M <= 64 ? launch_tiles<EPI_STORE_F32, 2>(a, nt, s)
         : a.M <= 96 ? launch_tiles<EPI_STORE_F32, 3>(a, nt, s) : launch_tiles<EPI_STORE_F32, 4>(a, nt, s);
}

}  // namespace spiral
