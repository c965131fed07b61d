// Large-M projection kernel (prefill and the scoring pass): out[m][n] = sum_k A[m][k] * W[n][k] with
// hundreds or thousands of rows, where the matrix cores, not HBM, are the bound.
//
// A workgroup (4 waves, one per SIMD) owns a 256 x 256 output tile and walks K in chunks of 64.  Both
// operand tiles of a chunk go global -> registers -> LDS (rows padded to 144 B so that operand reads
// are conflict free; the weights come from the fragment-ordered copies, 1 KB contiguous per wave
// load, already in the operand type).  Three chunks are in flight: chunk c is multiplied out of one
// LDS buffer, chunk c + 1 moves from registers into the other buffer, and the global loads of chunk
// c + 2 are issued; the one barrier of a chunk sits before its last k step, so that the first operand reads of the
// next chunk are issued under MFMAs like all the others.  Every wave owns a 128 x 128 quarter: per k step of 16 it reads 4 + 4 operand
// fragments from LDS (one step ahead of their use) for 16 v_mfma_f32_32x32x16 (256 accumulator
// registers), i.e. 128 flop per byte fetched from L2 against 64 for a 128 x 128 tile; the issue order of
// a step is pinned (8 LDS reads, then 4 x (4 MFMAs, 1 LDS write, 1 global load)) so that LDS and memory
// traffic run under the MFMAs: issued as one burst at the start of a chunk the 16 loads of a thread cost a
// sixth of the kernel, spread over the k steps nothing measurable.  An isolated loop of this shape runs at 71 %
// of the nominal MFMA rate (a pure MFMA stream at 82 %: the clock under this load is ~2.0 GHz); the kernel delivers
// 1.0-1.15 PFLOP/s on 16,384 rows, the matrix cores busy 52-57 % of the cycles at 1.9-2.0 GHz (the vendor GEMM:
// 0.9-1.4 PFLOP/s on these shapes).  The clock follows the operand bits: with all-zero operands the gate/up
// projection takes 1.09 ms instead of 1.41 (1.50 PFLOP/s; the vendor GEMM 1.3-1.4 -> 1.9-2.0 PFLOP/s).
// Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; the tile order is arranged so
// that each XCD (own L2) gets a contiguous run of tiles, ordered in bands of 4 row tiles.
// A second form has tiles of 128 x 256 (a wave 64 x 128, 128 accumulator registers), and K may be split over workgroups:
// at 788 rows of the 4B shape 256-row tiles leave O and down 40 workgroups.  A layer's projections there, before (streaming
// kernel for q/k/v, O and down, 256-row tiles for gate/up) and with the form and the split chosen by estimated time:
// q/k/v 67 + 17 (its post-processing) -> 50 us, O 51 -> 26, gate/up 133 -> 115, down 113 -> 50.

#include <algorithm>

#include "spiral_internal.h"
#include "mfma_ops.h"

namespace spiral {

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mma32t(const u32x4& w, const u32x4& a, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, a), c, 0, 0, 0);
}

constexpr int BN = 256, BK = 64;
constexpr int ROW = 144;                          // LDS bytes per tile row: 64 k x 2 B + 16 pad
constexpr int stage_bytes(int bm) { return (bm + BN) * ROW; }      // activation tile, then weight tile

}  // namespace

// The weights are the fragment-ordered copies (frag_block(); SWIGLU: the interleaved gate/up matrix, a
// workgroup covers 128 ffn columns and the epilogue applies SiLU(gate) * up in registers).
// TEPI: 0 stores the fp32 product, 1 is the SwiGLU epilogue, 2 the q/k/v epilogue (the product never reaches memory:
// bias, per-head RMSNorm of q and k, RoPE, q stored as half, k and v appended to the sequence's page; head_dim 128,
// so a wave's 128 columns are exactly one head), 3 the scoring epilogue (per row the maximum and the sum of
// exponentials over each 128 columns, and the target column's product; no product reaches memory).
// BM: activation rows of the tile, 256 (a wave's quarter is 128 x 128) or 128 (64 x 128).
// g.splits > 1 (TEPI 0): K is cut at multiples of 128, split s writes its partial product to out[s], as the streaming kernel does.
template <int TEPI, int BM>
__global__ __launch_bounds__(256) void gemm_tile_kernel(GemmArgs g, QkvPostArgs qa) {
    constexpr bool SWIGLU = TEPI == 1;
    constexpr int J = 4, I = BM / 64;               // 32-row weight tiles and batch tiles per wave
    constexpr int A_BYTES = BM * ROW;               // activation tile; the weight tile follows it
    constexpr int STAGE = stage_bytes(BM);
    constexpr int AU = BM / 32, UNITS = AU + 8, UQ = UNITS / 4;        // 16-byte units of a thread and chunk; a quarter per k step
    constexpr int GROUP_M = 1024 / BM;
    extern __shared__ uint4 lds_raw[];
    char* lds = (char*)lds_raw;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wm = wave & 1, wn = wave >> 1;        // this wave's quarter
    const int K = g.K;

    // ---- tile of this workgroup
    const int n_cols = SWIGLU ? 128 : 256;          // output columns per workgroup
    const int m_tiles = (g.M + BM - 1) / BM, n_tiles = (g.N + n_cols - 1) / n_cols;
    const int per_split = m_tiles * n_tiles, total = per_split * (TEPI == 0 ? g.splits : 1);
    const int per_xcd = (total + 7) / 8;
    int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || t >= total) return;
    const int split = TEPI == 0 ? t / per_split : 0;
    t -= split * per_split;
    const int band = t / (GROUP_M * n_tiles);
    const int band_rows = min(GROUP_M, m_tiles - band * GROUP_M);
    const int tile_m = band * GROUP_M + (t % (GROUP_M * n_tiles)) % band_rows;
    const int tile_n = (t % (GROUP_M * n_tiles)) / band_rows;
    const int m0 = tile_m * BM, n0 = tile_n * n_cols;

    // ---- chunks of this workgroup's share of K
    const int cb = TEPI == 0 && g.splits > 1 ? 2 * (int)(((long long)(K >> 7) * split) / g.splits) : 0;
    const int ce = TEPI == 0 && g.splits > 1 ? 2 * (int)(((long long)(K >> 7) * (split + 1)) / g.splits) : K / BK;
    const int NC = ce - cb;

    // ---- global -> LDS assignment, AU + 8 16-byte units per thread and chunk.
    //      Activations (row-major): unit i is row threadIdx.x / 8 + 32 i, 16-byte column threadIdx.x % 8
    //      (8 lanes read one 128-byte line).  Weights: a wave reads whole 1 KB fragment blocks, unit i is
    //      block (row tile i, k step threadIdx.x / 64) of the chunk, lane = threadIdx.x % 64.
    //      Offsets are 32-bit element offsets from the operand's base (the launcher checks that they fit).
    uint32_t a_off[AU], w_off[8];
    const int dst0 = (threadIdx.x >> 3) * ROW + (threadIdx.x & 7) * 16;       // unit i lands 32 rows further down
    const int wdst0 = A_BYTES + l32 * ROW + (threadIdx.x >> 6) * 32 + lh * 16;
    {
        const int t_all = SWIGLU ? (g.N + 15) / 16 : (g.N + 31) / 32;
#pragma unroll
        for (int i = 0; i < AU; ++i) {
            int m = m0 + (threadIdx.x >> 3) + 32 * i; if (m >= g.M) m = g.M - 1;
            a_off[i] = (uint32_t)m * (uint32_t)K + (uint32_t)cb * BK + (threadIdx.x & 7) * 8;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int t32 = min((SWIGLU ? n0 / 16 : n0 / 32) + i, t_all - 1);
            w_off[i] = (uint32_t)frag_block(t32, cb * (BK / 16) + (threadIdx.x >> 6), K) + lane * 8;
        }
    }
    // operand fragments: row (wm * BM / 2 + i * 32 + l32 or wn * 128 + j * 32 + l32), k = ks * 16 + lh * 8
    const int a_frag = (wm * (BM / 2) + l32) * ROW + lh * 16;
    const int w_frag = A_BYTES + (wn * 128 + l32) * ROW + lh * 16;

    f32x16 acc[J][I];                               // [weight tile j][batch tile i]
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int i = 0; i < I; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

    // Two register stages: a chunk's global loads are issued two chunks before it is multiplied and
    // one chunk before it is parked in LDS, so the staging writes never wait for memory.
    u32x4 rg[2][UNITS];                             // [stage][AU activation units, 8 weight units]
    auto load_unit = [&](const int st, const int cc, const int u) {
        if (u < AU) rg[st][u] = *(const u32x4*)((const uint16_t*)g.A + a_off[u < AU ? u : 0] + (size_t)cc * BK);
        else rg[st][u] = *(const u32x4*)((const uint16_t*)g.wf + w_off[u < AU ? 0 : u - AU] + (size_t)cc * (BK / 16) * 512);
    };
    auto load = [&](const int st, int c) {
        const int cc = c < NC ? c : NC - 1;           // past the end: a re-read of the last chunk
#pragma unroll
        for (int u = 0; u < UNITS; ++u) load_unit(st, cc, u);
    };
    auto park_unit = [&](char* buf, const int st, const int u) {
        if (u < AU) *(u32x4*)(buf + dst0 + u * 32 * ROW) = rg[st][u];
        else *(u32x4*)(buf + wdst0 + (u - AU) * 32 * ROW) = rg[st][u];
    };
    auto frags = [&](const char* buf, int ks, u32x4* af, u32x4* wf) {
#pragma unroll
        for (int i = 0; i < I; ++i) af[i] = *(const u32x4*)(buf + a_frag + i * 32 * ROW + ks * 32);
#pragma unroll
        for (int j = 0; j < J; ++j) wf[j] = *(const u32x4*)(buf + w_frag + j * 32 * ROW + ks * 32);
    };
    // Chunk c sits in LDS buffer c & 1 and came through register stage c & 1.  The barrier of a chunk sits before
    // its last k step, not after it: by then every wave has issued (and waited for) its last operand reads of the
    // chunk and has parked all of chunk c + 1, so the last k step already reads the first fragments of chunk c + 1
    // and starts parking chunk c + 2 into the buffer that just became free - no operand read is ever exposed
    // behind a barrier.  Per k step (BM = 256): the 8 operand reads of the next step, four units parked, four units
    // requested (each unit is requested four k steps before it is parked), 16 MFMAs; issue order pinned to 8 reads, then
    // 4 x (4 MFMAs, 1 write, 1 global load) (other orders of the same instructions measured within noise).
    u32x4 af[2][I], wf[2][J];
    auto chunk = [&](int c, const int cu, const int nx) {
        char* buf = lds + cu * STAGE;                 // cu == c & 1
        char* other = lds + nx * STAGE;
        const int c2 = c + 2 < NC ? c + 2 : NC - 1;   // past the end: a re-read of the last chunk
        const int c3 = c + 3 < NC ? c + 3 : NC - 1;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) {
                frags(buf, ks + 1, af[(ks + 1) & 1], wf[(ks + 1) & 1]);
#pragma unroll
                for (int u = 0; u < UQ; ++u) park_unit(other, nx, (ks + 1) * UQ + u);
#pragma unroll
                for (int u = 0; u < UQ; ++u) load_unit(cu, c2, (ks + 1) * UQ + u);
            } else {
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
                frags(other, 0, af[0], wf[0]);
#pragma unroll
                for (int u = 0; u < UQ; ++u) park_unit(buf, cu, u);
#pragma unroll
                for (int u = 0; u < UQ; ++u) load_unit(nx, c3, u);
            }
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int i = 0; i < I; ++i) acc[j][i] = mma32t(wf[ks & 1][j], af[ks & 1][i], acc[j][i]);
            __builtin_amdgcn_sched_group_barrier(0x100, I + J, 0);
#pragma unroll
            for (int r = 0; r < UQ; ++r) {
                __builtin_amdgcn_sched_group_barrier(0x008, I, 0);
                __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    load(0, 0);
    load(1, 1);
#pragma unroll
    for (int u = 0; u < UNITS; ++u) park_unit(lds, 0, u);
#pragma unroll
    for (int u = 0; u < UQ; ++u) park_unit(lds + STAGE, 1, u);
#pragma unroll
    for (int u = 0; u < UQ; ++u) load_unit(0, 2 < NC ? 2 : NC - 1, u);
    __syncthreads();
    frags(lds, 0, af[0], wf[0]);
    int c = 0;
    for (; c + 2 <= NC; c += 2) {
        chunk(c, 0, 1);
        chunk(c + 1, 1, 0);
    }
    if (c < NC) chunk(c, 0, 1);
    __syncthreads();                                  // the operand buffers are free for the epilogue

    // ---- epilogue.  In a 32 x 32 tile a lane holds batch row l32 and, in registers 4b..4b+3, weight rows 8b + 4*lh .. +3:
    //      written straight from there a store instruction touches 64 rows x 16 (or 8) bytes.  Each wave therefore
    //      turns its tile 32 rows at a time through a private LDS area (the operand buffers are free after the last
    //      barrier) and stores whole rows: 512 contiguous bytes per half wave (fp32), one 128-byte line per 8 lanes (SwiGLU).
    if (TEPI == 2) {
        const int head = (n0 + wn * 128) >> 7;
        const bool is_q = head < qa.n_q_heads, is_k = !is_q && head < qa.n_q_heads + qa.n_kv_heads;
        const int kvh = is_q ? 0 : (is_k ? head - qa.n_q_heads : head - qa.n_q_heads - qa.n_kv_heads);
        const uint16_t* bias = (const uint16_t*)(is_q ? qa.bq : (is_k ? qa.bk : qa.bv));      // bf16 like the weights, or null
        if (bias) bias += (is_q ? head : kvh) * 128;
        const float* gain = is_q ? qa.q_gain : (is_k ? qa.k_gain : nullptr);
        bool bad = false;
        // Rotation rows come in, q and k rows go out through a private LDS area of the wave, so that its global accesses are
        // whole rows: straight in the accumulator layout every instruction touches 32 rows (4B shape, 11,200 rows 442 us a
        // layer against 390; 256-row tiles, whose epilogue spills, 433).
        constexpr int RROW = 64 * 8 + 16, OROW = 128 * 2 + 16;      // staged rotation row, staged output row
        char* tb = lds + wave * (32 * RROW);
        if (head < qa.n_q_heads + 2 * qa.n_kv_heads) {
#pragma unroll
            for (int i = 0; i < I; ++i) {
                const int mb = m0 + wm * (BM / 2) + i * 32, m = mb + l32;
                if (is_q || is_k) {
                    u32x4 rr[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) rr[u] = *(const u32x4*)(qa.rope + (size_t)min(mb + 2 * u + lh, g.M - 1) * 64 + 2 * l32);
#pragma unroll
                    for (int u = 0; u < 16; ++u) *(u32x4*)(tb + (2 * u + lh) * RROW + l32 * 16) = rr[u];
                    __builtin_amdgcn_wave_barrier();
                }
                // this lane's 64 values of the head: dimension d = 32 j + 8 b + 4 lh + e sits in acc[j][i][4 b + e]
                if (bias) {
#pragma unroll
                    for (int j = 0; j < J; ++j)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const ushort4 bb = *(const ushort4*)(bias + 32 * j + 8 * b + 4 * lh);
                            acc[j][i][4 * b] += bf16_bits_to_f32(bb.x);
                            acc[j][i][4 * b + 1] += bf16_bits_to_f32(bb.y);
                            acc[j][i][4 * b + 2] += bf16_bits_to_f32(bb.z);
                            acc[j][i][4 * b + 3] += bf16_bits_to_f32(bb.w);
                        }
                }
                if (gain) {
                    // the pairs (d, d + 64), summed over the bits of d from the highest down as qkv_post_kernel's wave does
                    float e4[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float v[4];
#pragma unroll
                        for (int b = 0; b < 4; ++b)
                            v[b] = square_pair(acc[0][i][4 * b + e], acc[2][i][4 * b + e]) + square_pair(acc[1][i][4 * b + e], acc[3][i][4 * b + e]);
                        const float t4 = (v[0] + v[2]) + (v[1] + v[3]);
                        e4[e] = t4 + __shfl_xor(t4, 32, 64);
                    }
                    const float ss = (e4[0] + e4[2]) + (e4[1] + e4[3]);
                    const float rs = rsqrtf(ss / 128.f + qa.eps);
#pragma unroll
                    for (int j = 0; j < J; ++j)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const float4 gg = *(const float4*)(gain + 32 * j + 8 * b + 4 * lh);
                            acc[j][i][4 * b] = acc[j][i][4 * b] * rs * gg.x;
                            acc[j][i][4 * b + 1] = acc[j][i][4 * b + 1] * rs * gg.y;
                            acc[j][i][4 * b + 2] = acc[j][i][4 * b + 2] * rs * gg.z;
                            acc[j][i][4 * b + 3] = acc[j][i][4 * b + 3] * rs * gg.w;
                        }
                }
                if (is_q || is_k) {                      // rotate-half: d pairs with d + 64, i.e. tile j with tile j + 2
                    const float2* cs = (const float2*)(tb + l32 * RROW);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            const float4 c01 = *(const float4*)(cs + 32 * j + 8 * b + 4 * lh);
                            const float4 c23 = *(const float4*)(cs + 32 * j + 8 * b + 4 * lh + 2);
                            const float co[4] = {c01.x, c01.z, c23.x, c23.z}, si[4] = {c01.y, c01.w, c23.y, c23.w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float2 r2 = rotate_pair(acc[j][i][4 * b + e], acc[j + 2][i][4 * b + e], co[e], si[e]);
                                acc[j][i][4 * b + e] = r2.x;
                                acc[j + 2][i][4 * b + e] = r2.y;
                            }
                        }
                }
                if (is_q || is_k) {
                    __builtin_amdgcn_wave_barrier();     // the rotation rows have been read
#pragma unroll
                    for (int j = 0; j < J; ++j)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            bool out_of_range = false;
                            ushort4 o;
                            o.x = f32_to_act16_noting(acc[j][i][4 * b], out_of_range);
                            o.y = f32_to_act16_noting(acc[j][i][4 * b + 1], out_of_range);
                            o.z = f32_to_act16_noting(acc[j][i][4 * b + 2], out_of_range);
                            o.w = f32_to_act16_noting(acc[j][i][4 * b + 3], out_of_range);
                            bad = bad || (out_of_range && m < g.M);
                            *(ushort4*)(tb + l32 * OROW + (32 * j + 8 * b + 4 * lh) * 2) = o;
                        }
                    __builtin_amdgcn_wave_barrier();
                    if (is_q) {                          // 16 lanes a row of 256 bytes
                        const int c16 = lane & 15;
#pragma unroll
                        for (int ps = 0; ps < 8; ++ps) {
                            const int row = 4 * ps + (lane >> 4);
                            const u32x4 v = *(const u32x4*)(tb + row * OROW + c16 * 16);
                            if (mb + row < g.M) *(u32x4*)(qa.q + ((size_t)(mb + row) * qa.n_q_heads + head) * 128 + c16 * 8) = v;
                        }
                    } else {                             // 16 rows x 4 groups of 8 d: tokens of a page are neighbours
                        const int r16 = lane & 15;
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            const int row = half * 16 + r16;
                            const int2 pp = qa.row_page[min(mb + row, g.M - 1)];
                            uint16_t* dst = qa.pages + ((size_t)pp.x * qa.n_kv_heads + kvh) * (size_t)(2 * kPageTokens * 128);
#pragma unroll
                            for (int j = 0; j < 4; ++j) {
                                // K element (token, d) sits at (d/32)*512 + (((d%32)/8)*16 + token)*8 + d%8; this lane's d/8 is 4 j + lane/16
                                const int b = lane >> 4;
                                const u32x4 v = *(const u32x4*)(tb + row * OROW + (4 * j + b) * 16);
                                if (mb + row < g.M) *(u32x4*)(dst + j * 512 + ((b * 16 + (pp.y & (kPageTokens - 1))) << 3)) = v;
                            }
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                } else if (m < g.M) {
                    const int2 pp = qa.row_page[m];
                    const int slot = pp.y & (kPageTokens - 1);
                    uint16_t* dst = qa.pages + ((size_t)pp.x * qa.n_kv_heads + kvh) * (size_t)(2 * kPageTokens * 128) + kPageTokens * 128;
#pragma unroll
                    for (int j = 0; j < J; ++j)
#pragma unroll
                        for (int b = 0; b < 4; ++b) {
                            // V element (d, token) sits at (d/32)*512 + ((token/4)*16 + d%16)*8 + ((d/16)%2)*4 + token%4
                            uint16_t* vb = dst + j * 512 + (((slot >> 2) * 16 + 8 * (b & 1) + 4 * lh) << 3) + ((b >> 1) << 2) + (slot & 3);
                            vb[0] = f32_to_act16_noting(acc[j][i][4 * b], bad);
                            vb[8] = f32_to_act16_noting(acc[j][i][4 * b + 1], bad);
                            vb[16] = f32_to_act16_noting(acc[j][i][4 * b + 2], bad);
                            vb[24] = f32_to_act16_noting(acc[j][i][4 * b + 3], bad);
                        }
                }
            }
        }
        report_saturation(qa.sat_count, bad);
    } else if (TEPI == 3) {
        // A lane holds 64 of the 128 columns of four rows: it folds them, column tile by column tile, and the lane halves
        // merge theirs: one (max, sum exp) pair per row and 128 columns.  The streaming kernel folds in the same order, so
        // that repacked and row-major weights give the same bits.  The exponentials (256 a lane) are 5 % of the tile's
        // matrix time at K = 2560.  Bound by the matrix cores: 6,028 rows x 151,936 columns x 2560 take 4.4 ms
        // (1.09 PFLOP/s); the streaming kernel with 128-row tiles, which fetches twice the bytes per product from L2 and
        // reads twice the LDS per MFMA, took 6.5.
        const int c0 = n0 + wn * 128 + 4 * lh, pair = tile_n * 2 + wn;
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int m = m0 + wm * (BM / 2) + i * 32 + l32;
            const int tgt = m < g.M ? g.targets[m] : -1;
            float mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int col = c0 + 32 * j + 8 * (r >> 2) + (r & 3);
                    if (col >= g.N) acc[j][i][r] = -INFINITY;         // padding of the last tile (clamped weight rows)
                    if (col == tgt) g.tgt_logit[m] = acc[j][i][r];
                    mx = fmaxf(mx, acc[j][i][r]);
                }
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float ref = mx > -INFINITY ? mx : 0.f;              // nothing but -inf: all terms are zero
            float sum = 0.f;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                float sj = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) sj += __expf(acc[j][i][r] - ref);
                sum = j == 0 ? sj : sum + sj;
            }
            sum += __shfl_xor(sum, 32, 64);
            if (lh == 0 && m < g.M && pair < g.s_tiles) g.s_part[(size_t)pair * g.M + m] = make_float2(mx, sum);
        }
    } else if (!SWIGLU) {
        float* out = (float*)g.out + (size_t)split * g.M * g.N;
        constexpr int TROW = 128 * 4 + 16;              // staged row: 128 floats + pad
        char* tb = lds + wave * (32 * TROW);
        const int rr = lane >> 5, c4 = lane & 31;       // read side: row 2 p + rr, floats 4 c4 .. 4 c4 + 3
        const int n = n0 + wn * 128 + 4 * c4;
#pragma unroll
        for (int i = 0; i < I; ++i) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    *(float4*)(tb + l32 * TROW + (j * 32 + 8 * b + 4 * lh) * 4) =
                        make_float4(acc[j][i][4 * b], acc[j][i][4 * b + 1], acc[j][i][4 * b + 2], acc[j][i][4 * b + 3]);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ps = 0; ps < 16; ++ps) {
                const int row = 2 * ps + rr;
                const float4 v = *(const float4*)(tb + row * TROW + c4 * 16);
                const int m = m0 + wm * (BM / 2) + i * 32 + row;
                if (m < g.M && n < g.N) *(float4*)(out + (size_t)m * g.N + n) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
    } else {
        bool bad = false;
        constexpr int TROW = 64 * 2 + 16;               // staged row: 64 halves + pad
        char* tb = lds + wave * (32 * TROW);
        const int rr = lane >> 3, c8 = lane & 7;        // read side: row 8 p + rr, halves 8 c8 .. 8 c8 + 7
        const int f = n0 + wn * 64 + 8 * c8;
#pragma unroll
        for (int i = 0; i < I; ++i) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    ushort4 o;
                    o.x = f32_to_act16_noting(silu_f(acc[j][i][4 * b]) * acc[j][i][4 * b + 8], bad);
                    o.y = f32_to_act16_noting(silu_f(acc[j][i][4 * b + 1]) * acc[j][i][4 * b + 9], bad);
                    o.z = f32_to_act16_noting(silu_f(acc[j][i][4 * b + 2]) * acc[j][i][4 * b + 10], bad);
                    o.w = f32_to_act16_noting(silu_f(acc[j][i][4 * b + 3]) * acc[j][i][4 * b + 11], bad);
                    *(ushort4*)(tb + l32 * TROW + (j * 16 + 8 * b + 4 * lh) * 2) = o;
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int ps = 0; ps < 4; ++ps) {
                const int row = 8 * ps + rr;
                const u32x4 v = *(const u32x4*)(tb + row * TROW + c8 * 16);
                const int m = m0 + wm * (BM / 2) + i * 32 + row;
                if (m < g.M && f < g.N) *(u32x4*)((uint16_t*)g.out + (size_t)m * g.N + f) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
        report_saturation(g.sat_count, bad);
    }
}

template <int TEPI, int BM>
static hipError_t launch_tile_bm(const GemmArgs& a, const QkvPostArgs& qa, hipStream_t s) {
    const int cols = TEPI == 1 ? 128 : 256;
    const int m_tiles = (a.M + BM - 1) / BM;
    const int n_tiles = (a.N + cols - 1) / cols;
    const long long total = (long long)m_tiles * n_tiles * (TEPI == 0 ? a.splits : 1);
    if (total > (1ll << 30)) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8);
    const size_t lds_bytes = (size_t)2 * stage_bytes(BM);
    hipError_t e = hipFuncSetAttribute((const void*)gemm_tile_kernel<TEPI, BM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_tile_kernel<TEPI, BM>), dim3(per_xcd * 8), dim3(256), lds_bytes, s, a, qa);
    return hipGetLastError();
}

template <int TEPI>
static hipError_t launch_tile(const GemmArgs& a, const QkvPostArgs& qa, int bm, hipStream_t s) {
    return bm == 128 ? launch_tile_bm<TEPI, 128>(a, qa, s) : launch_tile_bm<TEPI, 256>(a, qa, s);
}

// needs the fragment-ordered weights (a.wf), K % 64 == 0 (% 128 with a split) and operands small enough for 32-bit element offsets
bool gemm_tile_usable(const GemmArgs& a) {
    return a.wf != nullptr && a.splits >= 1 && (a.K % (a.splits > 1 ? 128 : BK)) == 0 && a.splits <= std::max(1, a.K >> 7) && (a.N & 3) == 0 &&
           (long long)a.M * a.K < (1ll << 31) && ((long long)a.N + 32) * 2 * a.K < (1ll << 31);
}

// Estimated microseconds of one launch on 256 x 256 or 128 x 256 tiles (cols: output columns of a tile): rounds over the
// 256 compute units, one workgroup each, x (fixed part + 64-wide k chunks, which take a third longer on a full chip, where
// the clock follows the power limit).  Measured, 4B shape (us, one round): O on 40 tiles of 256 rows 84 and down 185
// (K = 4096, 9728), on 70 tiles of 128 rows 49 and 106; gate/up at 11,200 rows (13 and 26 rounds) 80 and 42.5 a round.
float gemm_tile_us(int M, int N, int K, int splits, int cols, int bm) {
    const long tiles = (long)((M + bm - 1) / bm) * ((N + cols - 1) / cols) * splits, rounds = (tiles + 255) / 256;
    const float chunk = bm == 256 ? 1.15f : 0.655f, fixed = bm == 256 ? 9.7f : 6.9f;
    return (float)rounds * (fixed + chunk * (K / (float)splits) / 64.f * (1.f + 0.35f * (float)tiles / (256.f * (float)rounds)));
}

// ... and of the streaming kernel on 128-row tiles of bn (128 or 64) columns.  Measured: O and down of the 4B shape at 788
// rows (140 workgroups of 128 columns) 51 and 113 us; O of the 0.6B shape (112 of 64 columns, K = 2048) 20.
float gemm_stream_us(int M, int N, int K, int splits, int bn) {
    const long tiles = (long)((M + 127) / 128) * ((N + bn - 1) / bn) * splits, rounds = (tiles + 255) / 256;
    const float chunks = (K / (float)splits) / 128.f;
    return (float)rounds * (bn >= 128 ? 5.8f + 1.41f * chunks : 2.6f + 0.92f * chunks * (1.f + 0.2f * (float)tiles / (256.f * (float)rounds)));
}

// The tile height for a launch: the cheaper of the two, 0 where the streaming kernel is cheaper still.  All three add
// the products of an output in the same order, so the choice never changes a result.  Shapes that the streaming kernel does not
// take (row-major weights go to a kernel with another order there) are tiled only where 256 x 256 tiles fill the chip.
int gemm_tile_height(int M, int N, int K, int splits, int cols, int bn) {
    if ((K & 127) || (N & 15))
        return M >= 512 && (long)((M + 255) / 256) * ((N + cols - 1) / cols) >= 200 ? 256 : 0;
    const float t256 = gemm_tile_us(M, N, K, splits, cols, 256), t128 = gemm_tile_us(M, N, K, splits, cols, 128);
    const float ts = gemm_stream_us(M, cols == 128 ? 2 * N : N, K, splits, bn == 64 ? 64 : 128);
    if (M <= 128 || ts < std::min(t256, t128)) return 0;
    return t128 < t256 ? 128 : 256;
}

int gemm_tile_rows(const GemmArgs& a, int epilogue, int bn) {
    if (!gemm_tile_usable(a) || (epilogue == EPI_SWIGLU && ((a.N & 7) || a.splits != 1))) return 0;     // SwiGLU rows are stored 8 halves at a time
    return gemm_tile_height(a.M, a.N, a.K, a.splits, epilogue == EPI_SWIGLU ? 128 : 256, bn);
}

// K splits of a projection over more than 128 rows, and the streaming kernel's tile width: the pair for which the estimated
// time of the launch plus that of the partial sums (written, and read by the norm kernel; 788 x 2560 of them cost 0.7 us
// of the norm kernel each, and the writes about as much again) is least.  It depends on the shape - the rows of the whole call
// among it - and not on how the weights are stored, so that repacked and row-major weights keep adding in the same order.
// The estimates err by 5 to 9 %, so splits that they prefer by less may go either way; measured (launch unsplit -> as chosen, and
// what the partial sums add to the norm kernel): down, 15,272 rows of the 4B shape (estimated gain 2.8 %) 712 -> 686 us and 21,
// 8,000 rows (3.1 %) 398 -> 399 and 10; down of the 7B shape, 15,272 rows (4.2 %) 1972 -> 1803 and 20, 11,000 (7.2 %)
// 1344 -> 1285 and 10; O of the 0.6B shape, 1,500 rows (3.0 %) 30.6 -> 21.5 and 0.8.  Asking for a gain of 8 % would lose all of
// these but the second.
float gemm_wide_shape(int M, int N, int K, int most, int& bn, int& splits) {
    float best = 1e30f;
    for (int s = 1; s <= std::max(1, most) && (s == 1 || (K % 128 == 0 && K / s >= 512)); ++s) {
        const float s128 = gemm_stream_us(M, N, K, s, 128), s64 = gemm_stream_us(M, N, K, s, 64);
        const float launch = std::min({gemm_tile_us(M, N, K, s, 256, 256), gemm_tile_us(M, N, K, s, 256, 128), s128, s64});
        const float us = launch + (float)(s - 1) * M * N * 4.f / 3.3e6f;
        if (us < best) { best = us; splits = s; bn = s64 < s128 ? 64 : 128; }
    }
    return best;
}

hipError_t launch_gemm_tile(const GemmArgs& a, int epilogue, int bm, hipStream_t s) {
    if (!gemm_tile_usable(a) || (epilogue == EPI_SWIGLU && ((a.N & 7) || a.splits != 1)) || (epilogue != EPI_SWIGLU && epilogue != EPI_STORE_F32))
        return hipErrorInvalidValue;
    const QkvPostArgs none = {};
    return epilogue == EPI_SWIGLU ? launch_tile<1>(a, none, bm, s) : launch_tile<0>(a, none, bm, s);
}

int gemm_tile_score_height(int M, int N, int K) { return gemm_tile_us(M, N, K, 1, 256, 128) < gemm_tile_us(M, N, K, 1, 256, 256) ? 128 : 256; }
// The LM head with the scoring epilogue: one (max, sum exp) pair per row and 128 columns.
hipError_t launch_gemm_tile_score(const GemmArgs& a, hipStream_t s) {
    if (!gemm_tile_usable(a) || a.splits != 1 || !a.s_part || !a.targets || !a.tgt_logit || a.s_tiles != (a.N + 127) / 128) return hipErrorInvalidValue;
    const QkvPostArgs none = {};
    return launch_tile<3>(a, none, gemm_tile_score_height(a.M, a.N, a.K), s);
}

// The q/k/v projection with the work of qkv_post_kernel in its epilogue (qa.qkv and qa.n_part are not used).
// The fused form has tiles of 128 rows; its epilogue costs a round 8 us.
bool gemm_tile_qkv_fits(int N, int K, const QkvPostArgs& qa) {
    return (K % BK) == 0 && qa.hd == 128 && (N & 255) == 0 && N == (qa.n_q_heads + 2 * qa.n_kv_heads) * 128;
}
// ... where the streaming kernel does not take the shape (K % 128 == 64) the alternative is 256 x 256 tiles once they fill the
// chip, with qkv_post_kernel behind them: 8,000 rows x 4096 x 1088 76 + 71 us,
// fused 98.
bool gemm_tile_qkv_fills(int M, int N) { return M >= 512 && (long)((M + 255) / 256) * (N / 256) >= 200; }
float gemm_tile_qkv_us(int M, int N, int K) {
    const long tiles = (long)((M + 127) / 128) * (N / 256);
    return gemm_tile_us(M, N, K, 1, 256, 128) + 8.f * (float)((tiles + 255) / 256);
}
hipError_t launch_gemm_tile_qkv(const GemmArgs& a, const QkvPostArgs& qa, hipStream_t s) {
    if (!gemm_tile_usable(a) || a.splits != 1 || qa.row_map || !gemm_tile_qkv_fits(a.N, a.K, qa)) return hipErrorInvalidValue;
    return launch_tile_bm<2, 128>(a, qa, s);
}

}  // namespace spiral
