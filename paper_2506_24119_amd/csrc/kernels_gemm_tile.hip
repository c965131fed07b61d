// Large-M projection kernel (prefill and the scoring pass): out[m][n] = sum_k A[m][k] * W[n][k] with
// hundreds or thousands of rows, where the matrix cores, not HBM, are the bound.
//
// A workgroup of 4 waves owns a tile of 256 or 128 rows x 256 columns, a wave a quarter of it (128 x 128 or 64 x 128, 256 or 128
// accumulator registers), and walks K in chunks of 64.  Both operands go from memory straight to LDS (buffer loads with an LDS
// destination): no registers, no LDS writes by the waves, and the 128-row tile, without staging registers and with 80 KB of LDS, fits a
// compute unit twice, so that one workgroup's first loads, epilogue and barriers run under the other's products.  LDS holds
// activations as whole 128-byte rows, their eight pieces permuted so that operand reads meet no bank twice, and weights as
// fragment blocks (frag_block(), already in the operand type), three (two) slots of 64 k of activations and four (three) of 32 k of
// weights.  What else was tried and measured, gate/up of the 4B shape at 15,272 rows (us in one session, in which the kernel that staged operands
// through registers, 256 rows, one chunk ahead, took 1412): both operands straight to LDS with two slots of 64 k 1656 to 1706 (loads one chunk ahead are too
// late); activations in slots of 32 k, whose loads touch half lines, 1357 (256 rows), 1375 (128); whole lines 1262 to 1290; the
// reads of a half's second k step as a burst instead of one behind each product +2 %; those behind the barrier spread likewise +1.5 %;
// s_setprio around the products +3 %; bands of 2048 or 4096 rows +1 and +7 %.
// The chip's power is the limit.  Counters of that launch, staged through registers -> now: matrix cores busy 58 -> 64 % of the cycles, clock 1.79 -> 1.73 GHz;
// traced with all-zero operands it takes 981 us instead of 1369 (1.55 PFLOP/s against 1.11).  A loop of nothing but products with random operands makes
// 1.70 PFLOP/s, with its operand reads from LDS 1.54.  Times of a launch, us between events, staged through registers -> now: gate/up 4B shape 15,272 rows
// 1399 -> 1309, 788 rows 115 -> 94, 0.6B shape 11,206 rows 184 -> 146; O and down 4B 15,272 rows 330 -> 291 and 700 -> 662, 788 rows (3 K splits)
// 29.0 -> 28.9 and 52.6 -> 51.2 (traced with the rest of a prefill 27.8 -> 28.1 and 51.9 -> 54.3); down 0.6B 11,206 rows 83 -> 75; q/k/v with its
// post-processing 4B 549 -> 465, 0.6B 161 -> 115; the scoring LM head, 6,028 rows 4527 -> 4160 (3780 by itself, 1.24 PFLOP/s).  Same bits throughout.
// Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; the tile order is arranged so
// that each XCD (own L2) gets a contiguous run of tiles, ordered in bands of 1024 rows.
// K may be split over workgroups: at 788 rows of the 4B shape 256-row tiles leave O and down 40 workgroups.

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "spiral_internal.h"
#include "mfma_ops.h"

namespace spiral {

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mma32t(const u32x4& w, const u32x4& a, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, a), c, 0, 0, 0);
}

constexpr int BK = 64;
constexpr int kAllBytes = 0x7FFFFFFF;

// The operand loads carry a buffer descriptor: one of size zero drops them, so that the steady loop runs to the end of K without a branch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_upto(const void* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00027000);
}
// 64 lanes x 16 bytes straight to 1 KB of LDS at dst (wave-uniform); IMM counts on both sides
template <int IMM, int AUX = 0>
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t r, char* dst, uint32_t off, int soff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, off, soff, IMM, AUX);
}
// which of a 128-byte row's eight 16-byte pieces sits where: 8 (and 16) lanes that read one piece of consecutive rows meet no bank twice
__device__ __forceinline__ int row_swizzle(int r) { return (r & 6) | ((r ^ (r >> 3)) & 1); }

// Slots in LDS: activations of 64 k, weights of 32 k; all 160 KB for the tall tile, half of them for the other, two of which share a compute unit.
template <int BM> struct Slots {
    static constexpr int A = BM == 256 ? 3 : 2, W = A + 1;
    static constexpr int A_BYTES = BM * 128, W_BYTES = 256 * 64, W_BASE = A * A_BYTES;
    static constexpr int TOTAL = W_BASE + W * W_BYTES;
};

}  // namespace

// The weights are the fragment-ordered copies (frag_block(); SWIGLU: the interleaved gate/up matrix, a
// workgroup covers 128 ffn columns and the epilogue applies SiLU(gate) * up in registers).
// TEPI: 0 stores the fp32 product, 1 is the SwiGLU epilogue, 2 the q/k/v epilogue (the product never reaches memory:
// bias, per-head RMSNorm of q and k, RoPE, q stored as half, k and v appended to the sequence's page; head_dim 128,
// so a wave's 128 columns are exactly one head), 3 the scoring epilogue (per row the maximum and the sum of
// exponentials over each 128 columns, and the target column's product; no product reaches memory).
// BM: activation rows of the tile, 256 (a wave's quarter is 128 x 128) or 128 (64 x 128).
// g.splits > 1 (TEPI 0): K is cut at multiples of 128, split s writes its partial product to out[s], as the streaming kernel does.
// NT: weights are read once, by non-temporal loads.
template <int TEPI, int BM, bool NT>
__device__ __forceinline__ void tile_body(const GemmArgs& g, const QkvPostArgs& qa) {
    constexpr bool SWIGLU = TEPI == 1;
    constexpr int J = 4, I = BM / 64;               // 32-row weight tiles and batch tiles per wave
    using L = Slots<BM>;
    constexpr int AU = BM / 32;                     // 8-row blocks of an activation chunk that a wave brings
    constexpr int GROUP_M = 1024 / BM;
    extern __shared__ uint4 lds_raw[];
    char* lds = (char*)lds_raw;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lh = lane >> 5;
    const int wm = wave & 1, wn = wave >> 1;        // this wave's quarter
    const int K = g.K;

    // ---- tile of this workgroup
    const int n_cols = SWIGLU ? 128 : 256;          // output columns per workgroup
    const int m_tiles = (g.M + BM - 1) / BM, n_tiles = (g.N + n_cols - 1) / n_cols;
    const int splits = TEPI == 0 ? g.splits : 1;
    // A last row tile at most half full is light work.  Its workgroups come last on every XCD, where they fill what the whole tiles leave (one after
    // the other with them, the last whole ones started when a light one ended), unless its second walk over the weights would be over
    // memory: the memory-side cache holds 256 MB.  us, all tiles alike / light ones multiplying what there is / and last: gate/up of the 4B shape,
    // 400 rows 60.6 / 57.5 / 53.5, 788 96 / 88 / 84, 1,300 134 / 134 / 128, q/k/v 1,300 68 / 65 / 58; scoring LM head 300 rows 286 / 268 / 329.
    const bool light = BM == 128 && TEPI <= 2 && m_tiles > 1 && g.M - (m_tiles - 1) * BM <= BM / 2 && (long long)g.N * K <= (SWIGLU ? 1 << 25 : 1 << 26);
    const int whole_m = m_tiles - light;             // row tiles of the first part
    const int per_split = whole_m * n_tiles, total = per_split * splits;
    const int per_xcd = (total + 7) / 8, xcd = blockIdx.x & 7, at = blockIdx.x >> 3;
    int split, tile_m, tile_n;
    if (at < per_xcd) {
        int t = xcd * per_xcd + at;
        if (t >= total) return;
        split = TEPI == 0 ? t / per_split : 0;
        t -= split * per_split;
        const int band = t / (GROUP_M * n_tiles);
        const int band_rows = min(GROUP_M, whole_m - band * GROUP_M);
        tile_m = band * GROUP_M + (t % (GROUP_M * n_tiles)) % band_rows;
        tile_n = (t % (GROUP_M * n_tiles)) / band_rows;
    } else {
        const int rest = light ? n_tiles * splits : 0, per_rest = (rest + 7) / 8, t = xcd * per_rest + at - per_xcd;
        if (at - per_xcd >= per_rest || t >= rest) return;
        split = TEPI == 0 ? t / n_tiles : 0;
        tile_m = whole_m;
        tile_n = t - split * n_tiles;
    }
    const int m0 = tile_m * BM, n0 = tile_n * n_cols;

    // ---- chunks of this workgroup's share of K
    const int cb = TEPI == 0 && g.splits > 1 ? 2 * (int)(((long long)(K >> 7) * split) / g.splits) : 0;
    const int ce = TEPI == 0 && g.splits > 1 ? 2 * (int)(((long long)(K >> 7) * (split + 1)) / g.splits) : K / BK;
    const int NC = ce - cb;

    // ---- global -> LDS.  Activations (row-major): an instruction brings 8 rows x 128 bytes, block u of a wave is rows 8 (4 u + wave) .. + 7;
    //      the LDS side of the load is linear, so a lane picks the piece of its row that belongs where it writes.  Weights: an
    //      instruction brings one fragment block, units 2 i and 2 i + 1 of a wave are the two k steps of row tile wave + 4 i.
    //      Offsets are bytes from the tile's own first row (the launcher bounds K).
    const int t_all = SWIGLU ? (g.N + 15) / 16 : (g.N + 31) / 32, tile0 = SWIGLU ? n0 / 16 : n0 / 32;
    const uint16_t* abase = (const uint16_t*)g.A + (size_t)m0 * K + (size_t)cb * BK;
    const uint16_t* wbase = (const uint16_t*)g.wf + frag_block(tile0, cb * (BK / 16), K);
    uint32_t a_off[AU], w_off[2];
#pragma unroll
    for (int u = 0; u < AU; ++u) {
        const int r = (u * 4 + wave) * 8 + (lane >> 3);
        a_off[u] = (uint32_t)min(r, g.M - 1 - m0) * (uint32_t)K * 2u + ((lane & 7) ^ row_swizzle(r)) * 16;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) w_off[i] = (uint32_t)min(wave + 4 * i, t_all - 1 - tile0) * (uint32_t)K * 64u + lane * 16;
    // operand fragments: row (wm * BM / 2 + i * 32 + l32 or wn * 128 + j * 32 + l32), k = ks * 16 + lh * 8
    int a_frag[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) a_frag[ks] = (wm * (BM / 2) + l32) * 128 + ((ks * 2 + lh) ^ row_swizzle(l32)) * 16;
    const int w_frag = L::W_BASE + wn * 8192 + lane * 16;

    f32x16 acc[J][I];                               // [weight tile j][batch tile i]
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int i = 0; i < I; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

    auto load_a = [&](int slot, int c, const int u) {
        load_to_lds<0>(buffer_upto(abase, c < NC ? kAllBytes : 0), lds + slot * L::A_BYTES + (u * 4 + wave) * 1024, a_off[u], c * 128);
    };
    auto load_w = [&](int slot, int h, const int u) {          // half chunk h
        const __amdgpu_buffer_rsrc_t r = buffer_upto(wbase, h < 2 * NC ? kAllBytes : 0);
        char* dst = lds + L::W_BASE + slot * L::W_BYTES + (wave + 4 * (u >> 1)) * 2048;
        if (u & 1) load_to_lds<1024, NT ? 2 : 0>(r, dst, w_off[u >> 1], h * 2048);
        else load_to_lds<0, NT ? 2 : 0>(r, dst, w_off[u >> 1], h * 2048);
    };
    auto frags = [&](auto ni, int as, int ws, int ks, u32x4* af, u32x4* wf) {
        constexpr int NI = decltype(ni)::value;
        if (NI == 0) return;
#pragma unroll
        for (int i = 0; i < NI; ++i) af[i] = *(const u32x4*)(lds + as * L::A_BYTES + a_frag[ks] + i * 32 * 128);
#pragma unroll
        for (int j = 0; j < J; ++j) wf[j] = *(const u32x4*)(lds + ws * L::W_BYTES + w_frag + (j * 2 + (ks & 1)) * 1024);
    };
    u32x4 af[2][I], wf[2][J];
    auto multiply = [&](auto ni, const int b) {                // up and down the batch tiles: one operand stays from one instruction to the next
        constexpr int NI = decltype(ni)::value;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int x = 0; x < NI; ++x) {
                const int i = (j & 1) ? NI - 1 - x : x;
                acc[j][i] = mma32t(wf[b][j], af[b][i], acc[j][i]);
            }
    };
    // The loop runs over halves of a chunk, two k steps each.  In the first the operands of the second are read from LDS; then, when the
    // wave has its operands and what the next half reads has landed, comes the half's one barrier: the weight slot (after a second
    // half the activation slot too) is free, the next half's first operands are read and the slot's next loads issued, three
    // halves (256 rows) or two before they are needed.  The waits count the loads that may still be in flight: per half four of weights
    // and, 256 rows, four of activations (a chunk's two fours after the barriers of the second half three chunks before and of the first
    // half two chunks before), or, 128 rows, four of activations after a second half only.
#pragma unroll
    for (int u = 0; u < AU; ++u) load_a(0, 0, u);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int u = 0; u < 4; ++u) load_w(h, h, u);
#pragma unroll
    for (int u = 0; u < AU; ++u) load_a(1, 1, u);
#pragma unroll
    for (int h = 2; h < L::W; ++h)
#pragma unroll
        for (int u = 0; u < 4; ++u) load_w(h, h, u);
    if (BM == 256)
#pragma unroll
        for (int u = 0; u < 4; ++u) load_a(2, 2, u);
    if (BM == 256) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // Waves of a last row tile that is partly empty multiply the 32-row blocks that there are.
    auto walk = [&](auto ni) {
        constexpr int NI = decltype(ni)::value;
        frags(ni, 0, 0, 0, af[0], wf[0]);
        int as = 0, ws = 0;                                        // the slots being multiplied
        for (int c = 0; c < NC; ++c) {
            const int a_next = as == L::A - 1 ? 0 : as + 1, a_last = as == 0 ? L::A - 1 : as - 1;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int w_next = ws == L::W - 1 ? 0 : ws + 1;
                __builtin_amdgcn_sched_barrier(0);
                frags(ni, as, ws, 2 * h + 1, af[1], wf[1]);
                multiply(ni, 0);
#pragma unroll
                for (int r = 0; NI > 0 && r < NI + J; ++r) {                  // a read behind each of the first products
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, NI == I ? I * J - I - J : 16, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (BM == 256) asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)" ::: "memory");
                else if (h == 0) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                frags(ni, h ? a_next : as, w_next, h ? 0 : 2, af[0], wf[0]);
#pragma unroll
                for (int u = 0; u < 4; ++u) load_w(ws, 2 * c + h + L::W, u);
                if (BM == 256) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (h) load_a(as, c + 3, u);
                        else load_a(a_last, c + 2, 4 + u);
                    }
                } else if (h) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) load_a(as, c + 2, u);
                }
                multiply(ni, 1);
                __builtin_amdgcn_sched_group_barrier(0x100, NI + J, 0);
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    __builtin_amdgcn_sched_group_barrier(0x008, NI == I ? I * J / 8 : 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                ws = w_next;
            }
            as = a_next;
        }
    };
    const int blocks = max(0, min(I, (g.M - m0 - wm * (BM / 2) + 31) >> 5));
    static_assert(BM == 256 || I == 2, "the wave's blocks are two, one or none");
    if (BM == 256 || blocks == I) walk(std::integral_constant<int, I>());
    else if (blocks == 1) walk(std::integral_constant<int, 1>());
    else walk(std::integral_constant<int, 0>());
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();                                  // the operand slots are free for the epilogue
    if (BM == 128 && blocks == 0) return;

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
                __builtin_amdgcn_wave_barrier();         // the rotation rows have been read
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
                } else if (is_k) {                       // 16 rows x 4 groups of 8 d: tokens of a page are neighbours
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
                } else {
                    // V element (d, token) sits at (d/32)*512 + ((token/4)*16 + d%16)*8 + ((d/16)%2)*4 + token%4: four tokens from a multiple of four on, at d
                    // and d + 16, are 16 neighbouring bytes, a lane's here (its d is 32 (lane/16) + lane%16).  Such runs start anywhere in
                    // the tile, as sequences do; the runs cut off at its ends or a sequence's go row by row.  (Two bytes a store, straight from the
                    // accumulators, was 64 stores of 16 pieces each for 32 rows.  us a launch, that -> this: 0.6B shape, 11,206 rows 140 -> 115; 4B, 788 rows 52.6 -> 46.7,
                    // 6,028 rows 217 -> 198, 15,272 rows 480 -> 465; traced, the last layer's k and v alone: 0.6B 83 -> 63, 4B 50 -> 44.5 and 193 -> 164.)
                    const int rows = min(32, g.M - mb);
                    const int2 mine = qa.row_page[min(m, g.M - 1)];
                    const int page_before = __shfl_up(mine.x, 1, 64), run_before = __shfl_up(mine.y >> 2, 1, 64);
                    const bool first = l32 == 0 || mine.x != page_before || (mine.y >> 2) != run_before;
                    uint32_t left = (uint32_t)__builtin_amdgcn_ballot_w64(first && l32 < rows);
                    const char* src = tb + (32 * (lane >> 4) + (lane & 15)) * 2;
                    while (left) {
                        const int r0 = __builtin_ctz(left);
                        left &= left - 1;
                        const int r1 = left ? __builtin_ctz(left) : rows;
                        const int page = __builtin_amdgcn_readlane(mine.x, r0), pos = __builtin_amdgcn_readlane(mine.y, r0);
                        uint16_t* dst = qa.pages + ((size_t)page * qa.n_kv_heads + kvh) * (size_t)(2 * kPageTokens * 128) + kPageTokens * 128 +
                                        (lane >> 4) * 512 + (((((pos & (kPageTokens - 1)) >> 2) * 16) + (lane & 15)) << 3);
                        if (r1 - r0 == 4) {
                            uint32_t x[8];
#pragma unroll
                            for (int t = 0; t < 4; ++t) {
                                x[t] = *(const uint16_t*)(src + (r0 + t) * OROW);
                                x[4 + t] = *(const uint16_t*)(src + (r0 + t) * OROW + 32);
                            }
                            *(u32x4*)dst = u32x4{x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6] | x[7] << 16};
                        } else {
                            for (int r = r0; r < r1; ++r) {
                                const int slot = __builtin_amdgcn_readlane(mine.y, r) & 3;
                                dst[slot] = *(const uint16_t*)(src + r * OROW);
                                dst[4 + slot] = *(const uint16_t*)(src + r * OROW + 32);
                            }
                        }
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        report_saturation(qa.sat_count, bad);
    } else if (TEPI == 3) {
        // A lane holds 64 of the 128 columns of four rows: it folds them, column tile by column tile, and the lane halves
        // merge theirs: one (max, sum exp) pair per row and 128 columns.  The streaming kernel folds in the same order, so
        // that repacked and row-major weights give the same bits.  The exponentials (128 a lane) are 5 % of the tile's
        // matrix time at K = 2560.  Bound by the matrix cores' power: 6,028 rows x 151,936 columns x 2560 take 3.8 to 4.2 ms
        // (1.24 to 1.13 PFLOP/s); the streaming kernel, which fetches twice the bytes per product from L2 and
        // reads twice the LDS per MFMA, took 6.5.
        const int c0 = n0 + wn * 128 + 4 * lh, pair = tile_n * 2 + wn;
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int m = m0 + wm * (BM / 2) + i * 32 + l32;
            const int tgt = m < g.M ? g.targets[m] : -1;
            const int mine = tgt - c0;                                // its place among this lane's columns, if it is one of them
            float mx = -INFINITY, found = 0.f;
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    if (c0 + 32 * j + 8 * (r >> 2) + (r & 3) >= g.N) acc[j][i][r] = -INFINITY;      // padding of the last tile
                    found = mine == 32 * j + 8 * (r >> 2) + (r & 3) ? acc[j][i][r] : found;
                    mx = fmaxf(mx, acc[j][i][r]);
                }
            if (tgt >= 0 && mine >= 0 && mine < 128 && (mine & 4) == 0 && tgt < g.N) g.tgt_logit[m] = found;
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
    } else if (TEPI == 4) {
        // score = logit / T + noise (the sampler's own expression); the best of the wave's 128 columns per row, a second kernel picks
        const int c0 = n0 + wn * 128 + 4 * lh, part = tile_n * 2 + wn;
        const float T = g.s_temperature;
#pragma unroll
        for (int i = 0; i < I; ++i) {
            const int m = m0 + wm * (BM / 2) + i * 32 + l32;
            const uint64_t key = (T > 0.f && m < g.M) ? g.s_keys[m] : 0ull;
            const uint64_t at = noise_at(key, c0);
            float bv = -INFINITY;
            int bi = 0x7FFFFFFF;
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int n = c0 + 32 * j + 8 * (r >> 2) + (r & 3);
                    float sc = acc[j][i][r];
                    if (T > 0.f) sc = sc / T + gumbel_noise(at + (uint64_t)(32 * j + 8 * (r >> 2) + (r & 3)) * kNoiseStep);
                    if (n < g.N && better(sc, n, bv, bi)) { bv = sc; bi = n; }
                }
            const float ov = __shfl_xor(bv, 32, 64);
            const int oi = __shfl_xor(bi, 32, 64);
            if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
            if (lh == 0 && m < g.M && part < g.s_tiles) g.s_part[(size_t)m * g.s_tiles + part] = make_float2(bv, __int_as_float(bi));
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
__global__ __launch_bounds__(256, BM == 128 ? 2 : 1) void gemm_tile_kernel(GemmArgs g, QkvPostArgs qa) { tile_body<TEPI, BM, false>(g, qa); }

// The LM head of a decode step: logits, or with SAMPLE the winners of each 128 columns.  NT: one tile of rows.
template <bool SAMPLE, bool NT>
__global__ __launch_bounds__(256, 2) void head_tile_kernel(GemmArgs g) { tile_body<SAMPLE ? 4 : 0, 128, NT>(g, QkvPostArgs{}); }

template <int TEPI, int BM>
static hipError_t launch_tile_bm(const GemmArgs& a, const QkvPostArgs& qa, hipStream_t s) {
    const int cols = TEPI == 1 ? 128 : 256;
    const int m_tiles = (a.M + BM - 1) / BM;
    const int n_tiles = (a.N + cols - 1) / cols;
    const long long total = (long long)m_tiles * n_tiles * (TEPI == 0 ? a.splits : 1);
    if (total > (1ll << 30)) return hipErrorInvalidValue;
    const int per_xcd = (int)((total + 7) / 8) + 1;          // the two parts of the grid are rounded up by themselves
    const size_t lds_bytes = Slots<BM>::TOTAL;
    hipError_t e = hipFuncSetAttribute((const void*)gemm_tile_kernel<TEPI, BM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((gemm_tile_kernel<TEPI, BM>), dim3(per_xcd * 8), dim3(256), lds_bytes, s, a, qa);
    return hipGetLastError();
}

template <int TEPI>
static hipError_t launch_tile(const GemmArgs& a, const QkvPostArgs& qa, int bm, hipStream_t s) {
    return bm == 128 ? launch_tile_bm<TEPI, 128>(a, qa, s) : launch_tile_bm<TEPI, 256>(a, qa, s);
}

// needs the fragment-ordered weights (a.wf), K % 64 == 0 (% 128 with a split), operands small enough for 32-bit element offsets and
// a tile's own rows (256 of activations, 8 x 32 of weights) within a buffer's 2^31 bytes
bool gemm_tile_usable(const GemmArgs& a) {
    return a.wf != nullptr && a.splits >= 1 && (a.K % (a.splits > 1 ? 128 : BK)) == 0 && a.splits <= std::max(1, a.K >> 7) && (a.N & 3) == 0 &&
           a.K < (1 << 22) && (long long)a.M * a.K < (1ll << 31) && ((long long)a.N + 32) * 2 * a.K < (1ll << 31);
}

// What the K splits, the q/k/v projection's form and the line to the streaming kernel go by: estimated microseconds of one launch
// on 256 x 256 or 128 x 256 tiles (cols: output columns of a tile), rounds over the 256 compute units x (fixed part + 64-wide k
// chunks, which take a third longer on a full chip).  They describe this kernel as it was with operands staged through
// registers, and stay because the order of an output's sums follows from them, for row-major weights (on the streaming kernel, as
// ever) too.  Checked against the kernel as it is, 60 pairs of shape and rows: O and down of the 4B, 0.6B and 7B shapes, 136 to
// 15,272 rows, launch and partial sums, lose nothing to the best of 1, 2, 3 or 6 splits on 41 of the 47 where the choice is one of these, and 4 to 25 %
// of 16 to 55 us on the others; fusing q/k/v's post-processing is right at all 15 row counts but 520 (34 us fused, 41 split).
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

// Which height is faster goes by estimates of the kernel as it is: a fixed part for each of the n tiles of the busiest compute unit, and
// per chunk the root of the squares of what that unit needs (n tall tiles one after the other, or pairs of the others and a
// single one) and of the chip's power for all tiles.  Fitted to 786 launches (the shapes above, gate/up among them, 136 to
// 15,272 rows): 3 % rms.  The tiles' bits are the same.
static float tile_us(long tiles, float chunks, bool swiglu, int bm) {
    const float n = (float)((tiles + 255) / 256), all = (float)tiles / 256.f;
    const float pairs = floorf(n / 2.f), odd = n - 2.f * pairs;
    auto hyp = [](float a, float b) { return sqrtf(a * a + b * b); };
    if (bm == 256) return swiglu ? 11.6f * n + chunks * hyp(0.96f * n, 1.20f * all) : 10.3f * n + chunks * hyp(0.965f * n, 1.35f * all);
    return swiglu ? 3.9f + 1.8f * n + chunks * hyp(1.16f * pairs + 0.64f * odd, 0.69f * all)
                  : 3.4f + 3.3f * n + chunks * hyp(1.03f * pairs + 0.55f * odd, 0.75f * all);
}

// The tile height for a launch, 0 where the streaming kernel takes it.  All three add
// the products of an output in the same order, so the choice never changes a result.  Shapes that the streaming kernel does not
// take (row-major weights go to a kernel with another order there) are tiled only where 256 x 256 tiles fill the chip.
// Gate/up leaves the tall tile for an estimated gain of 7 us.  Tall / not, us (its 256-row form with registers took 6 to 10 % more than tall):
// 8192 x 1024, 520 / 1,000 / 1,600 rows 33 / 38.5 / 68 and 30 / 37 / 61.5 (all tall), 4B shape, 1,000 / 2,100 / 4,200 / 8,000 / 15,272 rows
// 122 / 205 / 407 / 702 / 1264 and 100 / 205 / 359 / 678 / 1286, 7B shape, 1,000 / 1,600 / 3,000 / 8,000 271 / 451 / 691 / 1792 and
// 250 / 392 / 707 / 1830.
int gemm_tile_height(int M, int N, int K, int splits, int cols, int bn) {
    const bool swiglu = cols == 128;
    auto us = [&](int bm) { return tile_us((long)((M + bm - 1) / bm) * ((N + cols - 1) / cols) * splits, K / (float)splits / 64.f, swiglu, bm); };
    if ((K & 127) || (N & 15))
        return M >= 512 && (long)((M + 255) / 256) * ((N + cols - 1) / cols) >= 200 ? 256 : 0;
    const float t256 = gemm_tile_us(M, N, K, splits, cols, 256), t128 = gemm_tile_us(M, N, K, splits, cols, 128);
    const float ts = gemm_stream_us(M, cols == 128 ? 2 * N : N, K, splits, bn == 64 ? 64 : 128);
    if (M <= 128 || ts < std::min(t256, t128)) return 0;
    return us(128) + (swiglu ? 7.f : 0.f) < us(256) ? 128 : 256;
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

// The LM head of a decode step of more than 64 rows and at least 65,536 columns on tiles of 128 rows (two workgroups a compute unit), with
// logits or the sampler's winners.  Bound by the weights' way into the compute units, 4.8 TB/s with non-temporal loads (without, as on the
// streaming kernel, 4.2; zeros for operands change nothing).  Streaming kernel -> this, us, 151,936 columns: logits, K = 2560, 65 / 96 / 128 rows 164 / 173 / 180 ->
// 147 / 154 / 160, K = 1024 74 / 78 / 84 -> 64 / 67 / 71; 65,536 columns, K = 1024 30 / 33 / 35 -> 28 / 31 / 29.  Winners, whose noise keeps the
// vector units busy where nothing else runs: 128 rows, K = 2560 190 -> 180, 3584 244 -> 229, but 1024 101 -> 110, so from K = 2048 on; two row tiles (160 rows), for which the
// streaming kernel reads the weights twice, 1024 / 2560 / 3584 179 / 346 / 464 -> 157 / 259 / 331.  (Logits of more than 128 rows go by gemm_tile_rows().)
// 8,192 columns are too few tiles (160 rows 46 -> 60).
// Only the shapes that the streaming kernel takes: its sums are in the tiles' order, those of gemm_mfma_kernel, which row-major weights of the
// others go to, are not, and repacked weights have to give the same bits.
bool gemm_head_tiled(int M, int N, int K, int epilogue) {
    if (epilogue == EPI_SWIGLU || (K & 127) || (N & 15) || N < 65536 || M <= 64) return false;
    return epilogue == EPI_SAMPLE ? M > 128 || K >= 2048 : M <= 128;
}
bool gemm_head_tile_takes(const GemmArgs& a, int epilogue) {
    return a.head && a.splits == 1 && gemm_head_tiled(a.M, a.N, a.K, epilogue) && gemm_tile_usable(a);
}
template <bool SAMPLE, bool NT>
static hipError_t launch_head_tile_nt(const GemmArgs& a, hipStream_t s) {
    const int tiles = ((a.M + 127) / 128) * ((a.N + 255) / 256);
    const hipError_t e = hipFuncSetAttribute((const void*)head_tile_kernel<SAMPLE, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, Slots<128>::TOTAL);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((head_tile_kernel<SAMPLE, NT>), dim3((tiles + 7) / 8 * 8), dim3(256), Slots<128>::TOTAL, s, a);
    return hipGetLastError();
}
hipError_t launch_gemm_head_tile(const GemmArgs& a, int epilogue, hipStream_t s) {
    if (!gemm_head_tile_takes(a, epilogue)) return hipErrorInvalidValue;
    if (epilogue == EPI_STORE_F32) return launch_head_tile_nt<false, true>(a, s);
    if (!a.s_part || a.s_tiles != (a.N + 127) / 128 || (a.s_temperature > 0.f && !a.s_keys)) return hipErrorInvalidValue;
    return a.M <= 128 ? launch_head_tile_nt<true, true>(a, s) : launch_head_tile_nt<true, false>(a, s);
}

// The LM head with the scoring epilogue: one (max, sum exp) pair per row and 128 columns.
// Tiles of 128 rows: the exponentials run under another workgroup's products.  151,936 columns, K = 2560, 300 / 700 / 1,000 / 3,000
// rows 276 / 510 / 681 / 2012 us against 352 / 518 / 705 / 2022 on 256, K = 1024 113 / 216 / 289 / 839 against 167 / 243 / 340 / 939; 30,004
// columns, K = 256, 700 rows 19 against 29.
hipError_t launch_gemm_tile_score(const GemmArgs& a, hipStream_t s) {
    if (!gemm_tile_usable(a) || a.splits != 1 || !a.s_part || !a.targets || !a.tgt_logit || a.s_tiles != (a.N + 127) / 128) return hipErrorInvalidValue;
    const QkvPostArgs none = {};
    return launch_tile_bm<3, 128>(a, none, s);
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
