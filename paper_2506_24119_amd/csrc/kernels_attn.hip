// GQA attention over the paged KV cache on the gfx950 matrix cores.
//
// Page layout (per layer, page, kv head): K (16 tokens x hd) followed by V (hd x 16 tokens), 16-bit,
// each stored in MFMA operand order (see PageFrag) so that the operands come straight from HBM:
//   S^T[token][row] = sum_d K[token][d] * Q[row][d]     v_mfma_f32_16x16x32_bf16, A = K page (a lane
//                     reads 8 consecutive d of one token), B = the 16 query rows held in registers;
//   O^T[d][row]    += sum_token V^T[d][token] * P^T[token][row]   v_mfma_f32_16x16x16_bf16, A = V page
//                     (a lane reads 4 consecutive tokens of one d), B = P^T, which is exactly the
//                     register layout S^T came out in, so probabilities never leave the lane.
// A decode tile has 16 query rows: the G = Hq/Hkv query heads that share one kv head (padded to
// 16), so K and V are read once per group.
//
// Decode (attn_stream_kernel): the ordered stream of all (row, kv head, page) units of the batch is cut into equal
// ranges, one per workgroup; inside a range the four waves take pages round-robin, each with a private online
// softmax (running max m, sum l, unnormalised O), merged through LDS at the end of every (row, kv head) segment;
// a second small kernel merges the partial (m, l, O) of a pair that spans workgroups.  Batches whose longest pairs do not end much later than
// the rest give every (row, kv head) pair a workgroup instead, small ones every piece of a pair; the last rows of a prefill have pieces of
// a fixed number of pages (DecodeForm).
// Prefill (attn_prefill_kernel): tiles of 32 positions of one head on the 32x32x16 MFMA, four a workgroup, pages in LDS.
// Softmax is evaluated in base 2: scores are scaled by log2(e)/sqrt(hd) and v_exp_f32 is 2^x.
#include <type_traits>

#include "spiral_internal.h"

namespace spiral {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr float kNegBig = -1.0e30f;

// Decode reads every K/V byte once: non-temporal loads keep the stream from displacing q, the block
// tables and the partial results in L2 (measured: 13 us less per launch at C3, -7 % step time).
// Prefill re-reads pages across position tiles and keeps ordinary cached loads.
#ifndef ATTN_NT
#define ATTN_NT 1
#endif
#if ATTN_NT
#define KVLOAD(p) __builtin_nontemporal_load(p)
#else
#define KVLOAD(p) (*(p))
#endif

// q, the cached K/V and the probabilities share the 16-bit activation format (IEEE half by default:
// with bf16's 8 significant bits the attention output alone carries ~0.4 % error per layer)
__device__ __forceinline__ f32x4 mma_qk(const u32x4& k, const u32x4& q, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, k), __builtin_bit_cast(f16x8, q), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mma_pv(const u32x2& v, const u32x2& p, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, v), __builtin_bit_cast(f16x4, p), c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 mma32_f16(const u32x4& x, const u32x4& y, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, x), __builtin_bit_cast(f16x8, y), c, 0, 0, 0);
}

// One (page, kv head) holds K then V, each 16 tokens x HD elements, stored in the order the MFMA
// operand registers want them, so that every wave-wide 16-byte load reads 1 KB of consecutive memory:
//   K element (token t, d):  (d/32)*512 + (((d%32)/8)*16 + t)*8 + d%8
//   V element (d, token t):  (d/32)*512 + ((t/4)*16 + d%16)*8 + ((d/16)%2)*4 + t%4
template <int HD>
struct PageFrag {
    u32x4 k[HD / 32];     // K: lane = (d%32)/8 * 16 + token, 8 consecutive d
    u32x4 v[HD / 32];     // V: lane = (t/4)*16 + d%16; .xy = 4 tokens of d-tile 2m, .zw = of d-tile 2m+1
};

template <int HD>
__device__ __forceinline__ void load_page(PageFrag<HD>& f, const uint16_t* kp, int lane, bool real) {
    // !real: every lane reads the first 16 bytes of the page (a valid address, one cache line)
    const uint16_t* vp = kp + kPageTokens * HD;
    const int off = real ? lane * 8 : 0;
    const int step = real ? 512 : 0;
#pragma unroll
    for (int ks = 0; ks < HD / 32; ++ks) f.k[ks] = KVLOAD((const u32x4*)(kp + ks * step + off));
#pragma unroll
    for (int mp = 0; mp < HD / 32; ++mp) f.v[mp] = KVLOAD((const u32x4*)((real ? vp : kp) + mp * step + off));
}

// One (row, query head) by one wave, token by token, nothing read of a token that the row does not see: a lane scores one token
// of 64, then holds one dimension (of 128: two).  For rows whose sums met a NaN only; speed does not matter.
template <int HD, bool ACT32>
__device__ __forceinline__ void prefill_row_alone(const AttnArgs& a, const int32_t* bt, const uint16_t* head_pages, size_t page_elems, size_t out_row,
                                                  int last, int lane) {
    constexpr int DL = (HD + 63) / 64;
    const uint16_t* q = a.q + out_row * HD;
    float m_run = kNegBig, l_run = 0.f, o[DL];
#pragma unroll
    for (int j = 0; j < DL; ++j) o[j] = 0.f;
    for (int t0 = 0; t0 <= last; t0 += 64) {
        const int t = t0 + lane;
        float sc = -INFINITY;
        if (t <= last) {
            const uint16_t* kp = head_pages + (size_t)bt[t >> 4] * page_elems + (t & 15) * 8;
            sc = 0.f;
#pragma unroll 1
            for (int d = 0; d < HD; d += 8) {
                const f16x8 kv = *(const f16x8*)(kp + (d >> 5) * 512 + ((d & 31) >> 3) * 128), qv = *(const f16x8*)(q + d);
#pragma unroll
                for (int e = 0; e < 8; ++e) sc = fmaf((float)kv[e], (float)qv[e], sc);
            }
            sc *= a.scale_log2e;
        }
        float mx = sc;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        const float m_new = fmaxf(m_run, mx), alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        const float p = __builtin_amdgcn_exp2f(sc - m_new), ph = (float)(_Float16)p;
        l_run = l_run * alpha + wave_sum(p);
        m_run = m_new;
#pragma unroll
        for (int j = 0; j < DL; ++j) o[j] *= alpha;
#pragma unroll 1
        for (int i = 0; i < 64 && t0 + i <= last; ++i) {
            const int ti = t0 + i;
            const uint16_t* vp = head_pages + (size_t)bt[ti >> 4] * page_elems + kPageTokens * HD + ((ti & 15) >> 2) * 128 + (ti & 3);
            const float pi = __shfl(ph, i, 64);
#pragma unroll
            for (int j = 0; j < DL; ++j) {
                const int d = (lane + 64 * j) & (HD - 1);
                o[j] = fmaf(pi, (float)__builtin_bit_cast(_Float16, vp[(d >> 5) * 512 + (d & 15) * 8 + ((d >> 4) & 1) * 4]), o[j]);
            }
        }
    }
    const float inv = 1.0f / l_run;
#pragma unroll
    for (int j = 0; j < DL; ++j)
        if (lane + 64 * j < HD) {
            const int r = (int)(out_row / a.n_q_heads), col = (int)(out_row % a.n_q_heads) * HD + lane + 64 * j;
            ActStore<ACT32>::put(a.out, a.out_frag ? act_frag(r, col, a.n_rows, a.n_q_heads * HD) : out_row * HD + lane + 64 * j, o[j] * inv);
        }
}

// Grid of the prefill kernel: x = position blocks of eight pairs, y = groups of eight (sequence, kv head, head group) pairs.
// Everything a workgroup would divide for comes from the host, as a whole number or as a reciprocal: seven integer divisions in a
// row, and four look-ups one after the other, were half a microsecond of a launch before its first load.  Runs of 5 tokens without a
// history, 16 heads: 5.9 -> 5.2 us a launch (1.5 of it empty, 0.4 the look-ups, 1.2 the pages and q, 0.8 the step, 1.3 the output: few
// instructions, all of them fetched for the first time); 65 tokens, 32 heads 11.7 -> 10.1 with the events around it.
struct Reciprocal {
    uint32_t m;                                               // ceil(2^32 / d), 0 for d = 1
    __device__ __forceinline__ int of(int n) const { return m ? (int)__umulhi((uint32_t)n, m) : n; }      // n / d where n * d < 2^32
};
static Reciprocal reciprocal(int d) { return Reciprocal{d > 1 ? (uint32_t)(((1ull << 32) + d - 1) / d) : 0u}; }
struct PrefillGrid {
    int32_t pairs, group, heads_wg, head_groups, tiles;       // group: query heads per kv head; tiles: position tiles of a workgroup
    Reciprocal by_groups, by_kv_heads;                        // 1 / head_groups, 1 / n_kv_heads
};

// ---------------------------------------------------------------------------------------------
// Causal prefill attention.  A wave's tile is 32 consecutive positions of one query head, each row with its own causal
// limit; a workgroup holds four tiles that share a kv head: up to four heads of the group, or with groups of one or two
// heads also two or four consecutive position tiles.  The pages of 64 tokens (K and V, in their memory order) are
// copied to LDS by all four waves, double buffered, the next 64 tokens in flight in registers meanwhile; every wave
// then takes its operands from there:
//   S^T[token][row] = K q^T    v_mfma_f32_32x32x16, A = 32 tokens x 16 d of two pages, B = the query rows in registers;
//   O^T[d][row]    += V^T P^T  v_mfma_f32_32x32x16 over the 16 tokens of a page.  In S^T a lane holds the tokens
//                   4 lh .. + 3 and 8 + 4 lh .. + 3 of its row: they are the B operand as they are, and the A operand is
//                   read with the same order of the contraction index (two 8-byte groups of 4 tokens).
// Bound: a wave's own chain.  A 64-token step is 32 MFMAs (1024 cycles) and about 200 vector operations a lane (~1000, the
// exponentials half of them), in series but for the exponentials of a page under the products of the one before, then a barrier; two
// workgroups per compute unit hide half of it (matrix pipe busy 35 %, at 1.95 GHz; with zeros for q, k and v 15 % less time).
// Against 16-row tiles that walk single pages straight from L2 (16x16 MFMAs, no LDS), a layer of: 15,272 rows of U[256, 1024]
// tokens, 32 heads 353 -> 143 us; 11,206 rows of U[2048, 4096], 16 heads 484 -> 189 us (0.68 PFLOP/s); 788 rows appended to nine
// histories of U[400, 2000] 122 -> 61 us.  Of that, 175 -> 143, 213 -> 189 and 73 -> 61 came with unmasked steps in a loop of their
// own, K operands four reads ahead, rescaling only after a growth of 2^8, V reads without bank conflicts (a third of the LDS
// cycles; 4-byte stores to go with them cost more than they gave on short runs, 175 -> 208) and whole rows written through LDS.
// Without effect: the two score chains interleaved, sequences sorted by length, s_setprio around the scores (199 -> 204), two
// stages of pages in flight in registers (spills, 213 -> 233).
// ---------------------------------------------------------------------------------------------
template <int HD, bool ACT32>
__global__ __launch_bounds__(256, 2) void attn_prefill_kernel(AttnArgs a, PrefillGrid gr) {
    constexpr int KS = HD / 16, DT = HD / 32;
    constexpr int PAGE_B = 2 * kPageTokens * HD * 2;          // bytes of one (page, kv head): K then V
    constexpr int STAGE_B = 4 * PAGE_B;                       // 64 tokens
    constexpr int LD = PAGE_B / 1024;                         // 16-byte loads of a lane per page
    extern __shared__ float lds_f[];
    char* lds = (char*)lds_f;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, lh = lane >> 5;

    // blocks of one (sequence, kv head) run on one XCD (its L2 keeps the pages); the longest rows start first
    const int pair = blockIdx.y * 8 + (blockIdx.x & 7);
    if (pair >= gr.pairs) return;
    const int qb = (int)((gridDim.x - 1 - blockIdx.x) >> 3);
    const int seq_head = gr.by_groups.of(pair), hg = pair - seq_head * gr.head_groups;
    const int b = gr.by_kv_heads.of(seq_head), kvh = seq_head - b * a.n_kv_heads;
    const int r_first = a.cu_rows[b], r_end = a.cu_rows[b + 1];
    const int pos_base = a.base_pos[b], seq = a.seq_ids[b];   // position of the run's first row; requested together
    const int tiles = gr.tiles;                               // position tiles of the workgroup
    const int n_in_seq = r_end - r_first;
    const int first = qb * tiles * 32;                        // first position of the workgroup, counted from the run's start
    if (first >= n_in_seq) return;
    const int hw = tiles == 4 ? 0 : (tiles == 2 ? wave & 1 : wave), tile = tiles == 4 ? wave : (tiles == 2 ? wave >> 1 : 0);
    const int my_first = first + tile * 32;
    const int n_valid = min(32, n_in_seq - my_first);         // rows of this wave (<= 0: none)
    const bool active = hw < gr.heads_wg && hg * gr.heads_wg + hw < gr.group && n_valid > 0;
    const int h = kvh * gr.group + min(hg * gr.heads_wg + hw, gr.group - 1);
    const int row0 = r_first + my_first;
    const int pos0 = pos_base + my_first;
    const int limit = active && l32 < n_valid ? pos0 + l32 : -1;
    const int my_last = active ? pos0 + n_valid - 1 : -1;     // last visible position of the wave
    const int last = pos_base + min(first + tiles * 32, n_in_seq) - 1;       // ... of the workgroup
    const int last_page = last / kPageTokens;
    const int n_stages = last / 64 + 1;

    const int32_t* bt = a.block_table + (size_t)seq * a.max_blocks;
    const size_t page_elems = (size_t)a.n_kv_heads * (2 * kPageTokens * HD);
    const uint16_t* head_pages = a.pages + (size_t)kvh * (2 * kPageTokens * HD);

    // staging: wave w copies page 4 * stage + w (past the last page: that one again); pages are looked up a stage ahead of their load (a
    // scalar load and the LDS reads share a counter)
    u32x4 rg[LD];
    auto page_of = [&](int stage) { return bt[min(stage * 4 + wave, last_page)]; };
    auto load = [&](int page) {
        const uint16_t* src = head_pages + (size_t)page * page_elems + lane * 8;
#pragma unroll
        for (int u = 0; u < LD; ++u) rg[u] = *(const u32x4*)(src + u * 512);
    };
    auto park = [&](char* buf) {
#pragma unroll
        for (int u = 0; u < LD; ++u) *(u32x4*)(buf + wave * PAGE_B + u * 1024 + lane * 16) = rg[u];
    };
    load(page_of(0));
    int next_page = page_of(1);

    u32x4 qf[KS];
    {
        const bool real = active && l32 < n_valid;
        const uint16_t* qptr = a.q + ((size_t)(real ? row0 + l32 : r_first) * a.n_q_heads + h) * HD + lh * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const u32x4 v = *(const u32x4*)(qptr + ks * 16);
            qf[ks] = real ? v : u32x4{0u, 0u, 0u, 0u};
        }
    }
    f32x16 acc[DT];
#pragma unroll
    for (int d = 0; d < DT; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[d][r] = 0.f;
    float m_run = kNegBig, l_run = 0.f;

    // operand offsets: K of tokens 32 sub + l32 (two pages), V of d = 32 dt + l32 / 2 + 16 (l32 % 2) (4 tokens: 8 bytes).  With d in
    // the lanes' order sixteen lanes would read every other 8 bytes of 256, two to a bank.
    const int k_off = (l32 >> 4) * PAGE_B + lh * 256 + (l32 & 15) * 16;
    const int v_off = PAGE_B / 2 + lh * 256 + l32 * 8;

    // one step of a wave over the first NP pages of the staged four
    auto step = [&](const char* buf, int st, auto np) {
        constexpr int NP = decltype(np)::value, NS = (NP + 1) / 2, NR = NP == 1 ? 8 : 16;      // NR: scores of a lane per 32 tokens
        f32x16 s[NS];
#pragma unroll
        for (int sub = 0; sub < NS; ++sub) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[sub][r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const u32x4 kf = *(const u32x4*)(buf + sub * 2 * PAGE_B + k_off + (ks >> 1) * 1024 + (ks & 1) * 512);
                s[sub] = mma32_f16(kf, qf[ks], s[sub]);
            }
        }
        if (st * 64 + 63 > pos0) {                            // some row of the wave does not see all 64 tokens
#pragma unroll
            for (int sub = 0; sub < NS; ++sub)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (st * 64 + sub * 32 + 8 * (r >> 2) + 4 * lh + (r & 3) > limit) s[sub][r] = -INFINITY;
        }
        float mx = s[0][0];
#pragma unroll
        for (int sub = 0; sub < NS; ++sub)
#pragma unroll
            for (int r = 0; r < NR; ++r) mx = fmaxf(mx, s[sub][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx * a.scale_log2e);
        float ps = 0.f;
        u32x4 pb[NP];                                              // P^T of the pages
#pragma unroll
        for (int sub = 0; sub < NS; ++sub)
#pragma unroll
            for (int b2 = 0; b2 < NR / 4; ++b2) {
                f16x4 h4;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[sub][4 * b2 + e], a.scale_log2e, -m_new));
                    ps += p;
                    h4[e] = (_Float16)p;                      // in [0, 1]: no range to check
                }
                const u32x2 hb = __builtin_bit_cast(u32x2, h4);
                pb[2 * sub + (b2 >> 1)][2 * (b2 & 1)] = hb.x;
                pb[2 * sub + (b2 >> 1)][2 * (b2 & 1) + 1] = hb.y;
            }
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        l_run = l_run * alpha + ps;
        if (__builtin_amdgcn_ballot_w64(m_new != m_run) != 0) {
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[d][r] *= alpha;
        }
        m_run = m_new;
#pragma unroll
        for (int pg = 0; pg < NP; ++pg)
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                const char* vp = buf + pg * PAGE_B + v_off + d * 1024;
                const u32x2 lo = *(const u32x2*)vp, hi = *(const u32x2*)(vp + 512);
                acc[d] = mma32_f16(u32x4{lo.x, lo.y, hi.x, hi.y}, pb[pg], acc[d]);
            }
    };
    // the same over all four pages, none of whose tokens is hidden from a row of the wave
    auto whole_step = [&](const char* buf) {
        constexpr int KD = 4;                                 // K operands ahead
        f32x16 s[2];
        u32x4 kf[KD];
        auto read_k = [&](int i) { return *(const u32x4*)(buf + (i / KS) * 2 * PAGE_B + k_off + ((i % KS) >> 1) * 1024 + (i & 1) * 512); };
        auto read_v = [&](int i) {
            const char* vp = buf + (i / DT) * PAGE_B + v_off + (i % DT) * 1024;
            const u32x2 lo = *(const u32x2*)vp, hi = *(const u32x2*)(vp + 512);
            return u32x4{lo.x, lo.y, hi.x, hi.y};
        };
#pragma unroll
        for (int i = 0; i < KD; ++i) kf[i] = read_k(i);
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[sub][r] = 0.f;
        __builtin_amdgcn_sched_barrier(0);                    // left alone, the scheduler puts every read right before its use
#pragma unroll
        for (int i = 0; i < 2 * KS; ++i) {
            s[i / KS] = mma32_f16(kf[i % KD], qf[i % KS], s[i / KS]);
            if (i + KD < 2 * KS) kf[i % KD] = read_k(i + KD);
            __builtin_amdgcn_sched_barrier(0);
        }
        u32x4 vf[DT];                                         // the first page's V arrives under the exponentials
#pragma unroll
        for (int i = 0; i < DT; ++i) vf[i] = read_v(i);
        float mx = s[0][0];
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sub][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        // The weights are relative to m_run, which follows the row's maximum only when that has left it behind by 2^8: 32 rows raise
        // their maxima in most steps, and the accumulators' 64 products are a quarter of the vector operations.  A weight of up
        // to 256 is as exact in half as one of up to 1.
        const float m_new = fmaxf(m_run, mx * a.scale_log2e);
        if (__builtin_amdgcn_ballot_w64(m_new > m_run + 8.0f) != 0) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
            for (int d = 0; d < DT; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[d][r] *= alpha;
            l_run *= alpha;
            m_run = m_new;
        }
        float ps = 0.f;
#pragma unroll
        for (int pg = 0; pg < 4; ++pg) {
            u32x4 pb;                                         // P^T of the page
#pragma unroll
            for (int b2 = 0; b2 < 2; ++b2) {
                f16x4 h4;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[pg >> 1][8 * (pg & 1) + 4 * b2 + e], a.scale_log2e, -m_run));
                    ps += p;
                    h4[e] = (_Float16)p;
                }
                const u32x2 hb = __builtin_bit_cast(u32x2, h4);
                pb[2 * b2] = hb.x;
                pb[2 * b2 + 1] = hb.y;
            }
#pragma unroll
            for (int d = 0; d < DT; ++d) {
                acc[d] = mma32_f16(vf[d], pb, acc[d]);
                if (pg < 3) vf[d] = read_v((pg + 1) * DT + d);
            }
        }
        l_run += ps;
    };
    // Stages that every row of the workgroup sees in full: a step without a mask, in a loop of its own.  (With the three forms of a
    // step in one loop the accumulators were copied twice a step, and the registers of the copies left two operand reads in flight.)
    // Waves without rows multiply zeros along.
    const int n_whole = min((pos_base + first + 1) / 64, n_stages);
    int st = 0;
    for (; st < n_whole; ++st) {
        char* buf = lds + (st & 1) * STAGE_B;
        park(buf);
        __syncthreads();            // one barrier a step: the buffer written next was last read before this one
        load(next_page);            // past the last stage: its last page again
        whole_step(buf);
        next_page = page_of(st + 2);
    }
    for (; st < n_stages; ++st) {
        char* buf = lds + (st & 1) * STAGE_B;
        park(buf);
        __syncthreads();
        if (st + 1 < n_stages) {
            load(next_page);
            next_page = page_of(st + 2);
        }
        if (st * 64 + 32 <= my_last) step(buf, st, std::integral_constant<int, 4>());
        else if (st * 64 + 16 <= my_last) step(buf, st, std::integral_constant<int, 2>());
        else if (st * 64 <= my_last) step(buf, st, std::integral_constant<int, 1>());
    }

    // O^T[d][row]: lane (l32, lh) holds rows 8 b + 4 lh .. + 3 of each tile of 32 d; l is spread over the two lane halves
    l_run += __shfl_xor(l_run, 32, 64);
    bool nan = false;
    constexpr int OROW = HD * 2 + 16;
    static_assert(4 * 32 * OROW <= 2 * STAGE_B, "the output rows of four waves take the staged pages' place");
    char* rows_out = lds + wave * (32 * OROW);
    __syncthreads();                                          // every wave is done with the staged pages
    if (active && l32 < n_valid) {
        const float inv = 1.0f / l_run;
        f32x16 sum = acc[0];                                  // NaN where one is among its terms; far from overflow
#pragma unroll
        for (int d = 1; d < DT; ++d) sum += acc[d];
        float s1 = sum[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) s1 += sum[r];
        nan = s1 != s1;
        // Row i = 8 b2 + 4 lh + e of a tile is d = i / 2 + 16 (i % 2): a lane has two neighbours at 4 b2 + 2 lh and two 16 on.  Half
        // precision: the lane halves swap, so that one has four from 4 b2 on and the other the four 16 on, and the rows go out
        // through LDS, whole.
        const size_t o_idx = ((size_t)(row0 + l32) * a.n_q_heads + h) * HD;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
            for (int b2 = 0; b2 < 4; ++b2) {
                float o[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = acc[d][4 * b2 + e] * inv;
                if (ACT32) {
                    float* at = (float*)a.out + o_idx + d * 32 + b2 * 4 + lh * 2;
                    *(float2*)at = make_float2(o[0], o[2]);
                    *(float2*)(at + 16) = make_float2(o[1], o[3]);
                } else {                                      // the range as f32_to_act16 has it; a NaN is stored again below
                    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_fmed3f(o[e], -65504.0f, 65504.0f);
                    const uint32_t even = __builtin_bit_cast(uint32_t, f16x2{(_Float16)o[0], (_Float16)o[2]});
                    const uint32_t odd = __builtin_bit_cast(uint32_t, f16x2{(_Float16)o[1], (_Float16)o[3]});
                    const auto both = __builtin_amdgcn_permlane32_swap(even, odd, false, false);
                    *(u32x2*)(rows_out + l32 * OROW + (d * 32 + b2 * 4 + lh * 16) * 2) = u32x2{both[0], both[1]};
                }
            }
    }
    if (!ACT32) {
        constexpr int LPR = HD / 8;                           // lanes of 16 bytes to a row
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int ps = 0; ps < 32 * LPR / 64; ++ps) {
            const int row = ps * (64 / LPR) + lane / LPR;
            if (active && row < n_valid) {
                const size_t at = a.out_frag ? act_frag(row0 + row, h * HD + (lane % LPR) * 8, a.n_rows, a.n_q_heads * HD)
                                             : ((size_t)(row0 + row) * a.n_q_heads + h) * HD + (lane % LPR) * 8;
                *(u32x4*)((uint16_t*)a.out + at) = *(const u32x4*)(rows_out + row * OROW + (lane % LPR) * 16);
            }
        }
    }
    // A weight of zero does not stop a NaN: one in the V of a token that a row does not see (up to 63 further on in the row's
    // last 64) has reached its sums.  Such rows, and rows with a NaN of their own, are done again over their visible tokens only.
    const uint64_t lanes = __builtin_amdgcn_ballot_w64(nan);
    for (uint32_t rows = (uint32_t)lanes | (uint32_t)(lanes >> 32); rows; rows &= rows - 1) {
        const int row = __builtin_ctz(rows);
        prefill_row_alone<HD, ACT32>(a, bt, head_pages, page_elems, (size_t)(row0 + row) * a.n_q_heads + h, pos0 + row, lane);
    }
}

// ---------------------------------------------------------------------------------------------
// Decode attention as one balanced stream over all (row, kv head, page) units of the batch.
//
// The units are ordered by (row, kv head, page); row_page_start[] is the prefix sum of the rows'
// page counts, so unit u of row r is u - row_page_start[r] * Hkv = kvh * pages(r) + page.  Workgroup
// w owns units [w * U, (w + 1) * U): every workgroup streams the same number of pages whatever the
// mix of sequence lengths, and a workgroup's range is cut into segments at (row, kv head)
// boundaries.  Within a segment the four waves take pages round-robin; at the end
// of a segment they merge through LDS and write one partial (m, l, O) into slot
// (row, kv head, w - first workgroup of that pair).  While a wave finishes a segment its first page of
// the next segment is already in flight and the next query rows are loaded under the merge, so the
// page stream does not stop at segment boundaries (a workgroup per chunk pays a start-up and a
// drain for every 16 pages: 5.2 vs 5.9 TB/s measured).
// ---------------------------------------------------------------------------------------------
// FORM (a parameter of the template, since the test at run time costs the stream 8 registers and with them a workgroup of three a CU:
// 128 rows of 1,280 tokens, 7 % of a step):
//   DECODE_PAIR: a workgroup has one pair to itself and writes the output: no search, no partial results, no merging launch; the longest
//   pairs start first.  For contexts of up to 512 tokens (256 with few pairs) and, with heads of 128, thousands, wherever the estimated
//   end, when too few workgroups are left, costs less than that (decode_in_pairs()).  27 rows of 400 tokens, 0.6B shape: 6 us a layer less of 51.
//   DECODE_PIECES: the last rows of a prefill, and small batches: workgroup (x, y) has the y-th piece of pair x, if there is one, and
//   writes the pair's part y: no search, and one pair only.  Small batches are cut where the equal ranges cut them (a workgroup that would have
//   crossed from one pair to the next is two here), so that the two forms give the same bits.  A prefill's last rows (own_cut) are cut from each
//   pair's first page on: there the order of the sums follows from their own context, not from the call's others.
template <int HD, bool ACT32, int FORM>
__global__ __launch_bounds__(256) void attn_stream_kernel(AttnArgs a) {
    constexpr int KS = HD / 32, MT = HD / 16, OSTRIDE = HD + 4;
    constexpr bool STREAM = FORM == DECODE_STREAM;
    extern __shared__ float lds_f[];
    const int G = a.n_q_heads / a.n_kv_heads;
    const int Hkv = a.n_kv_heads;
    float* s_o = lds_f;                         // [4][G][OSTRIDE]
    float* s_m = s_o + 4 * G * OSTRIDE;         // [4][16]
    float* s_l = s_m + 64;                      // [4][16]

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lg = lane >> 4;
    const int U = a.units_per_wg;
    const int32_t* rps = a.row_page_start;
    const int T = a.total_units;
    int u = blockIdx.x * U;
    if (STREAM && u >= T) return;
    int u_end = min(u + U, T);

    struct Seg { int r, kvh, p0, p1, np, rs, pos; const int32_t* bt; };
    Seg cur;
    if (STREAM) {
        // the row that holds unit u: the largest r with row_page_start[r] * Hkv <= u.  The prefix sums
        // increase strictly, so r + 1 is the number of entries that satisfy it: the lanes test 64 entries
        // at a time (one round of independent loads instead of a chain of dependent ones).
        int below = 0;
        for (int base = 0; base < a.n_rows; base += 64) {
            const int j = min(base + lane, a.n_rows - 1);
            const bool hit = base + lane < a.n_rows && rps[j] * Hkv <= u;
            below += __builtin_popcountll(__builtin_amdgcn_ballot_w64(hit));
        }
        cur.r = __builtin_amdgcn_readfirstlane(below) - 1;
        cur.rs = rps[cur.r];
        cur.np = rps[cur.r + 1] - cur.rs;
        cur.pos = a.row_pos[cur.r];
        cur.kvh = (u - cur.rs * Hkv) / cur.np;
        cur.p0 = (u - cur.rs * Hkv) % cur.np;
    } else {
        // (the row, position and sequence as arguments by value instead: the larger launches cost the host more, 0.3 us each, than the
        // look-ups cost here; one row of a 0.6B model 938 -> 966 us a step)
        const int i = blockIdx.x / Hkv;
        cur.r = FORM == DECODE_PAIR && a.order ? a.order[i] : i;
        cur.rs = 0;
        cur.pos = a.row_pos[cur.r];
        cur.np = cur.pos / kPageTokens + 1;
        cur.kvh = blockIdx.x % Hkv;
        cur.p0 = 0;
        u_end = cur.np;
        if (FORM == DECODE_PIECES) {
            const int start = a.own_cut ? 0 : rps[cur.r] * Hkv + cur.kvh * cur.np;
            const int from = (start / U + (int)blockIdx.y) * U - start;
            cur.p0 = max(from, 0);
            u_end = from + U;
            if (cur.p0 >= cur.np) return;        // the longest pair has more pieces
        }
        u = cur.p0;
    }
    cur.p1 = min(cur.np, cur.p0 + (u_end - u));
    cur.bt = a.block_table + (size_t)a.row_seq[cur.r] * a.max_blocks;

    const size_t page_elems = (size_t)Hkv * (2 * kPageTokens * HD);
    constexpr int head_elems = 2 * kPageTokens * HD;

    u32x4 qf[KS];
    f32x4 acc[MT];
    float m_run, l_run;
    int limit;
    auto load_q = [&](const Seg& sg) {
        // rows >= G of the tile are padding: they read row 0's vector and are zeroed
        const uint16_t* qp = a.q + ((size_t)sg.r * a.n_q_heads + sg.kvh * G + (li < G ? li : 0)) * HD + lg * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const u32x4 v = *(const u32x4*)(qp + ks * 32);
            qf[ks] = li < G ? v : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto reset = [&](const Seg& sg) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run = kNegBig; l_run = 0.f; limit = sg.pos;
    };
    auto step = [&](const PageFrag<HD>& f, int pi) {
#include "attn_page_step.inc"
    };


    PageFrag<HD> cur_f, nxt_f;
    bool have = cur.p0 + wave < cur.p1;         // cur_f holds (or is being loaded with) this wave's first page of `cur`
    load_page<HD>(cur_f, a.pages + (size_t)cur.bt[have ? cur.p0 + wave : cur.p0] * page_elems + (size_t)cur.kvh * head_elems,
                  lane, have);
    load_q(cur);
    reset(cur);

    while (true) {
        // ---- where the next segment starts (if this workgroup has one)
        const int u_next = u + (cur.p1 - cur.p0);
        const bool has_next = STREAM && u_next < u_end;
        Seg nxt = cur;
        if (has_next) {                          // cur ended at the last page of its pair
            if (cur.kvh + 1 < Hkv) {
                nxt.kvh = cur.kvh + 1;
            } else {
                nxt.r = cur.r + 1;
                nxt.kvh = 0;
                nxt.rs = cur.rs + cur.np;
                nxt.np = rps[nxt.r + 1] - nxt.rs;
                nxt.pos = a.row_pos[nxt.r];
                nxt.bt = a.block_table + (size_t)a.row_seq[nxt.r] * a.max_blocks;
            }
            nxt.p0 = 0;
            nxt.p1 = min(nxt.np, u_end - u_next);
        }
        const int pn0 = nxt.p0 + wave;
        const bool cross = has_next && pn0 < nxt.p1;

        // ---- this wave's pages of the segment, the following page always in flight
        if (have) {
            int pi = cur.p0 + wave;
            while (true) {
                const int pn = pi + 4;
                const bool more = pn < cur.p1;
                const bool real = more || cross;
                const int32_t* btp = more ? cur.bt : nxt.bt;
                const int idx = more ? pn : (cross ? pn0 : nxt.p0);      // nxt.p0 is a valid entry (nxt = cur without a successor)
                const int kv = more ? cur.kvh : nxt.kvh;
                load_page<HD>(nxt_f, a.pages + (size_t)btp[idx] * page_elems + (size_t)kv * head_elems, lane, real);
                step(cur_f, pi);
                cur_f = nxt_f;
                if (!more) break;
                pi = pn;
            }
        } else if (cross) {
            load_page<HD>(cur_f, a.pages + (size_t)nxt.bt[pn0] * page_elems + (size_t)nxt.kvh * head_elems, lane, true);
        }

        // ---- merge the four waves and write this segment's partial result
        l_run += __shfl_xor(l_run, 16, 64);
        l_run += __shfl_xor(l_run, 32, 64);
        const float m_fin = m_run, l_fin = l_run;
        f32x4 o_fin[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) o_fin[mt] = acc[mt];
        if (has_next) { load_q(nxt); reset(nxt); }     // the query rows of the next segment arrive under the merge

        __syncthreads();                               // the previous segment's merge has been read
        if (lg == 0) { s_m[wave * 16 + li] = m_fin; s_l[wave * 16 + li] = l_fin; }
        if (li < G) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                *(float4*)&s_o[(wave * G + li) * OSTRIDE + mt * 16 + lg * 4] =
                    make_float4(o_fin[mt].x, o_fin[mt].y, o_fin[mt].z, o_fin[mt].w);
        }
        __syncthreads();
        {
            const int slot = STREAM ? blockIdx.x - (cur.rs * Hkv + cur.kvh * cur.np) / U : blockIdx.y;
            float* dst0 = a.part + (((size_t)cur.r * Hkv + cur.kvh) * a.n_chunks + slot) * G * (HD + 2);
            for (int e = threadIdx.x; e < G * HD; e += 256) {
                const int j = e / HD, i = e % HD;
                const float M = fmaxf(fmaxf(s_m[j], s_m[16 + j]), fmaxf(s_m[32 + j], s_m[48 + j]));
                float L = 0.f, O = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float sc = __builtin_amdgcn_exp2f(s_m[w * 16 + j] - M);
                    L += s_l[w * 16 + j] * sc;
                    O += s_o[(w * G + j) * OSTRIDE + i] * sc;
                }
                if (FORM == DECODE_PAIR) {
                    const int h = cur.kvh * G + j;
                    ActStore<ACT32>::put(a.out, a.out_frag ? act_frag(cur.r, h * HD + i, a.n_rows, a.n_q_heads * HD)
                                                           : ((size_t)cur.r * a.n_q_heads + h) * HD + i, O / L);
                    continue;
                }
                float* dst = dst0 + (size_t)j * (HD + 2);
                dst[i] = O;
                if (i == 0) { dst[HD] = M; dst[HD + 1] = L; }
            }
        }
        if (!has_next) break;
        u = u_next;
        cur = nxt;
        have = cross;
    }
}

// Merge the partial results of one (row, query head) written by attn_stream_kernel: one wave, a lane holds VEC neighbouring
// dimensions.  PRE parts are requested at once (past the end: the last one again, not counted): a loop that waits for each costs
// 0.45 us a part (1,450 tokens in 4-page pieces 10.8 us, eight at a time 3.4).  Four where no pair has more: further requests only
// repeat the last part.
template <int HD, bool ACT32, int PRE>
__global__ __launch_bounds__(64) void attn_stream_combine_kernel(AttnArgs a) {
    constexpr int VEC = HD >= 128 ? 2 : 1;
    const int r = blockIdx.x, h = blockIdx.y, i = threadIdx.x * VEC;
    if (i >= HD) return;
    const int G = a.n_q_heads / a.n_kv_heads, Hkv = a.n_kv_heads;
    const int kvh = h / G, j = h % G;
    const int rs = a.row_page_start[r], np = a.row_page_start[r + 1] - rs;
    const int start = a.own_cut ? 0 : rs * Hkv + kvh * np;
    const int first = start / a.units_per_wg;
    const int last = (start + np - 1) / a.units_per_wg;
    const int n_parts = last - first + 1;
    const float* base = a.part + (((size_t)r * Hkv + kvh) * a.n_chunks * G + j) * (HD + 2);       // a part is HD + 2 floats: 8-byte aligned
    const size_t cstride = (size_t)G * (HD + 2);
    float M = kNegBig, L = 0.f, O[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) O[e] = 0.f;
    for (int c0 = 0; c0 < n_parts; c0 += PRE) {
        float pm[PRE], pl[PRE], po[PRE][VEC];
#pragma unroll
        for (int c = 0; c < PRE; ++c) {
            const float* src = base + (size_t)min(c0 + c, n_parts - 1) * cstride;
            const float2 ml = *(const float2*)(src + HD);
            pm[c] = ml.x; pl[c] = ml.y;
            if (VEC == 2) {
                const float2 o = *(const float2*)(src + i);
                po[c][0] = o.x; po[c][VEC - 1] = o.y;
            } else po[c][0] = src[i];
        }
        float m_new = M;
#pragma unroll
        for (int c = 0; c < PRE; ++c)
            if (c0 + c < n_parts) m_new = fmaxf(m_new, pm[c]);
        if (c0 > 0) {
            const float sc = __builtin_amdgcn_exp2f(M - m_new);
            L *= sc;
#pragma unroll
            for (int e = 0; e < VEC; ++e) O[e] *= sc;
        }
        M = m_new;
#pragma unroll
        for (int c = 0; c < PRE; ++c)
            if (c0 + c < n_parts) {
                const float sc = __builtin_amdgcn_exp2f(pm[c] - M);
                L += pl[c] * sc;
#pragma unroll
                for (int e = 0; e < VEC; ++e) O[e] += po[c][e] * sc;
            }
    }
    const size_t at = a.out_frag ? act_frag(r, h * HD + i, a.n_rows, a.n_q_heads * HD) : ((size_t)r * a.n_q_heads + h) * HD + i;
    if (ACT32) {
        if (VEC == 2) *(float2*)((float*)a.out + at) = make_float2(O[0] / L, O[VEC - 1] / L);
        else ((float*)a.out)[at] = O[0] / L;
    } else {
        if (VEC == 2) *(uint32_t*)((uint16_t*)a.out + at) = (uint32_t)f32_to_act16(O[0] / L) | ((uint32_t)f32_to_act16(O[VEC - 1] / L) << 16);
        else ((uint16_t*)a.out)[at] = f32_to_act16(O[0] / L);
    }
}

template <int HD, bool ACT32>
static hipError_t stream_impl(const AttnArgs& a, hipStream_t s) {
    const int G = a.n_q_heads / a.n_kv_heads;
    const size_t lds = (size_t)(4 * G * (HD + 4) + 128) * sizeof(float);
    const int pairs = a.n_rows * a.n_kv_heads, wgs = (a.total_units + a.units_per_wg - 1) / a.units_per_wg;
    if (a.form == DECODE_PAIR) hipLaunchKernelGGL((attn_stream_kernel<HD, ACT32, DECODE_PAIR>), dim3(pairs), dim3(256), lds, s, a);
    else if (a.form == DECODE_PIECES)            // a pair that starts inside a piece has one more: of the two spare slots one is enough
        hipLaunchKernelGGL((attn_stream_kernel<HD, ACT32, DECODE_PIECES>), dim3(pairs, a.own_cut ? a.n_chunks : a.n_chunks - 1), dim3(256), lds, s, a);
    else hipLaunchKernelGGL((attn_stream_kernel<HD, ACT32, DECODE_STREAM>), dim3(wgs), dim3(256), lds, s, a);
    return hipGetLastError();
}

template <int HD, bool ACT32>
static hipError_t stream_combine_impl(const AttnArgs& a, hipStream_t s) {
    const dim3 g(a.n_rows, a.n_q_heads), b(64);
    if (a.n_chunks <= 4) hipLaunchKernelGGL((attn_stream_combine_kernel<HD, ACT32, 4>), g, b, 0, s, a);
    else hipLaunchKernelGGL((attn_stream_combine_kernel<HD, ACT32, 8>), g, b, 0, s, a);
    return hipGetLastError();
}

static bool stream_args_ok(const AttnArgs& a) {
    // every (row, kv head) pair of max_pages pages must fit its partial slots: pages / U + 2 <= n_chunks
    return a.n_rows > 0 && a.row_page_start && a.units_per_wg > 0 && a.total_units > 0 && a.n_chunks > 0 &&
           a.n_q_heads / a.n_kv_heads <= kMaxGroup;
}

hipError_t launch_attn_stream(const AttnArgs& a, int hd, bool act32, hipStream_t s) {
    if (!stream_args_ok(a)) return hipErrorInvalidValue;
    switch (hd) {
        case 32:  return act32 ? stream_impl<32, true>(a, s) : stream_impl<32, false>(a, s);
        case 64:  return act32 ? stream_impl<64, true>(a, s) : stream_impl<64, false>(a, s);
        case 128: return act32 ? stream_impl<128, true>(a, s) : stream_impl<128, false>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_attn_stream_combine(const AttnArgs& a, int hd, bool act32, hipStream_t s) {
    if (!stream_args_ok(a)) return hipErrorInvalidValue;
    switch (hd) {
        case 32:  return act32 ? stream_combine_impl<32, true>(a, s) : stream_combine_impl<32, false>(a, s);
        case 64:  return act32 ? stream_combine_impl<64, true>(a, s) : stream_combine_impl<64, false>(a, s);
        case 128: return act32 ? stream_combine_impl<128, true>(a, s) : stream_combine_impl<128, false>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int HD, bool ACT32>
static hipError_t prefill_impl(const AttnArgs& a, int B, int max_new, hipStream_t s) {
    PrefillGrid gr;
    gr.group = a.n_q_heads / a.n_kv_heads;
    gr.head_groups = (gr.group + 3) / 4;
    gr.heads_wg = (gr.group + gr.head_groups - 1) / gr.head_groups;       // at most four heads a workgroup
    gr.tiles = 4 / gr.heads_wg;
    gr.pairs = B * a.n_kv_heads * gr.head_groups;
    gr.by_groups = reciprocal(gr.head_groups);
    gr.by_kv_heads = reciprocal(a.n_kv_heads);
    if ((unsigned long long)gr.pairs * a.n_kv_heads >> 32) return hipErrorInvalidValue;       // no model: 2,000 kv heads in 1,024 sequences
    const int qblocks = (max_new + gr.tiles * 32 - 1) / (gr.tiles * 32);
    // (in one dimension a thousand sequences beside one of 65,600 tokens would pass the 2^32 threads that a dimension of a
    // launch may have)
    const dim3 grid(8 * qblocks, (gr.pairs + 7) / 8);
    constexpr size_t lds = (size_t)2 * 4 * (2 * kPageTokens * HD * 2);
    static_assert(lds <= 65536, "more needs hipFuncAttributeMaxDynamicSharedMemorySize");
    hipLaunchKernelGGL((attn_prefill_kernel<HD, ACT32>), grid, dim3(256), lds, s, a, gr);
    return hipGetLastError();
}

hipError_t launch_attn_prefill(const AttnArgs& a, int hd, int B, int max_new, bool act32, hipStream_t s) {
    if (B <= 0 || max_new <= 0) return hipErrorInvalidValue;
    switch (hd) {
        case 32:  return act32 ? prefill_impl<32, true>(a, B, max_new, s) : prefill_impl<32, false>(a, B, max_new, s);
        case 64:  return act32 ? prefill_impl<64, true>(a, B, max_new, s) : prefill_impl<64, false>(a, B, max_new, s);
        case 128: return act32 ? prefill_impl<128, true>(a, B, max_new, s) : prefill_impl<128, false>(a, B, max_new, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace spiral
