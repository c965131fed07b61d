// Learner-side scoring: log pi(target | context) for every row of a packed batch, without ever
// writing the [rows, vocab] logits.
//
// With fragment-ordered weights the LM head is the 256 x 256 tiled kernel with a scoring epilogue (gemm_tile_kernel<3>),
// which leaves one (max, sum of exp) pair per row and 128 columns for score_merge_pairs_kernel.
//
// Without them, or where that kernel's 32-bit offsets or the memory for its pairs do not suffice: score_lmhead_kernel is the
// LM-head GEMM of the decode path (32x32x16 MFMA, weights HBM/L2 -> registers in operand layout, activations through LDS)
// with another epilogue: a workgroup owns 128 rows and a range of 128-column vocabulary tiles.  FRAG: the weights come from
// the fragment-ordered copy (rows of narrow-head models, 800 and 6,000 of them, score 8 to 11 % slower from the row-major one).
// PAIRS: after each tile the four waves, 32 columns each, fold their logits in the tiled kernel's order (same bits) and
// write its pair.  Otherwise (a vocabulary whose pairs do not fit the workspace, with any weights): every lane folds its 16
// logits of each row into a private running pair over the whole range, the pairs of a row (2 lanes x 4 waves) are merged
// through LDS and written as one partial per (row, range); score_merge_kernel combines the ranges:
//     logp = logit[target] - (M + ln sum_i s_i * exp(m_i - M)).
// score_objective_kernel evaluates the clipped importance-ratio surrogate and the REINFORCE sum in
// float64 with a fixed reduction order.
#include "spiral_internal.h"
#include "mfma_ops.h"

namespace spiral {

namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mma32s(const u32x4& w, const u32x4& a, const f32x16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, a), c, 0, 0, 0);
}

constexpr int ROWB = 272;                 // LDS bytes per activation row (256 + 16 pad)
constexpr int BUF = 128 * ROWB;
constexpr int PD = 2;

}  // namespace

template <bool PAIRS, bool FRAG>
__global__ __launch_bounds__(256) void score_lmhead_kernel(ScoreArgs g) {
    extern __shared__ uint4 lds_raw[];
    char* lds = (char*)lds_raw;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l32 = lane & 31, lh = lane >> 5;
    const int tile_m = blockIdx.x % g.m_tiles;
    const int split = blockIdx.x / g.m_tiles;
    const int K = g.K;
    const int m0 = tile_m * 128;
    const int n_tiles = (g.V + 127) / 128;
    const int nt_begin = split * g.tiles_per_split;
    const int nt_end = min(nt_begin + g.tiles_per_split, n_tiles);

    const uint16_t* a_src[8];
    int a_dst[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int sgm = threadIdx.x + 256 * i;
        const int row = sgm >> 4, c16 = sgm & 15;
        int m = m0 + row; if (m >= g.M) m = g.M - 1;
        a_src[i] = (const uint16_t*)g.A + (size_t)m * K + c16 * 8;
        a_dst[i] = row * ROWB + c16 * 16;
    }
    const int frag_off = l32 * ROWB + lh * 16;
    const int NC = K >> 7;

    // this lane's rows (one per batch tile) and their targets
    int tgt[4];
    float m_run[4], s_run[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int m = m0 + t * 32 + l32;
        tgt[t] = m < g.M ? g.targets[m] : -1;
        m_run[t] = -INFINITY;
        s_run[t] = 0.f;
    }

    struct St { u32x4 a[8]; u32x4 w[8]; };
    for (int nt = nt_begin; nt < nt_end; ++nt) {
        const int n_first = nt * 128 + wave * 32;
        int n = n_first + l32; if (n >= g.V) n = g.V - 1;
        const uint16_t* wrow = FRAG ? (const uint16_t*)g.Wf + frag_block(min(nt * 4 + wave, (g.V + 31) / 32 - 1), 0, K) + lane * 8
                                    : (const uint16_t*)g.W + (size_t)n * K + lh * 8;

        f32x16 acc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

        St st[PD];
        auto load = [&](St& S, int chunk) {
            const int cc = chunk < NC ? chunk : NC - 1;
            const size_t off = (size_t)cc * 128;
#pragma unroll
            for (int i = 0; i < 8; ++i) S.a[i] = *(const u32x4*)(a_src[i] + off);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                S.w[ks] = FRAG ? *(const u32x4*)(wrow + ((size_t)cc * 8 + ks) * 512) : *(const u32x4*)(wrow + off + ks * 16);
        };
        auto iter = [&](St& S, int c) {
            char* buf = lds + (c & 1) * BUF;
#pragma unroll
            for (int i = 0; i < 8; ++i) *(u32x4*)(buf + a_dst[i]) = S.a[i];
            __syncthreads();
            u32x4 af[2][4];
#pragma unroll
            for (int t = 0; t < 4; ++t) af[0][t] = *(const u32x4*)(buf + frag_off + t * 32 * ROWB);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                if (ks + 1 < 8) {
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        af[(ks + 1) & 1][t] = *(const u32x4*)(buf + frag_off + t * 32 * ROWB + (ks + 1) * 32);
                }
                const u32x4 wp = FRAG ? S.w[ks] : prep_w(S.w[ks]);      // fragment-ordered copies are already widened
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[t] = mma32s(wp, af[ks & 1][t], acc[t]);
            }
            load(S, c + PD);
        };
#pragma unroll
        for (int i = 0; i < PD; ++i) load(st[i], i);
        int c = 0;
        for (; c + PD <= NC; c += PD) {
#pragma unroll
            for (int i = 0; i < PD; ++i) iter(st[i], c + i);
        }
#pragma unroll
        for (int i = 0; i < PD - 1; ++i)
            if (c + i < NC) iter(st[i], c + i);
        __syncthreads();                       // the next tile's first LDS write must not overtake a slow wave's reads

        // registers 4b..4b+3 of a tile hold columns n_first + 8b + 4*lh .. +3 of row l32
        if (PAIRS) {
            float* s_max = (float*)lds;                     // [4 waves][128 rows]
            float* s_sum = s_max + 512;                     // [4 waves][4 batch tiles][64 lanes]
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                float mx = -INFINITY;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int col = n_first + 8 * (r >> 2) + 4 * lh + (r & 3);
                    if (col >= g.V) acc[t][r] = -INFINITY;
                    mx = fmaxf(mx, acc[t][r]);
                    if (col == tgt[t]) g.tgt_logit[m0 + t * 32 + l32] = acc[t][r];
                }
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                if (lh == 0) s_max[wave * 128 + t * 32 + l32] = mx;
            }
            __syncthreads();
            float mine = -INFINITY;                         // the pair of batch tile `wave`: this wave writes it
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int row = t * 32 + l32;
                const float mx = fmaxf(fmaxf(s_max[row], s_max[128 + row]), fmaxf(s_max[256 + row], s_max[384 + row]));
                const float ref = mx > -INFINITY ? mx : 0.f;
                float sj = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) sj += __expf(acc[t][r] - ref);
                s_sum[(wave * 4 + t) * 64 + lane] = sj;
                if (t == wave) mine = mx;
            }
            __syncthreads();
            float sum = s_sum[wave * 64 + lane];
#pragma unroll
            for (int j = 1; j < 4; ++j) sum += s_sum[(j * 4 + wave) * 64 + lane];
            sum += __shfl_xor(sum, 32, 64);
            const int m = m0 + wave * 32 + l32;
            if (lh == 0 && m < g.M) g.pairs[(size_t)nt * g.M + m] = make_float2(mine, sum);
            __syncthreads();                                // the next tile's staging overwrites the exchange
            continue;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            float mx = -INFINITY;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int col = n_first + 8 * b + 4 * lh + r;
                    if (col >= g.V) acc[t][4 * b + r] = -INFINITY;
                    mx = fmaxf(mx, acc[t][4 * b + r]);
                    if (col == tgt[t]) g.tgt_logit[m0 + t * 32 + l32] = acc[t][4 * b + r];
                }
            if (mx > -INFINITY) {
                const float m_new = fmaxf(m_run[t], mx);
                float sum = 0.f;
#pragma unroll
                for (int r = 0; r < 16; ++r) sum += __expf(acc[t][r] - m_new);
                s_run[t] = s_run[t] * __expf(m_run[t] - m_new) + sum;
                m_run[t] = m_new;
            }
        }
    }

    if (PAIRS) return;
    // ---- merge the 8 (max, sum) pairs of every row: the two lane halves, then the four waves
    float* s_m = (float*)lds;                  // [4 waves][128 rows]
    float* s_s = s_m + 512;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float om = __shfl_xor(m_run[t], 32, 64), os = __shfl_xor(s_run[t], 32, 64);
        const float M = fmaxf(m_run[t], om);
        const float S = (m_run[t] > -INFINITY ? s_run[t] * __expf(m_run[t] - M) : 0.f) + (om > -INFINITY ? os * __expf(om - M) : 0.f);
        if (lh == 0) { s_m[wave * 128 + t * 32 + l32] = M; s_s[wave * 128 + t * 32 + l32] = S; }
    }
    __syncthreads();
    if (threadIdx.x < 128) {
        const int row = threadIdx.x, m = m0 + row;
        if (m < g.M) {
            float M = -INFINITY;
#pragma unroll
            for (int w = 0; w < 4; ++w) M = fmaxf(M, s_m[w * 128 + row]);
            float S = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float mw = s_m[w * 128 + row];
                if (mw > -INFINITY) S += s_s[w * 128 + row] * __expf(mw - M);
            }
            float2* dst = (float2*)g.part + (size_t)m * g.n_splits + split;
            *dst = make_float2(M, S);
        }
    }
}

__global__ __launch_bounds__(256) void score_merge_kernel(ScoreArgs g, float* out) {
    const int m = blockIdx.x * 256 + threadIdx.x;
    if (m >= g.M) return;
    if (g.targets[m] < 0) { out[m] = 0.f; return; }
    const float2* p = (const float2*)g.part + (size_t)m * g.n_splits;
    float M = -INFINITY;
    for (int i = 0; i < g.n_splits; ++i) M = fmaxf(M, p[i].x);
    float S = 0.f;
    for (int i = 0; i < g.n_splits; ++i)
        if (p[i].x > -INFINITY) S += p[i].y * expf(p[i].x - M);
    out[m] = g.tgt_logit[m] - (M + logf(S));
}

// The same merge for one pair per 128 columns, [n_pairs][M]: 32 rows a workgroup, eight threads to a row, so that a load
// instruction reads two 256-byte runs.
__global__ __launch_bounds__(256) void score_merge_pairs_kernel(ScoreArgs g, int n_pairs, float* out) {
    __shared__ float2 s_pair[8][32];
    const int r = threadIdx.x & 31, q = threadIdx.x >> 5;
    const int m = blockIdx.x * 32 + r;
    const int mc = m < g.M ? m : g.M - 1;
    float M = -INFINITY, S = 0.f;
    for (int t0 = q; t0 < n_pairs; t0 += 8 * 8) {              // eight loads in flight; past the end: the last pair, weight 0
        float2 p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = g.pairs[(size_t)min(t0 + 8 * u, n_pairs - 1) * g.M + mc];
        float mx = M;
#pragma unroll
        for (int u = 0; u < 8; ++u) mx = fmaxf(mx, p[u].x);
        if (mx > -INFINITY) {
            float sum = M > -INFINITY ? S * expf(M - mx) : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (t0 + 8 * u < n_pairs && p[u].x > -INFINITY) sum += p[u].y * expf(p[u].x - mx);
            S = sum;
            M = mx;
        }
    }
    s_pair[q][r] = make_float2(M, S);
    __syncthreads();
    if (q != 0 || m >= g.M) return;
    if (g.targets[m] < 0) { out[m] = 0.f; return; }
    M = -INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u) M = fmaxf(M, s_pair[u][r].x);
    S = 0.f;
#pragma unroll
    for (int u = 0; u < 8; ++u)
        if (s_pair[u][r].x > -INFINITY) S += s_pair[u][r].y * expf(s_pair[u][r].x - M);
    out[m] = g.tgt_logit[m] - (M + logf(S));
}

hipError_t launch_score_merge_pairs(const ScoreArgs& a, float* out, hipStream_t s) {
    if (a.M < 1 || a.V < 1 || !a.pairs || !a.targets || !a.tgt_logit) return hipErrorInvalidValue;
    hipLaunchKernelGGL(score_merge_pairs_kernel, dim3((a.M + 31) / 32), dim3(256), 0, s, a, (a.V + 127) / 128, out);
    return hipGetLastError();
}

// out[0] = sum mask * min(r * A, clip(r, 1 - eps, 1 + eps) * A), r = exp(new - old);  out[1] = sum mask * A * new
__global__ __launch_bounds__(1024) void score_objective_kernel(const float* logp_new, const float* logp_old, const float* adv,
                                                               const int32_t* mask, long long n, float eps, double* out) {
    __shared__ double s_a[1024], s_b[1024];
    double a = 0.0, b = 0.0;
    for (long long i = threadIdx.x; i < n; i += 1024) {
        if (mask && mask[i] == 0) continue;
        const double ln = logp_new[i], A = adv[i];
        const double r = exp(ln - (double)logp_old[i]);
        const double rc = fmin(fmax(r, 1.0 - (double)eps), 1.0 + (double)eps);
        a += fmin(r * A, rc * A);
        b += A * ln;
    }
    s_a[threadIdx.x] = a; s_b[threadIdx.x] = b;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (threadIdx.x < o) { s_a[threadIdx.x] += s_a[threadIdx.x + o]; s_b[threadIdx.x] += s_b[threadIdx.x + o]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) { out[0] = s_a[0]; out[1] = s_b[0]; }
}

hipError_t launch_score(const ScoreArgs& a, float* out, hipStream_t s) {
    if (a.M < 1 || a.V < 1 || (a.K & 127) || a.n_splits < 1 || a.tiles_per_split < 1) return hipErrorInvalidValue;
    ScoreArgs g = a;
    g.m_tiles = (a.M + 127) / 128;
    const dim3 grid(g.m_tiles * g.n_splits), b(256);
    const size_t lds = (size_t)2 * BUF;
    if (g.pairs && g.Wf) hipLaunchKernelGGL((score_lmhead_kernel<true, true>), grid, b, lds, s, g);
    else if (g.pairs) hipLaunchKernelGGL((score_lmhead_kernel<true, false>), grid, b, lds, s, g);
    else if (g.Wf) hipLaunchKernelGGL((score_lmhead_kernel<false, true>), grid, b, lds, s, g);
    else hipLaunchKernelGGL((score_lmhead_kernel<false, false>), grid, b, lds, s, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (g.pairs) return launch_score_merge_pairs(g, out, s);
    hipLaunchKernelGGL(score_merge_kernel, dim3((a.M + 255) / 256), dim3(256), 0, s, g, out);
    return hipGetLastError();
}

hipError_t launch_score_objective(const float* logp_new, const float* logp_old, const float* adv, const int32_t* mask,
                                  long long n, float eps, double* out, hipStream_t s) {
    hipLaunchKernelGGL(score_objective_kernel, dim3(1), dim3(1024), 0, s, logp_new, logp_old, adv, mask, n, eps, out);
    return hipGetLastError();
}

}  // namespace spiral
