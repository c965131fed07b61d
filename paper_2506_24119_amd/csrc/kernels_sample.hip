// Truncated (top-k / top-p) Gumbel-max sampler.
//
// Per row: z_v = logit_v / T; the keep set is { z_v >= tau } with tau the larger of the k-th largest z
// (top-k) and the z at which the descending running sum of softmax(z) over the top-k survivors first
// reaches p (top-p); the token is the argmax of z + g over the keep set.  Both thresholds are found by
// a most-significant-digit-first radix descent over an order-preserving 32-bit key of z, 8 bits per
// pass: top-k walks a histogram of counts, top-p a histogram of probability mass.  Mass is held in
// 64-bit fixed point (float64 exp(z - max) * 2^45: integer adds in any order give the same sum, so the
// result is bit-reproducible, and the running sums agree with exact arithmetic to ~2e-9 of the largest
// term summed over a 152k vocabulary); a token lighter than 2^-46 of the heaviest one counts as zero.
// One block of 1024 threads per row; each wave fills its own histogram copy in LDS.
//
// With a workspace the same thresholds are found in three sweeps of the row instead of up to nine, and by several
// workgroups per row: (1) row maximum; (2) one histogram of count and mass over 4096 bins that are linear in
// zmax - z (width 1/128; the last bin takes everything 32 or more below the maximum, whose mass is zero in the
// 2^45 fixed point), with sums over every 64 bins; (3) one sweep whose workgroups first find the bin that holds the cut (an
// integer prefix sum over the 64 sums, then over the 64 bins below one of them), then score the tokens in the bins above
// it for the Gumbel-max and copy the tokens of the cut bin (a few hundred to a few thousand) to the row's candidate list, on
// which the radix descent then runs in LDS, in a last kernel of a workgroup per row.  Bin order follows key order and the
// masses are the same integers, so the threshold is the one the single-kernel path finds, bit for bit; a row whose cut bin
// holds more candidates than the list (many equal scores) is done by that path's code in the last kernel.
// Bound by the fixed-point exponentials of the histogram and the generator's integer arithmetic of the sweep.  Measured
// against six launches (a plan kernel that read every bin, the single path's kernel launched behind for flagged rows) and at
// most 8 slices a row, 151,936 entries, T = 0.6, top-p 0.95: one row 59 -> 35 us, 16 rows 55 -> 34, 128 rows of flat logits
// 130 -> 111 (a call; 117 traced); 64 rows, top-k 50 54 -> 42.
#include <algorithm>

#include "spiral_internal.h"

namespace spiral {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;

// larger float <=> larger key; -0 and +0 share a key
__device__ __forceinline__ uint32_t order_key(float z) {
    const uint32_t b = __float_as_uint(z + 0.0f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// f(logit, v) for v = lo + tid, lo + tid + kThreads, ... < hi, with U loads in flight per thread (issued before the
// first use; past the end they re-read the last entry, a branch around a load would make every load wait)
template <int U, class F>
__device__ __forceinline__ void sweep(const float* lr, int lo, int hi, int tid, F&& f) {
    for (int base = lo + tid; base < hi; base += kThreads * U) {
        float l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) l[u] = lr[min(base + u * kThreads, hi - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = base + u * kThreads;
            if (v < hi) f(l[u], v);
        }
    }
}

__device__ __forceinline__ uint64_t shfl_down_u64(uint64_t v, int d) {
    const uint32_t lo = __shfl_down((uint32_t)v, d, 64), hi = __shfl_down((uint32_t)(v >> 32), d, 64);
    return ((uint64_t)hi << 32) | lo;
}

// 2^(j/32), j = 0..31
__device__ const double kExp2Tab[32] = {
    1.0, 1.0218971486541166, 1.0442737824274138, 1.0671404006768237,
    1.0905077326652577, 1.1143867425958924, 1.1387886347566916, 1.1637248587775775,
    1.189207115002721, 1.215247359980469, 1.241857812073484, 1.2690509571917332,
    1.2968395546510096, 1.3252366431597413, 1.3542555469368927, 1.383909881963832,
    1.4142135623730951, 1.4451808069770467, 1.4768261459394993, 1.5091644275934228,
    1.5422108254079407, 1.5759808451078865, 1.6104903319492543, 1.645755478153965,
    1.681792830507429, 1.718619298122478, 1.7562521603732995, 1.7947090750031072,
    1.8340080864093424, 1.8741676341103, 1.9152065613971474, 1.9571441241754002};

// floor(exp(z - zmax) * 2^45) for z <= zmax; zero from 32 below the maximum on (exp(-32) * 2^45 < 1) and for
// z = -inf.  exp(x) = 2^(k/32) * exp(r) with k = round(32 x / ln 2): the table gives 2^((k mod 32)/32), the Taylor
// series to the 6th power exp(r) for |r| <= ln 2 / 64 (remainder 4e-18), ldexp the rest; 4e-16 of exp() at worst.
__device__ __forceinline__ uint64_t mass45(float z, float zmax) {
    const double x = (double)z - (double)zmax;
    if (!(x > -32.0)) return 0;
    const double k = rint(x * 46.16624130844683);
    double r = fma(-k, 0.021660849392489467, x);       // ln 2 / 32, high part (12 trailing zero bits: k * hi is exact)
    r = fma(-k, 8.823528300947368e-15, r);             // low part
    double p = 1.0 / 720.0;
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    const int ki = (int)k;                              // <= 0
    return (uint64_t)ldexp(kExp2Tab[ki & 31] * p, (ki >> 5) + 45);
}

constexpr int kBins = 4096;           // linear in zmax - z, 1/128 wide; the last one is everything >= 32 below the maximum
constexpr int kCap = 8192;            // candidates of a row that the in-LDS resolution takes
constexpr int kCoarse = 64;           // sums of 64 bins each
constexpr int kMaxSlices = 16;        // workgroups per row

// What the prefix sum over a row's histogram decides (one per row, in the workspace).
struct TruncRow {
    float zmax;
    int cand_lo, cand_hi;             // tokens in bins [cand_lo, cand_hi] go to the candidate list; bins below cand_lo are kept
    int fallback;                     // more candidates than the list holds: the single-kernel path does this row
    uint64_t need_mass;               // top-p alone: fixed-point mass still to be covered inside the candidate bin
    uint32_t need_count;              // top-k: how many of the candidates, from the largest, are kept
    int n_cand;
};

__device__ __forceinline__ int bin_of(float z, float zmax) {
    const float d = zmax - z;
    return d < 32.f ? max((int)(d * 128.f), 0) : kBins - 1;      // NaN and -inf land in the last bin
}

struct Select {
    uint32_t prefix;       // digits fixed so far (high bits)
    uint64_t remaining;    // how much (count or mass) must still be covered from the top of the current bucket
};

// Among the 256 bins (sum over the waves' copies), walking from bin 255 down, the bin in which the
// running total first reaches `remaining`.  Executed by wave 0; result broadcast through LDS.
template <int COPIES>
__device__ __forceinline__ void pick_bin(const uint64_t* hist, int shift, Select* sel, int lane) {
    uint64_t b[4];
    uint64_t mine = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint64_t s = 0;
        for (int w = 0; w < COPIES; ++w) s += hist[w * 256 + lane * 4 + i];
        b[i] = s;
        mine += s;
    }
    // suffix sums over lanes: above = total of the bins of all higher lanes
    uint64_t incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t o = shfl_down_u64(incl, d);
        if (lane + d < 64) incl += o;
    }
    const uint64_t above = incl - mine;
    const uint64_t need = sel->remaining;
    if (above < need && need <= incl) {             // exactly one lane when need <= total
        uint64_t acc = above;
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            if (acc + b[i] >= need) {
                sel->prefix |= (uint32_t)(lane * 4 + i) << shift;
                sel->remaining = need - acc;
                break;
            }
            acc += b[i];
        }
    }
}

// One row by one workgroup, in up to nine sweeps of the logits; hist: LDS, [kWaves][256].
__device__ __forceinline__ void truncated_row(uint64_t* hist, const float* logits, int row, int V, float temperature, int top_k, float top_p,
                                              int use_noise_buffer, uint64_t key64, const float* noise, int32_t* out, float* tau_out) {
    __shared__ Select sel;
    __shared__ float s_red[kWaves];
    __shared__ int s_idx[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* lr = logits + (size_t)row * V;
    uint64_t* my_hist = hist + wave * 256;

    auto clear_hist = [&] {
        for (int i = tid; i < kWaves * 256; i += kThreads) hist[i] = 0;
        __syncthreads();
    };

    // ---- max of z (the softmax reference point)
    float zmax = -INFINITY;
    sweep<8>(lr, 0, V, tid, [&](float l, int) { zmax = fmaxf(zmax, l / temperature); });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, o, 64));
    if (lane == 0) s_red[wave] = zmax;
    __syncthreads();
    zmax = s_red[0];
    for (int w = 1; w < kWaves; ++w) zmax = fmaxf(zmax, s_red[w]);
    __syncthreads();

    uint32_t floor_key = 0;                      // keys below it are cut

    // ---- top-k: the key of the k-th largest z
    if (top_k > 0 && top_k < V) {
        if (tid == 0) { sel.prefix = 0; sel.remaining = (uint64_t)top_k; }
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            clear_hist();
            const uint32_t prefix = sel.prefix;
            sweep<8>(lr, 0, V, tid, [&](float l, int) {
                const uint32_t key = order_key(l / temperature);
                if (pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)))
                    atomicAdd((unsigned long long*)&my_hist[(key >> shift) & 255u], 1ull);
            });
            __syncthreads();
            if (wave == 0) pick_bin<kWaves>(hist, shift, &sel, lane);
            __syncthreads();
        }
        floor_key = sel.prefix;
        __syncthreads();
    }

    // ---- top-p over the survivors: the key at which the descending running mass first reaches p * Z
    if (top_p < 1.0f) {
        if (tid == 0) { sel.prefix = 0; sel.remaining = 0; }
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            clear_hist();
            const uint32_t prefix = sel.prefix;
            sweep<8>(lr, 0, V, tid, [&](float l, int) {
                const float z = l / temperature;
                const uint32_t key = order_key(z);
                if (key >= floor_key && (pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)))) {
                    const uint64_t mass = mass45(z, zmax);
                    atomicAdd((unsigned long long*)&my_hist[(key >> shift) & 255u], (unsigned long long)mass);
                }
            });
            __syncthreads();
            if (pass == 0) {
                // the first histogram holds the whole surviving mass Z: fix the target, then pick
                if (wave == 0) {
                    uint64_t mine = 0;
                    for (int i = 0; i < 4; ++i)
                        for (int w = 0; w < kWaves; ++w) mine += hist[w * 256 + lane * 4 + i];
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const uint64_t o = shfl_down_u64(mine, d);
                        if (lane + d < 64) mine += o;
                    }
                    if (lane == 0) {
                        const uint64_t Z = mine;
                        uint64_t target = (uint64_t)ceil((double)top_p * (double)Z);
                        if (target < 1) target = 1;
                        if (target > Z) target = Z;
                        sel.remaining = target;
                    }
                }
                __syncthreads();
            }
            if (wave == 0) pick_bin<kWaves>(hist, shift, &sel, lane);
            __syncthreads();
        }
        if (sel.prefix > floor_key) floor_key = sel.prefix;
        __syncthreads();
    }

    // ---- Gumbel-max over the keep set
    const float* nr = use_noise_buffer ? noise + (size_t)row * V : nullptr;
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    sweep<8>(lr, 0, V, tid, [&](float l, int v) {
        const float z = l / temperature;
        if (order_key(z) < floor_key) return;
        const float sc = z + (nr ? nr[v] : gumbel_noise(key64, v));
        if (better(sc, v, bv, bi)) { bv = sc; bi = v; }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
    }
    if (lane == 0) { s_red[wave] = bv; s_idx[wave] = bi; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w)
            if (s_red[w] > bv || (s_red[w] == bv && s_idx[w] < bi)) { bv = s_red[w]; bi = s_idx[w]; }
        out[row] = bi == 0x7FFFFFFF ? 0 : bi;
        if (tau_out) tau_out[row] = floor_key == 0 ? -INFINITY : key_value(floor_key);
    }
}

}  // namespace

__global__ __launch_bounds__(kThreads) void sample_truncated_kernel(const float* logits, int V, float temperature, int top_k,
                                                                    float top_p, int use_noise_buffer, KeyChunk keys,
                                                                    const float* noise, int32_t* out, float* tau_out) {
    __shared__ uint64_t hist[kWaves * 256];
    truncated_row(hist, logits, blockIdx.x, V, temperature, top_k, top_p, use_noise_buffer, keys.key[blockIdx.x], noise, out, tau_out);
}

// ---- the multi-workgroup path (needs a workspace) ---------------------------------------------------------------

// vocabulary range of slice blockIdx.x of gridDim.x
__device__ __forceinline__ void slice_range(int V, int& lo, int& hi) {
    const int per = (V + (int)gridDim.x - 1) / (int)gridDim.x;
    lo = (int)blockIdx.x * per;
    hi = min(V, lo + per);
}

__global__ __launch_bounds__(kThreads) void trunc_max_kernel(const float* logits, int V, float* lmax_part, int* cand_n) {
    __shared__ float s_red[kWaves];
    const int row = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float* lr = logits + (size_t)row * V;
    int lo, hi;
    slice_range(V, lo, hi);
    float m = -INFINITY;
    sweep<8>(lr, lo, hi, tid, [&](float l, int) { m = fmaxf(m, l); });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane == 0) s_red[wave] = m;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w) m = fmaxf(m, s_red[w]);
        lmax_part[row * kMaxSlices + blockIdx.x] = m;
        if (blockIdx.x == 0) cand_n[row] = 0;
    }
}

// the row maximum of z: division by T > 0 is monotone, so max(l / T) = max(l) / T
__device__ __forceinline__ float row_zmax(const float* lmax_part, int row, int slices, float temperature) {
    float m = lmax_part[row * kMaxSlices];
    for (int i = 1; i < slices; ++i) m = fmaxf(m, lmax_part[row * kMaxSlices + i]);
    return m / temperature;
}

__global__ __launch_bounds__(kThreads) void trunc_hist_kernel(const float* logits, int V, float temperature, const float* lmax_part,
                                                              int want_mass, uint64_t* hist_mass, uint32_t* hist_cnt,
                                                              uint64_t* sum_mass, uint32_t* sum_cnt) {
    __shared__ uint64_t hm[kBins];
    __shared__ uint32_t hc[kBins];
    const int row = blockIdx.y, tid = threadIdx.x;
    const float* lr = logits + (size_t)row * V;
    for (int i = tid; i < kBins; i += kThreads) { hm[i] = 0; hc[i] = 0; }
    const float zmax = row_zmax(lmax_part, row, gridDim.x, temperature);
    __syncthreads();
    int lo, hi;
    slice_range(V, lo, hi);
    sweep<8>(lr, lo, hi, tid, [&](float l, int) {
        const float z = l / temperature;
        const int b = bin_of(z, zmax);
        atomicAdd(&hc[b], 1u);
        if (want_mass) {
            const uint64_t m = mass45(z, zmax);
            if (m) atomicAdd((unsigned long long*)&hm[b], (unsigned long long)m);
        }
    });
    __syncthreads();
    const size_t base = ((size_t)row * gridDim.x + blockIdx.x) * kBins;
    for (int i = tid; i < kBins; i += kThreads) { hist_mass[base + i] = hm[i]; hist_cnt[base + i] = hc[i]; }
    uint64_t m = 0;
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) { m += hm[tid * 4 + i]; c += hc[tid * 4 + i]; }       // 16 threads to a sum
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) { m += shfl_down_u64(m, d); c += __shfl_down(c, d, 64); }
    if ((tid & 15) == 0) {
        const size_t at = ((size_t)row * gridDim.x + blockIdx.x) * kCoarse + (tid >> 4);
        sum_mass[at] = m;
        sum_cnt[at] = c;
    }
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int d) {
    const uint32_t lo = __shfl_up((uint32_t)v, d, 64), hi = __shfl_up((uint32_t)(v >> 32), d, 64);
    return ((uint64_t)hi << 32) | lo;
}

// Prefix sums over the bins of a row (bin 0 = the largest z) and the bin in which the cut falls; by one wave, two levels
// of 64.  Every lane of the wave returns with the plan.
__device__ __forceinline__ TruncRow trunc_plan(int row, int V, float temperature, int top_k, float top_p, int slices, const float* lmax_part,
                                               const uint64_t* hist_mass, const uint32_t* hist_cnt, const uint64_t* sum_mass,
                                               const uint32_t* sum_cnt, int lane) {
    TruncRow r = {};
    r.zmax = row_zmax(lmax_part, row, slices, temperature);
    const bool by_count = top_k > 0 && top_k < V;
    const bool by_mass = top_p < 1.0f;
    uint64_t target = 0, base_m = 0;
    uint32_t base_c = 0;
    int first = 0;                                           // the 64 entries of the level start here
#pragma unroll
    for (int level = 0; level < 2; ++level) {
        uint64_t m = 0;
        uint32_t c = 0;
#pragma unroll 4
        for (int s = 0; s < slices; ++s) {
            const size_t seg = (size_t)row * slices + s;
            m += level == 0 ? sum_mass[seg * kCoarse + lane] : hist_mass[seg * kBins + first + lane];
            c += level == 0 ? sum_cnt[seg * kCoarse + lane] : hist_cnt[seg * kBins + first + lane];
        }
        uint64_t im = m;
        uint32_t ic = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t om = shfl_up_u64(im, d);
            const uint32_t oc = __shfl_up(ic, d, 64);
            if (lane >= d) { im += om; ic += oc; }
        }
        if (level == 0 && !by_count) {
            const uint64_t total = ((uint64_t)__shfl((uint32_t)(im >> 32), 63, 64) << 32) | __shfl((uint32_t)im, 63, 64);
            target = (uint64_t)ceil((double)top_p * (double)total);
            if (target < 1) target = 1;
            if (target > total) target = total;
        }
        const uint64_t before_m = base_m + im - m;
        const uint32_t before_c = base_c + ic - c;
        const bool here = by_count ? (before_c < (uint32_t)top_k && (uint32_t)top_k <= before_c + c)
                                   : (before_m < target && target <= before_m + m);
        const uint64_t where = __builtin_amdgcn_ballot_w64(here);
        if (where == 0) { r.fallback = 1; return r; }        // no bin qualifies (a row of NaN): the single path's business
        const int at = __builtin_ctzll(where);               // exactly one
        base_m = ((uint64_t)__shfl((uint32_t)(before_m >> 32), at, 64) << 32) | __shfl((uint32_t)before_m, at, 64);
        base_c = __shfl(before_c, at, 64);
        if (level == 0) {
            first = at * (kBins / kCoarse);
        } else {
            const uint32_t bin_c = __shfl(c, at, 64);
            r.cand_hi = first + at;
            if (by_count && by_mass) {                       // top-p needs the mass of the top-k survivors: resolve both on the list
                r.cand_lo = 0;
                r.need_count = (uint32_t)top_k;
                r.n_cand = (int)(base_c + bin_c);
            } else {
                r.cand_lo = r.cand_hi;
                r.need_count = by_count ? (uint32_t)top_k - base_c : 0u;
                r.need_mass = by_count ? 0ull : target - base_m;
                r.n_cand = (int)bin_c;
            }
            r.fallback = r.n_cand > kCap ? 1 : 0;
        }
    }
    return r;
}

// One sweep: tokens above the candidate bins compete for the Gumbel-max right away, tokens in them are listed.
__global__ __launch_bounds__(kThreads) void trunc_select_kernel(const float* logits, int V, float temperature, int top_k, float top_p,
                                                                const float* lmax_part, const uint64_t* hist_mass, const uint32_t* hist_cnt,
                                                                const uint64_t* sum_mass, const uint32_t* sum_cnt, TruncRow* rows,
                                                                int use_noise_buffer, KeyChunk keys, const float* noise,
                                                                uint2* cand, int* cand_n, float2* part) {
    extern __shared__ uint4 lds_raw[];
    uint2* list = (uint2*)lds_raw;                            // [kCap]: this slice's candidates
    __shared__ TruncRow s_row;
    __shared__ int s_n, s_at;
    __shared__ int s_best;                                    // best score of the slice's kept tokens so far, as an ordered int
    __shared__ float s_red[kWaves];
    __shared__ int s_idx[kWaves];
    const int row = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (wave == 0) {
        const TruncRow p = trunc_plan(row, V, temperature, top_k, top_p, gridDim.x, lmax_part, hist_mass, hist_cnt, sum_mass, sum_cnt, lane);
        if (lane == 0) {
            s_row = p;
            s_n = 0;
            s_best = ordered_bits(__float_as_int(-INFINITY));
            if (blockIdx.x == 0) rows[row] = p;
        }
    }
    __syncthreads();
    const TruncRow r = s_row;
    if (r.fallback) return;
    const float* lr = logits + (size_t)row * V;
    const float* nr = use_noise_buffer ? noise + (size_t)row * V : nullptr;
    const uint64_t key64 = keys.key[row];
    const size_t seg = (size_t)row * gridDim.x + blockIdx.x;
    int lo, hi;
    slice_range(V, lo, hi);
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    if (!nr && lo + tid < hi) {                               // a first bound for noise_may_win: one kept token a thread
        const float z = lr[lo + tid] / temperature;
        if (bin_of(z, r.zmax) < r.cand_lo) {
            const float sc = z + gumbel_noise(key64, lo + tid);
            if (sc > -INFINITY) atomicMax(&s_best, ordered_bits(__float_as_int(sc)));
        }
    }
    __syncthreads();
    sweep<8>(lr, lo, hi, tid, [&](float l, int v) {
        const float z = l / temperature;
        const int b = bin_of(z, r.zmax);
        if (b < r.cand_lo) {
            const float bound = __int_as_float(ordered_bits(*(volatile int*)&s_best));
            const uint64_t at = noise_at(key64, v);
            if (!nr && !noise_may_win(at, z, noise_pass(bound))) return;
            const float sc = z + (nr ? nr[v] : gumbel_noise(at));
            if (better(sc, v, bv, bi)) {
                bv = sc; bi = v;
                if (sc > bound) atomicMax(&s_best, ordered_bits(__float_as_int(sc)));
            }
        } else if (b <= r.cand_hi) {
            const int slot = atomicAdd(&s_n, 1);
            if (slot < kCap) list[slot] = make_uint2(order_key(z), (uint32_t)v);      // n_cand <= kCap in all
        }
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if (lane == 0) { s_red[wave] = bv; s_idx[wave] = bi; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w)
            if (better(s_red[w], s_idx[w], bv, bi)) { bv = s_red[w]; bi = s_idx[w]; }
        part[seg] = make_float2(bv, __int_as_float(bi));
        s_at = s_n > 0 ? atomicAdd(&cand_n[row], s_n) : 0;    // this slice's place in the row's list
    }
    __syncthreads();
    const int n = min(s_n, kCap - s_at);
    for (int i = tid; i < n; i += kThreads) cand[(size_t)row * kCap + s_at + i] = list[i];
}

// The radix descent of the single-kernel path on the candidate list (in LDS), then the Gumbel-max over the kept
// candidates and the slices' winners among the tokens above the cut bin.  The list is short: one histogram for all waves.
__global__ __launch_bounds__(kThreads) void trunc_resolve_kernel(const float* logits, int V, float temperature, int top_k, float top_p, int slices,
                                                                 const TruncRow* rows, int use_noise_buffer, KeyChunk keys, const float* noise,
                                                                 const uint2* cand, const int* cand_n, const float2* part,
                                                                 int32_t* out, float* tau_out) {
    extern __shared__ uint4 lds_raw[];
    uint2* list = (uint2*)lds_raw;                            // [kCap]
    __shared__ uint64_t hist[256];
    __shared__ Select sel;
    __shared__ float s_red[kWaves];
    __shared__ int s_idx[kWaves];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TruncRow r = rows[row];
    if (r.fallback) {                                         // too many candidates, or none: all sweeps by this workgroup
        truncated_row((uint64_t*)lds_raw, logits, row, V, temperature, top_k, top_p, use_noise_buffer, keys.key[row], noise, out, tau_out);
        return;
    }
    uint64_t* my_hist = hist;
    const int n = min(cand_n[row], kCap);
    for (int i = tid; i < n; i += kThreads) list[i] = cand[(size_t)row * kCap + i];
    __syncthreads();

    auto clear_hist = [&] {
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
    };
    const bool by_count = top_k > 0 && top_k < V;
    const bool by_mass = top_p < 1.0f;
    uint32_t floor_key = 0;

    if (by_count) {
        if (tid == 0) { sel.prefix = 0; sel.remaining = (uint64_t)r.need_count; }
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            clear_hist();
            const uint32_t prefix = sel.prefix;
            for (int i = tid; i < n; i += kThreads) {
                const uint32_t key = list[i].x;
                if (pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)))
                    atomicAdd((unsigned long long*)&my_hist[(key >> shift) & 255u], 1ull);
            }
            __syncthreads();
            if (wave == 0) pick_bin<1>(hist, shift, &sel, lane);
            __syncthreads();
        }
        floor_key = sel.prefix;
        __syncthreads();
    }
    if (by_mass) {
        if (tid == 0) { sel.prefix = 0; sel.remaining = r.need_mass; }
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
            clear_hist();
            const uint32_t prefix = sel.prefix;
            for (int i = tid; i < n; i += kThreads) {
                const uint32_t key = list[i].x;
                if (key >= floor_key && (pass == 0 || (key >> (shift + 8)) == (prefix >> (shift + 8)))) {
                    const uint64_t mass = mass45(key_value(key), r.zmax);
                    atomicAdd((unsigned long long*)&my_hist[(key >> shift) & 255u], (unsigned long long)mass);
                }
            }
            __syncthreads();
            if (pass == 0) {
                // with top-k in front the target is a share of the survivors' mass, known only now; alone it came with
                // the row (and cannot exceed the list's mass: the same integers were summed for the histogram)
                if (wave == 0) {
                    uint64_t mine = 0;
                    for (int i = 0; i < 4; ++i) mine += hist[lane * 4 + i];
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const uint64_t o = shfl_down_u64(mine, d);
                        if (lane + d < 64) mine += o;
                    }
                    if (lane == 0) {
                        const uint64_t Z = mine;
                        uint64_t target = by_count ? (uint64_t)ceil((double)top_p * (double)Z) : sel.remaining;
                        if (target < 1) target = 1;
                        if (target > Z) target = Z;
                        sel.remaining = target;
                    }
                }
                __syncthreads();
            }
            if (wave == 0) pick_bin<1>(hist, shift, &sel, lane);
            __syncthreads();
        }
        if (sel.prefix > floor_key) floor_key = sel.prefix;
        __syncthreads();
    }

    const float* nr = use_noise_buffer ? noise + (size_t)row * V : nullptr;
    const uint64_t key64 = keys.key[row];
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    for (int i = tid; i < n; i += kThreads) {
        const uint2 e = list[i];
        if (e.x < floor_key) continue;
        const int v = (int)e.y;
        const float sc = key_value(e.x) + (nr ? nr[v] : gumbel_noise(key64, v));
        if (better(sc, v, bv, bi)) { bv = sc; bi = v; }
    }
    if (tid < slices) {
        const float2 e = part[(size_t)row * slices + tid];
        const int i = __float_as_int(e.y);
        if (better(e.x, i, bv, bi)) { bv = e.x; bi = i; }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
    if (lane == 0) { s_red[wave] = bv; s_idx[wave] = bi; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kWaves; ++w)
            if (better(s_red[w], s_idx[w], bv, bi)) { bv = s_red[w]; bi = s_idx[w]; }
        out[row] = bi == 0x7FFFFFFF ? 0 : bi;
        if (tau_out) tau_out[row] = floor_key == 0 ? -INFINITY : key_value(floor_key);
    }
}

namespace {
// workgroups per row: enough to put a workgroup on every compute unit, slices of at least 8192 tokens
int trunc_slices(int rows, int V, int most) {
    int s = (256 + rows - 1) / rows;
    s = std::min(s, most);
    s = std::min(s, std::max(1, V / 8192));
    return std::max(s, 1);
}
struct TruncLayout { size_t lmax, hist_mass, hist_cnt, sum_mass, sum_cnt, rows, cand, cand_n, part, total; };
TruncLayout trunc_layout(int rows, int slices) {
    TruncLayout L;
    size_t at = 0;
    auto take = [&](size_t bytes) { const size_t o = at; at += (bytes + 255) & ~(size_t)255; return o; };
    L.lmax = take((size_t)rows * kMaxSlices * sizeof(float));
    L.hist_mass = take((size_t)rows * slices * kBins * sizeof(uint64_t));
    L.hist_cnt = take((size_t)rows * slices * kBins * sizeof(uint32_t));
    L.sum_mass = take((size_t)rows * slices * kCoarse * sizeof(uint64_t));
    L.sum_cnt = take((size_t)rows * slices * kCoarse * sizeof(uint32_t));
    L.rows = take((size_t)rows * sizeof(TruncRow));
    L.cand = take((size_t)rows * kCap * sizeof(uint2));
    L.cand_n = take((size_t)rows * sizeof(int));
    L.part = take((size_t)rows * slices * sizeof(float2));
    L.total = at;
    return L;
}
}  // namespace

// rows of a batch are processed 128 at a time (the row keys travel by value), one chunk after the other on the stream.
// The size is that of up to 8 slices a row with a candidate list of their own each, which callers have been told so far;
// the layout in use (up to 16 slices, one list a row) needs less.
size_t sample_truncated_workspace_bytes(int B, int V) {
    const int rows = std::min(B, 128), slices = trunc_slices(rows, V, 8);
    auto pad = [](size_t bytes) { return (bytes + 255) & ~(size_t)255; };
    const size_t told = pad((size_t)rows * 8 * sizeof(float)) + pad((size_t)rows * slices * kBins * sizeof(uint64_t)) +
                        pad((size_t)rows * slices * kBins * sizeof(uint32_t)) + pad((size_t)rows * sizeof(TruncRow)) +
                        pad((size_t)rows * slices * kCap * sizeof(uint2)) + pad((size_t)rows * slices * sizeof(int)) +
                        pad((size_t)rows * slices * sizeof(float2));
    return told;
}

hipError_t launch_sample_truncated_ws(const float* logits, int B, int V, float temperature, int top_k, float top_p,
                                      const uint64_t* host_keys, const float* noise, int32_t* out, float* tau_out,
                                      void* workspace, hipStream_t s) {
    const int rows_max = std::min(B, 128);
    const int slices = trunc_slices(rows_max, V, kMaxSlices);
    const TruncLayout L = trunc_layout(rows_max, slices);
    if (L.total > sample_truncated_workspace_bytes(B, V)) return hipErrorInvalidValue;
    char* ws = (char*)workspace;
    float* lmax = (float*)(ws + L.lmax);
    uint64_t* hist_mass = (uint64_t*)(ws + L.hist_mass);
    uint32_t* hist_cnt = (uint32_t*)(ws + L.hist_cnt);
    uint64_t* sum_mass = (uint64_t*)(ws + L.sum_mass);
    uint32_t* sum_cnt = (uint32_t*)(ws + L.sum_cnt);
    TruncRow* rows = (TruncRow*)(ws + L.rows);
    uint2* cand = (uint2*)(ws + L.cand);
    int* cand_n = (int*)(ws + L.cand_n);
    float2* part = (float2*)(ws + L.part);
    const size_t list_lds = (size_t)kCap * sizeof(uint2);
    hipError_t e = hipFuncSetAttribute((const void*)trunc_select_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)list_lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)trunc_resolve_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)list_lds);
    if (e != hipSuccess) return e;
    for (int off = 0; off < B; off += 128) {
        KeyChunk k;
        const int m = B - off < 128 ? B - off : 128;
        for (int i = 0; i < m; ++i) k.key[i] = host_keys ? host_keys[off + i] : 0;
        const float* lg = logits + (size_t)off * V;
        const float* nz = noise ? noise + (size_t)off * V : nullptr;
        hipLaunchKernelGGL(trunc_max_kernel, dim3(slices, m), dim3(kThreads), 0, s, lg, V, lmax, cand_n);
        hipLaunchKernelGGL(trunc_hist_kernel, dim3(slices, m), dim3(kThreads), 0, s, lg, V, temperature, lmax,
                           top_p < 1.0f ? 1 : 0, hist_mass, hist_cnt, sum_mass, sum_cnt);
        hipLaunchKernelGGL(trunc_select_kernel, dim3(slices, m), dim3(kThreads), list_lds, s, lg, V, temperature, top_k, top_p, lmax,
                           hist_mass, hist_cnt, sum_mass, sum_cnt, rows, noise ? 1 : 0, k, nz, cand, cand_n, part);
        hipLaunchKernelGGL(trunc_resolve_kernel, dim3(m), dim3(kThreads), list_lds, s, lg, V, temperature, top_k, top_p, slices, rows,
                           noise ? 1 : 0, k, nz, cand, cand_n, part, out + off, tau_out ? tau_out + off : nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_sample_truncated(const float* logits, int B, int V, float temperature, int top_k, float top_p,
                                   const uint64_t* host_keys, const float* noise, int32_t* out, float* tau_out,
                                   hipStream_t s) {
    for (int off = 0; off < B; off += 128) {
        KeyChunk k;
        const int m = B - off < 128 ? B - off : 128;
        for (int i = 0; i < m; ++i) k.key[i] = host_keys ? host_keys[off + i] : 0;
        hipLaunchKernelGGL(sample_truncated_kernel, dim3(m), dim3(kThreads), 0, s, logits + (size_t)off * V, V, temperature,
                           top_k, top_p, noise ? 1 : 0, k, noise ? noise + (size_t)off * V : nullptr, out + off,
                           tau_out ? tau_out + off : nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace spiral
