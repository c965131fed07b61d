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
// workgroups per row: (1) row maximum; (2) one histogram over 4096 bins that are linear in zmax - z (width 1/128; the last bin takes
// everything 32 or more below the maximum, whose mass is zero in the 2^45 fixed point), with sums over every 64 bins: of counts where there is a
// top-k, by which the cut then goes (top-p is a share of the survivors' mass, which the last kernel finds), else of mass; (3) one sweep whose
// workgroups first find the bin that holds the cut (an integer prefix sum over the 64 sums, then over the 64 bins below one of them) and the least
// logits that lie in it and above it, then score the tokens above for the Gumbel-max and copy the tokens of the cut bin (one to a few
// hundred) to the row's candidate list, on which the radix descent then runs in LDS, in a last kernel of a workgroup per row.  Bin order
// follows key order and the masses are the same integers, so the threshold is the one the single-kernel path finds, bit for bit; a
// row whose cut bin holds more candidates than the list (many equal scores) is done by that path's code in the last kernel.
// Many rows: bound by the fixed-point exponentials of the histogram and the generator's integer arithmetic of the sweep; few: by four dependent
// launches, each a chain of a few loads, barriers and reductions.  151,936 entries, T = 0.6, top-p 0.95, us a call, with six launches and at most 8 slices a
// row / with both histograms, a division and a bin an entry in the sweep, one wave adding up the slices, four digits always and thread 0 comparing
// the waves' results / now: one row 59 / 30.7 / 22.4, 16 rows 55 / 35.0 / 27.4, 64 - / 57.6 / 47.8, 128 - / 94.8 / 72.3, of flat logits
// 130 / 111 / 86; 16 rows, top-k 50 - / 29.4 / 22.3, top-k 20 with top-p 0.9 - / 36.9 / 26.9.  (16 rows, traced: maximum 4.0 -> 3.4,
// histogram 11.9 -> 9.0, sweep 12.1 -> 10.0, last kernel 8.0 -> 6.1.)
#include <algorithm>
#include <type_traits>

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
// first use; past the end they re-read the last entry, a branch around a load would make every load wait).  Indices are unsigned: they
// run ahead of a row that may have 2^31 - 1 entries.
template <int U, class F>
__device__ __forceinline__ void sweep(const float* lr, uint32_t lo, uint32_t hi, int tid, F&& f) {
    for (uint32_t base = lo + tid; base < hi; base += kThreads * U) {
        float l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) l[u] = lr[min(base + u * kThreads, hi - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t v = base + u * kThreads;
            if (v < hi) f(l[u], (int)v);
        }
    }
}

// The same by threads that hold VEC neighbouring entries a load (4: rows of a multiple of four entries, 16-byte aligned, lo and hi multiples of
// four).  The first step's loads are issued by the constructor, so that what comes before run() hides them, every other step's under the step before.
template <int VEC>
struct Sweep {
    static constexpr int U = VEC == 4 ? 3 : 8, STEP = kThreads * VEC * U;
    typedef __attribute__((ext_vector_type(VEC))) float vec;
    const float* lr;
    uint32_t base, hi;
    vec next[U];
    __device__ __forceinline__ Sweep(const float* lr_, uint32_t lo, uint32_t hi_, int tid) : lr(lr_), base(lo + tid * VEC), hi(hi_) {
        if (base < hi) load(base);
    }
    __device__ __forceinline__ void load(uint32_t at) {
#pragma unroll
        for (int u = 0; u < U; ++u) next[u] = *(const vec*)(lr + min(at + u * kThreads * VEC, hi - VEC));
    }
    // step() before every step's entries, f(logit, v) for each
    template <class S, class F>
    __device__ __forceinline__ void run(S&& step, F&& f) {
        for (; base < hi; base += STEP) {
            vec l[U];
#pragma unroll
            for (int u = 0; u < U; ++u) l[u] = next[u];
            load(base + STEP);
            step();
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (base + u * kThreads * VEC < hi)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) f(l[u][e], (int)(base + u * kThreads * VEC + e));
        }
    }
};

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
// `tab`: the table, or a copy of it in LDS.
__device__ __forceinline__ uint64_t mass45(float z, float zmax, const double* tab = kExp2Tab) {
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
    // to an integer: below 2^52, floor(x) + 2^52 has it in its lower bits (the general conversion is several times that)
    const double m = floor(ldexp(tab[ki & 31] * p, (ki >> 5) + 45)) + 4503599627370496.0;
    return (uint64_t)__double_as_longlong(m) & 0xFFFFFFFFFFFFFull;
}

constexpr int kBins = 4096;           // linear in zmax - z, 1/128 wide; the last one is everything >= 32 below the maximum
constexpr int kCap = 8192;            // candidates of a row that the in-LDS resolution takes
constexpr int kCoarse = 64;           // sums of 64 bins each
constexpr int kMaxSlices = 16;        // workgroups per row
static_assert(kMaxSlices <= kWaves, "a wave of the last sweep reads one slice's sums");

// What the prefix sum over a row's histogram decides (one per row, in the workspace).
struct TruncRow {
    float zmax;
    int cand_lo, cand_hi;             // tokens in bins [cand_lo, cand_hi] go to the candidate list; bins below cand_lo are kept
    int fallback;                     // no cut found, or (top-k) more candidates than the list holds: the single-kernel path does this row
    uint64_t need_mass;               // top-p alone: fixed-point mass still to be covered inside the candidate bin
    uint32_t need_count;              // top-k: how many of the candidates, from the largest, are kept
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

// The best of the waves' (score, index) pairs, in every lane of the wave that calls this.
__device__ __forceinline__ void best_of_waves(const float* s_red, const int* s_idx, int lane, float& bv, int& bi) {
    bv = s_red[lane & (kWaves - 1)];
    bi = s_idx[lane & (kWaves - 1)];
#pragma unroll
    for (int o = kWaves / 2; o > 0; o >>= 1) {
        const float ov = __shfl_xor(bv, o, 64);
        const int oi = __shfl_xor(bi, o, 64);
        if (better(ov, oi, bv, bi)) { bv = ov; bi = oi; }
    }
}

// `per`: entries of a slice, blockIdx.x; a multiple of VEC.
template <int VEC>
__global__ __launch_bounds__(kThreads) void trunc_max_kernel(const float* logits, int V, int per, float* lmax_part, int* cand_n) {
    __shared__ float s_red[kWaves];
    const int row = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lo = (int)blockIdx.x * per;
    Sweep<VEC> sw(logits + (size_t)row * V, lo, min((uint32_t)V, (uint32_t)lo + per), tid);
    float m = -INFINITY;
    sw.run([] {}, [&](float l, int) { m = fmaxf(m, l); });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane == 0) s_red[wave] = m;
    __syncthreads();
    if (wave != 0) return;
    m = s_red[lane & (kWaves - 1)];
#pragma unroll
    for (int o = kWaves / 2; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if (lane == 0) {
        lmax_part[row * kMaxSlices + blockIdx.x] = m;
        if (blockIdx.x == 0) cand_n[row] = 0;
    }
}

// the row's largest logit, by a wave; z's maximum is that / T, as division by T > 0 is monotone
__device__ __forceinline__ float row_lmax(const float* lmax_part, int row, int slices, int lane) {
    float m = lane < slices ? lmax_part[row * kMaxSlices + lane] : -INFINITY;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    return __shfl(m, 0, 64);
}

__device__ __forceinline__ uint64_t shfl_down_any(uint64_t v, int d) { return shfl_down_u64(v, d); }
__device__ __forceinline__ uint32_t shfl_down_any(uint32_t v, int d) { return __shfl_down(v, d, 64); }

// H: uint64_t, the mass of every bin, or uint32_t, the number of its tokens (with top-k, which the cut then goes by).
template <int VEC, class H>
__global__ __launch_bounds__(kThreads) void trunc_hist_kernel(const float* logits, int V, int per, float temperature, const float* lmax_part,
                                                              H* hist, H* sums) {
    constexpr bool MASS = sizeof(H) == 8;
    __shared__ H h[kBins];
    __shared__ double s_exp2[32];
    const int row = blockIdx.y, tid = threadIdx.x;
    const int lo = (int)blockIdx.x * per;
    const float zmax = row_lmax(lmax_part, row, gridDim.x, tid & 63) / temperature;
    Sweep<VEC> sw(logits + (size_t)row * V, lo, min((uint32_t)V, (uint32_t)lo + per), tid);
    if (MASS && tid < 32) s_exp2[tid] = kExp2Tab[tid];
    for (int i = tid; i < kBins; i += kThreads) h[i] = 0;
    __syncthreads();
    sw.run([] {}, [&](float l, int) {
        const float z = l / temperature;
        const int b = bin_of(z, zmax);
        if constexpr (MASS) {
            const uint64_t m = mass45(z, zmax, s_exp2);
            if (m) atomicAdd((unsigned long long*)&h[b], (unsigned long long)m);
        } else {
            atomicAdd(&h[b], 1u);
        }
    });
    __syncthreads();
    const size_t seg = (size_t)row * gridDim.x + blockIdx.x;
    for (int i = tid; i < kBins; i += kThreads) hist[seg * kBins + i] = h[i];
    H sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) sum += h[tid * 4 + i];       // 16 threads to a sum
#pragma unroll
    for (int d = 8; d > 0; d >>= 1) sum += shfl_down_any(sum, d);
    if ((tid & 15) == 0) sums[seg * kCoarse + (tid >> 4)] = sum;
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int d) {
    const uint32_t lo = __shfl_up((uint32_t)v, d, 64), hi = __shfl_up((uint32_t)(v >> 32), d, 64);
    return ((uint64_t)hi << 32) | lo;
}

// Prefix sums over the bins of a row (bin 0 = the largest z) and the bin in which the cut falls, two levels of 64, by a
// workgroup: wave s brings the entries of slice s, all at once, the first wave adds and searches them.  (One wave that read four slices at a
// time waited eight times for memory.)  coarse: the sum of slice `wave` at `lane`; s_sum: LDS, [kMaxSlices][64].
// The first wave returns with the plan.
__device__ __forceinline__ TruncRow trunc_plan(int row, int V, float zmax, int top_k, float top_p, int slices,
                                               const uint64_t* hist_mass, const uint32_t* hist_cnt, uint64_t coarse, uint64_t* s_sum) {
    __shared__ int s_first;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    TruncRow r = {};
    r.zmax = zmax;
    const bool by_count = top_k > 0 && top_k < V;
    const bool by_mass = top_p < 1.0f;
    uint64_t target = (uint64_t)top_k, base = 0;              // of tokens, or of mass
    int first = 0;                                           // the 64 entries of the level start here
#pragma unroll
    for (int level = 0; level < 2; ++level) {
        if (level == 1) {
            if (threadIdx.x == 0) s_first = first;
            __syncthreads();
            first = s_first;
        }
        if (first < 0) continue;                             // no bin qualifies (every thread of the workgroup knows)
        if (wave < slices) {
            const size_t bin = ((size_t)row * slices + wave) * kBins + first + lane;
            s_sum[wave * 64 + lane] = level == 0 ? coarse : by_count ? (uint64_t)hist_cnt[bin] : hist_mass[bin];
        }
        __syncthreads();
        if (wave != 0) continue;
        uint64_t own = 0;
        for (int s = 0; s < slices; ++s) own += s_sum[s * 64 + lane];
        uint64_t sum = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint64_t o = shfl_up_u64(sum, d);
            if (lane >= d) sum += o;
        }
        if (level == 0 && !by_count) {
            const uint64_t total = ((uint64_t)__shfl((uint32_t)(sum >> 32), 63, 64) << 32) | __shfl((uint32_t)sum, 63, 64);
            target = (uint64_t)ceil((double)top_p * (double)total);
            if (target < 1) target = 1;
            if (target > total) target = total;
        }
        const uint64_t before = base + sum - own;
        const bool here = before < target && target <= before + own;
        const uint64_t where = __builtin_amdgcn_ballot_w64(here);
        if (where == 0) { r.fallback = 1; first = -1; continue; }        // no bin qualifies (a row of NaN): the single path's business
        const int at = __builtin_ctzll(where);               // exactly one
        base = ((uint64_t)__shfl((uint32_t)(before >> 32), at, 64) << 32) | __shfl((uint32_t)before, at, 64);
        if (level == 0) {
            first = at * (kBins / kCoarse);
        } else {
            r.cand_hi = first + at;
            if (by_count) {                                  // too many for the list: known here; by mass, when they have been listed
                const uint64_t through = base + (uint64_t)__shfl((uint32_t)own, at, 64);
                // top-p needs the mass of the top-k survivors: resolve both on the list
                r.cand_lo = by_mass ? 0 : r.cand_hi;
                r.need_count = (uint32_t)(by_mass ? target : target - base);
                r.fallback = (by_mass ? through : through - base) > kCap ? 1 : 0;
            } else {
                r.cand_lo = r.cand_hi;
                r.need_mass = target - base;
            }
        }
    }
    return r;
}

// The least logit whose bin is at most `most`, NaN (which no logit reaches) where there is none, in both halves of a wave with a `most` each.  Division by
// T > 0 and the binning are monotone, so entries can be told apart by this one comparison instead of a division and the arithmetic of the bin
// each.  Five bits of the logit's order-preserving key at a time: lane i of a half tries the last key of the i-th range.  Undefined
// and -inf logits lie in the last bin, which is not asked for here (most < kBins - 1); keys above the row's maximum count as it.
__device__ __forceinline__ float bin_threshold(int most, float zmax, float lmax, float temperature, int lane) {
    const uint32_t top = order_key(lmax), bottom = order_key(-INFINITY);
    const int i = lane & 31;
    auto reaches = [&](uint32_t key) { return key > bottom && bin_of((key < top ? key_value(key) : lmax) / temperature, zmax) <= most; };
    uint32_t at = 0;
#pragma unroll
    for (int shift = 30; shift >= 0; shift -= 5) {
        const uint32_t last = at + ((uint32_t)(shift == 30 ? i & 3 : i) << shift) + ((1u << shift) - 1u);
        const uint64_t hit = __builtin_amdgcn_ballot_w64(reaches(last));
        const uint32_t mine = (uint32_t)(hit >> (lane & 32));
        // a range whose last key reaches it exists, or (first step: the row's maximum does not) there is none at all
        at += (mine ? (uint32_t)__builtin_ctz(mine) : 0u) << shift;
    }
    return reaches(at) ? key_value(at) : NAN;
}

// One sweep: tokens above the candidate bins compete for the Gumbel-max right away, tokens in them are listed.
template <int VEC>
__global__ __launch_bounds__(kThreads) void trunc_select_kernel(const float* logits, int V, int per, float temperature, int top_k, float top_p,
                                                                const float* lmax_part, const uint64_t* hist_mass, const uint32_t* hist_cnt,
                                                                const uint64_t* sum_mass, const uint32_t* sum_cnt, TruncRow* rows,
                                                                int use_noise_buffer, KeyChunk keys, const float* noise,
                                                                uint2* cand, int* cand_n, float2* part) {
    extern __shared__ uint4 lds_raw[];
    uint2* list = (uint2*)lds_raw;                            // [kCap]: this slice's candidates; before, the plan's sums
    __shared__ int s_fallback;
    __shared__ float s_keep, s_list;                          // logits from s_keep on are kept, below it those from s_list on are listed
    __shared__ int s_n, s_at;
    __shared__ int s_best;                                    // best score of the slice's kept tokens so far, as an ordered int
    __shared__ float s_red[kWaves];
    __shared__ int s_idx[kWaves];
    const int row = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lo = (int)blockIdx.x * per, hi = (int)min((uint32_t)V, (uint32_t)lo + per);
    const float lmax = row_lmax(lmax_part, row, gridDim.x, lane);
    // (loads return in order: the plan's before the first logits)
    const size_t seg = (size_t)row * gridDim.x + blockIdx.x, seg_wave = (size_t)row * gridDim.x + min(wave, (int)gridDim.x - 1);
    const uint64_t coarse = top_k > 0 && top_k < V ? (uint64_t)sum_cnt[seg_wave * kCoarse + lane] : sum_mass[seg_wave * kCoarse + lane];
    Sweep<VEC> sw(logits + (size_t)row * V, lo, hi, tid);
    const TruncRow p = trunc_plan(row, V, lmax / temperature, top_k, top_p, gridDim.x, hist_mass, hist_cnt, coarse, (uint64_t*)lds_raw);
    if (wave == 0) {
        const int most = lane < 32 ? p.cand_lo - 1 : p.cand_hi;
        float t = bin_threshold(most, p.zmax, lmax, temperature, lane);
        if (most < 0) t = NAN;
        if (lane == 32) s_list = p.cand_hi == kBins - 1 ? -INFINITY : t;
        if (lane == 0) {
            s_keep = t;
            s_fallback = p.fallback;
            s_n = 0;
            s_best = ordered_bits(__float_as_int(-INFINITY));
            if (blockIdx.x == 0) rows[row] = p;
        }
    }
    __syncthreads();
    if (s_fallback) return;
    const float keep = s_keep, from = s_list;
    const bool all = from == -INFINITY;                       // undefined logits too
    const float* nr = use_noise_buffer ? noise + (size_t)row * V : nullptr;
    const uint64_t key64 = keys.key[row];
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    if (!nr && sw.base < (uint32_t)hi && sw.next[0][0] >= keep) {       // a first bound for the screen: one kept token a thread
        const float sc = sw.next[0][0] / temperature + gumbel_noise(key64, (int)sw.base);
        if (sc > -INFINITY) atomicMax(&s_best, ordered_bits(__float_as_int(sc)));
    }
    __syncthreads();
    const float scale = screen_scale(temperature);
    float bound = -INFINITY, pass = -INFINITY;
    bool full = false;                                        // more candidates than the list holds: the last kernel does the row
    sw.run([&] {
        bound = __int_as_float(ordered_bits(*(volatile int*)&s_best));
        pass = screen_pass(bound);
        full = *(volatile int*)&s_n > kCap;
    }, [&](float l, int v) {
        if (l >= keep) {
            const uint64_t at = noise_at(key64, v);
            if (!nr && !screen_may_win(at, l, scale, pass)) return;
            const float sc = l / temperature + (nr ? nr[v] : gumbel_noise(at));
            if (better(sc, v, bv, bi)) {
                bv = sc; bi = v;
                if (sc > bound) atomicMax(&s_best, ordered_bits(__float_as_int(sc)));
            }
        } else if ((l >= from || all) && !full) {
            const int slot = atomicAdd(&s_n, 1);
            if (slot < kCap) list[slot] = make_uint2(order_key(l / temperature), (uint32_t)v);
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
    if (wave == 0) best_of_waves(s_red, s_idx, lane, bv, bi);
    if (tid == 0) {
        part[seg] = make_float2(bv, __int_as_float(bi));
        s_at = s_n > 0 ? atomicAdd(&cand_n[row], s_n) : 0;    // this slice's place in the row's list
    }
    __syncthreads();
    const int n = min(s_n, kCap - s_at);
    for (int i = tid; i < n; i += kThreads) cand[(size_t)row * kCap + s_at + i] = list[i];
}

// The radix descent of the single-kernel path on the candidate list (in LDS), then the Gumbel-max over the kept
// candidates and the slices' winners among the tokens above the cut bin.  The list is short: one histogram for all waves.  Its keys mostly come
// from one bin and share their upper bits: the descent starts at the first digit in which any two differ.
__global__ __launch_bounds__(kThreads) void trunc_resolve_kernel(const float* logits, int V, float temperature, int top_k, float top_p, int slices,
                                                                 const TruncRow* rows, int use_noise_buffer, KeyChunk keys, const float* noise,
                                                                 const uint2* cand, const int* cand_n, const float2* part,
                                                                 int32_t* out, float* tau_out) {
    extern __shared__ uint4 lds_raw[];
    uint2* list = (uint2*)lds_raw;                            // [kCap]
    __shared__ uint64_t hist[256];
    __shared__ Select sel;
    __shared__ uint32_t s_diff;
    __shared__ double s_exp2[32];
    __shared__ float s_red[kWaves];
    __shared__ int s_idx[kWaves];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_listed = cand_n[row];
    const uint2 c0 = cand[(size_t)row * kCap], c_tid = cand[(size_t)row * kCap + tid];        // asked for before n is known, used below it
    const TruncRow r = rows[row];
    if (r.fallback || n_listed > kCap) {                      // too many candidates, or none: all sweeps by this workgroup
        truncated_row((uint64_t*)lds_raw, logits, row, V, temperature, top_k, top_p, use_noise_buffer, keys.key[row], noise, out, tau_out);
        return;
    }
    uint64_t* my_hist = hist;
    const int n = n_listed;
    if (tid == 0) s_diff = 0;
    if (tid < 32) s_exp2[tid] = kExp2Tab[tid];
    __syncthreads();
    uint32_t diff = 0;
    if (tid < n) { list[tid] = c_tid; diff = c_tid.x ^ c0.x; }
    for (int i = tid + kThreads; i < n; i += kThreads) {
        const uint2 e = cand[(size_t)row * kCap + i];
        list[i] = e;
        diff |= e.x ^ c0.x;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) diff |= __shfl_xor(diff, o, 64);
    if (lane == 0 && diff) atomicOr(&s_diff, diff);
    __syncthreads();
    // digits below which all keys agree; the digits above are the first key's
    const uint32_t any = s_diff;
    const int first_shift = any >> 24 ? 24 : any >> 16 ? 16 : any >> 8 ? 8 : 0;
    const uint32_t shared_bits = n > 0 && first_shift < 24 ? c0.x & ~((256u << first_shift) - 1u) : 0u;

    auto clear_hist = [&] {
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
    };
    const bool by_count = top_k > 0 && top_k < V;
    const bool by_mass = top_p < 1.0f;
    uint32_t floor_key = 0;

    if (by_count) {
        if (tid == 0) { sel.prefix = shared_bits; sel.remaining = (uint64_t)r.need_count; }
        for (int shift = first_shift; shift >= 0; shift -= 8) {
            clear_hist();
            const uint32_t prefix = sel.prefix;
            for (int i = tid; i < n; i += kThreads) {
                const uint32_t key = list[i].x;
                if (shift == first_shift || (key >> (shift + 8)) == (prefix >> (shift + 8)))
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
        if (tid == 0) { sel.prefix = shared_bits; sel.remaining = r.need_mass; }
        for (int shift = first_shift; shift >= 0; shift -= 8) {
            clear_hist();
            const uint32_t prefix = sel.prefix;
            for (int i = tid; i < n; i += kThreads) {
                const uint32_t key = list[i].x;
                if (key >= floor_key && (shift == first_shift || (key >> (shift + 8)) == (prefix >> (shift + 8)))) {
                    const uint64_t mass = mass45(key_value(key), r.zmax, s_exp2);
                    atomicAdd((unsigned long long*)&my_hist[(key >> shift) & 255u], (unsigned long long)mass);
                }
            }
            __syncthreads();
            if (by_count && shift == first_shift) {
                // with top-k in front the target is a share of the survivors' mass, known only now; alone it came with
                // the row (and is 1 at least and no more than the list's mass: the same integers were summed for the histogram)
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
                        uint64_t target = (uint64_t)ceil((double)top_p * (double)Z);
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
    if (wave == 0) best_of_waves(s_red, s_idx, lane, bv, bi);
    if (tid == 0) {
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
    const bool wide = (V & 3) == 0 && ((uintptr_t)logits & 15) == 0;
    int per = (int)(((long long)V + slices - 1) / slices);
    if (wide) per = (per + 3) & ~3;
    hipError_t e = hipFuncSetAttribute(wide ? (const void*)trunc_select_kernel<4> : (const void*)trunc_select_kernel<1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)list_lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)trunc_resolve_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)list_lds);
    if (e != hipSuccess) return e;
    for (int off = 0; off < B; off += 128) {
        KeyChunk k;
        const int m = B - off < 128 ? B - off : 128;
        for (int i = 0; i < m; ++i) k.key[i] = host_keys ? host_keys[off + i] : 0;
        const float* lg = logits + (size_t)off * V;
        const float* nz = noise ? noise + (size_t)off * V : nullptr;
        auto sweeps = [&](auto vec) {
            constexpr int VEC = decltype(vec)::value;
            const dim3 g(slices, m), b(kThreads);
            hipLaunchKernelGGL(trunc_max_kernel<VEC>, g, b, 0, s, lg, V, per, lmax, cand_n);
            if (top_k > 0 && top_k < V) hipLaunchKernelGGL((trunc_hist_kernel<VEC, uint32_t>), g, b, 0, s, lg, V, per, temperature, lmax, hist_cnt, sum_cnt);
            else hipLaunchKernelGGL((trunc_hist_kernel<VEC, uint64_t>), g, b, 0, s, lg, V, per, temperature, lmax, hist_mass, sum_mass);
            hipLaunchKernelGGL(trunc_select_kernel<VEC>, g, b, list_lds, s, lg, V, per, temperature, top_k, top_p, lmax, hist_mass, hist_cnt,
                               sum_mass, sum_cnt, rows, noise ? 1 : 0, k, nz, cand, cand_n, part);
        };
        if (wide) sweeps(std::integral_constant<int, 4>());
        else sweeps(std::integral_constant<int, 1>());
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
