// Eviction step kernels for gfx950: perturbed keys, segmented Gumbel-top-k
// selection with its ordered-subset log-probability, in-place compaction of
// the surviving K/V rows, and the row append used between rounds.
//
// The selection itself lives in ngc_select.h.  Compiled with -ffp-contract=off:
// the noise arithmetic is an exact operation sequence (see ngc_noise.h).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <map>
#include <mutex>

#include "../../include/ngc.h"
#include "ngc_device.h"
#include "ngc_noise.h"
#include "ngc_select.h"
#include "ngc_logsum.h"

namespace ngc {

__global__ __launch_bounds__(256) void perturbed_keys_kernel(
    const float *__restrict__ logits, const int32_t *__restrict__ len, float *__restrict__ keys_out,
    int seg0, SegGeom g, NoiseArgs na, int32_t *status)
{
    const int seg = seg0 + blockIdx.x;
    int l, b, h;
    seg_coords(seg, g, l, b, h);
    const int n = seg_rows(len, seg, g.cap, status);
    const int n_items = (n + g.block - 1) / g.block;
    const float *row = logits + (size_t)seg * g.cap;
    float *out = keys_out + (size_t)seg * g.cap;
    for (int quad = threadIdx.x; 4 * quad < n_items; quad += 256) {
        float s[4], key[4];
        keys_of_quad(row, n_items, quad, na, l, b, h, s, key);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * quad + i < n_items) out[4 * quad + i] = key[i];
    }
}

// ------------------------------------------- log-prob of given actions ----

struct LogprobArgs {
    const float *logits;
    const int32_t *n_items;
    const int32_t *sigma;
    const int32_t *keep;
    float *logp_out;
    int32_t *status;
    int64_t logit_stride;
    int sigma_stride;
    int stage_cap;   // floats of dynamic LDS for the picked items' terms (general route)
    int row_cap;     // floats of dynamic LDS for a segment's row
};

// Both kernels below (Eq. 2 for given actions, and its gradient) read a segment's row and its sigma once.  The row's
// weights exp(s - max s) are computed once, by the threads that read the row, and stand in LDS; a pick takes its item's
// weight from there and leaves a mark (an exchange, which also finds repeated picks); what stays unmarked was never
// picked.
// Thread i owns PICKS consecutive picks -- thread 0 the LAST ones, so that an ordinary exclusive scan over threads yields
// the mass of everything picked after a thread's own -- and keeps their weights in registers between the passes.  Rows
// that do not fit (N > row_cap) and rows whose logits span more than NGC_WIDE_SPREAD take the general route: a bitmap of
// picked items and re-reads of the row.
//
// What bounds them: the vector ALU, three quarters busy.  3584 segments of ~2970 items and ~2460 picks (84 MB in, for
// the gradient 43 MB out; ~15 and ~24 us of traffic): three reads of the row and up to three gathers per pick 61 and
// 102 us; one read of the row 35 and 44 (570 and 726 instructions a wave); one exponential per item instead of one per pick
// and one per item and whatever the lanes of a wave disagree about, maxima of three, reductions that fold into their
// additions, a reciprocal instead of a division: 22.4 and 29.3 us.  log p is added up in 64 bits from the threads on (error
// against 64 bits 5.0e-8 -> 2.6e-8: it is a sum of thousands).
constexpr float PICKED = -1.0f;      // in the LDS row, where every weight is >= 0
constexpr int PICKED_WORDS = 2048;   // general route: a bit per item
constexpr int SPARE_ITEMS = 64;      // LDS words behind the row for lanes without a pick to mark (one each)
typedef f32x4 f32x4_any __attribute__((aligned(4)));    // rows start anywhere: 16-byte accesses need 4-byte alignment only
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef i32x4 i32x4_any __attribute__((aligned(4)));

// a value that is the same in every lane, as a scalar: what is decided by it is a branch
__device__ __forceinline__ float scalar(float x)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x)));
}

// QUADS: a thread holds the items 4 (i THREADS + tid) .. + 3 of a row of up to 4 QUADS THREADS items in registers.
template <int THREADS, int PICKS, int QUADS>
struct PickedTerms {
    f32x4 row[QUADS];   // held rows: the logits and, with KEEP_ROW once the picks are marked, exp(s - max s) or PICKED
    bool held;
    float e[PICKS];     // exp(s - max s) of this thread's picks (latest pick last); 0 past the end
    int t[PICKS];       // item index; -1 past the end, -2 for an index outside the segment
    float after;        // mass of everything picked after them
    float unpicked;     // mass never picked (U of Eq. 2)
    int count;          // picks of this thread
    int per;            // the most any thread has
};

// Returns false (workgroup-uniform) when the segment needs the general route; LDS is then free for it.
// lds_row: row_cap + SPARE_ITEMS floats; on return exp(s - max s) of the items never picked and PICKED for the others.
// fmisc: 32 floats.
template <int THREADS, int PICKS, int QUADS, bool KEEP_ROW>
__device__ __forceinline__ bool gather_picked(const float *row, const int32_t *sig, int N, int K, int row_cap,
                                              float *lds_row, float *fmisc, int32_t *status,
                                              PickedTerms<THREADS, PICKS, QUADS> &pt)
{
    constexpr int NW = THREADS / NGC_WAVE;
    const int tid = threadIdx.x;
    if (N > row_cap || K > THREADS * PICKS) return false;
    pt.held = N <= 4 * QUADS * THREADS;
    const int per = (K + THREADS - 1) / THREADS;          // <= PICKS
    const int owners = (K + per - 1) / per;
    const int j_lo = tid < owners ? (owners - 1 - tid) * per : 0;
    pt.per = per;
    pt.count = tid < owners ? (j_lo + per <= K ? per : K - j_lo) : 0;
#pragma unroll
    for (int i = 0; i < PICKS; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) pt.t[i + u] = -1;
        if (i < per && tid < owners) {
            if (j_lo + i + 4 <= K) {
                const i32x4 v = *reinterpret_cast<const i32x4_any *>(sig + j_lo + i);
#pragma unroll
                for (int u = 0; u < 4; ++u) pt.t[i + u] = v[u];
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (j_lo + i + u < K) pt.t[i + u] = sig[j_lo + i + u];
            }
        }
    }
    // Four items; those past the end repeat the first.
    auto load_quad = [&](int q) -> f32x4 {
        const float *p = row + 4 * q;
        if (4 * q + 4 <= N) return *reinterpret_cast<const f32x4_any *>(p);
        f32x4 x = {p[0], p[0], p[0], p[0]};
#pragma unroll
        for (int u = 1; u < 3; ++u)
            if (4 * q + u < N) x[u] = p[u];
        return x;
    };
    // body(q, x): x is the registers' copy where the row is held, otherwise read by load(q)
    auto each_quad = [&](auto load, auto body) {
        if (pt.held) {
#pragma unroll
            for (int i = 0; i < QUADS; ++i)
                if (4 * i * THREADS < N)                      // uniform
                    if (4 * (i * THREADS + tid) < N) body(i * THREADS + tid, pt.row[i]);
        } else {
            for (int q = tid; 4 * q < N; q += THREADS) {
                f32x4 x = load(q);
                body(q, x);
            }
        }
    };
    if (pt.held) {
#pragma unroll
        for (int i = 0; i < QUADS; ++i)
            if (4 * i * THREADS < N)
                if (4 * (i * THREADS + tid) < N) pt.row[i] = load_quad(i * THREADS + tid);
    }
    // a row that is not held waits in LDS for the maximum
    auto staged_quad = [&](int q) { return reinterpret_cast<const f32x4 *>(lds_row)[q]; };
    if (tid < SPARE_ITEMS) lds_row[row_cap + tid] = PICKED;
    // Largest and smallest logit.  These maxima and minima are NaN if one of the logits is; such rows and those with masked
    // entries look again, at the others alone.
    float smax = -INFINITY, smin = INFINITY;
    each_quad(load_quad, [&](int q, f32x4 &x) {
        if (!pt.held) reinterpret_cast<f32x4 *>(lds_row)[q] = x;
        smax = max_or_nan(max_or_nan(x[0], x[1]), smax);
        smax = max_or_nan(max_or_nan(x[2], x[3]), smax);
        smin = min_or_nan(min_or_nan(x[0], x[1]), smin);
        smin = min_or_nan(min_or_nan(x[2], x[3]), smin);
    });
    block_max_min<THREADS>(smax, smin, fmisc);
    smax = scalar(smax);                                      // uniform, and everything that follows from them
    smin = scalar(smin);
    const bool masked = !(smin > -INFINITY);
    if (masked) {
        float neg_smin = -INFINITY;
        smax = -INFINITY;
        each_quad(staged_quad, [&](int, f32x4 &x) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (x[u] == x[u]) smax = fmaxf(smax, x[u]);
                if (x[u] > -INFINITY) neg_smin = fmaxf(neg_smin, -x[u]);
            }
        });
        block_max2_f<THREADS>(smax, neg_smin, fmisc);
        smax = scalar(smax);
        smin = -scalar(neg_smin);
    }
    if (smax > -INFINITY && smax - smin > NGC_WIDE_SPREAD) return false;
    if (smax == -INFINITY) smax = 0.f;                        // every entry masked: all weights are 0
    // (a masked entry's weight is 0)
    auto difference = [&](float x) { return masked && !(x > -INFINITY) ? -300.0f : x - smax; };
    each_quad(staged_quad, [&](int q, f32x4 &x) {
        f32x4 e;
        if (masked) {
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = difference(x[u]);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) e[u] = x[u] - smax;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) e[u] = exp_shifted_finite(e[u]);
        if (4 * q + 4 > N) {                                  // past the end: no weight
#pragma unroll
            for (int u = 1; u < 4; ++u)
                if (4 * q + u >= N) e[u] = 0.f;
        }
        reinterpret_cast<f32x4 *>(lds_row)[q] = e;
    });
    __syncthreads();
    float mass = 0.f;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < PICKS; ++i) pt.e[i] = 0.f;
    if (pt.count > 0) {
#pragma unroll
        for (int i = 0; i < PICKS; ++i)
            if (i < per) {                                    // uniform
                const int t = pt.t[i];
                const bool inside = (uint32_t)t < (uint32_t)N;
                const int at = inside ? t : row_cap + lane_id();       // (no pick: -1)
                pt.e[i] = __uint_as_float(atomicExch(reinterpret_cast<uint32_t *>(&lds_row[at]), __float_as_uint(PICKED)));
            }
#pragma unroll
        for (int i = 0; i < PICKS; ++i)
            if (i < per) {
                if (pt.e[i] < 0.f) {                          // no pick, out of range, or picked before
                    pt.e[i] = 0.f;
                    if (i < pt.count) {                       // counted, then taken from the row again
                        bad = true;
                        int t = pt.t[i];
                        if (t < 0 || t >= N) pt.t[i] = -2;
                        t = t < 0 ? 0 : (t >= N ? N - 1 : t);
                        pt.e[i] = exp_shifted_finite(difference(row[t]));
                    } else {
                        pt.t[i] = -1;
                    }
                }
                mass += pt.e[i];
            }
    }
    if (bad) atomicAdd(&status[NGC_STATUS_BAD_SIGMA], 1);
    __syncthreads();                                          // every pick has marked its item
    float unpicked = 0.f;
    each_quad([](int) { return f32x4{}; }, [&](int q, f32x4 &x) {
        const f32x4 v = reinterpret_cast<const f32x4 *>(lds_row)[q];
#pragma unroll
        for (int u = 0; u < 4; ++u) unpicked += max_no_nan(v[u], 0.f);
        if (KEEP_ROW) x = v;
    });
    // one exchange for the scan of the picked masses and the sum of the others
    const float incl = wave_incl_scan_f(mass);
    const float others = wave_sum_f(unpicked);
    if (lane_id() == NGC_WAVE - 1) { fmisc[2 * wave_id()] = incl; fmisc[2 * wave_id() + 1] = others; }
    __syncthreads();
    float all;
    const float base = below_waves<NW, 2>(fmisc, &all);
    pt.unpicked = across_waves<NW, 2>(fmisc + 1, OpAdd{});
    __syncthreads();
    pt.after = base + lane_below_f(incl);                     // sum of the lanes below, no subtraction
    return true;
}

// One workgroup per segment; on the general route an LDS bitmap of picked items (65536 bits).  Scalar registers: beyond 80 a
// SIMD holds seven waves instead of eight, i.e. a CU three workgroups of 512 threads instead of four (896 segments of
// 18000-20000 items, 5999 picks, general route: 95 us, 82 with at most 80).
template <int THREADS, int PICKS, int QUADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_num_sgpr(80))) void subset_logprob_kernel(LogprobArgs a)
{
    // row_cap + SPARE_ITEMS floats or, on the general route, PICKED_WORDS of the bitmap and stage_cap floats
    extern __shared__ __align__(16) float dynamic_lds[];
    __shared__ __align__(16) float fmisc[32];
    uint32_t *picked = reinterpret_cast<uint32_t *>(dynamic_lds);
    float *staged = dynamic_lds + PICKED_WORDS;
    const int tid = threadIdx.x;
    const int seg = blockIdx.x;
    int N = a.n_items[seg];
    if (N < 0) N = 0;
    if (N > 65536) N = 65536;
    int K = a.keep[seg];
    if (K < 0 || K > N) {
        if (tid == 0) atomicAdd(&a.status[NGC_STATUS_KEEP_CLAMPED], 1);
        K = K < 0 ? 0 : N;
    }
    const float *row = a.logits + (size_t)seg * a.logit_stride;
    const int32_t *sig = a.sigma + (size_t)seg * a.sigma_stride;
    if (K == 0) {
        if (tid == 0) a.logp_out[seg] = 0.f;
        return;
    }
    {
        PickedTerms<THREADS, PICKS, QUADS> pt;
        if (gather_picked<THREADS, PICKS, QUADS, false>(row, sig, N, K, a.row_cap, dynamic_lds, fmisc, a.status, pt)) {
            float R = pt.unpicked + pt.after;
            double acc = 0.0;
            if (pt.count > 0) {
                LogRatio ratio;                                // (a masked pick, weight 0, makes log p = -inf)
                static_assert(PICKS <= LogRatio::MAX_PICKS);
#pragma unroll
                for (int i = PICKS - 1; i >= 0; --i)
                    if (i < pt.per) {                          // uniform
                        R += pt.e[i];
                        if (i < pt.count) ratio.times(pt.e[i], R);
                    }
                acc = ratio.log_d();
            }
            // (thousands for a long sequence: rounded once)
            double *totals = reinterpret_cast<double *>(fmisc);
            const double total = wave_sum_d(acc);
            if (lane_id() == 0) totals[wave_id()] = total;
            __syncthreads();
            if (tid < NGC_WAVE) {
                const double lp = wave_sum_d(tid < THREADS / NGC_WAVE ? totals[tid] : 0.0);
                if (tid == 0) a.logp_out[seg] = (float)lp;
            }
            return;
        }
    }
    __syncthreads();
    for (int i = tid; i < PICKED_WORDS; i += THREADS) picked[i] = 0;
    __syncthreads();
    int bad = 0;
    for (int j = tid; j < K; j += THREADS) {
        const int t = sig[j];
        if (t < 0 || t >= N) { bad = 1; continue; }
        const uint32_t bit = 1u << (t & 31);
        if (atomicOr(&picked[t >> 5], bit) & bit) bad = 1;
    }
    if (bad) atomicAdd(&a.status[NGC_STATUS_BAD_SIGMA], 1);
    float smax = -INFINITY, neg_smin = -INFINITY;   // over the unmasked entries
    for (int t = tid; t < N; t += THREADS) {
        float x = row[t];
        if (x == x) smax = fmaxf(smax, x);
        if (x > -INFINITY) neg_smin = fmaxf(neg_smin, -x);
    }
    block_max2_f<THREADS>(smax, neg_smin, fmisc);   // barriers also publish `picked`
    // logits spanning more than NGC_WIDE_SPREAD: wide-range arithmetic (ngc_logsum.h); workgroup-uniform
    const bool wide = smax > -INFINITY && smax + neg_smin > NGC_WIDE_SPREAD;
    if (smax == -INFINITY) smax = 0.f;          // every entry masked: all weights are 0
    float unpicked = 0.f;
    LogSum unpicked_w = ls_empty();
    for (int t = tid; t < N; t += THREADS) {
        if (picked[t >> 5] & (1u << (t & 31))) continue;
        float x = row[t];
        if (x != x) x = -INFINITY;
        if (wide) unpicked_w = ls_add_term(unpicked_w, x);   // that route works on the logits as they came
        else unpicked += expf(x - smax);
    }
    const int chunk = (K + THREADS - 1) / THREADS;
    const int nchunks = (K + chunk - 1) / chunk;
    const int cidx = nchunks - 1 - tid;
    const int j_lo = cidx * chunk;
    const int j_hi = (cidx >= 0) ? ((j_lo + chunk < K) ? j_lo + chunk : K) : 0;
    auto logit_of = [&](int j) {
        int t = sig[j];
        t = t < 0 ? 0 : (t >= N ? N - 1 : t);
        float x = row[t];
        return (x != x) ? -INFINITY : x;
    };
    // When they fit, the picked items' terms are gathered into LDS first (all loads in flight at once), so
    // that the serial chunk loops do not wait for one gather after another.
    const bool use_stage = K <= a.stage_cap;
    const float shift = wide ? 0.f : smax;
    if (use_stage) {
        for (int j = tid; j < K; j += THREADS) staged[j] = logit_of(j) - shift;
        __syncthreads();
    }
    auto term = [&](int j) { return use_stage ? staged[j] : logit_of(j) - shift; };
    if (wide) {
        const LogSum Uw = block_sum_ls<THREADS>(unpicked_w, fmisc);
        const float lpw = sigma_logprob_wide<THREADS>(term, K, Uw, fmisc);
        if (tid == 0) a.logp_out[seg] = lpw;
        return;
    }
    const float U = block_sum_f<THREADS>(unpicked, fmisc);
    float mass = 0.f;
    if (cidx >= 0)
        for (int j = j_lo; j < j_hi; ++j) mass += expf(term(j));
    float total_mass;
    const float after = block_excl_scan_f<THREADS>(mass, fmisc, &total_mass);
    float acc = 0.f;
    if (cidx >= 0) {
        float R = U + after;
        LogRatio ratio;
        int n = 0;
        for (int j = j_hi - 1; j >= j_lo; --j) {
            const float e = expf(term(j));
            R += e;
            ratio.times(e, R);                                   // a masked pick: probability 0
            if (++n == LogRatio::MAX_PICKS) { acc += ratio.log(); ratio = LogRatio{}; n = 0; }
        }
        acc += ratio.log();
    }
    const float lp = block_sum_f<THREADS>(acc, fmisc);
    if (tid == 0) a.logp_out[seg] = lp;
}

// ------------------------------------------ gradient of the log-prob ------
//
// d log p / d s_t = 1[t in sigma] - e_t * C_{r(t)},  C_r = sum_{j <= r} 1 / R_j,
// r(t) = position of t in sigma (K if t was never picked), with e_t and R_j as
// in the forward form.  One reverse scan gives R_j, one forward scan of 1/R_j
// gives C_r; 1/R_j lives in LDS between the two.

struct LogprobBwdArgs {
    const float *logits;
    const int32_t *n_items;
    const int32_t *sigma;
    const int32_t *keep;
    const float *gout;     // upstream weight per segment, or nullptr for 1
    float *grad_out;
    int32_t *status;
    int64_t logit_stride;
    int sigma_stride;
    int keep_cap;
    int row_cap;
};

template <int THREADS, int PICKS, int QUADS>
__global__ __launch_bounds__(THREADS) void subset_logprob_backward_kernel(LogprobBwdArgs a)
{
    // row_cap + SPARE_ITEMS floats or, on the general route, PICKED_WORDS of the bitmap and keep_cap floats
    extern __shared__ __align__(16) float dynamic_lds[];
    __shared__ __align__(16) float fmisc[32];
    uint32_t *picked = reinterpret_cast<uint32_t *>(dynamic_lds);
    float *inv_r = dynamic_lds + PICKED_WORDS;
    const int tid = threadIdx.x;
    const int seg = blockIdx.x;
    int N = a.n_items[seg];
    N = N < 0 ? 0 : (N > 65536 ? 65536 : N);
    int K = a.keep[seg];
    {
        const int lim = N < a.keep_cap ? N : a.keep_cap;
        if (K < 0 || K > lim) {
            if (tid == 0) atomicAdd(&a.status[NGC_STATUS_KEEP_CLAMPED], 1);
            K = K < 0 ? 0 : lim;
        }
    }
    const float *row = a.logits + (size_t)seg * a.logit_stride;
    float *grow = a.grad_out + (size_t)seg * a.logit_stride;
    const int32_t *sig = a.sigma + (size_t)seg * a.sigma_stride;
    const float g = a.gout ? a.gout[seg] : 1.0f;
    if (K == 0) {
        for (int t = tid; t < N; t += THREADS) grow[t] = 0.f;
        return;
    }
    {
        PickedTerms<THREADS, PICKS, QUADS> pt;
        float *lds_row = dynamic_lds;
        if (gather_picked<THREADS, PICKS, QUADS, true>(row, sig, N, K, a.row_cap, lds_row, fmisc, a.status, pt)) {
            // 1 / R_j from the last pick backwards, then C_j = sum_{i <= j} 1 / R_i: the picks before a thread's own
            // are those of the threads ABOVE it
            float inv[PICKS], part = 0.f;
            {
                float R = pt.unpicked + pt.after;
#pragma unroll
                for (int i = PICKS - 1; i >= 0; --i) {
                    inv[i] = 0.f;
                    if (i < pt.per) {                          // uniform
                        R += pt.e[i];
                        if (i < pt.count) inv[i] = reciprocal(R);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < PICKS; ++i) part += inv[i];
            float c_all;
            float C = block_above_scan_f<THREADS>(part, fmisc, &c_all);
            float never = -g * c_all;                          // an item that was never picked: its weight times this
            if (!(scalar(fabsf(never)) < INFINITY)) {
                // The sum of the 1 / R_j reaches e^80, and times a large upstream weight it leaves fp32's range, which the
                // share e * c_all, at most the number of picks, does not: the weights become shares first.  (Always two
                // multiplications: 30 more registers, 3584 segments of 2150-3789 items 27.5 -> 30.9 us.)
                if (pt.held) {
#pragma unroll
                    for (int i = 0; i < QUADS; ++i)
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (4 * (i * THREADS + tid) < N && pt.row[i][u] >= 0.f) pt.row[i][u] *= c_all;
                } else {
                    for (int i = tid; i < N; i += THREADS)
                        if (lds_row[i] >= 0.f) lds_row[i] *= c_all;
                }
                never = -g;
            }
            if (!pt.held) {
                for (int i = tid; i < N; i += THREADS) {
                    const float e = lds_row[i];
                    if (e >= 0.f) lds_row[i] = e * never;
                }
                __syncthreads();
            }
            // the picks' gradients into the LDS row, then the row goes out in order
#pragma unroll
            for (int i = 0; i < PICKS; ++i)
                if (i < pt.per) {
                    C += inv[i];
                    if (pt.t[i] >= 0) lds_row[pt.t[i]] = g * __builtin_fmaf(-pt.e[i], C, 1.0f);
                }
            __syncthreads();
            auto store_quad = [&](int q, f32x4 w) {
                if (4 * q + 4 <= N) {
                    *reinterpret_cast<f32x4_any *>(grow + 4 * q) = w;
                } else {
#pragma unroll
                    for (int u = 0; u < 3; ++u)
                        if (4 * q + u < N) grow[4 * q + u] = w[u];
                }
            };
            if (pt.held) {
#pragma unroll
                for (int i = 0; i < QUADS; ++i) {
                    const int q = i * THREADS + tid;
                    if (4 * q < N) {
                        f32x4 w = reinterpret_cast<const f32x4 *>(lds_row)[q];
#pragma unroll
                        for (int u = 0; u < 4; ++u) w[u] = pt.row[i][u] >= 0.f ? pt.row[i][u] * never : w[u];
                        store_quad(q, w);
                    }
                }
            } else {
                for (int q = tid; 4 * q < N; q += THREADS) store_quad(q, reinterpret_cast<const f32x4 *>(lds_row)[q]);
            }
            return;
        }
    }
    __syncthreads();
    for (int i = tid; i < PICKED_WORDS; i += THREADS) picked[i] = 0;
    __syncthreads();
    int bad = 0;
    for (int j = tid; j < K; j += THREADS) {
        const int t = sig[j];
        if (t < 0 || t >= N) { bad = 1; continue; }
        const uint32_t bit = 1u << (t & 31);
        if (atomicOr(&picked[t >> 5], bit) & bit) bad = 1;
    }
    if (bad) atomicAdd(&a.status[NGC_STATUS_BAD_SIGMA], 1);
    float smax = -INFINITY, neg_smin = -INFINITY;   // over the unmasked entries
    for (int t = tid; t < N; t += THREADS) {
        const float x = row[t];
        if (x == x) smax = fmaxf(smax, x);
        if (x > -INFINITY) neg_smin = fmaxf(neg_smin, -x);
    }
    block_max2_f<THREADS>(smax, neg_smin, fmisc);
    const int chunk = (K + THREADS - 1) / THREADS;
    const int nchunks = (K + chunk - 1) / chunk;
    if (smax > -INFINITY && smax + neg_smin > NGC_WIDE_SPREAD) {
        // Logits spanning more than NGC_WIDE_SPREAD (workgroup-uniform): the same two scans in the wide-range
        // arithmetic of ngc_logsum.h.  LDS holds, per pick, first d_j = s_j - max, then -log R_j, then log C_j;
        // e_t C_r = exp(d_t + log C_r) is a sum of ratios e_t / R_j <= 1 and never leaves fp32's range.
        auto d_of = [&](int t) {
            const float x = row[t];
            return (x != x) ? -INFINITY : x - smax;
        };
        LogSum uw = ls_empty();
        for (int t = tid; t < N; t += THREADS)
            if (!(picked[t >> 5] & (1u << (t & 31)))) uw = ls_add_term(uw, d_of(t));
        const LogSum Uw = block_sum_ls<THREADS>(uw, fmisc);
        for (int j = tid; j < K; j += THREADS) {
            int t = sig[j];
            t = t < 0 ? 0 : (t >= N ? N - 1 : t);
            inv_r[j] = d_of(t);
        }
        __syncthreads();
        {   // reverse pass: thread 0 owns the last chunk; d -> -log R in place
            const int cidx = nchunks - 1 - tid;
            const int j_lo = cidx * chunk;
            const int j_hi = (cidx >= 0) ? ((j_lo + chunk < K) ? j_lo + chunk : K) : 0;
            LogSum mass = ls_empty();
            if (cidx >= 0)
                for (int j = j_lo; j < j_hi; ++j) mass = ls_add_term(mass, inv_r[j]);
            LogSum total;
            const LogSum after = block_excl_scan_ls<THREADS>(mass, fmisc, &total);
            if (cidx >= 0) {
                LogSum R = ls_add(Uw, after);
                for (int j = j_hi - 1; j >= j_lo; --j) {
                    R = ls_add_term(R, inv_r[j]);
                    inv_r[j] = -ls_log(R);
                }
            }
        }
        __syncthreads();
        LogSum c_all;
        {   // forward pass: thread i owns chunk i; -log R -> log C in place
            const int j_lo = tid * chunk;
            const int j_hi = (tid < nchunks) ? ((j_lo + chunk < K) ? j_lo + chunk : K) : j_lo;
            LogSum part = ls_empty();
            for (int j = j_lo; j < j_hi; ++j) part = ls_add_term(part, inv_r[j]);
            LogSum C = block_excl_scan_ls<THREADS>(part, fmisc, &c_all);
            for (int j = j_lo; j < j_hi; ++j) {
                C = ls_add_term(C, inv_r[j]);
                inv_r[j] = ls_log(C);
            }
        }
        __syncthreads();
        const float log_c_all = ls_log(c_all);
        for (int j = tid; j < K; j += THREADS) {
            const int t = sig[j];
            if (t >= 0 && t < N) grow[t] = g * (1.0f - expf(d_of(t) + inv_r[j]));
        }
        for (int t = tid; t < N; t += THREADS)
            if (!(picked[t >> 5] & (1u << (t & 31)))) grow[t] = -g * expf(d_of(t) + log_c_all);
        return;
    }
    float unpicked = 0.f;
    for (int t = tid; t < N; t += THREADS) {
        if (picked[t >> 5] & (1u << (t & 31))) continue;
        float x = row[t];
        if (x != x) x = -INFINITY;
        unpicked += expf(x - smax);
    }
    const float U = block_sum_f<THREADS>(unpicked, fmisc);
    auto mass_of = [&](int j) {
        int t = sig[j];
        t = t < 0 ? 0 : (t >= N ? N - 1 : t);
        const float x = row[t];
        return (x != x) ? 0.f : expf(x - smax);
    };
    // The masses of the picked items are gathered into LDS first, all loads in flight at once; the two
    // scans then run on LDS and never wait for a gather inside their serial chunk loops.
    for (int j = tid; j < K; j += THREADS) inv_r[j] = mass_of(j);
    __syncthreads();
    // reverse pass: thread 0 owns the last chunk; mass -> 1 / R in place
    {
        const int cidx = nchunks - 1 - tid;
        const int j_lo = cidx * chunk;
        const int j_hi = (cidx >= 0) ? ((j_lo + chunk < K) ? j_lo + chunk : K) : 0;
        float mass = 0.f;
        if (cidx >= 0)
            for (int j = j_lo; j < j_hi; ++j) mass += inv_r[j];
        float total;
        const float after = block_excl_scan_f<THREADS>(mass, fmisc, &total);
        if (cidx >= 0) {
            float R = U + after;
            for (int j = j_hi - 1; j >= j_lo; --j) {
                R += inv_r[j];
                inv_r[j] = 1.0f / R;
            }
        }
    }
    __syncthreads();
    // forward pass: thread i owns chunk i; 1 / R -> C in place
    float c_all;
    {
        const int j_lo = tid * chunk;
        const int j_hi = (tid < nchunks) ? ((j_lo + chunk < K) ? j_lo + chunk : K) : j_lo;
        float part = 0.f;
        for (int j = j_lo; j < j_hi; ++j) part += inv_r[j];
        const float before = block_excl_scan_f<THREADS>(part, fmisc, &c_all);
        float C = before;
        for (int j = j_lo; j < j_hi; ++j) {
            C += inv_r[j];
            inv_r[j] = C;
        }
    }
    __syncthreads();
    for (int j = tid; j < K; j += THREADS) {
        const int t = sig[j];
        if (t >= 0 && t < N) grow[t] = g * (1.0f - mass_of(j) * inv_r[j]);
    }
    for (int t = tid; t < N; t += THREADS) {
        if (picked[t >> 5] & (1u << (t & 31))) continue;
        float x = row[t];
        const float e = (x != x) ? 0.f : expf(x - smax);
        grow[t] = -g * e * c_all;
    }
}

// ------------------------------------------- eviction loss (Eq. 4) --------
//
// L^l = -(1/P) sum_prompts (1/G) sum_{i in prompt} A_i (1/n_i) sum_{t < n_i} sum_h logp[t][l][i][h],
// A_i = r_i - mean of r over the G rollouts of the prompt, n_i = rounds that fired for rollout i.
// One workgroup per layer; advantages and 1/n_i in LDS; fp64 accumulation in a fixed order (the
// advantages of a prompt sum to zero, so the terms cancel heavily).  Also writes d loss / d logp,
// the upstream weights of subset_logprob_backward_kernel.

struct LmemArgs {
    const float *logp;     // [R][L][B][H]
    const int32_t *rounds; // [B]
    const float *reward;   // [B]
    float *adv_out;        // [B] or nullptr
    float *loss_layer;     // [L]
    float *gout;           // [R][L][B][H] or nullptr
    int R, L, B, H, group;
};

constexpr int LMEM_THREADS = 256;
constexpr int LMEM_MAX_B = 8192;

__global__ __launch_bounds__(LMEM_THREADS) void lmem_layer_kernel(LmemArgs a)
{
    __shared__ float weight[LMEM_MAX_B];      // A_i / n_i (0 when no round fired)
    __shared__ int nrounds[LMEM_MAX_B];
    __shared__ double red[LMEM_THREADS];
    const int l = blockIdx.x, tid = threadIdx.x;
    for (int i = tid; i < a.B; i += LMEM_THREADS) {
        const int g0 = (i / a.group) * a.group;
        double mean = 0.0;
        for (int j = 0; j < a.group; ++j) mean += (double)a.reward[g0 + j];
        mean /= (double)a.group;
        const double adv = (double)a.reward[i] - mean;
        int n = a.rounds[i];
        n = n < 0 ? 0 : (n > a.R ? a.R : n);
        nrounds[i] = n;
        weight[i] = n > 0 ? (float)(adv / (double)n) : 0.f;
        if (l == 0 && a.adv_out) a.adv_out[i] = (float)adv;
    }
    __syncthreads();
    const int BH = a.B * a.H;
    double acc = 0.0;
    for (int t = 0; t < a.R; ++t) {
        const size_t base = ((size_t)t * a.L + l) * BH;
        for (int e = tid; e < BH; e += LMEM_THREADS) {
            const int i = e / a.H;
            const bool live = t < nrounds[i];
            if (live) acc += (double)a.logp[base + e] * (double)weight[i];
            if (a.gout) a.gout[base + e] = live ? -weight[i] / (float)a.B : 0.f;
        }
    }
    red[tid] = acc;
    __syncthreads();
    for (int s = LMEM_THREADS / 2; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) a.loss_layer[l] = (float)(-red[0] / (double)a.B);
}

// Advantages, layers, total and upstream weights in one launch by one workgroup, where there is little to add up or few
// layers to spread it over (lmem_in_one(): call after call 2 rounds x 7 layers x 128 rollouts x 4 heads 6.9 -> 5.9 us;
// 3 x 28 x 16 x 2 7.3 -> 5.8; 1 x 1 x 1024 x 32 38 -> 14).  A wave adds one layer's terms or, with fewer layers than waves,
// an equal share of them; with more, it takes one after another.
constexpr int LMEM_ONE_THREADS = 1024;
constexpr int LMEM_ONE_WAVES = LMEM_ONE_THREADS / NGC_WAVE;
constexpr int LMEM_ONE_MAX_B = 1024;
constexpr int LMEM_ONE_MAX_L = 128;
constexpr int LMEM_ONE_MAX_TERMS = 32768;

// x / d by a multiplication, exact for x and d up to 2^16: m = floor(2^32 / d) + 1 (0 stands for d = 1) is off by at most d,
// x m / 2^32 by less than 1 / d.  (One CU does all the work: with three integer divisions and one of floats per term the
// kernel took 8.5 us.)
inline uint32_t divide_by(uint32_t d) { return d > 1 ? (uint32_t)((1ull << 32) / d + 1) : 0; }
__device__ __forceinline__ int divided(int x, uint32_t m) { return m ? (int)__umulhi((uint32_t)x, m) : x; }

__global__ __launch_bounds__(LMEM_ONE_THREADS) void lmem_one_kernel(LmemArgs a, uint32_t by_h, uint32_t by_bh, float *loss)
{
    __shared__ float reward[LMEM_ONE_MAX_B], weight[LMEM_ONE_MAX_B], upstream[LMEM_ONE_MAX_B];
    __shared__ int nrounds[LMEM_ONE_MAX_B];
    __shared__ double share[LMEM_ONE_MAX_L > LMEM_ONE_WAVES ? LMEM_ONE_MAX_L : LMEM_ONE_WAVES];
    __shared__ float of_layer[LMEM_ONE_MAX_L];
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    // Terms x = 0 .. terms - 1 of a layer: (round x / BH, rollout and head x % BH).  Share `part` of a layer has those with
    // x / 64 % parts = part; lane k of a wave x = 64 (part + i parts) + k, BATCH values of i at a time.  The first
    // batch is asked for before the weights are known.
    constexpr int BATCH = 8;
    const int BH = a.B * a.H, terms = a.R * BH;
    const int parts = a.L < LMEM_ONE_WAVES ? LMEM_ONE_WAVES / a.L : 1;
    float lp[BATCH];
    auto load_batch = [&](int l, int x0) {
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            int x = x0 + i * parts * NGC_WAVE;
            x = x < terms ? x : terms - 1;
            const int t = divided(x, by_bh);
            lp[i] = a.logp[((size_t)t * a.L + l) * BH + (x - t * BH)];
        }
    };
    if (wv < a.L * parts) load_batch(wv / parts, (wv % parts) * NGC_WAVE + lane);
    int n = 0;
    if (tid < a.B) {
        reward[tid] = a.reward[tid];
        n = a.rounds[tid];
    }
    __syncthreads();
    if (tid < a.B) {
        const int g0 = (tid / a.group) * a.group;
        double mean = 0.0;
        for (int j = 0; j < a.group; ++j) mean += (double)reward[g0 + j];
        mean /= (double)a.group;
        const double adv = (double)reward[tid] - mean;
        n = n < 0 ? 0 : (n > a.R ? a.R : n);
        nrounds[tid] = n;
        weight[tid] = n > 0 ? (float)(adv / (double)n) : 0.f;
        upstream[tid] = -weight[tid] / (float)a.B;
        if (a.adv_out) a.adv_out[tid] = (float)adv;
    }
    __syncthreads();
    for (int idx = wv; idx < a.L * parts; idx += LMEM_ONE_WAVES) {
        const int l = idx / parts, part = idx - l * parts;
        double acc = 0.0;
        for (int x0 = part * NGC_WAVE + lane; x0 < terms; x0 += BATCH * parts * NGC_WAVE) {
            if (idx != wv || x0 >= BATCH * parts * NGC_WAVE) load_batch(l, x0);
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                const int x = x0 + i * parts * NGC_WAVE;
                if (x >= terms) break;
                const int t = divided(x, by_bh), e = x - t * BH, b = divided(e, by_h);
                const bool live = t < nrounds[b];
                if (live) acc += (double)lp[i] * (double)weight[b];
                if (a.gout) a.gout[((size_t)t * a.L + l) * BH + e] = live ? upstream[b] : 0.f;
            }
        }
        acc = wave_sum_d(acc);
        if (lane == 0) share[idx] = acc;
    }
    __syncthreads();
    if (tid < a.L) {
        double acc = 0.0;
        for (int i = 0; i < parts; ++i) acc += share[tid * parts + i];
        of_layer[tid] = (float)(-acc / (double)a.B);
        a.loss_layer[tid] = of_layer[tid];
    }
    __syncthreads();
    if (tid == 0) {
        double s = 0.0;
        for (int l = 0; l < a.L; ++l) s += (double)of_layer[l];
        *loss = (float)s;
    }
}

// One wave: 64 layers' losses per load, added in layer order.
__global__ __launch_bounds__(64) void lmem_total_kernel(const float *loss_layer, int L, float *loss)
{
    double s = 0.0;
    for (int l0 = 0; l0 < L; l0 += 64) {
        const int l = l0 + (int)threadIdx.x;
        const float x = l < L ? loss_layer[l] : 0.f;
        const int m = L - l0 < 64 ? L - l0 : 64;
        for (int i = 0; i < m; ++i) s += (double)__shfl(x, i, 64);
    }
    if (threadIdx.x == 0) *loss = (float)s;
}

// --------------------------------------------------------- compaction -----
//
// In place: the row that ends at slot j comes from a slot >= j, and once one
// kept row has moved every later one moves too (the kept list is ascending).
// A workgroup walks the rows from the first one that moves (row_start) to the
// end in tiles of TILE_ROWS destination rows: all of a tile's reads, a barrier, all of
// its writes, a barrier.  The first barrier is what correctness asks for (a row of the
// tile can be the source of another row of the same tile; the sources of tile
// i+1 lie at or beyond its first row, so earlier tiles' writes never touch them).  The second one is
// what the memory asks for: a CU that reads and writes in turns, in bursts of a whole
// tile, moves more than one whose waves mix both.  2048 segments of 4096-8192 rows, us per round: loads of tile i+1
// and stores of tile i in flight together (two register buffers) 956; stores held back until those loads have arrived 951, and
// with a barrier after that 934; this loop 923, without its second barrier 970.  It holds half the registers, so the
// 512-thread workgroups take 8 rows a thread (896 segments of 700 rows 77.4 us with 2, 74.4 with 8).  The row indices come
// from LDS (pooled rounds: from kept_out).  16-byte accesses, one full
// row per ROW_BYTES/16 consecutive lanes, K and V together; all of them carry
// the nontemporal hint (every row is touched once).  Offsets inside a segment
// are 32-bit (the host checks cap * ROW_BYTES < 2^31).
//
// POWER_OF_TWO: `block` is one, and the item of a row a shift instead of a division (20 instructions a row).
template <int ROW_BYTES, int THREADS, int UNROLL, bool POWER_OF_TWO, class Index>
__device__ __forceinline__ void compact_kv_inplace(unsigned char *kbase, unsigned char *vbase,
                                                   const Index *kept, int rows_new, int row_start, int block)
{
    constexpr int PIECES = ROW_BYTES / 16;           // 16-byte pieces per row
    constexpr int ROWS_PER_STEP = THREADS / PIECES;  // rows covered by one load per thread
    constexpr int TILE_ROWS = ROWS_PER_STEP * UNROLL;
    const int rsub = threadIdx.x / PIECES;
    const uint32_t col = (uint32_t)(threadIdx.x % PIECES) * 16u;
    const int last = rows_new - 1;
    if (row_start >= rows_new) return;   // workgroup-uniform
    const int shift = __builtin_ctz(block);

    // source rows of this thread's rows of a tile; rows past the end take the last row's source
    auto sources = [&](int tile, int (&src)[UNROLL]) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            int r = tile + u * ROWS_PER_STEP + rsub;
            r = r < last ? r : last;
            if constexpr (POWER_OF_TWO) {
                src[u] = ((int)kept[r >> shift] << shift) + (r & (block - 1));
            } else {
                const int item = r / block;
                src[u] = (int)kept[item] * block + (r - item * block);
            }
        }
    };
    auto load = [&](const int (&src)[UNROLL], u32x4 (&kb)[UNROLL], u32x4 (&vb)[UNROLL]) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t off = (uint32_t)src[u] * ROW_BYTES + col;
            kb[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(kbase + off));
            vb[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(vbase + off));
        }
    };
    auto store_full = [&](int tile, const u32x4 (&kb)[UNROLL], const u32x4 (&vb)[UNROLL]) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const uint32_t off = (uint32_t)(tile + u * ROWS_PER_STEP + rsub) * ROW_BYTES + col;
            __builtin_nontemporal_store(kb[u], reinterpret_cast<u32x4 *>(kbase + off));
            __builtin_nontemporal_store(vb[u], reinterpret_cast<u32x4 *>(vbase + off));
        }
    };
    auto store_tail = [&](int tile, const u32x4 (&kb)[UNROLL], const u32x4 (&vb)[UNROLL]) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int r = tile + u * ROWS_PER_STEP + rsub;
            if (r < rows_new) {
                const uint32_t off = (uint32_t)r * ROW_BYTES + col;
                __builtin_nontemporal_store(kb[u], reinterpret_cast<u32x4 *>(kbase + off));
                __builtin_nontemporal_store(vb[u], reinterpret_cast<u32x4 *>(vbase + off));
            }
        }
    };

    int src[UNROLL];
    u32x4 kb[UNROLL], vb[UNROLL];
    sources(row_start, src);
    for (int tile = row_start; ; tile += TILE_ROWS) {
        load(src, kb, vb);
        sources(tile + TILE_ROWS, src);
        __builtin_amdgcn_sched_barrier(0);
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                       // the whole tile has arrived, in every wave
        if (tile + TILE_ROWS >= rows_new) {
            store_tail(tile, kb, vb);
            break;
        }
        store_full(tile, kb, vb);
        __syncthreads();                       // all of it is on its way before the next tile is asked for
    }
}

__device__ __forceinline__ int source_row(const int32_t *kept, int r, int block)
{
    if (block == 1) return kept[r];
    const int item = r / block;
    return kept[item] * block + (r - item * block);
}

template <int THREADS>
__device__ __forceinline__ void compact_pos_inplace(int32_t *pos, const int32_t *kept, int rows_new,
                                                    int row_start, int block)
{
    constexpr int TILE = 4 * THREADS;
    for (int tile = (row_start / TILE) * TILE; tile < rows_new; tile += TILE) {
        int32_t val[4];
        bool moves[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = tile + u * THREADS + threadIdx.x;
            const int s = (r < rows_new) ? source_row(kept, r, block) : r;
            moves[u] = (s != r);
            val[u] = 0;
            if (moves[u]) val[u] = pos[s];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (moves[u]) pos[tile + u * THREADS + threadIdx.x] = val[u];
    }
}

// ------------------------------------------------- pooled-heads mode ------
//
// One selection problem per (layer, sequence): the items of all its KV heads
// compete for one budget, so heads whose logits are larger keep more rows.
// Item order (for ties and for the sampled sequence) is (head, row); the noise
// of item (head, row) is the one the per-head mode draws for it.
//
// What bounds it: one workgroup selects for all heads of a sequence, a chain of waits as long as its items are many, and
// the chip has as many workgroups to hide it as there are (layer, sequence) pairs.  Where LDS has room for a code and a
// bucket entry per item (16032 where all may be kept, 19200 where 6000), they are ranked by value buckets as in the per-head
// mode, every head's items filled up to a multiple of four so that a thread's four codes stay one access.  Beyond, and where
// ranking does not apply (masked items kept, many equal keys, a wide spread, no sequence wanted), pooled_general() selects by
// radix, from the codes in LDS if they are there; otherwise up to Hkv * cap = 65536 items, their codes in a workspace in
// global memory.
// The rows are moved by the same workgroup or, for few sequences, by a launch of one workgroup per head (see ngc_evict).
// Rounds of half the rows, us, before (radix always, one launch) and now:
//     sequences x heads x rows   16 x 2 x 500     16 x 8 x 300     16 x 8 x 2000   64 x 4 x 1500   128 x 2 x 4000
//                                25.9   18.1      53.7   24.7     217.5  100.0    103.3   67.5    144.8  134.1
//                              256 x 2 x 4000  448 x 4 x 500    896 x 4 x 1500   896 x 8 x 300
//                               240.3  225.6    128.7  107.0     618.0  564.1    335.9  250.4
// Selections that are not ranked, us, before ranking was tried, with keys made again after it, and from the codes in LDS
// (logits in steps of 1/8 at tau = 0; all equal; two thirds masked, some of them kept; a spread of 400):
//     sequences x heads x rows   quantised            equal                masked               spread
//               16 x 8 x  300     39.7  43.9  38.4    26.0  29.1  23.8    45.0  51.0  38.7     43.1  48.2  36.6
//               16 x 8 x 2000    125   137   127      90.0  97.5  82.8   137   159   138      104   124   103
//              128 x 2 x 4000     65.5  72.8  67.2    45.8  50.0  41.7    69.8  82.0  71.5     54.8  65.2  54.4
//              896 x 8 x  300    161   117   100     101    82.8  67.6   180   140   102      174   122    85.7

constexpr int POOL_MAX_HEADS = 16;
constexpr int POOL_FEW = 128;            // (layer, sequence) pairs up to which the rows take a second launch
constexpr int POOL_MANY = 256;           // beyond, with few items each, 512 threads
constexpr int POOL_SMALL_ITEMS = 2560;
// misc slots of the pooled kernel
constexpr int PM_N = 40;      // rows per head        [40, 56)
constexpr int PM_OFF = 56;    // item offset per head [56, 73)
constexpr int PM_BASE = 73;   // kept slots before each head [73, 90)
constexpr int PM_QUAD = 90;   // groups of four items before each head, every head's last one filled up [90, 107)
constexpr int PM_WORDS = 128;
constexpr int PM_MAXIMA = 64; // behind misc, where items are ranked: four words a wave

// What the attempt at ranking has made: the codes in LDS (null: nothing yet), groups of four over all heads, 0 where a head's
// last one is filled up; the largest code and logit (0: all masked), and whether the logits span more than NGC_WIDE_SPREAD.
struct PooledKeys {
    const uint32_t *code;
    uint32_t cmax;
    float smax;
    bool wide;
};

// Selection by radix.  The codes of all items are read in order by the select passes, from LDS if they have been made there
// (an item's index then counts the filled-up places too); the kept items' codes, logits and
// item indices stand in three dense arrays next to those in memory (K entries each, served by the L2 cache to the sort and to
// the log-probability), the index buffers of the sort in LDS.  Writes the kept lists, sigma and its log-probability, and
// leaves the kept slots before each head in misc.
template <int THREADS, bool RANK>
__device__ void pooled_general(const SelectArgs &a, int seg_first, int l, int b, int N, int K, const PooledKeys &keys,
                               uint32_t *hist, int *misc, uint16_t *idxA, uint16_t *idxB)
{
    constexpr int NW = THREADS / NGC_WAVE;
    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int Hkv = a.g.Hkv, cap = a.g.cap, lb = seg_first / Hkv;
    float *fmisc = reinterpret_cast<float *>(misc);
    // per (layer, sequence): [codes of all items][codes | logits | item indices of the kept items]
    uint32_t *code = a.pool_codes + (size_t)lb * Hkv * cap * 4;
    uint32_t *kcode = code + (size_t)Hkv * cap;
    float *klogit = reinterpret_cast<float *>(kcode + (size_t)Hkv * cap);
    uint16_t *items = reinterpret_cast<uint16_t *>(klogit + (size_t)Hkv * cap);
    const bool want_logp = a.logp_out != nullptr;
    const bool want_sort = want_logp || a.sigma_out != nullptr;
    auto head_of = [&](int i) {
        int h = 0;
        while (h + 1 < Hkv && i >= misc[PM_OFF + h + 1]) ++h;
        return h;
    };

    // ---- 1. keys (and the first histogram of the radix select) -------------
    const bool in_lds = RANK && keys.code != nullptr;
    if (in_lds) {
        N = 4 * misc[PM_QUAD + Hkv];
        if (tid <= Hkv) misc[PM_OFF + tid] = 4 * misc[PM_QUAD + tid];
    }
    for (int i = tid; i < SEL_BINS; i += THREADS) hist[i] = 0;
    __syncthreads();
    float smax = keys.smax;
    uint32_t cmax = keys.cmax;
    bool wide = keys.wide;   // logits spanning more than NGC_WIDE_SPREAD: wide-range arithmetic for Eq. 2
    if (in_lds) {
        for (int q = tid; 4 * q < N; q += THREADS) {
            const u32x4 c = reinterpret_cast<const u32x4 *>(keys.code)[q];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c[i] != 0u) {
                    // what comes here has many equal codes, masked ones or others: the bin of the first lane's is added to at
                    // once (8 heads of 2000 equal keys 93.7 -> 82.3 us)
                    const uint32_t bin = c[i] >> 21;
                    const uint64_t same = __ballot(bin == (uint32_t)__builtin_amdgcn_readfirstlane((int)bin));
                    const bool in = (same >> lane) & 1u;
                    if (!in || popc_below(same) == 0) atomicAdd(&hist[bin], in ? (uint32_t)__popcll(same) : 1u);
                }
        }
    } else {
        float neg_smin = -INFINITY;   // over the unmasked entries, as smax
        for (int h = 0; h < Hkv; ++h) {
            const int n = misc[PM_N + h], off = misc[PM_OFF + h];
            const float *row = a.logits + (size_t)(seg_first + h) * cap;
            for (int quad = tid; 4 * quad < n; quad += THREADS) {
                float s[4], key[4];
                keys_of_quad(row, n, quad, a.na, l, b, h, s, key);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (4 * quad + i < n) {
                        const uint32_t c = ordered_code(key[i]);
                        code[off + 4 * quad + i] = c;
                        atomicAdd(&hist[c >> 21], 1u);
                        cmax = c > cmax ? c : cmax;
                        smax = fmaxf(smax, s[i]);
                        if (s[i] > -INFINITY) neg_smin = fmaxf(neg_smin, -s[i]);
                    }
            }
        }
        if (want_logp) {
            block_max2_f<THREADS>(smax, neg_smin, fmisc);
            wide = smax > -INFINITY && smax + neg_smin > NGC_WIDE_SPREAD;
            if (smax == -INFINITY) smax = 0.f;
        }
        if (want_sort) cmax = block_max_u<THREADS>(cmax, reinterpret_cast<uint32_t *>(misc));
    }
    auto code_at = [&](int t) { return in_lds ? keys.code[t] : code[t]; };

    // ---- 2. radix select (the first histogram was accumulated with the keys) --
    int need;
    __syncthreads();   // publishes the codes and the histogram of step 1
    const uint32_t thr = radix_select_kth<THREADS>(code_at, N, K, hist, misc, need, true);

    // ---- 3. kept items, ascending in (head, row) order ----------------------
    // Slot j of the kept list gets its item index (items[j]) and its code (kcode[j]) in two dense arrays next to
    // the codes, so that everything after this step works on K entries read in order or from the L2 cache
    // instead of gathering from the N codes.
    const int per_wave = (((N + NW - 1) / NW) + NGC_WAVE - 1) & ~(NGC_WAVE - 1);
    const int w_begin = wv * per_wave;
    const int w_end = (w_begin + per_wave < N) ? (w_begin + per_wave) : N;
    {
        int gt = 0, eq = 0;
        for (int t0 = w_begin; t0 < w_end; t0 += NGC_WAVE) {
            const int t = t0 + lane;
            const uint32_t u = (t < w_end) ? code_at(t) : 0u;
            gt += __popcll(__ballot(u > thr));             // (a kept item's code is never 0)
            eq += __popcll(__ballot(u == thr));
        }
        if (lane == 0) { misc[wv] = gt; misc[16 + wv] = eq; }
    }
    __syncthreads();
    int gt_base = 0, eq_base = 0;
    for (int w = 0; w < wv; ++w) { gt_base += misc[w]; eq_base += misc[16 + w]; }
    float unpicked = 0.f;
    LogSum unpicked_w = ls_empty();
    for (int t0 = w_begin; t0 < w_end; t0 += NGC_WAVE) {
        const int t = t0 + lane;
        const uint32_t u = t < w_end ? code_at(t) : 0u;
        const bool in = u != 0u;
        const bool is_gt = u > thr, is_eq = u == thr;
        const uint64_t bgt = __ballot(is_gt), beq = __ballot(is_eq);
        const int gt_before = gt_base + popc_below(bgt);
        const int eq_before = eq_base + popc_below(beq);
        const bool sel = is_gt || (is_eq && eq_before < need);
        if (in && (want_logp || sel)) {
            float x = 0.f;
            if (want_logp) {
                const int h = head_of(t);
                x = a.logits[(size_t)(seg_first + h) * cap + (t - misc[PM_OFF + h])];
                if (x != x) x = -INFINITY;
            }
            if (sel) {
                const int slot = gt_before + (eq_before < need ? eq_before : need);
                items[slot] = (uint16_t)t;
                kcode[slot] = u;
                klogit[slot] = x;
                idxA[slot] = (uint16_t)slot;
            } else if (wide) {
                unpicked_w = ls_add_term(unpicked_w, x);
            } else {
                unpicked += expf(x - smax);
            }
        }
        gt_base += __popcll(bgt);
        eq_base += __popcll(beq);
    }
    __syncthreads();   // items, kcode (global, this workgroup's own) and idxA are complete
    // kept slots before each head: first slot whose item lies at or beyond the head's offset
    if (tid <= Hkv) {
        const int target = misc[PM_OFF + tid];
        int lo = 0, hi = K;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((int)items[mid] < target) lo = mid + 1; else hi = mid;
        }
        misc[PM_BASE + tid] = lo;
    }
    __syncthreads();
    auto head_of_slot = [&](int j) {
        int h = 0;
        while (h + 1 < Hkv && j >= misc[PM_BASE + h + 1]) ++h;
        return h;
    };
    for (int j = tid; j < K; j += THREADS) {
        const int h = head_of_slot(j);
        const int slot = j - misc[PM_BASE + h];
        if (slot < a.max_keep) a.kept_out[(size_t)(seg_first + h) * a.max_keep + slot] = (int)items[j] - misc[PM_OFF + h];
    }

    if (want_sort) {
        // ---- 4. sigma: the slots sorted by descending code ---------------------
        const uint16_t *src = sort_by_code_desc<THREADS>([&](uint16_t j) { return kcode[j]; }, K, cmax, thr, idxA, idxB,
                                                         hist, misc);
        auto logit_of_slot = [&](int j) { return klogit[j]; };
        if (a.sigma_out) {
            // the pooled sequence occupies the Hkv rows of this (layer, sequence) back to back
            int32_t *sig_row = a.sigma_out + (size_t)seg_first * a.max_keep;
            const int room = Hkv * a.max_keep;
            for (int j = tid; j < K && j < room; j += THREADS) {
                const int slot = src[j], h = head_of_slot(slot);
                sig_row[j] = h * cap + ((int)items[slot] - misc[PM_OFF + h]);
            }
        }
        if (want_logp) {
            // ---- 5. log-probability of the pooled sequence -------------------
            if (wide) {
                const LogSum Uw = block_sum_ls<THREADS>(unpicked_w, fmisc);
                const float lpw = sigma_logprob_wide<THREADS>([&](int j) { return logit_of_slot(src[j]); }, K, Uw,
                                                              fmisc);
                if (tid < Hkv) a.logp_out[seg_first + tid] = (tid == 0) ? lpw : 0.f;
            } else {
                const float U = block_sum_f<THREADS>(unpicked, fmisc);
                const int chunk = (K + THREADS - 1) / THREADS;
                const int nchunks = (K + chunk - 1) / chunk;
                const int cidx = nchunks - 1 - tid;
                const int j_lo = cidx * chunk;
                const int j_hi = (cidx >= 0) ? ((j_lo + chunk < K) ? j_lo + chunk : K) : 0;
                float mass = 0.f;
                if (cidx >= 0)
                    for (int j = j_lo; j < j_hi; ++j) mass += expf(logit_of_slot(src[j]) - smax);
                float total_mass;
                const float after = block_excl_scan_f<THREADS>(mass, fmisc, &total_mass);
                float acc = 0.f;
                if (cidx >= 0) {
                    float R = U + after;
                    for (int j = j_hi - 1; j >= j_lo; --j) {
                        const float d = logit_of_slot(src[j]) - smax;
                        R += expf(d);
                        acc += (d == -INFINITY) ? -INFINITY : d - logf(R);
                    }
                }
                const float lp = block_sum_f<THREADS>(acc, fmisc);
                if (tid < Hkv) a.logp_out[seg_first + tid] = (tid == 0) ? lp : 0.f;
            }
        }
    }
}

// RANK: LDS has been given for ranking (a.rank_cap).  Where it has not, a kernel without that code: 896 x 2 x 300 rows without
// sampled orders 34.8 -> 38.0 us with it, 16 x 2 x 500 10.5 -> 11.0.
template <int THREADS, int ROW_BYTES, int UNROLL, bool RANK>
__global__ __launch_bounds__(THREADS) void evict_pooled_kernel(SelectArgs a)
{
    constexpr int NW = THREADS / NGC_WAVE;
    constexpr int HIST = (SEL_BINS > SORT_BINS * NW) ? SEL_BINS : SORT_BINS * NW;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    uint32_t *hist = reinterpret_cast<uint32_t *>(smem_raw);
    int *misc = reinterpret_cast<int *>(hist + HIST);
    u32x4 *maxima = reinterpret_cast<u32x4 *>(misc + PM_WORDS);
    // ranking: rank_cap codes, then as many bits
    const int rank_cap = RANK ? a.rank_cap : 0;
    uint32_t *rank_code = reinterpret_cast<uint32_t *>(misc + PM_WORDS + (RANK ? PM_MAXIMA : 0));
    uint32_t *kept_bits = rank_code + rank_cap;
    uint16_t *idxA = reinterpret_cast<uint16_t *>(kept_bits + (rank_cap + 63) / 64 * 2);
    uint16_t *idxB = idxA + a.keep_cap;                                      // max(keep_cap, rank_cap) entries
    float *fmisc = reinterpret_cast<float *>(misc);

    const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
    const int Hkv = a.g.Hkv, cap = a.g.cap;
    const int lb = a.seg0 / Hkv + blockIdx.x;     // layer * B + sequence
    const int l = lb / a.g.B, b = lb - l * a.g.B;
    const int seg_first = lb * Hkv;

    // ---- 0. geometry of the pooled item space ------------------------------
    if (tid == 0) {
        int off = 0, ktot = 0, quads = 0;
        for (int h = 0; h < Hkv; ++h) {
            int n = a.len[seg_first + h];
            if (n < 0 || n > cap) {
                atomicAdd(&a.status[NGC_STATUS_LEN_CLAMPED], 1);
                n = n < 0 ? 0 : cap;
            }
            int kh = a.keep[seg_first + h];
            if (kh < 0) { atomicAdd(&a.status[NGC_STATUS_KEEP_CLAMPED], 1); kh = 0; }
            misc[PM_N + h] = n;
            misc[PM_OFF + h] = off;
            misc[PM_QUAD + h] = quads;
            off += n;
            quads += (n + 3) / 4;
            ktot += kh;
        }
        misc[PM_OFF + Hkv] = off;
        misc[PM_QUAD + Hkv] = quads;
        int lim = off < a.keep_cap ? off : a.keep_cap;
        if (ktot > lim) {
            atomicAdd(&a.status[NGC_STATUS_KEEP_CLAMPED], 1);
            ktot = lim;
        }
        misc[MISC_KEPT] = ktot;
    }
    __syncthreads();
    const int N = misc[PM_OFF + Hkv];
    const int K = misc[MISC_KEPT];
    const bool want_logp = a.logp_out != nullptr;
    const bool want_sort = want_logp || a.sigma_out != nullptr;
    if (K == 0) {
        if (tid < Hkv) {
            if (a.len_out) a.len_out[seg_first + tid] = 0;
            if (want_logp) a.logp_out[seg_first + tid] = 0.f;
        }
        return;
    }

    // ---- 1. ranking, where LDS holds a code and a bucket entry for every item (groups of four are dealt to the threads
    // over all heads: a head of few rows leaves none idle) ----
    const int quads = misc[PM_QUAD + Hkv];
    auto head_of_quad = [&](int q) {
        int h = 0;
        while (h + 1 < Hkv && q >= misc[PM_QUAD + h + 1]) ++h;
        return h;
    };
    bool ranked = false;
    float unpicked = 0.f, smax = -INFINITY;
    PooledKeys keys{nullptr, 0u, -INFINITY, false};
    if (RANK && want_sort && 4 * quads <= rank_cap) {
        for (int i = tid; i < HIST / 4; i += THREADS) reinterpret_cast<u32x4 *>(hist)[i] = u32x4{0u, 0u, 0u, 0u};
        for (int i = tid; i < (4 * quads + 63) / 64 * 2; i += THREADS) kept_bits[i] = 0;
        float neg_smin = -INFINITY;
        uint32_t cmax = 0, neg_cmin = 0;
        int unmasked = 0;
        constexpr int HELD = 2;      // groups of four logits a thread keeps until the kept items are known
        f32x4 held[HELD] = {};
        int group = 0;
#pragma unroll 1
        for (int q = tid; q < quads; q += THREADS, ++group) {
            const int h = head_of_quad(q), quad = q - misc[PM_QUAD + h], n = misc[PM_N + h];
            float x[4], key[4];
            keys_of_quad(a.logits + (size_t)(seg_first + h) * cap, n, quad, a.na, l, b, h, x, key);
            if (group == 0) held[0] = f32x4{x[0], x[1], x[2], x[3]};
            if (group == 1) held[1] = f32x4{x[0], x[1], x[2], x[3]};
            u32x4 c;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                c[i] = 4 * quad + i < n ? ordered_code(key[i]) : 0u;          // (0: below every masked item)
                cmax = c[i] > cmax ? c[i] : cmax;
                if (c[i] > CODE_MASKED) neg_cmin = ~c[i] > neg_cmin ? ~c[i] : neg_cmin;
                unmasked += c[i] > CODE_MASKED;
                smax = fmaxf(smax, x[i]);
                if (x[i] > -INFINITY) neg_smin = fmaxf(neg_smin, -x[i]);
            }
            reinterpret_cast<u32x4 *>(rank_code)[q] = c;
        }
        smax = wave_max_f(smax);
        neg_smin = wave_max_f(neg_smin);
        cmax = wave_reduce(cmax, OpMaxU{});
        neg_cmin = wave_reduce(neg_cmin, OpMaxU{});
        unmasked = wave_reduce(unmasked, OpAdd{});
        if (lane == 0) {
            maxima[wv] = u32x4{__float_as_uint(smax), __float_as_uint(neg_smin), cmax, neg_cmin};
            misc[wv] = unmasked;
        }
        __syncthreads();
        const u32x4 m = maxima[lane & (NW - 1)];
        smax = lanes_reduce<NW>(__uint_as_float(m[0]), OpMaxF{});
        neg_smin = lanes_reduce<NW>(__uint_as_float(m[1]), OpMaxF{});
        cmax = lanes_reduce<NW>(m[2], OpMaxU{});
        neg_cmin = lanes_reduce<NW>(m[3], OpMaxU{});
        unmasked = lanes_reduce<NW>(misc[lane & (NW - 1)], OpAdd{});
        const bool spread = want_logp && smax > -INFINITY && smax + neg_smin > NGC_WIDE_SPREAD;
        if (smax == -INFINITY) smax = 0.f;
        keys = PooledKeys{rank_code, cmax, smax, spread};
        ranked = !spread && K <= __builtin_amdgcn_readfirstlane(unmasked) &&
                 rank_items<THREADS>(rank_code, 4 * quads, K, cmax, ~neg_cmin, hist, reinterpret_cast<uint32_t *>(misc), idxB, idxA,
                                     kept_bits);
        if (ranked) {
            // kept slots before each head
            for (int h = wv; h <= Hkv; h += NW) {
                const int before = 4 * misc[PM_QUAD + h];
                int count = 0;
                for (int w = lane; 32 * w < before; w += NGC_WAVE) {
                    uint32_t bits = kept_bits[w];
                    if (32 * w + 32 > before) bits &= (1u << (before - 32 * w)) - 1u;
                    count += __popc(bits);
                }
                count = wave_reduce(count, OpAdd{});
                if (lane == 0) misc[PM_BASE + h] = count;
            }
            __syncthreads();
            const int words = (4 * quads + 63) / 64;
            const int per_wave = (words + NW - 1) / NW;
            const int w_begin = wv * per_wave;
            const int w_end = (w_begin + per_wave < words) ? (w_begin + per_wave) : words;
            const u32x2 *bits = reinterpret_cast<const u32x2 *>(kept_bits);
            int base = 0;
            for (int w = lane; w < w_begin; w += NGC_WAVE) base += __popc(bits[w][0]) + __popc(bits[w][1]);
            base = wave_reduce(base, OpAdd{});
            for (int w = w_begin; w < w_end; ++w) {
                const u32x2 pair = bits[w];
                const uint64_t sel_bits = ((uint64_t)pair[1] << 32) | pair[0];
                const int t = w * 64 + lane;
                if ((sel_bits >> lane) & 1u) {
                    const int h = head_of_quad(t >> 2);
                    const int slot = base + popc_below(sel_bits) - misc[PM_BASE + h];
                    if (slot < a.max_keep)
                        a.kept_out[(size_t)(seg_first + h) * a.max_keep + slot] = t - 4 * misc[PM_QUAD + h];
                }
                base += __popcll(sel_bits);
            }
            if (want_logp) {         // the weights of all items where their codes stood
                group = 0;
#pragma unroll 1
                for (int q = tid; q < quads; q += THREADS, ++group) {
                    f32x4 x = group == 0 ? held[0] : held[1];
                    if (group >= HELD) {
                        const int h = head_of_quad(q), first = 4 * (q - misc[PM_QUAD + h]), n = misc[PM_N + h];
                        const float *row = a.logits + (size_t)(seg_first + h) * cap;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            x[i] = first + i < n ? row[first + i] : -INFINITY;
                            if (x[i] != x[i]) x[i] = -INFINITY;
                        }
                    }
                    const uint32_t sel_bits = kept_bits[q >> 3] >> ((q & 7) * 4);
                    f32x4 e;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        e[i] = exp_shifted(x[i] - smax);
                        unpicked += (sel_bits >> i & 1u) ? 0.f : e[i];
                    }
                    reinterpret_cast<f32x4 *>(rank_code)[q] = e;
                }
            }
        }
    }
    if (!ranked) pooled_general<THREADS, RANK>(a, seg_first, l, b, N, K, keys, hist, misc, idxA, idxB);
    if (tid < Hkv) {
        const int kept = misc[PM_BASE + tid + 1] - misc[PM_BASE + tid];
        if (kept > a.max_keep) atomicAdd(&a.status[NGC_STATUS_KEEP_CLAMPED], 1);
        if (a.len_out) a.len_out[seg_first + tid] = kept < a.max_keep ? kept : a.max_keep;
    }
    __syncthreads();   // kept_out of this workgroup and the weights are complete and visible
    // ---- 2. per-head compaction; sums and logarithms come behind it ----
    if (a.k != nullptr)
        for (int h = 0; h < Hkv; ++h) {
            int Kh = misc[PM_BASE + h + 1] - misc[PM_BASE + h];
            Kh = Kh < a.max_keep ? Kh : a.max_keep;
            const size_t seg_off = (size_t)(seg_first + h) * cap * ROW_BYTES;
            const int32_t *kept = a.kept_out + (size_t)(seg_first + h) * a.max_keep;
            compact_kv_inplace<ROW_BYTES, THREADS, UNROLL, true>(reinterpret_cast<unsigned char *>(a.k) + seg_off,
                                                                 reinterpret_cast<unsigned char *>(a.v) + seg_off,
                                                                 kept, Kh, 0, 1);
            if (a.pos) compact_pos_inplace<THREADS>(a.pos + (size_t)(seg_first + h) * cap, kept, Kh, 0, 1);
        }
    if (ranked) {
        if (a.sigma_out) {
            // the pooled sequence occupies the Hkv rows of this (layer, sequence) back to back
            int32_t *sig_row = a.sigma_out + (size_t)seg_first * a.max_keep;
            const int room = Hkv * a.max_keep;
            for (int j = tid; j < K && j < room; j += THREADS) {
                const int t = idxA[j], h = head_of_quad(t >> 2);
                sig_row[j] = h * cap + (t - 4 * misc[PM_QUAD + h]);
            }
        }
        if (want_logp) {
            const float *weight = reinterpret_cast<const float *>(rank_code);
            const float lp = sigma_logprob<THREADS>([&](int j) { return weight[idxA[j]]; }, K, unpicked, fmisc);
            if (tid < Hkv) a.logp_out[seg_first + tid] = (tid == 0) ? lp : 0.f;
        }
    }
}

// The rows of a pooled round, one workgroup per segment: the selection has left each head's list and, as its length, how
// many it keeps.
template <int THREADS, int ROW_BYTES, int UNROLL>
__global__ __launch_bounds__(THREADS) void pooled_copy_kernel(SelectArgs a)
{
    const int seg = a.seg0 + (int)blockIdx.x;
    const int kept = a.len_out[seg];
    const int32_t *list = a.kept_out + (size_t)seg * a.max_keep;
    const size_t seg_off = (size_t)seg * a.g.cap * ROW_BYTES;
    compact_kv_inplace<ROW_BYTES, THREADS, UNROLL, true>(reinterpret_cast<unsigned char *>(a.k) + seg_off,
                                                         reinterpret_cast<unsigned char *>(a.v) + seg_off, list, kept, 0, 1);
    if (a.pos) compact_pos_inplace<THREADS>(a.pos + (size_t)seg * a.g.cap, list, kept, 0, 1);
}

// One segment at a time per workgroup: sample, score, then move the survivors.  While a workgroup is in its
// (ALU/LDS bound) selection phase, the other workgroups of the grid keep the memory system busy with their
// compaction phase.
template <int THREADS, int ROW_BYTES, int UNROLL>
__device__ __forceinline__ void evict_segment(const SelectArgs &a, int seg, unsigned char *smem_raw, int *misc)
{
    Selected sel;
    select_keep<THREADS>(a, seg, smem_raw, sel);
    if (a.k != nullptr) {
        __syncthreads();   // publishes misc[], the ascending list and this workgroup's kept_out writes
        const int rows_new = misc[MISC_ROWS], first = misc[MISC_FIRST];   // kept is ascending, kept[j] >= j
        if (threadIdx.x == 0) a.len_out[seg] = rows_new;
        if (first < sel.K) {
            const size_t seg_off = (size_t)seg * a.g.cap * ROW_BYTES;
            unsigned char *kbase = reinterpret_cast<unsigned char *>(a.k) + seg_off;
            unsigned char *vbase = reinterpret_cast<unsigned char *>(a.v) + seg_off;
            int32_t *pos = a.pos ? a.pos + (size_t)seg * a.g.cap : nullptr;
            if (a.unordered) {
                fill_holes_inplace<ROW_BYTES, THREADS, 4>(kbase, vbase, pos, sel.ascending, sel.K);
            } else {
                const int row_start = first * a.g.block;
                if ((a.g.block & (a.g.block - 1)) == 0)
                    compact_kv_inplace<ROW_BYTES, THREADS, UNROLL, true>(kbase, vbase, sel.ascending, rows_new, row_start,
                                                                         a.g.block);
                else
                    compact_kv_inplace<ROW_BYTES, THREADS, UNROLL, false>(kbase, vbase, sel.ascending, rows_new, row_start,
                                                                          a.g.block);
                if (pos)
                    compact_pos_inplace<THREADS>(pos, a.kept_out + (size_t)seg * a.max_keep, rows_new, row_start, a.g.block);
            }
        }
    }
    __syncthreads();       // the ascending list is free to be sorted
    select_score<THREADS>(a, seg, smem_raw, sel);
}

// The 1024-thread kernel (the host picks it for large segments, see ngc_evict) is persistent: one workgroup fills a CU, the grid
// holds as many workgroups as the chip keeps resident, and each takes the next segment from a counter in the
// workspace until none is left.  (With one workgroup per segment, a CU waited 7 us on average -- 20 us in one
// case out of ten -- between the end of one 1024-thread workgroup and the start of the next, with nothing else
// resident to cover the gap: 6 % of a round at 14336 segments of ~110 us each.)  The last workgroup to finish
// puts the two counters back to zero.  The smaller workgroups keep one workgroup per segment: two to four of
// them share a CU and cover each other's turnaround, and the loop costs them registers (values that do not
// change between segments stay live across the whole body: 69 -> 117 and 101 -> 171 vector registers, one
// workgroup fewer per CU, 6 % slower at 3584 segments of 4096 rows).
//
// Shape of the loop: the fetch by thread 0 sits between two barriers of its own, and the item index is made a
// scalar (it is the same in every lane).  Without the barrier in front of it the compiler merges the
// "thread 0 only" tail of one segment (the store of the new length) with the "thread 0 only" fetch of the
// next into one path, and the lanes that skip it are sent round an inner loop -- back to the barrier and the
// stale item -- that thread 0 never leaves: the grid never ends.
constexpr int PERSISTENT_THREADS = 1024;

template <int THREADS>
__device__ __forceinline__ int next_segment(const SelectArgs &a, int *slot)
{
    __syncthreads();   // every wave is done with the previous segment (its LDS, and the last read of *slot)
    if (threadIdx.x == 0) *slot = atomicAdd(&a.status[WS_QUEUE_NEXT], 1);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*slot);
}

template <int THREADS, int ROW_BYTES, int UNROLL>
__global__ __launch_bounds__(THREADS) void evict_kernel(SelectArgs a)
{
    constexpr int NW = THREADS / NGC_WAVE;
    constexpr int HIST = (SEL_BINS > SORT_BINS * NW) ? SEL_BINS : SORT_BINS * NW;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    int *misc = reinterpret_cast<int *>(reinterpret_cast<uint32_t *>(smem_raw) + a.items_cap + HIST);
    if constexpr (THREADS != PERSISTENT_THREADS) {
        evict_segment<THREADS, ROW_BYTES, UNROLL>(a, a.seg0 + (int)blockIdx.x, smem_raw, misc);
    } else {
        // The item index travels through the start of the sort buffer behind misc[], which a segment's selection writes
        // only after its first barrier: a word of static LDS would make the largest selections (all of a CU's 160 KB)
        // unlaunchable.
        int *next_item = misc + 64;
        for (int item = next_segment<THREADS>(a, next_item); item < a.nseg; item = next_segment<THREADS>(a, next_item))
            evict_segment<THREADS, ROW_BYTES, UNROLL>(a, a.seg0 + item, smem_raw, misc);
        if (threadIdx.x == 0) {
            const int done = atomicAdd(&a.status[WS_QUEUE_DONE], 1);
            if (done == (int)gridDim.x - 1) {   // every workgroup has taken its last item: nobody reads the counters any more
                __hip_atomic_store(&a.status[WS_QUEUE_NEXT], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&a.status[WS_QUEUE_DONE], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// --------------------------------------------------------- keep counts ----
//
// The fraction rule of Sec. 4.1 evaluated where the lengths live: K = ceil(N * num / den) items of the
// N = ceil(len / block) a segment has, in exact integer arithmetic, at least `min_keep` (and at least 1
// for a non-empty segment), at most N.  Saves the host a read-back of the ragged lengths per round.
__global__ __launch_bounds__(256) void keep_counts_kernel(const int32_t *__restrict__ len, int32_t *__restrict__ keep,
                                                          int seg0, int nseg, int cap, int block,
                                                          int64_t num, int64_t den, int min_keep)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= nseg) return;
    int n = len[seg0 + i];
    n = n < 0 ? 0 : (n > cap ? cap : n);
    const int64_t N = (n + block - 1) / block;
    int64_t K = (N * num + den - 1) / den;
    if (K < min_keep) K = min_keep;
    if (K < 1) K = 1;
    if (K > N) K = N;
    keep[seg0 + i] = (int32_t)K;
}

// -------------------------------------------------------------- append ----

struct AppendArgs {
    void *k;
    void *v;
    int32_t *pos;
    int32_t *len;
    const void *k_new;
    const void *v_new;
    const int32_t *new_pos;
    int32_t *status;
    int seg0;       // first segment of the launch
    int src_seg0;   // segment index that k_new[0] belongs to
    int B, Hkv, cap;
};

// One wave per segment: lanes [0, PIECES) copy the K row, the next PIECES the V row.
template <int ROW_BYTES>
__global__ __launch_bounds__(64) void append_kernel(AppendArgs a)
{
    constexpr int PIECES = ROW_BYTES / 16;
    const int seg = a.seg0 + blockIdx.x;
    const int lane = threadIdx.x;
    const int n = a.len[seg];
    if (n < 0 || n >= a.cap) {
        if (lane == 0) atomicAdd(&a.status[NGC_STATUS_APPEND_FULL], 1);
        return;
    }
    const size_t src_off = (size_t)(seg - a.src_seg0) * ROW_BYTES;
    const size_t dst_off = ((size_t)seg * a.cap + n) * ROW_BYTES;
    if (lane < 2 * PIECES) {
        const bool is_v = lane >= PIECES;
        const int piece = is_v ? lane - PIECES : lane;
        const unsigned char *s = reinterpret_cast<const unsigned char *>(is_v ? a.v_new : a.k_new) + src_off;
        unsigned char *d = reinterpret_cast<unsigned char *>(is_v ? a.v : a.k) + dst_off;
        *reinterpret_cast<uint4 *>(d + piece * 16) = *reinterpret_cast<const uint4 *>(s + piece * 16);
    }
    __syncthreads();
    if (lane == 0) {
        if (a.pos && a.new_pos) a.pos[(size_t)seg * a.cap + n] = a.new_pos[(seg / a.Hkv) % a.B];
        a.len[seg] = n + 1;
    }
}

}  // namespace ngc

// ============================================================ host side ====

using namespace ngc;

namespace {

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_cache(const ngc_cache *c)
{
    if (!c || !c->k || !c->v || !c->len) return NGC_EINVAL;
    if (!aligned16(c->k) || !aligned16(c->v)) return NGC_EINVAL;
    if (c->L <= 0 || c->B <= 0 || c->Hkv <= 0 || c->Hq <= 0 || c->cap <= 0) return NGC_EINVAL;
    if (c->D != 64 && c->D != 128) return NGC_EINVAL;
    if (c->Hq % c->Hkv != 0 || c->Hq / c->Hkv > 16) return NGC_EINVAL;
    if (c->L > 65535 || c->Hkv > 65534) return NGC_EINVAL;   // noise counter packs layer and head in 16 bits each
    return NGC_OK;
}

// The noise counter packs the global layer index into 16 bits.
int check_bases(const ngc_cache *c, const ngc_evict_params *p)
{
    if (p->layer_base < 0 || p->seq_base < 0) return NGC_EINVAL;
    if ((long long)p->layer_base + c->L > 65535) return NGC_EINVAL;
    if ((long long)p->seq_base + c->B > 0x7FFFFFFFLL) return NGC_EINVAL;
    return NGC_OK;
}

int layer_range(const ngc_cache *c, int layer, int *seg0, int *nseg)
{
    if (layer < -1 || layer >= c->L) return NGC_EINVAL;
    const int per_layer = c->B * c->Hkv;
    *seg0 = layer < 0 ? 0 : layer * per_layer;
    *nseg = layer < 0 ? c->L * per_layer : per_layer;
    return NGC_OK;
}

constexpr size_t STATUS_BYTES = NGC_STATUS_WORDS * sizeof(int32_t);

// Grid of a persistent kernel: as many workgroups as the device keeps resident at this workgroup size and LDS
// use (asked of the runtime once per device, kernel and LDS size, then remembered: the query costs tens of
// microseconds of host time; one per CU if the runtime does not say), but no more than there are items.
int resident_workgroups(const void *fn, int threads, size_t lds, int items)
{
    struct Key {
        int dev;
        const void *fn;
        size_t lds;
        bool operator<(const Key &o) const
        {
            return dev != o.dev ? dev < o.dev : (fn != o.fn ? fn < o.fn : lds < o.lds);
        }
    };
    static std::mutex lock;
    static std::map<Key, long long> known;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    long long slots;
    {
        std::lock_guard<std::mutex> g(lock);
        const Key key{dev, fn, lds};
        auto it = known.find(key);
        if (it == known.end()) {
            int cus = 0, per_cu = 0;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
                cus = 256;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds) != hipSuccess || per_cu <= 0) {
                (void)hipGetLastError();
                per_cu = 1;
            }
            it = known.emplace(key, (long long)cus * per_cu).first;
        }
        slots = it->second;
    }
    return (int)(slots < items ? slots : items);
}

// Eq. 2 and its gradient: the workgroup of a segment and how much of its row it holds in LDS.  The host knows the stride
// of the rows (no row that keeps to its own is longer), an upper bound on the picks, and the number of segments; a row or
// a sequence too long for the choice takes the general route.
//   - Strides up to 8192: by the stride.  Two rounds of Eq. 2 and its gradient, us: 2048 segments of 700-1400 items 53
//     with 256 threads, 67 with 512; of 1000-2000 items 69 and 76 (before the weights were computed once per item).  From
//     2049 to 4096 items a workgroup of 256 threads with 16 picks each runs fewer instructions in all but is a longer chain:
//     Eq. 2 of 512 segments of 2150-3789 items 7.2 us, 6.0 with 512 threads, of 2048 15.4 and 15.1, of 3584 22.4 and 24.3; the
//     gradient, whose 16 picks cost registers, 8.9 and 7.5, 20.1 and 19.2, 29.4 and 29.2.
//   - Strides up to 16384, as in a cache of that capacity: the rows in it are often far shorter, and with a whole stride in
//     LDS only two workgroups share a CU, so the picks decide.  Eq. 2 / gradient at a stride of 16384, us (one of 512
//     threads on the general route alone, then threads x picks per thread):
//         segments x items, picks       general     256 x 4/8     512 x 8/16    1024 x 16
//         3584 x 150-300,    240       15.2 / 17.2  17.3 / 20.0   20.6 / 24.8   42.9 / 60.2
//         3584 x 300-600,    480       18.2 / 21.2  17.3 / 20.9   21.2 / 25.3   43.8 / 61.5
//         3584 x 2150-3789, 1000       37.1 / 55.2  34.1 / 46.9   28.5 / 34.5   56.5 / 72.7
//         2048 x 700-1400,  1120       15.5 / 21.8  14.1 / 17.2   14.2 / 17.0   28.8 / 37.6
//         896 x 12000-16000, 1919      38.3 / 83.6  25.3 / 40.5   19.0 / 29.8   25.2 / 34.9
//         3584 x 2150-3789, 3144       52.3 / 93.6       -        33.6 / 39.4   59.9 / 76.6
//         896 x 6000-7000,  5599       34.6 / 95.4       -        16.3 / 21.4   23.1 / 30.1
//         400 x 6000-7000,  2000       12.0 / 19.9   7.2 / 11.4    6.0 /  8.2    9.6 / 13.0
//         16 x 12000-16000, 7128       23.6 / 38.0       -         8.4 / 12.2    7.1 /  8.6
//     Up to 1024 picks the rows may be short or long, and 256 threads are the slowest for neither; beyond, rows are as long
//     as their picks and 512 are never the slower ones (before the weights were computed once per item, 256 were, up to
//     2048 picks).  Up to 512 segments, all resident at once, the larger
//     workgroup is faster: it works through a row in fewer steps.
//   - Longer strides, or one row for all segments (stride 0): rows may be longer than any LDS row or far shorter (blocks of
//     rows as items).  LOGPROB_ROW_OF_FOUR items leave room for four workgroups of 512 threads, what the general route
//     wants: 896 x 18000-20000 items, 1999 picks: 49 / 110 us, with 16384 items in LDS 73 / 125 (1024 threads 67 / 106);
//     3584 x 2150-3789: 33 / 44 and 77 / 104.  Beyond 4096 picks the gradient's general route takes 1024 threads
//     (5999 picks: 161 us, 220 with 512), Eq. 2 does not (87 and 85).
constexpr int LOGPROB_MAX_ROW = 16384;
constexpr int LOGPROB_ROW_OF_FOUR = 8064;
constexpr int LOGPROB_FEW = 512;
constexpr int LOGPROB_MANY = 2048;

struct LogprobShape {
    int threads, picks, row_cap;
};

LogprobShape logprob_shape(int64_t stride, int64_t most_picks, int nseg, bool gradient)
{
    if (stride <= 0 || stride > LOGPROB_MAX_ROW) {
        if (most_picks <= 4096) return {512, 8, LOGPROB_ROW_OF_FOUR};
        if (most_picks <= 8192 && !gradient) return {512, 16, LOGPROB_ROW_OF_FOUR};
        return {1024, 16, LOGPROB_MAX_ROW};
    }
    const int row_cap = (int)((stride + 3) & ~(int64_t)3);
    most_picks = most_picks < stride ? most_picks : stride;
    if (row_cap <= 1024) return {256, 4, row_cap};
    if (row_cap <= 2048) return {256, 8, row_cap};
    if (row_cap <= 4096 && !gradient && nseg > LOGPROB_MANY) return {256, 16, row_cap};
    if (row_cap <= 8192) return {512, most_picks <= 4096 ? 8 : 16, row_cap};
    if (nseg > LOGPROB_FEW && most_picks <= 1024) return {256, 4, row_cap};
    if (most_picks <= 4096) return {512, 8, row_cap};
    if (most_picks <= 8192 && nseg > LOGPROB_FEW) return {512, 16, row_cap};
    return {1024, 16, row_cap};
}

// Whether Eq. 4 goes to one workgroup.  Nanoseconds, call after call: it takes about 3700 + 0.32 a term and, beyond the 16
// layers that its waves hold at once, 1.3 L^2; the two kernels 5900 + 240 for every 256 rollouts and heads of every round + 20
// a layer.  Microseconds of two kernels and of one (* where it is taken):
//      1 layer,   16 rounds, 8192 terms  14.6   5.7 *      20 layers,  1 round,  10240 terms   6.5   7.0
//      4 layers,   8 rounds, 16384        9.9   8.6 *      28 layers,  9 rounds,  8064         9.0   7.0 *
//      8 layers,   3 rounds, 12288        7.2   7.6        28 layers,  1 round,  14336         6.8   8.1
//     16 layers,   1 round,  8192         6.5   5.7 *      40 layers,  1 round,   1280         7.0   6.3 *
//     16 layers,   2 rounds, 16384        6.9   8.4        48 layers,  1 round,   1536         7.2   7.3
//     17 layers,   1 round,  8704         6.5   6.7       128 layers,  1 round,   4096        10.7  15.7
bool lmem_in_one(int64_t R, int64_t L, int64_t B, int64_t H)
{
    if (B > LMEM_ONE_MAX_B || L > LMEM_ONE_MAX_L || B * H > LMEM_ONE_MAX_TERMS || R > LMEM_ONE_MAX_TERMS ||
        R * L * B * H > LMEM_ONE_MAX_TERMS)
        return false;
    const int64_t one = 3700 + R * L * B * H * 32 / 100 + (L > LMEM_ONE_WAVES ? L * L * 13 / 10 : 0);
    const int64_t two = 5900 + 240 * R * ((B * H + LMEM_THREADS - 1) / LMEM_THREADS) + 20 * L;
    return one <= two;
}

// One of the five instantiations of a kernel by its workgroup.
#define NGC_PICK_SHAPE(KERNEL, shape) \
    ((shape).picks == 4       ? reinterpret_cast<const void *>(&KERNEL<256, 4, 1>) \
     : (shape).threads == 256 ? reinterpret_cast<const void *>(&KERNEL<256, 8, 2>) \
     : (shape).picks == 8     ? reinterpret_cast<const void *>(&KERNEL<512, 8, 4>) \
     : (shape).threads == 512 ? reinterpret_cast<const void *>(&KERNEL<512, 16, 4>) \
                              : reinterpret_cast<const void *>(&KERNEL<1024, 16, 4>))

// A segment's row and the spare words behind it or, on the general route, the bitmap and a value per pick.
size_t logprob_lds_bytes(const LogprobShape &shape, int picks)
{
    const int row = shape.row_cap + SPARE_ITEMS, general = PICKED_WORDS + picks;
    return (size_t)(row > general ? row : general) * sizeof(float);
}

}  // namespace

extern "C" int ngc_perturbed_keys(const ngc_cache *c, int32_t layer, const float *logits,
                                  const ngc_evict_params *p, float *keys_out,
                                  void *ws, size_t ws_bytes, void *stream)
{
    int rc = check_cache(c);
    if (rc) return rc;
    if (!logits || !keys_out || !p || !ws || p->block < 1) return NGC_EINVAL;
    if ((rc = check_bases(c, p)) != NGC_OK) return rc;
    if (ws_bytes < STATUS_BYTES) return NGC_ENOSPC;
    int seg0, nseg;
    rc = layer_range(c, layer, &seg0, &nseg);
    if (rc) return rc;
    SegGeom g{c->B, c->Hkv, c->cap, p->block};
    NoiseArgs na{p->seed, p->round, p->noise_scale, p->share_heads, p->layer_base, p->seq_base};
    hipLaunchKernelGGL(perturbed_keys_kernel, dim3(nseg), dim3(256), 0, (hipStream_t)stream,
                       logits, c->len, keys_out, seg0, g, na, reinterpret_cast<int32_t *>(ws));
    NGC_HIP_CHECK(hipGetLastError());
    return NGC_OK;
}

extern "C" int ngc_evict(const ngc_cache *c, int32_t layer, const float *logits,
                         const int32_t *keep, const ngc_evict_params *p, int32_t max_keep,
                         int32_t *kept_out, int32_t *sigma_out, float *logp_out,
                         void *ws, size_t ws_bytes, void *stream)
{
    int rc = check_cache(c);
    if (rc) return rc;
    if (!logits || !keep || !p || !kept_out || !ws || p->block < 1 || max_keep < 1) return NGC_EINVAL;
    if ((rc = check_bases(c, p)) != NGC_OK) return rc;
    if ((p->flags & NGC_EVICT_UNORDERED) && p->block != 1) return NGC_EUNSUPPORTED;
    if ((long long)c->cap * c->D * 2 > 0x7FFFFFFFLL) return NGC_EUNSUPPORTED;   // 32-bit byte offsets inside a segment
    int seg0, nseg;
    rc = layer_range(c, layer, &seg0, &nseg);
    if (rc) return rc;
    const int nseg_total = c->L * c->B * c->Hkv;
    if (ws_bytes < STATUS_BYTES + (size_t)nseg_total * 8) return NGC_ENOSPC;
    if (!aligned16(ws)) return NGC_EINVAL;

    if (p->flags & NGC_EVICT_POOL_HEADS) {
        // one selection per (layer, sequence) over the items of all its heads
        if (p->block != 1 || (p->flags & NGC_EVICT_UNORDERED)) return NGC_EUNSUPPORTED;
        if (c->Hkv > POOL_MAX_HEADS || (long long)c->Hkv * c->cap > 65536) return NGC_EUNSUPPORTED;
        const size_t codes_off = ngc_workspace_bytes(c, max_keep);
        const size_t codes_bytes = (size_t)c->L * c->B * c->Hkv * c->cap * sizeof(uint32_t) * 4;
        if (ws_bytes < codes_off + codes_bytes) return NGC_ENOSPC;
        long long kc = (long long)c->Hkv * max_keep;
        if (kc > (long long)c->Hkv * c->cap) kc = (long long)c->Hkv * c->cap;
        int keep_cap = (int)((kc + 7) & ~7LL);
        const long long quads = (long long)c->Hkv * ((c->cap + 3) / 4);
        // One workgroup per (layer, sequence) selects.  Up to POOL_FEW of them, half the CUs at most would copy, one head
        // after another: the rows get a launch of their own, a workgroup per head.  Microseconds with one launch and with two:
        //     sequences x heads x rows      8 x 4 x 500   32 x 2 x 1500   64 x 4 x 4000   128 x 4 x 1500   128 x 2 x 4000
        //                                  28.1  21.9     37.5  31.7     217.2  163.2    107.7  107.2     132.6  134.1
        //                               192 x 4 x 1500  192 x 4 x 4000   256 x 2 x 1500   448 x 4 x 500    896 x 4 x 1500
        //                                 141.2  146.0   345.5  373.4      91.0   97.9     109.5  119.2    564.1  627.8
        // 1024 threads; 512 where several workgroups share a CU and have little to select (us of 1024 and of 512: 448 x 2 x
        // 500 rows 59.2 and 55.8, 896 x 8 x 300 268 and 250, 896 x 2 x 1500 289 and 293, 448 x 8 x 1000 398 and 438; 256 x 4 x
        // 500 65.3 and 67.8; two launches, 16 x 8 x 300 24.7 and 27.8).
        const int sequences = nseg / c->Hkv;
        const bool split = sequences <= POOL_FEW;
        const int threads = sequences > POOL_MANY && (long long)c->Hkv * c->cap <= POOL_SMALL_ITEMS ? 512 : 1024;
        const int hist = (SEL_BINS > SORT_BINS * (threads / 64)) ? SEL_BINS : SORT_BINS * (threads / 64);
        const size_t fixed = (size_t)hist * 4 + PM_WORDS * 4;
        auto lds_for = [&](long long ranked) {
            const long long second = ranked > keep_cap ? ranked : keep_cap;
            return fixed + (ranked > 0 ? PM_MAXIMA * 4 : 0) + (size_t)ranked * 4 + (size_t)((ranked + 63) / 64) * 8 + (size_t)keep_cap * 2 + (size_t)second * 2;
        };
        // (without a sequence or its log-probability nothing is ranked, and the LDS for it would keep a second workgroup off the CU)
        int rank_cap = sigma_out || logp_out ? (int)((4 * quads + 7) & ~7LL) : 0;
        if (lds_for(rank_cap) > 160 * 1024) rank_cap = 0;
        size_t lds = lds_for(rank_cap);
        if (lds > 160 * 1024) {
            // Hkv * max_keep is only an upper bound of what a (layer, sequence) keeps (max_keep has to cover the
            // largest single head); the budget itself is on the device.  The index buffers take what LDS holds;
            // a budget above that is clamped by the kernel and counted in NGC_STATUS_KEEP_CLAMPED.
            keep_cap = (int)(((160 * 1024 - fixed) / 4) & ~7u);
            lds = lds_for(0);
        }
        SelectArgs sa;
        sa.logits = logits; sa.len = c->len; sa.keep = keep;
        sa.kept_out = kept_out; sa.sigma_out = sigma_out; sa.logp_out = logp_out;
        sa.status = reinterpret_cast<int32_t *>(ws);
        const bool move = !(p->flags & NGC_EVICT_SELECT_ONLY);       // (a second launch finds a.len_out, not a.k, set)
        sa.k = move && !split ? c->k : nullptr; sa.v = c->v; sa.pos = c->pos; sa.len_out = move ? c->len : nullptr;
        sa.unordered = 0;
        sa.seg0 = seg0; sa.max_keep = max_keep; sa.items_cap = 0; sa.keep_cap = keep_cap; sa.rank_cap = rank_cap;
        sa.pool_codes = reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(ws) + codes_off);
        sa.g = SegGeom{c->B, c->Hkv, c->cap, 1};
        sa.logit_stride = c->cap;
        sa.na = NoiseArgs{p->seed, p->round, p->noise_scale, p->share_heads, p->layer_base, p->seq_base};
#define NGC_PICK(KERNEL, T, ...) ((c->D == 128) ? reinterpret_cast<const void *>(&KERNEL<T, 256, __VA_ARGS__>) \
                                                : reinterpret_cast<const void *>(&KERNEL<T, 128, __VA_ARGS__>))
        const void *select = rank_cap > 0 ? (threads == 1024 ? NGC_PICK(evict_pooled_kernel, 1024, 4, true)
                                                             : NGC_PICK(evict_pooled_kernel, 512, 8, true))
                                          : (threads == 1024 ? NGC_PICK(evict_pooled_kernel, 1024, 4, false)
                                                             : NGC_PICK(evict_pooled_kernel, 512, 8, false));
        if (lds > 64 * 1024)
            NGC_HIP_CHECK(hipFuncSetAttribute(select, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        void *kargs[] = {&sa};
        NGC_HIP_CHECK(hipLaunchKernel(select, dim3(sequences), dim3(threads), kargs, lds, (hipStream_t)stream));
        if (!move || !split) return NGC_OK;
        sa.k = c->k;
        const int movers = c->cap > 4096 ? 1024 : (c->cap > 512 ? 512 : 256);    // (as in the per-head mode)
        const void *copy = movers == 1024  ? NGC_PICK(pooled_copy_kernel, 1024, 4)
                           : movers == 512 ? NGC_PICK(pooled_copy_kernel, 512, 8)
                                           : NGC_PICK(pooled_copy_kernel, 256, 6);
#undef NGC_PICK
        NGC_HIP_CHECK(hipLaunchKernel(copy, dim3(nseg), dim3(movers), kargs, 0, (hipStream_t)stream));
        return NGC_OK;
    }

    const int items_cap = (c->cap + p->block - 1) / p->block;
    if (items_cap > 16384) return NGC_EUNSUPPORTED;
    int keep_cap = max_keep < items_cap ? max_keep : items_cap;
    keep_cap = (keep_cap + 7) & ~7;
    const int items_cap_al = (items_cap + 3) & ~3;
    // Workgroup size and rows in flight per thread, all measured.  A round that moves rows in order is a copy with a
    // selection in front, and the size follows the rows of a segment, not its items.  One 1024-thread workgroup per CU, whose
    // reads and writes take turns, copies best, but has nothing beside it while it selects, and half a round of 256 of them
    // counts as a whole one: it is taken beyond 4096 rows and, with many segments and enough rows kept, from fewer.  Times of
    // 512 over 1024 threads by the share kept:
    //     segments x rows      a tenth  a fifth  a quarter  a third  0.4   half  nine tenths
    //        640 x 1600          0.81     0.84                0.93          0.98     1.04
    //       1152 x 1600          0.80     0.88     0.95       0.97  1.00    1.02     1.06
    //       1536 x 1300          0.69     0.82     0.85       0.95  0.95    1.00     1.05
    //       1792 x 3300          0.86     0.97     0.89       0.98  1.00    1.02     1.07
    //       2048 x 2048          0.77     0.90     0.94       0.99  1.00    1.05     1.06
    //       3584 x 1300          0.65     0.81     0.86       0.99  0.99    1.07     1.09
    //       3584 x 2304          0.78     0.98     0.98       1.05  1.08    1.09     1.11
    //       3584 x 4096          0.73     0.89     0.98       1.04  1.05    1.06     1.06
    // i.e. from half kept up and, beyond 2048 segments, from a third.  (In one job of ten 512 threads copied faster than
    // in all others, 2048 x 4096 rows, a third kept, in 478 us instead of 548, and the half-kept rounds were at 0.94-0.98;
    // the cause was not found.)  What is kept is on the device; max_keep is its bound.
    // Uneven budgets under a loose bound are taken for more than they are: 1536 x 1300 rows, a fifth kept of a bound of half,
    // 114 us where 512 threads take 102; a third of a bound of 0.83, 152 and 155.  512 threads from
    // 513 rows up (896 of 700: 74, 77 with 256), 256 below (896 of 300: 35 and 38).  A round that only selects, or fills
    // holes (few rows move), is bound by the selection's waits; two 512-thread workgroups per CU cover each other's up to
    // the 8192 rows at which two of them still fit in LDS (1024 segments of 8192: 96 us, 135 with 1024 threads), 256
    // threads up to 2048 rows (1024 of 1500: 25 us, 28 with 512) unless there are too few segments to fill the chip
    // that way (16 of 1500: 14.6 us with 512 threads, 17.2 with 256).  Their 512-thread kernel is the one with 2 rows a thread in
    // the ordered copy, which they do not run: 63 registers instead of the 113 that 8 rows cost, three workgroups a CU instead
    // of two (2048 segments of 4096 rows, kept lists only: 56 us, 66 with the other; 1024: 31.7 and 34.8).
    const bool move_rows = !(p->flags & NGC_EVICT_SELECT_ONLY);
    const bool copy_bound = move_rows && !(p->flags & NGC_EVICT_UNORDERED);
    const int few = (copy_bound || nseg <= 512) ? 512 : 2048;
    const long long kept_rows = (long long)max_keep * p->block;              // at most, of a segment
    int many = copy_bound ? 4096 : 8192;
    if (copy_bound && ((nseg > 2048 && 3 * kept_rows >= c->cap) || (nseg > 1024 && 2 * kept_rows >= c->cap))) many = 1280;
    else if (copy_bound && nseg > 512 && 2 * kept_rows >= c->cap) many = 1536;
    const int threads = c->cap > many ? 1024 : (c->cap > few ? 512 : 256);
    const int rank_cap = rank_capacity(threads, items_cap_al, keep_cap);
    const size_t lds = select_lds_bytes(threads, items_cap_al, keep_cap, rank_cap);
    if (lds > 160 * 1024) return NGC_EUNSUPPORTED;

    int32_t *status = reinterpret_cast<int32_t *>(ws);

    SelectArgs sa;
    sa.logits = logits; sa.len = c->len; sa.keep = keep;
    sa.kept_out = kept_out; sa.sigma_out = sigma_out; sa.logp_out = logp_out;
    sa.status = status;
    sa.k = move_rows ? c->k : nullptr; sa.v = c->v; sa.pos = c->pos; sa.len_out = c->len;
    sa.unordered = (p->flags & NGC_EVICT_UNORDERED) ? 1 : 0;
    sa.pool_codes = nullptr;
    sa.seg0 = seg0; sa.max_keep = max_keep; sa.items_cap = items_cap_al; sa.keep_cap = keep_cap; sa.rank_cap = rank_cap;
    sa.g = SegGeom{c->B, c->Hkv, c->cap, p->block};
    sa.logit_stride = c->cap;
    sa.na = NoiseArgs{p->seed, p->round, p->noise_scale, p->share_heads, p->layer_base, p->seq_base};

    hipStream_t st = (hipStream_t)stream;
    const void *fn;
#define NGC_PICK(T, U) ((c->D == 128) ? reinterpret_cast<const void *>(&evict_kernel<T, 256, U>) \
                                      : reinterpret_cast<const void *>(&evict_kernel<T, 128, U>))
    if (threads == 1024) fn = NGC_PICK(1024, 4);
    else if (threads == 512 && !copy_bound) fn = NGC_PICK(512, 2);
    else if (threads == 512) fn = NGC_PICK(512, 8);
    else fn = NGC_PICK(256, 6);
#undef NGC_PICK
    if (lds > 64 * 1024)
        NGC_HIP_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    sa.nseg = nseg;
    const int grid = threads == PERSISTENT_THREADS ? resident_workgroups(fn, threads, lds, nseg) : nseg;
    void *kargs[] = {&sa};
    NGC_HIP_CHECK(hipLaunchKernel(fn, dim3(grid), dim3(threads), kargs, lds, st));
    return NGC_OK;
}

extern "C" int ngc_subset_logprob(const float *logits, const int32_t *n_items,
                                  const int32_t *sigma, const int32_t *keep, int32_t nseg,
                                  int64_t logit_stride, int32_t sigma_stride,
                                  float *logp_out, void *ws, size_t ws_bytes, void *stream)
{
    if (!logits || !n_items || !sigma || !keep || !logp_out || !ws) return NGC_EINVAL;
    if (nseg < 0 || logit_stride < 0 || sigma_stride < 0) return NGC_EINVAL;
    if (ws_bytes < STATUS_BYTES) return NGC_ENOSPC;
    if (nseg == 0) return NGC_OK;
    const int stage_cap = sigma_stride < 16384 ? sigma_stride : 16384;     // at most 64 KB of LDS
    // (sigma_stride 0: one sequence for all segments, of any length)
    const LogprobShape shape = logprob_shape(logit_stride, sigma_stride > 0 ? sigma_stride : 65536, nseg, false);
    LogprobArgs la{logits, n_items, sigma, keep, logp_out, reinterpret_cast<int32_t *>(ws),
                   logit_stride, sigma_stride, stage_cap, shape.row_cap};
    const size_t lds = logprob_lds_bytes(shape, stage_cap);
    const void *fn = shape.threads == 256 && shape.picks == 16
                         ? reinterpret_cast<const void *>(&subset_logprob_kernel<256, 16, 4>)      // (Eq. 2 alone)
                         : NGC_PICK_SHAPE(subset_logprob_kernel, shape);
    if (lds > 48 * 1024)
        NGC_HIP_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    void *kargs[] = {&la};
    NGC_HIP_CHECK(hipLaunchKernel(fn, dim3(nseg), dim3(shape.threads), kargs, lds, (hipStream_t)stream));
    return NGC_OK;
}

extern "C" int ngc_subset_logprob_backward(const float *logits, const int32_t *n_items,
                                           const int32_t *sigma, const int32_t *keep, int32_t nseg,
                                           int64_t logit_stride, int32_t sigma_stride, int32_t max_keep,
                                           const float *gout, float *grad_out,
                                           void *ws, size_t ws_bytes, void *stream)
{
    if (!logits || !n_items || !sigma || !keep || !grad_out || !ws) return NGC_EINVAL;
    if (nseg < 0 || logit_stride < 0 || sigma_stride < 0 || max_keep < 1) return NGC_EINVAL;
    if (ws_bytes < STATUS_BYTES) return NGC_ENOSPC;
    if (max_keep > 32768) return NGC_EUNSUPPORTED;
    if (nseg == 0) return NGC_OK;
    const LogprobShape shape = logprob_shape(logit_stride, max_keep, nseg, true);
    LogprobBwdArgs la{logits, n_items, sigma, keep, gout, grad_out, reinterpret_cast<int32_t *>(ws),
                      logit_stride, sigma_stride, max_keep, shape.row_cap};
    const size_t lds = logprob_lds_bytes(shape, max_keep);
    const void *fn = NGC_PICK_SHAPE(subset_logprob_backward_kernel, shape);
    if (lds > 48 * 1024)
        NGC_HIP_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    void *kargs[] = {&la};
    NGC_HIP_CHECK(hipLaunchKernel(fn, dim3(nseg), dim3(shape.threads), kargs, lds, (hipStream_t)stream));
    return NGC_OK;
}

extern "C" int ngc_cache_append(const ngc_cache *c, int32_t layer, const void *k_new,
                                const void *v_new, const int32_t *new_pos,
                                void *ws, size_t ws_bytes, void *stream)
{
    int rc = check_cache(c);
    if (rc) return rc;
    if (!k_new || !v_new || !ws || !aligned16(k_new) || !aligned16(v_new)) return NGC_EINVAL;
    if (ws_bytes < STATUS_BYTES) return NGC_ENOSPC;
    int seg0, nseg;
    rc = layer_range(c, layer, &seg0, &nseg);
    if (rc) return rc;
    AppendArgs aa{c->k, c->v, c->pos, c->len, k_new, v_new, new_pos,
                  reinterpret_cast<int32_t *>(ws), seg0, seg0, c->B, c->Hkv, c->cap};
    if (c->D == 128)
        hipLaunchKernelGGL(append_kernel<256>, dim3(nseg), dim3(64), 0, (hipStream_t)stream, aa);
    else
        hipLaunchKernelGGL(append_kernel<128>, dim3(nseg), dim3(64), 0, (hipStream_t)stream, aa);
    NGC_HIP_CHECK(hipGetLastError());
    return NGC_OK;
}

extern "C" int ngc_lmem(const float *logp, const int32_t *rounds, const float *reward,
                        int32_t R, int32_t L, int32_t B, int32_t Hkv, int32_t group,
                        float *adv_out, float *loss_layer, float *loss, float *gout, void *stream)
{
    if (!logp || !rounds || !reward || !loss_layer || !loss) return NGC_EINVAL;
    if (R < 1 || L < 1 || B < 1 || Hkv < 1 || group < 1 || B % group != 0) return NGC_EINVAL;
    if (B > LMEM_MAX_B) return NGC_EUNSUPPORTED;
    LmemArgs la{logp, rounds, reward, adv_out, loss_layer, gout, R, L, B, Hkv, group};
    hipStream_t st = (hipStream_t)stream;
    if (lmem_in_one(R, L, B, Hkv)) {
        hipLaunchKernelGGL(lmem_one_kernel, dim3(1), dim3(LMEM_ONE_THREADS), 0, st, la,
                           divide_by((uint32_t)Hkv), divide_by((uint32_t)(B * Hkv)), loss);
        NGC_HIP_CHECK(hipGetLastError());
        return NGC_OK;
    }
    hipLaunchKernelGGL(lmem_layer_kernel, dim3(L), dim3(LMEM_THREADS), 0, st, la);
    NGC_HIP_CHECK(hipGetLastError());
    hipLaunchKernelGGL(lmem_total_kernel, dim3(1), dim3(64), 0, st, (const float *)loss_layer, (int)L, loss);
    NGC_HIP_CHECK(hipGetLastError());
    return NGC_OK;
}

extern "C" int ngc_keep_counts(const int32_t *len, int32_t seg0, int32_t nseg, int32_t cap, int32_t block,
                               int32_t num, int32_t den, int32_t min_keep, int32_t *keep_out, void *stream)
{
    if (!len || !keep_out) return NGC_EINVAL;
    if (seg0 < 0 || nseg < 0 || cap < 1 || block < 1 || num < 0 || den < 1 || num > den || min_keep < 0) return NGC_EINVAL;
    if (nseg == 0) return NGC_OK;
    hipLaunchKernelGGL(keep_counts_kernel, dim3((nseg + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       len, keep_out, (int)seg0, (int)nseg, (int)cap, (int)block, (int64_t)num, (int64_t)den, (int)min_keep);
    NGC_HIP_CHECK(hipGetLastError());
    return NGC_OK;
}
