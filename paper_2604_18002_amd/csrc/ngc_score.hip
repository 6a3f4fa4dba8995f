// Key scoring for the eviction policy on gfx950 (Sec. 4.2 of the paper): the
// attention weights that the w most recent queries put on every cached key,
// averaged over the query heads of a KV head and over the w queries, then
// (optionally) averaged over KV heads and over blocks of consecutive keys.
//
// One workgroup of 4 waves per (layer, sequence, KV head), several (or of 8 waves)
// where there are few of those (they ask for the queries, and for normalisers that
// are given, before the length is known).  The w*G query rows
// are padded to QT tiles of 16 and both passes run on the matrix cores:
//   pass 1  S^T = K Q^T   (queries on lane%16): running max / sum per query row
//   pass 2  S   = Q K^T   (keys on lane%16):    p = 2^(x - m) / l, summed over
//                                               the query rows of each key
// The two orientations use the same operand registers with the MFMA arguments
// swapped.  K is read twice (once per pass); nothing else touches HBM except
// the one fp32 score per key that is written.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/ngc.h"
#include "ngc_device.h"

namespace ngc {

constexpr int SC_WAVES = 4;
constexpr int SC_TILE = 32;
constexpr int MOST_SHARES = 32;

struct ScoreArgs {
    const unsigned char *k;
    const int32_t *len;
    const unsigned char *q;   // bf16 [lb][w][Hq][D]
    const float *lse;         // optional fp32 [lb][w][Hq]: log-sum-exp of every query's scaled scores
    float *psi_out;           // fp32 [seg][cap], one value per key or per tile
    int32_t *status;
    int seg0, nseg, lb0;
    int S;                    // workgroups per segment (1 for SCORE_BOTH) ...
    int share_rows;           // ... of at least so many rows; shorter ones are left to their first (SCORE_FIRST, SCORE_SECOND:
                              // as many of them as shares_of() says)
    int w, G, Hkv, cap, causal;
    float scale_log2e;
    // paged layout: k is the pool and a tile's base comes from the page table
    const int32_t *table;   // [seg][max_pages] or nullptr (contiguous layout)
    int max_pages, num_pages, tpp_shift;
    int block;                // a multiple of SC_TILE (TILES): tile t leaves the sum of its keys, their mean if the block is
                              // one tile, at psi[t]
};

// Where the shares of a segment leave their maxima and sums between the two launches: in the segment's own row of the scores,
// below its length, where every entry is either written again by the second launch or past the items.  (The workspace
// has no room to give: a call may bring the status words alone, or the workspace of another cache, whose tickets have to
// stay zero.)  Tiles' values end at the number of tiles, so one copy of all shares' parts fits behind them.  With a value
// per key a share reads its copy from the entries that itself will overwrite, so every share writes one for each of them:
// word e of the copy of share x stands in the e / 128-th of the rounds of 128 keys that x owns.
constexpr int SC_ROUND = SC_WAVES * SC_TILE;

template <bool TILES>
__host__ __device__ __forceinline__ bool parts_fit(int n, int shares, int R)
{
    const int words = 2 * R * shares;
    if (TILES) return words <= n - (n + SC_TILE - 1) / SC_TILE;
    return shares * ((words + SC_ROUND - 1) / SC_ROUND) * SC_ROUND <= n;
}

// The shares of a segment of n rows, `most` if their parts fit.  One: it leaves no parts, and its first workgroup does all
// of it in the first launch.
template <bool TILES>
__host__ __device__ __forceinline__ int shares_of(int n, int most, int R)
{
    const int rounds = TILES ? (n + SC_ROUND - 1) / SC_ROUND : n / SC_ROUND;      // (each share has a round)
    int shares = most < rounds ? most : rounds;
    while (shares > 1 && !parts_fit<TILES>(n, shares, R)) --shares;
    return shares > 1 ? shares : 1;
}

template <bool TILES>
__device__ __forceinline__ int part_at(int n, int shares, int reader, int word)
{
    if (TILES) return (n + SC_TILE - 1) / SC_TILE + word;
    return (word / SC_ROUND * shares + reader) * SC_ROUND + word % SC_ROUND;
}

// Up to three query tiles the kernel fits 168 registers per thread without spilling, i.e. three waves per SIMD
// (three workgroups per CU) instead of the two the compiler settles for by itself; with four tiles it does not.
// MODE: the normalisers are given (lse), one pass; both passes; or the two passes as launches of their own, which the
// workgroups of a segment share: the first leaves every share's maximum and sum of each query row, the second merges them;
// segments of one share are done by the first alone.
// TILES: `block` is a multiple of a tile, and a tile leaves one value (their own kernels: the choice at run time costs the
// others four registers and with them a workgroup per CU).
enum { SCORE_GIVEN, SCORE_BOTH, SCORE_FIRST, SCORE_SECOND };

template <int D, int QT, int MODE, bool TILES, int WAVES = SC_WAVES>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(WAVES == SC_WAVES && QT <= 3 ? 3 : 2)))
void score_keys_kernel(ScoreArgs a)
{
    constexpr bool GIVEN = MODE == SCORE_GIVEN, FIRST = MODE == SCORE_FIRST, SECOND = MODE == SCORE_SECOND;
    constexpr int ROW_BYTES = D * 2;
    constexpr int KCH = D / 32;
    constexpr int LROW = ROW_BYTES + 16;
    constexpr int K_LOADS = SC_TILE * ROW_BYTES / (64 * 16);
    constexpr int K_PIECES = ROW_BYTES / 16;
    constexpr int K_ROWS_PER_LOAD = 64 / K_PIECES;
    constexpr int WAVE_LDS = SC_TILE * LROW;

    __shared__ __align__(16) unsigned char lds[WAVES * WAVE_LDS];
    __shared__ float red_m[WAVES][QT * 16];
    __shared__ float red_l[WAVES][QT * 16];
    __shared__ float fin_m[QT * 16];
    __shared__ float fin_il[QT * 16];

    const int lane = lane_id(), wv = wave_id();
    const int li = lane & 15, kg = lane >> 4;
    // Workgroup -> (segment, share): the first shares of all segments come first.  Tile t of a segment belongs to wave
    // t % WAVES of share (t / WAVES) % shares.
    const int share = (int)(blockIdx.x / a.nseg);
    const int seg = a.seg0 + (int)(blockIdx.x - share * a.nseg);
    const int first_tile = share * WAVES;
    const int G = a.G, w = a.w, R = w * G;
    if (GIVEN && share > 0 && a.share_rows > 0 && a.len[seg] < a.share_rows) return;   // nothing to share
    // Asked for first, none of it waits for the length: the query operands -- row r = qt*16 + li  ->  (recent query
    // j = r / G, head g = r % G) -- and the normaliser of row threadIdx.x.
    const int h = seg % a.Hkv;
    const int lb = seg / a.Hkv - a.lb0;
    const int Hq = a.Hkv * G;
    bf16x8 qop[QT][KCH];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        const int r = qt * 16 + li;
        const int j = r / G, g = r - j * G;
        const bool ok = r < R;
        const unsigned char *qrow = a.q + (((size_t)lb * w + j) * Hq + (size_t)h * G + g) * ROW_BYTES;
#pragma unroll
        for (int c = 0; c < KCH; ++c) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (ok) v = *reinterpret_cast<const u32x4 *>(qrow + c * 64 + kg * 16);
            qop[qt][c] = __builtin_bit_cast(bf16x8, v);
        }
    }
    float given = -INFINITY;
    if constexpr (GIVEN) {
        if ((int)threadIdx.x < R) {
            const int j = threadIdx.x / G, g = threadIdx.x - j * G;
            given = a.lse[((size_t)lb * w + j) * Hq + (size_t)h * G + g] * 1.4426950408889634f;
        }
    }
    int n = a.len[seg];
    if (n < 0 || n > a.cap) {
        if (!SECOND && threadIdx.x == 0 && share == 0) atomicAdd(&a.status[NGC_STATUS_LEN_CLAMPED], 1);
        n = n < 0 ? 0 : a.cap;
    }
    const int shares = FIRST || SECOND ? shares_of<TILES>(n, a.S, R) : n < a.share_rows ? 1 : a.S;
    if (SECOND && shares == 1) return;
    const int tile_step = shares * WAVES;
    if (share >= shares || first_tile * SC_TILE >= n) return;
    const unsigned char *kseg = a.table ? a.k : a.k + (size_t)seg * a.cap * ROW_BYTES;
    const int32_t *tab = a.table ? a.table + (size_t)seg * a.max_pages : nullptr;
    float *psi = a.psi_out + (size_t)seg * a.cap;
    const int tiles = (n + SC_TILE - 1) / SC_TILE;
    const int last_row = n - 1;

    unsigned char *wlds = lds + wv * WAVE_LDS;
    u32x4 kbuf[K_LOADS];
    // Unconditional: a tile past the end re-reads the last tile, so that the number of loads in flight is
    // the same on every path and the wait for the current tile never also waits for the prefetch.
    auto load_tile = [&](int tile_raw) {
        const int tile = tile_raw < tiles ? tile_raw : tiles - 1;
        const int row0 = tile * SC_TILE;
        const unsigned char *kt = kseg;
        int first = 0;   // row number at offset 0 of kt
        if (tab) {       // a tile lies inside one page
            int page = tab[tile >> a.tpp_shift];
            page = (page < 0 || page >= a.num_pages) ? 0 : page;
            kt = kseg + (((size_t)page << a.tpp_shift) + (size_t)(tile & ((1 << a.tpp_shift) - 1))) *
                            (SC_TILE * ROW_BYTES);
            first = row0;
        }
#pragma unroll
        for (int r = 0; r < K_LOADS; ++r) {
            int row = row0 + r * K_ROWS_PER_LOAD + lane / K_PIECES;
            row = row < last_row ? row : last_row;
            kbuf[r] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4 *>(kt + (size_t)(row - first) * ROW_BYTES + (lane % K_PIECES) * 16));
        }
    };
    auto stage_tile = [&]() {
#pragma unroll
        for (int r = 0; r < K_LOADS; ++r) {
            const int rl = r * K_ROWS_PER_LOAD + lane / K_PIECES;
            *reinterpret_cast<u32x4 *>(wlds + rl * LROW + (lane % K_PIECES) * 16) = kbuf[r];
        }
    };

    // The first tile before the normalisers are there, except with one query tile, where the launches that are resident at
    // once (up to 512 segments) got slower for it: 400 segments of 2150-3789 keys 52.0 -> 55.0 us, 512 63.8 -> 65.6; with two
    // tiles 512 68.7 -> 67.9, 300 51.9 -> 49.9.
    constexpr bool ASK_EARLY = (GIVEN && QT > 1) || SECOND;
    if constexpr (ASK_EARLY) load_tile(first_tile + wv);
    // ------------------------------------------------ pass 1: max and sum ---
    // (skipped when the caller hands over the log-sum-exp that decode attention
    // already computed for these very queries: then K is read only once)
    if constexpr (GIVEN) {
        static_assert(QT * 16 <= WAVES * 64, "a thread per query row");
        if (threadIdx.x < QT * 16) fin_m[threadIdx.x] = given;
        __syncthreads();
    } else if constexpr (SECOND) {
        // four threads a row, each with every fourth share
        static_assert(WAVES == 4 && QT <= 4, "up to 64 query rows");
        const int r = threadIdx.x >> 2;
        float M = -INFINITY, L = 0.f;
        if (r < R) {
            f32x2 own[MOST_SHARES / 4];
#pragma unroll
            for (int i = 0; i < MOST_SHARES / 4; ++i) {
                const int x = 4 * i + (threadIdx.x & 3);
                own[i] = f32x2{-INFINITY, 0.f};
                if (x < shares) {
                    const float *part = psi + part_at<TILES>(n, shares, share, 2 * (x * R + r));
                    own[i] = f32x2{part[0], part[1]};
                }
            }
#pragma unroll
            for (int i = 0; i < MOST_SHARES / 4; ++i) M = fmaxf(M, own[i][0]);
            M = lanes_reduce<4>(M, OpMaxF{});
#pragma unroll
            for (int i = 0; i < MOST_SHARES / 4; ++i) L += own[i][0] == -INFINITY ? 0.f : own[i][1] * fast_exp2(own[i][0] - M);
            L = lanes_reduce<4>(L, OpAdd{});
        }
        if ((threadIdx.x & 3) == 0 && r < QT * 16) {
            fin_m[r] = M;
            fin_il[r] = (L > 0.f) ? 1.0f / L : 0.f;
        }
        __syncthreads();
    } else {
    float m_run[QT], l_run[QT];
    int vis_q[QT];   // number of rows the query row of this lane can see
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        m_run[qt] = -INFINITY;
        l_run[qt] = 0.f;
        const int r = qt * 16 + li, j = r / G;
        int vis = a.causal ? (n - w + j + 1) : n;
        vis = vis > n ? n : vis;
        vis_q[qt] = r < R && vis > 0 ? vis : 0;
    }
    {
        const int step = FIRST ? tile_step : WAVES;
        int tile = FIRST ? first_tile + wv : wv;
        load_tile(tile);
        for (; tile < tiles; tile += step) {
            stage_tile();
            const int row0 = tile * SC_TILE;
            load_tile(tile + step);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_wave_barrier();
            bf16x8 kop[2][KCH];
#pragma unroll
            for (int mt = 0; mt < 2; ++mt)
#pragma unroll
                for (int c = 0; c < KCH; ++c)
                    kop[mt][c] = __builtin_bit_cast(
                        bf16x8, *reinterpret_cast<const u32x4 *>(wlds + (mt * 16 + li) * LROW + c * 64 + kg * 16));
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int qt = 0; qt < QT; ++qt) {
                f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < KCH; ++c) {
                    s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[0][c], qop[qt][c], s0, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[1][c], qop[qt][c], s1, 0, 0, 0);
                }
                // lane (q = li, kg): keys row0 + 4kg + r (s0) and row0 + 16 + 4kg + r (s1)
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int t = row0 + ((e < 4) ? (4 * kg + e) : (16 + 4 * kg + e - 4));
                    const float sc = (e < 4) ? s0[e] : s1[e - 4];
                    x[e] = (t < vis_q[qt]) ? sc * a.scale_log2e : -INFINITY;
                }
                float tmax = x[0];
#pragma unroll
                for (int e = 1; e < 8; ++e) tmax = fmaxf(tmax, x[e]);
                tmax = quad_rows_max(tmax);
                const float m_new = fmaxf(m_run[qt], tmax);
                if (m_new > -INFINITY) {
                    float psum = 0.f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) psum += fast_exp2(x[e] - m_new);
                    l_run[qt] = l_run[qt] * fast_exp2(m_run[qt] - m_new) + psum;
                    m_run[qt] = m_new;
                }
            }
        }
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
        float l = l_run[qt];
        l = quad_rows_sum(l);
        if (kg == 0) { red_m[wv][qt * 16 + li] = m_run[qt]; red_l[wv][qt * 16 + li] = l; }
    }
    __syncthreads();
    for (int r = threadIdx.x; r < QT * 16; r += WAVES * 64) {
        float M = red_m[0][r];
#pragma unroll
        for (int x = 1; x < WAVES; ++x) M = fmaxf(M, red_m[x][r]);
        float L = 0.f;
#pragma unroll
        for (int x = 0; x < WAVES; ++x) {
            const float mw = red_m[x][r];
            L += (mw == -INFINITY) ? 0.f : red_l[x][r] * fast_exp2(mw - M);
        }
        if constexpr (FIRST) {
            if (shares > 1 && r < R)
                for (int x = 0; x < (TILES ? 1 : shares); ++x) {
                    float *part = psi + part_at<TILES>(n, shares, x, 2 * (share * R + r));
                    part[0] = M;
                    part[1] = L;
                }
        }
        fin_m[r] = M;
        fin_il[r] = (L > 0.f) ? 1.0f / L : 0.f;
    }
    if (FIRST && shares > 1) return;
    __syncthreads();
    }

    // ------------------------------------- pass 2: probabilities per key ---
    // lane (key = li, kg) holds query rows qt*16 + 4kg + r
    float m_row[QT][4], il_row[QT][4];
    int vis_row[QT][4];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = qt * 16 + 4 * kg + r;
            m_row[qt][r] = fin_m[row];
            if constexpr (!GIVEN) il_row[qt][r] = fin_il[row];
            const int j = row / G;
            int vis = a.causal ? (n - w + j + 1) : n;
            vis = vis > n ? n : vis;
            vis_row[qt][r] = (row < R && vis > 0) ? vis : 0;
        }
    const float inv_rows = 1.0f / (float)R;
    {
        int tile = first_tile + wv;
        if constexpr (!ASK_EARLY) load_tile(tile);
        for (; tile < tiles; tile += tile_step) {
            stage_tile();
            const int row0 = tile * SC_TILE;
            load_tile(tile + tile_step);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_wave_barrier();
            bf16x8 kop[2][KCH];
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int c = 0; c < KCH; ++c)
                    kop[nt][c] = __builtin_bit_cast(
                        bf16x8, *reinterpret_cast<const u32x4 *>(wlds + (nt * 16 + li) * LROW + c * 64 + kg * 16));
            __builtin_amdgcn_wave_barrier();
            float tile_sum = 0.f;
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int t = row0 + nt * 16 + li;   // the key of this lane
                float acc = 0.f;
#pragma unroll
                for (int qt = 0; qt < QT; ++qt) {
                    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int c = 0; c < KCH; ++c)
                        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qop[qt][c], kop[nt][c], s, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float p = fast_exp2(s[r] * a.scale_log2e - m_row[qt][r]);
                        if constexpr (!GIVEN) p *= il_row[qt][r];
                        if (t < vis_row[qt][r]) acc += p;
                    }
                }
                acc = quad_rows_sum(acc);
                if constexpr (TILES) tile_sum += t < n ? acc : 0.f;
                else if (kg == 0 && t < n) psi[t] = acc * inv_rows;
            }
            if constexpr (TILES) {
                tile_sum = lanes_reduce<16>(tile_sum, OpAdd{}) * inv_rows;
                if (a.block == SC_TILE) tile_sum /= (float)(n - row0 < SC_TILE ? n - row0 : SC_TILE);
                if (lane == 0) psi[tile] = tile_sum;
            }
        }
    }
}

// Block means and head pooling, in place over the per-key scores or the tiles' sums: item j of a segment becomes the mean
// over its rows; with pooling, the mean of that over the KV heads of the (layer, sequence) that have item j.
//
// Where an item's mean already stands at its own offset -- blocks of one tile, or of one key -- only the pooling is left, and
// every item of a (layer, sequence) is a thread's of its own, wherever it runs: pool_heads_kernel.  Before, a thread made the
// mean of 32 keys from memory, one after another, and one workgroup per (layer, sequence) went through all its items.
// Microseconds, before and now (normalisers given but in the last):
//     blocks of 32, pooled: 48 x 4 segments of 416 keys 20.0 and 11.6, 35 x 2 of 1692 at D = 64 13.6 and 8.5, 16 x 2 of 8000
//     23.7 and 14.6, 512 x 4 of 3000 290 and 238; not pooled: 3472 x 4 of 333 259 and 200, 512 x 2 of 3000 at D = 64 83 and 60;
//     blocks of 64, pooled: 40 x 2 of 3000 25.3 and 14.4; pooled per key: 128 x 8 of 2000 121 and 97; two passes: blocks of 32,
//     pooled, 20 x 8 of 447 31.6 and 13.1
//
// Otherwise (score_reduce_kernel) one workgroup per (layer, sequence); items are processed in ascending tiles and an item
// only reads values at or beyond its own index, so reading a tile, waiting, then writing it never clobbers what a later tile
// still reads.
struct ReduceArgs {
    float *scores;      // [lb][Hkv][cap]
    const int32_t *len;
    int lb0_seg;        // first (layer*B + sequence) of the launch
    int Hkv, cap, block, pool;
};

// UNIT: rows per value, 1, or SC_TILE where the tiles' sums are reduced.  (As an argument it is a division per value: blocks of
// 48, pooled, 64 x 4 segments of 1000 keys 30.6 -> 39.7 us in all.)
template <int UNIT>
__global__ __launch_bounds__(256) void score_reduce_kernel(ReduceArgs a)
{
    const int lb = a.lb0_seg + blockIdx.x;
    const int Hkv = a.Hkv, block = a.block;
    int max_items = 0;
    for (int h = 0; h < Hkv; ++h) {
        int n = a.len[lb * Hkv + h];
        n = n < 0 ? 0 : (n > a.cap ? a.cap : n);
        const int N = (n + block - 1) / block;
        max_items = N > max_items ? N : max_items;
    }
    float *base = a.scores + (size_t)lb * Hkv * a.cap;
    auto rows_of = [&](int h) {
        int n = a.len[lb * Hkv + h];
        return n < 0 ? 0 : (n > a.cap ? a.cap : n);
    };
    auto block_mean = [&](int h, int j, int n) {
        const int lo = j * block;
        const int hi = (lo + block < n) ? lo + block : n;
        float acc = 0.f;
        for (int t = lo; t < hi; t += UNIT) acc += base[(size_t)h * a.cap + t / UNIT];
        return acc / (float)(hi - lo);
    };
    for (int tile = 0; tile < max_items; tile += 256) {
        const int j = tile + threadIdx.x;
        if (a.pool) {
            float pooled = 0.f;
            int heads = 0;
            for (int h = 0; h < Hkv; ++h) {
                const int n = rows_of(h);
                if (j * block < n) { pooled += block_mean(h, j, n); ++heads; }
            }
            __syncthreads();
            for (int h = 0; h < Hkv; ++h)
                if (j * block < rows_of(h)) base[(size_t)h * a.cap + j] = pooled / (float)heads;
            __syncthreads();
        } else {
            for (int h = 0; h < Hkv; ++h) {
                const int n = rows_of(h);
                const bool have = j * block < n;
                const float v = have ? block_mean(h, j, n) : 0.f;
                __syncthreads();
                if (have) base[(size_t)h * a.cap + j] = v;
                __syncthreads();
            }
        }
    }
}

__global__ __launch_bounds__(256) void pool_heads_kernel(ReduceArgs a)
{
    const int lb = a.lb0_seg + blockIdx.x;
    float *base = a.scores + (size_t)lb * a.Hkv * a.cap;
    int longest = 0;
    for (int h = 0; h < a.Hkv; ++h) {
        const int n = a.len[lb * a.Hkv + h];
        longest = n > longest ? n : longest;
    }
    longest = longest < a.cap ? longest : a.cap;
    const int items = (longest + a.block - 1) / a.block;
    for (int j = (int)(blockIdx.y * 256 + threadIdx.x); j < items; j += (int)gridDim.y * 256) {
        auto has_item = [&](int h) {
            int n = a.len[lb * a.Hkv + h];
            n = n > a.cap ? a.cap : n;
            return j * a.block < n;
        };
        float pooled = 0.f;
        int heads = 0;
#pragma unroll 4
        for (int h = 0; h < a.Hkv; ++h)
            if (has_item(h)) { pooled += base[(size_t)h * a.cap + j]; ++heads; }
        pooled /= (float)heads;
#pragma unroll 4
        for (int h = 0; h < a.Hkv; ++h)
            if (has_item(h)) base[(size_t)h * a.cap + j] = pooled;
    }
}

}  // namespace ngc

using namespace ngc;

namespace {
// Workgroups per segment.  With the normalisers given, a key's score needs nothing from the other keys, so a segment can be
// shared freely.  Microseconds against the number S of workgroups per segment (D = 128, w = 5, 6 heads per KV head):
//     segments x keys     S=1     2     4     8    16    32
//         8 x 2000       17.6  10.8   7.5   6.5   5.8   5.9
//         8 x 8000       55.7  30.7  17.7  11.1   7.9   6.4
//        32 x 8000       74.8  40.3  23.5  15.7  13.7  16.6
//       128 x 2000       23.8  16.1  13.7  16.5  19.1  19.2
//       128 x 8000       85.2  52.5  46.2  48.8  49.3  52.5
//       400 x 2000       38.7  43.6  41.7  43.7  54.6  54.4
//      2048 x 2150-3789   284   282   294   327   382   470
// i.e. about two workgroups per CU, four at D = 64 (512 x 2000-6000: 64.9, 55.7 with two each).  Just beyond that, up to 640
// segments at D = 128, a second workgroup evens out what the last ones leave idle, if the segments are long (S = 1 -> 2:
// 520 x 2150-3789 78.5 -> 72.4, 640 x 2150-3789 92.7 -> 89.0; 768 x 4096 136 -> 138, 1536 x 4096 273 -> 279; at D = 64
// 640 x 2150-3789 45.5 -> 43.0, but 520 x 100-300 in a capacity of 2500 4.9 -> 5.2: not there).  The host does not know the
// lengths, so it launches the second one where the capacity permits; if the segment has fewer than SHARE_ROWS rows that
// leaves before it asks for anything else (640 x 100-300 in a capacity of 4096 9.8, 10.4 before there was one).
constexpr int SHARE_ROWS = 2048;

struct Shares {
    int S, rows;
};

Shares score_shares(int nseg, int cap, int D, bool have_lse)
{
    if (!have_lse) return {1, 0};
    const int rounds = (cap + SC_TILE * SC_WAVES - 1) / (SC_TILE * SC_WAVES);
    const int fill = (D == 128 ? 512 : 1024) / nseg;
    if (D == 128 && nseg > 512 && nseg <= 640 && cap >= SHARE_ROWS) return {2, SHARE_ROWS};
    const int s = rounds < fill ? rounds : fill;
    return {s > 1 ? s : 1, 0};
}

// Workgroups per segment where the normalisers are not given: the two passes as two launches, two workgroups per CU in all,
// where the capacity has room for the parts of four shares or more and is PASSES_ROWS or more; otherwise, up to a workgroup
// per CU, one with eight waves.  Microseconds (D = 128, 6 heads per KV head, w = 3) of one workgroup of four waves, of
// eight, and of two launches, lengths of the capacity:
//     segments     512           1024              2048              3000              8000 keys
//            8  10.7  9.1    17.5 13.8 10.0    30.7 22.4 12.1    45.0 32.6 14.4     119   84  17.6
//           32  10.9  9.4    17.7 14.0 10.6    35.3 26.7 14.4    50.7 37.0 16.8     127   89  25.1
//           64  12.3 10.5    18.5 14.9 11.1    35.9 26.9 16.6    52.3 38.2 20.4     131   93  44.6
//          128  12.9 11.1    20.8 16.8 15.6    38.1 29.1 24.8    55.9 42.0 34.6     139  102  85.7
//          160  13.1 11.2                      4096: 74.9 57.0;  256: 85.2 78.8;  512 x 3000 120 122
// The host does not know the lengths.  Far below the capacity the second launch only costs, 100 keys in 4096: 8 segments 5.6
// and 7.4, 64 5.7 and 8.6; 300 in 2048: 8.9, 8.0 (eight waves) and 11.0; 512 in 1024: 64 segments 10.7, 9.4 and 10.1, 128 11.6,
// 10.3 and 11.9.  So the capacities are those from which half of them still gains, and eight waves start beyond the rows that
// four have a tile or two each for (256 keys: 7.3 and 7.1, 100 keys 5.6 and 6.2).  (16 waves spill with two query tiles.)
constexpr int MORE_WAVES_SEGMENTS = 256;
constexpr int MORE_WAVES_ROWS = 2 * SC_ROUND;        // (more than so many)
constexpr int PASSES_ROWS = 1024;                    // ... up to 64 segments, twice that beyond

int passes_shares(int nseg, int cap, int R, bool tiles)
{
    if (cap < (nseg <= 64 ? PASSES_ROWS : 2 * PASSES_ROWS)) return 1;
    int S = 512 / nseg;
    if (S > MOST_SHARES) S = MOST_SHARES;
    S = tiles ? shares_of<true>(cap, S, R) : shares_of<false>(cap, S, R);
    return S >= 4 ? S : 1;
}

// Workgroups that pool heads: enough for every CU, then more items each.  One per 256 items of the capacity costs as much as the
// scores where the segments are short: per key, 448 x 2 segments, capacity 4000, us of one workgroup per sequence, of one per
// 256 items and of 2048: 60 keys 10.6, 17.2 and 10.4, 1000 50.4, 53.6 and 48.3, 4000 189, 179 and 178; 256 x 4, capacity
// 8000, 60 keys 11.5, 20.1 and 11.2, 2000 115, 109 and 102 (1024 and 4096 the same within 1 %).
constexpr int POOL_WORKGROUPS = 2048;

int launch_score(const ngc_cache *c, const ngc_paged_cache *pc, int32_t layer, const void *q_recent,
                 const float *lse_recent, int32_t w, float scale, uint32_t flags, int32_t block,
                 float *scores_out, void *ws, size_t ws_bytes, void *stream)
{
    if (!c->k || !c->len || !q_recent || !scores_out || !ws) return NGC_EINVAL;
    if ((reinterpret_cast<uintptr_t>(c->k) | reinterpret_cast<uintptr_t>(q_recent)) & 15u) return NGC_EINVAL;
    if (c->L <= 0 || c->B <= 0 || c->Hkv <= 0 || c->Hq <= 0 || c->cap <= 0) return NGC_EINVAL;
    if (c->D != 64 && c->D != 128) return NGC_EINVAL;
    if ((long long)c->cap * c->D * 2 > 0x7FFFFFFFLL) return NGC_EUNSUPPORTED;   // 32-bit byte offsets inside a segment
    if (c->Hq % c->Hkv != 0 || w < 1 || block < 1 || !(scale == scale)) return NGC_EINVAL;
    if (layer < -1 || layer >= c->L) return NGC_EINVAL;
    if (ws_bytes < NGC_STATUS_WORDS * sizeof(int32_t)) return NGC_ENOSPC;
    if (lse_recent && (flags & NGC_SCORE_NO_CAUSAL)) return NGC_EINVAL;   // decode's lse is the causal one
    const int G = c->Hq / c->Hkv;
    const int R = w * G;
    if (R > 64) return NGC_EUNSUPPORTED;
    const bool pool = (flags & NGC_SCORE_POOL_HEADS) != 0;
    const int per_layer = c->B * c->Hkv;
    const int seg0 = layer < 0 ? 0 : layer * per_layer;
    const int nseg = layer < 0 ? c->L * per_layer : per_layer;

    ScoreArgs sa;
    sa.k = reinterpret_cast<const unsigned char *>(c->k);
    sa.len = c->len;
    sa.q = reinterpret_cast<const unsigned char *>(q_recent);
    sa.lse = lse_recent;
    sa.psi_out = scores_out;
    sa.status = reinterpret_cast<int32_t *>(ws);
    sa.seg0 = seg0; sa.nseg = nseg;
    Shares shares = score_shares(nseg, c->cap, c->D, lse_recent != nullptr);   // nseg * S <= max(nseg, 1280)
    const bool tiles = block % SC_TILE == 0;
    if (!lse_recent) shares = {passes_shares(nseg, c->cap, R, tiles), 0};
    const bool two_passes = !lse_recent && shares.S > 1;
    const bool more_waves = !lse_recent && !two_passes && nseg <= MORE_WAVES_SEGMENTS && c->cap > MORE_WAVES_ROWS;
    sa.S = shares.S;
    sa.share_rows = shares.rows;
    sa.lb0 = layer < 0 ? 0 : layer * c->B;
    sa.w = w; sa.G = G; sa.Hkv = c->Hkv; sa.cap = c->cap;
    sa.causal = (flags & NGC_SCORE_NO_CAUSAL) ? 0 : 1;
    sa.block = block;
    sa.scale_log2e = scale * 1.4426950408889634f;
    sa.table = nullptr; sa.max_pages = 0; sa.num_pages = 0; sa.tpp_shift = 0;
    if (pc) {
        sa.table = pc->table; sa.max_pages = pc->max_pages; sa.num_pages = pc->num_pages;
        int tpp = pc->page_rows / SC_TILE, sh = 0;
        while ((1 << sh) < tpp) ++sh;
        sa.tpp_shift = sh;
    }
    hipStream_t st = (hipStream_t)stream;
    const int qt = (R + 15) / 16;
#define NGC_PICK_QT(DD, ...) \
    (qt == 1   ? reinterpret_cast<const void *>(&score_keys_kernel<DD, 1, __VA_ARGS__>) \
     : qt == 2 ? reinterpret_cast<const void *>(&score_keys_kernel<DD, 2, __VA_ARGS__>) \
     : qt == 3 ? reinterpret_cast<const void *>(&score_keys_kernel<DD, 3, __VA_ARGS__>) \
               : reinterpret_cast<const void *>(&score_keys_kernel<DD, 4, __VA_ARGS__>))
#define NGC_PICK_GIVEN(DD, TILES) \
    (lse_recent ? NGC_PICK_QT(DD, SCORE_GIVEN, TILES) \
     : two_passes ? NGC_PICK_QT(DD, SCORE_SECOND, TILES) \
     : more_waves ? NGC_PICK_QT(DD, SCORE_BOTH, TILES, 2 * SC_WAVES) : NGC_PICK_QT(DD, SCORE_BOTH, TILES))
    if (two_passes) {
        const void *first = c->D == 128 ? (tiles ? NGC_PICK_QT(128, SCORE_FIRST, true) : NGC_PICK_QT(128, SCORE_FIRST, false))
                                        : (tiles ? NGC_PICK_QT(64, SCORE_FIRST, true) : NGC_PICK_QT(64, SCORE_FIRST, false));
        const int rc = launch(first, dim3((unsigned)(nseg * sa.S)), dim3(SC_WAVES * 64), 0, st, sa);
        if (rc) return rc;
    }
    const void *fn = c->D == 128 ? (tiles ? NGC_PICK_GIVEN(128, true) : NGC_PICK_GIVEN(128, false))
                                 : (tiles ? NGC_PICK_GIVEN(64, true) : NGC_PICK_GIVEN(64, false));
#undef NGC_PICK_GIVEN
#undef NGC_PICK_QT
    // With two query tiles at D = 128 and the normalisers given four workgroups fit a CU.  Between 1024 and 1536 segments two
    // rounds of three are fuller than two of four: LDS that nobody uses keeps the fourth out (1536 x 1366-1800 keys 110 -> 107.5
    // us, 1030 77.4 -> 75.8; with four 1024 x 2150-3789 147 -> 139, 896 x 700 30.2 -> 29.0).
    const size_t keep_out = c->D == 128 && qt == 2 && lse_recent && nseg > 1024 && nseg <= 1536 ? 8192 : 0;
    const int rc = launch(fn, dim3((unsigned)(nseg * sa.S)), dim3((more_waves ? 2 : 1) * SC_WAVES * 64), keep_out, st, sa);
    if (rc) return rc;
    // scores_out is indexed by the global segment; what follows gets the global base
    const int sequences = nseg / c->Hkv;
    ReduceArgs ra{scores_out, c->len, seg0 / c->Hkv, c->Hkv, c->cap, block, pool ? 1 : 0};
    const bool whole = block == 1 || block == SC_TILE;       // an item's mean stands at its offset
    if (whole && pool) {
        const int columns = ((c->cap + block - 1) / block + 255) / 256;
        const int most = (POOL_WORKGROUPS + sequences - 1) / sequences;
        return launch(reinterpret_cast<const void *>(&pool_heads_kernel),
                      dim3((unsigned)sequences, (unsigned)(columns < most ? columns : most)), dim3(256), 0, st, ra);
    }
    if (!whole)
        return launch(tiles ? reinterpret_cast<const void *>(&score_reduce_kernel<SC_TILE>)
                            : reinterpret_cast<const void *>(&score_reduce_kernel<1>),
                      dim3((unsigned)sequences), dim3(256), 0, st, ra);
    return NGC_OK;
}
}  // namespace

extern "C" int ngc_score_keys(const ngc_cache *c, int32_t layer, const void *q_recent,
                              const float *lse_recent, int32_t w,
                              float scale, uint32_t flags, int32_t block, float *scores_out,
                              void *ws, size_t ws_bytes, void *stream)
{
    if (!c) return NGC_EINVAL;
    return launch_score(c, nullptr, layer, q_recent, lse_recent, w, scale, flags, block, scores_out,
                        ws, ws_bytes, stream);
}

extern "C" int ngc_paged_score_keys(const ngc_paged_cache *pc, int32_t layer, const void *q_recent,
                                    const float *lse_recent, int32_t w,
                                    float scale, uint32_t flags, int32_t block, float *scores_out,
                                    void *ws, size_t ws_bytes, void *stream)
{
    if (!pc || !pc->table) return NGC_EINVAL;
    if (pc->page_rows < SC_TILE || (pc->page_rows & (pc->page_rows - 1)) != 0) return NGC_EINVAL;
    if (pc->max_pages <= 0 || pc->num_pages <= 0) return NGC_EINVAL;
    if ((long long)pc->max_pages * pc->page_rows > 0x7FFFFFFFLL / 256) return NGC_EUNSUPPORTED;
    ngc_cache c{};
    c.k = pc->k_pool; c.v = pc->v_pool; c.len = pc->len; c.pos = nullptr;
    c.L = pc->L; c.B = pc->B; c.Hkv = pc->Hkv; c.Hq = pc->Hq; c.D = pc->D;
    c.cap = pc->max_pages * pc->page_rows;
    return launch_score(&c, pc, layer, q_recent, lse_recent, w, scale, flags, block, scores_out,
                        ws, ws_bytes, stream);
}
