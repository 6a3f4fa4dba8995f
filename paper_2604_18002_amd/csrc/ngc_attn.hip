// Decode attention over the surviving (compacted, ragged) cache rows on gfx950.
//
// One query token per sequence; every KV head serves G = Hq / Hkv query heads.
// The work is memory bound (each K and V row is read once and used by G
// queries), so the kernel is built around full-row 16-byte loads and keeps the
// vector ALU free by running both contractions on the matrix cores with the G
// query heads padded to a 16-wide tile:
//
//   S^T[row][q] = sum_d K[row][d] Q[q][d]     mfma 16x16x32 bf16, A = K rows
//   O^T[d][q]   = sum_row V[row][d] P[q][row] mfma 16x16x32 bf16, A = V^T
//
// Both products put the query head on the lane index (lane % 16), so all
// soft-max state (running max, running sum, rescale factor) is lane local.
//
// Data movement per 32-row tile and wave:
//   K: 8 (D=128) loads of 16 B per lane, one full row per 16 lanes -> wave
//      private LDS -> read back in the A-operand layout.
//   V: loaded straight into the registers that feed the second product.  Lane
//      (i, kg) loads, for each of the 8 rows that its lane group kg contracts
//      over, the 16 B holding d = 8i .. 8i+7; eight 2x2 16-bit transposes turn
//      them into the eight A operands for the d-tiles {8i + c}.  No LDS.
//   K and V rows are read exactly once, so their loads carry the nontemporal
//      hint (measured on MI355X: 7.1 TB/s streaming reads with it, 6.35 without).
//   P is split into a bf16 head and a bf16 remainder (two MFMAs) so the second
//      product is accurate to ~2^-16 relative, not bf16's 2^-8.
//
// Long segments are split over several workgroups (flash-decode); each writes
// an unnormalised partial (max, sum, O) and takes a ticket of its segment; the
// workgroup that takes the last ticket merges the partials.  One launch per
// call.  The partials and tickets cross workgroups (and the L2 caches of
// different XCDs) through device-scope stores and loads, which go to memory
// (16-byte buffer accesses for the O rows, relaxed atomics for the rest); the
// only wait is each writer's own wait for its stores before the workgroup's
// ticket -- no cache-wide write-back or invalidate is involved.
//
// The same kernel can first append the new token's K/V row (Sec. 4.1: the cache
// grows by one entry per token): every wave requests the new row together with
// its first tile; the wave that owns the last tile stores it into the cache and
// puts it in its place in that tile's operands, so no load waits for the store.
// The length is stored by whichever workgroup of the segment finishes last,
// after every other one has read it.
//
// Which tiles a wave works on does not depend on the segment's length (tile t
// belongs to wave t % 4 of workgroup (t / 4) % S), so in small launches and in
// those over long segments the first tile is requested before the length has
// arrived (first_tile_early() has the rule and its figures).  Rows at or beyond
// the length are switched off when their tile is computed (their scores by the
// mask, their V values by zeros: what lies there is unspecified and may be NaN).
//
// What bounds a launch: at a few segments the chain of memory round trips (first
// tile; then, if a segment is shared, partial -> ticket -> merge), at several
// hundred the read rate of the memory.  Per layer, from a HIP graph, before ->
// after the tiles were interleaved over the workgroups, the partials came in one
// batch, the last tile lost its prefetch and the first was asked for early:
// 2 segments x 2000 rows 8.2 -> 6.7 us, 32 x 525 rows (8.6 MB) 9.1 -> 7.0 us,
// 128 x 1494 rows (98 MB) 22.0 -> 19.7 us, 512 x 2700 rows (0.71 GB) 119 -> 117 us.
// Where the 5.75 us of 32 x 525 rows go (copies of the kernel that return early): launch 1.8, until the first
// tile is there 1.7, its products 0.4, the four waves' merge 0.3, partial stores until acknowledged 0.45, ticket 0.5
// (1.2 with the tickets of all segments on one cache line), merge 0.65.
//
// Paged layout (PAGED = true): a 32-row tile never straddles a page (pages hold
// a power-of-two number of rows >= 32), so only the tile's base address changes:
// it comes from the segment's page table.  Table entries are fetched two tiles
// ahead of their use so that the lookup never sits in front of the K/V loads.
#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "../../include/ngc.h"
#include "ngc_device.h"

namespace ngc {

constexpr int ATT_WAVES = 4;
constexpr int ATT_TILE = 32;   // rows per wave step
constexpr int MAX_SPLITS = 64;  // workgroups per segment at most

struct AttnArgs {
    const unsigned char *k;
    const unsigned char *v;
    const int32_t *len;
    const unsigned char *q;
    float *out;
    float *lse_out;   // optional: log-sum-exp of the scaled scores per query head, natural log
    float *part_o;    // [nseg_launch][S][G][D]
    float *part_ml;   // [nseg_launch][S][G][2]
    int32_t *status;
    int seg0;         // first segment of the launch
    int S;            // splits per segment
    int G, Hkv, cap;
    float scale_log2e;
    // paged layout only: k, v are the pools
    const int32_t *table;   // [seg][max_pages]
    int max_pages;
    int num_pages;
    int tpp_shift;          // log2(tiles per page)
    int32_t *ticket;        // [segments of the launch][ticket_step] workgroups of a segment that are done (the first word of
    int ticket_step;        // each); 0 between launches
    // fused append (APPEND kernels only)
    unsigned char *k_rw;    // the cache again, writable
    unsigned char *v_rw;
    int32_t *len_rw;
    int32_t *pos;           // or nullptr
    const unsigned char *k_new;   // [launch segments][D] bf16
    const unsigned char *v_new;
    const int32_t *new_pos;       // [B] or nullptr
    int B;
};

// Loads and stores that other workgroups' data travels through: device scope (served by memory, not by an XCD's own
// L2), 16 bytes wide for the partial O rows (a wave's stores land as whole cache lines instead of one 4-byte
// write-through per lane): raw buffer accesses with the device-scope bit, bounds-checked by the hardware against
// `bytes` (a load past the end returns 0, a store past the end is dropped).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t device_span(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}
constexpr int AUX_DEVICE_SCOPE = 16;   // sc1
__device__ __forceinline__ void st_device16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, f32x4 v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, byte_off, 0, AUX_DEVICE_SCOPE);
}
__device__ __forceinline__ f32x4 ld_device16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off)
{
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, AUX_DEVICE_SCOPE));
}
__device__ __forceinline__ void st_device8(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, f32x2 v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, byte_off, 0, AUX_DEVICE_SCOPE);
}
__device__ __forceinline__ f32x2 ld_device8(__amdgpu_buffer_rsrc_t r, uint32_t byte_off)
{
    return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, AUX_DEVICE_SCOPE));
}

// EARLY: a wave's first tile is requested before the length has arrived (see first_tile_early()).
template <int D, bool PAGED, bool APPEND, bool EARLY>
__global__ __launch_bounds__(ATT_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
void decode_kernel(AttnArgs a)
{
    constexpr int ROW_BYTES = D * 2;
    constexpr int DPL = D / 16;                 // bf16 per lane in a V row (8 or 4)
    constexpr int KCH = D / 32;                 // 32-wide d chunks of the first product
    constexpr int LROW = ROW_BYTES + 16;        // padded LDS row
    constexpr int K_LOADS = ATT_TILE * ROW_BYTES / (64 * 16);   // 16-B loads per lane per K tile
    constexpr int K_PIECES = ROW_BYTES / 16;    // lanes per K row
    constexpr int K_ROWS_PER_LOAD = 64 / K_PIECES;
    constexpr int WAVE_LDS = ATT_TILE * LROW;

    __shared__ __align__(16) unsigned char lds[ATT_WAVES * WAVE_LDS];
    __shared__ float red_m[ATT_WAVES][16];
    __shared__ float red_l[ATT_WAVES][16];
    __shared__ int is_last;
    __shared__ __align__(16) unsigned char fresh[APPEND ? 2 * ROW_BYTES : 16];   // the new K row and V row

    const int lane = lane_id(), wv = wave_id();
    const int li = lane & 15, kg = lane >> 4;
    // Workgroup -> (segment, run): run-major, i.e. the first runs of all segments come first, then the second runs,
    // ...  Consecutive workgroups go round-robin to the 8 XCDs: this way every XCD gets the same share of each
    // run index (with the run as the fastest coordinate and S = 2, all first runs land on four of the XCDs and all
    // second runs on the other four: measured 15 % slower at 1024 segments of 16K rows).
    // (A grid of two dimensions counts the same way; divisions, here and for the queries, would stand in front of the
    // first load.)
    const int split = (int)blockIdx.y;
    const int seg_local = (int)blockIdx.x;
    const int seg = a.seg0 + seg_local;
    const int G = a.G;

    const int n_raw = a.len[seg];
    if constexpr (!EARLY) __builtin_amdgcn_sched_barrier(0);   // asked for before anything else: the tile waits for it
    float *out_seg = a.out + (size_t)seg_local * G * D;    // [G][D] of this KV head

    const unsigned char *kseg = PAGED ? a.k : a.k + (size_t)seg * a.cap * ROW_BYTES;
    const unsigned char *vseg = PAGED ? a.v : a.v + (size_t)seg * a.cap * ROW_BYTES;
    const int wv_u = __builtin_amdgcn_readfirstlane(wv);
    const int step = a.S * ATT_WAVES;                      // tiles between two of a wave's own
    int tile = split * ATT_WAVES + wv_u;
    // Byte offset of a tile from the start of the segment's rows or, paged, of the pools (a tile lies inside one
    // page).  `top`: the last tile that may be looked up, taken in place of later ones.
    const int32_t *tab = PAGED ? a.table + (size_t)seg * a.max_pages : nullptr;
    auto tile_base = [&](int t, int top) -> size_t {
        const int tc = t < top ? t : top;
        if constexpr (!PAGED) return (size_t)tc * (ATT_TILE * ROW_BYTES);
        int page = tab[tc >> a.tpp_shift];
        page = (page < 0 || page >= a.num_pages) ? 0 : page;   // never leave the pool
        return ((size_t)page << a.tpp_shift) * (ATT_TILE * ROW_BYTES) +
               (size_t)(tc & ((1 << a.tpp_shift) - 1)) * (ATT_TILE * ROW_BYTES);
    };

    // rows this lane loads, relative to the tile: K in full-row order, V in the
    // order its lane group contracts over (matches the layout of the scores)
    int vrow_rel[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) vrow_rel[e] = (e < 4) ? (4 * kg + e) : (16 + 4 * kg + (e - 4));

    // 32-bit byte offsets inside the segment (a segment is at most cap * ROW_BYTES <= 2^31 bytes)
    const uint32_t k_col = (uint32_t)(lane % K_PIECES) * 16u;
    const uint32_t v_col = (uint32_t)li * (DPL * 2);
    u32x4 kbuf[K_LOADS];
    auto load_v_piece = [&](const unsigned char *p) -> u32x4 {
        if constexpr (DPL == 8) {
            return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        } else {
            const u32x2 t = __builtin_nontemporal_load(reinterpret_cast<const u32x2 *>(p));
            return u32x4{t[0], t[1], 0u, 0u};
        }
    };
    // Loads of tile t, whose rows start `base` bytes into K and V; rows beyond `last_row` are not touched (the last one
    // is read in their place).
    auto issue_loads = [&](int t, int last_row, size_t base, u32x4 (&vb)[8]) {
        const unsigned char *kt = kseg + base, *vt = vseg + base;      // wave-uniform
        const int lim = last_row - t * ATT_TILE;
#pragma unroll
        for (int r = 0; r < K_LOADS; ++r) {
            int rel = r * K_ROWS_PER_LOAD + lane / K_PIECES;
            rel = rel < lim ? rel : lim;
            kbuf[r] = __builtin_nontemporal_load(
                reinterpret_cast<const u32x4 *>(kt + ((uint32_t)rel * ROW_BYTES + k_col)));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int rel = vrow_rel[e] < lim ? vrow_rel[e] : lim;
            vb[e] = load_v_piece(vt + ((uint32_t)rel * ROW_BYTES + v_col));
        }
    };

    // Everything that does not need the length is requested first: the queries, the new row and, in small launches and
    // those over long segments (EARLY), the first tile (its rows are clamped to the capacity only; paged: table entries
    // beyond the pages in use hold anything, which tile_base() turns into some page of the pool).
    u32x4 new_piece = {0u, 0u, 0u, 0u};      // lanes [0, K_PIECES) hold the new K row, the next K_PIECES the V row
    if constexpr (APPEND) {
        const unsigned char *src = (lane / K_PIECES) & 1 ? a.v_new : a.k_new;
        new_piece = *reinterpret_cast<const u32x4 *>(src + (size_t)seg_local * ROW_BYTES + k_col);
    }
    // B operand of the first product: Q[q = li][32c + 8kg .. +7], zero for q >= G
    bf16x8 qop[KCH];
    {
        const unsigned char *qrow = a.q + ((size_t)seg_local * G + (li < G ? li : G - 1)) * ROW_BYTES;
#pragma unroll
        for (int c = 0; c < KCH; ++c)
            qop[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(qrow + c * 64 + kg * 16));
    }
    u32x4 v_a[8], v_b[8];
    const int cap_tile = (a.cap - 1) / ATT_TILE;
    // Bases of the first tile and of the two after it.  Paged: looked up before they are needed, and without the length
    // (a page that turns out not to be in use is not read from): with all three lookups after it 28.9 -> 29.9 us at 896
    // segments of 350 rows.  (Small launches would rather have the first tile on its way than the others' bases.)
    const size_t base0 = tile_base(tile, cap_tile);
    size_t base1 = 0, base2 = 0;
    if constexpr (!EARLY) {
        base1 = tile_base(tile + step, cap_tile);
        base2 = tile_base(tile + 2 * step, cap_tile);
    }
    if constexpr (EARLY) {
        issue_loads(tile < cap_tile ? tile : cap_tile, a.cap - 1, base0, v_a);
        __asm__ volatile("" ::: "memory");   // the requests stay in front of everything that waits for the length
    }

    int n = n_raw;
    if (n < 0 || n > a.cap) {
        if (threadIdx.x == 0 && split == 0) atomicAdd(&a.status[NGC_STATUS_LEN_CLAMPED], 1);
        n = n < 0 ? 0 : a.cap;
    }
    // fused append: this call's row goes to slot n and takes part in the attention
    bool grew = false;
    if constexpr (APPEND) {
        if (n < a.cap) {
            grew = true;
            n += 1;
        } else if (threadIdx.x == 0 && split == 0) {
            atomicAdd(&a.status[NGC_STATUS_APPEND_FULL], 1);
        }
    }
    // Every workgroup of a split segment takes a ticket when it is done (right away if its split is empty); the
    // one that takes the last ticket returns true here, all others false.  Whole workgroup calls it.
    auto took_last_ticket = [&]() -> bool {
        __syncthreads();   // this workgroup's partial stores have been waited for by their threads
        if (threadIdx.x == 0) {
            const int old = __hip_atomic_fetch_add(&a.ticket[seg_local * a.ticket_step], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_last = (old == a.S - 1) ? 1 : 0;
        }
        __syncthreads();
        return is_last != 0;
    };
    // What the last workgroup of a segment does besides merging: the tickets return to 0 for the next launch and
    // the appended row becomes part of the segment.
    auto close_segment = [&]() {
        if (threadIdx.x == 0) {
            if (a.S > 1) __hip_atomic_store(&a.ticket[seg_local * a.ticket_step], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (APPEND && grew) a.len_rw[seg] = n;
        }
    };

    if (n == 0) {
        if (split == 0) {
            if (a.lse_out && (int)threadIdx.x < G) a.lse_out[(size_t)seg_local * G + threadIdx.x] = -INFINITY;
            for (int i = threadIdx.x; i < G * D; i += ATT_WAVES * 64) out_seg[i] = 0.f;
            if (threadIdx.x == 0) atomicAdd(&a.status[NGC_STATUS_EMPTY_ATTN], 1);
        }
        return;
    }
    const int tiles = (n + ATT_TILE - 1) / ATT_TILE;
    const int groups = (tiles + ATT_WAVES - 1) / ATT_WAVES;
    const int s_eff = groups < a.S ? groups : a.S;            // workgroups of the segment that have rows
    const float *seg_po = a.part_o + (size_t)seg_local * a.S * G * D;
    const float *seg_pml = a.part_ml + (size_t)seg_local * a.S * G * 2;
    // Merge of the s_eff partials of this segment: out = sum_s O_s 2^(m_s - M) / sum_s l_s 2^(m_s - M).  A thread
    // owns four values of the output and asks for them and for their (max, sum) pairs of MERGE partials in one batch,
    // so up to MERGE partials cost one memory round trip (about 1 us).
    auto merge_batches = [&](auto batch) {
        constexpr int MERGE = decltype(batch)::value;
        __asm__ volatile("" ::: "memory");
        const __amdgpu_buffer_rsrc_t po = device_span(seg_po, (uint32_t)(s_eff * G * D * sizeof(float)));
        const __amdgpu_buffer_rsrc_t pml = device_span(seg_pml, (uint32_t)(s_eff * G * 2 * sizeof(float)));
        for (int i4 = threadIdx.x; i4 < G * D / 4; i4 += ATT_WAVES * 64) {
            const int qi = (i4 * 4) / D;
            f32x4 num = {0.f, 0.f, 0.f, 0.f};
            float M = -INFINITY, den = 0.f;
            for (int sp0 = 0; sp0 < s_eff; sp0 += MERGE) {
                f32x4 o[MERGE];
                f32x2 ml[MERGE];
#pragma unroll
                for (int u = 0; u < MERGE; ++u) {
                    const int sp = (sp0 + u < s_eff) ? sp0 + u : s_eff - 1;
                    o[u] = ld_device16(po, (uint32_t)((sp * G * D + i4 * 4) * sizeof(float)));
                    ml[u] = ld_device8(pml, (uint32_t)((sp * G + qi) * 2 * sizeof(float)));
                }
                float top = M;                       // finite from here on: every partial's maximum is
#pragma unroll
                for (int u = 0; u < MERGE; ++u) top = fmaxf(top, ml[u][0]);
                const float old = fast_exp2(M - top);
                den *= old;
                num *= old;
                M = top;
#pragma unroll
                for (int u = 0; u < MERGE; ++u) {
                    const float wgt = (sp0 + u < s_eff) ? fast_exp2(ml[u][0] - top) : 0.f;
                    den += ml[u][1] * wgt;
                    num += o[u] * wgt;
                }
            }
            const float inv = 1.0f / den;
            *reinterpret_cast<f32x4 *>(&out_seg[i4 * 4]) = num * inv;
            if (a.lse_out && i4 * 4 == qi * D)
                a.lse_out[(size_t)seg_local * G + qi] = (M + __log2f(den)) * 0.6931471805599453f;
        }
    };
    auto merge_partials = [&]() {
        if (s_eff <= 4) merge_batches(std::integral_constant<int, 4>{});
        else if (s_eff <= 8) merge_batches(std::integral_constant<int, 8>{});
        else merge_batches(std::integral_constant<int, 16>{});
    };
    if (split * ATT_WAVES >= tiles) {   // whole workgroup: no rows for this split
        if (took_last_ticket()) {
            close_segment();
            if (s_eff > 1) merge_partials();
        }
        return;
    }

    f32x4 oacc[DPL];
#pragma unroll
    for (int c = 0; c < DPL; ++c) oacc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The running maximum starts at the smallest finite number: exponents against it are never inf - inf, so rows that score
    // -inf add 0 to the sum and to O whatever comes before or after them (and a wave without rows has factor 0 in the merges).
    float m_run = -FLT_MAX, l_run = 0.f;

#pragma unroll
    for (int c = 0; c < KCH; ++c)
        if (li >= G) qop[c] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});   // (asked for without a branch)

    unsigned char *wlds = lds + wv * WAVE_LDS;
    const int last_row = n - 1;
    auto stage_k = [&]() {
#pragma unroll
        for (int r = 0; r < K_LOADS; ++r) {
            const int rl = r * K_ROWS_PER_LOAD + lane / K_PIECES;
            *reinterpret_cast<u32x4 *>(wlds + rl * LROW + k_col) = kbuf[r];
        }
    };
    // The segment's last tile: the new row takes its place (K in LDS, V in the operands), V rows past the end are 0.
    auto finish_last_tile = [&](int t, u32x4 (&vb)[8]) {
        const int row0 = t * ATT_TILE;
        if constexpr (APPEND) {
            if (grew) {
                if (lane < K_PIECES)
                    *reinterpret_cast<u32x4 *>(wlds + (last_row - row0) * LROW + k_col) =
                        *reinterpret_cast<const u32x4 *>(fresh + k_col);
                u32x4 piece = {0u, 0u, 0u, 0u};
                if constexpr (DPL == 8) {
                    piece = *reinterpret_cast<const u32x4 *>(fresh + ROW_BYTES + v_col);
                } else {
                    const u32x2 t2 = *reinterpret_cast<const u32x2 *>(fresh + ROW_BYTES + v_col);
                    piece = u32x4{t2[0], t2[1], 0u, 0u};
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (row0 + vrow_rel[e] == last_row) vb[e] = piece;
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (row0 + vrow_rel[e] > last_row) vb[e] = u32x4{0u, 0u, 0u, 0u};
    };
    // one 32-row tile: K from the wave's LDS area, V from registers
    auto compute_tile = [&](int tile, const u32x4 (&vcur)[8], auto masked) {
        const int row0 = tile * ATT_TILE;
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < KCH; ++c) {
            const u32x4 a0 = *reinterpret_cast<const u32x4 *>(wlds + li * LROW + c * 64 + kg * 16);
            const u32x4 a1 = *reinterpret_cast<const u32x4 *>(wlds + (16 + li) * LROW + c * 64 + kg * 16);
            s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0), qop[c], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1), qop[c], s1, 0, 0, 0);
        }
        // lane (q = li, kg) now holds rows 4kg+r (s0[r]) and 16+4kg+r (s1[r])
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float sc = (e < 4) ? s0[e] : s1[e - 4];
            x[e] = (!decltype(masked)::value || row0 + vrow_rel[e] < n) ? sc * a.scale_log2e : -INFINITY;
        }
        float tmax = x[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) tmax = fmaxf(tmax, x[e]);
        tmax = quad_rows_max(tmax);
        const float m_new = fmaxf(m_run, tmax);
        if (__ballot(m_new != m_run)) {                   // wave-uniform: the running max moved somewhere
            const float alpha = fast_exp2(m_run - m_new); // 0 on the first tile, 1 where nothing changed
            l_run *= alpha;
#pragma unroll
            for (int c = 0; c < DPL; ++c) oacc[c] *= alpha;
            m_run = m_new;
        }
        float p[8], psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            p[e] = fast_exp2(x[e] - m_run);
            psum += p[e];
        }
        l_run += psum;   // lane-local part; lane groups are summed at the end

        // P as bf16 head + bf16 remainder (B operands)
        uint32_t ph[4], pl[4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            const uint32_t b0 = __float_as_uint(p[2 * e2]), b1 = __float_as_uint(p[2 * e2 + 1]);
            const float r0 = p[2 * e2] - __uint_as_float(b0 & 0xFFFF0000u);
            const float r1 = p[2 * e2 + 1] - __uint_as_float(b1 & 0xFFFF0000u);
            ph[e2] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);                     // upper halves of b0, b1
            pl[e2] = __builtin_amdgcn_perm(__float_as_uint(r1), __float_as_uint(r0), 0x07060302u);
        }
        const bf16x8 p_hi = __builtin_bit_cast(bf16x8, u32x4{ph[0], ph[1], ph[2], ph[3]});
        const bf16x8 p_lo = __builtin_bit_cast(bf16x8, u32x4{pl[0], pl[1], pl[2], pl[3]});

        // O^T += V^T P
#pragma unroll
        for (int c = 0; c < DPL; ++c) {
            uint32_t va[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                const uint32_t w0 = vcur[2 * e2][c >> 1];       // row e = 2*e2,   d pair c/2
                const uint32_t w1 = vcur[2 * e2 + 1][c >> 1];   // row e = 2*e2+1
                // 2x2 transpose of 16-bit elements: one byte permute per output word
                va[e2] = (c & 1) ? __builtin_amdgcn_perm(w1, w0, 0x07060302u)
                                 : __builtin_amdgcn_perm(w1, w0, 0x05040100u);
            }
            const bf16x8 vop = __builtin_bit_cast(bf16x8, u32x4{va[0], va[1], va[2], va[3]});
            oacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, p_hi, oacc[c], 0, 0, 0);
            oacc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop, p_lo, oacc[c], 0, 0, 0);
        }
    };

    // Software pipeline, unrolled by two so that the V registers of the tile in
    // flight and of the tile being computed are distinct (no copies): the loads
    // of the next tile are issued before the current tile's math and are only
    // waited for at the top of the next step.  A wave's last tile is a copy of
    // the step without the loads (a prefetch inside a branch would make the wait
    // for the current tile wait for the prefetch too, and a prefetch past the
    // end, clamped to the last row, sends every wave of a segment to the same
    // two cache lines: 1.4 us of a 9.6 us launch of 16 segments x 12 workgroups);
    // only there can the segment end, so only there rows are masked.
    if constexpr (APPEND) {
        const int last_tile = tiles - 1;
        if (grew && last_tile / ATT_WAVES % a.S == split && last_tile % ATT_WAVES == wv_u) {
            const size_t at = ((size_t)seg * a.cap + last_row) * ROW_BYTES;
            if (lane < 2 * K_PIECES) {
                *reinterpret_cast<u32x4 *>((lane < K_PIECES ? a.k_rw : a.v_rw) + at + k_col) = new_piece;
                *reinterpret_cast<u32x4 *>(fresh + (lane / K_PIECES) * ROW_BYTES + k_col) = new_piece;
            }
            if (lane == 0 && a.pos && a.new_pos) a.pos[(size_t)seg * a.cap + last_row] = a.new_pos[(seg / a.Hkv) % a.B];
        }
    }

    if constexpr (!EARLY) {
        if (tile < tiles) issue_loads(tile, last_row, base0, v_a);
    } else {
        base1 = tile_base(tile + step, tiles - 1);
        base2 = tile_base(tile + 2 * step, tiles - 1);
    }
    bool staged = false;
    while (tile + step < tiles) {
        stage_k();
        issue_loads(tile + step, last_row, base1, v_b);
        base1 = base2;
        base2 = tile_base(tile + 3 * step, tiles - 1);
        __builtin_amdgcn_sched_barrier(0);
        compute_tile(tile, v_a, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        tile += step;
        if (tile + step >= tiles) {     // the last tile is in v_b: one copy of its step serves both buffers
            stage_k();
            staged = true;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 8; ++e) v_a[e] = v_b[e];
            break;
        }
        stage_k();
        issue_loads(tile + step, last_row, base1, v_a);
        base1 = base2;
        base2 = tile_base(tile + 3 * step, tiles - 1);
        __builtin_amdgcn_sched_barrier(0);
        compute_tile(tile, v_b, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        tile += step;
    }
    if (tile < tiles) {
        if (!staged) stage_k();
        __builtin_amdgcn_sched_barrier(0);
        if (tile == tiles - 1) finish_last_tile(tile, v_a);
        compute_tile(tile, v_a, std::true_type{});
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- merge the waves of this workgroup ----------------------------------
    // O of every wave, its maximum and its sum go to LDS as they are (O into the wave's own staging area, which is free now);
    // after one barrier a thread scales and adds the four waves' values of its own part of the output.
    // A row of 16-byte stores per query head and lane group, rows a multiple of 16 bytes but not of 256 apart: the 16
    // heads of a lane group meet 16 different sets of banks.  (Rows of D floats, stored a float at a time after a barrier and
    // an exchange of the maxima, had all of them meet in one bank: 0.7 us of a launch of 32 segments of 525 rows; per
    // layer from a HIP graph 6.9 -> 6.45 us, 2 x 300 rows of 128 bytes 4.3 -> 4.0, 128 x 1493 rows 19.8 -> 19.4.)
    constexpr int OROW = D + 4;                            // floats
    static_assert(16 * OROW * 4 <= WAVE_LDS, "staging area too small");
    l_run = quad_rows_sum(l_run);
    if (kg == 0) { red_m[wv][li] = m_run; red_l[wv][li] = l_run; }
    // lane (q = li, kg), register (c, r) holds d = DPL * (4kg + r) + c
    if (li < G) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < DPL; c += 4)
                reinterpret_cast<f32x4 *>(wlds)[(li * OROW + DPL * (4 * kg + r) + c) / 4] =
                    f32x4{oacc[c][r], oacc[c + 1][r], oacc[c + 2][r], oacc[c + 3][r]};
    }
    __syncthreads();
    // maximum and sum of query head qi over the waves, and the waves' factors (0 for a wave without rows)
    auto waves_of = [&](int qi, float (&f)[ATT_WAVES], float &m_all, float &l_all) {
        m_all = red_m[0][qi];
#pragma unroll
        for (int w = 1; w < ATT_WAVES; ++w) m_all = fmaxf(m_all, red_m[w][qi]);
        l_all = 0.f;
#pragma unroll
        for (int w = 0; w < ATT_WAVES; ++w) {
            f[w] = fast_exp2(red_m[w][qi] - m_all);
            l_all += red_l[w][qi] * f[w];
        }
    };
    auto sum_of_waves = [&](int qi, int d, const float (&f)[ATT_WAVES]) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < ATT_WAVES; ++w) acc += reinterpret_cast<const f32x4 *>(lds + w * WAVE_LDS)[(qi * OROW + d) / 4] * f[w];
        return acc;
    };
    float f[ATT_WAVES], m_all, l_all;
    const bool direct = (s_eff == 1);   // the only split of its segment with rows: finish here
    if (direct) {
        for (int i4 = threadIdx.x; i4 < G * D / 4; i4 += ATT_WAVES * 64) {
            const int qi = (i4 * 4) / D, d = i4 * 4 - qi * D;
            waves_of(qi, f, m_all, l_all);
            *reinterpret_cast<f32x4 *>(&out_seg[i4 * 4]) = sum_of_waves(qi, d, f) / l_all;
            if (a.lse_out && d == 0)
                a.lse_out[(size_t)seg_local * G + qi] = (m_all + __log2f(l_all)) * 0.6931471805599453f;
        }
        if (a.S == 1 || took_last_ticket()) close_segment();
        return;
    }
    float *dst_o = a.part_o + ((size_t)seg_local * a.S + split) * G * D;
    const __amdgpu_buffer_rsrc_t po = device_span(dst_o, (uint32_t)(G * D * sizeof(float)));
    const __amdgpu_buffer_rsrc_t pml =
        device_span(a.part_ml + ((size_t)seg_local * a.S + split) * G * 2, (uint32_t)(G * 2 * sizeof(float)));
    for (int i4 = threadIdx.x; i4 < G * D / 4; i4 += ATT_WAVES * 64) {
        const int qi = (i4 * 4) / D, d = i4 * 4 - qi * D;
        waves_of(qi, f, m_all, l_all);
        st_device16(po, (uint32_t)(i4 * 4 * sizeof(float)), sum_of_waves(qi, d, f));
        if (d == 0) st_device8(pml, (uint32_t)(qi * 2 * sizeof(float)), f32x2{m_all, l_all});
    }
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's partial stores have reached memory
    if (took_last_ticket()) {
        close_segment();
        merge_partials();
    }
}

}  // namespace ngc

// ============================================================ host side ====

using namespace ngc;

namespace {
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
constexpr size_t STATUS_BYTES = NGC_STATUS_WORDS * sizeof(int32_t);
// How many workgroups share a segment.  Microseconds per launch (MI355X, one launch per layer of 28 from a HIP graph, D = 128)
// against S, best in brackets:
//     segments x rows      S=1    2     3     4     5     6     7     8    10    12    16    24    32
//         2 x  525         8.0   6.8   6.4   5.8 [ 5.1]
//         2 x 2000        20.5  13.0  10.8   9.0   8.8   7.9         6.9   7.5   7.4 [ 6.0]
//         2 x 4000        37.8  22.0  16.5  13.6  12.3  11.3         9.5   9.8   8.7   7.7   8.7 [ 7.2]
//        16 x  525         8.5   7.5   6.9   6.1 [ 5.5]
//        16 x 2000        21.7  14.1  11.6   9.7   9.5   8.5         7.8   8.4   8.5 [ 7.5]
//        16 x 8000        74.7  41.2  29.4  24.1  20.7  18.5        16.0  16.0  16.0 [15.1]
//        32 x  300         6.2   6.3 [ 5.5]
//        32 x  800        11.0   9.0   7.7   7.2   7.5   6.7 [ 6.1]
//        32 x 2000        22.1  14.7  12.3  10.5  10.5 [ 9.7]        9.9
//        48 x  525         8.9   7.9   7.2   6.9 [ 6.2]
//        64 x  400         7.8   7.3   6.9 [ 6.1]
//        64 x 2000        24.5  15.9  15.2 [14.7]
//        64 x 8000        81.8  49.1 [42.4] 42.8
//       128 x  525         9.6 [ 9.5]
//       128 x 2000        26.6 [23.8]
// What they say: a launch should have no more workgroups than the chip has CUs, S <= 256 / segments.  Below that a
// workgroup works through rounds of four tiles (one per wave), so only the S that lower the number of rounds are worth
// their cost: sharing a segment at all (partial, ticket, merge: three memory round trips), a further such trip for every
// 16 partials more, and a little for workgroups beyond 128.  What these cost depends on how far apart the tickets lie
// (ticket_step()): the prices of a launch over words next to each other, 4 or more words apart, and half a line.  With one
// price for all, the one of the first row: 32 x 800 rows 7.2 us at S = 4 instead of 6.1 at 7, 48 x 525 7.2 (S = 3) instead of
// 6.2, 64 x 400 7.3 (2) and 6.1, 32 x 800 rows of 128 bytes 5.5 (4) and 5.0; with the last row's over tickets next to each other
// 16 x 2000 rows 9.6 us (S = 16) instead of 8.5 (8), 8 x 8000 12.9 (32) instead of 11.6 (16).
constexpr int COMPUTE_UNITS = 256;

int most_splits(int nseg_launch, int max_len)
{
    const int rounds_of_one = ((max_len + ATT_TILE - 1) / ATT_TILE + ATT_WAVES - 1) / ATT_WAVES;
    int s = COMPUTE_UNITS / (nseg_launch > 0 ? nseg_launch : 1);
    s = s < rounds_of_one ? s : rounds_of_one;
    s = s < MAX_SPLITS ? s : MAX_SPLITS;
    return s > 1 ? s : 1;
}

struct SplitPrice {
    float round, share, more, beyond;      // us: a round of tiles, sharing a segment, 16 partials more, a workgroup beyond 128
};

SplitPrice split_price(int row_bytes, int apart)
{
    const bool wide = row_bytes == 256;
    if (apart < 4) return wide ? SplitPrice{0.95f, 1.2f, 1.2f, 0.01f} : SplitPrice{0.58f, 1.2f, 1.2f, 0.01f};
    if (apart < 16) return wide ? SplitPrice{0.8f, 1.05f, 0.9f, 0.007f} : SplitPrice{0.45f, 1.1f, 0.9f, 0.004f};
    return wide ? SplitPrice{0.8f, 1.05f, 0.55f, 0.005f} : SplitPrice{0.45f, 1.1f, 0.6f, 0.003f};
}

// apart: words between the tickets of a workspace's launch (the static entry point splits the same way).
int splits_for(int nseg_launch, int max_len, int row_bytes, int apart)
{
    const int most = most_splits(nseg_launch, max_len);
    const int tiles = (max_len + ATT_TILE - 1) / ATT_TILE;
    const SplitPrice price = split_price(row_bytes, apart);
    int best = 1;
    float best_us = 3.0e38f;
    for (int s = most; s >= 1; --s) {
        const int rounds = (tiles + ATT_WAVES * s - 1) / (ATT_WAVES * s);
        if (s > 1 && (tiles + ATT_WAVES * (s - 1) - 1) / (ATT_WAVES * (s - 1)) == rounds) continue;   // one fewer does as well
        const int beyond = s * nseg_launch > 128 ? s * nseg_launch - 128 : 0;
        const float us = price.round * (float)rounds +
                         (s > 1 ? price.share + price.more * (float)((s - 1) / 16) + price.beyond * (float)beyond : 0.f);
        if (us < best_us) { best_us = us; best = s; }
    }
    return best;
}

// Whether a wave asks for its first tile before the length has arrived.  It saves part of a memory round trip in front of
// the launch, and reads rows nobody uses where a segment is shorter than the workgroup's four tiles.  Microseconds
// without -> with (D = 128, one kernel that takes the choice as an argument; the argument itself costs small launches
// up to 0.6 us, hence two kernels):
//     segments x rows        20-32          100-128        500-550        2000-3000
//           2             4.06 -> 4.25    4.53 -> 4.48    6.02 -> 5.83    7.74 -> 7.71
//          64             4.27 -> 4.47    4.72 -> 4.71    8.62 -> 8.49    17.9 -> 17.7
//         256             4.92 -> 5.84    6.38 -> 6.25    13.9 -> 13.8    53.5 -> 52.5
//         512             5.77 -> 8.45    8.04 -> 8.21    23.3 -> 23.5    103.6 -> 102.3
//        1024             9.83 -> 14.9    15.0 -> 15.6    44.6 -> 44.6    204.9 -> 203.9
//        8192             60.2 -> 108     102 -> 108      367 -> 366
// So it is done where every workgroup has a CU to itself (at most 16 MB are read in vain there) and the longest segment
// has more rows than two tiles; beyond, the other workgroups of a CU cover the wait, and it is done only if the caller
// knows the longest segment to have more than one round of tiles (the capacity alone says nothing about that).  With the
// two kernels 1024 segments of 20-32 rows take 8.6 us, 13.3 if all ask early; 384 of 100-200 rows 8.9 us if they ask early,
// 9.6 if not; 1792 of 700-1366 rows at D = 64 147 and 151 us.
bool first_tile_early(int nseg_launch, int S, int max_len, int max_len_hint)
{
    if (nseg_launch * S <= COMPUTE_UNITS) return max_len > 2 * ATT_TILE;
    return max_len_hint > ATT_WAVES * ATT_TILE;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// workspace layout: [status][per segment of the cache: 2 int32 of the paged layout's pool bookkeeping]
//                   [per segment of the cache: ticket][partial O][partial (max, sum)]
size_t ticket_offset(const ngc_cache *c)
{
    return STATUS_BYTES + (size_t)c->L * c->B * c->Hkv * 2 * sizeof(int32_t);
}
size_t attn_offset(const ngc_cache *c)
{
    return align256(ticket_offset(c) + (size_t)c->L * c->B * c->Hkv * sizeof(int32_t));
}
size_t partial_o_bytes(const ngc_cache *c, int nseg_launch, int S)
{
    return align256((size_t)nseg_launch * S * (c->Hq / c->Hkv) * c->D * sizeof(float));
}
size_t partial_ml_bytes(const ngc_cache *c, int nseg_launch, int S)
{
    return align256((size_t)nseg_launch * S * (c->Hq / c->Hkv) * 2 * sizeof(float));
}
size_t attn_partial_bytes(const ngc_cache *c, int nseg_launch, int S)
{
    return S > 1 ? partial_o_bytes(c, nseg_launch, S) + partial_ml_bytes(c, nseg_launch, S) : 0;
}

// Whether ngc_decode_attn_static takes a call is decided by this number of workgroups per segment, the one that ngc.h
// states, not by the one that is launched, so that a better split never turns a call away (nor lets one in).  It differs
// from "always" only for 16 query heads per KV head at D = 128.
int static_limit_splits(int nseg_launch, int max_len, int row_bytes)
{
    const double seg_mb = 2.0 * row_bytes * max_len * 1e-6;          // K and V of a segment
    int s = COMPUTE_UNITS / (nseg_launch > 0 ? nseg_launch : 1);
    const int by_merge = (int)sqrt(80.0 * seg_mb);
    const int by_length = (max_len + ATT_TILE - 1) / ATT_TILE / 4;
    s = s < by_merge ? s : by_merge;
    s = s < by_length ? s : by_length;
    s = s < MAX_SPLITS ? s : MAX_SPLITS;
    return s > 1 ? s : 1;
}

// `fixed_layout`: the scratch is not a workspace sized for this cache but the library's own fixed array, which
// serves caches of any geometry one after the other: tickets and partials then sit at offsets that do not depend
// on the geometry (a ticket region that moved with the geometry would land on an earlier call's partials).
// All words between the two offsets are tickets, ticket_step() apart, and zero between launches: they outnumber the
// COMPUTE_UNITS / 2 segments that a launch can have and still be split.
constexpr size_t FIXED_TICKET_OFFSET = STATUS_BYTES;
constexpr size_t FIXED_PARTIAL_OFFSET = 4096;
constexpr size_t FIXED_TICKETS = (FIXED_PARTIAL_OFFSET - FIXED_TICKET_OFFSET) / sizeof(int32_t);

// Words between the tickets of two segments.  Atomics on one cache line are served one after the other, so a launch's
// tickets lie as far apart as the words at hand allow, up to a line of 128 bytes.  A workspace has a word for every
// segment of the cache, so the launches of a model of L layers, one layer each, have L words for a segment; a launch
// over all layers has one, as does a cache of a single layer.  Microseconds per layer from a HIP graph of 28 layers, words
// next to each other -> 28 apart, D = 128 (no difference below 16 segments, where at most 64 atomics meet):
//     16 x 1500 rows   8.27 -> 6.69      32 x 1500   8.83 -> 8.11      64 x 1500        11.56 -> 11.06
//     32 x  300        5.70 -> 5.47      64 x  525   8.06 -> 7.79      128 x 525        10.18 ->  9.55
//     32 x  525        6.31 -> 5.74      48 x 676-1352 8.91 -> 8.64    64 x 3000-10000  41.18 -> 39.89
int ticket_step(size_t words, int nseg_launch)
{
    const size_t apart = words / (size_t)nseg_launch;
    return apart > 32 ? 32 : apart > 1 ? (int)apart : 1;
}

bool fits_static(const ngc_cache *c, int nseg_launch, int S)
{
    return FIXED_PARTIAL_OFFSET + attn_partial_bytes(c, nseg_launch, S) <= NGC_STATIC_SCRATCH_BYTES;
}
}  // namespace

extern "C" int ngc_version(void) { return 220; }

extern "C" const char *ngc_strerror(int code)
{
    switch (code) {
    case NGC_OK: return "ok";
    case NGC_EINVAL: return "invalid argument (null or misaligned pointer, bad shape or parameter)";
    case NGC_ENOSPC: return "workspace too small (ngc_decode_attn_static: the call needs more than its fixed scratch array)";
    case NGC_EHIP: return "a HIP runtime call failed";
    case NGC_EUNSUPPORTED: return "request outside the limits of this entry point";
    default: return "unknown error code";
    }
}

extern "C" size_t ngc_workspace_bytes(const ngc_cache *c, int32_t max_keep)
{
    (void)max_keep;
    if (!c || c->L <= 0 || c->B <= 0 || c->Hkv <= 0 || c->Hq <= 0 || c->cap <= 0) return 0;
    const int per_layer = c->B * c->Hkv;
    // the most any launch can ask for: one layer or all layers, any length hint (a launch that finds less
    // workspace than its preferred split needs falls back to fewer splits, so this is a guarantee, not a limit)
    const size_t one = attn_partial_bytes(c, per_layer, most_splits(per_layer, c->cap));
    const size_t all = attn_partial_bytes(c, per_layer * c->L, most_splits(per_layer * c->L, c->cap));
    const size_t most = one > all ? one : all;
    return attn_offset(c) + most;
}

namespace {
// Shared by both layouts.  `c` carries the logical geometry (for the paged
// layout: cap = max_pages * page_rows, k / v = the pools).
struct NewRows {            // fused append: the new token's rows, or all null
    const void *k_new;
    const void *v_new;
    const int32_t *new_pos;
};

int launch_decode(const ngc_cache *c, const ngc_paged_cache *pc, int32_t layer, const NewRows *nr, const void *q,
                  float scale, int32_t max_len_hint, float *out, float *lse_out, int32_t *status, void *ws,
                  size_t ws_bytes, void *stream, bool fixed_layout = false)
{
    if (nr && (!nr->k_new || !nr->v_new || !aligned16(nr->k_new) || !aligned16(nr->v_new) || pc)) return NGC_EINVAL;
    if (!c->k || !c->v || !c->len || !q || !out || !ws) return NGC_EINVAL;
    if (!aligned16(c->k) || !aligned16(c->v) || !aligned16(q) || !aligned16(out) || !aligned16(ws)) return NGC_EINVAL;
    if (c->L <= 0 || c->B <= 0 || c->Hkv <= 0 || c->Hq <= 0 || c->cap <= 0) return NGC_EINVAL;
    if (c->D != 64 && c->D != 128) return NGC_EINVAL;
    if ((long long)c->cap * c->D * 2 > 0x7FFFFFFFLL) return NGC_EUNSUPPORTED;   // 32-bit byte offsets inside a segment
    if (c->Hq % c->Hkv != 0 || c->Hq / c->Hkv > 16) return NGC_EINVAL;
    if (layer < -1 || layer >= c->L || max_len_hint < 0) return NGC_EINVAL;
    if (!(scale == scale)) return NGC_EINVAL;
    const int per_layer = c->B * c->Hkv;
    const int seg0 = layer < 0 ? 0 : layer * per_layer;
    const int nseg = layer < 0 ? c->L * per_layer : per_layer;
    const int max_len = (max_len_hint > 0 && max_len_hint < c->cap) ? max_len_hint : c->cap;
    const int apart = ticket_step((size_t)c->L * per_layer, nseg);
    int S = splits_for(nseg, max_len, c->D * 2, apart);
    if (nseg > COMPUTE_UNITS) S = 1;   // (what splits_for() returns anyway: the fixed ticket region relies on it)
    // A call that the fixed array serves is split the same way with a workspace: both return the same bits.
    const bool static_ok = fits_static(c, nseg, static_limit_splits(nseg, max_len, c->D * 2));
    if (fixed_layout && !static_ok) return NGC_ENOSPC;
    while (static_ok && S > 1 && !fits_static(c, nseg, S)) --S;
    const size_t off = fixed_layout ? FIXED_PARTIAL_OFFSET : attn_offset(c);
    if (ws_bytes < off) return NGC_ENOSPC;
    while (S > 1 && ws_bytes < off + attn_partial_bytes(c, nseg, S)) --S;   // fewer splits: same result, less scratch
    if ((long long)nseg * S > 0x7FFFFFFFLL) return NGC_EUNSUPPORTED;

    AttnArgs aa;
    aa.k = reinterpret_cast<const unsigned char *>(c->k);
    aa.v = reinterpret_cast<const unsigned char *>(c->v);
    aa.len = c->len;
    aa.q = reinterpret_cast<const unsigned char *>(q);
    aa.out = out;
    aa.lse_out = lse_out;
    aa.part_o = reinterpret_cast<float *>(reinterpret_cast<unsigned char *>(ws) + off);
    aa.part_ml = reinterpret_cast<float *>(reinterpret_cast<unsigned char *>(ws) + off +
                                           partial_o_bytes(c, nseg, S));
    aa.status = status ? status : reinterpret_cast<int32_t *>(ws);
    aa.seg0 = seg0;
    aa.S = S; aa.G = c->Hq / c->Hkv; aa.Hkv = c->Hkv; aa.cap = c->cap;
    aa.scale_log2e = scale * 1.4426950408889634f;
    aa.ticket = reinterpret_cast<int32_t *>(reinterpret_cast<unsigned char *>(ws) +
                                            (fixed_layout ? FIXED_TICKET_OFFSET : ticket_offset(c)));
    aa.ticket_step = fixed_layout ? ticket_step(FIXED_TICKETS, nseg) : apart;
    aa.k_rw = reinterpret_cast<unsigned char *>(c->k);
    aa.v_rw = reinterpret_cast<unsigned char *>(c->v);
    aa.len_rw = c->len;
    aa.pos = c->pos;
    aa.k_new = nr ? reinterpret_cast<const unsigned char *>(nr->k_new) : nullptr;
    aa.v_new = nr ? reinterpret_cast<const unsigned char *>(nr->v_new) : nullptr;
    aa.new_pos = nr ? nr->new_pos : nullptr;
    aa.B = c->B;
    aa.table = nullptr; aa.max_pages = 0; aa.num_pages = 0; aa.tpp_shift = 0;
    if (pc) {
        aa.table = pc->table; aa.max_pages = pc->max_pages; aa.num_pages = pc->num_pages;
        int tpp = pc->page_rows / ATT_TILE, sh = 0;
        while ((1 << sh) < tpp) ++sh;
        aa.tpp_shift = sh;
    }
    hipStream_t st = (hipStream_t)stream;
    const bool early = first_tile_early(nseg, S, max_len, max_len_hint);
#define NGC_PICK_DECODE(PAGED, APPEND) \
    (c->D == 128 ? (early ? reinterpret_cast<const void *>(&decode_kernel<128, PAGED, APPEND, true>) \
                          : reinterpret_cast<const void *>(&decode_kernel<128, PAGED, APPEND, false>)) \
                 : (early ? reinterpret_cast<const void *>(&decode_kernel<64, PAGED, APPEND, true>) \
                          : reinterpret_cast<const void *>(&decode_kernel<64, PAGED, APPEND, false>)))
    const void *fn = pc ? NGC_PICK_DECODE(true, false) : nr ? NGC_PICK_DECODE(false, true) : NGC_PICK_DECODE(false, false);
#undef NGC_PICK_DECODE
    return launch(fn, dim3(nseg, S), dim3(ATT_WAVES * 64), 0, st, aa);
}
}  // namespace

extern "C" int ngc_decode_attn(const ngc_cache *c, int32_t layer, const void *q, float scale,
                               int32_t max_len_hint, float *out, float *lse_out,
                               void *ws, size_t ws_bytes, void *stream)
{
    if (!c) return NGC_EINVAL;
    return launch_decode(c, nullptr, layer, nullptr, q, scale, max_len_hint, out, lse_out, nullptr, ws, ws_bytes,
                         stream);
}

extern "C" int ngc_decode_step(const ngc_cache *c, int32_t layer, const void *k_new, const void *v_new,
                               const int32_t *new_pos, const void *q, float scale, int32_t max_len_hint,
                               float *out, float *lse_out, void *ws, size_t ws_bytes, void *stream)
{
    if (!c) return NGC_EINVAL;
    const NewRows nr{k_new, v_new, new_pos};
    return launch_decode(c, nullptr, layer, &nr, q, scale, max_len_hint, out, lse_out, nullptr, ws, ws_bytes, stream);
}

// ---- the same call for callers that cannot allocate ------------------------
//
// The split partials and tickets (and, when the caller passes no status buffer,
// the status words) live in a fixed array inside the library's device image
// instead of a caller-provided workspace.  The array starts out zeroed when the
// image is loaded and every launch leaves the tickets at zero again.  Every GPU holds its own copy of the array; its
// address on a device is looked up once, with that device current, and kept.
constexpr size_t STATIC_SCRATCH_BYTES = NGC_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[MAX_DEVICES];      // device address of `scratch` per device, nullptr until looked up

int static_scratch(void **ptr)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return NGC_EHIP;
    if (dev < 0 || dev >= MAX_DEVICES) return NGC_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return NGC_EHIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return NGC_OK;
}
}  // namespace

extern "C" int ngc_decode_attn_static(const ngc_cache *c, int32_t layer, const void *q, float scale,
                                      int32_t max_len_hint, float *out, float *lse_out,
                                      int32_t *status, void *stream)
{
    if (!c) return NGC_EINVAL;
    void *ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc) return rc;
    return launch_decode(c, nullptr, layer, nullptr, q, scale, max_len_hint, out, lse_out, status, ws,
                         STATIC_SCRATCH_BYTES, stream, true);
}

extern "C" int ngc_paged_decode_attn(const ngc_paged_cache *pc, int32_t layer, const void *q, float scale,
                                     int32_t max_len_hint, float *out, float *lse_out,
                                     void *ws, size_t ws_bytes, void *stream)
{
    if (!pc || !pc->table) return NGC_EINVAL;
    if (pc->page_rows < ATT_TILE || (pc->page_rows & (pc->page_rows - 1)) != 0) return NGC_EINVAL;
    if (pc->max_pages <= 0 || pc->num_pages <= 0) return NGC_EINVAL;
    if ((long long)pc->max_pages * pc->page_rows > 0x7FFFFFFFLL / 256) return NGC_EUNSUPPORTED;
    ngc_cache c{};
    c.k = pc->k_pool; c.v = pc->v_pool; c.len = pc->len; c.pos = nullptr;
    c.L = pc->L; c.B = pc->B; c.Hkv = pc->Hkv; c.Hq = pc->Hq; c.D = pc->D;
    c.cap = pc->max_pages * pc->page_rows;
    return launch_decode(&c, pc, layer, nullptr, q, scale, max_len_hint, out, lse_out, nullptr, ws, ws_bytes, stream);
}
