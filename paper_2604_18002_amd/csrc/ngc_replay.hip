// Replay attention for the training forward pass (Sec. 4.5 and Appendix A.3 of
// the paper): all T positions of a trajectory at once, query i seeing key j iff
// j <= i and j had not been evicted when token i was generated.
//
// Instead of the paper's dense T x T boolean mask per layer, visibility is one
// int per key: death[j] = first query position that no longer sees key j, so
// visible(i, j) = (j <= i < death[j]).  For every tile of 128 query positions
// the keys that at least one of its queries can see are compacted into a list
// (j not after its last query, death[j] after its first); the attention kernel
// then only ever loads those rows: the work follows the retained cache, not the
// T x T triangle.  Over long trajectories a small first kernel makes the lists,
// shared by all query heads that share the decisions; over short ones every
// workgroup makes its own.
//
// Flash-attention forward on the matrix cores (S^T = K Q^T, O^T = V^T P, mfma 32x32x16: one query per lane % 32, so all
// soft-max state is lane local and crosses lanes once, between the two halves; P as bf16 head + remainder).  A workgroup
// = 4 waves x 32 query positions of one query head; tiles of 64 keys go from memory straight into double-buffered LDS
// (no registers, no LDS store instructions) and are shared by the waves; the V operand is read transposed from LDS.
//
// What bounds it: matrix and vector work of two waves per SIMD that overlap only in part, then the output.  B = 8,
// T = 4096, 28/4 heads, 27 % of the causal pairs visible (the issued products are worth 390 GFLOP): 546-557 us with
// 16-wide tiles and rows staged through registers, now 440-460 us; B = 16, T = 1050, 12/2 heads 123 -> 79 us.  On the
// way, at the first shape (552 us before): 32-wide tiles and loads straight to LDS 511 us; a reference for the
// exponents that moves only when outgrown by 2^8, and transposing reads of V instead of 32 byte permutes a step, 464 us;
// the output through LDS in whole lines, nontemporal, and the list kernel in one pass 440 us.  The version before the last
// of these took 470 us there, 403 without its tile loads, 281 without its products, 113 with neither (470 MB of output).
// Measured and not kept: two independent score accumulators (the chain
// already issues every 32 cycles), two steps per soft-max (spills at 256 registers, 668 us), 32-key tiles with two
// (+4 %) or three waves per SIMD (spills at 168 registers, +18 %), the remainder of P by a bf16 dot product (4 instead
// of 6 instructions a pair, no faster), output straight from the registers nontemporal (+20 %: partial lines).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/ngc.h"
#include "ngc_device.h"

namespace ngc {

constexpr int RP_WAVES = 4;
constexpr int RP_QW = 32;                    // query positions per wave
constexpr int RP_QT = RP_WAVES * RP_QW;      // query positions per workgroup
constexpr int RP_KT = 64;                    // keys per LDS tile (one barrier per tile)
constexpr int RP_MT = 32;                    // keys per step of the math (and per entry of tile_death)
// Start of the running max: finite and below every real score, so that 2^(x - m) is 0 for a masked
// x = -inf without a special case, and the first rescale factor 2^(m_init - m_new) is 0.
constexpr float RP_M_INIT = -1.0e30f;
constexpr float RP_LAZY = 8.0f;

// What the waves of a query tile have to know about RP_MT consecutive keys of its list, in terms of the wave index:
// waves below `after` have all their queries before the first of these keys; waves from `from` to `until` - 1 see all of
// the keys with all of their queries.  One word: after in the lowest byte, then from, then until.
constexpr uint32_t step_word(uint32_t after, uint32_t from, uint32_t until) { return after | from << 8 | until << 16; }

struct ReplayArgs {
    const unsigned char *q;    // bf16 [B][T][Hq][D]
    const unsigned char *k;    // bf16 [B][T][Hkv][D]
    const unsigned char *v;
    const int32_t *death;      // [B][Hd][T]
    uint16_t *klist;           // [B*Hd][nqt][T] visible keys per query tile, ascending
    int32_t *kcount;           // [B*Hd][nqt]
    uint32_t *steps;           // [B*Hd][nqt][ceil(T/32)] what the waves have to know about each RP_MT keys of a list
    float *out;                // fp32 [B][T][Hq][D]
    int B, T, Hq, Hkv, Hd;     // Hd = Hkv (a death row per KV head) or 1 (shared by the heads)
    float scale_log2e;
};

// What a wave-wide step of the list means for the tile's waves, from its first and last key and its earliest death.
__device__ __forceinline__ uint32_t step_of(int i0, int T, int first, int last, int lives_until)
{
    int after = 0, from = 0, until = 0;
#pragma unroll
    for (int w = 0; w < RP_WAVES; ++w) {
        const int q0 = i0 + w * RP_QW;                                   // the wave's first query and its last real one
        const int q1 = q0 + RP_QW - 1 < T - 1 ? q0 + RP_QW - 1 : T - 1;
        after += first > q1;
        from += last > q0;
        until += lives_until > q1;
    }
    return step_word(after, from, until);
}

// Ordered compaction, LIST_PASS keys per pass (one pass up to 4096 positions: its keys' death positions are all asked
// for at once).  Key j0 + 256 i + tid belongs to thread tid's i-th bit: ballots give the counts of every (i, wave),
// a scan over those 64 numbers their order.  What the attention kernel has to know about each RP_MT keys is gathered
// in LDS on the way.  (256 keys per pass, and a second walk over the list for the steps: 16 us at 256 lists of 4096
// positions, 9 us at 144 lists of 1050; now 6.4 and 5.0, most of it launch and two memory round trips.)
constexpr int LIST_THREADS = 256;
constexpr int LIST_BITS = 16;
constexpr int LIST_PASS = LIST_THREADS * LIST_BITS;
constexpr int LIST_WAVES = LIST_THREADS / NGC_WAVE;
constexpr int LIST_MAX_STEPS = 65536 / RP_MT;
constexpr uint16_t NO_KEY = 0xFFFF;          // beyond every key (T <= 65535): a last step of fewer keys needs the mask

__global__ __launch_bounds__(LIST_THREADS) void replay_lists_kernel(ReplayArgs a)
{
    static_assert(LIST_BITS * LIST_WAVES == NGC_WAVE, "a wave scans the counts of a pass");
    __shared__ int counts[LIST_BITS * LIST_WAVES];
    __shared__ int min_death[LIST_MAX_STEPS];
    __shared__ uint16_t first_key[LIST_MAX_STEPS], last_key[LIST_MAX_STEPS];
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int T = a.T;
    const int nqt = (T + RP_QT - 1) / RP_QT;
    const int qt = blockIdx.x, row = blockIdx.y;          // row = b * Hd + hd
    const int i0 = qt * RP_QT;
    const int last_pos = (i0 + RP_QT - 1 < T - 1) ? i0 + RP_QT - 1 : T - 1;
    const int32_t *death = a.death + (size_t)row * T;
    uint16_t *klist = a.klist + ((size_t)row * nqt + qt) * T;
    for (int s = tid; s * RP_MT <= last_pos; s += LIST_THREADS) {
        min_death[s] = 0x7FFFFFFF;
        last_key[s] = NO_KEY;
    }
    int n_list = 0;
    for (int j0 = 0; j0 <= last_pos; j0 += LIST_PASS) {
        int d[LIST_BITS];
#pragma unroll
        for (int i = 0; i < LIST_BITS; ++i) {
            const int j = j0 + i * LIST_THREADS + tid;
            d[i] = j <= last_pos ? death[j] : -1;          // (a key no query of the tile sees)
        }
        uint64_t seen[LIST_BITS];
#pragma unroll
        for (int i = 0; i < LIST_BITS; ++i) {
            seen[i] = __ballot(d[i] > i0);
            if (lane == 0) counts[i * LIST_WAVES + wv] = __popcll(seen[i]);
        }
        __syncthreads();
        const int mine = counts[lane];
        const int upto = wave_incl_scan_i(mine);
#pragma unroll
        for (int i = 0; i < LIST_BITS; ++i) {
            const int before = __builtin_amdgcn_readlane(upto - mine, i * LIST_WAVES + wv);
            if (d[i] > i0) {
                const int j = j0 + i * LIST_THREADS + tid;
                const int slot = n_list + before + popc_below(seen[i]);
                klist[slot] = (uint16_t)j;
                atomicMin(&min_death[slot / RP_MT], d[i]);
                if (slot % RP_MT == 0) first_key[slot / RP_MT] = (uint16_t)j;
                if (slot % RP_MT == RP_MT - 1) last_key[slot / RP_MT] = (uint16_t)j;
            }
        }
        n_list += __builtin_amdgcn_readlane(upto, NGC_WAVE - 1);
        __syncthreads();
    }
    if (tid == 0) a.kcount[(size_t)row * nqt + qt] = n_list;
    uint32_t *steps = a.steps + ((size_t)row * nqt + qt) * ((T + RP_MT - 1) / RP_MT);
    for (int s = tid; s * RP_MT < n_list; s += LIST_THREADS) {
        steps[s] = step_of(i0, T, first_key[s], last_key[s], min_death[s]);
    }
}

// The key list of one query tile in LDS, made by the workgroup itself, for trajectories of up to OWN_MAX positions.  A kernel of its
// own for the lists pays where many workgroups share a long one; over short trajectories it is mostly a launch and two
// memory round trips in front of the attention.  Microseconds, lists by a kernel -> by the workgroups:
//     B  heads         T = 130          350            600           1050            1500            2000
//     2  28/4      13.1 -> 10.0   15.7 -> 12.6   18.5 -> 15.1   26.3 -> 22.8    41.0 -> 37.8    50.8 -> 48.1
//    16  12/2      14.5 -> 11.0   25.5 -> 24.1   39.5 -> 36.1   75.8 -> 73.4   133.3 -> 132.0    197 -> 197
// i.e. nothing to gain beyond, where a list also no longer fits beside the tiles of two workgroups a CU.  A launch of many
// workgroups whose lists are shared by query heads hides the list kernel better than each workgroup its own list, beyond some
// 1600 positions: B = 32, 28/4 at D = 64, one set of decisions, T = 1600 / 1792 / 2048 357 -> 361, 401 -> 413, 477 -> 497; B = 64,
// 12/2 305 -> 308, 347 -> 357, 416 -> 431; 16, 28/4 at D = 128, a set per KV head, 358 -> 355 and 431 -> 429 (1792, 2048).  Up to 4096
// workgroups, or with a set of decisions for every query head, it stays the other way: 8, 28/4 at D = 64, T = 2048 129 -> 130 (one
// set), 16, 12/2 109 -> 110, 256, 4/4 at D = 128 1115 -> 1081 (a set per head).
constexpr int OWN_BITS = 8;
constexpr int OWN_MAX = LIST_THREADS * OWN_BITS;
constexpr int OWN_ALWAYS = 1536;              // positions
constexpr int OWN_WORKGROUPS = 4096;          // beyond them, where lists are shared
static_assert(LIST_THREADS == RP_WAVES * NGC_WAVE, "a workgroup of the attention kernel makes its list");
template <bool OWN>
struct OwnList {
    static constexpr int SLOTS = 1, STEPS = 1;
    uint16_t key[1], death[1];
    uint32_t steps[1];
};
template <>
struct OwnList<true> {
    static constexpr int SLOTS = OWN_MAX + RP_KT;           // the list, padded to a whole tile
    static constexpr int STEPS = SLOTS / RP_MT;
    __align__(16) uint16_t key[SLOTS], death[SLOTS];        // padding: key 0, which nobody sees
    uint32_t steps[STEPS];
    int min_death[STEPS];
    uint16_t first_key[STEPS], last_key[STEPS];
    int counts[OWN_BITS * LIST_WAVES];
};

// Returns the length of the list.  Whole workgroup; ends on a barrier.
__device__ __forceinline__ int replay_own_list(OwnList<true> &own, const int32_t *death, int i0, int T)
{
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int last_pos = (i0 + RP_QT - 1 < T - 1) ? i0 + RP_QT - 1 : T - 1;
    int d[OWN_BITS];
#pragma unroll
    for (int i = 0; i < OWN_BITS; ++i) {
        const int j = i * LIST_THREADS + tid;
        d[i] = j <= last_pos ? death[j] : -1;                            // (a key no query of the tile sees)
    }
    if (tid < OwnList<true>::STEPS) {
        own.min_death[tid] = 0x7FFFFFFF;
        own.last_key[tid] = NO_KEY;
    }
    uint64_t seen[OWN_BITS];
#pragma unroll
    for (int i = 0; i < OWN_BITS; ++i) {
        seen[i] = __ballot(d[i] > i0);
        if (lane == 0) own.counts[i * LIST_WAVES + wv] = __popcll(seen[i]);
    }
    __syncthreads();
    const int mine = lane < OWN_BITS * LIST_WAVES ? own.counts[lane] : 0;
    const int upto = wave_incl_scan_i(mine);
#pragma unroll
    for (int i = 0; i < OWN_BITS; ++i) {
        if (i * LIST_THREADS > last_pos) break;                          // uniform
        const int before = __builtin_amdgcn_readlane(upto - mine, i * LIST_WAVES + wv);
        if (d[i] > i0) {
            const int j = i * LIST_THREADS + tid;
            const int slot = before + popc_below(seen[i]);
            own.key[slot] = (uint16_t)j;
            own.death[slot] = (uint16_t)(d[i] < 0xFFFF ? d[i] : 0xFFFF);
            atomicMin(&own.min_death[slot / RP_MT], d[i]);
            if (slot % RP_MT == 0) own.first_key[slot / RP_MT] = (uint16_t)j;
            if (slot % RP_MT == RP_MT - 1) own.last_key[slot / RP_MT] = (uint16_t)j;
        }
    }
    const int n_list = __builtin_amdgcn_readlane(upto, NGC_WAVE - 1);
    if (tid < RP_KT) {
        own.key[n_list + tid] = 0;
        own.death[n_list + tid] = 0;
    }
    __syncthreads();
    if (tid * RP_MT < n_list) own.steps[tid] = step_of(i0, T, own.first_key[tid], own.last_key[tid], own.min_death[tid]);
    __syncthreads();
    return n_list;
}

// OWN: trajectories of up to OWN_MAX positions; a workgroup makes its key list itself, in LDS (see replay_own_list()).
template <int D, bool OWN>
__global__ __launch_bounds__(RP_WAVES * 64) __attribute__((amdgpu_waves_per_eu(2)))
void replay_attn_kernel(ReplayArgs a)
{
    constexpr int ROW_BYTES = D * 2;
    constexpr int DT = D / 32;                             // 32-wide d tiles of the second product
    constexpr int KCH = D / 16;                            // 16-wide d chunks of the first product
    constexpr int TILE_LDS = RP_KT * ROW_BYTES;
    constexpr int PIECES = ROW_BYTES / 16;                 // 16-byte pieces per row
    constexpr int LOAD_ROWS = 64 / PIECES;                 // rows one wave-wide load brings
    constexpr int LOADS = RP_KT / (RP_WAVES * LOAD_ROWS);  // per wave, per tensor
    constexpr int STEPS = RP_KT / RP_MT;

    __shared__ __align__(16) unsigned char lds_k0[TILE_LDS], lds_k1[TILE_LDS], lds_v0[TILE_LDS], lds_v1[TILE_LDS];
    __shared__ __align__(16) int32_t lds_death[2][OWN ? 1 : RP_KT];
    __shared__ __align__(16) int32_t lds_kidx[2][OWN ? 1 : RP_KT];
    __shared__ OwnList<OWN> own;

    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id());
    const int li = lane & 31, half = lane >> 5;
    const int T = a.T;
    const int nqt = (T + RP_QT - 1) / RP_QT;
    // Workgroup -> (query tile, head, trajectory).  The hardware deals consecutive workgroups round-robin to the
    // 8 XCDs, and a query tile's work grows with its position, so the tile index is the slowest coordinate,
    // heaviest first: every XCD gets the same mix of tiles at every moment.  Within one tile index the KV group
    // (trajectory, KV head) is the fastest coordinate: with a multiple of 8 groups an XCD always works on the
    // same groups, whose K/V rows then stay in its own L2 for all their query heads and tiles.
    const int G = a.Hq / a.Hkv;
    const int nkv = a.B * a.Hkv;
    const int per_tile = G * nkv;
    const int qt = nqt - 1 - (int)(blockIdx.x / per_tile);
    const int rem = (int)(blockIdx.x % per_tile);
    const int kvp = rem % nkv;
    const int b = kvp / a.Hkv, hkv = kvp % a.Hkv;
    const int head = hkv * G + rem / nkv;
    const int hd = a.Hd == 1 ? 0 : hkv;
    const int i0 = qt * RP_QT;
    const int32_t *death = a.death + ((size_t)b * a.Hd + hd) * T;
    // bytes between consecutive tokens; a sequence's K (or V) spans less than 2^32 bytes (checked on the host),
    // so a row's offset from the sequence's first row fits 32 bits
    const uint32_t kv_row = (uint32_t)a.Hkv * ROW_BYTES;
    const unsigned char *kbase = a.k + ((size_t)b * T * a.Hkv + hkv) * ROW_BYTES;
    const unsigned char *vbase = a.v + ((size_t)b * T * a.Hkv + hkv) * ROW_BYTES;
    const size_t list = ((size_t)b * a.Hd + hd) * nqt + qt;
    const uint16_t *klist = OWN ? nullptr : a.klist + list * T;
    const uint32_t *info = OWN ? nullptr : a.steps + list * ((T + RP_MT - 1) / RP_MT);
    int n_list;
    if constexpr (OWN) n_list = replay_own_list(own, death, i0, T);
    else n_list = a.kcount[list];
    const int t_end = (n_list + RP_KT - 1) / RP_KT;

    // Rows of a tile go straight from memory to LDS: a wave-wide load brings LOAD_ROWS whole rows, lane after lane.
    // The K pieces of row r are stored at slot (piece ^ (r & SWZ)), so that reading one piece of 32 consecutive rows
    // meets every bank; the V pieces at (piece ^ v_swizzle(r)), so that reading 32 bytes of 4 consecutive rows does.
    constexpr int SWZ = PIECES - 1;
    auto v_swizzle = [](int r) { return (2 * r) & (PIECES < 16 ? SWZ : 7) ; };
    const int lrow = lane / PIECES, lslot = lane % PIECES;
    struct IdxStage {
        int key[LOADS];   // key index of the rows this lane copies
        int mine;         // the entry of list slot s0 + tid % RP_KT, as stored
    };
    // Slots past the list's end hold whatever the workspace held: any value is clamped to a valid key, and such slots
    // are switched off by the mask.
    auto load_idx = [&](int t, IdxStage &ix) {
        const int s0 = t * RP_KT;
#pragma unroll
        for (int r = 0; r < LOADS; ++r) {
            int slot = s0 + (wv * LOADS + r) * LOAD_ROWS + lrow;
            if constexpr (OWN) {
                ix.key[r] = (int)own.key[slot < OwnList<OWN>::SLOTS ? slot : 0];
            } else {
                slot = slot < T ? slot : T - 1;         // a list row has T slots
                ix.key[r] = (int)klist[slot];
            }
        }
        if constexpr (!OWN) {
            int sl = s0 + (tid & (RP_KT - 1));
            sl = sl < T ? sl : T - 1;
            ix.mine = (int)klist[sl];
        }
    };
    auto load_rows = [&](const IdxStage &ix, unsigned char *dk, unsigned char *dv) {
#pragma unroll
        for (int r = 0; r < LOADS; ++r) {
            const int row0 = (wv * LOADS + r) * LOAD_ROWS;                  // wave-uniform
            const int key = ix.key[r] < T ? ix.key[r] : T - 1;              // whatever the list holds, stay inside k / v
            const uint32_t at = (uint32_t)key * kv_row;
            const uint32_t kp = (uint32_t)(lslot ^ ((row0 + lrow) & SWZ)) * 16u;
            load_to_lds16(kbase + (at + kp), dk + row0 * ROW_BYTES);
            const uint32_t vp = (uint32_t)(lslot ^ v_swizzle(row0 + lrow)) * 16u;
            load_to_lds16(vbase + (at + vp), dv + row0 * ROW_BYTES);
        }
    };
    // key index and death position of the tile's rows, for the steps that need a mask; 0x7FFFFFFF = a key no query
    // comes after: slots past the end of the list
    struct MaskStage {
        int d, i;
    };
    auto load_mask = [&](const IdxStage &ix, MaskStage &ms) {
        if constexpr (OWN) return;
        ms.i = ix.mine;
        ms.d = death[ix.mine < T ? ix.mine : T - 1];
    };
    auto store_mask = [&](int t, int buf, const MaskStage &ms) {
        if constexpr (OWN) return;
        const bool inside = t * RP_KT + tid < n_list;
        if (tid < RP_KT) {
            lds_death[buf][tid] = inside ? ms.d : 0;
            lds_kidx[buf][tid] = inside ? ms.i : 0x7FFFFFFF;
        }
    };
    // scalar loads: wave-uniform, from memory an earlier launch wrote
    struct TileInfo {
        uint32_t step[STEPS];
    };
    const int last_step = (T + RP_MT - 1) / RP_MT - 1;
    auto load_info = [&](int t) {
        TileInfo ti;
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const int at = t * STEPS + st;
            if constexpr (OWN) {
                ti.step[st] = (uint32_t)__builtin_amdgcn_readfirstlane((int)own.steps[at < OwnList<OWN>::STEPS ? at : 0]);
                continue;
            }
            ti.step[st] = reinterpret_cast<const __attribute__((address_space(4))) uint32_t *>(
                (uintptr_t)info)[at < last_step ? at : last_step];
        }
        return ti;
    };

    IdxStage ix_a, ix_b;   // take turns, so that a stage being filled is never copied
    MaskStage ms;
    load_idx(0, ix_a);

    // ---- query operands: 32 positions per wave, lane % 32 = position ----------
    const int wave_q0 = i0 + wv * RP_QW;               // first query position of this wave
    const int qpos = wave_q0 + li;
    bf16x8 qop[KCH];
    {
        const int p = qpos < T ? qpos : T - 1;
        const unsigned char *qrow = a.q + (((size_t)b * T + p) * a.Hq + head) * ROW_BYTES;
#pragma unroll
        for (int c = 0; c < KCH; ++c)
            qop[c] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(qrow + c * 32 + half * 16));
    }
    load_rows(ix_a, lds_k0, lds_v0);
    load_mask(ix_a, ms);
    load_idx(1, ix_b);
    TileInfo here = load_info(0), next = load_info(1);

    f32x16 oacc[DT];
#pragma unroll
    for (int c = 0; c < DT; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[c][r] = 0.f;
    float m_run = RP_M_INIT, l_run = 0.f;

    // LDS offsets of this lane's operands.  K: piece 2c + half of row li.  V: a transposing read gives lane x of 16 the
    // column d0 + x of 4 rows if lane x points at the 4 values from d0 + 4 (x % 4) of row x / 4; the rows are the keys
    // its half contracts over in a 16-key chunk (4 half .. +3 and 8 + 4 half .. +3: the order the scores come in).
    uint32_t koff[KCH];
#pragma unroll
    for (int c = 0; c < KCH; ++c) koff[c] = (uint32_t)(li * ROW_BYTES + (((2 * c + half) ^ (li & SWZ)) * 16));
    uint32_t vrd[DT];
    {
        const int row = 4 * half + (lane & 15) / 4;       // + 16 kc + 8 g: the same row modulo 8 for every g, kc
#pragma unroll
        for (int c = 0; c < DT; ++c) {
            const int d0 = 32 * c + (lane & 16) + 4 * (lane & 3);
            vrd[c] = (uint32_t)(row * ROW_BYTES + (((d0 / 8) ^ v_swizzle(row)) * 16) + (d0 % 8) * 2);
        }
    }

    // `slot`: where the step's keys stand in the list (OWN)
    auto compute_step = [&](const unsigned char *lk, const unsigned char *lv, const int32_t *ldeath, const int32_t *lkidx,
                            int slot, bool full) {
        f32x16 sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.f;
        u32x4 kop[KCH];
#pragma unroll
        for (int c = 0; c < KCH; ++c) kop[c] = *reinterpret_cast<const u32x4 *>(lk + koff[c]);
        __builtin_amdgcn_sched_barrier(0);     // all requests first: the products then wait for one after the other
#pragma unroll
        for (int c = 0; c < KCH; ++c)
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[c]), qop[c], sc, 0, 0, 0);
        // The V rows are requested as soon as the first product has been issued (the K operand registers are free from
        // here on) and arrive while the soft-max arithmetic runs.
        __builtin_amdgcn_sched_barrier(0);
        u32x2 vop[2][DT][2];      // [16-key chunk][d tile][keys 4 half .. +3, 8 + 4 half .. +3]
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int c = 0; c < DT; ++c)
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    vop[kc][c][g] = read_transposed16(lv + vrd[c] + (16 * kc + 8 * g) * ROW_BYTES);
        __builtin_amdgcn_sched_barrier(0);
        // lane (q = li, half), register r: key 8 (r / 4) + 4 half + r % 4 of this step.  Raw scores; the (positive)
        // scale is applied inside the exponent's multiply-add, the running max lives in the scaled domain.
        if (!full) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                int4 d, j;
                if constexpr (OWN) {
                    const u32x2 dd = *reinterpret_cast<const u32x2 *>(&own.death[slot + 8 * g + 4 * half]);
                    const u32x2 jj = *reinterpret_cast<const u32x2 *>(&own.key[slot + 8 * g + 4 * half]);
                    d = int4{(int)(dd[0] & 0xFFFFu), (int)(dd[0] >> 16), (int)(dd[1] & 0xFFFFu), (int)(dd[1] >> 16)};
                    j = int4{(int)(jj[0] & 0xFFFFu), (int)(jj[0] >> 16), (int)(jj[1] & 0xFFFFu), (int)(jj[1] >> 16)};
                } else {
                    d = *reinterpret_cast<const int4 *>(&ldeath[8 * g + 4 * half]);
                    j = *reinterpret_cast<const int4 *>(&lkidx[8 * g + 4 * half]);
                }
                sc[4 * g + 0] = ((j.x <= qpos) & (qpos < d.x)) ? sc[4 * g + 0] : -INFINITY;
                sc[4 * g + 1] = ((j.y <= qpos) & (qpos < d.y)) ? sc[4 * g + 1] : -INFINITY;
                sc[4 * g + 2] = ((j.z <= qpos) & (qpos < d.z)) ? sc[4 * g + 2] : -INFINITY;
                sc[4 * g + 3] = ((j.w <= qpos) & (qpos < d.w)) ? sc[4 * g + 3] : -INFINITY;
            }
        }
        // scores are finite or -inf, never NaN (finite inputs)
        float tmx = sc[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tmx = max_no_nan(tmx, sc[r]);
        tmx = half_rows_max(tmx) * a.scale_log2e;
        // The sums are rescaled only when a maximum has outgrown the reference by 2^RP_LAZY: any reference gives the
        // same quotients, and probabilities up to 2^RP_LAZY lose nothing in fp32 or in two bf16 parts.
        if (__ballot(tmx > m_run + RP_LAZY)) {
            // tmx is finite wherever it is larger; exp2(-1e30 - finite) = 0 on a first visible tile
            const float m_new = max_no_nan(m_run, tmx);
            const float alpha = (m_new == m_run) ? 1.0f : fast_exp2(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int c = 0; c < DT; ++c) oacc[c] *= alpha;
            m_run = m_new;
        }
        const float neg_m = -m_run;
        uint32_t ph[8], pl[8];
        float psum = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p0 = fast_exp2(__builtin_fmaf(sc[2 * e], a.scale_log2e, neg_m));       // -inf gives 0
            const float p1 = fast_exp2(__builtin_fmaf(sc[2 * e + 1], a.scale_log2e, neg_m));
            psum += p0 + p1;
            const uint32_t b0 = __float_as_uint(p0), b1 = __float_as_uint(p1);
            const float r0 = p0 - __uint_as_float(b0 & 0xFFFF0000u);
            const float r1 = p1 - __uint_as_float(b1 & 0xFFFF0000u);
            ph[e] = __builtin_amdgcn_perm(b1, b0, 0x07060302u);                     // upper halves of b0, b1
            pl[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{r0, r1}, bf16x2));   // rounded
        }
        l_run += psum;
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const bf16x8 p_hi = __builtin_bit_cast(bf16x8, u32x4{ph[4 * kc], ph[4 * kc + 1], ph[4 * kc + 2], ph[4 * kc + 3]});
            const bf16x8 p_lo = __builtin_bit_cast(bf16x8, u32x4{pl[4 * kc], pl[4 * kc + 1], pl[4 * kc + 2], pl[4 * kc + 3]});
            bf16x8 v[DT];
#pragma unroll
            for (int c = 0; c < DT; ++c)
                v[c] = __builtin_bit_cast(bf16x8, u32x4{vop[kc][c][0][0], vop[kc][c][0][1], vop[kc][c][1][0], vop[kc][c][1][1]});
#pragma unroll
            for (int c = 0; c < DT; ++c) oacc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[c], p_hi, oacc[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < DT; ++c) oacc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[c], p_lo, oacc[c], 0, 0, 0);
        }
    };
    auto compute_tile = [&](int t, const TileInfo &ti, const unsigned char *lk, const unsigned char *lv, int buf) {
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const int at = t * STEPS + st;
            if (at * RP_MT >= n_list || wave_q0 >= T) break;       // (a last tile may have waves without queries)
            const int after = (int)(ti.step[st] & 0xFFu), from = (int)((ti.step[st] >> 8) & 0xFFu);
            const int until = (int)(ti.step[st] >> 16);
            if (wv < after) break;                                 // the list ascends: all later keys come after them too
            const bool full = wv >= from && wv < until;            // no mask
            compute_step(lk + st * RP_MT * ROW_BYTES, lv + st * RP_MT * ROW_BYTES, &lds_death[buf][OWN ? 0 : st * RP_MT],
                         &lds_kidx[buf][OWN ? 0 : st * RP_MT], at * RP_MT, full);
        }
    };

    // Per tile: tile t is computed from one pair of LDS buffers while the rows of tile t+1 travel into the other and the
    // list entries of tile t+2 are fetched.
    store_mask(0, 0, ms);
    lds_loads_done();
    int t = 0;
    while (t < t_end) {
        if (t + 1 < t_end) {
            load_rows(ix_b, lds_k1, lds_v1);
            load_mask(ix_b, ms);
            load_idx(t + 2, ix_a);
        }
        __builtin_amdgcn_sched_barrier(0);
        compute_tile(t, here, lds_k0, lds_v0, 0);
        __builtin_amdgcn_sched_barrier(0);
        here = next;
        next = load_info(t + 2);
        if (++t >= t_end) break;
        store_mask(t, 1, ms);
        lds_loads_done();
        if (t + 1 < t_end) {
            load_rows(ix_a, lds_k0, lds_v0);
            load_mask(ix_a, ms);
            load_idx(t + 2, ix_b);
        }
        __builtin_amdgcn_sched_barrier(0);
        compute_tile(t, here, lds_k1, lds_v1, 1);
        __builtin_amdgcn_sched_barrier(0);
        here = next;
        next = load_info(t + 2);
        if (++t >= t_end) break;
        store_mask(t, 0, ms);
        lds_loads_done();
    }

    // ---- normalise and write -------------------------------------------------
    const float l = half_rows_sum(l_run);
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    // Through LDS, so that a row's D values leave as whole cache lines (a wave's own 32 rows, one of the four tile
    // buffers each): 16-byte piece p of row r at slot p ^ r.
    __syncthreads();                                       // every wave is done with the tiles
    {
        constexpr int OP = D / 4;                          // 16-byte pieces per output row
        unsigned char *mine = wv == 0 ? lds_k0 : wv == 1 ? lds_k1 : wv == 2 ? lds_v0 : lds_v1;
        static_assert(RP_QW * D * 4 == TILE_LDS, "a wave's output rows fill one tile buffer");
#pragma unroll
        for (int c = 0; c < DT; ++c)
#pragma unroll
            for (int g = 0; g < 4; ++g) {   // register (c, 4g + i) holds d = 32 c + 8 g + 4 half + i
                const int piece = 8 * c + 2 * g + half;
                *reinterpret_cast<f32x4 *>(mine + li * (D * 4) + ((piece ^ li) & (OP - 1)) * 16) =
                    f32x4{oacc[c][4 * g] * inv, oacc[c][4 * g + 1] * inv, oacc[c][4 * g + 2] * inv, oacc[c][4 * g + 3] * inv};
            }
        constexpr int ROWS = 64 / OP;                      // rows per wave-wide store
        const int piece = lane % OP;
#pragma unroll
        for (int r0 = 0; r0 < RP_QW; r0 += ROWS) {
            const int r = r0 + lane / OP;
            const f32x4 x = *reinterpret_cast<const f32x4 *>(mine + r * (D * 4) + ((piece ^ r) & (OP - 1)) * 16);
            if (wave_q0 + r < T) {
                f32x4 *dst = reinterpret_cast<f32x4 *>(a.out + (((size_t)b * T + wave_q0 + r) * a.Hq + head) * D) + piece;
                __builtin_nontemporal_store(x, dst);
            }
        }
    }
}

}  // namespace ngc

using namespace ngc;

extern "C" size_t ngc_replay_workspace_bytes(int32_t B, int32_t T, int32_t Hkv)
{
    if (B <= 0 || T <= 0 || Hkv <= 0) return 0;
    const size_t nqt = (size_t)(T + RP_QT - 1) / RP_QT;
    size_t lists = (size_t)B * Hkv * nqt * T * sizeof(uint16_t);
    lists = (lists + 255) & ~(size_t)255;
    size_t counts = (size_t)B * Hkv * nqt * sizeof(int32_t);
    counts = (counts + 255) & ~(size_t)255;
    const size_t tiles_max = (size_t)(T + RP_MT - 1) / RP_MT;
    return 256 + lists + counts + (size_t)B * Hkv * nqt * tiles_max * sizeof(uint32_t);
}

extern "C" int ngc_replay_attn(const void *q, const void *k, const void *v, const int32_t *death,
                               int32_t B, int32_t T, int32_t Hq, int32_t Hkv, int32_t D,
                               int32_t death_per_head, float scale, float *out,
                               void *ws, size_t ws_bytes, void *stream)
{
    if (!q || !k || !v || !death || !out || !ws) return NGC_EINVAL;
    if ((reinterpret_cast<uintptr_t>(q) | reinterpret_cast<uintptr_t>(k) | reinterpret_cast<uintptr_t>(v) |
         reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(ws)) & 15u)
        return NGC_EINVAL;
    if (B <= 0 || T <= 0 || Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0) return NGC_EINVAL;
    if (D != 64 && D != 128) return NGC_EINVAL;
    if (!(scale > 0.f) || scale > 3.0e38f) return NGC_EINVAL;   // positive and finite: the kernel takes maxima before scaling
    if ((long long)((T + RP_QT - 1) / RP_QT) * Hq * B > 0x7FFFFFFFLL) return NGC_EUNSUPPORTED;   // one workgroup each
    if ((unsigned long long)T * Hkv * D * 2 > 0xFFFFFFFFull) return NGC_EUNSUPPORTED;   // 32-bit row offsets inside a sequence
    if (T > 65535) return NGC_EUNSUPPORTED;   // 16-bit key lists
    if (ws_bytes < ngc_replay_workspace_bytes(B, T, Hkv)) return NGC_ENOSPC;
    ReplayArgs ra;
    ra.q = reinterpret_cast<const unsigned char *>(q);
    ra.k = reinterpret_cast<const unsigned char *>(k);
    ra.v = reinterpret_cast<const unsigned char *>(v);
    ra.death = death;
    ra.out = out;
    ra.B = B; ra.T = T; ra.Hq = Hq; ra.Hkv = Hkv; ra.Hd = death_per_head ? Hkv : 1;
    ra.scale_log2e = scale * 1.4426950408889634f;
    hipStream_t st = (hipStream_t)stream;
    const int nqt = (T + RP_QT - 1) / RP_QT;
    size_t lists = (size_t)B * ra.Hd * nqt * T * sizeof(uint16_t);
    lists = (lists + 255) & ~(size_t)255;
    ra.klist = reinterpret_cast<uint16_t *>(reinterpret_cast<unsigned char *>(ws) + 256);
    ra.kcount = reinterpret_cast<int32_t *>(reinterpret_cast<unsigned char *>(ws) + 256 + lists);
    size_t counts = (size_t)B * ra.Hd * nqt * sizeof(int32_t);
    counts = (counts + 255) & ~(size_t)255;
    ra.steps = reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(ws) + 256 + lists + counts);
    // (the list needs 8 KB beside the tiles: two workgroups still share a CU)
    const bool own = T <= OWN_ALWAYS || (T <= OWN_MAX && (ra.Hd == Hq || (long long)nqt * Hq * B <= OWN_WORKGROUPS));
    if (!own) {
        hipLaunchKernelGGL(replay_lists_kernel, dim3(nqt, B * ra.Hd), dim3(LIST_THREADS), 0, st, ra);
        NGC_HIP_CHECK(hipGetLastError());
    }
    const void *fn = D == 128 ? (own ? reinterpret_cast<const void *>(&replay_attn_kernel<128, true>)
                                     : reinterpret_cast<const void *>(&replay_attn_kernel<128, false>))
                              : (own ? reinterpret_cast<const void *>(&replay_attn_kernel<64, true>)
                                     : reinterpret_cast<const void *>(&replay_attn_kernel<64, false>));
    return launch(fn, dim3((unsigned)(nqt * Hq * B)), dim3(RP_WAVES * 64), 0, st, ra);
}

