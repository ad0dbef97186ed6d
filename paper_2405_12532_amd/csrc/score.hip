// Ensemble attention weights of the recent window (Algorithm 1,
// A_e = weighted_avg(A[-L:, :-L], dim=-2); Section 3.2.1), uniform weights, mean over heads:
//   scores[t] = 1/(Hq*L') * sum_h sum_{i=S-L'}^{S-1} A_h[i, t],   L' = min(w, S),
// or, with averaging weights omega (Section 4.1: more recent rows may weigh more; one weight
// per row of a full window, a shorter sequence uses the last L' of them),
//   scores[t] = 1/Hq * sum_h sum_i omega_i A_h[i, t] / sum_i omega_i.
//
// The weights of the last L' rows are rebuilt from the logits and the row denominators the
// attention kernel saved (log2 domain), so the S x S matrix is never stored:
//   A_h[i,t] = 2^(c * q_i.k_t - lse_h[i]);  a weight enters as  - log2(omega_i)  next to lse_h[i].
//
// Bound: reading K once from HBM.  So the window's queries stand still and K streams past them.  A
// wavefront owns a RANGE of consecutive keys and a list of TASKS: one KV head times up to two 32-row blocks of
// the window (of one query head, or of two of the head's group).  Per task the queries go into registers once
// and the range's keys follow in tiles of 32; with S = Q K^T in the MFMA accumulator a lane holds 16 window
// rows of ONE key, so the sum over the rows is a sum of registers, and a key's running sum over the tasks is
// one LDS word per half-wavefront.  Queries and keys are elements of one stream of 32-row tiles, loaded
// straight into a private ring of two LDS slots (global_load_lds, 16-byte chunks XOR-swizzled against bank
// conflicts), copied into registers, and the slot is requested again at once: no barrier until the end, where
// the wavefronts of a workgroup (they share out the tasks of one range) add their sums in a fixed order.
// No atomics: the result is bit-reproducible.  All S columns are written, the window's own columns too (so
// each sequence's scores sum to one).
// (Loads into registers pass the vector L1 at a quarter of the rate of LDS-direct loads, hence the ring.)
// Measured against the walk this one replaced (a workgroup per 64 keys with the keys standing still and every window
// row read once per 64 keys), us per launch: 64 x 2048, 32 heads 253 -> 188 (5.7 TB/s of K), 64 x 359 103 -> 49, 8 x 2048
// 45 -> 31, 4 x 32768 with 64/8 heads and w = 128 493 -> 370, one 2048-token prompt 20 -> 10, statistics of a
// 1537-row cache 49 -> 9.
//
// The same walk serves the generation-phase update of the cache (Algorithm 1 with a non-empty
// cache; Section 4.1): there the queries of the recent rows come in a buffer of their own
// ([B, w, Hq, d], right-aligned) and no attention pass has left row denominators behind, so a
// first pass (kStats; S^T = K Q^T there, a lane follows one window row over its keys) writes, per range, every
// window row's maximum and sum of exponentials, a small kernel folds them into denominators, and the score pass
// runs as above.  (Sequences of 2048 keys at most may get theirs by one walk instead: window_device.h, plan_update below.)
//
// Small batches.  When ranges times wavefronts leave the chip idle, the tasks of a range are also split over
// gridDim.y workgroups that write partial sums, one row of `sums` each; the selection kernel, which reads
// every score anyway, adds the rows up in order.
#include <float.h>
#include <math.h>

#include "score_device.h"

namespace pyr {
namespace {

constexpr int kMaxWaves = 8;         // wavefronts of a workgroup
constexpr int kMaxRangeTiles = 12;   // 32-key tiles of a range: eight wavefronts then fill the 160 KB of LDS at d = 128
constexpr int kRowArea = 512;        // LDS of one row block's denominators and weights, 64 floats each (32 used)
constexpr int kSlots = 2;            // tiles of a wavefront's ring

enum Mode { kScores = 0, kScoresWeighted = 1, kStats = 2 };

// Which range a workgroup takes.  Consecutive workgroup ids go round robin over the XCDs and, inside one, over its four shader
// engines, whether a workgroup finds work there or not.  A grid with places for ranges that do not exist therefore fills
// some engines' compute units twice while others stand idle (24 sequences of 235...2226 tokens on 40 heads, w = 256, ranges of
// 6 tiles: 175 workgroups, 354 us; 7 tiles, 152 workgroups, 232 us).
enum Order {
    kSeqPerXcd = 0,      // equal lengths, a multiple of the XCD count: all ranges of a sequence on one XCD
    kEqual = 1,          // as many ranges in every sequence: range after range, sequence after sequence
    kPacked = 2,         // ragged: the same, and the workgroup counts the ranges in front of it
    kGrid = 3,           // ragged: ranges_per_seq places for each sequence
};
// Counting costs a workgroup 0.3 us per 64 sequences.  Measured, packed / grid (us): 17 sequences of 3292...7710 tokens, 24
// heads, w = 512 404 / 691, 97 of 45...71, 24 heads, 12.0 / 18.6, 48 of 30...400 26 / 37, 128 of 60...1500 171 / 214; but 192 of 16...120,
// 8 heads, d = 64, 7.5 / 7.3, 256 12.5 / 10.7, 800 of 30...400 231 / 231.
constexpr int kMaxPackedSeqs = 256, kMaxPackedShortSeqs = 128, kShortLen = 256;
constexpr int kEnginesPerXcd = 4;

struct StripArgs {
    const uint16_t* q;
    const uint16_t* k;
    const float* lse;
    const int32_t* seq_offsets;
    int32_t n_seqs, group, n_kv_heads, w;     // (group: query heads per KV head)
    int32_t range_tiles, ranges_per_seq;      // tiles of a range; ranges of the longest sequence
    int32_t order, xcds, turn, head_step;     // order of the ranges over the workgroups, of the heads over the ranges
    int32_t q_window;                         // 0: q and lse by packed row; else by (sequence, window slot)
    float c;
    const float* row_weights;
    union {                                   // (arguments of 112 bytes and less, implicit ones among them, are 0.7 us less host time a launch)
        float* sums;                          // [groups, total_tokens]
        float2* part;                         // kStats: [range, sequence, query head, window slot]
    };
    int32_t total_tokens;
    int32_t waves, groups;                    // of a workgroup; workgroups a range's tasks are split over (the grid's y)
};
static_assert(sizeof(StripArgs) <= 112, "short arguments");

template <int D>
constexpr int wave_lds_bytes(int range_tiles) { return kSlots * 32 * D * 2 + 2 * kRowArea + 256 * range_tiles; }

// A position in a wavefront's stream of tiles.  All fields wave-uniform.
struct Cursor {
    int task;        // number of the task among all
    int hd, pair;    // KV head (before the rotation) and row-block pair of the task
    int e;           // element of the task: its row blocks, then its key tiles
};

// Accumulator register r of a lane: row 8*(r >> 2) + 4*gl + (r & 3) of the A operand, column li of the B operand.

// Score pass (rows: window rows, column: key): the key's probabilities over the 16 rows the lane holds, added up.
// nl: minus the rows' denominators.  Without kPlain, rows before the key are masked (q0: position of the lane's row 0).
template <bool kPlain>
__device__ __forceinline__ float tile_sum(const f32x16& s, float c, const float (&nl)[16], int key, int q0) {
    float p4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, nl[r]));
        if (!kPlain) p = key <= q0 + 8 * (r >> 2) + (r & 3) ? p : 0.f;
        p4[r & 3] += p;
    }
    return (p4[0] + p4[1]) + (p4[2] + p4[3]);
}

// Statistics pass (rows: keys, column: window row): the row's running maximum and sum of exponentials.  Without kPlain
// keys past the row, and rows past the sequence, are masked (key0: position of the lane's key 0).  m_run starts at the lowest
// finite value, so that a row whose keys so far all have logits of -inf has the sum zero and not the NaN of -inf - -inf.
template <bool kPlain>
__device__ __forceinline__ void tile_stats(f32x16& s, float c, int key0, int qpos, int S, float& m_run, float& l_run) {
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        s[r] *= c;
        if (!kPlain) s[r] = key0 + 8 * (r >> 2) + (r & 3) <= qpos && qpos < S ? s[r] : -INFINITY;
        mx = fmaxf(mx, s[r]);
    }
    const float m_new = fmaxf(m_run, mx);
    float l4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) l4[r & 3] += __builtin_amdgcn_exp2f(s[r] - m_new);
    l_run = l_run * __builtin_amdgcn_exp2f(m_run - m_new) + ((l4[0] + l4[1]) + (l4[2] + l4[3]));
    m_run = m_new;
}

// kStats writes part[((range * B + b) * Hq + h) * w + slot] = (max, sum of 2^(x - max)) over the
// range's visible keys, x = c * q.k, for every row that sees the range, and touches neither lse nor sums.
template <int D, int kMode>
__global__ __launch_bounds__(kMaxWaves * 64, D == 64 ? 3 : 2) void strip_kernel(StripArgs a) {
    constexpr bool kWeighted = kMode == kScoresWeighted;
    constexpr int kSteps = D / 16;
    constexpr int kChunks = D / 8;                  // 16-byte chunks per row
    constexpr int kRowBytes = D * 2;
    constexpr int kRowsPerLoad = 64 / kChunks;      // rows one load instruction covers
    constexpr int kTileBytes = 32 * kRowBytes;
    constexpr int kTileLoads = kTileBytes / 1024;   // load instructions of a tile
    constexpr int kRowLoads = kMode == kStats ? 0 : kWeighted ? 2 : 1;      // ... of a task's denominators and weights
    extern __shared__ __align__(1024) char smem[];

    const int lane = threadIdx.x & 63, waves = a.waves;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int li = lane & 31, gl = lane >> 5;
    // ---- which sequence, which range (uniform over the workgroup)
    int b, range, row0, S;
    if (a.order == kPacked) {
        // lane l counts the ranges of sequence first + l; a sum over the wavefront says which of them holds this workgroup's
        const int range_keys = 32 * a.range_tiles;
        int left = (int)blockIdx.x;
        for (int first = 0;; first += 64) {
            if (first >= a.n_seqs) return;
            const bool is_seq = first + lane < a.n_seqs;
            const int from = is_seq ? a.seq_offsets[first + lane] : 0, len = is_seq ? a.seq_offsets[first + lane + 1] - from : 0;
            const int mine = (len + range_keys - 1) / range_keys;
            int incl = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int up = __shfl_up(incl, d);
                if (lane >= d) incl += up;
            }
            const uint64_t past = __ballot(incl > left);
            if (past != 0) {
                const int at = __ffsll((unsigned long long)past) - 1;
                b = first + at;
                range = left - (__builtin_amdgcn_readlane(incl, at) - __builtin_amdgcn_readlane(mine, at));
                row0 = __builtin_amdgcn_readlane(from, at);
                S = __builtin_amdgcn_readlane(len, at);
                break;
            }
            left -= __builtin_amdgcn_readlane(incl, 63);
        }
    } else {
        const int id = (int)blockIdx.x, slot = a.order == kSeqPerXcd ? (int)((uint32_t)id / (uint32_t)a.xcds) : id;
        const int at = (int)((uint32_t)slot / (uint32_t)a.ranges_per_seq);
        b = a.order == kSeqPerXcd ? at * a.xcds + (id - slot * a.xcds) : at;
        if (b >= a.n_seqs) return;
        range = slot - at * a.ranges_per_seq;
        if (a.turn) range = (int)((uint32_t)(range + at) % (uint32_t)a.ranges_per_seq);       // (the same ranges of the sequence, from its at-th on)
        row0 = a.seq_offsets[b];
        S = a.seq_offsets[b + 1] - row0;
    }
    const int key_base = range * a.range_tiles * 32;
    if (key_base >= S) return;
    const int n_tiles = min(a.range_tiles, (S - key_base + 31) / 32);
    const int L = min(a.w, S);
    const int first_row = S - L;                      // local position of the first window row
    const int q_row_base = a.q_window ? b * a.w + (a.w - L) : row0 + first_row;   // row of q / lse holding the first window row
    const int n_rb = (L + 31) / 32;
    const int group = a.group, n_q_heads = group * a.n_kv_heads;
    const int blocks = group * n_rb;                  // row blocks per KV head
    const int pairs = (blocks + 1) / 2;
    // This workgroup's share of the tasks, dealt to its wavefronts one by one.  (All that stands in front of the first load is the time of
    // every workgroup: unsigned 32-bit divisions, and as few as can be, which the launcher's bounds allow: fewer than 2^26 tasks, kMaxScoreGroups
    // shares.  With signed and 64-bit ones and two per row block, 8 x 352 on 64/8 heads, w = 32 15.2 us, now 14.6.)
    const uint32_t n_tasks = (uint32_t)(a.n_kv_heads * pairs), groups = (uint32_t)a.groups;
    const int t_begin = (int)(n_tasks * blockIdx.y / groups), t_end = (int)(n_tasks * (blockIdx.y + 1) / groups);
    // Where the launcher asks for it (head_step != 0), neighbouring ranges start their walks head_step heads apart (a step of 8: at
    // two different heads of 16, four of 32; an odd step: at all of them): workgroups that run side by side then read different
    // columns of their token rows, which spreads them over the memory channels when the rows are a power of two apart.
    const int head_rot = a.head_step == 0 ? 0 : (int)((uint32_t)(range * a.head_step) % (uint32_t)a.n_kv_heads);

    // sum of the weights in use (fixed order: every lane strides over them, then a butterfly).
    // These are the only ordinary loads of the kernel and they are complete before the first
    // LDS-direct load is issued: the wait counts below assume no other load is in flight.
    float weight_sum = (float)L;
    if (kWeighted) {
        float part = 0.f;
        for (int j = lane; j < L; j += 64) part += a.row_weights[a.w - L + j];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) part += __shfl_xor(part, m, 64);
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(part) : : "memory");
        weight_sum = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, part)));   // uniform: a scalar register
    }

    // ---- this wavefront's LDS: ring, two row areas (denominators, then weights), key sums
    const int wave_bytes = wave_lds_bytes<D>(a.range_tiles);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    const uint32_t ring = lds0 + wave * wave_bytes;
    const uint32_t rows_at = ring + kSlots * kTileBytes;
    const uint32_t sums_at = rows_at + 2 * kRowArea;

    // ---- load side: lane -> (row inside an instruction's row group, physical chunk).  The LDS
    // slot of a lane is fixed by the instruction, so the swizzle picks the global chunk.
    const int ld_row = lane / kChunks, ld_chunk = lane % kChunks;
    const uint32_t k_row_bytes = (uint32_t)a.n_kv_heads * kRowBytes, q_row_bytes = (uint32_t)n_q_heads * kRowBytes;
    auto load_tile = [&](const char* base, uint32_t row_bytes, int last_row, uint32_t to) {      // rows past the last re-read it
#pragma unroll
        for (int i = 0; i < kTileLoads; ++i) {
            const int row = kRowsPerLoad * i + ld_row;
            // (24-bit multiply: full rate, where the 32-bit one takes four times as long; rows and strides are far below 2^24)
            lds_dma(base, __umul24((uint32_t)min(row, last_row), row_bytes) + 16 * (ld_chunk ^ (row & (kChunks - 1))), to + 1024 * i,
                    false);
        }
    };
    // a full key tile's offsets stay in registers: the loop over the keys issues nothing but its loads
    uint32_t k_off[kTileLoads];
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) {
        const int row = kRowsPerLoad * i + ld_row;
        k_off[i] = __umul24((uint32_t)row, k_row_bytes) + 16 * (ld_chunk ^ (row & (kChunks - 1)));
    }
    auto kv_head = [&](const Cursor& cu) { const int h = cu.hd + head_rot; return h >= a.n_kv_heads ? h - a.n_kv_heads : h; };
    auto n_blk = [&](const Cursor& cu) { return min(2, blocks - 2 * cu.pair); };
    auto next_task = [&](Cursor& cu) {
        cu.task += waves;
        cu.pair += waves;
        while (cu.pair >= pairs) {
            cu.pair -= pairs;
            ++cu.hd;
        }
    };
    // Request the element at the cursor into ring slot `slot` and move on; returns the number of load
    // instructions issued (0: the stream has ended).
    int of[2] = {0, 0}, rb[2] = {0, 0};               // the requested row blocks: query head of the KV head's, place in the window
    auto request = [&](Cursor& cu, int slot) -> int {
        if (cu.task >= t_end) return 0;
        const uint32_t to = ring + slot * kTileBytes;
        const int kvh = kv_head(cu), nb = n_blk(cu);
        int n = kTileLoads;
        if (cu.e < nb) {
            int of_blk, rb_blk;
            if (cu.e == 0) {
                of_blk = (int)((uint32_t)(2 * cu.pair) / (uint32_t)n_rb);
                rb_blk = 2 * cu.pair - of_blk * n_rb;
                of[0] = of_blk;
                rb[0] = rb_blk;
            } else {                                  // the block behind it
                const bool next = rb[0] + 1 == n_rb;
                of_blk = next ? of[0] + 1 : of[0];
                rb_blk = next ? 0 : rb[0] + 1;
                of[1] = of_blk;
                rb[1] = rb_blk;
            }
            const int h = kvh * group + of_blk;
            if (kMode != kStats) {
                const uint32_t row = (uint32_t)min(li, L - 1 - 32 * rb_blk), area = rows_at + cu.e * kRowArea;
                lds_dma((const char*)(a.lse + (size_t)(q_row_base + 32 * rb_blk) * n_q_heads + h), __umul24(row, (uint32_t)n_q_heads * 4), area, true);
                if (kWeighted) lds_dma((const char*)(a.row_weights + (a.w - L) + 32 * rb_blk), row * 4, area + 256, true);
                n += kRowLoads;
            }
            load_tile((const char*)(a.q + ((size_t)(q_row_base + 32 * rb_blk) * n_q_heads + h) * D), q_row_bytes, L - 1 - 32 * rb_blk, to);
        } else {
            const int key = key_base + 32 * (cu.e - nb);
            const char* base = (const char*)(a.k + ((size_t)(row0 + key) * a.n_kv_heads + kvh) * D);
            if (key + 32 <= S) {
#pragma unroll
                for (int i = 0; i < kTileLoads; ++i) lds_dma(base, k_off[i], to + 1024 * i, false);
            } else {
                load_tile(base, k_row_bytes, S - 1 - key, to);
            }
        }
        if (++cu.e == nb + n_tiles) {
            cu.e = 0;
            next_task(cu);
        }
        return n;
    };
    // wait until the element in front of the one requested last (`behind` instructions) has landed
    auto wait_front = [&](int behind) {
        if (behind == 0) wait_loads<0>();
        else if (kRowLoads == 0 || behind == kTileLoads) wait_loads<kTileLoads>();
        else wait_loads<kTileLoads + kRowLoads>();
    };

    // ---- fragment side: operand row li, logical chunk 2*ks + gl
    auto copy_tile = [&](bf16x8 (&f)[kSteps], int slot) {
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks) {
            const uint32_t p = ring + slot * kTileBytes + li * kRowBytes + (((2 * ks + gl) ^ (li & (kChunks - 1))) << 4);
            f[ks] = *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)p;
        }
    };

    // minus the denominators of row block rb (accumulator order), weights included
    auto copy_rows = [&](float (&nl)[16], int j, int rb) {
        if (kMode == kStats) return;
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            const uint32_t p = rows_at + j * kRowArea + 4 * (8 * a4 + 4 * gl);
            const f32x4 d4 = *(const f32x4 __attribute__((address_space(3)))*)(uintptr_t)p;
            f32x4 w4 = {1.f, 1.f, 1.f, 1.f};
            if (kWeighted) w4 = *(const f32x4 __attribute__((address_space(3)))*)(uintptr_t)(p + 256);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float x = -d4[i];
                if (kWeighted) x += __builtin_amdgcn_logf(w4[i]);      // omega * 2^x = 2^(x + log2 omega); a zero weight gives 2^-inf = 0
                nl[4 * a4 + i] = 32 * rb + 8 * a4 + 4 * gl + i < L ? x : -INFINITY;      // a row past the window adds nothing
            }
        }
    };

    auto product = [&](const bf16x8& qv, const bf16x8& kv, const f32x16& acc) {
        return kMode == kStats ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(kv, qv, acc, 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x16_bf16(qv, kv, acc, 0, 0, 0);
    };

    if (t_begin + wave >= t_end) {
        for (int t = 0; t < n_tiles; ++t) *(lfloat_t)(uintptr_t)(sums_at + 256 * t + 4 * lane) = 0.f;
    } else {
        Cursor now{t_begin + wave, 0, 0, 0};
        now.hd = (int)((uint32_t)now.task / (uint32_t)pairs);
        now.pair = now.task - now.hd * pairs;
        Cursor ahead = now;
        request(ahead, 0);
        int behind = request(ahead, 1);
        int slot = 0;
        bool first_task = true;
        for (; now.task < t_end; next_task(now)) {
            const int kvh = kv_head(now), nb = n_blk(now);
            bf16x8 qf[2][kSteps];
            float nl[2][16];                          // minus the rows' denominators (log2 domain), weights included
            int q_lo[2];                              // sequence positions of the row blocks' first rows
            // (the task's first two elements have been requested, no row block of the next task: it has a key tile at least)
            const int rb0 = rb[0], rb1 = rb[1], of0 = of[0], of1 = of[1];
            q_lo[0] = first_row + 32 * rb0;
            q_lo[1] = first_row + 32 * rb1;
            wait_front(behind);
            copy_tile(qf[0], slot);
            copy_rows(nl[0], 0, rb0);
            wait_lds();                               // in registers: the slot is free
            behind = request(ahead, slot);
            slot ^= 1;
            if (nb == 2) {
                wait_front(behind);
                copy_tile(qf[1], slot);
                copy_rows(nl[1], 1, rb1);
                wait_lds();
                behind = request(ahead, slot);
                slot ^= 1;
            }
            float m_run[2] = {-FLT_MAX, -FLT_MAX}, l_run[2] = {0.f, 0.f};         // kStats: this lane's window rows
            for (int t = 0; t < n_tiles; ++t) {
                bf16x8 kf[kSteps];
                wait_front(behind);
                copy_tile(kf, slot);
                wait_lds();
                behind = request(ahead, slot);
                slot ^= 1;
                const int key0 = key_base + 32 * t;
                float v = 0.f;
                if (nb == 2 && key0 + 31 <= q_lo[0] && key0 + 31 <= q_lo[1]) {
                    // the common tile: two row blocks, every row sees every key; their chains of products side by side
                    f32x16 s[2];
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int r = 0; r < 16; ++r) s[j][r] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < kSteps; ++ks)
#pragma unroll
                        for (int j = 0; j < 2; ++j) s[j] = product(qf[j][ks], kf[ks], s[j]);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        if (kMode == kStats) tile_stats<true>(s[j], a.c, 0, 0, 0, m_run[j], l_run[j]);
                        else v += tile_sum<true>(s[j], a.c, nl[j], 0, 0);
                } else {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        if ((j == 1 && nb < 2) || key0 > q_lo[j] + 31) continue;      // (the block precedes the keys)
                        f32x16 s;
#pragma unroll
                        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
                        for (int ks = 0; ks < kSteps; ++ks) s = product(qf[j][ks], kf[ks], s);
                        if (kMode == kStats) tile_stats<false>(s, a.c, key0 + 4 * gl, q_lo[j] + li, S, m_run[j], l_run[j]);
                        else v += tile_sum<false>(s, a.c, nl[j], key0 + li, q_lo[j] + 4 * gl);
                    }
                }
                if (kMode != kStats) {
                    lfloat_t at = (lfloat_t)(uintptr_t)(sums_at + 256 * t + 4 * lane);
                    *at = first_task ? v : *at + v;
                }
            }
            first_task = false;
            if (kMode == kStats) {
                // this half-wavefront's keys and the other's
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if (j == 1 && nb < 2) continue;
                    const float mo = __shfl_xor(m_run[j], 32, 64), so = __shfl_xor(l_run[j], 32, 64);
                    const float m_all = fmaxf(m_run[j], mo);
                    const int rb = j ? rb1 : rb0;
                    if (gl == 0 && 32 * rb + li < L && key_base <= q_lo[j] + li) {      // every range that the fold reads for this row
                        const float total = l_run[j] * __builtin_amdgcn_exp2f(m_run[j] - m_all) + so * __builtin_amdgcn_exp2f(mo - m_all);
                        const int h = kvh * group + (j ? of1 : of0), at = (a.w - L) + 32 * rb + li;
                        a.part[(((size_t)range * a.n_seqs + b) * n_q_heads + h) * a.w + at] = make_float2(m_all, total);   // 32 rows: 256 consecutive bytes
                    }
                }
            }
        }
    }
    // every load issued above has been waited for: nothing is in flight towards LDS here
    if (kMode == kStats) return;

    // ---- the sums of the two half-wavefronts (16 window rows of a block each) and of the wavefronts, fixed order
    const float norm = 1.0f / ((float)n_q_heads * weight_sum);
    __syncthreads();
    float* dst = a.sums + (size_t)blockIdx.y * a.total_tokens + row0 + key_base;
    for (int x = threadIdx.x; x < 32 * n_tiles && key_base + x < S; x += 64 * waves) {
        const uint32_t at = lds0 + kSlots * kTileBytes + 2 * kRowArea + 256 * (x >> 5) + 4 * (x & 31);
        float sum = 0.f;
        for (int wv = 0; wv < waves; ++wv) {
            const uint32_t p = at + wv * wave_bytes;
            sum += *(const lfloat_t)(uintptr_t)p + *(const lfloat_t)(uintptr_t)(p + 128);
        }
        dst[x] = sum * norm;
    }
}

// Row denominators of the window rows from the per-range statistics: for every (sequence,
// window slot, head) fold (max, sum) over the ranges the row can see, in a fixed order:
//   lse = M + log2(sum_r sum_r * 2^(m_r - M)),  M = max_r m_r.
// Bound: the latency of the loads, so eight lanes share a row (lane u takes ranges u, u + 8, ..., four of them in flight)
// and their eight results are folded through LDS; where a row has four ranges at most, one lane has them all in flight.
constexpr int kFoldThreads = 256;

__device__ __forceinline__ void fold_one(float& m_run, float& s_run, float m, float s) {
    const float m_new = fmaxf(m_run, m);
    if (m_new > -INFINITY) {      // (2^-inf = 0 for the side that is still empty)
        s_run = s_run * __builtin_amdgcn_exp2f(m_run - m_new) + s * __builtin_amdgcn_exp2f(m - m_new);
        m_run = m_new;
    }
}

template <int kFoldLanes>
__global__ __launch_bounds__(kFoldThreads) void fold_stats_kernel(const float2* __restrict__ part,
                                                         const int32_t* __restrict__ seq_offsets, int32_t n_seqs,
                                                         int32_t n_q_heads, int32_t w, int32_t range_keys, float* __restrict__ lse_win) {
    constexpr int kFoldRows = kFoldThreads / kFoldLanes;
    __shared__ float2 folded[kFoldLanes][kFoldRows + 1];
    const int row = threadIdx.x % kFoldRows, u = threadIdx.x / kFoldRows;
    const int64_t idx = (int64_t)blockIdx.x * kFoldRows + row;          // (b, h, slot), slot fastest, as in part
    const int64_t n_rows = (int64_t)n_seqs * w * n_q_heads;
    int slot = 0, h = 0, b = 0, n_ranges = 0;
    if (idx < n_rows) {
        slot = (int)(idx % w);
        h = (int)((idx / w) % n_q_heads);
        b = (int)(idx / ((int64_t)n_q_heads * w));
        const int S = seq_offsets[b + 1] - seq_offsets[b];
        const int L = min(w, S), i = slot - (w - L);
        if (i >= 0) n_ranges = (S - L + i) / range_keys + 1;            // ranges row S-L+i can see (0: slot not in use)
    }
    float m_run = -INFINITY, s_run = 0.f;
    constexpr int kAhead = 4;
    for (int r0 = u; r0 < n_ranges; r0 += kFoldLanes * kAhead) {
        float2 p[kAhead];
#pragma unroll
        for (int v = 0; v < kAhead; ++v) p[v] = part[(size_t)min(r0 + kFoldLanes * v, n_ranges - 1) * n_rows + idx];
#pragma unroll
        for (int v = 0; v < kAhead; ++v)
            if (r0 + kFoldLanes * v < n_ranges) fold_one(m_run, s_run, p[v].x, p[v].y);
    }
    if (kFoldLanes > 1) {
        folded[u][row] = make_float2(m_run, s_run);
        __syncthreads();
    }
    if (u != 0 || idx >= n_rows) return;
    for (int v = 1; v < kFoldLanes; ++v) fold_one(m_run, s_run, folded[v][row].x, folded[v][row].y);
    lse_win[((size_t)b * w + slot) * n_q_heads + h] = n_ranges > 0 ? m_run + __builtin_amdgcn_logf(s_run) : 0.f;
}

template <int kFoldLanes>
int launch_fold(const float2* part, const int32_t* seq_offsets_dev, const pyr_shape& s, int32_t w, int32_t range_keys, float* lse_win,
                hipStream_t stream) {
    constexpr int64_t kRows = kFoldThreads / kFoldLanes;
    const int64_t blocks = ((int64_t)s.n_seqs * w * s.n_q_heads + kRows - 1) / kRows;
    if (blocks >= (int64_t)1 << 31) return PYR_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((fold_stats_kernel<kFoldLanes>), dim3((unsigned)blocks), dim3(kFoldThreads), 0, stream, part, seq_offsets_dev,
                       s.n_seqs, s.n_q_heads, w, range_keys, lse_win);
    return check_launch();
}

// What the plan needs to know of a batch: tiles in all, and how many ranges there are if a range has that many tiles (counted in fp32).
struct BatchCut {
    bool equal;
    double tiles;
    int64_t ranges[kMaxRangeTiles + 1];
};

Order pick_order(const pyr_shape& s, bool equal, int64_t ranges, int64_t ranges_per_seq, int xcds) {
    if (equal && s.n_seqs % xcds == 0) return kSeqPerXcd;
    if (ranges == s.n_seqs * ranges_per_seq) return kEqual;
    return s.n_seqs <= (s.max_seqlen > kShortLen ? kMaxPackedSeqs : kMaxPackedShortSeqs) ? kPacked : kGrid;
}

int64_t count_ranges(const int32_t* seq_offsets_host, int32_t n_seqs, int32_t range_keys) {
    int64_t n = 0;
    for (int32_t b = 0; b < n_seqs; ++b) n += (seq_offsets_host[b + 1] - seq_offsets_host[b] + range_keys - 1) / range_keys;
    return n;
}

BatchCut cut_batch(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t min_seqlen) {
    BatchCut cut{};
    cut.equal = min_seqlen == s.max_seqlen;
    if (cut.equal) {
        cut.tiles = (double)s.n_seqs * ((s.max_seqlen + 31) / 32);
        for (int nt = 1; nt <= kMaxRangeTiles; ++nt) cut.ranges[nt] = (int64_t)s.n_seqs * (((s.max_seqlen + 31) / 32 + nt - 1) / nt);
        return cut;
    }
    // 256 sequences at a time, without divisions: the loops over them run on the host's vector unit
    constexpr int kBlock = 256;
    float tiles[kBlock];
    for (int32_t b0 = 0; b0 < s.n_seqs; b0 += kBlock) {
        const int n = s.n_seqs - b0 < kBlock ? s.n_seqs - b0 : kBlock;
        float sum_tiles = 0.f;
        for (int i = 0; i < n; ++i) sum_tiles += tiles[i] = (float)((seq_offsets_host[b0 + i + 1] - seq_offsets_host[b0 + i] + 31) / 32);
        cut.tiles += sum_tiles;
        for (int nt = 1; nt <= kMaxRangeTiles; ++nt) {
            const float inv = 1.0f / nt, up = (nt - 0.5f) * inv;
            int32_t sum = 0;
            for (int i = 0; i < n; ++i) sum += (int32_t)(tiles[i] * inv + up);
            cut.ranges[nt] += sum;
        }
    }
    return cut;
}

// The cut with the lowest cost, in microseconds, of two limits joined smoothly (the fourth root of the sum of fourth powers):
// - The chain.  An engine's compute units take its workgroups in rounds.  A round takes 1.9 until its first tiles are there, then a
//   wavefront goes through its tasks, each the range's tiles and the task's row blocks, one step after the other.  A step takes
//   `alone` where latency sets the time, and `shared` times the wavefronts of its SIMD where they wait for each other.
// - The stream.  A compute unit's share of the memory system delivers a tile of K in 0.35 from HBM, in 0.136 from L2 to every
//   further task of its KV head, and a tile of Q in 0.063 (d = 128; half of it at d = 64); a last round that leaves compute units
//   without a workgroup costs a tenth of what it leaves idle.
// Places for tiles that are not there (ranges that do not divide the sequences) add a tenth of their share.
// A row of partial sums costs the selection, one workgroup per sequence, 0.1 and 0.05 per 1000 tokens.
// The constants are fitted to 710 calls (d = 64 and 128, eleven head shapes, w = 16...512, one 16-token sequence to 200 x 655 and
// 3 x 40000 tokens, equal and ragged lengths, 173 of them powers of two), each timed with all cuts: nine in ten predictions near a
// call's best lie within 14 %, and the cut chosen takes 0.9 % longer than the best one in the mean, at most 6 % in 95 of 100
// calls (lengths of powers of two 0.3 %); the generation phase, with split tasks, 0.8 % (scores) and 1.3 % (statistics) of
// the whole call.  Fewer than four wavefronts per workgroup never were the best choice where there are tasks for four, nor fewer
// than eight where a KV head has 48 tasks or more, which then share its tiles (161 x 814, w >= 814, on 48/8 heads: eight 1880 us, four 2170).
StripPlan plan_strip(const pyr_shape& s, const BatchCut& cut, int32_t w, const DeviceInfo& dev, int min_range_tiles, int max_groups,
                     bool partial_sums) {
    const int L = w < s.max_seqlen ? w : s.max_seqlen;
    const int64_t blocks = (int64_t)(s.n_q_heads / s.n_kv_heads) * ((L + 31) / 32), pairs = (blocks + 1) / 2, tasks = s.n_kv_heads * pairs;
    const int64_t max_tiles = (s.max_seqlen + 31) / 32;
    const bool d64 = s.head_dim == 64;
    const double task_blocks = (double)blocks / pairs, size = s.head_dim / 128.0;
    const double alone = d64 ? 0.42 + 0.085 * task_blocks : 0.54 + 0.11 * task_blocks;
    const double shared = d64 ? 0.21 + 0.082 * task_blocks : 0.48;
    const int engines = kEnginesPerXcd * dev.xccs, engine_cus = dev.compute_units > engines ? dev.compute_units / engines : 1;
    const double per_row = partial_sums ? 0.1 + 5e-5 * s.max_seqlen : 0.0;
    StripPlan best{1, 1, 1, 1e300};
    for (int nt = kMaxRangeTiles; nt >= 1; --nt) {
        if (nt < min_range_tiles && nt < max_tiles) continue;
        const int64_t ranges_per_seq = (max_tiles + nt - 1) / nt, places = s.n_seqs * ranges_per_seq;
        if (nt > min_range_tiles && ranges_per_seq == (max_tiles + nt - 2) / (nt - 1)) continue;   // the same number of ranges, more evenly
        // (empty places of a grid: half of them count, as what they cost in balance)
        const double ranges = pick_order(s, cut.equal, cut.ranges[nt], ranges_per_seq, dev.xccs) == kGrid
                                  ? 0.5 * (cut.ranges[nt] + places) : (double)cut.ranges[nt];
        const double stream = (cut.tiles * (0.35 * s.n_kv_heads + 0.136 * (tasks - s.n_kv_heads)) + 0.063 * task_blocks * ranges * tasks) *
                              size / dev.compute_units;
        const double padding = 1.0 + 0.1 * (cut.ranges[nt] * (double)nt / cut.tiles - 1.0);
        for (int waves = kMaxWaves; waves >= 1; waves /= 2) {
            if ((waves > tasks && waves > 1) || (waves < 4 && 2 * waves <= tasks) || (waves < kMaxWaves && pairs >= 48)) continue;
            // workgroups a compute unit holds: 8 wavefronts at d = 128 and 12 at d = 64 by registers, 160 KB of LDS
            const int bytes = d64 ? wave_lds_bytes<64>(nt) : wave_lds_bytes<128>(nt);
            const int by_lds = 160 * 1024 / (waves * bytes), by_registers = (d64 ? 12 : 8) / waves;
            const int wgs_per_cu = by_lds < by_registers ? by_lds : by_registers;
            for (int g = 1; g <= max_groups && (g == 1 || (int64_t)g * waves < 2 * tasks); g *= 2) {
                const double wave_tasks = (double)((tasks + (int64_t)g * waves - 1) / ((int64_t)g * waves)), steps = wave_tasks * (nt + task_blocks);
                const int64_t queue = ((int64_t)(ranges * g) + engines - 1) / engines, round = (int64_t)engine_cus * wgs_per_cu;
                const int64_t per_cu = (queue + engine_cus - 1) / engine_cus, rest = queue % round;
                const double full = shared * wgs_per_cu * waves / 4, last = shared * (double)((rest + engine_cus - 1) / engine_cus * waves) / 4;
                const double chain = (double)(queue / round) * (1.9 + steps * (full > alone ? full : alone)) +
                                     (rest == 0 ? 0.0 : 1.9 + steps * (last > alone ? last : alone));
                const double flow = stream * (1.0 + 0.1 * ((double)per_cu * engine_cus / queue - 1.0));
                const double cost = sqrt(sqrt(chain * chain * chain * chain + flow * flow * flow * flow)) * padding + per_row * (g - 1);
                if (cost < best.cost) best = StripPlan{nt, waves, g, cost};
            }
        }
    }
    return best;
}

// By how many heads the walks of neighbouring ranges are apart, where K rows are a power of two apart.  Measured (us), steps of
// 0 / 2 / 7 / 8, d = 128 unless said: 64 x 2048 on 8 heads, d = 64, 30.6 / 28.5 / 28.5 / 30.8 (8 is a multiple of them), 16 heads
// 114 / 105 / 99 / 97, 32 heads 211 / 218 / 194 / 188, 64 heads 381 / 384 / 406 / 404; 4 x 32768 on 16 heads 112 / 103 / 97 / 93, 32
// heads 210 / 185 / 182 / 184, 64 heads 377 / 356 / 368 / 419; in short ranges, 8 x 2048 on 32 heads 28.5 / 27.6 / 27.2 / 35.6, 16 x 1000 on
// 64 heads 50.6 / 53.2 / 55.9 / 56.4.  Rows of 10 KB: no difference; 8 heads with four or more query heads each, where the window's
// Q rows that neighbouring ranges share count for more: 64 x 2048 on 32/8 heads 103 / 104 / 105 / 103, on 64/8 178 / 180 / 179 / 178.
int pick_head_step(const pyr_shape& s, int range_tiles) {
    const size_t k_row_bytes = (size_t)s.n_kv_heads * s.head_dim * 2;
    if ((k_row_bytes & (k_row_bytes - 1)) != 0) return 0;
    if (s.n_kv_heads <= 8) return s.n_q_heads > 2 * s.n_kv_heads ? 0 : 7;
    if (s.n_kv_heads > 32) return 2;
    return range_tiles >= 8 ? 8 : 7;
}

template <int D, int kMode>
int launch_strip_d(const StripArgs& a, dim3 grid, int waves, hipStream_t stream) {
    static std::atomic<uint64_t> lds_set{0};
    if (ensure_dynamic_lds((const void*)strip_kernel<D, kMode>, kMaxWaves * wave_lds_bytes<D>(kMaxRangeTiles), &lds_set) != PYR_OK)
        return PYR_ERR_LAUNCH;
    hipLaunchKernelGGL((strip_kernel<D, kMode>), grid, dim3(64 * waves), waves * wave_lds_bytes<D>(a.range_tiles), stream, a);
    return check_launch();
}

template <int kMode>
int launch_strip(const void* q, const void* k, const float* lse, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                 const pyr_shape& s, int32_t min_seqlen, int32_t w, int32_t q_window, float scale_log2, const float* row_weights, float* sums,
                 float2* part, const StripPlan& plan, const DeviceInfo& dev, hipStream_t stream) {
    StripArgs a{};
    a.q = (const uint16_t*)q;
    a.k = (const uint16_t*)k;
    a.lse = lse;
    a.seq_offsets = seq_offsets_dev;
    a.row_weights = row_weights;
    if (kMode == kStats) a.part = part;
    else a.sums = sums;
    a.n_seqs = s.n_seqs;
    a.w = w;
    a.total_tokens = s.total_tokens;
    a.group = s.n_q_heads / s.n_kv_heads;
    a.n_kv_heads = s.n_kv_heads;
    a.groups = plan.groups;
    a.waves = plan.waves;
    a.range_tiles = plan.range_tiles;
    a.ranges_per_seq = ((s.max_seqlen + 31) / 32 + plan.range_tiles - 1) / plan.range_tiles;
    // A whole sequence per XCD where that spreads the work evenly by construction (equal lengths, a multiple of the XCD
    // count: 64 x 2048 216 -> 196 us), so that the window's Q rows, which every range of the sequence re-reads, are found in that
    // XCD's L2; with ragged lengths the sequences of one XCD can be much longer than another's.  Where the places of a grid are
    // kept, an odd number per sequence keeps range r of all sequences from meeting on one XCD.
    a.xcds = dev.xccs;
    const int64_t ranges = min_seqlen == s.max_seqlen ? (int64_t)s.n_seqs * a.ranges_per_seq
                                                      : count_ranges(seq_offsets_host, s.n_seqs, 32 * plan.range_tiles);
    a.order = pick_order(s, min_seqlen == s.max_seqlen, ranges, a.ranges_per_seq, dev.xccs);
    if (a.order == kGrid) a.ranges_per_seq |= 1;
    // Where the window is a good part of the sequence, fewer of its rows see the later ranges; each sequence then starts at another
    // range, or the long ones would meet on the same engines (31 x 2048, w = 1024, on 32/8 heads 1038 us without, 809 with it; but
    // 30 x 1100, w = 128, on 32 heads 86.6 without, 91.1 with it).
    a.turn = (a.order == kSeqPerXcd || a.order == kEqual) && 2 * (int64_t)w >= s.max_seqlen ? 1 : 0;
    a.head_step = pick_head_step(s, plan.range_tiles);
    a.q_window = q_window;
    a.c = scale_log2;
    const int64_t n = a.order == kPacked ? ranges : (int64_t)s.n_seqs * a.ranges_per_seq;
    if (n >= (int64_t)1 << 31) return PYR_ERR_UNSUPPORTED;
    const dim3 grid((unsigned)n, (unsigned)plan.groups, 1);
    return s.head_dim == 128 ? launch_strip_d<128, kMode>(a, grid, plan.waves, stream)
                             : launch_strip_d<64, kMode>(a, grid, plan.waves, stream);
}

int launch_scores(const void* q, const void* k, const float* lse, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                  const pyr_shape& s, int32_t min_seqlen, int32_t w, int32_t q_window, float scale_log2, const float* row_weights, float* scores,
                  float* parts, const StripPlan& plan, const DeviceInfo& dev, hipStream_t stream) {
    float* sums = plan.groups > 1 ? parts : scores;
    return row_weights ? launch_strip<kScoresWeighted>(q, k, lse, seq_offsets_dev, seq_offsets_host, s, min_seqlen, w, q_window,
                                                       scale_log2, row_weights, sums, nullptr, plan, dev, stream)
                       : launch_strip<kScores>(q, k, lse, seq_offsets_dev, seq_offsets_host, s, min_seqlen, w, q_window, scale_log2,
                                               nullptr, sums, nullptr, plan, dev, stream);
}

}  // namespace

int launch_score(const void* q, const void* k, const float* lse, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                 const pyr_shape& s, int32_t min_seqlen, int32_t w, float scale_log2, const float* row_weights,
                 float* scores, hipStream_t stream) {
    if (s.n_seqs == 0 || s.max_seqlen == 0) return PYR_OK;
    DeviceInfo dev;
    if (device_info(&dev) != PYR_OK) return PYR_ERR_LAUNCH;
    const StripPlan plan = plan_strip(s, cut_batch(s, seq_offsets_host, min_seqlen), w, dev, 1, 1, true);
    return launch_scores(q, k, lse, seq_offsets_dev, seq_offsets_host, s, min_seqlen, w, 0, scale_log2, row_weights, scores, nullptr, plan, dev,
                         stream);
}

// (A prefill step only has room for partial sums where the batch has fewer than 1024 blocks of 64 keys: beyond that its ranges fill
// the chip.  The generation phase takes the room of the statistics, and may split larger batches where windows are wide.)
size_t score_parts_bytes(const pyr_shape& s) {
    const size_t blocks = (size_t)s.n_seqs * (((size_t)s.max_seqlen + 63) / 64);
    return blocks < 1024 ? (size_t)kMaxScoreGroups * s.total_tokens * sizeof(float) : 0;
}

int launch_score_groups(const StripPlan& plan, const void* q, const void* k, const float* lse, const int32_t* seq_offsets_dev,
                        const int32_t* seq_offsets_host, const pyr_shape& s, int32_t min_seqlen, int32_t w, float scale_log2, const float* row_weights,
                        float* scores, float* parts, hipStream_t stream) {
    if (s.n_seqs == 0 || s.max_seqlen == 0) return PYR_OK;
    DeviceInfo dev;
    if (device_info(&dev) != PYR_OK) return PYR_ERR_LAUNCH;
    return launch_scores(q, k, lse, seq_offsets_dev, seq_offsets_host, s, min_seqlen, w, 0, scale_log2, row_weights, scores, parts, plan, dev,
                         stream);
}

// How the generation phase gets its scores: by one walk over K (window.hip), or by two with the denominators folded between them.
struct UpdatePlan {
    bool one_walk;
    WindowPlan window;
    StripPlan stats, scores;
};

// Partial sums of the scores go where the statistics lie, which are dead once folded: as many rows as fit.
// One walk reads K once and is one launch where two walks are three, but it has the window's rows in blocks of 32 and its loads go by once
// per block: it wins where row blocks per KV head are few or sequences short.  Whole updates, two walks / one walk (us): 1 x 1024 rows on
// 32 heads, w = 64 28.2 / 23.1, 4 x 1537 71.8 / 61, 5 x 1330 on 8 heads, d = 64, w = 128 27.1 / 22.2, 48 of 689 at most on 24 heads, w = 32
// 135.6 / 100; but 18 x 826 on 64/8 heads, w = 16 55.8 / 74.5, 57 of 1066 at most on 32/8 heads, d = 64, w = 48 87 / 111.  Both costs
// are predicted (the two walks' with the fold and the selection, to 10 %) and one walk is taken where it is 8 % lower, 13 % with four to eight row blocks
// per KV head, where the prediction flatters it, 11.5 % with more than sixteen.  Of 1200 updates of random shapes up to 2048 rows, each timed both ways, the choice takes
// 0.5 % longer than the faster form in the mean (0.8 % with the lines 8 and 3 % lower that were drawn before the one walk's tasks went by KV head); it takes one walk
// against two that are more than 3 % faster in 6 (42 x 215 at most on 32/8 heads, d = 64, w = 100 43 / 51) and keeps two against one that is more than 3 % faster
// in 51, by 28 % at most (40 x 254...280 on 64/8 heads, w = 48 84 / 66, 4 x 841 on 64/8 heads, w = 128 46.5 / 36.9).  The lines stand where a batch's tasks go
// by query head too (window.hip, by_kv_head): 400 such updates between these lines and those take 0.918 of the two walks' time by one, 0.91 to 0.94 by
// the limit of that rule that keeps them out; 21 are more than 3 % slower, 16 % at most (48 x 75 on 64/8 heads, w = 48 45.6 / 52.9, 53 x 479 on 32/4, w = 16 50.7 / 57.4).
UpdatePlan plan_update(const pyr_shape& s, const BatchCut& cut, int32_t w, const DeviceInfo& dev) {
    UpdatePlan p{};
    const size_t room = window_score_part_bytes(s, w), row = (size_t)s.total_tokens * sizeof(float);
    int split = 1;
    while (split < kMaxScoreGroups && 2 * (size_t)split * row <= room) split *= 2;
    p.stats = plan_strip(s, cut, w, dev, 2, kMaxScoreGroups, false);
    p.scores = plan_strip(s, cut, w, dev, 1, split, true);
    p.window = plan_window(s, cut.tiles, w, room / row < 1 ? 1 : room / row > 256 ? 256 : (int)(room / row), dev);
    const int blocks = s.n_q_heads / s.n_kv_heads * (((w < s.max_seqlen ? w : s.max_seqlen) + 31) / 32);
    const double line = blocks >= 4 && blocks <= 8 ? 0.87 : blocks <= 16 ? 0.92 : 0.885;
    const double folded = (double)s.n_seqs * w * s.n_q_heads * ((s.max_seqlen + 63) / 64);
    p.one_walk = p.window.waves > 0 && p.window.cost < line * (11.5 + 1.16 * p.stats.cost + 0.86 * p.scores.cost + 7.6e-6 * folded);
    return p;
}

// A prefill step's scores: by the strip walk behind the attention launch, or by one walk in the launch of the attention tiles (layer.hip), where the
// windows' workgroups have the tiles' size, one or two groups of four wavefronts, and write a row of partial sums each.
// The one walk saves a launch and its latency and reads K beside the tiles that read it too, but takes the tiles' compute units: it wins where batches
// are small.  Both are predicted, in microseconds, from the attention's predicted time A and the strip walk's predicted C:
// - apart: A + 0.66 C + 4.1;
// - together: a workgroup takes 2.93 until its first tiles are there and then a task after the other, 0.43 and 0.88 per 32-key tile of a wavefront
//   (query rows count as one), 0.825 of that at d = 64; 0.86 of what all of them take adds to A as a share of the chip; joined with the longest workgroup as in
//   plan_strip.  A row of partial sums costs the selection 0.029.  At d = 64 five tiles a wavefront and more leave a compute unit
//   room for two workgroups instead of three: 12 % more for the tiles.  Where tiles of two groups fill their rounds, three at most, so far that the windows
//   open another: a tenth of A.  Two launches / one on both sides of two rounds, 512 tiles: 1 x 1900 on 32 heads (480) 68.5 / 65.7, 1 x 1920 68.8 / 65.9,
//   1 x 1985 (512) 72.2 / 73.9, 1 x 2048 74.2 / 75.6 (lengths between get tiles of one group, which go up to 1024 keys here); on 32/8 heads 1 x 1920 61.8 / 58.4, 1 x 2048 66.1 / 67.3.  A single round does not mind (1 x 1024 on 32 heads,
//   256 tiles 42.4 / 36.0), but 1 x 2048 on 16 heads is kept apart by the term: 55.7 / 49.4.
// Fitted to 1300 layers of random shapes (fifteen head shapes, w = 16...256, one sequence to 100, 32...2048 tokens, equal and ragged, with and without weights and
// hidden rows), each timed apart and with up to nine numbers of rows on inputs that change from call to call; one launch is taken where it is predicted to save
// 5 % of A, C and 10 us.  That chose it for 852 of them; over all 1300 the geometric mean of the time is 0.899 of that of the two launches (0.885 for
// the best choice each time), and four were more than 2 % slower, 4 % at most (91 x 44 tokens on 8 heads, d = 64 20.6 / 21.5, 24 x 284 on 12, d = 64 36.2 / 37.4).
// Two launches / one: 1 x 256 on 8 heads, d = 64 16.1 / 12.3, 1 x 473 on 32/8 heads, d = 64 19.7 / 15.8, 6 x 134 on 32/8 heads 25.8 / 20.7, 1 x 1058
// on 40 heads 43.1 / 38.9; but 64 x 359 on 32 heads 385 / 399, 16 x 694 on 32/8 heads, d = 64 89.7 / 98.9.
// Tried and taken back: the windows' workgroups behind the first rows of tiles, so that the longest tiles start first (within 1 %).
LayerPlan plan_layer(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len, int32_t min_seqlen, int32_t w, bool parts,
                     const AttentionChoice& choice, const DeviceInfo& dev) {
    LayerPlan plan{0, StripPlan{1, 1, 1, 0.0}};
    if (s.n_seqs == 0 || s.max_seqlen == 0) return plan;
    const BatchCut cut = cut_batch(s, seq_offsets_host, min_seqlen);
    plan.strip = plan_strip(s, cut, w, dev, 1, parts ? kMaxScoreGroups : 1, true);
    const int waves = 4 * choice.kernel, max_tiles = (s.max_seqlen + 31) / 32;
    const int L = w < s.max_seqlen ? w : s.max_seqlen, tasks = s.n_q_heads * ((L + 31) / 32);
    if (!parts || choice.kernel == 0 || s.max_seqlen > layer_max_keys(choice.kernel) || attention_tile_listed(s, seq_offsets_host, uniform_len)) return plan;
    // (one dimension of workgroups, of which a launch takes 2^32 lanes)
    if ((int64_t)s.n_seqs * (max_tiles + 3) / 4 * s.n_q_heads >= 1 << 20 || (int64_t)s.n_seqs * tasks >= 1 << 20) return plan;
    const bool d64 = s.head_dim == 64;
    const int wave_tiles = (max_tiles + waves - 1) / waves;
    const double k = d64 ? 0.825 : 1.0, longest = 0.43 + 0.88 * k * (wave_tiles + 1), mean = 0.43 + 0.88 * k * (cut.tiles / s.n_seqs / waves + 1);
    const double slots = (double)dev.compute_units * (choice.kernel == 2 ? 1 : d64 && wave_tiles <= 4 ? 3 : 2);
    const double tiles = choice.cost * (d64 && choice.kernel == 1 && wave_tiles > 4 ? 1.12 : 1.0);
    const int64_t places = attention_tiles(s, seq_offsets_host, uniform_len) * s.n_q_heads, cus = dev.compute_units;      // workgroups of the tiles
    const int64_t spare = choice.kernel == 2 && places <= 3 * cus ? (places + cus - 1) / cus * cus - places : (int64_t)1 << 40;
    double best = choice.cost + 0.66 * plan.strip.cost + 4.1 - 0.05 * (choice.cost + plan.strip.cost + 10.0);
    // (the workspace has room for a row per query head where the row statistics would lie, and for the strip walk's rows behind them)
    const int limit = tasks < s.n_q_heads + kMaxScoreGroups ? tasks : s.n_q_heads + kMaxScoreGroups;
    for (int g = 1;; g = g < 8 ? 2 * g : g + 8) {
        if (g > limit) g = limit;
        const double own = 2.93 + (tasks + g - 1) / g * longest;
        const double all = tiles + 0.86 * s.n_seqs * (g * 2.93 + tasks * mean) / slots;
        const double cost = sqrt(sqrt(all * all * all * all + own * own * own * own)) + 0.029 * (g - 1) + (s.n_seqs * (int64_t)g > spare ? 0.1 * choice.cost : 0.0);
        if (cost < best) {
            best = cost;
            plan.groups = g;
        }
        if (g == limit) break;
    }
    return plan;
}

void score_route(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t min_seqlen, int32_t w, bool parts, const DeviceInfo& dev,
                 pyr_route* out) {
    const BatchCut cut = cut_batch(s, seq_offsets_host, min_seqlen);
    const StripPlan score = plan_strip(s, cut, w, dev, 1, parts ? kMaxScoreGroups : 1, true);
    const UpdatePlan update = plan_update(s, cut, w, dev);
    out->score_tiles = score.range_tiles;
    out->score_waves = score.waves;
    out->score_groups = score.groups;
    out->score_order = pick_order(s, cut.equal, count_ranges(seq_offsets_host, s.n_seqs, 32 * score.range_tiles),
                                  ((s.max_seqlen + 31) / 32 + score.range_tiles - 1) / score.range_tiles, dev.xccs);
    if (!update.one_walk) {
        out->stats_tiles = update.stats.range_tiles;
        out->stats_waves = update.stats.waves;
        out->stats_groups = update.stats.groups;
    }
    out->window_tiles = update.one_walk ? ((s.max_seqlen + 31) / 32 + update.window.waves - 1) / update.window.waves : update.scores.range_tiles;
    out->window_waves = update.one_walk ? update.window.waves : update.scores.waves;
    out->window_groups = update.one_walk ? update.window.groups : update.scores.groups;
}

int update_route(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t min_seqlen, int32_t w, const DeviceInfo& dev, pyr_launches* out) {
    const BatchCut cut = cut_batch(s, seq_offsets_host, min_seqlen);
    const UpdatePlan update = plan_update(s, cut, w, dev);
    if (update.one_walk) return update.window.groups;
    const auto order = [&](const StripPlan& plan) {
        return pick_order(s, cut.equal, count_ranges(seq_offsets_host, s.n_seqs, 32 * plan.range_tiles),
                          ((s.max_seqlen + 31) / 32 + plan.range_tiles - 1) / plan.range_tiles, dev.xccs);
    };
    out->stats_order = order(update.stats);
    out->window_order = order(update.scores);
    return update.scores.groups;
}

int update_task_order(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t min_seqlen, int32_t w, const DeviceInfo& dev) {
    const BatchCut cut = cut_batch(s, seq_offsets_host, min_seqlen);
    return plan_update(s, cut, w, dev).one_walk ? window_task_order(s, cut.equal, w, dev) : -1;
}

size_t window_score_part_bytes(const pyr_shape& s, int32_t w) {
    const size_t ranges = ((size_t)s.max_seqlen + 63) / 64;           // (statistics ranges are at least 64 keys)
    return ranges * (size_t)s.n_seqs * (size_t)w * (size_t)s.n_q_heads * sizeof(float2);
}

int launch_window_score(const void* q_win, const void* k, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                        const pyr_shape& s, int32_t min_seqlen, int32_t w, float scale_log2, const float* row_weights, float* lse_win, void* part, float* scores,
                        int* groups, hipStream_t stream) {
    *groups = 1;
    if (s.n_seqs == 0 || s.max_seqlen == 0) return PYR_OK;
    DeviceInfo dev;
    if (device_info(&dev) != PYR_OK) return PYR_ERR_LAUNCH;
    const BatchCut cut = cut_batch(s, seq_offsets_host, min_seqlen);
    const UpdatePlan plan = plan_update(s, cut, w, dev);
    *groups = plan.one_walk ? plan.window.groups : plan.scores.groups;
    if (plan.one_walk)
        return launch_window(q_win, k, seq_offsets_dev, s, cut.equal, w, 1, scale_log2, row_weights, *groups > 1 ? (float*)part : scores,
                             plan.window, dev, stream);
    int rc = launch_strip<kStats>(q_win, k, nullptr, seq_offsets_dev, seq_offsets_host, s, min_seqlen, w, 1, scale_log2, nullptr, nullptr,
                                  (float2*)part, plan.stats, dev, stream);
    if (rc != PYR_OK) return rc;
    const int range_keys = 32 * plan.stats.range_tiles;
    rc = (s.max_seqlen + range_keys - 1) / range_keys <= 4
             ? launch_fold<1>((const float2*)part, seq_offsets_dev, s, w, range_keys, lse_win, stream)
             : launch_fold<8>((const float2*)part, seq_offsets_dev, s, w, range_keys, lse_win, stream);
    if (rc != PYR_OK) return rc;
    return launch_scores(q_win, k, lse_win, seq_offsets_dev, seq_offsets_host, s, min_seqlen, w, 1, scale_log2, row_weights, scores, (float*)part,
                         plan.scores, dev, stream);
}

}  // namespace pyr
