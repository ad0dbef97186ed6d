// Causal softmax attention for short sequences and small batches: one 128-row query tile of one (sequence, head) per
// workgroup, so that the hardware's dispatcher balances the load, two workgroups of a compute unit cover each
// other's beginnings and ends, and nothing is carried from tile to tile.  (The kernel in attention.hip keeps 256 rows
// per workgroup and walks a list of them: half the K/V traffic per product and no prologue per tile, which wins
// once tiles are long; its change of tile costs about as much as six key tiles.)
//
// Four wavefronts of 32 query rows each are a GROUP with a K/V stream of its own.  kGroups == 1: a workgroup is one group
// (80 KB of LDS at d = 128: two per compute unit).  kGroups == 2: two groups share the 128 rows and take the
// key tiles alternately, each with its own denominator, output and renewals of the exponent reference, which are merged through LDS
// at the end: a grid too small to put two wavefronts on every SIMD gets them that way, and its longest chain is halved.
//
// Everything inside a wavefront - MFMA mapping, transposed logits, the interleaving of products and exponentials,
// the exponent reference that is only moved when a row outgrows it - is as described in attention.hip.  The LDS
// ring is as short as that pipeline allows: two K tiles and three V tiles.  Synchronisation t sits in front of the last
// group of step t: every wavefront has read K(t+1) and finished with V(t-1) then, so K(t+3) and V(t+2) are requested
// into their slots, and K(t+2) and V(t+1), requested one step earlier, must have landed.
// Measured, lists of 256- or 128-row tiles as in attention.hip / this kernel (us): 1 x 2048, 32 heads 55 / 43, 64 x 359
// 190 / 173; d = 64: 64 x 2048 1550 / 1340, seven sequences of 100...3000 tokens on 32/8 heads 131 / 93.
#pragma once

#include "attention_device.h"

namespace pyr {

constexpr int kTileKeys = 64;              // key positions per LDS tile
constexpr int kTileRows = 128;             // query rows per workgroup
constexpr int kKRing = 2, kVRing = 3;

template <int D, int kGroups>
struct TileLds {
    static constexpr int kMatBytes = kTileKeys * D * 2;
    static constexpr int kGroupBytes = (kKRing + kVRing) * kMatBytes;
    static constexpr int kMergeBytes = kGroups == 2 ? 8 * (64 * (D / 4) * 4 + 2 * 256) : 0;      // per wavefront: half of O^T, reference, denominator
    static constexpr int kBytes = kGroups * kGroupBytes > kMergeBytes ? kGroups * kGroupBytes : kMergeBytes;
};

// (Kernel arguments of 112 bytes and less, implicit ones - the grid's and the workgroup's size - among them, are 0.7 us less host time a launch
// than longer ones, 2.8 / 3.5: so the grid's size is passed, and what does not go together does not travel together.)
struct TileArgs {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const int32_t* seq_offsets;
    uint16_t* out;
    int32_t n_seqs, uniform_len, n_q_heads, n_kv_heads;
    int32_t units_per_chunk, xcds;                // unit: one KV head of one sequence
    float c, lowest;                              // factor of the logits; lowest_reference()
};

// Launch arguments of a batch (attention_tile.hip), and the grid where its tiles are not listed (one launch below 8 million tokens a sequence).
int tile_args(const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
              const pyr_shape& s, int32_t uniform_len, float scale_log2, void* out, const DeviceInfo& dev, TileArgs* args);
dim3 tile_grid(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len, int groups, const DeviceInfo& dev, TileArgs* a);

// Grid: x = ((unit of the chunk's share of one XCD) * group + query head of the group) * xcds + xcd; y = query tile, the last
// one first; z = chunk.  Workgroup ids go round robin over the XCDs, so a unit's K and V are fetched into one L2 only;
// inside a chunk the long tiles of all its units start first.
// With a list (very unequal sequences, see the launch): x = (place * group + query head of the group) * xcds + xcd, where the
// places are the KV heads of a sequence that one XCD serves; y = position in the list of all sequences' tiles.
// Front: what the first `front.workgroups` workgroups of a one-dimensional grid do instead of a tile (layer.hip), or nothing, and the arguments that go with it.
struct NoFront {
    static constexpr bool kAny = false;
    static constexpr int kWaves = 2;              // wavefronts of a SIMD to leave registers for
    const int32_t* tile_map;                      // the list of a ragged batch's tiles (prefix sums of tiles per sequence), or nullptr
    float* lse;
    int32_t first_tile, tiles;                    // of the grid's y
};
template <int D, int kGroups, class Front>
__global__ __launch_bounds__(kGroups * 256, Front::kWaves) void attention_tile_kernel(TileArgs a, Front front) {
    using T = TileLds<D, kGroups>;
    constexpr int kRowBytes = D * 2;
    constexpr int kChunks = D / 8;                // 16-byte chunks per row
    constexpr int kMatBytes = T::kMatBytes;
    constexpr int NS = D / 16;                    // MFMAs per group of products = k-steps of QK^T = V fragments of a half
    constexpr int kDTiles = D / 32;               // 32-row tiles of O^T
    constexpr int EPS = 8 / NS;                   // logits of a chunk handled per slice (1 or 2)
    constexpr int kLook = NS - 2;                 // slices between the LDS read of a fragment and its MFMA
    constexpr int kRowsPerInstr = 1024 / kRowBytes;
    constexpr int kInstr = kMatBytes / 1024 / 4;  // load instructions of a wavefront per matrix tile
    constexpr int kQInstr = 32 * kRowBytes / 1024;
    constexpr int kLine = 256 / kRowBytes;        // rows per 256-byte bank line (1 or 2)
    static_assert(2 * kInstr == NS, "one load instruction per slice of a group");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int grid_x = (int)blockIdx.x, grid_y = (int)blockIdx.y, grid_z = (int)blockIdx.z, tiles, first_tile = 0;
    const int32_t* tile_map = nullptr;
    float* lse = nullptr;
    if constexpr (Front::kAny) {
        if (grid_x < front.workgroups) {
            front.run(a, grid_x, smem);
            return;
        }
        const int place = grid_x - front.workgroups, row = place / front.grid_x;
        tiles = front.grid_y;
        grid_x = place - row * front.grid_x;
        grid_z = row / tiles;
        grid_y = row - grid_z * tiles;
    } else {
        tiles = front.tiles;
        first_tile = front.first_tile;
        tile_map = front.tile_map;
        lse = front.lse;
    }

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int grp = kGroups == 2 ? wave >> 2 : 0, w4 = wave & 3;
    const int li = lane & 31, gl = lane >> 5;

    // ---- which tile
    const int head_group = a.n_q_heads / a.n_kv_heads;
    const int xcd = grid_x % a.xcds, slot = grid_x / a.xcds;
    int b, kvh, q_tile;
    if (tile_map != nullptr) {
        // The sequence: the last b with tile_map[b] <= position, found 64 candidates at a time (a binary search would be a chain of
        // a dozen loads in front of each tile).  [b, b + span) holds it; candidate lane l stands at b + l * step.
        const int pos = first_tile + grid_y;
        b = 0;
        for (int span = a.n_seqs; span > 1;) {
            const int step = (span + 63) / 64;
            const int cand = b + lane * step;
            const bool below = lane * step < span && tile_map[cand] <= pos;
            const int hits = __builtin_popcountll(__builtin_amdgcn_ballot_w64(below));
            b += (hits - 1) * step;               // (candidate 0 always is one)
            span = min(step, span - (hits - 1) * step);
        }
        q_tile = tile_map[b + 1] - 1 - pos;
        kvh = (xcd + a.xcds - (int)((int64_t)b * a.n_kv_heads % a.xcds)) % a.xcds + slot / head_group * a.xcds;      // the XCDs take turns at the odd heads
        if (kvh >= a.n_kv_heads) return;          // (uniform over the workgroup, like the others)
    } else {
        const int unit = (grid_z * a.units_per_chunk + slot / head_group) * a.xcds + xcd;
        b = unit / a.n_kv_heads;
        if (b >= a.n_seqs) return;
        kvh = unit % a.n_kv_heads;
        q_tile = first_tile + tiles - 1 - grid_y;
    }
    const int h = kvh * head_group + slot % head_group;
    int row0, S;
    if (a.uniform_len > 0) {
        row0 = b * a.uniform_len;
        S = a.uniform_len;
    } else {
        row0 = a.seq_offsets[b];
        S = a.seq_offsets[b + 1] - row0;
    }
    const int q_base = q_tile * kTileRows;
    if (q_base >= S) return;
    const int n_tiles = (min(S, q_base + kTileRows) + kTileKeys - 1) / kTileKeys;
    const int n_grp = (n_tiles - grp + kGroups - 1) / kGroups;       // key tiles of this group: grp, grp + kGroups, ...
    const int n_pos = (n_tiles + kGroups - 1) / kGroups;             // ... of the longer group: the workgroup's steps
    const int qlo = q_base + 32 * w4, qrow = qlo + li;
    const int H = qlo / 32 + 1;                   // 32-key halves this wavefront needs (the last one holds the diagonal)
    const int n_w = qlo < S ? (H + 1) / 2 : 0;
    const int n_my = n_w > grp ? (n_w - grp + kGroups - 1) / kGroups : 0;      // tiles of the group it takes part in

    // ---- LDS of the group: K ring, then V ring.  The query rows come through the V slots 1 and 2 before the stream needs them.
    const uint32_t lds_k = (uint32_t)(uintptr_t)(lptr_t)smem + grp * T::kGroupBytes;
    const uint32_t lds_v = lds_k + kKRing * kMatBytes;
    const uint32_t q_stage = lds_v + kMatBytes + w4 * 32 * kRowBytes;

    // ---- load side: instruction i of this wavefront fills rows (w4*kInstr + i)*kRowsPerInstr .. of a tile; lane l writes
    // physical chunk l % kChunks of row l / kChunks and fetches the logical chunk the swizzle stores there
    const uint32_t tok_bytes = (uint32_t)a.n_kv_heads * kRowBytes;
    const int l_row = lane / kChunks, l_chunk = lane % kChunks;
    uint32_t k_goff[kInstr], v_goff[kInstr];
#pragma unroll
    for (int i = 0; i < kInstr; ++i) {
        const int r = (w4 * kInstr + i) * kRowsPerInstr + l_row;
        k_goff[i] = (uint32_t)r * tok_bytes + ((l_chunk ^ ((r / kLine) & (kChunks - 1))) << 4);
        v_goff[i] = (uint32_t)r * tok_bytes + ((l_chunk ^ (((r / kLine) & (kChunks / 4 - 1)) << 2)) << 4);
    }
    const size_t unit_off = ((size_t)row0 * a.n_kv_heads + kvh) * D * 2;
    // instruction i of tile u (of the group) into its slot; rows past the end of the sequence re-read the last one
    auto load_piece = [&](const uint16_t* mat, const uint32_t (&goff)[kInstr], int u, uint32_t to, int i) __attribute__((always_inline)) {
        const int key = (kGroups * u + grp) * kTileKeys;
        const char* base = (const char*)mat + unit_off + (size_t)key * tok_bytes;
        uint32_t off = goff[i];
        if (key + kTileKeys > S) {
            const int r = (w4 * kInstr + i) * kRowsPerInstr + l_row;
            off -= (uint32_t)max(key + r - (S - 1), 0) * tok_bytes;
        }
        lds_dma16(base, off, to + (w4 * kInstr + i) * 1024);
    };
    int k_to = 0, v_to = 0;                       // ring slots the next K and V tile go to
    auto next_slots = [&]() __attribute__((always_inline)) {
        k_to ^= 1;
        v_to = v_to == kVRing - 1 ? 0 : v_to + 1;
    };
    auto k_piece = [&](int u, int i) __attribute__((always_inline)) {
        if (u < n_grp) load_piece(a.k, k_goff, u, lds_k + k_to * kMatBytes, i);
    };
    auto v_piece = [&](int u, int i) __attribute__((always_inline)) {
        if (u < n_grp) load_piece(a.v, v_goff, u, lds_v + v_to * kMatBytes, i);
    };

    // ---- fragment side (as in attention.hip)
    const int krow = (li & ~12) | ((li & 4) << 1) | ((li & 8) >> 1);
    const int k_lane = krow * kRowBytes + ((gl ^ ((krow / kLine) & (kChunks - 1))) << 4);
    const int vrow = 8 * gl + ((lane & 15) >> 2);
    const int v_lane = vrow * kRowBytes +
                       (((((vrow / kLine) & (kChunks / 4 - 1)) << 2) + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) << 4) +
                       8 * (lane & 1);
    int kaddr[NS], vaddr[kDTiles];                // in the K slot of the tile whose logits come next, in the V slot of the tile before
#pragma unroll
    for (int i = 0; i < NS; ++i) kaddr[i] = (int)lds_k + (k_lane ^ (i << 5));
#pragma unroll
    for (int dt = 0; dt < kDTiles; ++dt) vaddr[dt] = (int)lds_v + (kVRing - 1) * kMatBytes + (v_lane ^ (dt << 6));
    int kslot = 0, vslot = kVRing - 1;
    auto bump_k = [&]() __attribute__((always_inline)) {
        const int delta = kslot ? -kMatBytes : kMatBytes;
        kslot ^= 1;
#pragma unroll
        for (int i = 0; i < NS; ++i) kaddr[i] += delta;
    };
    auto bump_v = [&]() __attribute__((always_inline)) {
        const int delta = vslot == kVRing - 1 ? -(kVRing - 1) * kMatBytes : kMatBytes;
        vslot = vslot == kVRing - 1 ? 0 : vslot + 1;
#pragma unroll
        for (int dt = 0; dt < kDTiles; ++dt) vaddr[dt] += delta;
    };
    auto k_frag = [&](int half, int i) __attribute__((always_inline)) {
        return *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)(kaddr[i] + 32 * half * kRowBytes);
    };
    auto v_frag = [&](int half, int i) __attribute__((always_inline)) {
        const int p = vaddr[i % kDTiles] + 16 * (2 * half + i / kDTiles) * kRowBytes;
        const s16x4 lo = lds_read_tr(p);
        const s16x4 hi = lds_read_tr(p + 4 * kRowBytes);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    };

    bf16x8 qf[NS], F[NS];
    f32x16 oacc[kDTiles];                         // O^T
    f32x16 s0, s1;                                // logits of the two halves
    u32x4 p0[2], p1[2];                           // probabilities of the two halves
    float m_run = -INFINITY, nmc = 0.f, l_run = 0.f;      // exponent reference, -c * reference, denominators (this lane's keys)
    float ls0, ls1;
#pragma unroll
    for (int dt = 0; dt < kDTiles; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;

    auto fence = [&]() __attribute__((always_inline)) { __builtin_amdgcn_sched_barrier(0); };
    float pend = 0.f, last_e = 0.f;
    auto e_use = [&](int j, u32x4& pf, float& lsum) __attribute__((always_inline)) {
        lsum += last_e;
        asm volatile("" : "+v"(lsum));
        if (j & 1) {
            pf[j >> 1] = pack_bf16(pend, last_e);
            asm volatile("" : "+v"(pf[j >> 1]));
        } else {
            pend = last_e;
        }
    };
    auto e_slice = [&](const f32x16& sv, int base, int i, u32x4& pf, float& lsum) __attribute__((always_inline)) {
        if (EPS == 2) {
            float x = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[base + 2 * i], a.c, nmc));
            float y = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[base + 2 * i + 1], a.c, nmc));
            lsum += x;
            lsum += y;
            pf[i] = pack_bf16(x, y);
            asm volatile("" : "+v"(pf[i]), "+v"(lsum));
        } else {
            float x = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[base + i], a.c, nmc));
            asm volatile("" : "+v"(x));
            if (i > 0) e_use(i - 1, pf, lsum);
            last_e = x;
            if (i == NS - 1) e_use(i, pf, lsum);
        }
    };
    struct Chunk {                                // a chunk of exponentials: logits se[base ..+7] -> pe, lsum
        bool on;
        const f32x16* se;
        int base;
        u32x4* pe;
        float* lsum;
    };
    struct Frags { int kind, half; };             // NS fragments in LDS: kind 0 none, 1 K, 2 V
    auto frag = [&](const Frags& f, int j) __attribute__((always_inline)) -> bf16x8 {
        return f.kind == 1 ? k_frag(f.half, j) : v_frag(f.half, j);
    };
    auto prime = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kLook; ++j) F[j] = frag(f, j);
    };
    auto slice_load = [&](const Frags& own, const Frags& next, int i) __attribute__((always_inline)) {
        const int j = i + kLook;
        if (j < NS) {
            if (own.kind != 0) F[j] = frag(own, j);
        } else {
            if (next.kind != 0) F[j - NS] = frag(next, j - NS);
        }
    };
    auto qk_group = [&](f32x16& sd, const Chunk& e, const Frags& own, const Frags& next) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (i == 0) {
                f32x16 z;
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = 0.f;
                sd = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F[0], qf[0], z, 0, 0, 0);
            } else {
                sd = __builtin_amdgcn_mfma_f32_32x32x16_bf16(F[i], qf[i], sd, 0, 0, 0);
            }
            if (e.on) e_slice(*e.se, e.base, i, *e.pe, *e.lsum);
            slice_load(own, next, i);
            fence();
        }
    };
    // loads >= 0: every slice also requests one piece of K(loads + 1) and V(loads)
    auto pv_group = [&](const u32x4 (&pp)[2], const Chunk& e, const Frags& own, const Frags& next, int loads)
                        __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            oacc[i % kDTiles] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                F[i], __builtin_bit_cast(bf16x8, pp[i / kDTiles]), oacc[i % kDTiles], 0, 0, 0);
            if (e.on) e_slice(*e.se, e.base, i, *e.pe, *e.lsum);
            slice_load(own, next, i);
            if (loads >= 0) {
                if (i < kInstr) k_piece(loads + 1, i);
                else v_piece(loads, i - kInstr);
            }
            fence();
        }
    };
    auto e_group = [&](const f32x16& se, int ebase, u32x4& pe, float& lsum) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NS; ++i) e_slice(se, ebase, i, pe, lsum);
    };
    const Chunk no_e = {false, &s0, 0, &p0[0], &ls0};
    const Frags no_f = {0, 0};
    const Frags fk0 = {1, 0}, fk1 = {1, 1}, fv0 = {2, 0}, fv1 = {2, 1};

    // causal mask of a half: tile t of the group, half `half`
    const int diag = li - 8 * gl;                 // register r of a diagonal half is masked if 16*(r>>3) + (r&7) > diag
    auto mask_half = [&](f32x16& sv, int t, int half) __attribute__((always_inline)) {
        const int hh = 2 * (kGroups * t + grp) + half;
        if (hh >= H - 1) {
            int thr = hh > H - 1 ? -1 : diag;
            asm volatile("" : "+v"(thr));
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (16 * (r >> 3) + (r & 7) > thr) sv[r] = -INFINITY;
        }
    };
    auto max_of = [&](const f32x16& sv) __attribute__((always_inline)) {
        float mx = sv[0];
#pragma unroll
        for (int r = 1; r < 16; r += 2) {
            const float nxt = r + 1 < 16 ? sv[r + 1] : sv[r];
            mx = fmaxf(fmaxf(mx, sv[r]), nxt);
        }
        return max_with_other_half(mx);
    };
    auto settle_half = [&](const f32x16& sv, u32x4 (&pp)[2], float lsum) __attribute__((always_inline)) {
        if (__ballot(!(lsum <= 65536.0f)) != 0) {
            const float m_new = fmaxf(m_run, max_of(sv));
            const float alpha = m_new == m_run ? 1.0f : __builtin_amdgcn_exp2f((m_run - m_new) * a.c);
            l_run *= alpha;
#pragma unroll
            for (int dt = 0; dt < kDTiles; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
            m_run = m_new;
            nmc = -m_new * a.c;
            lsum = 0.f;
            e_group(sv, 0, pp[0], lsum);
            e_group(sv, 8, pp[1], lsum);
        }
        l_run += lsum;
    };
    auto sync = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- prologue: queries and K(0), then K(1) and V(0) behind them
    {
        const int first = min(qlo, S - 1);        // (rows past the end re-read the last one)
        const char* base = (const char*)(a.q + ((size_t)(row0 + first) * a.n_q_heads + h) * D);
#pragma unroll
        for (int i = 0; i < kQInstr; ++i) {
            const int row = kRowsPerInstr * i + l_row;
            lds_dma16(base, (uint32_t)min(row, S - 1 - first) * ((uint32_t)a.n_q_heads * kRowBytes) + ((l_chunk ^ (row & (kChunks - 1))) << 4),
                      q_stage + 1024 * i);
        }
    }
#pragma unroll
    for (int i = 0; i < kInstr; ++i) k_piece(0, i);
    k_to = 1;
#pragma unroll
    for (int i = 0; i < kInstr; ++i) k_piece(1, i);
#pragma unroll
    for (int i = 0; i < kInstr; ++i) v_piece(0, i);
    k_to = 0;
    v_to = 1;
    // K(1) may be absent, V(0) too (a second group without a tile): then everything is waited for
    if (n_grp > 1) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"(2 * kInstr) : "memory");
    else sync();
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        const uint32_t p = q_stage + li * kRowBytes + (((2 * j + gl) ^ (li & (kChunks - 1))) << 4);
        qf[j] = *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)p;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // in registers before the next synchronisation frees the area

    // ---- first logits: QK0(0), reference, QK1(0) | E0a(0), E0b(0)
    if (n_my > 0) {
        prime(fk0);
        qk_group(s0, no_e, fk0, fk1);
        mask_half(s0, 0, 0);
        m_run = max_of(s0);
    }
    // The reference is the row's maximum over its first 32 keys, for both groups: a reference of its own would have the second
    // group depend on keys 64...95, which may all be masked by the caller (logits of -inf), and round its probabilities apart from the
    // other kernels'.  Group 0 leaves it where the wavefront's queries were.  (One more barrier: 42.0 -> 42.3 us at 1 x 2048 on 32 heads,
    // 6.4 -> 6.6 at 1 x 256, d = 64, 8 heads.)
    if (kGroups == 2 && n_tiles > 1) {
        float __attribute__((address_space(3)))* ref =
            (float __attribute__((address_space(3)))*)(uintptr_t)(q_stage - grp * T::kGroupBytes + 4 * lane);
        if (grp == 0 && n_my > 0) *ref = m_run;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (grp == 1 && n_my > 0) m_run = *ref;
    }
    if (n_my > 0) {
        m_run = fmaxf(m_run, a.lowest);
        nmc = -m_run * a.c;
        ls0 = 0.f;
        fence();
        const Chunk e0a = {true, &s0, 0, &p0[0], &ls0};
        qk_group(s1, e0a, fk1, no_f);
        e_group(s0, 8, p0[1], ls0);
        if (grp == 0) l_run += ls0;
        else settle_half(s0, p0, ls0);            // (not these keys' own maximum)
        mask_half(s1, 0, 1);
        fence();
    }
    // requests after synchronisation t: K(t + 3), V(t + 2)
    auto request = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kInstr; ++i) k_piece(t + 3, i);
#pragma unroll
        for (int i = 0; i < kInstr; ++i) v_piece(t + 2, i);
        next_slots();
    };
    sync();                                       // synchronisation -1
    request(-1);
    bump_k();
    if (n_my > 1) prime(fk0);

    int t = 0;
#pragma unroll 1
    for (; t + 1 < n_my; ++t) {
        // tile t (probabilities, PV) and tile t+1 (logits)
        const Chunk e1a = {true, &s1, 0, &p1[0], &ls1}, e1b = {true, &s1, 8, &p1[1], &ls1};
        const Chunk e0a = {true, &s0, 0, &p0[0], &ls0}, e0b = {true, &s0, 8, &p0[1], &ls0};
        ls1 = 0.f;
        bump_v();
        qk_group(s0, e1a, fk0, fv0);              // QK0(t+1) | E1a(t)
        pv_group(p0, e1b, fv0, fk1, -1);          // PV0(t)   | E1b(t)
        settle_half(s1, p1, ls1);
        mask_half(s0, t + 1, 0);
        fence();
        ls0 = 0.f;
        qk_group(s1, e0a, fk1, fv1);              // QK1(t+1) | E0a(t+1)
        sync();
        bump_k();
        fence();
        pv_group(p1, e0b, fv1, fk0, t + 2);       // PV1(t)   | E0b(t+1) | loads
        next_slots();
        settle_half(s0, p0, ls0);
        mask_half(s1, t + 1, 1);
        fence();
    }
    // The wavefront's last tile.  V(t) stays in place until synchronisation t + 1, so the workgroup is not kept
    // waiting for it at synchronisation t.
    if (t <= n_pos - 2) {
        sync();
        request(t);
    }
    if (n_my > 0) {
        const Chunk e1b = {true, &s1, 8, &p1[1], &ls1};
        ls1 = 0.f;
        bump_v();
        prime(fv0);
        e_group(s1, 0, p1[0], ls1);
        fence();
        pv_group(p0, e1b, fv0, fv1, -1);          // PV0(t) | E1b(t)
        settle_half(s1, p1, ls1);
        fence();
        pv_group(p1, no_e, fv1, no_f, -1);        // PV1(t)
    }
#pragma unroll 1
    for (++t; t <= n_pos - 2; ++t) {
        sync();
        request(t);
    }
    // (the last synchronisation waited for every load that was issued)

    float l_tot = sum_with_other_half(l_run);
    int dt0 = 0;                                  // O^T tiles this wavefront stores: all, or its group's half
    if (kGroups == 2) {
        // The groups trade halves: each wavefront sends the half of O^T it does not store, and both send reference and denominator.
        constexpr int kHalf = kDTiles / 2, kSend = 64 * kHalf * 16 * 4;
        __syncthreads();                          // every fragment read is done
        const uint32_t box = (uint32_t)(uintptr_t)(lptr_t)smem;
        auto at = [&](int wv, int j) { return (f32x4 __attribute__((address_space(3)))*)(uintptr_t)(box + wv * (kSend + 512) + (j * 64 + lane) * 16); };
        auto stat = [&](int wv, int j) { return (float __attribute__((address_space(3)))*)(uintptr_t)(box + wv * (kSend + 512) + kSend + j * 256 + lane * 4); };
#pragma unroll
        for (int j = 0; j < kHalf * 4; ++j) {
            f32x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = grp == 0 ? oacc[kHalf + j / 4][4 * (j % 4) + e] : oacc[j / 4][4 * (j % 4) + e];
            *at(wave, j) = x;
        }
        *stat(wave, 0) = m_run;
        *stat(wave, 1) = l_tot;
        __syncthreads();
        const float m_oth = *stat(wave ^ 4, 0), l_oth = *stat(wave ^ 4, 1);
        const float m_all = fmaxf(m_run, m_oth);  // (finite: group 0 always has a tile)
        const float f_own = __builtin_amdgcn_exp2f((m_run - m_all) * a.c), f_oth = __builtin_amdgcn_exp2f((m_oth - m_all) * a.c);
        l_tot = l_tot * f_own + l_oth * f_oth;
        m_run = m_all;
        dt0 = grp * kHalf;
#pragma unroll
        for (int j = 0; j < kHalf * 4; ++j) {
            const f32x4 x = *at(wave ^ 4, j);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float own = grp == 0 ? oacc[j / 4][4 * (j % 4) + e] : oacc[kHalf + j / 4][4 * (j % 4) + e];
                oacc[j / 4][4 * (j % 4) + e] = own * f_own + x[e] * f_oth;
            }
        }
    }
    // ---- normalise, round to bf16, store (quads traded with the partner lane: 16 bytes per lane); log2 of the denominator
    const float inv = 1.0f / l_tot;
    constexpr int kStoreTiles = kDTiles / kGroups;
    u32x4 o16[kStoreTiles][2];
#pragma unroll
    for (int dt = 0; dt < kStoreTiles; ++dt)
#pragma unroll
        for (int ap = 0; ap < 2; ++ap) {
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t lo = pack_bf16(oacc[dt][8 * ap + 2 * e] * inv, oacc[dt][8 * ap + 2 * e + 1] * inv);
                const uint32_t hi = pack_bf16(oacc[dt][8 * ap + 4 + 2 * e] * inv, oacc[dt][8 * ap + 4 + 2 * e + 1] * inv);
                auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
                o16[dt][ap][e] = r[0];
                o16[dt][ap][2 + e] = r[1];
            }
        }
    if (qrow < S) {
        uint16_t* dst = a.out + ((size_t)(row0 + qrow) * a.n_q_heads + h) * D + 32 * dt0 + 8 * gl;
#pragma unroll
        for (int dt = 0; dt < kStoreTiles; ++dt)
#pragma unroll
            for (int ap = 0; ap < 2; ++ap) *(u32x4*)(dst + 32 * dt + 16 * ap) = o16[dt][ap];
        if (lse != nullptr && gl == 0 && grp == 0)
            lse[(size_t)(row0 + qrow) * a.n_q_heads + h] = m_run * a.c + __builtin_amdgcn_logf(l_tot);
    }
}

}  // namespace pyr
