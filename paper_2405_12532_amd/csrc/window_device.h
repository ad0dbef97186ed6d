// The scores of short sequences by one walk over K that finds the row denominators itself (Algorithm 1,
// A_e = weighted_avg(A[-L:, :-L]); see score.hip for the two-walk form and for what is computed).
//
// A workgroup of up to eight wavefronts holds the logits of 32 window rows (one query head) against ALL keys of a sequence in its
// registers: 16 accumulator registers per 32-key tile, up to kTiles tiles per wavefront, so 32 * kTiles keys a wavefront at most
// (2048 in eight with the 128 registers of kTiles = 8, half of the register file).  Per task (query head, row block) the wavefronts
// turn their tiles' logits into exponentials tile by tile, against a reference per row that is the row's logit of the wavefront's
// first key and is only moved (which the tiles before are told at the end) when a row outgrows it by 2^40; so the vector work hides
// behind the loads.  The wavefronts' references and sums per row then meet in LDS behind one barrier, and the exponentials, still
// in registers, are weighted and added up per key:
//   e = 2^(c*s - m_wave),  score += e * (omega_row * 2^(m_wave - M_row) / Z_row)
// A probability of 2^-126 and more may be a large exponential times a factor below the normal numbers (a wavefront whose first key is far below the
// row's other keys), so the factors, and the sums with them, stand 2^64 higher until the end; a reference's move is kept as an exponent.
// A key belongs to one wavefront, so its sum over the tasks is one LDS word per half-wavefront: no atomics, a fixed order.
//
// Bound at large batches: reading K, once from HBM (the row blocks and query heads that share a KV head run side by side on one XCD and
// find it in L2); else the chain of a wavefront's tiles (loads, 8 dependent products, 16 exponentials a lane: about 1 us a tile with
// two wavefronts on a SIMD, of which the vector port is busy 0.5).  Q and K rows are one stream of 32-row tiles per wavefront,
// through a private ring of two LDS slots filled by LDS-direct loads, as in score.hip.
// Measured against two walks and the fold between them, selection included (us): 64 x 2048 rows on 32 heads, w = 64, 418 -> 245, 88 x 692
// on 64 heads 410 -> 253, 22 of 286...914 on 32 heads, w = 32 61 -> 34, 5 x 199 on 16/2 heads, d = 64 19.5 -> 12.8.
// Tried and taken back: all logits first and the exponentials in a phase of their own (9.0 us a task of 8 tiles per wavefront, as now, and
// nothing hidden at short sequences); the loop over the tiles unrolled (55 KB of code, 12 us); the next tile's fragments read ahead (45
// registers spilled, 18 us).
#pragma once

#include <float.h>
#include <math.h>

#include "score_device.h"

namespace pyr {

constexpr int kWindowWaves = 8;                                  // wavefronts of a workgroup
constexpr int kWindowMaxTiles = 8;                               // 32-key tiles per wavefront, at most
constexpr float kWindowGrowth = 1099511627776.f;                 // 2^40: how far a row may outgrow its reference
constexpr int kWindowRaise = 64;                                 // factors and sums are kept times 2^64
constexpr int kWindowMaxKeys = kWindowWaves * 32 * kWindowMaxTiles;

struct WindowArgs {
    const uint16_t* q;
    const uint16_t* k;
    const int32_t* seq_offsets;
    const float* row_weights;
    float* sums;                              // [groups, total_tokens]
    int32_t n_seqs, n_q_heads, n_kv_heads, w, total_tokens;
    int32_t waves;                            // of a workgroup
    int32_t groups;                           // workgroups per sequence; workgroup g takes tasks g, g + groups, ...
    int32_t xcds;                             // > 0: equal lengths, a multiple of so many: a sequence's workgroups on one XCD
    int32_t q_window;                         // 0: q by packed row; else by (sequence, window slot)
    float c;
};
static_assert(sizeof(WindowArgs) <= 112, "short arguments");

// Sequence and place in it of workgroup `id`.
__device__ __forceinline__ void window_place(const WindowArgs& a, int id, int* b, int* g) {
    if (a.xcds > 0) {
        const int slot = (int)((uint32_t)id / (uint32_t)a.xcds), of_xcd = (int)((uint32_t)slot / (uint32_t)a.groups);
        *b = of_xcd * a.xcds + (id - slot * a.xcds);
        *g = slot - of_xcd * a.groups;
    } else {
        *b = (int)((uint32_t)id / (uint32_t)a.groups);
        *g = id - *b * a.groups;
    }
}

template <int D, int kTiles>
constexpr int window_lds_bytes(int waves) {                      // of a wavefront: ring, weights, factors, key sums and moves; statistics
    return waves * (2 * 32 * D * 2 + 256 + 128 + (256 + 128) * kTiles + 2 * 256);
}

template <int kCtrl>
__device__ __forceinline__ float dpp(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), kCtrl, 0xf, 0xf, false));
}
constexpr int kMirror16 = 0x140, kMirror8 = 0x141, kReverse4 = 0x1b, kSwap2 = 0xb1;      // inside 16, 8, 4 and 2 lanes

// The largest x of the 32 lanes of a half-wavefront, in all of them.
__device__ __forceinline__ float max_of_half(float x) {
    x = fmaxf(x, dpp<kMirror16>(x));
    x = fmaxf(x, dpp<kMirror8>(x));
    x = fmaxf(x, dpp<kReverse4>(x));
    x = fmaxf(x, dpp<kSwap2>(x));
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// v[r] added up over the 32 lanes of a half-wavefront; lane li receives the sum of register li & 15.  Lanes trade halves of
// their registers: 8 + 4 + 2 + 1 exchanges inside 16 lanes, then one between the two groups of 16.
__device__ __forceinline__ float sum_rows(const float (&v)[16], int li) {
    float a[8], b4[4], c2[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = (li & 8 ? v[8 + i] : v[i]) + dpp<kMirror16>(li & 8 ? v[i] : v[8 + i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) b4[i] = (li & 4 ? a[4 + i] : a[i]) + dpp<kMirror8>(li & 4 ? a[i] : a[4 + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) c2[i] = (li & 2 ? b4[2 + i] : b4[i]) + dpp<kReverse4>(li & 2 ? b4[i] : b4[2 + i]);
    const float x = (li & 1 ? c2[1] : c2[0]) + dpp<kSwap2>(li & 1 ? c2[0] : c2[1]);
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// v * 2^(x + up), also where 2^x by itself is no normal number.
__device__ __forceinline__ float times_exp2(float v, float x, int up) {
    const float bounded = fmaxf(x, -1000.f), whole = rintf(bounded);
    return __builtin_amdgcn_ldexpf(v * __builtin_amdgcn_exp2f(bounded - whole), (int)whole + up);
}

// The tasks of workgroup g of sequence b; at most kWindowWaves wavefronts, S <= 32 * kTiles * wavefronts, window_lds_bytes<D, kTiles>(wavefronts) of LDS at smem.
// kByKvHead: the tasks in turn over the KV heads; else query head after query head.
template <int D, int kTiles, bool kWeighted, bool kByKvHead>
__device__ void window_scores(const WindowArgs& a, int b, int g, char* smem) {
    constexpr int kSteps = D / 16;
    constexpr int kChunks = D / 8;                  // 16-byte chunks per row
    constexpr int kRowBytes = D * 2;
    constexpr int kRowsPerLoad = 64 / kChunks;      // rows one load instruction covers
    constexpr int kTileBytes = 32 * kRowBytes;
    constexpr int kTileLoads = kTileBytes / 1024;   // load instructions of a tile
    constexpr int kRowLoads = kWeighted ? 1 : 0;    // ... of a task's weights

    const int lane = threadIdx.x & 63;
    const int waves = a.waves, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int li = lane & 31, gl = lane >> 5;
    const int row0 = a.seq_offsets[b], S = a.seq_offsets[b + 1] - row0;
    if (S <= 0) return;
    const int L = min(a.w, S);
    const int first_row = S - L;                      // local position of the first window row
    const int q_row_base = a.q_window ? b * a.w + (a.w - L) : row0 + first_row;   // row of q holding the first window row
    const int n_rb = (L + 31) / 32;
    // (divisions unsigned, and as few as can be: what stands in front of the first load is the time of every workgroup:
    // signed ones, and a task's place found twice, 1 x 1537 on 32 heads 30.5 us, now 30.1)
    const int group = (int)((uint32_t)a.n_q_heads / (uint32_t)a.n_kv_heads);
    const int n_tasks = a.n_q_heads * n_rb;
    const int n_all = (S + 31) / 32;
    const int n_my = wave < n_all ? (int)((uint32_t)(n_all - wave + waves - 1) / (uint32_t)waves) : 0;     // tiles wave, wave + waves, ...

    // (the only ordinary loads; complete before the first LDS-direct load is issued)
    float weight_sum = (float)L;
    int raised = kWindowRaise;
    if (kWeighted) {
        float part = 0.f;
        for (int j = lane; j < L; j += 64) part += a.row_weights[a.w - L + j];
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) part += __shfl_xor(part, m, 64);
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(part) : : "memory");
        weight_sum = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, part)));
        if (!(weight_sum < 4294967296.f)) raised = max(0, kWindowRaise + 32 - __builtin_amdgcn_frexp_expf(weight_sum));      // (large weights leave less room)
    }

    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    const uint32_t ring = lds0 + wave * 2 * kTileBytes;
    const uint32_t weights_at = lds0 + waves * 2 * kTileBytes + wave * 256;
    const uint32_t factors_at = lds0 + waves * (2 * kTileBytes + 256) + wave * 128;
    const uint32_t sums_at = lds0 + waves * (2 * kTileBytes + 256 + 128) + wave * (256 + 128) * kTiles;
    const uint32_t moved_at = sums_at + 256 * kTiles + 16 * gl;
    const uint32_t stats_at = lds0 + waves * (2 * kTileBytes + 256 + 128 + (256 + 128) * kTiles);

    // ---- load side (as in score.hip): the LDS place of a lane is fixed by the instruction, so the swizzle picks the global chunk.
    // Rows kRowsPerLoad * i + ld_row: the swizzle of instruction i depends on i modulo kSwizzles only, the rest is wave-uniform.
    constexpr int kSwizzles = kChunks / kRowsPerLoad;
    const int ld_row = lane / kChunks, ld_chunk = lane % kChunks;
    const uint32_t k_row_bytes = (uint32_t)a.n_kv_heads * kRowBytes, q_row_bytes = (uint32_t)a.n_q_heads * kRowBytes;
    uint32_t k_off[kSwizzles];
#pragma unroll
    for (int j = 0; j < kSwizzles; ++j) k_off[j] = __umul24((uint32_t)ld_row, k_row_bytes) + 16 * (ld_chunk ^ ld_row ^ (kRowsPerLoad * j));
    auto load_part = [&](const char* base, uint32_t row_bytes, int last_row, uint32_t to) {      // rows past the last re-read it
#pragma unroll 1
        for (int i = 0; i < kTileLoads; ++i) {
            const int row = kRowsPerLoad * i + ld_row;
            lds_dma(base, __umul24((uint32_t)min(row, last_row), row_bytes) + 16 * (ld_chunk ^ (row & (kChunks - 1))), to + 1024 * i, false);
        }
    };
    // The stream's next element: the query rows of a task, then its key tiles.  (The divisions once per task, not in front of every tile.)
    int at_e = 0, at_task = n_my > 0 ? g : n_tasks, at_rb = 0;
    const char *at_q = nullptr, *at_k = nullptr;
    auto locate = [&]() {
        int h, kvh;
        if (kByKvHead) {
            const int r = (int)((uint32_t)at_task / (uint32_t)a.n_kv_heads), of_group = (int)((uint32_t)r / (uint32_t)n_rb);
            kvh = at_task - r * a.n_kv_heads;
            h = kvh * group + of_group;
            at_rb = r - of_group * n_rb;
        } else {
            h = (int)((uint32_t)at_task / (uint32_t)n_rb);
            kvh = (int)((uint32_t)h / (uint32_t)group);
            at_rb = at_task - h * n_rb;
        }
        at_q = (const char*)(a.q + ((size_t)(q_row_base + 32 * at_rb) * a.n_q_heads + __builtin_amdgcn_readfirstlane(h)) * D);
        at_k = (const char*)(a.k + ((size_t)(row0 + 32 * wave) * a.n_kv_heads + __builtin_amdgcn_readfirstlane(kvh)) * D);
    };
    auto request = [&](int slot) -> int {             // returns the number of load instructions issued (0: the stream has ended)
        if (at_task >= n_tasks) return 0;
        const uint32_t to = ring + slot * kTileBytes;
        int n = kTileLoads;
        if (at_e == 0) {
            locate();
            if (kWeighted) {
                lds_dma((const char*)(a.row_weights + (a.w - L) + 32 * at_rb), (uint32_t)min(li, L - 1 - 32 * at_rb) * 4, weights_at, true);
                n += kRowLoads;
            }
            load_part(at_q, q_row_bytes, L - 1 - 32 * at_rb, to);
        } else {
            const int key = 32 * (wave + waves * (at_e - 1));
            if (key + 32 <= S) {
#pragma unroll
                for (int i = 0; i < kTileLoads; ++i)
                    lds_dma(at_k + (size_t)(kRowsPerLoad * i) * k_row_bytes, k_off[i % kSwizzles], to + 1024 * i, false);
            } else {
                load_part(at_k, k_row_bytes, S - 1 - key, to);
            }
            at_k += (size_t)(32 * waves) * k_row_bytes;
        }
        if (++at_e > n_my) {
            at_e = 0;
            at_task += a.groups;
        }
        return n;
    };
    auto wait_front = [&](int behind) {               // until the element in front of the one requested last has landed
        if (behind == 0) wait_loads<0>();
        else if (kRowLoads == 0 || behind == kTileLoads) wait_loads<kTileLoads>();
        else wait_loads<kTileLoads + kRowLoads>();
    };
    const int f_row = li * kRowBytes, f_chunk = gl ^ (li & (kChunks - 1));      // operand row li, logical chunk 2*ks + gl
    auto copy_tile = [&](bf16x8 (&f)[kSteps], int slot) {
        int p = (int)ring + slot * kTileBytes + f_row, x = f_chunk;
        asm volatile("" : "+v"(p), "+v"(x));
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks)
            f[ks] = *(const bf16x8 __attribute__((address_space(3)))*)(uintptr_t)(uint32_t)(p + ((x ^ (2 * ks)) << 4));
    };

    // In front of LDS reads of what other lanes of the wavefront wrote: LDS serves a wavefront in order, but the compiler, which
    // knows nothing of other lanes, may have the lanes that did not write read first.
    auto lanes_meet = [&]() { asm volatile("" ::: "memory"); };
    auto rows_of = [&](uint32_t at, auto use) {   // a value per row to the lanes that hold the row's exponentials
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f32x4 x = ((const f32x4 __attribute__((address_space(3)))*)(uintptr_t)at)[2 * j];
#pragma unroll
            for (int e = 0; e < 4; ++e) use(4 * j + e, x[e]);
        }
    };

    for (int t = 0; t < n_my; ++t) *(lfloat_t)(uintptr_t)(sums_at + 256 * t + 4 * lane) = 0.f;
    const int my_row = 8 * ((li >> 2) & 3) + 4 * gl + (li & 3);      // the row whose sum sum_rows leaves in this lane
    request(0);
    int behind = request(1);
    int slot = 0;
    for (int i = 0, task = g; task < n_tasks; ++i, task += a.groups) {
        const int rb = at_rb;                         // (the task's first two elements have been requested, none of the next task)
        const int q_lo = first_row + 32 * rb;         // sequence position of the block's first row
        f32x16 s[kTiles];                             // exponentials of the wavefront's tiles
        float l[16], omega = 1.f;                     // the lane's share of the rows' sums
#pragma unroll
        for (int r = 0; r < 16; ++r) l[r] = 0.f;
        // The rows' references wait in LDS while the products run.  Finite, so that a row that has seen no key, or only
        // logits of -inf, keeps the sum zero.
        if (gl == 0) *(lfloat_t)(uintptr_t)(factors_at + 4 * li) = -FLT_MAX;
        lanes_meet();
        uint32_t moved = 0;                           // tiles in front of which references moved, by the exponents at moved_at
        if (n_my > 0) {
            bf16x8 qf[kSteps];
            wait_front(behind);
            copy_tile(qf, slot);
            if (kWeighted) omega = *(const lfloat_t)(uintptr_t)(weights_at + 4 * li);
            wait_lds();                               // in registers: the slot is free
            behind = request(slot);
            slot ^= 1;
#pragma unroll 1
            for (int t = 0; t < n_my; ++t) {
                bf16x8 kf[kSteps];
                f32x16 x, e;
                wait_front(behind);
                copy_tile(kf, slot);
                wait_lds();
                behind = request(slot);
                slot ^= 1;
#pragma unroll
                for (int r = 0; r < 16; ++r) x[r] = 0.f;
#pragma unroll
                for (int ks = 0; ks < kSteps; ++ks) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[ks], kf[ks], x, 0, 0, 0);
                const int key0 = 32 * (wave + waves * t);
                if (key0 + 31 > q_lo) {               // (uniform) keys that not every row sees
                    const int last = key0 + li - q_lo - 4 * gl;      // rows before this one do not see the lane's key
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (8 * (r >> 2) + (r & 3) < last) x[r] = -INFINITY;
                }
                if (t == 0 && li == 0) {              // the rows' logits of the first key (c > 0)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        f32x4 y;
#pragma unroll
                        for (int u = 0; u < 4; ++u) y[u] = fmaxf(-FLT_MAX, a.c * x[4 * j + u]);
                        ((f32x4 __attribute__((address_space(3)))*)(uintptr_t)(factors_at + 16 * gl))[2 * j] = y;
                    }
                }
                lanes_meet();
                float m[16], top = 0.f;
                rows_of(factors_at + 16 * gl, [&](int r, float y) { m[r] = y; });
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    e[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], a.c, -m[r]));
                    top = fmaxf(top, e[r]);
                }
                if (__ballot(!(top <= kWindowGrowth)) != 0) {
                    lanes_meet();
                    rows_of(factors_at + 16 * gl, [&](int r, float y) {
                        const int row = 8 * (r >> 2) + (r & 3);
                        const float to = fmaxf(y, a.c * max_of_half(x[r])), by = y - to;
                        l[r] *= __builtin_amdgcn_exp2f(by);
                        e[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], a.c, -to));
                        if (li == 0) {
                            ((lfloat_t)(uintptr_t)(factors_at + 16 * gl))[row] = to;
                            ((lfloat_t)(uintptr_t)moved_at)[32 * t + row] = by;
                        }
                    });
                    moved |= 1u << t;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) l[r] += e[r];
#pragma unroll
                for (int u = 0; u < kTiles; ++u)      // (t is wave-uniform: a branch and sixteen moves)
                    if (t == u) {
                        s[u] = e;
                        asm volatile("" : "+v"(s[u]));
                    }
            }
        }
        lanes_meet();
        const float l_row = sum_rows(l, li), m_own = *(const lfloat_t)(uintptr_t)(factors_at + 4 * li);
        const uint32_t stats = stats_at + (i & 1) * waves * 256;      // (two sets: one barrier per task is enough)
        if (gl == 0) *(lfloat_t)(uintptr_t)(stats + wave * 256 + 4 * li) = m_own;
        if (li < 16) *(lfloat_t)(uintptr_t)(stats + wave * 256 + 128 + 4 * my_row) = l_row;
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // lane li: row li over all wavefronts
        float ms[kWindowWaves], ls[kWindowWaves], m_all = -FLT_MAX, z = 0.f;
#pragma unroll
        for (int u = 0; u < kWindowWaves; ++u) {
            const uint32_t at = stats + min(u, waves - 1) * 256 + 4 * li;
            const float mu = *(const lfloat_t)(uintptr_t)at, lu = *(const lfloat_t)(uintptr_t)(at + 128);
            ms[u] = u < waves ? mu : -FLT_MAX;
            ls[u] = u < waves ? lu : 0.f;
            m_all = fmaxf(m_all, ms[u]);
        }
#pragma unroll
        for (int u = 0; u < kWindowWaves; ++u) z += ls[u] * __builtin_amdgcn_exp2f(ms[u] - m_all);
        float f = times_exp2(1.f, m_own - m_all, raised) / z;
        if (kWeighted) f *= omega;
        if (32 * rb + li >= L) f = 0.f;               // a row past the window adds nothing
        const uint32_t odd = (uint32_t)__ballot(!(f < INFINITY));
        if (__builtin_expect(odd != 0, 0)) {          // a row without a finite sum: NaN at the keys it sees, and not by way of 0 * NaN at later ones
            if (!(f < INFINITY)) f = 0.f;
#pragma unroll 1
            for (int t = 0; t < n_my; ++t)
                if (32 * (wave + waves * t) + li <= q_lo + 31 - __clz((int)odd)) *(lfloat_t)(uintptr_t)(sums_at + 256 * t + 4 * lane) = NAN;
        }
        if (gl == 0) *(lfloat_t)(uintptr_t)(factors_at + 4 * li) = f;
        lanes_meet();
        float fr[16];
        rows_of(factors_at + 16 * gl, [&](int r, float x) { fr[r] = x; });
#pragma unroll
        for (int t = kTiles - 1; t >= 0; --t) {
            if (t < n_my) {
                float p4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int r = 0; r < 16; ++r) p4[r & 3] = __builtin_fmaf(s[t][r], fr[r], p4[r & 3]);
                const lfloat_t at = (lfloat_t)(uintptr_t)(sums_at + 256 * t + 4 * lane);
                *at = *at + ((p4[0] + p4[1]) + (p4[2] + p4[3]));
            }
            if (moved >> t & 1) rows_of(moved_at + 128 * t, [&](int r, float x) { fr[r] = times_exp2(fr[r], x, 0); });
        }
    }
    // every load issued above has been waited for; the two half-wavefronts' rows
    const float norm = __builtin_amdgcn_ldexpf(1.0f / ((float)a.n_q_heads * weight_sum), -raised);
    float* dst = a.sums + (size_t)g * a.total_tokens + row0;
    for (int t = 0; t < n_my; ++t) {
        const float mine = *(lfloat_t)(uintptr_t)(sums_at + 256 * t + 4 * lane);
        const float sum = mine + __shfl_xor(mine, 32, 64);
        const int key = 32 * (wave + waves * t) + li;
        if (gl == 0 && key < S) dst[key] = sum * norm;
    }
}

}  // namespace pyr
