// Device code of the segmented top-k (Algorithm 1, TopP(A_e, p) with the retention ratio turned
// into a count, followed by the recent window that is always kept), written for a workgroup of
// 512 or 1024 lanes; the selection kernel (select.hip) runs it, one workgroup per sequence.
//
// The paper names the sort inside TopP as the one extra cost of the method that matters
// (Appendix A.1).  Nothing is sorted here: the workgroup finds the need-th largest context score and the position of the
// last key of that value that is admitted (ties go to the lower positions), by a histogram over the keys' distance from the
// smallest one, then emits the survivors with wavefront ballots and prefix counts, which yields ascending positions
// for free.
//
// Bound: latency (a few KB per sequence, one workgroup): loads that depend on each other, barriers, and atomics on one
// histogram bin, which LDS serves one after the other.  So
// - a wavefront owns consecutive positions from beginning to end and a lane keeps its keys in registers where there are kRegKeys of them at
//   most; else they are staged in LDS, and where that is too small re-read from memory in every pass;
// - the bins divide the span between the smallest and the largest key, not the bits in which keys differ: scores spread over
//   ten octaves fill all bins (with leading bits 120 of 2048: five lanes of a wavefront on one bin, and bins too full to stop at);
// - a bin of at most kCandidates keys ends the search: they are ranked against each other by value and position.  Of equal keys only
//   kEqualCandidates: more are counted in order, which costs two passes and not a look of every key at every other (scores of a few values,
//   250 keys of each, one sequence of 2048 tokens 9.0 ranked, 5.0 counted, 6.2 by digits; 64 of each 6.0 / 4.9 / 6.2, 40 of each 5.5 / 5.7 / 6.2).
// One pass over the bins at the score distributions of the method.
// - beyond the registers' reach, whole blocks of a wavefront's positions go without the checks of the last one (half the instructions, which
//   is what 16 keys a lane and more wait for: 16384 tokens 13.9 -> 10.8, 60000 69 -> 39).
// us per launch, leading bits in digits of 11 from LDS / now (a launch that does nothing takes 4 of these): one sequence of
// 256 tokens 5.1 / 4.2, of 2048 6.5 / 4.7, of 8192 11.4 / 8.2, four of 32768 28.6 / 17.0, two of 60000 73 / 39.
// Tried and taken back: 32 instead of 8 scores a lane has in flight while they are loaded (16384 tokens 13.9 -> 14.9); the whole blocks for
// keys in registers too, where the second copy of the code costs more than it saves (4096 tokens 6.4 -> 6.9, 8192 8.2 -> 9.0).
#pragma once

#include "pyr_internal.h"

namespace pyr {

constexpr int kRegKeys = 8;                 // keys of a lane in registers, at most
constexpr int kCandidates = 256;
constexpr int kEqualCandidates = 48;

// where a lane finds its keys after they have been loaded
enum KeySource { kInRegisters, kInLds, kInMemory };

template <int N> struct Int { static constexpr int value = N; };

// LDS the selection needs besides the staged keys
template <int kT>
struct SelectShared {
    uint2 hist[kT];                          // 2 * kT bins
    uint64_t cand[kCandidates];
    int count[16];                           // per wavefront
    int found[3];                            // bin, place of the threshold in it, keys in it
    uint32_t wave_min[16], wave_max[16], part[16];
    uint32_t n_cand;
    uint64_t threshold;
};

// Monotone map float -> uint32 (larger float, larger key); -0 is folded onto +0 so that
// equal floats always get equal keys.
__device__ __forceinline__ uint32_t ordered_key(float x) {
    uint32_t b = __float_as_uint(x);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// The order of the selection: by key, then the lower position first.
__device__ __forceinline__ uint64_t ranked(uint32_t key, int i) { return (uint64_t)key << 32 | (uint32_t)~i; }

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

template <int kCtrl, int kRowMask = 0xf>
__device__ __forceinline__ uint32_t lanes(uint32_t old, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, kCtrl, kRowMask, 0xf, false);
}

// op over the 64 lanes of a wavefront, in every lane: mirrors of 16 and 8 lanes, reversed quads, swapped pairs, then
// rows of 16 and halves.
template <class Op>
__device__ __forceinline__ uint32_t over_lanes(uint32_t x, Op op) {
    x = op(x, lanes<0x140>(x, x));
    x = op(x, lanes<0x141>(x, x));
    x = op(x, lanes<0x1b>(x, x));
    x = op(x, lanes<0xb1>(x, x));
    auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = op(r[0], r[1]);
    auto s = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return op(s[0], s[1]);
}

// The sum of x over this lane and the lanes before it: shifts inside rows of 16, then the rows' totals handed on.
__device__ __forceinline__ uint32_t sum_up_to_lane(uint32_t x) {
    x += lanes<0x111>(0u, x);
    x += lanes<0x112>(0u, x);
    x += lanes<0x114>(0u, x);
    x += lanes<0x118>(0u, x);
    x += lanes<0x142, 0xa>(0u, x);
    x += lanes<0x143, 0xc>(0u, x);
    return x;
}

// The sum of what the wavefronts before this one counted.
template <int kW>
__device__ __forceinline__ int sum_before(const int* count, int wave) {
    int n = 0;
#pragma unroll
    for (int u = 0; u < kW; ++u) n += u < wave ? count[u] : 0;
    return n;
}

// The smallest kept ranked() of the keys that `each` visits: the need-th largest, 0 < need <= number of keys.  Their
// minimum and maximum are known, sh->hist is zero and sh->n_cand too, all behind a barrier; ends behind one.
template <int kT, class Each>
__device__ uint64_t find_threshold(const Each& each, int need, uint32_t kmin, uint32_t kmax, SelectShared<kT>* sh) {
    constexpr int kW = kT / 64, kBinBits = kT == 512 ? 10 : 11;
    static_assert(2 * kT == 1 << kBinBits, "two bins a lane");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t* const hist = (uint32_t*)sh->hist;
    if (kmin == kmax) return ranked(kmin, need - 1);
    int remaining = need, bits = 32 - __clz((int)(kmax - kmin));      // the keys in question are base + less than 2^bits
    uint32_t base = kmin;
    bool whole = true;                                                // ... which are all of them
    while (true) {
        const int shift = bits > kBinBits ? bits - kBinBits : 0;
        each([&](uint32_t key, int, bool valid) {
            const uint32_t from = key - base;
            if (valid && (whole || from >> bits == 0)) {
                // equal bins throughout a wavefront (many equal scores) are counted by one lane
                const uint32_t bin = from >> shift, first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
                const uint64_t here = __ballot(true);
                if (__ballot(bin == first) == here) {
                    if (lane == __ffsll((unsigned long long)here) - 1) atomicAdd(&hist[first], (uint32_t)__popcll(here));
                } else {
                    atomicAdd(&hist[bin], 1u);
                }
            }
        });
        __syncthreads();
        // lane t owns the bins 2 * (kT - 1 - t) + 1 and + 0, in this (descending) order
        const uint2 h = sh->hist[kT - 1 - tid];
        const int mine = (int)(h.x + h.y), incl = (int)sum_up_to_lane(h.x + h.y);
        if (lane == 63) sh->count[wave] = incl;
        __syncthreads();
        const int before = incl - mine + sum_before<kW>(sh->count, wave);
        if (before < remaining && remaining <= before + mine) {
            const bool upper = remaining <= before + (int)h.y;
            sh->found[0] = 2 * (kT - 1 - tid) + upper;
            sh->found[1] = remaining - before - (upper ? 0 : (int)h.y);
            sh->found[2] = (int)(upper ? h.y : h.x);
        }
        __syncthreads();
        const uint32_t bin = (uint32_t)sh->found[0];
        const int in_bin = sh->found[2];
        remaining = sh->found[1];
        base += bin << shift;
        bits = shift;
        whole = false;
        if (in_bin <= kEqualCandidates || (bits > 0 && in_bin <= kCandidates)) {
            each([&](uint32_t key, int i, bool valid) {
                if (valid && (key - base) >> bits == 0) sh->cand[atomicAdd(&sh->n_cand, 1u)] = ranked(key, i);
            });
            __syncthreads();
            if (tid < in_bin) {
                const uint64_t my = sh->cand[tid];
                int larger = 0;
#pragma unroll 4
                for (int u = 0; u < in_bin; ++u) larger += sh->cand[u] > my;
                if (larger == remaining - 1) sh->threshold = my;
            }
            __syncthreads();
            return sh->threshold;
        }
        if (bits == 0) {                      // the bin's keys are equal: the remaining-th of them in order
            int n = 0;
            each([&](uint32_t key, int, bool valid) { n += __popcll(__ballot(valid && key == base)); });
            if (lane == 0) sh->count[wave] = n;
            __syncthreads();
            int at = remaining - sum_before<kW>(sh->count, wave);
            if (0 < at && at <= n) {
                each([&](uint32_t key, int i, bool valid) {
                    const bool equal = valid && key == base;
                    const uint64_t mask = __ballot(equal);
                    if (equal && __popcll(mask & lanemask_lt()) == at - 1) sh->threshold = ranked(key, i);
                    at -= __popcll(mask);
                });
            }
            __syncthreads();
            return sh->threshold;
        }
        sh->hist[tid] = make_uint2(0u, 0u);
        __syncthreads();
    }
}

// The selection of sequence b by the calling workgroup (all kT lanes take part; uniform control
// flow).  groups > 1: the scores are first added up from parts[groups][total_tokens], in order, and written by the workgroup that is to.
// kInRegisters: sequences of kRegKeys * kT tokens at most; kInLds: lds_keys has room for a sequence.
// sink.begin(first place, number of rows) is called once, sink(rank, row) for every kept row.
template <int kT, KeySource kSource, class Sink>
__device__ void select_sequence(int b, const float* __restrict__ parts, int groups, int32_t total_tokens, float* scores, bool write_scores,
                                const int32_t* __restrict__ seq_offsets, const int32_t* __restrict__ keep_len, int32_t w, uint32_t* lds_keys,
                                SelectShared<kT>* sh, Sink& sink) {
    constexpr int kW = kT / 64, kRegs = kSource == kInRegisters ? kRegKeys : 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t row0 = seq_offsets[b];
    const int S = seq_offsets[b + 1] - row0;
    const int L = min(w, S);
    const int k = min(max(keep_len[b], L), S);
    const int C = S - L;                        // context positions, the candidates
    const int need = k - L;                     // how many of them survive
    float* sc = scores + row0;

    // packed position of this sequence's output: sum of the keep counts before it
    uint32_t part = 0;
    for (int u = tid; u < b; u += kT) part += (uint32_t)keep_len[u];

    // wavefront `wave` owns the positions [lo, lo + seg) of the n that are loaded
    const int n = groups > 1 ? S : C;
    const int seg = (n + kT - 1) / kT * 64, lo = wave * seg;
    const bool decide = need > 0 && need < C;
    uint32_t keys[kRegs], kmin = 0xffffffffu, kmax = 0u;
    if (decide || groups > 1) {
        // kAhead scores a lane has in flight, kRows rows of partial sums of each (the latency of a row at a time is what this would wait for)
        const float* __restrict__ from = groups > 1 ? parts + row0 : sc;
        const int end = min(n, lo + seg);
        auto stage = [&](auto ahead, auto rows) {
            constexpr int kAhead = decltype(ahead)::value, kRows = decltype(rows)::value;
            auto block = [&](int at, auto whole) {      // kAhead * 64 positions; whole: all of them candidates
                constexpr bool kWhole = decltype(whole)::value != 0;
                const int i0 = at + lane;
                float x[kAhead];
                if (kRows == 1) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) x[u] = kWhole || i0 + 64 * u < end ? from[i0 + 64 * u] : 0.f;
                } else {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) x[u] = 0.f;
                    for (int g0 = 0; g0 < groups; g0 += kRows) {
                        float y[kRows][kAhead];
#pragma unroll
                        for (int g = 0; g < kRows; ++g)
#pragma unroll
                            for (int u = 0; u < kAhead; ++u)
                                y[g][u] = (kWhole || i0 + 64 * u < end) && g0 + g < groups ? from[(size_t)(g0 + g) * total_tokens + i0 + 64 * u] : 0.f;
#pragma unroll
                        for (int g = 0; g < kRows; ++g)
#pragma unroll
                            for (int u = 0; u < kAhead; ++u) x[u] += y[g][u];
                    }
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int i = i0 + 64 * u;
                    const uint32_t key = ordered_key(x[u]);
                    if (kSource == kInRegisters) keys[u] = key;
                    if (!kWhole && i >= end) continue;
                    if (groups > 1 && write_scores) sc[i] = x[u];
                    if (!kWhole && i >= C) continue;
                    if (kSource == kInLds) lds_keys[i] = key;
                    kmin = min(kmin, key);
                    kmax = max(kmax, key);
                }
            };
            int at = lo;
            if (kSource != kInRegisters)
                for (; at + 64 * kAhead <= min(end, C); at += 64 * kAhead) block(at, Int<1>{});
            for (; at < end; at += 64 * kAhead) block(at, Int<0>{});
        };
        if (groups <= 1) stage(Int<8>{}, Int<1>{});
        else if (seg > 256) stage(Int<8>{}, Int<4>{});
        else if (seg > 128) stage(Int<4>{}, Int<8>{});
        else stage(Int<2>{}, Int<16>{});
        sh->hist[tid] = make_uint2(0u, 0u);
    }
    kmin = over_lanes(kmin, [](uint32_t x, uint32_t y) { return min(x, y); });
    kmax = over_lanes(kmax, [](uint32_t x, uint32_t y) { return max(x, y); });
    part = over_lanes(part, [](uint32_t x, uint32_t y) { return x + y; });
    if (lane == 0) {
        sh->part[wave] = part;
        sh->wave_min[wave] = kmin;
        sh->wave_max[wave] = kmax;
        if (wave == 0) sh->n_cand = 0;
    }
    __syncthreads();                            // (also: the scores written above are visible to the workgroup)
    int out_base = 0;
#pragma unroll
    for (int u = 0; u < kW; ++u) {
        out_base += (int)sh->part[u];
        kmin = min(kmin, sh->wave_min[u]);
        kmax = max(kmax, sh->wave_max[u]);
    }
    sink.begin(out_base, k);

    // the recent window is always kept (A_e ranks the columns before it only)
    for (int i = tid; i < L; i += kT) sink(need + i, row0 + C + i);
    if (need == 0) return;
    if (need == C) {                            // nothing to evict: identity
        for (int i = tid; i < C; i += kT) sink(i, row0 + i);
        return;
    }

    auto key_at = [&](int i) { return kSource == kInLds ? lds_keys[i] : ordered_key(sc[i]); };
    // use(key, position, whether there is one) for the wavefront's keys in ascending order, all lanes together
    auto each = [&](auto use) {
        if constexpr (kSource == kInRegisters) {
#pragma unroll
            for (int u = 0; u < kRegs; ++u) {
                if (64 * u >= seg) break;
                use(keys[u], lo + 64 * u + lane, lo + 64 * u + lane < C);
            }
        } else {
            constexpr int kAhead = kSource == kInLds ? 4 : 8;
            const int hi = min(C, lo + seg);
            int at = lo;
            for (; at + 64 * kAhead <= hi; at += 64 * kAhead) {      // (nothing to check: half the instructions)
                uint32_t x[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) x[u] = key_at(at + lane + 64 * u);
#pragma unroll
                for (int u = 0; u < kAhead; ++u) use(x[u], at + lane + 64 * u, true);
            }
#pragma unroll 1
            for (; at < hi; at += 64) {
                const int i = at + lane;
                use(i < hi ? key_at(i) : 0u, i, i < hi);
            }
        }
    };
    const uint64_t threshold = find_threshold<kT>(each, need, kmin, kmax, sh);
    int kept = 0;
    each([&](uint32_t key, int i, bool valid) { kept += __popcll(__ballot(valid && ranked(key, i) >= threshold)); });
    if (lane == 0) sh->count[wave] = kept;
    __syncthreads();
    int to = sum_before<kW>(sh->count, wave);
    const uint64_t lt = lanemask_lt();
    each([&](uint32_t key, int i, bool valid) {
        const bool keep = valid && ranked(key, i) >= threshold;
        const uint64_t mask = __ballot(keep);
        if (keep) sink(to + __popcll(mask & lt), row0 + i);
        to += __popcll(mask);
    });
}

}  // namespace pyr
