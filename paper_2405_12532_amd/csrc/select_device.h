// Device code of the segmented top-k (Algorithm 1, TopP(A_e, p) with the retention ratio turned
// into a count, followed by the recent window that is always kept), written for a workgroup of
// any multiple of 64 lanes; the selection kernel (select.hip) runs it, one workgroup per sequence.
//
// The paper names the sort inside TopP as the one extra cost of the method that matters
// (Appendix A.1).  Nothing is sorted here: the workgroup finds the value of the need-th largest
// context score with a most-significant-digit-first radix select on the fp32 bit patterns, then
// emits the survivors with wavefront ballots and prefix counts, which yields ascending positions
// for free.  Ties at the threshold go to the lower positions.
//
// Bound: latency (a few KB per sequence, one workgroup): barriers and passes over the keys.  The radix
// select therefore skips the leading bits that all keys share (minimum and maximum are known from
// staging them), takes digits of 11 bits, and stops as soon as the digit's bin holds at most
// kCandidates keys, which are then ranked against each other directly: at the score distributions of
// the method that is one pass instead of the four that fixed 8-bit digits take (us per launch, before / now: one
// sequence of 256 tokens 6.4 / 4.9, of 2048 9.5 / 6.3, of 8192 27 / 10.4, four of 32768 64 / 25).
#pragma once

#include "pyr_internal.h"

namespace pyr {

constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;
constexpr int kCandidates = 256;

template <int N> struct Int { static constexpr int value = N; };

// LDS the selection needs besides the staged keys
struct SelectShared {
    uint32_t hist[kBins];
    uint32_t cand[kCandidates];
    int wave_cnt[2 * 16];
    int red[16];
    uint32_t wave_min[16], wave_max[16];
    int n_cand;
    int bcast[3];
    uint32_t tau;
};

// Monotone map float -> uint32 (larger float, larger key); -0 is folded onto +0 so that
// equal floats always get equal keys.
__device__ __forceinline__ uint32_t ordered_key(float x) {
    uint32_t b = __float_as_uint(x);
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ uint64_t lanemask_lt() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

template <bool kStaged>
__device__ __forceinline__ uint32_t get_key(const uint32_t* lds_keys, const float* __restrict__ g, int i) {
    if (kStaged) return lds_keys[i];
    return ordered_key(g[i]);
}

// The body after the keys are reachable through get_key<kStaged> and their minimum and maximum are known
// (sh->hist zeroed, both behind a barrier); kT lanes (a multiple of 64, at most 1024).
template <bool kStaged, int kT>
__device__ void select_body(const uint32_t* lds_keys, const float* __restrict__ sc, int C, int need, uint32_t kmin, uint32_t kmax,
                            int32_t row0, int32_t* __restrict__ out, SelectShared* sh) {
    constexpr int kW = kT / 64;
    constexpr int kPer = kBins / kT;            // bins a lane scans
    constexpr int kAhead = 4;                   // keys a lane fetches before it uses the first
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // ---- radix select: threshold key tau and the number of ties still to admit
    uint32_t tau = kmin;
    int ties = need;                            // (all keys equal: the first `need` of them)
    if (kmin != kmax) {
        int bits_left = 32 - __clz((int)(kmin ^ kmax));        // the keys differ in their low bits_left bits only
        int remaining = need;
        uint64_t prefix = (uint64_t)kmin >> bits_left;
        while (true) {
            const int nbits = min(kDigitBits, bits_left), shift = bits_left - nbits;
            for (int i0 = tid - lane; i0 < C; i0 += kAhead * kT) {      // (whole wavefronts: the ballots below)
                uint32_t keys[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int i = i0 + u * kT + lane;
                    keys[u] = i < C ? get_key<kStaged>(lds_keys, sc, i) : 0u;
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const bool match = i0 + u * kT + lane < C && ((uint64_t)keys[u] >> bits_left) == prefix;
                    const uint32_t digit = (keys[u] >> shift) & ((1u << nbits) - 1);
                    // equal digits throughout a wavefront (many equal scores) are counted by one lane
                    const uint64_t active = __ballot(match);
                    if (active == 0) continue;
                    const int leader = __ffsll((unsigned long long)active) - 1;
                    const uint32_t dl = __builtin_amdgcn_readlane(digit, leader);
                    if (__ballot(match && digit == dl) == active) {
                        if (lane == leader) atomicAdd(&sh->hist[dl], (uint32_t)__popcll(active));
                    } else if (match) {
                        atomicAdd(&sh->hist[digit], 1u);
                    }
                }
            }
            __syncthreads();
            // lane t owns bins kBins-1 - kPer*t downwards (descending order of value)
            const int top = kBins - 1 - kPer * tid;
            uint32_t h[kPer];
            int mine = 0;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                h[u] = sh->hist[top - u];
                mine += (int)h[u];
            }
            int incl = mine;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int up = __shfl_up(incl, d);
                if (lane >= d) incl += up;
            }
            if (lane == 63) sh->red[wave] = incl;
            if (tid == 0) sh->n_cand = 0;
            __syncthreads();
            int run = incl - mine;
            for (int u = 0; u < wave; ++u) run += sh->red[u];
            if (run < remaining && remaining <= run + mine) {
#pragma unroll
                for (int u = 0; u < kPer; ++u) {
                    if (run < remaining && remaining <= run + (int)h[u]) {
                        sh->bcast[0] = top - u;
                        sh->bcast[1] = remaining - run;
                        sh->bcast[2] = (int)h[u];
                    }
                    run += (int)h[u];
                }
            }
            __syncthreads();
            prefix = (prefix << nbits) | (uint32_t)sh->bcast[0];
            remaining = sh->bcast[1];
            const int in_bin = sh->bcast[2];
            bits_left = shift;
            if (bits_left == 0) {                              // every bit decided: the bin's keys are equal
                tau = (uint32_t)prefix;
                ties = remaining;
                break;
            }
            if (in_bin <= kCandidates) {
#pragma unroll 4
                for (int i = tid; i < C; i += kT) {
                    const uint32_t key = get_key<kStaged>(lds_keys, sc, i);
                    if (((uint64_t)key >> bits_left) == prefix) sh->cand[atomicAdd(&sh->n_cand, 1)] = key;
                }
                __syncthreads();
                if (tid < in_bin) {
                    const uint32_t my = sh->cand[tid];
                    int gt = 0, eq = 0;
                    for (int u = 0; u < in_bin; ++u) {
                        const uint32_t o = sh->cand[u];
                        gt += o > my;
                        eq += o == my;
                    }
                    if (gt < remaining && remaining <= gt + eq) {      // (equal candidates all write the same)
                        sh->tau = my;
                        sh->bcast[0] = remaining - gt;
                    }
                }
                __syncthreads();
                tau = sh->tau;
                ties = sh->bcast[0];
                break;
            }
            for (int i = tid; i < kBins; i += kT) sh->hist[i] = 0;
            __syncthreads();
        }
    }
    // ties >= 1 keys equal to tau are admitted, lowest positions first

    // ---- ordered emission: wavefront `wave` owns positions [wave*seg, (wave+1)*seg)
    const int seg = (C + kW * 64 - 1) / (kW * 64) * 64;
    const int lo = wave * seg;
    const int hi = min(C, lo + seg);
    int n_gt = 0, n_eq = 0;
#pragma unroll 4
    for (int i = lo + lane; i < hi; i += 64) {
        const uint32_t key = get_key<kStaged>(lds_keys, sc, i);
        n_gt += key > tau;
        n_eq += key == tau;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        n_gt += __shfl_xor(n_gt, d);
        n_eq += __shfl_xor(n_eq, d);
    }
    if (lane == 0) { sh->wave_cnt[2 * wave] = n_gt; sh->wave_cnt[2 * wave + 1] = n_eq; }
    __syncthreads();
    int gt_before = 0, eq_before = 0;
    for (int u = 0; u < wave; ++u) { gt_before += sh->wave_cnt[2 * u]; eq_before += sh->wave_cnt[2 * u + 1]; }
    int kept_cnt = gt_before + min(eq_before, ties);
    const uint64_t lt = lanemask_lt();
    for (int i0 = lo; i0 < hi; i0 += 64 * kAhead) {
        uint32_t keys[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + 64 * u + lane;
            keys[u] = i < hi ? get_key<kStaged>(lds_keys, sc, i) : 0u;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + 64 * u + lane;
            const bool gt = i < hi && keys[u] > tau;
            const bool eq = i < hi && keys[u] == tau;
            const uint64_t eq_mask = __ballot(eq);
            const int eq_rank = eq_before + __popcll(eq_mask & lt);
            const bool keep = gt || (eq && eq_rank < ties);
            const uint64_t keep_mask = __ballot(keep);
            if (keep) out[kept_cnt + __popcll(keep_mask & lt)] = row0 + i;
            kept_cnt += __popcll(keep_mask);
            eq_before += __popcll(eq_mask);
        }
    }
}

// The selection of sequence b by the calling workgroup (all kT lanes take part; uniform control
// flow).  groups > 1: the scores are first added up from parts[groups][total_tokens], in order, and written.
// lds_keys: room for lds_cap keys; scores of longer contexts are re-read from memory in
// every pass.  Also writes out_offsets[b + 1] (and out_offsets[0] for b == 0).
template <int kT>
__device__ void select_sequence(int b, const float* __restrict__ parts, int groups, int32_t total_tokens, float* scores,
                                const int32_t* __restrict__ seq_offsets, const int32_t* __restrict__ keep_len, int32_t w, uint32_t* lds_keys, int32_t lds_cap,
                                SelectShared* sh, int32_t* __restrict__ kept_idx, int32_t* __restrict__ out_offsets) {
    constexpr int kW = kT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t row0 = seq_offsets[b];
    const int S = seq_offsets[b + 1] - row0;
    const int L = min(w, S);
    const int k = min(max(keep_len[b], L), S);
    const int C = S - L;                        // context positions, the candidates
    const int need = k - L;                     // how many of them survive
    float* sc = scores + row0;

    // packed position of this sequence's output: sum of the keep counts before it
    int part = 0;
    for (int u = tid; u < b; u += kT) part += keep_len[u];

    // keys to LDS (if they fit), their minimum and maximum
    const bool staged = C <= lds_cap;
    const bool ranked = need > 0 && need < C;   // else there is nothing to decide
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    if (ranked || groups > 1) {
        // kAhead scores a lane has in flight, kRows rows of partial sums of each (the latency of a row at a time is what this would wait for)
        const float* __restrict__ from = groups > 1 ? parts + row0 : sc;
        const int n = groups > 1 ? S : C;
        auto stage = [&](auto ahead, auto rows) {
            constexpr int kAhead = decltype(ahead)::value, kRows = decltype(rows)::value;
            for (int i0 = tid; i0 < n; i0 += kAhead * kT) {
                float x[kAhead];
                if (kRows == 1) {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) x[u] = i0 + u * kT < n ? from[i0 + u * kT] : 0.f;
                } else {
#pragma unroll
                    for (int u = 0; u < kAhead; ++u) x[u] = 0.f;
                    for (int g0 = 0; g0 < groups; g0 += kRows) {
                        float y[kRows][kAhead];
#pragma unroll
                        for (int g = 0; g < kRows; ++g)
#pragma unroll
                            for (int u = 0; u < kAhead; ++u)
                                y[g][u] = i0 + u * kT < n && g0 + g < groups ? from[(size_t)(g0 + g) * total_tokens + i0 + u * kT] : 0.f;
#pragma unroll
                        for (int g = 0; g < kRows; ++g)
#pragma unroll
                            for (int u = 0; u < kAhead; ++u) x[u] += y[g][u];
                    }
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int i = i0 + u * kT;
                    if (i >= n) break;
                    if (groups > 1) sc[i] = x[u];
                    if (i >= C) break;
                    const uint32_t key = ordered_key(x[u]);
                    if (staged) lds_keys[i] = key;
                    kmin = min(kmin, key);
                    kmax = max(kmax, key);
                }
            }
        };
        if (groups <= 1) stage(Int<8>{}, Int<1>{});
        else if (n > 4 * kT) stage(Int<8>{}, Int<4>{});
        else if (n > 2 * kT) stage(Int<4>{}, Int<8>{});
        else stage(Int<2>{}, Int<16>{});
        for (int i = tid; i < kBins; i += kT) sh->hist[i] = 0;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        part += __shfl_xor(part, d);
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, d));
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, d));
    }
    if (lane == 0) {
        sh->red[wave] = part;
        sh->wave_min[wave] = kmin;
        sh->wave_max[wave] = kmax;
    }
    __syncthreads();                            // (also: the scores written above are visible to the workgroup)
    int out_base = 0;
#pragma unroll
    for (int u = 0; u < kW; ++u) {
        out_base += sh->red[u];
        kmin = min(kmin, sh->wave_min[u]);
        kmax = max(kmax, sh->wave_max[u]);
    }
    if (tid == 0) {
        out_offsets[b + 1] = out_base + k;
        if (b == 0) out_offsets[0] = 0;
    }
    int32_t* __restrict__ out = kept_idx + out_base;

    // the recent window is always kept (A_e ranks the columns before it only)
    for (int i = tid; i < L; i += kT) out[need + i] = row0 + C + i;
    if (need == 0) return;
    if (need == C) {                            // nothing to evict: identity
        for (int i = tid; i < C; i += kT) out[i] = row0 + i;
        return;
    }
    __syncthreads();                            // (red is used again below)
    if (staged) select_body<true, kT>(lds_keys, sc, C, need, kmin, kmax, row0, out, sh);
    else select_body<false, kT>(lds_keys, sc, C, need, kmin, kmax, row0, out, sh);
}

}  // namespace pyr
