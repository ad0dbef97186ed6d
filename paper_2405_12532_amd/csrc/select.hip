// Launch of the segmented top-k (Algorithm 1, TopP(A_e, p); see select_device.h): one workgroup per sequence.
#include "select_device.h"

namespace pyr {
namespace {

constexpr int kFusedLanes = 512;
constexpr int kLdsKeys = 36864;            // 144 KiB of the 160 KiB LDS of a gfx950 compute unit

// kept_idx and out_offsets of sequence b
struct ToMemory {
    int32_t *kept_idx, *out_offsets;
    int b;
    __device__ void begin(int base, int rows) {
        kept_idx += base;
        if (threadIdx.x != 0) return;
        out_offsets[b + 1] = base + rows;
        if (b == 0) out_offsets[0] = 0;
    }
    __device__ void operator()(int rank, int32_t row) { kept_idx[rank] = row; }
};

// The same, by the workgroups of a sequence together: this one keeps the ranks [lo, hi) in LDS and writes them.
struct ToPart {
    ToMemory memory;
    int32_t* rows;                     // LDS
    int part, parts, room, base, lo, hi;
    __device__ void begin(int first, int n) {
        const int size = (n + parts - 1) / parts;
        base = first;
        lo = min(n, part * size);
        hi = min(n, lo + min(size, room));
        if (part == 0) memory.begin(first, n);
        else memory.kept_idx += first;
    }
    __device__ void operator()(int rank, int32_t row) {
        if (rank < lo || rank >= hi) return;
        rows[rank - lo] = row;
        memory(rank, row);
    }
};

template <int kT, KeySource kSource>
__global__ __launch_bounds__(kT) void select_topk_kernel(
    const float* __restrict__ parts, int32_t groups, int32_t total_tokens, float* scores,
    const int32_t* __restrict__ seq_offsets, const int32_t* __restrict__ keep_len, int32_t w,
    int32_t* __restrict__ kept_idx, int32_t* __restrict__ out_offsets) {
    extern __shared__ uint32_t lds_keys[];
    __shared__ SelectShared<kT> sh;
    ToMemory sink{kept_idx, out_offsets, (int)blockIdx.x};
    select_sequence<kT, kSource>(blockIdx.x, parts, groups, total_tokens, scores, true, seq_offsets, keep_len, w, lds_keys, &sh, sink);
}

// The selection and the gather of a small batch in one launch: `split` workgroups per sequence, each of which finds the threshold for
// itself and copies its part of the kept rows (`room` at most).  Bound: latency, and a launch less of it.  The copy goes by 16 bytes and not by rows,
// so that all of a workgroup's (16 KB where the batch is as large as this launch takes) are on their way at once whatever a row's
// length: whole calls, two launches / one with a wavefront per row / one (us): 203 x 55 tokens on 2/1 heads, d = 64 17.8 / 22.0 / 13.8, 16 x 370
// 20.2 / 21.8 / 17.8, 1 x 64 on 32 heads, d = 128 17.9 / 16.7 / 15.3.  (Held
// to 64 registers, as if a compute unit had more than one of these workgroups, it spills: 1 to 3 % on the whole call.)
// Sources: GatherSources, or K and V alone, which leaves the arguments at 108 bytes (112 and less are 0.7 us less host time a launch).
struct TwoSources {
    const u32x4* src[2];
    u32x4* dst[2];
    int32_t row_chunks;                // of either
    __device__ __forceinline__ int32_t all() const { return 2 * row_chunks; }
    __device__ __forceinline__ int32_t piece(int32_t c, const u32x4** from, u32x4** to, int32_t* chunks) const {
        const bool y = c >= row_chunks;
        *from = y ? src[1] : src[0];
        *to = y ? dst[1] : dst[0];
        *chunks = row_chunks;
        return y ? c - row_chunks : c;
    }
    __device__ __forceinline__ void position(int32_t, int64_t) const {}
};
static_assert(6 * sizeof(void*) + sizeof(TwoSources) + 5 * sizeof(int32_t) <= 112, "short arguments");
struct AnySources {
    GatherSources g;
    __device__ __forceinline__ int32_t end1() const { return g.chunks[0] + (g.n > 1 ? g.chunks[1] : 0); }
    __device__ __forceinline__ int32_t all() const { return end1() + (g.n > 2 ? g.chunks[2] : 0); }
    __device__ __forceinline__ int32_t piece(int32_t c, const u32x4** from, u32x4** to, int32_t* chunks) const {      // its place in the row of its source
        const int y = (c >= g.chunks[0]) + (c >= end1());
        // (Opaque, in scalar registers: of a choice between three arguments the compiler makes a load of each lane from the one it needs, two trips to memory
        // in front of every 16 bytes.  Updates of 20 x 125 rows with ids on 32/8 heads, d = 64 14.6 us, now 14.1, 2 x 200 tokens on 32/8 heads with
        // hidden rows and ids 16.8 / 16.1.)
        const u32x4 *s0 = g.src[0], *s1 = g.src[1], *s2 = g.src[2];
        u32x4 *d0 = g.dst[0], *d1 = g.dst[1], *d2 = g.dst[2];
        asm("" : "+s"(s0), "+s"(s1), "+s"(s2), "+s"(d0), "+s"(d1), "+s"(d2));
        *from = y == 0 ? s0 : y == 1 ? s1 : s2;
        *to = y == 0 ? d0 : y == 1 ? d1 : d2;
        *chunks = y == 0 ? g.chunks[0] : y == 1 ? g.chunks[1] : g.chunks[2];
        return c - (y == 0 ? 0 : y == 1 ? g.chunks[0] : end1());
    }
    __device__ __forceinline__ void position(int32_t row, int64_t at) const {
        if (g.pos != nullptr) g.pos_out[at] = g.pos[row];
    }
};
template <class Sources>
__global__ __launch_bounds__(kFusedLanes) void select_gather_kernel(
    const float* __restrict__ parts, float* scores, const int32_t* __restrict__ seq_offsets, const int32_t* __restrict__ keep_len,
    int32_t* __restrict__ kept_idx, int32_t* __restrict__ out_offsets, Sources g, int32_t groups, int32_t total_tokens, int32_t w, int32_t split, int32_t room) {
    extern __shared__ int32_t rows[];
    __shared__ SelectShared<kFusedLanes> sh;
    const int b = (int)blockIdx.x / split, part = (int)blockIdx.x - b * split;
    ToPart sink{{kept_idx, out_offsets, b}, rows, part, split, room, 0, 0, 0};
    select_sequence<kFusedLanes, kInRegisters>(b, parts, groups, total_tokens, scores, part == 0, seq_offsets, keep_len, w, nullptr, &sh, sink);
    __syncthreads();
    // item i: the 16 bytes at i % all of row i / all, which is its row of every source, one after the other
    constexpr int kAhead = 4;
    const int n = sink.hi - sink.lo;
    const int64_t first = (int64_t)sink.base + sink.lo;
    const int32_t all = g.all();
    for (int i0 = threadIdx.x; i0 < n * all; i0 += kAhead * kFusedLanes) {
        u32x4 x[kAhead];
        u32x4* to[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = i0 + u * kFusedLanes;
            if (i >= n * all) break;
            const int j = i / all;
            const u32x4* src;
            u32x4* dst;
            int32_t chunks;
            const int32_t at = g.piece(i - j * all, &src, &dst, &chunks);
            x[u] = __builtin_nontemporal_load(src + (int64_t)rows[j] * chunks + at);
            to[u] = dst + (first + j) * chunks + at;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (i0 + u * kFusedLanes < n * all) __builtin_nontemporal_store(x[u], to[u]);
    }
    for (int j = threadIdx.x; j < n; j += kFusedLanes) g.position(rows[j], first + j);
}

template <int kT, KeySource kSource>
int launch_select_t(const float* parts, int groups, int32_t total_tokens, float* scores,
                    const int32_t* seq_offsets_dev, const int32_t* keep_len_dev, int32_t n_seqs, int32_t max_seqlen,
                    int32_t w, int32_t* kept_idx, int32_t* out_offsets_dev, hipStream_t stream) {
    size_t lds_bytes = 0;
    if (kSource == kInLds) {
        lds_bytes = (size_t)max_seqlen * sizeof(uint32_t);
        static std::atomic<uint64_t> lds_set{0};      // the limit is raised once per device, to the most the kernel ever asks for
        if (ensure_dynamic_lds((const void*)select_topk_kernel<kT, kSource>, kLdsKeys * (int)sizeof(uint32_t), &lds_set) != PYR_OK)
            return PYR_ERR_LAUNCH;
    }
    hipLaunchKernelGGL((select_topk_kernel<kT, kSource>), dim3(n_seqs), dim3(kT), lds_bytes, stream,
                       parts, (int32_t)groups, total_tokens, scores, seq_offsets_dev, keep_len_dev, w, kept_idx, out_offsets_dev);
    return check_launch();
}

}  // namespace

int launch_select(const float* parts, int groups, int32_t total_tokens, float* scores,
                  const int32_t* seq_offsets_dev, const int32_t* keep_len_dev, int32_t n_seqs, int32_t max_seqlen,
                  int32_t w, int32_t* kept_idx, int32_t* out_offsets_dev, hipStream_t stream) {
    if (n_seqs == 0) return PYR_OK;
    // Few keys: the barriers' latency counts, and eight wavefronts reach them sooner than sixteen; many: the passes over the keys do
    // (8 keys of a lane either way: 4096 tokens on 512 lanes 6.3 us, 8192 on 1024 lanes 8.2).
    const bool few = max_seqlen <= 512 * kRegKeys && (int64_t)groups * max_seqlen <= 32768;
    const auto launch = few ? launch_select_t<512, kInRegisters>
                      : max_seqlen <= 1024 * kRegKeys ? launch_select_t<1024, kInRegisters>
                      : max_seqlen <= kLdsKeys ? launch_select_t<1024, kInLds> : launch_select_t<1024, kInMemory>;
    return launch(parts, groups, total_tokens, scores, seq_offsets_dev, keep_len_dev, n_seqs, max_seqlen, w, kept_idx, out_offsets_dev, stream);
}

// Rows of partial sums that would take the selection's one workgroup longer than a launch that adds them with the whole chip (1.7 us).
// What that launch adds to an update (us; 180 of random shapes, 1 to 12 sequences): 16 rows of up to 800 tokens +1.2...+2.5, of 1000...1600
// +0.4...+0.8, 24 rows of up to 1000 +0.3...+1.1, of 1140...1410 -0.2...-0.4, of 1810...1950 -1.0, 32 rows of up to 1010 0...+0.7, of 1040...1130
// -0.5...-1.0 (beyond 32768 sums the selection goes to 1024 lanes; the line at 36864 leaves these), of 1240...1980 -0.3...-1.8, 40 rows of
// 190...710 -0.4...+0.2, 48 of up to 640 -0.2...-0.7, of 730...1240 -1.8, 64 of 100...500 -1.1...-1.8, of 540...1700 -1.4...-4.7.
// One launch where the rows to copy are so few that the selection's own workgroups are enough for them; counted as if every
// sequence kept as many as the one that keeps most, because all get the same number of workgroups.  Whole calls, two launches / one
// (us): a 64-token layer on 32 heads (1.0 MB) 17.9 / 15.3, 256 tokens on 8 heads, d = 64 (0.3 MB) 17.0 / 15.9, 16 x 183 on 8/4 heads, d = 64
// (2.9 MB) 18.6 / 17.1; of 139 calls below the line one launch takes 0.78 to 0.99 of the time.  The line was drawn where the copy with a wavefront per
// row lost (updates of 1 x 176 rows, 3.1 MB 15.2 / 15.7, of 6 x 368, 5.4 MB 14.9 / 16.1); 256 workgroups instead of 192 differed by 1 % either
// way then, 64 cost up to 10 % at the upper end.
SelectPlan plan_select(int groups, int32_t n_seqs, int32_t max_seqlen, int32_t max_kept, int64_t row_chunks) {
    constexpr int64_t kFewBytes = 3000000;
    constexpr int kFusedGroups = 192;
    SelectPlan p{};
    p.sums = groups > 1 && sums_pay(groups, max_seqlen);
    if (n_seqs > 0 && max_kept > 0 && row_chunks > 0 && max_seqlen <= kFusedLanes * kRegKeys && row_chunks <= kFewBytes / 16 &&
        row_chunks * max_kept <= kFewBytes / 16 && row_chunks * max_kept * n_seqs <= kFewBytes / 16)
        p.split = (kFusedGroups + n_seqs - 1) / n_seqs;
    return p;
}

int launch_select_gather(const float* parts, int groups, int32_t total_tokens, float* scores, const int32_t* seq_offsets_dev,
                         const int32_t* keep_len_dev, int32_t n_seqs, int32_t max_seqlen, int32_t max_kept, int64_t n_kept, int32_t w,
                         int32_t* kept_idx, int32_t* out_offsets_dev, const GatherSources& g, hipStream_t stream) {
    int64_t row_chunks = 0;
    for (int i = 0; i < g.n; ++i) row_chunks += g.chunks[i];
    const SelectPlan plan = plan_select(groups, n_seqs, max_seqlen, max_kept, row_chunks);
    if (plan.sums) {
        const int rc = launch_sum_parts(parts, groups, total_tokens, scores, stream);
        if (rc != PYR_OK) return rc;
        groups = 1;
    }
    // (offsets written over the ones that are read, which one sequence can afford where one workgroup does both: not with several)
    const auto overlap = [](const int32_t* a, int64_t n, const int32_t* b, int64_t m) { return a < b + m && b < a + n; };
    const bool in_place = overlap(out_offsets_dev, n_seqs + (int64_t)1, seq_offsets_dev, n_seqs + (int64_t)1) ||
                          overlap(out_offsets_dev, n_seqs + (int64_t)1, keep_len_dev, n_seqs);
    if (plan.split > 0 && !in_place) {
        const int32_t room = (max_kept + plan.split - 1) / plan.split;
        const auto launch = [&](auto sources) {
            hipLaunchKernelGGL((select_gather_kernel<decltype(sources)>), dim3((unsigned)(plan.split * n_seqs)), dim3(kFusedLanes), (size_t)room * sizeof(int32_t),
                               stream, parts, scores, seq_offsets_dev, keep_len_dev, kept_idx, out_offsets_dev, sources, (int32_t)groups, total_tokens, w,
                               (int32_t)plan.split, room);
            return check_launch();
        };
        if (g.n == 2 && g.chunks[0] == g.chunks[1] && g.pos == nullptr) return launch(TwoSources{{g.src[0], g.src[1]}, {g.dst[0], g.dst[1]}, g.chunks[0]});
        return launch(AnySources{g});
    }
    const int rc = launch_select(parts, groups, total_tokens, scores, seq_offsets_dev, keep_len_dev, n_seqs, max_seqlen, w, kept_idx, out_offsets_dev, stream);
    return rc != PYR_OK ? rc : launch_gather_multi(g, kept_idx, n_kept, stream);
}

}  // namespace pyr
