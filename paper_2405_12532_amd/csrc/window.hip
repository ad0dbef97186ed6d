// Launch of the one-walk scores (window_device.h): its cut, and the rule that says when it is taken.
#include <type_traits>

#include "window_device.h"

namespace pyr {
namespace {

// scores[t] = the sum of parts[0 .. groups)[t]: 64 tokens a workgroup, whose wavefronts take every kSumWaves-th row and meet in LDS.
// Bound: the latency of one trip to memory up to 64 rows, 1.7 us with its launch; the selection's one workgroup, which has room for 16 rows
// of 1024 tokens on their way at a time, took 5 us for 64 rows of 1537.
constexpr int kSumWaves = 8;
__global__ __launch_bounds__(64 * kSumWaves) void sum_parts_kernel(const float* __restrict__ parts, int32_t groups, int32_t total_tokens,
                                                                   float* __restrict__ scores) {
    __shared__ float sums[kSumWaves][64];
    constexpr int kAhead = 8;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t t = (int64_t)blockIdx.x * 64 + lane;
    float x = 0.f;
    for (int g0 = wave; g0 < groups; g0 += kSumWaves * kAhead) {
        float y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) y[u] = t < total_tokens && g0 + u * kSumWaves < groups ? parts[(size_t)(g0 + u * kSumWaves) * total_tokens + t] : 0.f;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) x += y[u];
    }
    sums[wave][lane] = x;
    __syncthreads();
    if (wave != 0 || t >= total_tokens) return;
#pragma unroll
    for (int u = 1; u < kSumWaves; ++u) x += sums[u][lane];
    scores[t] = x;
}

template <int D, int kTiles, bool kWeighted, bool kByKvHead>
__global__ __launch_bounds__(64 * kWindowWaves, 2) void window_kernel(WindowArgs a) {
    extern __shared__ __align__(1024) char smem[];
    int b, g;
    window_place(a, (int)blockIdx.x, &b, &g);
    window_scores<D, kTiles, kWeighted, kByKvHead>(a, b, g, smem);
}

int window_bytes(bool d64, int tiles, int waves) {
    const auto of = [&](auto t) { return d64 ? window_lds_bytes<64, decltype(t)::value>(waves) : window_lds_bytes<128, decltype(t)::value>(waves); };
    return tiles <= 2 ? of(std::integral_constant<int, 2>{}) : tiles <= 4 ? of(std::integral_constant<int, 4>{}) : of(std::integral_constant<int, 8>{});
}

template <int D, int kTiles, bool kWeighted, bool kByKvHead>
int launch_window_t(const WindowArgs& a, unsigned grid, int waves, hipStream_t stream) {
    static std::atomic<uint64_t> lds_set{0};
    const void* kernel = (const void*)window_kernel<D, kTiles, kWeighted, kByKvHead>;
    if (ensure_dynamic_lds(kernel, window_lds_bytes<D, kTiles>(kWindowWaves), &lds_set) != PYR_OK) return PYR_ERR_LAUNCH;
    const int lds = window_lds_bytes<D, kTiles>(waves);
    hipLaunchKernelGGL((window_kernel<D, kTiles, kWeighted, kByKvHead>), dim3(grid), dim3(64 * waves), lds, stream, a);
    return check_launch();
}

// Equal lengths, a multiple of the XCDs: a sequence's workgroups on one of them.
bool seq_per_xcd(const pyr_shape& s, bool equal, const DeviceInfo& dev) { return equal && s.n_seqs % dev.xccs == 0; }

// The order of the tasks.  Where a sequence's workgroups are not on one XCD anyway, those of a KV head come together on one, or on few, if its
// tasks are as many apart as there are KV heads, since workgroups go round robin over the XCDs; else every XCD fetches the keys of every head.  Short
// sequences gain less than the divisions by the number of KV heads take (0.2 us), and more than sixteen row blocks per KV head find the keys in L2 either way.
// Whole updates, query head after query head / by KV head (us): 1 x 1537 rows on 32 heads, w = 64 31.2 / 30.55, 4 x 1605 at most on 32/8, w = 64 37.3 / 30.5,
// 4 x 1378 on 40 heads, w = 64 58.7 / 55.3, 28 x 345 on 8 heads, w = 100 31.5 / 29.1.  Of 460 updates by KV head, geometric means of the time: 256
// tokens and more on 8, 24, 32 or 40 KV heads 0.95...0.98 (the worst 1.02), below 0.97...1.01; on 2, 4 or 12 from 768 tokens and four row blocks on
// 0.94...0.98, else 0.99...1.015; 24 row blocks per KV head and more 1.00...1.02.  With a sequence's workgroups on one XCD 64 x 2048 901 / 1055.
bool by_kv_head(const pyr_shape& s, bool equal, int32_t w, const DeviceInfo& dev) {
    const int blocks = s.n_q_heads / s.n_kv_heads * (((w < s.max_seqlen ? w : s.max_seqlen) + 31) / 32);
    const bool even = s.n_kv_heads % dev.xccs == 0;
    return !seq_per_xcd(s, equal, dev) && blocks >= (even ? 2 : 4) && blocks <= 16 && s.max_seqlen >= (even ? 256 : 768);
}

template <int D, int kTiles>
int launch_window_w(const WindowArgs& a, unsigned grid, int waves, bool by_kv, hipStream_t stream) {
    if (by_kv) return a.row_weights ? launch_window_t<D, kTiles, true, true>(a, grid, waves, stream) : launch_window_t<D, kTiles, false, true>(a, grid, waves, stream);
    return a.row_weights ? launch_window_t<D, kTiles, true, false>(a, grid, waves, stream) : launch_window_t<D, kTiles, false, false>(a, grid, waves, stream);
}

template <int D>
int launch_window_d(const WindowArgs& a, int32_t max_seqlen, unsigned grid, int waves, bool by_kv, hipStream_t stream) {
    const int tiles = (max_seqlen + 32 * waves - 1) / (32 * waves);
    return tiles <= 2 ? launch_window_w<D, 2>(a, grid, waves, by_kv, stream)
         : tiles <= 4 ? launch_window_w<D, 4>(a, grid, waves, by_kv, stream) : launch_window_w<D, 8>(a, grid, waves, by_kv, stream);
}

}  // namespace

// The cut with the lowest cost, in microseconds (selection included), joined as in plan_strip from
// - the chain: 3.1 until the first tiles are there, then a workgroup's tasks one after the other; a task takes a wavefront 1.02 per tile
//   (query rows count as one) where its latencies set the time, and 0.2 + 0.55 per tile times the wavefronts of its SIMD where they
//   wait for each other, 0.79 of that at d = 64;
// - the stream: a tile of K takes a compute unit's share of the memory system 0.236 from HBM and 0.218 from L2 to every task.
// A row of partial sums costs the selection 0.03; where they are added in a launch of their own, that costs 1.7 and 3 per million.
// Fitted to 270 calls (eleven head shapes, w = 16...256, one sequence to 160, 33...2048 tokens, equal and ragged), each timed with
// up to 50 cuts: predictions near a call's best have a standard deviation of 11 %, the cut chosen takes 2.9 % longer than the best one in
// the mean (before that launch).  Seven wavefronts are left out where there is work for eight, which were 1 to 5 % faster at every such
// choice (2 x 889 on 12 heads, d = 64 16.2 / 15.4 us a call).  One wavefront is left to sequences of one tile: more of them hide each other's latency less well than predicted.
WindowPlan plan_window(const pyr_shape& s, double tiles, int32_t w, int max_groups, const DeviceInfo& dev) {
    WindowPlan best{0, 0, 1e300};
    if (s.max_seqlen > kWindowMaxKeys) return best;
    const bool d64 = s.head_dim == 64;
    const int L = w < s.max_seqlen ? w : s.max_seqlen, max_tiles = (s.max_seqlen + 31) / 32;
    const int64_t tasks = (int64_t)s.n_q_heads * ((L + 31) / 32);
    const int fewest = (max_tiles + kWindowMaxTiles - 1) / kWindowMaxTiles, most = max_tiles < kWindowWaves ? max_tiles : kWindowWaves;
    const double size = s.head_dim / 128.0, k = d64 ? 0.79 : 1.0;
    const double flow = tiles * (0.236 * s.n_kv_heads + 0.218 * tasks) * size / dev.compute_units;
    const int limit = (int)(tasks < max_groups ? tasks : max_groups);
    for (int waves = fewest > 1 || most == 1 ? fewest : 2; waves <= most; ++waves) {
        if (waves == 7 && most == 8) continue;
        const int wave_tiles = (max_tiles + waves - 1) / waves;
        // (workgroups a compute unit holds: 8 wavefronts by registers, 12 of up to two tiles; 160 KB of LDS)
        const int by_registers = (wave_tiles <= 2 ? 12 : 8) / waves;
        const int bytes = window_bytes(d64, wave_tiles, waves);
        const int by_lds = 160 * 1024 / bytes, per_cu = by_lds < by_registers ? by_lds : by_registers;
        const double per_wave = (double)max_tiles / waves;
        const double mean_tiles = tiles == (double)s.n_seqs * max_tiles ? wave_tiles : tiles / s.n_seqs / waves + 0.5 * (1.0 - 1.0 / waves);
        for (int g = 1, last = 0; !last; g = 2 * g) {
            if (g >= limit || g >= 256) {
                last = 1;
                g = limit < 256 ? limit : 256;
            }
            const double task_rounds = (double)((tasks + g - 1) / g), wgs = (double)s.n_seqs * g, slots = (double)dev.compute_units * per_cu;
            const double there = ceil(wgs / dev.compute_units), on_simd = (there < per_cu ? there : per_cu) * waves / 4;
            const double own = on_simd > 1.0 ? on_simd : 1.0;
            const auto task = [&](double t) {
                const double alone = 1.02 * k * (t + 1), shared = (0.2 + 0.55 * k * (t < per_wave ? t + 1 : per_wave + 1)) * own;
                return alone > shared ? alone : shared;
            };
            const double longest = task_rounds * task(wave_tiles);
            double chain = 3.1 + longest;
            if (wgs > slots) {
                const double mean = task_rounds * task(mean_tiles), all = wgs * mean / slots;
                chain = 3.1 + (all > longest ? all : longest) + (wgs < 8 * slots ? 0.5 : 0.25) * mean;
            }
            const double cost = 6.0 + sqrt(sqrt(chain * chain * chain * chain + flow * flow * flow * flow)) + (sums_pay(g, s.max_seqlen) ? 1.7 + 3e-6 * g * s.total_tokens : 0.03 * (g - 1));
            if (cost <= best.cost) best = WindowPlan{waves, g, cost};
        }
    }
    return best;
}

int launch_window(const void* q, const void* k, const int32_t* seq_offsets_dev, const pyr_shape& s, bool equal, int32_t w, int32_t q_window,
                  float scale_log2, const float* row_weights, float* sums, const WindowPlan& plan, const DeviceInfo& dev, hipStream_t stream) {
    WindowArgs a{};
    a.q = (const uint16_t*)q;
    a.k = (const uint16_t*)k;
    a.seq_offsets = seq_offsets_dev;
    a.row_weights = row_weights;
    a.sums = sums;
    a.n_seqs = s.n_seqs;
    a.w = w;
    a.total_tokens = s.total_tokens;
    a.n_q_heads = s.n_q_heads;
    a.n_kv_heads = s.n_kv_heads;
    a.groups = plan.groups;
    a.xcds = seq_per_xcd(s, equal, dev) ? dev.xccs : 0;
    a.waves = plan.waves;
    a.q_window = q_window;
    a.c = scale_log2;
    const int64_t n = (int64_t)s.n_seqs * plan.groups;
    if (n >= (int64_t)1 << 31) return PYR_ERR_UNSUPPORTED;
    const bool by_kv = by_kv_head(s, equal, w, dev);
    return s.head_dim == 128 ? launch_window_d<128>(a, s.max_seqlen, (unsigned)n, plan.waves, by_kv, stream)
                             : launch_window_d<64>(a, s.max_seqlen, (unsigned)n, plan.waves, by_kv, stream);
}

int window_task_order(const pyr_shape& s, bool equal, int32_t w, const DeviceInfo& dev) { return by_kv_head(s, equal, w, dev) ? 1 : 0; }

int launch_sum_parts(const float* parts, int groups, int32_t total_tokens, float* scores, hipStream_t stream) {
    hipLaunchKernelGGL(sum_parts_kernel, dim3((unsigned)((total_tokens + (int64_t)63) / 64)), dim3(64 * kSumWaves), 0, stream, parts, (int32_t)groups,
                       total_tokens, scores);
    return check_launch();
}

}  // namespace pyr
