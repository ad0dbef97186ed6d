// A small prefill batch's attention and scores in one launch: the first workgroups take the scores by one walk over K that finds
// the row denominators itself (window_device.h), so that it need not wait for the attention's, the others an attention tile each
// (attention_tile_device.h).  When: plan_layer in score.hip.
// Bound: as its parts are, a tile's chain of steps and a window's chain of tasks.  A window's workgroup has the registers and the LDS of a tile's, so a
// compute unit takes either, and its tasks go in turn over the KV heads, so that it reads K where the tiles of that head do.
// us per layer, apart / in one launch: 1 x 256 on 8 heads, d = 64 16.2 / 12.2 (7.0 + 4.2 in the two launches), 3 x 343 on 32 heads 33.0 / 29.2.
#include <type_traits>

#include "attention_tile_device.h"
#include "window_device.h"

namespace pyr {
namespace {

template <int D, int kGroups, int kTiles, bool kWeighted>
struct WindowFront {
    static constexpr bool kAny = true;
    // As many tiles a compute unit as without it.  At d = 64 with four tiles a wavefront that holds the kernel to 168 registers, two to four of which
    // wait in scratch memory: 30 such layers take 7 % longer (0.93 to 1.16) with two workgroups a compute unit and none there.  (d = 128, eight
    // tiles a wavefront: one to four with 256 registers.  Their accesses make the counted waits for a walk's tiles stricter, never shorter.)
    static constexpr int kWaves = D == 64 && kGroups == 1 && kTiles < 8 ? 3 : 2;
    const float* row_weights;
    float* sums;                                      // [groups, total_tokens]
    int32_t w, total_tokens, groups;
    int32_t workgroups, grid_x, grid_y;               // ... and the grid of the tiles behind them
    __device__ __forceinline__ void run(const TileArgs& t, int id, char* smem) const {
        const WindowArgs a{t.q, t.k, t.seq_offsets, row_weights, sums, t.n_seqs, t.n_q_heads, t.n_kv_heads, w, total_tokens, 4 * kGroups, groups, 0, 0, t.c};
        const int b = id / groups;
        if (b < t.n_seqs) window_scores<D, kTiles, kWeighted, true>(a, b, id - b * groups, smem);
    }
};

struct Windows {
    const float* row_weights;
    float* sums;
    int32_t w, total_tokens, groups, workgroups;
};

template <int D, int kGroups, int kTiles, bool kWeighted>
int launch_layer_t(const TileArgs& t, const Windows& w, dim3 grid, hipStream_t stream) {
    using Front = WindowFront<D, kGroups, kTiles, kWeighted>;
    static_assert(sizeof(TileArgs) + sizeof(Front) <= 112, "short arguments");
    constexpr int tile = TileLds<D, kGroups>::kBytes, window = window_lds_bytes<D, kTiles>(4 * kGroups), lds = tile > window ? tile : window;
    static std::atomic<uint64_t> lds_set{0};
    if (ensure_dynamic_lds((const void*)attention_tile_kernel<D, kGroups, Front>, lds, &lds_set) != PYR_OK) return PYR_ERR_LAUNCH;
    hipLaunchKernelGGL((attention_tile_kernel<D, kGroups, Front>), dim3((unsigned)w.workgroups + grid.x * grid.y * grid.z), dim3(kGroups * 256), lds, stream, t,
                       Front{w.row_weights, w.sums, w.w, w.total_tokens, w.groups, w.workgroups, (int32_t)grid.x, (int32_t)grid.y});
    return check_launch();
}

template <int D, int kGroups>
int launch_layer_d(const TileArgs& t, const Windows& w, int32_t max_seqlen, dim3 grid, hipStream_t stream) {
    const auto tiles = [&](auto n) {
        constexpr int kTiles = decltype(n)::value;
        return w.row_weights ? launch_layer_t<D, kGroups, kTiles, true>(t, w, grid, stream)
                             : launch_layer_t<D, kGroups, kTiles, false>(t, w, grid, stream);
    };
    const int per_wave = (max_seqlen + 128 * kGroups - 1) / (128 * kGroups);
    return per_wave <= 2 ? tiles(std::integral_constant<int, 2>{}) : per_wave <= 4 ? tiles(std::integral_constant<int, 4>{}) : tiles(std::integral_constant<int, 8>{});
}

}  // namespace

int launch_layer(const AttentionChoice& choice, int groups, const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev,
                 const int32_t* seq_offsets_host, const pyr_shape& s, int32_t uniform_len, int32_t w, float scale_log2,
                 const float* row_weights, void* out, float* sums, hipStream_t stream) {
    DeviceInfo dev;
    if (device_info(&dev) != PYR_OK) return PYR_ERR_LAUNCH;
    TileArgs t;
    const int rc = tile_args(q, k, v, seq_offsets_dev, seq_offsets_host, s, uniform_len, scale_log2, out, dev, &t);
    if (rc != PYR_OK) return rc;
    const dim3 grid = tile_grid(s, seq_offsets_host, uniform_len, choice.kernel, dev, &t);
    const int workgroups = (s.n_seqs * groups + dev.xccs - 1) / dev.xccs * dev.xccs;      // (the tiles keep their XCDs)
    const Windows a{row_weights, sums, w, s.total_tokens, groups, workgroups};
    if (s.head_dim == 128)
        return choice.kernel == 2 ? launch_layer_d<128, 2>(t, a, s.max_seqlen, grid, stream) : launch_layer_d<128, 1>(t, a, s.max_seqlen, grid, stream);
    return choice.kernel == 2 ? launch_layer_d<64, 2>(t, a, s.max_seqlen, grid, stream) : launch_layer_d<64, 1>(t, a, s.max_seqlen, grid, stream);
}

}  // namespace pyr
