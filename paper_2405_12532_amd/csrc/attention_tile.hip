// Launch of the 128-row attention tiles (attention_tile_device.h): the grid, its order, the list of a very ragged batch.
#include "attention_tile_device.h"

namespace pyr {
namespace {

// prefix sums of the number of query tiles per sequence
__global__ __launch_bounds__(1024) void tile_map_kernel(const int32_t* __restrict__ seq_offsets, int32_t n_seqs,
                                                        int32_t* __restrict__ tile_map) {
    __shared__ int part[1024];
    const int tid = threadIdx.x;
    const int chunk = (n_seqs + 1023) / 1024;
    const int lo = min(tid * chunk, n_seqs), hi = min(lo + chunk, n_seqs);
    int sum = 0;
    for (int b = lo; b < hi; ++b) sum += (seq_offsets[b + 1] - seq_offsets[b] + kTileRows - 1) / kTileRows;
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int add = tid >= d ? part[tid - d] : 0;
        __syncthreads();
        part[tid] += add;
        __syncthreads();
    }
    int run = part[tid] - sum;
    for (int b = lo; b < hi; ++b) {
        tile_map[b] = run;
        run += (seq_offsets[b + 1] - seq_offsets[b] + kTileRows - 1) / kTileRows;
    }
    if (tid == 1023) tile_map[n_seqs] = part[1023];
}

template <int D, int kGroups>
int launch_tile(const TileArgs& a, const NoFront& rest, dim3 grid, hipStream_t stream) {
    using T = TileLds<D, kGroups>;
    static_assert(sizeof(TileArgs) + sizeof(NoFront) <= 112, "short arguments");
    static std::atomic<uint64_t> lds_set{0};
    if (ensure_dynamic_lds((const void*)attention_tile_kernel<D, kGroups, NoFront>, T::kBytes, &lds_set) != PYR_OK) return PYR_ERR_LAUNCH;
    hipLaunchKernelGGL((attention_tile_kernel<D, kGroups, NoFront>), grid, dim3(kGroups * 256), T::kBytes, stream, a, rest);
    return check_launch();
}

// The work of the XCD that has most of it, relative to an equal share, if unit u goes to XCD u % xcds.  Where that is far from one
// (few KV heads and few sequences, or one sequence far longer than the others) units are not bound to XCDs: each L2 then
// fetches the K/V rows itself. Measured, bound / not (us): 32768 and 255 x 64 tokens on 16/2 heads 15600 / 3930,
// d = 64: the same on 12/12 heads 2230 / 1680.
double xcd_share(const pyr_shape& s, const int32_t* off, int32_t uniform_len, int xcds) {
    const int odd = s.n_kv_heads % xcds;
    if (odd == 0) return 1.0;
    if (uniform_len > 0) {
        const int64_t units = (int64_t)s.n_seqs * s.n_kv_heads;
        return (double)((units + xcds - 1) / xcds * xcds) / units;
    }
    constexpr int kMaxXcds = 64;
    if (xcds > kMaxXcds) return xcds;
    double extra[kMaxXcds] = {}, even = 0, all = 0;
    for (int32_t b = 0, at = 0; b < s.n_seqs; ++b, at = (at + odd) % xcds) {
        const double len = off[b + 1] - off[b], work = len * (len + 512);      // (a tile costs what four steps do, besides its own)
        even += work * (s.n_kv_heads / xcds);
        all += work * s.n_kv_heads;
        for (int i = 0; i < odd; ++i) extra[(at + i) % xcds] += work;
    }
    double most = 0;
    for (int i = 0; i < xcds; ++i) most = extra[i] > most ? extra[i] : most;
    return all > 0 ? (even + most) * xcds / all : 1.0;
}

int64_t count_tiles(const pyr_shape& s, const int32_t* seq_offsets_host) {
    int64_t tiles = 0;
    for (int32_t b = 0; b < s.n_seqs; ++b) tiles += (seq_offsets_host[b + 1] - seq_offsets_host[b] + kTileRows - 1) / kTileRows;
    return tiles;
}

constexpr int kMaxGrid = 65535;              // of y and z

int bound_xcds(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len, const DeviceInfo& dev) {
    return xcd_share(s, seq_offsets_host, uniform_len, dev.xccs) <= 1.15 ? dev.xccs : 1;
}

// A chunk: the units one XCD works on at a time, long tiles first.  Half the workgroups an XCD holds, in units that come in
// fours (rows a power of two apart) or, in a ragged batch, in whole sequences' worth of heads, which are equally long: the
// tiles that run together then share their K/V rows in L2 (us, two rounds of workgroups to a chunk / now: 64 x 359
// 190 / 173, 64 x 269 154 / 136, 64 x 512 282 / 258; d = 64: 64 x 500 153 / 147).  All units where they are few and the
// grid is at most eight rounds: what counts there is that nothing long starts late (3 x 5000 tokens, 24 heads,
// nine units per XCD: 533 in chunks of four, 459 in one).  At d = 64 ragged batches, whose
// chunks end unevenly, go in one up to 2/5 of the slots (38 units an XCD, 16 for equal sequences), and where the longest sequence has at most
// 9/8 of the mean's tiles up to 3/10 (28).  Over 300 batches of 6 to 38 units (eleven head shapes, 130 to 6000 tokens at most, the shortest 0.1
// to 1 of that), chunks / one (us): 17 x 609...3417 on 8 heads 127 / 101, 19 x 144...720 on 12 22.7 / 16.6, 12 x 1486...1500 on 12 67 / 55.
// Nearly equal with more than 28 units: 24 x 326...330 on 12 15.0 / 15.7, 33 x 264...330 on 8 13.2 / 14.0, 34 x 267...276 on 8 12.7 / 13.8, of
// 60 such batches 0.90 to 1.08.  All others take 0.73 to 1.06 of the time in one, 0.92 in the middle (the worst, 32 x 221...542 on 2 heads 9.9 / 10.4).
// At d = 128, twenty batches took 0.88 to 1.07.
struct Chunks {
    int units, count, per_xcd;          // units of a chunk, chunks, units of an XCD
};

Chunks cut_chunks(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len, int groups, int xcds, const DeviceInfo& dev) {
    const int64_t unit_tiles = (int64_t)((s.max_seqlen + kTileRows - 1) / kTileRows) * (s.n_q_heads / s.n_kv_heads);
    const int slots = dev.compute_units / xcds * (groups == 2 ? 1 : s.head_dim == 128 ? 2 : 3);
    const int units_per_xcd = (int)(((int64_t)s.n_seqs * s.n_kv_heads + xcds - 1) / xcds);
    const int target = (int)((slots + unit_tiles) / (2 * unit_tiles));                   // (rounded)
    int chunk = target < 6 ? 4 : (target + 2) / 4 * 4;
    int few = slots / 6;
    if (uniform_len == 0) {
        const int per_seq = s.n_kv_heads % xcds == 0 ? s.n_kv_heads / xcds : 1;
        chunk = per_seq * (target < 2 * per_seq ? 1 : (target + per_seq / 2) / per_seq);
        if (s.head_dim == 64) {
            const int most = 2 * slots / 5, nearly_equal = 3 * slots / 10;
            const int64_t places = (int64_t)s.n_seqs * ((s.max_seqlen + kTileRows - 1) / kTileRows);
            few = units_per_xcd > nearly_equal && units_per_xcd <= most && 8 * places <= 9 * count_tiles(s, seq_offsets_host) ? nearly_equal : most;
        }
    }
    if (units_per_xcd <= few && units_per_xcd * unit_tiles <= 8 * (int64_t)slots) chunk = units_per_xcd;
    if (chunk > units_per_xcd) chunk = units_per_xcd;
    if (chunk < (units_per_xcd + kMaxGrid - 1) / kMaxGrid) chunk = (units_per_xcd + kMaxGrid - 1) / kMaxGrid;
    const int chunks = (units_per_xcd + chunk - 1) / chunk;
    return Chunks{(units_per_xcd + chunks - 1) / chunks, chunks, units_per_xcd};          // (equal chunks)
}

}  // namespace

// A list of the tiles that exist, where the grid would mostly hold workgroups that find no rows.  One of those costs about 0.8 ns;
// finding its place in the list costs a tile about 1.2 us, 2.3 ns of the whole device, and the list is a launch of its own, 4.5 us.
// Measured, grid / list (us): 32768 and 255 x 64 tokens 10310 / 8280, 4096 and 2000 x 16 2400 / 721, d = 64: 8192 and
// 500 x 100 on 12 heads 530 / 180; but 32 sequences of 512...4096 on 32/8 heads 1946 / 2000.
bool attention_tile_listed(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len) {
    if (uniform_len > 0) return false;
    const int tiles = (s.max_seqlen + kTileRows - 1) / kTileRows;
    return ((int64_t)s.n_seqs * tiles - 4 * count_tiles(s, seq_offsets_host)) * s.n_q_heads > 6000;
}

int64_t attention_tiles(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len) {
    return uniform_len > 0 ? (int64_t)s.n_seqs * ((uniform_len + kTileRows - 1) / kTileRows) : count_tiles(s, seq_offsets_host);
}

void attention_tile_route(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len, int groups, const DeviceInfo& dev, pyr_launches* out) {
    if (attention_tile_listed(s, seq_offsets_host, uniform_len)) return;
    const Chunks cut = cut_chunks(s, seq_offsets_host, uniform_len, groups, bound_xcds(s, seq_offsets_host, uniform_len, dev), dev);
    out->attention_chunk = cut.units;
    out->attention_units = cut.per_xcd;
}

int tile_args(const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
              const pyr_shape& s, int32_t uniform_len, float scale_log2, void* out, const DeviceInfo& dev, TileArgs* args) {
    TileArgs a{};
    a.q = (const uint16_t*)q;
    a.k = (const uint16_t*)k;
    a.v = (const uint16_t*)v;
    a.seq_offsets = seq_offsets_dev;
    if ((int64_t)s.n_seqs * s.n_kv_heads >= (int64_t)1 << 31) return PYR_ERR_UNSUPPORTED;
    a.n_seqs = s.n_seqs;
    a.n_q_heads = s.n_q_heads;
    a.n_kv_heads = s.n_kv_heads;
    a.xcds = bound_xcds(s, seq_offsets_host, uniform_len, dev);
    a.uniform_len = uniform_len;
    a.c = scale_log2;
    a.lowest = lowest_reference(scale_log2);
    a.out = (uint16_t*)out;
    *args = a;
    return PYR_OK;
}

dim3 tile_grid(const pyr_shape& s, const int32_t* seq_offsets_host, int32_t uniform_len, int groups, const DeviceInfo& dev, TileArgs* a) {
    const Chunks cut = cut_chunks(s, seq_offsets_host, uniform_len, groups, a->xcds, dev);
    a->units_per_chunk = cut.units;
    return dim3((unsigned)(a->xcds * cut.units * (s.n_q_heads / s.n_kv_heads)), (unsigned)((s.max_seqlen + kTileRows - 1) / kTileRows), (unsigned)cut.count);
}

int launch_attention_tile(const void* q, const void* k, const void* v, const int32_t* seq_offsets_dev, const int32_t* seq_offsets_host,
                          const pyr_shape& s, int32_t uniform_len, float scale_log2, void* out, float* lse, int32_t* tile_map,
                          int groups, hipStream_t stream) {
    if (s.n_seqs == 0 || s.max_seqlen == 0) return PYR_OK;
    DeviceInfo dev;
    if (device_info(&dev) != PYR_OK) return PYR_ERR_LAUNCH;
    TileArgs a;
    int rc = tile_args(q, k, v, seq_offsets_dev, seq_offsets_host, s, uniform_len, scale_log2, out, dev, &a);
    if (rc != PYR_OK) return rc;
    const int tiles = (s.max_seqlen + kTileRows - 1) / kTileRows, head_group = s.n_q_heads / s.n_kv_heads;
    NoFront rest{nullptr, lse, 0, 0};
    const auto launch = [&](dim3 grid) {
        rest.tiles = (int32_t)grid.y;
        if (s.head_dim == 128) return groups == 2 ? launch_tile<128, 2>(a, rest, grid, stream) : launch_tile<128, 1>(a, rest, grid, stream);
        return groups == 2 ? launch_tile<64, 2>(a, rest, grid, stream) : launch_tile<64, 1>(a, rest, grid, stream);
    };
    // (sequence after sequence with the last tile first, the order a chunk of one sequence has)
    if (attention_tile_listed(s, seq_offsets_host, uniform_len)) {
        const int64_t listed = count_tiles(s, seq_offsets_host);
        hipLaunchKernelGGL(tile_map_kernel, dim3(1), dim3(1024), 0, stream, seq_offsets_dev, s.n_seqs, tile_map);
        rc = check_launch();
        rest.tile_map = tile_map;
        const int64_t x = (int64_t)(s.n_kv_heads + a.xcds - 1) / a.xcds * head_group * a.xcds;
        if (x * 256 * groups >= (int64_t)1 << 32) return PYR_ERR_UNSUPPORTED;
        for (int64_t first = 0; rc == PYR_OK && first < listed; first += kMaxGrid) {
            rest.first_tile = (int32_t)first;
            rc = launch(dim3((unsigned)x, (unsigned)(listed - first < kMaxGrid ? listed - first : kMaxGrid)));
        }
        return rc;
    }
    dim3 grid = tile_grid(s, seq_offsets_host, uniform_len, groups, dev, &a);
    for (int left = tiles; left > 0; left -= kMaxGrid) {         // (one launch below 8 million tokens a sequence)
        const int n = left < kMaxGrid ? left : kMaxGrid;
        rest.first_tile = left - n;
        grid.y = (unsigned)n;
        rc = launch(grid);
        if (rc != PYR_OK) return rc;
    }
    return PYR_OK;
}

}  // namespace pyr
