// Launch of the segmented top-k (Algorithm 1, TopP(A_e, p); see select_device.h): one workgroup per sequence.
#include "select_device.h"

namespace pyr {
namespace {

constexpr int kLdsKeys = 36864;            // 144 KiB of the 160 KiB LDS of a gfx950 compute unit

template <int kT, KeySource kSource>
__global__ __launch_bounds__(kT) void select_topk_kernel(
    const float* __restrict__ parts, int32_t groups, int32_t total_tokens, float* scores,
    const int32_t* __restrict__ seq_offsets, const int32_t* __restrict__ keep_len, int32_t w,
    int32_t* __restrict__ kept_idx, int32_t* __restrict__ out_offsets) {
    extern __shared__ uint32_t lds_keys[];
    __shared__ SelectShared<kT> sh;
    select_sequence<kT, kSource>(blockIdx.x, parts, groups, total_tokens, scores, seq_offsets, keep_len, w, lds_keys, &sh, kept_idx, out_offsets);
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

}  // namespace pyr
