// Greedy channel selection of Sec. 3.4 on the channel maxima.
//
// The paper splits one channel at a time, always the one that currently holds the largest
// magnitude in the layer.  Halving a channel halves its maximum exactly and its copy has the
// same maximum, so the whole sequence of choices depends only on the C channel maxima: the
// tensor itself is never re-scanned.  One workgroup keeps the (growing) list of maxima in
// LDS and performs the splits in rounds (select_lds.h).
#include <atomic>

#include "ocs_internal.h"
#include "select_lds.h"

namespace ocs {

// What bounds it: the latency of one workgroup's passes over LDS, its barriers and one trip to memory.
// 3000 channels, 150 splits, the column maxima outside the caches: 78 us with one split per step (0.2 us a step on one wave, 0.5 us
// on four), 14 in rounds, 11.7 with a round's list in registers; 1075 channels, 52 splits: the whole weight path 33 -> 14 us; a few splits of up to 1024 channels are
// taken step by step (select_lds.h).  NT: sixteen waves where the list or its column maxima give every lane something to do.  HELD: pieces of NT
// entries that the list is at most, as few as hold it: every one more is code to fetch.
template <int NT, bool FEW, bool BLOCKS, int HELD>
__global__ __launch_bounds__(NT) void select_kernel(
    const float* __restrict__ colmax, int C, int g, int s, int mode,
    const int32_t* split_in, int32_t* split_src,
    int32_t* __restrict__ chan_src, int32_t* __restrict__ chan_depth, float* __restrict__ max_out,
    float clip_ratio, float qmax, float* __restrict__ scale_out, int blocks) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int E = C + s;
    unsigned long long* cand = reinterpret_cast<unsigned long long*>(smem);
    float* vals = reinterpret_cast<float*>(cand + E);
    unsigned short* src = reinterpret_cast<unsigned short*>(vals + E);
    unsigned short* dep = src + E;
    __shared__ GreedyScratch sc;
    const int tid = threadIdx.x;

    channel_maxima_to_lds<NT, BLOCKS>(colmax, blocks, C, g, vals, src, dep);

    if (mode == 0) {
        greedy_select<NT, FEW, HELD>(vals, src, dep, cand, sc, C, s, split_src);
    } else {
        if (tid == 0) {
            for (int i = 0; i < s; ++i) {
                const int cur = C + i;
                int j = split_in[i];
                j = j < 0 ? 0 : (j >= cur ? cur - 1 : j);
                unsigned short d = (unsigned short)(dep[j] + 1);
                dep[j] = d;
                vals[cur] = vals[j];  // copies are not halved: the maximum stays
                src[cur] = src[j];
                dep[cur] = d;
            }
        }
        __syncthreads();
    }

    unsigned m = 0;   // bit pattern of the largest entry (all entries are non-negative)
    for (int j = tid; j < E; j += NT) {
        chan_src[j] = src[j];
        chan_depth[j] = dep[j];
        const unsigned u = __float_as_uint(vals[j]);
        m = u > m ? u : m;
    }
    m = group_umax<NT>(m, sc.red);
    if (tid == 0) {
        const float mx = __uint_as_float(m);
        if (max_out) *max_out = mx;
        if (scale_out) {
            float T = clip_ratio * mx;
            scale_out[0] = T;
            scale_out[1] = T / qmax;
        }
    }
}

constexpr unsigned kSelectMaxLds = 128 * 1024;   // holds the list of kMaxExpanded channels

template <int NT, bool FEW, bool BLOCKS, int HELD>
static hipError_t run_select(const float* colmax, int blocks, int C, int g, int s, int mode, const int32_t* split_in,
                             int32_t* split_src, int32_t* chan_src, int32_t* chan_depth, float* max_out,
                             float clip_ratio, float qmax, float* scale_out, hipStream_t stream) {
    const unsigned lds = greedy_list_bytes(C + s);
    if (lds > kSelectMaxLds) return hipErrorInvalidValue;
    if (lds > 60 * 1024) {
        // more than 64 KB of LDS has to be opted into, once per kernel and device
        static std::atomic<bool> opted_in[64];
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        if (!opted_in[dev].load(std::memory_order_acquire)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel<NT, FEW, BLOCKS, HELD>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSelectMaxLds);
            if (e != hipSuccess) return e;
            opted_in[dev].store(true, std::memory_order_release);
        }
    }
    select_kernel<NT, FEW, BLOCKS, HELD><<<1, NT, lds, stream>>>(colmax, C, g, s, mode, split_in, split_src, chan_src, chan_depth,
                                              max_out, clip_ratio, qmax, scale_out, blocks);
    return hipGetLastError();
}

hipError_t launch_select(const float* colmax, int blocks, int C, int g, int s, int mode,
                         const int32_t* split_in, int32_t* split_src, int32_t* chan_src,
                         int32_t* chan_depth, float* max_out, float clip_ratio, float qmax,
                         float* scale_out, hipStream_t stream) {
    // E = C + s <= kMaxExpanded is checked by the caller
    const bool few = mode == 0 && few_steps(C, s);
    const bool narrow = C + s <= 512 && (int64_t)C * g <= 1024 && (int64_t)blocks * C * g <= 8192;
    static_assert(kMaxExpanded <= 8 * 1024, "pieces of the longest list");
    auto instance = [&](auto blk) {
        constexpr bool BLOCKS = decltype(blk)::value;
        if (narrow) return few ? run_select<256, true, BLOCKS, 2> : run_select<256, false, BLOCKS, 2>;
        if (few) return run_select<1024, true, BLOCKS, 2>;
        if (C + s <= 2048) return run_select<1024, false, BLOCKS, 2>;
        return C + s <= 4096 ? run_select<1024, false, BLOCKS, 4> : run_select<1024, false, BLOCKS, 8>;
    };
    const auto run = blocks > 1 ? instance(std::true_type()) : instance(std::false_type());
    return run(colmax, blocks, C, g, s, mode, split_in, split_src, chan_src, chan_depth, max_out, clip_ratio, qmax, scale_out,
               stream);
}

}  // namespace ocs
