// Worker step on the GPU: forward and backward pass of the paper's CNN (model endnote) for n
// workers x B images in one batch of launches.  Worker w reads the weights of ring slot
// meta[w].slot in place (a stale snapshot costs no copy) and its gradient is written straight into
// queue entry meta[w].q (Section 3.3 worker step: read weights, compute gradient, append).
// This file holds the launch order, the final fixed-order reduction of partial sums, and the debug
// mask kernel; the layers live in ps_conv1.hip, ps_conv2.hip, ps_fc1.hip and ps_fc2.hip.
#include "ps_common.h"
#include "ps_philox.h"

namespace ps {

namespace {

// Sums the partial slots in fixed order into the worker's queue entry: conv1 tensors have one partial
// per image (of conv2's input-gradient kernel), conv2 tensors one per block of its weight-gradient kernel, fc2
// tensors, fc1 bias and the loss one per block of the fc2 kernel.  Nothing but memory latency at few workers:
// the up to 16 slots of a conv2 or fc2 value are loaded together by one thread; the 160 conv1 values have a slot
// per image and get C1_LANES threads each (thread j adds slots j, j + 8, ..., 16 at a time, and the 8 sums
// are added in order), 32 values to each of the first 5 blocks of a worker.  How many blocks a worker
// gets does not change any sum.
constexpr int REDUCE_SLOTS = 16, C1_LANES = 8, C1_VALUES = 32, C1_BLOCKS = OFF_W2 / C1_VALUES;
static_assert(C1_VALUES * C1_BLOCKS == OFF_W2 && C1_VALUES * C1_LANES == 256, "conv1 values over the first blocks");
constexpr int REDUCE_ITEMS = CONV2_PART + FC2_PART_LOSS + 1;  // conv2 values, then fc2's

// p[0] + p[step] + ... in order, `count` values; of each REDUCE_SLOTS the sum first, which keeps the sums over a slot
// per image as close to 64 bits as the others (batches of 4096: conv1's gradient off by 1.2e-7 in one chain, 0.56e-7 so)
__device__ __forceinline__ float ordered_sum(const float* __restrict__ p, size_t step, int count)
{
    float sum = 0.f;
    for (int c0 = 0; c0 < count; c0 += REDUCE_SLOTS) {
        float v[REDUCE_SLOTS];
#pragma unroll
        for (int c = 0; c < REDUCE_SLOTS; ++c) v[c] = p[(size_t)min(c0 + c, count - 1) * step];
        float part = v[0];
#pragma unroll
        for (int c = 1; c < REDUCE_SLOTS; ++c)
            if (c0 + c < count) part += v[c];
        sum += part;
    }
    return sum;
}

__global__ __launch_bounds__(256) void grad_reduce_kernel(WorkerBuffers wb, int fc2_slots, int c1_slots, int c2_slots)
{
    __shared__ float c1_sum[C1_LANES][C1_VALUES];
    const int w = blockIdx.x;
    float* grad = worker_grad(wb, w);
    if (blockIdx.y < C1_BLOCKS) {
        const int e = threadIdx.x % C1_VALUES, j = threadIdx.x / C1_VALUES, v = blockIdx.y * C1_VALUES + e;
        c1_sum[j][e] = ordered_sum(wb.part1 + ((size_t)w * c1_slots + j) * OFF_W2 + v, C1_LANES * OFF_W2, (c1_slots - j + C1_LANES - 1) / C1_LANES);
        __syncthreads();
        if (j == 0) {
            float sum = 0.f;
#pragma unroll
            for (int k = 0; k < C1_LANES; ++k) sum += c1_sum[k][e];
            grad[v] = sum;
        }
    }
    const float* part = wb.part + (size_t)w * c2_slots * CONV2_PART;
    const float* fpart = wb.fpart + (size_t)w * fc2_slots * FC2_PART;
    for (int i = blockIdx.y * 256 + threadIdx.x; i < REDUCE_ITEMS; i += gridDim.y * 256) {
        if (i < CONV2_PART) {
            const float sum = ordered_sum(part + i, CONV2_PART, c2_slots);
            // register r = i / 64 of lane i % 64 of that kernel: tile row mt = r / 36, tap r % 36 / 4
            const int r = i / 64, o = 16 * (r / 36) + 4 * (i % 64 / 16) + r % 4;
            grad[i < CONV2_PART_B2 ? OFF_W2 + (o * C1 + i % 16) * 9 + r % 36 / 4 : OFF_B2 + i - CONV2_PART_B2] = sum;
        } else {
            const int f = i - CONV2_PART;
            const float sum = ordered_sum(fpart + f, FC2_PART, fc2_slots);
            if (f < FC2_PART_B4)
                grad[OFF_W4 + f] = sum;
            else if (f < FC2_PART_B3)
                grad[OFF_B4 + f - FC2_PART_B4] = sum;
            else if (f < FC2_PART_LOSS)
                grad[OFF_B3 + f - FC2_PART_B3] = sum;
            else if (wb.loss)
                wb.loss[w] = sum / (float)wb.B;
        }
    }
}

__global__ __launch_bounds__(256) void keep_mask_kernel(uint8_t* keep, int B, uint32_t mb_lo, uint32_t mb_hi,
                                                        uint32_t seed_lo, uint32_t seed_hi, uint32_t threshold)
{
    const int i = blockIdx.x * 256 + threadIdx.x;  // one Philox call = 4 units
    if (i >= B * (FC1 / 4)) return;
    const int s = i / (FC1 / 4), u4 = i % (FC1 / 4);
    const uint4 r = philox4x32_10(make_uint4(mb_lo, mb_hi, (uint32_t)s, (uint32_t)u4), make_uint2(seed_lo, seed_hi));
    uint8_t* k = keep + (size_t)s * FC1 + u4 * 4;
    k[0] = r.x >= threshold;
    k[1] = r.y >= threshold;
    k[2] = r.z >= threshold;
    k[3] = r.w >= threshold;
}

}  // namespace

// Wavefronts take as many images (up to `most_images`) as leave two wavefronts for every SIMD: each reads and splits a
// filter bank (conv2) or reads its weights (conv1) once per launch.  Where there is not
// one for every SIMD, as many (a power of two up to `most_wavefronts`) share an image as still find SIMDs to run on, one
// each; the kernels count on those having that image alone.
// A launch of nothing else (`alone`) lasts as long as the compute unit with the most blocks: it takes fewer images at a time
// where that makes its share smaller.  100 workers of 128 images: conv1 70 -> 60 us, conv2's forward pass 142 -> 128
// (eight images: 400 blocks, two on some compute units; one: 3200, thirteen at most); 200 of 30 37 -> 33 and 74 -> 70.  What
// a wavefront of conv2's forward pass does once is a sixteenth of an image's time (64 of 128, four, two and one image: 79.6,
// 80.8, 83.3 us), and no more in conv1, for which the same figure serves.
ImageSplit split_images(const WorkerBuffers& wb, int most_images, int most_wavefronts, int wavefronts_per_block, bool alone)
{
    ImageSplit sp{most_images, 1, 0};
    while (sp.wavefronts < most_wavefronts && 2 * sp.wavefronts * wb.n * wb.B <= 4 * wb.compute_units) sp.wavefronts *= 2;
    while (sp.images > 1 && (sp.wavefronts > 1 || wb.n * ((wb.B + sp.images - 1) / sp.images) < 2 * 4 * wb.compute_units)) sp.images /= 2;
    auto blocks = [&](int images) { return ((wb.B + images - 1) / images * sp.wavefronts + wavefronts_per_block - 1) / wavefronts_per_block; };
    auto longest = [&](int images) { return (int64_t)((wb.n * blocks(images) + wb.compute_units - 1) / wb.compute_units) * (16 * images + 1); };
    if (alone)
        for (int images = sp.images / 2; images > 0; images /= 2)
            if (longest(images) < longest(sp.images)) sp.images = images;
    sp.blocks = blocks(sp.images);
    return sp;
}

#define PS_TIMED(id, ...)      \
    do {                       \
        prof.begin(id, s);     \
        __VA_ARGS__;           \
        prof.end(s);           \
    } while (0)

hipError_t launch_worker_forward(const WorkerBuffers& wb, hipStream_t s, Profiler& prof)
{
    if (wb.n * wb.B <= 0) return hipSuccess;
    PS_TIMED(K_CONV1_FWD, launch_conv1_fwd(wb, s));
    PS_TIMED(K_CONV2_FWD, launch_conv2_fwd(wb, s));
    PS_TIMED(K_FC1_FWD, launch_fc1_fwd(wb, s));
    return hipGetLastError();
}

hipError_t launch_worker_backward(const WorkerBuffers& wb, hipStream_t s, Profiler& prof)
{
    if (wb.n * wb.B <= 0) return hipSuccess;
    PS_TIMED(K_FC2, launch_fc2(wb, s));
    if (!fc1_dw_in_backward(wb)) PS_TIMED(K_FC1_DW, launch_fc1_dw(wb, s));
    PS_TIMED(K_FC1_DX, launch_fc1_dx(wb, s));
    PS_TIMED(fc1_dw_in_backward(wb) ? K_BACKWARD_FC1 : K_BACKWARD, launch_backward(wb, s));
    // one value per thread while the chip has room, at least the blocks that the conv1 values take
    const int reduce_y = wb.n * (REDUCE_ITEMS / 256 + 1) <= 8 * wb.compute_units ? REDUCE_ITEMS / 256 + 1 : 8;
    PS_TIMED(K_GRAD_REDUCE, hipLaunchKernelGGL(grad_reduce_kernel, dim3(wb.n, reduce_y), dim3(256), 0, s, wb, fc2_split(wb.n),
                                                conv1_part_slots(wb.B), conv2_part_slots(wb.B)));
    return hipGetLastError();
}

const char* kernel_name(int id)
{
    static const char* const names[K_COUNT] = {
        "conv1_fwd_kernel", "conv2_fwd_kernel", "gemm_split<Fc1FwdEpi>", "fc2_kernel", "gemm_split<Fc1DwEpi>", "gemm_split<Fc1DxEpi>",
        "backward_kernel", "backward_kernel<fc1>", "grad_reduce_kernel", "apply_kernel<0>", "apply_kernel<1>", "grad_sqnorm_kernel",
        "apply_kernel<0, clip>", "apply_kernel<1, clip>", "apply_adadelta_kernel", "local_step_kernel",
        "elastic_average_kernel"};
    return id >= 0 && id < K_COUNT ? names[id] : "";
}

hipError_t launch_keep_mask(uint8_t* keep_dev, int B, uint32_t mb_lo, uint32_t mb_hi, uint32_t seed_lo,
                            uint32_t seed_hi, uint32_t threshold, hipStream_t s)
{
    hipLaunchKernelGGL(keep_mask_kernel, dim3((B * (FC1 / 4) + 255) / 256), dim3(256), 0, s, keep_dev, B, mb_lo, mb_hi,
                       seed_lo, seed_hi, threshold);
    return hipGetLastError();
}

}  // namespace ps
