// conv1 (1 -> 16 channels, 3x3, pad 1, on the 28x28 input) forward with fused ReLU + 2x2 max pool.
// K = 9 is too short for the matrix cores; it runs on the vector ALU with the zero-padded image in
// LDS.  (Its weight gradient is fused into conv2's input-gradient kernel.)
#include "ps_common.h"
#include "ps_split.h"

namespace ps {

namespace {

// Bound by vector-ALU issue: 36 of the about 50 instructions per (pooled position, channel) are FMAs.  A
// wavefront works on whole images by itself (no block barrier); lane (p, j) = (lane / 4, lane % 4) computes
// channels 4j .. 4j + 3 of positions p, p + 16, ..., 13 passes of which the last has 16 lanes: the 40 weights
// of its channels stay in registers, the 4x4 input patch is read for four channels at once, and what a
// wavefront stores in a pass is one contiguous KB of pool1 ([position][channel], as conv2 reads it).  In launches
// that would leave SIMDs idle, `parts` wavefronts share an image, each with every parts-th pass.
// 65,536 images: 0.313 -> 0.265 ms against a lane per position that walked all channels with weights from LDS
// and stored [channel][position] (0.37 ms when that kernel stored [position][channel], 16 bytes at a time 64
// bytes apart); two workers of 32 images: 11 -> 8 us.  Two images at most: with eight 262 us instead of 254, 64 workers of 128
// images 43.6 instead of 41.
// Up to eight wavefronts share an image: two workers of 32 images, whole step 61.7 -> 59.9 us with eight, one of 16 59.0 -> 58.1.
// Each as a block of its own, two to a SIMD, gained 1 % more on images that the caches held, and lost as much on others, which
// each of them then fetched.
constexpr int CONV1_NW = 4, CONV1_NT = 64 * CONV1_NW, CONV1_IPW = 2, CONV1_PARTS = 8;  // wavefronts per block, most images per wavefront, most wavefronts per image
constexpr int CONV1_XW = 30;

// N_META > 0: the workers' metadata are in the arguments, and the first block of a worker puts its own where the
// later kernels of the call look for it (an upload in front costs 4 us of copy and 5 us until conv1 starts).
template <int N_META>
__global__ __launch_bounds__(CONV1_NT) void conv1_fwd_kernel(WorkerBuffers wb, int blocks_per_worker, int ipw, int parts, MetaArgs<N_META> args)
{
    __shared__ __attribute__((aligned(16))) float images[CONV1_NW][CONV1_XW * CONV1_XW];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), c0 = 4 * (lane & 3);
    const int w = blockIdx.x / blocks_per_worker, chunk = blockIdx.x % blocks_per_worker;
    const int unit = chunk * CONV1_NW + wave, part = unit % parts;
    const int B = wb.B, s_begin = unit / parts * ipw, s_end = min(B, s_begin + ipw);
    if (N_META > 0 && chunk == 0 && threadIdx.x == 0) wb.meta[w] = args.m[w];
    if (s_begin >= s_end) return;
    float* __restrict__ xs = images[wave];
    const float* __restrict__ theta = N_META > 0 ? wb.ring + (ptrdiff_t)args.m[w].slot * PSTRIDE : worker_theta(wb, w);

    floatx4 xv[4];  // 196 float4 of an image (lanes past the end repeat the last one)
    auto prefetch = [&](size_t g) {
#pragma unroll
        for (int k = 0; k < 4; ++k) xv[k] = reinterpret_cast<const floatx4*>(wb.x + g * IMG_PIX)[min(lane + 64 * k, IMG_PIX / 4 - 1)];
    };
    prefetch((size_t)w * B + s_begin);
    float wk[4][9], bias[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int i = 0; i < 9; ++i) wk[j][i] = theta[OFF_W1 + (c0 + j) * 9 + i];
        bias[j] = theta[OFF_B1 + c0 + j];
    }
    for (int i = lane; i < CONV1_XW * CONV1_XW; i += 64) xs[i] = 0.f;  // the border stays zero

    for (int s = s_begin; s < s_end; ++s) {
        const size_t g = (size_t)w * B + s;
        wave_lds_fence();  // the last image has been read
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = lane + 64 * k;
            if (64 * (k + 1) <= IMG_PIX / 4 || i < IMG_PIX / 4) {
                float* dst = xs + (4 * i / IMG_W + 1) * CONV1_XW + 4 * i % IMG_W + 1;  // 28 % 4 == 0: one image row
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[e] = xv[k][e];
            }
        }
        wave_lds_fence();
        if (s + 1 < s_end) prefetch(g + 1);
#pragma unroll 1
        for (int pos = lane / 4 + 16 * part; pos < P1_POS; pos += 16 * parts) {
            const float* window = xs + (pos / P1_W * CONV1_XW + pos % P1_W) * 2;
            float patch[4][4];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) patch[a][b] = window[a * CONV1_XW + b];
            floatx4 out;
            uint32_t bytes = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = bias[j];
#pragma unroll
                    for (int i = 0; i < 9; ++i) v[e] = fmaf(wk[j][i], patch[e / 2 + i / 3][e % 2 + i % 3], v[e]);
                }
                // first maximum in scan order; the winner is kept as its offset in a 30-wide padded input image
                float best = v[0];
                uint32_t off = 0;
                if (v[1] > best) { best = v[1]; off = 1; }
                if (v[2] > best) { best = v[2]; off = 30; }
                if (v[3] > best) { best = v[3]; off = 31; }
                out[j] = fmaxf(best, 0.f);
                bytes |= (off | (best > 0.f ? AM1_GATE : 0)) << (8 * j);
            }
            *reinterpret_cast<floatx4*>(wb.p1 + g * P1_SIZE + pos * C1 + c0) = out;
            *reinterpret_cast<uint32_t*>(wb.am1 + g * P1_SIZE + pos * C1 + c0) = bytes;
        }
    }
}

}  // namespace

template <int N_META>
static void start_conv1_fwd(const WorkerBuffers& wb, hipStream_t s)
{
    const ImageSplit sp = split_images(wb, CONV1_IPW, CONV1_PARTS, CONV1_NW, true);
    MetaArgs<N_META> args;
    if (N_META > 0) std::copy(wb.meta_host, wb.meta_host + wb.n, args.m);
    hipLaunchKernelGGL(conv1_fwd_kernel<N_META>, dim3(wb.n * sp.blocks), dim3(CONV1_NT), 0, s, wb, sp.blocks, sp.images, sp.wavefronts, args);
}

void launch_conv1_fwd(const WorkerBuffers& wb, hipStream_t s)
{
    if (!wb.meta_host)
        start_conv1_fwd<0>(wb, s);
    else if (wb.n <= 16)
        start_conv1_fwd<16>(wb, s);
    else
        start_conv1_fwd<META_IN_ARGS>(wb, s);
}

}  // namespace ps
