// conv2 (16 -> 32 channels, 3x3, pad 1, on 14x14 maps) on the gfx950 bf16 matrix cores with operands split in
// three (ps_split.h): forward with fused ReLU + 2x2 max pool, input gradient fused with conv1's weight
// gradient, and per-worker weight gradient.  In all three a wavefront works on whole images by itself, its
// operands go from memory to registers, are split there once and reused for several taps, and what a
// wavefront needs to turn round inside an image goes through LDS of its own: no block barrier in any loop.
#include "ps_common.h"
#include "ps_fc1_dw.h"
#include "ps_split.h"

namespace ps {

namespace {

// Pool2 window bytes of an image: [channel][7 rows][AM2_PITCH], the byte past a row's seven is 0.
// Bits 0-3: bit (2 dy + dx) of the winner, set only where the winner's activation is > 0; bits 4-5: the winner.
// The input gradient reads bits 0-3 from a second copy, [window][channel].

// ---------------------------------------------------------------------------------------------
// Forward (32x32x16).  GEMM rows are two rows of the map, 16 padded columns each; columns the 32 output
// channels; one k-step the 16 input channels of one tap.  Lane (h, e, column) of the A operand holds eight
// channels of one position of row R + e, which is 32 consecutive bytes of pool1.  The rows read for tap row
// dy are R = 2t - 1 + dy for pooled row t; each pair of rows is split once per tap row, the three dx are the
// same operand moved by 0, 1, 2 lanes, and the pair of dy = 2 is that of dy = 0 one pooled row further on.
// A lane ends up with both rows of four windows of one output channel, so pooling stays in its registers;
// the pooled image is turned to [channel][position] in LDS and leaves in 16-byte stores.
// In launches that would leave SIMDs idle, `parts` wavefronts share an image: four, two or one pooled rows each.
// 14 of 16 columns are real: 378 MFMAs per image, 12,100 cycles of a SIMD's matrix pipe.
// 65,536 images: 1.005 -> 0.61 ms against the fp32 MFMA kernel that staged padded planes in LDS (matrix pipe busy
// 69 % of the cycles); two workers of 32 images: 41 -> 13 us.
constexpr int FWD_NW = 4, FWD_NT = 64 * FWD_NW, FWD_IPW = 8;  // wavefronts per block, most images per wavefront
// Most wavefronts per image, seven of which have a row.  Whole steps with eight against four: one worker of three images
// 58.8 -> 57.3 us, two of 32 62.8 -> 61.6; where two of them would share a SIMD they split the filter bank twice as often: ten of
// 100 145.9 -> 148.9.
constexpr int FWD_PARTS = 8;

// Scale of the gradients of image g, as a scalar.
__device__ __forceinline__ float image_scale(const WorkerBuffers& wb, size_t g) { return __int_as_float(uniform(__float_as_int(wb.grad_scale[g]))); }

struct FwdImage {  // one wavefront's pooled image
    float p2[P2_SIZE];
    uint8_t am2[AM2_SIZE];
    uint8_t am2t[P2_SIZE];
};

// The sums of rows 2t, 2t + 1 for which the split does not hold (ps_split.h), formed again with fp32 matrix
// instructions, operands straight from memory.
__device__ __forceinline__ void conv2_fwd_again(const float* __restrict__ p1, const float* __restrict__ W2, int t, int lane, floatx16& sums)
{
    const uint32_t which = lost_sums<16, 16>(sums);
    lane = rarely(lane);
    const int h = lane >> 5, l32 = lane & 31, e = l32 >> 4, column = lane & 15;
    floatx16 again;
#pragma unroll
    for (int i = 0; i < 16; ++i) again[i] = 0.f;
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
        const int y = 2 * t + e + tap / 3 - 1, x = column + tap % 3 - 1;
        const bool inside = y >= 0 && y < P1_W && x >= 0 && x < P1_W;
        const float* p = p1 + (inside ? y * P1_W + x : 0) * C1 + 8 * h;
        const float* w = W2 + (l32 * C1 + 8 * h) * 9 + tap;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float v = p[j];
            again = __builtin_amdgcn_mfma_f32_32x32x2f32(inside ? v : 0.f, w[9 * j], again, 0, 0, 0);
        }
        if (!worth_going_on<16>(which, again)) break;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (which >> i & 1) sums[i] = again[i];
}

__global__ __launch_bounds__(FWD_NT, 2) void conv2_fwd_kernel(WorkerBuffers wb, int blocks_per_worker, int ipw, int parts)
{
    __shared__ __attribute__((aligned(16))) FwdImage images[FWD_NW];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int h = lane >> 5, l32 = lane & 31, e = l32 >> 4, x = (lane & 15) - 1;
    const int w = blockIdx.x / blocks_per_worker, chunk = blockIdx.x % blocks_per_worker;
    const int unit = chunk * FWD_NW + wave, t_begin = unit % parts * 8 / parts, t_end = min(P2_W, t_begin + 8 / parts);
    const int B = wb.B, s_begin = unit / parts * ipw, s_end = min(B, s_begin + ipw);
    if (s_begin >= s_end || t_begin >= t_end) return;
    FwdImage& im = images[wave];
    const float* __restrict__ W2 = worker_theta(wb, w) + OFF_W2;

    constexpr uint32_t ROW_BYTES = P1_W * C1 * 4, IMAGE_BYTES = P1_SIZE * 4;
    const uint32_t at = (x >= 0 && x < P1_W) ? (uint32_t)e * ROW_BYTES + (uint32_t)(x * C1 + 8 * h) * 4 : BUFFER_NOWHERE;
    floatx4 raw[2][2];  // rows (R, R + 1) of the next pooled row: R = 2t and R = 2t + 1
    auto prefetch = [&](size_t g, int t) {
        const Buffer b = buffer_of(wb.p1 + g * P1_SIZE, IMAGE_BYTES);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 2; ++k) raw[i][k] = buffer_float4(b, at + (uint32_t)(2 * t + i) * ROW_BYTES + 16 * k);
    };
    auto split_raw = [&](int i) {
        const float v[8] = {raw[i][0][0], raw[i][0][1], raw[i][0][2], raw[i][0][3], raw[i][1][0], raw[i][1][1], raw[i][1][2], raw[i][1][3]};
        return split8(v);
    };
    Split8 up;  // rows 2t - 1 and 2t; for an image shared by wavefronts, the rows above the first of this one's
    if (t_begin > 0) {
        const Buffer b = buffer_of(wb.p1 + ((size_t)w * B + s_begin) * P1_SIZE, IMAGE_BYTES);
#pragma unroll
        for (int k = 0; k < 2; ++k) raw[0][k] = buffer_float4(b, at + (uint32_t)(2 * t_begin - 1) * ROW_BYTES + 16 * k);
        up = split_raw(0);
    }
    prefetch((size_t)w * B + s_begin, t_begin);

    Split8 wt[9];  // lane (h, l32): W2[o = l32][c = 8h + j][tap]
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = W2[(l32 * C1 + 8 * h + j) * 9 + t];
        wt[t] = split8(v);
    }
    const float bias = W2[C2 * C1 * 9 + l32];

    for (int s = s_begin; s < s_end; ++s) {
        const size_t g = (size_t)w * B + s;
        wave_lds_fence();  // the last image has been stored
#pragma unroll 1
        for (int t = t_begin; t < t_end; ++t) {
            const Split8 mid = split_raw(0), low = split_raw(1);  // rows 2t, 2t + 1 and 2t + 1, 2t + 2
            if (t == 0) {  // rows -1 (zero) and 0: the odd groups of 16 lanes take what the even ones of `mid` hold
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) up.p[i][j] = __builtin_amdgcn_permlane16_swap(0u, mid.p[i][j], false, false)[0];
            }
            if (t + 1 < t_end)
                prefetch(g, t + 1);
            else if (s + 1 < s_end)
                prefetch(g + 1, 0);
            SplitSum<floatx16> sum;
            sum.clear();
            const Split8* const rows[3] = {&up, &mid, &low};
#pragma unroll
            for (int dy = 0; dy < 3; ++dy) {
                sum.add(*rows[dy], wt[3 * dy]);
                sum.add(lanes_up<1>(*rows[dy]), wt[3 * dy + 1]);
                sum.add(lanes_up<2>(*rows[dy]), wt[3 * dy + 2]);
            }
            up = low;
            floatx16 acc = sum.value();
            // register i of lane (h, l32): channel l32 at row 2t + i / 8, column 8 (i / 4 % 2) + 4h + i % 4
            if (any_lost<16, 16>(acc)) conv2_fwd_again(wb.p1 + g * P1_SIZE, W2, t, lane, acc);
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                uint32_t bytes = 0;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int px = 4 * half + 2 * h + m, i = 4 * half + 2 * m;
                    int code;
                    // the four values of a window share their channel's bias: it is added to the winner only
                    const float best = pool_first_max(acc[i], acc[i + 1], acc[i + 8], acc[i + 9], code) + bias;
                    const uint32_t b = (uint32_t)(code << 4) | (best > 0.f ? 1u << code : 0u);
                    if (half == 0 || m == 0 || h == 0) {  // px = 7 does not exist
                        im.p2[l32 * P2_POS + t * P2_W + px] = fmaxf(best, 0.f);
                        im.am2t[(t * P2_W + px) * C2 + l32] = (uint8_t)(b & 15u);
                        bytes |= b << (8 * m);
                    }
                }
                *reinterpret_cast<uint16_t*>(im.am2 + (l32 * P2_W + t) * AM2_PITCH + 4 * half + 2 * h) = (uint16_t)bytes;
            }
        }
        wave_lds_fence();
        if (parts > 1) {  // windows 7 t_begin .. of every channel
            const int first = P2_W * t_begin, count = P2_W * (t_end - t_begin);
            for (int i = lane; i < count * C2; i += 64) {
                const int o = i / count, p = first + i % count;
                wb.p2[g * P2_SIZE + o * P2_POS + p] = im.p2[o * P2_POS + p];
                wb.am2t[g * P2_SIZE + first * C2 + i] = im.am2t[first * C2 + i];
            }
            const int pitch = AM2_PITCH * (t_end - t_begin);
            for (int i = lane; i < pitch * C2; i += 64) {
                const int at2 = i / pitch * P2_W * AM2_PITCH + t_begin * AM2_PITCH + i % pitch;
                wb.am2[g * AM2_SIZE + at2] = im.am2[at2];
            }
            continue;
        }
#pragma unroll
        for (int k = 0; k < 7; ++k)
            if (64 * (k + 1) <= P2_SIZE / 4 || lane + 64 * k < P2_SIZE / 4)
                reinterpret_cast<floatx4*>(wb.p2 + g * P2_SIZE)[lane + 64 * k] = reinterpret_cast<const floatx4*>(im.p2)[lane + 64 * k];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (64 * (k + 1) <= AM2_SIZE / 16 || lane + 64 * k < AM2_SIZE / 16)
                reinterpret_cast<uintx4*>(wb.am2 + g * AM2_SIZE)[lane + 64 * k] = reinterpret_cast<const uintx4*>(im.am2)[lane + 64 * k];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (64 * (k + 1) <= P2_SIZE / 16 || lane + 64 * k < P2_SIZE / 16)
                reinterpret_cast<uintx4*>(wb.am2t + g * P2_SIZE)[lane + 64 * k] = reinterpret_cast<const uintx4*>(im.am2t)[lane + 64 * k];
    }
}

// ---------------------------------------------------------------------------------------------
// Input gradient of conv2 fused with the weight gradient of conv1.
//   d pool1[c][Y][X] = sum_{o,dy,dx} d2pad[o][Y+2-dy][X+2-dx] * W2[o][c][dy][dx], zeroed where pool1 == 0.
// 16x16x32: GEMM rows are the 16 columns of a padded row of the 14x14 map, columns the 16 input channels, one
// k-step the 32 output channels of one tap.  The pooled gradients are split once per image, on their way into
// LDS; a row of d2 is those parts masked by the window bytes and serves all nine taps: the three dx are the
// same operand moved by 0, 1, 2 lanes, the three dy go to the accumulators of three output rows, which rotate.
// The 9 x 3 operands of the filter bank stay in 108 registers.
// The result never goes to memory: conv1 has no input gradient, so each value is routed to its pool1
// window's winner and multiplied right away with the 3x3 neighbourhood of input pixels there,
//   d W1[c][dy][dx] += d pool1[c][p] * xpad[winner(c,p) + (dy,dx)],   d b1[c] += d pool1[c][p],
// on the vector ALU.  A wavefront works on whole images by itself and writes one partial slot of conv1 sums per
// image: the sum over rows 0-6 plus the sum over rows 7-13.  In launches that would leave SIMDs idle, two
// wavefronts of a block share an image, a half each, and add up the same two sums: nothing depends on how a
// launch is cut up.
// 65,536 images, this and the weight gradient when both were dense: 2.09 -> 1.35 ms against the fp32 MFMA kernels (this one in
// two-wavefront blocks); two workers of 32 images: 87 -> 16 us (a wavefront walked eight images there, now one).  The
// scratch that the compiler reports for the launch is a pair of registers, kept there outside the loops of products.
constexpr int DX_NW = 4, DX_NT = 64 * DX_NW, DX_IPW = 8;  // wavefronts per block, most images per wavefront
constexpr int DX_XW = 30, DX_XS = 30 * DX_XW + 16;        // padded input image (and what lanes 14, 15 read past it)
// A d2 operand lane holds eight output channels 8q + DX_CHANNEL(i); the order is the one in which a word of
// window bytes turns into 16-bit masks.
constexpr int DX_WIN = 40;  // pitch of a window in the planes of parts, in values: 80 bytes, eight windows in different banks
__device__ __forceinline__ constexpr int dx_channel(int i) { return i < 4 ? 2 * i : 2 * i - 7; }   // 0 2 4 6 1 3 5 7
__device__ __forceinline__ int dx_place(int o) { return (o & ~7) + (o & 1) * 4 + (o & 7) / 2; }    // its inverse over all channels

struct DxImage {  // one wavefront's image
    uint16_t dp2[3][P2_POS * DX_WIN];  // pool2 gradient, its three parts, [window][place of channel]
    uint8_t am2t[P2_SIZE];             // pool2 window bytes, [window][channel]
    uint8_t am1[P1_SIZE + 32];         // pool1 window bytes, [position][channel]
    float xs[DX_XS];
};

// The same as conv2_fwd_again for d pool1 row Y of image g, times `scale`: lane (q, l16) holds channel l16 at X = 4q
// .. 4q + 3.
__device__ __forceinline__ void conv2_dx_again(const WorkerBuffers& wb, size_t g, float scale, const float* __restrict__ W2, int Y, int lane, floatx4& sums)
{
    const uint32_t which = lost_sums<4, 4>(sums);
    lane = rarely(lane);
    const int q = lane >> 4, l16 = lane & 15;
    const uint8_t* codes = wb.am2t + g * P2_SIZE;
    const float* dp = wb.dp2g + g * P2_SIZE;
    floatx4 again = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
        const int y = Y + 1 - tap / 3, x = l16 + 1 - tap % 3;  // of d2, for the result at X = l16
        const bool inside = y >= 0 && y < P1_W && x >= 0 && x < P1_W;
        const int p = inside ? (y >> 1) * P2_W + (x >> 1) : 0, bit = 2 * (y & 1) + (x & 1);
#pragma unroll 2
        for (int k = 0; k < C2 / 4; ++k) {
            const int o = 4 * k + q;
            const float d = scale * dp[o * P2_POS + p];
            const bool winner = inside & (codes[p * C2 + o] >> bit & 1);
            again = __builtin_amdgcn_mfma_f32_16x16x4f32(winner ? d : 0.f, W2[(o * C1 + l16) * 9 + tap], again, 0, 0, 0);
        }
        if (!worth_going_on<4>(which, again)) break;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (which >> i & 1) sums[i] = again[i];
}

struct Conv1Sums {
    float v[10];
};

// conv1's sums of image g, channel c: the first half's plus the second half's, without the image's scale.
__device__ __forceinline__ void store_conv1_sums(const WorkerBuffers& wb, size_t g, int c, const float* first, const float (&second)[10], float unscale)
{
    float* part = wb.part1 + g * OFF_W2;
#pragma unroll
    for (int i = 0; i < 9; ++i) part[OFF_W1 + c * 9 + i] = (first[c * 10 + i] + second[i]) * unscale;
    part[OFF_B1 + c] = (first[c * 10 + 9] + second[9]) * unscale;
}

// How conv2's gradients are cut up: blocks of the input gradient, then blocks of the weight gradient.
struct BwdShape {
    int dx_blocks, dx_blocks_per_worker, dx_ipw, dx_parts;
    int dw_blocks, dw_slots, dw_ipw, dw_shared;
};

__device__ __forceinline__ void conv2_dx_block(const WorkerBuffers& wb, const BwdShape& sh, int block, DxImage* images)
{
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), q = lane >> 4, l16 = lane & 15;
    const int w = block / sh.dx_blocks_per_worker, chunk = block % sh.dx_blocks_per_worker;
    const int unit = chunk * DX_NW + wave, half = unit % sh.dx_parts;
    const int B = wb.B, s_begin = min(B, unit / sh.dx_parts * sh.dx_ipw), s_end = min(B, s_begin + sh.dx_ipw);
    // rows of d pool1 to finish; d2 rows from one before to one behind them
    const int Y_begin = P1_W / 2 * half, Y_end = half + 1 == sh.dx_parts ? P1_W : P1_W / 2;
    const int py_begin = half == 0 ? 0 : 3, py_end = Y_end == P1_W ? P2_W : 4;
    DxImage& im = images[wave];
    const float* __restrict__ W2 = worker_theta(wb, w) + OFF_W2;

    Split8 wt[9];  // lane (q, l16): W2[o = 8q + dx_channel(i)][c = l16][tap]
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = W2[((8 * q + dx_channel(i)) * C1 + l16) * 9 + t];
        wt[t] = split8(v);
    }
    for (int i = lane; i < DX_XS; i += 64) im.xs[i] = 0.f;  // the border stays zero
    if (lane < 32) im.am1[P1_SIZE + lane] = 0;

    // column l16 of the padded map is x = l16 - 1; columns 0 and 15 are border, whose shift finds a bit that is never set
    const int x = l16 - 1, px = min(max(x >> 1, 0), P2_W - 1);
    const bool border = x < 0 || x >= P1_W;
    const uint32_t shift[2] = {border ? 0u : 7u - (x & 1), border ? 0u : 5u - (x & 1)};  // bit of (row, x) -> bit 7 of its byte
    const uint32_t real = q == 3 ? 0u : ~0u;  // positions X = 4q + 2, 4q + 3 exist
    // lane (o, half) = (lane / 2, lane % 2) brings in windows 25 half .. of channel o: 25 or 24 of them
    const int o_in = lane >> 1, win_in = 25 * (lane & 1), last_in = o_in * P2_POS + (lane & 1 ? P2_POS - 1 : 24);

    Conv1Sums shared_sum{};
    float unscale = 1.f;
    for (int s = s_begin; s < s_end; ++s) {
        const size_t g = (size_t)w * B + s;
        // the image's pooled gradients, window bytes (98 uint4), pool1 window bytes and pixels (196 of either;
        // lanes past the end repeat the last one).  The other wavefront of the SIMD works meanwhile.
        float pv[26];
        floatx4 xv[4];
        uintx4 pc[2], bv[4];
        const float scale = image_scale(wb, g);
        const float* dp = wb.dp2g + g * P2_SIZE;
#pragma unroll
        for (int k = 0; k < 6; ++k) __builtin_memcpy(&pv[4 * k], dp + o_in * P2_POS + win_in + 4 * k, 16);
        pv[24] = pv[25] = dp[last_in];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            pc[k] = reinterpret_cast<const uintx4*>(wb.am2t + g * P2_SIZE)[min(lane + 64 * k, P2_SIZE / 16 - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = min(lane + 64 * k, IMG_PIX / 4 - 1);
            xv[k] = reinterpret_cast<const floatx4*>(wb.x + g * IMG_PIX)[i];
            bv[k] = reinterpret_cast<const uintx4*>(wb.am1 + g * P1_SIZE)[i];
        }
        unscale = scale == 1.f ? 1.f : 0x1p-64f;
        if (__builtin_expect(scale != 1.f, 0)) {  // an image whose gradients are tiny: see grad_scale
#pragma unroll
            for (int k = 0; k < 26; ++k) pv[k] *= scale;
        }
        wave_lds_fence();  // the last image has been read
        const int at = win_in * DX_WIN + dx_place(o_in);
#pragma unroll
        for (int m = 0; m < 26; m += 2) {
            uint32_t part[3];
            split2(pv[m], pv[m + 1], part[0], part[1], part[2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if (m < 24 || !(lane & 1)) im.dp2[i][at + m * DX_WIN] = (uint16_t)part[i];
                if (m < 24) im.dp2[i][at + (m + 1) * DX_WIN] = (uint16_t)(part[i] >> 16);
            }
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (64 * (k + 1) <= P2_SIZE / 16 || lane + 64 * k < P2_SIZE / 16) reinterpret_cast<uintx4*>(im.am2t)[lane + 64 * k] = pc[k];
        wave_lds_fence();

        float g1[10];  // this lane's share of d W1[l16][.] and d b1[l16]
#pragma unroll
        for (int i = 0; i < 10; ++i) g1[i] = 0.f;
        float* half_sum = reinterpret_cast<float*>(im.am1);  // [16][10], in the place of window bytes that have been used
        // folds the four lane quarters: every lane then holds the sums for channel l16
        auto fold = [&]() {
#pragma unroll
            for (int i = 0; i < 10; ++i) {
                g1[i] += __shfl_xor(g1[i], 16, 64);
                g1[i] += __shfl_xor(g1[i], 32, 64);
            }
        };

        // conv1's gradient from d pool1 row Y: lane (q, l16) holds channel l16 at X = 4q .. 4q + 3
        auto finish_row = [&](int Y, floatx4 acc) {
            if (any_lost<4, 4>(acc)) conv2_dx_again(wb, g, scale, W2, Y, lane, acc);
            const uint8_t* bytes = im.am1 + (P1_W * Y + 4 * q) * C1 + l16;
            const float* row = im.xs + 2 * Y * DX_XW + 8 * q;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t b = bytes[C1 * i];
                if (i >= 2) b &= real;
                const float* p = row + 2 * i + (b & 0x7fu);
                const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)b, 7, 1);  // gate bit -> all ones or zero
                const float v = __uint_as_float(__float_as_uint(acc[i]) & keep);
                g1[9] += v;
#pragma unroll
                for (int k = 0; k < 9; ++k) g1[k] = fmaf(v, p[(k / 3) * DX_XW + k % 3], g1[k]);
            }
        };

        SplitSum<floatx4> acc[3];  // d pool1 rows y - 1, y, y + 1
#pragma unroll
        for (int i = 0; i < 3; ++i) acc[i].clear();
#pragma unroll 1
        for (int py = py_begin; py < py_end; ++py) {
            const int win = py * P2_W + px;
            uintx4 part[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) part[i] = *reinterpret_cast<const uintx4*>(&im.dp2[i][win * DX_WIN + 8 * q]);
            const uint32_t* code = reinterpret_cast<const uint32_t*>(im.am2t + win * C2 + 8 * q);
            const uint32_t code0 = code[0], code1 = code[1];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int y = 2 * py + r;
                // the window's bit of this row and column in bit 7 of every byte; bits 15 and 31 fill half words
                const uint32_t c0 = code0 << shift[r], c1 = code1 << shift[r];
                const uintx4 mask = {__builtin_amdgcn_perm(0u, c0 << 8, 0x09090808u), __builtin_amdgcn_perm(0u, c1 << 8, 0x09090808u),
                                     __builtin_amdgcn_perm(0u, c0, 0x09090808u), __builtin_amdgcn_perm(0u, c1, 0x09090808u)};
                Split8 a0;
#pragma unroll
                for (int i = 0; i < 3; ++i) a0.p[i] = part[i] & mask;
                // row y of d2 is tap row dy of row y - 1 + dy of the result (row -1 does not exist)
#pragma unroll
                for (int dx = 2; dx >= 0; --dx) {
                    const Split8 a = dx == 2 ? a0 : dx == 1 ? lanes_up<1>(a0) : lanes_up<2>(a0);
#pragma unroll
                    for (int t = 0; t <= SPLIT_SMALL; ++t) {
                        if (r == 1 || py > 0) acc[0].add(t, a, wt[dx]);
                        acc[1].add(t, a, wt[3 + dx]);
                        acc[2].add(t, a, wt[6 + dx]);
                    }
                }
                if (y == 2 * py_begin) {  // the rest of the image, which the first finished row needs first
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int i = lane + 64 * k;
                        if (64 * (k + 1) <= IMG_PIX / 4 || i < IMG_PIX / 4) {
                            float* dst = im.xs + (4 * i / IMG_W + 1) * DX_XW + 4 * i % IMG_W + 1;  // 28 % 4 == 0: one image row
#pragma unroll
                            for (int e = 0; e < 4; ++e) dst[e] = xv[k][e];
                            reinterpret_cast<uintx4*>(im.am1)[i] = bv[k];
                        }
                    }
                    wave_lds_fence();
                } else if (y - 1 >= Y_begin) {
                    finish_row(y - 1, acc[0].value());
                    if (y == P1_W / 2 && Y_end == P1_W) {  // the first half is complete: rows 0-6 of the window bytes are free
                        fold();
                        wave_lds_fence();
                        if (q == 0) {
#pragma unroll
                            for (int i = 0; i < 10; ++i) half_sum[l16 * 10 + i] = g1[i];
                        }
#pragma unroll
                        for (int i = 0; i < 10; ++i) g1[i] = 0.f;
                    }
                }
                acc[0] = acc[1];
                acc[1] = acc[2];
                acc[2].clear();
            }
        }
        if (Y_end == P1_W) finish_row(P1_W - 1, acc[0].value());
        fold();
        wave_lds_fence();
        if (sh.dx_parts == 1) {
            if (q == 0) store_conv1_sums(wb, g, l16, half_sum, g1, unscale);
        } else {
            if (half == 0 && q == 0) {
#pragma unroll
                for (int i = 0; i < 10; ++i) half_sum[l16 * 10 + i] = g1[i];
            }
            #pragma unroll
            for (int i = 0; i < 10; ++i) shared_sum.v[i] = g1[i];
        }
    }
    if (sh.dx_parts == 2) {  // one image (or none) per wavefront
        __syncthreads();
        if (half == 1 && s_begin < s_end && q == 0)
            store_conv1_sums(wb, (size_t)w * B + s_begin, l16, reinterpret_cast<const float*>(images[wave - 1].am1), shared_sum.v, unscale);
    }
}

// ---------------------------------------------------------------------------------------------
// Weight gradient (sparse 16x16x64): d W2[o][c][dy][dx] = sum over the worker's images and positions of
// d2[o][y][x] * pool1pad[c][y+dy][x+dx];  d b2[o] = sum d2[o].  GEMM rows are the output channels (two tiles), columns
// the 16 input channels of one tap (nine tiles).  Of the four values of a pooling window only the winner's is not zero, so
// d2 is the operand of v_smfmac_f32_16x16x64_bf16, which holds two of every four consecutive k and says which: k = 4 window +
// (map row, column), a k-step is 16 windows, which is a pooled row (seven and a pad) of each of two images, or of the
// upper and the lower half of one.  Half the matrix instructions, and half the splits, that a dense k-step of 32 takes.
// d2: lane (q, l16) holds channel l16, windows 4 (q % 2) .. + 3 of half q / 2; each pooled value is split once into both
// halves of a register, and the winner's column says which of them stays, its row where the two are taken.
// pool1: lane (q, l16) holds channel l16, the windows 2q and 2q + 1 of both halves.  A register is two columns of a map row;
// tap row dy meets rows 2py - 1 + dy and 2py + dy, of which one is even and one odd: they have the even and the
// odd registers of an operand, so that the next tap row needs one new row, in the place of the one before last.  (The
// winner's row then takes the places of the other row in every other tap row: a second index.)
// Bound by issue: next to 108 smfmac of 16 cycles, which leave room for one vector instruction each, a k-step has about
// 430 (a third of them splits, a quarter adding and clearing the small terms' sums).
// A block's four wavefronts take conv2_dw_ipw(B) images each at most, meet in LDS once, and write one partial slot;
// the slots depend on the batch alone, so that the order of a worker's sums does not depend on the launch.
// The 72 registers of a second accumulator (ps_split.h) do not fit next to the operands: the five small terms of
// a k-step are summed from zero and added on the vector ALU.  What is then cut off towards minus infinity is
// of one sign, and the odd wavefronts take d2 negated and are subtracted, so that it cancels in a slot.  Against 64 bits
// d W2 is off by 0.62-0.79e-7 (1.09-1.51e-7 with fp32 MFMAs), d b2, summed on the vector ALU, by 0.54-0.74e-7 (0.55-0.76e-7 as
// a product with a column of ones).
// 65,536 images, this and the input gradient: 1.35 ms with dense 16x16x32, 1.07 with the sparse form (this alone 0.73 ->
// 0.43), matrix pipe busy 51 % of the cycles; 64 workers of 128 images 172 -> 139 us, 16 of 64 27.8 -> 23.6, one of 256
// 24.7 -> 22.7.
constexpr int DW_NW = 4, DW_NT = 64 * DW_NW, DW_MAX_SLOTS = 16;
constexpr int DW_REGS = 2 * 9 * 4;  // sums per lane without the bias

typedef uint32_t uintx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));

// Two map rows of pool1 as the dense operands of three tap columns, part by part: register 4 image + 2 window + (odd row).
struct DwRows {
    uintx8 t[3][3];  // [tap column][part]
    // columns 4q - 1 .. 4q + 4 of a row of one of the two images
    template <int ODD>
    __device__ __forceinline__ void put(int image, const float (&v)[6])
    {
        uint32_t p[3][3];
#pragma unroll
        for (int j = 0; j < 3; ++j) split2(v[2 * j], v[2 * j + 1], p[0][j], p[1][j], p[2][j]);
        const int at = 4 * image + ODD;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            t[0][i][at] = p[i][0];
            t[0][i][at + 2] = p[i][1];
            t[1][i][at] = __builtin_amdgcn_alignbit(p[i][1], p[i][0], 16);
            t[1][i][at + 2] = __builtin_amdgcn_alignbit(p[i][2], p[i][1], 16);
            t[2][i][at] = p[i][1];
            t[2][i][at + 2] = p[i][2];
        }
    }
    template <int ODD>
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 8; j += 2) t[dx][i][j + ODD] = 0;
    }
};

// The parts of one value, each in both halves.
__device__ __forceinline__ void split_twice(float x, uint32_t (&p)[3])
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        p[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{x, x}, bf16x2));
        x -= __uint_as_float(p[i] << 16);
    }
}

// Zeros, made where they are wanted: the compiler would make them all at the top of the loop.
__device__ __forceinline__ floatx4 cleared()
{
    floatx4 zero = {0.f, 0.f, 0.f, 0.f};
    asm volatile("" : "+s"(zero));
    return zero;
}

// Four pooled gradients of an output channel as the sparse operand.
struct DwGrads {
    Split8 value;   // window by window: in the low half if the winner is in the left column, in the high half if in the right one
    int place[2];   // four bits a window: where in the window's four values they are taken; [1]: with the two map rows exchanged
    float sum;      // of the values, for the bias
};

__device__ __forceinline__ DwGrads dw_grads(const floatx4& pooled, uint32_t bytes, float scale)
{
    DwGrads d;
    // the winner's column: bits 0 and 2 of a byte the left one, bits 1 and 3 the right one; to the top of every byte
    const uint32_t any = bytes | bytes >> 2, left = any << 7, right = any << 6;
    const uint32_t mask[4] = {__builtin_amdgcn_perm(right << 8, left << 8, 0x0a0a0808u), __builtin_amdgcn_perm(right, left, 0x0a0a0808u),
                              __builtin_amdgcn_perm(right << 8, left << 8, 0x0b0b0909u), __builtin_amdgcn_perm(right, left, 0x0b0b0909u)};
    float v[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        uint32_t p[3];
        v[m] = scale * pooled[m];
        split_twice(v[m], p);
#pragma unroll
        for (int i = 0; i < 3; ++i) d.value.p[i][m] = p[i] & mask[m];
        v[m] = mask[m] ? v[m] : 0.f;
    }
    d.sum = (v[0] + v[1]) + (v[2] + v[3]);
    // the winner's row, bit 5 of a byte: its two places are 0, 1 (0b0100) or 2, 3 (0b1110)
    uint32_t row = bytes >> 5 & 0x01010101u;
    row = (row | row >> 4) & 0x00110011u;
    row = (row | row >> 8) & 0x1111u;
    d.place[0] = (int)(0x4444u + 10u * row);
    d.place[1] = d.place[0] ^ 0xaaaa;
    return d;
}

// The same as conv2_fwd_again for the sums over images [s_begin, s_end) of worker w: output channels 16 mt + 4q + i,
// input channel l16, tap 0..8.  The sums are times `scale`.  An infinite activation does not count: d2 is zero at every place that
// sees it, whose products are left out (as where windows are multiplied, of which most places never meet an operand), or NaN,
// which is in the sums without it.  Were it neither, an infinite pool2 value would have come of it, and with that an image
// whose fc1 units are all off or whose logits are not numbers.
__device__ __forceinline__ void conv2_dw_again(const WorkerBuffers& wb, int w, int s_begin, int s_end, int mt, int tap, float scale, int lane, floatx4& sums)
{
    const uint32_t which = lost_sums<4, 4>(sums);
    lane = rarely(lane);
    const int q = lane >> 4, l16 = lane & 15, o = 16 * mt + l16;
    floatx4 again = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s = s_begin; s < s_end; ++s) {
        const size_t g = (size_t)w * wb.B + s;
#pragma unroll 7
        for (int k = 0; k < P1_POS / 4; ++k) {
            const int pos = 4 * k + q, y = pos / P1_W, x = pos % P1_W, r = o * P2_W + (y >> 1);
            const bool winner = wb.am2[g * AM2_SIZE + r * AM2_PITCH + (x >> 1)] >> (2 * (y & 1) + (x & 1)) & 1;
            const float d = scale * wb.dp2g[g * P2_SIZE + r * P2_W + (x >> 1)];
            const int yy = y + tap / 3 - 1, xx = x + tap % 3 - 1;
            const bool inside = yy >= 0 && yy < P1_W && xx >= 0 && xx < P1_W;
            const float v = wb.p1[g * P1_SIZE + (inside ? yy * P1_W + xx : 0) * C1 + l16];
            again = __builtin_amdgcn_mfma_f32_16x16x4f32(winner ? d : 0.f, inside && fabsf(v) < INFINITY ? v : 0.f, again, 0, 0, 0);
        }
        if (!worth_going_on<4>(which, again)) break;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (which >> i & 1) sums[i] = again[i];
}

typedef float DwSums[DW_NW][DW_REGS + 2][64];  // 75,776 B

// A wavefront's two images: pooled gradients and window bytes as they lie in memory, in whole KB.
struct DwImages {
    float dp2[2][7 * 256];
    uint8_t am2[2][2048];
};
union DwShared {
    DwImages images[DW_NW];
    DwSums red;
};

// SHARED: a launch that would leave SIMDs idle has six blocks for a slot, one for every (tap row, half of the
// output channels); each sum is formed as in the one block, only fewer of them.  A share repeats its images' splits, so what
// it saves grows with the images of a wavefront.  Whole steps, shared and not: up to three wavefronts for four SIMDs one worker
// of 64 images 56.0 and 56.9 us, of 128 71.7 and 77.3, of 256 86.6 and 101.6, two of 128 87.4 and 87.8, of 256 103.7 and
// 113.6 (but two of 64 61.6 and 60.9).  With more, three of 64 68.4 and 67.2, of 100 95.4 and 93.4; but where a wavefront has three
// images and more, up to four and a half for four SIMDs three of 160 104.8 and 108.2, of 192 126.3 and 126.0, of 288
// 148.9 and 154.3, of 512 188.6 and 194.1, and beyond, four of 192 134.6 and 131.2, of 256 148.5 and 143.0.
constexpr int DW_SHARES = 6;

template <bool SHARED>
__device__ __forceinline__ void conv2_dw_block(const WorkerBuffers& wb, const BwdShape& sh, int block, DwShared& lds)
{
    constexpr int MTS = SHARED ? 1 : 2, DYS = SHARED ? 1 : 3;  // halves of the output channels and tap rows of this block
    const int share = SHARED ? block % DW_SHARES : 0, mt0 = share / 3, dy0 = share % 3;
    if (SHARED) block /= DW_SHARES;
    const int slots = sh.dw_slots, ipw = sh.dw_ipw;
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6), q = lane >> 4, l16 = lane & 15;
    const int w = block / slots, slot = block % slots;
    const int B = wb.B, s_begin = min(B, (slot * DW_NW + wave) * ipw), s_end = min(B, s_begin + ipw);

    float unscale = s_begin < s_end ? 0x1p-64f : 1.f;  // of a wavefront's sums, if all its images have tiny gradients
    for (int s = s_begin; s < s_end; ++s)
        if (image_scale(wb, (size_t)w * B + s) == 1.f) unscale = 1.f;
    const float scale = (wave & 1 ? -1.f : 1.f) * (unscale == 1.f ? 1.f : 0x1p64f);
    floatx4 acc[MTS][3 * DYS];
    float acc_b[MTS];
#pragma unroll
    for (int mt = 0; mt < MTS; ++mt) {
        acc_b[mt] = 0.f;
#pragma unroll
        for (int j = 0; j < 3 * DYS; ++j) acc[mt][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }

    constexpr uint32_t POS_BYTES = C1 * 4, ROW_BYTES = P1_W * POS_BYTES;
    // columns 4q - 1 .. 4q + 4; the first of them, and the last three of the last quarter, are outside the map
    const uint32_t at = (uint32_t)(4 * q) * POS_BYTES + 4 * l16, at_first = q == 0 ? BUFFER_NOWHERE : at - POS_BYTES;
    const uint32_t at_last = q == 3 ? BUFFER_NOWHERE : at + 2 * POS_BYTES;
    // What the two halves of a contraction are: two images, or, where a wavefront has but one left, the upper four rows of
    // windows of it and the lower three.
    auto alone = [&](int s) { return s + 1 >= s_end; };
    auto load_row = [&](int s, int set, int R, float (&v)[6]) {
        const int image = alone(s) ? 0 : set;
        if (alone(s)) R += 8 * set;
        // a descriptor of the row alone: a map's own would have to take the row as the scalar offset, of which the compiler's
        // definition says that bounds do not count it, and rows 14 to 16 are the next image's
        const bool here = s + image < s_end && R >= 0 && R < P1_W;
        const float* row = wb.p1 + ((size_t)w * B + (here ? s + image : s_begin)) * P1_SIZE + (here ? R * P1_W * C1 : 0);
        const Buffer b = buffer_of(row, here ? ROW_BYTES : 0);
        v[0] = buffer_float(b, at_first);
#pragma unroll
        for (int k = 0; k < 2; ++k) v[1 + k] = buffer_float(b, at + k * POS_BYTES);
#pragma unroll
        for (int k = 0; k < 3; ++k) v[3 + k] = buffer_float(b, at_last + k * POS_BYTES);
    };
    // map rows of a step: 2py + 2 and 2py + 1; SHARED, the two that tap row dy0 meets
    const int even_row = SHARED && dy0 < 2 ? 0 : 2, odd_row = SHARED && dy0 == 0 ? -1 : 1;
    float even[2][6], odd[2][6];
    DwImages& im = lds.images[wave];
    // The images' gradients and bytes straight to LDS: by lanes, as they are used, each would touch 64 cache lines for a
    // quarter KB.
    auto bring_images = [&](int s) {
#pragma unroll
        for (int image = 0; image < 2; ++image) {
            if (alone(s) && image == 1) break;
            const size_t g = (size_t)w * B + s + image;
            const Buffer d = buffer_of(wb.dp2g + g * P2_SIZE, P2_SIZE * 4);
            const Buffer b = buffer_of(reinterpret_cast<const float*>(wb.am2 + g * AM2_SIZE), AM2_SIZE);
#pragma unroll
            for (int k = 0; k < 7; ++k) buffer_to_lds16(d, im.dp2[image] + 256 * k, 16 * lane + 1024 * k);
#pragma unroll
            for (int k = 0; k < 2; ++k) buffer_to_lds16(b, im.am2[image] + 1024 * k, 16 * lane + 1024 * k);
        }
    };
    auto load_rows = [&](int s, int py) {
#pragma unroll
        for (int image = 0; image < 2; ++image) {
            load_row(s, image, 2 * py + odd_row, odd[image]);
            load_row(s, image, 2 * py + even_row, even[image]);
        }
    };

    if (s_begin < s_end) {
        bring_images(s_begin);
        load_rows(s_begin, 0);
    }
    for (int s = s_begin; s < s_end; s += 2) {
        const bool one_image = alone(s);
        const int steps = one_image ? 4 : P2_W;
        // windows px = 4 (q % 2) .. + 3 of half q / 2 (px = 7: whatever follows, masked)
        const int image_of = one_image ? 0 : q >> 1, py_of = one_image ? 4 * (q >> 1) : 0;
        const float* const pooled = im.dp2[image_of] + (16 * mt0 + l16) * P2_POS + py_of * P2_W + 4 * (q & 1);
        const uint8_t* const bytes = im.am2[image_of] + ((16 * mt0 + l16) * P2_W + py_of) * AM2_PITCH + 4 * (q & 1);
        DwRows rows;
        rows.clear<1>();  // row -1
        if (!SHARED) {
            float first[2][6];
#pragma unroll
            for (int set = 0; set < 2; ++set) load_row(s, set, 0, first[set]);
#pragma unroll
            for (int set = 0; set < 2; ++set) rows.put<0>(set, first[set]);
            if (one_image) {
                load_row(s, 1, -1, first[1]);
                rows.put<1>(1, first[1]);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the images are in LDS
#pragma unroll 1
        for (int py = 0; py < steps; ++py) {
            const int next_s = py + 1 < steps ? s : s + 2, next_py = py + 1 < steps ? py + 1 : 0;
            DwGrads d2[MTS];
#pragma unroll
            for (int mt = 0; mt < MTS; ++mt) {
                const float* p = pooled + 16 * mt * P2_POS + py * P2_W;
                uint32_t b = *reinterpret_cast<const uint32_t*>(bytes + (16 * mt * P2_W + py) * AM2_PITCH);
                if (py + py_of >= P2_W) b = 0;
                d2[mt] = dw_grads(floatx4{p[0], p[1], p[2], p[3]}, b, scale);
                acc_b[mt] += d2[mt].sum;
            }
            if (py + 1 == steps) {  // these were the last values of the images: the next ones take their place
                // what comes straight to LDS does not wait for reads that are on their way: with fc1's blocks next to this one
                // they were late enough, now and then, to find the next image
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (s + 2 < s_end) bring_images(s + 2);
            }
#pragma unroll
            for (int dy = 0; dy < DYS; ++dy) {
                if (SHARED || dy == 1) {
#pragma unroll
                    for (int image = 0; image < 2; ++image) rows.put<1>(image, odd[image]);
                }
                if (SHARED || dy == 2) {
#pragma unroll
                    for (int image = 0; image < 2; ++image) rows.put<0>(image, even[image]);
                    load_rows(next_s, next_py);
                }
                if (!SHARED) __builtin_amdgcn_sched_barrier(0);
                const bool exchanged = SHARED ? dy0 != 1 : dy != 1;
                // tile by tile; a tile's small terms are added to its sums under the next one's products
                floatx4 small[2];
                auto settle = [&](int n) { acc[n % MTS][3 * dy + n / MTS] += small[n % 2]; };
#pragma unroll
                for (int n = 0; n < 3 * MTS; ++n) {
                    const int mt = n % MTS, dx = n / MTS, place = exchanged ? d2[mt].place[1] : d2[mt].place[0];
                    const auto product = [&](int ta, int tb, floatx4 sum) {
                        return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(d2[mt].value.part(ta), __builtin_bit_cast(bf16x16, rows.t[dx][tb]), sum, place, 0, 0);
                    };
                    small[n % 2] = cleared();
#pragma unroll
                    for (int t = 0; t < SPLIT_SMALL; ++t) small[n % 2] = product(TERM_A[t], TERM_B[t], small[n % 2]);
                    acc[mt][3 * dy + dx] = product(0, 0, acc[mt][3 * dy + dx]);
                    if (n > 0) settle(n - 1);
                }
                settle(3 * MTS - 1);
            }
        }
    }

    DwSums& red = lds.red;
    __syncthreads();  // everybody has read its images, whose place the sums take
    // register i of tile (mt, j): output channel 16 mt + 4q + i, input channel l16, tap j
    bool lost = false;
#pragma unroll
    for (int mt = 0; mt < MTS; ++mt) {
#pragma unroll
        for (int j = 0; j < 3 * DYS; ++j) {
            lost |= any_lost<4, 4>(acc[mt][j]);
#pragma unroll
            for (int i = 0; i < 4; ++i) red[wave][((mt0 + mt) * 9 + 3 * dy0 + j) * 4 + i][lane] = acc[mt][j][i];
        }
        acc_b[mt] += __shfl_xor(acc_b[mt], 16, 64);
        acc_b[mt] += __shfl_xor(acc_b[mt], 32, 64);
        if (q == 0) red[wave][DW_REGS + mt0 + mt][l16] = acc_b[mt];
    }
    const int r_begin = (mt0 * 9 + 3 * dy0) * 4;  // of this block's DYS * MTS * 12 registers
    if (lost) {
#pragma unroll 1
        for (int r = r_begin; r < r_begin + 12 * DYS * MTS; r += 4) {
            floatx4 sums;
#pragma unroll
            for (int i = 0; i < 4; ++i) sums[i] = red[wave][r + i][lane];
            if (!any_lost<4, 4>(sums)) continue;
            conv2_dw_again(wb, w, s_begin, s_end, r / 36, r % 36 / 4, scale, lane, sums);
#pragma unroll
            for (int i = 0; i < 4; ++i) red[wave][r + i][lane] = sums[i];
        }
    }
    if (__builtin_expect(unscale != 1.f, 0)) {
        wave_lds_fence();
#pragma unroll 1
        for (int r = r_begin; r < r_begin + 12 * DYS * MTS; ++r) red[wave][r][lane] *= unscale;
        if (lane < 16 * MTS) red[wave][DW_REGS + mt0 + lane / 16][lane % 16] *= unscale;
    }
    __syncthreads();
    float* part = wb.part + ((size_t)w * slots + slot) * CONV2_PART;
#pragma unroll
    for (int i = 0; i < 12 * DYS * MTS / DW_NW; ++i) {
        const int r = r_begin + (threadIdx.x >> 6) + DW_NW * i;
        part[r * 64 + lane] = (red[0][r][lane] - red[1][r][lane]) + (red[2][r][lane] - red[3][r][lane]);
    }
    if (dy0 == 0 && threadIdx.x < 16 * MTS) {
        const int r = DW_REGS + mt0 + threadIdx.x / 16, j = threadIdx.x % 16;
        part[CONV2_PART_B2 + 16 * mt0 + threadIdx.x] = (red[0][r][j] - red[1][r][j]) + (red[2][r][j] - red[3][r][j]);
    }
}

// conv2's two gradients in one launch, and with up to 42 workers fc1's weight gradient (ps_fc1_dw.h) with them: none needs
// another, the one fills the SIMDs that the others leave idle, and one or two launches are saved.
struct NoFc1Dw {
    static constexpr int STAGE = 0;
};
template <class Fc1Dw, bool RAGGED>  // fc1's tiles, and whether the batch is not a multiple of their stages
__global__ __launch_bounds__(256, 2) void backward_kernel(WorkerBuffers wb, BwdShape sh, GemmShape fc1)
{
    static_assert(DX_NT == 256 && DW_NT == 256, "one block size");
    __shared__ __attribute__((aligned(16))) union {
        DxImage images[DX_NW];
        DwShared dw;
        char stages[2 * Fc1Dw::STAGE + 1];
    } lds;
    int block = blockIdx.x;
    if (block < sh.dx_blocks) return conv2_dx_block(wb, sh, block, lds.images);
    block -= sh.dx_blocks;
    if (block < sh.dw_blocks) return sh.dw_shared ? conv2_dw_block<true>(wb, sh, block, lds.dw) : conv2_dw_block<false>(wb, sh, block, lds.dw);
    // fc1's blocks start at a multiple of 8: block number mod 8 says which XCD a tile runs on
    if constexpr (Fc1Dw::STAGE > 0) {
        block = blockIdx.x - (sh.dx_blocks + sh.dw_blocks + 7) / 8 * 8;
        if (block >= 0) fc1_dw_block<Fc1Dw, RAGGED>(wb, fc1, block, lds.stages);
    }
}

}  // namespace

void launch_conv2_fwd(const WorkerBuffers& wb, hipStream_t s)
{
    const ImageSplit sp = split_images(wb, FWD_IPW, FWD_PARTS, FWD_NW, true);
    hipLaunchKernelGGL(conv2_fwd_kernel, dim3(wb.n * sp.blocks), dim3(FWD_NT), 0, s, wb, sp.blocks, sp.images, sp.wavefronts);
}

int conv1_part_slots(int batch) { return batch; }

// Images per wavefront.  They are taken in pairs, seven k-steps each, and the last of an odd number in halves, in four.  (An even
// number in its place is fewer and longer wavefronts: one worker of 160 images 76.7 against 80.9 us, five of 192 138 and 143, five of
// 320 178 and 182; large launches, which lose the empty half of a k-step, 64 of 192 885 against 871, 256 of 160 3009 and 2969.)
static int conv2_dw_ipw(int batch) { return (batch + DW_NW * DW_MAX_SLOTS - 1) / (DW_NW * DW_MAX_SLOTS); }

int conv2_part_slots(int batch)
{
    const int per_slot = DW_NW * conv2_dw_ipw(batch);
    return (batch + per_slot - 1) / per_slot;
}

template <class Fc1Dw>
static void start_backward(const WorkerBuffers& wb, const BwdShape& sh, const GemmShape& fc1, hipStream_t s)
{
    const int conv_blocks = (sh.dx_blocks + sh.dw_blocks + 7) / 8 * 8;
    auto kernel = backward_kernel<Fc1Dw, false>;
    int blocks = conv_blocks;
    if constexpr (Fc1Dw::STAGE > 0) {
        if (wb.B % Fc1Dw::KS != 0) kernel = backward_kernel<Fc1Dw, true>;
        blocks += gemm_grid(fc1);
    }
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, s, wb, sh, fc1);
}

void launch_backward(const WorkerBuffers& wb, hipStream_t s)
{
    BwdShape sh;
    const ImageSplit dx = split_images(wb, DX_IPW, 2, DX_NW, false);
    sh.dx_ipw = dx.images;
    sh.dx_parts = dx.wavefronts;
    sh.dx_blocks_per_worker = dx.blocks;
    sh.dx_blocks = wb.n * sh.dx_blocks_per_worker;
    sh.dw_slots = conv2_part_slots(wb.B);
    sh.dw_ipw = conv2_dw_ipw(wb.B);
    sh.dw_shared = 2 * DW_SHARES * DW_NW * wb.n * sh.dw_slots <= (sh.dw_ipw < 3 ? 6 : 9) * wb.compute_units;
    sh.dw_blocks = wb.n * sh.dw_slots * (sh.dw_shared ? DW_SHARES : 1);
    const Fc1DwWhere where = fc1_dw_where(wb);
    if (where == FC1_DW_FEW)
        start_backward<Fc1DwFew>(wb, sh, fc1_dw_shape<Fc1DwFew>(wb), s);
    else if (where == FC1_DW_SEVERAL)
        start_backward<Fc1DwSeveral>(wb, sh, fc1_dw_shape<Fc1DwSeveral>(wb), s);
    else
        start_backward<NoFc1Dw>(wb, sh, GemmShape{}, s);
}

bool fc1_dw_in_backward(const WorkerBuffers& wb) { return fc1_dw_where(wb) != FC1_DW_ALONE; }

}  // namespace ps
