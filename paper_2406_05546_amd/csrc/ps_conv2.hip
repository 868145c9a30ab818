// conv2 (16 -> 32 channels, 3x3, pad 1, on 14x14 maps) as implicit GEMMs on the gfx950 matrix cores
// (v_mfma_f32_16x16x4_f32): forward with fused ReLU + 2x2 max pool, input gradient, and per-worker
// weight gradient.  Zero-padded feature maps are staged in LDS as [channel][16][16] planes (plane
// pitch a little above 256 floats), so that a 3x3 tap is a compile-time address offset (dy*16 + dx)
// from a lane's base address.
// The 32x16x9 filter bank lives in registers for the whole block (72 VGPRs per lane) in exactly the
// layout the MFMA B operand wants; it is read from the worker's ring slot once per block.
#include "ps_common.h"
#include "ps_split.h"

namespace ps {

namespace {

// LDS pitch (floats) of one padded 16x16 plane, chosen per kernel so that the 32 lanes an LDS read
// serves per cycle fall into 32 different banks: the lane quarters of the forward A operand are four
// channels over 8+8 window columns (pitch = 8 mod 32), those of the input-gradient A operand two
// channels over 16 consecutive positions (pitch = 16 mod 32), and the weight-gradient operands put 16
// channels on 16 lanes at 2 neighbouring positions (pitch = 2 mod 32).
constexpr int CHS_FWD = 264, CHS_DW = 258;

__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Staging is split in two so that the global loads of the next group of images are in flight while
// the matrix cores work on the current one: prefetch_* issues the loads into registers, commit_*
// writes the registers into the padded LDS planes after the barrier that ends the current group.

// pool1 planes of COUNT images (16 channels, 14x14 interiors); NV float4 per thread of a block of NT.
template <int COUNT, int CHS, int NT = 256>
struct Pool1Stage {
    static constexpr int P1_IMS = C1 * CHS;
    static constexpr int N4 = COUNT * (P1_SIZE / 4), NV = (N4 + NT - 1) / NT;
    floatx4 v[NV];
    uint32_t src[NV];  // float offset of this thread's k-th float4 inside a group of COUNT images
    __device__ __forceinline__ void init(int tid)
    {
#pragma unroll
        for (int k = 0; k < NV; ++k) src[k] = (uint32_t)min(tid + NT * k, N4 - 1) * 4;  // threads without an element repeat the last one
    }
    // images [g0, g0 + valid) exist; the rest of the group repeats the last existing image (its
    // results are never stored), so the loads need no branches
    __device__ __forceinline__ void prefetch(const float* __restrict__ p1, size_t g0, int valid, int tid)
    {
        const float* group = p1 + g0 * P1_SIZE;
        if (valid >= COUNT) {  // uniform over the block
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = *reinterpret_cast<const floatx4*>(group + src[k]);
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const uint32_t img = min(src[k] / P1_SIZE, (uint32_t)(valid - 1));
                v[k] = *reinterpret_cast<const floatx4*>(group + img * P1_SIZE + src[k] % P1_SIZE);
            }
        }
    }
    // Where the float4s land does not change from group to group: a table (bits 0-14 the offset of
    // the first element, bit 15 set when the four positions run over the end of a 14-wide row after two
    // elements) replaces that arithmetic by one 2-byte LDS read per float4.
    static __device__ __forceinline__ void build_table(uint16_t* __restrict__ tab, int tid)
    {
        static_assert(COUNT * P1_IMS < (1 << 15), "offsets must fit 15 bits");
        for (int i4 = tid; i4 < N4; i4 += NT) {
            const int img = i4 / (P1_SIZE / 4), r = (i4 % (P1_SIZE / 4)) * 4, c = r / P1_POS, pos = r % P1_POS;
            const int base = img * P1_IMS + c * CHS + 17 + (pos / P1_W) * 16 + pos % P1_W;  // interior starts at (1,1)
            tab[i4] = (uint16_t)(base | (pos % P1_W == P1_W - 2 ? 0x8000 : 0));
        }
    }
    __device__ __forceinline__ void commit(float* __restrict__ tile, const uint16_t* __restrict__ tab, int tid) const
    {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i4 = tid + NT * k;
            if (NT * (k + 1) <= N4 || i4 < N4) {
                const uint32_t e = tab[i4];
                float* dst = tile + (e & 0x7fffu);
                const uint32_t hop = (e >> 15) * 2;  // the next row starts 16 - 14 further on
                dst[0] = v[k][0];
                dst[1] = v[k][1];
                dst[2 + hop] = v[k][2];
                dst[3 + hop] = v[k][3];
            }
        }
    }
};

// Gated pool2 gradient of COUNT images, routed to the window winners of padded planes
// d2[o][16][16] (interior at (1,1)).  A thread moves four consecutive values at a time (one 16-byte load
// of gradients, one 4-byte load of window bytes); where a value lands apart from its winner's place in
// the window never changes, so those offsets are computed once per block (two 16-bit offsets per
// register) and a commit costs a handful of vector instructions per value instead of the divisions by 49
// and 7.  Before the next commit the planes are cleared as a whole with 16-byte stores.
template <int COUNT, int CHS, int NT = 256>
struct D2Stage {
    static constexpr int D2_IMS = C2 * CHS;
    static constexpr int N4 = COUNT * (P2_SIZE / 4), NV = (N4 + NT - 1) / NT;
    static_assert(P2_SIZE % 4 == 0, "a group of four values never straddles two images");
    static_assert(COUNT * D2_IMS < (1 << 16), "offsets must fit 16 bits");
    floatx4 v[NV];
    uint32_t code[NV];
    uint32_t base[NV][2];  // offsets of the four values' windows (winner (0,0)), 16 bits each
    __device__ __forceinline__ void init(int tid)
    {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            uint32_t b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = min(4 * (tid + NT * k), COUNT * P2_SIZE - 4) + j;
                const int img = e / P2_SIZE, r = e % P2_SIZE, o = r / P2_POS, p = r % P2_POS;
                b[j] = (uint32_t)(img * D2_IMS + o * CHS + (2 * (p / P2_W) + 1) * 16 + 2 * (p % P2_W) + 1);
            }
            base[k][0] = b[0] | (b[1] << 16);
            base[k][1] = b[2] | (b[3] << 16);
        }
    }
    __device__ __forceinline__ void prefetch(const WorkerBuffers& wb, size_t g0, int valid, int tid)
    {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i4 = tid + NT * k;
            const bool ok = (NT * (k + 1) <= N4 || i4 < N4) && (4 * i4) / P2_SIZE < valid;
            v[k] = ok ? *reinterpret_cast<const floatx4*>(wb.dp2g + g0 * P2_SIZE + (size_t)i4 * 4) : floatx4{0.f, 0.f, 0.f, 0.f};
            code[k] = ok ? *reinterpret_cast<const uint32_t*>(wb.am2 + g0 * P2_SIZE + (size_t)i4 * 4) : 0u;
        }
    }
    __device__ __forceinline__ void commit(float* __restrict__ d2, int tid) const
    {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            if (!(NT * (k + 1) <= N4 || tid + NT * k < N4)) break;
            // winner (dy, dx) of every byte -> dy * 16 + dx, four at once
            const uint32_t off = (code[k] & 0x01010101u) | ((code[k] & 0x02020202u) << 3);
            d2[(base[k][0] & 0xffffu) + (off & 0xffu)] = v[k][0];
            d2[(base[k][0] >> 16) + ((off >> 8) & 0xffu)] = v[k][1];
            d2[(base[k][1] & 0xffffu) + ((off >> 16) & 0xffu)] = v[k][2];
            d2[(base[k][1] >> 16) + (off >> 24)] = v[k][3];
        }
    }
    // zeroes all COUNT * D2_IMS floats of the planes
    static __device__ __forceinline__ void clear(float* __restrict__ d2, int tid)
    {
        static_assert(COUNT * D2_IMS % 4 == 0, "16-byte stores");
        constexpr int T4 = COUNT * D2_IMS / 4;
#pragma unroll
        for (int i = 0; i < (T4 + NT - 1) / NT; ++i)
            if (NT * (i + 1) <= T4 || tid + NT * i < T4)
                reinterpret_cast<floatx4*>(d2)[tid + NT * i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
};

// ---------------------------------------------------------------------------------------------
// Forward.  GEMM rows are conv outputs ordered (pooled position, window element) so that the four
// accumulators of a lane are one 2x2 pool window; columns are the 32 output channels (two 16-wide
// MFMA tiles sharing the A operand); K = (tap, channel).  A block owns up to FWD_IPB images of one
// worker and walks them FWD_G at a time (FWD_G * 49 pooled positions, four per row tile), FWD_NW wavefronts
// per block.
constexpr int FWD_G = 4, FWD_NW = 4, FWD_NT = 64 * FWD_NW, FWD_IPB = 32;
constexpr int FWD_TILES = (FWD_G * P2_POS + 3) / 4;

__global__ __launch_bounds__(FWD_NT, 512 / FWD_NT) void conv2_fwd_kernel(WorkerBuffers wb, int blocks_per_worker, int ipb)
{
    constexpr int CHS = CHS_FWD, P1_IMS = C1 * CHS;
    __shared__ __attribute__((aligned(16))) float tile[FWD_G * P1_IMS];  // 16,896 B per image
    // pooled position of the group -> offset of its window in the planes / of its output.  On this chip
    // fp32 MFMAs and vector-ALU instructions do not overlap, so index arithmetic inside the tile loop
    // is paid for in matrix time: look it up.
    // (entries past the group's last position, in a last tile that is not full, point at position 0: read, never stored)
    __shared__ int win_off[4 * FWD_TILES], out_off[4 * FWD_TILES];
    __shared__ uint16_t stage_tab[Pool1Stage<FWD_G, CHS_FWD, FWD_NT>::N4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, l16 = lane & 15;
    const int w = blockIdx.x / blocks_per_worker, chunk = blockIdx.x % blocks_per_worker;
    const int B = wb.B, s_begin = chunk * ipb, s_end = min(B, s_begin + ipb);
    const float* __restrict__ W2 = worker_theta(wb, w) + OFF_W2;
    for (int i = tid; i < 4 * FWD_TILES; i += FWD_NT) {
        const int e = i < FWD_G * P2_POS ? i : 0, img = e / P2_POS, pos = e % P2_POS;
        win_off[i] = img * P1_IMS + 2 * (pos / P2_W) * 16 + 2 * (pos % P2_W);
        out_off[i] = img * P2_SIZE + pos;
    }
    Pool1Stage<FWD_G, CHS, FWD_NT>::build_table(stage_tab, tid);

    // B operand of k-step s (channels 4*(s/9) .. +3, tap = s%9): lane (q, l16) holds W2[o][4*(s/9)+q][tap].
    // Taps innermost: the nine A reads of a channel group then share one LDS base address.
    float wreg[36][2];
#pragma unroll
    for (int s = 0; s < 36; ++s)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) wreg[s][hf] = W2[((l16 + 16 * hf) * C1 + 4 * (s / 9) + q) * 9 + s % 9];
    const float bias0 = W2[C2 * C1 * 9 + l16], bias1 = W2[C2 * C1 * 9 + 16 + l16];

    for (int i = tid; i < FWD_G * P1_IMS / 4; i += FWD_NT)
        reinterpret_cast<float4*>(tile)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();

    // this lane's part of the A operand address: channel quarter, window element
    const float* a_lane = tile + q * CHS + ((l16 >> 1) & 1) * 16 + (l16 & 1);
    Pool1Stage<FWD_G, CHS, FWD_NT> stage;
    stage.init(tid);
    stage.prefetch(wb.p1, (size_t)w * B + s_begin, min(FWD_G, s_end - s_begin), tid);
    int rot = 0;
    for (int s0 = s_begin; s0 < s_end; s0 += FWD_G, ++rot) {
        const size_t g0 = (size_t)w * B + s0;
        const int valid = min(FWD_G, s_end - s0);
        stage.commit(tile, stage_tab, tid);
        __syncthreads();
        if (s0 + FWD_G < s_end) stage.prefetch(wb.p1, g0 + FWD_G, min(FWD_G, s_end - s0 - FWD_G), tid);
        for (int t = (wave + rot) % FWD_NW; t < FWD_TILES; t += FWD_NW) {  // which wavefront takes the odd tile rotates
            // A operand: lane row l16 = (pooled position 4t + l16/4, window element l16%4)
            const float* a = a_lane + win_off[4 * t + (l16 >> 2)];
            floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 36; ++s) {
                const float av = a[4 * (s / 9) * CHS + ((s % 9) / 3) * 16 + (s % 9) % 3];
                acc0 = mfma16(av, wreg[s][0], acc0);
                acc1 = mfma16(av, wreg[s][1], acc1);
            }
            // lane (q, l16) now holds the 2x2 window of pooled position 4t + q for channels l16, l16+16
            const int ppo = 4 * t + q;
            if (ppo < valid * P2_POS) {
                const size_t out = g0 * P2_SIZE + out_off[ppo];
                // the four values of a window share their channel's bias: it is added to the winner only
                int code;
                float best = pool_first_max(acc0[0], acc0[1], acc0[2], acc0[3], code) + bias0;
                wb.p2[out + l16 * P2_POS] = fmaxf(best, 0.f);
                wb.am2[out + l16 * P2_POS] = (uint8_t)(code | (best > 0.f ? 4 : 0));
                best = pool_first_max(acc1[0], acc1[1], acc1[2], acc1[3], code) + bias1;
                wb.p2[out + (l16 + 16) * P2_POS] = fmaxf(best, 0.f);
                wb.am2[out + (l16 + 16) * P2_POS] = (uint8_t)(code | (best > 0.f ? 4 : 0));
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------
// Input gradient of conv2 fused with the weight gradient of conv1.
//   d pool1[c][Y][X] = sum_{o,dy,dx} d2pad[o][Y+2-dy][X+2-dx] * W2[o][c][dy][dx], zeroed where pool1 == 0.
// On the bf16 matrix cores (ps_split.h, 16x16x32): GEMM rows are the 16 columns of a padded row of the 14x14
// map, columns the 16 input channels, one k-step the 32 output channels of one tap.  A row of d2 is put
// together in registers from the pooled gradients and the window winners, split once and used for all nine
// taps: the three dx are the same operand moved by 0, 1, 2 lanes, the three dy go to the accumulators of
// three output rows, which rotate.  The 9 x 3 operands of the filter bank stay in 108 registers.
// The result never goes to memory: conv1 has no input gradient, so each value is routed to its pool1
// window's winner and multiplied right away with the 3x3 neighbourhood of input pixels there,
//   d W1[c][dy][dx] += d pool1[c][p] * xpad[winner(c,p) + (dy,dx)],   d b1[c] += d pool1[c][p],
// on the vector ALU.  A wavefront works on whole images by itself (no block barrier anywhere) and writes
// one partial slot of conv1 sums per image, so that nothing depends on how a launch is cut up.
// 65,536 images: 1.146 -> 0.600 ms against the fp32 MFMA kernel in two-wavefront blocks it replaced; two
// workers of 32 images: 87 -> 17 us (a wavefront walked eight images there, now one).
constexpr int DX_NW = 4, DX_NT = 64 * DX_NW, DX_IPW = 8;  // wavefronts per block, most images per wavefront
constexpr int DX_XW = 30, DX_XS = 30 * DX_XW + 16;        // padded input image (and what lanes 14, 15 read past it)

struct DxImage {  // one wavefront's image
    float dp2[P2_SIZE];            // gated pool2 gradient
    uint32_t code[P2_SIZE / 4];    // window winners 0..3, bytes
    uint8_t am1[P1_SIZE + 32];     // pool1 window bytes, [position][channel]
    float xs[DX_XS];
};

// d pool1 of channel c at (Y, X) with fp32 FMAs: for sums the split cannot hold (see ps_split.h).
__device__ __forceinline__ float conv2_dx_plain(const DxImage& im, const float* __restrict__ W2, int c, int Y, int X)
{
    const uint8_t* code = reinterpret_cast<const uint8_t*>(im.code);
    float sum = 0.f;
#pragma unroll 1
    for (int o = 0; o < C2; ++o)
#pragma unroll 1
        for (int t = 0; t < 9; ++t) {
            const int y = Y + 1 - t / 3, x = X + 1 - t % 3;
            float v = 0.f;
            if (y >= 0 && y < P1_W && x >= 0 && x < P1_W) {
                const int p = o * P2_POS + (y >> 1) * P2_W + (x >> 1);
                v = code[p] == 2 * (y & 1) + (x & 1) ? im.dp2[p] : 0.f;
            }
            sum = fmaf(v, W2[(o * C1 + c) * 9 + t], sum);
        }
    return sum;
}

__global__ __launch_bounds__(DX_NT, 2) void conv2_dx_kernel(WorkerBuffers wb, int blocks_per_worker, int ipw)
{
    __shared__ __attribute__((aligned(16))) DxImage images[DX_NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = lane >> 4, l16 = lane & 15;
    const int w = blockIdx.x / blocks_per_worker, chunk = blockIdx.x % blocks_per_worker;
    const int B = wb.B, s_begin = (chunk * DX_NW + wave) * ipw, s_end = min(B, s_begin + ipw);
    if (s_begin >= s_end) return;
    DxImage& im = images[wave];
    const float* __restrict__ W2 = worker_theta(wb, w) + OFF_W2;

    Split8 wt[9];  // lane (q, l16): W2[o = 8q + j][c = l16][tap]
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = W2[((8 * q + j) * C1 + l16) * 9 + t];
        wt[t] = split8(v);
    }
    for (int i = lane; i < DX_XS; i += 64) im.xs[i] = 0.f;  // the border stays zero
    if (lane < 32) im.am1[P1_SIZE + lane] = 0;

    // column l16 of the padded map is x = l16 - 1; columns 0 and 15 are border
    const int x = l16 - 1;
    const uint32_t want0 = (x >= 0 && x < P1_W) ? (uint32_t)(x & 1) : 0x100u;  // winner code of an even row at x; never for the border
    const int d2_at = 8 * q * P2_POS + min(max(x >> 1, 0), P2_W - 1);
    const uint32_t real = q == 3 ? 0u : ~0u;  // positions X = 4q + 2, 4q + 3 exist

    for (int s = s_begin; s < s_end; ++s) {
        const size_t g = (size_t)w * B + s;
        // pooled gradients and winners: 392 float4 and 98 uint4; pool1 window bytes and pixels: 196 of either
        // (lanes past the end repeat the last one).  The other wavefront of the SIMD works meanwhile.
        floatx4 pv[7], xv[4];
        uintx4 pc[2], bv[4];
#pragma unroll
        for (int k = 0; k < 7; ++k)
            pv[k] = reinterpret_cast<const floatx4*>(wb.dp2g + g * P2_SIZE)[min(lane + 64 * k, P2_SIZE / 4 - 1)];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            pc[k] = reinterpret_cast<const uintx4*>(wb.am2 + g * P2_SIZE)[min(lane + 64 * k, P2_SIZE / 16 - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = min(lane + 64 * k, IMG_PIX / 4 - 1);
            xv[k] = reinterpret_cast<const floatx4*>(wb.x + g * IMG_PIX)[i];
            bv[k] = reinterpret_cast<const uintx4*>(wb.am1 + g * P1_SIZE)[i];
        }
        wave_lds_fence();  // the last image has been read
#pragma unroll
        for (int k = 0; k < 7; ++k)
            if (64 * (k + 1) <= P2_SIZE / 4 || lane + 64 * k < P2_SIZE / 4) reinterpret_cast<floatx4*>(im.dp2)[lane + 64 * k] = pv[k];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (64 * (k + 1) <= P2_SIZE / 16 || lane + 64 * k < P2_SIZE / 16)
                reinterpret_cast<uintx4*>(im.code)[lane + 64 * k] = pc[k] & 0x03030303u;
        wave_lds_fence();

        float g1[9], gb1 = 0.f;  // this lane's share of d W1[l16][.] and d b1[l16]
#pragma unroll
        for (int i = 0; i < 9; ++i) g1[i] = 0.f;

        // conv1's gradient from d pool1 row Y: lane (q, l16) holds channel l16 at X = 4q .. 4q + 3
        auto finish_row = [&](int Y, floatx4 acc) {
            if (__any(__builtin_isunordered(acc[0], acc[1]) || __builtin_isunordered(acc[2], acc[3])))
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] = conv2_dx_plain(im, W2, l16, Y, 4 * q + i);
            const uint8_t* bytes = im.am1 + (P1_W * Y + 4 * q) * C1 + l16;
            const float* row = im.xs + 2 * Y * DX_XW + 8 * q;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                uint32_t b = bytes[C1 * i];
                if (i >= 2) b &= real;
                const float* px = row + 2 * i + (b & 0x7fu);
                const uint32_t keep = (uint32_t)((int32_t)(b << 24) >> 31);  // gate bit -> all ones or zero
                const float v = __uint_as_float(__float_as_uint(acc[i]) & keep);
                gb1 += v;
#pragma unroll
                for (int k = 0; k < 9; ++k) g1[k] = fmaf(v, px[(k / 3) * DX_XW + k % 3], g1[k]);
            }
        };

        floatx4 acc[3];  // d pool1 rows y - 1, y, y + 1
#pragma unroll
        for (int i = 0; i < 3; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int py = 0; py < P2_W; ++py) {
            float v[8];
            uint32_t code[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                v[j] = im.dp2[d2_at + j * P2_POS + py * P2_W];
                code[j] = reinterpret_cast<const uint8_t*>(im.code)[d2_at + j * P2_POS + py * P2_W];
            }
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int y = 2 * py + r;
                float d[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) d[j] = code[j] == want0 + 2 * r ? v[j] : 0.f;
                const Split8 a0 = split8(d), a1 = lanes_up<1>(a0), a2 = lanes_up<2>(a0);
                // row y of d2 is tap row dy of row y - 1 + dy of the result (row -1 does not exist)
                const Split8* const moved[3] = {&a2, &a1, &a0};
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) {
                    if (r == 1 || py > 0)
                        mfma_split<3>(*moved[dx], {&wt[dx], &wt[3 + dx], &wt[6 + dx]}, {&acc[0], &acc[1], &acc[2]});
                    else
                        mfma_split<2>(*moved[dx], {&wt[3 + dx], &wt[6 + dx]}, {&acc[1], &acc[2]});
                }
                if (y == 0) {  // the rest of the image, which row 0 of the result needs first
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
                } else {
                    finish_row(y - 1, acc[0]);
                }
                acc[0] = acc[1];
                acc[1] = acc[2];
                acc[2] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
        }
        finish_row(P1_W - 1, acc[0]);

        // fold the four lane quarters; lanes of quarter 0 hold the image's sums for channel l16
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            g1[i] += __shfl_xor(g1[i], 16, 64);
            g1[i] += __shfl_xor(g1[i], 32, 64);
        }
        gb1 += __shfl_xor(gb1, 16, 64);
        gb1 += __shfl_xor(gb1, 32, 64);
        if (q == 0) {
            float* part = wb.part1 + g * OFF_W2;
#pragma unroll
            for (int i = 0; i < 9; ++i) part[OFF_W1 + l16 * 9 + i] = g1[i];
            part[OFF_B1 + l16] = gb1;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Weight gradient: d W2[o][c][dy][dx] = sum over the worker's images and positions of
// d2[o][y][x] * pool1pad[c][y+dy][x+dx];  d b2[o] = sum d2[o].  GEMM rows are the 32 output channels
// (two tiles), columns (tap, input channel) (nine tiles), K = positions, four per MFMA step.  A block
// owns one chunk of a worker's images; its four wavefronts split every image's 49 k-steps and keep
// their 18 accumulator tiles across images; each wavefront's sum goes to its own partial slot.
__global__ __launch_bounds__(256, 2) void conv2_dw_kernel(WorkerBuffers wb)
{
    constexpr int CHS = CHS_DW, D2_IMS = C2 * CHS, P1_IMS = C1 * CHS;
    __shared__ __attribute__((aligned(16))) float d2[D2_IMS];   // 33,024 B
    __shared__ __attribute__((aligned(16))) float p1t[P1_IMS];  // 16,512 B
    // position -> offset inside a padded plane.  On this chip fp32 MFMAs and vector-ALU instructions do
    // not overlap, so index arithmetic inside the MFMA loops is paid for in matrix time: look it up.
    __shared__ int plane_off[P1_POS];
    __shared__ uint16_t stage_tab[Pool1Stage<1, CHS_DW>::N4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = lane >> 4, l16 = lane & 15;
    const int w = blockIdx.x, chunk = blockIdx.y, B = wb.B;
    const int per = (B + N_CHUNK - 1) / N_CHUNK;
    const int s_begin = chunk * per, s_end = min(B, s_begin + per);

    floatx4 acc[2][9];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int j = 0; j < 9; ++j) acc[mt][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    float sum0 = 0.f, sum1 = 0.f;

    for (int i = tid; i < D2_IMS / 4; i += 256) reinterpret_cast<float4*>(d2)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int i = tid; i < P1_IMS / 4; i += 256) reinterpret_cast<float4*>(p1t)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (tid < P1_POS) plane_off[tid] = (tid / P1_W) * 16 + tid % P1_W;
    Pool1Stage<1, CHS>::build_table(stage_tab, tid);
    __syncthreads();
    const float* d2_lane = d2 + l16 * CHS + 17;
    const float* p1_lane = p1t + l16 * CHS;

    D2Stage<1, CHS> sd;
    sd.init(tid);
    Pool1Stage<1, CHS> sp;
    sp.init(tid);
    if (s_begin < s_end) {
        sd.prefetch(wb, (size_t)w * B + s_begin, 1, tid);
        sp.prefetch(wb.p1, (size_t)w * B + s_begin, 1, tid);
    }
    int rot = 0;
    for (int s = s_begin; s < s_end; ++s, ++rot) {
        const size_t g = (size_t)w * B + s;
        sd.commit(d2, tid);
        sp.commit(p1t, stage_tab, tid);
        __syncthreads();
        if (s + 1 < s_end) {
            sd.prefetch(wb, g + 1, 1, tid);
            sp.prefetch(wb.p1, g + 1, 1, tid);
        }
        for (int pos = 4 * ((wave + rot) & 3) + q; pos < P1_POS; pos += 16) {
            const int off = plane_off[pos];
            const float a0 = d2_lane[off], a1 = d2_lane[16 * CHS + off];
            sum0 += a0;
            sum1 += a1;
            const float* b = p1_lane + off;
#pragma unroll
            for (int j = 0; j < 9; ++j) {
                const float bv = b[(j / 3) * 16 + j % 3];
                acc[0][j] = mfma16(a0, bv, acc[0][j]);
                acc[1][j] = mfma16(a1, bv, acc[1][j]);
            }
        }
        __syncthreads();
        sd.clear(d2, tid);
        __syncthreads();  // cleared by all threads before the next commit scatters into the planes
    }

    // accumulator i of tile (mt, j): output channel 16*mt + 4q + i, input channel l16, tap j
    float* part = wb.part + ((size_t)w * N_PART + chunk * 4 + wave) * CONV_PART;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int j = 0; j < 9; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) part[OFF_W2 + ((16 * mt + 4 * q + i) * C1 + l16) * 9 + j] = acc[mt][j][i];
    sum0 += __shfl_xor(sum0, 16, 64);
    sum0 += __shfl_xor(sum0, 32, 64);
    sum1 += __shfl_xor(sum1, 16, 64);
    sum1 += __shfl_xor(sum1, 32, 64);
    if (q == 0) {
        part[OFF_B2 + l16] = sum0;
        part[OFF_B2 + 16 + l16] = sum1;
    }
}

}  // namespace

static int compute_units()
{
    static int cus = 0;
    if (cus == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
    }
    return cus;
}

// Images per block: as many as FWD_IPB when the launch still gives every compute unit as many blocks as fit
// it, else fewer (16, 8), so that a small launch does not leave part of the chip idle.
static int images_per_block(int n, int batch, int most, int blocks_per_cu)
{
    int ipb = most;
    while (ipb > 8 && n * ((batch + ipb - 1) / ipb) < blocks_per_cu * compute_units()) ipb /= 2;
    return ipb;
}

void launch_conv2_fwd(const WorkerBuffers& wb, hipStream_t s)
{
    const int ipb = images_per_block(wb.n, wb.B, FWD_IPB, 512 / FWD_NT), bpw = (wb.B + ipb - 1) / ipb;
    hipLaunchKernelGGL(conv2_fwd_kernel, dim3(wb.n * bpw), dim3(FWD_NT), 0, s, wb, bpw, ipb);
}

int conv1_part_slots(int batch) { return batch; }

// A wavefront walks as many images (up to DX_IPW) as leave two wavefronts for every SIMD: reading and
// splitting the filter bank, once per wavefront, takes about a quarter of an image's time.
void launch_conv2_dx(const WorkerBuffers& wb, hipStream_t s)
{
    int ipw = DX_IPW;
    while (ipw > 1 && wb.n * ((wb.B + ipw - 1) / ipw) < 2 * 4 * compute_units()) ipw /= 2;
    const int bpw = (wb.B + DX_NW * ipw - 1) / (DX_NW * ipw);
    hipLaunchKernelGGL(conv2_dx_kernel, dim3(wb.n * bpw), dim3(DX_NT), 0, s, wb, bpw, ipw);
}

void launch_conv2_dw(const WorkerBuffers& wb, hipStream_t s)
{
    hipLaunchKernelGGL(conv2_dw_kernel, dim3(wb.n, N_CHUNK), dim3(256), 0, s, wb);
}

}  // namespace ps
