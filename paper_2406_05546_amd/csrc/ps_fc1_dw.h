// Weight gradient of the 1568 -> 512 fully connected layer: rows = 512 units (d3, row-contiguous), columns = 1568
// features (pool2, row-contiguous), contraction over the worker's samples.
#pragma once
#include <type_traits>

#include "ps_common.h"
#include "ps_gemm.h"

namespace ps {

constexpr int FEAT_WIDE = P2_SIZE / 128 * 128;  // 1536: features in whole 128-wide tiles

// Per-worker d fc1.W[u][i] = sum_s d3[s][u] * pool2[s][i], written into the worker's queue entry.
// Rows m are units, columns n features, so a wavefront's lanes run along contiguous memory.  STREAM: stored past the
// caches, in launches that write more than those hold on to (64 workers of 128 images: 122 -> 112 us).  Next to conv2's
// gradients, up to 56 workers, neither kind is ahead always, with the update that reads the rows: plain stores take 0.98-1.02 of the
// time (16 of 64 132.8 and 132.6 us, 42 of 128 416 and 410, of 512 1306 and 1327), but for two to five workers of up to 32 images,
// which store plainly and in wide tiles lose 1 us by it (2 of 32 58.8 and 57.5).
template <bool STREAM>
struct Fc1DwEpi {
    WorkerBuffers wb;
    __device__ const float* a_ptr(int z) const { return wb.d3 + (size_t)z * wb.B * FC1; }
    __device__ const float* b_ptr(int z) const { return wb.p2 + (size_t)z * wb.B * P2_SIZE; }
    __device__ void operator()(int z, int m, int n, float4 acc) const
    {
        float* g = worker_grad(wb, z) + OFF_W3 + (size_t)m * P2_SIZE + n;
        const float v[4] = {acc.x, acc.y, acc.z, acc.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (STREAM)
                __builtin_nontemporal_store(v[i], g + i * P2_SIZE);
            else
                g[i * P2_SIZE] = v[i];
        }
    }
};

// A launch of its own: 128 x 128 tiles and 128 x 32 at the edge.
typedef GemmCfg<false, false, 2, 2, 2, 2, 2> Fc1DwMain;
typedef GemmCfg<false, false, 1, 1, 4, 1, 2> Fc1DwEdge;

// Next to conv2's gradients, which it needs as little as they need it: its blocks fill what those leave idle, and their stores
// run under the others' products.  Tiles are counted, which depend on the workers alone: the batch is the contraction.
// FEW workers (up to ten, less than two wide tiles for a compute unit) have 128 x 64 tiles, SEVERAL 128 x 128.  Steps in us, with
// the update that reads the rows:
//   workers x images   1x64  1x256  2x100  2x256  3x192  4x256  5x37  8x64  8x256  10x128  11x64  12x256  16x64  20x256  40x128
//   128 x 64           56.7   86.7   82.3  103.5  125.9  142.8  68.8  88.9  189.9   158.0  112.6   259.0  133.8   375.3   397.2
//   128 x 128          57.3   91.0   86.3  109.3  129.4  145.2  68.9  89.1  188.2   156.6  113.4   260.3  132.8   368.8   388.8
//   64 x 64            57.6   88.1   88.8  106.5  126.4  143.6  74.1  92.8  196.2   162.8  117.3   270.4
// The narrow ones gain where a few long tiles would be what the launch waits for, the wide ones bring less for a product;
// between eight and twelve workers either is ahead, by 1.5 % at most.
// SEVERAL are up to 42 (eight wide tiles for a compute unit); with more, its blocks hold up conv2's in large batches, and in a
// launch of its own the edge blocks run among the wide ones:
//   workers x images   16x64  20x64  32x256  40x128  42x128  44x128  48x32  48x128  48x256  56x128  64x128  64x256  80x100  80x512
//   here               132.6  168.0   551.7   385.7   410.3   433.1  220.5   463.4   804.8   548.7   594.7  1013.3   668.8  2428.2
//   in its own         135.8  182.6   551.3   395.3   423.3   444.4  233.6   461.4   798.4   539.0   584.5  1006.0   649.9  2418.8
// (Batches up to 64 gain here with more workers too, 2-5 %.)
//
// Alone, a wide tile of a short contraction is what it takes to bring the first stages and to store, and two blocks of a compute
// unit leave much of that uncovered; of 64 x 128 tiles, which need two thirds of the registers, there are three.  Long
// contractions pay for splitting operands more often, and launches of many images for reading them more often, once their operands,
// 8,320 bytes an image, outgrow the last-level cache (edge blocks among the narrow tiles gain nothing: 64 of 128 95, 250 of 250 741).  The
// launch alone, us, events included; 128 x 64 instead of 64 x 128 is up to 4 % behind:
//   workers x images   43x40  250x3  250x64  500x40  64x96  340x64  240x96  256x96  350x64  400x64  600x64  1000x24
//   128 x 128           48.0  171.6   260.1   432.8   84.6   337.3   321.2   365.1   386.1   499.3   753.0    927.2
//   64 x 128            42.5  149.8   235.6   387.4   77.0   310.9   319.5   366.3   387.1   521.4   799.0    984.8
//   workers x images   64x128  100x128  160x128  176x128  200x112  225x100  250x100  190x128  200x128  64x192  80x200  43x250  250x250
//   128 x 128           100.5    150.8    243.4    269.5    276.0    318.4    385.2    317.1    347.7   134.2   177.9   116.0    704.5
//   64 x 128             94.7    146.8    239.0    260.6    259.8    302.7    395.8    319.1    354.2   129.5   181.0   118.5    742.0
typedef GemmCfg<false, false, 1, 2, 2, 2, 2> Fc1DwShort;
inline bool fc1_dw_short(const WorkerBuffers& wb) { return wb.B <= 128 && wb.n * wb.B <= 22500; }
typedef GemmCfg<false, false, 2, 1, 2, 2, 2> Fc1DwFew;
typedef Fc1DwMain Fc1DwSeveral;
enum Fc1DwWhere { FC1_DW_FEW, FC1_DW_SEVERAL, FC1_DW_ALONE };

inline Fc1DwWhere fc1_dw_where(const WorkerBuffers& wb)
{
    const int wide_tiles = FC1 / 128 * (FEAT_WIDE / 128) * wb.n;
    return wide_tiles < 2 * wb.compute_units ? FC1_DW_FEW : wide_tiles < 8 * wb.compute_units ? FC1_DW_SEVERAL : FC1_DW_ALONE;
}

template <class Cfg>
GemmShape fc1_dw_shape(const WorkerBuffers& wb)
{
    return gemm_shape<Cfg>(FC1, P2_SIZE, wb.B, FC1, P2_SIZE, wb.n, 0, FC1, 0, P2_SIZE);
}

template <class Cfg, bool RAGGED>
__device__ __forceinline__ void fc1_dw_block(const WorkerBuffers& wb, const GemmShape& sh, int block, char* lds)
{
    gemm_block<Cfg, RAGGED, 0>(sh, Fc1DwEpi<std::is_same<Cfg, Fc1DwSeveral>::value>{wb}, block, lds);
}

}  // namespace ps
