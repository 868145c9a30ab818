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
// caches, in launches that write more than those hold on to (64 workers of 128 images: 122 -> 112 us); in small
// ones the update that follows reads the rows 0.4 us faster out of them.
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
// FEW workers (up to ten, less than two wide tiles for a compute unit) have 128 x 64 tiles: 8 workers of 64 images,
// everything together, 28.5 us (64 x 64 tiles, four times as many loads and waits for them as products: 33; 128 x 128: 28.3), 5 of
// 37 18.5 (23.5; 18.0), 1 of 256 21.9 (22.6; 25.4), 10 of 128 46.8 (53.7; 43.7).  SEVERAL (up to 42) have 128 x 128:
// 16 of 64 44.8 us (128 x 64: 46; in a launch of its own 48-50), 20 of 64 52 (53; 66), 40 of 64 92 (97; 102), 40 of 250
// 268 (288; 275).  With more its rows outgrow the caches: 64 of 128 243 us, in a launch of its own 229; 100 of 64 244 and 217.
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
