// Weight gradient of the 1568 -> 512 fully connected layer: rows = 512 units (d3, row-contiguous), columns = 1568
// features (pool2, row-contiguous), contraction over the worker's samples.
#pragma once
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

// 128 x 128 tiles and 128 x 32 at the edge, or 64 x 64 (FEW) for a launch in which those would leave compute units idle.
typedef GemmCfg<false, false, 2, 2, 2, 2, 2> Fc1DwMain;
typedef GemmCfg<false, false, 1, 1, 4, 1, 2> Fc1DwEdge;
typedef GemmCfg<false, false, 1, 1, 2, 2, 4, 32> Fc1DwFew;

// 64 x 64 tiles next to conv2's gradients (8 workers of 64 images: 34 us together) against a launch of wide ones, which
// alone leave the compute units idle that conv2's gradients then have to themselves (16 + 22 us), up to two wide
// tiles for a compute unit (16 of 64: 57 against 24 + 27 us).  Tiles are counted, which depend on the workers alone:
// the batch is the contraction.
inline bool fc1_dw_few(const WorkerBuffers& wb) { return gemm_few_tiles(FC1 / 128 * (FEAT_WIDE / 128) * wb.n / 2, wb.compute_units); }

inline GemmShape fc1_dw_few_shape(int n, int B) { return gemm_shape<Fc1DwFew>(FC1, P2_SIZE, B, FC1, P2_SIZE, n, 0, FC1, 0, P2_SIZE); }

template <bool RAGGED>
__device__ __forceinline__ void fc1_dw_few_block(const WorkerBuffers& wb, const GemmShape& sh, int block, char* lds)
{
    gemm_block<Fc1DwFew, RAGGED, 0>(sh, Fc1DwEpi<false>{wb}, block, lds);
}

}  // namespace ps
