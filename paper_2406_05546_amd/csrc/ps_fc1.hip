// The three contractions of the 1568 -> 512 fully connected layer on the matrix cores: forward with fused bias +
// ReLU + dropout, input gradient, and the per-worker weight gradient (which in small launches runs next to
// conv2's gradients instead, ps_fc1_dw.h).
#include "ps_common.h"
#include "ps_fc1_dw.h"
#include "ps_gemm.h"
#include "ps_philox.h"

namespace ps {

namespace {

// fc1 on the matrix cores.  Rows m are fc1 units, columns n are the worker's samples, so that the
// four accumulators a lane holds for one column are four consecutive units of one sample: exactly
// the four words of one Philox call.
struct Fc1FwdEpi {
    WorkerBuffers wb;
    __device__ const float* a_ptr(int z) const { return worker_theta(wb, z) + OFF_W3; }
    __device__ const float* b_ptr(int z) const { return wb.p2 + (size_t)z * wb.B * P2_SIZE; }
    __device__ void operator()(int z, int m, int n, float4 acc) const
    {
        const float4 b = *reinterpret_cast<const float4*>(worker_theta(wb, z) + OFF_B3 + m);
        const WorkerMeta mt = wb.meta[z];
        const uint4 r = philox4x32_10(make_uint4(mt.mb_lo, mt.mb_hi, (uint32_t)n, (uint32_t)(m >> 2)),
                                      make_uint2(wb.seed_lo, wb.seed_hi));
        float4 o;
        o.x = r.x >= wb.drop_threshold ? fmaxf(acc.x + b.x, 0.f) * wb.drop_scale : 0.f;
        o.y = r.y >= wb.drop_threshold ? fmaxf(acc.y + b.y, 0.f) * wb.drop_scale : 0.f;
        o.z = r.z >= wb.drop_threshold ? fmaxf(acc.z + b.z, 0.f) * wb.drop_scale : 0.f;
        o.w = r.w >= wb.drop_threshold ? fmaxf(acc.w + b.w, 0.f) * wb.drop_scale : 0.f;
        *reinterpret_cast<float4*>(wb.ht + ((size_t)z * wb.B + n) * FC1 + m) = o;
    }
};

// d pool2 = d3 . W3 (the conv2 kernels that read it apply the ReLU gate).
// Rows m are pool2 features, columns n samples, contraction over the 512 units.
struct Fc1DxEpi {
    WorkerBuffers wb;
    __device__ const float* a_ptr(int z) const { return worker_theta(wb, z) + OFF_W3; }
    __device__ const float* b_ptr(int z) const { return wb.d3 + (size_t)z * wb.B * FC1; }
    __device__ void operator()(int z, int m, int n, float4 acc) const
    {
        *reinterpret_cast<float4*>(wb.dp2g + ((size_t)z * wb.B + n) * P2_SIZE + m) = acc;
    }
};

}  // namespace

// Block tiles are 128 x 128 (four wavefronts of 64 x 64).  The 1568 features are 12 such tiles plus 32: that
// edge is covered with 32-wide tiles (four wavefronts of 32 x 32 side by side) instead of a thirteenth wide
// tile that would be three quarters empty, by extra blocks of the same launch that run next to the last wide
// tiles.  A launch with fewer wide tiles than compute units takes as long as the serial loop over K of one
// tile, and is cut up: into 64 x 64 tiles (32 x 32, with wavefronts that only multiply, where those find a compute unit
// each), or, in the forward and the input gradient of batches up to 64, into
// 32 x 32 or 32 x 64 tiles with a wavefront for every chunk of K (1568 = 7 x 14 stages, 512 = 4 x 8).  Whether a batch
// is summed in chunks depends on its size alone, so that these sums have the same bits whatever else is in the
// launch; beyond 64 the chunks' totals would not fit the registers of 64 x 64 wavefront tiles.
// Those tiles serve larger launches too (us, in 32 x 32, 32 x 64 and 128 x 64 tiles; of batches up to 32 only the first are full):
//   workers x images     4x64  8x64  12x64  16x64  20x40  40x64  48x64  64x32  64x64  100x64  128x32  256x32  256x64
//   forward, 32 x 32     11.9  12.6   18.4   19.8   24.4   38.9   52.6   34.2   65.4    93.1    65.0   116.6   230.3
//            32 x 64           12.6   17.8   18.8   30.0   44.3
//            128 x 64                                       51     55.6   57.4   58.2    80.4    83.7   159.7   174.1
//   backward, 32 x 32     9.3  13.1   15.8   20.0   21.2   38.5   45.7   33.1                    57.3   107.2
//             32 x 64     9.9  12.5   16.0   19.9   20.0   36.9   43.9          54.9    78.9                   185.7
//             128 x 64                                      41.8   48.0   53.9   55.2    79.9    91.7   167.9   181.6
// Beyond batches of 64 the forward pass is summed in two parts of 784, which two sets of wavefronts form side by side where there
// are no more wide tiles than compute units.
constexpr int FWD_CHUNKS = 7, FWD_CHUNK = 14, DX_CHUNKS = 4, DX_CHUNK = 8, CHUNKED_BATCH = 64;
static_assert(FWD_CHUNKS * FWD_CHUNK * GEMM_K == P2_SIZE && DX_CHUNKS * DX_CHUNK * GEMM_K == FC1, "whole chunks");

// forward: rows = 512 units (W3, k-contiguous), columns = the worker's samples (pool2, k-contiguous)
// Beyond batches of 64, by how many tiles find a compute unit (the launch alone, us; all of K in one part: 1 x 256 23.7, 8 x 128
// 39.8, 21 x 129 50.5, 32 x 128 53.6, 48 x 128 74.3, 64 x 128 87.0, 33 x 176 106.4).  64 x 64 tiles come two to a compute unit, and where there are
// more 128 x 128 tiles than compute units, two rounds of them are ahead of those, whose second half of the batch may be empty:
//   workers x images          1x256   8x128  16x128  21x129  24x80  32x128  22x129  24x200  40x128  56x128  64x128
//   32 x 32, roles              18.0
//   64 x 64, side by side               26.5    29.5    48.3   43.1    49.9    64.7    68.9    67.5    88.8
//   128 x 128, side by side             59.2    59.4    64.8   59.1    60.3    65.3    62.3    61.0    69.5    75.6
//   workers x images         33x129  33x176  25x320  42x160  43x192  72x128  256x256
//   64 x 64, side by side      83.8    87.2    94.2    91.3   110.1
//   128 x 128, side by side   121.7   125.8   128.2   124.1   128.1   128.1    587.9
//   128 x 128, parts in turn  112.7   114.2   117.5   116.6   118.0   112.0    528.0
void launch_fc1_fwd(const WorkerBuffers& wb, hipStream_t s)
{
    const int wide_tiles = FC1 / 128 * ((wb.B + 127) / 128) * wb.n, square_tiles = FC1 / 64 * ((wb.B + 63) / 64) * wb.n;
    const Fc1FwdEpi epi{wb};
    if (wb.B <= CHUNKED_BATCH) {
        const int tiles = FC1 / 32 * wb.n;  // of a worker's samples 32 or 64 at a time
        const bool narrow = wb.B <= 32 || 2 * tiles <= wb.compute_units || tiles > wb.compute_units;
        if (wb.B <= 32 || gemm_few_tiles(wide_tiles, wb.compute_units))
            gemm_launch_chunks<true, true, FWD_CHUNKS, FWD_CHUNK>(FC1, wb.B, P2_SIZE, P2_SIZE, wb.n, narrow, epi, s);
        else
            gemm_launch<GemmCfg<true, true, 2, 1, 2, 2, 2>, FWD_CHUNK, 2>(FC1, wb.B, P2_SIZE, P2_SIZE, P2_SIZE, wb.n, epi, s);
    } else if (gemm_roles_fit<1>(FC1, wb.B, wb.n, wb.compute_units)) {
        gemm_launch_roles<true, true, 2, 1>(FC1, wb.B, P2_SIZE, P2_SIZE, P2_SIZE, wb.n, epi, s);
    } else if (square_tiles <= (wide_tiles > wb.compute_units ? 4 : 2) * wb.compute_units) {
        gemm_launch_sides<GemmCfg<true, true, 1, 1, 2, 2, 4>>(FC1, wb.B, P2_SIZE, P2_SIZE, P2_SIZE, wb.n, epi, s);
    } else if (wide_tiles <= wb.compute_units) {
        gemm_launch_sides<GemmCfg<true, true, 2, 2, 2, 2, 2>>(FC1, wb.B, P2_SIZE, P2_SIZE, P2_SIZE, wb.n, epi, s);
    } else {
        gemm_launch_parts<GemmCfg<true, true, 2, 2, 2, 2, 2>, P2_SIZE>(FC1, wb.B, P2_SIZE, P2_SIZE, wb.n, epi, s);
    }
}

// weight gradient in a launch of its own (see ps_fc1_dw.h)
void launch_fc1_dw(const WorkerBuffers& wb, hipStream_t s)
{
    if (fc1_dw_short(wb))
        gemm_launch_edge<Fc1DwShort, Fc1DwEdge, false, 0, 3>(FC1, P2_SIZE, wb.B, FC1, P2_SIZE, wb.n, FC1, FEAT_WIDE, Fc1DwEpi<true>{wb}, s);
    else
        gemm_launch_edge<Fc1DwMain, Fc1DwEdge, true, 0, 2>(FC1, P2_SIZE, wb.B, FC1, P2_SIZE, wb.n, FC1, FEAT_WIDE, Fc1DwEpi<true>{wb}, s);
}

// input gradient: rows = 1568 features (W3, row-contiguous), columns = samples (d3, k-contiguous),
// contraction over the 512 units
void launch_fc1_dx(const WorkerBuffers& wb, hipStream_t s)
{
    // 64 x 64 tiles already fall behind where there is a wide tile for two compute units (8 workers of 128 images, 96
    // tiles: 22 against 28 us; 16 of 128: 37 against 31); where each finds a compute unit, some wavefronts only multiply (two of
    // 128: 16.6 -> 13.4 us)
    const int wide_tiles = FEAT_WIDE / 128 * ((wb.B + 127) / 128) * wb.n;
    const bool few = gemm_few_tiles(2 * wide_tiles, wb.compute_units);
    const Fc1DxEpi epi{wb};
    if (wb.B <= CHUNKED_BATCH) {
        const bool narrow = wb.B <= 32 || 4 * (P2_SIZE / 32) * wb.n <= 5 * wb.compute_units;
        if (wb.B <= 32 || wide_tiles < 5 * wb.compute_units)
            gemm_launch_chunks<false, true, DX_CHUNKS, DX_CHUNK>(P2_SIZE, wb.B, P2_SIZE, FC1, wb.n, narrow, epi, s);
        else
            gemm_launch_edge<GemmCfg<false, true, 2, 1, 2, 2, 2>, GemmCfg<false, true, 1, 1, 1, 4, 2>, false, DX_CHUNK, 2>(P2_SIZE, wb.B, FC1, P2_SIZE, FC1, wb.n,
                                                                                                          FEAT_WIDE, wb.B, epi, s);
    } else if (gemm_roles_fit<1>(P2_SIZE, wb.B, wb.n, wb.compute_units)) {
        gemm_launch_roles<false, true, 1, 1>(P2_SIZE, wb.B, FC1, P2_SIZE, FC1, wb.n, epi, s);
    } else if (gemm_roles_fit<2>(P2_SIZE, wb.B, wb.n, wb.compute_units)) {
        gemm_launch_roles<false, true, 1, 2>(P2_SIZE, wb.B, FC1, P2_SIZE, FC1, wb.n, epi, s);
    } else if (few) {
        gemm_launch<GemmCfg<false, true, 1, 1, 2, 2, 4, 32>, 0, 2>(P2_SIZE, wb.B, FC1, P2_SIZE, FC1, wb.n, epi, s);
    } else {
        gemm_launch_edge<GemmCfg<false, true, 2, 2, 2, 2, 2>, GemmCfg<false, true, 1, 1, 1, 4, 2>, false, 0, 2>(P2_SIZE, wb.B, FC1, P2_SIZE, FC1, wb.n,
                                                                                               FEAT_WIDE, wb.B, epi, s);
    }
}

}  // namespace ps
