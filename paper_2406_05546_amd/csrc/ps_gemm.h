// Batched fp32 GEMM on the gfx950 bf16 matrix cores with operands split in three (ps_split.h), used for the
// three contractions of the 1568 -> 512 fully connected layer (forward, input gradient, per-worker weight
// gradient).
//
//   C[m][n] = sum_k A(m,k) * B(n,k)        one problem per batch index z (= worker)
//
// Either operand may be stored k-contiguous ("KC": element (r,k) at base[r*ld + k]) or row-contiguous ("RC":
// element (r,k) at base[k*ld + r]).  A 256-thread block (4 wavefronts arranged WM x WN) owns a (WM*TM*32) x
// (WN*TN*32) tile of C; each wavefront owns TM x TN MFMA tiles of 32x32.  K advances 16 at a time through
// double-buffered LDS: a thread loads eight consecutive values (AHEAD + 1 stages ahead), splits them once and
// writes the three parts with 16-byte stores, so that splitting costs 88 vector instructions per thread and
// stage next to the wavefront's 24 MFMAs.  The parts of a KC operand lie as [k / 8][row][8 k] and a lane's
// operand is one 16-byte LDS read; those of an RC operand lie as [k][row], and the transposing LDS read
// (ds_read_b64_tr_b16: 16 lanes read four k of 16 rows and each gets the four k of its row) turns them.
//
// Blocks are numbered so that the blocks of one batch index run next to each other on one XCD (work
// groups are handed to the 8 XCDs round-robin, each XCD has its own L2): the operand that belongs to
// the batch index is then fetched from HBM once and re-used out of that L2.
//
// The epilogue functor names the operands (a_ptr(z), b_ptr(z)) and receives four consecutive rows m..m+3 of
// one column n: epi(z, m, n, float4 sums)   with m % 4 == 0.
#pragma once
#include "ps_common.h"
#include "ps_split.h"

namespace ps {

constexpr int GEMM_XCDS = 8;
constexpr int GEMM_KS = 16;  // contraction indices per stage

struct GemmShape {
    int M, N, K;     // rows of an RC operand: a multiple of 8; K % 16 == 0 when an operand is KC
    int lda, ldb;
    int gx, gy, gz;  // tiles along M, along N, batch size
    int m_base, n_base;  // origin of the tile grid inside C (a launch may cover only part of C)
};

// Operand tiles are read with unconditional loads from addresses that are clamped into the operand, so the
// loop carries no branches and no 64-bit address arithmetic (uniform base + 32-bit offset): rows past the end
// repeat the last ones (they only reach rows or columns of C that are never stored); if K is not a multiple
// of 16 (RAGGED, RC operands only), a k past the end reads k = K-1 and is replaced by zeros.
template <int ROWS, bool KC, bool RAGGED>
struct GemmOperand {
    static_assert(KC ? !RAGGED : true, "KC operands come in whole stages");
    static constexpr int PIECES = ROWS * GEMM_KS / 8;  // of eight values each; at most one per thread
    static_assert(PIECES <= 256, "one piece per thread");
    // KC: the second k / 8 plane starts 64 bytes on, so that four rows of both planes fill all banks on a
    // write.  RC: 32-byte groups of 16 rows are exchanged by k % 4, so that the four k of a transposing
    // read lie in different banks.
    static constexpr int PLANE8 = ROWS * 16 + 64;                            // KC: bytes of one k / 8 plane
    static constexpr int PART = KC ? 2 * PLANE8 : GEMM_KS * ROWS * 2, BYTES = 3 * PART;
    static constexpr int SWAP = ROWS / 16 - 1 < 3 ? ROWS / 16 - 1 : 3;

    const float* base;
    uint32_t off, stage_step;  // float offset of this thread's piece in stage 0; floats between stages
    int k0, k_last, ld;        // RC: k of the piece in stage 0

    __device__ __forceinline__ void init(const float* b, int ld_, int row0, int nrows, int K, int tid)
    {
        const int f = min(tid, PIECES - 1);
        base = b;
        ld = ld_;
        k_last = K - 1;
        stage_step = KC ? GEMM_KS : GEMM_KS * ld;
        if (KC) {
            k0 = 0;
            off = (uint32_t)min(row0 + f / 2, nrows - 1) * ld + (f & 1) * 8;
        } else {
            k0 = f / (ROWS / 8);
            off = (uint32_t)min(row0 + f % (ROWS / 8) * 8, nrows - 8);
            if (!RAGGED) off += (uint32_t)k0 * ld;
        }
    }

    // Global -> registers for stage kt.
    __device__ __forceinline__ void load(int kt, floatx4 (&r)[2]) const
    {
        uint32_t o = off;
        bool inside = true;
        if (RAGGED) {
            const int k = kt * GEMM_KS + k0;
            inside = k <= k_last;
            o += (uint32_t)min(k, k_last) * ld;
        } else {
            o += (uint32_t)kt * stage_step;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            r[i] = *reinterpret_cast<const floatx4*>(base + o + 4 * i);
            if (RAGGED) r[i] = inside ? r[i] : floatx4{0.f, 0.f, 0.f, 0.f};
        }
    }

    static __device__ __forceinline__ void store(char* __restrict__ tile, int tid, const floatx4 (&r)[2])
    {
        const float v[8] = {r[0][0], r[0][1], r[0][2], r[0][3], r[1][0], r[1][1], r[1][2], r[1][3]};
        const Split8 s = split8(v);
        int at;
        if (KC) {
            at = (tid & 1) * PLANE8 + tid / 2 * 16;
        } else {
            const int k = tid / (ROWS / 8), r8 = tid % (ROWS / 8);
            at = k * ROWS * 2 + ((r8 / 2) ^ (k & SWAP)) * 32 + r8 % 2 * 16;
        }
        if (PIECES == 256 || tid < PIECES) {
#pragma unroll
            for (int i = 0; i < 3; ++i) *reinterpret_cast<uintx4*>(tile + i * PART + at) = s.p[i];
        }
    }

    // The operand of rows 32 * rt .. +31: lane (h, l32) gets k = 8h .. 8h + 7 of row l32.
    static __device__ __forceinline__ Split8 fetch(const char* __restrict__ tile, int rt, int lane)
    {
        Split8 s;
        if (KC) {
            const char* p = tile + (lane >> 5) * PLANE8 + (32 * rt + (lane & 31)) * 16;
#pragma unroll
            for (int i = 0; i < 3; ++i) s.p[i] = *reinterpret_cast<const uintx4*>(p + i * PART);
        } else {
            typedef short shortx4 __attribute__((ext_vector_type(4)));
            typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
            const int t = lane & 15, k = 8 * (lane >> 5) + (t >> 2), group = (2 * rt + (lane >> 4 & 1)) ^ ((t >> 2) & SWAP);
            const char* p = tile + k * ROWS * 2 + group * 32 + (t & 3) * 8;
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {  // k and k + 4
                    typedef __attribute__((address_space(3))) shortx4* LdsPtr;
                    const shortx4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsPtr)(shortx4*)(p + i * PART + j * 4 * ROWS * 2));
                    const uintx2 d = __builtin_bit_cast(uintx2, v);
                    s.p[i][2 * j] = d[0];
                    s.p[i][2 * j + 1] = d[1];
                }
        }
        return s;
    }
};

// One element of C with fp32 FMAs (see ps_split.h).
template <bool A_KC, bool B_KC>
__device__ __forceinline__ float gemm_plain(const GemmShape& sh, const float* __restrict__ A, const float* __restrict__ B, int m, int n)
{
    float sum = 0.f;
#pragma unroll 1
    for (int k = 0; k < sh.K; ++k)
        sum = fmaf(A[A_KC ? (size_t)m * sh.lda + k : (size_t)k * sh.lda + m], B[B_KC ? (size_t)n * sh.ldb + k : (size_t)k * sh.ldb + n], sum);
    return sum;
}

// Hands rows m .. m + 3 of column n to the epilogue.
template <bool A_KC, bool B_KC, class Epi>
__device__ __forceinline__ void gemm_store(const GemmShape& sh, const Epi& epi, int z, int m, int n, float v0, float v1, float v2, float v3)
{
    if (m >= sh.M || n >= sh.N) return;
    float4 v = make_float4(v0, v1, v2, v3);
    if (__builtin_isunordered(v0, v1) || __builtin_isunordered(v2, v3)) {
        const float* A = epi.a_ptr(z);
        const float* B = epi.b_ptr(z);
        v = make_float4(gemm_plain<A_KC, B_KC>(sh, A, B, m, n), gemm_plain<A_KC, B_KC>(sh, A, B, m + 1, n),
                        gemm_plain<A_KC, B_KC>(sh, A, B, m + 2, n), gemm_plain<A_KC, B_KC>(sh, A, B, m + 3, n));
    }
    epi(z, m, n, v);
}

// Stores one 32x32 tile of sums at (m0, n0): register i of lane (h, l32) is row 8*(i/4) + 4*h + i%4, column l32.
template <bool A_KC, bool B_KC, class Epi>
__device__ __forceinline__ void gemm_finish(const GemmShape& sh, const Epi& epi, int z, int m0, int n0, int lane, const floatx16& acc)
{
#pragma unroll
    for (int g = 0; g < 4; ++g)
        gemm_store<A_KC, B_KC>(sh, epi, z, m0 + 8 * g + 4 * (lane >> 5), n0 + (lane & 31), acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
}

// Tile configuration of one launch.
template <bool A_KC_, bool B_KC_, int TM_, int TN_, int WM_, int WN_, int AHEAD_>
struct GemmCfg {
    static constexpr bool A_KC = A_KC_, B_KC = B_KC_;
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, AHEAD = AHEAD_;
    static constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    static_assert(WM * WN == 4, "four wavefronts per block");
    static constexpr int STAGE = GemmOperand<BM, A_KC, false>::BYTES + GemmOperand<BN, B_KC, false>::BYTES;  // one of the two stage buffers
};

// Where block `block` of a launch over `total` tiles works: XCD x (= block number mod 8) walks a contiguous
// range of (z, y, x) triples.
__device__ __forceinline__ int gemm_tile(int block, int total)
{
    const int per_xcd = (total + GEMM_XCDS - 1) / GEMM_XCDS;
    return block % GEMM_XCDS * per_xcd + block / GEMM_XCDS;
}

// One block's tile: `block` of `sh.gx * sh.gy * sh.gz` (rounded up to the XCD count), stage buffers in lds.
// CHUNK > 0: the sum is formed as the sum, in order, of the sums over CHUNK stages each.  The order in which a
// value's products are added up depends on CHUNK alone, not on the tile shape.
template <class Cfg, bool RAGGED, int CHUNK, class Epi>
__device__ __forceinline__ void gemm_block(const GemmShape& sh, const Epi& epi, int block, char* __restrict__ lds)
{
    constexpr int TM = Cfg::TM, TN = Cfg::TN, WM = Cfg::WM, BM = Cfg::BM, BN = Cfg::BN;
    using OpA = GemmOperand<BM, Cfg::A_KC, RAGGED>;
    using OpB = GemmOperand<BN, Cfg::B_KC, RAGGED>;

    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int v = gemm_tile(block, sh.gx * sh.gy * sh.gz);
    if (v >= sh.gx * sh.gy * sh.gz) return;
    const int m0 = sh.m_base + (v % sh.gx) * BM, n0 = sh.n_base + (v / sh.gx % sh.gy) * BN, z = v / (sh.gx * sh.gy);

    SplitSum<floatx16> acc[TM][TN];
    floatx16 total[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            acc[a][b].clear();
            total[a][b] = acc[a][b].big;
        }

    // Pipeline: while the matrix cores consume stage kt out of one LDS buffer, stage kt + 1 is split and written
    // into the other, out of one of AHEAD register sets, which then takes the loads of stage kt + 1 + AHEAD.
    constexpr int AHEAD = Cfg::AHEAD;
    floatx4 ra[AHEAD][2], rb[AHEAD][2];
    const int nk = (sh.K + GEMM_KS - 1) / GEMM_KS;
    OpA opa;
    OpB opb;
    opa.init(epi.a_ptr(z), sh.lda, m0, sh.M, sh.K, tid);
    opb.init(epi.b_ptr(z), sh.ldb, n0, sh.N, sh.K, tid);
    {
        floatx4 ra0[2], rb0[2];
        opa.load(0, ra0);
        opb.load(0, rb0);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            opa.load(min(1 + i, nk - 1), ra[i]);
            opb.load(min(1 + i, nk - 1), rb[i]);
        }
        OpA::store(lds, tid, ra0);
        OpB::store(lds + OpA::BYTES, tid, rb0);
    }
    __syncthreads();

    static_assert(AHEAD % 2 == 0, "the LDS buffer of an unrolled stage is fixed");
    for (int kt0 = 0; kt0 < nk; kt0 += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int kt = kt0 + u;
            if (u > 0 && kt >= nk) break;
            const char* ta = lds + (u & 1) * Cfg::STAGE;
            char* na = lds + (~u & 1) * Cfg::STAGE;
            Split8 fa[TM], fb[TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) fa[a] = OpA::fetch(ta, wm * TM + a, lane);
#pragma unroll
            for (int b = 0; b < TN; ++b) fb[b] = OpB::fetch(ta + OpA::BYTES, wn * TN + b, lane);
            // unconditional on purpose (straight-line code): past the end the last stage is simply loaded and
            // stored again where nobody reads it
            OpA::store(na, tid, ra[u]);
            OpB::store(na + OpA::BYTES, tid, rb[u]);
            opa.load(min(kt + 1 + AHEAD, nk - 1), ra[u]);
            opb.load(min(kt + 1 + AHEAD, nk - 1), rb[u]);
#pragma unroll
            for (int t = 0; t <= SPLIT_SMALL; ++t)
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) acc[a][b].add(t, fa[a], fb[b]);
            if (CHUNK > 0 && (kt + 1) % (CHUNK > 0 ? CHUNK : 1) == 0) {
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        total[a][b] += acc[a][b].value();
                        acc[a][b].clear();
                    }
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
            gemm_finish<Cfg::A_KC, Cfg::B_KC>(sh, epi, z, m0 + (wm * TM + a) * 32, n0 + (wn * TN + b) * 32, lane, CHUNK > 0 ? total[a][b] : acc[a][b].value());
}

// The same sums for a launch with too few tiles to fill the chip: a block owns one 32x32 tile and its wavefronts
// one CHUNK of stages each, every wavefront with its operands straight from memory; the chunks' sums meet in
// LDS and are added up in order, so that a value is bit for bit what gemm_block<..., CHUNK> makes of it.
template <bool KC>
struct GemmLane {  // the operand rows of one lane
    const float* p;
    int ld;
    __device__ __forceinline__ void init(const float* b, int ld_, int row, int nrows, int lane)
    {
        ld = ld_;
        row = min(row, nrows - 1);
        p = KC ? b + (size_t)row * ld + 8 * (lane >> 5) : b + (size_t)(8 * (lane >> 5)) * ld + row;
    }
    __device__ __forceinline__ void load(int kt, float (&v)[8]) const
    {
        if (KC) {
            const floatx4* q = reinterpret_cast<const floatx4*>(p + (size_t)kt * GEMM_KS);
            const floatx4 a = q[0], b = q[1];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[j] = a[j];
                v[4 + j] = b[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[((size_t)kt * GEMM_KS + j) * ld];
        }
    }
};

template <bool A_KC, bool B_KC, int CHUNKS, int CHUNK, class Epi>
__global__ __launch_bounds__(64 * CHUNKS) void gemm_split_chunks(GemmShape sh, Epi epi)
{
    static_assert(CHUNKS >= 4, "four wavefronts store the tile");
    __shared__ float part[CHUNKS][16][64];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int t = gemm_tile(blockIdx.x, sh.gx * sh.gy * sh.gz);
    if (t >= sh.gx * sh.gy * sh.gz) return;
    const int m0 = t % sh.gx * 32, n0 = t / sh.gx % sh.gy * 32, z = t / (sh.gx * sh.gy);
    GemmLane<A_KC> la;
    GemmLane<B_KC> lb;
    la.init(epi.a_ptr(z), sh.lda, m0 + (lane & 31), sh.M, lane);
    lb.init(epi.b_ptr(z), sh.ldb, n0 + (lane & 31), sh.N, lane);
    SplitSum<floatx16> sum;
    sum.clear();
    const int k0 = wave * CHUNK;
    constexpr int AHEAD = 2;  // stages in flight
    float a[AHEAD][8], b[AHEAD][8];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
        la.load(k0 + i, a[i]);
        lb.load(k0 + i, b[i]);
    }
#pragma unroll
    for (int kt = 0; kt < CHUNK; ++kt) {
        const Split8 sa = split8(a[kt % AHEAD]), sb = split8(b[kt % AHEAD]);
        if (kt + AHEAD < CHUNK) {
            la.load(k0 + kt + AHEAD, a[kt % AHEAD]);
            lb.load(k0 + kt + AHEAD, b[kt % AHEAD]);
        }
        sum.add(sa, sb);
    }
    const floatx16 acc = sum.value();
#pragma unroll
    for (int i = 0; i < 16; ++i) part[wave][i][lane] = acc[i];
    __syncthreads();
    if (wave >= 4) return;
    float v[4];  // wavefront g stores rows 8g + 4h .. +3
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = part[0][4 * wave + i][lane];
#pragma unroll
        for (int c = 1; c < CHUNKS; ++c) v[i] += part[c][4 * wave + i][lane];
    }
    gemm_store<A_KC, B_KC>(sh, epi, z, m0 + 8 * wave + 4 * (lane >> 5), n0 + (lane & 31), v[0], v[1], v[2], v[3]);
}

constexpr int gemm_grid(const GemmShape& sh) { return (sh.gx * sh.gy * sh.gz + GEMM_XCDS - 1) / GEMM_XCDS * GEMM_XCDS; }

template <class Cfg, bool RAGGED, int CHUNK, int MINW, class Epi>
__global__ __launch_bounds__(256, MINW) void gemm_split(GemmShape sh, Epi epi)
{
    __shared__ __attribute__((aligned(16))) char lds[2 * Cfg::STAGE];
    gemm_block<Cfg, RAGGED, CHUNK>(sh, epi, blockIdx.x, lds);
}

// Two tile shapes in one launch: the first `main_blocks` blocks cover the main part of C with Main tiles,
// the rest cover an edge strip with Edge tiles.  The edge blocks are dispatched last and run next to the
// last main blocks instead of as a launch of their own behind them.
template <class Main, class Edge, bool RAGGED, int CHUNK, int MINW, class Epi>
__global__ __launch_bounds__(256, MINW) void gemm_split_edge(GemmShape sh_main, GemmShape sh_edge, int main_blocks, Epi epi)
{
    constexpr int STAGE = Main::STAGE > Edge::STAGE ? Main::STAGE : Edge::STAGE;
    __shared__ __attribute__((aligned(16))) char lds[2 * STAGE];
    if ((int)blockIdx.x < main_blocks)  // uniform over the block
        gemm_block<Main, RAGGED, CHUNK>(sh_main, epi, blockIdx.x, lds);
    else
        gemm_block<Edge, RAGGED, CHUNK>(sh_edge, epi, blockIdx.x - main_blocks, lds);
}

template <class Cfg>
GemmShape gemm_shape(int M, int N, int K, int lda, int ldb, int batch, int m_begin, int m_end, int n_begin, int n_end)
{
    return GemmShape{M, N, K, lda, ldb, (m_end - m_begin + Cfg::BM - 1) / Cfg::BM, (n_end - n_begin + Cfg::BN - 1) / Cfg::BN,
                     batch, m_begin, n_begin};
}

// One problem per batch index, all of C covered with Cfg tiles over a 1-D grid padded to a multiple of
// the XCD count.
template <class Cfg, int CHUNK, int MINW, class Epi>
void gemm_launch(int M, int N, int K, int lda, int ldb, int batch, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh = gemm_shape<Cfg>(M, N, K, lda, ldb, batch, 0, M, 0, N);
    constexpr bool CAN_BE_RAGGED = !Cfg::A_KC && !Cfg::B_KC;
    if (!CAN_BE_RAGGED || K % GEMM_KS == 0)
        hipLaunchKernelGGL((gemm_split<Cfg, false, CHUNK, MINW, Epi>), dim3(gemm_grid(sh)), dim3(256), 0, s, sh, epi);
    else
        hipLaunchKernelGGL((gemm_split<Cfg, CAN_BE_RAGGED, CHUNK, MINW, Epi>), dim3(gemm_grid(sh)), dim3(256), 0, s, sh, epi);
}

// One problem per batch index in 32x32 tiles, K = CHUNKS * CHUNK stages.
template <bool A_KC, bool B_KC, int CHUNKS, int CHUNK, class Epi>
void gemm_launch_chunks(int M, int N, int lda, int ldb, int batch, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh{M, N, CHUNKS * CHUNK * GEMM_KS, lda, ldb, (M + 31) / 32, (N + 31) / 32, batch, 0, 0};
    hipLaunchKernelGGL((gemm_split_chunks<A_KC, B_KC, CHUNKS, CHUNK, Epi>), dim3(gemm_grid(sh)), dim3(64 * CHUNKS), 0, s, sh, epi);
}

// Rows [0, m_split) x columns [0, n_split) of C with Main tiles and the rest with Edge tiles, where exactly
// one of the splits is inside C (the other equals M or N) and is a multiple of Main's tile: covering a
// ragged edge with narrow tiles avoids a mostly empty wide tile.
template <class Main, class Edge, int CHUNK, int MINW, class Epi>
void gemm_launch_edge(int M, int N, int K, int lda, int ldb, int batch, int m_split, int n_split, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh_main = gemm_shape<Main>(M, N, K, lda, ldb, batch, 0, m_split, 0, n_split);
    const GemmShape sh_edge = m_split < M ? gemm_shape<Edge>(M, N, K, lda, ldb, batch, m_split, M, 0, N)
                                          : gemm_shape<Edge>(M, N, K, lda, ldb, batch, 0, M, n_split, N);
    const int main_blocks = gemm_grid(sh_main), grid = main_blocks + gemm_grid(sh_edge);
    constexpr bool CAN_BE_RAGGED = !Main::A_KC && !Main::B_KC;
    if (!CAN_BE_RAGGED || K % GEMM_KS == 0)
        hipLaunchKernelGGL((gemm_split_edge<Main, Edge, false, CHUNK, MINW, Epi>), dim3(grid), dim3(256), 0, s, sh_main, sh_edge, main_blocks, epi);
    else
        hipLaunchKernelGGL((gemm_split_edge<Main, Edge, CAN_BE_RAGGED, CHUNK, MINW, Epi>), dim3(grid), dim3(256), 0, s, sh_main, sh_edge, main_blocks, epi);
}

}  // namespace ps
