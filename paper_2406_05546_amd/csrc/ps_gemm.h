// Batched fp32 GEMM on the gfx950 bf16 matrix cores with operands split in three (ps_split.h), used for the
// three contractions of the 1568 -> 512 fully connected layer (forward, input gradient, per-worker weight
// gradient).
//
//   C[m][n] = sum_k A(m,k) * B(n,k)        one problem per batch index z (= worker)
//
// Either operand may be stored k-contiguous ("KC": element (r,k) at base[r*ld + k]) or row-contiguous ("RC":
// element (r,k) at base[k*ld + r]).  A 256-thread block (4 wavefronts arranged WM x WN) owns a (WM*TM*32) x
// (WN*TN*32) tile of C; each wavefront owns TM x TN MFMA tiles of 32x32.  K advances 16 (or 32) at a time through
// double-buffered LDS: a thread loads four times four consecutive values (AHEAD + 1 stages ahead), splits them
// once and writes the parts, so that splitting costs 88 vector instructions per thread and stage next to the
// wavefront's 24 MFMAs.  The parts of a KC operand lie as [k / 8][row][8 k] and a lane's
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
constexpr int GEMM_K = 16;  // contraction indices of one MFMA; a stage has one or two of them

struct GemmShape {
    int M, N, K;     // rows of an RC operand: a multiple of 8; whole stages when an operand is KC
    int lda, ldb;
    int gx, gy, gz;  // tiles along M, along N, batch size
    int m_base, n_base;  // origin of the tile grid inside C (a launch may cover only part of C)
};

// Operand tiles are read with unconditional loads from addresses that are clamped into the operand, so the
// loop carries no branches and no 64-bit address arithmetic (uniform base + 32-bit offset): rows past the end
// repeat the last ones (they only reach rows or columns of C that are never stored); if K is not a multiple
// of a stage (RAGGED, RC operands only), a k past the end reads k = K-1 and is replaced by zeros.
// NT threads bring a stage of KS contraction indices in, four consecutive values at a time, and consecutive
// threads take consecutive ones: what a load instruction costs, where that is the limit, is the cache lines it
// touches, about 2.8 cycles each.
template <int ROWS, bool KC, bool RAGGED, int NT, int KS>
struct GemmOperand {
    static_assert(KC ? !RAGGED : true, "KC operands come in whole stages");
    static constexpr int N4 = ROWS * KS / 4, NV = (N4 + NT - 1) / NT;  // groups of four values, per stage and per thread
    // KC: a k / 8 plane starts 64 bytes past the rows of the one before, so that rows of two planes fill all banks
    // on a write.  RC: 32-byte groups of 16 rows are exchanged by k % 4, so that the four k of a transposing read
    // lie in different banks.
    static constexpr int PLANE8 = ROWS * 16 + 64;  // KC: bytes of one k / 8 plane
    static constexpr int PART = KC ? KS / 8 * PLANE8 : KS * ROWS * 2, BYTES = 3 * PART;
    static constexpr int SWAP = ROWS / 16 - 1 < 3 ? ROWS / 16 - 1 : 3;

    const float* base;
    uint32_t off[NV], stage_step;  // float offset of this thread's groups in stage 0; floats between stages
    int k0[NV], k_last, ld;        // RC: k of the groups in stage 0

    __device__ __forceinline__ void init(const float* b, int ld_, int row0, int nrows, int K, int t)
    {
        base = b;
        ld = ld_;
        k_last = K - 1;
        stage_step = KC ? KS : KS * ld;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int f = min(t + NT * i, N4 - 1);  // threads without a group repeat the last one
            if (KC) {
                k0[i] = 0;
                off[i] = (uint32_t)min(row0 + f / (KS / 4), nrows - 1) * ld + f % (KS / 4) * 4;
            } else {
                k0[i] = f / (ROWS / 4);
                off[i] = (uint32_t)min(row0 + f % (ROWS / 4) * 4, nrows - 4);
                if (!RAGGED) off[i] += (uint32_t)k0[i] * ld;
            }
        }
    }

    // Global -> registers for a stage that begins at k, anywhere.
    __device__ __forceinline__ void load_at(int k, floatx4 (&r)[NV]) const
    {
        static_assert(!RAGGED, "whole stages");
#pragma unroll
        for (int i = 0; i < NV; ++i) r[i] = *reinterpret_cast<const floatx4*>(base + (off[i] + (uint32_t)k * (KC ? 1 : ld)));
    }

    // Global -> registers for stage kt.
    __device__ __forceinline__ void load(int kt, floatx4 (&r)[NV]) const
    {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (RAGGED) {
                const int k = kt * KS + k0[i];
                const floatx4 v = *reinterpret_cast<const floatx4*>(base + (off[i] + (uint32_t)min(k, k_last) * ld));
                r[i] = k <= k_last ? v : floatx4{0.f, 0.f, 0.f, 0.f};
            } else {
                r[i] = *reinterpret_cast<const floatx4*>(base + (off[i] + (uint32_t)kt * stage_step));
            }
        }
    }

    static __device__ __forceinline__ void store(char* __restrict__ tile, int t, const floatx4 (&r)[NV])
    {
        typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int f = t + NT * i;
            uint32_t p[2][3];
            split2(r[i][0], r[i][1], p[0][0], p[0][1], p[0][2]);
            split2(r[i][2], r[i][3], p[1][0], p[1][1], p[1][2]);
            int at;
            if (KC) {
                at = f % (KS / 4) / 2 * PLANE8 + f / (KS / 4) * 16 + f % 2 * 8;
            } else {
                const int k = f / (ROWS / 4), r4 = f % (ROWS / 4);
                at = k * ROWS * 2 + ((r4 / 4) ^ (k & SWAP)) * 32 + r4 % 4 * 8;
            }
            if (NT * (i + 1) <= N4 || f < N4) {
#pragma unroll
                for (int j = 0; j < 3; ++j) *reinterpret_cast<uintx2*>(tile + j * PART + at) = uintx2{p[0][j], p[1][j]};
            }
        }
    }

    // The operand of rows 32 * rt .. +31 in the `sub`-th MFMA of the stage: lane (h, l32) gets k = 16 sub + 8h + 0..7 of
    // row l32.
    static __device__ __forceinline__ Split8 fetch(const char* __restrict__ tile, int rt, int sub, int lane)
    {
        Split8 s;
        if (KC) {
            const char* p = tile + (2 * sub + (lane >> 5)) * PLANE8 + (32 * rt + (lane & 31)) * 16;
#pragma unroll
            for (int i = 0; i < 3; ++i) s.p[i] = *reinterpret_cast<const uintx4*>(p + i * PART);
        } else {
            typedef short shortx4 __attribute__((ext_vector_type(4)));
            typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
            const int t = lane & 15, k = 16 * sub + 8 * (lane >> 5) + (t >> 2), group = (2 * rt + (lane >> 4 & 1)) ^ ((t >> 2) & SWAP);
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

// Four consecutive k of one row of an operand, from memory; zero past K (RC).
template <bool KC>
__device__ __forceinline__ floatx4 gemm_operand4(const float* __restrict__ base, int ld, int row, int k, int K)
{
    if (KC) return *reinterpret_cast<const floatx4*>(base + (size_t)row * ld + k);
    floatx4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x = base[(size_t)min(k + i, K - 1) * ld + row];
        v[i] = k + i < K ? x : 0.f;
    }
    return v;
}

// The sums `which` of a 32x32 tile at (m0, n0), for which the split does not hold (ps_split.h), formed again with fp32 matrix
// instructions, whose registers lie as those of the bf16 ones do.  Operands come straight from memory, so it takes
// about four times as long as the tile did, unless the sums turn out NaN anyway: a network of NaN weights is not
// slowed down by more than that first look.
// EARLY: 32 k ahead.  Tiny weights, forward of 2 x 32 66.2 -> 51.1 us, of 64 x 128 279 -> 267.  Not in gemm_block, whose launches
// that have nothing to form again it slows down: input gradient of 8 x 176 29.0 -> 30.4 us, of the whole range 5 to 16 x 65 to 512 3-5 %.
template <bool A_KC, bool B_KC, bool EARLY, class Epi>
__device__ __forceinline__ void gemm_again(const GemmShape& sh, const Epi& epi, int z, int m0, int n0, int lane, uint32_t which, floatx16& sums)
{
    lane = rarely(lane);
    const float* __restrict__ A = epi.a_ptr(z);
    const float* __restrict__ B = epi.b_ptr(z);
    const int row = min(m0 + (lane & 31), sh.M - 1), col = min(n0 + (lane & 31), sh.N - 1), h = lane >> 5;
    floatx16 again;
#pragma unroll
    for (int i = 0; i < 16; ++i) again[i] = 0.f;
    floatx4 a[4], b[4];  // of the next 32 k; past K, a multiple of 8 where an operand does not read as zero there, the last ones
    auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = (A_KC || B_KC ? min(k0 + 8 * i, sh.K - 8) : k0 + 8 * i) + 4 * h;
            a[i] = gemm_operand4<A_KC>(A, sh.lda, row, k, sh.K);
            b[i] = gemm_operand4<B_KC>(B, sh.ldb, col, k, sh.K);
        }
    };
    if (EARLY) load(0);
#pragma unroll 1
    for (int k0 = 0; k0 < sh.K; k0 += 32) {
        floatx4 x[4], y[4];
        if (EARLY) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[i] = a[i];
                y[i] = b[i];
            }
            load(k0 + 32);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (k0 + 8 * i >= sh.K) break;  // K is a multiple of 8, or the operands read as zero past it
            if (!EARLY) {
                x[i] = gemm_operand4<A_KC>(A, sh.lda, row, k0 + 8 * i + 4 * h, sh.K);
                y[i] = gemm_operand4<B_KC>(B, sh.ldb, col, k0 + 8 * i + 4 * h, sh.K);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) again = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][j], y[i][j], again, 0, 0, 0);
        }
        if (!worth_going_on<16>(which, again)) break;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
        if (which >> i & 1) sums[i] = again[i];
}

// Stores one 32x32 tile of sums at (m0, n0): register i of lane (h, l32) is row 8*(i/4) + 4*h + i%4, column l32.
template <bool A_KC, bool B_KC, bool EARLY, class Epi>
__device__ __forceinline__ void gemm_finish(const GemmShape& sh, const Epi& epi, int z, int m0, int n0, int lane, floatx16 sums)
{
    constexpr int G = A_KC || B_KC ? 4 : 16;  // as gemm_split_chunks looks at them, where that may have the same sums to form
    if (any_lost<16, G>(sums)) gemm_again<A_KC, B_KC, EARLY>(sh, epi, z, m0, n0, lane, lost_sums<16, G>(sums), sums);
    const int n = n0 + (lane & 31);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int m = m0 + 8 * g + 4 * (lane >> 5);
        if (m < sh.M && n < sh.N) epi(z, m, n, make_float4(sums[4 * g], sums[4 * g + 1], sums[4 * g + 2], sums[4 * g + 3]));
    }
}

// Tile configuration of one launch.
template <bool A_KC_, bool B_KC_, int TM_, int TN_, int WM_, int WN_, int AHEAD_, int KS_ = GEMM_K>
struct GemmCfg {
    static constexpr bool A_KC = A_KC_, B_KC = B_KC_;
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, AHEAD = AHEAD_, KS = KS_;
    static constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    static_assert(WM * WN == 4, "four wavefronts per block");
    static constexpr int STAGE = GemmOperand<BM, A_KC, false, 256, KS>::BYTES + GemmOperand<BN, B_KC, false, 256, KS>::BYTES;  // one of the two stage buffers
};

// Where block `block` of a launch over `total` tiles works: XCD x (= block number mod 8) walks a contiguous
// range of (z, y, x) triples.
__device__ __forceinline__ int gemm_tile(int block, int total)
{
    const int per_xcd = (total + GEMM_XCDS - 1) / GEMM_XCDS;
    return block % GEMM_XCDS * per_xcd + block / GEMM_XCDS;
}

// One block's tile: `block` of `sh.gx * sh.gy * sh.gz` (rounded up to the XCD count), stage buffers in lds.
// CHUNK > 0: the sum is formed as the sum, in order, of the sums over CHUNK stages each (KS = 16).  The order in which a
// value's products are added up depends on CHUNK alone, not on the tile shape.
template <class Cfg, bool RAGGED, int CHUNK, class Epi>
__device__ __forceinline__ void gemm_block(const GemmShape& sh, const Epi& epi, int block, char* __restrict__ lds)
{
    constexpr int TM = Cfg::TM, TN = Cfg::TN, WM = Cfg::WM, BM = Cfg::BM, BN = Cfg::BN, KS = Cfg::KS;
    // With tiles up to 64 wide the first two wavefronts bring in A and the others B.
    constexpr bool HALVES = BM <= 64 && BN <= 64;
    static_assert(CHUNK == 0 || KS == GEMM_K, "chunks are counted in MFMAs");
    using OpA = GemmOperand<BM, Cfg::A_KC, RAGGED, HALVES ? 128 : 256, KS>;
    using OpB = GemmOperand<BN, Cfg::B_KC, RAGGED, HALVES ? 128 : 256, KS>;

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
    static_assert(!HALVES || OpA::NV == OpB::NV, "one register set for either operand");
    floatx4 ra[AHEAD][OpA::NV], rb[HALVES ? 1 : AHEAD][OpB::NV];
    const int nk = (sh.K + KS - 1) / KS;
    const bool brings_b = HALVES && wave >= 2;
    OpA opa;
    OpB opb;
    opa.init(epi.a_ptr(z), sh.lda, m0, sh.M, sh.K, tid);
    opb.init(epi.b_ptr(z), sh.ldb, n0, sh.N, sh.K, HALVES ? tid & 127 : tid);
    auto load = [&](int kt, floatx4 (&a)[OpA::NV], floatx4 (&b)[OpB::NV]) {
        if (!brings_b) opa.load(kt, a);
        if constexpr (!HALVES)
            opb.load(kt, b);
        else if (brings_b)
            opb.load(kt, a);
    };
    auto store = [&](char* stage, const floatx4 (&a)[OpA::NV], const floatx4 (&b)[OpB::NV]) {
        if (!brings_b) OpA::store(stage, tid, a);
        if constexpr (!HALVES)
            OpB::store(stage + OpA::BYTES, tid, b);
        else if (brings_b)
            OpB::store(stage + OpA::BYTES, tid & 127, a);
    };
    {
        floatx4 ra0[OpA::NV], rb0[OpB::NV];
        load(0, ra0, rb0);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load(min(1 + i, nk - 1), ra[i], rb[HALVES ? 0 : i]);
        store(lds, ra0, rb0);
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
#pragma unroll
            for (int sub = 0; sub < KS / GEMM_K; ++sub) {
                Split8 fa[TM], fb[TN];
#pragma unroll
                for (int a = 0; a < TM; ++a) fa[a] = OpA::fetch(ta, wm * TM + a, sub, lane);
#pragma unroll
                for (int b = 0; b < TN; ++b) fb[b] = OpB::fetch(ta + OpA::BYTES, wn * TN + b, sub, lane);
                if (sub == 0) {
                    // unconditional on purpose (straight-line code): past the end the last stage is simply loaded
                    // and stored again where nobody reads it
                    store(na, ra[u], rb[HALVES ? 0 : u]);
                    load(min(kt + 1 + AHEAD, nk - 1), ra[u], rb[HALVES ? 0 : u]);
                }
#pragma unroll
                for (int t = 0; t <= SPLIT_SMALL; ++t)
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b) acc[a][b].add(t, fa[a], fb[b]);
            }
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
            gemm_finish<Cfg::A_KC, Cfg::B_KC, false>(sh, epi, z, m0 + (wm * TM + a) * 32, n0 + (wn * TN + b) * 32, lane, CHUNK > 0 ? total[a][b] : acc[a][b].value());
}

// One block's tile with eight wavefronts, two to a SIMD: four form the sum over the first half of the contraction, the others
// that over the rest, in one loop, and the sums meet in LDS.  For launches of up to one tile for a compute unit, which otherwise
// leave every SIMD a single wavefront and its waits (64 workers of 128 images: 87 -> 76 us).  The loop is bound by issue: a stage
// has about 100 vector instructions next to its 24 MFMAs, and the clock falls to 1.8-2.1 GHz under either.  The two fours
// taking turns, one multiplying out of registers while the other reads, splits and writes, is slower (91 us): reads, splits and
// writes after each other take 1,300 cycles of a SIMD to the products' 790.
template <class Cfg, class Epi>
__device__ __forceinline__ void gemm_sides_block(const GemmShape& sh, const Epi& epi, int block, char* __restrict__ lds)
{
    constexpr int TM = Cfg::TM, TN = Cfg::TN, WM = Cfg::WM, BM = Cfg::BM, BN = Cfg::BN, KS = Cfg::KS, AHEAD = Cfg::AHEAD;
    constexpr bool HALVES = BM <= 64 && BN <= 64;  // the first two wavefronts of a four bring in A and the others B
    using OpA = GemmOperand<BM, Cfg::A_KC, false, HALVES ? 128 : 256, KS>;
    using OpB = GemmOperand<BN, Cfg::B_KC, false, HALVES ? 128 : 256, KS>;
    static_assert(!HALVES || OpA::NV == OpB::NV, "one register set for either operand");
    static_assert(AHEAD % 2 == 0, "the LDS buffer of an unrolled stage is fixed");

    const int tid = threadIdx.x & 255, lane = tid & 63, wave = uniform(tid >> 6), half = uniform(threadIdx.x >> 8);
    const int wm = wave % WM, wn = wave / WM;
    const int v = gemm_tile(block, sh.gx * sh.gy * sh.gz);
    if (v >= sh.gx * sh.gy * sh.gz) return;
    const int m0 = sh.m_base + (v % sh.gx) * BM, n0 = sh.n_base + (v / sh.gx % sh.gy) * BN, z = v / (sh.gx * sh.gy);
    const int k_first = half * (sh.K / 2), nk = sh.K / (2 * KS);
    char* const stages = lds + half * 2 * Cfg::STAGE;

    SplitSum<floatx16> acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b].clear();

    floatx4 ra[AHEAD][OpA::NV], rb[HALVES ? 1 : AHEAD][OpB::NV];
    const bool brings_b = HALVES && wave >= 2;
    OpA opa;
    OpB opb;
    opa.init(epi.a_ptr(z), sh.lda, m0, sh.M, sh.K, HALVES ? tid & 127 : tid);
    opb.init(epi.b_ptr(z), sh.ldb, n0, sh.N, sh.K, HALVES ? tid & 127 : tid);
    auto load = [&](int kt, floatx4 (&a)[OpA::NV], floatx4 (&b)[OpB::NV]) {  // past the end the last stage again, which nobody reads
        const int k = k_first + min(kt, nk - 1) * KS;
        if (!brings_b) opa.load_at(k, a);
        if constexpr (!HALVES)
            opb.load_at(k, b);
        else if (brings_b)
            opb.load_at(k, a);
    };
    auto store = [&](char* stage, const floatx4 (&a)[OpA::NV], const floatx4 (&b)[OpB::NV]) {
        if (!brings_b) OpA::store(stage, HALVES ? tid & 127 : tid, a);
        if constexpr (!HALVES)
            OpB::store(stage + OpA::BYTES, tid, b);
        else if (brings_b)
            OpB::store(stage + OpA::BYTES, tid & 127, a);
    };
    {
        floatx4 ra0[OpA::NV], rb0[OpB::NV];
        load(0, ra0, rb0);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            __builtin_amdgcn_sched_barrier(0);  // in this order, or the loop waits for younger loads than it needs
            load(1 + i, ra[i], rb[HALVES ? 0 : i]);
        }
        __builtin_amdgcn_sched_barrier(0);
        store(stages, ra0, rb0);
    }
    __syncthreads();
    auto multiply = [&](int u, int kt) __attribute__((always_inline)) {
        const char* ta = stages + (u & 1) * Cfg::STAGE;
        char* na = stages + (~u & 1) * Cfg::STAGE;
#pragma unroll
        for (int sub = 0; sub < KS / GEMM_K; ++sub) {
            Split8 fa[TM], fb[TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) fa[a] = OpA::fetch(ta, wm * TM + a, sub, lane);
#pragma unroll
            for (int b = 0; b < TN; ++b) fb[b] = OpB::fetch(ta + OpA::BYTES, wn * TN + b, sub, lane);
            if (sub == 0) {
                store(na, ra[u], rb[HALVES ? 0 : u]);
                load(kt + 1 + AHEAD, ra[u], rb[HALVES ? 0 : u]);
            }
#pragma unroll
            for (int t = 0; t <= SPLIT_SMALL; ++t)
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) acc[a][b].add(t, fa[a], fb[b]);
        }
        __syncthreads();
    };
    int kt0 = 0;
    for (; kt0 + AHEAD <= nk; kt0 += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) multiply(u, kt0 + u);
    }
#pragma unroll
    for (int u = 0; u < AHEAD - 1; ++u) {
        if (kt0 + u >= nk) break;
        multiply(u, kt0 + u);
    }

    // The parts meet in LDS, in the place of the stages; each four finish half of a wavefront's tiles, or the first all of one.
    constexpr bool SHARED = TM % 2 == 0;
    typedef float Meet[2][4][SHARED ? TM / 2 : TM][TN][16][64];  // [for which four]
    static_assert(sizeof(Meet) <= 4 * Cfg::STAGE, "the sums fit where the stages were");
    Meet& meet = *reinterpret_cast<Meet*>(lds);
    auto finishes = [&](int a) { return SHARED ? (a >= TM / 2) == (half != 0) : half == 0; };
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            if (finishes(a)) continue;
            const floatx16 x = acc[a][b].value();
#pragma unroll
            for (int i = 0; i < 16; ++i) meet[!half][wave][SHARED ? a % (TM / 2) : a][b][i][lane] = x[i];
        }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            if (!finishes(a)) continue;
            floatx16 x = acc[a][b].value();
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] += meet[half][wave][SHARED ? a % (TM / 2) : a][b][i][lane];
            gemm_finish<Cfg::A_KC, Cfg::B_KC, true>(sh, epi, z, m0 + (wm * TM + a) * 32, n0 + (wn * TN + b) * 32, lane, x);
        }
}

// An operand that a wavefront brings for itself alone: 32 contraction indices at a time, straight to LDS as they are, and split
// on their way from there into the MFMA layout.  KC: a row of the stage is 128 bytes, whose 16-byte pieces are exchanged by bits
// 1-3 of the row, so that 16 rows read the same piece from different banks.  RC: one k is 128 bytes.
template <int ROWS, bool KC>
struct GemmOwnOperand {
    static constexpr int KS = 2 * GEMM_K, BYTES = ROWS * KS * 4, LOADS = BYTES / 1024;
    static_assert(KC || ROWS == 32, "a k of an RC operand is one line");
    Buffer buffer;
    uint32_t off[LOADS];  // of this lane's 16 bytes in stage 0
    uint32_t stage_step;

    __device__ __forceinline__ void init(const float* base, int ld, int row0, int nrows, int K, int k_first, int lane)
    {
        buffer = buffer_of(base, (uint32_t)(KC ? nrows : K) * ld * 4);
        stage_step = (KC ? KS : KS * ld) * 4;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int r = 8 * i + lane / 8, piece = KC ? lane % 8 ^ (r >> 1 & 7) : lane % 8;  // r: row, or k
            if (KC)
                off[i] = ((uint32_t)min(row0 + r, nrows - 1) * ld + k_first + 4 * piece) * 4;
            else
                off[i] = ((uint32_t)(k_first + r) * ld + min(row0 + 4 * piece, nrows - 4)) * 4;
        }
    }
    __device__ __forceinline__ void bring(int kt, char* tile) const
    {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) buffer_to_lds16(buffer, tile + 1024 * i, off[i] + (uint32_t)kt * stage_step);
    }
    // The operand of rows 32 * rt .. +31 in the `sub`-th MFMA of the stage: lane (h, l32) gets k = 16 sub + 8h + 0..7 of row l32.
    static __device__ __forceinline__ void read(const char* tile, int rt, int sub, int lane, float (&v)[8])
    {
        const int h = lane >> 5, l32 = lane & 31;
        if (KC) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const floatx4 x = *reinterpret_cast<const floatx4*>(tile + (32 * rt + l32) * 128 + ((4 * sub + 2 * h + i) ^ (l32 >> 1 & 7)) * 16);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[4 * i + j] = x[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float*>(tile + (16 * sub + 8 * h + j) * 128 + l32 * 4);
        }
    }
};

// The same sums for small batches: a block owns one tile of 32 x 32 NT and its wavefronts one CHUNK of MFMA steps each; the
// chunks' sums meet in LDS and are added up in order, so that a value is bit for bit what gemm_block<..., CHUNK> makes of it.
// A wavefront brings its operands to LDS of its own, 32 contraction indices at a time, so that a load touches whole cache
// lines (straight into the MFMA layout it touches 32, which took all of the 14 us of the forward pass of two workers of 32 images),
// and without a way through registers: next to matrix instructions of the other wavefronts of its SIMD a load into registers gets
// 32 bytes a cycle of a compute unit, one into LDS 64, and the parts need not be written to LDS.  Through registers and split
// before LDS, and so (us): forward 2 x 32 13.5 -> 11.7, 8 x 64 14.5 -> 12.6, 40 x 64 51 -> 39; input gradient 8.4 -> 7.8, 14.2 -> 12.5,
// 40 -> 37.  Two stages on their way are no faster (forward 2 x 32 12.2) and leave room for fewer blocks.
template <bool A_KC, bool B_KC, int NT, int CHUNKS, int CHUNK, class Epi>
__global__ __launch_bounds__(64 * CHUNKS, NT == 1 ? 4 : CHUNKS == 4 ? 3 : 2) void gemm_split_chunks(GemmShape sh, Epi epi)
{
    static_assert(CHUNKS >= 4 && NT <= 2, "four wavefronts store the tile");
    using OpA = GemmOwnOperand<32, A_KC>;
    using OpB = GemmOwnOperand<32 * NT, B_KC>;
    constexpr int SUBS = OpA::KS / GEMM_K, STAGES = CHUNK / SUBS;
    static_assert(CHUNK % SUBS == 0, "whole stages");
    __shared__ __attribute__((aligned(16))) union {
        char stage[CHUNKS][OpA::BYTES + OpB::BYTES];
        float part[CHUNKS][NT][16][64];
    } lds;
    __shared__ int lost[NT];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int t = gemm_tile(blockIdx.x, sh.gx * sh.gy * sh.gz);
    if (t >= sh.gx * sh.gy * sh.gz) return;
    if (threadIdx.x < NT) lost[threadIdx.x] = 0;
    const int m0 = t % sh.gx * 32, n0 = t / sh.gx % sh.gy * 32 * NT, z = t / (sh.gx * sh.gy);
    OpA opa;
    OpB opb;
    opa.init(epi.a_ptr(z), sh.lda, m0, sh.M, sh.K, wave * CHUNK * GEMM_K, lane);
    opb.init(epi.b_ptr(z), sh.ldb, n0, sh.N, sh.K, wave * CHUNK * GEMM_K, lane);
    char* const tile_a = lds.stage[wave];
    char* const tile_b = tile_a + OpA::BYTES;
    opa.bring(0, tile_a);
    opb.bring(0, tile_b);
    SplitSum<floatx16> sum[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) sum[i].clear();
#pragma unroll
    for (int kt = 0; kt < STAGES; ++kt) {
        float a[SUBS][8], b[SUBS][NT][8];
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stage is in LDS
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            OpA::read(tile_a, 0, sub, lane, a[sub]);
#pragma unroll
            for (int i = 0; i < NT; ++i) OpB::read(tile_b, i, sub, lane, b[sub][i]);
        }
        if (kt + 1 < STAGES) {
            // what comes straight to LDS does not wait for reads that are on their way
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            opa.bring(kt + 1, tile_a);
            opb.bring(kt + 1, tile_b);
        }
        __builtin_amdgcn_sched_barrier(0);  // the next stage is on its way before this one is split
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            const Split8 fa = split8(a[sub]);
            Split8 fb[NT];
#pragma unroll
            for (int i = 0; i < NT; ++i) fb[i] = split8(b[sub][i]);
#pragma unroll
            for (int t = 0; t <= SPLIT_SMALL; ++t)
#pragma unroll
                for (int i = 0; i < NT; ++i) sum[i].add(t, fa, fb[i]);
        }
        __builtin_amdgcn_sched_barrier(0);  // and is not waited for in front of that
    }
    __syncthreads();  // everybody has read its stages, whose place the sums take
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const floatx16 acc = sum[j].value();
#pragma unroll
        for (int i = 0; i < 16; ++i) lds.part[wave][j][i][lane] = acc[i];
    }
    __syncthreads();
    floatx4 v[NT];  // wavefront g stores rows 8g + 4h .. +3
    if (wave < 4) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[j][i] = lds.part[0][j][4 * wave + i][lane];
#pragma unroll
                for (int c = 1; c < CHUNKS; ++c) v[j][i] += lds.part[c][j][4 * wave + i][lane];
            }
            if (any_lost<4, 4>(v[j])) lost[j] = 1;
        }
    }
    __syncthreads();
    int again[NT], redo = 0;
#pragma unroll
    for (int j = 0; j < NT; ++j) redo |= again[j] = uniform(lost[j]);
    if (__builtin_expect(redo, 0)) {  // a tile's lost sums are formed again by one wavefront for all four
        uint32_t(*which)[4][64] = reinterpret_cast<uint32_t(*)[4][64]>(lds.part[1]);
        float(*sums)[16][64] = lds.part[0];
        if (wave < 4) {
#pragma unroll
            for (int j = 0; j < NT; ++j) which[j][wave][lane] = lost_sums<4, 4>(v[j]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (!again[j] || wave != j) continue;
            uint32_t all = 0;
#pragma unroll
            for (int g = 0; g < 4; ++g) all |= which[j][g][lane] << (4 * g);
            floatx16 x;
            gemm_again<A_KC, B_KC, true>(sh, epi, z, m0, n0 + 32 * j, lane, all, x);
#pragma unroll
            for (int i = 0; i < 16; ++i) sums[j][i][lane] = x[i];
        }
        __syncthreads();
        if (wave < 4) {
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (which[j][wave][lane] >> i & 1) v[j][i] = sums[j][4 * wave + i][lane];
        }
    }
    if (wave >= 4) return;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int m = m0 + 8 * wave + 4 * (lane >> 5), n = n0 + 32 * j + (lane & 31);
        if (m < sh.M && n < sh.N) epi(z, m, n, make_float4(v[j][0], v[j][1], v[j][2], v[j][3]));
    }
}

// The same sums for a launch with so few tiles that its time is that of one block's serial loop over K: for each of PARTS
// halves of the contraction (or all of it, the sums of gemm_block<..., 0>) T x T wavefronts that do nothing but multiply, a tile of
// 32 x 32 each, and four T that bring their operands in and split them, 32 contraction indices at a time.  (A last stage of fewer
// begins earlier instead, and what comes twice is passed over.)  Bound by the chain of the five small terms of a step, each of which
// waits 66 cycles for the one before, 330 to a step of 16, and up to 200 more where splits are issued on the same SIMD.
// Forward of one worker of 256 images or four of 128: 64 x 64 tiles, whose wavefronts do everything, 38 us, in one part 24, in
// two 18.  Input gradient, one part, of one of 100 15.4 -> 9.4 us, of two 15.4 -> 16.3.  T = 2, a multiplying wavefront on each
// SIMD, input gradient of two of 100 to one of 512 16.6 -> 13.4 us, of one of 640 and five of 128 17.3 -> 14.3 (events included; with four that bring 15.2, and two such
// blocks to a compute unit, eight of 128, 25.6 against 21.3 in 64 x 64 tiles).  In two parts there is room for four of them to a part
// only: forward of five to ten of 128 32.4 against 26.4 us side by side.
constexpr int roles_bring(int T) { return 4 * T; }  // wavefronts of a part that bring operands; T * T multiply
template <bool A_KC, bool B_KC, int PARTS, int T, class Epi>
__global__ __launch_bounds__(64 * PARTS * (T * T + roles_bring(T))) void gemm_split_roles(GemmShape sh, Epi epi)
{
    constexpr int KS = 2 * GEMM_K, SUBS = KS / GEMM_K, AHEAD = 4;  // stages on their way in registers
    constexpr int MULT = T * T, BRING = roles_bring(T), NT = 64 * BRING / 2;
    static_assert(T == 1 || (T == 2 && PARTS == 1), "the parts of one tile meet");
    using OpA = GemmOperand<32 * T, A_KC, false, NT, KS>;
    using OpB = GemmOperand<32 * T, B_KC, false, NT, KS>;
    constexpr int STAGE = OpA::BYTES + OpB::BYTES;
    static_assert(OpA::NV == OpB::NV, "one register set for either operand");
    __shared__ __attribute__((aligned(16))) char lds[PARTS][3 * STAGE];
    __shared__ float meet[PARTS][16][64];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int v = gemm_tile(blockIdx.x, sh.gx * sh.gy * sh.gz);
    if (v >= sh.gx * sh.gy * sh.gz) return;
    const int m0 = v % sh.gx * (32 * T), n0 = v / sh.gx % sh.gy * (32 * T), z = v / (sh.gx * sh.gy);
    const bool multiplies = wave < PARTS * MULT;
    const int half = multiplies ? wave / MULT : (int)((uint32_t)(wave - PARTS * MULT) / BRING);
    const int bringer = (wave - PARTS * MULT) & (BRING - 1), t = (64 * bringer + lane) & (NT - 1);
    const int mt = wave & (T - 1), nt = wave / T & (T - 1);  // tile of a multiplying wavefront
    const int K = sh.K / PARTS, k_first = half * K, nk = (K + KS - 1) / KS, tail = (nk * KS - K) / GEMM_K;  // MFMA steps that the last stage repeats

    // While stage kt is multiplied, out of one buffer, stage kt + 1 lies in the second and stage kt + 2 comes into the
    // third: the multiplying wavefront reads one MFMA step ahead, also from one stage into the next.
    // The two kinds of wavefronts run loops of their own: the same barriers (nk + 1, and one behind), but in a common loop
    // the compiler would wait for every load in flight where their ways meet.
    char *now = lds[half], *next = now + STAGE, *later = now + 2 * STAGE;
    auto turn = [&]() __attribute__((always_inline)) {
        char* const read = now;
        now = next;
        next = later;
        later = read;
    };
    if (!multiplies) {
        const bool brings_b = bringer >= BRING / 2;
        OpA opa;
        OpB opb;
        if (brings_b)
            opb.init(epi.b_ptr(z), sh.ldb, n0, sh.N, sh.K, t);
        else
            opa.init(epi.a_ptr(z), sh.lda, m0, sh.M, sh.K, t);
        auto load = [&](int kt, floatx4 (&x)[OpA::NV]) {  // past the end the last stage again, which nobody reads
            const int k = k_first + min(kt * KS, K - KS);
            if (brings_b)
                opb.load_at(k, x);
            else
                opa.load_at(k, x);
        };
        auto store = [&](char* stage, const floatx4 (&x)[OpA::NV]) {
            if (brings_b)
                OpB::store(stage + OpA::BYTES, t, x);
            else
                OpA::store(stage, t, x);
        };
        floatx4 r[AHEAD][OpA::NV];  // stage kt + 2 .. kt + 1 + AHEAD; stage s in r[s % AHEAD]
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            load(i, r[i]);
            __builtin_amdgcn_sched_barrier(0);  // in this order
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            store(i ? next : now, r[i]);
            load(AHEAD + i, r[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        auto stage = [&](int u, int kt) __attribute__((always_inline)) {
            store(later, r[(u + 2) % AHEAD]);
            load(kt + 2 + AHEAD, r[(u + 2) % AHEAD]);
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);  // or the next stages are split, and so waited for, up here
            turn();
        };
        int kt0 = 0;
        for (; kt0 + AHEAD <= nk; kt0 += AHEAD) {
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) stage(u, kt0 + u);
        }
#pragma unroll
        for (int u = 0; u < AHEAD - 1; ++u) {
            if (kt0 + u >= nk) break;
            stage(u, kt0 + u);
        }
        __syncthreads();
        return;
    }
    __syncthreads();

    SplitSum<floatx16> acc;
    acc.clear();
    Split8 fa, fb;
    auto fetch = [&](const char* stage, int sub) {
        fa = OpA::fetch(stage, mt, sub, lane);
        fb = OpB::fetch(stage + OpA::BYTES, nt, sub, lane);
    };
    fetch(now, nk == 1 ? tail : 0);
    for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
        for (int sub = 0; sub < SUBS; ++sub) {
            if (kt == nk - 1 && sub < tail) continue;
            const Split8 a = fa, b = fb;
            if (sub + 1 < SUBS)
                fetch(now, sub + 1);
            else
                fetch(next, kt + 2 == nk ? tail : 0);
            acc.add(a, b);
        }
        __syncthreads();
        turn();
    }
    floatx16 sums = acc.value();
    if (half > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) meet[half][i][lane] = sums[i];
    }
    __syncthreads();
    if (half > 0) return;
#pragma unroll
    for (int p = 1; p < PARTS; ++p)
#pragma unroll
        for (int i = 0; i < 16; ++i) sums[i] += meet[p][i][lane];
    gemm_finish<A_KC, B_KC, true>(sh, epi, z, m0 + 32 * mt, n0 + 32 * nt, lane, sums);
}

// Whether a launch over this many 128 x 128 tiles leaves compute units idle.
inline bool gemm_few_tiles(int wide_tiles, int compute_units) { return wide_tiles < compute_units; }

constexpr int gemm_grid(const GemmShape& sh) { return (sh.gx * sh.gy * sh.gz + GEMM_XCDS - 1) / GEMM_XCDS * GEMM_XCDS; }

template <class Cfg, int CHUNK, int MINW, class Epi>
__global__ __launch_bounds__(256, MINW) void gemm_split(GemmShape sh, Epi epi)
{
    __shared__ __attribute__((aligned(16))) char lds[2 * Cfg::STAGE];
    gemm_block<Cfg, false, CHUNK>(sh, epi, blockIdx.x, lds);
}

template <class Cfg, class Epi>
__global__ __launch_bounds__(512, 2) void gemm_split_sides(GemmShape sh, Epi epi)
{
    __shared__ __attribute__((aligned(16))) char lds[4 * Cfg::STAGE];
    gemm_sides_block<Cfg>(sh, epi, blockIdx.x, lds);
}

// The same sums for launches of many tiles: four wavefronts to a block, two blocks to a compute unit, which need not keep in
// step, one half after the other.  The first half's sums, 64 a lane, wait in LDS (28) and in registers (36), for which loads run
// one stage ahead instead of two.  256 workers of 256 images 528 us (28, 20 and the rest in the tile's own place in C 4 us more, all
// of them there 37 more; gemm_sides_block 60 more).
template <class Cfg, class Epi>
__global__ __launch_bounds__(256, 2) void gemm_split_parts(GemmShape sh, Epi epi)
{
    constexpr int TM = Cfg::TM, TN = Cfg::TN, WM = Cfg::WM, BM = Cfg::BM, BN = Cfg::BN, KS = Cfg::KS;
    using OpA = GemmOperand<BM, Cfg::A_KC, false, 256, KS>;
    using OpB = GemmOperand<BN, Cfg::B_KC, false, 256, KS>;
    static_assert(KS == GEMM_K, "one MFMA step to a stage");
    constexpr int GROUPS = TM * TN * 4, IN_LDS = 7, IN_REGS = GROUPS - IN_LDS;  // groups of four sums: where those of the first part wait
    __shared__ __attribute__((aligned(16))) char lds[2 * Cfg::STAGE];
    __shared__ floatx4 waiting[IN_LDS][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6), wm = wave % WM, wn = wave / WM;
    const int v = gemm_tile(blockIdx.x, sh.gx * sh.gy * sh.gz);
    if (v >= sh.gx * sh.gy * sh.gz) return;
    const int m0 = v % sh.gx * BM, n0 = v / sh.gx % sh.gy * BN, z = v / (sh.gx * sh.gy), nk = sh.K / KS;
    OpA opa;
    OpB opb;
    opa.init(epi.a_ptr(z), sh.lda, m0, sh.M, sh.K, tid);
    opb.init(epi.b_ptr(z), sh.ldb, n0, sh.N, sh.K, tid);
    SplitSum<floatx16> acc[TM][TN];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) acc[a][b].clear();
    };
    clear();
    floatx4 held[IN_REGS] = {};
    floatx4 ra[OpA::NV], rb[OpB::NV];  // of the stage after the next
    {
        floatx4 ra0[OpA::NV], rb0[OpB::NV];
        opa.load(0, ra0);
        opb.load(0, rb0);
        opa.load(min(1, nk - 1), ra);
        opb.load(min(1, nk - 1), rb);
        OpA::store(lds, tid, ra0);
        OpB::store(lds + OpA::BYTES, tid, rb0);
    }
    __syncthreads();
    for (int kt0 = 0; kt0 < nk; kt0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int kt = kt0 + u;
            if (u > 0 && kt >= nk) break;
            const char* ta = lds + (u & 1) * Cfg::STAGE;
            char* na = lds + (~u & 1) * Cfg::STAGE;
            Split8 fa[TM], fb[TN];
#pragma unroll
            for (int a = 0; a < TM; ++a) fa[a] = OpA::fetch(ta, wm * TM + a, 0, lane);
#pragma unroll
            for (int b = 0; b < TN; ++b) fb[b] = OpB::fetch(ta + OpA::BYTES, wn * TN + b, 0, lane);
            OpA::store(na, tid, ra);
            OpB::store(na + OpA::BYTES, tid, rb);
            opa.load(min(kt + 2, nk - 1), ra);
            opb.load(min(kt + 2, nk - 1), rb);
#pragma unroll
            for (int t = 0; t <= SPLIT_SMALL; ++t)
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) acc[a][b].add(t, fa[a], fb[b]);
            __syncthreads();
            if (u == 0 && __builtin_expect(kt == nk / 2 - 1, 0)) {  // the first part is done
#pragma unroll
                for (int i = 0; i < GROUPS; ++i) {
                    const int a = i / (4 * TN), b = i / 4 % TN, g = i % 4;
                    const SplitSum<floatx16>& x = acc[a][b];
                    const floatx4 first = {x.big[4 * g] + x.small[4 * g], x.big[4 * g + 1] + x.small[4 * g + 1], x.big[4 * g + 2] + x.small[4 * g + 2],
                                           x.big[4 * g + 3] + x.small[4 * g + 3]};
                    if (i < IN_LDS)
                        waiting[i][tid] = first;
                    else
                        held[i - IN_LDS] = first;
                }
                clear();
            }
        }
    }
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) {
            floatx16 x = acc[a][b].value();
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const floatx4 first = (a * TN + b) * 4 + g < IN_LDS ? waiting[(a * TN + b) * 4 + g][tid] : held[(a * TN + b) * 4 + g - IN_LDS];
#pragma unroll
                for (int k = 0; k < 4; ++k) x[4 * g + k] += first[k];
            }
            gemm_finish<Cfg::A_KC, Cfg::B_KC, true>(sh, epi, z, m0 + (wm * TM + a) * 32, n0 + (wn * TN + b) * 32, lane, x);
        }
}

// Two tile shapes in one launch: `main_blocks` blocks cover the main part of C with Main tiles, the rest cover an
// edge strip with Edge tiles.  The edge blocks are dispatched last and run next to the last main blocks instead of
// as a launch of their own behind them; or, with MIXED, evenly among the main blocks, a block for every XCD at a time.
// Blocks of one shape all reach their stores at the same time, over and over: where those make up a fifth of a
// tile's time, the shorter blocks among them put the compute units out of step and the stores of some run under the
// products of others (fc1 weight gradient, 256 workers of 256 images: 0.77 -> 0.68 ms; nothing stored at all 0.61).
// The input gradient stores half as much per product and loses more at the end than it wins (0.607 -> 0.621).
template <class Main, class Edge, bool RAGGED, bool MIXED, int CHUNK, int MINW, class Epi>
__global__ __launch_bounds__(256, MINW) void gemm_split_edge(GemmShape sh_main, GemmShape sh_edge, int main_blocks, Epi epi)
{
    static_assert(Main::KS == Edge::KS, "one stage for both tile shapes");
    constexpr int STAGE = Main::STAGE > Edge::STAGE ? Main::STAGE : Edge::STAGE;
    __shared__ __attribute__((aligned(16))) char lds[2 * STAGE];
    int block = blockIdx.x;
    bool main = block < main_blocks;  // uniform over the block
    if (MIXED) {  // of every `period` groups of blocks the first is an edge group, until there are none left
        const int group = block / GEMM_XCDS, edge_groups = (gridDim.x - main_blocks) / GEMM_XCDS, period = gridDim.x / (gridDim.x - main_blocks);
        main = group % period != 0 || group / period >= edge_groups;
        block -= GEMM_XCDS * (main ? min(edge_groups, group / period + 1) : group - group / period);
    } else if (!main) {
        block -= main_blocks;
    }
    if (main)
        gemm_block<Main, RAGGED, CHUNK>(sh_main, epi, block, lds);
    else
        gemm_block<Edge, RAGGED, CHUNK>(sh_edge, epi, block, lds);
}

template <class Cfg>
GemmShape gemm_shape(int M, int N, int K, int lda, int ldb, int batch, int m_begin, int m_end, int n_begin, int n_end)
{
    return GemmShape{M, N, K, lda, ldb, (m_end - m_begin + Cfg::BM - 1) / Cfg::BM, (n_end - n_begin + Cfg::BN - 1) / Cfg::BN,
                     batch, m_begin, n_begin};
}

// One problem per batch index (K in whole stages), all of C covered with Cfg tiles over a 1-D grid padded to a
// multiple of the XCD count.
template <class Cfg, int CHUNK, int MINW, class Epi>
void gemm_launch(int M, int N, int K, int lda, int ldb, int batch, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh = gemm_shape<Cfg>(M, N, K, lda, ldb, batch, 0, M, 0, N);
    hipLaunchKernelGGL((gemm_split<Cfg, CHUNK, MINW, Epi>), dim3(gemm_grid(sh)), dim3(256), 0, s, sh, epi);
}

template <class Cfg, class Epi>
void gemm_launch_sides(int M, int N, int K, int lda, int ldb, int batch, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh = gemm_shape<Cfg>(M, N, K, lda, ldb, batch, 0, M, 0, N);
    hipLaunchKernelGGL((gemm_split_sides<Cfg, Epi>), dim3(gemm_grid(sh)), dim3(512), 0, s, sh, epi);
}

template <class Cfg, int K, class Epi>
void gemm_launch_parts(int M, int N, int lda, int ldb, int batch, const Epi& epi, hipStream_t s)
{
    static_assert(K % (4 * Cfg::KS) == 2 * Cfg::KS, "the first half's last stage is an even one");
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh = gemm_shape<Cfg>(M, N, K, lda, ldb, batch, 0, M, 0, N);
    hipLaunchKernelGGL((gemm_split_parts<Cfg, Epi>), dim3(gemm_grid(sh)), dim3(256), 0, s, sh, epi);
}

// Whether every tile of 32 T x 32 T finds a compute unit of its own (both sides measured: gemm_split_roles).
template <int T>
bool gemm_roles_fit(int M, int N, int batch, int compute_units)
{
    return (M + 32 * T - 1) / (32 * T) * ((N + 32 * T - 1) / (32 * T)) * batch <= compute_units;
}

// K / PARTS: at least 32, a multiple of 16.
template <bool A_KC, bool B_KC, int PARTS, int T, class Epi>
void gemm_launch_roles(int M, int N, int K, int lda, int ldb, int batch, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh{M, N, K, lda, ldb, (M + 32 * T - 1) / (32 * T), (N + 32 * T - 1) / (32 * T), batch, 0, 0};
    hipLaunchKernelGGL((gemm_split_roles<A_KC, B_KC, PARTS, T, Epi>), dim3(gemm_grid(sh)), dim3(64 * PARTS * (T * T + roles_bring(T))), 0, s, sh, epi);
}

// One problem per batch index in tiles of 32 x 32 (narrow) or 32 x 64; K = CHUNKS * CHUNK MFMA steps.
template <bool A_KC, bool B_KC, int CHUNKS, int CHUNK, class Epi>
void gemm_launch_chunks(int M, int N, int lda, int ldb, int batch, bool narrow, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh{M, N, CHUNKS * CHUNK * GEMM_K, lda, ldb, (M + 31) / 32, narrow ? (N + 31) / 32 : (N + 63) / 64, batch, 0, 0};
    auto kernel = narrow ? gemm_split_chunks<A_KC, B_KC, 1, CHUNKS, CHUNK, Epi> : gemm_split_chunks<A_KC, B_KC, 2, CHUNKS, CHUNK, Epi>;
    hipLaunchKernelGGL(kernel, dim3(gemm_grid(sh)), dim3(64 * CHUNKS), 0, s, sh, epi);
}

// Rows [0, m_split) x columns [0, n_split) of C with Main tiles and the rest with Edge tiles, where exactly
// one of the splits is inside C (the other equals M or N) and is a multiple of Main's tile: covering a
// ragged edge with narrow tiles avoids a mostly empty wide tile.
template <class Main, class Edge, bool MIXED, int CHUNK, int MINW, class Epi>
void gemm_launch_edge(int M, int N, int K, int lda, int ldb, int batch, int m_split, int n_split, const Epi& epi, hipStream_t s)
{
    if (M <= 0 || N <= 0 || batch <= 0) return;
    const GemmShape sh_main = gemm_shape<Main>(M, N, K, lda, ldb, batch, 0, m_split, 0, n_split);
    const GemmShape sh_edge = m_split < M ? gemm_shape<Edge>(M, N, K, lda, ldb, batch, m_split, M, 0, N)
                                          : gemm_shape<Edge>(M, N, K, lda, ldb, batch, 0, M, n_split, N);
    const int main_blocks = gemm_grid(sh_main), grid = main_blocks + gemm_grid(sh_edge);
    constexpr bool CAN_BE_RAGGED = !Main::A_KC && !Main::B_KC;
    if (!CAN_BE_RAGGED || K % Main::KS == 0)
        hipLaunchKernelGGL((gemm_split_edge<Main, Edge, false, MIXED, CHUNK, MINW, Epi>), dim3(grid), dim3(256), 0, s, sh_main, sh_edge, main_blocks, epi);
    else
        hipLaunchKernelGGL((gemm_split_edge<Main, Edge, CAN_BE_RAGGED, MIXED, CHUNK, MINW, Epi>), dim3(grid), dim3(256), 0, s, sh_main, sh_edge, main_blocks, epi);
}

}  // namespace ps
