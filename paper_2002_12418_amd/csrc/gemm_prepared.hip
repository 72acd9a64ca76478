// Pointwise layers and Winograd products with weights prepared as bf16 parts in operand order (parts and terms as in gemm_split.hip).
//
// gemm_split.hip and gemm_short.hip cut both operands into parts anew for every tile, the weights among them, which never change: half of their vector
// instructions, and in the staged tiles half of what goes through LDS.  Here the weights go from the L2 straight to the registers that the matrix instruction
// reads, 16 bytes per lane and load, one step ahead; only the columns are cut.  What bounds it then: 64 x 64 and 128 x 64 tiles the bytes of
// both operands that a CU takes from the L2 (some 30 per clock), large ones the matrix cores.
// Measured against the best of those two, us (images x plane, channels): 16 x 28 x 28 512 -> 256 31.6 -> 25.4, 32 x 14 x 15 1024 -> 512 57.7 -> 46.3,
// 4 x 27 x 28 1024 -> 1024 48.3 -> 43.6, one of 56 x 56 512 -> 512 18.7 -> 16.6, 16 x 28 x 28 256 -> 256 19.3 -> 15.4, 8 x 28 x 28 128 -> 256 7.6 -> 7.0,
// 16 x 13 x 13 1024 -> 195 17.3 -> 15.8; divided, 8 x 27 x 29 96 -> 130 6.5 -> 5.4, 16 x 7 x 7 512 -> 1024 12.4 -> 11.8.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels.hpp"
#include "lds_barrier.hpp"
#include "xcd_remap.hpp"
#include "gemm_epilogue.hpp"
#include "bf16_parts.hpp"
#include "fast_div.hpp"

namespace mnnconv {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

// Weights: blocks of 32 rows and 16 reduction rows, as conv_patch.hip prepares them for one tap
struct PreparedArgs {
    int tilesM, tilesN, total;
    unsigned a_bytes, b_bytes;
    int blocks, steps;           // 32-row blocks of the weights; steps of 16 reduction rows
    int vecD;
    ConstDiv by_l, by_tm, by_tiles;
};

__device__ __forceinline__ void* parts_of(const GemmProblem& p, const PreparedArgs& g, int b) { return static_cast<char*>(const_cast<void*>(p.a_parts)) + (long long)b * g.a_bytes; }

// Products of parts: six of three parts (fp32), three of two ("bf16x3", gemm_split.hip)
template <int NP> struct Terms;
template <> struct Terms<3> { static constexpr int end = 6, pa[6] = {1, 1, 0, 2, 0, 0}, pb[6] = {1, 0, 1, 0, 2, 0}; };
template <> struct Terms<2> { static constexpr int end = 3, pa[3] = {1, 0, 0}, pb[3] = {0, 1, 0}; };

// LDS slot of a column: a lane holds two of them and writes one at a time, a matrix operand is 32 in a row; both spread over all banks
template <int BN>
__device__ __forceinline__ int column_slot(int col) { return (col & 1) * (BN / 2) + ((col >> 1) ^ ((col & 1) << 3)); }

// BATCH: Winograd products, one per position; a pointwise layer is spared the division.
// Columns staged in LDS, two buffers, one barrier per chunk: planes of an even size (pairs of columns, aligned to 4 bytes).  RAGGED: a reduction that is no multiple of 8.
template <int BM, int BN, int WM, int WN, bool RAGGED, bool BATCH, int NP>
__global__ __launch_bounds__(WM * WN * 64, 2) void gemm_prepared_kernel(GemmProblem p, PreparedArgs g)
{
    constexpr int NW = WM * WN, THREADS = NW * 64;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int KG = THREADS * 2 / BN, BK = KG * 8, KS = BK / 16;      // a lane stages eight rows of two columns
    constexpr int GROUP = BN * 16, BUF = NP * KG * GROUP;
    constexpr int EPI = NW * kStageFloats * 4;
    __shared__ __attribute__((aligned(16))) char smem[2 * BUF > EPI ? 2 * BUF : EPI];
    __shared__ int wave_lost[NW];
    unsigned lost = 0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lrow = lane >> 5, lcol = lane & 31;

    const int wg = (int)xcd_contiguous(blockIdx.x, (unsigned)g.total);
    const int b = BATCH ? (int)const_div((unsigned)wg, g.by_tiles) : 0, tile = wg - b * (g.tilesM * g.tilesN);
    const int tn = (int)const_div((unsigned)tile, g.by_tm), tm = tile - tn * g.tilesM;
    const int m0 = tm * BM, n0 = tn * BN;

    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(parts_of(p, g, b), 0, (int)g.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.B) + b * p.strideB_batch, 0, (int)g.b_bytes, 0x00020000);

    auto column = [&](int col) -> unsigned {             // byte offset in row 0, or kOutsideBytes
        const int img = (int)const_div((unsigned)col, g.by_l), rest = col - img * p.L;
        return col < p.Ncols ? (unsigned)(img * (int)p.strideB_img + rest) * 4u : kOutsideBytes;
    };

    // ---- staging
    const unsigned row_bytes = (unsigned)p.strideB_row * 4u;
    const int pair = tid % (BN / 2), grp = tid / (BN / 2);
    const unsigned base = column(n0 + 2 * pair);
    float st[16];
    auto load_b = [&](int ch) __attribute__((always_inline)) {
        const int r = (ch * KG + grp) * 8;
        const unsigned o = r < p.R && base != kOutsideBytes ? base + (unsigned)r * row_bytes : kOutsideBytes;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uintx2 v = __builtin_bit_cast(uintx2, __builtin_amdgcn_raw_buffer_load_b64(rsB, (int)(!RAGGED || r + i < p.R ? o : kOutsideBytes), (int)(i * row_bytes), 0));
            st[2 * i] = __uint_as_float(v.x);
            st[2 * i + 1] = __uint_as_float(v.y);
        }
    };
    auto store_b = [&](int buf) __attribute__((always_inline)) {
        char* d0 = smem + buf * BUF + grp * GROUP;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            unsigned part[4][NP];
#pragma unroll
            for (int h = 0; h < 4; ++h) split_pair<NP>(st[4 * h + j], st[4 * h + 2 + j], part[h], lost);
            const int slot = column_slot<BN>(2 * pair + j);
#pragma unroll
            for (int q = 0; q < NP; ++q)
                *reinterpret_cast<uintx4*>(d0 + q * (KG * GROUP) + slot * 16) = uintx4{part[0][q], part[1][q], part[2][q], part[3][q]};
        }
    };
    floatx16 acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    clear();

    const int block0 = m0 / 32 + wm * TM;
    uintx4 av[2][TM][NP];
    auto read_a = [&](int step, uintx4 (&a)[TM][NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const bool in = block0 + i < g.blocks && step < g.steps;     // uniform
            const unsigned from = in ? (unsigned)((block0 + i) * g.steps + step) * (NP * 1024u) : 0u;
#pragma unroll
            for (int q = 0; q < NP; ++q)
                a[i][q] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rsA, in ? lane * 16 + q * 1024 : (int)kOutsideBytes, (int)from, 0));
        }
    };
    int b_slot[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) b_slot[j] = column_slot<BN>(wn * (BN / WN) + j * 32 + lcol) * 16 + lrow * GROUP;
    // A chunk has sums of its own, which start from nothing and are added to the others': 64 steps in one chain have an error of 4.8e-7 (2-norm,
    // 1024 channels), in chunks of four 1.4e-7, and the time is the same.
    floatx16 part[TM][TN];
    auto multiply = [&](const char* s0, const uintx4 (&a)[TM][NP], bool begin) __attribute__((always_inline)) {
        bf16x8 bv[TN][NP];
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int j = 0; j < TN; ++j) bv[j][q] = *reinterpret_cast<const bf16x8*>(s0 + q * (KG * GROUP) + b_slot[j]);
        // the product of the leading parts last; every accumulator is touched once per round of tiles
#pragma unroll
        for (int t = 0; t < Terms<NP>::end; ++t) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    part[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i][Terms<NP>::pa[t]]), bv[j][Terms<NP>::pb[t]],
                                                                         begin && t == 0 ? floatx16{} : part[i][j], 0, 0, 0);
        }
    };

    const int nchunks = (p.R + BK - 1) / BK;
    load_b(0);
    read_a(0, av[0]);
    store_b(0);
    if (nchunks > 1) load_b(1);
#pragma unroll 1
    for (int c = 0; c < nchunks; ++c) {
        const char* s0 = smem + (c & 1) * BUF;
        lds_barrier();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            read_a(c * KS + ks + 1, av[(ks + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            multiply(s0 + 2 * ks * GROUP, av[ks & 1], ks == 0);
        }
        if (c + 1 < nchunks) {
            store_b((c + 1) & 1);
            if (c + 2 < nchunks) load_b(c + 2);
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] += part[i][j];
    }
    if constexpr (NP == 3) {
        const bool l = parts_lost(lost);
        if (lane == 0) wave_lost[wave] = l ? 1 : 0;
    }
    lds_barrier();

    // A wavefront with sums that are not finite, and every wavefront of a workgroup that staged a value its parts do not hold, repeats its
    // block on the fp32 matrix instructions, columns straight from memory (as in conv_patch.hip)
    if constexpr (NP == 3) {
        FiniteCheck check;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) check.add(acc[i][j][r]);
        int any_lost = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) any_lost |= wave_lost[w];
        if (check.failed() || __builtin_amdgcn_readfirstlane(any_lost) != 0) {
            clear();
            unsigned bc[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) bc[j] = column(n0 + wn * (BN / WN) + j * 32 + lcol);
#pragma unroll 1
            for (int step = 0; step < g.steps; ++step) {
                read_a(step, av[0]);
                const int r0 = step * 16 + 8 * lrow;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float x[TN];
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        x[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                            rsB, (int)(r0 + e < p.R && bc[j] != kOutsideBytes ? bc[j] + (unsigned)(r0 + e) * row_bytes : kOutsideBytes), 0, 0));
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const float wv = weight_value(av[0][i], e);
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, x[j], acc[i][j], 0, 0, 0);
                    }
                }
            }
        }
    }

    const TileDest dest = tile_dest(p, b, 0, 1, 0);
    store_tiles<TM, TN, true>(acc, dest, p.M, p.Ncols, m0 + wm * (BM / WM), n0 + wn * (BN / WN), lane,
                              reinterpret_cast<float*>(smem) + wave * kStageFloats, g.vecD);
}

// Few columns and a long reduction (as gemm_short.hip): the WK wavefronts divide the reduction, each loads its columns straight into registers, and
// their sums are added through LDS in wavefront order.
template <int TM, int TN, int WK, bool RAGGED, bool BATCH, int NP>
__global__ __launch_bounds__(WK * 64) void gemm_prepared_short_kernel(GemmProblem p, PreparedArgs g)
{
    constexpr int THREADS = WK * 64;
    __shared__ __attribute__((aligned(16))) float red[WK * TM * TN * 1024];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ls = lane & 31, lg = lane >> 5;

    const int wg = (int)xcd_contiguous(blockIdx.x, (unsigned)g.total);
    const int b = BATCH ? (int)const_div((unsigned)wg, g.by_tiles) : 0, tile = wg - b * (g.tilesM * g.tilesN);
    const int tn = (int)const_div((unsigned)tile, g.by_tm), tm = tile - tn * g.tilesM;

    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(parts_of(p, g, b), 0, (int)g.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.B) + b * p.strideB_batch, 0, (int)g.b_bytes, 0x00020000);

    // steps of this wavefront: a contiguous run
    const int per_wave = (g.steps + WK - 1) / WK, first = wave * per_wave;
    const int steps = g.steps - first < per_wave ? g.steps - first : per_wave;         // <= 0: none

    const unsigned row_bytes = (unsigned)p.strideB_row * 4u;
    unsigned b_base[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = (tn * TN + j) * 32 + ls;
        const int img = (int)const_div((unsigned)col, g.by_l), rest = col - img * p.L;
        b_base[j] = col < p.Ncols ? (unsigned)(img * (int)p.strideB_img + rest) * 4u : kOutsideBytes;
    }
    auto read_a = [&](int step, uintx4 (&a)[TM][NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = tm * TM + i;
            const bool in = mb < g.blocks && step < g.steps;             // uniform
#pragma unroll
            for (int q = 0; q < NP; ++q)
                a[i][q] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(
                    rsA, in ? lane * 16 + q * 1024 : (int)kOutsideBytes, in ? (int)((unsigned)(mb * g.steps + step) * (NP * 1024u)) : 0, 0));
        }
    };
    auto read_b = [&](int step, float (&b)[TN][8]) __attribute__((always_inline)) {
        const int r = step * 16 + lg * 8;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const unsigned o = r < p.R && b_base[j] != kOutsideBytes ? b_base[j] + (unsigned)r * row_bytes : kOutsideBytes;
            // rows past the end may be the next image's, whose infinities and NaN a zero weight does not cancel
#pragma unroll
            for (int e = 0; e < 8; ++e)
                b[j][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsB, (int)(!RAGGED || r + e < p.R ? o : kOutsideBytes), (int)(e * row_bytes), 0));
        }
    };

    floatx16 acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    clear();
    unsigned lost = 0;
    uintx4 av[TM][NP];
    float bv[TN][8];
    if (steps > 0) {
        read_b(first, bv);
        read_a(first, av);
    }
#pragma unroll 1
    for (int s = 0; s < steps; ++s) {
        uintx4 a[TM][NP];
        bf16x8 v[TN][NP];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < NP; ++q) a[i][q] = av[i][q];
#pragma unroll
        for (int j = 0; j < TN; ++j) split_octet<NP>(bv[j], v[j], lost);
        if (s + 1 < steps) {
            read_b(first + s + 1, bv);
            read_a(first + s + 1, av);
        }
#pragma unroll
        for (int t = 0; t < Terms<NP>::end; ++t)              // the product of the leading parts last
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i][Terms<NP>::pa[t]]), v[j][Terms<NP>::pb[t]], acc[i][j], 0, 0, 0);
    }

    // as above, the wavefront's own steps
    if constexpr (NP == 3) {
        FiniteCheck check;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) check.add(acc[i][j][r]);
        if (check.failed() || parts_lost(lost)) {
            clear();
#pragma unroll 1
            for (int q = 0; q < steps; ++q) {
                read_a(first + q, av);
                const int r0 = (first + q) * 16 + lg * 8;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float x[TN];
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        x[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                            rsB, (int)(r0 + e < p.R && b_base[j] != kOutsideBytes ? b_base[j] + (unsigned)(r0 + e) * row_bytes : kOutsideBytes), 0, 0));
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const float wv = weight_value(av[i], e);
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, x[j], acc[i][j], 0, 0, 0);
                    }
                }
            }
        }
    }

    // ---- partial tiles added in wavefront order, then bias and store
    constexpr int OUT = TM * TN * 1024, IT = OUT / THREADS;
    auto out_row = [&](int o) -> int { const int r = (o >> 6) & 15, l = o & 63; return (tm * TM + (o >> 10) / TN) * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); };
    float bias[IT];                           // on its way while the partial tiles cross LDS
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int m = out_row(tid + t * THREADS);
        bias[t] = p.bias ? p.bias[m < p.M ? m : p.M - 1] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[((wave * TM * TN + i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int o = tid + t * THREADS;
        float v = red[o];
#pragma unroll
        for (int w = 1; w < WK; ++w) v += red[w * OUT + o];
        const int m = out_row(o), col = (tn * TN + (o >> 10) % TN) * 32 + (o & 31);
        if (m < p.M && col < p.Ncols) {
            const int img = (int)const_div((unsigned)col, g.by_l);
            p.D[b * p.strideD_batch + (long long)img * p.strideD_img + (long long)m * p.strideD_row + (col - img * p.L)] = v + bias[t];
        }
    }
}

bool prepared_args(const GemmProblem& p, int bm, int bn, int threads, PreparedArgs* g)
{
    unsigned plain = 0;
    if (!p.a_parts || p.splitk > 1 || !gemm_prepared_covers(p) || !gemm_operand_extents(p, &plain, &g->b_bytes)) return false;
    g->a_bytes = (unsigned)gemm_parts_bytes(p.prec, p.M, p.R);
    g->blocks = (p.M + 31) / 32;
    g->steps = (p.R + 15) / 16;
    g->tilesM = (p.M + bm - 1) / bm;
    g->tilesN = (p.Ncols + bn - 1) / bn;
    const long long total = (long long)g->tilesM * g->tilesN * p.batch;
    if (!grid_fits(total, threads)) return false;
    g->total = (int)total;
    g->vecD = result_rows_vectorisable(p);
    g->by_l = make_constdiv((unsigned)p.L);
    g->by_tm = make_constdiv((unsigned)g->tilesM);
    g->by_tiles = make_constdiv((unsigned)(g->tilesM * g->tilesN));
    return true;
}

template <int TM, int TN, int WK>
hipError_t launch_prepared_short_cfg(const GemmProblem& p, bool, hipStream_t s)
{
    PreparedArgs g{};
    if (!prepared_args(p, 32 * TM, 32 * TN, WK * 64, &g)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)g.total), block(WK * 64);
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, p, g); };
    if (p.prec == 2) {
        if (p.R & 7) run(gemm_prepared_short_kernel<TM, TN, WK, true, true, 2>);
        else run(gemm_prepared_short_kernel<TM, TN, WK, false, true, 2>);
    } else if (p.batch > 1) {
        if (p.R & 7) run(gemm_prepared_short_kernel<TM, TN, WK, true, true, 3>);
        else run(gemm_prepared_short_kernel<TM, TN, WK, false, true, 3>);
    } else if (p.R & 7) run(gemm_prepared_short_kernel<TM, TN, WK, true, false, 3>);
    else run(gemm_prepared_short_kernel<TM, TN, WK, false, false, 3>);
    return hipGetLastError();
}

template <int BM, int BN, int WM, int WN>
hipError_t launch_prepared_cfg(const GemmProblem& p, bool vec, hipStream_t s)
{
    PreparedArgs g{};
    if (p.L % 2 != 0) return launch_prepared_short_cfg<2, 2, 8>(p, vec, s);          // a choice saved for another plane: a pair of columns may lie in two images
    if (!prepared_args(p, BM, BN, WM * WN * 64, &g)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)g.total), block(WM * WN * 64);
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, p, g); };
    if (p.prec == 2) {
        if (p.R & 7) run(gemm_prepared_kernel<BM, BN, WM, WN, true, true, 2>);
        else run(gemm_prepared_kernel<BM, BN, WM, WN, false, true, 2>);
    } else if (p.batch > 1) {
        if (p.R & 7) run(gemm_prepared_kernel<BM, BN, WM, WN, true, true, 3>);
        else run(gemm_prepared_kernel<BM, BN, WM, WN, false, true, 3>);
    } else if (p.R & 7) run(gemm_prepared_kernel<BM, BN, WM, WN, true, false, 3>);
    else run(gemm_prepared_kernel<BM, BN, WM, WN, false, false, 3>);
    return hipGetLastError();
}

// One workgroup per 32 output channels x 64 channels of one position: rows of U, prepared as parts (as the preparation of the rows, bound by memory; it runs once).
template <int NP>
__global__ __launch_bounds__(256) void parts_of_rows_kernel(const float* __restrict__ U, uintx4* __restrict__ Up, int K, int C, int ldk, int blocks, int steps, int quads)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = blockIdx.x % quads, r1 = blockIdx.x / quads, kb = r1 % blocks, b = r1 / blocks;
    const int step = q * 4 + wave, k = kb * 32 + (lane & 31), c = step * 16 + (lane >> 5) * 8;
    if (step >= steps) return;
    const float* u = U + ((long long)b * C + c) * ldk + k;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = k < K && c + e < C ? u[(long long)e * ldk] : 0.f;
    unsigned part[4][NP];
    if constexpr (NP == 3) weight_parts(v, part);
    else {
        unsigned lost = 0;
#pragma unroll
        for (int h = 0; h < 4; ++h) split_pair<NP>(v[2 * h], v[2 * h + 1], part[h], lost);
    }
    uintx4* up = Up + (((long long)b * blocks + kb) * steps + step) * (NP * 64) + lane;
#pragma unroll
    for (int t = 0; t < NP; ++t) up[t * 64] = uintx4{part[0][t], part[1][t], part[2][t], part[3][t]};
}

const GemmVariant kPrepared[] = {
    {"x6_prepared_128x128x32_w2x2", launch_prepared_cfg<128, 128, 2, 2>, 128, 128, 32},
    {"x6_prepared_128x64x64_w2x2", launch_prepared_cfg<128, 64, 2, 2>, 128, 64, 64},
    {"x6_prepared_64x128x32_w2x2", launch_prepared_cfg<64, 128, 2, 2>, 64, 128, 32},
    {"x6_prepared_64x64x64_w2x2", launch_prepared_cfg<64, 64, 2, 2>, 64, 64, 64},
    {"x6_prepared_32x32_k8", launch_prepared_short_cfg<1, 1, 8>, 32, 32, 128},
    {"x6_prepared_64x64_k8", launch_prepared_short_cfg<2, 2, 8>, 64, 64, 128},
};

}  // namespace

int gemm_prepared_variant_count() { return (int)(sizeof(kPrepared) / sizeof(kPrepared[0])); }
const GemmVariant& gemm_prepared_variant(int i) { return kPrepared[i]; }

// Results of 48 MB and more go to the plain tiles: they are bound by memory, and past the caches these lose 3 to 15 % (32 x 28 x 28 256 -> 1024 86 against
// 93 us, 32 x 32 x 32 96 -> 1024 56 against 64; at 45 MB, 8 x 56 x 57 128 -> 442, 26.5 against 25.4).  Staged tiles where 64 x 64 tiles fill half the
// chip (below, the divided ones always won: one of 56 x 56 405 -> 96, 98 tiles, 6.8 against 11.4), 128 x 128 where they fill it three times (16 x 14 x 14
// 512 -> 512, 392 tiles, 26.5 against 16.6; 8 x 28 x 29 256 -> 1024, 1632 tiles, 25.4 against 27.1).  Divided ones up to two 64 x 64 tiles per CU, and
// 64 x 64 among them from half the chip on and with two steps for each wavefront (32 x 14 x 15 1024 -> 256, 420 tiles, 28.4 against 29.5 staged; 2 x 28
// x 28 1024 -> 128, 50 tiles, 14.3 against 8.2 in 32 x 32).  Planes of an odd size have the divided tiles alone.
// Single products with a long reduction and few 32 x 32 tiles keep the plain divided ones: the weights' six bytes count more there, and timing, on operands
// that are in the L2, does not show it.  Of 30 such layers (454 to 1211 channels, three plans in turn, whole calls) these take 0.99 to 1.42 times as long as
// the plain ones below 130 tiles, and a planner that may take them does so wrongly for 1199 -> 956 on 10 x 10 (120 tiles, 9.9 against 10.3 us) and 896 -> 546
// on 14 x 14 (126, 7.7 against 8.1); from 140 to 190 tiles it is 0.96 to 1.01 (502 -> 641 on 18 x 13 6.4 both).  From 192 tiles on (17 layers) and with
// up to 448 channels the planner's choice is the better one within 3 %.  Loads two steps ahead are slower everywhere (up to 0.4 us).
// Winograd products take the same rules over all positions: 64 of 93 x 248 x 67 8.2 -> 7.6, 36 of 256 x 512 x 256 25.0 -> 22.3, 36 of 512 x 392 x 512 56.8 ->
// 50.7, 64 of 256 x 124 x 256 12.7 -> 11.6, 16 of 256 x 1600 x 256 29.0 -> 27.7; 50 MB and more lose: 100 of 256 x 4096 x 256 304 against 337, 64 of
// 128 x 4096 x 128 64 against 73, 64 of 256 x 1600 x 256 83 against 84.  Of few columns it is the weights that count, six bytes instead of four: more than
// 12 MB of them for fewer than 64 columns stay as they are (whole calls, 100 of 115 x 36 x 254, 20 MB, 15.6 against 15.4; 16 of 512 x 52 x 512, 25 MB,
// 13.1 against 13.0; 36 of 128 x 52 x 300, 8 MB, 12.0 against 12.6; 36 of 512 x 64 x 512, 57 MB, 21.0 against 21.2).  128 x 128 in fp32 is for reductions beyond four
// chunks: of 24 layers with 35 to 128 channels a planner that may take it did so in none (three processes each), and with it the whole call takes 0.97 to 1.25
// times as long, 1.08 on average (F(4,3) 128 -> 128 on 32 x 28 x 28 38.7 against 39.1 us, 128 -> 135 F(4,5) on 3 x 42 x 42 26.3 against 24.3).  bf16x3: 36 of 256 x 512 x 256
// 17.7 -> 16.5, 64 of 90 x 92 x 400 10.4 -> 7.3, 36 of 128 x 1600 x 128 14.9 -> 13.8.
bool gemm_prepared_offered(const GemmProblem& p, int i)
{
    if (!gemm_prepared_covers(p)) return false;
    if ((long long)p.M * p.Ncols * p.batch > 12ll << 20) return false;
    if (p.batch > 1 && p.Ncols < 64 && (long long)p.batch * gemm_parts_bytes(p.prec, p.M, p.R) > 12ll << 20) return false;
    const long long tiles64 = (long long)((p.M + 63) / 64) * ((p.Ncols + 63) / 64) * p.batch;
    const long long tiles32 = (long long)((p.M + 31) / 32) * ((p.Ncols + 31) / 32);
    switch (i) {
        case 0: return p.L % 2 == 0 && tiles64 >= 768 && (p.batch == 1 || p.prec != 0 || p.R > 128);
        case 1: case 2: case 3: return p.L % 2 == 0 && tiles64 >= 128;
        case 4: return tiles64 < 512 && (p.batch > 1 || p.R <= 448 || tiles32 >= 192);
        default: return p.R >= 256 && tiles64 >= 128 && tiles64 < 512;
    }
}

size_t gemm_parts_bytes(int prec, int K, int C) { return conv_patch_weight_bytes(K, C, 1) / 3 * (prec == 2 ? 2 : 3); }

hipError_t launch_parts_of_rows(int prec, const float* U, void* Up, int K, int C, int ldk, int batch, hipStream_t s)
{
    if (!U || !Up || K <= 0 || C <= 0 || ldk < K || batch <= 0 || (prec != 0 && prec != 2)) return hipErrorInvalidValue;
    const int blocks = (K + 127) / 128 * 4, steps = (C + 15) / 16, quads = (steps + 3) / 4;        // whole blocks of 128 rows (conv_patch_weight_bytes)
    const long long total = (long long)blocks * quads * batch;
    if (!grid_fits(total, 256)) return hipErrorInvalidValue;
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(256), 0, s, U, static_cast<uintx4*>(Up), K, C, ldk, blocks, steps, quads); };
    if (prec == 0) run(parts_of_rows_kernel<3>);
    else run(parts_of_rows_kernel<2>);
    return hipGetLastError();
}

bool gemm_prepared_covers(const GemmProblem& p)
{
    unsigned a = 0, b = 0;
    return (p.prec == 0 || (p.prec == 2 && p.batch > 1)) && !p.gather && p.batch > 0 && p.M > 0 && p.R >= 16 && p.L > 0 && conv_patch_weight_bytes(p.M, p.R, 1) < ((size_t)1 << 31) &&
           7ll * p.strideB_row * 4 < (1ll << 30) && gemm_operand_extents(p, &a, &b);
}

}  // namespace mnnconv
