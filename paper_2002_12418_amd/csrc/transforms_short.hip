// The Winograd transforms for grids too short to fill the chip (batch-1 layers, small planes).
//
// transforms.hip gives a lane a whole tile: alpha^2 values, two transforms one after the other, some 900 vector instructions at alpha = 8.  Where
// a SIMD holds one such wavefront or none, each instruction that needs the one before it takes 8 cycles, and the kernel's time is that chain
// (F(6,3) on 5 x 67 x 37 x 41: 7.2 us on 65 workgroups, for 4 MB).  Here a lane owns one row or column of a tile: alpha times the wavefronts, a chain
// an alpha-th as long, the two one-dimensional transforms meet in LDS.  Same layouts, same precision.
// Whole calls, us, a lane per tile -> here: F(6,3) 5 x 67 -> 93 x 37 x 41 25.6 -> 19.5, 4 x 100 -> 90 x 60 x 60 F(4,5) 34.8 -> 31.3, F(8,3) 4 x 128 x 64 x 64 34.0 -> 27.6, F(4,7)
// 2 x 64 x 56 x 56 27.3 -> 22.7, F(4,3) 8 x 128 x 28 x 28 22.3 -> 20.7; with the weights in every call: F(2,3) one image 64 -> 64 56 x 56 18.2 -> 14.2, F(4,3) one
// image 128 -> 128 28 x 28 24.6 -> 14.7, F(6,3) 5 x 67 -> 93 39 x 39 38.6 -> 20.4.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels.hpp"
#include "xcd_remap.hpp"
#include "wino_paired.hpp"
#include "tile_row.hpp"
#include "fast_div.hpp"

namespace mnnconv {
namespace {

constexpr int kShortTiles = 32;              // tiles per workgroup: a lane is (row or column) * 32 + tile

struct ShortInArgs {
    int cblocks, input_blocks;               // blocks of 32 tiles per channel; workgroups of the input transform (the others: weights)
    unsigned x_bytes;
    long long plane, row;                    // floats between positions, and between channels (tiled: between runs of 64 tiles)
    ConstDiv by_tw, by_th, by_cblocks, by_ldk, by_c;
};

constexpr int short_threads(int alpha) { return (alpha * kShortTiles + 63) / 64 * 64; }

// 32 tiles of one channel.  Tiles past the last one (the padding of V's rows) are zeros.
template <int A>
__device__ __forceinline__ void input_short(const WinoGeom& g, const ShortInArgs& sa, const MatArg<A, A>& bt, const float* __restrict__ x,
                                            float* __restrict__ V, int wg, float* lds)
{
    const int c = (int)const_div((unsigned)wg, sa.by_cblocks);
    const int t = threadIdx.x % kShortTiles, i = threadIdx.x / kShortTiles;
    const int p = (wg - c * sa.cblocks) * kShortTiles + t;
    const bool row_ok = short_threads(A) == A * kShortTiles || i < A;
    {
        const int r1 = (int)const_div((unsigned)p, sa.by_tw), tx = p - r1 * g.tw;
        const int img = (int)const_div((unsigned)r1, sa.by_th), ty = r1 - img * g.th;
        const int y = ty * g.n - g.pad_h + i, x0 = tx * g.n - g.pad_w;
        const bool ok = row_ok && p < g.P && (unsigned)y < (unsigned)g.H;
        const int first = ((img * g.C + c) * g.H + y) * g.W + x0;        // elements; the tensor has fewer than 2^29
        float d[A];
        load_tile_row<A>(x, sa.x_bytes, first, x0, g.W, ok, d);
        if (row_ok) {
#pragma unroll
            for (int e = 0; e < A; ++e) lds[(e * A + i) * kShortTiles + t] = d[e];
        }
    }
    __syncthreads();
    // columns first, as everywhere else: which intermediate values overflow depends on it
    float in[A], out[A];
    if (row_ok) {
        float* col = lds + i * A * kShortTiles + t;
#pragma unroll
        for (int a = 0; a < A; ++a) in[a] = col[a * kShortTiles];
        bt_apply<A>(bt, in, out);
#pragma unroll
        for (int a = 0; a < A; ++a) col[a * kShortTiles] = out[a];
    }
    __syncthreads();
    if (!row_ok || p >= g.ldp) return;
#pragma unroll
    for (int b = 0; b < A; ++b) in[b] = lds[(b * A + i) * kShortTiles + t];
    bt_apply<A>(bt, in, out);
    float* dst = V + (g.tiled ? ((long long)c * g.pb + (p >> 6)) * sa.row + (p & 63) : (long long)c * sa.row + p) + (long long)i * A * sa.plane;
#pragma unroll
    for (int b = 0; b < A; ++b) dst[b * sa.plane] = out[b];
}

template <int A>
__global__ __launch_bounds__(short_threads(A)) void input_short_kernel(WinoGeom g, ShortInArgs sa, MatArg<A, A> bt, const float* __restrict__ x,
                                                                       float* __restrict__ V)
{
    __shared__ float lds[A * A * kShortTiles];
    input_short<A>(g, sa, bt, x, V, (int)xcd_contiguous(blockIdx.x, gridDim.x), lds);
}

// The input transform and the weights' in one launch, for a call that prepares its weights: the first workgroups take tiles, the others U, one
// lane per (row of G w G^T, input channel, output channel), the padding of U's rows included.
struct ShortFilterMat { float g[kMaxAlphaT][7]; };

template <int A, int KT>
__global__ __launch_bounds__(short_threads(A)) void input_filter_short_kernel(WinoGeom g, ShortInArgs sa, MatArg<A, A> bt, ShortFilterMat gm,
                                                                              const float* __restrict__ x, const float* __restrict__ w,
                                                                              float* __restrict__ V, float* __restrict__ U)
{
    __shared__ float lds[A * A * kShortTiles];
    if ((int)blockIdx.x < sa.input_blocks) {
        input_short<A>(g, sa, bt, x, V, (int)xcd_contiguous(blockIdx.x, (unsigned)sa.input_blocks), lds);
        return;
    }
    const int idx = ((int)blockIdx.x - sa.input_blocks) * short_threads(A) + (int)threadIdx.x;
    const int r1 = (int)const_div((unsigned)idx, sa.by_ldk), kk = idx - r1 * g.ldk;
    const int i = (int)const_div((unsigned)r1, sa.by_c), c = r1 - i * g.C;
    if (i >= A) return;
    const float* wp = w + ((long long)(kk < g.K ? kk : 0) * g.C + c) * KT * KT;
    float wl[KT][KT], row[KT];
#pragma unroll
    for (int r = 0; r < KT; ++r)
#pragma unroll
        for (int s = 0; s < KT; ++s) wl[r][s] = kk < g.K ? wp[r * KT + s] : 0.f;
#pragma unroll
    for (int s = 0; s < KT; ++s) {
        float acc = 0.f;
#pragma unroll
        for (int r = 0; r < KT; ++r) {
            float gi = gm.g[0][r];                        // row i of G: i differs between lanes, so it is picked from scalars
#pragma unroll
            for (int h = 1; h < A; ++h) gi = i == h ? gm.g[h][r] : gi;
            acc = fmaf(gi, wl[r][s], acc);
        }
        row[s] = acc;
    }
    float* up = U + ((long long)i * A * g.C + c) * g.ldk + kk;
#pragma unroll
    for (int j = 0; j < A; ++j) {
        float acc = 0.f;
#pragma unroll
        for (int s = 0; s < KT; ++s) acc = fmaf(row[s], gm.g[j][s], acc);
        up[(long long)j * g.C * g.ldk] = acc;
    }
}

struct ShortOutArgs {
    int pblocks;
    int vec;                                  // 2: 16-byte stores of whole tile rows, 1: pairs, 0: single values
    long long plane, row;                     // as ShortInArgs, of M
    ConstDiv by_tw, by_th, by_pblocks;
};

// 32 tiles of one output channel: a lane sums one column of m, then writes one row of the tile
template <int NT, int A>
__global__ __launch_bounds__(short_threads(A)) void output_short_kernel(WinoGeom g, ShortOutArgs sa, MatArg<NT, A> at, const float* __restrict__ M,
                                                                        const float* __restrict__ bias, float* __restrict__ y)
{
    __shared__ float lds[NT * A * kShortTiles];
    const int wg = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int k = (int)const_div((unsigned)wg, sa.by_pblocks);
    const int t = threadIdx.x % kShortTiles, i = threadIdx.x / kShortTiles;
    const int p = (wg - k * sa.pblocks) * kShortTiles + t;
    const bool pok = p < g.P;
    const float bv = bias ? bias[k] : 0.f;
    if ((short_threads(A) == A * kShortTiles || i < A) && pok) {
        const float* src = M + (g.tiled ? ((long long)k * g.pb + (p >> 6)) * sa.row + (p & 63) : (long long)k * sa.row + p) + i * sa.plane;
        float m[A], o[NT];
#pragma unroll
        for (int a = 0; a < A; ++a) m[a] = src[(long long)a * A * sa.plane];
        at_apply<NT, A>(at, m, 0.f, o);
#pragma unroll
        for (int r = 0; r < NT; ++r) lds[(r * A + i) * kShortTiles + t] = o[r];
    }
    __syncthreads();
    if (i >= NT || !pok) return;
    const int r1 = (int)const_div((unsigned)p, sa.by_tw), tx = p - r1 * g.tw;
    const int img = (int)const_div((unsigned)r1, sa.by_th), ty = r1 - img * g.th;
    const int oy = ty * NT + i;
    if (oy >= g.Ho) return;
    float s[A], o[NT];
#pragma unroll
    for (int b = 0; b < A; ++b) s[b] = lds[(i * A + b) * kShortTiles + t];
    at_apply<NT, A>(at, s, bv, o);
    float* row = y + (((long long)img * g.K + k) * g.Ho + oy) * g.Wo + tx * NT;
    if (NT == 4 && sa.vec == 2) {
        *reinterpret_cast<float4*>(row) = make_float4(o[0], o[1 % NT], o[2 % NT], o[3 % NT]);
    } else if (NT % 2 == 0 && sa.vec >= 1 && tx * NT + NT <= g.Wo) {
#pragma unroll
        for (int j = 0; j + 1 < NT; j += 2) *reinterpret_cast<float2*>(row + j) = make_float2(o[j], o[j + 1]);
    } else {
#pragma unroll
        for (int j = 0; j < NT; ++j)
            if (tx * NT + j < g.Wo) row[j] = o[j];
    }
}

ShortInArgs short_in_args(const WinoGeom& g)
{
    ShortInArgs a{};
    a.cblocks = (g.ldp + kShortTiles - 1) / kShortTiles;
    a.input_blocks = a.cblocks * g.C;
    a.x_bytes = (unsigned)((long long)g.N * g.C * g.H * g.W * 4);
    a.plane = g.tiled ? 64 : (long long)g.C * g.ldp;
    a.row = g.tiled ? 64ll * g.alpha * g.alpha : g.ldp;
    a.by_tw = make_constdiv((unsigned)g.tw); a.by_th = make_constdiv((unsigned)g.th); a.by_cblocks = make_constdiv((unsigned)a.cblocks);
    a.by_ldk = make_constdiv((unsigned)g.ldk); a.by_c = make_constdiv((unsigned)g.C);
    return a;
}

template <int A>
MatArg<A, A> short_bt(const float* BT)
{
    MatArg<A, A> m;
    for (int i = 0; i < A; ++i)
        for (int j = 0; j < A; ++j) m.v[i][j] = BT[i * A + j];
    return m;
}

template <int A>
hipError_t launch_input_filter_t(const WinoGeom& g, const ShortInArgs& a, const float* BT, const float* G, const float* x, const float* w, float* V,
                                 float* U, hipStream_t s)
{
    ShortFilterMat m;
    for (int i = 0; i < kMaxAlphaT; ++i)
        for (int j = 0; j < 7; ++j) m.g[i][j] = (i < g.alpha && j < g.k) ? G[i * g.k + j] : 0.f;
    const long long rows = (long long)A * g.C * g.ldk;
    const dim3 grid((unsigned)(a.input_blocks + (rows + short_threads(A) - 1) / short_threads(A))), block(short_threads(A));
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, s, g, a, short_bt<A>(BT), m, x, w, V, U); };
#define MNN_KT(KT_) \
    if constexpr (A - KT_ + 1 >= 2 && A - KT_ + 1 <= 8) { if (g.k == KT_) { launch(input_filter_short_kernel<A, KT_>); return hipGetLastError(); } }
    MNN_KT(2) MNN_KT(3) MNN_KT(4) MNN_KT(5) MNN_KT(6) MNN_KT(7)
#undef MNN_KT
    return hipErrorInvalidValue;
}

}  // namespace

// Where the lane's chain is what counts.  Whole planned calls of the separate kernels, a lane per tile against a lane per row of one, 473 + 349 shapes of
// 16 to 1024 channels: up to 65536 pairs of channel and tile, a wavefront of whole tiles per SIMD or fewer, 1.00 (alpha 3) to 1.12 (9 and 10) times the
// speed.  Beyond, for the long chains of a large alpha: alpha 6 and 7 up to 150000 pairs 1.00 to 1.15, but F(2,5) 4 x 602 -> 445 21 x 21 (291368 pairs) 82.9 us
// a lane per tile and 85.0 here, and F(2,5) one image 400 -> 512 40 x 40 (160000) 59.5 and 60.5: the products read V a little slower afterwards,
// which few output channels do not show (-> 64 28.2 and 25.4).  Alpha 8, two paired transforms, up to 600000 pairs 1.03 on average and 0.98 at worst; 10 up to
// 200000 1.05, at 390000 0.95 to 1.04; 9, whose matrices have no pairs, 0.96 on average from 100000 on, and 0.89 at 480000.
bool input_transform_short(const WinoGeom& g)
{
    const long long pairs = (long long)g.C * g.P;
    if (g.blocked || (long long)g.N * g.C * g.H * g.W >= (1ll << 29) - 1024) return false;
    if (pairs <= 65536) return true;
    switch (g.alpha) {
        case 6: case 7: return pairs <= 150000 || (pairs <= 200000 && g.K <= 256);
        case 8: return pairs <= 625000;
        case 10: return pairs <= 250000;
        default: return false;
    }
}

// The call that prepares its weights saves a launch as well, and its scratch array bounds the grid.
// Many weights: a lane per row of G w G^T reads them alpha times over (allocation-free F(4,3) 32 x 512 -> 512 x 7 x 7 54 us in two launches, 73 in one;
// 256 -> 256 x 14 x 14 49 both), and each is a run of k^2 values of its own, so that the line lies sooner for larger kernels (one image of 14 x 14, F(4,5)
// 160 -> 160 channels 31 and 28, 192 33.7 and 33.8, 224 37 and 41, 254 46 and 63; F(2,6) 128 26.2 and 24.5, 160 28.4 and 31.6).
bool input_filter_short(const WinoGeom& g)
{
    const long long pairs = (long long)g.C * g.P;
    if (g.blocked || (long long)g.N * g.C * g.H * g.W >= (1ll << 29) - 1024) return false;
    if (pairs > 65536 && (g.alpha < 6 || pairs * g.alpha * g.alpha > 40000000)) return false;
    return (long long)g.K * g.C <= 65536 && (long long)g.K * g.C * g.k * g.k <= 800000;
}

// Of the same calls: up to 65536 pairs 1.00 (alpha 8) to 1.01 (9 and 10), up to 200000 1.01 to 1.02 from alpha 8 on, beyond 0.95 to 1.04, 1.00 on average.
bool output_transform_short(const WinoGeom& g)
{
    const long long pairs = (long long)g.K * g.P;
    return pairs <= 65536 || (g.alpha >= 8 && pairs <= 200000);
}

hipError_t launch_input_short(const WinoGeom& g, const float* BT, const float* x, float* V, hipStream_t s)
{
    const ShortInArgs a = short_in_args(g);
    const dim3 grid((unsigned)a.input_blocks);
    switch (g.alpha) {
#define MNN_A(A_) case A_: hipLaunchKernelGGL(input_short_kernel<A_>, grid, dim3(short_threads(A_)), 0, s, g, a, short_bt<A_>(BT), x, V); break;
        MNN_A(3) MNN_A(4) MNN_A(5) MNN_A(6) MNN_A(7) MNN_A(8) MNN_A(9) MNN_A(10)
#undef MNN_A
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_input_filter_short(const WinoGeom& g, const float* BT, const float* G, const float* x, const float* w, float* V, float* U, hipStream_t s)
{
    const ShortInArgs a = short_in_args(g);
    if ((long long)g.alpha * g.C * g.ldk >= (1ll << 30)) return hipErrorInvalidValue;
    switch (g.alpha) {
#define MNN_A(A_) case A_: return launch_input_filter_t<A_>(g, a, BT, G, x, w, V, U, s);
        MNN_A(3) MNN_A(4) MNN_A(5) MNN_A(6) MNN_A(7) MNN_A(8) MNN_A(9) MNN_A(10)
#undef MNN_A
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_output_short(const WinoGeom& g, const float* AT, const float* M, const float* bias, float* y, hipStream_t s)
{
    ShortOutArgs a{};
    a.pblocks = (g.P + kShortTiles - 1) / kShortTiles;
    a.plane = g.tiled ? 64 : (long long)g.K * g.ldp;
    a.row = g.tiled ? 64ll * g.alpha * g.alpha : g.ldp;
    a.vec = (g.n == 4 && g.Wo % 4 == 0 && (reinterpret_cast<uintptr_t>(y) & 15u) == 0) ? 2
            : (g.n % 2 == 0 && g.Wo % 2 == 0 && (reinterpret_cast<uintptr_t>(y) & 7u) == 0) ? 1 : 0;
    a.by_tw = make_constdiv((unsigned)g.tw); a.by_th = make_constdiv((unsigned)g.th); a.by_pblocks = make_constdiv((unsigned)a.pblocks);
    const dim3 grid((unsigned)((long long)a.pblocks * g.K));
    auto launch = [&](auto nt, auto al) -> hipError_t {
        constexpr int NT = decltype(nt)::value, A = decltype(al)::value;
        MatArg<NT, A> m;
        for (int i = 0; i < NT; ++i)
            for (int j = 0; j < A; ++j) m.v[i][j] = AT[i * A + j];
        hipLaunchKernelGGL((output_short_kernel<NT, A>), grid, dim3(short_threads(A)), 0, s, g, a, m, M, bias, y);
        return hipGetLastError();
    };
#define MNN_NA(NN, AA) \
    if constexpr (AA - NN + 1 >= 2 && AA - NN + 1 <= 7) { if (g.n == NN && g.alpha == AA) return launch(std::integral_constant<int, NN>{}, std::integral_constant<int, AA>{}); }
#define MNN_ALL_A(NN) MNN_NA(NN, 3) MNN_NA(NN, 4) MNN_NA(NN, 5) MNN_NA(NN, 6) MNN_NA(NN, 7) MNN_NA(NN, 8) MNN_NA(NN, 9) MNN_NA(NN, 10)
    MNN_ALL_A(2) MNN_ALL_A(3) MNN_ALL_A(4) MNN_ALL_A(5) MNN_ALL_A(6) MNN_ALL_A(7) MNN_ALL_A(8)
#undef MNN_ALL_A
#undef MNN_NA
    return hipErrorInvalidValue;
}

}  // namespace mnnconv
