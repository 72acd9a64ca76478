// Winograd products and inverse transform of a short grid in one kernel, for the call that prepares its weights every time.
//
// After the launch that transforms input and weights, products and inverse transform took two more, each some 3 us of launch, arguments, first loads and
// drain around little work, and as long again on the host.  Here a workgroup owns 16 tiles x 16 output channels at all positions: wavefront w takes positions
// w, w + 8, ... and the whole reduction of each, loads operands straight into the registers the fp32 matrix instruction reads (as gemm_short.hip),
// and leaves its 16 x 16 sums in LDS; then each pair of tile and channel is one lane per share of the tile's rows.
// What bounds it are the 4-byte loads, 6 cycles of a CU each, 16 per wavefront, position and 32 channels: so few positions and channels only
// (products_output_short).  Whole calls, us: F(2,3) one image 64 -> 64 56 x 56 13.1 -> 12.4, 25 -> 22 48 x 49 10.1 -> 8.3, 2 images 21 -> 89 25 x 28 12.7 -> 8.4, F(2,5)
// one image 9 -> 115 10 x 14 13.9 -> 12.2.  Loads four steps ahead instead of two: no difference.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels.hpp"
#include "xcd_remap.hpp"
#include "wino_paired.hpp"
#include "bf16_parts.hpp"
#include "fast_div.hpp"

namespace mnnconv {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kWaves = 8;

struct ProductsArgs {
    int K, C, P, Ho, Wo, ldk, ldp, tw, th;
    int kblocks, total, steps;               // steps of 32 channels
    unsigned u_bytes, v_bytes;
    int vec;                                 // 2: 16-byte stores of whole tile rows, 1: pairs, 0: single values
    ConstDiv by_kblocks, by_tw, by_th, by_steps;
};

// RAGGED: a channel count that is no multiple of 8
template <int NT, int A, bool RAGGED>
__global__ __launch_bounds__(kWaves * 64) void products_output_kernel(ProductsArgs g, MatArg<NT, A> at, const float* __restrict__ U, const float* __restrict__ V,
                                                                      const float* __restrict__ bias, float* __restrict__ y)
{
    constexpr int RING = 3;
    __shared__ float sums[A * A * 256];                   // [position][channel][tile]
    const int tid = threadIdx.x, lane = tid & 63, ls = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = (int)xcd_contiguous(blockIdx.x, (unsigned)g.total);
    const int pb = (int)const_div((unsigned)wg, g.by_kblocks), kb = wg - pb * g.kblocks;
    const int k0 = kb * 16, p0 = pb * 16;

    const __amdgpu_buffer_rsrc_t rsU = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(U), 0, (int)g.u_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsV = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(V), 0, (int)g.v_bytes, 0x00020000);
    const int u_row = g.ldk * 4, v_row = g.ldp * 4;       // bytes
    const unsigned u_lane = k0 + ls < g.ldk ? (unsigned)(lg * 8 * g.ldk + k0 + ls) * 4u : kOutsideBytes;
    const unsigned v_lane = p0 + ls < g.ldp ? (unsigned)(lg * 8 * g.ldp + p0 + ls) * 4u : kOutsideBytes;

    // step u: 32 channels of one of this wavefront's positions
    const int positions = (A * A - wave + kWaves - 1) / kWaves, all = positions * g.steps;
    float a[RING][8], b[RING][8];
    auto load = [&](int u, float (&av)[8], float (&bv)[8]) __attribute__((always_inline)) {
        const int q = (int)const_div((unsigned)u, g.by_steps), c0 = (u - q * g.steps) * 32;
        const int row = (wave + q * kWaves) * g.C + c0;
        const int left = g.C - c0 - lg * 8;               // channels of this lane's group: behind them lie the next position's
        const bool in = u < all && left > 0;
        const unsigned uo = in && u_lane != kOutsideBytes ? u_lane + (unsigned)row * u_row : kOutsideBytes;
        const unsigned vo = in && v_lane != kOutsideBytes ? v_lane + (unsigned)row * v_row : kOutsideBytes;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            av[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsU, (int)(!RAGGED || e < left ? uo : kOutsideBytes), e * u_row, 0));
            bv[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsV, (int)(!RAGGED || e < left ? vo : kOutsideBytes), e * v_row, 0));
        }
    };
#pragma unroll
    for (int r = 0; r < RING - 1; ++r) load(r, a[r], b[r]);
    floatx4 acc[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
    int in_position = 0, position = wave;
    auto step = [&](int u, auto slot) __attribute__((always_inline)) {
        constexpr int I = decltype(slot)::value;
        load(u + RING - 1, a[(I + RING - 1) % RING], b[(I + RING - 1) % RING]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[I][e], b[I][e], acc[e & 1], 0, 0, 0);
        if (++in_position == g.steps) {
            if (u < all)
#pragma unroll
                for (int r = 0; r < 4; ++r) sums[position * 256 + (4 * lg + r) * 16 + ls] = acc[0][r] + acc[1][r];
            acc[0] = acc[1] = floatx4{0.f, 0.f, 0.f, 0.f};
            in_position = 0;
            position += kWaves;
        }
    };
#pragma unroll 1
    for (int u = 0; u < all; u += RING) {
        step(u, std::integral_constant<int, 0>{});
        step(u + 1, std::integral_constant<int, 1>{});
        step(u + 2, std::integral_constant<int, 2>{});
    }
    __syncthreads();

    // a lane per (channel, tile) and share of the tile's rows
    constexpr int SHARES = kWaves * 64 / 256, ROWS = (NT + SHARES - 1) / SHARES;
    const int kk = (tid >> 4) & 15, share = tid >> 8;
    const int k = k0 + kk, p = p0 + ls;
    if (k >= g.K || p >= g.P) return;
    const float bv = bias ? bias[k] : 0.f;
    float t[ROWS][A];
#pragma unroll
    for (int c = 0; c < A; ++c) {
        float m[A], o[NT];
#pragma unroll
        for (int r = 0; r < A; ++r) m[r] = sums[(r * A + c) * 256 + kk * 16 + ls];
        at_apply<NT, A>(at, m, 0.f, o);
#pragma unroll
        for (int i = 0; i < ROWS; ++i) t[i][c] = share == 0 ? o[i] : o[ROWS + i < NT ? ROWS + i : NT - 1];
    }
    const int r1 = (int)const_div((unsigned)p, g.by_tw), tx = p - r1 * g.tw;
    const int img = (int)const_div((unsigned)r1, g.by_th), ty = r1 - img * g.th;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const int row = share * ROWS + i, oy = ty * NT + row;
        if (row >= NT || oy >= g.Ho) break;
        float o[NT];
        at_apply<NT, A>(at, t[i], bv, o);
        float* dst = y + (((long long)img * g.K + k) * g.Ho + oy) * g.Wo + tx * NT;
        if (NT == 4 && g.vec == 2) {
            *reinterpret_cast<float4*>(dst) = make_float4(o[0], o[1 % NT], o[2 % NT], o[3 % NT]);
        } else if (NT % 2 == 0 && g.vec >= 1 && tx * NT + NT <= g.Wo) {
#pragma unroll
            for (int j = 0; j + 1 < NT; j += 2) *reinterpret_cast<float2*>(dst + j) = make_float2(o[j], o[j + 1]);
        } else {
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (tx * NT + j < g.Wo) dst[j] = o[j];
        }
    }
}

}  // namespace

// Of 70 shapes (1 to 4 images, 8 to 500 channels), time of one kernel over that of two: alpha^2 positions times steps of 32 channels up to 36 0.65 to 0.98
// (F(2,3) up to 64 channels, alpha 5 and 6 up to 32), 48 to 75 0.90 to 1.26, 108 1.2 to 1.6 and more beyond.
bool products_output_short(const WinoGeom& g)
{
    return !g.blocked && !g.tiled && g.alpha <= 6 && g.alpha * g.alpha * ((g.C + 31) / 32) <= 36;
}

hipError_t launch_products_output(const WinoGeom& g, const float* AT, const float* U, const float* V, const float* bias, float* y, hipStream_t s)
{
    if (!AT || !U || !V || !y || !products_output_short(g) || (g.alpha % 2 == 0 && !at_is_paired(AT, g.n, g.alpha))) return hipErrorNotSupported;
    ProductsArgs a{};
    a.K = g.K; a.C = g.C; a.P = g.P; a.Ho = g.Ho; a.Wo = g.Wo; a.ldk = g.ldk; a.ldp = g.ldp; a.tw = g.tw; a.th = g.th;
    const long long rows = (long long)g.alpha * g.alpha * g.C;
    if (rows * g.ldk >= (1ll << 29) || rows * g.ldp >= (1ll << 29)) return hipErrorNotSupported;
    a.u_bytes = (unsigned)(rows * g.ldk * 4);
    a.v_bytes = (unsigned)(rows * g.ldp * 4);
    a.kblocks = (g.K + 15) / 16;
    const long long total = (long long)a.kblocks * ((g.P + 15) / 16);
    if (!grid_fits(total, kWaves * 64)) return hipErrorNotSupported;
    a.total = (int)total;
    a.steps = (g.C + 31) / 32;
    a.vec = (g.n == 4 && g.Wo % 4 == 0 && (reinterpret_cast<uintptr_t>(y) & 15u) == 0) ? 2
            : (g.n % 2 == 0 && g.Wo % 2 == 0 && (reinterpret_cast<uintptr_t>(y) & 7u) == 0) ? 1 : 0;
    a.by_kblocks = make_constdiv((unsigned)a.kblocks);
    a.by_tw = make_constdiv((unsigned)g.tw);
    a.by_th = make_constdiv((unsigned)g.th);
    a.by_steps = make_constdiv((unsigned)a.steps);
    auto launch = [&](auto nt, auto al) -> hipError_t {
        constexpr int NT = decltype(nt)::value, A = decltype(al)::value;
        MatArg<NT, A> m;
        for (int i = 0; i < NT; ++i)
            for (int j = 0; j < A; ++j) m.v[i][j] = AT[i * A + j];
        auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(kWaves * 64), 0, s, a, m, U, V, bias, y); };
        if (g.C & 7) run(products_output_kernel<NT, A, true>);
        else run(products_output_kernel<NT, A, false>);
        return hipGetLastError();
    };
#define MNN_NA(NN, AA) \
    if constexpr (AA - NN + 1 >= 2 && AA - NN + 1 <= 7) { if (g.n == NN && g.alpha == AA) return launch(std::integral_constant<int, NN>{}, std::integral_constant<int, AA>{}); }
#define MNN_ALL_A(NN) MNN_NA(NN, 3) MNN_NA(NN, 4) MNN_NA(NN, 5) MNN_NA(NN, 6)
    MNN_ALL_A(2) MNN_ALL_A(3) MNN_ALL_A(4) MNN_ALL_A(5)
#undef MNN_ALL_A
#undef MNN_NA
    return hipErrorNotSupported;
}

}  // namespace mnnconv
