// Sliding window as an implicit product whose right operand is staged as a patch of the image (fp32-grade on the bf16 matrix cores: parts and
// terms as in gemm_split.hip).
//
// The gather of gemm_split.hip stages every column once per tap: a 3 x 3 window loads, cuts into parts and writes to LDS each input value
// nine times (2.25 times at stride 2, where it is still nine loads for four new values).  Here a workgroup owns a rectangle of output pixels
// (NI images x TY rows x TX columns, up to BN) and keeps the patch of the input that they see in LDS, 16 channels at a time, cut into parts once.
// A tap is then one more offset into the patch, the same for all lanes.  The weights are prepared as parts in operand order and go from the L2
// straight to registers, one tap ahead.
//
// What bounds it (3 x 3 stride 2, 64 -> 128 on 32 x 56 x 56, 128 x 64 tiles, 29 us): 15 us of matrix instructions, which the power holds at 1.5 to 1.7 GHz; the rest
// does not overlap with them, because the 448 workgroups are one round in step: launch and first patch 6 us, LDS reads and taps 3, the later
// patches 3, the stores 3 (measured by leaving each out).  A wavefront owns 32 output channels and all columns of the rectangle: 64 x 32 and 64 x 64
// blocks read more weights per product than the L1 delivers (64 bytes per cycle and CU; 35 and 41 us).
// Measured against the best of the other configurations, us: that layer 41.5 -> 29.3; stride 2 128 -> 256 on 32 x 28 x 28 41.6 -> 30; stride 1 64 -> 64 on
// 16 x 56 x 56 39.4 -> 29, 2 x 2 24.4 -> 20.  Short grids belong to conv_short.hip (3 x 3 128 -> 128 on 4 x 28 x 28: 10.8 there, 18.2 here): the
// planner times both.  Relative error of the first layer 1.4e-7 -> 1.0e-7, 5 x 5 128 -> 128 on 8 x 28 x 28
// 3.0e-7 -> 2.2e-7 (one sum for all six products would give 3.6e-7 and 8.5e-7).
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels.hpp"
#include "lds_barrier.hpp"
#include "xcd_remap.hpp"
#include "gemm_epilogue.hpp"
#include "bf16_parts.hpp"
#include "fast_div.hpp"
#include "patch_rect.hpp"

namespace mnnconv {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
constexpr int kPatchChannels = 16;           // channels per chunk: the depth of one matrix instruction

struct PatchArgs : PatchRect {
    int tilesM, total;
    int nch;                     // chunks of channels
    int nbuf;                    // patch buffers: 2 where they fit
    int N, Ho;
    unsigned a_bytes, b_bytes;
    ConstDiv by_pw, by_ph, by_tx, by_ty, by_sw, by_tm, by_tiles_x, by_tiles_y;
};

// Wp[m/32][c/16][tap]: lane l holds output channel l % 32 and channels 8 * (l / 32) .. + 7 of the chunk, as [part][lane][8 bf16] (weight_parts):
// the matrix operand as it is read.  Channels past K and C hold zeros.
__global__ __launch_bounds__(256) void patch_weights_kernel(const float* __restrict__ w, uintx4* __restrict__ Wp, int K, int C, int taps, int nch)
{
    const int mb = blockIdx.x / nch, ch = blockIdx.x % nch;
    const int lane = threadIdx.x & 63;
    const int m = mb * 32 + (lane & 31), c0 = ch * kPatchChannels + (lane >> 5) * 8;
#pragma unroll 1
    for (int tap = threadIdx.x >> 6; tap < taps; tap += 4) {
        float v[8];
        unsigned part[4][3];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = m < K && c0 + e < C ? w[((long long)m * C + c0 + e) * taps + tap] : 0.f;
        weight_parts(v, part);
        uintx4* up = Wp + ((long long)blockIdx.x * taps + tap) * 3 * 64 + lane;
#pragma unroll
        for (int q = 0; q < 3; ++q) up[q * 64] = uintx4{part[0][q], part[1][q], part[2][q], part[3][q]};
    }
}

// LDS: nbuf patches [part][8-channel group][slot][8 bf16].  WM x WN wavefronts multiply.  NS = 0: they stage, too.  NS > 0: that many more stage.  Loads
// of one wavefront return in order, and weights that follow pixels wait for those, a trip to memory in every chunk: it pays where chunks
// are many and workgroups few (stride 2 128 -> 256 on 32 x 28 x 28 35 -> 30 us, 256 -> 512 on 32 x 14 x 14 50 -> 40), not where more workgroups
// per CU hide it (64 -> 128 on 32 x 56 x 56 30 -> 32, stride 1 64 -> 64 on 16 x 56 x 56 29 -> 31).
//
// Two workgroups of four wavefronts per CU also in registers: left to itself the compiler takes so many for the 64 x 128 tile that one fits (whole calls,
// us: stride 2 32 -> 64 on 16 x 112 x 112 27.7 -> 19.4, 64 -> 64 on 16 x 56 x 56 36.2 -> 27.9, although ten scalar registers spill), and the others are 1 to 4 % slower
// (128 x 64, stride 2 64 -> 128 on 32 x 56 x 56 31.5 -> 30.8; 64 x 64, 48 -> 96 on 24 x 40 x 40 27.4 -> 26.5; 5 x 5 128 -> 128 on 8 x 28 x 28 41.1 -> 40.9).
template <int BM, int BN, int WM, int WN, int ITEMS, int NS>
__global__ __launch_bounds__((WM * WN + NS) * 64, 2) void conv_patch_kernel(GemmProblem p, PatchArgs g)
{
    constexpr int NW = WM * WN;
    constexpr int SW = NS > 0 ? NS : NW, S0 = NS > 0 ? NW : 0, LANES = SW * 64;          // wavefronts that stage, the first of them
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int wave_lost[SW];
    unsigned lost = 0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lrow = lane >> 5, lcol = lane & 31;

    const int wg = (int)xcd_contiguous(blockIdx.x, (unsigned)g.total);
    const int t1 = (int)const_div((unsigned)wg, g.by_tm);
    const int m0 = (wg - t1 * g.tilesM) * BM;
    const int t2 = (int)const_div((unsigned)t1, g.by_tiles_x);
    const int ox0 = (t1 - t2 * g.tilesX) * g.tx;
    const int t3 = (int)const_div((unsigned)t2, g.by_tiles_y);
    const int oy0 = (t2 - t3 * g.tilesY) * g.ty;
    const int img0 = t3 * g.ni;

    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.a_parts), 0, (int)g.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p.B), 0, (int)g.b_bytes, 0x00020000);
    const int taps = p.cv_kh * p.cv_kw;
    const int plane = p.cv_H * p.cv_W;
    const int C = p.cv_C;
    const int PBUF = 3 * 2 * g.pp * 16;                 // bytes of one patch

    // ---- staging items: (pixel of the patch, group of 8 channels)
    unsigned boff[ITEMS];        // byte offset in channel 0 of the chunk, or kOutsideBytes
    int bslot[ITEMS];            // LDS byte offset of the leading part, -1: nothing to stage
    int bgrp[ITEMS];
#pragma unroll
    for (int t = 0; t < ITEMS; ++t) {
        const int id = t * LANES + tid - S0 * 64;
        const int grp = id >= g.ppr ? 1 : 0, q = id - grp * g.ppr;
        const int r1 = (int)const_div((unsigned)q, g.by_pw), px = q - r1 * g.pw;
        const int i = (int)const_div((unsigned)r1, g.by_ph), py = r1 - i * g.ph;
        const int iy = oy0 * p.cv_sh - p.cv_ph + py, ix = ox0 * p.cv_sw - p.cv_pw + px;
        const bool ok = q < g.ppr && img0 + i < g.N && (unsigned)iy < (unsigned)p.cv_H && (unsigned)ix < (unsigned)p.cv_W;
        const int xq = (int)const_div((unsigned)px, g.by_sw), xr = px - xq * p.cv_sw;
        bgrp[t] = grp;
        boff[t] = ok ? (unsigned)(((img0 + i) * C + grp * 8) * plane + iy * p.cv_W + ix) * 4u : kOutsideBytes;
        bslot[t] = q < g.ppr ? (grp * g.pp + (r1 * p.cv_sw + xr) * g.pws + xq) * 16 : -1;
    }

    float bst[ITEMS][8];
    auto load_b = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            if (t > 0 && t * LANES >= 2 * g.ppr) break;                  // uniform
            const int left = C - ch * kPatchChannels - bgrp[t] * 8;      // channels of the group
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = ch * kPatchChannels + e;                   // a scalar offset past the tensor would defeat the range check
                bst[t][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsB, (int)(e < left ? boff[t] : kOutsideBytes),
                                                                                 (int)((unsigned)((c < C ? c : C - 1) * plane) * 4u), 0));
            }
        }
    };
    auto store_b = [&](int buf) __attribute__((always_inline)) {
        char* d0 = smem + buf * PBUF;
#pragma unroll
        for (int t = 0; t < ITEMS; ++t) {
            if (t > 0 && t * LANES >= 2 * g.ppr) break;
            unsigned part[4][3];
#pragma unroll
            for (int h = 0; h < 4; ++h) split_pair<3>(bst[t][2 * h], bst[t][2 * h + 1], part[h], lost);
            if (bslot[t] >= 0) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<uintx4*>(d0 + bslot[t] + q * 2 * g.pp * 16) = uintx4{part[0][q], part[1][q], part[2][q], part[3][q]};
            }
        }
    };
    auto flag_lost = [&]() {                            // read behind a barrier
        const bool l = parts_lost(lost);
        if (lane == 0) wave_lost[wave - S0] = l ? 1 : 0;
    };

    if (NS > 0 && wave >= NW) {
        // patch ch + 1 is staged while the taps of chunk ch are multiplied, from pixels loaded during the chunk before
        load_b(0);
        store_b(0);
        if (g.nch > 1) load_b(1);
        lds_barrier();
#pragma unroll 1
        for (int ch = 0; ch < g.nch; ++ch) {
            if (g.nbuf == 1) lds_barrier();                  // the taps of this chunk have been read
            if (ch + 1 < g.nch) {
                store_b(g.nbuf == 2 ? (ch + 1) & 1 : 0);
                load_b(ch + 2 < g.nch ? ch + 2 : ch + 1);
            }
            if (ch + 1 == g.nch) flag_lost();
            lds_barrier();
        }
        return;
    }

    // ---- this lane's columns
    struct Col { int y, x, img; bool ok; };
    auto column = [&](int c) -> Col {
        const int u = (int)const_div((unsigned)c, g.by_tx), tx = c - u * g.tx;
        const int i = (int)const_div((unsigned)u, g.by_ty), ty = u - i * g.ty;
        Col r;
        r.img = i; r.y = ty; r.x = tx;
        r.ok = i < g.ni && img0 + i < g.N && oy0 + ty < g.Ho && ox0 + tx < p.cv_Wo;
        return r;
    };
    int b_slot[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const Col c = column(wn * (BN / WN) + j * 32 + lcol);
        b_slot[j] = (lrow * g.pp + (c.ok ? (c.img * g.ph + c.y * p.cv_sh) * (p.cv_sw * g.pws) + c.x : 0)) * 16;
    }

    // The products of the leading parts have sums of their own, one for every other tap: those round once per two taps, the small products round where
    // it does not show.
    floatx16 acc[TM][TN], odd[TM][TN], small[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = odd[i][j][r] = small[i][j][r] = 0.f;
    };
    clear();

    // Operands: the patch's one tap ahead, the weights' too, or three where a tap has few products (a trip to the L2 is longer) and the registers
    // hold them.  Weights: tap `u` of the whole reduction (chunk by chunk).
    constexpr int RING = NS == 0 || TM * TN > 1 ? 2 : 4;
    const int all_taps = g.nch * taps;
    const int mb0 = (m0 + wm * (BM / WM)) / 32;
    uintx4 av[RING][TM][3];
    bf16x8 bv[2][TN][3];
    auto read_a = [&](int u, uintx4 (&a)[TM][3]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                a[i][q] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rsA, lane * 16 + q * 1024,
                                                                                           (int)((unsigned)((mb0 + i) * all_taps + u) * 3072u), 0));
    };
    auto read_b = [&](const char* b0, bf16x8 (&b)[TN][3]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < 3; ++q) b[j][q] = *reinterpret_cast<const bf16x8*>(b0 + q * 2 * g.pp * 16 + b_slot[j]);
    };
    auto multiply = [&](const uintx4 (&a)[TM][3], const bf16x8 (&b)[TN][3], floatx16 (&lead)[TM][TN]) __attribute__((always_inline)) {
        constexpr int pa[6] = {0, 1, 1, 0, 2, 0}, pb[6] = {0, 1, 0, 1, 0, 2};
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    floatx16& sum = t == 0 ? lead[i][j] : small[i][j];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i][pa[t]]), b[j][pb[t]], sum, 0, 0, 0);
                }
    };
    // LDS byte offset of the tap after (ky, kx), the first one's behind the last
    int ky = 0, kx = 0;
    auto next_tap = [&]() -> int {
        if (++kx == p.cv_kw) { kx = 0; if (++ky == p.cv_kh) ky = 0; }
        const int dx = kx * p.cv_dw, xq = (int)const_div((unsigned)dx, g.by_sw), xr = dx - xq * p.cv_sw;
        return ((ky * p.cv_dh * p.cv_sw + xr) * g.pws + xq) * 16;
    };

    if (NS == 0) load_b(0);
#pragma unroll
    for (int r = 0; r < RING - 1; ++r) read_a(r < all_taps ? r : 0, av[r]);
    if (NS == 0) store_b(0);
    int u = RING - 2;                                   // the last tap whose weights were loaded
#pragma unroll 1
    for (int ch = 0; ch < g.nch; ++ch) {
        const char* patch = smem + (g.nbuf == 2 ? (ch & 1) * PBUF : 0);
        const bool more = NS == 0 && ch + 1 < g.nch;
        lds_barrier();
        if (more) load_b(ch + 1);
        read_b(patch, bv[0]);
        auto tap = [&](auto slot) __attribute__((always_inline)) {
            constexpr int I = decltype(slot)::value;
            ++u;
            read_a(u < all_taps ? u : 0, av[(I + RING - 1) % RING]);
            read_b(patch + next_tap(), bv[(I + 1) % 2]);
            __builtin_amdgcn_sched_barrier(0);          // or the reads move down to their use
            multiply(av[I], bv[I % 2], I % 2 == 0 ? acc : odd);
        };
        // the slots behind an incomplete round start the next chunk
        auto rotate = [&](auto by) __attribute__((always_inline)) {
            uintx4 t[RING][TM][3];
#pragma unroll
            for (int r = 0; r < RING; ++r)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int q = 0; q < 3; ++q) t[r][i][q] = av[(r + decltype(by)::value) % RING][i][q];
#pragma unroll
            for (int r = 0; r < RING - 1; ++r)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int q = 0; q < 3; ++q) av[r][i][q] = t[r][i][q];
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>;
        int t = 0;
#pragma unroll 1
        for (; t + RING <= taps; t += RING) {
            tap(I0{});
            tap(I1{});
            if constexpr (RING == 4) { tap(I2{}); tap(I3{}); }
        }
        const int rest = taps - t;
        if (rest == 1) { tap(I0{}); rotate(I1{}); }
        if constexpr (RING == 4) {
            if (rest == 2) { tap(I0{}); tap(I1{}); rotate(I2{}); }
            if (rest == 3) { tap(I0{}); tap(I1{}); tap(I2{}); rotate(I3{}); }
        }
        if (NS > 0 && g.nbuf == 1) lds_barrier();
        if (more) {
            if (g.nbuf == 1) lds_barrier();
            store_b(g.nbuf == 2 ? (ch + 1) & 1 : 0);
        }
    }
    if (NS == 0) flag_lost();
    lds_barrier();

    // A wavefront with sums that are not finite, and every wavefront of a workgroup that staged a value its parts do not hold, repeats its
    // block on the fp32 matrix instructions, inputs straight from memory (as in gemm_split.hip; the weights come out of their stored form with
    // all their bits)
    FiniteCheck check;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] += odd[i][j][r] + small[i][j][r];
                check.add(acc[i][j][r]);
            }
    int any_lost = 0;
#pragma unroll
    for (int w = 0; w < SW; ++w) any_lost |= wave_lost[w];
    if (check.failed() || __builtin_amdgcn_readfirstlane(any_lost) != 0) {
        clear();
        Col cs[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) cs[j] = column(wn * (BN / WN) + j * 32 + lcol);
#pragma unroll 1
        for (int v = 0; v < all_taps; ++v) {
            const int ch = v / taps, tap = v - ch * taps, fy = tap / p.cv_kw, fx = tap - fy * p.cv_kw;
            read_a(v, av[0]);
            const int c0 = ch * kPatchChannels + 8 * lrow;
            unsigned bc[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int iy = (oy0 + cs[j].y) * p.cv_sh - p.cv_ph + fy * p.cv_dh, ix = (ox0 + cs[j].x) * p.cv_sw - p.cv_pw + fx * p.cv_dw;
                const bool ok = cs[j].ok && (unsigned)iy < (unsigned)p.cv_H && (unsigned)ix < (unsigned)p.cv_W;
                bc[j] = ok ? (unsigned)(((img0 + cs[j].img) * C + c0) * plane + iy * p.cv_W + ix) * 4u : kOutsideBytes;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float xv[TN];
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    xv[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        rsB, (int)(c0 + e < C && bc[j] != kOutsideBytes ? bc[j] + (unsigned)(e * plane) * 4u : kOutsideBytes), 0, 0));
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const float wv = weight_value(av[0][i], e);
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, xv[j], acc[i][j], 0, 0, 0);
                }
            }
        }
    }

    // accumulator layout of v_mfma_f32_32x32x*: lane l holds column l % 32, rows 8 * (r / 4) + 4 * (l / 32) + r % 4
    if (g.vecD) {
        // four columns are four floats in a row: through a wavefront's own 32 x 32 tile in LDS, where the patch was, 16 bytes per lane and store
        // (gemm_epilogue.hpp)
        float* stage = reinterpret_cast<float*>(smem) + wave * kStageFloats;
        const int rrow = lane >> 3, rc4 = (lane & 7) * 4;
        float bias[TM][4];                                 // all at once: behind the bounds check of a row each would be a trip of its own
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int ps = 0; ps < 4; ++ps) {
                const int m = m0 + wm * (BM / WM) + i * 32 + ps * 8 + rrow;
                bias[i][ps] = p.bias ? p.bias[m < p.M ? m : p.M - 1] : 0.f;
            }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const Col c = column(wn * (BN / WN) + j * 32 + rc4);
            float* d0 = p.D + (long long)(img0 + c.img) * p.strideD_img + (long long)(oy0 + c.y) * p.cv_Wo + ox0 + c.x;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
#pragma unroll
                for (int r = 0; r < 16; ++r) stage[(8 * (r / 4) + 4 * lrow + (r % 4)) * kStageStride + lcol] = acc[i][j][r];
#pragma unroll
                for (int ps = 0; ps < 4; ++ps) {
                    const int row = ps * 8 + rrow, m = m0 + wm * (BM / WM) + i * 32 + row;
                    float4 v = *reinterpret_cast<const float4*>(&stage[row * kStageStride + rc4]);
                    if (c.ok && m < p.M) {
                        v.x += bias[i][ps]; v.y += bias[i][ps]; v.z += bias[i][ps]; v.w += bias[i][ps];
                        *reinterpret_cast<float4*>(d0 + (long long)m * p.strideD_row) = v;
                    }
                }
            }
        }
        return;
    }
    float bias[TM][16];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm * (BM / WM) + i * 32 + 8 * (r / 4) + 4 * lrow + r % 4;
            bias[i][r] = p.bias ? p.bias[m < p.M ? m : p.M - 1] : 0.f;
        }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const Col c = column(wn * (BN / WN) + j * 32 + lcol);
        if (!c.ok) continue;
        float* d0 = p.D + (long long)(img0 + c.img) * p.strideD_img + (long long)(oy0 + c.y) * p.cv_Wo + ox0 + c.x;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wm * (BM / WM) + i * 32 + 8 * (r / 4) + 4 * lrow + r % 4;
                if (m < p.M) d0[(long long)m * p.strideD_row] = acc[i][j][r] + bias[i][r];
            }
    }
}

constexpr int kPatchLds = 160 * 1024 - 1024;
constexpr int kPatchPixels = 768;            // of a patch that 128 columns see

bool choose_rectangle(const GemmProblem& p, int bn, PatchRect* out)
{
    return choose_patch_rect(p, bn, kPatchPixels * bn / 128, kPatchLds / 96, true, out);
}

template <int BM, int BN, int WM, int WN, int ITEMS, int NS>
hipError_t launch_patch_cfg(const GemmProblem& p, bool, hipStream_t s)
{
    constexpr int LANES = (NS > 0 ? NS : WM * WN) * 64, THREADS = (WM * WN + NS) * 64;
    static_assert(ITEMS * LANES / 2 >= kPatchPixels * BN / 128, "staging items for the largest patch");
    PatchArgs g{};
    unsigned plain = 0;
    if (!conv_patch_covers(p) || !p.a_parts || !choose_rectangle(p, BN, &g) || !gemm_operand_extents(p, &plain, &g.b_bytes)) return hipErrorInvalidValue;
    g.a_bytes = (unsigned)conv_patch_weight_bytes(p.M, p.cv_C, p.cv_kh * p.cv_kw);
    g.tilesM = (p.M + BM - 1) / BM;
    g.N = p.Ncols / p.L;
    g.Ho = p.L / p.cv_Wo;
    const long long total = (long long)g.tilesM * g.tilesX * g.tilesY * ((g.N + g.ni - 1) / g.ni);
    if (!grid_fits(total, THREADS)) return hipErrorInvalidValue;
    g.total = (int)total;
    g.nch = (p.cv_C + kPatchChannels - 1) / kPatchChannels;
    // a second patch buffer while two workgroups still fit a CU, or if one alone does
    const int one = g.pp * 96, stage = WM * WN * kStageFloats * 4;
    g.nbuf = g.nch > 1 && (2 * one <= kPatchLds / 2 || total <= 256) && 2 * one <= kPatchLds ? 2 : 1;
    g.vecD = g.vecD && (reinterpret_cast<uintptr_t>(p.D) & 15u) == 0 && p.strideD_img % 4 == 0 && p.strideD_row % 4 == 0;
    g.by_pw = make_constdiv((unsigned)g.pw);
    g.by_ph = make_constdiv((unsigned)g.ph);
    g.by_tx = make_constdiv((unsigned)g.tx);
    g.by_ty = make_constdiv((unsigned)g.ty);
    g.by_sw = make_constdiv((unsigned)p.cv_sw);
    g.by_tm = make_constdiv((unsigned)g.tilesM);
    g.by_tiles_x = make_constdiv((unsigned)g.tilesX);
    g.by_tiles_y = make_constdiv((unsigned)g.tilesY);
    hipLaunchKernelGGL((conv_patch_kernel<BM, BN, WM, WN, ITEMS, NS>), dim3((unsigned)total), dim3(THREADS), (size_t)(g.nbuf * one > stage ? g.nbuf * one : stage), s, p, g);
    return hipGetLastError();
}

const GemmVariant kPatch[] = {
    {"x6_patch_128x64_w4x1", launch_patch_cfg<128, 64, 4, 1, 3, 0>, 128, 64, 16},
    {"x6_patch_64x128_w2x2", launch_patch_cfg<64, 128, 2, 2, 6, 0>, 64, 128, 16},
    {"x6_patch_64x64_w2x2", launch_patch_cfg<64, 64, 2, 2, 3, 0>, 64, 64, 16},
    {"x6_patch_128x64_w4x1s4", launch_patch_cfg<128, 64, 4, 1, 3, 4>, 128, 64, 16},
    {"x6_patch_64x64_w2x2s4", launch_patch_cfg<64, 64, 2, 2, 3, 4>, 64, 64, 16},
};

}  // namespace

int conv_patch_variant_count() { return (int)(sizeof(kPatch) / sizeof(kPatch[0])); }
const GemmVariant& conv_patch_variant(int i) { return kPatch[i]; }

size_t conv_patch_weight_bytes(int K, int C, int taps)
{
    return (size_t)((K + 127) / 128 * 4) * ((C + kPatchChannels - 1) / kPatchChannels) * taps * 3072;      // whole blocks of 128 channels
}

// Fewer channels would leave a chunk of 16 more than half empty; one tap reads each value of a patch once.
bool conv_patch_offered(const GemmProblem& p) { return p.gather && p.prec == 0 && p.cv_C >= 8 && p.cv_kh * p.cv_kw > 1; }

bool conv_patch_covers(const GemmProblem& p)
{
    if (!p.gather || p.batch != 1 || p.prec != 0 || p.splitk > 1 || p.M <= 0 || p.L <= 0 || p.cv_Wo <= 0 || p.Ncols % p.L != 0) return false;
    if ((long long)p.M * p.R >= (1ll << 28) || conv_patch_weight_bytes(p.M, p.cv_C, p.cv_kh * p.cv_kw) >= ((size_t)1 << 31)) return false;
    unsigned a = 0, b = 0;
    PatchArgs g{};
    return gemm_operand_extents(p, &a, &b) && choose_rectangle(p, 64, &g) && choose_rectangle(p, 128, &g);
}

hipError_t launch_patch_weights(const float* w, void* Wp, int K, int C, int taps, hipStream_t s)
{
    if (!w || !Wp || K <= 0 || C <= 0 || taps <= 0) return hipErrorInvalidValue;
    const int nch = (C + kPatchChannels - 1) / kPatchChannels;
    const long long blocks = (long long)((K + 127) / 128 * 4) * nch;
    if (!grid_fits(blocks, 256)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(patch_weights_kernel, dim3((unsigned)blocks), dim3(256), 0, s, w, (uintx4*)Wp, K, C, taps, nch);
    return hipGetLastError();
}

}  // namespace mnnconv
