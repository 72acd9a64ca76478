// Winograd convolution one axis at a time (Section 3.3.1 of the MNN paper): V = B^T (d B) and y = A^T (m A) are two one-dimensional transforms
// each, and only the halves along the image width pass through memory.
//
//   rows in:   T[b][c][y][tx] = (d B)[y][b], every image row once: alpha / n values per input value, where V holds (alpha / n)^2
//   columns:   for one column b of the positions and all alpha rows a: V = B^T T in registers and LDS, the channel sums on the matrix cores,
//              S[b][i] = sum_a A^T[i][a] m[a][b]: alpha n values per tile and output channel, where M holds alpha^2
//   rows out:  y[i][j] = sum_b A^T[j][b] S[b][i] + bias
//
// F(4,7) on 16 x 64 x 112 x 112 moves 514 MB this way where separate transforms move 1.39 GB, for more vector instructions: a block of output channels
// transforms its tiles anew.  So it pays for few outputs per tile and many taps: kernels of 5 taps and more (F(6,3) on 16 x 128 x 64 x 64: 69 us against 72
// for separate kernels, F(8,3) 83 against 68).
// Measured against the best of the other arrangements, us: F(4,5) 16 x 128 x 64 x 64 125 -> 100, 8 x 256 x 56 x 56 139 -> 126; F(4,7) 16 x 64 x 112 x 112 222 -> 188;
// F(2,7) there 458 -> 357, 96 -> 192 channels on 8 x 80 x 80 367 -> 325.  Behind them where tiles are few (F(4,7) 4 x 128 x 28 x 28 39, 32; wino_cols_offered) and where
// channels are (F(4,5) 16 x 32 x 112 x 112 95, 60): the planner times all.
// Of the 188: rows in 30 and rows out 35 at 5 to 6 TB/s, columns 112 to 134, where the matrix cores are busy 23 % and the vector units 50 % of the cycles
// (F(4,5): 61 of 100, matrix cores 55 %).  Tried for that kernel: four wavefronts that stage and four that multiply, walking over blocks (F(4,7) 115,
// F(4,5) 85: one wavefront of a SIMD issues a vector instruction every 8 cycles where each needs the one before); the same walk with all
// eight doing both (registers spill); matrix and vector instructions interleaved by the compiler (F(4,5) 71); one buffer and two workgroups of
// four wavefronts per CU (F(4,5) 70, F(4,7) 192, spills).
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels.hpp"
#include "lds_barrier.hpp"
#include "xcd_remap.hpp"
#include "wino_paired.hpp"
#include "row_shares.hpp"
#include "tile_row.hpp"
#include "bf16_parts.hpp"
#include "fast_div.hpp"

namespace mnnconv {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kColsChunk = 16;               // channels per chunk
constexpr int kColsTiles = 64;               // tiles per workgroup

// 32-channel blocks per workgroup: four would be half empty up to 64 channels, and need more registers than there are from alpha = 9
inline int cols_kw(int K, int alpha) { return K <= 64 || alpha > 8 ? 2 : 4; }
inline int cols_mblocks(int K, int alpha) { const int kw = cols_kw(K, alpha); return (K + 32 * kw - 1) / (32 * kw) * kw; }
inline int cols_pblocks(int P) { return (P + kColsTiles - 1) / kColsTiles; }
inline int cols_chunks(int C) { return (C + kColsChunk - 1) / kColsChunk; }

// ---------------------------------------------------------------- prepared weights
// Uc[b][k/32][c/16][a]: lane l holds output channel l % 32 and channels 8 * (l / 32) .. + 7 of the chunk, as [part][lane][8 bf16] (weight_parts).
// Channels past K and C hold zeros.
struct ColsFilterMat { float g[kMaxAlphaT][7]; };

// One workgroup per 32 output channels x 16 input channels and share of the rows of G w G^T: rows grp, grp + groups, ... of `groups` shares, one
// for each `row_waves` wavefronts, which take turns at its columns.  Few blocks are a handful of workgroups, bound by the trips to memory for
// their weights: many loads at once, and a share per row.  us, a workgroup per block and a load at a time -> here: F(4,7) 64 -> 64 36 -> 12 (8 blocks, ten
// shares), F(4,5) 128 -> 128 18 -> 8, 256 -> 256 23 -> 13; F(4,7) 512 -> 512 99 -> 57 (one share; 157 MB of parts).
template <int KT>
__global__ __launch_bounds__(256) void cols_filter_kernel(int K, int C, int alpha, int mblocks, ColsFilterMat gm, const float* __restrict__ w,
                                                          uintx4* __restrict__ U, int nch, int groups, int row_waves)
{
    constexpr int RUN = kColsChunk * KT * KT, LD = RUN + 1, LOADS = 32 * RUN / 256;
    __shared__ float ws[32 * LD];
    const int block = (int)blockIdx.x / groups, grp = (int)blockIdx.x - block * groups;
    const int kb = block / nch, ch = block % nch;
    const int c_run = (C - ch * kColsChunk < kColsChunk ? C - ch * kColsChunk : kColsChunk) * KT * KT;
    constexpr int STEP = LOADS % 14 == 0 ? 14 : LOADS % 12 == 0 ? 12 : 10;
    static_assert(32 * RUN % 256 == 0 && LOADS % STEP == 0, "whole rounds of loads");
#pragma unroll 1
    for (int r = 0; r < LOADS; r += STEP) {
        float v[STEP];
#pragma unroll
        for (int t = 0; t < STEP; ++t) {
            const int i = (r + t) * 256 + (int)threadIdx.x, k = i / RUN, j = i % RUN;
            const bool ok = kb * 32 + k < K && j < c_run;
            v[t] = w[((long long)(ok ? kb * 32 + k : 0) * C + ch * kColsChunk) * KT * KT + (ok ? j : 0)];
            v[t] = ok ? v[t] : 0.f;
        }
#pragma unroll
        for (int t = 0; t < STEP; ++t) {
            const int i = (r + t) * 256 + (int)threadIdx.x;
            ws[i / RUN * LD + i % RUN] = v[t];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wrow = wave % row_waves, wcol = wave / row_waves, col_waves = 4 / row_waves;
    const float* wp = ws + (lane & 31) * LD + (lane >> 5) * 8 * KT * KT;
#pragma unroll 1
    for (int i = grp + groups * wrow; i < alpha; i += groups * row_waves) {
        float row[8][KT];                                     // row i of G w, 8 channels
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int s = 0; s < KT; ++s) {
                float acc = 0.f;
#pragma unroll
                for (int r = 0; r < KT; ++r) acc = fmaf(gm.g[i][r], wp[e * KT * KT + r * KT + s], acc);
                row[e][s] = acc;
            }
#pragma unroll 1
        for (int j = wcol; j < alpha; j += col_waves) {
            unsigned part[4][3];
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] = 0.f;
#pragma unroll
                for (int s = 0; s < KT; ++s) v[e] = fmaf(row[e][s], gm.g[j][s], v[e]);
            }
            weight_parts(v, part);
            uintx4* up = U + ((((long long)j * mblocks + kb) * nch + ch) * alpha + i) * 3 * 64 + lane;
#pragma unroll
            for (int q = 0; q < 3; ++q) up[q * 64] = uintx4{part[0][q], part[1][q], part[2][q], part[3][q]};
        }
    }
}

// ---------------------------------------------------------------- rows in
struct RowsArgs {
    int lanes;                   // C * N * H * tw
    int N, C, H, W, tw, pad_w, n;
    unsigned x_bytes;
    ConstDiv by_tw, by_h, by_n;
};

// One lane per (channel, image, row, tile of the row): a row's alpha values in 16- and 8-byte loads, alpha stores whose lanes are consecutive.
template <int A>
__global__ __launch_bounds__(256) void cols_rows_in_kernel(RowsArgs g, MatArg<A, A> bt, const float* __restrict__ x, float* __restrict__ T)
{
    const int idx = (int)(xcd_contiguous(blockIdx.x, gridDim.x) * 256 + threadIdx.x);
    const bool live = idx < g.lanes;
    const int r1 = (int)const_div((unsigned)idx, g.by_tw), tx = idx - r1 * g.tw;
    const int r2 = (int)const_div((unsigned)r1, g.by_h), y = r1 - r2 * g.H;
    const int c = (int)const_div((unsigned)r2, g.by_n), img = r2 - c * g.N;
    const int x0 = tx * g.n - g.pad_w;
    const int first = ((img * g.C + c) * g.H + y) * g.W + x0;            // elements; the tensor has fewer than 2^29
    float d[A];
    load_tile_row<A>(x, g.x_bytes, first, x0, g.W, live, d);
    float out[A];
    bt_apply<A>(bt, d, out);
    if (!live) return;
#pragma unroll
    for (int b = 0; b < A; ++b) (T + (long long)b * g.lanes)[idx] = out[b];
}

// ---------------------------------------------------------------- columns
struct ColsArgs {
    int C, H, th, tw, P, pad_h;
    int kblocks, pblocks, mblocks, nch;
    unsigned plane_bytes;        // of one channel of T[b]: N * H * tw floats
    unsigned t_bytes, u_bytes;   // of one column b
    ConstDiv by_kblocks, by_pblocks, by_tw, by_th;
};

// KW blocks of 32 output channels x 64 tiles, eight wavefronts: wavefront kt + KW grp owns block kt and a share of the alpha rows for both
// 32-tile blocks, so that a weight operand serves two products and the two wavefronts of a SIMD have alpha / 2 (KW = 2) or alpha (KW = 4) rows.
// LDS: V as [a][part][channel pair][tile][2 bf16], lane = tile when it is written; two buffers, and the wavefronts of a SIMD take turns: one
// stages the next chunk while the other multiplies.
template <int NT, int A, int KW>
__global__ __launch_bounds__(512, 2) void cols_kernel(ColsArgs g, MatArg<A, A> bt, MatArg<NT, A> at, const float* __restrict__ T,
                                                      const void* __restrict__ U, float* __restrict__ S)
{
    constexpr int NW = 8, Q = NW / KW;                    // wavefronts, shares of the rows
    constexpr int A0 = (A + Q - 1) / Q;                   // rows of the larger shares
    constexpr int POS = 3 * 8 * 256;                      // bytes of one position
    constexpr int VBUF = A * POS;
    constexpr int XSLOT = NW * (Q - 1) * 4096;            // one exchange of sums
    constexpr int LDS = 2 * VBUF > XSLOT ? 2 * VBUF : XSLOT;
    static_assert(LDS <= 160 * 1024 - 64, "LDS");
    __shared__ __attribute__((aligned(16))) char smem[LDS];
    __shared__ int redo;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kt = wave % KW, grp = wave / KW;
    const int lh = lane >> 5, l32 = lane & 31;

    // output-channel blocks fastest: they share the tiles; the position column slowest: its weights stay in an XCD's L2
    const int wg = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int t1 = (int)const_div((unsigned)wg, g.by_kblocks);
    const int kb = wg - t1 * g.kblocks;
    const int b = (int)const_div((unsigned)t1, g.by_pblocks);
    const int pb = t1 - b * g.pblocks;
    const int mb = kb * KW + kt;

    const float* Tb = T + (long long)b * (g.t_bytes / 4u);
    const char* Ub = static_cast<const char*>(U) + (long long)b * g.u_bytes;
    const __amdgpu_buffer_rsrc_t rsT = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Tb), 0, (int)g.t_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsU = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Ub), 0, (int)g.u_bytes, 0x00020000);

    // byte offsets in channel 0 of the alpha rows that tile p sees, kOutsideBytes above and below the image
    auto rows = [&](int p, unsigned (&off)[A]) __attribute__((always_inline)) {
        const int r1 = (int)const_div((unsigned)p, g.by_tw), tx = p - r1 * g.tw;
        const int img = (int)const_div((unsigned)r1, g.by_th), ty = r1 - img * g.th;
        const int y0 = ty * NT - g.pad_h;
#pragma unroll
        for (int a = 0; a < A; ++a)
            off[a] = p < g.P && (unsigned)(y0 + a) < (unsigned)g.H ? (unsigned)((img * g.H + y0 + a) * g.tw + tx) * 4u : kOutsideBytes;
    };
    unsigned off[A];
    rows(pb * kColsTiles + lane, off);

    unsigned lost = 0;
    float tv[2][A];
    // a channel past the last reads that one again: its weights are zero
    auto load_t = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int c = ch * kColsChunk + wave * 2 + e;
            const unsigned so = (unsigned)(c < g.C ? c : g.C - 1) * g.plane_bytes;
#pragma unroll
            for (int a = 0; a < A; ++a) tv[e][a] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsT, (int)off[a], (int)so, 0));
        }
    };
    auto stage = [&](int buf) __attribute__((always_inline)) {
        float v0[A], v1[A];
        bt_apply<A>(bt, tv[0], v0);
        bt_apply<A>(bt, tv[1], v1);
        char* d0 = smem + buf * VBUF + wave * 256 + lane * 4;
#pragma unroll
        for (int a = 0; a < A; ++a) {
            unsigned part[3];
            split_pair<3>(v0[a], v1[a], part, lost);
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<unsigned*>(d0 + a * POS + q * 2048) = part[q];
        }
    };
    floatx16 acc[A0][2];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < A0; ++q)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[q][j][r] = 0.f;
    };
    // rows a0 .. a0 + mine - 1
    constexpr int MORE = A % Q;
    const int mine = row_share(A, Q, grp).rows, a0 = row_share(A, Q, grp).first;
    const unsigned u0 = (unsigned)(mb * g.nch * A + a0) * 3072u;
    uintx4 u[2][3];
    auto load_u = [&](int ch, int q, uintx4 (&v)[3]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 3; ++s)
            v[s] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(rsU, lane * 16 + s * 1024, (int)(u0 + (unsigned)(ch * A + q) * 3072u), 0));
    };
    auto multiply = [&](int ch, int buf) __attribute__((always_inline)) {
        const char* v0 = smem + buf * VBUF + a0 * POS + lh * 1024 + l32 * 4;
        const int next = ch + 1 < g.nch ? ch + 1 : ch;
        uintx4 bv[2][3];
        auto load_v = [&](int q, int j) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) bv[j][s][e] = *reinterpret_cast<const unsigned*>(v0 + q * POS + s * 2048 + e * 256 + j * 128);
        };
        load_v(0, 0);
#pragma unroll
        for (int q = 0; q < A0; ++q) {
            const bool final = q + 1 == A0;
            if (MORE != 0 && final && q >= mine) {                  // a smaller share
                load_u(next, 0, u[(q + 1) & 1]);
                continue;
            }
            // operands one product ahead: weights a row, V a tile block
            const int ahead = row_of_step(A, Q, grp, q + 1);
            load_u(final ? next : ch, final ? 0 : ahead, u[(q + 1) & 1]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (j == 0) load_v(q, 1);
                else if (!final) load_v(ahead, 0);
                __builtin_amdgcn_sched_barrier(0);                  // or the reads move down to their use
                constexpr int pa[6] = {1, 2, 0, 1, 0, 0}, pv[6] = {1, 0, 2, 0, 1, 0};     // small products first
#pragma unroll
                for (int s = 0; s < 6; ++s)
                    acc[q][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u[q & 1][pa[s]]), __builtin_bit_cast(bf16x8, bv[j][pv[s]]),
                                                                       acc[q][j], 0, 0, 0);
            }
        }
        if (A0 % 2 != 0) {
#pragma unroll
            for (int s = 0; s < 3; ++s) u[0][s] = u[1][s];
        }
    };

    clear();
    load_t(0);
    load_u(0, 0, u[0]);
    const int last = g.nch - 1;
    auto ahead = [&](int c) { return c + 2 < last ? c + 2 : last; };
    stage(0);
    load_t(last < 1 ? last : 1);
    lds_barrier();
    if (wave < NW / 2) {
#pragma unroll 1
        for (int c = 0; c < last; ++c) {
            multiply(c, c & 1);
            stage((c + 1) & 1);
            load_t(ahead(c));
            lds_barrier();
        }
    } else {
#pragma unroll 1
        for (int c = 0; c < last; ++c) {
            stage((c + 1) & 1);
            load_t(ahead(c));
            multiply(c, c & 1);
            lds_barrier();
        }
    }
    multiply(last, last & 1);

    // A workgroup with sums that are not finite, or with a transformed input that its parts do not hold, repeats the channels on the fp32 matrix
    // instructions (as in gemm_split.hip; the weights come out of their stored form with all their bits)
    if (tid == 0) redo = 0;
    lds_barrier();
    FiniteCheck check;
#pragma unroll
    for (int q = 0; q < A0; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) check.add(acc[q][j][r]);
    if ((check.failed() || parts_lost(lost)) && lane == 0) redo = 1;
    lds_barrier();
    if (__builtin_amdgcn_readfirstlane(redo) != 0) {
        clear();
#pragma unroll 1
        for (int cc = 0; cc < g.nch * 8; ++cc) {          // channel e of either half's octet
            const int ch = cc >> 3, e = cc & 7, c = ch * kColsChunk + 8 * lh + e;
#pragma unroll 1
            for (int j = 0; j < 2; ++j) {
                unsigned o[A];
                float t[A], v[A];
                rows(pb * kColsTiles + j * 32 + l32, o);
#pragma unroll
                for (int a = 0; a < A; ++a)
                    t[a] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        rsT, (int)(c < g.C && o[a] != kOutsideBytes ? o[a] + (unsigned)c * g.plane_bytes : kOutsideBytes), 0, 0));
                bt_apply<A>(bt, t, v);
#pragma unroll
                for (int q = 0; q < A0; ++q) {
                    if (q >= mine) continue;
                    unsigned part[3];
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        const unsigned two = __builtin_amdgcn_raw_buffer_load_b32(rsU, lane * 16 + s * 1024 + (e >> 1) * 4,
                                                                                 (int)(u0 + (unsigned)(ch * A + q) * 3072u), 0);
                        part[s] = e & 1 ? two & 0xFFFF0000u : two << 16;
                    }
                    const float wv = weight_value(part);
                    float vv = v[q];
#pragma unroll
                    for (int h = 1; h < Q; ++h) {
                        constexpr int kLast = A - 1;
                        const int a = q + row_share(A, Q, h).first;
                        if (grp == h) vv = v[a < A ? a : kLast];
                    }
                    if (j == 0) acc[q][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, vv, acc[q][0], 0, 0, 0);
                    else acc[q][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, vv, acc[q][1], 0, 0, 0);
                }
            }
        }
    }

    // ---- A^T along the rows: every share sums its own, then the wavefronts of a channel block exchange.  Of Q results (tile block o % 2, row
    // i + o / 2) share o finishes one: it adds the others in their order and stores it.
    const int pairs = 2 * g.pblocks;
    auto fold = [&](auto h) __attribute__((always_inline)) {
        constexpr int H = decltype(h)::value;
        constexpr int FIRST = row_share(A, Q, H).first, COUNT = row_share(A, Q, H).rows;
        constexpr int RI = Q / 2, MERGE = LDS / XSLOT;                  // rows of S per exchange slot, slots per pair of barriers
        auto sum = [&](int i, int j, int r) __attribute__((always_inline)) {
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < COUNT; ++q) s = fmaf(at.v[i][FIRST + q], acc[q][j][r], s);
            return s;
        };
#pragma unroll
        for (int i0 = 0; i0 < NT; i0 += RI * MERGE) {
            lds_barrier();                                    // V, or what the round before left, has been read
#pragma unroll
            for (int m = 0; m < MERGE; ++m)
#pragma unroll
                for (int o = 0; o < Q; ++o) {
                    const int i = i0 + m * RI + o / 2;
                    if (o == H || i >= NT) continue;
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4)
                        *reinterpret_cast<float4*>(smem + ((m * NW + wave) * (Q - 1) + o - (o > H ? 1 : 0)) * 4096 + r4 * 1024 + lane * 16) =
                            make_float4(sum(i, o % 2, 4 * r4), sum(i, o % 2, 4 * r4 + 1), sum(i, o % 2, 4 * r4 + 2), sum(i, o % 2, 4 * r4 + 3));
                }
            lds_barrier();
#pragma unroll
            for (int m = 0; m < MERGE; ++m) {
                const int i = i0 + m * RI + H / 2;
                if (i >= NT) continue;
                float* dst = S + ((((long long)b * NT + i) * g.mblocks + mb) * pairs + pb * 2 + H % 2) * 1024;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                    for (int o = 0; o < Q; ++o) {
                        float4 v;
                        if (o == H) v = make_float4(sum(i, H % 2, 4 * r4), sum(i, H % 2, 4 * r4 + 1), sum(i, H % 2, 4 * r4 + 2), sum(i, H % 2, 4 * r4 + 3));
                        else v = *reinterpret_cast<const float4*>(smem + ((m * NW + kt + KW * o) * (Q - 1) + H - (H > o ? 1 : 0)) * 4096 + r4 * 1024 + lane * 16);
                        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
                    }
                    *reinterpret_cast<float4*>(dst + r4 * 256 + lane * 4) = t;
                }
            }
        }
    };
    if (grp == 0) fold(std::integral_constant<int, 0>{});
    else if (grp == 1) fold(std::integral_constant<int, 1>{});
    else if constexpr (Q == 4) {
        if (grp == 2) fold(std::integral_constant<int, 2>{});
        else fold(std::integral_constant<int, 3>{});
    }
}

// ---------------------------------------------------------------- rows out
struct RowsOutArgs {
    int K, Ho, Wo, th, tw, P;
    int mblocks, pairs;          // 32-channel and 32-tile blocks of S
    int vec;                     // 2: 16-byte stores of whole tile rows, 1: pairs, 0: single values
    ConstDiv by_pairs, by_n, by_tw, by_th;
};

// One workgroup per (32 channels, row i of the tiles, 32 tiles); a lane holds four channels of one tile, as the accumulators left them.
// STREAM: S is too large to stay in the last-level cache, and this, its last read, goes past the caches instead of evicting what comes next.  Whole
// calls, us, through the caches and past them: S of 67 MB (F(4,5) 16 x 128 x 64 x 64) 94.9 and 95.9, 101 MB (24 images) 142 and 146, 113 MB (F(4,7)
// 14 x 64 x 112 x 112) 154 and 158, 128 MB (16) 187 and 179, 134 MB 203 and 196, 154 MB (F(2,7), 12) 270 and 259, 179 MB (F(6,5) 16 x 64 -> 128) 238 and 217.
template <int NT, int A, bool STREAM>
__global__ __launch_bounds__(256) void cols_rows_out_kernel(RowsOutArgs g, MatArg<NT, A> at, const float* __restrict__ S,
                                                            const float* __restrict__ bias, float* __restrict__ y)
{
    const int wg = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int t1 = (int)const_div((unsigned)wg, g.by_n), i = wg - t1 * NT;
    const int mb = (int)const_div((unsigned)t1, g.by_pairs), pp = t1 - mb * g.pairs;
    const int lane = threadIdx.x & 63, r4 = threadIdx.x >> 6;
    const float* src = S + (((long long)i * g.mblocks + mb) * g.pairs + pp) * 1024 + r4 * 256 + lane * 4;
    const long long step = (long long)NT * g.mblocks * g.pairs * 1024;
    float in[4][A];
#pragma unroll
    for (int b = 0; b < A; ++b) {
        const floatx4* q = reinterpret_cast<const floatx4*>(src + b * step);
        const floatx4 v = STREAM ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
        for (int e = 0; e < 4; ++e) in[e][b] = v[e];
    }
    const int p = pp * 32 + (lane & 31), k0 = mb * 32 + 8 * r4 + 4 * (lane >> 5);
    const int r1 = (int)const_div((unsigned)p, g.by_tw), tx = p - r1 * g.tw;
    const int img = (int)const_div((unsigned)r1, g.by_th), ty = r1 - img * g.th;
    const int oy = ty * NT + i;
    if (p >= g.P || oy >= g.Ho) return;
    const bool whole = tx * NT + NT <= g.Wo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int k = k0 + e;
        if (k >= g.K) break;
        float o[NT];
        at_apply<NT, A>(at, in[e], bias ? bias[k] : 0.f, o);
        float* row = y + (((long long)img * g.K + k) * g.Ho + oy) * g.Wo + tx * NT;
        if (NT % 4 == 0 && g.vec == 2) {
#pragma unroll
            for (int j = 0; j + 3 < NT; j += 4) *reinterpret_cast<float4*>(row + j) = make_float4(o[j], o[j + 1], o[j + 2], o[j + 3]);
        } else if (NT % 2 == 0 && g.vec >= 1 && whole) {
#pragma unroll
            for (int j = 0; j + 1 < NT; j += 2) *reinterpret_cast<float2*>(row + j) = make_float2(o[j], o[j + 1]);
        } else {
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if (tx * NT + j < g.Wo) row[j] = o[j];
        }
    }
}

template <int A>
MatArg<A, A> bt_arg(const float* BT)
{
    MatArg<A, A> m;
    for (int i = 0; i < A; ++i)
        for (int j = 0; j < A; ++j) m.v[i][j] = BT[i * A + j];
    return m;
}

template <int NT, int A>
MatArg<NT, A> at_arg(const float* AT)
{
    MatArg<NT, A> m;
    for (int i = 0; i < NT; ++i)
        for (int j = 0; j < A; ++j) m.v[i][j] = AT[i * A + j];
    return m;
}

size_t cols_column_bytes(const WinoGeom& g) { return (size_t)cols_mblocks(g.K, g.alpha) * cols_chunks(g.C) * g.alpha * 3072; }
long long cols_row_tiles(const WinoGeom& g) { return (long long)g.N * g.H * g.tw; }

bool cols_geom_ok(const WinoGeom& g)
{
    if (g.nw != g.n || g.kw != g.k || g.alpha != g.n + g.k - 1 || g.N <= 0 || g.C <= 0 || g.H <= 0 || g.W <= 0 || g.K <= 0) return false;
    if (g.Ho != g.H + 2 * g.pad_h - g.k + 1 || g.Wo != g.W + 2 * g.pad_w - g.k + 1 || g.Ho <= 0 || g.Wo <= 0) return false;
    if (g.th != (g.Ho + g.n - 1) / g.n || g.tw != (g.Wo + g.n - 1) / g.n || (long long)g.P != (long long)g.N * g.th * g.tw) return false;
    return wino_cols_covers(g);
}

}  // namespace

bool wino_cols_available(int n, int k) { return k >= 5 && n >= 2 && n + k - 1 >= 7 && winograd_kernels_available(n, k); }

// Every product below is of values below 2^31, and is checked before the next factor.
bool wino_cols_covers(const WinoGeom& g)
{
    if (!wino_cols_available(g.n, g.k) || g.C <= 0 || g.K <= 0 || g.N <= 0 || g.H <= 0 || g.W <= 0 || g.th <= 0 || g.tw <= 0) return false;
    const long long limit = (1ll << 31) - 4096;
    const long long plane = (long long)g.N * g.H, rows = plane < limit ? plane * g.tw : limit;
    if (plane >= limit || plane * g.W >= limit || plane * g.W * g.C * 4 >= limit || rows >= limit || rows * g.C * 4 >= limit) return false;
    const long long P = (long long)g.N * g.th * g.tw;                    // below 2^31: as rows, but for padding
    if ((long long)g.N * g.th >= limit || P >= (1ll << 30) || (long long)g.K * g.C >= (1ll << 27)) return false;
    if (cols_column_bytes(g) >= (size_t)limit) return false;
    const long long mb = cols_mblocks(g.K, g.alpha), pb = cols_pblocks((int)P), kb = mb / cols_kw(g.K, g.alpha);
    if (!grid_fits((rows * g.C + 255) / 256, 256) || !grid_fits(kb * pb * g.alpha, 512)) return false;
    return pb < (1ll << 24) && mb < (1ll << 20) && mb * pb < (1ll << 28) && grid_fits(mb * 2 * pb * g.n, 256);
}

// Few workgroups of the columns kernel walk all channels each while the others' products fill the chip: of 75 layers with fewer than 32 it won none (0.83 of
// the speed at best), of 50 with 32 to 63 two (1.14), of 62 with 64 to 255 twelve (1.50).  Timing it took as long as the other arrangements together
// (planning F(6,5) 2 x 85 -> 175 9 x 11 4.4 ms, 2.8 without it).
bool wino_cols_offered(const WinoGeom& g)
{
    const long long P = (long long)g.N * g.th * g.tw;
    return (P + kColsTiles - 1) / kColsTiles * (cols_mblocks(g.K, g.alpha) / cols_kw(g.K, g.alpha)) * g.alpha >= 32;
}

size_t wino_cols_weight_bytes(const WinoGeom& g) { return cols_column_bytes(g) * g.alpha; }
size_t wino_cols_input_bytes(const WinoGeom& g) { return (size_t)cols_row_tiles(g) * g.C * g.alpha * sizeof(float); }
size_t wino_cols_sum_bytes(const WinoGeom& g) { return (size_t)g.alpha * g.n * cols_mblocks(g.K, g.alpha) * 2 * cols_pblocks(g.P) * 4096; }

hipError_t launch_cols_filter(const WinoGeom& g, const float* G, const float* w, void* U, hipStream_t s)
{
    if (!G || !w || !U || !cols_geom_ok(g)) return hipErrorInvalidValue;
    ColsFilterMat m;
    for (int i = 0; i < kMaxAlphaT; ++i)
        for (int j = 0; j < 7; ++j) m.g[i][j] = (i < g.alpha && j < g.k) ? G[i * g.k + j] : 0.f;
    const int mb = cols_mblocks(g.K, g.alpha), nch = cols_chunks(g.C);
    const int blocks = mb * nch;                          // K C < 2^27: fewer than 2^19
    const int groups = blocks >= 256 ? 1 : 256 / blocks < g.alpha ? 256 / blocks : g.alpha;
    const int rows = (g.alpha + groups - 1) / groups, row_waves = rows >= 4 ? 4 : rows >= 2 ? 2 : 1;
    const dim3 grid((unsigned)(blocks * groups));
    switch (g.k) {
#define MNN_FILTER(KT_) case KT_: hipLaunchKernelGGL(cols_filter_kernel<KT_>, grid, dim3(256), 0, s, g.K, g.C, g.alpha, mb, m, w, (uintx4*)U, nch, groups, row_waves); break;
        MNN_FILTER(5) MNN_FILTER(6) MNN_FILTER(7)
#undef MNN_FILTER
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_cols_rows_in(const WinoGeom& g, const float* BT, const float* x, float* T, hipStream_t s)
{
    if (!BT || !x || !T || !cols_geom_ok(g) || (g.alpha % 2 == 0 && !bt_is_paired(BT, g.alpha))) return hipErrorInvalidValue;
    RowsArgs a{};
    a.lanes = (int)(cols_row_tiles(g) * g.C);
    a.N = g.N; a.C = g.C; a.H = g.H; a.W = g.W; a.tw = g.tw; a.pad_w = g.pad_w; a.n = g.n;
    a.x_bytes = (unsigned)((long long)g.N * g.C * g.H * g.W * 4);
    a.by_tw = make_constdiv((unsigned)g.tw); a.by_h = make_constdiv((unsigned)g.H); a.by_n = make_constdiv((unsigned)g.N);
    const dim3 grid((unsigned)((a.lanes + 255ll) / 256));
    switch (g.alpha) {
#define MNN_A(A_) case A_: hipLaunchKernelGGL(cols_rows_in_kernel<A_>, grid, dim3(256), 0, s, a, bt_arg<A_>(BT), x, T); break;
        MNN_A(7) MNN_A(8) MNN_A(9) MNN_A(10)
#undef MNN_A
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

namespace {

template <int NT, int A>
hipError_t launch_cols_t(const WinoGeom& g, const float* BT, const float* AT, const float* T, const void* U, float* S, hipStream_t s)
{
    const int kw = cols_kw(g.K, g.alpha);
    ColsArgs a{};
    a.C = g.C; a.H = g.H; a.th = g.th; a.tw = g.tw; a.P = g.P; a.pad_h = g.pad_h;
    a.mblocks = cols_mblocks(g.K, g.alpha); a.kblocks = a.mblocks / kw; a.pblocks = cols_pblocks(g.P); a.nch = cols_chunks(g.C);
    a.plane_bytes = (unsigned)(cols_row_tiles(g) * 4);
    a.t_bytes = (unsigned)(cols_row_tiles(g) * g.C * 4);
    a.u_bytes = (unsigned)cols_column_bytes(g);
    a.by_kblocks = make_constdiv((unsigned)a.kblocks); a.by_pblocks = make_constdiv((unsigned)a.pblocks);
    a.by_tw = make_constdiv((unsigned)g.tw); a.by_th = make_constdiv((unsigned)g.th);
    const dim3 grid((unsigned)((long long)a.kblocks * a.pblocks * A)), block(512);
    if constexpr (A <= 8) {
        if (kw == 4) {
            hipLaunchKernelGGL((cols_kernel<NT, A, 4>), grid, block, 0, s, a, bt_arg<A>(BT), at_arg<NT, A>(AT), T, U, S);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((cols_kernel<NT, A, 2>), grid, block, 0, s, a, bt_arg<A>(BT), at_arg<NT, A>(AT), T, U, S);
    return hipGetLastError();
}

template <int NT, int A>
hipError_t launch_rows_out_t(const WinoGeom& g, const float* AT, const float* S, const float* bias, float* y, hipStream_t s)
{
    RowsOutArgs a{};
    a.K = g.K; a.Ho = g.Ho; a.Wo = g.Wo; a.th = g.th; a.tw = g.tw; a.P = g.P;
    a.mblocks = cols_mblocks(g.K, g.alpha); a.pairs = 2 * cols_pblocks(g.P);
    a.vec = (NT % 4 == 0 && g.Wo % NT == 0 && (reinterpret_cast<uintptr_t>(y) & 15u) == 0) ? 2
            : (NT % 2 == 0 && g.Wo % 2 == 0 && (reinterpret_cast<uintptr_t>(y) & 7u) == 0) ? 1 : 0;
    a.by_pairs = make_constdiv((unsigned)a.pairs); a.by_n = make_constdiv((unsigned)NT);
    a.by_tw = make_constdiv((unsigned)g.tw); a.by_th = make_constdiv((unsigned)g.th);
    const dim3 grid((unsigned)((long long)a.mblocks * a.pairs * NT));
    if (wino_cols_sum_bytes(g) > 120000000)
        hipLaunchKernelGGL((cols_rows_out_kernel<NT, A, true>), grid, dim3(256), 0, s, a, at_arg<NT, A>(AT), S, bias, y);
    else
        hipLaunchKernelGGL((cols_rows_out_kernel<NT, A, false>), grid, dim3(256), 0, s, a, at_arg<NT, A>(AT), S, bias, y);
    return hipGetLastError();
}

}  // namespace

#define MNN_COLS_ALL(X) \
    X(3, 5) X(4, 5) X(5, 5) X(6, 5) X(2, 6) X(3, 6) X(4, 6) X(5, 6) X(2, 7) X(3, 7) X(4, 7)

hipError_t launch_cols(const WinoGeom& g, const float* BT, const float* AT, const float* T, const void* U, float* S, hipStream_t s)
{
    if (!BT || !AT || !T || !U || !S || !cols_geom_ok(g) || (g.alpha % 2 == 0 && !bt_is_paired(BT, g.alpha))) return hipErrorInvalidValue;
#define MNN_X(NN, KK) if (g.n == NN && g.k == KK) return launch_cols_t<NN, NN + KK - 1>(g, BT, AT, T, U, S, s);
    MNN_COLS_ALL(MNN_X)
#undef MNN_X
    return hipErrorInvalidValue;
}

hipError_t launch_cols_rows_out(const WinoGeom& g, const float* AT, const float* S, const float* bias, float* y, hipStream_t s)
{
    if (!AT || !S || !y || !cols_geom_ok(g) || (g.alpha % 2 == 0 && !at_is_paired(AT, g.n, g.alpha))) return hipErrorInvalidValue;
#define MNN_X(NN, KK) if (g.n == NN && g.k == KK) return launch_rows_out_t<NN, NN + KK - 1>(g, AT, S, bias, y, s);
    MNN_COLS_ALL(MNN_X)
#undef MNN_X
    return hipErrorInvalidValue;
}

}  // namespace mnnconv
