// Sliding window for grids too short to fill the chip several times over, with weights prepared in operand order and staged patches.
//
// gemm_short.hip gathers every operand value by itself: a 16 x 16 tile spends, per tap and 32 channels, sixteen 4-byte loads on 256 cycles of matrix
// instructions, and an input value is loaded (and cut into parts) once per tap.  Here the weights lie as the matrix instruction reads them (two or three
// 16-byte loads), and a workgroup keeps the patch of the image that its pixels see in LDS, all channels at once where they fit: one trip to memory, one
// barrier.  A tap is an offset into the patch.  The wavefronts divide the steps (64 / S times 8 channels, tap) evenly, each into sums of its own, which
// are added through LDS in wavefront order (the same bits every run).
//
// What bounds it, 3 x 3 256 -> 256 on one 14 x 14 image, 16 x 16 tiles in fp32, us into the kernel (6.0 of the 7.2 that a call takes): arguments 0.4, places
// worked out 0.6, patch in LDS 2.6 (one trip 1.1, the rest its 24 loads per lane), products 4.9 (2.0 of matrix instructions), partial tiles across LDS
// and stored 5.9.  512 -> 512 on 7 x 7: 128 workgroups, on which weights arrive at 30 bytes per cycle, whether as fp32 (10.8 us) or as bf16 parts (11.4).
// Measured against the best of the other configurations, us per call, weights not in the L2: one image, 64 -> 64 56 x 56 7.1 -> 6.2, stride 2 128 -> 256
// 28 x 28 7.6 -> 6.3, 256 -> 256 14 x 14 11.1 -> 7.2, stride 2 256 -> 512 14 x 14 12.7 -> 8.6, 512 -> 512 7 x 7 11.4 with a second kernel -> 10.8; 8 images
// stride 2 256 -> 512 14 x 14 20.0 -> 15.9, 16 images 512 -> 512 7 x 7 40 -> 29; 5 x 5 264 -> 84 on 2 x 32 x 36 36.8 -> 24.3.  The planner times them next to
// the others, which stay ahead where a patch is mostly halo or channels leave a step half empty (stride 2 64 -> 128 56 x 56 6.4 against 6.8).
// Relative error of 256 -> 256 3.1e-7 in fp32 before, 2.2e-7 here (two sums per wavefront), in parts 1.1e-7.
// Tried: 32 x 16 tiles in fp32 (7.7 to 15, never ahead), 16 x 16 in parts (no faster: weights), sixteen wavefronts (slower everywhere).
#include <hip/hip_runtime.h>
#include <type_traits>
#include "kernels.hpp"
#include "lds_barrier.hpp"
#include "xcd_remap.hpp"
#include "fast_div.hpp"
#include "patch_rect.hpp"
#include "bf16_parts.hpp"

namespace mnnconv {
namespace {

constexpr int kShortPixels = 512;            // of a patch: a lane each
constexpr int kShortTaps = 64;               // a lane each
constexpr int kShortLds = 160 * 1024 - 1024;

// S x S matrix instructions.  Eight reduction rows per lane and step, 64 / S lanes per row or column.  An operand of eight values is NP times 16 bytes:
// two halves in fp32, or three bf16 parts.
template <bool PARTS> struct Matrix;
template <> struct Matrix<false> {
    typedef float acc_t __attribute__((ext_vector_type(4)));
    static constexpr int S = 16, NP = 2, REGS = 4;
    static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + r; }
    // the sums take turns
    static __device__ __forceinline__ void multiply(const uintx4 (&a)[NP], const uintx4 (&b)[NP], acc_t (&sums)[2])
    {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            sums[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e / 4][e % 4]), __uint_as_float(b[e / 4][e % 4]), sums[e & 1], 0, 0, 0);
    }
};
template <> struct Matrix<true> {
    typedef float acc_t __attribute__((ext_vector_type(16)));
    static constexpr int S = 32, NP = 3, REGS = 16;
    static __device__ __forceinline__ int row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
    // the products of the leading parts have a sum of their own
    static __device__ __forceinline__ void multiply(const uintx4 (&a)[NP], const uintx4 (&b)[NP], acc_t (&sums)[2])
    {
        constexpr int pa[6] = {0, 1, 1, 0, 2, 0}, pb[6] = {0, 1, 0, 1, 0, 2};
#pragma unroll
        for (int t = 0; t < 6; ++t)
            sums[t > 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[pa[t]]), __builtin_bit_cast(bf16x8, b[pb[t]]), sums[t > 0], 0, 0, 0);
    }
};
constexpr int kOctetRows = Matrix<false>::S, kOctetChannels = 512 / kOctetRows;

struct ConvShortArgs : PatchRect {
    const void* w; const float* x; float* y; const float* bias;
    long long sImg, sRow;
    int M, C, H, W, N, Ho, Wo;
    int kw, taps, sh, sw, pad_h, pad_w, dh, dw;
    int tilesM, tilesP, total;
    int m_first;                 // workgroups that follow each other share the pixels, not the weights
    int nch, cpr;                // chunks of channels, as many as LDS holds at once
    int gstep;                   // groups of 8 channels that the workgroup stages at a time, a lane per pixel and group
    unsigned a_bytes, b_bytes;
    ConstDiv by_inner, by_pw, by_ph, by_ppr, by_tx, by_ty, by_sw, by_kw, by_taps, by_tiles_x, by_tiles_y;
};

// Wq[m/16][c/32][tap][half][lane][4]: lane l holds output channel l % 16 and channels 8 * (l / 16) + 4 * half .. + 3 of the chunk.  Channels past
// K and C hold zeros.
__global__ __launch_bounds__(256) void octet_weights_kernel(const float* __restrict__ w, float4* __restrict__ Wq, int K, int C, int taps, int nch)
{
    const int mb = blockIdx.x / nch, ch = blockIdx.x % nch;
    const int lane = threadIdx.x & 63;
    const int m = mb * kOctetRows + (lane & 15);
#pragma unroll 1
    for (int u = threadIdx.x >> 6; u < 2 * taps; u += 4) {
        const int tap = u >> 1, c0 = ch * kOctetChannels + (lane >> 4) * 8 + (u & 1) * 4;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = m < K && c0 + e < C ? w[((long long)m * C + c0 + e) * taps + tap] : 0.f;
        Wq[((long long)blockIdx.x * taps * 2 + u) * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
    }
}

// TM x TN matrix tiles, WK wavefronts.  RAGGED: a channel count that is no multiple of 8.  BATCH: groups of channels that a lane has in flight.
template <bool PARTS, int TM, int TN, int WK, int BATCH, bool RAGGED>
__global__ __launch_bounds__(WK * 64, PARTS || BATCH > 2 ? 2 : 4) void conv_short_kernel(ConvShortArgs g)
{
    typedef Matrix<PARTS> Mx;
    typedef typename Mx::acc_t acc_t;
    constexpr int S = Mx::S, NP = Mx::NP, REGS = Mx::REGS, GPS = 64 / S, CHANNELS = GPS * 8;
    constexpr int THREADS = WK * 64, RING = PARTS && TM * TN > 1 ? 2 : 4;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ int wave_lost[WK];
    unsigned lost = 0;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ls = lane % S, lg = lane / S;

    const int wg = (int)xcd_contiguous(blockIdx.x, (unsigned)g.total);
    const int outer = (int)const_div((unsigned)wg, g.by_inner), inner = wg - outer * (int)g.by_inner.d;
    const int tm = g.m_first ? inner : outer, t1 = g.m_first ? outer : inner;
    const int t2 = (int)const_div((unsigned)t1, g.by_tiles_x);
    const int ox0 = (t1 - t2 * g.tilesX) * g.tx;
    const int t3 = (int)const_div((unsigned)t2, g.by_tiles_y);
    const int oy0 = (t2 - t3 * g.tilesY) * g.ty;
    const int img0 = t3 * g.ni;

    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.w), 0, (int)g.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(g.x), 0, (int)g.b_bytes, 0x00020000);
    const int plane = g.H * g.W;
    const int mblocks = (g.M + S - 1) / S;

    // ---- staging: a lane keeps its pixel of the patch and walks over groups of 8 channels, so that its place is worked out once.  LDS holds
    // [group][half or part][slot][16 bytes].
    const int grp0 = (int)const_div((unsigned)tid, g.by_ppr), gstep = g.gstep;
    unsigned x_off;              // byte offset of its pixel in channel 0, or kOutsideBytes
    int x_slot;                  // LDS bytes
    {
        const int q = tid - grp0 * g.ppr;
        const int r1 = (int)const_div((unsigned)q, g.by_pw), px = q - r1 * g.pw;
        const int i = (int)const_div((unsigned)r1, g.by_ph), py = r1 - i * g.ph;
        const int iy = oy0 * g.sh - g.pad_h + py, ix = ox0 * g.sw - g.pad_w + px;
        const bool ok = img0 + i < g.N && (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
        const int xq = (int)const_div((unsigned)px, g.by_sw), xr = px - xq * g.sw;
        x_off = ok ? (unsigned)((img0 + i) * g.C * plane + iy * g.W + ix) * 4u : kOutsideBytes;
        x_slot = ((r1 * g.sw + xr) * g.pws + xq) * 16;
    }
    // groups first + t * gstep of the round, which starts at channel c_first
    auto load_batch = [&](float (&st)[BATCH][8], int first, int c_first) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < BATCH; ++t) {
            const int c0 = c_first + (first + t * gstep + grp0) * 8;
            const unsigned o = c0 < g.C && x_off != kOutsideBytes ? x_off + (unsigned)(c0 * plane) * 4u : kOutsideBytes;
            // channels past the end may be the next image's, whose infinities and NaN a zero weight does not cancel
#pragma unroll
            for (int e = 0; e < 8; ++e)
                st[t][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsB, (int)(!RAGGED || c0 + e < g.C ? o : kOutsideBytes), e * plane * 4, 0));
        }
    };
    auto store_batch = [&](const float (&st)[BATCH][8], int first, int groups) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < BATCH; ++t) {
            const int grp = first + t * gstep + grp0;
            uintx4 v[NP];
            if constexpr (PARTS) {
                bf16x8 part[NP];
                split_octet<NP>(st[t], part, lost);
#pragma unroll
                for (int q = 0; q < NP; ++q) v[q] = __builtin_bit_cast(uintx4, part[q]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e / 4][e % 4] = __float_as_uint(st[t][e]);
            }
            char* to = smem + grp * NP * g.pp * 16 + x_slot;
            if (grp0 < gstep && grp < groups) {
#pragma unroll
                for (int q = 0; q < NP; ++q) *reinterpret_cast<uintx4*>(to + q * g.pp * 16) = v[q];
            }
        }
    };
    const int all_taps = g.nch * g.taps;
    // weights of step u of the whole reduction
    auto read_a = [&](int u, uintx4 (&a)[TM][NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int mb = tm * TM + i;
            const bool in = mb < mblocks;                                // uniform
#pragma unroll
            for (int q = 0; q < NP; ++q)
                a[i][q] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(
                    rsA, in ? lane * 16 + q * 1024 : (int)kOutsideBytes, in ? (int)((unsigned)(mb * all_taps + u) * (NP * 1024u)) : 0, 0));
        }
    };
    // A round: the channels that LDS holds at once.  Its steps, a contiguous run for each wavefront, and its first loads
    int ch0 = 0, chunks = 0, u0 = 0, n = 0;
    float early[BATCH][8];
    uintx4 av[RING][TM][NP];
    auto begin = [&]() __attribute__((always_inline)) {
        chunks = g.nch - ch0 < g.cpr ? g.nch - ch0 : g.cpr;
        const int units = chunks * g.taps, per = (units + WK - 1) / WK;
        u0 = wave * per;
        n = units - u0 < per ? units - u0 : per;
        load_batch(early, 0, ch0 * CHANNELS);
#pragma unroll
        for (int r = 0; r < RING - 1; ++r) read_a(ch0 * g.taps + (r < n ? u0 + r : 0), av[r]);
    };
    begin();
    __builtin_amdgcn_sched_barrier(0);                   // what follows is worked out while those are on their way

    // ---- this lane's column
    struct Col { int y, x, img; bool ok; };
    auto column = [&](int c) -> Col {
        const int u = (int)const_div((unsigned)c, g.by_tx), tx = c - u * g.tx;
        const int i = (int)const_div((unsigned)u, g.by_ty), ty = u - i * g.ty;
        Col r;
        r.img = i; r.y = ty; r.x = tx;
        r.ok = i < g.ni && img0 + i < g.N && oy0 + ty < g.Ho && ox0 + tx < g.Wo;
        return r;
    };
    Col mine[TN];
    int b_lane[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const Col c = mine[j] = column(j * S + ls);
        b_lane[j] = (lg * NP * g.pp + (c.ok ? (c.img * g.ph + c.y * g.sh) * (g.sw * g.pws) + c.x : 0)) * 16;
    }

    // lane t: LDS bytes of tap t
    int tap_offset;
    {
        const int ky = (int)const_div((unsigned)lane, g.by_kw), dx = (lane - ky * g.kw) * g.dw;
        const int xq = (int)const_div((unsigned)dx, g.by_sw), xr = dx - xq * g.sw;
        tap_offset = ((ky * g.dh * g.sw + xr) * g.pws + xq) * 16;
    }

    // the outputs of this thread, and their bias on the way
    constexpr int OUT = TM * TN * REGS * 64, IT = (OUT + THREADS - 1) / THREADS;
    auto out_row = [&](int o) -> int { return (tm * TM + o / (REGS * 64) / TN) * S + Mx::row((o >> 6) % REGS, o & 63); };
    float bias[IT];
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int m = out_row(tid + t * THREADS);
        bias[t] = g.bias ? g.bias[m < g.M ? m : g.M - 1] : 0.f;
    }

    acc_t acc[TM][TN][2];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < REGS; ++r) acc[i][j][0][r] = acc[i][j][1][r] = 0.f;
    };
    clear();

    auto read_b = [&](int off, uintx4 (&b)[TN][NP]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int q = 0; q < NP; ++q) b[j][q] = *reinterpret_cast<const uintx4*>(smem + off + b_lane[j] + q * g.pp * 16);
    };

#pragma unroll 1
    for (;;) {
        const int groups = chunks * GPS, ubase = ch0 * g.taps + u0;
        if (ch0 > 0) lds_barrier();                          // the patch before has been read
        store_batch(early, 0, groups);
#pragma unroll 1
        for (int first = BATCH * gstep; first < groups; first += BATCH * gstep) {
            float st[BATCH][8];
            load_batch(st, first, ch0 * CHANNELS);
            store_batch(st, first, groups);
        }
        lds_barrier();
        int chunk = (int)const_div((unsigned)u0, g.by_taps), tap = u0 - chunk * g.taps;
        // LDS bytes of the step; behind the last one some other's
        auto offset = [&]() -> int { return (chunk < chunks ? chunk : 0) * GPS * NP * 16 * g.pp + __builtin_amdgcn_readlane(tap_offset, tap); };
        auto advance = [&]() {
            const bool wrap = ++tap == g.taps;
            tap = wrap ? 0 : tap;
            chunk += wrap ? 1 : 0;
        };
        uintx4 bv[2][TN][NP];
        if (n > 0) read_b(offset(), bv[0]);
        int u = 0;
        auto step = [&](auto slot_) __attribute__((always_inline)) {
            constexpr int I = decltype(slot_)::value;
            const int ahead = u + RING - 1;
            read_a(ubase + (ahead < n ? ahead : 0), av[(I + RING - 1) % RING]);
            advance();
            read_b(offset(), bv[(I + 1) % 2]);
            __builtin_amdgcn_sched_barrier(0);           // or the reads move down to their use
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) Mx::multiply(av[I][i], bv[I % 2][j], acc[i][j]);
            ++u;
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>;
#pragma unroll 1
        while (u + RING <= n) {
            step(I0{});
            step(I1{});
            if constexpr (RING == 4) { step(I2{}); step(I3{}); }
        }
        if (u < n) {
            step(I0{});
            if constexpr (RING == 4) {
                if (u < n) {
                    step(I1{});
                    if (u < n) step(I2{});
                }
            }
        }
        ch0 += g.cpr;
        if (ch0 >= g.nch) break;
        begin();
    }

    if constexpr (PARTS) {
        const bool l = parts_lost(lost);
        if (lane == 0) wave_lost[wave] = l ? 1 : 0;
    }
    lds_barrier();                                           // the patch has been read
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < REGS; ++r) acc[i][j][0][r] += acc[i][j][1][r];

    if constexpr (PARTS) {
        // sums that are not finite, or values that their parts do not hold: the wavefront repeats its steps on the fp32 matrix instructions, inputs
        // straight from memory (as in conv_patch.hip)
        FiniteCheck check;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int r = 0; r < REGS; ++r) check.add(acc[i][j][0][r]);
        int any_lost = 0;
#pragma unroll
        for (int w = 0; w < WK; ++w) any_lost |= wave_lost[w];
        if (check.failed() || __builtin_amdgcn_readfirstlane(any_lost) != 0) {
            clear();
#pragma unroll 1
            for (ch0 = 0; ch0 < g.nch; ch0 += g.cpr) {
                const int units = (g.nch - ch0 < g.cpr ? g.nch - ch0 : g.cpr) * g.taps, per = (units + WK - 1) / WK;
                const int first = wave * per, last = first + per < units ? first + per : units;
#pragma unroll 1
                for (int u = first; u < last; ++u) {
                    const int ch = (int)const_div((unsigned)u, g.by_taps), tap = u - ch * g.taps;
                    const int ky = (int)const_div((unsigned)tap, g.by_kw), kx = tap - ky * g.kw;
                    read_a(ch0 * g.taps + u, av[0]);
                    const int c0 = (ch0 + ch) * CHANNELS + lg * 8;
                    unsigned from[TN];
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int iy = (oy0 + mine[j].y) * g.sh - g.pad_h + ky * g.dh, ix = (ox0 + mine[j].x) * g.sw - g.pad_w + kx * g.dw;
                        const bool ok = mine[j].ok && (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
                        from[j] = ok ? (unsigned)(((img0 + mine[j].img) * g.C + c0) * plane + iy * g.W + ix) * 4u : kOutsideBytes;
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        float xv[TN];
#pragma unroll
                        for (int j = 0; j < TN; ++j)
                            xv[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                rsB, (int)(c0 + e < g.C && from[j] != kOutsideBytes ? from[j] + (unsigned)(e * plane) * 4u : kOutsideBytes), 0, 0));
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const float wv = weight_value(av[0][i], e);
#pragma unroll
                            for (int j = 0; j < TN; ++j) acc[i][j][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, xv[j], acc[i][j][0], 0, 0, 0);
                        }
                    }
                }
            }
        }
    }

    // ---- partial tiles added in wavefront order, then bias and store
    float* red = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < REGS; ++r) red[(((wave * TM + i) * TN + j) * REGS + r) * 64 + lane] = acc[i][j][0][r];
    lds_barrier();
#pragma unroll
    for (int t = 0; t < IT; ++t) {
        const int o = tid + t * THREADS;
        if (OUT % THREADS != 0 && o >= OUT) break;
        float s = red[o];
#pragma unroll
        for (int w = 1; w < WK; ++w) s += red[w * OUT + o];
        const int m = out_row(o);
        const Col c = mine[t * THREADS / (REGS * 64) % TN];              // o % S is this lane's column, and TN > 1 only where a round stays in one tile
        if (c.ok && m < g.M) g.y[(long long)(img0 + c.img) * g.sImg + (long long)m * g.sRow + (oy0 + c.y) * g.Wo + ox0 + c.x] = s + bias[t];
    }
}

bool short_rect(const GemmProblem& p, int columns, int channel_bytes, ConvShortArgs* g)
{
    return choose_patch_rect(p, columns, kShortPixels, kShortLds / channel_bytes, false, g);       // one chunk of channels at least
}

bool conv_short_takes(const GemmProblem& p)
{
    if (!p.gather || p.batch != 1 || p.prec != 0 || p.splitk > 1 || p.M <= 0 || p.L <= 0 || p.cv_Wo <= 0 || p.Ncols % p.L != 0) return false;
    const int taps = p.cv_kh * p.cv_kw;
    return p.cv_C >= 8 && taps <= kShortTaps && octet_weight_bytes(p.M, p.cv_C, taps) < ((size_t)1 << 31) &&
           conv_patch_weight_bytes(p.M, p.cv_C, taps) < ((size_t)1 << 31);
}

template <bool PARTS, int TM, int TN, int WK>
hipError_t launch_conv_short(const GemmProblem& p, bool, hipStream_t s)
{
    typedef Matrix<PARTS> Mx;
    constexpr int GPS = 64 / Mx::S, CHUNK = GPS * Mx::NP * 16;            // LDS bytes of a slot in a chunk of channels
    static_assert(TN == 1 || (Mx::REGS * 64) % (WK * 64) == 0, "the epilogue's rounds stay in a tile");
    ConvShortArgs g{};
    unsigned plain = 0;
    g.w = PARTS ? p.a_parts : p.a_octets;
    if (!g.w || !conv_short_takes(p) || !short_rect(p, Mx::S * TN, CHUNK, &g) || !gemm_operand_extents(p, &plain, &g.b_bytes)) return hipErrorInvalidValue;
    g.x = p.B; g.y = p.D; g.bias = p.bias;
    g.sImg = p.strideD_img; g.sRow = p.strideD_row;
    g.M = p.M; g.C = p.cv_C; g.H = p.cv_H; g.W = p.cv_W; g.N = p.Ncols / p.L; g.Ho = p.L / p.cv_Wo; g.Wo = p.cv_Wo;
    g.kw = p.cv_kw; g.taps = p.cv_kh * p.cv_kw; g.sh = p.cv_sh; g.sw = p.cv_sw; g.pad_h = p.cv_ph; g.pad_w = p.cv_pw; g.dh = p.cv_dh; g.dw = p.cv_dw;
    g.a_bytes = (unsigned)(PARTS ? conv_patch_weight_bytes(p.M, p.cv_C, g.taps) : octet_weight_bytes(p.M, p.cv_C, g.taps));
    g.tilesM = (p.M + TM * Mx::S - 1) / (TM * Mx::S);
    const long long tilesP = (long long)g.tilesX * g.tilesY * ((g.N + g.ni - 1) / g.ni), total = tilesP * g.tilesM;
    if (!grid_fits(total, WK * 64)) return hipErrorInvalidValue;
    g.tilesP = (int)tilesP;
    g.total = (int)total;
    // the larger operand is the one that an XCD should not read whole
    g.m_first = g.a_bytes < g.b_bytes ? 1 : 0;
    g.nch = (g.C + GPS * 8 - 1) / (GPS * 8);
    const int chunk = CHUNK * g.pp, lds = total <= 256 ? kShortLds : kShortLds / 2;
    g.cpr = lds / chunk < g.nch ? (lds / chunk < 1 ? 1 : lds / chunk) : g.nch;
    const int rounds = (g.nch + g.cpr - 1) / g.cpr;
    g.cpr = (g.nch + rounds - 1) / rounds;
    g.gstep = WK * 64 / g.ppr;
    g.by_inner = make_constdiv((unsigned)(g.m_first ? g.tilesM : g.tilesP));
    g.by_pw = make_constdiv((unsigned)g.pw);
    g.by_ph = make_constdiv((unsigned)g.ph);
    g.by_ppr = make_constdiv((unsigned)g.ppr);
    g.by_tx = make_constdiv((unsigned)g.tx);
    g.by_ty = make_constdiv((unsigned)g.ty);
    g.by_sw = make_constdiv((unsigned)g.sw);
    g.by_kw = make_constdiv((unsigned)g.kw);
    g.by_taps = make_constdiv((unsigned)g.taps);
    g.by_tiles_x = make_constdiv((unsigned)g.tilesX);
    g.by_tiles_y = make_constdiv((unsigned)g.tilesY);
    const int red = WK * TM * TN * Mx::REGS * 256, patch = g.cpr * chunk;
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(WK * 64), (size_t)(patch > red ? patch : red), s, g); };
    auto ragged_or_not = [&](auto batch) {
        constexpr int B = decltype(batch)::value;
        if (g.C & 7) launch(conv_short_kernel<PARTS, TM, TN, WK, B, true>);
        else launch(conv_short_kernel<PARTS, TM, TN, WK, B, false>);
    };
    const int batches = (g.cpr * GPS + g.gstep - 1) / g.gstep;
    if (batches == 1) ragged_or_not(std::integral_constant<int, 1>{});
    else if (batches == 2) ragged_or_not(std::integral_constant<int, 2>{});
    else if (batches == 3 || PARTS) ragged_or_not(std::integral_constant<int, 3>{});
    else ragged_or_not(std::integral_constant<int, PARTS ? 3 : 6>{});
    return hipGetLastError();
}

const GemmVariant kConvShort[] = {
    {"f32_patch_16x16_k8", launch_conv_short<false, 1, 1, 8>, 16, 16, 256},
    {"x6_patch_32x32_k8", launch_conv_short<true, 1, 1, 8>, 32, 32, 128},
    {"x6_patch_64x32_k8", launch_conv_short<true, 2, 1, 8>, 64, 32, 128},
    {"x6_patch_32x64_k8", launch_conv_short<true, 1, 2, 8>, 32, 64, 128},
};
constexpr int kOctetVariants = 1;            // of these, the first

}  // namespace

int conv_short_variant_count() { return (int)(sizeof(kConvShort) / sizeof(kConvShort[0])); }
const GemmVariant& conv_short_variant(int i) { return kConvShort[i]; }
bool conv_short_takes_octets(int i) { return i < kOctetVariants; }

size_t octet_weight_bytes(int K, int C, int taps)
{
    return (size_t)((K + kOctetRows - 1) / kOctetRows) * ((C + kOctetChannels - 1) / kOctetChannels) * taps * 2048;
}

// Not where 64 x 64 tiles fill the chip one and a half times: of 33 such layers none was fastest here, the best of these took 1.04 to 2.3 times as long as the
// best of the others (16 x 16 tiles up to 3.9 times), and timing them costs every plan (64 -> 64 on 16 x 56 x 56, 784 tiles).  But for few output channels,
// which leave a larger tile half empty: 453 -> 13 7 x 7 on 34 x 26 x 26 313 -> 216 us, 280 -> 15 3 x 3 on 34 x 45 x 45, 1076 tiles, 102 -> 83.
bool conv_short_offered(const GemmProblem& p, int i)
{
    const long long tiles64 = (long long)((p.M + 63) / 64) * ((p.Ncols + 63) / 64);
    return (conv_short_takes_octets(i) ? p.a_octets : p.a_parts) && (p.M <= 32 || tiles64 < 384) && conv_short_covers(p);
}

bool conv_short_covers(const GemmProblem& p)
{
    unsigned a = 0, b = 0;
    ConvShortArgs g{};
    return conv_short_takes(p) && gemm_operand_extents(p, &a, &b) && short_rect(p, 16, 128, &g) && short_rect(p, 32, 96, &g) && short_rect(p, 64, 96, &g);
}

hipError_t launch_octet_weights(const float* w, void* Wq, int K, int C, int taps, hipStream_t s)
{
    if (!w || !Wq || K <= 0 || C <= 0 || taps <= 0) return hipErrorInvalidValue;
    const int nch = (C + kOctetChannels - 1) / kOctetChannels;
    const long long blocks = (long long)((K + kOctetRows - 1) / kOctetRows) * nch;
    if (!grid_fits(blocks, 256)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(octet_weights_kernel, dim3((unsigned)blocks), dim3(256), 0, s, w, (float4*)Wq, K, C, taps, nch);
    return hipGetLastError();
}

}  // namespace mnnconv
