// Launch functions of the gfx950 kernels.  Raw device pointers and a hipStream_t;
// every launcher validates what its kernel assumes and returns hipError_t.
#pragma once
#include <hip/hip_runtime_api.h>
#include <cstddef>
#include <cstdint>

namespace mnnconv {

// Largest alpha = n + k - 1 the Winograd kernels are built for.  In fp32 the error of the generated
// transforms grows quickly with alpha: about 3e-4 of the output range at alpha = 10 and above 1e-2 from
// alpha = 11 on, which is outside the accuracy this library promises.
constexpr int kMaxAlphaT = 10;

// Transform matrix handed to kernels by value (lands in SGPRs).
template <int R, int C>
struct MatArg { float v[R][C]; };

// A launch holds fewer than 2^32 work-items: one over that runs, without an error, on what is left modulo 2^32.
constexpr bool grid_fits(long long workgroups, int threads) { return workgroups > 0 && workgroups < (1ll << 31) && workgroups * threads < (1ll << 32); }

struct WinoGeom {
    int N, C, H, W, K;          // input x[N][C][H][W], K output channels
    int Ho, Wo;                 // output plane
    int pad_h, pad_w;
    int n, k, alpha;            // F(n, k), alpha = n + k - 1 (along H when the kernel is not square)
    int nw, kw, alpha_w;        // the same along W; equal to n, k, alpha for square kernels.  An axis along
                                // which the kernel has one tap is left untransformed: n = k = alpha = 1.
    int th, tw;                 // tiles per image: ceil(Ho/n), ceil(Wo/nw)
    int P;                      // N * th * tw
    int ldp;                    // row length of V / M rows (P rounded up to 4)
    int ldk;                    // row length of U rows (K rounded up to 4)
    // Blocked ("MFMA-native") layout used by the fused kernel instead of the row layouts
    // (xi = a*alpha + b):  Ub[b][c/4][a][k/16][c%4][k%16],  Vb[b][c/4][a][p/16][c%4][p%16]
    int blocked;                // 0: row layouts U[xi][c][ldk], V[xi][c][ldp];  1: blocked
    int kg, pg;                 // allocated 16-column groups along K and along P
    int cchunks;                // allocated 4-channel groups (>= ceil(C/4), padded to whole chunks)
    // Tiled row layout (blocked == 0, tiled == 1): V[c][p/64][xi][p%64], M[k][p/64][xi][p%64] -- the alpha^2 values of 64
    // consecutive tiles of one channel are one contiguous run, which is exactly what one wavefront of the transform kernels
    // writes or reads; ldp = 64 * pb.
    int tiled;
    int pb;                     // 64-tile blocks: ceil(P / 64)
    int itx_waves;              // input transform: resident wavefronts per CU to allow (10, 12, 16 or 20), 0 = as many as fit
};

// U[xi][c][k] = (G w[k][c] G^T)[xi/alpha][xi%alpha]          (Section 3.3.1, G W G^T)
hipError_t launch_filter_transform(const WinoGeom& g, const float* G /*host, alpha x k*/,
                                   const float* w, float* U, hipStream_t s);

// V[xi][c][p] = (B^T d B)[xi/alpha][xi%alpha], d = input tile p of channel c   (B^T X B)
hipError_t launch_input_transform(const WinoGeom& g, const float* BT /*host, alpha x alpha*/,
                                  const float* x, float* V, hipStream_t s);

// y[img][k][ty*n+i][tx*n+j] = (A^T m A)[i][j] + bias[k], m[a][b] = M[a*alpha+b][k][p]   (A^T [.] A)
hipError_t launch_output_transform(const WinoGeom& g, const float* AT /*host, n x alpha*/,
                                   const float* M, const float* bias, float* y, hipStream_t s);

// The same for few (channel, tile) pairs (transforms_short.hip; the launchers above take them where these rules say so), and the input transform
// together with the weights': V and U with all their padding, which the two alone leave as it is.  Geometry and matrices as the launchers above
// check them, alpha even or odd, matrices of an even alpha with the structure that the generated ones have.
bool input_transform_short(const WinoGeom& g);
bool input_filter_short(const WinoGeom& g);
bool output_transform_short(const WinoGeom& g);
hipError_t launch_input_short(const WinoGeom& g, const float* BT, const float* x, float* V, hipStream_t s);
hipError_t launch_output_short(const WinoGeom& g, const float* AT, const float* M, const float* bias, float* y, hipStream_t s);
hipError_t launch_input_filter_short(const WinoGeom& g, const float* BT, const float* G, const float* x, const float* w, float* V, float* U, hipStream_t s);
hipError_t launch_input_filter(const WinoGeom& g, const float* BT, const float* G, const float* x, const float* w, float* V, float* U, hipStream_t s);

// Products and inverse transform of few tiles in one launch, U and V in the row layouts (products_short.hip): M is never stored.
bool products_output_short(const WinoGeom& g);
hipError_t launch_products_output(const WinoGeom& g, const float* AT, const float* U, const float* V, const float* bias, float* y, hipStream_t s);

bool input_transform_capped(const WinoGeom& g, const float* BT);       // whether the kernel that itx_waves limits is launched

bool winograd_kernels_available(int n, int k);

// One-dimensional Winograd for kernels with a single row or column (1 x k, k x 1; Section 3.3.1: "kernels of
// any size"): F(n, k) along the long axis, identity along the other.  Row layouts only (g.blocked == 0):
// U[(i*alpha_w + j)][c][ldk], V and M likewise.  Matrices of the untransformed axis are the 1 x 1 identity.
bool winograd_rect_kernels_available(int nh, int kh, int nw, int kw);
hipError_t launch_filter_transform_rect(const WinoGeom& g, const float* Gh, const float* Gw, const float* w, float* U,
                                        hipStream_t s);
hipError_t launch_input_transform_rect(const WinoGeom& g, const float* BTh, const float* BTw, const float* x, float* V,
                                       hipStream_t s);
hipError_t launch_output_transform_rect(const WinoGeom& g, const float* ATh, const float* ATw, const float* M,
                                        const float* bias, float* y, hipStream_t s);

// Winograd-domain product with the inverse transform and bias fused in:
// y = A^T [ sum_c U (.) V ] A + bias, operands in the blocked layout.  M is never stored.
// config 0: 32 channels x 32 tiles per workgroup; config 1: 64 x 64 (only where wino_fused_has_big_block), with the
// tiles of a mostly empty last round of workgroups handed to 32 x 32 workgroups (up to two launches).
bool wino_fused_available(int n, int k);
bool wino_fused_has_big_block(int n, int k);
hipError_t launch_wino_fused(const WinoGeom& g, int config, const float* AT /*host*/, const float* Ub,
                             const float* Vb, const float* bias, float* y, hipStream_t s);
int wino_fused_launch_count(const WinoGeom& g, int config);      // kernels one such call enqueues

// The whole convolution in one kernel (alpha <= 6, x below 2 GiB): y = A^T [ sum_c U (.) B^T x B ] A + bias.  U: the prepared weights as
// bf16 parts in matrix-operand order, wino_full_weight_bytes, written by launch_filter_full.
bool wino_full_available(int n, int k);
int wino_full_block_channels(int alpha);            // output channels per workgroup
// Sizes the one-kernel arrangement takes: 32-bit byte offsets into the input (with room for the over-read of a tile row) and the weights,
// a grid the hardware counts.  Reads N, C, H, W, K, n, k, alpha, th and tw.
bool wino_full_covers(const WinoGeom& g);
size_t wino_full_weight_bytes(const WinoGeom& g);
hipError_t launch_filter_full(const WinoGeom& g, const float* G /*host*/, const float* w, void* U, hipStream_t s);
hipError_t launch_wino_full(const WinoGeom& g, const float* BT /*host*/, const float* AT /*host*/, const float* x, const void* U,
                            const float* bias, float* y, hipStream_t s);

// One axis at a time (alpha 7 to 10, x and its row transform below 2 GiB): T[b] = x B by rows, then for each column b of the positions the
// transform along the image height, the channel sums and A^T along the height in one kernel (S), then A^T along the rows.  U: bf16 parts in
// matrix-operand order.  T, U and S have the sizes below.
bool wino_cols_available(int n, int k);
bool wino_cols_covers(const WinoGeom& g);           // reads N, C, H, W, K, n, k, alpha, th and tw
bool wino_cols_offered(const WinoGeom& g);          // whether the planner times it where it covers; reads the same
size_t wino_cols_weight_bytes(const WinoGeom& g);
size_t wino_cols_input_bytes(const WinoGeom& g);
size_t wino_cols_sum_bytes(const WinoGeom& g);
hipError_t launch_cols_filter(const WinoGeom& g, const float* G /*host*/, const float* w, void* U, hipStream_t s);
hipError_t launch_cols_rows_in(const WinoGeom& g, const float* BT /*host*/, const float* x, float* T, hipStream_t s);
hipError_t launch_cols(const WinoGeom& g, const float* BT /*host*/, const float* AT /*host*/, const float* T, const void* U, float* S, hipStream_t s);
hipError_t launch_cols_rows_out(const WinoGeom& g, const float* AT /*host*/, const float* S, const float* bias, float* y, hipStream_t s);

// Batched GEMM  D_b[m][col] = sum_r At_b[r][m] * B_b[r][col] (+ bias[m]).
//   At: [batch][R][lda]  (A stored transposed, m contiguous; lda % 4 == 0, 16-byte aligned)
//   B : element (r, col) at  B + b*strideB_batch + (col / L)*strideB_img + r*strideB_row + (col % L)
//   D : element (m, col) at  D + b*strideD_batch + (col / L)*strideD_img + m*strideD_row + (col % L)
// L is the number of consecutive columns that are contiguous in memory (the whole
// row for the Winograd-domain product, H*W for the 1x1 convolution of one image).
struct GemmArgs {
    const float* At; const float* B; float* D; const float* bias;
    int M, Ncols, R, batch;
    int lda;
    int L;
    long long strideA_batch;
    long long strideB_batch, strideB_img, strideB_row;
    long long strideD_batch, strideD_img, strideD_row;
    int variant;                // 0 = choose from the shape; > 0 = a specific tile configuration (tuning, tests)
    int prec;                   // 0: fp32 MFMA; 1: bf16 operands; 2: bf16x3 (hi/lo split, three bf16 MFMAs per product)
    // Split-K (register-staged kernels only): splitk > 1 cuts the reduction of every tile into that many
    // workgroups, which write partial results to splitk_partial (gemm_splitk_workspace floats, 16-byte
    // aligned); a second kernel adds them up in slice order.  0 or 1 = off.
    int splitk;
    float* splitk_partial;
    // Implicit-GEMM gather for the sliding-window scheme (gather != 0): B is the input tensor x[N][C][H][W],
    // row r = (c, kr, ks), column = (img, oy, ox), element = x[img][c][oy*sh - ph + kr*dh][ox*sw - pw + ks*dw] or 0.
    // L must be H_o*W_o; the strideB_* fields are ignored.
    int gather;
    int cv_C, cv_H, cv_W, cv_kh, cv_kw, cv_sh, cv_sw, cv_ph, cv_pw, cv_dh, cv_dw, cv_Wo;
};
// What the product kernels do not read stays out of their arguments (gemm_split.hip says why it matters).
struct GemmProblem : GemmArgs {
    const void* a_parts;        // weights of the patch kernels and of pointwise layers (launch_patch_weights), U of Winograd (launch_parts_of_rows); At is then unused
    const void* a_octets;       // the same for those of them that read fp32 (launch_octet_weights)
};
hipError_t launch_gemm_f32(const GemmProblem& p, hipStream_t s);
int gemm_f32_variant_count();
const char* gemm_f32_variant_name(int variant);
// Tile shape of a variant of precision `prec` (false for variants that cannot split K) and the scratch a
// split-K launch needs: floats of partial sums and number of tile counters.
bool gemm_variant_tile(int prec, int variant, int* bm, int* bn, int* bk);
inline int gemm_splitk_ldc(const GemmProblem& p) { return (p.Ncols + 3) / 4 * 4; }    // row length of the partial results
long long gemm_splitk_workspace(const GemmProblem& p, int splitk);                    // floats
hipError_t launch_splitk_reduce(const GemmProblem& p, hipStream_t s);
// Bytes one batch of each operand spans (descriptor sizes); false when the 32-bit loaders cannot address them.
bool gemm_operand_extents(const GemmProblem& p, unsigned* a_bytes, unsigned* b_bytes);
// fp32-grade products on the bf16 matrix cores (gemm_split.hip): variants of prec 0 that follow the fp32 kernels'
struct GemmVariant { const char* name; hipError_t (*fn)(const GemmProblem&, bool, hipStream_t); int bm, bn, bk; };
int gemm_split6_variant_count();
const GemmVariant& gemm_split6_variant(int i);
constexpr int kStaged128 = 0, kStaged128x64 = 1, kStaged64x128 = 2, kStaged64 = 3;        // its tiles of that size
// the same for grids too short to fill the chip (gemm_short.hip); these follow
int gemm_short_variant_count();
const GemmVariant& gemm_short_variant(int i);
constexpr int kShort16 = 0, kShort32 = 2, kShort64 = 4;
// and the sliding window on staged patches (conv_patch.hip), with weights of a form of their own; these come last
int conv_patch_variant_count();
const GemmVariant& conv_patch_variant(int i);
bool conv_patch_covers(const GemmProblem& p);       // whether the patch kernels take this product
bool conv_patch_offered(const GemmProblem& p);      // whether the planner times them
size_t conv_patch_weight_bytes(int K, int C, int taps);
hipError_t launch_patch_weights(const float* w, void* Wp, int K, int C, int taps, hipStream_t s);
// the same for short grids (conv_short.hip), which have numbers after theirs and no public names
int conv_short_variant_count();
const GemmVariant& conv_short_variant(int i);
bool conv_short_takes_octets(int i);
bool conv_short_covers(const GemmProblem& p);
bool conv_short_offered(const GemmProblem& p, int i);      // whether the planner times it
size_t octet_weight_bytes(int K, int C, int taps);
hipError_t launch_octet_weights(const float* w, void* Wq, int K, int C, int taps, hipStream_t s);
// pointwise layers with weights as parts, of the same form for one tap (gemm_prepared.hip); numbers after those
int gemm_prepared_variant_count();
const GemmVariant& gemm_prepared_variant(int i);
bool gemm_prepared_covers(const GemmProblem& p);
bool gemm_prepared_offered(const GemmProblem& p, int i);      // whether the planner times it
int gemm_first_prepared_variant(int prec);
// the same of Winograd-domain weights: rows of U of `batch` positions as three parts (prec 0) or two (prec 2), gemm_parts_bytes each
size_t gemm_parts_bytes(int prec, int K, int C);
hipError_t launch_parts_of_rows(int prec, const float* U, void* Up, int K, int C, int ldk, int batch, hipStream_t s);
// what a variant reads the weights of a planned layer from: At, a_parts or a_octets
enum class WeightForm { Rows, Parts, Octets };
WeightForm gemm_variant_weights(int prec, int variant);
// bf16 / bf16x3 operands (gemm_split.hip; operands of 2 GiB and more: gemm_bf16.hip); launch_gemm_f32 forwards to them when prec != 0
int gemm_bf16_variant_count();
int gemm_bf16_named_count();
const char* gemm_bf16_variant_name(int variant);
hipError_t launch_gemm_bf16(const GemmProblem& p, hipStream_t s);
hipError_t launch_gemm_bf16_wide(const GemmProblem& p, int config, bool vec, hipStream_t s);     // config: gemm_bf16_variant - 1
bool gemm_bf16_variant_tile(int variant, int* bm, int* bn, int* bk);
bool gemm_variant_tuned(const GemmProblem& p, int variant);     // whether the planner times it
// variants of the table that serves precision `prec`
inline int gemm_variant_count(int prec) { return prec == 0 ? gemm_f32_variant_count() : gemm_bf16_variant_count(); }
int gemm_named_variant_count(int prec);         // of these, the ones with a public name
int gemm_product_variant_count(int prec);       // of these, the ones that take any product: all but the patch kernels
inline const char* gemm_variant_name(int prec, int v) { return prec == 0 ? gemm_f32_variant_name(v) : gemm_bf16_variant_name(v); }

// Strassen's algorithm (Section 3.3.2), one level = expand both operands, one batched GEMM, combine.
// A view addresses element (r, c) of a row-major operand at  (c / L) * sImg + r * sRow + c % L  (the column
// mapping of the GEMM: L consecutive columns are contiguous, the next L belong to the next image).
// All of L, sImg, sRow and the half widths must be multiples of 4, bases 16-byte aligned.
struct StrassenView { int L; long long sImg, sRow; };
// src: nb operands [2*rows_half][2*cols_half] (batch stride in floats) -> dst [7*nb][rows_half][cols_half] dense.
// left: the operand is A stored transposed (At[r][m]); otherwise it is B.
hipError_t launch_strassen_expand(bool left, const StrassenView& v, const float* src, long long src_batch_stride, int rows_half,
                                  int cols_half, int nb, float* dst, hipStream_t s);
// src: [7*nb][rows_half][cols_half] dense products -> dst: nb results [2*rows_half][2*cols_half] (+ bias per row, nb = 1).
hipError_t launch_strassen_combine(const StrassenView& v, const float* src, int rows_half, int cols_half, int nb, float* dst,
                                   long long dst_batch_stride, const float* bias, hipStream_t s);

// Wt[r][k] = w[k][r], r < R = C*kh*kw, row length ldk (zero padded)
hipError_t launch_weight_transpose(const float* w, float* Wt, int K, int R, int ldk, hipStream_t s);

// Seeded pseudo-random floats in [lo, hi] (scratch tensors of the timing planner) and zeros written by a kernel
// (dst 16-byte aligned), for memory that code under graph capture has to clear.
hipError_t launch_fill_pattern(float* dst, size_t n_floats, unsigned seed, float lo, float hi, hipStream_t s);
hipError_t launch_fill_zero(float* dst, size_t n_floats, hipStream_t s);

// Device address, on the current device, of the library's fixed scratch array of kStaticScratchBytes bytes (256-byte
// aligned; part of the code object, never allocated or freed; every device holds its own copy, which keeps the contents
// of the last call).  Looks the address up on the first call per device; allocates nothing.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
hipError_t static_scratch(float** ptr);

// Device-rate probes: `workgroups` x 4 waves each issuing 4*iters fp32 32x32x2 matrix-core instructions
// (out: workgroups*256 floats), and a 16-byte-per-lane copy of n_floats (multiple of 4, 16-byte aligned).
hipError_t launch_mfma_issue(float* out, int workgroups, int iters, hipStream_t s);
hipError_t launch_stream_copy(const float* src, float* dst, size_t n_floats, hipStream_t s);

}  // namespace mnnconv
