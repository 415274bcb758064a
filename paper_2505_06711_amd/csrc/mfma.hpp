// Matrix-core (MFMA) dense layers for the hidden layers of the atomic NNs and their
// vector-Jacobian products: C[rows x out] = A[rows x in] * Wt^T with FP32 accumulation.
// Operands are FP32, bfloat16 or OCP FP8 e4m3 (per-tensor scales); A is FP32 in memory and
// is rounded to the operand type while it is staged to LDS.
#pragma once

#include "mlp.hpp"

namespace reann {

enum class OpType { F32 = 0, BF16 = 1, FP8 = 2, F64 = 3 };   // F64: the packed operands of the FP64 NN only

constexpr int kMfmaKC = 32;   // K chunk staged per iteration; weight rows are padded to it

__host__ __device__ inline int pad_k(int in) { return (in + kMfmaKC - 1) / kMfmaKC * kMfmaKC; }

// Wt: operand-typed [out][ldw] (ldw = pad_k(in), zero padded).  FP8 only: sA / sW are the
// device scales of A (amax/448, see amax_scale) and of Wt; the product is rescaled by both.
void gemm_mfma(hipStream_t st, OpType op, Epi epi, int64_t rows, int in, int out, const float *A, int lda,
               const void *Wt, int ldw, const float *bias, float *Z, int ldz, float *C, int ldc, const float *sA,
               const float *sW);

// *d_scale = max(|A|) / 448 over rows x cols (row stride lda), or 1 if A is all zero.
void amax_scale(hipStream_t st, const float *A, int64_t rows, int cols, int lda, float *d_scale, uint32_t *d_tmp);

// Convert FP32 [rows][cols] (row stride ld_src) into operand type [rows][ld_dst] (zero padded);
// for FP8 the values are divided by *scale first.
void convert_operand(hipStream_t st, OpType op, const float *src, int rows, int cols, int ld_src, void *dst,
                     int ld_dst, const float *scale);

// Operands of the fused kernels, stored as the fragments their lanes read: for K chunk kc (4 RUN
// values of k) and block j of 16 rows, lane l holds the RUN values W[16 j + l % 16][4 RUN kc +
// RUN (l / 16) ..], RUN = 4 (FP32) or 8, at ((kc nblk + j) 64 + l) RUN; zero past the matrix.
__host__ __device__ constexpr int op_run(OpType op) { return op == OpType::F32 ? 4 : 8; }
inline size_t packed_elems(OpType op, int rows, int cols) {
    const int kc = 4 * op_run(op);
    return (size_t)((rows + 15) / 16 * 16) * (size_t)((cols + kc - 1) / kc * kc);
}
// Pack FP32 [rows][cols] (row stride ld_src); for FP8 the values are divided by *scale first.
void pack_operand(hipStream_t st, OpType op, const float *src, int rows, int cols, int ld_src, void *dst,
                  const float *scale);

// Multinomial weight l! / (lx! ly! lz!) of Cartesian component q (components by order, then lx, ly
// descending).
constexpr float lambda_weight(int L, int q) {
    int k = 0;
    for (int l = 0; l <= L; ++l)
        for (int x = l; x >= 0; --x)
            for (int y = l - x; y >= 0; --y, ++k)
                if (k == q) {
                    int w = 1;
                    for (int j = 2; j <= l; ++j) w *= j;
                    for (int j = 2; j <= x; ++j) w /= j;
                    for (int j = 2; j <= y; ++j) w /= j;
                    for (int j = 2; j <= l - x - y; ++j) w /= j;
                    return (float)w;
                }
    return 0.0f;
}

// Features of the NN input (L = 0: the radial form's K sums), and their chunks.
constexpr int fused_features(int L, int K) { return L == 0 ? K : n_feat(L, K); }
constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Fused atomic NN (every layer of one element's NN in one launch, FP32 or BF16 operands).
constexpr int kFuseBM = 32;      // rows per workgroup
constexpr int kFuseSmallBM = 16; // rows per workgroup of a launch with few rows
constexpr int kFuseMaxH = 128;   // hidden width (64 or 128)
constexpr int kFuseMaxF = 256;   // input width
constexpr int kFuseMaxNh = 4;    // hidden layers
constexpr int kFuseMaxOut = 16;  // output width
constexpr int kFuseMaxNLK = 160; // orbital sums per row (NL * K)

template <typename R> struct FusedNNT {
    int64_t rows;                 // rows of this element's segment
    int F, H, nh, dout;           // input width, hidden width, hidden layers, output width
    int L, K;                     // angular order and radial channels of the density input
    const R *S;               // orbital sums [rows][NL*K] (the NN input is their density)
    // packed operands (pack_operand): forward, layer k [out][in]; adjoint, its transpose
    const void *W[kFuseMaxNh];
    const R *b[kFuseMaxNh];       // forward: hidden-layer biases
    R *Z[kFuseMaxNh];             // pre-activations [rows][H]: written by forward, read by adjoint
    const R *Wout, *bout;         // output layer [dout][H], [dout]
    const double *Wout64, *bout64;   // FP32 data, forward with dout = 1 (the energy NN): the same in FP64
    // FP8 forward only (1 / 1 / NULL otherwise): layer k's product is multiplied by zscale[k]
    // before its bias; the input of hidden layer k >= 1 is stored as h * hinv[k]; the layer-0
    // input (the density) as rho_f * xinv[f] (the calibrated per-feature scales, whose inverses
    // are folded into the layer-0 operand)
    float zscale[kFuseMaxNh];
    float hinv[kFuseMaxNh];
    const float *xinv;
    // The exchange around a message NN, done by the launch itself.  copy_rng (or NULL: no copies):
    // row r's ghost copies are copy_idx[copy_rng[r].x .. y).  Forward: the outputs are also written
    // to the copies' rows of Cg.  Adjoint: the copies' rows of Gg are added to G, in that order.
    const int2 *copy_rng;
    const int32_t *copy_idx;
    R *Cg;
    const R *Gg;
    // Radial form's residual (NULL otherwise), [rows][K].  Forward: resid is added to the outputs.
    // Adjoint: next_in is added to G (after the copies), and the sum is kept in next_out.
    const R *resid;
    const R *next_in;
    R *next_out;
    // Adjoint of the energy NN (dout = 1), which takes no G: row r's output adjoint is
    // seed_scale g w[perm[r]] (g = *seed_g or 1; w = seed_w in caller order or 1)
    double seed_scale;
    const double *seed_g, *seed_w;
    const int32_t *perm;
    const R *G;                   // adjoint of a message NN: output adjoint [rows][K]
    R *C;                         // forward: outputs [rows][dout]; adjoint: dE/dS [rows][NL*K]
};
using FusedNN = FusedNNT<float>;
using FusedNN64 = FusedNNT<double>;

// Segments of the same NN shape (the elements' rows of one layer, or locals and ghosts) for
// one launch of the fused kernels.  Kernel arguments stay well under 4 KiB.
constexpr int kFuseMaxSeg = 4;
template <typename R> struct FusedMultiT {
    int n;
    int64_t tile0[kFuseMaxSeg + 1];   // first block of each segment; tile0[n] = total blocks
    FusedNNT<R> seg[kFuseMaxSeg];
};
using FusedMulti = FusedMultiT<float>;
static_assert(sizeof(FusedMulti) < 3072, "kernel arguments");

// Whether the fused kernels take these shapes (every operand type: FP8 runs the forward only,
// its adjoint takes BF16 operands).
bool fused_nn_ok(int F, int H, int nh, int dout, int NLK);

// FP8 calibration from FP32 activations: out[f] = max over the rows of |rho_f| of the density of
// S [rows][NL*K] (f = (l, a <= b) in the feature order); out[F] must be zero on entry.
void density_absmax(hipStream_t st, int L, int K, int64_t rows, const DensityConsts &dc, const float *S, float *out);
// out[0] = max(out[0], max |SiLU(z)|) over Z [rows][ld], H columns; out must be zero initially.
void silu_absmax(hipStream_t st, int64_t rows, int H, int ld, const float *Z, float *out);
// Forward (fwd = true: density of S, hidden layers, Z stores, output layer with FP64
// accumulation) or adjoint (fwd = false: output layer, hidden layers, first layer, density
// adjoint to dE/dS) over nseg segments of one NN shape, kFuseMaxSeg to a launch; returns the
// launches.
int mlp_fused_segments(hipStream_t st, OpType op, bool fwd, const FusedNN *segs, int nseg);

// The same in FP64 (data, operands and accumulation): whether its kernels take a model, its operands
// (for K chunk kc of 8 and block j of 16 rows, lane l holds the pair k = 8 kc + 2 (l / 16) .. of row
// 16 j + l % 16 at ((kc nblk + j) 64 + l) 2, zero past the matrix), and the launches.
bool fused64_ok(int L, int K, int F, int H, int nh);
size_t packed64_elems(int rows, int cols);
// The matrices of one NN: element (r, c) at src + r ld_row + c ld_col of the NN's weights, its packed
// form from dst of the NN's operands; the NNs are src_stride and dst_stride elements apart.
struct Pack64Matrix { int rows, cols, ld_row, ld_col; int64_t src, dst; };
struct Pack64 { int n; int64_t src_stride, dst_stride; Pack64Matrix m[2 * kFuseMaxNh]; };
void pack_operands64(hipStream_t st, const Pack64 &pk, int count, const double *src, double *dst);
int mlp64_segments(hipStream_t st, bool fwd, const FusedNN64 *segs, int nseg);

inline size_t op_bytes(OpType op) { return op == OpType::F32 ? 4 : (op == OpType::BF16 ? 2 : 1); }

}  // namespace reann
