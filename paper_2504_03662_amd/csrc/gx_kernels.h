// Internal launcher interface between the layer driver and the kernel translation units.
#pragma once
#include "gx_common.h"

namespace gx {

// true when the current device is the architecture this library is built for (cached per process)
bool device_is_gfx950();

// C[M,N] = op(A) * op(B), all matrices row-major with leading dimensions in elements.
//   NN: A is [M,K], B is [K,N]      (forward: activations times "in x out" weights)
//   NT: A is [M,K], B is [N,K]      (input gradient: dY times W^T, reduction over W's columns)
//   TN: A is [K,M], B is [K,N]      (weight gradient: X^T times dY, reduction over tokens)
enum Layout { LAY_NN = 0, LAY_NT = 1, LAY_TN = 2 };

enum Epilogue {
  EPI_STORE = 0,   // C = acc                                   (storage type)
  EPI_BIAS,        // C = acc + bias[n]            (bias may be null)
  EPI_RESID,       // p = acc + bias[n]; aux = p if aux; C = resid + p
  EPI_GELU,        // z = acc + bias[n]; C = gelu'(z); aux = gelu(z)  (erf form, or tanh form if gelu_tanh)
  EPI_DGELU,       // C = acc * z[m,n], z holding what EPI_GELU left in C
  EPI_F32,         // C (fp32) = acc
  EPI_F32_ACC,     // C (fp32) += acc
  EPI_PART         // C[part] (fp32) = acc over the part's reduction steps (the bf16 launcher's own: gemm_bf16_split)
};

struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  int M, N, K;
  int lda, ldb, ldc;
  const void* bias;    // [N], storage type
  const void* resid;   // [M, ldc], storage type
  void* aux;           // [M, ldc], storage type
  union {
    const void* z;     // [M, ldc], storage type: EPI_DGELU's multiplier
    const void* next;  // bf16 NN only, optional: weights that the next product of the chain reads (its B), 16-byte
  };                   // aligned; compute units that this product leaves idle may bring them nearer
  int gelu_tanh;       // EPI_GELU: tanh form of GELU instead of the erf form
  unsigned next_bytes;
  float* colpart;      // bf16 EPI_DGELU, optional: partial column sums of the stored C over blocks of 64
                       // rows, [ceil(M / 64)][N] fp32 (stage 1 of the bias gradient; finished by colsum_finish).
                       // fp32 TN, optional: column sums of B, [N], stored or, with EPI_F32_ACC, added to (a slower instance)
  // set by the bf16 launcher only (callers leave them 0): a launch that covers the super-tiles
  // (2 x 2 kernel tiles) numbered tile_first onwards in the tile walk, four workgroups each, the
  // tile-rows that the walk takes at a time, and how many workgroups have a tile; EPI_PART: tile_first holds
  // the reduction steps of a part
  int tail, tile_first, group, tiles;
};
static_assert(sizeof(GemmArgs) == 112, "a launch copies it: 136 bytes cost a product 0.2 us");

hipError_t gemm_bf16(Layout lay, Epilogue epi, const GemmArgs& g, hipStream_t s);
// Which tile gemm_bf16 takes for an M x N x K product (column_sums: EPI_DGELU), host code, so that tests can
// tell what their sizes reach: 0 256x256, 1 256x192, 2 192x256, 3 256x128, 4 128x128, 5 64x128, 6 64x64,
// 7 256x256 with the remainder in 128x128.
extern "C" int gx_bf16_tile(int M, int N, int K, int column_sums);
// Whether reading ahead can pay for a product of own_bytes of weights before one of next_bytes in a call of call_bytes
bool read_ahead_pays(long own_bytes, long next_bytes, long call_bytes);
// Workgroups without a tile with which gemm_bf16 then launches an NN product (host code, for tests)
extern "C" int gx_bf16_read_ahead(int M, int N, int K, long next_bytes, long call_bytes);
// Forward products of few tokens: into how many parts gemm_bf16_split cuts the reduction (1: it is not for this product),
// and the scratch that takes, one fp32 copy of C per part.  extern "C": host code, for tests.
extern "C" int gx_bf16_split(int M, int N, int K);
size_t gemm_bf16_split_bytes(int M, int N, int K);
// The NN product with its reduction cut into parts, and a second launch that adds them in order and does the epilogue
hipError_t gemm_bf16_split(Epilogue epi, const GemmArgs& g, float* scratch, hipStream_t s);
// Which kernel gemm_f32 takes (host code, for tests): 0 32x32 tiles with four wavefronts, 64x64 with 1 two and 2 one per 32x32
// block, 3 and 4 the same for short reductions
extern "C" int gx_f32_tile(int M, int N, int K);
hipError_t gemm_f32(Layout lay, Epilogue epi, const GemmArgs& g, hipStream_t s);
// An NT product and a TN product (fp32, stored or added to) in one launch, both in 32 x 32 tiles
hipError_t gemm_f32_pair(Epilogue nt_epi, const GemmArgs& nt, bool accumulate, const GemmArgs& tn, hipStream_t s);

// Causal attention over the local heads.  qkv is [T, 3*Hl] with column blocks [Q | K | V], each
// head's dh columns contiguous; ctx / dctx are [T, Hl]; lse and dsum are [B, nl, S] fp32.
struct AttnArgs {
  const void* qkv;
  void* ctx;          // fwd out / bwd in
  float* lse;         // fwd out / bwd in: log-sum-exp of the scaled, masked scores per row
  const void* dctx;   // bwd in
  void* dqkv;         // bwd out, same layout as qkv
  float* dsum;        // bwd scratch: rowsum(dctx * ctx)
  int B, S, nl, dh;
  bool alone;         // bf16 bwd: no weight gradient runs beside it (a rule on sizes: it may decide which kernel is taken)
  // dropout of the probabilities (rowbits == nullptr: none): keep bits from attn_mask, row-major for
  // the forward and dQ kernels, column-major for dK / dV (bf16 path; the fp32 path reads rowbits
  // throughout), wpr words per row, kept probabilities multiplied by keep_scale
  const unsigned* rowbits;
  const unsigned* colbits;
  int wpr;
  float keep_scale;
};
hipError_t attn_fwd_bf16(const AttnArgs& a, hipStream_t s);
hipError_t attn_bwd_bf16(const AttnArgs& a, hipStream_t s);
// Over how many wavefronts the forward (backward: the dQ) kernel spreads the keys of a query block: 1, 2 or 4 (host code,
// so that tests can tell which kernel their sizes reach)
extern "C" int gx_attn_key_shares(int B, int S, int nl, int dh, int backward);
// Whether the backward kernels of a pass share a launch (bf16: of a pass that stays on one stream; host code)
extern "C" int gx_attn_bf16_one_launch(int B, int S, int nl);
extern "C" int gx_attn_f32_one_launch(int B, int S, int nl, int dh);
hipError_t attn_fwd_f32(const AttnArgs& a, hipStream_t s);
hipError_t attn_bwd_f32(const AttnArgs& a, hipStream_t s);

// Dropout (Philox4x32-10 bytes; an element is dropped iff its byte < t, t in 0..255).
// Keep bits of the attention probabilities of B x nl (sample, local head) pairs, heads `head0`..
// of a model with `heads` heads: rowbits / colbits are [B * nl * S * attn_mask_wpr(S)] words
// (colbits may be null).  Counter (i, j / 16, b * heads + head0 + h, 1), byte j % 16.
int attn_mask_wpr(int S);
hipError_t attn_mask(unsigned* rowbits, unsigned* colbits, int B, int nl, int S, int heads, int head0, unsigned k0,
                     unsigned k1, int t, hipStream_t s);
// out = (resid ? resid : 0) + keep * 256 / (256 - t) * in over [rows, cols]; counter
// (row, column / 16, 0, stream), byte column % 16.  out may alias in.  The fourth counter word
// separates the masks: 1 attention probabilities (attn_mask), 2 and 3 the two halves' outputs.
constexpr unsigned DROP_STREAM_ATTN_OUT = 2, DROP_STREAM_MLP_OUT = 3;
hipError_t dropout_rows(bool bf16, const void* in, const void* resid, void* out, int rows, int cols,
                        unsigned stream, unsigned k0, unsigned k1, int t, hipStream_t s);

// Row-wise and column-sum kernels, templated on storage type through the `bf16` switch.
// LayerNorm forward: y = g * (x - mean) * rstd + b; writes mean/rstd per row.
hipError_t ln_fwd(bool bf16, const void* x, const void* g, const void* b, void* y, float* mean, float* rstd,
                  int rows, int cols, float eps, hipStream_t s);
// Column reductions are two-stage and fixed-order: a producer leaves per-block partial rows
// part[nblk][cols] (fp32), and ONE launch at the end of a pass finishes all of them.
struct FinishSeg {
  const float* part;   // [nblk][cols]
  float* out;          // [cols], written or, with accumulate, added to
  int nblk, cols, accumulate;
  int wg0;             // set by colsum_finish
};
constexpr int FINISH_MAX = 10;
struct FinishArgs {
  FinishSeg seg[FINISH_MAX];
  int nseg;
};
hipError_t colsum_finish(const FinishSeg* segs, int nseg, hipStream_t s);
// LayerNorm backward in one pass: dx = (resid ? resid : 0) + LNbwd(dy), and partial column sums
// part[a][ln_bwd_blocks(..)][cols]: a = 0 sum dy * xhat (gain gradient), 1 sum dy (bias gradient) and,
// with nsum = 4 (resid required), 2 sum resid, 3 sum dx.
hipError_t ln_bwd(bool bf16, const void* dy, const void* x, const void* g, const float* mean, const float* rstd,
                  const void* resid, void* dx, int rows, int cols, int nsum, float* part, hipStream_t s);
int ln_bwd_blocks(bool bf16, int rows, int cols);
// Stage 1 of the column sums of a [rows, cols] matrix: part[colsum_blocks(rows)][cols].
hipError_t colsum_partial(bool bf16, const void* a, int rows, int cols, int ld, float* part, hipStream_t s);
int colsum_blocks(int rows);

}  // namespace gx
