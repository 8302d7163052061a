// Dropout masks for the dropout variant of the block: a counter-based generator (Philox4x32 with
// 10 rounds, Salmon et al., SC 2011) turned into keep bits.
//
// Attention probabilities: the masks are materialised once per pass as bit arrays, because the
// attention kernels hold the score tile in MFMA accumulator layouts (a lane of the forward and dQ
// kernels owns 16 keys of one query, a lane of the dK/dV kernel 16 queries of one key) and
// regenerating 16-byte counters in those layouts would cost several generator calls per element.
// One wavefront covers 64 queries and 128 keys; per group of 16 keys every lane makes one
// generator call for its query, keeps the 16 bits for the row-major array and contributes them to
// 16 wavefront ballots, each of which is the column-major word pair "64 queries of one key".
//   rowbits[(bh * S + i) * wpr + j / 32]  bit j % 32  = keep(i, j)        (forward, dQ)
//   colbits[(bh * S + j) * wpr + i / 32]  bit i % 32  = keep(i, j)        (dK / dV)
// What bounds it is vector arithmetic: a call's 20 products of 32 x 32 bits, each at a quarter of the rate, about 60 plain
// operations around them, and 16 comparisons with what places their bits.  20 of the plain ones are exclusive ors of three
// values, one instruction each instead of two.  A ballot is the comparison's own mask, put into its lane by v_writelane (a select
// per lane and half took four instructions).  us, with selects / v_writelane / one instruction for three values: 64 pairs of
// S 1024, row-major alone 17.0 / 14.0 / 12.5, both 26.9 / 18.1 / 17.1; 64 of S 2048, row-major 41.0 before, 36.9 now, both 89.5 /
// 57.6 / 53.4.
// wpr = 2 * ceil(S / 64) words per row.  Only words that a causal kernel can touch are written:
// keys below 64 * (i / 64 + 1).
//
// Outputs of the two halves: one pass, out = residual + keep * scale * in (forward) or
// out = keep * scale * in (backward), one generator call per 16 consecutive columns.
#include "gx_kernels.h"

namespace gx {
namespace {

struct Philox {
  unsigned x[4];
};

GX_DEVINL Philox philox4x32_10(unsigned c0, unsigned c1, unsigned c2, unsigned c3, unsigned k0, unsigned k1) {
  constexpr unsigned M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; r++) {
    const unsigned long long p0 = (unsigned long long)M0 * c0, p1 = (unsigned long long)M1 * c2;
    const unsigned hi0 = (unsigned)(p0 >> 32), lo0 = (unsigned)p0, hi1 = (unsigned)(p1 >> 32), lo1 = (unsigned)p1;
    c0 = __builtin_amdgcn_bitop3_b32(hi1, c1, k0, 0x96);      // hi1 ^ c1 ^ k0 in one instruction
    c1 = lo1;
    c2 = __builtin_amdgcn_bitop3_b32(hi0, c3, k1, 0x96);
    c3 = lo0;
    k0 += W0;
    k1 += W1;
  }
  return Philox{{c0, c1, c2, c3}};
}

// element e is kept: byte e of the 16 random bytes >= t
GX_DEVINL bool keep_of(const Philox& r, int e, unsigned t) { return ((r.x[e >> 2] >> (8 * (e & 3))) & 0xFFu) >= t; }
GX_DEVINL unsigned keep_bits16(const Philox& r, unsigned t) {
  unsigned bits = 0;
#pragma unroll
  for (int e = 0; e < 16; e++) bits |= keep_of(r, e, t) ? 1u << e : 0u;
  return bits;
}

// One wavefront: 64 queries x MASK_GROUPS groups of 16 keys.
constexpr int MASK_GROUPS = 8;

template <bool COLS>
__global__ void __launch_bounds__(64) attn_mask_kernel(unsigned* __restrict__ rowbits, unsigned* __restrict__ colbits,
                                                       int S, int wpr, int nchunk, int heads, int head0, unsigned k0,
                                                       unsigned k1, unsigned t) {
  const int lane = threadIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int blk = blockIdx.x / nchunk, chunk = blockIdx.x % nchunk;
  const int nl = gridDim.y;
  const int groups = min(4 * (blk + 1), 2 * wpr);      // 16-key groups up to the end of the diagonal tile
  const int jg0 = chunk * MASK_GROUPS;
  if (jg0 >= groups) return;                           // wavefront-uniform
  const int jg1 = min(jg0 + MASK_GROUPS, groups);      // jg0, jg1 and groups are even
  const int i = 64 * blk + lane;
  const size_t bh = (size_t)b * nl + h;
  const unsigned c2 = (unsigned)(b * heads + head0 + h);
  unsigned word = 0;
  for (int jg = jg0; jg < jg1; jg++) {
    const Philox r = philox4x32_10((unsigned)i, (unsigned)jg, c2, 1u, k0, k1);
    // lane e of (lo, hi): the 64 queries of key e, which is the wavefront's mask of the comparison itself
    unsigned kb = 0, lo = 0, hi = 0;
#pragma unroll
    for (int e = 0; e < 16; e += 4) {
      unsigned long long col[4];
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const bool keep = keep_of(r, e + k, t);
        kb |= keep ? 1u << (e + k) : 0u;
        if (COLS) col[k] = __builtin_amdgcn_ballot_w64(keep);
      }
      // (two wait states between a comparison and the read of its mask)
      if (COLS)
        asm("s_nop 1\n\t"
            "v_writelane_b32 %0, %2, %10\n\tv_writelane_b32 %1, %3, %10\n\t"
            "v_writelane_b32 %0, %4, %11\n\tv_writelane_b32 %1, %5, %11\n\t"
            "v_writelane_b32 %0, %6, %12\n\tv_writelane_b32 %1, %7, %12\n\t"
            "v_writelane_b32 %0, %8, %13\n\tv_writelane_b32 %1, %9, %13"
            : "+v"(lo), "+v"(hi)
            : "s"((unsigned)col[0]), "s"((unsigned)(col[0] >> 32)), "s"((unsigned)col[1]), "s"((unsigned)(col[1] >> 32)),
              "s"((unsigned)col[2]), "s"((unsigned)(col[2] >> 32)), "s"((unsigned)col[3]), "s"((unsigned)(col[3] >> 32)),
              "n"(e), "n"(e + 1), "n"(e + 2), "n"(e + 3));
    }
    word |= kb << (16 * (jg & 1));
    if (jg & 1) {
      if (i < S) rowbits[(bh * S + i) * wpr + (jg >> 1)] = word;
      word = 0;
    }
    if (COLS) {
      const int j = 16 * jg + lane;
      if (lane < 16 && j < S)
        *reinterpret_cast<unsigned long long*>(colbits + (bh * S + j) * wpr + 2 * blk) =
            (unsigned long long)hi << 32 | lo;
    }
  }
}

template <typename T>
struct Vec16B;                       // 16 bytes of T
template <>
struct Vec16B<float> {
  using type = f32x4;
  static constexpr int N = 4;
};
template <>
struct Vec16B<bf16> {
  using type = bf16x8;
  static constexpr int N = 8;
};

// one lane: the 16 consecutive columns of one generator call, moved as 16-byte vectors
template <typename T>
__global__ void __launch_bounds__(256) dropout_rows_kernel(const T* __restrict__ in, const T* __restrict__ resid,
                                                           T* __restrict__ out, int rows, int cols, int groups,
                                                           unsigned stream, unsigned k0, unsigned k1, unsigned t,
                                                           float scale) {
  using V = typename Vec16B<T>::type;
  constexpr int N = Vec16B<T>::N;
  const long id = (long)blockIdx.x * 256 + threadIdx.x;
  if (id >= (long)rows * groups) return;
  const int r = (int)(id / groups), cg = (int)(id % groups);
  const unsigned kb = keep_bits16(philox4x32_10((unsigned)r, (unsigned)cg, 0u, stream, k0, k1), t);
#pragma unroll
  for (int q = 0; q < 16 / N; q++) {
    const int c = 16 * cg + N * q;
    if (c >= cols) break;                                // cols is a multiple of N
    const size_t idx = (size_t)r * cols + c;
    const V v = *reinterpret_cast<const V*>(in + idx);
    V o;
    if (resid) o = *reinterpret_cast<const V*>(resid + idx);
#pragma unroll
    for (int e = 0; e < N; e++) {
      const float x = ((kb >> (N * q + e)) & 1u) ? (float)v[e] * scale : 0.f;
      o[e] = (T)(resid ? (float)o[e] + x : x);
    }
    *reinterpret_cast<V*>(out + idx) = o;
  }
}

}  // namespace

int attn_mask_wpr(int S) { return 2 * cdiv(S, 64); }

hipError_t attn_mask(unsigned* rowbits, unsigned* colbits, int B, int nl, int S, int heads, int head0, unsigned k0,
                     unsigned k1, int t, hipStream_t s) {
  if (!rowbits || S <= 0 || t < 0 || t > 255) return hipErrorInvalidValue;
  const int wpr = attn_mask_wpr(S), nchunk = cdiv(2 * wpr, MASK_GROUPS);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(S, 64) * nchunk, nl, B), dim3(64), 0, s, rowbits, colbits, S, wpr, nchunk, heads,
                       head0, k0, k1, (unsigned)t);
  };
  if (colbits) go(attn_mask_kernel<true>);
  else go(attn_mask_kernel<false>);
  return hipGetLastError();
}

hipError_t dropout_rows(bool bf, const void* in, const void* resid, void* out, int rows, int cols, unsigned stream,
                        unsigned k0, unsigned k1, int t, hipStream_t s) {
  if (t < 0 || t > 255 || (cols & (bf ? 7 : 3))) return hipErrorInvalidValue;
  const int groups = cdiv(cols, 16);
  const long n = (long)rows * groups;
  const float scale = 256.0f / (256.0f - (float)t);
  const dim3 grid((unsigned)cdiv(n, 256L));
  if (bf)
    hipLaunchKernelGGL(dropout_rows_kernel<bf16>, grid, dim3(256), 0, s, static_cast<const bf16*>(in),
                       static_cast<const bf16*>(resid), static_cast<bf16*>(out), rows, cols, groups, stream, k0, k1,
                       (unsigned)t, scale);
  else
    hipLaunchKernelGGL(dropout_rows_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(in),
                       static_cast<const float*>(resid), static_cast<float*>(out), rows, cols, groups, stream, k0,
                       k1, (unsigned)t, scale);
  return hipGetLastError();
}

}  // namespace gx
