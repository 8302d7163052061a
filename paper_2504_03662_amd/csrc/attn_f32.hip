// fp32 causal attention on v_mfma_f32_32x32x2_f32: every product and sum is a full fp32 one, in a
// fixed order.
//
// A workgroup owns 32 query rows (forward, dQ) or 32 key rows (dK / dV) of one (sample, head); its
// 4 wavefronts take every 4th 32-row tile of the other side and their partial results are merged
// through LDS in wavefront order.  Scores are taken transposed to the owner (a lane owns one query,
// or one key, of every accumulator), so that an accumulator register is, as it stands, an operand
// of the next product: register v of a lane in half g holds tile row 8 (v / 4) + 4 g + v % 4, and a
// 32x32x2 product takes one row from each half.  Operands therefore come straight from global
// memory (16 B per lane along the head dimension, or 128 B runs of one row per half wavefront) with
// no staging and no barrier inside the loop; a tile costs a wavefront 4096 to 16384 cycles of the
// matrix pipe against 0.5 to 1 kB per row pair of cache reads, so the matrix pipe is the bound once
// a few wavefronts share a SIMD.
// With few blocks dQ and dK / dV share a launch (one_launch()).
// Head dimensions up to 128 are padded with zeros to 32, 64 or 128.  With 16 heads of 64, S 512, batch 2:
// forward 1031 -> 25 us, dQ 2222 -> 41 us, dK / dV 2426 -> 47 us against one wavefront per row with
// scalar multiply-adds; with 8 heads of 128 forward 1251 -> 43 us, backward 5448 -> 142 us, although dK / dV then
// needs more than the 512 registers there are and spills 43 (176 bytes a lane; 28, 116 bytes, with padding).  In the launch that
// holds both kernels it spills 94 (380 bytes; 34, 124 bytes, with padding), which is still the faster form where it is taken: 8
// heads of 128, S 512, 118 -> 79 us.  dQ with padding to 64 spills one register: its text in a function that two kernels share
// takes 256 instead of 251 (16 heads of 50, S 512, batch 2: both kernels 139.7 -> 141 us), but the same function is faster at head
// dim 64 (16 heads, S 1024, batch 2: 240 -> 224).
#include "gx_kernels.h"

namespace gx {
namespace {

constexpr int PARTS = 4;          // wavefronts of a workgroup

GX_DEVINL f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; v++) z[v] = 0.f;
  return z;
}
GX_DEVINL int acc_row(int v, int g) { return 8 * (v >> 2) + 4 * g + (v & 3); }
GX_DEVINL f32x16 mfma(float a, float b, const f32x16& c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// One lane's share of 32 rows by DHP columns whose reduction index is the column: chunk c holds columns
// 8 c + 4 g .. + 3 of the lane's row.  EXACT: the head dimension is DHP, so that rows start at 16-byte
// boundaries and none is padded; otherwise columns beyond dh read as zero, one at a time.
template <int DHP, bool EXACT>
GX_DEVINL void load_rows(const float* row, int dh, int g, f32x4 (&out)[DHP / 8]) {
#pragma unroll
  for (int c = 0; c < DHP / 8; c++) {
    const int d = 8 * c + 4 * g;
    if (EXACT) {
      out[c] = *reinterpret_cast<const f32x4*>(row + d);
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++) out[c][e] = (d + e < dh) ? row[d + e] : 0.f;
    }
  }
}
// a per-row vector's values for the 16 tile rows of this lane's accumulator registers
GX_DEVINL void load_row_stats(const float* tile, int rows, int g, float (&out)[16]) {
  typedef f32x4 __attribute__((aligned(4))) f32x4_u;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    if (rows >= 32) {
      const f32x4 t = *reinterpret_cast<const f32x4_u*>(tile + 8 * q + 4 * g);
#pragma unroll
      for (int e = 0; e < 4; e++) out[4 * q + e] = t[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; e++) out[4 * q + e] = tile[min(8 * q + 4 * g + e, rows - 1)];
    }
  }
}
// 32 x 32 scores: sum over columns of a[row] * b[col]
template <int DHP>
GX_DEVINL f32x16 row_product(const f32x4 (&a)[DHP / 8], const f32x4 (&b)[DHP / 8]) {
  f32x16 s = zero16();
#pragma unroll
  for (int c = 0; c < DHP / 8; c++)
#pragma unroll
    for (int e = 0; e < 4; e++) s = mfma(a[c][e], b[c][e], s);
  return s;
}

// acc[dt][d][col] += sum over the 32 rows r of the tile of src[r][d] * w[r][col], w being an
// accumulator.  On the tile that touches the diagonal some weights stand for masked pairs, on a partial
// last tile for rows that are not there, and are 0; a value of src that is not finite must not reach the
// columns it is masked for (0 * inf), so such a tile then takes the second form: weights through LDS and
// one multiply-add per pair that counts.
// LATER: a row is masked for the columns below it (keys for queries); else for those above it.
template <int DHP, bool EXACT, bool LATER>
GX_DEVINL void col_product(f32x16 (&acc)[DHP / 32], const f32x16& w, const float* src, int ld, int rows, int dh,
                           bool diagonal, float* spill, int lane) {
  const int g = lane >> 5, l32 = lane & 31;
  constexpr int CH = DHP >= 64 ? 2 : 1;                      // column blocks in registers at a time
#pragma unroll
  for (int d0 = 0; d0 < DHP / 32; d0 += CH) {
    float x[CH][16];
#pragma unroll
    for (int c = 0; c < CH; c++) {
      const int dd = 32 * (d0 + c) + l32;
      const int d = EXACT ? dd : min(dd, dh - 1);            // columns beyond dh are never stored
      if (rows >= 32) {
        const unsigned off = (unsigned)(4 * g * ld + d);
#pragma unroll
        for (int v = 0; v < 16; v++) x[c][v] = (src + (size_t)acc_row(v, 0) * ld)[off];
      } else {
        // rows beyond the tensor have weight 0 and take the last row's values; where that row is not finite
        // the second form leaves them out
#pragma unroll
        for (int v = 0; v < 16; v++) x[c][v] = src[(unsigned)(min(acc_row(v, g), rows - 1) * ld + d)];
      }
    }
    bool bad = false;
    if (diagonal || rows < 32) {
#pragma unroll
      for (int c = 0; c < CH; c++)
#pragma unroll
        for (int v = 0; v < 16; v++) bad |= !(fabsf(x[c][v]) < INFINITY);
    }
    if (__builtin_amdgcn_ballot_w64(bad)) {
#pragma unroll
      for (int v = 0; v < 16; v++) spill[acc_row(v, g) * 33 + l32] = w[v];
      for (int r = 0; r < min(rows, 32); r++) {
        const float wr = spill[r * 33 + l32];
        if (diagonal && (LATER ? r > l32 : r < l32)) continue;
#pragma unroll
        for (int c = 0; c < CH; c++)
#pragma unroll
          for (int v = 0; v < 16; v++) {
            const int d = 32 * (d0 + c) + acc_row(v, g);
            if (d < dh) acc[d0 + c][v] = fmaf(wr, src[(size_t)r * ld + d], acc[d0 + c][v]);
            if ((v & 3) == 3) asm volatile("" ::: "memory");     // a rare path: few loads in flight, few registers
          }
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; v++)
#pragma unroll
        for (int c = 0; c < CH; c++) acc[d0 + c] = mfma(x[c][v], w[v], acc[d0 + c]);
    }
  }
}

// Adds the parts' accumulators in the order of the wavefronts; the sum is complete in wavefront 0.
template <int DT>
GX_DEVINL void merge_parts(f32x16 (&acc)[DT], float* park, int part, int lane) {
  __syncthreads();
  if (part > 0)
#pragma unroll
    for (int dt = 0; dt < DT; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) park[((part - 1) * DT * 16 + 16 * dt + v) * 64 + lane] = acc[dt][v];
  __syncthreads();
  if (part == 0)
    for (int p = 0; p < PARTS - 1; p++)
#pragma unroll
      for (int dt = 0; dt < DT; dt++)
#pragma unroll
        for (int v = 0; v < 16; v++) acc[dt][v] += park[(p * DT * 16 + 16 * dt + v) * 64 + lane];
}
// one column (= one row of the tensor) of a transposed result: dst[d] = acc * scale
template <int DHP, bool EXACT>
GX_DEVINL void store_column(const f32x16 (&acc)[DHP / 32], float* dst, float scale, int dh, int g) {
#pragma unroll
  for (int dt = 0; dt < DHP / 32; dt++)
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int d = 32 * dt + 8 * q + 4 * g;
      const f32x4 v = {acc[dt][4 * q] * scale, acc[dt][4 * q + 1] * scale, acc[dt][4 * q + 2] * scale,
                       acc[dt][4 * q + 3] * scale};
      if (EXACT) {
        *reinterpret_cast<f32x4*>(dst + d) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
          if (d + e < dh) dst[d + e] = v[e];
      }
    }
}

// LDS: the parts' (O, m, l) or the spilled weights of a diagonal tile (one area per wavefront)
template <int DHP>
constexpr int lds_floats() {
  const int merge = (PARTS - 1) * (DHP / 2 + 2) * 64, spill = PARTS * 32 * 33;
  return merge > spill ? merge : spill;
}

struct Args {
  const float *qkv, *ctx, *dctx;
  float *out, *lse, *dsum;      // out: ctx (forward) or dqkv (backward)
  int S, nl, dh, npair;
  const unsigned* rowbits;      // dropout: keep bits, [pair][S][wpr] words, bit j % 32 of word j / 32; or null
  int wpr;
  float keep_scale;
};
// the (sample, head) pair and tile of workgroup `blk`; the tiles with most work come first
struct Where {
  int b, h, tile, ld;
  const float *q, *k, *v;
  GX_DEVINL Where(const Args& a, int blk, bool last_first) {
    const int pair = blk % a.npair, n = (a.S + 31) / 32, i = blk / a.npair;
    tile = last_first ? n - 1 - i : i;
    h = pair % a.nl;
    b = pair / a.nl;
    ld = 3 * a.nl * a.dh;
    q = a.qkv + (size_t)b * a.S * ld + h * a.dh;
    k = q + a.nl * a.dh;
    v = k + a.nl * a.dh;
  }
};

// What exponents are taken relative to.  The largest score that a part has seen is -inf while all of them
// are (products that leave the fp32 range); such keys get weight 0, not that of -inf - -inf.
GX_DEVINL float finite_ref(float m) { return m == -INFINITY ? 0.f : m; }

template <int DHP, bool EXACT>
__global__ void __launch_bounds__(64 * PARTS, DHP <= 64 ? 2 : 1) attn_fwd_f32_kernel(Args a) {
  __shared__ float lds[lds_floats<DHP>()];
  const int lane = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  const Where w(a, blockIdx.x, true);
  const int i0 = 32 * w.tile, i = i0 + l32;
  const float scale = rsqrtf((float)a.dh);
  const size_t row = ((size_t)w.b * a.nl + w.h) * a.S + min(i, a.S - 1);
  f32x4 qf[DHP / 8];
  load_rows<DHP, EXACT>(w.q + (size_t)min(i, a.S - 1) * w.ld, a.dh, g, qf);
  f32x16 o[DHP / 32];
#pragma unroll
  for (int dt = 0; dt < DHP / 32; dt++) o[dt] = zero16();
  float m = -INFINITY, l = 0.f;
  for (int t = part; t <= w.tile; t += PARTS) {
    const int j0 = 32 * t;
    f32x4 kf[DHP / 8];
    load_rows<DHP, EXACT>(w.k + (size_t)min(j0 + l32, a.S - 1) * w.ld, a.dh, g, kf);
    f32x16 s = row_product<DHP>(kf, qf);                         // S^T[j][i]
    float mx = -INFINITY;
    const float mold = m;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      s[v] = (j0 + acc_row(v, g) <= i) ? s[v] * scale : -INFINITY;
      mx = fmaxf(mx, s[v]);
    }
    m = fmaxf(m, max_across_halves(mx));
    const float ref = finite_ref(m), alpha = expf(mold - ref);
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      s[v] = (j0 + acc_row(v, g) <= i) ? expf(s[v] - ref) : 0.f;
      sum += s[v];
    }
    l = l * alpha + sum;                                         // of the undropped probabilities
    if (a.rowbits) {
      const unsigned bits = a.rowbits[row * a.wpr + t];
#pragma unroll
      for (int v = 0; v < 16; v++) s[v] = ((bits >> acc_row(v, g)) & 1u) ? s[v] * a.keep_scale : 0.f;
    }
#pragma unroll
    for (int dt = 0; dt < DHP / 32; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) o[dt][v] *= alpha;
    col_product<DHP, EXACT, true>(o, s, w.v + (size_t)j0 * w.ld, w.ld, a.S - j0, a.dh, t == w.tile, lds + part * 32 * 33,
                           lane);
  }
  // merge the parts' (m, l, O); a part without a tile has m = -inf, l = 0, O = 0 and adds nothing
  constexpr int VALS = DHP / 2 + 2;
  __syncthreads();
  if (part > 0) {
    float* p = lds + (part - 1) * VALS * 64 + lane;
    p[0] = m;
    p[64] = l;
#pragma unroll
    for (int dt = 0; dt < DHP / 32; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) p[(2 + 16 * dt + v) * 64] = o[dt][v];
  }
  __syncthreads();
  if (part > 0) return;
  for (int pp = 0; pp < min(PARTS - 1, w.tile); pp++) {          // part 0 always has a tile; part p when tile >= p
    const float* p = lds + pp * VALS * 64 + lane;
    const float mm = fmaxf(m, p[0]), ref = finite_ref(mm), a0 = expf(m - ref), a1 = expf(p[0] - ref);
    l = l * a0 + p[64] * a1;
    m = mm;
#pragma unroll
    for (int dt = 0; dt < DHP / 32; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) o[dt][v] = o[dt][v] * a0 + p[(2 + 16 * dt + v) * 64] * a1;
  }
  l += __shfl_xor(l, 32, 64);
  if (i >= a.S) return;
  store_column<DHP, EXACT>(o, a.out + ((size_t)w.b * a.S + i) * (a.nl * a.dh) + w.h * a.dh, 1.0f / l, a.dh, g);
  if (g == 0) a.lse[row] = m + logf(l);
}

// D_i = dO_i . O_i, dS_ij = P_ij (dO_i . V_j - D_i), dQ_i = scale sum_j dS_ij K_j
template <int DHP, bool EXACT>
GX_DEVINL void dq_block(const Args& a, int blk, float* lds) {
  const int lane = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  const Where w(a, blk, true);
  const int i0 = 32 * w.tile, i = i0 + l32, ic = min(i, a.S - 1);
  const float scale = rsqrtf((float)a.dh);
  const size_t row = ((size_t)w.b * a.nl + w.h) * a.S + ic;
  const size_t head_row = ((size_t)w.b * a.S + ic) * (a.nl * a.dh) + w.h * a.dh;
  f32x4 qf[DHP / 8], dof[DHP / 8];
  load_rows<DHP, EXACT>(w.q + (size_t)ic * w.ld, a.dh, g, qf);
  load_rows<DHP, EXACT>(a.dctx + head_row, a.dh, g, dof);
  float dd = 0.f;
  {
    f32x4 of[DHP / 8];
    load_rows<DHP, EXACT>(a.ctx + head_row, a.dh, g, of);
#pragma unroll
    for (int c = 0; c < DHP / 8; c++)
#pragma unroll
      for (int e = 0; e < 4; e++) dd = fmaf(dof[c][e], of[c][e], dd);
  }
  dd += __shfl_xor(dd, 32, 64);
  const float lse = a.lse[row];
  if (part == 0 && g == 0 && i < a.S) a.dsum[row] = dd;
  f32x16 dq[DHP / 32];
#pragma unroll
  for (int dt = 0; dt < DHP / 32; dt++) dq[dt] = zero16();
  for (int t = part; t <= w.tile; t += PARTS) {
    const int j0 = 32 * t;
    f32x16 s, dp;
    {
      f32x4 kf[DHP / 8];
      load_rows<DHP, EXACT>(w.k + (size_t)min(j0 + l32, a.S - 1) * w.ld, a.dh, g, kf);
      s = row_product<DHP>(kf, qf);                              // S^T[j][i]
      if (DHP > 64) __builtin_amdgcn_sched_barrier(0);           // one operand in registers at a time
      load_rows<DHP, EXACT>(w.v + (size_t)min(j0 + l32, a.S - 1) * w.ld, a.dh, g, kf);
      dp = row_product<DHP>(kf, dof);                            // dP^T[j][i]
    }
    if (a.rowbits) {
      const unsigned bits = a.rowbits[row * a.wpr + t];
#pragma unroll
      for (int v = 0; v < 16; v++) dp[v] *= ((bits >> acc_row(v, g)) & 1u) ? a.keep_scale : 0.f;
    }
#pragma unroll
    for (int v = 0; v < 16; v++) s[v] = (j0 + acc_row(v, g) <= i) ? expf(s[v] * scale - lse) * (dp[v] - dd) : 0.f;
    if (DHP > 64) __builtin_amdgcn_sched_barrier(0);
    col_product<DHP, EXACT, true>(dq, s, w.k + (size_t)j0 * w.ld, w.ld, a.S - j0, a.dh, t == w.tile, lds + part * 32 * 33,
                           lane);
  }
  merge_parts(dq, lds, part, lane);
  if (part == 0 && i < a.S)
    store_column<DHP, EXACT>(dq, a.out + ((size_t)w.b * a.S + i) * w.ld + w.h * a.dh, scale, a.dh, g);
}

// dV_j = sum_{i >= j} P_ij dO_i, dK_j = scale sum_{i >= j} dS_ij Q_i
// OWN_D: D is formed here once more, from the rows of dO that are in registers and those of O, in the order of the dQ
// kernel; else it is what that kernel has left.
template <int DHP, bool EXACT, bool OWN_D>
GX_DEVINL void dkv_block(const Args& a, int blk, float* lds) {
  const int lane = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  const Where w(a, blk, false);
  const int j0 = 32 * w.tile, j = j0 + l32, jc = min(j, a.S - 1);
  const float scale = rsqrtf((float)a.dh);
  const size_t pair_row = ((size_t)w.b * a.nl + w.h) * a.S;
  const int Hl = a.nl * a.dh;
  const float* dob = a.dctx + (size_t)w.b * a.S * Hl + w.h * a.dh;
  const float* ob = a.ctx + (size_t)w.b * a.S * Hl + w.h * a.dh;
  f32x4 kf[DHP / 8], vf[DHP / 8];
  load_rows<DHP, EXACT>(w.k + (size_t)jc * w.ld, a.dh, g, kf);
  load_rows<DHP, EXACT>(w.v + (size_t)jc * w.ld, a.dh, g, vf);
  f32x16 dk[DHP / 32], dv[DHP / 32];
#pragma unroll
  for (int dt = 0; dt < DHP / 32; dt++) dk[dt] = dv[dt] = zero16();
  const int nt = (a.S + 31) / 32;
  for (int t = w.tile + part; t < nt; t += PARTS) {
    const int i0 = 32 * t, ir = min(i0 + l32, a.S - 1);
    f32x16 p, ds;
    float dd = 0.f;                        // OWN_D: D of row i0 + l32
    {
      f32x4 xf[DHP / 8];
      load_rows<DHP, EXACT>(w.q + (size_t)ir * w.ld, a.dh, g, xf);
      p = row_product<DHP>(xf, kf);                              // S[i][j]
      if (DHP > 64) __builtin_amdgcn_sched_barrier(0);           // one operand in registers at a time
      load_rows<DHP, EXACT>(dob + (size_t)ir * Hl, a.dh, g, xf);
      ds = row_product<DHP>(xf, vf);                             // dP[i][j]
      if (OWN_D) {
        f32x4 of[DHP / 8];
        load_rows<DHP, EXACT>(ob + (size_t)ir * Hl, a.dh, g, of);
#pragma unroll
        for (int c = 0; c < DHP / 8; c++)
#pragma unroll
          for (int e = 0; e < 4; e++) dd = fmaf(xf[c][e], of[c][e], dd);
        dd += __shfl_xor(dd, 32, 64);
      }
    }
    float st[16];
    load_row_stats(a.lse + pair_row + i0, a.S - i0, g, st);
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int i = i0 + acc_row(v, g);
      p[v] = (i >= j && i < a.S) ? expf(p[v] * scale - st[v]) : 0.f;
    }
    unsigned kept = 0xffffu;
    if (a.rowbits) {
      kept = 0;
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const size_t r = pair_row + min(i0 + acc_row(v, g), a.S - 1);
        kept |= ((a.rowbits[r * a.wpr + w.tile] >> l32) & 1u) << v;
        ds[v] = ((kept >> v) & 1u) ? ds[v] * a.keep_scale : 0.f;
      }
    }
    if (OWN_D) {
#pragma unroll
      for (int v = 0; v < 16; v++) st[v] = __shfl(dd, acc_row(v, g), 64);
    } else {
      load_row_stats(a.dsum + pair_row + i0, a.S - i0, g, st);
    }
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int i = i0 + acc_row(v, g);
      ds[v] = (i >= j && i < a.S) ? p[v] * (ds[v] - st[v]) : 0.f;
    }
    if (a.rowbits)
#pragma unroll
      for (int v = 0; v < 16; v++) p[v] = ((kept >> v) & 1u) ? p[v] * a.keep_scale : 0.f;
    const bool diagonal = t == w.tile;
    if (DHP >= 64) __builtin_amdgcn_sched_barrier(0);
    col_product<DHP, EXACT, false>(dv, p, dob + (size_t)i0 * Hl, Hl, a.S - i0, a.dh, diagonal, lds + part * 32 * 33, lane);
    if (DHP > 64) __builtin_amdgcn_sched_barrier(0);
    col_product<DHP, EXACT, false>(dk, ds, w.q + (size_t)i0 * w.ld, w.ld, a.S - i0, a.dh, diagonal, lds + part * 32 * 33,
                            lane);
  }
  merge_parts(dk, lds, part, lane);
  merge_parts(dv, lds, part, lane);
  if (part != 0 || j >= a.S) return;
  float* dst = a.out + ((size_t)w.b * a.S + j) * w.ld + Hl + w.h * a.dh;
  store_column<DHP, EXACT>(dk, dst, scale, a.dh, g);
  store_column<DHP, EXACT>(dv, dst + Hl, 1.0f, a.dh, g);
}

template <int DHP, bool EXACT>
__global__ void __launch_bounds__(64 * PARTS, DHP <= 64 ? 2 : 1) attn_bwd_dq_f32_kernel(Args a) {
  __shared__ float lds[lds_floats<DHP>()];
  dq_block<DHP, EXACT>(a, blockIdx.x, lds);
}
template <int DHP, bool EXACT>
__global__ void __launch_bounds__(64 * PARTS, 1) attn_bwd_dkv_f32_kernel(Args a) {
  __shared__ float lds[lds_floats<DHP>()];
  dkv_block<DHP, EXACT, false>(a, blockIdx.x, lds);
}
// Both in one launch, first the blocks of dK / dV, which have more to do (dQ's store D here too, which nobody reads).
template <int DHP, bool EXACT>
__global__ void __launch_bounds__(64 * PARTS, 1) attn_bwd_f32_kernel(Args a) {
  __shared__ float lds[lds_floats<DHP>()];
  const int blk = blockIdx.x, n = gridDim.x / 2;
  if (blk < n) dkv_block<DHP, EXACT, true>(a, blk, lds);
  else dq_block<DHP, EXACT>(a, blk - n, lds);
}

bool shape_ok(const AttnArgs& a) {
  return a.S > 0 && a.S <= 8192 && a.dh > 0 && a.dh <= 128 && a.nl > 0 && a.B > 0 &&
         (long)a.B * a.nl * cdiv(a.S, 32) < (1L << 31) && (!a.rowbits || a.wpr >= cdiv(a.S, 32));
}

// Whether dQ and dK / dV share a launch: where their blocks find places at the same time, so that neither waits for the
// other's longest.  One workgroup per compute unit (two at head dim 32, which takes fewer registers); many pairs of short
// sequences fill the chip with each kernel alone, and forming D twice then costs more than it saves.  Layers forward and
// backward, us, two launches / one (blocks of 32 rows, pairs):
//   256 x 4 heads of 64, 2 x 128 tokens (32, 8) 107 / 98    512 x 8 of 64, 512 tokens (128, 8) 252 / 228
//   128 x 2 of 64, 1024 tokens (64, 2) 224 / 185            200 x 4 of 50, 900 tokens (116, 4) 322 / 273
//   768 x 6 of 128, 1024 tokens (192, 6) 720 / 693          640 x 10 of 64, 512 tokens (160, 10) 341 / 335
//   512 x 8 of 64, 1024 tokens (256, 8) 403 / 390           512 x 8 of 64, 4 x 256 tokens (256, 32) 329 / 334
//   256 x 8 of 32, 2 x 512 tokens (256, 16) 179 / 166       256 x 8 of 32, 4 x 256 tokens (256, 32) 159 / 163
//   512 x 16 of 32, 1024 tokens (512, 16) 384 / 382         1024 x 16 of 64, 2 x 512 tokens (512, 32) 782 / 802
// Up to 128 blocks also with many pairs; the attention kernels alone: 32 x 4 heads of 32, S 32 (128 pairs) 17.1 / 10.2; 16 x 8 of
// 64, S 32 25 / 13.7; 8 x 16 of 128, S 32 49 / 31; 4 x 16 of 64, S 64 25 / 13.9; 8 x 4 of 128, S 128 (32 pairs) 51 / 36; 8 x 4 of
// 64, S 128 26 / 15.7.
bool one_launch(int B, int S, int nl, int dh) {
  const long pairs = (long)B * nl, blocks = pairs * cdiv(S, 32);
  return blocks <= 128 || (pairs <= 16 && blocks <= (dh <= 32 ? 512 : 256));
}

Args make_args(const AttnArgs& a, float* out) {
  return Args{(const float*)a.qkv, (const float*)a.ctx, (const float*)a.dctx, out, a.lse, a.dsum, a.S, a.nl, a.dh,
              a.nl * a.B, a.rowbits, a.wpr, a.keep_scale};
}

// Head dimensions of exactly 32, 64 or 128 read rows 16 B at a time; every other one takes the next
// larger of the three, padded.
#define GX_F32_ATTN(KERNEL, ARGS, TIMES)                                                           \
  do {                                                                                             \
    const dim3 grid((unsigned)((TIMES) * (ARGS).npair * cdiv((ARGS).S, 32))), block(64 * PARTS);    \
    switch ((ARGS).dh) {                                                                           \
      case 32: hipLaunchKernelGGL((KERNEL<32, true>), grid, block, 0, s, (ARGS)); break;            \
      case 64: hipLaunchKernelGGL((KERNEL<64, true>), grid, block, 0, s, (ARGS)); break;            \
      case 128: hipLaunchKernelGGL((KERNEL<128, true>), grid, block, 0, s, (ARGS)); break;          \
      default:                                                                                     \
        if ((ARGS).dh < 32) hipLaunchKernelGGL((KERNEL<32, false>), grid, block, 0, s, (ARGS));     \
        else if ((ARGS).dh < 64) hipLaunchKernelGGL((KERNEL<64, false>), grid, block, 0, s, (ARGS)); \
        else hipLaunchKernelGGL((KERNEL<128, false>), grid, block, 0, s, (ARGS));                   \
    }                                                                                              \
  } while (0)

}  // namespace

extern "C" int gx_attn_f32_one_launch(int B, int S, int nl, int dh) { return one_launch(B, S, nl, dh); }

hipError_t attn_fwd_f32(const AttnArgs& a, hipStream_t s) {
  if (!shape_ok(a)) return hipErrorInvalidValue;
  const Args f = make_args(a, (float*)a.ctx);
  GX_F32_ATTN(attn_fwd_f32_kernel, f, 1);
  return hipGetLastError();
}

hipError_t attn_bwd_f32(const AttnArgs& a, hipStream_t s) {
  if (!shape_ok(a)) return hipErrorInvalidValue;
  const Args f = make_args(a, (float*)a.dqkv);
  if (one_launch(a.B, a.S, a.nl, a.dh)) {
    GX_F32_ATTN(attn_bwd_f32_kernel, f, 2);
    return hipGetLastError();
  }
  GX_F32_ATTN(attn_bwd_dq_f32_kernel, f, 1);      // also leaves D for the next kernel
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  GX_F32_ATTN(attn_bwd_dkv_f32_kernel, f, 1);
  return hipGetLastError();
}

}  // namespace gx
