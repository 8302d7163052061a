// Body of the bf16 attention kernels for one head dimension.  Included by attn_bf16.hip once per
// supported head dimension, inside a namespace of its own, with GX_ATTN_DH defined.
constexpr int DH = GX_ATTN_DH;         // head dimension of this instantiation (128 or 64)
constexpr int ROWB = DH * 2;           // bytes per tile row
constexpr int CPR = DH / 8;            // 16 B chunks per tile row
static_assert(DH == 128 || DH == 64, "tile swizzles are worked out for these two row lengths");

// 16 B chunk c of tile row r lives at chunk c ^ swz(r), chosen so that both access patterns of a
// tile are free of bank conflicts: ds_read_b128 of 16 consecutive rows at one logical chunk, and
// the transposing read of 4 consecutive rows x 64 B.
//   256 B rows: the low row bits move whole 64 B groups (the 4 rows of a transposing read fall in
//   distinct banks); the next two bits permute inside a group.
//   128 B rows: two rows share a 256 B bank window, so the swizzle depends on r / 2: its low bit
//   flips the 64 B group (rows r and r + 2 of a transposing read), the rest permutes inside it;
//   it is a bijection of (r / 2) % 8 onto the 8 chunks, which keeps 16 consecutive rows distinct.
GX_DEVINL int swz(int r) {
  if (DH == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  const int x = (r >> 1) & 7;
  return ((x & 1) << 2) | (x >> 1);
}

// Direct-to-LDS loads of tiles of ROWS x DH, column blocks of one sample's rows: the buffer ends with the sample's last
// row, so that rows beyond it read as zeros without a comparison, and the column block goes into the instruction's scalar
// offset.  Instruction i of this wave's share of the tile that starts at byte row0_bytes = first row * row bytes.
template <int ROWS, int NW>
struct RowStream {
  static constexpr int RPI = 64 / CPR, PER_WAVE = ROWS / RPI / NW;
  static_assert(PER_WAVE >= 1, "tile too small for the workgroup");
  unsigned voff[PER_WAVE];
  GX_DEVINL void init(int ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < PER_WAVE; i++) {
      const int r = RPI * (wave * PER_WAVE + i) + lane / CPR;
      const int c = (lane % CPR) ^ swz(r);
      voff[i] = (unsigned)(r * ld + c * 8) * 2u;
    }
  }
  GX_DEVINL void issue(__amdgpu_buffer_rsrc_t rsrc, unsigned row0_bytes, int col_bytes, char* dst, int wave, int i) const {
    const unsigned off = voff[i] + row0_bytes;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + (wave * PER_WAVE + i) * 1024), 16, off,
                                             col_bytes, 0, 0);
  }
  GX_DEVINL void load(__amdgpu_buffer_rsrc_t rsrc, unsigned row0_bytes, int col_bytes, char* dst, int wave) const {
#pragma unroll
    for (int i = 0; i < PER_WAVE; i++) issue(rsrc, row0_bytes, col_bytes, dst, wave, i);
  }
};

// MFMA operand whose 32 rows are tile rows r0..r0+31 and whose reduction index is the head
// dimension (step s covers d = 16 s .. 16 s + 15)
GX_DEVINL bf16x8 frag_rows(const char* tile, int r, int s, int g) {
  const int c = (2 * s + g) ^ swz(r);
  return *reinterpret_cast<const bf16x8*>(tile + r * ROWB + (c << 4));
}
// MFMA operands whose 32 rows are head-dim columns 32 dt .. 32 dt + 31 and whose reduction index
// runs over 16 tile rows starting at a multiple of 16, in the slot order of an accumulator column
// (slot (g, e) <-> row 8 (e / 4) + 4 g + e % 4 of the group), come from transposing reads issued
// as untracked asm (see lds_read_tr_issue): the four
// head-dim blocks of the 16 tile rows starting at 16 * GI, from per-lane addresses prepared by
// cols_lane_offsets() plus the tile's LDS address.  The caller waits (lds_wait_le) and pins.
GX_DEVINL void cols_lane_offsets(int lane, unsigned (&off)[2][DH / 32]) {
  const int g = lane >> 5, s = lane & 15, hb = (lane >> 4) & 1;
#pragma unroll
  for (int half = 0; half < 2; half++) {
    const int r = 4 * g + (s >> 2) + 8 * half;       // swz(16 k + r) == swz(r)
#pragma unroll
    for (int dt = 0; dt < DH / 32; dt++) {
      const int d0 = 32 * dt + 16 * hb + 4 * (s & 3);
      off[half][dt] = (unsigned)(r * ROWB + (((d0 >> 3) ^ swz(r)) << 4) + (d0 & 7) * 2);
    }
  }
}
struct ColFrags {
  bf16x4 lo[DH / 32], hi[DH / 32];
};
template <int GI>
GX_DEVINL void cols_issue(unsigned tile, const unsigned (&off)[2][DH / 32], ColFrags& f) {
#pragma unroll
  for (int dt = 0; dt < DH / 32; dt++) {
    f.lo[dt] = lds_read_tr_issue<GI * 16 * ROWB>(tile + off[0][dt]);
    f.hi[dt] = lds_read_tr_issue<GI * 16 * ROWB>(tile + off[1][dt]);
  }
}
GX_DEVINL bf16x8 cols_get(ColFrags& f, int dt) {
  lds_pin(f.lo[dt]);
  lds_pin(f.hi[dt]);
  return __builtin_shufflevector(f.lo[dt], f.hi[dt], 0, 1, 2, 3, 4, 5, 6, 7);
}

// registers v = 8 h .. 8 h + 7 of an accumulator, rounded to bf16, as an MFMA operand
GX_DEVINL bf16x8 pack_half(const f32x16& a, int h) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; e++) o[e] = (bf16)a[8 * h + e];
  return o;
}

GX_DEVINL f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int v = 0; v < 16; v++) z[v] = 0.f;
  return z;
}

template <class F, int... I>
GX_DEVINL void unroll_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
// f(0) .. f(N - 1) with the index as a constant
template <int N, class F>
GX_DEVINL void unroll(F&& f) {
  unroll_seq(f, std::make_integer_sequence<int, N>());
}

// N products whose LDS fragments are requested DEPTH products ahead: read(i) returns fragment i, mul(i, f)
// issues product i.  Left to itself the compiler asks for a fragment one product ahead.
template <int N, int DEPTH, class Read, class Mul>
GX_DEVINL void streamed(Read read, Mul mul) {
  bf16x8 f[DEPTH];
#pragma unroll
  for (int i = 0; i < DEPTH && i < N; i++) f[i] = read(i);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < N; i++) {
    mul(i, f[i % DEPTH]);
    __builtin_amdgcn_sched_barrier(0);
    if (i + DEPTH < N) f[i % DEPTH] = read(i + DEPTH);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// this lane's 8 steps of a 32-row operand read straight from global memory (row clamped)
GX_DEVINL void load_row_frags(const bf16* base, int ld, int row, int nrows, int g, bf16x8 (&out)[DH / 16]) {
  const bf16* p = base + (size_t)min(row, nrows - 1) * ld + 8 * g;
#pragma unroll
  for (int s = 0; s < DH / 16; s++) out[s] = *reinterpret_cast<const bf16x8*>(p + 16 * s);
}


// acc[dt] += product of the transposed fragments of a tile of 16 * NG16 rows (groups of 16 rows at LDS address `ct`)
// with xf[group]; rows of the result are head-dim columns.  Groups 0 and 1 must have been issued into cf[0], cf[1] by the
// caller (as early as it likes, to cover LDS latency with its own work); with four groups, groups 2 and 3
// are issued here, so that two groups are always in flight.
template <int NG16>
GX_DEVINL void tr_product(f32x16 (&acc)[DH / 32], unsigned ct, const unsigned (&coff)[2][DH / 32],
                          ColFrags (&cf)[2], const bf16x8 (&xf)[NG16]) {
  static_assert(NG16 == 2 || NG16 == 4, "tiles of 32 or 64 rows");
#define GX_TR_GROUP(U, BUF) \
  _Pragma("unroll") for (int dt = 0; dt < DH / 32; dt++) acc[dt] = MFMA(cols_get(cf[BUF], dt), xf[U], acc[dt])
  lds_wait_le<2 * (DH / 32)>();
  GX_TR_GROUP(0, 0);
  if (NG16 == 4) {
    cols_issue<2>(ct, coff, cf[0]);
    lds_wait_le<2 * (DH / 32)>();
    GX_TR_GROUP(1, 1);
    cols_issue<3>(ct, coff, cf[1]);
    lds_wait_le<2 * (DH / 32)>();
    GX_TR_GROUP(NG16 - 2, 0);
    lds_wait_all();
    GX_TR_GROUP(NG16 - 1, 1);
  } else {
    lds_wait_all();
    GX_TR_GROUP(1, 1);
  }
#undef GX_TR_GROUP
}
// ------------------------------------------------------------------------------- forward
// A workgroup owns 32 NQ query rows of one (sample, head); its NQ * SPLIT wavefronts are NQ blocks
// of 32 rows times SPLIT shares of the keys: every step brings SPLIT tiles of BKV keys (K and V)
// into LDS and wavefront (q, part) works on tile `part`; the SPLIT partial softmax states
// (max, sum, O) of a row block are merged through LDS at the end, in the order of `part`.
//   many (sample, head) pairs : NQ 4, SPLIT 1, BKV 64 (4 wavefronts, two workgroups per compute unit)
//   few pairs                 : NQ 2, SPLIT 2, BKV 32 (the same), or NQ 2, SPLIT 4, BKV 32 (8 wavefronts, one workgroup
//     per unit: see keys_over_four()): the causal triangle gives query blocks between 1 and S / 32 NQ
//     units of work, so with few pairs the chip is filled by short blocks cut fine, each with its keys spread
//     over two or four wavefronts.
// Workgroups are numbered longest query block first over the whole launch (all pairs' last blocks, then all pairs'
// next-to-last blocks, ...): the hardware hands them out in that order.  With SPLIT 2 the second half of the
// launch runs shortest first: with two workgroups per compute unit and a launch of twice the number of units,
// workgroups x and x + gridDim.x / 2 tend to share a unit, and their work then adds up to the same total.
// Dropout of the probabilities: keep bits (1 = kept) of the whole launch, `wpr` 32-bit words per
// row; row-major (a query's keys) for the forward and dQ kernels, column-major (a key's queries)
// for the dK / dV kernel.  Kept probabilities are multiplied by `scale`.
struct KeepArgs {
  const unsigned* bits;
  int wpr;
  float scale;
};
// The keep bits of a lane's NJT 32 x 32 accumulator tiles: zero the values whose bit is clear.
// Accumulator register v of tile jt sits at bit 32 jt + 8 (v / 4) + 4 g + v % 4.
template <int NJT>
GX_DEVINL void drop_unkept(f32x16 (&a)[NJT], unsigned long long kw, int g) {
#pragma unroll
  for (int jt = 0; jt < NJT; jt++) {
    const unsigned w = (unsigned)(kw >> (32 * jt)) >> (4 * g);
#pragma unroll
    for (int v = 0; v < 16; v++)
      if (!((w >> (8 * (v >> 2) + (v & 3))) & 1u)) a[jt][v] = 0.f;
  }
}
// registers 8 h .. 8 h + 7 of one tile, w = its word shifted down by 4 g
GX_DEVINL void drop_unkept_half(f32x16& a, unsigned w, int h) {
#pragma unroll
  for (int v = 8 * h; v < 8 * h + 8; v++)
    if (!((w >> (8 * (v >> 2) + (v & 3))) & 1u)) a[v] = 0.f;
}
// this lane's keep bits of the BKV keys starting at key j0 of one query row (bits: the row's words)
template <int NJT>
GX_DEVINL unsigned long long keep_bits_of_step(const unsigned* row_words, int j0) {
  if (NJT == 2) return *reinterpret_cast<const unsigned long long*>(row_words + (j0 >> 5));
  return row_words[j0 >> 5];
}

// End of a forward workgroup: merge the SPLIT partial softmax states of each row block through LDS
// (the tiles are no longer needed), then normalise and store the block's rows of ctx and lse.
constexpr int FWD_REGION = (4 + DH / 2) * 64;          // a wavefront's parked state, in floats
// LDS: two buffers for K and two for V, or what the merge parks
constexpr int fwd_smem(int nq, int split, int bkv) {
  const int tiles = 4 * bkv * split * ROWB, parked = split > 1 ? nq * split * FWD_REGION * 4 : 0;
  return tiles > parked ? tiles : parked;
}
template <int NQ, int SPLIT, bool DROP>
GX_DEVINL void fwd_merge_store(char* smem, f32x16 (&o)[DH / 32], float m, float lsum, int part, int qs, int lane,
                               int iw, int b, int h, int S, int nl, bf16* __restrict__ ctx,
                               float* __restrict__ lse, const KeepArgs& keep) {
  constexpr int NDT = DH / 32, OWN = NDT / SPLIT > 0 ? NDT / SPLIT : 1, OWNERS = NDT / OWN;
  const int g = lane >> 5, l32 = lane & 31;
  const int Hl = nl * DH;
  lsum += __shfl_xor(lsum, 32, 64);
  // Part p finishes the head-dim blocks p * OWN ..: every part parks its maximum, sum and blocks in LDS (the tiles
  // are no longer needed) as [row block][part][2 values, then blocks of 16 values][64 lanes], 16 B per lane and write.
  // A part that saw no key has m = -inf, l = 0, O = 0 and counts for nothing (part 0 always saw key 0).
  if constexpr (SPLIT > 1) {
    constexpr int REGION = FWD_REGION;
    float* mine = reinterpret_cast<float*>(smem) + (qs * SPLIT + part) * REGION;
    *reinterpret_cast<f32x2*>(mine + lane * 4) = f32x2{m, lsum};
#pragma unroll
    for (int dt = 0; dt < NDT; dt++)
#pragma unroll
      for (int q = 0; q < 4; q++)
        if (dt / OWN != part)
          *reinterpret_cast<f32x4*>(mine + 256 + ((dt * 4 + q) * 64 + lane) * 4) =
              f32x4{o[dt][4 * q], o[dt][4 * q + 1], o[dt][4 * q + 2], o[dt][4 * q + 3]};
    __syncthreads();
    if (part >= OWNERS) return;
    const float* all = reinterpret_cast<const float*>(smem) + qs * SPLIT * REGION;
    float mp[SPLIT], lp[SPLIT], mm = -INFINITY;
#pragma unroll
    for (int p = 0; p < SPLIT; p++) {
      const f32x2 v = *reinterpret_cast<const f32x2*>(all + p * REGION + lane * 4);
      mp[p] = v[0];
      lp[p] = v[1];
      mm = fmaxf(mm, mp[p]);
    }
    lsum = 0.f;
#pragma unroll
    for (int p = 0; p < SPLIT; p++) {
      mp[p] = __builtin_amdgcn_exp2f(mp[p] - mm);
      lsum += lp[p] * mp[p];
    }
    m = mm;
    f32x16 t[OWN];
#pragma unroll
    for (int k = 0; k < OWN; k++) {
      t[k] = zero16();
#pragma unroll
      for (int p = 0; p < SPLIT; p++) {
        // this part's own share comes from its registers
        f32x16 x;
        if (p == part) {
#pragma unroll
          for (int dt = 0; dt < NDT; dt++)
            if (dt == part * OWN + k) x = o[dt];
        } else {
#pragma unroll
          for (int q = 0; q < 4; q++) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(all + p * REGION + 256 +
                                                            (((part * OWN + k) * 4 + q) * 64 + lane) * 4);
#pragma unroll
            for (int e = 0; e < 4; e++) x[4 * q + e] = v[e];
          }
        }
#pragma unroll
        for (int v = 0; v < 16; v++) t[k][v] += x[v] * mp[p];
      }
    }
#pragma unroll
    for (int k = 0; k < OWN; k++) o[k] = t[k];
  }
  const int i = iw + l32;
  if (i < S) {
    const float inv = (DROP ? keep.scale : 1.0f) / lsum;
    bf16* orow = ctx + ((size_t)b * S + i) * Hl + h * DH + 32 * (SPLIT > 1 ? part * OWN : 0);
#pragma unroll
    for (int dt = 0; dt < (SPLIT > 1 ? OWN : NDT); dt++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        bf16x4 pk;
#pragma unroll
        for (int e = 0; e < 4; e++) pk[e] = (bf16)(o[dt][4 * q4 + e] * inv);
        *reinterpret_cast<bf16x4*>(orow + 32 * dt + 8 * q4 + 4 * g) = pk;
      }
    if (g == 0 && part == 0) lse[((size_t)b * nl + h) * S + i] = (m + __builtin_amdgcn_logf(lsum)) * LN2;
  }
}

// What bounds it: 64 scores cost 32 cycles of the matrix pipe (512 FLOP each at DH 128) and about nine issue
// slots of 4 cycles of vector work (an exponential alone takes four), so neither pipe may wait for the other.  The
// wavefronts of a SIMD do not take turns by themselves: they pass the same barrier, then want the same pipe.  So one
// wavefront's stream mixes the two: in step t the products of the step before (O += V P, t - 1) and the
// scores of the next one (S, t + 1) are issued one by one, and behind each goes its share of the softmax of step t, held in
// that order by scheduling barriers and by pinning the results (else the exponentials sink to their use).
// K and V have two buffers each: step t requests K(t + 2) where K(t) was and V(t) where V(t - 2) was, in its first four
// or eight slots (later, the step's end waits for them; all at once, the wavefronts queue for the load unit).
// LAZY: the reference maximum m follows the true one only when some row exceeds it by more than 2^8, so exponentials
// stay below 2^8 and the rescaling of O (as many multiplies as a step's vector work has otherwise) becomes rare; any
// reference gives the same softmax up to rounding, and lse = m + log2(l) holds for any m.  Without it m is the
// running maximum itself, so that a row's largest probability is exactly 1 in bf16, which leaves outputs 0.1 to 1.5 %
// nearer to the fp64 ones (64 pairs of S 2048).
// Measured against one kernel without the mix (many pairs) and one with only the scores ahead (few), in turn
// between the products of a layer, us: 64 pairs of S 2048 105 -> 94, 64 of S 1024 34.4 -> 31.7, 4 of S 8192 109 -> 99.6, 8 of
// S 2048 29.2 -> 24.7, 16 of S 2048 33.4 -> 32.9, 20 of S 2048 38.6 -> 37.0, 20 of S 128 8.0 -> 7.2; DH 64: 64 of S 1024
// 22.6 -> 20.6, 12 of S 1024 12.7 -> 10.9.  Distances from fp64 (2-norm,
// four key shares against two, five calls, two to six seeds each): outputs -0.5 to +0.1 %, gradient matrices -0.5 to +0.1 % from
// S 2048 on and +-1.4 % at 1024 tokens, gradient vectors of some hundred elements +-6 %, without a direction: P is rounded
// to bf16 relative to another maximum.  Deeper rings (80 KB) leave one workgroup per unit: 64 pairs of S 2048 take twice as long.
template <int NQ, int SPLIT, int BKV, bool LAZY, bool DROP>
__global__ void __launch_bounds__(64 * NQ * SPLIT, 2)
    attn_fwd_kernel(const bf16* __restrict__ qkv, bf16* __restrict__ ctx, float* __restrict__ lse, int S, int nl,
                    int npair, KeepArgs keep) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr int NW = NQ * SPLIT, BQ = 32 * NQ, ROWS = BKV * SPLIT, TILE = ROWS * ROWB, NS = DH / 16;
  constexpr int NJT = BKV / 32, NG = 2 * NJT, NDT = DH / 32;
  static_assert((NQ & (NQ - 1)) == 0 && (BKV == 32 || BKV == 64), "shape of the step");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qs = wave % NQ, part = wave / NQ;
  const int g = lane >> 5, l32 = lane & 31;
  const int nq = (S + BQ - 1) / BQ;
  const int pair = blockIdx.x % npair;
  const int rq = blockIdx.x / npair, hq = (nq + 1) / 2;
  const int qt = (SPLIT != 2 || rq < hq) ? nq - 1 - rq : rq - hq;
  const int h = pair % nl, b = pair / nl;
  const int Hl = nl * DH, ld = 3 * Hl;
  const int i0 = qt * BQ, iw = i0 + qs * 32;          // this wave's first query row
  const bf16* sample = qkv + (size_t)b * S * ld;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(sample), 0,
                                                                        (unsigned)(S * ld) * 2u, 0x00020000);
  bf16x8 qf[NS];
  load_row_frags(sample + h * DH, ld, iw + l32, S, g, qf);

  f32x16 o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; dt++) o[dt] = zero16();
  float m = -INFINITY, lsum = 0.f;
  const float c2 = rsqrtf((float)DH) * LOG2E;
  unsigned coff[2][NDT];
  cols_lane_offsets(lane, coff);

  char* const kst = smem;                             // K(t) at kst + (t & 1) * TILE
  char* const vst = smem + 2 * TILE;                  // V(t) at vst + (t & 1) * TILE
  const int jend = min(S, i0 + BQ);                   // keys 0 .. jend-1 can be visible
  const int nt = (jend + ROWS - 1) / ROWS;
  RowStream<ROWS, NW> src;
  constexpr int PER = RowStream<ROWS, NW>::PER_WAVE;
  src.init(ld, wave, lane);
  const int kcol = (Hl + h * DH) * 2, vcol = (2 * Hl + h * DH) * 2;
  const unsigned tile_bytes = (unsigned)(ROWS * ld) * 2u, none = (unsigned)(S * ld) * 2u;   // none: nothing but zeros
  src.load(rsrc, 0, kcol, kst, wave);
  src.load(rsrc, 0, vcol, vst, wave);
  src.load(rsrc, nt > 1 ? tile_bytes : none, kcol, kst + TILE, wave);
  const unsigned* kwords = DROP ? keep.bits + (((size_t)b * nl + h) * S + min(iw + l32, S - 1)) * keep.wpr : nullptr;
  auto keep_of = [&](int t) -> unsigned long long {
    const int j = t * ROWS + part * BKV;
    return j <= iw + 31 && j < S ? keep_bits_of_step<NJT>(kwords, j) : 0ull;
  };
  unsigned long long kw = 0, kw_next = 0;
  if (DROP) kw_next = keep_of(0);
  WAIT_VM0();
  __syncthreads();
  f32x16 s_even[NJT], s_odd[NJT];                     // scores of an even and an odd step
#pragma unroll
  for (int jt = 0; jt < NJT; jt++) s_even[jt] = zero16();
  if (part * BKV <= iw + 31) {
    const char* k0 = kst + part * BKV * ROWB;
    streamed<NJT * NS, 4>([&](int q) { return frag_rows(k0, 32 * (q / NS) + l32, q % NS, g); },
                          [&](int q, bf16x8 f) { s_even[q / NS] = MFMA(f, qf[q % NS], s_even[q / NS]); });
  }
  __syncthreads();                                    // K(2) goes into the buffer of K(0)
  bf16x8 pf[NG];                                      // P of the step before, 16 keys per entry
  struct VFrag { bf16x4 lo, hi; };
  auto v_request = [&](unsigned vt, auto P, VFrag& f) __attribute__((always_inline)) {
    constexpr int p = decltype(P)::value, dt = p / NG, u = p % NG;
    f.lo = lds_read_tr_issue<u * 16 * ROWB>(vt + coff[0][dt]);
    f.hi = lds_read_tr_issue<u * 16 * ROWB>(vt + coff[1][dt]);
  };
  auto v_get = [&](VFrag& f) __attribute__((always_inline)) {
    lds_pin(f.lo);
    lds_pin(f.hi);
    return __builtin_shufflevector(f.lo, f.hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  constexpr int NPV = NG * NDT, NSC = NJT * NS, VD = 4 < NPV ? 4 : NPV, KD = 4 < NSC ? 4 : NSC;
  auto flush = [&](unsigned vt) __attribute__((always_inline)) {       // O^T += V^T P^T of the step before, on its own
    VFrag vf[VD];
    unroll<VD>([&](auto P) __attribute__((always_inline)) { v_request(vt, P, vf[P]); });
    unroll<NPV>([&](auto P) __attribute__((always_inline)) {
      constexpr int p = decltype(P)::value, newer = 2 * ((p + VD < NPV ? p + VD : NPV) - p - 1);
      lds_wait_le<newer>();
      o[p / NG] = MFMA(v_get(vf[p % VD]), pf[p % NG], o[p / NG]);
      if constexpr (p + VD < NPV) v_request(vt, std::integral_constant<int, p + VD>(), vf[p % VD]);
    });
  };
  // this wave's steps with a visible key are 0 .. tv - 1 (wave-uniform)
  const int ahead = iw + 31 - part * BKV, tv = ahead < 0 ? 0 : min(nt, ahead / ROWS + 1);
  // request i of a step: first its share of K(t + 2), then of V(t)
  auto request = [&](int t, int i) __attribute__((always_inline)) {
    if (i < PER) src.issue(rsrc, t + 2 < nt ? (unsigned)(t + 2) * tile_bytes : none, kcol, kst + (t & 1) * TILE, wave, i);
    else src.issue(rsrc, (unsigned)t * tile_bytes, vcol, vst + (t & 1) * TILE, wave, i - PER);
  };
  auto meet = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  auto step = [&](int t, f32x16 (&sacc)[NJT], f32x16 (&snxt)[NJT], auto first_tag) __attribute__((always_inline)) {
    constexpr bool FIRST = decltype(first_tag)::value;
    if (DROP) {
      kw = kw_next;
      kw_next = keep_of(t + 1);
    }
    const int j0 = t * ROWS + part * BKV;              // this wave's keys of the step
    const unsigned vt = lds_addr(vst + ((t - 1) & 1) * TILE + part * BKV * ROWB);
    {
      const char* kn = kst + ((t + 1) & 1) * TILE + part * BKV * ROWB;
      constexpr int NP = FIRST ? 0 : NPV, NM = NP + NSC, RS = NM / 4;
      constexpr int NREQ = FIRST ? PER : 2 * PER;      // V(0) came with K(0)
      VFrag vf[VD];
      bf16x8 kf[KD];
      if constexpr (!FIRST) unroll<VD>([&](auto P) __attribute__((always_inline)) { v_request(vt, P, vf[P]); });
      if constexpr (FIRST) {
#pragma unroll
        for (int q = 0; q < KD; q++) kf[q] = frag_rows(kn, 32 * (q / NS) + l32, q % NS, g);
      }
#pragma unroll
      for (int jt = 0; jt < NJT; jt++) snxt[jt] = zero16();
      const int i = iw + l32;
      float psum = 0.f, alpha = 1.f;
      bool moved = false;
      // the softmax of step t for query column i (base-2 exponentials, scale folded into the exponent's multiply-add)
      // in pieces: 0 mask, 1 reference, then EPP scores each, a head-dim block of O to rescale each, 16 keys to round each
      // SPREAD: the keep bits of each 16 keys where these are rounded, not all at once.  At head dim 64 that also takes 166
      // registers instead of 173, three wavefronts per SIMD instead of two (128 pairs of S 2048 118 -> 111 us); at 128
      // it is slower (64 pairs of S 2048 98.0, 99.7).
      constexpr bool SPREAD = DROP && DH == 64;
      constexpr int EPP = 2;
      constexpr int NE = 16 * NJT / EPP, P_E = 2, P_R = P_E + NE, P_P = P_R + NDT, NPIECE = P_P + NG;
      auto piece = [&](auto K) __attribute__((always_inline)) {
        constexpr int k = decltype(K)::value;
        if constexpr (k == 0) {
          if (j0 + BKV - 1 > iw) {                     // the tile touches the diagonal
#pragma unroll
            for (int jt = 0; jt < NJT; jt++)
#pragma unroll
              for (int v = 0; v < 16; v++)
                if (j0 + 32 * jt + 8 * (v >> 2) + 4 * g + (v & 3) > i) sacc[jt][v] = -INFINITY;
          }
        } else if constexpr (k == 1) {
          float mloc = sacc[0][0];
#pragma unroll
          for (int jt = 0; jt < NJT; jt++)
#pragma unroll
            for (int v = 0; v < 16; v++) mloc = fmaxf(mloc, sacc[jt][v]);
          mloc = max_across_halves(mloc) * c2;
          float mnew = fmaxf(m, mloc);
          if (LAZY) {
            moved = __builtin_amdgcn_ballot_w64(mloc > m + 8.f) != 0;
            mnew = moved ? mnew : m;
          }
          alpha = __builtin_amdgcn_exp2f(m - mnew);
          m = mnew;
          lsum *= alpha;
          asm volatile("" : "+v"(m), "+v"(alpha));
        } else if constexpr (k < P_R) {
          constexpr int e = EPP * (k - P_E), jt = e / 16, v0 = e % 16;
#pragma unroll
          for (int v = v0; v < v0 + EPP; v++) {
            const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[jt][v], c2, -m));
            sacc[jt][v] = p;
            psum += p;
          }
          asm volatile("" : "+v"(psum));
        } else if constexpr (k < P_P) {
          constexpr int dt = k - P_R;
          if constexpr (!LAZY && !FIRST) {
#pragma unroll
            for (int v = 0; v < 16; v++) o[dt][v] *= alpha;
            asm volatile("" : "+v"(o[dt]));
          } else if constexpr (LAZY && !FIRST && dt == 0) {
            if (moved) {
#pragma unroll
              for (int d = 0; d < NDT; d++)
#pragma unroll
                for (int v = 0; v < 16; v++) o[d][v] *= alpha;
            }
          }
        } else {
          constexpr int u = k - P_P;
          if (DROP && u == 0) lsum += psum;            // the undropped sum
          if constexpr (SPREAD) drop_unkept_half(sacc[u >> 1], (unsigned)(kw >> (32 * (u >> 1))) >> (4 * g), u & 1);
          else if (DROP && u == 0) drop_unkept<NJT>(sacc, kw, g);
          pf[u] = pack_half(sacc[u >> 1], u & 1);
        }
      };
      // cost of the pieces in issue slots, for spreading them over the matrix instructions
      constexpr auto cost = [](int k) constexpr {
        return k == 0 ? 4 : k == 1 ? 12 + 8 * NJT : k < P_R ? 6 * EPP : k < P_P ? (LAZY ? 1 : 16) : SPREAD ? 20 : 4;
      };
      constexpr auto upto = [cost](int k) constexpr { int c = 0; for (int x = 0; x < k; x++) c += cost(x); return c; };
      constexpr int TOTAL = upto(NPIECE);
      // piece k goes behind matrix instruction slot_of(k); rescaling behind the last product into O
      constexpr auto slot_of = [upto, cost](int k) constexpr {
        int sl = (upto(k) + cost(k) / 2) * NM / TOTAL;
        if (k >= P_R && sl < NP) sl = NP;
        return sl < NM ? sl : NM - 1;
      };
      __builtin_amdgcn_sched_barrier(0);
      piece(std::integral_constant<int, 0>());
      unroll<NM>([&](auto I) __attribute__((always_inline)) {
        constexpr int x = decltype(I)::value;
        if constexpr (x < NP) {
          // untracked reads younger than this product's, and the K fragments requested so far
          constexpr int newer = 2 * ((x + VD < NPV ? x + VD : NPV) - x - 1) + (x > NPV - KD ? x - (NPV - KD) : 0);
          lds_wait_le<newer>();
          o[x / NG] = MFMA(v_get(vf[x % VD]), pf[x % NG], o[x / NG]);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (x + VD < NPV) v_request(vt, std::integral_constant<int, x + VD>(), vf[x % VD]);
          if constexpr (x >= NPV - KD) {
            constexpr int q = x - (NPV - KD);
            kf[q] = frag_rows(kn, 32 * (q / NS) + l32, q % NS, g);
          }
        } else {
          constexpr int q = x - NP;
          snxt[q / NS] = MFMA(kf[q % KD], qf[q % NS], snxt[q / NS]);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (q + KD < NSC) kf[q % KD] = frag_rows(kn, 32 * ((q + KD) / NS) + l32, (q + KD) % NS, g);
        }
#pragma unroll
        for (int i = x * NREQ / RS; i < (x + 1) * NREQ / RS && i < NREQ; i++) request(t, i);
        unroll<NPIECE>([&](auto K) __attribute__((always_inline)) {
          if constexpr (decltype(K)::value > 0 && slot_of(decltype(K)::value) == x) piece(K);
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      if (!DROP) lsum += psum;
      // also where no step follows: the waits above count the reads of these products
#pragma unroll
      for (int jt = 0; jt < NJT; jt++) asm volatile("" : "+v"(snxt[jt]));
    }
    meet();
  };
  int t = 0;
  if (tv > 0) {
    step(0, s_even, s_odd, std::true_type());
    for (t = 1; t + 1 < tv; t += 2) {
      step(t, s_odd, s_even, std::false_type());
      step(t + 1, s_even, s_odd, std::false_type());
    }
    if (t < tv) {
      step(t, s_odd, s_even, std::false_type());
      t++;
    }
    flush(lds_addr(vst + ((t - 1) & 1) * TILE + part * BKV * ROWB));
  }
  for (; t < nt; t++) {                               // what the other wavefronts still need
#pragma unroll
    for (int i = 0; i < 2 * PER; i++)
      if (i < PER || t > 0) request(t, i);
    meet();
  }
  if (SPLIT > 1) __syncthreads();                     // the merge reuses the tile buffers
  fwd_merge_store<NQ, SPLIT, DROP>(smem, o, m, lsum, part, qs, lane, iw, b, h, S, nl, ctx, lse, keep);
}

// ------------------------------------------------------------------------------- backward: dK, dV
// A workgroup owns 64 key rows as 2 blocks of 32; each block belongs to a PAIR of wavefronts that split
// the work by output: wavefront `pair` (role V) forms S = Q K^T, the probabilities P and dV += P^T dO;
// wavefront `pair + 2` (role K) forms dP = dO V^T, then dS = P (dP - D) and dK += dS^T Q.  P crosses
// from one to the other through LDS as bf16, in the accumulator's own lane layout (16 B per lane per
// half sub-tile, conflict-free).  Each wavefront thus keeps one operand (K or V) and one 32 x DH
// accumulator in registers.
//
// What bounds it: a phase (one query tile of 32 rows) written as a chain (LDS reads, products, exponentials,
// exchange, barrier) keeps the matrix pipe busy for a third of its length.  So a wavefront's stream mixes the
// first products of the next tile with the vector work of its own, product by product, as in the forward kernel, and a
// second, independent workgroup on the compute unit (76 KB of LDS at DH 128) fills the rest.  In phase n
//   role V: S(n+1) = Q(n+1) K^T, mixed with P(n) -> LDS; then dV += P(n)^T dO(n)
//   role K: dP(n) = dO(n) V^T, mixed with dS(n-1) from P(n-1) and dP(n-1); then dK += dS(n-1)^T Q(n-1)
// with one barrier per phase; Q(n+3) and dO(n+2) are requested in its first slots.  Tiles need two phases to arrive:
// with one (and the second products a phase later, mixed too, in the same LDS) every phase waited for them.
// This kernel, us, as a chain / as it is, in turn between the products of a layer: 64 pairs of S 2048 198 / 182,
// 16 pairs 62.1 / 56.2, 4 pairs of S 8192 221 / 198, 64 of S 1024 58.2 / 57.6, 20 of S 128 9.4 / 9.8; DH 64: 12 pairs of S 1024
// 22.8 / 19.4, 64 of S 2048 with dropout 125 / 119, 64 of S 1024 with dropout 41.8 / 40.8, without 32.8 / 34.2 (three
// workgroups share a unit instead of four).  In a step of 64 pairs of S 2048, where power holds the clock down, 173 / 171.
// The chain with two workgroups per unit against 128 key rows, query tiles of 64 and one workgroup of 8 wavefronts (the whole
// backward pass, nothing else on the chip, us): 64 pairs of S 2048 at DH 128 394 -> 292, 16 pairs 112 -> 101, 4 pairs of
// S 8192 372 -> 334.
constexpr int KV_PAIRS = 2, KV_NW = 2 * KV_PAIRS, KV_BJ = 32 * KV_PAIRS, KV_BI = 32;
// LDS: Q tiles (+ their D rows) in a ring (tiles n-1 .. n+3), dO tiles (+ lse rows) in a ring (tiles
// n .. n+2), two P exchange buffers, and a 256 B sink (see the requests).
constexpr int KV_PAIRED = 512;                               // launches that are resident all at once
constexpr int KV_NQ = 5, KV_NDO = 3;
constexpr int KV_TILE = KV_BI * ROWB + 256;                  // rows of Q or dO | their D or lse (64 lanes' worth)
constexpr int KV_PX = KV_PAIRS * 2 * 1024;                   // P exchange: [pair][half][lane] x 16 B
constexpr int KV_OFF_DO = KV_NQ * KV_TILE, KV_OFF_PX = KV_OFF_DO + KV_NDO * KV_TILE;
constexpr int KV_OFF_SINK = KV_OFF_PX + 2 * KV_PX, KV_SMEM = KV_OFF_SINK + 256;
static_assert(2 * KV_SMEM <= 160 * 1024, "two workgroups per compute unit");

// What both kernels of the backward pass are given.
struct BwdArgs {
  const bf16 *qkv, *ctx, *dctx;
  const float* lse;
  float* dsum;
  bf16* dqkv;
  int S, nl, npair;
};

// Block `blk` of the launch order.  PAIRED: the second half of the blocks runs those with fewest tiles first.
// OWN_D: D of the rows that see these keys is formed here first, from dO and O, into LDS behind the rings; else it is what the
// dQ kernel has left.
template <bool DROP, bool OWN_D>
GX_DEVINL void dkv_block(const BwdArgs& a, const KeepArgs& keep, int blk, bool paired, char* smem) {
  const bf16* __restrict__ const qkv = a.qkv;
  const bf16* __restrict__ const dctx = a.dctx;
  const float* __restrict__ const lse = a.lse;
  bf16* __restrict__ const dqkv = a.dqkv;
  const int S = a.S, nl = a.nl, npair = a.npair;
  constexpr int NS = DH / 16, NDT = DH / 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool role_v = wave < KV_PAIRS;
  const int pair = wave & (KV_PAIRS - 1);
  const int g = lane >> 5, l32 = lane & 31;
  // Blocks with most query tiles (the first keys) first.  In a launch that is resident all at once, two
  // workgroups per unit, the second half runs those with fewest first, as in the forward kernel (16 pairs
  // of S 2048 2 % faster, 4 pairs of S 8192 4 %; with four times as many workgroups as places plain order is 8 %
  // faster).
  const int kp = blk % npair, rk = blk / npair, nkb = (S + KV_BJ - 1) / KV_BJ, hk = (nkb + 1) / 2;
  const int kb = rk < hk || !paired ? rk : nkb - 1 - (rk - hk);
  const int h = kp % nl, b = kp / nl;
  const int Hl = nl * DH, ld = 3 * Hl;
  const int j0 = kb * KV_BJ, jw = j0 + pair * 32;
  const bf16* sample = qkv + (size_t)b * S * ld;
  const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(sample), 0,
                                                                      (unsigned)(S * ld) * 2u, 0x00020000);
  const __amdgpu_buffer_rsrc_t rdo = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16*>(dctx + (size_t)b * S * Hl), 0, (unsigned)(S * Hl) * 2u, 0x00020000);
  bf16x8 kvf[NS];                           // role V: this block's K rows; role K: its V rows
  load_row_frags(sample + h * DH + (role_v ? Hl : 2 * Hl), ld, jw + l32, S, g, kvf);
  f32x16 acc[NDT];                          // role V: dV; role K: dK
#pragma unroll
  for (int dt = 0; dt < NDT; dt++) acc[dt] = zero16();
  const float scale = rsqrtf((float)DH), c2 = scale * LOG2E;
  const float* lrow = lse + ((size_t)b * nl + h) * S;
  const float* drow = a.dsum + ((size_t)b * nl + h) * S;
  char* const px = smem + KV_OFF_PX + pair * (KV_PX / KV_PAIRS) + lane * 16;
  unsigned coff[2][NDT];
  cols_lane_offsets(lane, coff);

  // query tiles t0 .. nt - 1 see these keys, tiles tp .. nt - 1 those of this pair of wavefronts
  const int t0 = j0 / KV_BI, tp = t0 + pair, nt = (S + KV_BI - 1) / KV_BI;
  // lse and D rows of a query tile go to LDS by the same direct path, 4 B per lane (wavefront 0:
  // lse, wavefront 1: D; the others send an out-of-range load to a sink, so that every wavefront has the same
  // number of loads in flight).  Rows beyond the sequence read as 0
  // everywhere (Q, dO, lse, D): their probabilities are 1 but their contributions to dV and dK
  // are exactly 0, and whole tiles beyond the sequence may be requested harmlessly.
  const __amdgpu_buffer_rsrc_t raux = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(wave == 0 ? lrow : drow), 0, (unsigned)S * 4u, 0x00020000);
  RowStream<KV_BI, KV_NW> srcq, srcdo;
  constexpr int PER = RowStream<KV_BI, KV_NW>::PER_WAVE, NREQ = 2 * PER + 1;
  srcq.init(ld, wave, lane);
  srcdo.init(Hl, wave, lane);
  const unsigned q_bytes = (unsigned)(KV_BI * ld) * 2u, do_bytes = (unsigned)(KV_BI * Hl) * 2u;
  const int col = h * DH * 2;
  auto q_slot = [&](int slot) { return smem + slot * KV_TILE; };
  auto do_slot = [&](int slot) { return smem + KV_OFF_DO + slot * KV_TILE; };
  auto aux_load = [&](int t, char* dst, bool on) {
    const int i = t * KV_BI + lane;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(raux, (lds_void_ptr)(on ? dst : smem + KV_OFF_SINK), 4,
                                             (on && lane < KV_BI && i < S) ? (unsigned)i * 4u : OOB, 0, 0, 0);
  };
  srcq.load(rq, (unsigned)t0 * q_bytes, col, q_slot(0), wave);
  srcq.load(rq, (unsigned)(t0 + 1) * q_bytes, col, q_slot(1), wave);
  srcdo.load(rdo, (unsigned)t0 * do_bytes, col, do_slot(0), wave);
  const bool lse_or_d = wave < (OWN_D ? 1 : 2), d_too = !OWN_D && wave == 1;
  aux_load(t0, wave == 0 ? do_slot(0) + KV_BI * ROWB : q_slot(0) + KV_BI * ROWB, lse_or_d);
  aux_load(t0 + 1, q_slot(1) + KV_BI * ROWB, d_too);
  srcq.load(rq, (unsigned)(t0 + 2) * q_bytes, col, q_slot(2), wave);
  srcdo.load(rdo, (unsigned)(t0 + 1) * do_bytes, col, do_slot(1), wave);
  aux_load(wave == 0 ? t0 + 1 : t0 + 2, (wave == 0 ? do_slot(1) : q_slot(2)) + KV_BI * ROWB, lse_or_d);
  float* const own_d = reinterpret_cast<float*>(smem + KV_SMEM);     // of rows j0 .. 32 nt - 1
  if constexpr (OWN_D) {
    // CPR lanes to a row, 16 bytes of it each
    constexpr int RPS = 64 * KV_NW / CPR, AHEAD = 4;
    const int rows = nt * KV_BI - j0, r0 = threadIdx.x / CPR, c = threadIdx.x % CPR;
    const size_t at = ((size_t)b * S + j0) * Hl + h * DH + c * 8;
    for (int base = 0; base < rows; base += AHEAD * RPS) {
      bf16x8 x[AHEAD], y[AHEAD];
#pragma unroll
      for (int k = 0; k < AHEAD; k++) {
        const size_t row = at + (size_t)min(base + k * RPS + r0, S - 1 - j0) * Hl;
        x[k] = *reinterpret_cast<const bf16x8*>(dctx + row);
        y[k] = *reinterpret_cast<const bf16x8*>(a.ctx + row);
      }
#pragma unroll
      for (int k = 0; k < AHEAD; k++) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 8; e++) d = __builtin_fmaf((float)x[k][e], (float)y[k][e], d);
#pragma unroll
        for (int o = CPR / 2; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
        const int r = base + k * RPS + r0;
        if (c == 0 && r < rows) own_d[r] = j0 + r < S ? d : 0.f;
      }
    }
  }
  const int j = jw + l32;
  // dropout: this key's column of keep bits, KV_BI bits per query tile (both roles read them; they are
  // fetched one phase before their use)
  const unsigned* kcol = DROP ? keep.bits + (((size_t)b * nl + h) * S + min(j, S - 1)) * keep.wpr : nullptr;
  auto keep_word = [&](int t) -> unsigned long long { return t < t0 || t >= nt ? 0ull : kcol[t]; };
  // all that was requested before this phase has landed, and this wavefront is done with its reads
  auto meet = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NREQ) : "memory");
  };
  meet();

  int qs = 0, ds = 0;                       // ring positions of tile n
  auto q_of = [&](int d) { return q_slot(qs + d < KV_NQ ? qs + d : qs + d - KV_NQ); };       // tile n + d, d in 0 .. 4
  auto do_of = [&](int d) { return do_slot(ds + d < KV_NDO ? ds + d : ds + d - KV_NDO); };   // tile n + d, d in 0 .. 2
  // request i of phase n: this wavefront's share of Q(n + 3), of dO(n + 2), then D(n + 3) or lse(n + 2)
  auto request = [&](int n, int i) __attribute__((always_inline)) {
    if (i < PER) srcq.issue(rq, (unsigned)(n + 3) * q_bytes, col, q_of(3), wave, i);
    else if (i < 2 * PER) srcdo.issue(rdo, (unsigned)(n + 2) * do_bytes, col, do_of(2), wave, i - PER);
    else aux_load(wave == 0 ? n + 2 : n + 3, (wave == 0 ? do_of(2) : q_of(3)) + KV_BI * ROWB, lse_or_d);
  };
  auto request_all = [&](int n) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NREQ; i++) request(n, i);
  };
  auto advance = [&]() __attribute__((always_inline)) {
    qs = qs == KV_NQ - 1 ? 0 : qs + 1;
    ds = ds == KV_NDO - 1 ? 0 : ds + 1;
  };
  struct CFrag { bf16x4 lo, hi; };
  constexpr int NPC = 2 * NDT, VD = 4, KD = 4;       // products with a transposed tile; fragments requested ahead
  static_assert(NPC >= VD && NS >= KD && NREQ <= NS, "slots of a phase");
  // product p takes head-dim block p % NDT and rows 16 (p / NDT) .. + 15 of the tile
  auto c_request = [&](unsigned ct, auto P, CFrag& f) __attribute__((always_inline)) {
    constexpr int p = decltype(P)::value, dt = p % NDT, u = p / NDT;
    f.lo = lds_read_tr_issue<u * 16 * ROWB>(ct + coff[0][dt]);
    f.hi = lds_read_tr_issue<u * 16 * ROWB>(ct + coff[1][dt]);
  };
  auto c_get = [&](CFrag& f) __attribute__((always_inline)) {
    lds_pin(f.lo);
    lds_pin(f.hi);
    return __builtin_shufflevector(f.lo, f.hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // S or dP of one tile on its own
  auto first_product = [&](const char* rows, f32x16& out) __attribute__((always_inline)) {
    out = zero16();
    streamed<NS, KD>([&](int s) { return frag_rows(rows, l32, s, g); },
                     [&](int s, bf16x8 f) { out = MFMA(f, kvf[s], out); });
  };
  unsigned long long kw = 0, kw_next = 0;   // keep bits: role V: tile n; role K: tile n - 1
  // One phase.  cur: S(n) (role V) or dP(n - 1) (role K), worked on in place; nxt: S(n + 1) or dP(n).  DIAGONAL: role
  // V's tile has keys behind their queries.
  auto phase = [&](int n, f32x16& cur, f32x16& nxt, auto role_tag, auto diagonal_tag) __attribute__((always_inline)) {
    constexpr bool ROLE_V = decltype(role_tag)::value, DIAGONAL = decltype(diagonal_tag)::value;
    if (DROP) {
      kw = kw_next;
      kw_next = keep_word(ROLE_V ? n + 1 : n);
    }
    const char* rows = ROLE_V ? q_of(1) : do_of(0);
    const char* own = ROLE_V ? do_of(0) : q_of(4);                    // dO(n) and lse(n), or Q(n - 1) and D(n - 1)
    const unsigned ct = lds_addr(own);
    const float* aux = OWN_D && !ROLE_V ? own_d + (n - 1) * KV_BI - j0 : reinterpret_cast<const float*>(own + KV_BI * ROWB);
    char* const pxn = px + ((ROLE_V ? n : n - 1) & 1) * KV_PX;
    f32x4 row_value[4];
#pragma unroll
    for (int q4 = 0; q4 < 4; q4++) row_value[q4] = *reinterpret_cast<const f32x4*>(aux + 8 * q4 + 4 * g);
    bf16x8 pb[2];
    if (!ROLE_V) {
#pragma unroll
      for (int u = 0; u < 2; u++) pb[u] = *reinterpret_cast<const bf16x8*>(pxn + u * 1024);
    }
    CFrag cf[VD];
    bf16x8 rf[KD], xf[2];                   // xf: P or dS, 16 query rows per entry
#pragma unroll
    for (int q = 0; q < KD; q++) rf[q] = frag_rows(rows, l32, q, g);
    nxt = zero16();
    // the vector work in pieces: two values each, then 16 query rows to round each
    constexpr int EPP = 2, NE = 16 / EPP, NPIECE = NE + 2;
    auto piece = [&](auto K) __attribute__((always_inline)) {
      constexpr int k = decltype(K)::value;
      if constexpr (k < NE) {
        constexpr int v0 = EPP * k;
        if constexpr (ROLE_V) {
#pragma unroll
          for (int v = v0; v < v0 + EPP; v++) {
            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[v], c2, -LOG2E * row_value[v >> 2][v & 3]));
            if (DIAGONAL && j > n * KV_BI + 8 * (v >> 2) + 4 * g + (v & 3)) p = 0.f;
            cur[v] = p;
          }
        } else {
          if (DROP && k == 0) {                                   // gradient w.r.t. the undropped probabilities
            f32x16 (&one)[1] = reinterpret_cast<f32x16 (&)[1]>(cur);
            drop_unkept<1>(one, kw, g);
          }
#pragma unroll
          for (int v = v0; v < v0 + EPP; v++) {
            const float dp = DROP ? cur[v] * keep.scale : cur[v];
            cur[v] = (float)pb[v >> 3][v & 7] * (dp - row_value[v >> 2][v & 3]);
          }
        }
      } else {
        constexpr int u = k - NE;
        xf[u] = pack_half(cur, u);
        if constexpr (ROLE_V) *reinterpret_cast<bf16x8*>(pxn + u * 1024) = xf[u];
        if constexpr (ROLE_V && DROP && u == 1) {                 // dV takes the dropped probabilities
          f32x16 (&one)[1] = reinterpret_cast<f32x16 (&)[1]>(cur);
          drop_unkept<1>(one, kw, g);
#pragma unroll
          for (int w = 0; w < 2; w++) xf[w] = pack_half(cur, w);
        }
      }
    };
    constexpr auto cost = [](int k) constexpr { return k < NE ? (ROLE_V ? 7 : 3) * EPP : 6; };
    constexpr auto upto = [cost](int k) constexpr { int c = 0; for (int x = 0; x < k; x++) c += cost(x); return c; };
    constexpr int TOTAL = upto(NPIECE);
    // piece k goes behind first product slot_of(k)
    constexpr auto slot_of = [upto, cost](int k) constexpr { return (upto(k) + cost(k) / 2) * NS / TOTAL; };
    __builtin_amdgcn_sched_barrier(0);
    unroll<NS>([&](auto I) __attribute__((always_inline)) {
      constexpr int x = decltype(I)::value;
      nxt = MFMA(rf[x % KD], kvf[x], nxt);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (x + KD < NS) rf[x % KD] = frag_rows(rows, l32, x + KD, g);
      if constexpr (x >= NS - VD) c_request(ct, std::integral_constant<int, x - (NS - VD)>(), cf[x - (NS - VD)]);
      if constexpr (x < NREQ) request(n, x);
      unroll<NPIECE>([&](auto K) __attribute__((always_inline)) {
        if constexpr (slot_of(decltype(K)::value) == x) piece(K);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    unroll<NPC>([&](auto P) __attribute__((always_inline)) {
      constexpr int p = decltype(P)::value, newer = 2 * ((p + VD < NPC ? p + VD : NPC) - p - 1);   // untracked, younger
      lds_wait_le<newer>();
      acc[p % NDT] = MFMA(xf[p / NDT], c_get(cf[p % VD]), acc[p % NDT]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (p + VD < NPC) c_request(ct, std::integral_constant<int, p + VD>(), cf[p % VD]);
    });
    asm volatile("" : "+v"(nxt));           // also where no tile follows
  };
  // One loop per role (the branch is wavefront-uniform; both pass a barrier after each of the phases t0 .. nt - 1).
  f32x16 sa, sb;
  int n = t0;
  if (role_v) {
    if (DROP) kw_next = keep_word(tp);
    if (tp == t0) first_product(q_of(0), sa);
    for (; n < tp && n < nt; n++) {
      request_all(n);
      if (n + 1 == tp) first_product(q_of(1), sa);
      meet();
      advance();
    }
    if (n < nt) {
      auto next = [&](f32x16& cur, f32x16& nxt, auto diagonal_tag) __attribute__((always_inline)) {
        phase(n, cur, nxt, std::true_type(), diagonal_tag);
        meet();
        advance();
        n++;
      };
      next(sa, sb, std::true_type());
      while (n + 1 < nt) {
        next(sb, sa, std::false_type());
        next(sa, sb, std::false_type());
      }
      if (n < nt) next(sb, sa, std::false_type());
    }
  } else {
    for (; n <= tp && n < nt; n++) {
      request_all(n);
      if (n == tp) first_product(do_of(0), sa);
      meet();
      advance();
    }
    if (tp < nt) {                          // n is tp + 1; phases up to nt
      if (DROP) kw_next = keep_word(tp);
      auto next = [&](f32x16& cur, f32x16& nxt) __attribute__((always_inline)) {
        phase(n, cur, nxt, std::false_type(), std::false_type());
        if (n < nt) meet();
        advance();
        n++;
      };
      while (n < nt) {
        next(sa, sb);
        next(sb, sa);
      }
      if (n <= nt) next(sa, sb);
    }
  }
  WAIT_VM0();   // requests for tiles beyond the last one (zero fill) must not outlive the workgroup's LDS
  // accumulator register v of lane l is row 8 (v/4) + 4 g + v%4, column l%32 of its 32x32 tile
  const float oscale = role_v ? (DROP ? keep.scale : 1.f) : scale;
  bf16* obase = dqkv + (size_t)b * S * ld + h * DH + (role_v ? 2 * Hl : Hl);
#pragma unroll
  for (int dt = 0; dt < NDT; dt++)
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int jr = jw + 8 * (v >> 2) + 4 * g + (v & 3);
      if (jr < S) obase[(size_t)jr * ld + 32 * dt + l32] = (bf16)(acc[dt][v] * oscale);
    }
}

// ------------------------------------------------------------------------------- backward: dQ
// Shapes and workgroup order as in the forward kernel; the parts' dQ partial sums are added
// through LDS in the order of `part`.  It runs before the dK / dV kernel and leaves D[b, h, s] = sum_d dO * O for it.
// The rows of dO are here anyway; those of O are read as row fragments, once by every share of the keys, and waited for before
// the first tile, so the kernel takes longer by about what a launch of D's own took (64 pairs of S 2048 130 + 14.3 -> 146 us,
// 64 of S 1024 41.6 + 8.8 -> 44.3, 16 of S 2048 42.7 + 7.4 -> 43.6; DH 64: 64 of S 2048 65.8 + 8.4 -> 75.7, 64 of S 1024 25.1 +
// 7.7 -> 28.0).  What is gained is that launch's wait for compute units beside the weight gradients of the other stream, up to
// 250 us: steps of hidden 768, 1024 tokens 198.5 -> 193, hidden 2048, 8192 tokens 2486 -> 2465, attention half of 4 heads and
// S 8192 958 -> 934; the order of the kernels beside those gradients changes with it, and a step with dropout of hidden 896,
// 2976 tokens, is 3 % slower (252 -> 260) although its kernels one by one take 300 -> 288.
// Block `blk` of the launch order; PAIRED as in the other kernel.
template <int NQ, int SPLIT, int BKV, bool DROP>
GX_DEVINL void dq_block(const BwdArgs& a, const KeepArgs& keep, int blk, bool paired, char* smem) {
  const bf16* __restrict__ const qkv = a.qkv;
  const bf16* __restrict__ const ctx = a.ctx;
  const bf16* __restrict__ const dctx = a.dctx;
  const float* __restrict__ const lse = a.lse;
  float* __restrict__ const dsum = a.dsum;
  bf16* __restrict__ const dqkv = a.dqkv;
  const int S = a.S, nl = a.nl, npair = a.npair;
  constexpr int NW = NQ * SPLIT, BQ = 32 * NQ, ROWS = BKV * SPLIT, STAGE = 2 * ROWS * ROWB;
  constexpr int NJT = BKV / 32;
  static_assert((SPLIT - 1) * NQ * (DH / 2) * 256 <= 2 * STAGE, "merge area fits the tile buffers");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qs = wave % NQ, part = wave / NQ;
  const int g = lane >> 5, l32 = lane & 31;
  const int nq = (S + BQ - 1) / BQ;
  const int pair = blk % npair;
  // longest blocks first; with two workgroups per compute unit (4 wavefronts each), the second
  // half of the launch runs shortest first, as in the forward kernel
  const int rq = blk / npair, hq = (nq + 1) / 2;
  const int qt = (paired && rq >= hq) ? rq - hq : nq - 1 - rq;
  const int h = pair % nl, b = pair / nl;
  const int Hl = nl * DH, ld = 3 * Hl;
  const int i0 = qt * BQ, iw = i0 + qs * 32;
  const bf16* sample = qkv + (size_t)b * S * ld;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(sample), 0,
                                                                        (unsigned)(S * ld) * 2u, 0x00020000);
  bf16x8 qf[DH / 16], dof[DH / 16];
  load_row_frags(sample + h * DH, ld, iw + l32, S, g, qf);
  load_row_frags(dctx + (size_t)b * S * Hl + h * DH, Hl, iw + l32, S, g, dof);
  bf16x8 of[DH / 16];
  load_row_frags(ctx + (size_t)b * S * Hl + h * DH, Hl, iw + l32, S, g, of);
  const int i = iw + l32;
  const int ic = min(i, S - 1);
  const float scale = rsqrtf((float)DH), c2 = scale * LOG2E;
  const float lse2 = lse[((size_t)b * nl + h) * S + ic] * LOG2E;
  unsigned coff[2][DH / 32];
  cols_lane_offsets(lane, coff);
  f32x16 dq[DH / 32];
#pragma unroll
  for (int dt = 0; dt < DH / 32; dt++) dq[dt] = zero16();

  const int jend = min(S, i0 + BQ);
  const int nt = (jend + ROWS - 1) / ROWS;
  RowStream<ROWS, NW> src;
  src.init(ld, wave, lane);
  const int kcol = (Hl + h * DH) * 2, vcol = (2 * Hl + h * DH) * 2;
  const unsigned tile_bytes = (unsigned)(ROWS * ld) * 2u;
  src.load(rsrc, 0, kcol, smem, wave);
  src.load(rsrc, 0, vcol, smem + ROWS * ROWB, wave);
  float d4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < DH / 16; s++)
#pragma unroll
    for (int e = 0; e < 8; e++) d4[e & 3] = __builtin_fmaf((float)of[s][e], (float)dof[s][e], d4[e & 3]);
  float dd = (d4[0] + d4[1]) + (d4[2] + d4[3]);
  dd += __shfl_xor(dd, 32, 64);
  if (part == 0 && g == 0 && i < S) dsum[((size_t)b * nl + h) * S + i] = dd;
  const unsigned* kwords = DROP ? keep.bits + (((size_t)b * nl + h) * S + ic) * keep.wpr : nullptr;
  WAIT_VM0();
  __syncthreads();
  for (int t = 0; t < nt; t++) {
    if (t + 1 < nt) {
      char* nxt = smem + ((t + 1) & 1) * STAGE;
      src.load(rsrc, (unsigned)(t + 1) * tile_bytes, kcol, nxt, wave);
      src.load(rsrc, (unsigned)(t + 1) * tile_bytes, vcol, nxt + ROWS * ROWB, wave);
    }
    const int j0 = t * ROWS + part * BKV;
    if (j0 <= iw + 31) {
      const char* kt = smem + (t & 1) * STAGE + part * BKV * ROWB;
      const char* vt = kt + ROWS * ROWB;
      unsigned long long kw = 0;                        // keep bits of this query's keys of the step
      if (DROP) kw = keep_bits_of_step<NJT>(kwords, j0);
      f32x16 sacc[NJT], pacc[NJT];
#pragma unroll
      for (int jt = 0; jt < NJT; jt++) {
        sacc[jt] = zero16();
        pacc[jt] = zero16();
#pragma unroll
        for (int s = 0; s < DH / 16; s++) {
          sacc[jt] = MFMA(frag_rows(kt, 32 * jt + l32, s, g), qf[s], sacc[jt]);    // S^T[j][i]
          pacc[jt] = MFMA(frag_rows(vt, 32 * jt + l32, s, g), dof[s], pacc[jt]);   // dP^T[j][i]
        }
      }
      if (DROP) {                                      // gradient w.r.t. the undropped probabilities
        // Left to mix the masks into the products the compiler needs 12 registers more than there are at head dim 128
        // (64 pairs of S 2048: 209 us, 150 as it is) and 175 at head dim 64, two wavefronts per SIMD (128 pairs 176, 160).
        asm volatile("" : "+v"(kw));                   // the keep bits are waited for here, after the products (164 without)
        drop_unkept<NJT>(pacc, kw, g);
#pragma unroll
        for (int jt = 0; jt < NJT; jt++)
#pragma unroll
          for (int v = 0; v < 16; v++) pacc[jt][v] *= keep.scale;
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int jt = 0; jt < NJT; jt++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[jt][v], c2, -lse2));
          pacc[jt][v] = p * (pacc[jt][v] - dd);                                    // dS^T
        }
      // the scores are dead: their registers take the first transposed K fragments
      const unsigned ct = lds_addr(kt);
      ColFrags cf[2];
      cols_issue<0>(ct, coff, cf[0]);
      cols_issue<1>(ct, coff, cf[1]);
      if (j0 + BKV - 1 > iw) {                         // the tile touches the diagonal
#pragma unroll
        for (int jt = 0; jt < NJT; jt++)
#pragma unroll
          for (int v = 0; v < 16; v++)
            if (j0 + 32 * jt + 8 * (v >> 2) + 4 * g + (v & 3) > i) pacc[jt][v] = 0.f;
      }
      bf16x8 dsf[2 * NJT];
#pragma unroll
      for (int u = 0; u < 2 * NJT; u++) dsf[u] = pack_half(pacc[u >> 1], u & 1);
      tr_product<2 * NJT>(dq, ct, coff, cf, dsf);       // dQ^T[d][i] += K^T dS^T
    }
    WAIT_VM0();
    __syncthreads();
  }
  if (SPLIT > 1) {
    constexpr int REGION = (DH / 2) * 64;
    if (part > 0) {
      float* park = reinterpret_cast<float*>(smem) + ((part - 1) * NQ + qs) * REGION + lane;
#pragma unroll
      for (int dt = 0; dt < DH / 32; dt++)
#pragma unroll
        for (int v = 0; v < 16; v++) park[(16 * dt + v) * 64] = dq[dt][v];
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int pp = 1; pp < SPLIT; pp++) {
      const float* park = reinterpret_cast<const float*>(smem) + ((pp - 1) * NQ + qs) * REGION + lane;
#pragma unroll
      for (int dt = 0; dt < DH / 32; dt++)
#pragma unroll
        for (int v = 0; v < 16; v++) dq[dt][v] += park[(16 * dt + v) * 64];
    }
  }
  if (i < S) {
    bf16* row = dqkv + ((size_t)b * S + i) * ld + h * DH;
#pragma unroll
    for (int dt = 0; dt < DH / 32; dt++)
#pragma unroll
      for (int q4 = 0; q4 < 4; q4++) {
        bf16x4 pk;
#pragma unroll
        for (int e = 0; e < 4; e++) pk[e] = (bf16)(dq[dt][4 * q4 + e] * scale);
        *reinterpret_cast<bf16x4*>(row + 32 * dt + 8 * q4 + 4 * g) = pk;
      }
  }
}

// ------------------------------------------------------------------------------- backward: launches
template <bool DROP>
__global__ void __launch_bounds__(64 * KV_NW, DH == 64 ? 3 : 2) attn_bwd_dkv_kernel(BwdArgs a, KeepArgs keep) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  dkv_block<DROP, false>(a, keep, blockIdx.x, gridDim.x <= KV_PAIRED, smem);
}
template <int NQ, int SPLIT, int BKV, bool DROP>
__global__ void __launch_bounds__(64 * NQ * SPLIT, NQ * SPLIT == 4 ? 2 : 1) attn_bwd_dq_kernel(BwdArgs a, KeepArgs keep) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  dq_block<NQ, SPLIT, BKV, DROP>(a, keep, blockIdx.x, NQ * SPLIT == 4, smem);
}
// Both in one launch (see one_launch()), first the blocks of dK / dV, which have more to do.  dQ's blocks store D here too, 4 bytes
// a row that nobody reads.
template <bool DROP>
__global__ void __launch_bounds__(256, 2) attn_bwd_both_kernel(BwdArgs a, KeepArgs rows, KeepArgs cols) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int blk = blockIdx.x, n = gridDim.x / 2;
  if (blk < n) dkv_block<DROP, true>(a, cols, blk, false, smem);
  else dq_block<2, 2, 32, DROP>(a, rows, blk - n, false, smem);
}

template <typename K>
hipError_t set_smem(K kernel, int bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             bytes);
}

bool attn_shape_ok(const AttnArgs& a) {
  if (a.dh != DH || a.B <= 0 || a.S <= 0 || a.nl <= 0) return false;
  const size_t bytes = (size_t)a.B * a.S * 3 * a.nl * DH * 2;
  return bytes < (1ul << 31);
}

// With few (sample, head) pairs the chip is filled by cutting the query blocks fine and spreading
// each block's keys over two or four wavefronts (see the forward kernel).
bool few_pairs(const AttnArgs& a) { return (long)a.B * a.nl * cdiv(a.S, 128) <= 384; }

// Few pairs, forward: the keys of a step over four wavefronts instead of two where the workgroups of 64 query rows
// then still find a compute unit each, or are at most two per unit of fewer than 16 pairs, whose sequences are then so long
// that a unit's two would spend most of their time one after the other (a long and a short one together).  Each has a longer
// start and end, so the keys must be many.  us, two / four: 12 pairs of S 1024 14.7 / 14.0, of S 512 10.0 / 10.5, 12 of S 2048
// 27.9 / 25.9, 16 of S 2048 28.1 / 28.9, 8 of S 4096 50.1 / 46.6, 4 of S 8192 108 / 87.
bool keys_over_four(const AttnArgs& a) {
  const long pairs = (long)a.B * a.nl, blocks = pairs * cdiv(a.S, 64);
  return a.S >= 768 && (blocks <= 256 || (blocks <= 512 && pairs < 16));
}

// The same for the dQ kernel, whose steps are longer, so that the start and the end matter more.  us, two / four, head dim
// 128: 12 pairs of S 1024 21.4 / 22.1, 4 of S 1024 20.2 / 20.7, 2 of S 2048 33.5 / 30.6, 8 of S 2048 34.8 / 33.6, 12 of S 2048
// 40.9 / 40.0, 4 of S 4096 61.4 / 55.2, 7 of S 4096 73.6 / 68.3, 8 of S 4096 76.4 / 77.1, 4 of S 8192 140.5 / 132.3, 5 of S 8192
// (640 workgroups, one per unit: a third round) 153.7 / 183.2, 6 184.3 / 198.1, with dropout 226 / 251.  Head dim 64, where two
// share a unit: 12 of S 1024 14.8 / 14.7, 8 of S 2048 22.6 / 19.4, 7 of S 4096 43.5 / 37.9, 4, 5, 6 of S 8192 81.5 / 71.2, 89.5 /
// 81.1, 95.0 / 92.5.
bool dq_keys_over_four(const AttnArgs& a) {
  const long pairs = (long)a.B * a.nl, blocks = pairs * cdiv(a.S, 64);
  return a.S >= 2048 && (blocks <= 256 || (pairs < 8 && (blocks <= 512 || DH == 64)));
}

// over how many wavefronts the keys of a query block are spread (1: many pairs)
int fwd_key_shares(const AttnArgs& a) { return !few_pairs(a) ? 1 : keys_over_four(a) ? 4 : 2; }
int dq_key_shares(const AttnArgs& a) { return !few_pairs(a) ? 1 : dq_keys_over_four(a) ? 4 : 2; }

// the dQ kernel in its three shapes, <4, 1, 64>, <2, 2, 32> and <2, 4, 32>: two stages of 64 or 128 rows of K and of V
constexpr int SMEM_MANY = 2 * 2 * 64 * ROWB, SMEM_FEW = 2 * 2 * 64 * ROWB, SMEM_FOUR_DQ = 2 * 2 * 128 * ROWB;

hipError_t fwd(const AttnArgs& a, hipStream_t s) {
  if (!attn_shape_ok(a)) return hipErrorInvalidValue;
  static bool configured = false;
  constexpr int SMEM_MANY_FWD = fwd_smem(4, 1, 64), SMEM_TWO = fwd_smem(2, 2, 32), SMEM_FOUR = fwd_smem(2, 4, 32);
  if (!configured) {
    hipError_t e = set_smem(attn_fwd_kernel<4, 1, 64, false, false>, SMEM_MANY_FWD);
    if (e == hipSuccess) e = set_smem(attn_fwd_kernel<2, 2, 32, true, false>, SMEM_TWO);
    if (e == hipSuccess) e = set_smem(attn_fwd_kernel<2, 4, 32, true, false>, SMEM_FOUR);
    if (e == hipSuccess) e = set_smem(attn_fwd_kernel<4, 1, 64, false, true>, SMEM_MANY_FWD);
    if (e == hipSuccess) e = set_smem(attn_fwd_kernel<2, 2, 32, true, true>, SMEM_TWO);
    if (e == hipSuccess) e = set_smem(attn_fwd_kernel<2, 4, 32, true, true>, SMEM_FOUR);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const KeepArgs keep{a.rowbits, a.wpr, a.keep_scale};
  const bool drop = a.rowbits != nullptr;
  if (drop && a.wpr != 2 * cdiv(a.S, 64)) return hipErrorInvalidValue;
  const int npair = a.nl * a.B;
  auto go = [&](auto kernel, int bq, int threads, int smem) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(a.S, bq) * npair), dim3(threads), smem, s, (const bf16*)a.qkv, (bf16*)a.ctx,
                       a.lse, a.S, a.nl, npair, keep);
  };
  const int shares = fwd_key_shares(a);
  if (shares == 1) {
    if (drop) go(attn_fwd_kernel<4, 1, 64, false, true>, 128, 256, SMEM_MANY_FWD);
    else go(attn_fwd_kernel<4, 1, 64, false, false>, 128, 256, SMEM_MANY_FWD);
  } else if (shares == 4) {
    if (drop) go(attn_fwd_kernel<2, 4, 32, true, true>, 64, 512, SMEM_FOUR);
    else go(attn_fwd_kernel<2, 4, 32, true, false>, 64, 512, SMEM_FOUR);
  } else {
    if (drop) go(attn_fwd_kernel<2, 2, 32, true, true>, 64, 256, SMEM_TWO);
    else go(attn_fwd_kernel<2, 2, 32, true, false>, 64, 256, SMEM_TWO);
  }
  return hipGetLastError();
}

// Whether dQ and dK / dV share a launch: where nothing of another stream runs beside them, all of their workgroups find a place
// at once, and forming D twice takes less than the dQ kernel.  Forward and backward on one stream, us, two launches / one: hidden
// 512 (head dim 64) 64 tokens 117.6 / 112.8, 256 131 / 126.5, 1024 166 / 161.5, 2048 212.6 / 213.2; hidden 1024, degree 4, 1024
// tokens 161.6 / 156.8; attention half of hidden 768, 1024 tokens 114 / 110.  Beside the weight gradients of larger layers it
// gains (hidden 1024, 1024 tokens 237 / 227) and loses (hidden 2048, 1024 tokens 454 / 467; hidden 768, degree 2, 2 x 1024 191 /
// 197) and is not taken.
constexpr int ONE_LAUNCH_S = 1024;
bool fits_one_launch(int B, int S, int nl) { return S <= ONE_LAUNCH_S && (long)B * nl * cdiv(S, KV_BJ) <= 256; }
bool one_launch(const AttnArgs& a) { return a.alone && fits_one_launch(a.B, a.S, a.nl); }
int one_launch_smem(int S) {
  const int kv = KV_SMEM + 4 * KV_BI * cdiv(S, KV_BI);
  return kv > SMEM_FEW ? kv : SMEM_FEW;
}

// dQ with D, then dK / dV.
hipError_t bwd(const AttnArgs& a, hipStream_t s) {
  if (!attn_shape_ok(a)) return hipErrorInvalidValue;
  static bool configured = false;
  if (!configured) {
    hipError_t e = set_smem(attn_bwd_dkv_kernel<false>, KV_SMEM);
    if (e == hipSuccess) e = set_smem(attn_bwd_dkv_kernel<true>, KV_SMEM);
    if (e == hipSuccess) e = set_smem(attn_bwd_both_kernel<false>, one_launch_smem(ONE_LAUNCH_S));
    if (e == hipSuccess) e = set_smem(attn_bwd_both_kernel<true>, one_launch_smem(ONE_LAUNCH_S));
    if (e == hipSuccess) e = set_smem(attn_bwd_dq_kernel<4, 1, 64, false>, SMEM_MANY);
    if (e == hipSuccess) e = set_smem(attn_bwd_dq_kernel<2, 2, 32, false>, SMEM_FEW);
    if (e == hipSuccess) e = set_smem(attn_bwd_dq_kernel<2, 4, 32, false>, SMEM_FOUR_DQ);
    if (e == hipSuccess) e = set_smem(attn_bwd_dq_kernel<2, 4, 32, true>, SMEM_FOUR_DQ);
    if (e == hipSuccess) e = set_smem(attn_bwd_dq_kernel<4, 1, 64, true>, SMEM_MANY);
    if (e == hipSuccess) e = set_smem(attn_bwd_dq_kernel<2, 2, 32, true>, SMEM_FEW);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const bool drop = a.rowbits != nullptr;
  if (drop && (!a.colbits || a.wpr != 2 * cdiv(a.S, 64))) return hipErrorInvalidValue;
  const KeepArgs keep_rows{a.rowbits, a.wpr, a.keep_scale}, keep_cols{a.colbits, a.wpr, a.keep_scale};
  const int npair = a.nl * a.B;
  const BwdArgs args{(const bf16*)a.qkv, (const bf16*)a.ctx, (const bf16*)a.dctx, a.lse, a.dsum, (bf16*)a.dqkv,
                     a.S, a.nl, npair};
  if (one_launch(a)) {
    static_assert(KV_BJ == 64, "as many blocks of keys as of queries");
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(2 * cdiv(a.S, KV_BJ) * npair), dim3(256), one_launch_smem(a.S), s, args, keep_rows,
                         keep_cols);
    };
    if (drop) go(attn_bwd_both_kernel<true>);
    else go(attn_bwd_both_kernel<false>);
    return hipGetLastError();
  }
  auto go_dq = [&](auto kernel, int bq, int threads, int smem) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(a.S, bq) * npair), dim3(threads), smem, s, args, keep_rows);
  };
  const int shares = dq_key_shares(a);
  if (shares == 4) {
    if (drop) go_dq(attn_bwd_dq_kernel<2, 4, 32, true>, 64, 512, SMEM_FOUR_DQ);
    else go_dq(attn_bwd_dq_kernel<2, 4, 32, false>, 64, 512, SMEM_FOUR_DQ);
  } else if (shares == 2) {
    if (drop) go_dq(attn_bwd_dq_kernel<2, 2, 32, true>, 64, 256, SMEM_FEW);
    else go_dq(attn_bwd_dq_kernel<2, 2, 32, false>, 64, 256, SMEM_FEW);
  } else {
    if (drop) go_dq(attn_bwd_dq_kernel<4, 1, 64, true>, 128, 256, SMEM_MANY);
    else go_dq(attn_bwd_dq_kernel<4, 1, 64, false>, 128, 256, SMEM_MANY);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto go_dkv = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(a.S, KV_BJ) * npair), dim3(64 * KV_NW), KV_SMEM, s, args, keep_cols);
  };
  if (drop) go_dkv(attn_bwd_dkv_kernel<true>);
  else go_dkv(attn_bwd_dkv_kernel<false>);
  return hipGetLastError();
}

