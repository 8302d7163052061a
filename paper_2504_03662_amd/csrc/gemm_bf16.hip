// bf16 MFMA GEMM family for gfx950: the dense contractions of one rank's transformer-block share
// (column-parallel QKV / FC1, row-parallel out-proj / FC2, their input and weight gradients).
//
// One workgroup computes a tile of C through LDS stages that loads fill straight from HBM
// (buffer_load ... lds, 16 B per lane, no register staging): 256 x 256 by 8 wavefronts of 128 x 64 and a
// double buffer of 64 reduction steps, and six smaller tiles for products that would leave compute
// units without one, the smallest of them with several wavefronts per place that share every stage's
// reduction steps (see the tiles and their prices below).
// Products are v_mfma_f32_16x16x32_bf16: on this chip the large products run at the board's power
// limit, and a register-only loop on normal data holds 2030 TFLOP/s with that instruction against
// 1811 with 32x32x16 (on zeros 2411 and 2472): it reads and writes an accumulator half as often.
// Fragments come from ds_read_b128 when the reduction index is contiguous in memory ("K-major" tiles)
// and from the transposing ds_read_b64_tr_b16 when it is strided ("MN-major" tiles), so no operand is
// ever transposed in HBM.  LDS positions are XOR-swizzled on the global-address side because a
// direct-to-LDS load fixes each lane's LDS slot.
// Measured, TFLOP/s at 4096^3 / 8192^3 (warm, normal data) against the 32x32x16 form of the same loop:
// NN 1262 / 1360 -> 1383 / 1443, NT 1275 / 1368 -> 1407 / 1448, TN 1224 / 1337 -> 1285 / 1355; the 128 x 128
// tile against one with 8 wavefronts of 64 x 32: 4096 x 1024 x 4096 NT 40.1 -> 31.7 us, NN 42.5 -> 33.0,
// 1024 x 4096 x 4096 TN 44.0 -> 35.0.
#include "gx_kernels.h"
#include <type_traits>

namespace gx {
namespace {

constexpr unsigned OOB = 0x80000000u;           // beyond num_records: the load writes zeros

// A workgroup's tile: BM x BN of C by WGM x WGN wavefronts, times KW wavefronts that share each of
// those places and take interleaved shares of every stage of KE reduction steps; STAGES stages in LDS.
template <int BM_, int BN_, int WGM_, int WGN_, int KW_, int KE_, int STAGES_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, KW = KW_, KE = KE_, STAGES = STAGES_;
  static constexpr int NW = WGM * WGN * KW, THREADS = 64 * NW;
  static constexpr int WM = BM / WGM, WN = BN / WGN;           // a wavefront's part of C
  static constexpr int TM = WM / 16, TN = WN / 16;             // in 16 x 16 accumulators
  static constexpr int KS = KE / KW / 32;                      // sub-steps of a wavefront's share of a stage
  static constexpr int A_BYTES = BM * KE * 2, B_BYTES = BN * KE * 2;
  static constexpr int RING = STAGES * (A_BYTES + B_BYTES);
  static constexpr int PADN = BN + 4;                          // row of a parked tile, in floats (KW > 1)
  static constexpr int PARK = KW > 1 ? KW * BM * PADN * 4 + NW * BN * 4 : 0;
  static constexpr int SMEM = RING > PARK ? RING : PARK;
  static_assert(KE <= 128 || KE == 256, "swizzle");
  static_assert(KS == 1 || KS == 2, "the loop over tiles alternates fragment buffers");
};

// K-major tile: [R rows][BK k], 2 BK bytes per row, 16 B chunk c of row r stored at c ^ swz_k(r):
// the 16 rows that one ds_read_b128 pass covers at a fixed chunk then fall in distinct banks.
template <int BK>
GX_DEVINL int swz_k(int r) { return BK >= 128 ? (r & 15) : ((r >> 1) & 7); }
// MN-major tile: [BK k-rows][R cols], 2R B per k-row, 16 B chunk c of k-row kr stored at
// c ^ swz_mn(kr): whole 64 B groups move so that 4 consecutive k-rows fall in distinct banks (where
// rows are an odd multiple of 128 B, consecutive rows already alternate between bank halves), and the
// 32 B halves of a group swap every 8 k-rows, because one pass of the transposing read takes 32 B
// of 4 consecutive k-rows and of the 4 that lie 8 further on.
template <int R>
GX_DEVINL int swz_mn(int kr) {
  return (R % 128 == 0 ? (kr & 3) << 2 : ((kr >> 1) & 1) << 2) | (((kr >> 3) & 1) << 1);
}

GX_DEVINL __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}

// This wave's share of the direct-to-LDS loads of one operand tile (R rows/columns by BK reduction
// steps): R * BK / (512 NW) instructions of 64 lanes x 16 B each.
template <bool KMAJOR, int R, int BK, int NW>
struct TileLoader {
  static constexpr int PER = R * BK / (512 * NW);
  static_assert(PER * 512 * NW == R * BK, "whole instructions per wavefront");
  unsigned base[PER];   // k-invariant part of the lane's element offset, or OOB
  int kc[PER];          // K-major: k offset of the chunk; MN-major: k-row of the chunk
  unsigned voff[PER];   // the same as a byte offset (or OOB): the vector offset of the cheap form
  __amdgpu_buffer_rsrc_t rsrc;
  int ld, K;

  GX_DEVINL void init(const bf16* ptr, unsigned bytes, int ld_, int K_, int origin, int extent, int wave,
                      int lane) {
    rsrc = make_rsrc(ptr, bytes);
    ld = ld_;
    K = K_;
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const int q = wave * PER + i;
      if (KMAJOR) {
        constexpr int CPR = BK / 8;                // 16 B chunks per row
        constexpr int RPI = 64 / CPR;              // rows per instruction
        const int r = RPI * q + lane / CPR;
        const int c = (lane % CPR) ^ swz_k<BK>(r);
        kc[i] = c * 8;
        base[i] = (origin + r < extent) ? (unsigned)((origin + r) * ld + c * 8) : OOB;
      } else {
        constexpr int CPR = R / 8;                 // 16 B chunks per k-row
        const int kr = (64 * q + lane) / CPR;
        const int c = ((64 * q + lane) % CPR) ^ swz_mn<R>(kr);
        kc[i] = kr;
        base[i] = (origin + c * 8 < extent) ? (unsigned)(kr * ld + origin + c * 8) : OOB;
      }
      voff[i] = (base[i] != OOB) ? base[i] * 2u : OOB;
    }
  }
  // instruction i of this wave's share of the tile that starts at reduction index k0, into LDS at
  // `dst`; lanes beyond the operand or beyond K get zeros
  GX_DEVINL void issue_one(char* dst, int k0, int wave, int i) const {
    unsigned off;
    if (KMAJOR) off = (base[i] != OOB && k0 + kc[i] < K) ? (base[i] + (unsigned)k0) * 2u : OOB;
    else        off = (base[i] != OOB && k0 + kc[i] < K) ? (base[i] + (unsigned)(k0 * ld)) * 2u : OOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + (wave * PER + i) * 1024), 16, off, 0, 0,
                                             0);
  }
  GX_DEVINL void issue(char* dst, int k0, int wave) const {
#pragma unroll
    for (int i = 0; i < PER; i++) issue_one(dst, k0, wave, i);
  }
  // The cheap form, for a tile that lies wholly inside K: the tile's reduction index goes into the
  // instruction's scalar offset (which takes no part in the range check, hence the condition) and
  // the lane's vector offset never changes, so a load costs no vector arithmetic at all.
  GX_DEVINL unsigned tile_offset(int k0) const { return KMAJOR ? (unsigned)k0 * 2u : (unsigned)(k0 * ld) * 2u; }
  GX_DEVINL void issue_inside(char* dst, unsigned tile_off, int wave, int i) const {
    unsigned off = voff[i];
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + (wave * PER + i) * 1024), 16, off,
                                             tile_off, 0, 0);
  }
};

// Operands of v_mfma_f32_16x16x32_bf16: lane l holds row (or column) l % 16 and reduction steps
// 8 (l / 16) .. + 7 of the sub-step.  A fragment being fetched is either complete (K-major tile, one
// ds_read_b128 the compiler tracks) or two untracked transposing reads of an MN-major tile, which
// the loop waits for by count.
struct Frag {
  bf16x8 full;
  bf16x4 lo, hi;
};
template <int BK>
GX_DEVINL bf16x8 frag_k(const char* tile, int row, int k32, int q) {
  const int c = (4 * k32 + q) ^ swz_k<BK>(row);
  return *reinterpret_cast<const bf16x8*>(tile + row * (2 * BK) + (c << 4));
}
template <int R>
GX_DEVINL void frag_mn_issue(const char* tile, int col0, int k32, int lane, Frag& f) {
  const int q = lane >> 4, s = lane & 15;
  const int kr = 32 * k32 + 8 * q + (s >> 2);
  const int ne = col0 + 4 * (s & 3);
  const int c = (ne >> 3) ^ swz_mn<R>(kr);
  const unsigned addr = lds_addr(tile + kr * (2 * R) + (c << 4) + (ne & 7) * 2);
  f.lo = lds_read_tr_issue<0>(addr);
  f.hi = lds_read_tr_issue<4 * (2 * R)>(addr);
}
GX_DEVINL bf16x8 frag_mn_finish(Frag& f) {
  lds_pin(f.lo);
  lds_pin(f.hi);
  return __builtin_shufflevector(f.lo, f.hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// wait until at most n LDS operations of this wavefront are outstanding; n is a constant once the
// caller's loops are unrolled (one short of the counter's maximum at most)
GX_DEVINL void lds_wait_most(int n) {
#define GX_W(N) case N: lds_wait_le<N>(); break;
  switch (n) {
    GX_W(0) GX_W(1) GX_W(2) GX_W(3) GX_W(4) GX_W(5) GX_W(6) GX_W(7) GX_W(8) GX_W(9) GX_W(10) GX_W(11) GX_W(12)
    GX_W(13)
    default: lds_wait_le<14>();
  }
#undef GX_W
}

// What nothing reads soon after goes past the caches (non-temporal): weight gradients (the TN products'
// outputs, read again by a later micro-batch or the optimizer) and gelu'(z) (kept for the backward
// pass), as does gelu'(z) on its only read.  The next kernel's operands stay cached instead: layer steps
// 2587 -> 2545 us (hidden 2048, 8192 tokens), 1292 -> 1280 (hidden 4096, degree 4), 583 -> 560 (hidden 1024,
// dropout, bf16 gradients), the pipeline stage with accumulation 20720 -> 20450; none slower.
// Side inputs of an epilogue: what it reads besides the accumulators (the residual, gelu'(z), the
// weight gradient being added to), one run of 4 columns.
template <int EPI>
struct Side {
  static constexpr bool B16 = (EPI == EPI_RESID || EPI == EPI_DGELU), F32 = (EPI == EPI_F32_ACC), ANY = B16 || F32;
  bf16x4 h;
  f32x4 f;
  GX_DEVINL void fetch(const GemmArgs& g, size_t idx) {
    if (EPI == EPI_RESID) h = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(g.resid) + idx);
    if (EPI == EPI_DGELU)
      h = __builtin_nontemporal_load(reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(g.z) + idx));
    if (F32) f = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(static_cast<const float*>(g.C) + idx));
  }
};
template <int EPI>
GX_DEVINL void load_bias(const GemmArgs& g, int col, float (&bv)[4]) {
#pragma unroll
  for (int e = 0; e < 4; e++) bv[e] = 0.f;
  if ((EPI == EPI_BIAS || EPI == EPI_RESID || EPI == EPI_GELU) && g.bias && col < g.N) {
    const bf16x4 b4 = *reinterpret_cast<const bf16x4*>(static_cast<const bf16*>(g.bias) + col);
#pragma unroll
    for (int e = 0; e < 4; e++) bv[e] = (float)b4[e];
  }
}
// One run of 4 columns of C from its sums: bias, the epilogue's arithmetic, the stores.  cs (EPI_DGELU):
// the stored values are added to it.
template <int LAY, int EPI>
GX_DEVINL void finish_run(const GemmArgs& g, size_t idx, const f32x4& xv, const float (&bv)[4], const Side<EPI>& side,
                          float (&cs)[4]) {
  float x[4] = {xv[0] + bv[0], xv[1] + bv[1], xv[2] + bv[2], xv[3] + bv[3]};
  bf16* aux = static_cast<bf16*>(g.aux);
  if (EPI == EPI_PART) {
    *reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + idx) = f32x4{x[0], x[1], x[2], x[3]};
    return;
  }
  if (EPI == EPI_F32) {
    __builtin_nontemporal_store(f32x4{x[0], x[1], x[2], x[3]},
                                reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + idx));
    return;
  }
  if (EPI == EPI_F32_ACC) {
    __builtin_nontemporal_store(f32x4{side.f[0] + x[0], side.f[1] + x[1], side.f[2] + x[2], side.f[3] + x[3]},
                                reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + idx));
    return;
  }
  bf16x4 o;
  if (EPI == EPI_RESID) {
    if (aux) {
#pragma unroll
      for (int e = 0; e < 4; e++) o[e] = (bf16)x[e];
      *reinterpret_cast<bf16x4*>(aux + idx) = o;
    }
#pragma unroll
    for (int e = 0; e < 4; e++) x[e] += (float)side.h[e];
  } else if (EPI == EPI_GELU) {
    bf16x4 ga;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      float y, dy;
      if (g.gelu_tanh) gelu_tanh_both_fast(x[e], y, dy);
      else gelu_both_fast(x[e], y, dy);
      ga[e] = (bf16)y;
      x[e] = dy;                                     // C receives gelu'(z)
    }
    *reinterpret_cast<bf16x4*>(aux + idx) = ga;
  } else if (EPI == EPI_DGELU) {
#pragma unroll
    for (int e = 0; e < 4; e++) x[e] *= (float)side.h[e];
  }
#pragma unroll
  for (int e = 0; e < 4; e++) o[e] = (bf16)x[e];
  bf16x4* c = reinterpret_cast<bf16x4*>(static_cast<bf16*>(g.C) + idx);
  if (EPI == EPI_GELU || LAY == LAY_TN) __builtin_nontemporal_store(o, c);
  else *c = o;
  if (EPI == EPI_DGELU) {
#pragma unroll
    for (int e = 0; e < 4; e++) cs[e] += (float)o[e];
  }
}

// Workgroups beyond the tiles read the next product's weights, so that it finds them in the memory-side cache.  With few
// tokens a product is bound by what one compute unit can have in flight (20 GB/s of weights from memory, 30 from that cache,
// for a 64 x 64 tile with 4 stages of 32 KB), and has fewer tiles than the chip has units: 128 x 5120 x 10240 on 160 of
// them 64 -> 44 us.  Where: read_ahead_pays(), read_ahead_workgroups(), and only in calls without GX_FWD_PARTS; with it the
// reductions are cut into parts, which is faster (gemm_bf16_split; 128 tokens of hidden 5120, degree 2, 161 us against 132).
// A workgroup reads at most what one with a tile reads, so that it does not outlast the product.
// The values go to LDS, where nobody reads them: no registers, and nothing that could be optimised away.
template <class T>
GX_DEVINL void read_ahead(const GemmArgs& g, char* smem, int wave, int lane) {
  constexpr int U = 8, CHUNK = U * T::THREADS * 16;
  static_assert(CHUNK <= T::SMEM, "landing area");
  const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(g.next, g.next_bytes);
  const unsigned n = gridDim.x - g.tiles, me = blockIdx.x - g.tiles;
  const unsigned chunks = g.next_bytes / CHUNK + 1, most = (unsigned)((long)g.K * ((T::BM + T::BN) * 2) / CHUNK);
  const unsigned mine = min((chunks + n - 1 - me) / n, most);
  for (unsigned k = 0; k < mine; k++) {
#pragma unroll
    for (int i = 0; i < U; i++)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(smem + (wave * U + i) * 1024), 16,
                                               (me + k * n) * CHUNK + (unsigned)((wave * U + i) * 1024 + lane * 16), 0,
                                               0, 0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(U) : "memory");
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                // nothing may land after this workgroup's LDS is given away
}

// READ_AHEAD: the instance with workgroups beyond the tiles.  One of its own, because products of a few microseconds feel the
// branch (forward half of hidden 768, 423 tokens, two products: 19.4 us, 19.9 with it in every instance and 136 bytes of
// arguments instead of 112, which a launch copies).
template <int LAY, int EPI, class T, bool READ_AHEAD>
__global__ void __launch_bounds__(T::THREADS, 2) gemm_kernel(GemmArgs g) {
  constexpr int BM = T::BM, BN = T::BN, KE = T::KE, KS = T::KS, STAGES = T::STAGES, TM = T::TM, TN = T::TN;
  constexpr int WM = T::WM, WN = T::WN, NW = T::NW, KW = T::KW;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  constexpr bool A_K = (LAY != LAY_TN);
  constexpr bool B_K = (LAY == LAY_NT);
  constexpr int A_BYTES = T::A_BYTES, B_BYTES = T::B_BYTES;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kw = wave / (T::WGM * T::WGN), place = wave % (T::WGM * T::WGN);
  const int wm = place / T::WGN, wn = place % T::WGN;
  const int q4 = lane >> 4, l16 = lane & 15;

  // tile index: spread consecutive tiles over the 8 XCDs' round-robin dispatch so that each XCD
  // (own L2) works on a compact block of tiles, then walk tiles in groups of 8 tile-rows, or of 4
  // where a launch takes several rounds (8192^3 NT 779 -> 748 us, NN 807 -> 791; 28672 x 8192 x 4096 TN
  // 1606 -> 1554; within one round the two are equal).  Grids that are not a multiple of 8 are spread too
  // (2327 x 9752 x 7168 NT with GELU', 1463 tiles: 447 -> 353 us against consecutive numbering).
  if constexpr (READ_AHEAD)
    if ((int)blockIdx.x >= g.tiles) return read_ahead<T>(g, smem, wave, lane);
  int pid = blockIdx.x;
  const int nwg = g.tiles;
  if constexpr (EPI == EPI_PART) {
    // parts of a tile are consecutive workgroups; each is a product of its own over its share of the reduction
    const int parts = gridDim.x / nwg, part = pid % parts, k0 = part * g.tile_first;
    pid /= parts;
    g.A = static_cast<const bf16*>(g.A) + k0;
    g.B = static_cast<const bf16*>(g.B) + (size_t)k0 * g.ldb;
    g.C = static_cast<float*>(g.C) + (size_t)part * g.M * g.ldc;
    g.K = min(g.K - k0, g.tile_first);
  }
  const int xcd = pid & 7;
  pid = xcd * (nwg >> 3) + min(xcd, nwg & 7) + (pid >> 3);      // XCD's share: nwg / 8, one more for the first nwg % 8
  // tail launch: the walk runs over super-tiles of 2BM x 2BN (the tiles of the large-tile launch
  // that took the whole rounds), starting at g.tile_first; four consecutive workgroups share one
  const int sub = g.tail ? (pid & 3) : 0;
  const int SB = g.tail ? 2 : 1;
  if (g.tail) pid = g.tile_first + (pid >> 2);
  const int tm = (g.M + SB * BM - 1) / (SB * BM), tn = (g.N + SB * BN - 1) / (SB * BN);
  const int group = g.group;
  const int in_group = group * tn;
  const int first_m = (pid / in_group) * group;
  const int gsize = min(tm - first_m, group);
  const int pm = first_m + (pid % in_group) % gsize;
  const int pn = (pid % in_group) / gsize;
  const int m0 = (SB * pm + (sub >> 1)) * BM, n0 = (SB * pn + (sub & 1)) * BN;
  if (m0 >= g.M || n0 >= g.N) return;      // quarter of a ragged super-tile that lies outside C

  const bf16* A = static_cast<const bf16*>(g.A);
  const bf16* B = static_cast<const bf16*>(g.B);
  TileLoader<A_K, BM, KE, NW> la;
  TileLoader<B_K, BN, KE, NW> lb;
  la.init(A, (unsigned)((size_t)(A_K ? g.M : g.K) * g.lda * 2), g.lda, g.K, m0, g.M, wave, lane);
  lb.init(B, (unsigned)((size_t)(B_K ? g.N : g.K) * g.ldb * 2), g.ldb, g.K, n0, g.N, wave, lane);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Epilogue set-up; it sits ahead of the K loop because the first block of what the epilogue
  // reads is requested before the loop ends.
  //   KW == 1: a wavefront finishes its own WM x WN part, 32 rows at a time through a private LDS
  //     region; a row is WN / 4 runs of 4 columns, NJ runs per lane and 32 rows.  Where WN / 4 does not
  //     divide 64 a lane meets NC different column places in turn.
  //   KW > 1: all partial tiles go to LDS and wavefront w finishes rows w BM / NW onwards.
  constexpr int LPR = (KW == 1 ? WN : BN) / 4;         // runs per row
  constexpr int EROWS = KW == 1 ? 32 : BM / NW;        // rows of a block
  constexpr int NJ = EROWS * LPR / 64, NC = (64 % LPR == 0) ? 1 : 3;
  static_assert(EROWS * LPR == NJ * 64 && (NC == 1 || (64 * NC) % LPR == 0), "runs of an epilogue block");
  static_assert(NC == 1 || EPI != EPI_DGELU, "column sums need one column place per lane");
  constexpr int NBLK = KW == 1 ? WM / 32 : 1;
  const int erow0 = m0 + (KW == 1 ? wm * WM : wave * EROWS), ecol0 = n0 + (KW == 1 ? wn * WN : 0);
  auto run_row = [&](int j) { return (64 * j + lane) / LPR; };
  auto run_col = [&](int j) { return 4 * ((64 * (j % NC) + lane) % LPR); };
  float bv[NC][4];
  // Side inputs are fetched one 32-row block ahead, all of a block's loads together.  Written as
  // load - use - store per row, every load sits behind the previous row's store (the compiler
  // cannot know that the two tensors do not overlap) and the epilogue pays a memory latency per
  // row: 52 k cycles instead of 11 k for the residual form.
  constexpr bool AHEAD = NBLK > 1 && !(Side<EPI>::F32 && NC > 1);   // two blocks' worth of registers
  Side<EPI> side[AHEAD ? 2 : 1][NJ];
  auto fetch = [&](int blk, int buf) {
    if (blk == 0) {
#pragma unroll
      for (int c = 0; c < NC; c++) load_bias<EPI>(g, ecol0 + run_col(c), bv[c]);
    }
    if (!Side<EPI>::ANY) return;
#pragma unroll
    for (int j = 0; j < NJ; j++) {
      const int row = erow0 + 32 * blk + run_row(j), col = ecol0 + run_col(j);
      if (row < g.M && col < g.N) side[buf][j].fetch(g, (size_t)row * g.ldc + col);
    }
  };

  // The first block is fetched before the last tiles where the registers allow it (nothing may
  // spill there: a fragment read in flight must not be moved), else after them.  Gradients added to on 256 x 128 tiles, operands
  // not in the caches, us: 4096 x 2048 x 3003 57.5 without, 56.0 with it, 2048 x 4096 x 3003 55.5 / 54.1; on 128 x 128
  // 1024 x 3072 x 4096 31.2 / 30.2.
  constexpr int SIDE_VGPRS = 2 * NJ * (Side<EPI>::F32 ? 2 : Side<EPI>::B16) + 4 * NC;
  constexpr bool EARLY = SIDE_VGPRS <= (TM * TN >= 32 ? 8 : TM * TN >= 24 ? 24 : 40);
  char* sa = smem;                       // A[STAGES]
  char* sb = smem + STAGES * A_BYTES;    // B[STAGES]
  const int nk = (g.K + KE - 1) / KE;
  // Fragments of a sub-step are requested during the one before it.  B fragments, which every row of
  // products uses, alternate between two sets of registers; the A fragment of a row is requested
  // into its own registers once the row's products are issued.
  Frag fa[TM], fb[2][TN];
  auto request_a = [&](const char* ta, int ks, int mi) {
    if (A_K) fa[mi].full = frag_k<KE>(ta, wm * WM + mi * 16 + l16, kw * KS + ks, q4);
    else     frag_mn_issue<BM>(ta, wm * WM + mi * 16, kw * KS + ks, lane, fa[mi]);
  };
  auto request_b = [&](const char* tb, int ks, int buf, int ni) {
    if (B_K) fb[buf][ni].full = frag_k<KE>(tb, wn * WN + ni * 16 + l16, kw * KS + ks, q4);
    else     frag_mn_issue<BN>(tb, wn * WN + ni * 16, kw * KS + ks, lane, fb[buf][ni]);
  };
  // The loop is written as a fixed sequence of slots: every matrix instruction is followed by its
  // share of the fragment reads and tile loads, and a scheduling barrier on either side keeps the
  // compiler from regrouping them.  Left to itself it gathers a tile's loads and their address
  // arithmetic into one block behind the workgroup barrier, during which both wavefronts of a SIMD
  // leave the matrix pipe idle at the same moment (measured: 2 - 8 % per product).
  //   sub-step before the last: products; B fragments of the next sub-step in its first row, the A
  //                        fragment of each row at the end of the row (an earlier row's at the same time)
  //   last sub-step:       products of row 0; wait for tile kt + 1, workgroup barrier; the other rows'
  //                        products, with the first fragments of tile kt + 1 requested in the same
  //                        pattern, and tile kt + STAGES requested into the stage just retired
  // The last tile requests nothing: a fragment read in flight whose destination nobody uses any
  // more would land in registers that already hold something else.
  constexpr int LA = TileLoader<A_K, BM, KE, NW>::PER, LPT = LA + TileLoader<B_K, BN, KE, NW>::PER;
  constexpr int RA = A_K ? 1 : 2, RB = B_K ? 1 : 2;          // LDS reads per fragment
  static_assert((STAGES - 1) * LPT < 64, "vmcnt immediate");
  enum { INSIDE, CHECKED, LAST };
  int slot = 0;
  auto tile = [&](int kt, auto mode_tag, auto par_tag) __attribute__((always_inline)) {
    constexpr int MODE = decltype(mode_tag)::value, PAR = decltype(par_tag)::value;
    char* ta = sa + slot * A_BYTES;
    char* tb = sb + slot * B_BYTES;
    slot = (STAGES & (STAGES - 1)) == 0 ? (slot + 1) & (STAGES - 1) : (slot == STAGES - 1 ? 0 : slot + 1);
    const char* na = sa + slot * A_BYTES;
    const char* nb = sb + slot * B_BYTES;
    const unsigned offa = la.tile_offset((kt + STAGES) * KE), offb = lb.tile_offset((kt + STAGES) * KE);
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
      const int buf = (PAR + ks) & 1;
      const bool last = ks == KS - 1, hand_over = MODE != LAST && last;
      const bool requests = !last || hand_over;
      const int row0 = hand_over ? 1 : 0;                    // first row that requests
      const char* ra = last ? na : ta;
      const char* rb = last ? nb : tb;
      const int rks = last ? 0 : ks + 1;
      bf16x8 bfr[TN];
#pragma unroll
      for (int mi = 0; mi < TM; mi++) {
        // untracked reads still outstanding that are younger than what this row needs: the A
        // fragments of later rows, and this sub-step's requests so far
        const int newer = (!requests || mi <= row0) ? 0 : TN * RB + mi * RA;
        if (!(hand_over && mi >= 1)) {
          if (!A_K || (!B_K && mi == 0)) lds_wait_most((TM - 1 - mi) * RA + newer);
        } else if (mi == 1) {
          // every LDS read of tile kt by this wavefront has completed; its share of tile kt + 1 has
          // landed when only the younger tiles' requests are outstanding
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((STAGES - 2) * LPT) : "memory");
        }
        if (mi == 0) {
#pragma unroll
          for (int ni = 0; ni < TN; ni++) bfr[ni] = B_K ? fb[buf][ni].full : frag_mn_finish(fb[buf][ni]);
        }
        const bf16x8 af = A_K ? fa[mi].full : frag_mn_finish(fa[mi]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ni = 0; ni < TN; ni++) {
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[ni], af, acc[mi][ni], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (requests && mi == row0) request_b(rb, rks, buf ^ 1, ni);
          if (requests && mi >= row0 && ni == TN - 1) {
            if (mi == row0) {
#pragma unroll
              for (int m = 0; m < row0; m++) request_a(ra, rks, m);
            }
            request_a(ra, rks, mi);
          }
          if (hand_over && mi >= 1) {
            constexpr int SL = (TM - 1) * TN;
            const int sl = (mi - 1) * TN + ni;
#pragma unroll
            for (int i = sl * LPT / SL; i < (sl + 1) * LPT / SL; i++) {
              if (MODE == INSIDE) {
                if (i < LA) la.issue_inside(ta, offa, wave, i);
                else lb.issue_inside(tb, offb, wave, i - LA);
              } else {
                // a ragged last tile, or nothing at all beyond K (every lane out of range: zeros, no
                // memory traffic; the count of loads in flight stays the same)
                if (i < LA) la.issue_one(ta, (kt + STAGES) * KE, wave, i);
                else lb.issue_one(tb, (kt + STAGES) * KE, wave, i - LA);
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
#define GX_TILE(KT, MODE, PAR) tile(KT, std::integral_constant<int, MODE>(), std::integral_constant<int, PAR>())
#pragma unroll
  for (int t = 0; t < STAGES; t++) {
    la.issue(sa + t * A_BYTES, t * KE, wave);
    lb.issue(sb + t * B_BYTES, t * KE, wave);
  }
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((STAGES - 1) * LPT) : "memory");   // tile 0 is there
#pragma unroll
  for (int ni = 0; ni < TN; ni++) request_b(sb, 0, 0, ni);
#pragma unroll
  for (int mi = 0; mi < TM; mi++) request_a(sa, 0, mi);
  const int ninside = max(0, g.K / KE - STAGES);   // tiles kt whose prefetch target kt + STAGES lies wholly inside K
  int kt = 0;
  if constexpr (KS == 2) {
    for (; kt < ninside; kt++) GX_TILE(kt, INSIDE, 0);
    if (EARLY) fetch(0, 0);
    for (; kt < nk - 1; kt++) GX_TILE(kt, CHECKED, 0);
    GX_TILE(nk - 1, LAST, 0);
  } else {                                         // one sub-step per tile: the B registers alternate by tile
    for (; kt + 1 < ninside; kt += 2) {
      GX_TILE(kt, INSIDE, 0);
      GX_TILE(kt + 1, INSIDE, 1);
    }
    if (EARLY) fetch(0, 0);
    for (; kt + 2 < nk; kt += 2) {
      GX_TILE(kt, CHECKED, 0);
      GX_TILE(kt + 1, CHECKED, 1);
    }
    GX_TILE(kt, CHECKED, 0);
    if (kt + 1 < nk) {
      GX_TILE(kt + 1, LAST, 1);
    } else {                                       // nothing left: see the reads of the next stage's zeros in
      lds_wait_all();
#pragma unroll
      for (int mi = 0; mi < TM; mi++)
        if (!A_K) lds_pin(fa[mi].lo), lds_pin(fa[mi].hi);
#pragma unroll
      for (int ni = 0; ni < TN; ni++)
        if (!B_K) lds_pin(fb[1][ni].lo), lds_pin(fb[1][ni].hi);
    }
  }
#undef GX_TILE
  if (!EARLY) fetch(0, 0);
  // the zero-fill requests beyond K must have landed, and every wavefront must be done with the
  // tiles, before the staging below reuses LDS
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  // epilogue.  The MFMAs were issued with the B fragment as the row operand, so accumulator
  // register v of lane l holds C[m = l % 16][n = 4 * (l / 16) + v] of its block: a run of 4
  // consecutive columns.  Blocks pass through LDS (row stride of 4 floats more than the columns
  // keeps the 16 B writes conflict-free) and are read back so that consecutive lanes cover a row:
  // every global access of the epilogue (C, residual, pre-activation, second output) is a 16 B
  // or 8 B vector in fully used lines.
  // EPI_DGELU may also leave partial column sums of what it stores (stage 1 of the bias gradient of
  // the product that made z), one row of sums per block of 64 rows of C, by one writer each.
  float cs[4] = {0.f, 0.f, 0.f, 0.f};
  if constexpr (KW == 1) {
    static_assert(EPI != EPI_DGELU || WM % 64 == 0, "column-sum blocks of 64 rows");
    constexpr int EPAD = WN + 4;
    float* stage = reinterpret_cast<float*>(smem + wave * (32 * EPAD * 4));
#pragma unroll
    for (int mi = 0; mi < NBLK; mi++) {
      if (AHEAD && mi + 1 < NBLK) fetch(mi + 1, (mi + 1) & 1);
      if (!AHEAD && mi > 0) fetch(mi, 0);
#pragma unroll
      for (int h = 0; h < 2; h++)
#pragma unroll
        for (int ni = 0; ni < TN; ni++)
          *reinterpret_cast<f32x4*>(stage + (16 * h + l16) * EPAD + ni * 16 + 4 * q4) = acc[2 * mi + h][ni];
#pragma unroll
      for (int j = 0; j < NJ; j++) {
        const f32x4 xv = *reinterpret_cast<const f32x4*>(stage + run_row(j) * EPAD + run_col(j));
        const int row = erow0 + 32 * mi + run_row(j), col = ecol0 + run_col(j);
        if (row >= g.M || col >= g.N) continue;            // N is a multiple of 4: whole run in or out
        finish_run<LAY, EPI>(g, (size_t)row * g.ldc + col, xv, bv[j % NC], side[AHEAD ? mi & 1 : 0][j], cs);
      }
      if (EPI == EPI_DGELU && (mi & 1) && g.colpart) {
        // each lane has added its rows of the block; lanes that share columns combine by shuffles
#pragma unroll
        for (int e = 0; e < 4; e++) {
#pragma unroll
          for (int o = LPR; o < 64; o <<= 1) cs[e] += __shfl_xor(cs[e], o, 64);
        }
        const int row0 = erow0 + (mi - 1) * 32, col = ecol0 + run_col(0);      // first row of this block of 64
        if (lane < LPR && row0 < g.M && col < g.N)
          *reinterpret_cast<f32x4*>(g.colpart + (size_t)(row0 >> 6) * g.N + col) = f32x4{cs[0], cs[1], cs[2], cs[3]};
#pragma unroll
        for (int e = 0; e < 4; e++) cs[e] = 0.f;
      }
    }
  } else {
    constexpr int PADN = T::PADN;
    float* park = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int mi = 0; mi < TM; mi++)
#pragma unroll
      for (int ni = 0; ni < TN; ni++)
        *reinterpret_cast<f32x4*>(park + (kw * BM + wm * WM + mi * 16 + l16) * PADN + wn * WN + ni * 16 + 4 * q4) =
            acc[mi][ni];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; j++) {
      const int r = wave * EROWS + run_row(j);
      f32x4 xv = *reinterpret_cast<const f32x4*>(park + r * PADN + run_col(j));
#pragma unroll
      for (int k = 1; k < KW; k++) {
        const f32x4 p = *reinterpret_cast<const f32x4*>(park + (k * BM + r) * PADN + run_col(j));
#pragma unroll
        for (int e = 0; e < 4; e++) xv[e] += p[e];
      }
      const int row = m0 + r, col = ecol0 + run_col(j);
      if (row >= g.M || col >= g.N) continue;
      finish_run<LAY, EPI>(g, (size_t)row * g.ldc + col, xv, bv[j % NC], side[0][j], cs);
    }
    if (EPI == EPI_DGELU && g.colpart) {
      constexpr int WPB = 64 / EROWS;                                          // wavefronts per block of 64 rows
      float* red = park + KW * BM * PADN;                                      // [NW][BN]
#pragma unroll
      for (int e = 0; e < 4; e++) {
#pragma unroll
        for (int o = LPR; o < 64; o <<= 1) cs[e] += __shfl_xor(cs[e], o, 64);
      }
      if (lane < LPR) *reinterpret_cast<f32x4*>(red + wave * BN + run_col(0)) = f32x4{cs[0], cs[1], cs[2], cs[3]};
      __syncthreads();
      for (int i = threadIdx.x; i < BM / 64 * BN; i += T::THREADS) {
        const int blk = i / BN, c = i % BN;
        float t = red[blk * WPB * BN + c];
#pragma unroll
        for (int w = 1; w < WPB; w++) t += red[(blk * WPB + w) * BN + c];
        if (m0 + 64 * blk < g.M && n0 + c < g.N) g.colpart[(size_t)((m0 >> 6) + blk) * g.N + n0 + c] = t;
      }
    }
  }
}

constexpr int ROUND = 256;                     // workgroups at work at once: one per compute unit
// How many workgroups read ahead.  They cost the product bandwidth, and other streams the compute units that they hold, so:
//  - the weights of the whole call exceed the memory-side cache; smaller ones may still be in it from the call before (one
//    layer again and again: hidden 2048 64 tokens 79.6 us with nothing read ahead, 86.6 with, hidden 4096 degree 4 74.3 / 81.1,
//    hidden 8192 degree 8 105.8 / 115.7; other layers in between 106.6 / 94.2, 100.4 / 92.4 and 152.8 / 145.3 are given up).
//  - this product's weights and the next one's fit the cache together, or what is read ahead is gone by the time it is used
//    (hidden 8192, degree 2: 512 tokens 428 / 442, 1024 701 / 714; hidden 5120, degree 1: 200 tokens 328 / 340).
//  - more than 64 tokens and up to 256: fewer are bound by the bandwidth itself (1 token of hidden 4096 4.5 % slower, a stage
//    of two blocks and two streams, 64 tokens, hidden 8192 degree 4, 2 %); more mostly by operands (hidden 8192, degree 4: 400
//    tokens 238 / 253; hidden 6144, degree 2: 312 / 323; hidden 5120, degree 2: 512 tokens 280 / 254 are given up).
//  - beyond 128 tokens a quarter of the compute units at least has no tile (hidden 5120, degree 1: 129 tokens 2.3 % slower with
//    fewer, that stage with 256 tokens 0.7 %); up to 128 a few are enough (hidden 8192, degree 4: 100 tokens 1.7 to 3 % faster).
// Forward passes within that, other layers in between, without / with, us: hidden 5120, degree 2: 72 tokens 163 / 147, 128
// 183 / 161, 256 226 / 195; hidden 4096: 128 205 / 197; hidden 8192, degree 4: 160 214 / 203; hidden 6144, degree 2: 256 271 /
// 262; hidden 3584: 100 178 / 164.  What still loses: one layer's 300 to 400 MB again and again, which the cache half holds
// (hidden 3584, 72 tokens 151 / 156, 160 tokens 168 / 169; forward and backward of hidden 4096, 100 tokens 553 / 573, with other
// layers in between 587 / 572), and a stage of two blocks on two streams at one size of eleven (hidden 8192, degree 4, 128 tokens
// 1.3 %; the others within 0.6 %).
constexpr long CACHE = 256L << 20;
constexpr int READ_AHEAD_TILE = 128 * 128;     // so few tokens do not take larger ones in calls of so many weights
template <class T>
int read_ahead_workgroups(int M, int tiles) {
  if (T::BM * T::BN > READ_AHEAD_TILE || M <= 64 || M > 256) return 0;
  return tiles <= (M <= 128 ? ROUND : ROUND / 4 * 3) ? ROUND - tiles : 0;
}

template <int LAY, int EPI, class T, bool READ_AHEAD>
hipError_t start(const GemmArgs& g, hipStream_t s, int grid) {
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_kernel<LAY, EPI, T, READ_AHEAD>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, T::SMEM);
    if (e != hipSuccess) return e;
    configured = true;
  }
  hipLaunchKernelGGL((gemm_kernel<LAY, EPI, T, READ_AHEAD>), dim3(grid), dim3(T::THREADS), T::SMEM, s, g);
  return hipGetLastError();
}
template <int LAY, int EPI, class T>
hipError_t launch_tile(const GemmArgs& g, hipStream_t s, int grid) {
  GemmArgs a = g;
  if (!a.tail) a.group = grid > 256 ? 4 : 8;
  a.tiles = grid;
  if constexpr (LAY == LAY_NN && T::BM * T::BN <= READ_AHEAD_TILE)
    if (a.next && !a.tail)
      if (const int more = read_ahead_workgroups<T>(a.M, grid)) return start<LAY, EPI, T, true>(a, s, grid + more);
  return start<LAY, EPI, T, false>(a, s, grid);
}
template <int LAY, int EPI, class T>
hipError_t launch_whole(const GemmArgs& g, hipStream_t s) {
  return launch_tile<LAY, EPI, T>(g, s, cdiv(g.M, T::BM) * cdiv(g.N, T::BN));
}

// The tiles.  `fixed` and `per_k` price one round of a tile (at most 256 workgroups, one per compute
// unit): microseconds that do not depend on K, and per 1024 reduction steps.
struct Large : Tile<256, 256, 2, 4, 1, 64, 2> { static constexpr float fixed = 9.0f, per_k = 24.8f; };
struct Wide : Tile<256, 192, 4, 2, 1, 64, 2> { static constexpr float fixed = 8.7f, per_k = 18.7f; };
struct Tall : Tile<192, 256, 2, 4, 1, 64, 2> { static constexpr float fixed = 8.7f, per_k = 18.7f; };
struct Half : Tile<256, 128, 4, 2, 1, 64, 3> { static constexpr float fixed = 6.5f, per_k = 14.5f; };
struct Small : Tile<128, 128, 2, 2, 2, 64, 4> { static constexpr float fixed = 5.1f, per_k = 7.2f; };
struct Flat : Tile<64, 128, 1, 2, 4, 128, 3> { static constexpr float fixed = 4.8f, per_k = 4.7f; };
struct Tiny : Tile<64, 64, 1, 1, 4, 128, 4> { static constexpr float fixed = 3.8f, per_k = 3.4f; };

// Which tile: the one whose rounds are cheapest.  A product's time is the number of rounds of 256
// workgroups it takes times the price of a round, whether the last round is full or not, so the larger
// tiles (less traffic per product) win where they fill the chip and the smaller ones where a larger
// one would leave compute units without work.  The prices are fits to products of 1 to 4096 tiles
// and K 768 to 10240; measured (us, the same operands again and again), chosen tile first:
//   NN 4096 x 3072 x 4096   Wide 79.0 (256 tiles)  Large 86.5 (192)  Small 90.4   Half 103
//   NT 2048 x 5120 x 10240  Tall 164 (220)         Wide 161 (216)    Large 177    Small 190
//   NN 3003 x 4096 x 2048   Tall 42.5 (256)        Large 44.4 (192)  Wide 73.8    Half 55.3
//   NT 2048 x 2560 x 5120   Half 55.2 (160)        Small 66.5 (320)  Flat 72.7    Large 92.0
//   NT 4096 x 1024 x 4096   Small 29.9 (256)       Flat 40.4         Half 43.9    Large 71.2
//   TN 512 x 4096 x 8192    Flat 40.7 (256)        Small 49.7 (128)  Tiny 59.9    Large 150
//   TN 1024 x 1024 x 4096   Tiny 17.1 (256)        Flat 21.6 (128)   Small 27.1   Large 78.5
//   NN 128 x 7680 x 5120    Tiny 22.4 (240)        Flat 27.9 (120)   Small 35.2   Large 85.0
// Beyond whole rounds of large tiles, the remaining ones can also be cut into 128 x 128 tiles in a second
// launch (TAIL is what that launch costs): NN 2048 x 10240 x 5120, 320 large tiles, 157 against 175
// (Tall), 182 (Small) and 203 (Large alone).
constexpr float TAIL = 3.0f;
template <class T>
float price(long tiles, int K) {
  return (float)((tiles + ROUND - 1) / ROUND) * (T::fixed + T::per_k * (float)K * (1.0f / 1024));
}
// Another tile than the large one has to be 3 % cheaper: where it only evens out, the large one leaves more
// to the product of the other stream that shares the chip (two products of 5466 x 6528 x 19584 and its
// transpose, equal alone, 1.5 % slower together with 256 x 192 tiles).  192 x 256 before 256 x 192: the same
// price, but its rows are read back from LDS without a remainder.  Where both take the same number of rounds
// 256 x 192 took 1.3 % longer on the mean of 70 products, whichever has fewer tiles (6618 x 1216 x 16952 NT, 175
// and 182 tiles, 421 us against 439; 2048 x 5120 x 10240 NT, 220 and 216 tiles, 215 against 218, operands not
// in the caches; a pipeline stage of hidden 5120 is 0.3 % faster than with the fewer tiles first).
enum Pick { PICK_LARGE, PICK_WIDE, PICK_TALL, PICK_HALF, PICK_SMALL, PICK_FLAT, PICK_TINY, PICK_LARGE_TAIL };
Pick pick(int M, int N, int K, bool column_sums) {
  const long big = (long)cdiv(M, 256) * cdiv(N, 256), rem = big % ROUND;
  Pick best = PICK_LARGE;
  float least = price<Large>(big, K);
  if (big > ROUND && rem) {
    const float with_tail = price<Large>(big - rem, K) + price<Small>(4 * rem, K) + TAIL;
    if (with_tail < least) least = with_tail, best = PICK_LARGE_TAIL;
  }
  least *= 0.97f;
  auto consider = [&](Pick t, int bm, int bn, auto tile) {
    const float p = price<decltype(tile)>((long)cdiv(M, bm) * cdiv(N, bn), K);
    if (p < least) least = p, best = t;
  };
  // the 192-wide tiles have no column sums: their wavefronts' parts are not whole blocks of 64 rows
  if (!column_sums) {
    consider(PICK_TALL, Tall::BM, Tall::BN, Tall());
    consider(PICK_WIDE, Wide::BM, Wide::BN, Wide());
  }
  consider(PICK_HALF, Half::BM, Half::BN, Half());
  consider(PICK_SMALL, Small::BM, Small::BN, Small());
  consider(PICK_FLAT, Flat::BM, Flat::BN, Flat());
  consider(PICK_TINY, Tiny::BM, Tiny::BN, Tiny());
  return best;
}
template <int LAY, int EPI>
hipError_t launch(const GemmArgs& g, hipStream_t s) {
  switch (pick(g.M, g.N, g.K, EPI == EPI_DGELU)) {
    case PICK_LARGE: return launch_whole<LAY, EPI, Large>(g, s);
    case PICK_WIDE:
      if constexpr (EPI != EPI_DGELU) return launch_whole<LAY, EPI, Wide>(g, s);
      break;
    case PICK_TALL:
      if constexpr (EPI != EPI_DGELU) return launch_whole<LAY, EPI, Tall>(g, s);
      break;
    case PICK_HALF: return launch_whole<LAY, EPI, Half>(g, s);
    case PICK_SMALL: return launch_whole<LAY, EPI, Small>(g, s);
    case PICK_FLAT: return launch_whole<LAY, EPI, Flat>(g, s);
    case PICK_TINY: return launch_whole<LAY, EPI, Tiny>(g, s);
    case PICK_LARGE_TAIL: {
      const long big = (long)cdiv(g.M, 256) * cdiv(g.N, 256), rem = big % ROUND;
      hipError_t e = launch_tile<LAY, EPI, Large>(g, s, (int)(big - rem));
      if (e != hipSuccess) return e;
      GemmArgs t = g;
      t.tail = 1;
      t.group = big - rem > 256 ? 4 : 8;             // the walk of the launch above
      t.tile_first = (int)(big - rem);
      return launch_tile<LAY, EPI, Small>(t, s, (int)(4 * rem));
    }
  }
  return hipErrorInvalidValue;
}

// Few tokens: the reduction is cut into parts, so that every compute unit streams weights, and a second launch adds the parts in
// order and does the epilogue.  A unit takes 40 to 50 bytes per ns of weights and operands from memory, whatever the tile (rows of
// weights lie tens of KB apart; reading 128 columns instead of 64 and deeper rings change little), so what counts is how little
// each has to take: wide tiles on as many units as there are.  Without the second launch, weights not in the caches, us,
// one launch of the best tile / parts of 128 x 128 tiles: 128 x 10240 x 5120 45 / 27 (3 parts), 128 x 5120 x 10240 63 / 28 (6),
// 128 x 7680 x 5120 33 / 22 (4); the second takes 4 to 5.
template <int EPI>
__global__ void __launch_bounds__(256) split_finish_kernel(GemmArgs g, const float* __restrict__ part, int parts) {
  const long run = (long)blockIdx.x * 256 + threadIdx.x, per_row = g.N / 4;
  if (run >= g.M * per_row) return;
  const int row = (int)(run / per_row), col = 4 * (int)(run % per_row);
  const size_t idx = (size_t)row * g.ldc + col, stride = (size_t)g.M * g.ldc;
  Side<EPI> side;
  if (Side<EPI>::ANY) side.fetch(g, idx);
  float bv[4], cs[4];
  load_bias<EPI>(g, col, bv);
  f32x4 x = *reinterpret_cast<const f32x4*>(part + idx);
#pragma unroll 4
  for (int k = 1; k < parts; k++) {
    const f32x4 p = *reinterpret_cast<const f32x4*>(part + k * stride + idx);
    x = f32x4{x[0] + p[0], x[1] + p[1], x[2] + p[2], x[3] + p[3]};
  }
  finish_run<LAY_NN, EPI>(g, idx, x, bv, side, cs);
}
// steps of a part: whole stages of every tile used; parts that are at least SPLIT_K long
constexpr int SPLIT_UNIT = 128, SPLIT_K = 256, SPLIT_TOKENS = 256, SPLIT_N = 128;
int split_steps(int N, int K) {
  const int most = ROUND / cdiv(N, SPLIT_N);
  if (most < 2) return K;
  const int steps = cdiv(cdiv(K, most), SPLIT_UNIT) * SPLIT_UNIT;
  return steps < SPLIT_K ? SPLIT_K : steps;
}
template <class T>
hipError_t launch_parts(const GemmArgs& g, int parts, hipStream_t s) {
  GemmArgs a = g;
  a.group = 8;
  a.tiles = cdiv(a.M, T::BM) * cdiv(a.N, T::BN);
  return start<LAY_NN, EPI_PART, T, false>(a, s, a.tiles * parts);
}

// The combinations that the layer driver asks for.
template <int LAY>
hipError_t dispatch_epi(Epilogue epi, const GemmArgs& g, hipStream_t s) {
  if constexpr (LAY == LAY_NN) {
    if (epi == EPI_BIAS) return launch<LAY, EPI_BIAS>(g, s);
    if (epi == EPI_RESID) return launch<LAY, EPI_RESID>(g, s);
    if (epi == EPI_GELU) return launch<LAY, EPI_GELU>(g, s);
  } else if constexpr (LAY == LAY_NT) {
    if (epi == EPI_STORE) return launch<LAY, EPI_STORE>(g, s);
    if (epi == EPI_DGELU) return launch<LAY, EPI_DGELU>(g, s);
  } else {
    if (epi == EPI_F32) return launch<LAY, EPI_F32>(g, s);
    if (epi == EPI_F32_ACC) return launch<LAY, EPI_F32_ACC>(g, s);
    if (epi == EPI_STORE) return launch<LAY, EPI_STORE>(g, s);
    if (epi == EPI_RESID) return launch<LAY, EPI_RESID>(g, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace

extern "C" int gx_bf16_tile(int M, int N, int K, int column_sums) { return pick(M, N, K, column_sums != 0); }

bool read_ahead_pays(long own_bytes, long next_bytes, long call_bytes) {
  return call_bytes > CACHE && own_bytes + next_bytes <= CACHE / 8 * 7;
}

extern "C" int gx_bf16_read_ahead(int M, int N, int K, long next_bytes, long call_bytes) {
  if (!read_ahead_pays((long)N * K * 2, next_bytes, call_bytes)) return 0;
  auto of = [&](auto tile) {
    using T = decltype(tile);
    return read_ahead_workgroups<T>(M, cdiv(M, T::BM) * cdiv(N, T::BN));
  };
  switch (pick(M, N, K, false)) {
    case PICK_LARGE: return of(Large());
    case PICK_WIDE: return of(Wide());
    case PICK_TALL: return of(Tall());
    case PICK_HALF: return of(Half());
    case PICK_SMALL: return of(Small());
    case PICK_FLAT: return of(Flat());
    case PICK_TINY: return of(Tiny());
    case PICK_LARGE_TAIL: break;                 // more than a round of tiles
  }
  return 0;
}

namespace {
bool args_ok(Layout lay, const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
  // 16-byte chunks along each operand's contiguous index; 31-bit byte offsets in buffer loads
  const long a_rows = (lay == LAY_TN) ? g.K : g.M, b_rows = (lay == LAY_NT) ? g.N : g.K;
  if ((g.lda & 7) || (g.ldb & 7)) return false;
  if (lay != LAY_TN && (g.K & 7)) return false;
  if (lay == LAY_TN && (g.M & 7)) return false;
  if (lay != LAY_NT && (g.N & 7)) return false;
  // the epilogue moves runs of 4 columns as one vector
  if ((g.N & 3) || (g.ldc & 3) || (reinterpret_cast<uintptr_t>(g.C) & 15)) return false;
  if (a_rows * g.lda * 2 >= (1L << 31) || b_rows * g.ldb * 2 >= (1L << 31)) return false;
  return !((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B)) & 15);
}
}  // namespace

hipError_t gemm_bf16(Layout lay, Epilogue epi, const GemmArgs& args, hipStream_t s) {
  GemmArgs g = args;
  g.tail = g.tile_first = g.group = g.tiles = 0;       // the launcher's own fields
  if (!args_ok(lay, g)) return hipErrorInvalidValue;
  switch (lay) {
    case LAY_NN: return dispatch_epi<LAY_NN>(epi, g, s);
    case LAY_NT: return dispatch_epi<LAY_NT>(epi, g, s);
    case LAY_TN: return dispatch_epi<LAY_TN>(epi, g, s);
  }
  return hipErrorInvalidValue;
}

extern "C" int gx_bf16_split(int M, int N, int K) {
  if (M > SPLIT_TOKENS) return 1;
  return cdiv(K, split_steps(N, K));
}
size_t gemm_bf16_split_bytes(int M, int N, int K) {
  const int parts = gx_bf16_split(M, N, K);
  return parts > 1 ? (size_t)parts * M * N * 4 : 0;
}

hipError_t gemm_bf16_split(Epilogue epi, const GemmArgs& args, float* scratch, hipStream_t s) {
  const int parts = gx_bf16_split(args.M, args.N, args.K);
  if (parts < 2 || !scratch || !args_ok(LAY_NN, args) || args.ldc != args.N) return hipErrorInvalidValue;
  GemmArgs p = args;
  p.C = scratch;
  p.bias = p.resid = p.next = nullptr;
  p.aux = nullptr;
  p.tail = 0;
  p.tile_first = split_steps(args.N, args.K);
  hipError_t e = p.M <= 64 ? launch_parts<Flat>(p, parts, s) : p.M <= 128 ? launch_parts<Small>(p, parts, s)
                                                                        : launch_parts<Half>(p, parts, s);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)cdiv((long)args.M * (args.N / 4), 256L));
  switch (epi) {
    case EPI_BIAS: hipLaunchKernelGGL(split_finish_kernel<EPI_BIAS>, grid, dim3(256), 0, s, args, scratch, parts); break;
    case EPI_RESID: hipLaunchKernelGGL(split_finish_kernel<EPI_RESID>, grid, dim3(256), 0, s, args, scratch, parts); break;
    case EPI_GELU: hipLaunchKernelGGL(split_finish_kernel<EPI_GELU>, grid, dim3(256), 0, s, args, scratch, parts); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gx
