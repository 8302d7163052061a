// fp32 GEMM for the full-precision configuration on v_mfma_f32_32x32x2_f32 (full fp32 products and
// sums, twice the rate of the vector units' multiply-add), with the layouts and epilogues of the
// bf16 family.
//
// A workgroup owns a BM x BM tile of C as 32 x 32 blocks, one per wavefront; KW wavefronts share a
// block by taking KW interleaved shares of the reduction, added in order through LDS at the end.
// Operand tiles of 32 KW reduction steps go from memory straight into LDS through a ring of STAGES
// stages, one barrier per stage.  A matrix instruction holds the pipe for 64 cycles and needs one
// or two LDS reads, so the matrix pipe is the bound as soon as every SIMD has a wavefront with data:
// the tile is chosen to give the chip enough wavefronts, not to save LDS traffic.  Against a 64 x 64
// tile of scalar multiply-adds: 256 x 256 x 1024 60 -> 9 us, 1024 x 1024 x 4096 (NT) 240 -> 70 us.
#include "gx_kernels.h"
#include <type_traits>

namespace gx {
namespace {

constexpr unsigned OOB = 0x80000000u;    // beyond num_records: the load writes zeros

// Loads of one operand's share of a stage: KW sub-tiles of 32 reduction steps.  K-major (reduction
// index contiguous in memory): [BM rows][32 k], 16 B chunk c of row r at c ^ ((r >> 1) & 7), so that
// the 16 rows of one LDS read pass fall in distinct banks.  MN-major: [32 k][BM columns].
template <bool KMAJOR, int BM, int KW, int NW>
struct TileLoader {
  static constexpr int PER = BM * 32 * KW * 4 / 1024 / NW;     // 1 KB instructions per wavefront
  unsigned base[PER];      // element offset without the stage's reduction index, or OOB
  int kc[PER];             // reduction index of the lane's chunk within the stage
  __amdgpu_buffer_rsrc_t rsrc;
  int ld, K;
  GX_DEVINL void init(const float* p, size_t bytes, int ld_, int K_, int origin, int extent, int wave, int lane) {
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (unsigned)bytes, 0x00020000);
    ld = ld_;
    K = K_;
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const int q = (wave * PER + i) * 64 + lane, per_sub = BM * 8;     // 16 B slots; BM * 8 in a sub-tile
      const int sub = q / per_sub, s = q % per_sub;
      if (KMAJOR) {
        const int r = s >> 3, c = (s & 7) ^ ((r >> 1) & 7);
        kc[i] = 32 * sub + 4 * c;
        base[i] = (origin + r < extent) ? (unsigned)((origin + r) * ld + kc[i]) : OOB;
      } else {
        const int k = s / (BM / 4), c = s % (BM / 4);
        kc[i] = 32 * sub + k;
        base[i] = (origin + 4 * c < extent) ? (unsigned)(kc[i] * ld + origin + 4 * c) : OOB;
      }
    }
  }
  GX_DEVINL void issue(char* dst, int k0, int wave) const {
#pragma unroll
    for (int i = 0; i < PER; i++) {
      const unsigned off =
          (base[i] != OOB && k0 + kc[i] < K) ? (base[i] + (unsigned)(KMAJOR ? k0 : k0 * ld)) * 4u : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(dst + (wave * PER + i) * 1024), 16, off, 0, 0, 0);
    }
  }
};

// This lane's operand of the four 32x32x2 products that cover reduction steps 8 c .. 8 c + 7: step e
// pairs 8 c + e (lower half of the wavefront) with 8 c + 4 + e (upper half).
template <bool KMAJOR, int BM>
GX_DEVINL f32x4 frag(const char* sub, int row, int c, int g) {
  if (KMAJOR) return *reinterpret_cast<const f32x4*>(sub + row * 128 + (((2 * c + g) ^ ((row >> 1) & 7)) << 4));
  const float* p = reinterpret_cast<const float*>(sub) + (8 * c + 4 * g) * BM + row;
  return f32x4{p[0], p[BM], p[2 * BM], p[3 * BM]};
}

// One tile of one product: workgroup `pid` of the `nwg` that the product has.
// AHEAD: the next stage's fragments are read between the products; else at the start of their own stage (see pick()).
// SUMS (LAY_TN, g.colpart): column sums of B, the bias gradient of the product whose weight gradient this is.  B passes through
// the registers of the first tile-row's wavefronts anyway, so they add it up there, eight stages at a time: no pass over the
// tensor and no partial sums in memory (hidden 256, 256 tokens, forward and backward: two launches fewer, 141 -> 137 us).  It makes
// a product 3 to 4 % slower (2048 x 8192 x 1024 271 -> 278 us, x 2048 533 -> 553), so the others are instances without it; which
// products have it: sums_in_product().
template <int LAY, int EPI, int BM, int KW, int STAGES, bool AHEAD, bool SUMS = false>
GX_DEVINL void tile_of_product(const GemmArgs& g, int pid, int nwg, char* smem) {
  constexpr bool A_K = (LAY != LAY_TN), B_K = (LAY == LAY_NT);
  constexpr int WR = BM / 32, NW = WR * WR * KW, NT = 64 * NW;
  constexpr int SUB = BM * 128, OPER = KW * SUB, STAGE = 2 * OPER;
  constexpr int PADN = BM + 4;
  static_assert(KW * BM * (PADN + 1) * 4 <= STAGES * STAGE, "partial blocks and column sums fit the stages");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kw = wave % KW, wm = (wave / KW) / WR, wn = (wave / KW) % WR;
  const int grp = lane >> 5, l32 = lane & 31;

  // consecutive tiles spread over the 8 XCDs' round-robin dispatch, 8 tile-rows at a time
  if ((nwg & 7) == 0) pid = (pid & 7) * (nwg >> 3) + (pid >> 3);
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BM - 1) / BM;
  const int first = (pid / (8 * tn)) * 8, gsize = min(tm - first, 8);
  const int m0 = (first + (pid % (8 * tn)) % gsize) * BM, n0 = ((pid % (8 * tn)) / gsize) * BM;

  TileLoader<A_K, BM, KW, NW> la;
  TileLoader<B_K, BM, KW, NW> lb;
  la.init(static_cast<const float*>(g.A), (size_t)(A_K ? g.M : g.K) * g.lda * 4, g.lda, g.K, m0, g.M, wave, lane);
  lb.init(static_cast<const float*>(g.B), (size_t)(B_K ? g.N : g.K) * g.ldb * 4, g.ldb, g.K, n0, g.N, wave, lane);
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; v++) acc[v] = 0.f;

  constexpr int LPT = la.PER + lb.PER;                  // loads per wavefront and stage
  static_assert((STAGES - 1) * LPT < 64, "vmcnt immediate");
  const int nk = (g.K + 32 * KW - 1) / (32 * KW);
  auto request = [&](int t, int slot) __attribute__((always_inline)) {   // stages beyond K: out of range, zeros, no traffic
    la.issue(smem + slot * STAGE, t * 32 * KW, wave);
    lb.issue(smem + slot * STAGE + OPER, t * 32 * KW, wave);
  };
  f32x4 fa[AHEAD ? 2 : 1][4], fb[AHEAD ? 2 : 1][4];
  auto read = [&](int slot, int set, int c) __attribute__((always_inline)) {
    const char* ta = smem + slot * STAGE + kw * SUB;
    fa[set][c] = frag<A_K, BM>(ta, 32 * wm + l32, c, grp);
    fb[set][c] = frag<B_K, BM>(ta + OPER, 32 * wn + l32, c, grp);
  };
  const bool sums = SUMS && g.colpart && m0 == 0, my_sums = sums && wm == 0;    // wavefront-uniform
  float cs = 0.f, cs_before = 0.f;                       // of column n0 + 32 wn + l32, this wavefront's share of the rows
  auto products = [&](int set, int c) __attribute__((always_inline)) {
    if (SUMS && my_sums) cs += (fb[set][c][0] + fb[set][c][1]) + (fb[set][c][2] + fb[set][c][3]);
#pragma unroll
    for (int e = 0; e < 4; e++)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[set][c][e], fb[set][c][e], acc, 0, 0, 0);
  };
  auto sums_of_stage = [&](int kt) __attribute__((always_inline)) {
    if (SUMS && (kt & 7) == 7) {
      cs_before += cs;
      cs = 0.f;
    }
  };
  // (__syncthreads() would wait for the younger requests too)
  int slot = 0;
  if constexpr (AHEAD) {
    // The fragments of stage kt + 1 are read between the products of stage kt, so that no product waits for LDS;
    // a stage's slot is free for stage kt + STAGES as soon as every wavefront holds its fragments.
#pragma unroll
    for (int t = 0; t < STAGES; t++) request(t, t);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * LPT) : "memory");
#pragma unroll
    for (int c = 0; c < 4; c++) read(0, 0, c);
    auto stage = [&](int kt, auto set_tag) __attribute__((always_inline)) {
      constexpr int SET = decltype(set_tag)::value;
#pragma unroll
      for (int c = 0; c < 4; c++) {
        if (c == 1) {
          // this wavefront holds stage kt, and its share of stage kt + 1 has landed
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((STAGES - 2) * LPT) : "memory");
          request(kt + STAGES, slot);
          slot = (slot == STAGES - 1) ? 0 : slot + 1;
          read(slot, SET ^ 1, 0);
        }
        if (c > 0) read(slot, SET ^ 1, c);
        __builtin_amdgcn_sched_barrier(0);
        products(SET, c);
        __builtin_amdgcn_sched_barrier(0);
      }
      sums_of_stage(kt);
    };
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
      stage(kt, std::integral_constant<int, 0>());
      stage(kt + 1, std::integral_constant<int, 1>());
    }
    if (kt < nk) stage(kt, std::integral_constant<int, 0>());
  } else {
    // Two stages are requested at once, of more all but the last; stage kt's slot takes stage kt + STAGES when all wavefronts
    // have finished with it.
    constexpr int UP = STAGES == 2 ? 2 : STAGES - 1;
#pragma unroll
    for (int t = 0; t < UP; t++) request(t, t);
    for (int kt = 0; kt < nk; kt++) {
      if (UP == STAGES && kt == 0) {
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((STAGES - 1) * LPT) : "memory");
      } else {
        // stage kt has landed (STAGES - 2 younger ones may be in flight) and every wavefront has finished
        // with stage kt - 1, whose slot takes the next request
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((STAGES - 2) * LPT) : "memory");
        request(kt + STAGES - 1, slot == 0 ? STAGES - 1 : slot - 1);
      }
#pragma unroll
      for (int c = 0; c < 4; c++) read(slot, 0, c);
#pragma unroll
      for (int c = 0; c < 4; c++) products(0, c);
      sums_of_stage(kt);
      slot = (slot == STAGES - 1) ? 0 : slot + 1;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // requests beyond K must not land in what follows
  __syncthreads();

  // blocks through LDS: [kw][BM rows][BM columns + 4], then whole 16 B runs of a row
  float* part = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int v = 0; v < 16; v++)
    part[(kw * BM + 32 * wm + 8 * (v >> 2) + 4 * grp + (v & 3)) * PADN + 32 * wn + l32] = acc[v];
  float* const col_sums = part + KW * BM * PADN;        // [kw][BM columns]
  if (SUMS && my_sums) {
    cs += cs_before;
    cs += __shfl_xor(cs, 32, 64);
    if (grp == 0) col_sums[kw * BM + 32 * wn + l32] = cs;
  }
  __syncthreads();
  if (SUMS && sums && threadIdx.x < BM && n0 + (int)threadIdx.x < g.N) {
    float t = col_sums[threadIdx.x];
#pragma unroll
    for (int k = 1; k < KW; k++) t += col_sums[k * BM + threadIdx.x];
    float* out = g.colpart + n0 + threadIdx.x;
    *out = EPI == EPI_F32_ACC ? *out + t : t;
  }
  const float* bias = static_cast<const float*>(g.bias);
  const float* resid = static_cast<const float*>(g.resid);
  const float* zin = static_cast<const float*>(g.z);
  float* aux = static_cast<float*>(g.aux);
  float* C = static_cast<float*>(g.C);
#pragma unroll
  for (int i = 0; i < BM * BM / 4 / NT; i++) {
    const int s = threadIdx.x + i * NT, r = s / (BM / 4), c = 4 * (s % (BM / 4));
    const int row = m0 + r, col = n0 + c;
    if (row >= g.M || col >= g.N) continue;             // N is a multiple of 4: whole run in or out
    f32x4 x = *reinterpret_cast<const f32x4*>(part + r * PADN + c);
#pragma unroll
    for (int k = 1; k < KW; k++) {
      const f32x4 p = *reinterpret_cast<const f32x4*>(part + (k * BM + r) * PADN + c);
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] += p[e];
    }
    const size_t idx = (size_t)row * g.ldc + col;
    if ((EPI == EPI_BIAS || EPI == EPI_RESID || EPI == EPI_GELU) && bias) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(bias + col);
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] += b[e];
    }
    if (EPI == EPI_RESID) {
      if (aux) *reinterpret_cast<f32x4*>(aux + idx) = x;
      const f32x4 o = *reinterpret_cast<const f32x4*>(resid + idx);
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] += o[e];
    } else if (EPI == EPI_GELU) {
      f32x4 y;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        float ye, dye;
        if (g.gelu_tanh) gelu_tanh_both_f(x[e], ye, dye);
        else gelu_both_f(x[e], ye, dye);
        y[e] = ye;
        x[e] = dye;
      }
      *reinterpret_cast<f32x4*>(aux + idx) = y;
    } else if (EPI == EPI_DGELU) {
      const f32x4 z = *reinterpret_cast<const f32x4*>(zin + idx);
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] *= z[e];
    } else if (EPI == EPI_F32_ACC) {
      const f32x4 o = *reinterpret_cast<const f32x4*>(C + idx);
#pragma unroll
      for (int e = 0; e < 4; e++) x[e] += o[e];
    }
    *reinterpret_cast<f32x4*>(C + idx) = x;
  }
}

template <int LAY, int EPI, int BM, int KW, int STAGES, bool AHEAD, bool SUMS>
__global__ void __launch_bounds__(BM * BM * KW / 16) gemm_f32_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  tile_of_product<LAY, EPI, BM, KW, STAGES, AHEAD, SUMS>(g, blockIdx.x, gridDim.x, smem);
}

// An input gradient and a weight gradient that need nothing of each other, in one launch: workgroups 0 .. nt_tiles - 1 have a
// tile of the first.  For layers so small that a launch, or handing work to another stream, costs more than the product: hidden
// 256, 256 tokens, forward and backward, 137 us with the weight gradients on a second stream, 125 with all launches in a row,
// 107 with the four pairs (15 launches instead of 21).
template <int EPI_NT, int EPI_TN, int STAGES>
__global__ void __launch_bounds__(256) gemm_f32_pair_kernel(GemmArgs nt, GemmArgs tn, int nt_tiles) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int pid = blockIdx.x;
  if (pid < nt_tiles) tile_of_product<LAY_NT, EPI_NT, 32, 4, STAGES, false>(nt, pid, nt_tiles, smem);
  else tile_of_product<LAY_TN, EPI_TN, 32, 4, STAGES, false, true>(tn, pid - nt_tiles, gridDim.x - nt_tiles, smem);
}

template <int LAY, int EPI, int BM, int KW, int STAGES, bool AHEAD, bool SUMS = false>
hipError_t launch_tile(const GemmArgs& g, hipStream_t s) {
  if constexpr (LAY == LAY_TN && !SUMS)
    if (g.colpart) return launch_tile<LAY, EPI, BM, KW, STAGES, AHEAD, true>(g, s);
  constexpr int SMEM = STAGES * 2 * KW * BM * 128;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_kernel<LAY, EPI, BM, KW, STAGES, AHEAD, SUMS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return e;
    configured = true;
  }
  hipLaunchKernelGGL((gemm_f32_kernel<LAY, EPI, BM, KW, STAGES, AHEAD, SUMS>), dim3(cdiv(g.M, BM) * cdiv(g.N, BM)),
                     dim3(BM * BM * KW / 16), SMEM, s, g);
  return hipGetLastError();
}

// The smaller tile is for products that leave most of the 256 compute units without one of 64 x 64;
// two wavefronts per block while that gives no unit more than three tiles, one beyond.  Two stages are enough with
// the fragments of the next one in registers, and leave room for two or four workgroups per unit, so that the last
// ones do not run alone.  Measured (NN, us; <32, KW 4> / <64, KW 2> / <64, KW 1>):
//   tiles of 64 x 64      64               128              256              320             1024             4096
//   (M, N, K)             512 512 1024     512 1024 1024    1024 1024 1024   1024 1280 1024  1024 4096 1024   4096 4096 1024
//                         9.8/20.0/22.0    18.0/20/22       31/20.4/21.6     42/36.5/37.1    130/71/69.5      502/276/270
// and at 768 tiles 99/54.0/54.3.  With fragments read at the start of their own stage, three and four stages: 768 tiles 58,
// 1024 tiles 77, 4096 tiles 280, 1024 1024 4096 (NT) 75.6 against 70.  The largest is 127 TFLOP/s of a peak of 157.
// Short reductions, the weight gradients of few tokens, end before the extra start has paid and keep that older form
// (forward and backward, us, without / with it: hidden 768, 128 tokens 217 / 210, hidden 1024, 128 tokens 255 / 248, hidden
// 2048, 33 tokens 428 / 410; with it from 192 tokens on hidden 768 is 2 to 5 % slower).  Hidden 512, whose weight gradients
// are one round of tiles beside the other stream, would be 1 to 2 % faster with it up to 512 tokens (256 tokens 205 / 201),
// hidden 768 and 1024 1 to 2 % slower, by the same tiles.
enum Pick { PICK_32, PICK_64_TWO, PICK_64_ONE, PICK_64_TWO_SHORT, PICK_64_ONE_SHORT };
Pick pick(int M, int N, int K) {
  const long t64 = (long)cdiv(M, 64) * cdiv(N, 64);
  if (t64 <= 128) return PICK_32;
  if (K <= 160) return t64 <= 256 ? PICK_64_TWO_SHORT : PICK_64_ONE_SHORT;
  return t64 <= 768 ? PICK_64_TWO : PICK_64_ONE;
}
template <int LAY, int EPI>
hipError_t launch(const GemmArgs& g, hipStream_t s) {
  switch (pick(g.M, g.N, g.K)) {
    case PICK_32: return launch_tile<LAY, EPI, 32, 4, 4, false>(g, s);
    case PICK_64_TWO: return launch_tile<LAY, EPI, 64, 2, 2, true>(g, s);
    case PICK_64_ONE: return launch_tile<LAY, EPI, 64, 1, 2, true>(g, s);
    case PICK_64_TWO_SHORT: return launch_tile<LAY, EPI, 64, 2, 4, false>(g, s);
    case PICK_64_ONE_SHORT: return launch_tile<LAY, EPI, 64, 1, 3, false>(g, s);
  }
  return hipErrorInvalidValue;
}

template <int EPI_NT, int EPI_TN, int STAGES>
hipError_t launch_pair_kernel(const GemmArgs& nt, const GemmArgs& tn, hipStream_t s) {
  constexpr int SMEM = STAGES * 2 * 4 * 32 * 128;
  static bool configured = false;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_f32_pair_kernel<EPI_NT, EPI_TN, STAGES>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles = cdiv(nt.M, 32) * cdiv(nt.N, 32);
  hipLaunchKernelGGL((gemm_f32_pair_kernel<EPI_NT, EPI_TN, STAGES>), dim3(tiles + cdiv(tn.M, 32) * cdiv(tn.N, 32)), dim3(256),
                     SMEM, s, nt, tn, tiles);
  return hipGetLastError();
}
// Two stages hold the whole of reductions of up to 256 steps and leave room for two workgroups per compute unit.
template <int EPI_NT, int EPI_TN>
hipError_t launch_pair(const GemmArgs& nt, const GemmArgs& tn, hipStream_t s) {
  return nt.K <= 256 && tn.K <= 256 ? launch_pair_kernel<EPI_NT, EPI_TN, 2>(nt, tn, s)
                                    : launch_pair_kernel<EPI_NT, EPI_TN, 4>(nt, tn, s);
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
  }
  return hipErrorInvalidValue;
}

}  // namespace

extern "C" int gx_f32_tile(int M, int N, int K) { return pick(M, N, K); }

namespace {
// 16-byte chunks along each operand's contiguous index, 31-bit byte offsets in buffer loads
bool args_ok(Layout lay, const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
  const long a_rows = (lay == LAY_TN) ? g.K : g.M, b_rows = (lay == LAY_NT) ? g.N : g.K;
  if ((g.lda | g.ldb | g.ldc | g.N) & 3) return false;
  if ((lay != LAY_TN && (g.K & 3)) || (lay == LAY_TN && (g.M & 3))) return false;
  if (a_rows * g.lda * 4 >= (1L << 31) || b_rows * g.ldb * 4 >= (1L << 31)) return false;
  return !((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B) | reinterpret_cast<uintptr_t>(g.C)) & 15);
}
}  // namespace

hipError_t gemm_f32(Layout lay, Epilogue epi, const GemmArgs& g, hipStream_t s) {
  if (!args_ok(lay, g)) return hipErrorInvalidValue;
  switch (lay) {
    case LAY_NN: return dispatch_epi<LAY_NN>(epi, g, s);
    case LAY_NT: return dispatch_epi<LAY_NT>(epi, g, s);
    case LAY_TN: return dispatch_epi<LAY_TN>(epi, g, s);
  }
  return hipErrorInvalidValue;
}

hipError_t gemm_f32_pair(Epilogue nt_epi, const GemmArgs& nt, bool accumulate, const GemmArgs& tn, hipStream_t s) {
  if (!args_ok(LAY_NT, nt) || !args_ok(LAY_TN, tn)) return hipErrorInvalidValue;
  if (nt_epi == EPI_STORE)
    return accumulate ? launch_pair<EPI_STORE, EPI_F32_ACC>(nt, tn, s) : launch_pair<EPI_STORE, EPI_F32>(nt, tn, s);
  if (nt_epi == EPI_DGELU)
    return accumulate ? launch_pair<EPI_DGELU, EPI_F32_ACC>(nt, tn, s) : launch_pair<EPI_DGELU, EPI_F32>(nt, tn, s);
  return hipErrorInvalidValue;
}

}  // namespace gx
