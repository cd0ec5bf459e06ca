// bf16 MFMA GEMM for the prefill projections [Q~ | V] = X [W~^Q | W^V]
// (Eq. 2: no key projection), against weights packed once before inference,
// and for the large products of the backward pass through the projections.
//
// C (M x N) = A0 W0^T + A1 W1^T, where A0 [M, K0] and W0 [N, K0] (row n =
// output column n) are both K-major, the layout the MFMA fragments want; the
// optional second term (K1 > 0) continues the same k loop on another pair of
// operands. For the projections A0 = X, W0 = the packed weights and K1 = 0.
// Columns below n_split go to C0 (the routed queries), the rest to C1 (the
// values). fp32 accumulation in v_mfma_f32_16x16x32_bf16, one rounding to
// bf16 on store.
//
// Large products: tile 256 x 256 x 64, 16 waves (4 x 4), each wave 64 x 64 of C
// (64 fp32 accumulators per lane, four waves per SIMD: while some waves restart a
// k-tile with their LDS reads after the barrier, others keep the matrix pipe
// busy). Each operand tile is rows of 128 bytes in LDS with the 16-byte chunks of
// row r XOR-swizzled by (r >> 1) & 7, so the fragment reads (16 rows per access)
// are free of bank conflicts. Tiles move from memory straight into LDS
// (global_load_lds, 16 bytes per lane, no register staging); the swizzle is
// applied to the global addresses. Two LDS stages (128 KiB): the next tile is in
// flight while the current one is multiplied.
// A product with few such tiles leaves most CUs idle (a prompt of 517 tokens at
// N 1792: 21 tiles for 256 CUs), and what bounds it is the latency of its k-steps
// (0.4 us each whatever their size), so it takes 128 x 128 or 64 x 64 tiles: more
// workgroups, shorter steps, and a third stage where one CU holds few waves. The
// rule and its measurements stand at launch_gemm_bf16.
// Workgroup ids are remapped so each XCD owns a band of tile rows walked
// column-major, which keeps concurrently running tiles in that XCD's L2.

#include <cmath>
#include <type_traits>

#include "kl_device.h"
#include "kl_internal.h"

namespace kl {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((address_space(3))) unsigned char lds_u8;

constexpr int BK = 64;
static_assert(BK == 64, "the fragment schedule assumes two 32-wide k-steps per tile");

// An output tile of BM x BN on WM x WN waves, ST stages of LDS.
template <int BM_, int BN_, int WM_, int WN_, int ST_>
struct Shape {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, ST = ST_;
  static constexpr int WAVES = WM * WN, THREADS = WAVES * 64;
  static constexpr int TA = BM * BK * 2, TW = BN * BK * 2;  // bytes of an operand tile
  static constexpr int STAGE = TA + TW, LDS = ST * STAGE;
  static constexpr int CA = BM / 8 / WAVES;  // copies per wave and operand tile
  static constexpr int RM = BM / WM / 16, RN = BN / WN / 16;      // 16-wide blocks per wave
  static constexpr int EU = WAVES >= 8 ? 4 : 2;                   // waves per SIMD to fit
  static_assert(ST == 2 || ST == 3, "the loop's waits");
  static_assert(CA * 8 * WAVES == BM && BM == BN, "whole copies per wave");
};
using Shape256 = Shape<256, 256, 4, 4, 2>;  // one workgroup per CU
using Shape128 = Shape<128, 128, 2, 2, 2>;  // two
using Shape128Deep = Shape<128, 128, 2, 4, 3>;  // one: 8 waves, two k-tiles in flight
using Shape64 = Shape<64, 64, 2, 2, 3>;     // three

struct GemmParams2 {
  const uint16_t* A0;  // [M, K0], row stride lda0 (elements)
  const uint16_t* W0;  // [N, K0], row stride ldw0
  const uint16_t* A1;  // [M, K1], row stride lda1 (K1 = 0: no second term)
  const uint16_t* W1;  // [N, K1], row stride ldw1
  void* C0;            // columns [0, n_split): bf16, or fp32 for the F32 form
  void* C1;            // columns [n_split, N)
  int M, N, K0, K1, n_split;
  long lda0, ldw0, lda1, ldw1;
  long ldc0, ldc1;
  long sA0, sW0, sC0, sC1;  // element strides between batch items (blockIdx.y)
  long zA0, zW0, zC0;       // and along blockIdx.z (a second batch index)
};

// Byte offset of (row, 16-byte chunk) inside a swizzled operand tile.
__device__ __forceinline__ int swz(int row, int chunk) {
  return row * (BK * 2) + ((chunk ^ ((row >> 1) & 7)) << 4);
}

// Four waves per SIMD (the 128 KiB of LDS allow one workgroup per CU): the
// register budget is 128, the accumulators and one k-step's fragments.
// TWO: the second term is present (one more pair of copy offsets per lane and
// a uniform choice per k-tile; the projections take the plain form). F32: the
// outputs are stored in fp32 (partial products of a split contraction).
template <class SH, bool TWO, bool F32>
__global__ __launch_bounds__(SH::THREADS) __attribute__((amdgpu_waves_per_eu(SH::EU, 4)))
void gemm_bf16_kernel(GemmParams2 p) {
  constexpr int BM = SH::BM, BN = SH::BN, RM = SH::RM, RN = SH::RN, ST = SH::ST;
  using CT = std::conditional_t<F32, float, uint16_t>;
  const int tilesM = (p.M + BM - 1) / BM, tilesN = (p.N + BN - 1) / BN;
  const int ntiles = tilesM * tilesN;
  CT* C0 = static_cast<CT*>(p.C0);
  CT* C1 = static_cast<CT*>(p.C1);
  if (blockIdx.y > 0 || blockIdx.z > 0) {  // batch item: the first term's operands and the outputs move
    p.A0 += (size_t)blockIdx.y * p.sA0 + (size_t)blockIdx.z * p.zA0;
    p.W0 += (size_t)blockIdx.y * p.sW0 + (size_t)blockIdx.z * p.zW0;
    C0 += (size_t)blockIdx.y * p.sC0 + (size_t)blockIdx.z * p.zC0;
    C1 += (size_t)blockIdx.y * p.sC1 + (size_t)blockIdx.z * p.zC0;
  }
  int wg = blockIdx.x;
  // XCD-aware order: hardware places workgroup i on XCD i % 8; each XCD takes a
  // contiguous run of tiles.
  wg = (wg & 7) * (ntiles >> 3) + min(wg & 7, ntiles & 7) + (wg >> 3);
  constexpr int GM = 4;
  const int group = wg / (GM * tilesN);
  const int first_m = group * GM;
  const int gsize = min(tilesM - first_m, GM);
  const int in_group = wg % (GM * tilesN);
  const int m0 = (first_m + in_group % gsize) * BM;
  const int n0 = (in_group / gsize) * BN;

  // ST pipeline stages, each an A tile and a W tile: [stage][A | W].
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / SH::WN, wn = wave % SH::WN;  // wave tile: rows 16 RM wm.., columns 16 RN wn..

  // Direct-to-LDS copies: one wave instruction fills 8 rows (1 KiB) of a tile,
  // lane L landing at byte 16 L, i.e. row L / 8, physical chunk L % 8, which
  // holds logical chunk (L % 8) ^ ((row >> 1) & 7). Each wave fills CA row groups
  // of each operand. Rows past the end are clamped: they only feed output rows
  // or columns that are never stored. Per-lane byte offsets for each term.
  constexpr int NT = TWO ? 2 : 1;
  uint32_t offA[NT][SH::CA], offW[NT][SH::CA];  // [term][row group]
  auto lane_offsets = [&](auto& off, int row0, int rows, long ld0, long ld1) {
#pragma unroll
    for (int i = 0; i < SH::CA; ++i) {
      const int r = (i * SH::WAVES + wave) * 8 + (lane >> 3);
      const int lc = (lane & 7) ^ ((r >> 1) & 7);
      const int rc = min(row0 + r, rows - 1);
      off[0][i] = (uint32_t)(((size_t)rc * ld0 + lc * 8) * 2);
      if constexpr (TWO) off[NT - 1][i] = (uint32_t)(((size_t)rc * ld1 + lc * 8) * 2);
    }
  };
  lane_offsets(offA, m0, p.M, p.lda0, p.lda1);
  lane_offsets(offW, n0, p.N, p.ldw0, p.ldw1);
  const int nk0 = p.K0 / BK;  // k-tiles of the first term
  // Copies of k-tile kt (of the concatenated k range) into one stage.
  auto issue = [&](lds_u8* sa, lds_u8* sw, int kt) {
    const bool second = TWO && kt >= nk0;  // uniform
    const int k0 = (second ? kt - nk0 : kt) * BK;
    const unsigned char* ga = reinterpret_cast<const unsigned char*>(second ? p.A1 : p.A0) + (size_t)k0 * 2;
    const unsigned char* gw = reinterpret_cast<const unsigned char*>(second ? p.W1 : p.W0) + (size_t)k0 * 2;
#pragma unroll
    for (int i = 0; i < SH::CA; ++i) {
      const uint32_t grp_off = (uint32_t)((i * SH::WAVES + wave) * 1024);
      copy_to_lds(ga, second ? offA[NT - 1][i] : offA[0][i], (uint32_t)(uintptr_t)sa + grp_off);
      copy_to_lds(gw, second ? offW[NT - 1][i] : offW[0][i], (uint32_t)(uintptr_t)sw + grp_off);
    }
  };

  f32x4_t acc[RM][RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int fr = lane & 15, grp = lane >> 4;
  // Per 32-wide k-step: the wave's RM A and RN W fragments, then their products
  // (one fragment set; the other waves on the SIMD cover the read latency).
  auto compute = [&](const lds_u8* a, const lds_u8* w) {
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
      const int chunk = ks * 4 + grp;
      bf16x8_t af[RM], bf[RN];
#pragma unroll
      for (int i = 0; i < RM; ++i)
        af[i] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t*>(
            a + swz(wm * (RM * 16) + i * 16 + fr, chunk));
#pragma unroll
      for (int j = 0; j < RN; ++j)
        bf[j] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8_t*>(
            w + swz(wn * (RN * 16) + j * 16 + fr, chunk));
      // W as the A operand: the result block is C^T, so a lane holds four
      // consecutive output columns of one row (one 8-byte store in bf16).
#pragma unroll
      for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], af[i], acc[i][j], 0, 0, 0);
    }
  };

  lds_u8* const base = (lds_u8*)smem;
  auto stageA = [&](int st) { return base + st * SH::STAGE; };
  auto stageW = [&](int st) { return base + st * SH::STAGE + SH::TA; };
  const int nk = TWO ? nk0 + p.K1 / BK : nk0;
#pragma unroll
  for (int i = 0; i < ST - 1; ++i)
    if (i < nk) issue(stageA(i), stageW(i), i);
  // One barrier per k-tile. Before it, each wave waits for its copies of tile
  // kt (those of the later tiles may stay in flight) and for its own LDS reads
  // of tile kt - 1 (the barrier does not wait for those); after it, both hold
  // for every wave, so the copies of tile kt + ST - 1 may refill the stage of
  // tile kt - 1 while tile kt is multiplied.
  constexpr int PER = 2 * SH::CA;
  int ring = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const int ahead = nk - 1 - kt;  // tiles after kt, of which ST - 2 may be in flight
    if (ST == 3 && ahead >= 1) KL_WAIT_VMCNT(PER);
    else KL_WAIT_VMCNT(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    const int cur = ST == 2 ? kt & 1 : ring;
    const int refill = ST == 2 ? cur ^ 1 : (cur == 0 ? ST - 1 : cur - 1);
    if (kt + ST - 1 < nk) issue(stageA(refill), stageW(refill), kt + ST - 1);
    compute(stageA(cur), stageW(cur));
    ring = cur == ST - 1 ? 0 : cur + 1;
  }

  // Lane holds C[row 16 i + fr][col 16 j + 4 grp + r] of the wave's block:
  // four consecutive columns, stored as one 8-byte (bf16) or 16-byte (fp32)
  // store when they lie on one side of n_split, inside N, and the outputs' row
  // strides and bases keep them aligned (uniform); otherwise element by element.
  // A tile whose rows all exist stores without a per-row check.
  constexpr int VB = 4 * (int)sizeof(CT);  // bytes of four outputs
  const bool vec = p.ldc0 % 4 == 0 && p.ldc1 % 4 == 0 && p.n_split % 4 == 0 &&
                   reinterpret_cast<uintptr_t>(C0) % VB == 0 &&
                   reinterpret_cast<uintptr_t>(C1) % VB == 0;
  auto store = [&](auto check_rows) {
    constexpr bool CHECK = decltype(check_rows)::value;
#pragma unroll
    for (int i = 0; i < RM; ++i) {
      const int row = m0 + wm * (RM * 16) + i * 16 + fr;
      if (CHECK && row >= p.M) continue;
#pragma unroll
      for (int j = 0; j < RN; ++j) {
        const int col = n0 + wn * (RN * 16) + j * 16 + grp * 4;
        if (vec && col + 4 <= p.N && (col + 4 <= p.n_split || col >= p.n_split)) {
          CT* dst = col < p.n_split ? C0 + (size_t)row * p.ldc0 + col
                                    : C1 + (size_t)row * p.ldc1 + (col - p.n_split);
          if constexpr (F32) {
            *reinterpret_cast<f32x4_t*>(dst) = acc[i][j];
          } else {
            typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;
            const bf16x4_t v = {(__bf16)acc[i][j][0], (__bf16)acc[i][j][1], (__bf16)acc[i][j][2],
                                (__bf16)acc[i][j][3]};
            *reinterpret_cast<bf16x4_t*>(dst) = v;
          }
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int c = col + r;
            if (c >= p.N) continue;
            CT* dst = c < p.n_split ? C0 + (size_t)row * p.ldc0 + c
                                    : C1 + (size_t)row * p.ldc1 + (c - p.n_split);
            if constexpr (F32) *dst = acc[i][j][r];
            else *dst = __builtin_bit_cast(uint16_t, (__bf16)acc[i][j][r]);
          }
        }
      }
    }
  };
  if (m0 + BM <= p.M) store(std::false_type{});
  else store(std::true_type{});
}

}  // namespace

const char* gemm_bf16_unsupported(const GemmBf16Args& a) {
  if (a.M <= 0 || a.N <= 0) return "empty product";
  if (a.K0 < BK || a.K0 % BK != 0 || a.K1 < 0 || a.K1 % BK != 0)
    return "the contraction lengths must be multiples of 64 (the first one positive)";
  if (a.lda0 % 8 != 0 || a.lda0 < a.K0 || a.ldw0 % 8 != 0 || a.ldw0 < a.K0)
    return "operand row strides must be multiples of 8 and at least the contraction length";
  if (a.K1 > 0 && (a.lda1 % 8 != 0 || a.lda1 < a.K1 || a.ldw1 % 8 != 0 || a.ldw1 < a.K1))
    return "operand row strides must be multiples of 8 and at least the contraction length";
  if (a.ldc0 <= 0 || a.ldc1 <= 0) return "output row strides must be positive";
  if ((a.batch > 1 || a.zbatch > 1) &&
      (a.K1 > 0 || a.batch > 65535 || a.zbatch > 65535 || a.sA0 % 8 != 0 || a.sW0 % 8 != 0 ||
       a.zA0 % 8 != 0 || a.zW0 % 8 != 0))
    return "a batched product has one term, at most 65535 items per index, and 16-byte aligned items";
  if (a.c_f32 && a.K1 > 0) return "fp32 outputs are for one-term products";
  // Operand offsets are 32-bit byte offsets.
  const size_t lim = 1ull << 32;
  if ((size_t)a.M * a.lda0 * 2 >= lim || (size_t)a.N * a.ldw0 * 2 >= lim ||
      (a.K1 > 0 && ((size_t)a.M * a.lda1 * 2 >= lim || (size_t)a.N * a.ldw1 * 2 >= lim)))
    return "an operand exceeds 4 GiB (32-bit operand offsets)";
  return nullptr;
}

const char* gemm_bf16_unsupported(int M, int N, int K, long lda, long ldc0, long ldc1) {
  GemmBf16Args a{};
  a.M = M;
  a.N = N;
  a.K0 = K;
  a.lda0 = lda;
  a.ldw0 = K;
  a.ldc0 = ldc0;
  a.ldc1 = ldc1;
  const char* why = gemm_bf16_unsupported(a);
  if (why && (K < BK || K % BK != 0)) return "d_model must be a positive multiple of 64 for bf16";
  if (why && (lda % 8 != 0 || lda < K))
    return "the row stride of x must be a multiple of 8 and >= d_model";
  return why;
}

namespace {

template <class SH, bool TWO, bool F32>
hipError_t launch_shape(const GemmParams2& p, int batch, int zbatch, hipStream_t st) {
  static std::atomic<uint32_t> done{0};
  hipError_t e = set_max_lds((const void*)gemm_bf16_kernel<SH, TWO, F32>, SH::LDS, done);
  if (e != hipSuccess) return e;
  const int tiles = ((p.M + SH::BM - 1) / SH::BM) * ((p.N + SH::BN - 1) / SH::BN);
  hipLaunchKernelGGL((gemm_bf16_kernel<SH, TWO, F32>), dim3(tiles, batch, zbatch), dim3(SH::THREADS),
                     SH::LDS, st, p);
  return hipGetLastError();
}

template <class SH>
hipError_t launch_form(const GemmParams2& p, int batch, int zbatch, bool f32, hipStream_t st) {
  if (p.K1 > 0) return launch_shape<SH, true, false>(p, batch, zbatch, st);
  return f32 ? launch_shape<SH, false, true>(p, batch, zbatch, st)
             : launch_shape<SH, false, false>(p, batch, zbatch, st);
}

}  // namespace

hipError_t launch_gemm_bf16(const GemmBf16Args& a, hipStream_t st) {
  GemmParams2 p{};
  p.A0 = static_cast<const uint16_t*>(a.A0);
  p.W0 = static_cast<const uint16_t*>(a.W0);
  p.A1 = static_cast<const uint16_t*>(a.K1 > 0 ? a.A1 : a.A0);
  p.W1 = static_cast<const uint16_t*>(a.K1 > 0 ? a.W1 : a.W0);
  p.C0 = a.C0;
  p.C1 = a.C1;
  p.M = a.M;
  p.N = a.N;
  p.K0 = a.K0;
  p.K1 = a.K1;
  p.n_split = a.n_split;
  p.lda0 = a.lda0;
  p.ldw0 = a.ldw0;
  p.lda1 = a.K1 > 0 ? a.lda1 : a.lda0;
  p.ldw1 = a.K1 > 0 ? a.ldw1 : a.ldw0;
  p.ldc0 = a.ldc0;
  p.ldc1 = a.ldc1;
  p.sA0 = a.sA0;
  p.sW0 = a.sW0;
  p.sC0 = a.sC0;
  p.sC1 = a.sC1;
  p.zA0 = a.zA0;
  p.zW0 = a.zW0;
  p.zC0 = a.zC0;
  const int batch = a.batch > 1 ? a.batch : 1, zbatch = a.zbatch > 1 ? a.zbatch : 1;
  auto tiles = [&](int T) {
    return (double)((a.M + T - 1) / T) * ((a.N + T - 1) / T) * batch * zbatch;
  };
  // The shape whose workgroups take the least time, from the time of one k-step
  // (64 deep) measured at K 1024 to 4096, in us: 256 x 256 tiles 1.7 per full
  // round of 256 (one per CU), 1.3 for a last round that is partly empty; 128 x
  // 128 tiles 0.95 per round of 512 (two per CU) or 0.65 for a last one of at
  // most 256; 64 x 64 tiles 0.15 + 0.22 per 256. At N 1792, K 1536 (256 / 128 /
  // 64, us): M 517: 37 / 18 / 9.3; M 2000: 38 / 17 / 23; M 4096: 40 / 28 / 41;
  // at N = 8192, K = 4096: M 1000: 83 / 62 / 100, M 8192: 422 / 470 / 778. The number
  // of k-steps cancels as long as they outweigh a tile's entry and store: over 771
  // shapes (K 64 to 8192) no choice is slower than 256-wide tiles by 2.5%, but with one to
  // four k-steps the fastest shape is up to 30% faster (M 3000, N 3072, K 256: 14 / 16 /
  // 18 for 64 / 128 / 256), and so are one-k-loop batches of 128 x 128 outputs (96 items
  // over K 2048: 20 on 128-wide tiles, 39 on the 64-wide ones that are taken).
  auto rounds = [](double t, double per, double full, double part, double few) {
    const double whole = std::floor(t / per), rest = t - whole * per;
    return whole * full + (rest == 0 ? 0. : (2 * rest <= per ? few : part));
  };
  const double t256 = rounds(tiles(256), 256, 1.7, 1.3, 1.3);
  const double t128 = rounds(tiles(128), 512, 0.95, 0.95, 0.65);
  const double t64 = 0.15 + 0.22 * tiles(64) / 256;
  if (t64 < t128 && t64 < t256) return launch_form<Shape64>(p, batch, zbatch, a.c_f32, st);
  if (t256 <= t128) return launch_form<Shape256>(p, batch, zbatch, a.c_f32, st);
  if (tiles(128) <= 256) return launch_form<Shape128Deep>(p, batch, zbatch, a.c_f32, st);
  return launch_form<Shape128>(p, batch, zbatch, a.c_f32, st);
}

namespace {

// out[i] = bf16(sum over s < S of part[s n + i]), in order of s; four elements a
// thread (n is a multiple of 4: whole heads).
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ part, int S,
                                                           size_t n, uint16_t* __restrict__ out) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
  for (int s = 0; s < S; ++s) acc += *reinterpret_cast<const f32x4_t*>(part + (size_t)s * n + i);
#pragma unroll
  for (int e = 0; e < 4; ++e) out[i + e] = __builtin_bit_cast(uint16_t, (__bf16)acc[e]);
}

}  // namespace

hipError_t launch_sum_partials_bf16(const float* part, int S, size_t n, void* out, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (S <= 0 || n % 4 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n / 4 + 255) / 256)), dim3(256), 0, st, part,
                     S, n, static_cast<uint16_t*>(out));
  return hipGetLastError();
}

hipError_t launch_gemm_bf16_packed(const void* A, int M, int K, long lda, const void* Wp, int N,
                                   int n_split, void* C0, long ldc0, void* C1, long ldc1,
                                   hipStream_t st) {
  GemmBf16Args a{};
  a.A0 = A;
  a.lda0 = lda;
  a.W0 = Wp;
  a.ldw0 = K;
  a.K0 = K;
  a.M = M;
  a.N = N;
  a.n_split = n_split;
  a.C0 = C0;
  a.ldc0 = ldc0;
  a.C1 = C1;
  a.ldc1 = ldc1;
  return launch_gemm_bf16(a, st);
}

}  // namespace kl

