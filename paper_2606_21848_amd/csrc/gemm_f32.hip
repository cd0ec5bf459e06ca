// GEMM in fp32 arithmetic on the matrix cores (v_mfma_f32_16x16x4_f32), for the
// fp32 layer (projections, routing fold, weight gradients) and for the bf16
// products that the bf16 kernel does not take (operands widened as they are
// loaded). Operands are addressed by two strides each, so transposed operands
// are a choice of strides.
//
// Bound by the fp32 matrix rate (1/16 of bf16: 32 cycles per 16x16x4), which
// one LDS read of four k per 16 rows feeds for four products, so LDS and its
// staging cost little and the tile is chosen for the number of workgroups, not
// for reuse: 128 x 128, 64 x 64 or 32 x 32 (see launch_e). M 512, K 1024, N 1024
// + 1024: 31 us = 69 TFLOP/s, where a loop of the same products without operands
// takes 19 us; the two vector-ALU launches before it took 117 us. An 8-wave form
// that splits k over waves with private LDS and no barriers: 30 us.
//
// LDS holds an operand tile as quads of k: quad (k / 4, row) is 16 bytes, rows
// consecutive, one quad of padding per k-quad row, so a wave's fragment read
// (16 rows of 4 quad rows) is conflict-free. The contraction order is free as
// long as both operands agree: product j of a fragment pair contracts the k
// with k % 4 = j. A thread stages 4 x 4 blocks: four loads along the contiguous
// index, then four quads (transposed in registers where the rows, not k, are
// contiguous). Three tiles of loads are in flight while a tile is multiplied
// (one behind: 47 us); two LDS buffers, one barrier per tile.

#include "kl_device.h"
#include "kl_internal.h"

namespace kl {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;

// How an operand is loaded: four k of one row at once, four rows of one k at
// once, or element by element (no alignment, any strides).
enum LoadMode { kAlongK = 0, kAlongRows = 1, kScalar = 2 };

struct Operand {
  const void* p;
  long rs, ks;  // strides of the row (m or n) and of k, in elements
  int mode;
};

struct GemmF32Params {
  Operand A[2], B[2], Bd;  // two terms of the contraction; Bd: B of the second column block
  int K[2];
  int M, N, Nd;            // N columns to C, then Nd to Cd (the second column block, same A)
  void* C;
  void* Cd;
  long ldc, ldcd;
  long sA, sB, sC;         // between batch items (blockIdx.z)
  int tiles_n;             // column tiles of C
};

__device__ __forceinline__ f32x4_t load4(const float* p) {
  return *reinterpret_cast<const f32x4_t*>(p);
}
__device__ __forceinline__ f32x4_t load4(const uint16_t* p) {
  const u32x2 w = *reinterpret_cast<const u32x2*>(p);
  return f32x4_t{bf16_lo(w.x), bf16_hi(w.x), bf16_lo(w.y), bf16_hi(w.y)};
}
__device__ __forceinline__ float load1(const float* p) { return *p; }
__device__ __forceinline__ float load1(const uint16_t* p) {
  return __uint_as_float((uint32_t)*p << 16);
}
__device__ __forceinline__ void store1(float* p, float v) { *p = v; }
__device__ __forceinline__ void store1(uint16_t* p, float v) { *p = (uint16_t)f32_to_bf16(v); }

// One wave's (or two waves') share of staging an operand: a 4 x 4 block of rows
// rr .. rr + 3 and k 4 kq .. 4 kq + 3 of a tile, for lane x of TR rows x KQ quads.
template <typename E, int TR, int KQ, bool VEC>
struct Stager {
  const E *base0, *base1;  // of each term: scalars, so that the choice between them is a select
  uint32_t st0, st1;
  long rs0, ks0, rs1, ks1;
  int K0, K1, nk0, rows, r, rr, kq;
  bool along_k;  // uniform
  // Lanes run along k where k is contiguous (whole rows of a tile); else 16
  // lanes take 4 row blocks of 4 k quads, whose LDS writes then hit distinct
  // banks. Both terms of a product have the same layout.
  __device__ __forceinline__ Stager(const Operand& o0, const Operand& o1, size_t batch, int K0, int K1,
                                    int nk0, int rows, int first_row, int x)
      : base0(static_cast<const E*>(o0.p) + batch), base1(static_cast<const E*>(o1.p) + batch),
        rs0(o0.rs), ks0(o0.ks), rs1(o1.rs), ks1(o1.ks), K0(K0), K1(K1), nk0(nk0), rows(rows) {
    along_k = VEC ? o0.mode == kAlongK : o0.ks == 1;
    st0 = (uint32_t)(along_k ? o0.rs : o0.ks);
    st1 = (uint32_t)(along_k ? o1.rs : o1.ks);
    kq = along_k ? x % KQ : (x >> 2) % KQ;
    rr = along_k ? x / KQ * 4 : (x / (4 * KQ) * 4 + (x & 3)) * 4;
    r = first_row + rr;
  }
  // v[i]: row r + i (along k, scalar) or k + i (along rows) of tile kt. Indices
  // past the end are clamped: such rows are never stored, such k are zeroed as
  // the block is staged.
  __device__ __forceinline__ void load(int kt, f32x4_t (&v)[4]) const {
    const bool term = kt >= nk0;  // uniform: selects, no branch between the loads in flight
    const int k = (kt - (term ? nk0 : 0)) * (4 * KQ) + kq * 4, K = term ? K1 : K0;
    const E* base = term ? base1 : base0;
    if constexpr (VEC) {
      const E* src = base + (along_k ? min(k, K - 4) : min(r, rows - 4));
      const uint32_t st = term ? st1 : st0;
      const int first = along_k ? r : k, last = (along_k ? rows : K) - 1;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = load4(src + (size_t)(uint32_t)min(first + i, last) * st);
    } else {
      const long rs = term ? rs1 : rs0, ks = term ? ks1 : ks0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          v[i][j] = load1(base + (size_t)min(r + i, rows - 1) * rs + (size_t)min(k + j, K - 1) * ks);
    }
  }
  __device__ __forceinline__ void stage(int kt, const f32x4_t (&v)[4], f32x4_t* buf) const {
    const bool term = kt >= nk0;
    const int k0 = (kt - (term ? nk0 : 0)) * (4 * KQ), K = term ? K1 : K0;
    f32x4_t* dst = buf + kq * (TR + 1) + rr;
    f32x4_t q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) q[i][j] = !VEC || along_k ? v[i][j] : v[j][i];
    if (k0 + 4 * KQ > K) {  // uniform
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) q[i][j] = k0 + kq * 4 + j < K ? q[i][j] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) dst[i] = q[i];
  }
};

// Four consecutive columns of a row.
template <typename E>
__device__ __forceinline__ void store4(E* C, long ldc, int m, int n, int N, f32x4_t x) {
  E* dst = C + (size_t)m * ldc + n;
  if (sizeof(E) == 4 && ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0 && n + 4 <= N) {
    *reinterpret_cast<f32x4_t*>(dst) = x;
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (n + r < N) store1(dst + r, x[r]);
  }
}

// T x T output tile, k-steps of BK, 4 waves of T/2 x T/2, PF tiles of loads in
// flight. VEC: every operand is loaded four elements at a time.
template <typename E, int T, int BK, bool VEC>
__global__ __launch_bounds__(kThreads) void gemm_f32_kernel(GemmF32Params p) {
  constexpr int KQ = BK / 4;              // quads of k per tile
  constexpr int QP = T + 1;               // quads per k-quad row (padded)
  constexpr int BUF = 2 * KQ * QP;        // quads per buffer (A then B)
  constexpr int RB = T / 32;              // 16-row blocks per wave and operand
  constexpr int PF = VEC ? 3 : 1;
  static_assert(T / 4 * KQ * 2 == kThreads, "one 4 x 4 block per thread and tile");
  __shared__ f32x4_t lds[2 * BUF];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r16 = lane & 15, grp = lane >> 4;
  const int m0 = blockIdx.y * T;
  const bool second = (int)blockIdx.x >= p.tiles_n;  // uniform: the second column block
  const int n0 = (second ? blockIdx.x - p.tiles_n : blockIdx.x) * T;
  const int N = second ? p.Nd : p.N;
  const int nk0 = (p.K[0] + BK - 1) / BK, nk = nk0 + (p.K[1] + BK - 1) / BK;
  // Waves 0 and 1 stage A, waves 2 and 3 stage B.
  const bool is_a = wave < 2;
  const Operand o0 = is_a ? p.A[0] : (second ? p.Bd : p.B[0]);
  const Operand o1 = is_a ? p.A[1] : p.B[1];
  const Stager<E, T, KQ, VEC> sg(o0, o1, (size_t)blockIdx.z * (is_a ? p.sA : p.sB), p.K[0], p.K[1],
                                 nk0, is_a ? p.M : N, is_a ? m0 : n0, t % (kThreads / 2));
  const int place = is_a ? 0 : KQ * QP;
  f32x4_t v[PF][4];

  f32x4_t acc[RB][RB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < RB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int wm = (wave >> 1) * (T / 2) + r16, wn = (wave & 1) * (T / 2) + r16;
  auto step = [&](int kt, f32x4_t (&v)[4], bool more) {
    f32x4_t* buf = lds + (kt & 1) * BUF;
    sg.stage(kt, v, buf + place);
    __syncthreads();
    if (more) sg.load(min(kt + PF, nk - 1), v);
#pragma unroll
    for (int s = 0; s < BK / 16; ++s) {
      f32x4_t a[RB], b[RB];
      const f32x4_t* qa = buf + (s * 4 + grp) * QP;
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        a[i] = qa[wm + i * 16];
        b[i] = qa[KQ * QP + wn + i * 16];
      }
      // B as the first operand: the result is C^T, four consecutive columns per lane.
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int im = 0; im < RB; ++im)
#pragma unroll
          for (int in = 0; in < RB; ++in)
            acc[im][in] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[in][j], a[im][j], acc[im][in], 0, 0, 0);
    }
  };
  // The loop body is straight-line, its loads unconditional (past the end: the
  // last tile again), so that the compiler counts the loads in flight; behind a
  // branch it would wait for all of them at once.
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < PF; ++i) sg.load(min(i, nk - 1), v[i]);
    int kt = 0;
    for (; kt + PF <= nk; kt += PF) {
#pragma unroll
      for (int i = 0; i < PF; ++i) step(kt + i, v[i], true);
    }
#pragma unroll
    for (int i = 0; i + 1 < PF; ++i)
      if (kt + i < nk) step(kt + i, v[i], false);
  }

  // Lane holds C[wm + 16 im][n0 + (wave & 1) T / 2 + 16 in + 4 grp .. + 3].
  E* C = static_cast<E*>(second ? p.Cd : p.C) + (size_t)blockIdx.z * p.sC;
  const long ldc = second ? p.ldcd : p.ldc;
#pragma unroll
  for (int im = 0; im < RB; ++im) {
    const int m = m0 + wm + im * 16;
    if (m >= p.M) continue;
#pragma unroll
    for (int in = 0; in < RB; ++in) {
      const int n = n0 + (wave & 1) * (T / 2) + in * 16 + grp * 4;
      if (n < N) store4(C, ldc, m, n, N, acc[im][in]);
    }
  }
}

// The widest load that the operand's strides, base and extents allow. A chunk
// along the contiguous index is then whole or absent.
Operand operand(const void* ptr, long rs, long ks, int rows, int K, long batch_stride, size_t elem) {
  Operand o{ptr, rs, ks, kScalar};
  const bool al = reinterpret_cast<uintptr_t>(ptr) % (4 * elem) == 0 && batch_stride % 4 == 0 &&
                  rs < (1L << 31) && ks < (1L << 31);
  if (al && ks == 1 && rs % 4 == 0 && K % 4 == 0) o.mode = kAlongK;
  else if (al && rs == 1 && ks % 4 == 0 && rows % 4 == 0) o.mode = kAlongRows;
  return o;
}

template <typename E, int T, int BK>
hipError_t launch_t(GemmF32Params& p, bool vec, int batch, hipStream_t st) {
  p.tiles_n = (p.N + T - 1) / T;
  const dim3 grid(p.tiles_n + (p.Nd + T - 1) / T, (p.M + T - 1) / T, batch);
  if (vec) hipLaunchKernelGGL((gemm_f32_kernel<E, T, BK, true>), grid, dim3(kThreads), 0, st, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<E, T, BK, false>), grid, dim3(kThreads), 0, st, p);
  return hipGetLastError();
}

template <typename E>
hipError_t launch_e(GemmF32Params& p, bool vec, int batch, hipStream_t st) {
  auto tiles = [&](int T) {
    return (long)((p.N + T - 1) / T + (p.Nd + T - 1) / T) * ((p.M + T - 1) / T) * batch;
  };
  // The largest tile that fills the 256 CUs: 128-wide from one per CU on, 64-wide from
  // two (a training layer of 1400 tokens at d_model 1024: 469 us, against 490 from one
  // and 479 with 32-wide tiles only). Over 803 shapes 28 take more than 5% longer than the
  // best tile, most with 1 to 1.4 128-wide tiles per CU (M 1400, N 4096, K 1024, 352 of
  // them: 146, 64-wide 120), 2000 x 64 products over K 64 the most (16 items, us: 10.9,
  // 64-wide 7.6).
  if (tiles(128) >= 256) return launch_t<E, 128, 16>(p, vec, batch, st);
  if (tiles(64) >= 512) return launch_t<E, 64, 32>(p, vec, batch, st);
  return launch_t<E, 32, 64>(p, vec, batch, st);
}

}  // namespace

hipError_t launch_gemm_f32(const GemmParams& g, hipStream_t st) {
  if (g.M == 0 || (g.N == 0 && g.N2 == 0) || g.batch == 0) return hipSuccess;
  const size_t e = g.dtype == KL_BF16 ? 2 : 4;
  auto one = [](long s) { return s ? s : 1L; };
  GemmF32Params p{};
  p.A[0] = operand(g.A, g.lda, one(g.a_cs), g.M, g.K, g.strideA, e);
  p.B[0] = operand(g.Bm, one(g.b_cs), g.ldb, g.N, g.K, g.strideB, e);
  p.K[0] = g.K;
  if (g.K1 > 0) {
    p.A[1] = operand(g.A1, g.lda1, one(g.a_cs), g.M, g.K1, g.strideA, e);
    p.B[1] = operand(g.B1, one(g.b_cs1), g.ldb1, g.N, g.K1, g.strideB, e);
    p.K[1] = g.K1;
  }
  if (g.N2 > 0) p.Bd = operand(g.B2, one(g.b_cs), g.ldb2, g.N2, g.K, g.strideB, e);
  p.M = g.M;
  p.N = g.N;
  p.Nd = g.N2;
  p.C = g.C;
  p.Cd = g.C2;
  p.ldc = g.ldc;
  p.ldcd = g.ldc2;
  p.sA = g.strideA;
  p.sB = g.strideB;
  p.sC = g.strideC;
  bool vec = p.A[0].mode != kScalar && p.B[0].mode != kScalar;
  if (g.N2 > 0) vec = vec && p.Bd.mode != kScalar;
  if (g.K1 > 0) {  // both terms in one layout
    vec = vec && p.A[1].mode == p.A[0].mode && p.B[1].mode == p.B[0].mode;
  }
  return g.dtype == KL_BF16 ? launch_e<uint16_t>(p, vec, g.batch, st)
                            : launch_e<float>(p, vec, g.batch, st);
}

}  // namespace kl
