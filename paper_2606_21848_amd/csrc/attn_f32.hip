// fp32 keyless attention on the matrix cores (v_mfma_f32_16x16x4_f32: fp32
// products, fp32 sums), forward (Eq. 2 with the score of Eq. 4, and Eq. 14) and
// backward (Section 2.3), for 16-byte aligned operands.
//
// A 16 x 16 block of scores costs D / 4 products of 32 cycles, so with 16-byte
// loads and one LDS round trip per block the kernels are bound by the matrix
// rate once enough waves run. A short fp32 layer (a few hundred tokens, a few
// heads) has few 16-row blocks: a workgroup therefore owns one 16-row block
// (queries for the output and dQ~, values for dV) and its NW waves share the
// blocks it meets, block t to wave t % NW, each with a private LDS tile and no
// barrier until the waves' partial results are merged. At N 512, 8 heads x 128,
// causal: forward 17.5 us, dQ~ 25 us, dV 35 us (0.27, 0.40 and 0.54 GFLOP; the
// CU with the heaviest block is the bound, 8 of the forward's 17.5 us), where
// the vector-ALU kernels took 117, 1904 and 1100 us.
//
// Layouts. Row blocks are read from memory straight into the first operand's
// layout (lane (r, g) = (lane % 16, lane / 16) holds columns 16 s + 4 g .. + 3
// of row r: product j of step s contracts the columns with 4 g + j, an order
// both operands share). The scores come out with one row of the workgroup's own
// block per lane column and rows 4 g + i of the other block in register i,
// which is the second product's second operand as it stands (step i contracts
// rows 4 g + i); its first operand, the other block transposed, is read from
// the LDS copy of the block, row pitch D + 4 floats so that the four lane
// groups hit distinct banks.

#include <algorithm>

#include "kl_device.h"
#include "kl_internal.h"

namespace kl {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.69314718055994531f;

template <int D>
struct Block {  // a 16-row block staged by one wave
  static constexpr int S = D / 16;      // 16-byte pieces per lane
  static constexpr int PITCH = D + 4;   // floats
  static constexpr int FLOATS = 16 * PITCH;
};

// Row `row` (zeros when it is not below `rows`) of a [rows, ...] matrix, in the
// layout above.
template <int D>
__device__ __forceinline__ void load_rows(const float* base, long stride, int row, int rows, int g,
                                          f32x4_t (&v)[D / 16]) {
  const bool live = row < rows;
  const float* src = base + (size_t)(live ? row : 0) * stride + 4 * g;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    const f32x4_t x = *reinterpret_cast<const f32x4_t*>(src + 16 * s);
    v[s] = live ? x : f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
}

template <int D>
__device__ __forceinline__ void stage_rows(float* tile, int r, int g, const f32x4_t (&v)[D / 16]) {
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
    *reinterpret_cast<f32x4_t*>(tile + r * Block<D>::PITCH + 16 * s + 4 * g) = v[s];
}

// acc[a row][b row] += sum over the D columns.
template <int D>
__device__ __forceinline__ f32x4_t dot_rows(const f32x4_t (&a)[D / 16], const f32x4_t (&b)[D / 16],
                                            f32x4_t acc) {
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][j], b[s][j], acc, 0, 0, 0);
  return acc;
}

// acc[db] (columns 16 db + 4 g + i of the result, own row r) += tile^T w over
// the tile's 16 rows.
template <int D>
__device__ __forceinline__ void add_weighted(const float* tile, int r, int g, f32x4_t w,
                                             f32x4_t (&acc)[D / 16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
      acc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(
          tile[(4 * g + i) * Block<D>::PITCH + 16 * db + r], w[i], acc[db], 0, 0, 0);
}

// The same on a diagonal block that holds an infinity or a NaN: rows the own row
// does not see (`first` .. `last` are seen) must not reach it, not even as 0 x inf.
template <int D>
__device__ __forceinline__ void add_weighted_seen(const float* tile, int r, int g, f32x4_t w,
                                                  int first, int last, f32x4_t (&acc)[D / 16]) {
#pragma unroll 1
  for (int k = 0; k < 16; ++k) {
    const float x = (k & 2) ? ((k & 1) ? w[3] : w[2]) : ((k & 1) ? w[1] : w[0]);
    const float wk = __shfl(x, (k >> 2) * 16 + r, 64);
    const bool seen = k >= first && k <= last;
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = tile[k * Block<D>::PITCH + 16 * db + 4 * g + i];
        acc[db][i] = seen ? fmaf(wk, v, acc[db][i]) : acc[db][i];
      }
  }
}

template <int D>
__device__ __forceinline__ bool any_not_finite(const f32x4_t (&v)[D / 16]) {
  bool bad = false;
#pragma unroll
  for (int s = 0; s < D / 16; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) bad |= !(fabsf(v[s][j]) < INFINITY);
  return __builtin_amdgcn_ballot_w64(bad) != 0;
}

// Sums the waves' acc (scaled by `f`) into out(row, column, value) calls, one
// per element of the 16 x D result, in wave order. Uses every wave's tile.
template <int D, int NW, class Out>
__device__ __forceinline__ void merge_sum(float* lds, float* tile, int r, int g, float f,
                                          const f32x4_t (&acc)[D / 16], Out out) {
#pragma unroll
  for (int db = 0; db < D / 16; ++db)
    *reinterpret_cast<f32x4_t*>(tile + r * Block<D>::PITCH + 16 * db + 4 * g) = acc[db] * f;
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * D / 4; e += NW * 64) {
    const int row = e / (D / 4), c = e % (D / 4) * 4;
    f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w)
      sum += *reinterpret_cast<const f32x4_t*>(lds + w * Block<D>::FLOATS + row * Block<D>::PITCH + c);
    out(row, c, sum);
  }
}

// Forward: 16 query rows of one head per workgroup.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_f32_kernel(AttnParams p) {
  constexpr int S = D / 16;
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  __shared__ float s_ml[NW][16][2];
  const int nq = (p.N + 15) / 16;
  // Heads fastest, the heaviest causal blocks first.
  const int q0 = (p.causal ? nq - 1 - (int)blockIdx.y : (int)blockIdx.y) * 16;
  const int h = blockIdx.x, b = blockIdx.z, kg = h / (p.H / p.G);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const tile = lds_f32 + wave * Block<D>::FLOATS;
  const float* V = static_cast<const float*>(p.v) + (size_t)b * p.Nk * p.v_stride + (size_t)kg * D;

  const int nblk = ((p.causal ? min(q0 + 16, p.Nk) : p.Nk) + 15) / 16;
  f32x4_t v[S], q[S], o[S];
  if (wave < nblk) load_rows<D>(V, p.v_stride, wave * 16 + r, p.Nk, g, v);
  load_rows<D>(static_cast<const float*>(p.q) + (size_t)b * p.N * p.q_stride + (size_t)h * D,
               p.q_stride, q0 + r, p.N, g, q);
#pragma unroll
  for (int s = 0; s < S; ++s) {
    q[s] *= p.scale_log2;
    o[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY, l = 0.f;
  for (int t = wave; t < nblk; t += NW) {
    const int j0 = t * 16;
    stage_rows<D>(tile, r, g, v);
    f32x4_t sc = dot_rows<D>(v, q, f32x4_t{0.f, 0.f, 0.f, 0.f});
    const bool diag = p.causal && j0 + 15 > q0;  // uniform
    const bool apart = diag && any_not_finite<D>(v);
    if (t + NW < nblk) load_rows<D>(V, p.v_stride, j0 + NW * 16 + r, p.Nk, g, v);
    if (diag || j0 + 16 > p.Nk) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = j0 + 4 * g + i;
        if (j >= p.Nk || (p.causal && j > q0 + r)) sc[i] = -INFINITY;
      }
    }
    float mt = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(m, fmaxf(mt, __shfl_xor(mt, 32)));
    const float ms = mt == -INFINITY ? 0.f : mt;
    const float alpha = fast_exp2(m - ms);
    m = mt;
    f32x4_t w;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = fast_exp2(sc[i] - ms);
    l = fmaf(l, alpha, (w[0] + w[1]) + (w[2] + w[3]));
#pragma unroll
    for (int s = 0; s < S; ++s) o[s] *= alpha;
    if (apart) add_weighted_seen<D>(tile, r, g, w, 0, q0 + r - j0, o);
    else add_weighted<D>(tile, r, g, w, o);
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (g == 0) {
    s_ml[wave][r][0] = m;
    s_ml[wave][r][1] = l;
  }
  __syncthreads();
  auto total = [&](int row, float& mx) {
    mx = s_ml[0][row][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_ml[w][row][0]);
    const float ms = mx == -INFINITY ? 0.f : mx;
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) sum = fmaf(s_ml[w][row][1], fast_exp2(s_ml[w][row][0] - ms), sum);
    return sum;
  };
  float mx;
  const float sum = total(r, mx);
  const float ms = mx == -INFINITY ? 0.f : mx;
  if (p.lse && wave == 0 && g == 0 && q0 + r < p.N)
    p.lse[((size_t)b * p.H + h) * p.N + q0 + r] = sum > 0.f ? (mx + __log2f(sum)) * kLn2 : -INFINITY;
  // No value rows: a zero row.
  const float f = sum > 0.f ? fast_exp2(m - ms) / sum : 0.f;
  float* O = static_cast<float*>(p.out);
  merge_sum<D, NW>(lds_f32, tile, r, g, f, o, [&](int row, int c, f32x4_t x) {
    if (q0 + row >= p.N) return;
    const size_t bq = (size_t)b * p.N + q0 + row;
    *reinterpret_cast<f32x4_t*>(O + bq * p.o_stride + (size_t)h * D + c) = x;
    if (p.out_f32) *reinterpret_cast<f32x4_t*>(p.out_f32 + (bq * p.H + h) * D + c) = x;
  });
}

// dQ~ = tau dS V for 16 query rows of one head per workgroup; forms Dd =
// rowsum(dO * O) for its rows and publishes it for the dV kernel.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void bwd_dq_f32_kernel(BwdParams p) {
  constexpr int S = D / 16;
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int nq = (p.N + 15) / 16, blk = p.block0 + blockIdx.y;
  const int q0 = (p.causal ? nq - 1 - blk : blk) * 16;
  const int h = blockIdx.x, b = blockIdx.z, kg = h / (p.H / p.G);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const tile = lds_f32 + wave * Block<D>::FLOATS;
  const float* V = static_cast<const float*>(p.v) + (size_t)b * p.N * p.v_stride + (size_t)kg * D;

  const int nblk = ((p.causal ? min(q0 + 16, p.N) : p.N) + 15) / 16;
  f32x4_t v[S], q[S], go[S], acc[S];
  if (wave < nblk) load_rows<D>(V, p.v_stride, wave * 16 + r, p.N, g, v);
  load_rows<D>(static_cast<const float*>(p.q) + (size_t)b * p.N * p.q_stride + (size_t)h * D,
               p.q_stride, q0 + r, p.N, g, q);
  const size_t orow = (size_t)b * p.N;
  load_rows<D>(static_cast<const float*>(p.dout) + orow * p.o_stride + (size_t)h * D, p.o_stride,
               q0 + r, p.N, g, go);
  const int qc = min(q0 + r, p.N - 1);
  const size_t row = ((size_t)b * p.H + h) * p.N + qc;
  const float lse2 = p.lse[row] * kLog2e;
  // Dd from the forward's fp32 output when it was kept in its own tensor (which
  // need not be aligned), else from the output, fp32 as well.
  const float* O = p.out_f32 ? p.out_f32 + ((orow + qc) * p.H + h) * D
                             : static_cast<const float*>(p.out) + (orow + qc) * p.o_stride + (size_t)h * D;
  float dd = 0.f;
#pragma unroll
  for (int s = 0; s < S; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      dd = fmaf(O[16 * s + 4 * g + j], go[s][j], dd);
      q[s][j] *= p.scale_log2;
      acc[s][j] = 0.f;
    }
  dd += __shfl_xor(dd, 16);
  dd += __shfl_xor(dd, 32);
  if (wave == 0 && g == 0 && q0 + r < p.N) p.Dd[row] = dd;

  for (int t = wave; t < nblk; t += NW) {
    const int j0 = t * 16;
    stage_rows<D>(tile, r, g, v);
    const f32x4_t sc = dot_rows<D>(v, q, f32x4_t{0.f, 0.f, 0.f, 0.f});
    const f32x4_t dp = dot_rows<D>(v, go, f32x4_t{0.f, 0.f, 0.f, 0.f});
    const bool diag = p.causal && j0 + 15 > q0;
    const bool apart = diag && any_not_finite<D>(v);
    if (t + NW < nblk) load_rows<D>(V, p.v_stride, j0 + NW * 16 + r, p.N, g, v);
    f32x4_t ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int j = j0 + 4 * g + i;
      ds[i] = fast_exp2(sc[i] - lse2) * (dp[i] - dd);
      if (j >= p.N || (p.causal && j > q0 + r)) ds[i] = 0.f;
    }
    if (apart) add_weighted_seen<D>(tile, r, g, ds, 0, q0 + r - j0, acc);
    else add_weighted<D>(tile, r, g, ds, acc);
  }
  float* out = static_cast<float*>(p.dq);
  merge_sum<D, NW>(lds_f32, tile, r, g, p.scale, acc, [&](int rr, int c, f32x4_t x) {
    if (q0 + rr < p.N)
      *reinterpret_cast<f32x4_t*>(out + (orow + q0 + rr) * p.dq_stride + (size_t)h * D + c) = x;
  });
}

// dV = P^T dO + tau dS^T Q~ for 16 value rows of one group per workgroup; the
// waves share the (head of the group, query block) pairs.
template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2) void bwd_dv_f32_kernel(BwdParams p) {
  constexpr int S = D / 16;
  extern __shared__ __attribute__((aligned(16))) float lds_f32[];
  const int kv0 = (p.block0 + blockIdx.y) * 16;  // block 0 is the heaviest under the causal mask
  const int kg = blockIdx.x, b = blockIdx.z, R = p.H / p.G;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float* const tq = lds_f32 + wave * 2 * Block<D>::FLOATS;
  float* const tg = tq + Block<D>::FLOATS;
  const float* Q = static_cast<const float*>(p.q) + (size_t)b * p.N * p.q_stride;
  const float* dO = static_cast<const float*>(p.dout) + (size_t)b * p.N * p.o_stride;
  const int qb0 = p.causal ? kv0 / 16 : 0;
  const int per_head = (p.N + 15) / 16 - qb0, items = R * per_head;
  f32x4_t v[S], q[S], go[S], acc[S];
  float lse[4], dd[4];
  auto load = [&](int it) {
    const int h = kg * R + it / per_head, q0 = (qb0 + it % per_head) * 16;
    load_rows<D>(Q + (size_t)h * D, p.q_stride, q0 + r, p.N, g, q);
    load_rows<D>(dO + (size_t)h * D, p.o_stride, q0 + r, p.N, g, go);
    const size_t row = ((size_t)b * p.H + h) * p.N;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int qq = min(q0 + 4 * g + i, p.N - 1);
      lse[i] = p.lse[row + qq];
      dd[i] = p.Dd[row + qq];
    }
  };
  if (wave < items) load(wave);
  load_rows<D>(static_cast<const float*>(p.v) + (size_t)b * p.N * p.v_stride + (size_t)kg * D,
               p.v_stride, kv0 + r, p.N, g, v);
#pragma unroll
  for (int s = 0; s < S; ++s) acc[s] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int it = wave; it < items; it += NW) {
    const int q0 = (qb0 + it % per_head) * 16;
    stage_rows<D>(tq, r, g, q);
    stage_rows<D>(tg, r, g, go);
    const f32x4_t sc = dot_rows<D>(q, v, f32x4_t{0.f, 0.f, 0.f, 0.f});
    const f32x4_t dp = dot_rows<D>(go, v, f32x4_t{0.f, 0.f, 0.f, 0.f});
    const bool diag = p.causal && q0 < kv0 + 15;
    const bool apart = diag && (any_not_finite<D>(q) | any_not_finite<D>(go));
    f32x4_t pr, ds;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int qq = q0 + 4 * g + i;
      pr[i] = fast_exp2(fmaf(sc[i], p.scale_log2, -lse[i] * kLog2e));
      ds[i] = pr[i] * (dp[i] - dd[i]) * p.scale;
      if (qq >= p.N || (p.causal && qq < kv0 + r)) pr[i] = ds[i] = 0.f;
    }
    if (it + NW < items) load(it + NW);
    if (apart) {
      add_weighted_seen<D>(tg, r, g, pr, kv0 + r - q0, 15, acc);
      add_weighted_seen<D>(tq, r, g, ds, kv0 + r - q0, 15, acc);
    } else {
      add_weighted<D>(tg, r, g, pr, acc);
      add_weighted<D>(tq, r, g, ds, acc);
    }
  }
  // The waves' results through their first tiles' places, packed.
  __syncthreads();
  float* out = static_cast<float*>(p.dv);
  merge_sum<D, NW>(lds_f32, lds_f32 + wave * Block<D>::FLOATS, r, g, 1.f, acc,
                   [&](int rr, int c, f32x4_t x) {
    if (kv0 + rr < p.N)
      *reinterpret_cast<f32x4_t*>(out + ((size_t)b * p.N + kv0 + rr) * p.dv_stride + (size_t)kg * D + c) = x;
  });
}

// Waves per workgroup: eight share a block's work (two per SIMD at the kernels'
// registers); the results of all are merged once.
constexpr int kNW = 8;
constexpr int kMaxGridY = 65535;

template <class K, class P>
hipError_t launch(K kern, const P& p, dim3 grid, int lds, std::atomic<uint32_t>& done, hipStream_t st) {
  hipError_t e = set_max_lds(reinterpret_cast<const void*>(kern), lds, done);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(kNW * 64), lds, st, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_fwd(const AttnParams& p, hipStream_t st) {
  static std::atomic<uint32_t> done{0};
  return launch(attn_f32_kernel<D, kNW>, p, dim3(p.H, (p.N + 15) / 16, p.B),
                kNW * Block<D>::FLOATS * 4, done, st);
}

template <int D>
hipError_t launch_bwd(const BwdParams& p, hipStream_t st) {
  static std::atomic<uint32_t> done_q{0}, done_v{0};
  // A grid takes 65535 row blocks; above a million rows both kernels run in several
  // launches. dV reads the Dd of every query, so all of dQ~ runs first.
  const int nblk = (p.N + 15) / 16;
  auto all = [&](auto kern, int heads, int lds, std::atomic<uint32_t>& done) {
    hipError_t e = hipSuccess;
    BwdParams q = p;
    for (q.block0 = 0; q.block0 < nblk && e == hipSuccess; q.block0 += kMaxGridY)
      e = launch(kern, q, dim3(heads, std::min(nblk - q.block0, kMaxGridY), p.B), lds, done, st);
    return e;
  };
  const hipError_t e = all(bwd_dq_f32_kernel<D, kNW>, p.H, kNW * Block<D>::FLOATS * 4, done_q);
  if (e != hipSuccess) return e;
  return all(bwd_dv_f32_kernel<D, kNW>, p.G, 2 * kNW * Block<D>::FLOATS * 4, done_v);
}

bool aligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

bool attn_f32_supported(const AttnParams& p) {
  // Up to four rows on four (64 wide: eight): one or two updates of the vector-ALU
  // kernel, which has no merge. 8 heads, causal, us (that kernel / here): 64 wide, one
  // row 3.4 / 4.0, eight 3.8 / 4.0, sixteen 4.5 / 4.0; 128 wide, four 5.0 / 5.5, eight 5.7 /
  // 5.7 (unmasked 5.7 / 5.3).
  const int few = p.D == 64 ? 8 : 4;
  if (p.N <= few && p.Nk <= few && p.H <= 65535) return false;
  return p.dtype == KL_F32 && (p.D == 64 || p.D == 128) && p.Nk > 0 && p.q_stride % 4 == 0 &&
         p.v_stride % 4 == 0 && p.o_stride % 4 == 0 && aligned(p.q) && aligned(p.v) &&
         aligned(p.out) && aligned(p.out_f32) && (p.N + 15) / 16 <= kMaxGridY;
}

hipError_t launch_attention_f32(const AttnParams& p, hipStream_t st) {
  if (p.N == 0 || p.B == 0) return hipSuccess;
  if (p.causal && p.Nk != p.N) return hipErrorInvalidValue;
  return p.D == 128 ? launch_fwd<128>(p, st) : launch_fwd<64>(p, st);
}

hipError_t launch_attention_backward_f32(const BwdParams& p, hipStream_t st) {
  if (p.B == 0 || p.N == 0) return hipSuccess;
  return p.D == 128 ? launch_bwd<128>(p, st) : launch_bwd<64>(p, st);
}

}  // namespace kl
