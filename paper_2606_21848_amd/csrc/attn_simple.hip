// Vector-ALU keyless attention (fp32 arithmetic), for what the matrix-core
// kernels do not take: no value rows, a few fp32 rows, fp32 operands that are
// not 16-byte aligned, strides past their limits. A flash-style kernel where one
// LDS tile of values serves both the scores (Eq. 4) and the weighted sum, 16
// lanes per query row.

#include "kl_device.h"
#include "kl_internal.h"

namespace kl {
namespace {

template <typename T>
__device__ __forceinline__ float ld(const T* p, size_t i);
template <>
__device__ __forceinline__ float ld<float>(const float* p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float ld<uint16_t>(const uint16_t* p, size_t i) {
  return __uint_as_float((uint32_t)p[i] << 16);
}
template <typename T>
__device__ __forceinline__ void st(T* p, size_t i, float v);
template <>
__device__ __forceinline__ void st<float>(float* p, size_t i, float v) { p[i] = v; }
template <>
__device__ __forceinline__ void st<uint16_t>(uint16_t* p, size_t i, float v) {
  p[i] = (uint16_t)f32_to_bf16(v);
}

// A workgroup of 4 waves owns 16 query rows of one head; each query row
// has 16 lanes, lane c holding columns c E .. c E + E - 1 (E = D / 16) of the
// routed query and of the running output. Value tiles of 64 rows are staged in
// LDS once and serve both the scores (Eq. 4) and the weighted sum; a score is
// the lanes' partial dot products summed over the 16 lanes, and the online
// softmax (m, l, acc) is updated once per value row.
constexpr int SQ_ROWS = 16;  // query rows per workgroup
constexpr int SV_ROWS = 64;  // value rows per staged tile

template <typename T, int D>
__global__ __launch_bounds__(256) void attn_simple_kernel(AttnParams p) {
  constexpr int E = D / 16;
  typedef float f32xE __attribute__((ext_vector_type(E)));
  const int i0 = blockIdx.x * SQ_ROWS;
  const int h = blockIdx.y, b = blockIdx.z;
  const int g = h / (p.H / p.G);
  const int t = threadIdx.x, c = t & 15;
  const int i = i0 + (t >> 4);  // this lane group's query row
  const T* Q = reinterpret_cast<const T*>(p.q);
  const T* V = reinterpret_cast<const T*>(p.v);
  __shared__ __attribute__((aligned(16))) float sV[SV_ROWS][D];
  const bool live = i < p.N;
  f32xE q, acc;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    q[e] = live ? ld(Q, ((size_t)b * p.N + i) * p.q_stride + (size_t)h * D + c * E + e) * p.scale_log2
                : 0.f;
    acc[e] = 0.f;
  }
  float m = -INFINITY, l = 0.f;
  // Rows this lane group sees, and the rows any group of the workgroup sees.
  const int seen = live ? (p.causal ? min(i + 1, p.Nk) : p.Nk) : 0;
  const int jend = p.causal ? min(p.Nk, min(p.N, i0 + SQ_ROWS)) : p.Nk;
  for (int j0 = 0; j0 < jend; j0 += SV_ROWS) {
    __syncthreads();
    for (int e = t; e < SV_ROWS * D; e += 256) {
      const int jj = e / D, cc = e % D;
      const int j = j0 + jj;
      sV[jj][cc] = (j < p.Nk) ? ld(V, ((size_t)b * p.Nk + j) * p.v_stride + (size_t)g * D + cc) : 0.f;
    }
    __syncthreads();
    // Four value rows per update: four independent score chains, one rescale.
    // Rows past what this group sees (or past the tile's end) get no weight,
    // and their values are replaced by zeros so that nothing non-finite in them
    // can reach the sum.
    const int jn = min(SV_ROWS, jend - j0);
    for (int jj = 0; jj < jn; jj += 4) {
      f32xE v[4];
      float s[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = *reinterpret_cast<const f32xE*>(&sV[jj + u][c * E]);
        s[u] = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) s[u] = fmaf(q[e], v[u][e], s[u]);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s[u] = group_sum<16>(s[u]);
        if (j0 + jj + u >= seen || jj + u >= jn) {
          s[u] = -INFINITY;
          v[u] = f32xE{};
        }
      }
      const float mn = fmaxf(fmaxf(m, fmaxf(s[0], s[1])), fmaxf(s[2], s[3]));
      const float ms = mn == -INFINITY ? 0.f : mn;  // nothing seen yet: no shift
      const float alpha = fast_exp2(m - ms);
      float w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = fast_exp2(s[u] - ms);
      l = fmaf(l, alpha, (w[0] + w[1]) + (w[2] + w[3]));
#pragma unroll
      for (int e = 0; e < E; ++e)
        acc[e] = fmaf(w[3], v[3][e], fmaf(w[2], v[2][e], fmaf(w[1], v[1][e], fmaf(w[0], v[0][e], acc[e] * alpha))));
      m = mn;
    }
  }
  if (live) {
    T* O = reinterpret_cast<T*>(p.out);
    const float inv = l > 0.f ? 1.f / l : 0.f;  // no value rows: a zero row
    if (p.lse && c == 0)  // m and the scores are in log2 units
      p.lse[((size_t)b * p.H + h) * p.N + i] =
          l > 0.f ? (m + __log2f(l)) * 0.69314718055994531f : -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e)
      st(O, ((size_t)b * p.N + i) * p.o_stride + (size_t)h * D + c * E + e, acc[e] * inv);
    if (p.out_f32) {
#pragma unroll
      for (int e = 0; e < E; ++e)
        p.out_f32[(((size_t)b * p.N + i) * p.H + h) * D + c * E + e] = acc[e] * inv;
    }
  }
}

}  // namespace

hipError_t launch_prefill_attention_simple(const AttnParams& p, hipStream_t st) {
  if (p.N == 0 || p.B == 0) return hipSuccess;
  if (p.Nk < 0 || (p.causal && p.Nk != p.N)) return hipErrorInvalidValue;
  dim3 grid((p.N + SQ_ROWS - 1) / SQ_ROWS, p.H, p.B);
  if (p.dtype == KL_BF16) {
    if (p.D == 64) hipLaunchKernelGGL((attn_simple_kernel<uint16_t, 64>), grid, dim3(256), 0, st, p);
    else if (p.D == 128) hipLaunchKernelGGL((attn_simple_kernel<uint16_t, 128>), grid, dim3(256), 0, st, p);
    else return hipErrorInvalidValue;
  } else {
    if (p.D == 64) hipLaunchKernelGGL((attn_simple_kernel<float, 64>), grid, dim3(256), 0, st, p);
    else if (p.D == 128) hipLaunchKernelGGL((attn_simple_kernel<float, 128>), grid, dim3(256), 0, st, p);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace kl
