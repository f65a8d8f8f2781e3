// LayerNorm and GELU of the transformer-block stage (gfx950): token-major
// [T][C] bf16 activations; one wave per token for the LayerNorm, each lane
// holding whole 8-channel vectors in registers; statistics in fp32.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "tkernels.hpp"

namespace pulse {

namespace {

constexpr int LN_VEC = 4;        // 8-channel vectors per lane: C <= 64 * 8 * LN_VEC = 2048
constexpr int LN_BLOCKS = 512;   // of the backward pass: two per CU

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__device__ __forceinline__ void up8bf(const uint4& q, float v[8]) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

__device__ __forceinline__ void ld8bf(const uint16_t* p, float v[8]) {
  up8bf(*reinterpret_cast<const uint4*>(p), v);
}

__device__ __forceinline__ void st8bf(uint16_t* p, const float v[8]) {
  uint4 q;
  q.x = pack2(v[0], v[1]);
  q.y = pack2(v[2], v[3]);
  q.z = pack2(v[4], v[5]);
  q.w = pack2(v[6], v[7]);
  *reinterpret_cast<uint4*>(p) = q;
}

// y = (x - mean) * rstd * g + b per token; stats[t] = (mean, rstd)
__global__ __launch_bounds__(256) void k_ln_fwd(const uint16_t* x, long T, int C, float eps,
                                                const float* g, const float* b, uint16_t* y,
                                                float2* stats) {
  const long t = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (t >= T) return;
  const int nv = C / 8;
  float v[LN_VEC][8];
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < LN_VEC; ++j) {
    const int vi = lane + 64 * j;
    if (vi < nv) {
      ld8bf(x + t * C + vi * 8, v[j]);
#pragma unroll
      for (int i = 0; i < 8; ++i) s += v[j][i];
    }
  }
  const float mean = wave_sum(s) / C;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < LN_VEC; ++j)
    if (lane + 64 * j < nv)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float d = v[j][i] - mean;
        q += d * d;
      }
  const float rstd = rsqrtf(wave_sum(q) / C + eps);
#pragma unroll
  for (int j = 0; j < LN_VEC; ++j) {
    const int vi = lane + 64 * j;
    if (vi < nv) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = (v[j][i] - mean) * rstd * g[vi * 8 + i] + b[vi * 8 + i];
      st8bf(y + t * C + vi * 8, o);
    }
  }
  if (lane == 0) stats[t] = make_float2(mean, rstd);
}

// dx = add + rstd * (dxh - mean(dxh) - xh * mean(dxh * xh)), dxh = dy * g.
// A wave takes every (4 x blocks)-th token, the next token's rows in flight
// while the current one is reduced, and keeps its column sums of dy * xh, dy
// and dx (as stored) in registers over its tokens; the block's four waves
// meet in LDS and part[block][3][C] receives those sums.  Bound by HBM (three
// rows read, one written per token).  NV, the 8-channel vectors per lane, is
// the width's own: with registers for 2048 channels and one token per wave,
// 4096 tokens of 768 channels wrote as many bytes of partials as of
// activations and found little room beside the weight GEMMs of the other
// stream: 34.6 us there on average against 16.5 now (10 us alone; 1408
// channels, 8192 tokens: 39 -> 31 us alone).
template <int NV>
__global__ __launch_bounds__(256) void k_ln_bwd(const uint16_t* dy, const uint16_t* x,
                                                const float2* stats, const float* g,
                                                const uint16_t* add, long T, int C, uint16_t* dx,
                                                float* part) {
  __shared__ float sm[3][4][64 * 8];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int nv = C / 8;
  const long step = (long)gridDim.x * 4;
  float acc[3][NV][8];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[r][j][i] = 0.f;
  uint4 xr[NV], dr[NV], ar[NV];
  float2 st = make_float2(0.f, 0.f);
  auto load = [&](long t) __attribute__((always_inline)) {
    st = stats[t];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int vi = min(lane + 64 * j, nv - 1);  // lanes past the row reload its end
      xr[j] = *reinterpret_cast<const uint4*>(x + t * C + vi * 8);
      dr[j] = *reinterpret_cast<const uint4*>(dy + t * C + vi * 8);
      if (add) ar[j] = *reinterpret_cast<const uint4*>(add + t * C + vi * 8);
    }
  };
  long t = (long)blockIdx.x * 4 + w;
  if (t < T) load(t);
  for (; t < T; t += step) {
    float xh[NV][8], gy[NV][8], a[NV][8];
    float s1 = 0.f, s2 = 0.f;
    const float rs = st.y;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int vi = lane + 64 * j;
      float dv[8];
      up8bf(xr[j], xh[j]);
      up8bf(dr[j], dv);
#pragma unroll
      for (int i = 0; i < 8; ++i) a[j][i] = 0.f;
      if (add) up8bf(ar[j], a[j]);
      if (vi < nv) {
        const float4 g0 = reinterpret_cast<const float4*>(g)[2 * vi];
        const float4 g1 = reinterpret_cast<const float4*>(g)[2 * vi + 1];
        const float gv[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          xh[j][i] = (xh[j][i] - st.x) * rs;
          gy[j][i] = dv[i] * gv[i];
          s1 += gy[j][i];
          s2 += gy[j][i] * xh[j][i];
          acc[0][j][i] += dv[i] * xh[j][i];
          acc[1][j][i] += dv[i];
        }
      }
    }
    if (t + step < T) load(t + step);
    const float m1 = wave_sum(s1) / C, m2 = wave_sum(s2) / C;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int vi = lane + 64 * j;
      if (vi < nv) {
        float o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          o[i] = a[j][i] + rs * (gy[j][i] - m1 - xh[j][i] * m2);
          acc[2][j][i] += bf2f(f2bf(o[i]));  // the value as stored
        }
        st8bf(dx + t * C + vi * 8, o);
      }
    }
  }
  // the four waves' column sums, in wave order, one vector slice at a time
  float* out = part + (long)blockIdx.x * 3 * C;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (j) __syncthreads();
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int i = 0; i < 8; ++i) sm[r][w][lane + 64 * i] = acc[r][j][i];
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * 512; e += 256) {
      const int r = e >> 9, c = e & 511;  // column c of this slice
      if (j * 512 + c >= C) continue;
      const int at = (c >> 3) + 64 * (c & 7);
      float s = sm[r][0][at];
#pragma unroll
      for (int ww = 1; ww < 4; ++ww) s += sm[r][ww][at];
      out[(long)r * C + j * 512 + c] = s;
    }
  }
}

// dg += row 0, db += row 1, dsum (or null) += row 2 of part[rows][3][C]: 8
// columns x 32 row lanes per block, each lane's rows in ascending order (8
// loads in flight), the lanes in a fixed tree.
__global__ __launch_bounds__(256) void k_ln_totals(const float* part, int rows, int C, float* dg,
                                                   float* db, float* dsum) {
  __shared__ float sm[32][8];
  const int tx = threadIdx.x & 7, ty = threadIdx.x >> 3;
  const int r = blockIdx.y, c = blockIdx.x * 8 + tx;
  const float* p = part + (long)r * C + c;
  float s = 0.f;
  constexpr int NB = 8;
  for (int i0 = ty; i0 < rows; i0 += NB * 32) {
    float v[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) v[k] = i0 + 32 * k < rows ? p[(long)(i0 + 32 * k) * 3 * C] : 0.f;
#pragma unroll
    for (int k = 0; k < NB; ++k) s += v[k];
  }
  sm[ty][tx] = s;
  __syncthreads();
  for (int off = 16; off > 0; off >>= 1) {
    if (ty < off) sm[ty][tx] += sm[ty + off][tx];
    __syncthreads();
  }
  if (ty == 0) {
    float* dst = r == 0 ? dg : (r == 1 ? db : dsum);
    dst[c] += sm[0][tx];
  }
}

__global__ __launch_bounds__(256) void k_gelu_fwd(const uint16_t* z, uint16_t* m, long n8) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n8;
       i += (long)gridDim.x * blockDim.x) {
    float v[8];
    ld8bf(z + i * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = gelu_f(v[k]);
    st8bf(m + i * 8, v);
  }
}

__global__ __launch_bounds__(256) void k_gelu_bwd(const uint16_t* dm, const uint16_t* z,
                                                  uint16_t* dz, long n8) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n8;
       i += (long)gridDim.x * blockDim.x) {
    float a[8], v[8];
    ld8bf(dm + i * 8, a);
    ld8bf(z + i * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) a[k] *= gelu_d(v[k]);
    st8bf(dz + i * 8, a);
  }
}

unsigned grid_of(long n, long cap = 8192) {
  long b = (n + 255) / 256;
  return (unsigned)(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

int ln_bwd_blocks(long T) { return (int)std::min<long>((T + 3) / 4, LN_BLOCKS); }

hipError_t launch_ln_fwd(const void* x, long T, int C, float eps, const float* g, const float* b,
                         void* y, float* stats, hipStream_t st) {
  if (C % 8 || C > 64 * 8 * LN_VEC) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_ln_fwd, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st,
                     static_cast<const uint16_t*>(x), T, C, eps, g, b, static_cast<uint16_t*>(y),
                     reinterpret_cast<float2*>(stats));
  return hipGetLastError();
}

hipError_t launch_ln_bwd(const void* dy, const void* x, const float* stats, const float* g,
                         const void* add, long T, int C, void* dx, float* part, hipStream_t st,
                         hipEvent_t done) {
  if (C % 8 || C > 64 * 8 * LN_VEC) return hipErrorInvalidValue;
  auto kern = C <= 512 ? k_ln_bwd<1> : C <= 1024 ? k_ln_bwd<2> : C <= 1536 ? k_ln_bwd<3>
                                                                            : k_ln_bwd<4>;
  const dim3 grid((unsigned)ln_bwd_blocks(T)), block(256);
  const uint16_t* d = static_cast<const uint16_t*>(dy);
  const uint16_t* xi = static_cast<const uint16_t*>(x);
  const float2* ss = reinterpret_cast<const float2*>(stats);
  const uint16_t* ad = static_cast<const uint16_t*>(add);
  uint16_t* o = static_cast<uint16_t*>(dx);
  if (done)  // the event completes with the kernel (no marker packet of its own)
    hipExtLaunchKernelGGL(kern, grid, block, 0, st, nullptr, done, 0, d, xi, ss, g, ad, T, C, o,
                          part);
  else
    hipLaunchKernelGGL(kern, grid, block, 0, st, d, xi, ss, g, ad, T, C, o, part);
  return hipGetLastError();
}

hipError_t launch_ln_totals(const float* part, int rows, int C, float* dg, float* db, float* dsum,
                            hipStream_t st) {
  hipLaunchKernelGGL(k_ln_totals, dim3(C / 8, dsum ? 3 : 2), dim3(256), 0, st, part, rows, C, dg,
                     db, dsum);
  return hipGetLastError();
}

hipError_t launch_gelu_fwd(const void* z, void* m, long n, hipStream_t st) {
  if (n % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gelu_fwd, dim3(grid_of(n / 8)), dim3(256), 0, st,
                     static_cast<const uint16_t*>(z), static_cast<uint16_t*>(m), n / 8);
  return hipGetLastError();
}


hipError_t launch_gelu_bwd(const void* dm, const void* z, void* dz, long n, hipStream_t st) {
  if (n % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gelu_bwd, dim3(grid_of(n / 8)), dim3(256), 0, st,
                     static_cast<const uint16_t*>(dm), static_cast<const uint16_t*>(z),
                     static_cast<uint16_t*>(dz), n / 8);
  return hipGetLastError();
}

}  // namespace pulse
