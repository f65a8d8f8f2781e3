// LayerNorm and GELU of the transformer-block stage (gfx950): token-major
// [T][C] bf16 activations; one wave per token for the LayerNorm, each lane
// holding whole 8-channel vectors in registers; statistics in fp32.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "tkernels.hpp"

namespace pulse {

namespace {

constexpr int LN_VEC = 4;        // 8-channel vectors per lane: C <= 64 * 8 * LN_VEC = 2048
constexpr int LN_BLOCKS = 512;   // of the backward pass, at most: two per CU

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
// WR waves hold one token's row, 8 channels per lane, so that a lane's column
// sums of dy * xh, dy and dx (as stored), kept over the tokens of its row
// group, take 24 registers whatever the width: the kernel stays within the 96
// that a weight-gradient GEMM of the other stream (two waves of 208 per SIMD)
// leaves, instead of waiting for its blocks to end.  A block holds RG row
// groups; the next token's rows are in flight while the current one is
// reduced (wave shuffles, then the WR waves through LDS, one barrier per
// token).  part[block][3][C] receives the block's column sums.  Bound by HBM:
// three rows read, one written per token.
template <int WR, int RG>
__global__ __launch_bounds__(64 * WR * RG, 5) void k_ln_bwd(const uint16_t* dy, const uint16_t* x,
                                                            const float2* stats, const float* g,
                                                            const uint16_t* add, int T, int C,
                                                            uint16_t* dx, float* part) {
  __shared__ float2 red[2][RG][WR];
  __shared__ float sm[RG > 1 ? RG * 3 * WR * 512 : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wr = wave % WR, rg = wave / WR;
  const int nv = C / 8, vi = wr * 64 + lane;
  const bool on = vi < nv;
  const int vc = (on ? vi : nv - 1) * 8;  // lanes past the row reload its end
  const int step = gridDim.x * RG;
  float acc[3][8], gv[8];
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[r][i] = 0.f;
  {
    const float4 g0 = reinterpret_cast<const float4*>(g + vc)[0];
    const float4 g1 = reinterpret_cast<const float4*>(g + vc)[1];
    gv[0] = g0.x; gv[1] = g0.y; gv[2] = g0.z; gv[3] = g0.w;
    gv[4] = g1.x; gv[5] = g1.y; gv[6] = g1.z; gv[7] = g1.w;
  }
  uint4 xr, dr, ar = {0u, 0u, 0u, 0u};
  float2 st;
  // every row group runs the same count of steps (a barrier each); past T
  // the loads repeat the last token and nothing is stored or summed
  auto load = [&](int t) __attribute__((always_inline)) {
    const int tc = t < T ? t : T - 1;
    const int e = tc * C + vc;  // T * C elements stay below 2^30
    st = stats[tc];
    xr = *reinterpret_cast<const uint4*>(x + e);
    dr = *reinterpret_cast<const uint4*>(dy + e);
    if (add) ar = *reinterpret_cast<const uint4*>(add + e);
  };
  int t = blockIdx.x * RG + rg;
  load(t);
  int buf = 0;
#pragma unroll 1
  for (int tb = blockIdx.x * RG; tb < T; tb += step, t += step, buf ^= 1) {
    float xh[8], gy[8];
    float s1 = 0.f, s2 = 0.f;
    const float rs = st.y;
    const bool ok = on && t < T;
    const uint4 ac = ar;
    up8bf(xr, xh);
    up8bf(dr, gy);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      xh[i] = (xh[i] - st.x) * rs;
      const float d = ok ? gy[i] : 0.f;
      acc[0][i] += d * xh[i];
      acc[1][i] += d;
      gy[i] = d * gv[i];
      s1 += gy[i];
      s2 += gy[i] * xh[i];
    }
    if (tb + step < T) load(t + step);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if constexpr (WR > 1) {
      if (lane == 0) red[buf][rg][wr] = make_float2(s1, s2);
      __syncthreads();
      s1 = s2 = 0.f;
#pragma unroll
      for (int q = 0; q < WR; ++q) {
        s1 += red[buf][rg][q].x;
        s2 += red[buf][rg][q].y;
      }
    }
    const float m1 = s1 / C, m2 = s2 / C;
    if (ok) {
      float o[8];
      up8bf(ac, o);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        o[i] += rs * (gy[i] - m1 - xh[i] * m2);
        acc[2][i] += bf2f(f2bf(o[i]));  // the value as stored
      }
      st8bf(dx + (t * C + vc), o);
    }
  }
  float* out = part + (long)blockIdx.x * 3 * C;
  if constexpr (RG == 1) {
    if (on) {
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        float4* p = reinterpret_cast<float4*>(out + (long)r * C + vc);
        p[0] = make_float4(acc[r][0], acc[r][1], acc[r][2], acc[r][3]);
        p[1] = make_float4(acc[r][4], acc[r][5], acc[r][6], acc[r][7]);
      }
    }
  } else {
    // the row groups' sums, in group order (element i of lane l at 64 i + l)
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        sm[((rg * 3 + r) * WR + wr) * 512 + 64 * i + lane] = acc[r][i];
    __syncthreads();
    for (int e = threadIdx.x; e < 3 * C; e += 64 * WR * RG) {
      const int r = e / C, c = e - r * C;
      const int at = (r * WR + (c >> 9)) * 512 + 64 * (c & 7) + ((c & 511) >> 3);
      float s = sm[at];
#pragma unroll
      for (int q = 1; q < RG; ++q) s += sm[q * 3 * WR * 512 + at];
      out[e] = s;
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

namespace {
// waves per row and row groups per block of the backward for C channels
int ln_wr(int C) { return (C + 511) / 512; }
int ln_rg(int C) { return ln_wr(C) == 1 ? 4 : ln_wr(C) == 2 ? 2 : 1; }
}  // namespace

int ln_bwd_blocks(long T, int C) {
  return (int)std::min<long>((T + ln_rg(C) - 1) / ln_rg(C), LN_BLOCKS);
}

hipError_t launch_ln_fwd(const void* x, long T, int C, float eps, const float* g, const float* b,
                         void* y, float* stats, hipStream_t st) {
  if (C % 8 || C > 64 * 8 * LN_VEC) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_ln_fwd, dim3((unsigned)((T + 3) / 4)), dim3(256), 0, st,
                     static_cast<const uint16_t*>(x), T, C, eps, g, b, static_cast<uint16_t*>(y),
                     reinterpret_cast<float2*>(stats));
  return hipGetLastError();
}

hipError_t launch_ln_bwd(const void* dy, const void* x, const float* stats, const float* g,
                         const void* add, long T, int C, void* dx, float* part, hipStream_t st) {
  if (C % 8 || C > 64 * 8 * LN_VEC) return hipErrorInvalidValue;
  auto kern = C <= 512 ? k_ln_bwd<1, 4> : C <= 1024 ? k_ln_bwd<2, 2> : C <= 1536 ? k_ln_bwd<3, 1>
                                                                                  : k_ln_bwd<4, 1>;
  const dim3 grid((unsigned)ln_bwd_blocks(T, C)), block(64 * ln_wr(C) * ln_rg(C));
  const uint16_t* d = static_cast<const uint16_t*>(dy);
  const uint16_t* xi = static_cast<const uint16_t*>(x);
  const float2* ss = reinterpret_cast<const float2*>(stats);
  const uint16_t* ad = static_cast<const uint16_t*>(add);
  uint16_t* o = static_cast<uint16_t*>(dx);
  hipLaunchKernelGGL(kern, grid, block, 0, st, d, xi, ss, g, ad, (int)T, C, o, part);
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
