// Timestep-embedding projection, weight re-layouts and conversions (gfx950).
// All small or streaming; none is on the MFMA path.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace pulse {

namespace {

__device__ __forceinline__ float ld_any(const void* p, int dtype, long i) {
  return dtype == DT_BF16 ? bf2f(static_cast<const uint16_t*>(p)[i])
                          : static_cast<const float*>(p)[i];
}

__device__ __forceinline__ void st_any(void* p, int dtype, long i, float v) {
  if (dtype == DT_BF16)
    static_cast<uint16_t*>(p)[i] = f2bf(v);
  else
    static_cast<float*>(p)[i] = v;
}

// Every block's projection of one stage half in one launch.  Block
// (row tile, stage block k, image group) of 4 waves, each wave 2 rows o of
// Wl_k for 8 images.  Per slice of d every memory read is issued at once:
// the wave's Wl rows (16-byte loads into registers) and SiLU(temb) of the 8
// images (16-byte loads, activated into LDS); the lanes' 2 x 8 partial dot
// products then meet in LDS in a fixed order.  The blocks of the first row
// tile of stage block 0 also write the temb copy.
constexpr int TP_ROWS = 2;                      // rows per wave
constexpr int TP_IMG = 8;                       // images per block
constexpr int TP_DS = 2048;                     // d slice
constexpr int TP_J = TP_DS / 256;               // float4 loads per lane and row

__global__ __launch_bounds__(256) void k_temb_fwd_multi(const void* temb, int dtype, int B,
                                                        int D, TembFwdSet set, void* copy) {
  __shared__ __attribute__((aligned(16))) float st[TP_IMG][TP_DS];
  __shared__ float red[4][TP_ROWS * TP_IMG][65];
  const int k = blockIdx.y;
  const TembFwdBlock& blk = set.blk[k];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int b0 = blockIdx.z * TP_IMG;
  const int o0 = (blockIdx.x * 4 + wave) * TP_ROWS;
  const bool do_copy = copy && blockIdx.x == 0 && k == 0;
  const bool vec = dtype == DT_BF16 && (D % 8) == 0;
  float acc[TP_ROWS][TP_IMG];
#pragma unroll
  for (int r = 0; r < TP_ROWS; ++r)
#pragma unroll
    for (int i = 0; i < TP_IMG; ++i) acc[r][i] = 0.f;
  for (int dc = 0; dc < D; dc += TP_DS) {
    const int dn = min(TP_DS, D - dc);
    // the wave's weight rows, all loads in flight together
    float4 wv[TP_ROWS][TP_J];
#pragma unroll
    for (int r = 0; r < TP_ROWS; ++r) {
      const int o = min(o0 + r, blk.O - 1);
      const float* w = blk.Wl + (long)o * D + dc;
#pragma unroll
      for (int j = 0; j < TP_J; ++j) {
        const int d = 4 * lane + 256 * j;
        if ((D & 3) == 0 && d + 3 < dn) {
          wv[r][j] = *reinterpret_cast<const float4*>(w + d);
        } else {
          wv[r][j].x = d < dn ? w[d] : 0.f;
          wv[r][j].y = d + 1 < dn ? w[d + 1] : 0.f;
          wv[r][j].z = d + 2 < dn ? w[d + 2] : 0.f;
          wv[r][j].w = d + 3 < dn ? w[d + 3] : 0.f;
        }
      }
    }
    __syncthreads();  // the previous slice's LDS reads are done
    if (vec) {
      // 8-element pieces: TP_IMG * dn / 8 of them, at most 8 per thread
      constexpr int NP = TP_IMG * TP_DS / 8 / 256;
      uint4 q[NP];
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int e = threadIdx.x + 256 * j;
        const int i = e / (TP_DS / 8), d = (e - i * (TP_DS / 8)) * 8;
        q[j] = uint4{0u, 0u, 0u, 0u};
        if (b0 + i < B && d < dn)
          q[j] = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(temb) +
                                                 (long)(b0 + i) * D + dc + d);
      }
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int e = threadIdx.x + 256 * j;
        const int i = e / (TP_DS / 8), d = (e - i * (TP_DS / 8)) * 8;
        if (do_copy && b0 + i < B && d < dn)
          *reinterpret_cast<uint4*>(static_cast<uint16_t*>(copy) + (long)(b0 + i) * D + dc + d) =
              q[j];
        const uint32_t w4[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
        float v[8];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          v[2 * h] = silu_f(__uint_as_float(w4[h] << 16));
          v[2 * h + 1] = silu_f(__uint_as_float(w4[h] & 0xffff0000u));
        }
        if (!(b0 + i < B && d < dn)) {
#pragma unroll
          for (int h = 0; h < 8; ++h) v[h] = 0.f;
        }
        float4* dst = reinterpret_cast<float4*>(&st[i][d]);
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
      }
    } else {
      for (int e = threadIdx.x; e < TP_IMG * TP_DS; e += 256) {
        const int i = e / TP_DS, d = e - i * TP_DS;
        float v = 0.f;
        if (b0 + i < B && d < dn) {
          const long at = (long)(b0 + i) * D + dc + d;
          const float t = ld_any(temb, dtype, at);
          if (do_copy) st_any(copy, dtype, at, t);
          v = silu_f(t);
        }
        st[i][d] = v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TP_J; ++j) {
      const int d = 4 * lane + 256 * j;
      if (d >= dn) break;
#pragma unroll
      for (int i = 0; i < TP_IMG; ++i) {
        const float4 sv = *reinterpret_cast<const float4*>(&st[i][d]);
#pragma unroll
        for (int r = 0; r < TP_ROWS; ++r)
          acc[r][i] += wv[r][j].x * sv.x + wv[r][j].y * sv.y + wv[r][j].z * sv.z +
                       wv[r][j].w * sv.w;
      }
    }
  }
  // lane sums -> LDS; lane q < 16 of the wave then adds the 64 lanes of
  // (row q / 8, image q % 8) in order
#pragma unroll
  for (int r = 0; r < TP_ROWS; ++r)
#pragma unroll
    for (int i = 0; i < TP_IMG; ++i) red[wave][r * TP_IMG + i][lane] = acc[r][i];
  __syncthreads();
  if (lane < TP_ROWS * TP_IMG) {
    const int r = lane / TP_IMG, i = lane - r * TP_IMG;
    const int o = o0 + r, b = b0 + i;
    if (o < blk.O && b < B) {
      float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
      for (int l = 0; l < 64; l += 4) {
        s0 += red[wave][lane][l];
        s1 += red[wave][lane][l + 1];
        s2 += red[wave][lane][l + 2];
        s3 += red[wave][lane][l + 3];
      }
      float bias = blk.bias_a[o];
      if (blk.bias_b) bias += blk.bias_b[o];
      blk.e[(long)b * blk.ldE + o] = ((s0 + s1) + (s2 + s3)) + bias;
    }
  }
}

// dWl[o][d] += sum_b de[b][o] * SiLU(temb[b][d]) over a 64 (d) x 16 (o)
// tile per block: the tile's SiLU(temb) columns and de rows are staged in
// LDS for up to 32 images at a time (each SiLU evaluated once per tile, not
// once per output), and thread (d lane, row group g) owns rows 4 g .. 4 g + 3.
// The blocks of the first d tile also sum de over the images for the bias
// gradients.  Every sum runs over b in increasing order.
constexpr int TB_D = 64, TB_O = 16, TB_B = 32;
__global__ __launch_bounds__(256) void k_temb_bwd_w(const float* de, const void* temb, int dtype,
                                                    int B, int D, int O, float* dWl, float* dbl,
                                                    float* db1) {
  __shared__ float sv[TB_B][TB_D];
  __shared__ __attribute__((aligned(16))) float se[TB_B][TB_O];
  const int tx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int d0 = blockIdx.x * TB_D, o0 = blockIdx.y * TB_O;
  const bool bias = blockIdx.x == 0 && threadIdx.x < TB_O;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float sb = 0.f;
  for (int b0 = 0; b0 < B; b0 += TB_B) {
    const int nb = min(TB_B, B - b0);
    __syncthreads();
    for (int e = threadIdx.x; e < nb * TB_D; e += 256) {
      const int bb = e / TB_D, c = e - bb * TB_D;
      sv[bb][c] = d0 + c < D ? silu_f(ld_any(temb, dtype, (long)(b0 + bb) * D + d0 + c)) : 0.f;
    }
    for (int e = threadIdx.x; e < nb * TB_O; e += 256) {
      const int bb = e / TB_O, c = e - bb * TB_O;
      se[bb][c] = o0 + c < O ? de[(long)(b0 + bb) * O + o0 + c] : 0.f;
    }
    __syncthreads();
    for (int bb = 0; bb < nb; ++bb) {
      const float v = sv[bb][tx];
      const float4 w = reinterpret_cast<const float4*>(&se[bb][0])[g];
      acc[0] += w.x * v;
      acc[1] += w.y * v;
      acc[2] += w.z * v;
      acc[3] += w.w * v;
    }
    if (bias)
      for (int bb = 0; bb < nb; ++bb) sb += se[bb][threadIdx.x];
  }
  const int d = d0 + tx;
  if (d < D) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = o0 + 4 * g + j;
      if (o < O) dWl[(long)o * D + d] += acc[j];
    }
  }
  if (bias && o0 + threadIdx.x < O) {
    dbl[o0 + threadIdx.x] += sb;
    if (db1) db1[o0 + threadIdx.x] += sb;
  }
}

// block (64 d x 16 o-lanes) per (d block, image b):
// dtemb[b][d] += SiLU'(temb[b][d]) * sum_o Wl[o][d] de[b][o]
__global__ __launch_bounds__(1024) void k_temb_bwd_x(const float* de, const void* temb,
                                                     int dtype, int B, int D, int O,
                                                     const float* Wl, float* dtemb) {
  __shared__ float sm[16][64];
  const int d = blockIdx.x * 64 + threadIdx.x;
  const int b = blockIdx.y;
  float s = 0.f;
  if (d < D) {
    int o = threadIdx.y;
    for (; o + 48 < O; o += 64) {
      const float w0 = Wl[(long)o * D + d], w1 = Wl[(long)(o + 16) * D + d];
      const float w2 = Wl[(long)(o + 32) * D + d], w3 = Wl[(long)(o + 48) * D + d];
      s += w0 * de[(long)b * O + o];
      s += w1 * de[(long)b * O + o + 16];
      s += w2 * de[(long)b * O + o + 32];
      s += w3 * de[(long)b * O + o + 48];
    }
    for (; o < O; o += 16) s += Wl[(long)o * D + d] * de[(long)b * O + o];
  }
  sm[threadIdx.y][threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.y == 0 && d < D) {
    float t = sm[0][threadIdx.x];
#pragma unroll
    for (int y = 1; y < 16; ++y) t += sm[y][threadIdx.x];
    const long i = (long)b * D + d;
    dtemb[i] += t * dsilu_f(ld_any(temb, dtype, i));
  }
}

// Refresh of a stage's weight copies: one launch over a table of jobs, each
// 64 x 64 tile of an fp32 master [O][taps * C] read once (16-byte loads,
// coalesced) and written twice: the row-major compute copy straight from
// registers, and the data-gradient copy dst[c][taps - 1 - t][o] through LDS,
// so that its stores are 16-byte pieces of 8 consecutive o as well.  Bound
// by HBM: 4 bytes read and 2 x 2 written per bf16 weight.  The 161 M
// weights of a 1280-channel stage take 221-244 us in one launch (5.3-5.8
// TB/s); one kernel per copy with one element per thread, which read the
// master twice and, for the transposed copies, in strides of a whole row,
// took 1384 us in 26 launches.
// LDS rows of 65 floats: the 16-lane row pieces of the stores and the
// 8-row column pieces of the reads both touch 64 different banks.
constexpr int RF_T = 64;

template <int DT>
__global__ __launch_bounds__(256) void k_refresh(RefreshSet set) {
  __shared__ float sm[RF_T][RF_T + 1];
  int j = 0;
  while (j + 1 < set.n && (int)blockIdx.x >= set.job[j + 1].first) ++j;
  const RefreshJob& job = set.job[j];
  const int tile = (int)blockIdx.x - job.first;
  const int t = threadIdx.x;
  if (job.taps == 0) {  // fp32 vector: row = src + src2 (null: zero)
    const int i = tile * 256 + t;
    if (i < job.O)
      static_cast<float*>(job.row)[i] =
          (job.src ? job.src[i] : 0.f) + (job.src2 ? job.src2[i] : 0.f);
    return;
  }
  const int K = job.taps * job.C;
  const int tk = (K + RF_T - 1) / RF_T;
  const int o0 = tile / tk * RF_T, k0 = (tile - tile / tk * tk) * RF_T;
  const int kq = (t & 15) * 4;  // this thread's 4 columns
  float4 v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int o = o0 + (t >> 4) + 16 * i;
    v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (o < job.O && k0 + kq < K)
      v[i] = *reinterpret_cast<const float4*>(job.src + (long)o * K + k0 + kq);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = (t >> 4) + 16 * i;
    sm[r][kq] = v[i].x;
    sm[r][kq + 1] = v[i].y;
    sm[r][kq + 2] = v[i].z;
    sm[r][kq + 3] = v[i].w;
    if (o0 + r < job.O && k0 + kq < K) {
      const long e = (long)(o0 + r) * job.ldd + job.coff + k0 + kq;
      if constexpr (DT == DT_BF16)
        *reinterpret_cast<uint2*>(static_cast<uint16_t*>(job.row) + e) =
            make_uint2(pack2(v[i].x, v[i].y), pack2(v[i].z, v[i].w));
      else
        *reinterpret_cast<float4*>(static_cast<float*>(job.row) + e) = v[i];
    }
  }
  __syncthreads();
  const int oc = (t & 7) * 8;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int kk = (t >> 3) + 32 * i;
    if (k0 + kk >= K || o0 + oc >= job.O) continue;
    const int tap = (k0 + kk) / job.C, c = k0 + kk - tap * job.C;
    float w[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) w[q] = sm[oc + q][kk];
    st8(job.tr, DT, job.O, (long)c * job.taps + job.taps - 1 - tap, o0 + oc, w);
  }
}

// dst = (ddt) (a + b), a of dtype adt, b fp32
__global__ void k_add_cast(const void* a, int adt, const float* b, void* dst, int ddt, long n) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (long)gridDim.x * blockDim.x)
    st_any(dst, ddt, i, ld_any(a, adt, i) + b[i]);
}

// dst = a + b over n = 8 * n8 elements, 8 per thread per step (16- or
// 32-byte accesses); the element types are template arguments
template <int ADT, int DDT>
__global__ __launch_bounds__(256) void k_add_cast8(const void* a, const float* b, void* dst,
                                                   long n8) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n8;
       i += (long)gridDim.x * blockDim.x) {
    float v[8];
    ld8(Src{a, ADT, 8}, i, 0, v);
    const float4* q = reinterpret_cast<const float4*>(b) + 2 * i;
    const float4 b0 = q[0], b1 = q[1];
    v[0] += b0.x; v[1] += b0.y; v[2] += b0.z; v[3] += b0.w;
    v[4] += b1.x; v[5] += b1.y; v[6] += b1.z; v[7] += b1.w;
    st8(dst, DDT, 8, i, 0, v);
  }
}

}  // namespace

hipError_t launch_temb_fwd_multi(const void* temb, int dtype, int B, int D,
                                 const TembFwdSet& set, void* copy, hipStream_t st) {
  if (set.n < 1 || set.n > TEMB_MAX_BLOCKS) return hipErrorInvalidValue;
  int omax = 0;
  for (int k = 0; k < set.n; ++k) omax = std::max(omax, set.blk[k].O);
  const int rows_per_block = 4 * TP_ROWS;
  hipLaunchKernelGGL(k_temb_fwd_multi,
                     dim3((omax + rows_per_block - 1) / rows_per_block, set.n,
                          (B + TP_IMG - 1) / TP_IMG),
                     dim3(256), 0, st, temb, dtype, B, D, set, copy);
  return hipGetLastError();
}

hipError_t launch_temb_bwd(const float* de, const void* temb, int dtype, int B, int D, int O,
                           const float* Wl, float* dWl, float* dbl, float* db1, float* dtemb,
                           hipStream_t st) {
  if (O <= 0) return hipSuccess;
  // at least one d tile: its blocks also produce the bias gradients
  const int dt = std::max(1, (D + TB_D - 1) / TB_D);
  hipLaunchKernelGGL(k_temb_bwd_w, dim3(dt, (O + TB_O - 1) / TB_O), dim3(256), 0, st, de, temb,
                     dtype, B, D, O, dWl, dbl, db1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !dtemb) return e;
  hipLaunchKernelGGL(k_temb_bwd_x, dim3((D + 63) / 64, B), dim3(64, 16), 0, st, de, temb, dtype,
                     B, D, O, Wl, dtemb);
  return hipGetLastError();
}

hipError_t RefreshList::flush() {
  if (set_.n == 0) return hipSuccess;
  auto kern = dtype_ == DT_BF16 ? k_refresh<DT_BF16> : k_refresh<DT_F32>;
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks_), dim3(256), 0, st_, set_);
  set_.n = 0;
  blocks_ = 0;
  return hipGetLastError();
}

hipError_t RefreshList::add(RefreshJob job, long blocks) {
  hipError_t e = hipSuccess;
  // A full table goes first.  Its grid stays below 2^24 blocks, HIP's limit of
  // 2^32 threads: a 3x3 weight of 8192 by 8192 channels, the largest a stage
  // takes, has 147456.
  if (set_.n == REFRESH_MAX_JOBS) e = flush();
  job.first = (int)blocks_;
  set_.job[set_.n++] = job;
  blocks_ += blocks;
  return e;
}

hipError_t RefreshList::weight(const float* src, int O, int C, int taps, void* row, int ldd,
                               int coff, void* tr) {
  if (O % 8 || C % 4 || ldd % 4 || coff % 4) return hipErrorInvalidValue;
  RefreshJob j{};
  j.src = src;
  j.row = row;
  j.tr = tr;
  j.O = O;
  j.C = C;
  j.taps = taps;
  j.ldd = ldd;
  j.coff = coff;
  const long K = (long)taps * C;
  return add(j, ((O + RF_T - 1) / RF_T) * ((K + RF_T - 1) / RF_T));
}

hipError_t RefreshList::vec(const float* a, const float* b, float* dst, int n) {
  RefreshJob j{};
  j.src = a;
  j.src2 = b;
  j.row = dst;
  j.O = n;
  return add(j, (n + 255) / 256);
}

hipError_t launch_add_cast(const void* a, int adt, const float* b, void* dst, int ddt, long n,
                           hipStream_t st) {
  const bool aligned = ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) |
                         reinterpret_cast<uintptr_t>(dst)) & 15) == 0;
  if (n % 8 == 0 && aligned) {
    long blocks = (n / 8 + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    auto kern = adt == DT_BF16 ? (ddt == DT_BF16 ? k_add_cast8<DT_BF16, DT_BF16>
                                                 : k_add_cast8<DT_BF16, DT_F32>)
                               : (ddt == DT_BF16 ? k_add_cast8<DT_F32, DT_BF16>
                                                 : k_add_cast8<DT_F32, DT_F32>);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, st, a, b, dst, n / 8);
    return hipGetLastError();
  }
  long blocks = (n + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_add_cast, dim3((unsigned)blocks), dim3(256), 0, st, a, adt, b, dst, ddt,
                     n);
  return hipGetLastError();
}

}  // namespace pulse
