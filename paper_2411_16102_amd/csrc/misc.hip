// Small kernels around the GEMMs: RMSNorm preparation of the layer input, the
// RoPE angle table, and conversion between token-major K/V arrays and the
// library's KV page layout.
#include "misc.hpp"
#include "common.hpp"

namespace bs {
namespace {

// Workgroup blockIdx.x of an upload: 4 KB of pinned host memory into the device's copy, one 16-byte load per
// thread, so that everything asks at once.  Bound by the host link (486 KB 13.5 us).  hipMemcpyAsync instead kept
// the stream idle for 20 to 27 us between two steps (the copy engine and the handover to it and back), or, for
// descriptors of a few KB, 9 us (a copy kernel and the gap behind it).
__device__ __forceinline__ void upload_block(const Upload &up) {
  const int i = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (i < up.n16) up.dst[i] = up.src[i];
}

__global__ __launch_bounds__(256) void upload_kernel(const Upload up) { upload_block(up); }

// xg = bf16(x * g) (the GEMM operand of the normalised row; the 1/rms factor commutes with the
// contraction and is applied in the GEMM epilogue) and rstd = 1 / sqrt(mean(x^2) + eps).
// The first `up.blocks` workgroups bring the step's descriptor over (see upload_block).  They hide under the rows in part:
// the launch takes 2 us longer with a descriptor of 209 KB and 1580 rows of 4096, 5 with 345 KB and 2560 rows, 11 with
// 928 KB and 5120 rows of 8192 (43 us).
// WPR wavefronts per row.  One wavefront per row where there are
// rows enough for the chip (8192 rows of 4096: 26 us, the bytes at the rate of a copy); with few rows the
// kernel is the round trips of one row, and four wavefronts share them (see launch_norm_prep).
template <int WPR>
__global__ __launch_bounds__(256) void norm_prep_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ g,
                                                       uint16_t *__restrict__ xg, float *__restrict__ rstd, int rows, int d,
                                                       float eps, unsigned *__restrict__ zero_words, int n_zero, const Upload up) {
  if ((int)blockIdx.x < up.blocks) return upload_block(up);
  const int bid = (int)blockIdx.x - up.blocks;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // the first kernel of a step also clears the step's counters (a fill in a kernel, not a
  // memset on the stream, so that a captured step replays it like any other launch)
  if (bid == 0 && (int)threadIdx.x < n_zero) zero_words[threadIdx.x] = 0u;
  const int row = WPR == 1 ? bid * 4 + wave : bid;
  if (row >= rows) return;  // (with four wavefronts per row: all of the workgroup or none)
  const uint16_t *xr = x + (size_t)row * d;
  uint16_t *outr = xg + (size_t)row * d;
  float s = 0.f;
  const int first = (WPR == 1 ? lane : (int)threadIdx.x) * 8;
  constexpr int STEP = WPR * 64 * 8;
  auto eight = [&](int c) __attribute__((always_inline)) {
    const u32x4_t xv = *reinterpret_cast<const u32x4_t *>(xr + c);
    const u32x4_t gv = *reinterpret_cast<const u32x4_t *>(g + c);
    u32x4_t ov;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x0 = __uint_as_float(xv[i] << 16), x1 = __uint_as_float(xv[i] & 0xFFFF0000u);
      const float g0 = __uint_as_float(gv[i] << 16), g1 = __uint_as_float(gv[i] & 0xFFFF0000u);
      s += x0 * x0 + x1 * x1;
      ov[i] = pack_bf16x2(x0 * g0, x1 * g1);
    }
    *reinterpret_cast<u32x4_t *>(outr + c) = ov;
  };
  if constexpr (WPR == 1) {
    for (int c = first; c < d; c += STEP) eight(c);
  } else {
#pragma unroll 4
    for (int c = first; c < d; c += STEP) eight(c);
  }
  s = wave_sum(s);
  if constexpr (WPR > 1) {
    __shared__ float part[WPR];
    if (lane == 0) part[wave] = s;
    __syncthreads();
    s = (part[0] + part[1]) + (part[2] + part[3]);
  }
  if ((WPR == 1 ? lane : (int)threadIdx.x) == 0) rstd[row] = rsqrtf(s / (float)d + eps);
}

// rstd[m] = 1 / sqrt(sum_p part[p][m] / d + eps): closes the row sums of squares that
// the output projection's epilogue leaves per column tile.  A workgroup covers 64 rows;
// its four wavefronts each add every fourth partial (coalesced along the rows, the loads
// of a thread independent of each other) and meet in LDS.
__global__ __launch_bounds__(256) void rstd_finalize_kernel(const float *part, int n_part, int stride, float *rstd,
                                                            int rows, float d, float eps) {
  __shared__ float sh[4][64];
  const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int m = blockIdx.x * 64 + r;
  float s = 0.f;
  if (m < rows) {
#pragma unroll 8
    for (int p = q; p < n_part; p += 4) s += part[(size_t)p * stride + m];
  }
  sh[q][r] = s;
  __syncthreads();
  if (q == 0 && m < rows) rstd[m] = rsqrtf((sh[0][r] + sh[1][r] + sh[2][r] + sh[3][r]) / d + eps);
}

// cos/sin of pos * theta^(-2i/dh), evaluated in double and stored as float
__global__ void rope_table_kernel(float *cos_t, float *sin_t, int max_pos, int half, double theta) {
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (long)max_pos * half) return;
  const int pos = (int)(idx / half), i = (int)(idx % half);
  const double freq = pow(theta, -(double)i / (double)half);
  double s, c;
  sincos((double)pos * freq, &s, &c);
  cos_t[idx] = (float)c;
  sin_t[idx] = (float)s;
}

// token-major k, v [n_pages][16][Hkv][dh]  <->  pages of K [Hkv][16][dh] and V^T [Hkv][dh][16]
__global__ void kv_pack_kernel(const uint16_t *k, const uint16_t *v, uint16_t *pool, long n_pages, int hkv, int dh,
                               int unpack, uint16_t *k_out, uint16_t *v_out) {
  const long per_page = (long)16 * hkv * dh;
  const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_pages * per_page) return;
  const long page = idx / per_page;
  long r = idx % per_page;
  const int slot = (int)(r / (hkv * dh));
  r %= (long)hkv * dh;
  const int head = (int)(r / dh), e = (int)(r % dh);
  const long tile = (long)16 * dh;
  const long kd = ((page * 2 + 0) * hkv + head) * tile + (long)slot * dh + e;
  const long vd = ((page * 2 + 1) * hkv + head) * tile + (long)e * 16 + slot;
  if (unpack) {
    k_out[idx] = pool[kd];
    v_out[idx] = pool[vd];
  } else {
    pool[kd] = k[idx];
    pool[vd] = v[idx];
  }
}

}  // namespace

// Up to here four wavefronts share a row.  Measured, rows of 4096 (8192): 7 rows 8.6 -> 6.3 us (12.9 -> 6.9),
// 256 rows 9.5 -> 7.3 (13.8 -> 7.8), 1024 rows 10.4 -> 8.5 (16.0 -> 11.7), all with the 4 us of a timed launch.
constexpr int NORM_SHARED_ROWS = 1024;

hipError_t launch_norm_prep(const uint16_t *x, const uint16_t *g, uint16_t *xg, float *rstd, int rows, int d,
                            float eps, unsigned *zero_words, int n_zero, const Upload &up, hipStream_t stream) {
  if (rows <= 0) return hipErrorInvalidValue;
  const int nz = zero_words ? n_zero : 0;
  if (rows <= NORM_SHARED_ROWS)
    hipLaunchKernelGGL(norm_prep_kernel<4>, dim3(up.blocks + rows), dim3(256), 0, stream, x, g, xg, rstd, rows, d, eps, zero_words, nz, up);
  else
    hipLaunchKernelGGL(norm_prep_kernel<1>, dim3(up.blocks + (rows + 3) / 4), dim3(256), 0, stream, x, g, xg, rstd, rows, d, eps, zero_words, nz, up);
  return hipGetLastError();
}

hipError_t launch_upload(const Upload &up, hipStream_t stream) {
  if (up.blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(upload_kernel, dim3(up.blocks), dim3(256), 0, stream, up);
  return hipGetLastError();
}

hipError_t launch_rstd_finalize(const float *part, int n_part, int stride, float *rstd, int rows, int d, float eps,
                                hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(rstd_finalize_kernel, dim3((rows + 63) / 64), dim3(256), 0, stream, part, n_part, stride, rstd,
                     rows, (float)d, eps);
  return hipGetLastError();
}

hipError_t launch_rope_table(float *cos_t, float *sin_t, int max_pos, int half, double theta, hipStream_t stream) {
  const long n = (long)max_pos * half;
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, cos_t, sin_t,
                     max_pos, half, theta);
  return hipGetLastError();
}

hipError_t launch_kv_pack(const uint16_t *k, const uint16_t *v, uint16_t *pool, long n_pages, int hkv, int dh,
                          hipStream_t stream) {
  const long n = n_pages * 16 * hkv * dh;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(kv_pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, k, v, pool, n_pages,
                     hkv, dh, 0, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t launch_kv_unpack(const uint16_t *pool, uint16_t *k, uint16_t *v, long n_pages, int hkv, int dh,
                            hipStream_t stream) {
  const long n = n_pages * 16 * hkv * dh;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(kv_pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, nullptr, nullptr,
                     const_cast<uint16_t *>(pool), n_pages, hkv, dh, 1, k, v);
  return hipGetLastError();
}

}  // namespace bs
