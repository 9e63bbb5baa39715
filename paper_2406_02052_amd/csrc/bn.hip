// Batch-normalisation statistics, BN backward coefficients and the fused
// elementwise passes of the reversible coupling (gfx950).
//
// Statistics arrive as per-tile partial sums written by the producing kernel
// (the conv epilogue or combine_bwd); the finalize kernels combine them in a
// fixed order in fp64, so results are run-to-run deterministic.
#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace petra {

namespace bnk {

// Finalize kernels: one block of NW waves per channel.  Thread t takes tiles
// t, t + 64 NW, ..., U of them in flight, then the block's sums are combined in a
// fixed tree: xor levels inside each wave, then the wave results in order.
// Deterministic run to run, and the order does not depend on U.
//
// What bounds them is latency: a launch (about 2.3 us), one trip to memory for the
// partials, the reduction and a scalar tail, 60 to 90 times in a tick of a 4-stage
// schedule.  Hence the tail's operands are fetched beside the partials, the
// reduction's first four levels are DPP moves (an LDS permute has some 100 clocks),
// the row count comes from the host with its reciprocal, and the tile counts take
// a fast reciprocal in place of a division.  About 1.1 us less per launch than with
// each of these after the other (forwards with 24 statistics of 256 tiles of 128
// channels 781 -> 756 us, with 8 of 32 tiles of 32 channels 83.3 -> 75.3 us, with 18
// of 128 and 32 channels at 64x56x56 430 -> 409 us).
constexpr int FIN_WAVES = 4;

// The sum over the wave's lanes, in every lane: xor levels 1, 2, 4, 8 with DPP (once
// the levels below agree, the half mirror and the mirror bring xor 4 and 8's values),
// then 16 and 32.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
  const u32x2_t w = __builtin_bit_cast(u32x2_t, v);
  const u32x2_t x{
      static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w.x), CTRL, 0xF, 0xF, false)),
      static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w.y), CTRL, 0xF, 0xF, false))};
  return v + __builtin_bit_cast(double, x);
}
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0xB1>(v);    // [1,0,3,2]
  v = dpp_add<0x4E>(v);    // [2,3,0,1]
  v = dpp_add<0x141>(v);   // half mirror
  v = dpp_add<0x140>(v);   // mirror
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// (a, b) summed over the block, in every thread of its first wave.
template <int NW>
__device__ __forceinline__ void block_sum(double& a, double& b) {
  a = wave_sum(a);
  b = wave_sum(b);
  if constexpr (NW > 1) {
    static_assert(NW == 4, "the wave results are combined as four");
    __shared__ double red[2][NW];
    const int tid = threadIdx.x;
    if ((tid & 63) == 0) {
      red[0][tid >> 6] = a;
      red[1][tid >> 6] = b;
    }
    __syncthreads();
    a = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    b = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
  }
}

__device__ __forceinline__ float buf_load4(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, static_cast<int>(off), 0, 0));
}

// 1 / n of a positive tile count: hardware estimate and two Newton steps, correct
// to the last bits of fp64.
__device__ __forceinline__ double recip(double n) {
  double r = __builtin_amdgcn_rcp(n);
  r = fma(fma(-n, r, 1.0), r, r);
  return fma(fma(-n, r, 1.0), r, r);
}

// partials[tile][3][c] = (rows n_t, sum S_t, centred sum of squares Q_t).  Every tile
// is re-centred on one shift K near the first tile's mean: with e_t = S_t - n_t K,
// sum_x (x - K) = sum_t e_t and sum_x (x - K)^2 = sum_t [Q_t + e_t^2 / n_t].  Those
// are plain sums (one fixed-order block reduction of two fp64 values, B and A), and
// mean = K + B/m, M2 = A - B^2/m.  K lies within a tile's spread of the mean, so the
// subtraction loses a few bits of fp64 at most.  Tiles past the end read zeros.
template <int NW, int U>
__global__ __launch_bounds__(64 * NW) void bn_stats_finalize_kernel(
    const float* partials, int tiles, int c, double inv_m, double unbias, const float* gamma,
    const float* beta, float eps, float* scale, float* shift, float* mean_out, float* rstd_out,
    float* run_mean, float* run_var, float momentum) {
  const int ch = blockIdx.x;
  const uint32_t row = static_cast<uint32_t>(c) * 4u, cho = static_cast<uint32_t>(ch) * 4u;
  const __amdgpu_buffer_rsrc_t r = make_rsrc(partials, static_cast<long>(tiles) * 3 * c * 4);
  float vn[U], vs[U], vq[U];
  auto load = [&](int base) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t off = static_cast<uint32_t>(base + u * 64 * NW) * 3u * row + cho;
      vn[u] = buf_load4(r, off);
      vs[u] = buf_load4(r, off + row);
      vq[u] = buf_load4(r, off + 2u * row);
    }
  };
  // all of a one-pass call's loads at once: the shift, the tiles, the tail's operands
  const bool run = run_mean != nullptr;
  const float n0 = buf_load4(r, cho), s0 = buf_load4(r, row + cho);
  load(threadIdx.x);
  const float g = buf_load4(make_rsrc(gamma, row), cho), be = buf_load4(make_rsrc(beta, row), cho);
  const float rm = buf_load4(make_rsrc(run_mean, run ? row : 0), cho);
  const float rv = buf_load4(make_rsrc(run_var, run ? row : 0), cho);
  __builtin_amdgcn_sched_barrier(0);
  const double k = n0 > 0.f ? static_cast<double>(s0 * __builtin_amdgcn_rcpf(n0)) : 0.0;
  double a = 0.0, b = 0.0;
  for (int base = 0;;) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (vn[u] > 0.f) {
        const double nt = vn[u], e = fma(-nt, k, static_cast<double>(vs[u]));
        b += e;
        a += fma(e * e, recip(nt), static_cast<double>(vq[u]));
      }
    }
    base += 64 * NW * U;
    if (base >= tiles) break;
    load(base + static_cast<int>(threadIdx.x));
  }
  block_sum<NW>(a, b);
  if (threadIdx.x != 0) return;
  const double mean = k + b * inv_m;
  const double var = fmax(a - b * b * inv_m, 0.0) * inv_m;   // biased batch variance
  const double rstd = rsqrt(var + static_cast<double>(eps));
  const double sc = static_cast<double>(g) * rstd;
  scale[ch] = static_cast<float>(sc);
  shift[ch] = static_cast<float>(static_cast<double>(be) - mean * sc);
  mean_out[ch] = static_cast<float>(mean);
  rstd_out[ch] = static_cast<float>(rstd);
  if (run) {
    const double mom = momentum;
    run_mean[ch] = static_cast<float>((1.0 - mom) * rm + mom * mean);
    run_var[ch] = static_cast<float>((1.0 - mom) * rv + mom * (var * unbias));
  }
}

// partials[tile][2][c]: sums of d and of d xhat.
template <int NW, int U>
__global__ __launch_bounds__(64 * NW) void bn_bwd_finalize_kernel(
    const float* partials, int tiles, int c, double inv_m, const float* gamma, const float* rstd,
    float inv_k, float* dgamma, float* dbeta, float* ca, float* cb, float* cc) {
  const int ch = blockIdx.x;
  const uint32_t row = static_cast<uint32_t>(c) * 4u, cho = static_cast<uint32_t>(ch) * 4u;
  const __amdgpu_buffer_rsrc_t rs = make_rsrc(partials, static_cast<long>(tiles) * 2 * c * 4);
  float va[U], vb[U];
  auto load = [&](int base) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t off = static_cast<uint32_t>(base + u * 64 * NW) * 2u * row + cho;
      va[u] = buf_load4(rs, off);
      vb[u] = buf_load4(rs, off + row);
    }
  };
  load(threadIdx.x);
  const float gf = buf_load4(make_rsrc(gamma, row), cho), rf = buf_load4(make_rsrc(rstd, row), cho);
  const float dg = buf_load4(make_rsrc(dgamma, row), cho), db = buf_load4(make_rsrc(dbeta, row), cho);
  __builtin_amdgcn_sched_barrier(0);
  double sd = 0.0, sdx = 0.0;
  for (int base = 0;;) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sd += va[u];
      sdx += vb[u];
    }
    base += 64 * NW * U;
    if (base >= tiles) break;
    load(base + static_cast<int>(threadIdx.x));
  }
  block_sum<NW>(sd, sdx);
  if (threadIdx.x != 0) return;
  dbeta[ch] = db + inv_k * static_cast<float>(sd);
  dgamma[ch] = dg + inv_k * static_cast<float>(sdx);
  const double g = gf, r = rf;
  // dh = g*r*(d - sd/m - xhat*sdx/m), xhat = (h - mean)*r
  ca[ch] = static_cast<float>(g * r);
  cb[ch] = static_cast<float>(-g * r * r * sdx * inv_m);
  cc[ch] = static_cast<float>(-g * r * sd * inv_m);
}

template <typename T>
__global__ __launch_bounds__(256) void combine_fwd_kernel(const T* r, const T* h,
                                                          const float* scale, const float* shift,
                                                          T* y, long total8, int c8) {
  for (long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; i < total8;
       i += static_cast<long>(gridDim.x) * 256) {
    const int ch = static_cast<int>(i % c8) * 8;
    float rv[8], hv[8], o[8];
    Vec8<T>::load(r + i * 8, rv);
    Vec8<T>::load(h + i * 8, hv);
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = rv[j] + fmaf(scale[ch + j], hv[j], shift[ch + j]);
    Vec8<T>::store(y + i * 8, o);
  }
}

// x = v - (scale*h + shift): the reconstruction of a coupling input.
template <typename T>
__global__ __launch_bounds__(256) void combine_rec_kernel(const T* v, const T* h,
                                                          const float* scale, const float* shift,
                                                          T* x, long total8, int c8) {
  for (long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; i < total8;
       i += static_cast<long>(gridDim.x) * 256) {
    const int ch = static_cast<int>(i % c8) * 8;
    float vv[8], hv[8], o[8];
    Vec8<T>::load(v + i * 8, vv);
    Vec8<T>::load(h + i * 8, hv);
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = vv[j] - fmaf(scale[ch + j], hv[j], shift[ch + j]);
    Vec8<T>::store(x + i * 8, o);
  }
}

// Each block owns rows [tile*rows_per_tile, ...) and writes one partial row.
template <typename T>
__global__ __launch_bounds__(256) void combine_bwd_kernel(const T* v, const T* h, const T* d,
                                                          const float* scale, const float* shift,
                                                          const float* mean, const float* rstd,
                                                          T* x, float* partials, long m, int c,
                                                          int rows_per_tile) {
  const int c8 = c / 8;
  const int rows_per_pass = 256 / c8;
  const int tid = threadIdx.x;
  const int cg = tid % c8, rr = tid / c8;
  const int ch = cg * 8;
  const long row0 = static_cast<long>(blockIdx.x) * rows_per_tile;
  const long row1 = min(m, row0 + rows_per_tile);
  float s1[8], s2[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) s1[j] = s2[j] = 0.f;
  if (rr < rows_per_pass) {
    float sc[8], sh[8], mu[8], rs[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      sc[j] = scale[ch + j];
      sh[j] = shift[ch + j];
      mu[j] = mean[ch + j];
      rs[j] = rstd[ch + j];
    }
    for (long row = row0 + rr; row < row1; row += rows_per_pass) {
      const long off = row * c + ch;
      float vv[8], hv[8], dv[8], o[8];
      Vec8<T>::load(v + off, vv);
      Vec8<T>::load(h + off, hv);
      Vec8<T>::load(d + off, dv);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        o[j] = vv[j] - fmaf(sc[j], hv[j], sh[j]);
        s1[j] += dv[j];
        s2[j] += dv[j] * ((hv[j] - mu[j]) * rs[j]);
      }
      Vec8<T>::store(x + off, o);
    }
  }
  // Fixed-order reduction over the rows_per_pass thread rows of each channel.
  __shared__ float buf[2][256][9];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    buf[0][tid][j] = s1[j];
    buf[1][tid][j] = s2[j];
  }
  __syncthreads();
  for (int i = tid; i < 2 * c; i += 256) {
    const int which = i / c, chh = i - which * c;
    const int g = chh / 8, j = chh - g * 8;
    float t = 0.f;
    for (int q = 0; q < rows_per_pass; ++q) t += buf[which][q * c8 + g][j];
    partials[(static_cast<long>(blockIdx.x) * 2 + which) * c + chh] = t;
  }
}

int ew_rows_per_tile(long m, int c) {
  const int rows_per_pass = 256 / (c / 8);
  long want = (m + 1023) / 1024;
  long rpt = ((want + rows_per_pass - 1) / rows_per_pass) * rows_per_pass;
  if (rpt < rows_per_pass) rpt = rows_per_pass;
  return static_cast<int>(rpt);
}

unsigned ew_grid(long total8) {
  long b = (total8 + 255) / 256;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return static_cast<unsigned>(b);
}

}  // namespace bnk
using namespace bnk;

int ew_tiles(long m, int c) {
  const int rpt = ew_rows_per_tile(m, c);
  return static_cast<int>((m + rpt - 1) / rpt);
}

// One wave and no barrier while every lane has at most one tile; else four waves,
// with as many tiles in flight per thread as one pass needs, up to four.
#define PETRA_FINALIZE(KERNEL, ...)                                                        \
  do {                                                                                     \
    const dim3 grid(c), one(64), four(64 * FIN_WAVES);                                     \
    if (tiles <= 64)                                                                       \
      PETRA_LAUNCH((KERNEL<1, 1>), grid, one, 0, st, __VA_ARGS__);                         \
    else if (tiles <= 256)                                                                 \
      PETRA_LAUNCH((KERNEL<FIN_WAVES, 1>), grid, four, 0, st, __VA_ARGS__);                \
    else if (tiles <= 512)                                                                 \
      PETRA_LAUNCH((KERNEL<FIN_WAVES, 2>), grid, four, 0, st, __VA_ARGS__);                \
    else                                                                                   \
      PETRA_LAUNCH((KERNEL<FIN_WAVES, 4>), grid, four, 0, st, __VA_ARGS__);                \
  } while (0)

void bn_stats_finalize(const float* partials, int tiles, int c, long m, const float* gamma,
                       const float* beta, float eps, float* scale, float* shift, float* mean,
                       float* rstd, float* run_mean, float* run_var, float momentum,
                       hipStream_t st) {
  const double rows = static_cast<double>(m);
  const double inv_m = m > 0 ? 1.0 / rows : 0.0, unbias = m > 1 ? rows / (rows - 1.0) : 1.0;
  PETRA_FINALIZE(bn_stats_finalize_kernel, partials, tiles, c, inv_m, unbias, gamma, beta, eps,
                 scale, shift, mean, rstd, run_mean, run_var, momentum);
}

void bn_bwd_finalize(const float* partials, int tiles, int c, long m, const float* gamma,
                     const float* rstd, float inv_k, float* dgamma, float* dbeta, float* ca,
                     float* cb, float* cc, hipStream_t st) {
  const double inv_m = m > 0 ? 1.0 / static_cast<double>(m) : 0.0;
  PETRA_FINALIZE(bn_bwd_finalize_kernel, partials, tiles, c, inv_m, gamma, rstd, inv_k, dgamma,
                 dbeta, ca, cb, cc);
}
#undef PETRA_FINALIZE

void combine_fwd(int dtype, const void* r, const void* h, const float* scale, const float* shift,
                 void* y, long m, int c, hipStream_t st) {
  const long total8 = m * c / 8;
  if (dtype == DT_BF16)
    PETRA_LAUNCH(combine_fwd_kernel<bf16_t>, dim3(ew_grid(total8)), dim3(256), 0, st,
                       static_cast<const bf16_t*>(r), static_cast<const bf16_t*>(h), scale, shift,
                       static_cast<bf16_t*>(y), total8, c / 8);
  else
    PETRA_LAUNCH(combine_fwd_kernel<float>, dim3(ew_grid(total8)), dim3(256), 0, st,
                       static_cast<const float*>(r), static_cast<const float*>(h), scale, shift,
                       static_cast<float*>(y), total8, c / 8);
}

void combine_rec(int dtype, const void* v, const void* h, const float* scale, const float* shift,
                 void* x, long m, int c, hipStream_t st) {
  const long total8 = m * c / 8;
  if (dtype == DT_BF16)
    PETRA_LAUNCH(combine_rec_kernel<bf16_t>, dim3(ew_grid(total8)), dim3(256), 0, st,
                       static_cast<const bf16_t*>(v), static_cast<const bf16_t*>(h), scale, shift,
                       static_cast<bf16_t*>(x), total8, c / 8);
  else
    PETRA_LAUNCH(combine_rec_kernel<float>, dim3(ew_grid(total8)), dim3(256), 0, st,
                       static_cast<const float*>(v), static_cast<const float*>(h), scale, shift,
                       static_cast<float*>(x), total8, c / 8);
}

void combine_bwd(int dtype, const void* v, const void* h, const void* d, const float* scale,
                 const float* shift, const float* mean, const float* rstd, void* x,
                 float* partials, long m, int c, hipStream_t st) {
  const int rpt = ew_rows_per_tile(m, c);
  const int tiles = static_cast<int>((m + rpt - 1) / rpt);
  if (dtype == DT_BF16)
    PETRA_LAUNCH(combine_bwd_kernel<bf16_t>, dim3(tiles), dim3(256), 0, st,
                       static_cast<const bf16_t*>(v), static_cast<const bf16_t*>(h),
                       static_cast<const bf16_t*>(d), scale, shift, mean, rstd,
                       static_cast<bf16_t*>(x), partials, m, c, rpt);
  else
    PETRA_LAUNCH(combine_bwd_kernel<float>, dim3(tiles), dim3(256), 0, st,
                       static_cast<const float*>(v), static_cast<const float*>(h),
                       static_cast<const float*>(d), scale, shift, mean, rstd,
                       static_cast<float*>(x), partials, m, c, rpt);
}

}  // namespace petra
