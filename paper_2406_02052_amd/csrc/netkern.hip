// Kernels of the multi-stage network: image ingest, the non-reversible front
// layers' BN passes on split activations, the stride-2 input-gradient scatter,
// the softmax cross-entropy head and the padded-channel split-K reduce.
#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace petra {

namespace netk {

unsigned grid_of(long n, long per_block = 256) {
  long b = (n + per_block - 1) / per_block;
  if (b > 65536) b = 65536;
  if (b < 1) b = 1;
  return static_cast<unsigned>(b);
}

template <typename T>
__global__ __launch_bounds__(256) void pad8_kernel(const T* src, int c_img, T* dst, long m) {
  for (long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; i < m * 8;
       i += static_cast<long>(gridDim.x) * 256) {
    const long row = i >> 3;
    const int c = static_cast<int>(i & 7);
    dst[i] = c < c_img ? src[row * c_img + c] : T{};
  }
}

__global__ void copy_i32_kernel(const int32_t* src, int32_t* dst, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

template <typename T>
__global__ __launch_bounds__(256) void bn_apply_split_kernel(const T* h, const float* scale,
                                                             const float* shift, int relu, T* o1,
                                                             T* o2, long m, int c) {
  const int c8 = c / 8, half = c / 2;
  for (long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; i < m * c8;
       i += static_cast<long>(gridDim.x) * 256) {
    const long row = i / c8;
    const int ch = static_cast<int>(i - row * c8) * 8;
    float v[8];
    Vec8<T>::load(h + row * c + ch, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = fmaf(scale[ch + j], v[j], shift[ch + j]);
      if (relu) v[j] = fmaxf(v[j], 0.f);
    }
    T* dst = ch < half ? o1 + row * half + ch : o2 + row * half + (ch - half);
    Vec8<T>::store(dst, v);
  }
}

// Gradient of the BN output (optionally masked by the ReLU after it), read
// from the two half tensors.
template <typename T>
__device__ __forceinline__ void load_dz(const T* d1, const T* d2, const T* h, const float* scale,
                                        const float* shift, int relu, long row, int ch, int c,
                                        float* dz, float* hv) {
  const int half = c / 2;
  const T* src = ch < half ? d1 + row * half + ch : d2 + row * half + (ch - half);
  Vec8<T>::load(src, dz);
  Vec8<T>::load(h + row * c + ch, hv);
  if (relu) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (!(fmaf(scale[ch + j], hv[j], shift[ch + j]) > 0.f)) dz[j] = 0.f;
  }
}

int split_rows_per_tile(long m, int c) {
  const int rows_per_pass = 256 / (c / 8);
  long want = (m + 1023) / 1024;
  long rpt = ((want + rows_per_pass - 1) / rows_per_pass) * rows_per_pass;
  if (rpt < rows_per_pass) rpt = rows_per_pass;
  return static_cast<int>(rpt);
}

template <typename T>
__global__ __launch_bounds__(256) void split_bwd_partials_kernel(
    const T* d1, const T* d2, const T* h, const float* scale, const float* shift,
    const float* mean, const float* rstd, int relu, float* partials, long m, int c,
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
    for (long row = row0 + rr; row < row1; row += rows_per_pass) {
      float dz[8], hv[8];
      load_dz(d1, d2, h, scale, shift, relu, row, ch, c, dz, hv);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        s1[j] += dz[j];
        s2[j] += dz[j] * ((hv[j] - mean[ch + j]) * rstd[ch + j]);
      }
    }
  }
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

// Elementwise over (row, 8 channels); a block's 256 threads cover whole rows
// (c / 8 divides 256), so a thread keeps its channels' constants over APPLY_ROWS
// rows: with one row per thread the 48 constant loads cost more than the three
// 16-byte tensor accesses (128x32x32x64: 24.2 us).
constexpr int APPLY_ROWS = 4;
template <typename T>
__global__ __launch_bounds__(256) void split_bwd_apply_kernel(
    const T* d1, const T* d2, const T* h, const float* scale, const float* shift, const float* ca,
    const float* cb, const float* cc, const float* mean, int relu, T* dh, long m, int c) {
  const int c8 = c / 8, half = c / 2;
  const int rows = 256 / c8, ch = (threadIdx.x % c8) * 8;
  const T* src = ch < half ? d1 + ch : d2 + (ch - half);
  float ks[8], kh[8], ka[8], kb[8], kc[8], km[8];
  Vec8<float>::load(scale + ch, ks);
  Vec8<float>::load(shift + ch, kh);
  Vec8<float>::load(ca + ch, ka);
  Vec8<float>::load(cb + ch, kb);
  Vec8<float>::load(cc + ch, kc);
  Vec8<float>::load(mean + ch, km);
  const long row0 = static_cast<long>(blockIdx.x) * rows * APPLY_ROWS + threadIdx.x / c8;
  Raw8<T> rz[APPLY_ROWS], rh[APPLY_ROWS];
#pragma unroll
  for (int r = 0; r < APPLY_ROWS; ++r) {
    const long row = min(row0 + static_cast<long>(r) * rows, m - 1);
    rz[r].load(src + row * half);
    rh[r].load(h + row * c + ch);
  }
#pragma unroll
  for (int r = 0; r < APPLY_ROWS; ++r) {
    const long row = row0 + static_cast<long>(r) * rows;
    if (row >= m) break;
    float dz[8], hv[8], o[8];
    rz[r].to_f32(dz);
    rh[r].to_f32(hv);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (relu && !(fmaf(ks[j], hv[j], kh[j]) > 0.f)) dz[j] = 0.f;
      o[j] = fmaf(ka[j], dz[j], fmaf(kb[j], hv[j] - km[j], kc[j]));
    }
    Vec8<T>::store(dh + row * c + ch, o);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void scatter2_kernel(const T* src, T* dst1, T* dst2, int n,
                                                       int h, int w, int c) {
  const int c8 = c / 8, half = c / 2;
  const int h2 = h / 2, w2 = w / 2;
  const long total = static_cast<long>(n) * h * w * c8;
  for (long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; i < total;
       i += static_cast<long>(gridDim.x) * 256) {
    const long pix = i / c8;
    const int ch = static_cast<int>(i - pix * c8) * 8;
    const int x = static_cast<int>(pix % w);
    const int y = static_cast<int>((pix / w) % h);
    const long img = pix / (static_cast<long>(h) * w);
    float v[8];
    if ((x & 1) == 0 && (y & 1) == 0 && (y >> 1) < h2 && (x >> 1) < w2) {
      const long srow = (img * h2 + (y >> 1)) * w2 + (x >> 1);
      Vec8<T>::load(src + srow * c + ch, v);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = 0.f;
    }
    T* dst = ch < half ? dst1 + pix * half + ch : dst2 + pix * half + (ch - half);
    Vec8<T>::store(dst, v);
  }
}

// One block per image.  c <= 1024, k <= 64.  Latency-bound (a few KB per image):
// the pixels are summed 8 channels at a time by all threads, and the softmax runs
// over the lanes of one wave (one thread did it class by class in fp64, 26 us in
// all at 128x4x4x512).
template <typename T>
__global__ __launch_bounds__(256) void head_kernel(const T* x1, const T* x2, int hw, int c,
                                                   const float* wfc, const float* bfc, int k,
                                                   const int32_t* labels, int n, float* pooled,
                                                   float* dlogits, float* loss_n, T* g1, T* g2) {
  __shared__ __attribute__((aligned(16))) float part[2048];
  __shared__ __attribute__((aligned(16))) float sp[1024];
  __shared__ float sl[64];
  const int img = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int half = c / 2, c8 = c / 8;
  const int groups = 256 / c8;   // pixel groups (c8 <= 128 divides 256)
  const int ch8 = (tid % c8) * 8, grp = tid / c8;
  const T* src = ch8 < half ? x1 + static_cast<long>(img) * hw * half + ch8
                            : x2 + static_cast<long>(img) * hw * half + (ch8 - half);
  {
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
#pragma unroll 4
    for (int p = grp; p < hw; p += groups) {
      float v[8];
      Vec8<T>::load(src + static_cast<long>(p) * half, v);
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] += v[j];
    }
    Vec8<float>::store(part + tid * 8, acc);   // [group][channel]
  }
  __syncthreads();
  for (int ch = tid; ch < c; ch += 256) {
    float acc = 0.f;
    for (int g = 0; g < groups; ++g) acc += part[g * c + ch];
    const float v = acc / static_cast<float>(hw);
    sp[ch] = v;
    pooled[static_cast<long>(img) * c + ch] = v;
  }
  __syncthreads();
  for (int j = wave; j < k; j += 4) {
    float acc = 0.f;
#pragma unroll 4
    for (int ch = lane; ch < c; ch += 64) acc += sp[ch] * wfc[static_cast<long>(j) * c + ch];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) sl[j] = acc + bfc[j];
  }
  __syncthreads();
  if (wave == 0) {
    const float v = lane < k ? sl[lane] : sl[0];
    float mx = v;
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    const double z = static_cast<double>(v - mx);
    double se = lane < k ? exp(z) : 0.0;
    for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off, 64);
    const double lse = log(se);
    const int raw = labels[img];
    const bool valid = raw >= 0 && raw < k;   // an out-of-range label yields a NaN loss
    const int lab = valid ? raw : 0;
    if (lane == lab) loss_n[img] = valid ? static_cast<float>(lse - z) : __int_as_float(0x7fc00000);
    if (lane < k) {
      const float p = static_cast<float>((exp(z - lse) - (lane == lab ? 1.0 : 0.0)) / n);
      sl[lane] = p;
      dlogits[static_cast<long>(img) * k + lane] = p;
    }
  }
  __syncthreads();
  // the gradient of every pixel, 8 channels per thread
  float d[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) d[j] = 0.f;
#pragma unroll 2
  for (int q = 0; q < k; ++q) {
    float w[8];
    Vec8<float>::load(wfc + static_cast<long>(q) * c + ch8, w);
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] += sl[q] * w[j];
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) d[j] = d[j] / static_cast<float>(hw);
  T* dst = ch8 < half ? g1 + static_cast<long>(img) * hw * half + ch8
                      : g2 + static_cast<long>(img) * hw * half + (ch8 - half);
  for (int p = grp; p < hw; p += groups) Vec8<T>::store(dst + static_cast<long>(p) * half, d);
}

// Blocks [0, k * ceil(c / 32)): 32 channels of one class, 8 groups of images whose
// sums are added in order; the last block: bias gradients (a wave per class, lanes
// over images) and the mean loss.  One thread per weight over all images took 46 us
// at 128 images, 512 channels, 10 classes: a chain of 128 dependent loads.
__global__ __launch_bounds__(256) void head_grads_kernel(const float* pooled, const float* dlogits,
                                                         const float* loss_n, int n, int c, int k,
                                                         float inv_k, float* gw, float* gb,
                                                         float* loss) {
  const int tid = threadIdx.x;
  const int cblocks = (c + 31) / 32;
  if (static_cast<int>(blockIdx.x) < k * cblocks) {
    __shared__ float red[8][33];
    const int j = blockIdx.x / cblocks;
    const int cl = tid & 31, g = tid >> 5, ch = (blockIdx.x - j * cblocks) * 32 + cl;
    float acc = 0.f;
    if (ch < c) {
#pragma unroll 8
      for (int r = g; r < n; r += 8)
        acc += dlogits[static_cast<long>(r) * k + j] * pooled[static_cast<long>(r) * c + ch];
    }
    red[g][cl] = acc;
    __syncthreads();
    if (g == 0 && ch < c) {
#pragma unroll
      for (int q = 1; q < 8; ++q) acc += red[q][cl];
      gw[static_cast<long>(j) * c + ch] += inv_k * acc;
    }
    return;
  }
  const int lane = tid & 63, wave = tid >> 6;
  for (int j = wave; j < k; j += 4) {
    float acc = 0.f;
    for (int r = lane; r < n; r += 64) acc += dlogits[static_cast<long>(r) * k + j];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) gb[j] += inv_k * acc;
  }
  if (wave == 0 && loss != nullptr) {
    double acc = 0.0;
    for (int r = lane; r < n; r += 64) acc += loss_n[r];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) *loss = static_cast<float>(acc / n);
  }
}

// A block owns 32 consecutive weights; its 8 thread rows take interleaved splits,
// four loads in flight, and the row sums are combined in a fixed order (one thread
// per weight over all 256 splits took 102 us at 64 x 27 weights).
__global__ __launch_bounds__(256) void wgrad_reduce_pad_kernel(const float* part, int splits,
                                                               int c_out, int taps, int c_pad,
                                                               int c_real, float inv_k,
                                                               float* grad) {
  __shared__ float red[8][33];
  const long numel = static_cast<long>(c_out) * taps * c_real;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const long i = static_cast<long>(blockIdx.x) * 32 + tx;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  if (i < numel) {
    const float* src = part + (i / c_real) * c_pad + i % c_real;
    const long stride = static_cast<long>(c_out) * taps * c_pad;
    int t = ty;
    for (; t + 24 < splits; t += 32) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += src[(t + 8 * u) * stride];
    }
    for (; t < splits; t += 8) acc[0] += src[t * stride];
  }
  red[ty][tx] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (ty == 0 && i < numel) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) s += red[r][tx];
    grad[i] += inv_k * s;
  }
}

}  // namespace netk
using namespace netk;

void pad_channels8(int dtype, const void* src, int c_img, void* dst, long m, hipStream_t st) {
  if (dtype == DT_BF16)
    PETRA_LAUNCH(pad8_kernel<bf16_t>, dim3(grid_of(m * 8)), dim3(256), 0, st,
                       static_cast<const bf16_t*>(src), c_img, static_cast<bf16_t*>(dst), m);
  else
    PETRA_LAUNCH(pad8_kernel<float>, dim3(grid_of(m * 8)), dim3(256), 0, st,
                       static_cast<const float*>(src), c_img, static_cast<float*>(dst), m);
}

void copy_i32(const int32_t* src, int32_t* dst, int n, hipStream_t st) {
  PETRA_LAUNCH(copy_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, st, src, dst, n);
}

void bn_apply_split(int dtype, const void* h, const float* scale, const float* shift, int relu,
                    void* out1, void* out2, long m, int c, hipStream_t st) {
  const unsigned g = grid_of(m * (c / 8));
  if (dtype == DT_BF16)
    PETRA_LAUNCH(bn_apply_split_kernel<bf16_t>, dim3(g), dim3(256), 0, st,
                       static_cast<const bf16_t*>(h), scale, shift, relu,
                       static_cast<bf16_t*>(out1), static_cast<bf16_t*>(out2), m, c);
  else
    PETRA_LAUNCH(bn_apply_split_kernel<float>, dim3(g), dim3(256), 0, st,
                       static_cast<const float*>(h), scale, shift, relu,
                       static_cast<float*>(out1), static_cast<float*>(out2), m, c);
}

int split_tiles(long m, int c) {
  const int rpt = split_rows_per_tile(m, c);
  return static_cast<int>((m + rpt - 1) / rpt);
}

void split_bwd_partials(int dtype, const void* d1, const void* d2, const void* h,
                        const float* scale, const float* shift, const float* mean,
                        const float* rstd, int relu, float* partials, long m, int c,
                        hipStream_t st) {
  const int rpt = split_rows_per_tile(m, c);
  const int tiles = static_cast<int>((m + rpt - 1) / rpt);
  if (dtype == DT_BF16)
    PETRA_LAUNCH(split_bwd_partials_kernel<bf16_t>, dim3(tiles), dim3(256), 0, st,
                       static_cast<const bf16_t*>(d1), static_cast<const bf16_t*>(d2),
                       static_cast<const bf16_t*>(h), scale, shift, mean, rstd, relu, partials, m,
                       c, rpt);
  else
    PETRA_LAUNCH(split_bwd_partials_kernel<float>, dim3(tiles), dim3(256), 0, st,
                       static_cast<const float*>(d1), static_cast<const float*>(d2),
                       static_cast<const float*>(h), scale, shift, mean, rstd, relu, partials, m,
                       c, rpt);
}

void split_bwd_apply(int dtype, const void* d1, const void* d2, const void* h,
                     const float* scale, const float* shift, const float* ca, const float* cb,
                     const float* cc, const float* mean, int relu, void* dh, long m, int c,
                     hipStream_t st) {
  const long rows = 256 / (c / 8) * APPLY_ROWS;
  const unsigned g = static_cast<unsigned>((m + rows - 1) / rows);
  if (dtype == DT_BF16)
    PETRA_LAUNCH(split_bwd_apply_kernel<bf16_t>, dim3(g), dim3(256), 0, st,
                       static_cast<const bf16_t*>(d1), static_cast<const bf16_t*>(d2),
                       static_cast<const bf16_t*>(h), scale, shift, ca, cb, cc, mean, relu,
                       static_cast<bf16_t*>(dh), m, c);
  else
    PETRA_LAUNCH(split_bwd_apply_kernel<float>, dim3(g), dim3(256), 0, st,
                       static_cast<const float*>(d1), static_cast<const float*>(d2),
                       static_cast<const float*>(h), scale, shift, ca, cb, cc, mean, relu,
                       static_cast<float*>(dh), m, c);
}

void scatter_stride2_split(int dtype, const void* src, void* dst1, void* dst2, int n, int h,
                           int w, int c, hipStream_t st) {
  const unsigned g = grid_of(static_cast<long>(n) * h * w * (c / 8));
  if (dtype == DT_BF16)
    PETRA_LAUNCH(scatter2_kernel<bf16_t>, dim3(g), dim3(256), 0, st,
                       static_cast<const bf16_t*>(src), static_cast<bf16_t*>(dst1),
                       static_cast<bf16_t*>(dst2), n, h, w, c);
  else
    PETRA_LAUNCH(scatter2_kernel<float>, dim3(g), dim3(256), 0, st,
                       static_cast<const float*>(src), static_cast<float*>(dst1),
                       static_cast<float*>(dst2), n, h, w, c);
}

void head_forward_backward(int dtype, const void* x1, const void* x2, int n, int hw, int c,
                           const float* wfc, const float* bfc, int k, const int32_t* labels,
                           float* pooled, float* dlogits, float* loss_n, void* g1, void* g2,
                           hipStream_t st) {
  if (dtype == DT_BF16)
    PETRA_LAUNCH(head_kernel<bf16_t>, dim3(n), dim3(256), 0, st,
                       static_cast<const bf16_t*>(x1), static_cast<const bf16_t*>(x2), hw, c, wfc,
                       bfc, k, labels, n, pooled, dlogits, loss_n, static_cast<bf16_t*>(g1),
                       static_cast<bf16_t*>(g2));
  else
    PETRA_LAUNCH(head_kernel<float>, dim3(n), dim3(256), 0, st,
                       static_cast<const float*>(x1), static_cast<const float*>(x2), hw, c, wfc,
                       bfc, k, labels, n, pooled, dlogits, loss_n, static_cast<float*>(g1),
                       static_cast<float*>(g2));
}

void head_param_grads(const float* pooled, const float* dlogits, const float* loss_n, int n,
                      int c, int k, float inv_k, float* grad_w, float* grad_b, float* loss,
                      hipStream_t st) {
  const long blocks = static_cast<long>(k) * ((c + 31) / 32) + 1;
  PETRA_LAUNCH(head_grads_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, pooled, dlogits,
                     loss_n, n, c, k, inv_k, grad_w, grad_b, loss);
}

void wgrad_reduce_pad(const float* part, int splits, int c_out, int taps, int c_pad, int c_real,
                      float inv_k, float* grad, hipStream_t st) {
  const long numel = static_cast<long>(c_out) * taps * c_real;
  PETRA_LAUNCH(wgrad_reduce_pad_kernel, dim3(static_cast<unsigned>((numel + 31) / 32)), dim3(256), 0, st, part, splits,
                     c_out, taps, c_pad, c_real, inv_k, grad);
}

}  // namespace petra
